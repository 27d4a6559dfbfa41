// kernels.hip -- device side of the cold exact mask and the -inf apply (gfx950).
//
// grid_mask launches, on the caller's stream:
//  1. prologue (one 1024-thread workgroup per row; the dense action and GOTO
//     tables and the top of the row's stack in LDS): thread t runs terminal t's
//     reduce chain and shift from sigma, so A(sigma) (section 3.2, allowed
//     terminals under table compression) is the ballot of those that shifted, and
//     each one's post-shift stack (an overlay above the shared read-only stack) is
//     recorded; the allowed set of every post-shift stack follows the same way, a
//     wave per 64 terminals, the end of input as one more; then the
//     end-of-sequence gate (section 3.2), the pending lexeme's winner and the
//     bytes that continue the pending lexeme in the schema lexicon.
//  2. judge (one thread per lexeme-program class of the row's lexer state):
//     tokens whose lexeme programs from that state are equal share a class (the
//     verdict-equivalence idea of section 4.2, fixed at compile time per state);
//     each class is judged once against A(sigma) and the allowed sets after a
//     first shift -- reject, allow, walk (a second shift or more than three lexeme
//     ends) or lexicon (the verdict depends on the token's own lexicon flags,
//     section 2 L3).
//  3. stream (512 ids per wave step): the mask in token-id order straight from
//     the class map, a byte per lane; lexicon classes are settled by a shortcut
//     where the token's first byte or its token-flag entry answers the class's
//     first lexicon question; the ids left open go to the row's list.
//  4. residue (one 1024-thread workgroup per compute unit): the open ids of the
//     whole batch dealt evenly, a few per wave; each is judged to its end, from
//     its class's record with its own lexicon flags and, past the record, by DFA
//     steps over its bytes (section 4.1), later shifts on the lane's LDS overlay;
//     the allowed ids are OR-ed into the mask.  An id whose stack area is too
//     small is judged again with a large one.  The last chunk of a row writes its
//     status (Proposition 8: a viable configuration has a nonempty mask).
//  5. with a mask cache or a context-independent word cache: the rows' new entries
//     are published.
// grid_apply is a streaming in-place -inf fill of the masked logits.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <mutex>
#include <cstdint>
#include <string>

#include "fill.h"
#include "host.h"
#include "lexhash.h"
#include "rolling_hash.h"

namespace grid {
int fail(int code, const std::string& msg);
void clear_error();
}  // namespace grid

using namespace grid;

namespace {

constexpr int kBlock = 256;          // workgroup size of most kernels
constexpr int kProThreads = 1024;    // prologue workgroup size (one per row)
constexpr int kStackWin = 256;       // top of the row's stack kept in LDS (prologue)
constexpr int kPostCap = 14;         // overlay states recorded per first shift
constexpr int kGuard = 4096;         // reduce-chain steps without the stack falling, at most: only empty
                                     // reductions can take more (see lr_chain and chain_shift)
constexpr int kUnitGuard = 1 << 14;  // reductions of one entry in a row, at most: LR states have 14 bits
constexpr uint32_t kRowValid = 0x600D;
constexpr size_t kWsHead = 256;      // workspace head (reserved)

constexpr int kWalkWin = 64;         // top stack entries of each row in the walk's LDS
constexpr int kJudgeThreads = 512;   // workgroup size of the judge kernel

// stream kernel
constexpr int kStreamThreads = 512;
constexpr int kStreamWaves = kStreamThreads / 64;
constexpr int kStepIds = 512;        // ids of one wave step (8 per lane)
constexpr int kOpenList = 8192;      // open ids a row lists at most
constexpr int kOpenLocal = 1024;     // and one stream workgroup
constexpr uint32_t kListFull = 1u << 30;  // in a row's count: some open ids are not listed

// residue kernel
constexpr int kResThreads = 1024;
constexpr int kResWaves = kResThreads / 64;
constexpr int kChunkMin = 64;        // open ids a workgroup takes at a time, about
constexpr int kChunkMax = 512;
constexpr int kQueue = kChunkMax + kStepIds;  // and at most (a whole last step)
constexpr int kTableThreads = kResThreads - kChunkMax;  // those that take no listed id stage the tables
constexpr int kCountRegs = 4;        // rows' counts a lane keeps
constexpr int kLanesMax = 32;        // ids a wave takes at a time, at most
constexpr int kFastLane = 16;        // per-lane stack area of a walk: its overlay
constexpr int kSlowLane = 512;       // the same for a walk that outgrew it
constexpr int kSlowWaves = kResWaves * kLanesMax * kFastLane / kSlowLane;  // walks that fit in its place
static_assert(kStackWin <= kProThreads, "a prologue thread per stack-window entry");
constexpr uint32_t kLdsMax = 160 * 1024;
constexpr uint32_t kLdsStatic = 4096;     // LDS the judge and mask kernels declare statically, at most
constexpr uint32_t kTablesMax = 133328;   // lexer and LR tables, the largest that are supported

struct Tables {
  const uint16_t* dfa;        // [S*C]
  const uint8_t* bclass;      // [256]
  const uint32_t* acc_off;    // [S+1]
  const uint8_t* acc_list;
  const uint32_t* live;       // [S*8]
  const uint16_t* action;     // [NS*(T+1)] LALR actions
  const uint32_t* prod;       // [P] lhs | length << 16
  const uint16_t* mact;       // [NS*(T+1)] the mask kernels' actions
  const uint32_t* mred;       // their reductions, when entries are indices
  int mbits;                  // bits of the left side in a reduce entry, 0: an index
  const uint32_t* term_info;  // [T]
  const uint32_t* pstate;     // [NS][parse_record_words(tw)]
  const uint32_t* predx;
  const uint2* ghash;         // [H]: key, target
  const uint4* spell_rec;     // [spellings]: head lo, head hi, first id | multi << 31, length | chunk << 8
  const uint4* spell_tail;    // chunk u: bytes 8..23 of spelling u; overflow chunks after
  const uint32_t* spell_of_id;  // [V]
  const uint16_t* lex_flags;
  const uint32_t* lex_hash;
  const uint32_t* lex_slots;
  const uint4* lex_prefix;
  const uint4* lex_stride;    // [entries][2]
  const uint32_t* lex_token;  // [slots][V] token flags at start offsets 0 and 1
  const uint32_t* id_head;    // [V] first byte | second byte << 8 | 0x10000 if it has one
  const uint8_t* lex_toksum;  // [slots][V] nonzero bytes of each token-flag entry
  const uint32_t* lex_child;  // [nodes][8] child bytes of every lexicon-trie node
  const uint16_t* cmap;       // class of each token per lexer state [S][V]
  const uint32_t* coff;       // [S+1] first class record of each state
  const uint4* crec;          // class records
  int S, C, T, N, NS, V, W, n_slots, eos_id;
  int max_classes;            // largest class count of one lexer state
  int prog;                   // the classes are those of the reduced programs
  const uint16_t* pshift;      // shift targets per LR state
  const uint16_t* go;          // dense GOTO [states][N], kNoGoto none
  int tw, n_pstate, n_predx, n_pshift, n_acc, hbits;
  const uint32_t* state_sym;  // [NS] accessing symbol of each LR state (rolling hash)
  const uint64_t* stack_hash; // rolling hash of every stack entry, or null (mask cache key)
  uint8_t* cache;             // mask cache (null: off)
  uint32_t cache_mask;        // entries - 1
  uint32_t cache_flags;       // GRID_CACHE_*
  uint32_t cache_stride;      // bytes per entry
  uint32_t fp;                // fingerprint of the compiled handle
  uint8_t* ci_cache;          // context-independent-words cache (null: off)
  uint32_t ci_mask;           // entries - 1
  uint32_t ci_flags;          // GRID_CI_*
  uint32_t ci_stride;         // bytes per entry
  uint32_t family_fp;         // fingerprint of the lexer and vocabulary (the grammar family)
  uint32_t ign[8];            // the ignored terminals (term_info bit 0), one bit each
};

// ------------------------------------------------------------- mask cache
// Entry: a 64-byte key/state header, then the row's W mask words.  state 0
// empty, 1 claimed (being written), 2 published.
struct CacheEntry {
  uint32_t state, fp, q, slot, flags, rem_len, rem_lo, rem_hi, lexnode, depth;
  uint32_t h[4];  // 128-bit content hash of the stack
  uint32_t eos, status;
};
static_assert(sizeof(CacheEntry) == 64, "cache entry header is 64 bytes");
constexpr int kCacheProbes = 8;
constexpr uint64_t kRollingKeyTag = 0x524F4C4C494E4748ull;  // key words of a rolling-hash key
constexpr uint32_t kRowCached = 0xCAC4;  // RowHeader::valid of a row served from the cache

__host__ __device__ inline uint32_t cache_stride_of(int W) { return 64u + ((uint32_t)W * 4u + 15u) / 16u * 16u; }

// Context-independent-words cache entry: a 96-byte header (state word: 0
// empty, 1 claimed, 2 published; the key), then W words holding the allowed
// bits of the row's context-independent tokens -- those whose lexeme program
// from the scan state ends no lexeme, so that their verdict depends only on
// the scan state, the pending remainder, A(sigma) and the lexicon (section
// 4.2, CI / CD split; the end-of-sequence bit is never stored).
constexpr int kCiKeyWords = 17;
constexpr uint32_t kCiHeader = 96;
__host__ __device__ inline uint32_t ci_stride_of(int W) { return kCiHeader + ((uint32_t)W * 4u + 15u) / 16u * 16u; }
// A class whose tokens end no lexeme: byte 0 continues the pending lexeme and
// no later byte ends one.
__host__ __device__ inline bool ci_class(uint32_t w0) { return (w0 & (kClassEndsMask | kClassP0 | kClassWalk)) == 0u; }

// One stack entry's share of the stack hash: a 64-bit mix of (position,
// state) under a salt; the hash is the sum over the stack, so every thread
// adds its positions in any order.
__device__ inline uint64_t stack_mix(uint32_t i, uint32_t s, uint64_t salt) {
  uint64_t z = ((uint64_t)i << 32 | s) + salt;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

// ---------------------------------------------------------------- workspace
// Row header, written by the prologue: everything the walk needs of a row
// besides the tables that follow it (the walk copies header, tables and
// stack window to LDS in one piece).
struct RowHeader {
  uint32_t A[8];              // allowed terminals of sigma
  uint32_t R[8];              // terminals whose category the row's lexicon restricts
  uint32_t slot[kSlotWords];  // the row's lexicon slot record (the words Slot holds; the rest 0)
  uint32_t cont[8];           // bytes b such that (pending lexeme) b prefixes a lexicon word
  uint32_t eos_ok;
  uint32_t valid;
  int32_t winner;             // pending lexeme's winner at an emission, -1 none
  uint32_t wkind;             // 0 no winner, 1 the winner is ignored, 2 it shifts
  uint32_t stk_off, stk_depth, q, lexnode;
  uint32_t rem_lo, rem_hi, rem_len;  // first 8 bytes and length of the pending lexeme
  int32_t pstat;              // status bits from the prologue
  unsigned long long done;    // the row's residue chunks that ended (see residue_kernel)
  uint32_t nonempty;          // the stream allowed some id
  int32_t cache_slot;         // mask-cache entry this row publishes to, -1 none
  int32_t fstat;              // final row status
  uint32_t cls_base, n_cls;   // the row's lexer state's class records
  uint32_t slot_id;           // the row's lexicon slot
  int32_t ci_hit;             // context-independent-words entry serving this row, -1 none
  int32_t ci_claim;           // such an entry this row publishes to, -1 none
  uint32_t pad[6];
};
static_assert(sizeof(RowHeader) == 256, "row header is 256 bytes");

struct Post {                 // stack after shifting one allowed terminal
  uint16_t k;                 // shared base entries kept
  uint8_t m;                  // overlay entries
  uint8_t ok;
  uint16_t ov[kPostCap];
};
static_assert(sizeof(Post) == 32, "post entry is 32 bytes");
static_assert(kPostCap == 14, "the walk decodes a post entry as two 16-byte halves");

struct RowLayout {
  size_t win, usets, acc, block, post, codes, cats, cont2, open, n_open, list, total;
};

__host__ __device__ inline uint32_t pad16(uint32_t x) { return (x + 15u) & ~15u; }

// One row's workspace: header; the top kWalkWin states of the stack; the allowed sets with the ignored terminals added, from
// sigma and after each allowed terminal's shift; the packed accept lists; the
// stacks after each allowed terminal's shift; [the block the residue kernel keeps in LDS ends here]; a
// verdict byte per class of the row's lexer state and, where the stream settles
// it by prefix flags, its categories; for every byte b that continues the pending lexeme in
// the lexicon, the bytes that continue it after b (256 bits per b, rows of
// other b unwritten); the ids the stream kernel left open, a bit each (16 words per wave step, written
// where the step has some), their number per step (u16), and, when the row's
// are few enough, a list of them (id, class | its code << 16).
__host__ __device__ inline int open_list_cap(int V) { return V < kOpenList ? V : kOpenList; }
__host__ __device__ inline int stream_steps(int V) { return (V + kStepIds - 1) / kStepIds; }
__host__ __device__ inline RowLayout row_layout(int T, int S, int V, int max_classes) {
  RowLayout L;
  size_t o = sizeof(RowHeader);
  L.win = o;
  o += kWalkWin * 2;
  L.usets = o;
  o += (size_t)(1 + T) * 32;
  L.acc = o;
  o += pad16((uint32_t)S * 4u);
  L.post = o;
  o += (size_t)T * sizeof(Post);
  L.block = o;
  L.codes = o;
  o += (size_t)pad16((uint32_t)max_classes);
  L.cats = o;
  o += (size_t)pad16((uint32_t)max_classes);
  L.cont2 = o;
  o += 256 * 32;
  L.open = o;
  o += (size_t)stream_steps(V) * (kStepIds / 8);
  L.n_open = o;
  o += (size_t)stream_steps(V) * 2;
  o = (o + 15) & ~(size_t)15;
  L.list = o;
  o += (size_t)open_list_cap(V) * 8;
  L.total = (o + 255) & ~(size_t)255;
  return L;
}

__host__ __device__ inline RowLayout row_layout(const Tables& tb) { return row_layout(tb.T, tb.S, tb.V, tb.max_classes); }

#define GRID_LDS_VOID __attribute__((address_space(3))) void
struct StageRegion {
  const uint8_t* src;
  uint8_t* dst;
  uint32_t bytes;
};

// Global -> LDS copies by direct global-to-LDS loads (global_load_lds, 16
// bytes a lane): no registers hold the data on the way, so every load of the
// staging is issued before any is waited for and the whole staging costs
// about one memory round trip.  A region's full 16-byte chunks are cut into
// blocks of 64 (one wave instruction writes 1 KB at a wave-uniform LDS
// address, lane l at +16 l), dealt to the waves of the workgroup round-robin
// across all regions (first = the running block number); a region's last
// partial chunk is copied byte by byte by one thread.  Both ends of every
// region are 16-byte aligned.  The caller runs dma_wait() and a barrier
// before reading the copies.
__device__ inline uint32_t dma_region(const StageRegion& rg, int tid, int nt, uint32_t first) {
  const uint32_t lane = (uint32_t)tid & 63u, wave = (uint32_t)tid >> 6, nw = (uint32_t)nt >> 6;
  const uint32_t full = rg.bytes / 16u, nblk = (full + 63u) / 64u;
  for (uint32_t b = (wave + nw - first % nw) % nw; b < nblk; b += nw) {
    const uint32_t c = b * 64u + lane;
    if (c < full)
      __builtin_amdgcn_global_load_lds((const void*)(rg.src + 16u * c), (GRID_LDS_VOID*)(rg.dst + 64u * 16u * b), 16, 0,
                                       0);
  }
  const uint32_t tail = rg.bytes & 15u;
  if (tail && (uint32_t)tid == (first + nblk) % (uint32_t)nt)
    for (uint32_t i = rg.bytes - tail; i < rg.bytes; ++i) rg.dst[i] = rg.src[i];
  return first + nblk;
}

template <int N>
__device__ inline uint32_t dma_regions(const StageRegion (&rg)[N], int tid, int nt, uint32_t first = 0) {
#pragma unroll
  for (int j = 0; j < N; ++j) first = dma_region(rg[j], tid, nt, first);
  return first;
}

// Waits for this thread's outstanding loads, direct-to-LDS ones included.
__device__ inline void dma_wait() { __builtin_amdgcn_s_waitcnt(0); }

// ------------------------------------------------------- compact LR tables
// Those of the device advance.  The tables and the stack sit in LDS (L = true),
// where LDS-typed pointers make every access an LDS load; a row whose stack
// outgrows its area, or tables too large, are read from global memory (L = false).
#define GRID_LDS __attribute__((address_space(3)))
template <bool L, class T>
struct MemSpace;
template <class T>
struct MemSpace<true, T> {
  typedef GRID_LDS T* ptr;
};
template <class T>
struct MemSpace<false, T> {
  typedef T* ptr;
};
template <bool L, class T>
using mptr = typename MemSpace<L, T>::ptr;
// plain vector types for 8- and 16-byte loads through typed pointers
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
template <bool L, class T>
__device__ inline mptr<L, T> in_mem(T* p) {
  return (mptr<L, T>)p;
}

template <bool L>
struct ParseTabs {
  mptr<L, const uint32_t> st;    // state records, parse_record_words(MW) words each
  mptr<L, const uint32_t> redx;  // extra reduce groups
  mptr<L, const u32x2> gh;       // GOTO (key, target) slots
  mptr<L, const uint16_t> sl;    // shift targets (runs per state)
  mptr<L, const uint16_t> gd;    // dense GOTO [states][N] when dense, else unused
  int T, hbits, N, dense;
};

struct ParseLds {  // byte offsets of the staged tables
  uint32_t st, redx, ghash, sl, gdense, total;
  int dense;  // GOTO as the dense table (else as the hash)
};

__host__ __device__ inline ParseLds parse_lds(const Tables& tb, uint32_t base, bool dense = false) {
  ParseLds L;
  uint32_t o = base;
  L.dense = dense ? 1 : 0;
  L.st = o;
  o += pad16((uint32_t)tb.n_pstate * 4);
  L.redx = o;
  o += pad16((uint32_t)tb.n_predx * 4);
  L.ghash = o;
  if (!dense) o += 8u << tb.hbits;
  L.gdense = o;
  if (dense) o += pad16((uint32_t)(tb.NS * tb.N * 2));
  L.sl = o;
  o += pad16((uint32_t)tb.n_pshift * 2);
  L.total = o - base;
  return L;
}

// The prologue's LR tables in LDS: GOTO as the dense table when it fits
// beside the prologue's own arrays, else as the hash.
constexpr uint32_t kPrologueParseMax = 92 * 1024;
__host__ __device__ inline ParseLds prologue_parse_lds(const Tables& tb) {
  const ParseLds d = parse_lds(tb, 0, true);
  return d.total <= kPrologueParseMax ? d : parse_lds(tb, 0, false);
}

__device__ inline StageRegion parse_region(const Tables& tb, uint8_t* lds, const ParseLds& L, int which) {
  if (which == 0) return {(const uint8_t*)tb.pstate, lds + L.st, (uint32_t)tb.n_pstate * 4};
  if (which == 1) return {(const uint8_t*)tb.predx, lds + L.redx, (uint32_t)tb.n_predx * 4};
  if (which == 3) return {(const uint8_t*)tb.pshift, lds + L.sl, (uint32_t)tb.n_pshift * 2};
  if (L.dense) return {(const uint8_t*)tb.go, lds + L.gdense, (uint32_t)(tb.NS * tb.N * 2)};
  return {(const uint8_t*)tb.ghash, lds + L.ghash, 8u << tb.hbits};
}

// The LR tables in LDS (the caller stages them, see parse_region).
__device__ inline ParseTabs<true> lds_parse(const Tables& tb, uint8_t* lds, const ParseLds& L) {
  return {in_mem<true>((const uint32_t*)(lds + L.st)), in_mem<true>((const uint32_t*)(lds + L.redx)),
          in_mem<true>((const u32x2*)(lds + L.ghash)), in_mem<true>((const uint16_t*)(lds + L.sl)),
          in_mem<true>((const uint16_t*)(lds + L.gdense)), tb.T, tb.hbits, tb.N, L.dense};
}

__device__ inline ParseTabs<false> global_parse(const Tables& tb) {
  return {in_mem<false>(tb.pstate), in_mem<false>(tb.predx), in_mem<false>((const u32x2*)tb.ghash),
          in_mem<false>(tb.pshift), in_mem<false>(tb.go), tb.T, tb.hbits, tb.N, 1};
}

template <bool L>
struct BaseStack {  // the shared read-only stack of one row
  const uint16_t* pool;           // states [0, depth), global
  mptr<L, const uint16_t> win;    // copy of states [lo, depth), or unused with lo = depth
  uint32_t depth, lo;
  __device__ uint16_t at(uint32_t i) const { return i >= lo ? win[i - lo] : pool[i]; }
};

template <bool L>
__device__ __forceinline__ uint16_t goto_of(const ParseTabs<L>& pt, uint32_t s, uint32_t a) {
  if (pt.dense) return pt.gd[__umul24(s, (uint32_t)pt.N) + a];  // states and N below 2^24
  const uint32_t key = goto_key(s, a);
  const uint32_t mask = (1u << pt.hbits) - 1u;
  uint32_t h = goto_slot(key, pt.hbits);
  u32x2 e = pt.gh[h];
  // linear probing; the load factor (at most 2/3) keeps an empty slot
  for (uint32_t i = 0; e.x != key && e.x != 0u && i < mask; ++i) {
    h = (h + 1) & mask;
    e = pt.gh[h];
  }
  return e.x == key ? (uint16_t)e.y : kNoGoto;
}

constexpr uint32_t kNoProd = 0xFFFFFFFFu;  // no production

// Action of the terminal with set word w and bit `bit` in state s:
// kActShiftP (shift, or accept for the end-of-input column), kNoProd
// (error), else the production to reduce.
constexpr uint32_t kActShiftP = 0xFFFFFFFEu;
constexpr uint32_t kNoState = 0xFFFFFFFFu;
template <bool L, int MW>
__device__ __forceinline__ uint32_t action_of(const ParseTabs<L>& pt, uint32_t s, uint32_t w, uint32_t bit) {
  constexpr int R = parse_record_words(MW);
  const mptr<L, const uint32_t> rec = pt.st + s * (uint32_t)R;
  const uint32_t sh = rec[w], rd = rec[MW + w];  // both loads issued together
  const u32x2 me = *(mptr<L, const u32x2>)(rec + 2 * MW);
  const uint32_t hit = (sh | rd) & bit;
  uint32_t a = (sh & bit) ? kActShiftP : (hit ? me.x : kNoProd);
  const uint32_t nx = hit ? 0u : (me.y & 0xFFu);
  mptr<L, const uint32_t> g = pt.redx + (me.y >> 8);
  for (uint32_t e = 0; e < nx; ++e, g += MW + 1)  // the state's other reduce groups
    if (g[1 + w] & bit) {
      a = g[0];
      break;
    }
  return a;
}

// LALR target of the shift of terminal x in state s (x's shift bit is set): entry
// (shift bits below x) of the state's run of shift targets.
template <bool L, int MW>
__device__ __forceinline__ uint16_t shift_target(const ParseTabs<L>& pt, uint32_t s, int x) {
  constexpr int R = parse_record_words(MW);
  static_assert(2 * MW + 2 < R, "the record holds its shift run");
  const mptr<L, const uint32_t> rec = pt.st + s * (uint32_t)R;
  const uint32_t w = (uint32_t)x >> 5;
  uint32_t rank = 0, base = rec[2 * MW + 2];
#pragma unroll
  for (int k = 0; k < MW; ++k) {
    const uint32_t bits = rec[k];
    if ((uint32_t)k < w) rank += (uint32_t)__popc(bits);
    if ((uint32_t)k == w) rank += (uint32_t)__popc(bits & ((1u << (x & 31)) - 1u));
  }
  return pt.sl[base + rank];
}

// Virtual stack base[0,k) ++ ov[0,m) ++ tmp[0,t) (k >= 1): its top state.
// In LDS the three places are one address space, so the address is selected
// and read once; a base entry below the LDS window is read from the pool.
template <bool L>
__device__ __forceinline__ uint16_t stack_at_top(const BaseStack<L>& bs, uint32_t k, int m,
                                                 mptr<L, const uint16_t> ov, int t,
                                                 mptr<L, const uint16_t> tmp) {
  if constexpr (L) {
    const uint32_t i = k - 1u;
    const bool deep = t == 0 && m == 0 && i < bs.lo;
    const mptr<L, const uint16_t> p = t > 0 ? tmp + (t - 1) : (m > 0 ? ov + (m - 1) : bs.win + (deep ? 0u : i - bs.lo));
    uint16_t v = *p;  // a valid LDS address in every case
    if (deep) v = bs.pool[i];
    return v;
  } else {
    if (t > 0) return tmp[t - 1];
    if (m > 0) return ov[m - 1];
    return bs.at(k - 1u);
  }
}

// Pops len entries from base[0,k) ++ ov[0,m) ++ tmp[0,t) (tmp first); false
// if that would empty the stack.
__device__ __forceinline__ bool pop_len(uint32_t len, uint32_t& k, int& m, int& t) {
  const uint32_t dt = min((uint32_t)t, len);
  const uint32_t dm = min((uint32_t)m, len - dt);
  const uint32_t dk = len - dt - dm;
  if (dk >= k) return false;
  t -= (int)dt;
  m -= (int)dm;
  k -= dk;
  return true;
}

// A chain step needs the state under the popped entries.  With one entry
// popped it is the state that was under the top (`below`, when known); with
// none, the top itself; else it is read -- only then, so a run of unit
// reductions waits for no stack read.
template <bool L>
__device__ __forceinline__ uint32_t goto_source(const BaseStack<L>& bs, uint32_t len, uint32_t s, uint32_t below,
                                                uint32_t k, int m, mptr<L, const uint16_t> ov, int t,
                                                mptr<L, const uint16_t> tmp) {
  uint32_t sb = len == 0 ? s : below;
  if (len > 1 || sb == kNoState) sb = stack_at_top<L>(bs, k, m, ov, t, tmp);
  return sb;
}

// ---------------------------------------------------- reduce chains of the mask
// The mask kernels run every reduce chain on two dense tables: the action of
// (state, terminal) with all that these two decide done ahead (host:
// build_mask_actions), and GOTO.  At every step a chain holds one state above a
// prefix of its stack, so a step is one action read, at most one stack read and
// one GOTO read, with no pushes to keep -- a step of the compact tables (state
// record, bit tests, extra reduce groups, overlay) took about twice as long.
template <bool L>
struct LrTabs {
  mptr<L, const uint16_t> act, go;  // [states][T + 1], [states][N]
  const uint32_t* red;              // reductions of indexed entries (bits = 0), global
  uint32_t T1, N;
  int bits;
};

struct LrLds {  // byte offsets of the two tables in LDS
  uint32_t act, go, total;
};
__host__ __device__ inline LrLds lr_lds(const Tables& tb, uint32_t base) {
  LrLds l;
  l.act = base;
  l.go = l.act + pad16((uint32_t)tb.NS * (uint32_t)(tb.T + 1) * 2u);
  l.total = l.go + pad16((uint32_t)tb.NS * (uint32_t)tb.N * 2u) - base;
  return l;
}
// The largest tables the mask kernels keep in LDS beside what else they stage;
// larger ones are read from global memory.
constexpr uint32_t kLrLdsMax = 96 * 1024;
__host__ __device__ inline bool lr_in_lds(const Tables& tb) { return lr_lds(tb, 0).total <= kLrLdsMax; }

__device__ inline uint32_t dma_lr(const Tables& tb, uint8_t* lds, const LrLds& l, int tid, int nt, uint32_t first) {
  const StageRegion rg[2] = {{(const uint8_t*)tb.mact, lds + l.act, (uint32_t)tb.NS * (uint32_t)(tb.T + 1) * 2u},
                             {(const uint8_t*)tb.go, lds + l.go, (uint32_t)tb.NS * (uint32_t)tb.N * 2u}};
  return dma_regions<2>(rg, tid, nt, first);
}
template <bool L>
__device__ inline LrTabs<L> lr_tabs(const Tables& tb, uint8_t* lds, const LrLds& l) {
  if constexpr (L)
    return {in_mem<true>((const uint16_t*)(lds + l.act)), in_mem<true>((const uint16_t*)(lds + l.go)), tb.mred,
            (uint32_t)tb.T + 1u, (uint32_t)tb.N, tb.mbits};
  else
    return {in_mem<false>(tb.mact), in_mem<false>(tb.go), tb.mred, (uint32_t)tb.T + 1u, (uint32_t)tb.N, tb.mbits};
}

// A row's stack as the chains see it: base[0, k) ++ ov[0, m), the base read
// from its LDS window (entries from lo on) or the pool.
struct ChainStack {
  const uint16_t* pool;
  mptr<true, const uint16_t> win;
  uint32_t lo, k;
  mptr<true, const uint16_t> ov;
  uint32_t m;
  __device__ __forceinline__ uint32_t at(uint32_t i) const {
    const bool over = i >= k, deep = !over && i < lo;
    const mptr<true, const uint16_t> p = over ? ov + (i - k) : win + (deep ? 0u : i - lo);
    uint32_t v = *p;  // a valid LDS address in every case
    if (deep) v = pool[i];
    return v;
  }
};

// Reduce chain of terminal x from the stack: in, s is its top state and n the
// entries below it; out, the stack that x is shifted on is its first n entries
// and s, moved tells whether some reduction ran.  Returns the last action: 0
// (refused), or a kMactShift entry.  A legal chain can be as long as the stack is
// deep, so only the steps since the stack last fell are counted: those put one
// state after another above the same entry, never one of them twice (a grammar
// where they did would be ambiguous), so no chain reaches the count.
template <bool L>
__device__ __forceinline__ uint32_t lr_chain(const LrTabs<L>& lt, const ChainStack& st, uint32_t x, uint32_t& n,
                                             uint32_t& s, bool& moved) {
  uint32_t a = lt.act[__umul24(s, lt.T1) + x];
  uint32_t e = n ? st.at(n - 1u) : 0u;  // the state below s
  moved = false;
  for (int guard = 0; guard < kUnitGuard && a - 1u < kMactShift - 1u; ++guard) {  // a reduction
    uint32_t lhs = a & ((1u << lt.bits) - 1u), pops = a >> lt.bits;
    if (lt.bits == 0) {  // uniform
      const uint32_t r = lt.red[a - 1u];
      lhs = r & 0xFFFFu;
      pops = r >> 16;
    }
    if (pops > n) return 0u;  // it would empty the stack
    if (pops > 1u) {
      n -= pops - 1u;
      e = st.at(n - 1u);
      guard = 0;
    }
    s = lt.go[__umul24(e, lt.N) + lhs];
    moved = true;
    if (s == kNoGoto) return 0u;
    a = lt.act[__umul24(s, lt.T1) + x];
  }
  return a & kMactShift ? a : 0u;
}

// The stack after a chain's shift (a its last action): base entries kept and
// overlay, written over ov[0, m).  False if the overlay outgrows cap, or empty
// reductions before the shift take more than kGuard steps.
__device__ __forceinline__ bool lr_commit(const Tables& tb, uint32_t a, uint32_t x, uint32_t n, uint32_t s, bool moved,
                                          uint32_t& k, uint32_t& m, mptr<true, uint16_t> ov, uint32_t cap) {
  if (moved) {
    m = n > k ? n - k : 0u;
    k = min(k, n);
    if (m >= cap) return false;
    ov[m++] = (uint16_t)s;
  }
  if (a & kMactPushed) {  // the states the empty reductions push first (rare: the LALR tables in global memory)
    const uint32_t floor = m, T1 = (uint32_t)tb.T + 1u;
    uint32_t top = s;
    int guard = 0;
    for (; guard < kGuard; ++guard) {
      const uint32_t la = tb.action[top * T1 + x];
      if ((la & 0xC000u) != kActReduce) break;
      const uint32_t pr = tb.prod[la & 0x3FFFu], len = pr >> 16;
      if (len > m - floor) return false;
      m -= len;
      const uint32_t g = tb.go[(m > floor ? (uint32_t)ov[m - 1u] : s) * (uint32_t)tb.N + (pr & 0xFFFFu)];
      if (g == kNoGoto || m >= cap) return false;
      ov[m++] = (uint16_t)g;
      top = g;
    }
    if (guard == kGuard) return false;
  }
  if (m >= cap) return false;
  ov[m++] = (uint16_t)(a & 0x3FFFu);
  return true;
}

// ---------------------------------------------------------- lexicon helpers
struct Slot {
  uint32_t fbase, hbase, hmask, restricted, nodes, pbase, pmask, sbase, smask;
};

__device__ inline Slot slot_of(const uint32_t* r) { return {r[0], r[1], r[2], r[3], r[4], r[5], r[6], r[7], r[8]}; }

__device__ inline Slot load_slot(const Tables& tb, int s) { return slot_of(tb.lex_slots + (size_t)s * kSlotWords); }

__device__ inline uint32_t lex_child(const Tables& tb, const Slot& sl, uint32_t node, uint32_t b) {
  if (node == kNoLex) return kNoLex;
  uint32_t key = lex_key(node, b);
  uint32_t h = lex_hash(key) & sl.hmask;
  for (uint32_t probe = 0; probe <= sl.hmask; ++probe, h = (h + 1) & sl.hmask) {
    uint2 e = reinterpret_cast<const uint2*>(tb.lex_hash)[sl.hbase + h];
    if (e.x == key) return e.y;
    if (e.x == 0) return kNoLex;
  }
  return kNoLex;
}

__device__ inline uint32_t lex_flags_of(const Tables& tb, const Slot& sl, uint32_t node) {
  return node == kNoLex ? 0u : tb.lex_flags[sl.fbase + node];
}

// Lexicon node and flags of the prefix given by its bytes (length 1..8): one
// probe in the slot's prefix table.  (0, kNoLex) if it is no word's prefix.
__device__ inline uint2 lexp_find(const Tables& tb, const Slot& sl, uint64_t bytes, uint32_t len) {
  const uint32_t lo = (uint32_t)bytes, hi = (uint32_t)(bytes >> 32);
  uint32_t h = lexp_hash(lo, hi, len) & sl.pmask;
  for (uint32_t probe = 0; probe <= sl.pmask; ++probe, h = (h + 1) & sl.pmask) {
    const uint4 e = tb.lex_prefix[sl.pbase + h];
    const uint32_t el = e.z & 0xFFFFu;
    if (el == 0) break;
    if (e.x == lo && e.y == hi && el == len) return make_uint2(e.z >> 16, e.w);
  }
  return make_uint2(0u, kNoLex);
}

// Flags and node of the lexicon-trie node below node anc (at a depth that is
// a multiple of 8) reached by len (1..8) more bytes: one probe in the slot's
// stride table.  (0, kNoLex) if no word has that prefix.
__device__ inline uint2 lexs_find(const Tables& tb, const Slot& sl, uint32_t anc, uint64_t bytes, uint32_t len) {
  const uint32_t lo = (uint32_t)bytes, hi = (uint32_t)(bytes >> 32);
  uint32_t h = lexs_hash(anc, lo, hi, len) & sl.smask;
  for (uint32_t probe = 0; probe <= sl.smask; ++probe, h = (h + 1) & sl.smask) {
    const uint4 e = tb.lex_stride[2 * (size_t)(sl.sbase + h)];
    const uint32_t el = e.w & 0xFFFFu;
    if (el == 0) break;
    if (e.x == anc && e.y == lo && e.z == hi && el == len) return make_uint2(e.w >> 16, tb.lex_stride[2 * (size_t)(sl.sbase + h) + 1].x);
  }
  return make_uint2(0u, kNoLex);
}

__device__ inline uint64_t low_bytes(uint64_t w, uint32_t n) { return n >= 8 ? w : w & ((1ull << (8 * n)) - 1ull); }

// Lexicon flags of a lexeme of len (1..24) bytes held in b0 b1 b2
// (little-endian, 8 bytes a word): at most three probes (prefix table, then
// stride table).
__device__ __forceinline__ uint32_t lex_flags_bytes(const Tables& tb, const Slot& sl, uint64_t b0, uint64_t b1,
                                                    uint64_t b2, uint32_t len) {
  uint32_t n = min(len, 8u);
  uint2 f = lexp_find(tb, sl, low_bytes(b0, n), n);  // (flags, node)
  while (len > 8u) {                                 // eight more bytes a stride
    if (f.y == kNoLex) return 0u;
    len -= 8u;
    b0 = b1;
    b1 = b2;
    n = min(len, 8u);
    f = lexs_find(tb, sl, f.y, low_bytes(b0, n), n);
  }
  return f.x;
}

__device__ inline bool bit_of(const uint32_t* s, int t) { return (s[t >> 5] >> (t & 31)) & 1u; }

// What a lane needs to judge terminals: term info, ignored set I, the row's
// restricted set R and the live-terminal sets of the lexer DFA (MW words per
// state, stride lstride).
struct TermView {
  const uint32_t* tinfo;
  const uint32_t* I;
  const uint32_t* R;
  const uint32_t* live;
  int lstride;
};

// Pending lexeme's winner at an emission: the first accept-list entry (highest
// priority, ties to the lower id) that is ignored or allowed and passes the
// lexicon word test.  -1 if none.  lf_of() yields the lexeme's lexicon flags
// and is called at most once, only for an allowed candidate whose category is
// restricted.
template <int MW, class LexFlags>
__device__ inline int winner_of(const TermView& tv, const uint32_t* acc_off, const uint8_t* acc_list,
                                const uint32_t (&acur)[MW], int q, LexFlags lf_of) {
  uint32_t lf = 0;
  bool have_lf = false;
  for (uint32_t j = acc_off[q]; j < acc_off[q + 1]; ++j) {
    const int t = acc_list[j];
    bool ok = bit_of(tv.I, t);
#pragma unroll
    for (int w = 0; w < MW; ++w)
      if (w == (t >> 5)) ok = ok || ((acur[w] >> (t & 31)) & 1u);
    if (!ok) continue;
    if (bit_of(tv.R, t)) {
      if (!have_lf) {
        lf = lf_of();
        have_lf = true;
      }
      if (!((lf >> (8 + ((tv.tinfo[t] >> 8) & 0xFFu))) & 1u)) continue;
    }
    return t;
  }
  return -1;
}

// -------------------------------------------------- CI-words cache key
// The key of a row's context-independent words (section 4.3): per handle
// (T1, Definition 5's key) -- the handle's fingerprint, the scan state q, the
// lexicon slot, the pending remainder (empty flag, length, first 8 bytes,
// lexicon node) and A(sigma) -- or, with GRID_CI_FAMILY (the cross-family
// tier T2), the grammar family's fingerprint (lexer and vocabulary: every
// role projection of one dialect shares it, since projections never
// renumber terminals) and the slot's schema fingerprint, which scopes every
// entry of a lexicon-bearing producer (Remark 1).  With GRID_CI_GENN the T2
// remainder is taken in the genN scanner normal form: under this build's
// gap-free lexers a remainder that has accepted has its last accept at its
// end, so (p, q, v) = (q, q, empty) and the bytes drop out of the key -- only
// under the lexicon-visibility guard (no terminal the row's lexicon
// restricts is live or accepting in q); otherwise, or while the remainder
// has not accepted, the raw remainder stays in the key.
__device__ inline void ci_key(const Tables& tb, const grid_config& cfg, const Slot& sl, const uint32_t (&a_sig)[8],
                              const uint32_t* R, uint32_t (&key)[kCiKeyWords]) {
  const bool family = (tb.ci_flags & GRID_CI_FAMILY) != 0;
  const bool empty = (cfg.flags & 1u) != 0;
  bool genn = false;
  if (family && (tb.ci_flags & GRID_CI_GENN)) {
    bool guard = true;
    const uint32_t* lv = tb.live + (size_t)cfg.q * 8;
    for (int w = 0; w < 8; ++w) guard = guard && (lv[w] & R[w]) == 0u;
    const bool accepting = tb.acc_off[cfg.q + 1] > tb.acc_off[cfg.q];
    for (uint32_t j = tb.acc_off[cfg.q]; j < tb.acc_off[cfg.q + 1]; ++j) guard = guard && !bit_of(R, tb.acc_list[j]);
    genn = guard && (accepting || empty);
  }
  const uint32_t rem_lo = (uint32_t)cfg.rem_head[0] | (uint32_t)cfg.rem_head[1] << 8 |
                          (uint32_t)cfg.rem_head[2] << 16 | (uint32_t)cfg.rem_head[3] << 24;
  const uint32_t rem_hi = (uint32_t)cfg.rem_head[4] | (uint32_t)cfg.rem_head[5] << 8 |
                          (uint32_t)cfg.rem_head[6] << 16 | (uint32_t)cfg.rem_head[7] << 24;
  // (which tokens are context-independent depends on the class tables in use)
  key[0] = (family ? (genn ? 3u : 2u) : 1u) | (tb.prog ? 8u : 0u);
  key[1] = family ? tb.family_fp : tb.fp;
  key[2] = cfg.q;
  key[3] = family ? tb.lex_slots[(size_t)cfg.slot * kSlotWords + 9] : (uint32_t)cfg.slot;
  key[4] = empty ? 1u : 0u;
  key[5] = genn || empty ? 0u : cfg.rem_len;
  key[6] = genn || empty ? 0u : rem_lo;
  key[7] = genn || empty ? 0u : rem_hi;
  key[8] = genn || empty ? 0u : cfg.lexnode;
#pragma unroll
  for (int k = 0; k < 8; ++k) key[9 + k] = a_sig[k];
  (void)sl;
}

// Accept list of a state in one word: its first three terminals, its length in
// the top byte.
__device__ __forceinline__ uint32_t pack_accepts(const uint32_t* acc_off, const uint8_t* acc_list, int q) {
  const uint32_t o = acc_off[q], n = acc_off[q + 1] - o;
  uint32_t w = n << 24;
  for (uint32_t j = 0; j < 3u; ++j)
    if (j < n) w |= (uint32_t)acc_list[o + j] << (8u * j);
  return w;
}

// The number of open ids of each of the B rows (after the rows' areas).
__device__ __forceinline__ uint32_t* open_counts(uint8_t* ws, size_t rbytes, int B) {
  return (uint32_t*)(ws + kWsHead + (size_t)B * rbytes);
}

// The prologue's dynamic LDS: the chains' tables (when they fit), then (when they
// fit beside them) the lexer's accept lists and live sets and the terminal
// info.
struct ProLds {
  LrLds lr;
  uint32_t acc_off, acc_list, live, tinfo, total;
  int lexer;  // the lexer tables are staged (else read from global memory)
};
constexpr uint32_t kPrologueLdsMax = 128 * 1024;
__host__ __device__ inline ProLds prologue_lds(const Tables& tb) {
  ProLds P;
  P.lr = lr_lds(tb, 0);
  uint32_t o = lr_in_lds(tb) ? P.lr.total : 0u;
  const uint32_t base = o;
  P.acc_off = o;
  o += pad16((uint32_t)(tb.S + 1) * 4u);
  P.acc_list = o;
  o += pad16((uint32_t)tb.n_acc);
  P.live = o;
  o += pad16((uint32_t)tb.S * 32u);
  P.tinfo = o;
  o += pad16((uint32_t)tb.T * 4u);
  P.lexer = o <= kPrologueLdsMax ? 1 : 0;
  P.total = P.lexer ? o : base;
  return P;
}

// ---------------------------------------------------------------- prologue
// One workgroup per row.  Phase 1: every terminal's reduce chain and shift from
// sigma, a thread each (A(sigma) is the ballot of those that shifted), with the
// lexicon continuation bits of the pending lexeme beside them; then the allowed
// set of the stack after each allowed terminal's shift, a wave per 64 terminals,
// the end of input one of them; then the pending lexeme's winner and the row
// block.  Bound by the longest reduce chain and the staging of the tables: 12.9 us
// at 32 DML rows (V = 151,936), 17.7 with the compact tables and a set simulation.
template <int MW, bool L>
__global__ __launch_bounds__(kProThreads) void prologue_kernel(Tables tb, const grid_config* __restrict__ cfgs,
                                                          const uint16_t* __restrict__ pool,
                                                          uint32_t* __restrict__ mask,
                                                          uint8_t* __restrict__ eos_out,
                                                          int32_t* __restrict__ status,
                                                          uint8_t* __restrict__ ws, size_t rbytes) {
  extern __shared__ __align__(16) uint8_t plds[];
  const int row = blockIdx.x;
  const int tid = threadIdx.x;
  if (tid == 0) open_counts(ws, rbytes, (int)gridDim.x)[row] = 0u;
  __shared__ uint16_t win[kStackWin];
  __shared__ uint32_t A[8], I[8], R[8];
  __shared__ int bad, overflow, winner, eos_ok, eos_sigma, cache_hit;
  __shared__ uint8_t eos_after[256];  // end-of-sequence test after shifting each candidate winner
  __shared__ Post posts[256];          // stack after shifting each allowed terminal
  __shared__ uint32_t a2_s[256][MW];   // allowed set after shifting each allowed terminal
  __shared__ uint8_t alist[256];       // the allowed terminals in order
  __shared__ unsigned long long hacc[2];
  uint8_t* rw = ws + kWsHead + (size_t)row * rbytes;
  RowHeader* hdr = (RowHeader*)rw;
  const RowLayout RL = row_layout(tb);
  Post* post = (Post*)(rw + RL.post);
  uint32_t* usets = (uint32_t*)(rw + RL.usets);
  const grid_config cfg = cfgs[row];
  const ProLds PR = prologue_lds(tb);
  const uint32_t depth = cfg.stk_depth;
  const uint32_t lo = depth > (uint32_t)kStackWin ? depth - kStackWin : 0;
  // one round trip to memory: the LR tables (and the lexer's accept lists and
  // live sets and the terminal info) go straight to LDS while every thread
  // loads one entry of the top kStackWin stack entries
  const bool shape_ok = cfg.q < tb.S && cfg.slot < tb.n_slots && depth >= 1;  // uniform
  uint32_t first = 0;
  if (L) first = dma_lr(tb, plds, PR.lr, tid, kProThreads, 0);
  if (PR.lexer) {
    const StageRegion rg[4] = {{(const uint8_t*)tb.acc_off, plds + PR.acc_off, (uint32_t)(tb.S + 1) * 4u},
                               {tb.acc_list, plds + PR.acc_list, (uint32_t)tb.n_acc},
                               {(const uint8_t*)tb.live, plds + PR.live, (uint32_t)tb.S * 32u},
                               {(const uint8_t*)tb.term_info, plds + PR.tinfo, (uint32_t)tb.T * 4u}};
    dma_regions<4>(rg, tid, kProThreads, first);
  }
  const uint32_t* acc_off = PR.lexer ? (const uint32_t*)(plds + PR.acc_off) : tb.acc_off;
  const uint8_t* acc_list = PR.lexer ? (const uint8_t*)(plds + PR.acc_list) : tb.acc_list;
  const uint32_t* live = PR.lexer ? (const uint32_t*)(plds + PR.live) : tb.live;
  const uint32_t* tinfo = PR.lexer ? (const uint32_t*)(plds + PR.tinfo) : tb.term_info;
  uint32_t s_top = 0;
  if (shape_ok && tid < kStackWin && lo + (uint32_t)tid < depth) s_top = pool[cfg.stk_off + lo + tid];
  // the row's lexicon slot, its class range and this thread's terminal info,
  // in the same round trip
  const Slot sl = shape_ok ? load_slot(tb, cfg.slot) : Slot{0, 0, 0, 0, 0, 0, 0, 0, 0};
  const uint32_t cls_lo = shape_ok ? tb.coff[cfg.q] : 0u, cls_hi = shape_ok ? tb.coff[cfg.q + 1] : 0u;
  const uint32_t ti = tid < tb.T ? tb.term_info[tid] : 0u;
  const LrTabs<L> lt = lr_tabs<L>(tb, plds, PR.lr);
  if (tid == 0) {
    int b = shape_ok ? 0 : 1;
    if (!b && cfg.lexnode != kNoLex && cfg.lexnode >= sl.nodes) b = 1;
    bad = b;
    overflow = 0;
    winner = -1;
    eos_ok = 0;
    eos_sigma = 0;
    cache_hit = -1;
    hacc[0] = 0;
    hacc[1] = 0;
  }
  dma_wait();
  __syncthreads();
  const bool sum_hash = tb.cache && !tb.stack_hash;  // the cache key needs the whole stack's content
  if (!bad) {  // every entry is an LR state; the window goes to LDS; the content hash for the cache
    uint64_t h1 = 0, h2 = 0;
    if (tid < kStackWin && lo + (uint32_t)tid < depth) {
      const uint32_t i = lo + (uint32_t)tid;
      if (s_top >= (uint32_t)tb.NS) bad = 1;
      win[tid] = (uint16_t)s_top;
      if (sum_hash) {
        h1 += stack_mix(i, s_top, 0x9E3779B97F4A7C15ull);
        h2 += stack_mix(i, s_top, 0xD1B54A32D192ED03ull);
      }
    }
    for (uint32_t i = tid; i < lo; i += kProThreads) {  // entries below the window
      const uint16_t v = pool[cfg.stk_off + i];
      if (v >= tb.NS) bad = 1;
      if (sum_hash) {
        h1 += stack_mix(i, v, 0x9E3779B97F4A7C15ull);
        h2 += stack_mix(i, v, 0xD1B54A32D192ED03ull);
      }
    }
    if (sum_hash) {
      atomicAdd(&hacc[0], (unsigned long long)h1);
      atomicAdd(&hacc[1], (unsigned long long)h2);
    }
  }
  __syncthreads();
  if (bad) {
    if (tid == 0) {
      hdr->pstat = GRID_ROW_BAD_CONFIG;
      hdr->fstat = GRID_ROW_BAD_CONFIG;
      if (status) status[row] = GRID_ROW_BAD_CONFIG;
      hdr->valid = 0;
      hdr->eos_ok = 0;
      hdr->cache_slot = -1;
      hdr->ci_hit = -1;
      hdr->ci_claim = -1;
      if (eos_out) eos_out[row] = 0;
    }
    return;
  }
  // mask cache: probe the row's key; a published entry is the row's mask, an
  // empty slot on the way is claimed for the row when inserting
  if (tb.cache && tid == 0) {
    // the stack's part of the key: its rolling hash H(top) when the caller
    // keeps one (O(1) to read), else the content sums over every entry
    uint64_t h1 = hacc[0], h2 = hacc[1];
    if (tb.stack_hash) {
      h1 = tb.stack_hash[cfg.stk_off + depth - 1];
      h2 = kRollingKeyTag;
    }
    const uint32_t key[13] = {tb.fp,
                              cfg.q,
                              cfg.slot,
                              cfg.flags & 1u,
                              cfg.rem_len,
                              (uint32_t)cfg.rem_head[0] | (uint32_t)cfg.rem_head[1] << 8 |
                                  (uint32_t)cfg.rem_head[2] << 16 | (uint32_t)cfg.rem_head[3] << 24,
                              (uint32_t)cfg.rem_head[4] | (uint32_t)cfg.rem_head[5] << 8 |
                                  (uint32_t)cfg.rem_head[6] << 16 | (uint32_t)cfg.rem_head[7] << 24,
                              cfg.lexnode,
                              depth,
                              (uint32_t)h1,
                              (uint32_t)(h1 >> 32),
                              (uint32_t)h2,
                              (uint32_t)(h2 >> 32)};
    // home slot: every key word mixed in (rows on one stack but another
    // schema or scan state start elsewhere)
    uint64_t home = h1;
    for (int k = 0; k < 9; ++k) home = stack_mix((uint32_t)k, key[k], home);
    int hit = -1, claim = -1;
    for (int pr = 0; pr < kCacheProbes; ++pr) {
      const uint32_t idx = (uint32_t)(home + (uint64_t)pr) & tb.cache_mask;
      CacheEntry* e = (CacheEntry*)(tb.cache + (size_t)idx * tb.cache_stride);
      const uint32_t st = __hip_atomic_load(&e->state, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT);
      if (st == 2u) {
        const uint32_t* ek = &e->fp;
        bool same = true;
        for (int k = 0; k < 13; ++k) same = same && ek[k] == key[k];
        if (same && (tb.cache_flags & GRID_CACHE_LOOKUP)) {
          hit = (int)idx;
          break;
        }
        continue;
      }
      if (st == 0u) {
        if (!(tb.cache_flags & GRID_CACHE_INSERT)) break;
        if (atomicCAS(&e->state, 0u, 1u) == 0u) {
          uint32_t* ek = &e->fp;
          for (int k = 0; k < 13; ++k) ek[k] = key[k];
          claim = (int)idx;
          break;
        }
      }
    }
    cache_hit = hit;
    hdr->cache_slot = claim;
  } else if (tid == 0) {
    hdr->cache_slot = -1;
  }
  __syncthreads();
  if (cache_hit >= 0) {  // the cached row: mask, EOS byte, status
    const CacheEntry* e = (const CacheEntry*)(tb.cache + (size_t)cache_hit * tb.cache_stride);
    const uint32_t* src = (const uint32_t*)(e + 1);
    uint32_t* dst = mask + (size_t)row * tb.W;
    for (int i = tid; i < tb.W; i += kProThreads) dst[i] = src[i];
    if (tid == 0) {
      hdr->valid = kRowCached;
      hdr->pstat = (int32_t)e->status;
      if (status) status[row] = (int32_t)e->status;
      hdr->eos_ok = e->eos;
      hdr->cache_slot = -1;
      hdr->ci_hit = -1;
      hdr->ci_claim = -1;
      if (eos_out) eos_out[row] = (uint8_t)e->eos;
    }
    return;
  }
  if (tid < 8) {
    I[tid] = tb.ign[tid];
    R[tid] = 0;
    A[tid] = 0;
  }
  const uint32_t s_sigma = win[depth - 1u - lo];  // the top of the stack
  __syncthreads();
  if (tid < tb.T) {  // restricted terminals, one per thread
    const uint32_t c = (ti >> 8) & 0xFFu;
    if (c != 0xFFu && ((sl.restricted >> c) & 1u)) atomicOr(&R[tid >> 5], 1u << (tid & 31));
  }
  const mptr<true, const uint16_t> win_l = in_mem<true>((const uint16_t*)win);
  const TermView tv{tinfo, I, R, live, 8};
  __syncthreads();

  // phase 1: thread x runs terminal x's reduce chain from sigma (x = T: the end
  // of input, so that is the end-of-sequence gate for an empty remainder or an
  // ignored winner): A(sigma) is the set that shifts, and their stacks after
  // the shift go to LDS and the row's workspace.  Meanwhile the threads from
  // 256 on find the bytes that continue the pending lexeme in the lexicon
  // (thread 256 + b for byte b) and, after each, the bytes that continue it
  // further (the child bitmap of that trie node).
  static_assert(kProThreads == 1024, "threads 256 to 511 probe one byte value each");
  const bool rem_empty = (cfg.flags & 1u) != 0;
  const int G = (tb.T + 64) / 64;  // waves over the terminals and the end of input
  const int lane = tid & 63, wave = tid >> 6;
  if (tid >= 256 && tid < 512) {  // whole waves
    const uint32_t b = (uint32_t)tid - 256u;
    const uint32_t n1 = rem_empty ? kNoLex : lex_child(tb, sl, cfg.lexnode, b);
    const bool c = n1 != kNoLex;
    const uint64_t bal = __ballot(c);
    if ((b & 31) == 0) hdr->cont[b >> 5] = (uint32_t)(bal >> (b & 32));
    if (c) {
      const uint4* src = reinterpret_cast<const uint4*>(tb.lex_child + (size_t)(sl.fbase + n1) * 8u);
      uint4* dst = reinterpret_cast<uint4*>(rw + RL.cont2 + (size_t)b * 32u);
      dst[0] = src[0];
      dst[1] = src[1];
    }
  } else if (tid >= 512) {  // the packed accept lists, for the verdicts
    uint32_t* acc = (uint32_t*)(rw + RL.acc);
    for (int q = tid - 512; q < tb.S; q += kProThreads - 512) acc[q] = pack_accepts(acc_off, acc_list, q);
  } else if (wave < G) {
    const ChainStack st{pool + cfg.stk_off, win_l, lo, depth, win_l, 0u};
    uint32_t n = depth - 1u, s = s_sigma, a = 0;
    bool moved = false;
    if (tid <= tb.T) a = lr_chain<L>(lt, st, (uint32_t)tid, n, s, moved);
    const uint64_t bal = __ballot(a != 0u && tid < tb.T);
    if (lane == 0) {
      A[2 * wave] = (uint32_t)bal;
      A[2 * wave + 1] = (uint32_t)(bal >> 32);
    }
    if (tid == tb.T) {
      eos_sigma = a != 0u;
    } else if (a) {
      uint32_t k = depth, m = 0;
      Post& p = posts[tid];
      if (!lr_commit(tb, a, (uint32_t)tid, n, s, moved, k, m, in_mem<true>((uint16_t*)p.ov), kPostCap) || k > 0xFFFFu)
        overflow = 1;
      p.k = (uint16_t)k;
      p.m = (uint8_t)m;
      p.ok = 1;
      uint4* dst = reinterpret_cast<uint4*>(&post[tid]);
      const uint4* src = reinterpret_cast<const uint4*>(&p);
      dst[0] = src[0];
      dst[1] = src[1];
    }
  }
  __syncthreads();
  // phase 2: the allowed set after each allowed terminal's shift, a wave per 64
  // terminals of one set (the ballot is the set), with the end-of-sequence gate
  // after that shift on the end-of-input lane; the last wave finds the pending
  // lexeme's winner and probes the CI words meanwhile
  int nA = 0;
#pragma unroll
  for (int w = 0; w < MW; ++w) nA += __popc(A[w]);
  if (tid < tb.T && bit_of(A, tid)) {
    int rank = 0;  // allowed terminals below tid
#pragma unroll
    for (int w = 0; w < MW; ++w)
      if (w < (tid >> 5)) rank += __popc(A[w]);
      else if (w == (tid >> 5)) rank += __popc(A[w] & ((1u << (tid & 31)) - 1u));
    alist[rank] = (uint8_t)tid;
  }
  __syncthreads();
  constexpr int kSetWaves = kProThreads / 64 - 1;
  for (int j = wave; wave < kSetWaves && j < nA * G; j += kSetWaves) {  // uniform per wave
    const int t = alist[j / G], g = j % G, x = g * 64 + lane;
    const Post& p = posts[t];
    const ChainStack st{pool + cfg.stk_off, win_l, lo, p.k, in_mem<true>((const uint16_t*)p.ov), p.m};
    uint32_t n = (uint32_t)p.k + p.m - 1u, a = 0;
    uint32_t s = st.at(n);
    bool moved = false;
    if (x <= tb.T) a = lr_chain<L>(lt, st, (uint32_t)x, n, s, moved);
    const uint64_t bal = __ballot(a != 0u && x < tb.T);
    if (lane == 0) {
      if (2 * g < MW) a2_s[t][2 * g < MW ? 2 * g : 0] = (uint32_t)bal;
      if (2 * g + 1 < MW) a2_s[t][2 * g + 1 < MW ? 2 * g + 1 : 0] = (uint32_t)(bal >> 32);
    }
    if (x == tb.T) eos_after[t] = a != 0u;
  }
  constexpr int kSetThreads = kSetWaves * 64;
  // the pending lexeme's winner if a byte ends it (the gate wave's first
  // thread, while the set jobs run)
  if (tid == kSetThreads && !rem_empty) {
    uint32_t a0[MW];
#pragma unroll
    for (int w = 0; w < MW; ++w) a0[w] = A[w];
    winner = winner_of<MW>(tv, acc_off, acc_list, a0, cfg.q, [&]() { return lex_flags_of(tb, sl, cfg.lexnode); });
  }
  if (tid == kProThreads - 1) {
    // context-independent words, by the gate wave's last thread while the set
    // jobs run: probe the row's key (A(sigma) is known); a published entry
    // serves the row's CI tokens, an empty slot on the way is claimed
    int ci_hit = -1, ci_claim = -1;
    if (tb.ci_cache && !overflow) {
      uint32_t a_sig[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) a_sig[k] = A[k];
      uint32_t key[kCiKeyWords];
      ci_key(tb, cfg, sl, a_sig, R, key);
      uint64_t home = 0x8F1BBCDC2C2D6A1Bull;
      for (int k = 0; k < kCiKeyWords; ++k) home = stack_mix((uint32_t)k, key[k], home);
      for (int pr = 0; pr < kCacheProbes; ++pr) {
        const uint32_t idx = (uint32_t)(home + (uint64_t)pr) & tb.ci_mask;
        uint32_t* e = (uint32_t*)(tb.ci_cache + (size_t)idx * tb.ci_stride);
        const uint32_t st = __hip_atomic_load(e, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT);
        if (st == 2u) {
          bool same = true;
          for (int k = 0; k < kCiKeyWords; ++k) same = same && e[1 + k] == key[k];
          if (same && (tb.ci_flags & GRID_CI_LOOKUP)) {
            ci_hit = (int)idx;
            break;
          }
          continue;
        }
        if (st == 0u) {
          if (!(tb.ci_flags & GRID_CI_INSERT)) break;
          if (atomicCAS(e, 0u, 1u) == 0u) {
            for (int k = 0; k < kCiKeyWords; ++k) e[1 + k] = key[k];
            ci_claim = (int)idx;
            break;
          }
        }
      }
    }
    hdr->ci_hit = ci_hit;
    hdr->ci_claim = ci_claim;
  }
  __syncthreads();
  const int w = winner;
  const bool w_shifts = w >= 0 && !bit_of(I, w);
  if (tid < tb.T && bit_of(A, tid)) {
#pragma unroll
    for (int k = 0; k < MW; ++k) usets[(1 + tid) * 8 + k] = a2_s[tid][k] | I[k];
  }
  if (tid >= 256 && tid < 264) usets[tid - 256] = A[tid - 256] | I[tid - 256];
  if (tid == 0) eos_ok = (rem_empty || (w >= 0 && !w_shifts)) ? eos_sigma : (w >= 0 ? (int)eos_after[w] : 0);
  __syncthreads();
  {  // the top of the stack for the walks
    uint16_t* wwin = (uint16_t*)(rw + RL.win);
    const uint32_t wlo = depth > (uint32_t)kWalkWin ? depth - kWalkWin : 0u;
    if ((uint32_t)tid < depth - wlo) wwin[tid] = win[wlo + tid - lo];
  }
  if (tid < 8) {
    hdr->A[tid] = A[tid];
    hdr->R[tid] = R[tid];
  }
  if (tid == 0) {  // the slot's table bases and masks (its other words are not used on the device side)
    const uint32_t sw[kSlotWords] = {sl.fbase, sl.hbase, sl.hmask, sl.restricted, sl.nodes, sl.pbase,
                                     sl.pmask, sl.sbase, sl.smask, 0u,       0u,       0u};
#pragma unroll
    for (int k = 0; k < kSlotWords; ++k) hdr->slot[k] = sw[k];
  }
  if (tid == 0) {
    hdr->eos_ok = (uint32_t)eos_ok;
    if (eos_out) eos_out[row] = (uint8_t)eos_ok;
    hdr->winner = w;
    hdr->wkind = w < 0 ? 0u : (w_shifts ? 2u : 1u);
    hdr->stk_off = cfg.stk_off;
    hdr->stk_depth = depth;
    hdr->q = cfg.q;
    hdr->lexnode = cfg.lexnode;
    hdr->rem_lo = (uint32_t)cfg.rem_head[0] | (uint32_t)cfg.rem_head[1] << 8 | (uint32_t)cfg.rem_head[2] << 16 |
                  (uint32_t)cfg.rem_head[3] << 24;
    hdr->rem_hi = (uint32_t)cfg.rem_head[4] | (uint32_t)cfg.rem_head[5] << 8 | (uint32_t)cfg.rem_head[6] << 16 |
                  (uint32_t)cfg.rem_head[7] << 24;
    hdr->rem_len = rem_empty ? 0u : cfg.rem_len;
    hdr->nonempty = 0;
    hdr->done = 0;
    hdr->slot_id = cfg.slot;
    hdr->cls_base = cls_lo;
    hdr->n_cls = cls_hi - cls_lo;
    hdr->pstat = overflow ? GRID_ROW_OVERFLOW : GRID_ROW_OK;
    hdr->valid = kRowValid;
  }
}

struct DfaView {  // lexer DFA by byte class (LDS copy or global)
  const uint16_t* next_;
  const uint8_t* cls_;
  int C;
  __device__ uint32_t cls(uint32_t b) const { return cls_[b]; }
  __device__ int next(int q, uint32_t c) const { return next_[q * C + c]; }
};

// ----------------------------------------------------------- class verdicts
// Codes of a class for a row (2 bits per class in the row's verdict table).
// kVerdictLexicon: the verdict depends on the schema lexicon (a lexeme's
// winner or the trailing lexeme's viability), so each token of the class is
// judged again with its own lexemes' lexicon flags.
constexpr uint32_t kVerdictReject = 0, kVerdictAllow = 1, kVerdictWalk = 2, kVerdictLexicon = 3;
constexpr uint32_t kCodeCi = 4;  // beside kVerdictAllow in a class's byte: its tokens are context-independent

// A lexeme whose lexicon flags were not asked for yet.
constexpr uint32_t kLexOpen = 0xFFFFFFFFu;

// Verdict of one lexeme-program class, or of one of its tokens, for a row.  The
// lexemes the token ends are judged in order against the allowed set the parser
// has at that point: A(sigma) before any shift, the prologue's set after the
// first, the set after the second where it is known.
// Each ended lexeme's winner is the first accept-list entry (priority order)
// that is ignored or allowed and, for a restricted terminal, whose category has
// the lexeme as a word (section 2, L3); the trailing lexeme (state after the
// last byte) must still complete to an allowed or ignored terminal, a restricted
// one only where the lexeme prefixes a word of its category (Definition 2).  An
// ignored unrestricted terminal live there accepts it under any stack.  Lexicon
// flags come from lex.word(i) (lexeme i) and lex.trail().
// With a second shift, or more ends than the record holds, the verdict is
// kVerdictWalk.  An accept list is one packed word, and the
// first three candidates' bits are read side by side, so a lexeme costs two
// dependent LDS reads and hardly a branch.

template <int MW>
__device__ __forceinline__ bool set_has(const uint32_t (&set)[MW], uint32_t t) {
  uint32_t w = 0;  // masked, not selected: a select of array elements becomes an indexed load from scratch
#pragma unroll
  for (int i = 0; i < MW; ++i) w |= set[i] & (0u - (uint32_t)((t >> 5) == (uint32_t)i));
  return (w >> (t & 31u)) & 1u;
}

// What a verdict reads of the row and the grammar.  The allowed sets are in LDS
// with the ignored terminals added: usets[0] from sigma, usets[1 + t] after
// shifting t, 8 words each.
template <int MW>
struct RowView {
  uint32_t R[MW], I[MW];     // restricted and ignored terminals (uniform)
  const uint32_t* R_s;       // R in LDS
  const uint32_t* usets;     // [1 + T][8]
  const uint32_t* live;      // [S][8]
  const uint32_t* acc;       // packed accept lists [S]
  const uint32_t* acc_off;   // the lists themselves, past the packed three
  const uint8_t* acc_list;
  const uint32_t* tinfo;
  int winner;
  uint32_t wkind;
  __device__ __forceinline__ int accept(uint32_t q, uint32_t packed, uint32_t j) const {
    return j < 3u ? (int)((packed >> (8u * j)) & 0xFFu) : (int)acc_list[acc_off[q] + j];
  }
  __device__ __forceinline__ const uint32_t* after(int t) const { return usets + (1 + t) * 8; }
  // The winner of a lexeme that ends in state q when set is the allowed set:
  // the first accept-list entry in the set that, if restricted, has its
  // category's word flag in flags() (asked for at most once).  -1 if none.
  template <class Flags>
  __device__ __forceinline__ int winner_in(uint32_t q, const uint32_t* set, Flags flags) const {
    const uint32_t packed = acc[q], n = packed >> 24;
    const uint32_t c0 = packed & 0xFFu, c1 = (packed >> 8) & 0xFFu, c2 = (packed >> 16) & 0xFFu;
    const uint32_t u0 = set[c0 >> 5] >> (c0 & 31u), u1 = set[c1 >> 5] >> (c1 & 31u), u2 = set[c2 >> 5] >> (c2 & 31u);
    const uint32_t r0 = R_s[c0 >> 5] >> (c0 & 31u), r1 = R_s[c1 >> 5] >> (c1 & 31u), r2 = R_s[c2 >> 5] >> (c2 & 31u);
    const uint32_t ok = ((u0 & 1u) | (u1 & 1u) << 1 | (u2 & 1u) << 2) & ((1u << min(n, 3u)) - 1u);
    const uint32_t rs = (r0 & 1u) | (r1 & 1u) << 1 | (r2 & 1u) << 2;
    if (ok == 0u && n <= 3u) return -1;
    const uint32_t f = ok & (0u - ok);
    if (f & ~rs) return (int)(f == 1u ? c0 : (f == 2u ? c1 : c2));
    uint32_t wf = 0;
    bool have = false;
    for (uint32_t j = 0; j < n; ++j) {  // a restricted candidate first, or a long list
      const int c = accept(q, packed, j);
      if (!((set[c >> 5] >> (c & 31)) & 1u)) continue;
      if ((R_s[c >> 5] >> (c & 31)) & 1u) {
        if (!have) wf = flags();
        have = true;
        if (!((wf >> (8 + ((tinfo[c] >> 8) & 7u))) & 1u)) continue;
      }
      return c;
    }
    return -1;
  }
};

// A view of the row whose block is in LDS.
template <int MW>
__device__ __forceinline__ void view_row(RowView<MW>& rv, const Tables& tb, const RowLayout& RL, const uint8_t* block) {
  const RowHeader& h = *(const RowHeader*)block;
#pragma unroll
  for (int w = 0; w < MW; ++w) {
    rv.R[w] = __builtin_amdgcn_readfirstlane(h.R[w]);
    rv.I[w] = tb.ign[w];
  }
  rv.R_s = h.R;
  rv.usets = (const uint32_t*)(block + RL.usets);
  rv.acc = (const uint32_t*)(block + RL.acc);
  rv.acc_off = tb.acc_off;
  rv.acc_list = tb.acc_list;
  rv.winner = __builtin_amdgcn_readfirstlane(h.winner);
  rv.wkind = __builtin_amdgcn_readfirstlane(h.wkind);
}

// Definition 2's test of a trailing lexeme in state q against the set cur
// (known: the parser's whole allowed set; else only what holds under any stack).
template <int MW, class Trail>
__device__ __forceinline__ uint32_t trail_verdict(const RowView<MW>& rv, const uint32_t* set, bool known, uint32_t q,
                                                  Trail trail) {
  const uint32_t* lv = rv.live + (size_t)q * 8;
  uint32_t unres = 0, res = 0, ign = 0, rw[MW];
#pragma unroll
  for (int w = 0; w < MW; ++w) {
    const uint32_t l = lv[w], bits = l & set[w];
    unres |= bits & ~rv.R[w];
    rw[w] = bits & rv.R[w];
    res |= rw[w];
    ign |= l & rv.I[w] & ~rv.R[w];
  }
  if (ign || (known && unres)) return kVerdictAllow;
  if (!known) return kVerdictWalk;
  if (!res) return kVerdictReject;
  uint32_t cats = 0;
#pragma unroll
  for (int w = 0; w < MW; ++w)
    for (uint32_t r = rw[w]; r; r &= r - 1) cats |= 1u << ((rv.tinfo[w * 32 + __ffs(r) - 1] >> 8) & 7u);
  return (trail(cats) & cats) ? kVerdictAllow : kVerdictReject;
}

template <int MW, class Lex>
__device__ __forceinline__ uint32_t class_verdict(const RowView<MW>& rv, uint4 rec, Lex& lex) {
  const uint32_t w0 = rec.x;
  if (w0 & kClassReject) return kVerdictReject;
  if (w0 & kClassWalk) return kVerdictWalk;
  const uint32_t ends = w0 & kClassEndsMask;
  const uint32_t* set = rv.usets;  // the set in force
  int sel = -1;                    // -1 from sigma, t >= 0 after shifting t, -2 unknown
  for (uint32_t i = 0; i < min(ends, (uint32_t)kClassEnds); ++i) {
    int t;
    if (i == 0 && (w0 & kClassP0)) {  // byte 0 ends the pending lexeme: the prologue's winner
      if (rv.wkind == 0) return kVerdictReject;
      t = rv.winner;
    } else {
      if (sel == -2) return kVerdictWalk;
      const uint32_t q = i == 0 ? rec.y >> 16 : (i == 1 ? rec.z & 0xFFFFu : rec.z >> 16);
      t = rv.winner_in(q, set, [&]() { return lex.word(i); });
      if (t < 0) return kVerdictReject;
    }
    if (set_has<MW>(rv.I, t)) continue;
    if (sel == -1) {
      sel = t;
      set = rv.after(t);
    } else {
      sel = -2;
    }
  }
  if (ends > (uint32_t)kClassEnds) return kVerdictWalk;
  return trail_verdict<MW>(rv, set, sel != -2, rec.y & 0xFFFFu, [&](uint32_t cats) { return lex.trail(cats); });
}

// Whether lexeme i of a class record (i = 0 with no end: the trailing one) holds
// the pending bytes, and the byte it starts at; trail: the trailing lexeme.
__device__ __forceinline__ bool holds_pending(const uint4& rec, uint32_t i) { return i == 0 && !(rec.x & kProgFresh); }
__device__ __forceinline__ uint32_t lexeme_start(const uint4& rec, int prog, uint32_t i, bool trail) {
  if (!prog) return i == 0 ? 0u : (rec.w >> (8u * (i - 1u))) & 0xFFu;  // where the lexeme before it ended
  if (trail) return rec.x >> 24;
  return i == 0 ? rec.w >> 24 : (i == 1 ? (rec.x >> 8) & 0xFFu : (rec.x >> 16) & 0xFFu);
}

// Lexicon policy that answers the class's first lexicon question with "no
// flags" and records it (kind, start offset in the token, whether the lexeme
// holds the pending bytes); it notes whether a second question is asked.
struct LexNo {
  uint4 rec;
  int prog;
  bool pending_empty;
  int kind;           // first question: -1 none yet, 0 trailing prefix, 1 word
  int start;          // its start offset in the token where the token-flag table
                      // (GRID_ART_LEX_TOKEN: bytes 0 and 1, in the start state) answers for it, or -1
  bool pending;       // its lexeme holds the pending bytes
  bool second;        // a second question was asked
  uint32_t cats;      // the categories a trailing question asks about
  __device__ void first(uint32_t i, int k) {
    kind = k;
    const bool hp = holds_pending(rec, i);
    const uint32_t o = lexeme_start(rec, prog, i, k == 0);
    pending = hp && !pending_empty;
    start = hp ? (pending_empty ? 0 : -1) : (o <= 1u ? (int)o : -1);
  }
  __device__ uint32_t word(uint32_t i) {
    if (kind >= 0) second = true;
    else first(i, 1);
    return 0u;
  }
  __device__ uint32_t trail(uint32_t c) {
    if (kind >= 0) second = true;
    else first(rec.x & kClassEndsMask, 0);
    cats = c;
    return 0u;
  }
};

// Shortcut of a class the lexicon decides: its verdict v_no when the answer
// to its first lexicon question is "no flags", valid when that answer leads
// to no second question.  The stream kernel knows the answer is "no flags"
// when the question's lexeme starts with the pending bytes and the token's
// first byte does not continue them in the lexicon (the row's cont table) or,
// when the lexeme also holds the token's second byte, that byte does not
// continue them after the first (the row's second-byte table); or when the
// lexeme starts at token byte 0 or 1 in the start state and the token-flag
// entry has no flags there.  Encoded as 3 (the class code) | kind << 2 (0
// pending bytes, 1 trailing prefix at o, 2 word at o) | o << 4 | v_no << 5 |
// valid << 7; for kind 0, bit 4 says the lexeme holds the token's second byte
// when the token has one (a trailing lexeme, or a word ending at offset 2 or
// later).
constexpr uint32_t kNoValid = 1u << 7;
// The class's byte from one verdict run: the run under "no flags" follows the
// run without token bytes up to the first lexicon question, so a class that asks
// none has its final verdict there, and one that asks is a lexicon class whose
// verdict under "no flags" is the run's result.  A trailing question on a lexeme
// the token-flag table covers is settled by the stream either way: *cats are the
// categories whose prefix allows the token.
template <int MW>
__device__ __forceinline__ uint32_t class_code(const RowView<MW>& rv, int prog, bool pending_empty, uint4 rec,
                                               uint32_t* cats) {
  LexNo ln{rec, prog, pending_empty, -1, -1, false, false, 0u};
  const uint32_t v = class_verdict<MW>(rv, rec, ln);
  *cats = ln.cats;
  if (ln.kind < 0) return v;  // no lexicon question: the class's verdict
  if (ln.second) return kVerdictLexicon;
  if (ln.pending) {
    const bool two = ln.kind == 0 || (rec.w & 0xFFu) >= 2u;
    return kVerdictLexicon | (two ? 1u << 4 : 0u) | v << 5 | kNoValid;
  }
  if (ln.start < 0) return kVerdictLexicon;
  return kVerdictLexicon | (ln.kind == 0 ? 1u : 2u) << 2 | (uint32_t)ln.start << 4 | v << 5 | kNoValid;
}

// LDS of a judge workgroup: the row's block up to its stacks, live sets,
// terminal info.
struct JudgeLds {
  uint32_t block, live, tinfo, total;
};

__host__ __device__ inline JudgeLds judge_lds(const Tables& tb) {
  JudgeLds L;
  uint32_t o = 0;
  L.block = o;
  o += pad16((uint32_t)row_layout(tb).post);
  L.live = o;
  o += (uint32_t)tb.S * 32u;
  L.tinfo = o;
  o += pad16((uint32_t)tb.T * 4u);
  L.total = o;
  return L;
}

// After the prologue: the verdict byte of every class of the row's lexer state,
// from A(sigma) and the allowed sets after one shift; a class with a second shift
// is left to the walk.  Workgroups (row, part), a part being every parts-th block
// of kJudgeThreads classes.
// (The sets after two shifts can be had too: a row's classes ask for some 15 pairs
// of terminals.  Finding them and judging those classes again took each workgroup
// 5 us, in all 8 to 12 us of a step of 1 to 47 rows; walking their ids as well costs
// the residue kernel 1 to 3 us.  At 256 rows, 20 us less residue paid for it.
// Measured when a step of 32 rows took 89 us and one of 256 rows 350.)
template <int MW>
__global__ __launch_bounds__(kJudgeThreads, 8) void judge_kernel(Tables tb, uint8_t* __restrict__ ws, size_t rbytes,
                                                              int parts) {
  extern __shared__ __align__(16) uint8_t lds[];
  const int tid = threadIdx.x;
  const int row = (int)blockIdx.x / parts, part = (int)blockIdx.x - row * parts;
  uint8_t* rw = ws + kWsHead + (size_t)row * rbytes;
  const RowHeader* hdr = (const RowHeader*)rw;
  const uint32_t n = hdr->n_cls, cls_base = hdr->cls_base;
  const uint32_t first = (uint32_t)part * kJudgeThreads, stride = (uint32_t)parts * kJudgeThreads;
  if (hdr->valid != kRowValid || first >= n) return;  // uniform
  const JudgeLds JL = judge_lds(tb);
  const RowLayout RL = row_layout(tb);
  uint4 rec = make_uint4(0, 0, 0, 0);
  if (first + (uint32_t)tid < n) rec = tb.crec[cls_base + first + (uint32_t)tid];
  const StageRegion rg[3] = {{rw, lds + JL.block, (uint32_t)RL.post},
                             {(const uint8_t*)tb.live, lds + JL.live, (uint32_t)tb.S * 32u},
                             {(const uint8_t*)tb.term_info, lds + JL.tinfo, (uint32_t)tb.T * 4u}};
  dma_regions<3>(rg, tid, kJudgeThreads);
  const RowHeader& h = *(const RowHeader*)(lds + JL.block);
  RowView<MW> rv;
  rv.live = (const uint32_t*)(lds + JL.live);
  rv.tinfo = (const uint32_t*)(lds + JL.tinfo);
  dma_wait();
  __syncthreads();
  view_row(rv, tb, RL, lds + JL.block);
  const bool empty = h.rem_len == 0;
  uint8_t* codes = rw + RL.codes;
  uint8_t* cats = rw + RL.cats;
  for (uint32_t c = first + (uint32_t)tid; c < n; c += stride) {
    const uint4 cur = rec;
    if (c + stride < n) rec = tb.crec[cls_base + c + stride];
    const bool ci = ci_class(cur.x);
    uint32_t code = kVerdictReject;
    if (!(h.ci_hit >= 0 && ci)) {  // (else served by the row's cached context-independent words)
      uint32_t ct = 0;
      code = class_code<MW>(rv, tb.prog, empty, cur, &ct);
      if (((code >> 2) & 3u) == 1u) cats[c] = (uint8_t)ct;  // (only a trailing question has that kind)
      if (code == kVerdictAllow && ci) code |= kCodeCi;
    }
    codes[c] = (uint8_t)code;
  }
}

// ------------------------------------------------------------------ stream
// LDS of a stream workgroup: the row's class bytes, a queue of open ids per
// wave, those it leaves open.
struct StreamLds {
  uint32_t codes, queue, list, total;
};
__host__ __device__ inline StreamLds stream_lds(const Tables& tb) {
  StreamLds L;
  uint32_t o = 0;
  L.codes = o;
  o += pad16((uint32_t)tb.max_classes);
  L.queue = o;
  o += kStreamWaves * kStepIds * 4;
  L.list = o;
  o += kOpenLocal * 8;
  L.total = o;
  return L;
}

// Eight consecutive class ids (u16), a class-map row being aligned to 2 bytes.
struct __attribute__((packed, aligned(2))) Ids8 {
  uint32_t w[4];
};

// Position of this lane among the lanes of bal.
__device__ __forceinline__ int lane_rank(uint64_t bal) {
  return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0u));
}

// The mask in token-id order straight from the class map, one row against one
// slice of the vocabulary per workgroup.  A wave step covers 512 ids, 8 per
// lane: one 16-byte load of the class map, eight class bytes gathered from LDS,
// the allowed bits as one byte of the mask.  The ids the class byte leaves
// open go to the wave's own queue and are taken 64 at a time, so that their
// lookups cost what the open ids need and not what the step has: a class the
// lexicon decides takes its shortcut verdict when the answer to its first
// lexicon question is "no flags" for the token (from its first two bytes and
// the row's continuation tables, or from its token-flag summary), or when that
// question is a trailing one the token's prefix flags answer.  What stays
// open is listed for the residue kernel, and marked in the row's open bitmap for
// the row that has more than its list holds.  16 bytes of class map per lane: 13.1 us
// at 32 rows of 151,936 ids and 59 us at 256 (64 ids per wave and one 2-byte load
// per lane: 20.8 and 123 us).  Bound by the open ids' chains of dependent lookups:
// reading a batch's first lookups while the one before it is settled took it from 65
// to 58 us at 256 rows; neither packing the queue with half the instructions nor
// settling the lexicon classes in place before it (from 96 open ids on) made it
// faster.  Rows served from the mask cache are skipped; rows with a bad
// configuration get zero words.
__global__ __launch_bounds__(kStreamThreads, 8) void stream_kernel(Tables tb, uint32_t* __restrict__ mask,
                                                                uint8_t* __restrict__ ws, size_t rbytes, int B,
                                                                int n_slices, int slice_ids) {
  extern __shared__ __align__(16) uint8_t slds[];
  __shared__ int open_s, base_s;
  __shared__ uint8_t cont[256];  // first bytes that continue the pending bytes in the lexicon
  __shared__ uint32_t mbits[kStreamWaves][kStepIds / 32], cbits[kStreamWaves][kStepIds / 32],
      obits[kStreamWaves][kStepIds / 32];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int row = (int)blockIdx.x / n_slices, slice = (int)blockIdx.x - row * n_slices;
  const int lo = slice * slice_ids, hi = min(lo + slice_ids, tb.V);
  uint8_t* rw = ws + kWsHead + (size_t)row * rbytes;
  RowHeader* hdr = (RowHeader*)rw;
  const uint32_t valid = hdr->valid;
  if (valid == kRowCached) return;
  uint32_t* mrow = mask + (size_t)row * tb.W;
  if (valid != kRowValid) {  // bad configuration: an empty row
    for (int w = (lo >> 5) + tid; w < min((lo + slice_ids) >> 5, tb.W); w += kStreamThreads) mrow[w] = 0u;
    return;
  }
  const StreamLds SL = stream_lds(tb);
  const RowLayout RL = row_layout(tb);
  const uint16_t* cm = tb.cmap + (size_t)hdr->q * tb.V;
  const uint32_t cls_base = hdr->cls_base;
  {
    const StageRegion rg[1] = {{rw + RL.codes, slds + SL.codes, pad16(hdr->n_cls)}};
    dma_regions<1>(rg, tid, kStreamThreads);
  }
  const uint8_t* codes = slds + SL.codes;
  const uint32_t* cont2 = (const uint32_t*)(rw + RL.cont2);
  uint32_t* queue = (uint32_t*)(slds + SL.queue) + wave * kStepIds;
  const int eos = hdr->eos_ok ? tb.eos_id : -1;
  const uint8_t* tsum = tb.lex_toksum + (size_t)hdr->slot_id * tb.V;
  const uint32_t* tok = tb.lex_token + (size_t)hdr->slot_id * tb.V;
  const uint8_t* cats = rw + RL.cats;
  // a row served by cached context-independent words ORs them into its words
  const int ci = hdr->ci_hit, claim = hdr->ci_claim;
  const uint32_t* ciw = ci >= 0 ? (const uint32_t*)(tb.ci_cache + (size_t)ci * tb.ci_stride + kCiHeader) : nullptr;
  // a row that claimed an entry writes its CI tokens' bits there (the residue
  // pass adds those it decides)
  uint32_t* cdst = claim >= 0 ? (uint32_t*)(tb.ci_cache + (size_t)claim * tb.ci_stride + kCiHeader) : nullptr;
  if (tid < 256) cont[tid] = (uint8_t)((hdr->cont[tid >> 5] >> (tid & 31)) & 1u);
  // the class ids of this lane in a step, 0 (rejected) past the vocabulary
  auto load_ids = [&](int id0) -> Ids8 {
    Ids8 v = {{0, 0, 0, 0}};
    if (id0 + 8 <= tb.V) {
      v = *reinterpret_cast<const Ids8*>(cm + id0);
    } else {
#pragma unroll
      for (int j = 0; j < 8; ++j)
        if (id0 + j < tb.V) v.w[j >> 1] |= (uint32_t)cm[id0 + j] << (16 * (j & 1));
    }
    return v;
  };
  bool any = false;
  uint2* list = (uint2*)(slds + SL.list);
  int wb = lo + wave * kStepIds;
  Ids8 ids = {{0, 0, 0, 0}};
  if (wb < hi) ids = load_ids(wb + lane * 8);
  if (tid == 0) open_s = 0;
  dma_wait();
  __syncthreads();
  for (; wb < hi; wb += kStreamWaves * kStepIds) {
    const Ids8 cur = ids;
    if (wb + kStreamWaves * kStepIds < hi) ids = load_ids(wb + kStreamWaves * kStepIds + lane * 8);
    uint32_t bits = 0, open = 0, cib = 0;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const uint32_t cd = codes[(cur.w[j >> 1] >> (16 * (j & 1))) & 0xFFFFu];
      bits |= ((cd & 3u) == kVerdictAllow ? 1u : 0u) << j;
      cib |= ((cd & 7u) == (kVerdictAllow | kCodeCi) ? 1u : 0u) << j;
      open |= ((cd >> 1) & 1u) << j;
    }
    if ((uint32_t)(eos - (wb + lane * 8)) < 8u) bits |= 1u << (eos - (wb + lane * 8));
    ((uint8_t*)mbits[wave])[lane] = (uint8_t)bits;
    ((uint8_t*)obits[wave])[lane] = 0;
    if (cdst) ((uint8_t*)cbits[wave])[lane] = (uint8_t)cib;
    int n = 0;  // open ids of the step (uniform)
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const bool o = (open >> j) & 1u;
      const uint64_t bal = __ballot(o);
      if (o)
        queue[n + lane_rank(bal)] = ((cur.w[j >> 1] >> (16 * (j & 1))) & 0xFFFFu) << 16 | (uint32_t)(lane * 8 + j);
      n += __popcll(bal);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    int left = 0;  // of them, left to the residue (uniform)
    // a batch's entries and what their shortcuts ask first, read a batch ahead
    uint32_t e = 0, rule = 0, word = 0;
    auto fetch = [&](int i0) {
      e = rule = word = 0;
      if (i0 + lane < n) {
        e = queue[i0 + lane];
        rule = codes[e >> 16];
        const int id = wb + (int)(e & 0xFFFFu);
        if ((rule & (3u | kNoValid)) == (kVerdictLexicon | kNoValid))
          word = (rule >> 2) & 3u ? (uint32_t)tsum[id] : tb.id_head[id];
      }
    };
    fetch(0);
    for (int i0 = 0; i0 < n; i0 += 64) {
      const uint32_t cls = e >> 16, lid = e & 0xFFFFu, rl = rule, wd0 = word;
      const int id = wb + (int)lid;
      fetch(i0 + 64);
      uint32_t cd = rl & 3u;
      if (cd == kVerdictLexicon && (rl & kNoValid)) {
        const uint32_t kind = (rl >> 2) & 3u;
        bool no;
        if (kind == 0) {  // on the pending bytes: the token's first byte, then its second
          const uint32_t fb = wd0 & 0xFFu, sb = (wd0 >> 8) & 0xFFu;
          no = !cont[fb];
          if (!no && ((rl >> 4) & 1u) && (wd0 & 0x10000u)) no = !((cont2[fb * 8u + (sb >> 5)] >> (sb & 31u)) & 1u);
        } else {
          const uint32_t o = (rl >> 4) & 1u;
          no = ((wd0 >> (2u * o + (kind == 2u ? 1u : 0u))) & 1u) == 0u;
          // a trailing question is the last one: the token's prefix flags settle it
          if (!no && kind == 1u) cd = (tok[id] >> (16u * o)) & cats[cls] & 0xFFu ? kVerdictAllow : kVerdictReject;
        }
        if (no) cd = (rl >> 5) & 3u;
      }
      if (cd == kVerdictAllow) {
        atomicOr(&mbits[wave][lid >> 5], 1u << (lid & 31u));
        if (cdst && ci_class(tb.crec[cls_base + cls].x)) atomicOr(&cbits[wave][lid >> 5], 1u << (lid & 31u));
      }
      const uint64_t bal = __ballot(cd >= kVerdictWalk);
      if (bal) {  // uniform
        int base = 0;
        if (lane == 0) base = atomicAdd(&open_s, __popcll(bal));
        base = __builtin_amdgcn_readfirstlane(base);
        if (cd >= kVerdictWalk) {
          atomicOr(&obits[wave][lid >> 5], 1u << (lid & 31u));
          const int at = base + lane_rank(bal);
          if (at < kOpenLocal) list[at] = make_uint2((uint32_t)id, cls | (rl & 3u) << 16);
        }
        left += __popcll(bal);
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    const int wd = (wb >> 5) + lane;
    if (lane < kStepIds / 32) {
      if (wd < tb.W) {
        uint32_t v = mbits[wave][lane];
        if (ciw) v |= ciw[wd];
        any = any || v != 0u;
        mrow[wd] = v;
        if (cdst) cdst[wd] = cbits[wave][lane];
      }
      if (left) ((uint32_t*)(rw + RL.open))[wd] = obits[wave][lane];
    }
    if (lane == 0) ((uint16_t*)(rw + RL.n_open))[wb / kStepIds] = (uint16_t)left;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  }
  if (__any(any) && lane == 0) hdr->nonempty = 1u;
  __syncthreads();
  const int n = open_s;
  if (n == 0) return;  // uniform
  if (tid == 0) {  // this workgroup's place in the row's list
    uint32_t* cnt = open_counts(ws, rbytes, B) + row;
    base_s = (int)(atomicAdd(cnt, (uint32_t)n) & (kListFull - 1u));
    if (n > kOpenLocal) atomicOr(cnt, kListFull);
  }
  __syncthreads();
  uint2* out = (uint2*)(rw + RL.list);
  for (int i = tid; i < min(n, kOpenLocal); i += kStreamThreads)
    if (base_s + i < open_list_cap(tb.V)) out[base_s + i] = list[i];
}

// ----------------------------------------------------------------- residue
// The next value of an LDS counter for the whole wave (one atomic).
__device__ inline int wave_grab(int* ctr) {
  int v = 0;
  if ((threadIdx.x & 63) == 0) v = atomicAdd(ctr, 1);
  return __builtin_amdgcn_readfirstlane(v);
}

// The live sets, allowed sets and accept lists of a verdict.
inline uint32_t verdict_bytes(const Tables& tb) {
  return (uint32_t)tb.S * 32u + (uint32_t)tb.T * 32u + pad16((uint32_t)tb.T * 4u) + pad16((uint32_t)(tb.S + 1) * 4u) +
         pad16((uint32_t)tb.n_acc);
}

// The lexer's and the parser's tables (LR with GOTO as the hash) and two bytes
// per lexer state: what the supported grammars are bounded by.
inline uint32_t table_bytes(const Tables& tb) {
  return pad16((uint32_t)(tb.S * tb.C * 2)) + pad16((uint32_t)(tb.S + 1) * 4u) + pad16((uint32_t)tb.n_acc) +
         (uint32_t)tb.S * 32u + 2u * pad16((uint32_t)tb.S) + parse_lds(tb, 0, false).total;
}

struct ResLds {  // byte offsets into dynamic LDS
  uint32_t block, bcls, tinfo, live, dfa, areas, qid, qcls, slow, total;
  int full;  // the chains' tables, the DFA and the live sets are in LDS too
  LrLds lr;
};

__host__ __device__ inline ResLds res_lds(const Tables& tb) {
  ResLds w;
  uint32_t o = 0;
  w.block = o;
  o += (uint32_t)row_layout(tb).block;
  w.bcls = o;
  o += 256;
  w.tinfo = o;
  o += pad16((uint32_t)tb.T * 4u);
  w.areas = o;
  o += kResWaves * kLanesMax * kFastLane * 2;
  w.qid = o;
  o += kQueue * 4;
  w.qcls = o;
  o += kQueue * 2;
  w.slow = o;
  o += kQueue * 4;
  const uint32_t live = (uint32_t)tb.S * 32u;  // as in global memory, 8 words per state
  const uint32_t dfa = pad16((uint32_t)(tb.S * tb.C * 2));
  w.lr = lr_lds(tb, o);
  w.full = o + w.lr.total + live + dfa <= kLdsMax - kLdsStatic ? 1 : 0;
  w.live = w.dfa = 0;
  if (w.full) {
    o += w.lr.total;
    w.live = o;
    o += live;
    w.dfa = o;
    o += dfa;
  }
  w.total = o;
  return w;
}
static_assert(kSlowWaves >= 1 && kSlowWaves * kSlowLane <= kResWaves * kLanesMax * kFastLane,
              "the slow walks' areas fit where the fast ones were");

// Bytes [s, s + 8) of the 24-byte window b0 b1 b2 (zero beyond it).
__device__ __forceinline__ uint64_t window8(uint64_t b0, uint64_t b1, uint64_t b2, uint32_t s) {
  const uint32_t w = s >> 3, sh = (s & 7u) * 8u;
  const uint64_t lo = w == 0 ? b0 : (w == 1 ? b1 : (w == 2 ? b2 : 0ull));
  const uint64_t hi = w == 0 ? b1 : (w == 1 ? b2 : 0ull);
  return sh ? (lo >> sh) | (hi << (64 - sh)) : lo;
}

// Lexicon policy of a token judged with its own bytes: lexeme i of the
// class record (the pending bytes and the token's bytes before end 0, or the
// bytes between ends i-1 and i) and the trailing lexeme.  A lexeme starting
// in the start state at byte 0 or 1 is answered by the token-flag entry tf;
// others are looked up in the prefix and stride tables, and one that does not
// lie in the token's first 24 bytes is out of reach.  The pending bytes are
// known up to 8; beyond that the lexeme continues from the pending lexeme's
// trie node.  Plain scalar members only, so the policy lives in registers.
struct LexLane {
  const Tables* tb;
  Slot sl;
  uint64_t b0, b1, b2;  // token bytes 0..23, zero padded
  uint32_t n;           // token length
  uint64_t rem;         // pending bytes (first 8)
  uint32_t rem_len, lexnode;
  uint32_t tf;          // token-flag entry
};

// What a byte walk reads besides the row's sets.
template <int MW, bool L>
struct WalkView {
  const Tables* tb;
  RowView<MW> rv;
  LrTabs<L> lt;
  DfaView step;
  const uint16_t* pool;       // the row's stack
  mptr<true, const uint16_t> win;
  uint32_t lo, depth;
  const uint4* post;          // stacks after one shift, two 16-byte halves each
  uint32_t q;                 // the row's scan state
};

// A Post record's two halves unpacked onto a lane's stack area: false if it is
// unusable (not a stack, or more entries than the area holds).
__device__ __forceinline__ bool load_post(const uint4& h1, const uint4& h2, uint32_t depth, uint32_t cap, uint32_t& k,
                                          uint32_t& m, mptr<true, uint16_t> ov) {
  const uint32_t pk = h1.x & 0xFFFFu, pm = (h1.x >> 16) & 0xFFu, pok = h1.x >> 24;
  if (!pok || pk == 0 || pk > depth || pm > (uint32_t)kPostCap || pm > cap) return false;
  k = pk;
  m = pm;
  const uint32_t w[7] = {h1.y, h1.z, h1.w, h2.x, h2.y, h2.z, h2.w};
#pragma unroll
  for (uint32_t j = 0; j < 14; ++j)
    if (j < m) ov[j] = (uint16_t)(w[j >> 1] >> (16 * (j & 1)));
  return true;
}

// Verdicts of a walk besides reject and allow.
constexpr uint32_t kWalkTrail = 4;  // some terminal of X must be shiftable from the lane's stack
constexpr uint32_t kWalkFull = 5;   // the stack area is too small

// One token judged to its end: lexemes as in class_verdict, from the class
// record while it has them, else by running the DFA over the bytes; past the
// first shift the parser's stack is the lane's own (base[0, k) and m overlay
// entries in its area of cap), a lexeme's candidates are tried in priority order
// by their reduce chains, and the first that shifts is committed -- no allowed
// set is needed until the trailing lexeme, whose terminals X are left to the
// whole wave (see residue_kernel).
// (The lookup of a lexeme's flags appears here four times and is kept small: with
// the strides and the two placings of the bytes written out it made the kernel 40 %
// larger, past what the instruction cache holds, and every call 2 to 5 % slower.)
template <int MW, bool L>
__device__ __forceinline__ uint32_t walk_token(const WalkView<MW, L>& wv, uint4 rec, const LexLane& lex, uint32_t chunk,
                                               mptr<true, uint16_t> ov, uint32_t cap, uint32_t& k, uint32_t& m,
                                               uint32_t (&X)[MW]) {
  const Tables& tb = *wv.tb;
  const RowView<MW>& rv = wv.rv;
  const uint32_t w0 = rec.x, ends = w0 & kClassEndsMask, n_rec = min(ends, (uint32_t)kClassEnds);
  const uint32_t* set = rv.usets;  // the set in force, while it is kept
  int sel = -1;                    // -1 from sigma, t >= 0 after shifting t, -4 the lane's own stack
  bool scan = (w0 & kClassWalk) != 0;
  uint32_t o = 0, si = 0, sq = wv.q, q = 0;  // the current lexeme's first byte; the scan's position and state
  bool pending = true;                       // the lexeme holds the pending bytes
  // byte i of the token
  auto byte_at = [&](uint32_t i) -> uint32_t {
    if (i >= 24u) return reinterpret_cast<const uint8_t*>(tb.spell_tail + chunk)[i - 24u];
    const uint64_t b = (lex.b0 & (0ull - (uint64_t)(i < 8u))) | (lex.b1 & (0ull - (uint64_t)(i >= 8u && i < 16u))) |
                       (lex.b2 & (0ull - (uint64_t)(i >= 16u)));
    return (uint32_t)(b >> (8u * (i & 7u))) & 0xFFu;
  };
  // lexicon flags of bytes [o, e) (with the pending bytes before them)
  auto flags = [&](uint32_t e) -> uint32_t {
    const bool cont = pending && lex.rem_len > 0;  // (then o is 0)
    if (!cont && o <= 1u) return (lex.tf >> (16u * o)) & 0xFFFFu;  // the token-flag table
    const uint32_t len = e - o + (cont ? lex.rem_len : 0u);
    if (e <= 24u && len <= 24u && !(cont && lex.rem_len > 8u)) {  // the prefix and stride tables
      const uint32_t sh = 8u * lex.rem_len;  // the pending bytes go before: 8..64 bits
      uint64_t c0 = window8(lex.b0, lex.b1, lex.b2, o), c1 = window8(lex.b0, lex.b1, lex.b2, o + 8),
               c2 = window8(lex.b0, lex.b1, lex.b2, o + 16);
      if (cont) {
        c2 = (c1 >> (64 - sh)) | (sh < 64 ? c2 << sh : 0ull);
        c1 = (c0 >> (64 - sh)) | (sh < 64 ? c1 << sh : 0ull);
        c0 = lex.rem | (sh < 64 ? c0 << sh : 0ull);
      }
      return lex_flags_bytes(tb, lex.sl, c0, c1, c2, len);
    }
    // byte by byte through the lexicon trie
    uint32_t node = cont ? lex.lexnode : 0u;
    for (uint32_t i = o; i < e && node != kNoLex; ++i) node = lex_child(tb, lex.sl, node, byte_at(i));
    return lex_flags_of(tb, lex.sl, node);
  };
  for (uint32_t i = 0;; ++i) {
    uint32_t e;
    if (!scan && i == n_rec) {
      if (ends <= (uint32_t)kClassEnds) {
        q = rec.y & 0xFFFFu;
        o = lexeme_start(rec, tb.prog, ends, true);
        pending = holds_pending(rec, ends);
        break;
      }
      scan = true;
      si = o;
      sq = kStart;
    }
    if (scan) {
      while (si < lex.n) {
        const int nq = wv.step.next((int)sq, wv.step.cls(byte_at(si)));
        if (nq == kDead) break;
        sq = (uint32_t)nq;
        ++si;
      }
      q = sq;
      e = si;
      if (si == lex.n) break;
      if (si == o && !(pending && lex.rem_len > 0)) return kVerdictReject;  // a byte that starts no lexeme
    } else {
      q = i == 0 ? rec.y >> 16 : (i == 1 ? rec.z & 0xFFFFu : rec.z >> 16);
      o = lexeme_start(rec, tb.prog, i, false);
      e = (rec.w >> (8u * i)) & 0xFFu;
      pending = holds_pending(rec, i);
    }
    // the lexeme's winner
    int t = -1;
    uint32_t a = 0, n = 0, s = 0;
    bool moved = false;
    if (!scan && i == 0 && (w0 & kClassP0)) {
      if (rv.wkind == 0) return kVerdictReject;
      t = rv.winner;
    } else {
      if (sel != -4) {
        t = rv.winner_in(q, set, [&]() { return flags(e); });
      } else {
        const uint32_t acc = rv.acc[q];
        uint32_t wf = kLexOpen;
        for (uint32_t j = 0; j < acc >> 24; ++j) {
          const int c = rv.accept(q, acc, j);
          if (set_has<MW>(rv.R, c)) {
            if (wf == kLexOpen) wf = flags(e);
            if (!((wf >> (8 + ((rv.tinfo[c] >> 8) & 7u))) & 1u)) continue;
          }
          if (!set_has<MW>(rv.I, c)) {
            n = k + m - 1u;
            const ChainStack st{wv.pool, wv.win, wv.lo, k, ov, m};
            s = st.at(n);
            a = lr_chain<L>(wv.lt, st, (uint32_t)c, n, s, moved);
            if (!a) continue;
          }
          t = c;
          break;
        }
      }
      if (t < 0) return kVerdictReject;
    }
    o = e;
    pending = false;
    if (scan) sq = kStart;
    if (set_has<MW>(rv.I, t)) continue;
    // its shift
    if (sel == -1) {
      sel = t;
      set = rv.after(t);
      continue;
    }
    if (sel != -4) {  // from the kept stack after sel: t is in its allowed set, its chain is still to run
      if (!load_post(wv.post[2 * sel], wv.post[2 * sel + 1], wv.depth, cap, k, m, ov)) return kWalkFull;
      n = k + m - 1u;
      const ChainStack st{wv.pool, wv.win, wv.lo, k, ov, m};
      s = st.at(n);
      a = lr_chain<L>(wv.lt, st, (uint32_t)t, n, s, moved);
      if (!a) return kVerdictReject;
      sel = -4;
    }
    if (!lr_commit(tb, a, (uint32_t)t, n, s, moved, k, m, ov, cap)) return kWalkFull;
  }
  // the trailing lexeme, in state q
  if (sel != -4) return trail_verdict<MW>(rv, set, true, q, [&](uint32_t) { return flags(lex.n); });
  const uint32_t* lv = rv.live + (size_t)q * 8;
  uint32_t any = 0, res = 0, ign = 0;
#pragma unroll
  for (int w = 0; w < MW; ++w) {
    X[w] = lv[w];
    ign |= X[w] & rv.I[w] & ~rv.R[w];
    res |= X[w] & rv.R[w];
  }
  if (ign) return kVerdictAllow;
  if (res) {  // restricted terminals count where the lexeme prefixes a word of their category
    const uint32_t pf = flags(lex.n);
    ign = 0;
#pragma unroll
    for (int w = 0; w < MW; ++w)
      for (uint32_t r = X[w] & rv.R[w]; r; r &= r - 1)
        if (!((pf >> ((rv.tinfo[w * 32 + __ffs(r) - 1] >> 8) & 7u)) & 1u)) X[w] &= ~(r & (0u - r));
#pragma unroll
    for (int w = 0; w < MW; ++w) ign |= X[w] & rv.I[w];
    if (ign) return kVerdictAllow;
  }
#pragma unroll
  for (int w = 0; w < MW; ++w) {
    X[w] &= ~rv.I[w];
    any |= X[w];
  }
  return any ? kWalkTrail : kVerdictReject;
}

// The trailing lexemes a wave's walks left (lanes with todo): does any terminal of
// the lane's set X shift from the lane's stack?  The (lane, terminal) pairs of all
// lanes are dealt to the 64 lanes in turn, so a round runs 64 chains side by side
// whichever walks they belong to.  (A round per walk took 4 us of a wave's 13 at
// 32 DML rows, up to 15 in the slowest.)
template <int MW, bool L>
__device__ __forceinline__ bool trail_pairs(const WalkView<MW, L>& wv, bool todo, const uint32_t (&X)[MW], uint32_t k,
                                            uint32_t m, mptr<true, const uint16_t> base) {
  const int lane = threadIdx.x & 63;
  uint32_t cnt = 0;
  if (todo) {
#pragma unroll
    for (int w = 0; w < MW; ++w) cnt += (uint32_t)__popc(X[w]);
  }
  uint32_t incl = cnt;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t x = __shfl_up(incl, d);
    if (lane >= d) incl += x;
  }
  const uint32_t excl = incl - cnt, all = __builtin_amdgcn_readlane(incl, 63);
  bool ok = false;
  for (uint32_t p0 = 0; p0 < all; p0 += 64) {  // uniform
    const uint32_t p = p0 + (uint32_t)lane;
    int src = 0;  // the first lane whose pairs end after p
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1)
      if ((uint32_t)__shfl(incl, src + d - 1) <= p) src += d;
    src &= 63;
    uint32_t j = p - (uint32_t)__shfl(excl, src), word = 0, at = 0;
    bool found = false;
#pragma unroll
    for (int w = 0; w < MW; ++w) {  // the set's j-th terminal: its word
      const uint32_t x = (uint32_t)__shfl(X[w], src), c = (uint32_t)__popc(x);
      const bool here = !found && j < c;
      word = here ? x : word;
      at = here ? (uint32_t)w * 32u : at;
      j -= found || here ? 0u : c;
      found = found || here;
    }
#pragma unroll
    for (uint32_t h = 16; h >= 1; h >>= 1) {  // and its bit
      const uint32_t low = word & ((1u << h) - 1u), c = (uint32_t)__popc(low);
      const bool up = j >= c;
      j -= up ? c : 0u;
      word = up ? word >> h : low;
      at += up ? h : 0u;
    }
    const uint32_t sk = (uint32_t)__shfl(k, src), sm = (uint32_t)__shfl(m, src);
    uint32_t a = 0;
    if (p < all) {
      const ChainStack st{wv.pool, wv.win, wv.lo, sk, base + src * kFastLane, sm};
      uint32_t n = sk + sm - 1u, sv = st.at(n);
      bool moved = false;
      a = lr_chain<L>(wv.lt, st, at, n, sv, moved);
    }
    const uint64_t hit = __ballot(a != 0u);
    // this lane's pairs of the round: [excl, incl) less p0
    const uint32_t b0 = excl > p0 ? min(excl - p0, 64u) : 0u, b1 = incl > p0 ? min(incl - p0, 64u) : 0u;
    const uint64_t below1 = b1 >= 64u ? ~0ull : (1ull << b1) - 1ull, below0 = b0 >= 64u ? ~0ull : (1ull << b0) - 1ull;
    ok = ok || (hit & below1 & ~below0) != 0ull;
  }
  return ok;
}

// Sum of v over the threads below this one (workgroup of kResThreads), and the
// total; sums holds a word per wave.  Every thread calls it.
__device__ __forceinline__ uint32_t block_scan(uint32_t v, uint32_t* sums, uint32_t* total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t incl = v;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t x = __shfl_up(incl, d);
    if (lane >= d) incl += x;
  }
  __syncthreads();  // the previous scan's sums are read
  if (lane == 63) sums[wave] = incl;
  __syncthreads();
  uint32_t below = 0, all = 0;
#pragma unroll
  for (int w = 0; w < kResWaves; ++w) {
    if (w < wave) below += sums[w];
    all += sums[w];
  }
  *total = all;
  return below + incl - v;
}

// The row and the chunk in it that hold chunk c of the batch when every row's
// open ids are dealt K at a time; row -1 past the last.  By one wave.
// first: this lane's counts of the first kCountRegs * 64 rows.
__device__ __forceinline__ int find_chunk(const uint32_t* counts, const uint32_t (&first)[kCountRegs], int B, uint32_t K,
                                          uint32_t c, uint32_t* in_row) {
  const int lane = threadIdx.x & 63;
  uint32_t run = 0;
  auto in_rows = [&](int r0, uint32_t n) -> int {  // rows r0.., n open ids in this lane's
    const uint32_t nc = (n + K - 1u) / K;
    uint32_t incl = nc;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const uint32_t x = __shfl_up(incl, d);
      if (lane >= d) incl += x;
    }
    const uint64_t at = __ballot(c < run + incl);
    if (at) {  // uniform
      const int l = __ffsll((unsigned long long)at) - 1;
      *in_row = c - run - (__builtin_amdgcn_readlane(incl, l) - __builtin_amdgcn_readlane(nc, l));
      return r0 + l;
    }
    run += __builtin_amdgcn_readlane(incl, 63);
    return -1;
  };
#pragma unroll
  for (int j = 0; j < kCountRegs; ++j) {
    if (j * 64 >= B) return -1;
    const int r = in_rows(j * 64, first[j]);
    if (r >= 0) return r;
  }
  for (int r0 = kCountRegs * 64; r0 < B; r0 += 64) {
    const int r = in_rows(r0, r0 + lane < B ? counts[r0 + lane] & (kListFull - 1u) : 0u);
    if (r >= 0) return r;
  }
  return -1;
}

// The largest part of a call: 37 to 40 us at 32 DML rows (V = 151,936) by what the
// rows allow, 147 at 256 with a schema each (55.9 and 261 when a workgroup took
// whole words of a row's bitmap and simulated allowed sets), 18 to 28 us for the
// smallest calls, where a single id's chain is all of it.
// The ids the stream left open, dealt evenly to the workgroups: a chunk is K
// open ids of one row, K set by the batch's total, so a row with many costs no
// workgroup more than a row with few.  The waves of the workgroup take a few ids
// at a time, one per lane (a wave's time is that of its slowest lane), and judge
// them to the end: the first shift from the sets and stacks kept for the row, later
// ones by reduce chains, with the chains' tables and the DFA in LDS.
// An id whose lane's stack area was too small is judged again at the end with a
// large one.  Allowed ids are OR-ed into the mask.  The last chunk of a row to
// end writes the row's status (a row without open ids gets it from one thread).
// (Per id the work is a chain of dependent reads and branches, up to some 15,000
// cycles long, so what counts is how few ids a lane takes one after the other
// and that no wave waits for another in between.)
template <int MW, bool Full>
__global__ __launch_bounds__(kResThreads) void residue_kernel(Tables tb, const uint16_t* __restrict__ pool,
                                                              uint32_t* __restrict__ mask, uint8_t* __restrict__ ws,
                                                              size_t rbytes, int B, int32_t* __restrict__ status) {
  extern __shared__ __align__(16) uint8_t lds[];
  __shared__ int q_cnt, n_walk, n_lex, s_cnt, group_ctr, slow_ctr, any_s, ovf_s, step_lo, step_hi;
  __shared__ uint32_t sums[kResWaves];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const uint32_t* counts = open_counts(ws, rbytes, B);
  const ResLds WL = res_lds(tb);
  const RowLayout RL = row_layout(tb);
  // the batch's open ids, and the chunk size that deals them evenly (every wave
  // for itself)
  uint32_t mine = 0, first[kCountRegs];
#pragma unroll
  for (int j = 0; j < kCountRegs; ++j) {
    const int r = j * 64 + lane;
    first[j] = r < B ? counts[r] & (kListFull - 1u) : 0u;
  }
  const bool tables = tid >= kResThreads - kTableThreads;
  if (tables) {  // what every row needs, on its way while the chunk is found
    const int tt = tid - (kResThreads - kTableThreads);
    const StageRegion rg[2] = {{tb.bclass, lds + WL.bcls, 256u},
                               {(const uint8_t*)tb.term_info, lds + WL.tinfo, (uint32_t)tb.T * 4u}};
    const uint32_t blk = dma_regions<2>(rg, tt, kTableThreads);
    if (Full) {
      const StageRegion rl[2] = {{(const uint8_t*)tb.live, lds + WL.live, (uint32_t)tb.S * 32u},
                                 {(const uint8_t*)tb.dfa, lds + WL.dfa, (uint32_t)(tb.S * tb.C * 2)}};
      dma_lr(tb, lds, WL.lr, tt, kTableThreads, dma_regions<2>(rl, tt, kTableThreads, blk));
    }
  }
#pragma unroll
  for (int j = 0; j < kCountRegs; ++j) mine += first[j];
  for (int r = kCountRegs * 64 + lane; r < B; r += 64) mine += counts[r] & (kListFull - 1u);
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) mine += __shfl_xor(mine, d);
  const uint32_t all = __builtin_amdgcn_readfirstlane(mine);
  for (int r = (int)blockIdx.x * kResThreads + tid; r < B; r += (int)gridDim.x * kResThreads) {
    RowHeader* hr = (RowHeader*)(ws + kWsHead + (size_t)r * rbytes);
    if (counts[r] == 0u && hr->valid == kRowValid) {  // nothing open: the status is known
      const int32_t st = hr->pstat | (!hr->nonempty && !hr->eos_ok ? GRID_ROW_EMPTY : 0);
      if (status) status[r] = st;
      hr->fstat = st;
    }
  }
  // (a row's last chunk may be short, so up to B chunks more than full ones)
  const uint32_t room = gridDim.x - min((uint32_t)B, gridDim.x / 2u);
  const uint32_t per = (all + room - 1) / room;
  const uint32_t K = min((uint32_t)kChunkMax, max((uint32_t)kChunkMin, (per + 31u) / 32u * 32u));
  uint32_t in_row = 0;
  int row = all ? find_chunk(counts, first, B, K, blockIdx.x, &in_row) : -1;
  if (row < 0) {  // uniform over the workgroup
    dma_wait();
    return;
  }
  const uint8_t* rowblk = lds + WL.block;
  const RowHeader& h = *(const RowHeader*)rowblk;
  WalkView<MW, Full> wv;
  wv.tb = &tb;
  wv.lt = lr_tabs<Full>(tb, lds, WL.lr);
  wv.step = DfaView{Full ? (const uint16_t*)(lds + WL.dfa) : tb.dfa, lds + WL.bcls, tb.C};
  wv.win = in_mem<true>((const uint16_t*)(rowblk + RL.win));
  RowView<MW>& rv = wv.rv;
  rv.live = Full ? (const uint32_t*)(lds + WL.live) : tb.live;
  rv.tinfo = (const uint32_t*)(lds + WL.tinfo);
  wv.post = (const uint4*)(rowblk + RL.post);
  uint32_t* qid = (uint32_t*)(lds + WL.qid);
  uint16_t* qcls = (uint16_t*)(lds + WL.qcls);
  uint32_t* slow = (uint32_t*)(lds + WL.slow);
  uint16_t* areas = (uint16_t*)(lds + WL.areas);
  const int steps = stream_steps(tb.V);
  for (uint32_t c = blockIdx.x;;) {
    const uint32_t from = in_row * K;
    uint8_t* rw = ws + kWsHead + (size_t)row * rbytes;
    const RowHeader* hdr = (const RowHeader*)rw;
    const uint32_t have = counts[row];
    if (tid == 0) {
      q_cnt = 0;
      n_walk = 0;
      n_lex = 0;
      s_cnt = 0;
      group_ctr = kResWaves;  // the first groups are taken by wave number
      slow_ctr = 0;
      any_s = 0;
      ovf_s = 0;
      step_lo = steps;
      step_hi = 0;
    }
    const bool listed = have <= (uint32_t)open_list_cap(tb.V);  // uniform
    static_assert(kQueue <= kResThreads && kChunkMax % 64 == 0, "one id per thread");
    const int n_listed = (int)min(K, have - from);
    uint2 ent = make_uint2(0u, 0u);  // this thread's id and class
    if (listed && tid < n_listed) ent = ((const uint2*)(rw + RL.list))[from + tid];
    if (!tables) {
      const StageRegion rg[1] = {{rw, lds + WL.block, (uint32_t)RL.block}};
      dma_regions<1>(rg, tid, kChunkMax);
    }
    if (listed && tid < n_listed) {
      // what the id's lane will read is asked for here, beside the staging: its
      // first bytes are then in the cache
      const uint32_t u = tb.spell_of_id[ent.x];
      const uint32_t tf = tb.lex_token[(size_t)hdr->slot_id * tb.V + ent.x];
      const uint32_t r0 = tb.crec[hdr->cls_base + (ent.y & 0xFFFFu)].x;
      const uint32_t k0 = tb.spell_rec[u].x, t0 = tb.spell_tail[u].x;
      asm volatile("" ::"v"(tf), "v"(r0), "v"(k0), "v"(t0));
    }
    if (!listed) {  // from the open bitmap: the wave steps whose open ids start at a position in [from, from + K)
      const uint16_t* n_open = (const uint16_t*)(rw + RL.n_open);
      uint32_t run = 0;
      for (int s0 = 0; s0 < steps; s0 += kResThreads) {
        const int s = s0 + tid;
        const uint32_t v = s < steps ? n_open[s] : 0u;
        uint32_t tot = 0;
        const uint32_t ex = run + block_scan(v, sums, &tot);
        if (v && ex >= from && ex < from + K) {
          atomicMin(&step_lo, s);
          atomicMax(&step_hi, s + 1);
        }
        run += tot;
      }
      __syncthreads();
      for (int s = step_lo + wave; s < step_hi; s += kResWaves) {  // a wave per step: its ids to the queue
        if (n_open[s] == 0) continue;  // uniform
        const uint32_t b = ((const uint8_t*)(rw + RL.open))[s * (kStepIds / 8) + lane];
        int base = 0;
        if (lane == 0) base = atomicAdd(&q_cnt, (int)n_open[s]);
        base = __builtin_amdgcn_readfirstlane(base);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const bool o = (b >> j) & 1u;
          const uint64_t bal = __ballot(o);
          if (o) qid[base + lane_rank(bal)] = (uint32_t)(s * kStepIds + lane * 8 + j);
          base += __popcll(bal);
        }
      }
    }
    dma_wait();
    __syncthreads();
    const int n_ids = listed ? n_listed : q_cnt;
    uint32_t* mrow = mask + (size_t)row * tb.W;
    // a CI token of a row that claimed a CI-words entry also goes there
    uint32_t* cdst =
        h.ci_claim >= 0 ? (uint32_t*)(tb.ci_cache + (size_t)h.ci_claim * tb.ci_stride + kCiHeader) : nullptr;
    view_row(rv, tb, RL, rowblk);
    wv.pool = pool + h.stk_off;
    wv.depth = h.stk_depth;
    wv.lo = h.stk_depth > (uint32_t)kWalkWin ? h.stk_depth - kWalkWin : 0u;
    wv.q = h.q;
    // the ids in two kinds, those of walk classes from the queue's start, those
    // of lexicon classes from its end: a wave takes ids of one kind, so its lanes
    // mostly take the same branches
    const bool in = tid < n_ids;
    if (!listed) {
      const uint8_t* codes = rw + RL.codes;
      if (in) {
        const uint32_t cls = tb.cmap[(size_t)h.q * tb.V + qid[tid]];
        ent = make_uint2(qid[tid], cls | (uint32_t)(codes[cls] & 3u) << 16);
      }
      __syncthreads();  // the queue is read before it is filled again
    }
    {
      const bool walk = in && (ent.y >> 16) == kVerdictWalk;
      const uint64_t bw = __ballot(walk), bl = __ballot(in && !walk);
      int w0 = 0, l0 = 0;
      if (lane == 0) {
        if (bw) w0 = atomicAdd(&n_walk, __popcll(bw));
        if (bl) l0 = atomicAdd(&n_lex, __popcll(bl));
      }
      w0 = __builtin_amdgcn_readfirstlane(w0);
      l0 = __builtin_amdgcn_readfirstlane(l0);
      const int at = walk ? w0 + lane_rank(bw) : kQueue - 1 - (l0 + lane_rank(bl));
      if (in) {
        qid[at] = ent.x;
        qcls[at] = (uint16_t)ent.y;
      }
    }
    __syncthreads();
    // groups, one id per lane: the waves are shared out by the kinds' costs (a
    // walk takes about three times a lexicon id's time)
    const int nw = n_walk, nl = n_lex;
    const int w_waves = nw == 0 ? 0 : (nl == 0 ? kResWaves : min(kResWaves - 1, max(1, kResWaves * 3 * nw / (3 * nw + nl))));
    const int w_lanes = nw ? min(kLanesMax, (nw + w_waves - 1) / w_waves) : 1;
    const int l_lanes = nl ? min(kLanesMax, (nl + kResWaves - w_waves - 1) / (kResWaves - w_waves)) : 1;
    const int w_groups = (nw + w_lanes - 1) / w_lanes, groups = w_groups + (nl + l_lanes - 1) / l_lanes;
    bool any = false;
    for (int pass = 0; pass < 2; ++pass) {  // pass 1: the ids whose stack area was too small
      const int n_all = pass == 0 ? groups : s_cnt;
      const uint32_t cap = pass == 0 ? kFastLane : kSlowLane;
      for (int g = pass == 0 ? wave : (wave < kSlowWaves ? wave_grab(&slow_ctr) : n_all); g < n_all;
           g = wave_grab(pass == 0 ? &group_ctr : &slow_ctr)) {  // uniform per wave
        const bool gw = pass == 0 && g < w_groups;  // a group of walk ids
        const int pos = gw ? g * w_lanes + lane : (g - w_groups) * l_lanes + lane;
        const bool in = pass == 1 ? lane == 0 : (gw ? lane < w_lanes && pos < nw : lane < l_lanes && pos < nl);
        const mptr<true, uint16_t> base =
            in_mem<true>(areas + (pass == 0 ? wave * kLanesMax * kFastLane : wave * kSlowLane));
        uint32_t v = kVerdictReject, k = 0, m = 0, X[MW];
        int id = 0, here = 0;
        uint4 rec = make_uint4(0, 0, 0, 0);
        if (in) {
          const int at = pass == 1 ? (int)slow[g] : (gw ? pos : kQueue - 1 - pos);
          id = (int)qid[at];
          here = at;
          const uint32_t cls = qcls[at], u = tb.spell_of_id[id];
          LexLane lx;
          lx.tf = tb.lex_token[(size_t)h.slot_id * tb.V + id];
          rec = tb.crec[h.cls_base + cls];
          const uint4 rk = tb.spell_rec[u], tl = tb.spell_tail[u];
          lx.tb = &tb;
          lx.sl = slot_of(h.slot);
          lx.n = rk.w & 0xFFu;
          lx.b0 = (uint64_t)rk.x | (uint64_t)rk.y << 32;
          lx.b1 = lx.n > 8 ? (uint64_t)tl.x | (uint64_t)tl.y << 32 : 0ull;
          lx.b2 = lx.n > 8 ? (uint64_t)tl.z | (uint64_t)tl.w << 32 : 0ull;
          lx.rem = (uint64_t)h.rem_lo | (uint64_t)h.rem_hi << 32;
          lx.rem_len = h.rem_len;
          lx.lexnode = h.lexnode;
          v = walk_token<MW, Full>(wv, rec, lx, rk.w >> 8, base + lane * kFastLane, cap, k, m, X);
        }
        if (__any(v == kWalkTrail)) {  // trailing lexemes past the kept stacks
          const bool ok = trail_pairs<MW, Full>(wv, v == kWalkTrail, X, k, m, base);
          if (v == kWalkTrail) v = ok ? kVerdictAllow : kVerdictReject;
        }
        if (in) {
          if (v == kVerdictAllow) {
            atomicOr(mrow + (id >> 5), 1u << (id & 31));
            if (cdst && ci_class(rec.x)) atomicOr(cdst + (id >> 5), 1u << (id & 31));
            any = true;
          } else if (v == kWalkFull) {
            if (pass == 0) slow[atomicAdd(&s_cnt, 1)] = (uint32_t)here;
            else ovf_s = 1;
          }
        }
      }
      if (pass == 0 && any) any_s = 1;
      __syncthreads();
      if (s_cnt == 0) break;  // uniform
      if (pass == 1) {
        if (any) any_s = 1;
        __syncthreads();
      }
    }
    if (tid == 0) {
      // chunks ended, those that allowed an id, those that overflowed, 21 bits
      // each in one word: the last chunk needs no other memory of the others
      const unsigned long long add = 1ull | (any_s ? 1ull << 21 : 0ull) | (ovf_s ? 1ull << 42 : 0ull);
      const unsigned long long sum = atomicAdd(&((RowHeader*)rw)->done, add) + add;
      constexpr unsigned long long kField = (1ull << 21) - 1ull;
      if ((sum & kField) == ((have & (kListFull - 1u)) + K - 1u) / K) {
        int32_t st = h.pstat;
        if (sum >> 42) st |= GRID_ROW_OVERFLOW;
        if (!((sum >> 21) & kField) && !h.nonempty && !h.eos_ok) st |= GRID_ROW_EMPTY;
        if (status) status[row] = st;
        ((RowHeader*)rw)->fstat = st;
        ((RowHeader*)rw)->done = 0ull;
      }
    }
    c += gridDim.x;
    row = find_chunk(counts, first, B, K, c, &in_row);
    if (row < 0) break;  // uniform
    __syncthreads();  // the row's block and counters are free
  }
}

// The rows' statuses when the last phase is asked for them in a call of its own.
__global__ __launch_bounds__(64) void status_kernel(const uint8_t* __restrict__ ws, size_t rbytes, int B,
                                                    int32_t* __restrict__ status) {
  const int row = (int)(blockIdx.x * 64u + threadIdx.x);
  if (row >= B) return;
  const RowHeader* hdr = (const RowHeader*)(ws + kWsHead + (size_t)row * rbytes);
  status[row] = hdr->valid == kRowValid ? hdr->fstat : hdr->pstat;
}

// Publishes the CI-words entry of every row that claimed one and ended OK, or
// gives the slot back.
__global__ __launch_bounds__(64) void ci_publish_kernel(Tables tb, const uint8_t* __restrict__ ws, size_t rbytes, int B) {
  const int row = (int)(blockIdx.x * 64u + threadIdx.x);
  if (row >= B) return;
  const RowHeader* hdr = (const RowHeader*)(ws + kWsHead + (size_t)row * rbytes);
  if (hdr->valid != kRowValid || hdr->ci_claim < 0) return;
  uint32_t* e = (uint32_t*)(tb.ci_cache + (size_t)hdr->ci_claim * tb.ci_stride);
  __threadfence();
  __hip_atomic_store(e, hdr->fstat == GRID_ROW_OK ? 2u : 0u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
}

// Mask cache write-back: each row that claimed an entry in the prologue
// copies its finished mask row, EOS flag and status into it, then publishes
// it (a device-scope fence orders the copy before the state word).
__global__ __launch_bounds__(kBlock) void cache_publish_kernel(Tables tb, const uint32_t* __restrict__ mask,
                                                               const uint8_t* __restrict__ ws, size_t rbytes) {
  const int row = blockIdx.x;
  const RowHeader* hdr = (const RowHeader*)(ws + kWsHead + (size_t)row * rbytes);
  if (hdr->valid != kRowValid || hdr->cache_slot < 0) return;  // uniform
  CacheEntry* e = (CacheEntry*)(tb.cache + (size_t)hdr->cache_slot * tb.cache_stride);
  uint32_t* dst = (uint32_t*)(e + 1);
  const uint32_t* src = mask + (size_t)row * tb.W;
  for (int i = threadIdx.x; i < tb.W; i += kBlock) dst[i] = src[i];
  if (threadIdx.x == 0) {
    e->eos = hdr->eos_ok;
    e->status = (uint32_t)hdr->fstat;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    __threadfence();
    __hip_atomic_store(&e->state, 2u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// Empties a mask cache: every entry's state word to 0.
__global__ __launch_bounds__(kBlock) void cache_clear_kernel(uint8_t* cache, uint32_t n, uint32_t stride) {
  for (uint32_t i = blockIdx.x * kBlock + threadIdx.x; i < n; i += gridDim.x * kBlock)
    ((CacheEntry*)(cache + (size_t)i * stride))->state = 0u;
}

// ------------------------------------------------------------------- apply
// Each thread covers 8 consecutive logits of one row; the mask byte for them
// comes from one word.  (Logit by logit in every unaligned row, the fill of
// 47 rows of 50,257 cost 2 us more, 71.4 against 69.2 for mask and fill.)
template <typename T>
__global__ __launch_bounds__(kBlock) void apply_kernel(const uint32_t* __restrict__ mask, T* logits, int B,
                                                       int V, int W, int64_t stride, uint32_t neg_inf_bits,
                                                       bool aligned) {
  // row blockIdx.y; groups of 8 logits along it, grid-stride in x
  const int groups = (V + 7) >> 3;
  const int row = (int)blockIdx.y;
  (void)B;
  for (int grp = (int)(blockIdx.x * kBlock + threadIdx.x); grp < groups; grp += (int)(gridDim.x * kBlock)) {
    const int col = grp * 8;
    const uint32_t bits = (mask[(size_t)row * W + (col >> 5)] >> (col & 31)) & 0xFFu;
    if (bits == 0xFFu) continue;
    fill_group<T>(logits + (int64_t)row * stride + col, bits, V - col, aligned, neg_inf_bits);
  }
}

// ------------------------------------------------------------- rolling hash
// x of lane (me + k) % 4 of the quad, by DPP quad_perm.
template <int K>
__device__ __forceinline__ uint64_t quad_rot(uint64_t x) {
  constexpr int ctrl = (K & 3) | ((K + 1) & 3) << 2 | ((K + 2) & 3) << 4 | ((K + 3) & 3) << 6;
  const int lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)x, ctrl, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(x >> 32), ctrl, 0xF, 0xF, true);
  return (uint64_t)(uint32_t)lo | (uint64_t)(uint32_t)hi << 32;
}

// node_hash by the four lanes of a quad, all with the same arguments: lane j
// holds column j of BLAKE2b's 4 x 4 state, so the four G of a half round run
// side by side and the rows are turned by lane moves for the diagonals.  Two of
// the 16 message words are not zero; each is kept masked for each lane, and a
// half round adds only where its schedule has one of the two.
// (One hash is a serial chain of 24 G, about 1 us; by one lane, 96 of them took
// 4.5 us: 32 rows of depth 30 hashed in 140 us.)
__device__ __forceinline__ uint64_t node_hash4(uint64_t parent, uint32_t state, uint32_t sym) {
  const uint32_t j = threadIdx.x & 3u;
  const uint64_t m[2] = {parent, (uint64_t)state | (uint64_t)sym << 32};
  uint64_t mine[2][4];
#pragma unroll
  for (int w = 0; w < 2; ++w)
#pragma unroll
    for (uint32_t l = 0; l < 4; ++l) mine[w][l] = m[w] & (0ull - (uint64_t)(j == l));
  auto pick = [&](uint64_t x0, uint64_t x1, uint64_t x2, uint64_t x3) {
    return j == 0 ? x0 : (j == 1 ? x1 : (j == 2 ? x2 : x3));
  };
  constexpr uint64_t h0 = kBlake2bIv[0] ^ 0x01010000ull ^ 16ull;  // digest length 16, no key, fanout 1, depth 1
  uint64_t a = pick(h0, kBlake2bIv[1], kBlake2bIv[2], kBlake2bIv[3]);
  uint64_t b = pick(kBlake2bIv[4], kBlake2bIv[5], kBlake2bIv[6], kBlake2bIv[7]);
  uint64_t c = pick(kBlake2bIv[0], kBlake2bIv[1], kBlake2bIv[2], kBlake2bIv[3]);
  uint64_t d = pick(kBlake2bIv[4] ^ 16ull, kBlake2bIv[5], ~kBlake2bIv[6], kBlake2bIv[7]);  // counter 16, final block
#pragma unroll
  for (int r = 0; r < 12; ++r) {
#pragma unroll
    for (int half = 0; half < 2; ++half) {  // columns, then diagonals
#pragma unroll
      for (int y = 0; y < 2; ++y) {  // a's two additions
        a += b;
#pragma unroll
        for (int l = 0; l < 4; ++l) {
          const int w = kBlake2bSigma[r % 10][8 * half + 2 * l + y];
          if (w < 2) a += mine[w][l];
        }
        d = rotr64(d ^ a, y ? 16 : 32);
        c += d;
        b = rotr64(b ^ c, y ? 63 : 24);
      }
      b = half ? quad_rot<3>(b) : quad_rot<1>(b);
      c = quad_rot<2>(c);
      d = half ? quad_rot<1>(d) : quad_rot<3>(d);
    }
  }
  const uint64_t v = a ^ c;  // lane 0: words 0 and 8
  const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)v, 0, 0xF, 0xF, true);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(v >> 32), 0, 0xF, 0xF, true);
  return h0 ^ ((uint64_t)lo | (uint64_t)hi << 32);
}

// ------------------------------------------------------------------ accept
// The whole stack stk[0, d) as a read-only base for simulations: in LDS it
// is the window, in global memory the pool.
template <bool L>
__device__ inline BaseStack<L> whole_stack(mptr<L, uint16_t> stk, uint32_t d) {
  if constexpr (L) return BaseStack<L>{nullptr, stk, d, 0u};
  else return BaseStack<L>{stk, nullptr, d, d};
}

// Reduce chain of terminal x on the stack stk[0, d), pushes above d (the
// stack below stays as it is).  1 shift, 2 accept (x is the end of input), 0
// error, -1 capacity (the area, or more than kGuard steps since the stack last
// fell).  With commit, a shift makes the chain's result the
// stack: the pushed states move down onto the popped entries, then x's
// shift target goes on top (so a winner costs one chain, not two).
template <bool L, int MW>
__device__ int chain_shift(const ParseTabs<L>& pt, mptr<L, uint16_t> stk, uint32_t& d, uint32_t cap, int x,
                           bool commit, uint32_t& lo_mod) {
  if (d >= cap) return -1;
  const BaseStack<L> bs = whole_stack<L>(stk, d);
  const mptr<L, uint16_t> tmp = stk + d;
  const int tmpcap = (int)(cap - d);
  const uint32_t w = (uint32_t)x >> 5, bit = 1u << (x & 31);
  uint32_t k = d;
  int m = 0, t = 0;
  uint32_t s = stack_at_top<L>(bs, k, m, tmp, 0, tmp), below = kNoState;
  for (int guard = 0; guard < kGuard; ++guard) {
    const uint32_t a = action_of<L, MW>(pt, s, w, bit);
    if (a >= kActShiftP) {
      if (a != kActShiftP) return 0;
      if (x == pt.T) return 2;
      if (commit) {
        for (int i = 0; i < t; ++i) stk[k + (uint32_t)i] = tmp[i];  // k <= d: a forward move is safe
        lo_mod = min(lo_mod, k);
        d = k + (uint32_t)t;
        if (d >= cap) return -1;
        stk[d++] = shift_target<L, MW>(pt, s, x);
      }
      return 1;
    }
    const uint32_t len = a >> 16, k0 = k;
    if (!pop_len(len, k, m, t)) return 0;
    if (k < k0) guard = 0;
    const uint32_t sb = goto_source<L>(bs, len, s, below, k, m, tmp, t, tmp);
    const uint16_t g = goto_of<L>(pt, sb, a & 0xFFFFu);
    if (g == kNoGoto) return 0;
    if (t >= tmpcap) return -1;
    tmp[t++] = g;
    below = sb;
    s = g;
  }
  return -1;
}

// The same without commit, one lane's: the pushes go to the lane's own area tmp
// of kAccLane entries; 3 when the chain needs a larger one.
constexpr int kAccLane = 16;
template <bool L, int MW>
__device__ int chain_test(const ParseTabs<L>& pt, mptr<L, const uint16_t> stk, uint32_t d, uint32_t cap, uint32_t x,
                          mptr<true, uint16_t> tmp) {
  if (d >= cap) return -1;
  const uint32_t w = x >> 5, bit = 1u << (x & 31);
  uint32_t k = d, t = 0, s = stk[d - 1u];
  for (int guard = 0; guard < kGuard; ++guard) {
    const uint32_t a = action_of<L, MW>(pt, s, w, bit);
    if (a >= kActShiftP) return a == kActShiftP ? 1 : 0;
    const uint32_t len = a >> 16, dt = min(t, len);
    if (len - dt >= k) return 0;
    if (len > dt) guard = 0;
    t -= dt;
    k -= len - dt;
    uint32_t sb = s;
    if (len) {
      if (t) sb = tmp[t - 1u];
      else sb = stk[k - 1u];
    }
    s = goto_of<L>(pt, sb, a & 0xFFFFu);
    if (s == kNoGoto) return 0;
    if (t >= cap - d) return -1;
    if (t >= (uint32_t)kAccLane) return 3;
    tmp[t++] = (uint16_t)s;
  }
  return -1;
}

// The lexer tables an advance reads (global memory, or their LDS copies).
struct LexPtrs {
  const uint16_t* dfa;
  const uint8_t* bclass;
  const uint32_t* term_info;
  const uint32_t* acc_off;
  const uint8_t* acc_list;
  const uint32_t* live;
};

// A row's lexer side: DFA state, lexicon node and its flags, pending lexeme
// (length, first 8 bytes).
struct AccLex {
  uint32_t q, lex, flags, rem;
  uint64_t head;
};

// A token's bytes: the first kAccBytes in registers, the rest in the tail table.
constexpr uint32_t kAccBytes = 24;
struct AccToken {
  uint64_t b0, b1, b2;
  uint32_t n, chunk;  // length (0: special or empty), first overflow chunk
  __device__ __forceinline__ uint32_t at(const Tables& tb, uint32_t i) const {
    if (i >= kAccBytes) return reinterpret_cast<const uint8_t*>(tb.spell_tail + chunk)[i - kAccBytes];
    return (uint32_t)(window8(b0, b1, b2, i) & 0xFFu);
  }
};

// The lexicon nodes the token's bytes lead to, and their flags: entry
// [o * kAccBytes + i] after bytes o..i from the trie's root, and, for o =
// kAccBytes, after bytes 0..i from the pending lexeme's node.
struct AccTrie {
  uint32_t node[(kAccBytes + 1) * kAccBytes], flags[(kAccBytes + 1) * kAccBytes];
};

// One row's advance by token tok (section 6.1, per-token step 7), by one wave, on
// the stack stk[0, d) of capacity cap, with the LR tables pt; lo_mod falls to the
// lowest stack index the advance rewrites (entries below it are unchanged).  The
// token's bytes go through the lexer with maximal munch; a byte that kills the DFA
// emits the pending lexeme as the highest-priority candidate that is ignored or
// shifts and passes its category's lexicon, and a shifted terminal runs its reduce
// chain on the stack (lane 0).  The new pending lexeme must still complete to an
// allowed or ignored terminal (Definition 2; a lane per terminal, the lowest that
// does not fail decides, as if tried in order).  The end-of-sequence token is
// accepted when the end-of-sequence gate holds (section 3.2).  Returns the row
// status in every lane; with GRID_ROW_OK, d and lx (lane 0's) are the new
// configuration's.
template <bool L, int MW>
__device__ __forceinline__ int advance_row(const Tables& tb, const LexPtrs lp, const ParseTabs<L>& pt, const Slot& sl,
                           mptr<L, uint16_t> stk, uint32_t& d, uint32_t cap, int tok, const AccToken& tk,
                           const AccTrie& trie, mptr<true, uint16_t> areas, AccLex& lx, uint32_t& lo_mod) {
  const uint32_t lane = threadIdx.x & 63u;
  auto ignored = [&](int t) { return (lp.term_info[t] & 1u) != 0; };
  auto restricted_cat = [&](int t) -> int {  // category the row's lexicon restricts, or -1
    const uint32_t c = (lp.term_info[t] >> 8) & 0xFFu;
    return c != 0xFFu && ((sl.restricted >> c) & 1u) ? (int)c : -1;
  };
  // can terminal t be shifted from the stack now (reduce chain only, pushes
  // above the stack, which stays as it is)?
  // 1 shift, 2 accept (the end of input), 0 error, -1 capacity
  auto shifts = [&](int t) -> int { return chain_shift<L, MW>(pt, stk, d, cap, t, false, lo_mod); };
  // the pending lexeme's winner in state q, its reduce chain and shift applied to
  // the stack when it is not ignored: -1 none, else the terminal; capacity
  // problems surface as -2
  auto winner = [&]() -> int {
    for (uint32_t j = lp.acc_off[lx.q]; j < lp.acc_off[lx.q + 1]; ++j) {
      const int t = lp.acc_list[j];
      const int c = restricted_cat(t);
      if (c >= 0 && !((lx.flags >> (8 + c)) & 1u)) continue;
      if (ignored(t)) return t;
      const int r = chain_shift<L, MW>(pt, stk, d, cap, t, true, lo_mod);
      if (r < 0) return -2;
      if (r == 1) return t;
    }
    return -1;
  };
  constexpr int kTrailing = -1;  // all bytes taken: the pending lexeme's test is left
  auto bytes = [&]() -> int {
    if (tok == tb.eos_id) {  // the configuration itself stays as it is
      int ok = 0;
      if (lx.rem == 0) {
        ok = shifts(tb.T) == 2;
      } else {
        const int w = winner();
        if (w == -2) return GRID_ROW_OVERFLOW;
        if (w >= 0) ok = shifts(tb.T) == 2;
      }
      return ok ? GRID_ROW_FINISHED : GRID_ROW_NOT_VIABLE;
    }
    if (tk.n == 0) return GRID_ROW_NOT_VIABLE;  // special or empty token
    uint32_t from = kAccBytes;                  // where the lexeme starts (kAccBytes: the pending one)
    for (uint32_t i = 0; i < tk.n; ++i) {
      const uint32_t b = tk.at(tb, i), bc = lp.bclass[b];
      int nq = lp.dfa[lx.q * tb.C + bc];
      if (nq == kDead) {  // b kills the pending lexeme: emit it
        if (lx.rem == 0 || lp.acc_off[lx.q + 1] == lp.acc_off[lx.q]) return GRID_ROW_NOT_VIABLE;
        const int w = winner();
        if (w == -2) return GRID_ROW_OVERFLOW;
        if (w < 0) return GRID_ROW_NOT_VIABLE;
        nq = lp.dfa[kStart * tb.C + bc];
        if (nq == kDead) return GRID_ROW_NOT_VIABLE;
        lx.lex = 0;
        lx.rem = 0;
        lx.head = 0;
        from = i;
      }
      lx.q = (uint32_t)nq;
      if (i < kAccBytes) {
        lx.lex = trie.node[from * kAccBytes + i];
        lx.flags = trie.flags[from * kAccBytes + i];
      } else {
        lx.lex = lex_child(tb, sl, lx.lex, b);
        lx.flags = lex_flags_of(tb, sl, lx.lex);
      }
      if (lx.rem < 8) lx.head = (lx.head & ~(0xFFull << (8u * lx.rem))) | (uint64_t)b << (8u * lx.rem);
      ++lx.rem;
    }
    return kTrailing;
  };
  int st = 0;
  if (lane == 0) st = bytes();
  st = __builtin_amdgcn_readfirstlane(st);
  if (st != kTrailing) return st;
  // Definition 2 for the pending lexeme
  const uint32_t q = __builtin_amdgcn_readfirstlane(lx.q), fl = __builtin_amdgcn_readfirstlane(lx.flags);
  const uint32_t dd = __builtin_amdgcn_readfirstlane(d);
  const uint32_t* lv = lp.live + (size_t)q * 8;
  for (int g = 0; g < (tb.T + 63) / 64; ++g) {
    const int t = g * 64 + (int)lane;
    int r = 0;
    if (t < tb.T && ((lv[t >> 5] >> (t & 31)) & 1u)) {
      const int c = restricted_cat(t);
      if (c < 0 || ((fl >> c) & 1u))
        r = ignored(t) ? 1 : chain_test<L, MW>(pt, stk, dd, cap, (uint32_t)t, areas + lane * kAccLane);
    }
    uint64_t todo = __ballot(r != 0);
    while (todo) {
      const int f = __ffsll((unsigned long long)todo) - 1;
      int rf = __builtin_amdgcn_readlane(r, f);
      if (rf == 3) {  // its area was too small: above the stack, by lane 0
        if (lane == 0) rf = shifts(g * 64 + f);
        rf = __builtin_amdgcn_readfirstlane(rf);
      }
      if (rf < 0) return GRID_ROW_OVERFLOW;
      if (rf == 1) return GRID_ROW_OK;
      todo &= todo - 1ull;
    }
  }
  return GRID_ROW_NOT_VIABLE;
}

// LDS bytes of the lexer tables an accept workgroup stages beside the LR
// tables and the stack: DFA, byte classes, terminal info, accept lists, live
// sets (offsets from the start of the area).
struct AccLexLds {
  uint32_t dfa, bclass, tinfo, acc_off, acc_list, live, total;
};
__host__ __device__ inline AccLexLds accept_lex_lds(const Tables& tb) {
  AccLexLds L;
  uint32_t o = 0;
  L.dfa = o;
  o += pad16((uint32_t)(tb.S * tb.C * 2));
  L.bclass = o;
  o += 256;
  L.tinfo = o;
  o += pad16((uint32_t)tb.T * 4u);
  L.acc_off = o;
  o += pad16((uint32_t)(tb.S + 1) * 4u);
  L.acc_list = o;
  o += pad16((uint32_t)tb.n_acc);
  L.live = o;
  o += pad16((uint32_t)tb.S * 32u);
  L.total = o;
  return L;
}
constexpr uint32_t kAcceptLdsMax = 152 * 1024;

constexpr uint32_t kAccStack = 8192;  // stack entries an accept workgroup keeps in LDS

__host__ __device__ inline uint32_t accept_stack_cap(uint32_t cap) { return cap < kAccStack ? cap : kAccStack; }

// Device incremental advance: one workgroup per row.  The LR tables, the lexer
// tables and the row's stack are staged in LDS and one wave advances the row
// there (the chain of dependent table reads is the cost, so every read is an LDS
// read).  While the other waves stage, wave 0 reads the token's bytes and follows
// the lexicon trie from every byte it may start a lexeme at, a lane each, and
// wave 1 copies the stack: read by the advancing thread in turn, a byte's trie
// node was a global read each.  256 DML rows out of place take 14.4 us (2.5 more with
// one thread reading the token and the trie after the staging and trying the
// trailing lexeme's terminals in turn).
// Every row's output is self-contained, whatever its status: the input stack
// is copied to the row's own area pool_out + b * cap (checking every entry is
// an LR state) and the configuration written to cfg_out points there; an
// advance then rewrites only the entries from the lowest one it changed.  A
// stack that outgrows the LDS area while cap allows more is advanced again
// from the start, by the same routine, on that global copy with the tables in
// global memory; so is every row when the LR tables are too large to stage
// (use_lds = 0).  A row whose stack does not fit cap gets depth 0 (a
// configuration every call rejects).
//
// In place (inplace = 1; cfg_out == cfgs, pool_out == pool): row b's stack
// lives in pool[b * cap, (b + 1) * cap) and is its persistent arena -- the
// entries below the lowest one a step rewrites are neither copied nor
// written, the rewritten ones are written back from LDS, and, with hash, the
// rolling hash of every rewritten entry is recomputed from its parent's (one
// hash per pushed node).  A row that is not advanced keeps its stack and
// configuration untouched; a stack too deep for the LDS area is reported as
// an overflow (the out-of-place call handles it).
constexpr int kAccThreads = 512;
constexpr uint32_t kAccFirst = 1024;  // stack entries wave 1 copies alone
template <int MW>
__global__ __launch_bounds__(kAccThreads) void accept_kernel(Tables tb, const grid_config* cfgs, const uint16_t* pool,
                                                             const int32_t* __restrict__ tokens, grid_config* cfg_out,
                                                             uint16_t* pool_out, uint64_t* hash, uint32_t cap,
                                                             int32_t* status, int use_lds, int use_lex, int inplace,
                                                             int tok_stride, int late) {
  extern __shared__ __align__(16) uint8_t alds[];
  __shared__ int s_st, s_bad;
  __shared__ uint32_t s_d, s_lo;
  __shared__ AccTrie trie;
  __shared__ uint16_t areas[64 * kAccLane];
  const int row = (int)blockIdx.x, tid = (int)threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const ParseLds PL = prologue_parse_lds(tb);
  const uint32_t lcap = accept_stack_cap(cap);
  const mptr<true, uint16_t> stk_l = in_mem<true>((uint16_t*)(alds + PL.total));
  // the tables by waves 2 and up; the lexer's too when they fit: every byte step
  // is then an LDS read
  const AccLexLds XL = accept_lex_lds(tb);
  uint8_t* xl = alds + PL.total + pad16(lcap * 2u);
  LexPtrs lp{tb.dfa, tb.bclass, tb.term_info, tb.acc_off, tb.acc_list, tb.live};
  if (use_lds && use_lex)
    lp = LexPtrs{(const uint16_t*)(xl + XL.dfa), xl + XL.bclass, (const uint32_t*)(xl + XL.tinfo),
                 (const uint32_t*)(xl + XL.acc_off), xl + XL.acc_list, (const uint32_t*)(xl + XL.live)};
  if (use_lds && wave >= 2 && (!late || (uint32_t)tokens[(size_t)row * tok_stride] < (uint32_t)tb.V)) {
    const int t2 = tid - 128, nt = kAccThreads - 128;
    const StageRegion rg[4] = {parse_region(tb, alds, PL, 0), parse_region(tb, alds, PL, 1),
                               parse_region(tb, alds, PL, 2), parse_region(tb, alds, PL, 3)};
    const uint32_t first = dma_regions<4>(rg, t2, nt);
    if (use_lex) {
      const StageRegion rx[6] = {{(const uint8_t*)tb.dfa, xl + XL.dfa, (uint32_t)(tb.S * tb.C * 2)},
                                 {tb.bclass, xl + XL.bclass, 256u},
                                 {(const uint8_t*)tb.term_info, xl + XL.tinfo, (uint32_t)tb.T * 4u},
                                 {(const uint8_t*)tb.acc_off, xl + XL.acc_off, (uint32_t)(tb.S + 1) * 4u},
                                 {tb.acc_list, xl + XL.acc_list, (uint32_t)tb.n_acc},
                                 {(const uint8_t*)tb.live, xl + XL.live, (uint32_t)tb.S * 32u}};
      dma_regions<6>(rx, t2, nt, first);
    }
  }
  const grid_config cfg = cfgs[row];
  const int tok = tokens[(size_t)row * tok_stride];
  const uint32_t d0 = cfg.stk_depth;
  uint16_t* out_stk = pool_out + (size_t)row * cap;
  const bool copyable = d0 >= 1 && d0 <= cap && (!inplace || cfg.stk_off == (uint32_t)row * cap);  // uniform
  bool bad = !copyable || cfg.q >= (uint32_t)tb.S || cfg.q == (uint32_t)kDead || cfg.slot >= (uint32_t)tb.n_slots ||
             tok < 0 || tok >= tb.V;
  if (bad && inplace) {  // nothing to do (uniform)
    dma_wait();
    __syncthreads();  // every wave has its row
    if (tid == 0 && status) status[row] = GRID_ROW_BAD_CONFIG;
    return;
  }
  const bool fits = use_lds && d0 < lcap;  // uniform
  Slot sl{};
  AccToken tk{};
  uint32_t flags0 = 0;
  if (wave == 0 && !bad) {
    sl = load_slot(tb, (int)cfg.slot);
    bad = cfg.lexnode != kNoLex && cfg.lexnode >= sl.nodes;
  }
  if (wave == 0 && !bad) {
    const uint32_t su = tb.spell_of_id[tok];
    if (su != 0xFFFFFFFFu) {
      const uint4 rk = tb.spell_rec[su], tl = tb.spell_tail[su];
      tk.n = rk.w & 0xFFu;
      tk.chunk = rk.w >> 8;
      tk.b0 = (uint64_t)rk.x | (uint64_t)rk.y << 32;
      if (tk.n > 8) {
        tk.b1 = (uint64_t)tl.x | (uint64_t)tl.y << 32;
        tk.b2 = (uint64_t)tl.z | (uint64_t)tl.w << 32;
      }
    }
    flags0 = lex_flags_of(tb, sl, cfg.lexnode);
    const uint32_t n = min(tk.n, kAccBytes);
    if (lane <= (int)kAccBytes) {  // lane o follows the trie from byte o, lane kAccBytes from the pending node
      uint32_t node = lane < (int)kAccBytes ? 0u : cfg.lexnode;
      for (uint32_t i = lane < (int)kAccBytes ? (uint32_t)lane : 0u; i < n; ++i) {
        node = lex_child(tb, sl, node, (uint32_t)(window8(tk.b0, tk.b1, tk.b2, i) & 0xFFu));
        trie.node[lane * kAccBytes + i] = node;
        trie.flags[lane * kAccBytes + i] = lex_flags_of(tb, sl, node);
      }
    }
  }
  bool foreign = false;  // an entry that is no LR state
  auto copy = [&](uint32_t i) {  // the input stack to the row's output area and to LDS, entries checked
    const uint16_t v = pool[cfg.stk_off + i];
    foreign = foreign || v >= (uint32_t)tb.NS;
    if (!inplace) out_stk[i] = v;
    if (fits) stk_l[i] = v;
  };
  if (wave == 1) {
    if (copyable)
      for (uint32_t i = (uint32_t)lane; i < min(d0, kAccFirst); i += 64u) copy(i);
    foreign = __any(foreign);
    if (lane == 0) s_bad = foreign ? 1 : 0;
  }
  dma_wait();
  __syncthreads();  // the tables and the stack's first entries are in LDS
  if (copyable && d0 > kAccFirst) {  // uniform
    for (uint32_t i = kAccFirst + (uint32_t)tid; i < d0; i += kAccThreads) copy(i);
    if (foreign) s_bad = 1;
    __syncthreads();
  }
  grid_config out = cfg;
  if (!inplace) {
    if (copyable) out.stk_off = (uint32_t)row * cap;
    else out.stk_depth = 0;
  }
  int st = -1;  // -1: not advanced in LDS
  uint32_t d = d0, lo = d0;
  AccLex lx{};
  if (wave == 0) {
    uint64_t head0 = 0;
    for (int k = 0; k < 8; ++k) head0 |= (uint64_t)cfg.rem_head[k] << (8 * k);
    auto start = [&]() {
      lx.q = cfg.q;
      lx.lex = cfg.lexnode;
      lx.flags = flags0;
      lx.rem = (cfg.flags & 1u) ? 0u : cfg.rem_len;
      lx.head = lx.rem > 0 ? head0 : 0ull;
      d = d0;
      lo = d0;
    };
    if (bad || s_bad) {
      st = GRID_ROW_BAD_CONFIG;
    } else {
      const mptr<true, uint16_t> ar = in_mem<true>(areas);
      if (fits) {
        start();
        st = advance_row<true, MW>(tb, lp, lds_parse(tb, alds, PL), sl, stk_l, d, lcap, tok, tk, trie, ar, lx, lo);
        if (st == GRID_ROW_OVERFLOW && lcap < cap) st = -1;
      }
      if (inplace && st == -1) st = GRID_ROW_OVERFLOW;  // in place, only the LDS route
      if (st == -1) {  // the global route, from the start, on the output copy
        start();
        const LexPtrs lg{tb.dfa, tb.bclass, tb.term_info, tb.acc_off, tb.acc_list, tb.live};
        st = advance_row<false, MW>(tb, lg, global_parse(tb), sl, in_mem<false>(out_stk), d, cap, tok, tk, trie, ar, lx, lo);
        if (lane == 0) {
          if (st != GRID_ROW_OK)  // a refused token leaves the row's input stack in its area
            for (uint32_t i = lo; i < d0; ++i) out_stk[i] = pool[cfg.stk_off + i];
          s_st = -1;
        }
      } else if (lane == 0) {
        s_st = st;
      }
    }
    if (lane == 0) {
      if (st == GRID_ROW_BAD_CONFIG) s_st = st;
      s_d = d;
      s_lo = lo;
    }
  }
  __syncthreads();
  if (s_st == GRID_ROW_OK)  // the entries the advance rewrote
    for (uint32_t i = s_lo + (uint32_t)tid; i < s_d; i += kAccThreads) out_stk[i] = stk_l[i];
  if (s_st == GRID_ROW_OK && hash && tid < 4) {  // rolling hashes of the rewritten entries, each from its parent's
    const uint32_t off = out.stk_off, top = s_d;
    uint64_t hv = hash[off + s_lo - 1];  // s_lo >= 1: the bottom entry is never popped
    for (uint32_t i = s_lo; i < top; ++i) {
      const uint32_t sv = stk_l[i];
      hv = node_hash4(hv, sv, tb.state_sym[sv]);
      if (tid == 0) hash[off + i] = hv;
    }
  }
  if (tid != 0) return;
  if (inplace && st != GRID_ROW_OK) {
    if (status) status[row] = st;
    return;
  }
  if (st == GRID_ROW_OK) {
    out.stk_depth = d;
    out.lexnode = lx.lex;
    out.q = (uint16_t)lx.q;
    out.flags = lx.rem == 0 ? 1u : 0u;
    out.rem_len = lx.rem;
    for (int k = 0; k < 8; ++k) out.rem_head[k] = (uint8_t)(lx.head >> (8 * k));
  }
  cfg_out[row] = out;
  if (status) status[row] = st;
}

// Rolling hash of every stack entry of every row: entry 0 is the root (hash 0),
// entry i > 0 hashes the one below it, its LR state and that state's accessing
// symbol.  Four lanes per row, 16 rows per wave; each entry's hash needs its
// parent's, so a row's time is its depth times one hash, and the next entries'
// states and symbols are read while it runs.
__global__ __launch_bounds__(64) void stack_hash_kernel(Tables tb, const grid_config* __restrict__ cfgs,
                                                       const uint16_t* __restrict__ pool, uint64_t* __restrict__ hash,
                                                       int B) {
  const int row = (int)(blockIdx.x * 16u + threadIdx.x / 4u);
  if (row >= B) return;  // uniform over the four lanes
  const grid_config cfg = cfgs[row];
  const uint32_t n = cfg.stk_depth;
  const uint16_t* st = pool + cfg.stk_off;
  uint64_t* out = hash + cfg.stk_off;
  auto state = [&](uint32_t i) -> uint32_t { return i < n ? st[i] : kNoState; };
  auto symbol = [&](uint32_t sv) -> uint32_t { return sv < (uint32_t)tb.NS ? tb.state_sym[sv] : kNoSymbol; };
  const bool writes = (threadIdx.x & 3u) == 0u;
  if (n && writes) out[0] = 0ull;
  uint64_t h = 0;
  uint32_t s0 = state(1), s1 = state(2), y0 = symbol(s0);
  for (uint32_t i = 1; i < n; ++i) {
    const uint32_t s2 = state(i + 2), y1 = symbol(s1);
    h = node_hash4(h, s0, y0);
    if (writes) out[i] = h;
    s0 = s1;
    s1 = s2;
    y0 = y1;
  }
}

// An artifact that is empty needs no device copy.
bool bound(const grid_compiled* g, int which) {
  const void* p = nullptr;
  size_t n = 0;
  return g->dev[which] != nullptr || (grid_artifact(g, which, &p, &n) == GRID_OK && n == 0);
}

// Raises a kernel's dynamic-LDS limit (needed above 64 KB of LDS in total) once
// per (kernel, device, size); the record of what was raised is shared by all host
// threads.
bool raise_lds(const void* fn, uint32_t bytes) {
  struct Entry {
    const void* fn;
    int dev;
    uint32_t bytes;
  };
  static std::mutex mu;
  static Entry done[64];
  static int n_done = 0;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return false;
  std::lock_guard<std::mutex> lock(mu);
  for (int i = 0; i < n_done; ++i)
    if (done[i].fn == fn && done[i].dev == dev && done[i].bytes >= bytes) return true;
  if (hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes) != hipSuccess) return false;
  if (n_done < 64) done[n_done++] = {fn, dev, bytes};
  return true;
}

// Compute units of the current device, looked up once per device.
int compute_units() {
  constexpr int kDevices = 64;
  static std::atomic<int> seen[kDevices];
  int dev = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kDevices) return 256;
  cus = seen[dev].load(std::memory_order_relaxed);
  if (cus == 0) {
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0) cus = 256;
    seen[dev].store(cus, std::memory_order_relaxed);
  }
  return cus;
}

template <int MW>
int launch_mask(const Tables& tb, int B, const grid_config* cfg_dev, const uint16_t* pool, uint32_t* mask,
                uint8_t* eos, int32_t* status, uint8_t* ws, size_t rb, uint32_t phases, hipStream_t s) {
  if (phases & GRID_PHASE_PROLOGUE) {
    const uint32_t pro = prologue_lds(tb).total, jud = judge_lds(tb).total;
    const bool in_lds = lr_in_lds(tb);
    const auto prologue = in_lds ? prologue_kernel<MW, true> : prologue_kernel<MW, false>;
    if (!raise_lds((const void*)prologue, pro) || !raise_lds((const void*)judge_kernel<MW>, jud))
      return fail(GRID_E_HIP, "grid_mask: cannot raise the LDS limit");
    hipLaunchKernelGGL(prologue, dim3(B), dim3(kProThreads), pro, s, tb, cfg_dev, pool, mask, eos, status, ws, rb);
    // a row's classes: as many parts as make four workgroups per compute unit over
    // the batch (each stages the tables anew), at least one block of classes each
    const int blocks = std::max(1, (tb.max_classes + kJudgeThreads - 1) / kJudgeThreads);
    const int parts = std::max(1, std::min(4 * compute_units() / B, blocks));
    hipLaunchKernelGGL(judge_kernel<MW>, dim3((uint32_t)B * (uint32_t)parts), dim3(kJudgeThreads), jud, s, tb, ws, rb, parts);
  }
  if (phases & GRID_PHASE_WALK) {
    const uint32_t lds = stream_lds(tb).total;
    if (!raise_lds((const void*)stream_kernel, lds)) return fail(GRID_E_HIP, "grid_mask: cannot raise the LDS limit");
    // a row's slices: three workgroups per compute unit over the batch (their
    // LDS lets them share one), at least one wave step each
    const int steps = stream_steps(tb.V);
    const int want = std::max(1, std::min(3 * compute_units() / B, steps));
    const int slice_ids = (steps + want - 1) / want * kStepIds;
    const int slices = (tb.V + slice_ids - 1) / slice_ids;
    const long long blocks = (long long)B * slices;
    if (blocks > 0x7FFFFFFFll) return fail(GRID_E_CAPACITY, "grid_mask: batch x vocabulary too large");
    hipLaunchKernelGGL(stream_kernel, dim3((uint32_t)blocks), dim3(kStreamThreads), lds, s, tb, mask, ws, rb, B, slices,
                       slice_ids);
  }
  if (phases & GRID_PHASE_RESIDUE) {
    const ResLds RL = res_lds(tb);
    const void* fn = RL.full ? (const void*)residue_kernel<MW, true> : (const void*)residue_kernel<MW, false>;
    if (!raise_lds(fn, RL.total)) return fail(GRID_E_HIP, "grid_mask: cannot raise the LDS limit");
    // one workgroup per compute unit, no more than the batch can have chunks
    const long long chunks = (long long)B * ((tb.V + kChunkMin - 1) / kChunkMin);
    const dim3 grid((uint32_t)std::min((long long)compute_units(), chunks));
    if (RL.full)
      hipLaunchKernelGGL((residue_kernel<MW, true>), grid, dim3(kResThreads), RL.total, s, tb, pool, mask, ws, rb, B,
                         status);
    else
      hipLaunchKernelGGL((residue_kernel<MW, false>), grid, dim3(kResThreads), RL.total, s, tb, pool, mask, ws, rb, B,
                         status);
  }
  if (phases & GRID_PHASE_FINALIZE) {
    // (beside the residue phase the statuses are written there)
    if (status && !(phases & GRID_PHASE_RESIDUE))
      hipLaunchKernelGGL(status_kernel, dim3((uint32_t)(B + 63) / 64), dim3(64), 0, s, ws, rb, B, status);
    if (tb.ci_cache && (tb.ci_flags & GRID_CI_INSERT))
      hipLaunchKernelGGL(ci_publish_kernel, dim3((uint32_t)(B + 63) / 64), dim3(64), 0, s, tb, ws, rb, B);
    if (tb.cache && (tb.cache_flags & GRID_CACHE_INSERT))
      hipLaunchKernelGGL(cache_publish_kernel, dim3(B), dim3(kBlock), 0, s, tb, mask, ws, rb);
  }
  return GRID_OK;
}

}  // namespace

int grid::overlay_capacity() { return kFastLane; }

// 0 when the class tables, built here if nothing has asked for them yet, do not
// fit into memory.
static size_t row_bytes(const grid_compiled* g) {
  try {
    return row_layout(g->parser.T, g->dfa.S, g->vocab.V, (int)g->max_classes()).total;
  } catch (const std::exception&) {
    return 0;
  }
}

// head, B rows, then the number of open ids of every row (0 as row_bytes)
static size_t workspace_size(const grid_compiled* g, int B) {
  const size_t rb = row_bytes(g);
  return rb ? kWsHead + rb * (size_t)B + (((size_t)B * 4 + 255) & ~(size_t)255) : 0;
}

extern "C" size_t grid_mask_workspace_bytes(const grid_compiled* g, int32_t B) {
  if (!g || B <= 0) return 0;
  return workspace_size(g, B);
}

// What a call's kernels read.
enum class Reads { kMask, kAdvance, kAdvanceHash, kStackHash };

// GRID_E_UNBOUND if something is not bound that the call's kernels read.
static int check_bound(const grid_compiled* g, Reads reads) {
  static const int lexer[] = {GRID_ART_DFA_CLASS, GRID_ART_BYTE_CLASS,  GRID_ART_DFA_ACCEPT_OFF, GRID_ART_DFA_ACCEPT_LIST,
                              GRID_ART_DFA_LIVE,  GRID_ART_TERM_INFO,   GRID_ART_SPELL_REC,      GRID_ART_SPELL_TAIL,
                              GRID_ART_LEX_FLAGS, GRID_ART_LEX_HASH,    GRID_ART_LEX_SLOTS,      GRID_ART_SPELL_OF_ID,
                              GRID_ART_GOTO_SKIP, GRID_ART_PARSE_SHIFT};
  static const int mask[] = {GRID_ART_ACTION,     GRID_ART_PROD,    GRID_ART_LEX_PREFIX, GRID_ART_LEX_STRIDE,
                             GRID_ART_LEX_TOKEN,  GRID_ART_LEX_CHILD, GRID_ART_ID_HEAD,  GRID_ART_LEX_TOKSUM};
  static const int advance[] = {GRID_ART_PARSE_STATE, GRID_ART_PARSE_REDX, GRID_ART_GOTO_HASH};
  auto missing = [&](int w) { return fail(GRID_E_UNBOUND, "artifact " + std::to_string(w) + " is not bound"); };
  if (reads != Reads::kStackHash)
    for (int w : lexer)
      if (!bound(g, w)) return missing(w);
  if (reads == Reads::kMask) {
    for (int w : mask)
      if (!bound(g, w)) return missing(w);
    if (!g->uses_progs() && !g->uses_classes())  // the classes are never empty
      for (int w : {GRID_ART_CLASS_MAP, GRID_ART_CLASS_OFF, GRID_ART_CLASS_REC})
        if (!g->dev[w]) return missing(w);
  } else if (reads != Reads::kStackHash) {
    for (int w : advance)
      if (!bound(g, w)) return missing(w);
  }
  if ((reads == Reads::kAdvanceHash || reads == Reads::kStackHash) && !bound(g, GRID_ART_STATE_SYMBOL))
    return missing(GRID_ART_STATE_SYMBOL);
  return GRID_OK;
}

// The device tables of a compiled handle for a call (GRID_E_UNBOUND as above).
static int bind_tables(const grid_compiled* g, Tables& tb, Reads reads) {
  const int rc = check_bound(g, reads);
  if (rc != GRID_OK) return rc;
  // the classes: of the reduced programs, or of the full ones where those are not bound
  const bool prog = g->uses_progs();
  tb.dfa = (const uint16_t*)g->dev[GRID_ART_DFA_CLASS];
  tb.bclass = (const uint8_t*)g->dev[GRID_ART_BYTE_CLASS];
  tb.acc_off = (const uint32_t*)g->dev[GRID_ART_DFA_ACCEPT_OFF];
  tb.acc_list = (const uint8_t*)g->dev[GRID_ART_DFA_ACCEPT_LIST];
  tb.live = (const uint32_t*)g->dev[GRID_ART_DFA_LIVE];
  tb.action = (const uint16_t*)g->dev[GRID_ART_ACTION];
  tb.term_info = (const uint32_t*)g->dev[GRID_ART_TERM_INFO];
  tb.pstate = (const uint32_t*)g->dev[GRID_ART_PARSE_STATE];
  tb.predx = (const uint32_t*)g->dev[GRID_ART_PARSE_REDX];
  tb.pshift = (const uint16_t*)g->dev[GRID_ART_PARSE_SHIFT];
  tb.go = (const uint16_t*)g->dev[GRID_ART_GOTO_SKIP];
  tb.ghash = (const uint2*)g->dev[GRID_ART_GOTO_HASH];
  tb.spell_rec = (const uint4*)g->dev[GRID_ART_SPELL_REC];
  tb.spell_tail = (const uint4*)g->dev[GRID_ART_SPELL_TAIL];
  tb.lex_flags = (const uint16_t*)g->dev[GRID_ART_LEX_FLAGS];
  tb.lex_hash = (const uint32_t*)g->dev[GRID_ART_LEX_HASH];
  tb.lex_slots = (const uint32_t*)g->dev[GRID_ART_LEX_SLOTS];
  tb.lex_prefix = (const uint4*)g->dev[GRID_ART_LEX_PREFIX];
  tb.lex_stride = (const uint4*)g->dev[GRID_ART_LEX_STRIDE];
  tb.lex_token = (const uint32_t*)g->dev[GRID_ART_LEX_TOKEN];
  tb.id_head = (const uint32_t*)g->dev[GRID_ART_ID_HEAD];
  tb.lex_toksum = (const uint8_t*)g->dev[GRID_ART_LEX_TOKSUM];
  tb.lex_child = (const uint32_t*)g->dev[GRID_ART_LEX_CHILD];
  tb.spell_of_id = (const uint32_t*)g->dev[GRID_ART_SPELL_OF_ID];
  tb.state_sym = (const uint32_t*)g->dev[GRID_ART_STATE_SYMBOL];
  tb.stack_hash = nullptr;
  tb.prog = prog ? 1 : 0;
  tb.cmap = (const uint16_t*)g->dev[prog ? GRID_ART_PROG_MAP : GRID_ART_CLASS_MAP];
  tb.coff = (const uint32_t*)g->dev[prog ? GRID_ART_PROG_OFF : GRID_ART_CLASS_OFF];
  tb.crec = (const uint4*)g->dev[prog ? GRID_ART_PROG_REC : GRID_ART_CLASS_REC];
  tb.max_classes = 0;  // (only the mask reads classes)
  tb.S = g->dfa.S;
  tb.C = g->dfa.C;
  tb.T = g->parser.T;
  tb.N = g->parser.N;
  tb.NS = g->parser.n_states;
  tb.V = g->vocab.V;
  tb.W = (g->vocab.V + 31) / 32;
  tb.n_slots = g->lex.n_slots;
  tb.eos_id = g->vocab.eos_id;
  tb.tw = g->parser.tw;
  tb.n_pstate = (int)g->parser.pstate.size();
  tb.n_predx = (int)g->parser.predx.size();
  tb.n_pshift = (int)g->parser.n_shift_runs;
  tb.mact = tb.pshift + g->parser.mact_off;
  tb.mred = (const uint32_t*)(tb.pshift + g->parser.mact_red_off);
  tb.mbits = g->parser.mact_bits;
  tb.prod = (const uint32_t*)g->dev[GRID_ART_PROD];
  tb.n_acc = (int)g->dfa.accept_list.size();
  tb.hbits = g->parser.goto_hbits;
  for (int w = 0; w < 8; ++w) tb.ign[w] = 0;
  for (int t = 0; t < tb.T && t < 256; ++t)
    if (g->term_info[t] & 1u) tb.ign[t >> 5] |= 1u << (t & 31);
  return GRID_OK;
}

static int mask_call(const grid_compiled* g, int32_t B, const grid_config* cfg_dev, const uint16_t* stack_pool_dev,
                     uint32_t* mask_dev, uint8_t* eos_dev, int32_t* status_dev, void* workspace_dev,
                     size_t workspace_bytes, void* cache_dev, size_t cache_bytes, uint32_t cache_flags,
                     uint32_t phases, void* stream, const uint64_t* stack_hash_dev = nullptr,
                     void* ci_dev = nullptr, size_t ci_bytes = 0, uint32_t ci_flags = 0) {
  clear_error();
  if (phases & ~GRID_PHASE_ALL) return fail(GRID_E_ARG, "grid_mask: unknown phase bits");
  if (cache_flags & ~(GRID_CACHE_LOOKUP | GRID_CACHE_INSERT)) return fail(GRID_E_ARG, "grid_mask: unknown cache flags");
  if (ci_flags & ~(GRID_CI_LOOKUP | GRID_CI_INSERT | GRID_CI_FAMILY | GRID_CI_GENN))
    return fail(GRID_E_ARG, "grid_mask_warm: unknown flags");
  if ((ci_flags & GRID_CI_GENN) && !(ci_flags & GRID_CI_FAMILY))
    return fail(GRID_E_ARG, "grid_mask_warm: the genN normal form belongs to the cross-family tier");
  if (!g || B <= 0 || B > 65535 || !cfg_dev || !stack_pool_dev || !mask_dev || !workspace_dev)
    return fail(GRID_E_ARG, "grid_mask: null pointer or batch size out of range");
  const size_t rb = row_bytes(g);
  if (rb == 0) return fail(GRID_E_CAPACITY, "grid_mask: out of memory for the class tables");
  if (workspace_bytes < workspace_size(g, B)) return fail(GRID_E_ARG, "grid_mask: workspace too small");
  if (((uintptr_t)workspace_dev & 255) != 0) return fail(GRID_E_ARG, "grid_mask: workspace not 256-byte aligned");
  Tables tb;
  const int brc = bind_tables(g, tb, Reads::kMask);
  if (brc != GRID_OK) return brc;
  tb.max_classes = (int)g->max_classes();  // (built above)
  tb.cache = nullptr;
  tb.cache_mask = 0;
  tb.cache_flags = 0;
  tb.cache_stride = cache_stride_of(tb.W);
  tb.fp = g->fingerprint;
  if (cache_dev && cache_flags) {
    const size_t n = cache_bytes / tb.cache_stride;
    if (n == 0 || (n & (n - 1)) != 0 || n > 0x80000000ull || n * tb.cache_stride != cache_bytes)
      return fail(GRID_E_ARG, "grid_mask: cache size is not grid_cache_bytes of a power of two");
    if (((uintptr_t)cache_dev & 15) != 0) return fail(GRID_E_ARG, "grid_mask: cache not 16-byte aligned");
    tb.cache = (uint8_t*)cache_dev;
    tb.cache_mask = (uint32_t)(n - 1);
    tb.cache_flags = cache_flags;
    tb.stack_hash = stack_hash_dev;
  }
  tb.ci_cache = nullptr;
  tb.ci_mask = 0;
  tb.ci_flags = 0;
  tb.ci_stride = ci_stride_of(tb.W);
  tb.family_fp = g->family_fp;
  if (ci_dev && (ci_flags & (GRID_CI_LOOKUP | GRID_CI_INSERT))) {
    const size_t n = ci_bytes / tb.ci_stride;
    if (n == 0 || (n & (n - 1)) != 0 || n > 0x80000000ull || n * tb.ci_stride != ci_bytes)
      return fail(GRID_E_ARG, "grid_mask_warm: cache size is not grid_ci_cache_bytes of a power of two");
    if (((uintptr_t)ci_dev & 15) != 0) return fail(GRID_E_ARG, "grid_mask_warm: cache not 16-byte aligned");
    tb.ci_cache = (uint8_t*)ci_dev;
    tb.ci_mask = (uint32_t)(n - 1);
    tb.ci_flags = ci_flags;
  }
  const int mw = tb.tw;
  if (tb.T > 255 || (mw != 2 && mw != 4 && mw != 8) || table_bytes(tb) > kTablesMax ||
      res_lds(tb).total > kLdsMax - kLdsStatic || stream_lds(tb).total > kLdsMax - kLdsStatic || prologue_parse_lds(tb).total > kPrologueParseMax ||
      verdict_bytes(tb) > 64 * 1024)
    return fail(GRID_E_CAPACITY, "grid_mask: lexer DFA or LR tables too large for the LDS staging");
  hipStream_t s = (hipStream_t)stream;
  uint8_t* ws = (uint8_t*)workspace_dev;
  int rc;
  if (mw == 2)
    rc = launch_mask<2>(tb, B, cfg_dev, stack_pool_dev, mask_dev, eos_dev, status_dev, ws, rb, phases, s);
  else if (mw == 4)
    rc = launch_mask<4>(tb, B, cfg_dev, stack_pool_dev, mask_dev, eos_dev, status_dev, ws, rb, phases, s);
  else
    rc = launch_mask<8>(tb, B, cfg_dev, stack_pool_dev, mask_dev, eos_dev, status_dev, ws, rb, phases, s);
  if (rc != GRID_OK) return rc;
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(GRID_E_HIP, std::string("grid_mask launch: ") + hipGetErrorString(e));
  return GRID_OK;
}

extern "C" int grid_mask_phases(const grid_compiled* g, int32_t B, const grid_config* cfg_dev,
                                const uint16_t* stack_pool_dev, uint32_t* mask_dev, uint8_t* eos_dev,
                                int32_t* status_dev, void* workspace_dev, size_t workspace_bytes,
                                uint32_t phases, void* stream) {
  return mask_call(g, B, cfg_dev, stack_pool_dev, mask_dev, eos_dev, status_dev, workspace_dev, workspace_bytes,
                   nullptr, 0, 0, phases, stream);
}

extern "C" int grid_mask(const grid_compiled* g, int32_t B, const grid_config* cfg_dev,
                         const uint16_t* stack_pool_dev, uint32_t* mask_dev, uint8_t* eos_dev,
                         int32_t* status_dev, void* workspace_dev, size_t workspace_bytes, void* stream) {
  return mask_call(g, B, cfg_dev, stack_pool_dev, mask_dev, eos_dev, status_dev, workspace_dev, workspace_bytes,
                   nullptr, 0, 0, GRID_PHASE_ALL, stream);
}

extern "C" int grid_mask_cached(const grid_compiled* g, int32_t B, const grid_config* cfg_dev,
                                const uint16_t* stack_pool_dev, const uint64_t* stack_hash_dev, uint32_t* mask_dev,
                                uint8_t* eos_dev, int32_t* status_dev, void* workspace_dev, size_t workspace_bytes,
                                void* cache_dev, size_t cache_bytes, uint32_t cache_flags, void* stream) {
  return mask_call(g, B, cfg_dev, stack_pool_dev, mask_dev, eos_dev, status_dev, workspace_dev, workspace_bytes,
                   cache_dev, cache_bytes, cache_flags, GRID_PHASE_ALL, stream, stack_hash_dev);
}

extern "C" int grid_stack_hash(const grid_compiled* g, int32_t B, const grid_config* cfg_dev,
                               const uint16_t* stack_pool_dev, uint64_t* stack_hash_dev, void* stream) {
  clear_error();
  if (!g || B <= 0 || !cfg_dev || !stack_pool_dev || !stack_hash_dev)
    return fail(GRID_E_ARG, "grid_stack_hash: null pointer or bad batch size");
  Tables tb;
  const int rc = bind_tables(g, tb, Reads::kStackHash);
  if (rc != GRID_OK) return rc;
  hipLaunchKernelGGL(stack_hash_kernel, dim3((unsigned)((B + 15) / 16)), dim3(64), 0, (hipStream_t)stream, tb, cfg_dev,
                     stack_pool_dev, stack_hash_dev, B);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(GRID_E_HIP, std::string("grid_stack_hash launch: ") + hipGetErrorString(e));
  return GRID_OK;
}

// ------------------------------------------------------ no-alloc mask entry
// The workspace of grid_mask_noalloc: a device array of the code object, one
// copy per GPU, held until the process ends.  Host code never passes the
// array's name to a kernel (on the host it is only a stand-in for the
// symbol); it uses the device address hipGetSymbolAddress returns, looked up
// once per device with that device current.
constexpr size_t kScratchBytes = size_t(32) << 20;
static __device__ __align__(256) uint8_t scratch[kScratchBytes];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};

// Device address of the current device's scratch array, or nullptr (the
// error is recorded).
void* scratch_on_current_device() {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) {
    fail(GRID_E_HIP, "grid_mask_noalloc: no current device");
    return nullptr;
  }
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !ptr) {
      fail(GRID_E_HIP, std::string("grid_mask_noalloc: hipGetSymbolAddress: ") + hipGetErrorString(e));
      return nullptr;
    }
    g_scratch_ptr[dev] = ptr;
  }
  return g_scratch_ptr[dev];
}
}  // namespace

extern "C" size_t grid_mask_noalloc_max_bytes(void) { return kScratchBytes; }

extern "C" int grid_mask_noalloc(const grid_compiled* g, int32_t B, const grid_config* cfg_dev,
                                 const uint16_t* stack_pool_dev, uint32_t* mask_dev, uint8_t* eos_dev,
                                 int32_t* status_dev, void* stream) {
  clear_error();
  if (!g || B <= 0 || B > 65535) return fail(GRID_E_ARG, "grid_mask_noalloc: null handle or batch size out of range");
  const size_t need = workspace_size(g, B);
  if (need > kScratchBytes)
    return fail(GRID_E_CAPACITY, "grid_mask_noalloc: " + std::to_string(B) + " rows need " + std::to_string(need) +
                                     " workspace bytes, more than the " + std::to_string(kScratchBytes) +
                                     " of the static scratch array");
  void* ws = scratch_on_current_device();
  if (!ws) return GRID_E_HIP;
  return mask_call(g, B, cfg_dev, stack_pool_dev, mask_dev, eos_dev, status_dev, ws, kScratchBytes, nullptr, 0, 0,
                   GRID_PHASE_ALL, stream);
}

extern "C" size_t grid_cache_bytes(const grid_compiled* g, int32_t n_entries) {
  if (!g || n_entries < 1 || (n_entries & (n_entries - 1)) != 0) return 0;
  return (size_t)n_entries * cache_stride_of((g->vocab.V + 31) / 32);
}

extern "C" int grid_cache_clear(const grid_compiled* g, void* cache_dev, size_t cache_bytes, void* stream) {
  clear_error();
  if (!g || !cache_dev) return fail(GRID_E_ARG, "grid_cache_clear: null argument");
  const uint32_t stride = cache_stride_of((g->vocab.V + 31) / 32);
  const size_t n = cache_bytes / stride;
  if (n == 0 || (n & (n - 1)) != 0 || n > 0x80000000ull || n * stride != cache_bytes)
    return fail(GRID_E_ARG, "grid_cache_clear: cache size is not grid_cache_bytes of a power of two");
  const int blocks = (int)std::min<size_t>((n + kBlock - 1) / kBlock, 1024);
  hipLaunchKernelGGL(cache_clear_kernel, dim3(blocks), dim3(kBlock), 0, (hipStream_t)stream, (uint8_t*)cache_dev,
                     (uint32_t)n, stride);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(GRID_E_HIP, std::string("grid_cache_clear launch: ") + hipGetErrorString(e));
  return GRID_OK;
}

static int accept_call(const grid_compiled* g, int32_t B, const grid_config* cfg_dev, const uint16_t* stack_pool_dev,
                       const int32_t* token_dev, grid_config* cfg_out_dev, uint16_t* stack_out_dev, uint64_t* hash_dev,
                       uint32_t stack_cap, int32_t* status_dev, int inplace, void* stream, int tok_stride = 1,
                       bool few_tokens = false) {
  Tables tb;
  const int rc = bind_tables(g, tb, hash_dev ? Reads::kAdvanceHash : Reads::kAdvance);
  if (rc != GRID_OK) return rc;
  if (tb.T > 255) return fail(GRID_E_CAPACITY, "grid_accept: more than 255 terminals");
  const ParseLds PL = prologue_parse_lds(tb);
  const int use_lds = PL.total <= kPrologueParseMax ? 1 : 0;
  uint32_t lds = use_lds ? PL.total + pad16(accept_stack_cap(stack_cap) * 2u) : 0u;
  const int use_lex = use_lds && lds + accept_lex_lds(tb).total <= kAcceptLdsMax ? 1 : 0;
  if (use_lex) lds += accept_lex_lds(tb).total;
  const void* fn = tb.tw == 2 ? (const void*)accept_kernel<2>
                              : (tb.tw == 4 ? (const void*)accept_kernel<4> : (const void*)accept_kernel<8>);
  if (!raise_lds(fn, lds)) return fail(GRID_E_HIP, "grid_accept: cannot raise the LDS limit");
  // The tables are staged before the row's token is known, which saves a row that
  // has one a read's latency (256 rows: 14.5 us against 15.2), unless rows without a
  // token would stage for nothing in others' time: in a forced span, where most
  // rows have none (16 rows, 4 steps: 324 us against 336), and when the rows
  // queue for the compute units (1,024 without: 9.9 us against 20.1, in place
  // 8.1 against 19.6; with: 32.3 against 32.0).
  const int late = few_tokens || B > compute_units() ? 1 : 0;
  hipStream_t s = (hipStream_t)stream;
  const dim3 grid((unsigned)B), block(kAccThreads);
  if (tb.tw == 2)
    hipLaunchKernelGGL(accept_kernel<2>, grid, block, lds, s, tb, cfg_dev, stack_pool_dev, token_dev, cfg_out_dev,
                       stack_out_dev, hash_dev, stack_cap, status_dev, use_lds, use_lex, inplace, tok_stride, late);
  else if (tb.tw == 4)
    hipLaunchKernelGGL(accept_kernel<4>, grid, block, lds, s, tb, cfg_dev, stack_pool_dev, token_dev, cfg_out_dev,
                       stack_out_dev, hash_dev, stack_cap, status_dev, use_lds, use_lex, inplace, tok_stride, late);
  else
    hipLaunchKernelGGL(accept_kernel<8>, grid, block, lds, s, tb, cfg_dev, stack_pool_dev, token_dev, cfg_out_dev,
                       stack_out_dev, hash_dev, stack_cap, status_dev, use_lds, use_lex, inplace, tok_stride, late);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(GRID_E_HIP, std::string("grid_accept launch: ") + hipGetErrorString(e));
  return GRID_OK;
}

extern "C" size_t grid_ci_cache_bytes(const grid_compiled* g, int32_t n_entries) {
  if (!g || n_entries < 1 || (n_entries & (n_entries - 1)) != 0) return 0;
  return (size_t)n_entries * ci_stride_of((g->vocab.V + 31) / 32);
}

extern "C" int grid_ci_cache_clear(const grid_compiled* g, void* cache_dev, size_t cache_bytes, void* stream) {
  clear_error();
  if (!g || !cache_dev) return fail(GRID_E_ARG, "grid_ci_cache_clear: null argument");
  const uint32_t stride = ci_stride_of((g->vocab.V + 31) / 32);
  const size_t n = cache_bytes / stride;
  if (n == 0 || (n & (n - 1)) != 0 || n > 0x80000000ull || n * stride != cache_bytes)
    return fail(GRID_E_ARG, "grid_ci_cache_clear: cache size is not grid_ci_cache_bytes of a power of two");
  const int blocks = (int)std::min<size_t>((n + kBlock - 1) / kBlock, 1024);
  hipLaunchKernelGGL(cache_clear_kernel, dim3(blocks), dim3(kBlock), 0, (hipStream_t)stream, (uint8_t*)cache_dev,
                     (uint32_t)n, stride);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(GRID_E_HIP, std::string("grid_ci_cache_clear launch: ") + hipGetErrorString(e));
  return GRID_OK;
}

extern "C" int grid_mask_warm(const grid_compiled* g, int32_t B, const grid_config* cfg_dev,
                              const uint16_t* stack_pool_dev, uint32_t* mask_dev, uint8_t* eos_dev, int32_t* status_dev,
                              void* workspace_dev, size_t workspace_bytes, void* ci_cache_dev, size_t ci_cache_bytes,
                              uint32_t ci_flags, void* stream) {
  return mask_call(g, B, cfg_dev, stack_pool_dev, mask_dev, eos_dev, status_dev, workspace_dev, workspace_bytes,
                   nullptr, 0, 0, GRID_PHASE_ALL, stream, nullptr, ci_cache_dev, ci_cache_bytes, ci_flags);
}

extern "C" int grid_accept(const grid_compiled* g, int32_t B, const grid_config* cfg_dev,
                           const uint16_t* stack_pool_dev, const int32_t* token_dev, grid_config* cfg_out_dev,
                           uint16_t* stack_out_dev, uint32_t stack_cap, int32_t* status_dev, void* stream) {
  clear_error();
  if (!g || B <= 0 || !cfg_dev || !stack_pool_dev || !token_dev || !cfg_out_dev || !stack_out_dev || stack_cap < 2)
    return fail(GRID_E_ARG, "grid_accept: null pointer or bad size");
  return accept_call(g, B, cfg_dev, stack_pool_dev, token_dev, cfg_out_dev, stack_out_dev, nullptr, stack_cap,
                     status_dev, 0, stream);
}

extern "C" int grid_accept_inplace(const grid_compiled* g, int32_t B, grid_config* cfg_dev, uint16_t* stack_pool_dev,
                                   uint64_t* stack_hash_dev, uint32_t stack_cap, const int32_t* token_dev,
                                   int32_t* status_dev, void* stream) {
  clear_error();
  if (!g || B <= 0 || !cfg_dev || !stack_pool_dev || !token_dev || stack_cap < 2)
    return fail(GRID_E_ARG, "grid_accept_inplace: null pointer or bad size");
  return accept_call(g, B, cfg_dev, stack_pool_dev, token_dev, cfg_dev, stack_pool_dev, stack_hash_dev, stack_cap,
                     status_dev, 1, stream);
}

// Jump-forward step i (section 6.1 step 6): a row whose mask allows exactly
// one token (the end-of-sequence token counts when its bit is set) takes it
// as span[row][i]; any other row, a row whose mask call did not end OK, and a
// row whose span already stopped (a non-forced step, or the end-of-sequence
// token) gets -1.  Before that, a row whose advance by span[row][i - 1]
// failed (acc_status neither OK nor FINISHED; its configuration is then
// unchanged) has that token taken back and stops.  span_len[row] counts the
// forced tokens.  With take == 0 only the check of the last advance runs.
__global__ __launch_bounds__(kBlock) void singleton_kernel(const uint32_t* __restrict__ mask,
                                                           const int32_t* __restrict__ status,
                                                           const int32_t* __restrict__ acc_status, int32_t* span,
                                                           int32_t* span_len, int W, int max_len, int i, int eos_id,
                                                           int take) {
  const int row = (int)blockIdx.x, tid = (int)threadIdx.x;
  __shared__ int count, word;
  if (tid == 0) {
    count = 0;
    word = -1;
  }
  __syncthreads();
  const uint32_t* m = mask + (size_t)row * W;
  int c = 0, wd = -1;
  if (take) {
    for (int w = tid; w < W; w += kBlock) {
      const int k = __popc(m[w]);
      c += k;
      if (k) wd = w;
    }
  }
  if (c) atomicAdd(&count, c);
  if (wd >= 0) atomicMax(&word, wd);
  __syncthreads();
  if (tid != 0) return;
  int32_t* sp = span + (size_t)row * max_len;
  if (i == 0) span_len[row] = 0;
  bool open = i == 0 || (sp[i - 1] >= 0 && sp[i - 1] != eos_id);
  if (i > 0 && sp[i - 1] >= 0 && acc_status[row] != GRID_ROW_OK && acc_status[row] != GRID_ROW_FINISHED) {
    sp[i - 1] = -1;  // not applied: the row keeps the configuration before it
    span_len[row] = i - 1;
    open = false;
  }
  if (!take) return;
  int tok = -1;
  if (open && count == 1 && (!status || status[row] == GRID_ROW_OK)) tok = word * 32 + __ffs((int)m[word]) - 1;
  sp[i] = tok;
  if (tok >= 0) span_len[row] = i + 1;
}

extern "C" int grid_forced_span(const grid_compiled* g, int32_t B, grid_config* cfg_dev, uint16_t* stack_pool_dev,
                                uint64_t* stack_hash_dev, uint32_t stack_cap, int32_t max_len, int32_t* span_dev,
                                int32_t* span_len_dev, uint32_t* mask_dev, uint8_t* eos_dev, int32_t* status_dev,
                                void* workspace_dev, size_t workspace_bytes, void* stream) {
  clear_error();
  if (!g || B <= 0 || !cfg_dev || !stack_pool_dev || !span_dev || !span_len_dev || !mask_dev || !status_dev ||
      !workspace_dev || max_len < 1 || stack_cap < 2)
    return fail(GRID_E_ARG, "grid_forced_span: null pointer or bad size");
  const size_t mask_ws = workspace_size(g, B);
  if (workspace_bytes < mask_ws + (size_t)B * 4u)
    return fail(GRID_E_ARG, "grid_forced_span: workspace smaller than grid_forced_span_workspace_bytes");
  // the advances' statuses live after the mask workspace
  int32_t* acc_status = (int32_t*)((uint8_t*)workspace_dev + mask_ws);
  const int W = (g->vocab.V + 31) / 32;
  hipStream_t s = (hipStream_t)stream;
  for (int i = 0; i <= max_len; ++i) {
    int rc = mask_call(g, B, cfg_dev, stack_pool_dev, mask_dev, eos_dev, status_dev, workspace_dev, mask_ws, nullptr,
                       0, 0, GRID_PHASE_ALL, stream);
    if (rc != GRID_OK) return rc;
    const int take = i < max_len ? 1 : 0;  // the last round only checks the last advance
    hipLaunchKernelGGL(singleton_kernel, dim3((unsigned)B), dim3(kBlock), 0, s, mask_dev, status_dev, acc_status,
                       span_dev, span_len_dev, W, max_len, i, g->vocab.eos_id, take);
    if (!take) break;
    // rows with -1 are left as they are (their status is not needed)
    rc = accept_call(g, B, cfg_dev, stack_pool_dev, span_dev + i, cfg_dev, stack_pool_dev, stack_hash_dev, stack_cap,
                     acc_status, 1, stream, max_len, true);
    if (rc != GRID_OK) return rc;
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(GRID_E_HIP, std::string("grid_forced_span launch: ") + hipGetErrorString(e));
  return GRID_OK;
}

extern "C" size_t grid_forced_span_workspace_bytes(const grid_compiled* g, int32_t B) {
  if (!g || B <= 0) return 0;
  return workspace_size(g, B) + (size_t)B * 4u;
}

extern "C" int grid_apply(const uint32_t* mask_dev, void* logits_dev, int32_t dtype, int32_t B, int32_t V,
                          int64_t row_stride, void* stream) {
  clear_error();
  if (!mask_dev || !logits_dev || B <= 0 || V <= 0 || row_stride < V)
    return fail(GRID_E_ARG, "grid_apply: null pointer or bad shape");
  if (dtype != GRID_DTYPE_F32 && dtype != GRID_DTYPE_BF16) return fail(GRID_E_ARG, "grid_apply: dtype");
  const int W = (V + 31) / 32;
  if (B > 65535) return fail(GRID_E_ARG, "grid_apply: more than 65535 rows");
  const int groups = (V + 7) / 8;
  // one grid row per batch row; along it enough workgroups for every group
  // of 8 logits, at most 512 (a grid-stride loop covers the rest)
  const dim3 blocks((unsigned)std::min((groups + kBlock - 1) / kBlock, 512), (unsigned)B);
  hipStream_t s = (hipStream_t)stream;
  const int64_t esz = dtype == GRID_DTYPE_BF16 ? 2 : 4;
  const bool aligned = (uintptr_t)logits_dev % 16 == 0 && row_stride * esz % 16 == 0;
  if (dtype == GRID_DTYPE_BF16)
    hipLaunchKernelGGL(apply_kernel<uint16_t>, blocks, dim3(kBlock), 0, s, mask_dev,
                       (uint16_t*)logits_dev, B, V, W, row_stride, 0xFF80u, aligned);
  else
    hipLaunchKernelGGL(apply_kernel<uint32_t>, blocks, dim3(kBlock), 0, s, mask_dev,
                       (uint32_t*)logits_dev, B, V, W, row_stride, 0xFF800000u, aligned);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(GRID_E_HIP, std::string("grid_apply launch: ") + hipGetErrorString(e));
  return GRID_OK;
}
