// The fill of a group of eight logits on the host: every bit pattern at every
// alignment against one logit at a time, and, in an unaligned group, no write to
// a logit it keeps (those lie in a page that may only be read).
#include <sys/mman.h>

#include <cstdio>
#include <cstring>

#include "../../paper_2607_11951_amd/csrc/fill.h"

template <typename T>
static int check(uint32_t neg_inf) {
  alignas(16) T buf[32];
  for (int at = 0; at < 8; ++at)
    for (int n = 1; n <= 9; ++n)
      for (uint32_t bits = 0; bits < 256; ++bits) {
        T want[32];
        for (int i = 0; i < 32; ++i) buf[i] = want[i] = (T)(0x9E3779B1u * (uint32_t)(i + 1));
        const bool aligned = at * sizeof(T) % 16 == 0;
        for (int j = 0; j < 8 && j < n; ++j)
          if (!((bits >> j) & 1u)) want[at + j] = (T)neg_inf;
        grid::fill_group<T>(buf + at, bits, n, aligned, neg_inf);
        if (memcmp(buf, want, sizeof(buf))) return printf("size %zu at %d n %d bits %x\n", sizeof(T), at, n, bits), 1;
      }
  const size_t page = 65536;
  for (int k = 1; k < 8; ++k) {  // the last 8 - k logits of the group in the second page, kept
    if (k * sizeof(T) % 16 == 0) continue;
    uint8_t* m = (uint8_t*)mmap(nullptr, 2 * page, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS, -1, 0);
    if (m == MAP_FAILED || mprotect(m + page, page, PROT_READ)) return printf("mmap\n"), 1;
    T* p = (T*)(m + page) - k;
    for (uint32_t low = 0; low < (1u << k); ++low) {
      for (int j = 0; j < k; ++j) p[j] = (T)(j + 1);
      grid::fill_group<T>(p, low | (0xFFu << k & 0xFFu), 8, false, neg_inf);
      for (int j = 0; j < k; ++j)
        if (p[j] != ((low >> j) & 1u ? (T)(j + 1) : (T)neg_inf)) return printf("size %zu k %d low %x\n", sizeof(T), k, low), 1;
    }
    munmap(m, 2 * page);
  }
  return 0;
}

int main() { return check<uint16_t>(0xFF80u) | check<uint32_t>(0xFF800000u); }
