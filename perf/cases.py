"""The calls a user of the library makes, at the sizes they are made at.

One pass (`run`) is one step of a program that decodes under a grammar: the
exact mask of a batch of configurations, the -inf fill of the logits, the
device advance by the sampled tokens, the two caches, forced spans.  Grammars,
vocabularies, schemas and sentences come from the `workloads` package; the
compiled handle of a (grammar, vocabulary, schemas) triple is kept for the
life of the process, as a server keeps it, and everything else -- the rows'
prefixes, their continuations, the logits -- is made anew from the seed.

Every result is a set of bits fixed by the language (mask words, bytes,
states, token ids, 64-bit hashes) or an untouched / -inf logit, so the outputs
of two correct implementations are equal.
"""

import functools
import math
import random

import numpy as np
import torch

import paper_2607_11951_amd as G
from workloads import configs as W
from workloads import grammar_text
from workloads import schema as sch
from workloads import sentences as sen
from workloads import vocab as voc

DEV = "cuda:0"
CAP = 1024            # stack entries per row of an advance's arena
V_FULL = 151936       # the large vocabulary of the DML workloads
SCHEMAS = 64          # tenants of the multi-schema server

DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}


def _case(name, kind, grammar, V, B, dtype="bf16", schemas=1, depth=0, prefix=0, steps=1):
    c = {"kind": kind, "grammar": grammar, "V": V, "B": B, "dtype": dtype, "schemas": schemas, "depth": depth,
         "prefix": prefix, "steps": steps}
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # one user, a calculator-sized grammar: the call is launches and latency only
        _case("expr_b1_mask", "mask", "expr", 1024, 1),
        # a read-only query box on a 32k vocabulary; its logits are float32
        _case("select_b32_step_f32", "step", "sql_select", 32000, 32, dtype="f32"),
        # one user on the full vocabulary: time to the next token
        _case("dml_b1_step", "step", "sql_dml", V_FULL, 1),
        # the ordinary serving step: a batch of 32 on the full vocabulary
        _case("dml_b32_step", "step", "sql_dml", V_FULL, 32),
        # a large batch whose rows belong to many tenants, each with its own schema lexicon
        _case("schemas_b256_step", "step", "sql_dml", V_FULL, 256, schemas=SCHEMAS),
        # a vocabulary that is a multiple of nothing and an odd batch: unaligned logits rows
        _case("dml_odd_b47_step", "step", "sql_dml", 50257, 47),
        # long outputs: deep stacks (nested queries) after tens of kilobytes of text
        _case("long_b32_mask", "mask", "sql_dml", 128256, 32, depth=32, prefix=40000),
        # the decode loop: mask, fill and in-place advance with rolling hashes, eight tokens
        _case("dml_b32_decode8", "decode", "sql_dml", V_FULL, 32, steps=8),
        # the advance alone, out of place, for a large batch (speculative verification)
        _case("dml_b256_accept", "accept", "sql_dml", V_FULL, 256),
        # the mask cache: a batch that misses and is inserted, then the same batch served
        _case("dml_b64_cached", "cached", "sql_dml", V_FULL, 64),
        # the warm path: context-independent words inserted, then reused with live verdicts
        _case("dml_b32_warm", "warm", "sql_dml", 128256, 32),
        # jump-forward: up to four forced tokens a row
        _case("select_b16_span4", "span", "sql_select", 32000, 16, steps=4),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: kind by how often a program makes the call, sizes over the logarithm of their ranges."""
    kind = rng.choice(["step", "step", "step", "mask", "mask", "decode", "accept", "cached", "warm", "span"])
    grammar = rng.choice(["expr", "sql_select", "sql_dml", "sql_dml"]) if kind in ("mask", "step") else \
        rng.choice(["sql_select", "sql_dml", "sql_dml"])
    if grammar == "expr":
        V = 1024
    elif grammar == "sql_select":
        V = _log_int(rng, 4000, 48000)
    else:
        V = _log_int(rng, 8000, V_FULL)
    if rng.random() < 0.5 and grammar != "expr":
        V = max(4000, V // 64 * 64)
    most = {"mask": 256, "step": 256, "accept": 256, "cached": 64, "warm": 64, "decode": 48, "span": 24}[kind]
    B = _log_int(rng, 1, most)
    steps = {"decode": rng.randint(2, 8), "span": rng.randint(1, 4)}.get(kind, 1)
    schemas = rng.choice([1, 1, SCHEMAS]) if grammar == "sql_dml" else 1
    depth, prefix = (rng.randint(1, 128), _log_int(rng, 400, 40000)) if grammar == "sql_dml" and kind == "mask" and \
        rng.random() < 0.5 else (0, 0)
    return _case(None, kind, grammar, V, B, rng.choice(["bf16", "f32"]), schemas, depth, prefix, steps)


# ------------------------------------------------------------- what a server keeps
@functools.lru_cache(maxsize=None)
def _schemas(grammar, n):
    banned = sch.keyword_spellings(W.GRAMMAR_DIR / f"{grammar}.grid")
    if grammar == "sql_select":
        return [sch.make_schema(np.random.default_rng(2002), 8, 12, 12, banned)]
    if n == 1:
        return [sch.make_schema(np.random.default_rng(3002), 200, 30, 30, banned)]
    out = []
    for i in range(n):
        rng = np.random.default_rng(5000 + 7 * i)
        out.append(sch.make_schema(rng, int(rng.integers(50, 501)), 5, 60, banned))
    return out


@functools.lru_cache(maxsize=None)
def _vocab(grammar, V):
    if grammar == "expr":
        return voc.config1_vocab(1000), [], -1
    kws = sorted(sch.keyword_spellings(W.GRAMMAR_DIR / f"{grammar}.grid"))
    s = _schemas(grammar, 1)[0]
    if grammar == "sql_select":
        return voc.config2_vocab(2000, kws, list(s.tables) + s.all_columns(), V)
    return voc.geometric_vocab(3000, kws, list(s.tables) + s.all_columns()[:2000], V)


@functools.lru_cache(maxsize=None)
def _handle(grammar, V, schemas):
    """(compiled grammar on the device, its lexicon slots)."""
    vocab, specials, eos = _vocab(grammar, V)
    drop = W.READ_ONLY_ROLE if grammar == "sql_dml" else ()
    grid = G.Grid(grammar_text(grammar), drop, vocab, specials, eos)
    slots = [0]
    if grammar != "expr":
        slots = [grid.add_lexicon(s.lexicon(with_alias=grammar == "sql_dml")) for s in _schemas(grammar, schemas)]
    return grid.to_device(DEV), slots


@functools.lru_cache(maxsize=None)
def _token_ids(grammar, V):
    return {sp: i for i, sp in reversed(list(enumerate(_vocab(grammar, V)[0]))) if sp}


# ----------------------------------------------------------------------- inputs
def _sentence(case, r, schema):
    if case["grammar"] == "expr":
        return sen.gen_expr(r).encode()
    if case["grammar"] == "sql_select":
        return sen.SelectSubsetGen(r, schema).sentence().encode()
    g = sen.DmlQueryGen(r, schema)
    return (g.long_sentence(case["depth"], case["prefix"] + 64) if case["depth"] else g.sentence()).encode()


def _greedy(ids, text, n):
    """The first n tokens of text by greedy longest match; None if it holds fewer."""
    out, i = [], 0
    while len(out) < n:
        for k in range(min(32, len(text) - i), 0, -1):
            t = ids.get(text[i:i + k])
            if t is not None:
                break
        else:
            return None
        out.append(t)
        i += k
    return out


def _rows(case, r, tokens):
    """(prefix, slot index, next tokens) of every row: sentences of the row's
    schema cut at a uniform byte (at the case's prefix length when it has one)."""
    schemas = _schemas(case["grammar"], case["schemas"]) if case["grammar"] != "expr" else [None]
    ids = _token_ids(case["grammar"], case["V"]) if tokens else None
    out = []
    while len(out) < case["B"]:
        s = r.randrange(len(schemas))
        text = _sentence(case, r, schemas[s])
        cut = case["prefix"] - r.randint(0, min(64, case["prefix"])) if case["depth"] else r.randint(0, len(text))
        nxt = _greedy(ids, text[cut:], tokens) if tokens else []
        if nxt is not None:
            out.append((text[:cut], s, nxt))
    return out


def prepare(case, seed):
    grid, slots = _handle(case["grammar"], case["V"], case["schemas"])
    kind, B = case["kind"], case["B"]
    r = random.Random(f"{seed} {kind} {B}")
    n_tok = {"decode": case["steps"], "accept": 1}.get(kind, 0)
    rows = _rows(case, r, n_tok)
    cfgs, pool = grid.configs([w for w, _, _ in rows], [slots[s] for _, s, _ in rows])
    arena = kind in ("decode", "span")
    if arena:  # every row's stack in its own region
        region = np.zeros(B * CAP, dtype=np.uint16)
        for b in range(B):
            off, d = int(cfgs["stk_off"][b]), int(cfgs["stk_depth"][b])
            region[b * CAP:b * CAP + d] = pool[off:off + d]
            cfgs["stk_off"][b] = b * CAP
        pool = region
    cfg, pool = grid.configs_to_device(cfgs, pool, DEV)
    st = {"case": case, "grid": grid, "cfg": cfg, "pool": pool}
    if n_tok:
        st["tokens"] = torch.tensor([t for _, _, t in rows], dtype=torch.int32).t().contiguous().to(DEV)
    if arena:
        st["cfg0"], st["pool0"] = cfg.clone(), pool.clone()
        st["hash"] = torch.zeros(B * CAP, dtype=torch.int64, device=DEV)
    if kind == "accept":
        st["cfg_out"] = torch.zeros(B * 32, dtype=torch.uint8, device=DEV)
        st["pool_out"] = torch.zeros(B * CAP, dtype=torch.int16, device=DEV)
        st["acc"] = torch.zeros(B, dtype=torch.int32, device=DEV)
        return st
    if kind == "span":
        n = G.lib().grid_forced_span_workspace_bytes(grid.h, B)
        st["ws"] = torch.empty(n, dtype=torch.uint8, device=DEV)
        return st
    steps = case["steps"] if kind == "decode" else 2 if kind in ("cached", "warm") else 1
    st["mask"] = torch.zeros((steps, B, grid.W), dtype=torch.int32, device=DEV)
    st["eos"] = torch.zeros((steps, B), dtype=torch.uint8, device=DEV)
    st["status"] = torch.zeros((steps, B), dtype=torch.int32, device=DEV)
    st["ws"] = grid.new_workspace(B, DEV)
    if kind in ("step", "decode"):
        gen = torch.Generator(device=DEV).manual_seed(seed)
        st["logits"] = (2.0 * torch.randn((steps, B, grid.V), generator=gen, device=DEV)).to(DTYPES[case["dtype"]])
    if kind == "decode":
        st["acc"] = torch.zeros((steps, B), dtype=torch.int32, device=DEV)
    if kind == "cached":
        st["cache"] = grid.new_cache(1024, DEV)
        st["hash"] = grid.stack_hash(cfg, pool, B)
    if kind == "warm":
        st["cache"] = grid.new_ci_cache(1024, DEV)
    return st


def run(st):
    case, grid, cfg, pool = st["case"], st["grid"], st["cfg"], st["pool"]
    kind, B = case["kind"], case["B"]
    if kind == "accept":
        return list(grid.accept(cfg, pool, st["tokens"][0], B, CAP, st["cfg_out"], st["pool_out"], st["acc"]))
    if kind == "span":  # advances the rows in place: from their starting configurations
        cfg.copy_(st["cfg0"])
        pool.copy_(st["pool0"])
        grid.stack_hash(cfg, pool, B, out=st["hash"])
        out = grid.forced_span(cfg, pool, B, CAP, case["steps"], stack_hash=st["hash"], workspace=st["ws"])
        return list(out) + [cfg, pool, st["hash"]]
    mask, eos, status, ws = st["mask"], st["eos"], st["status"], st["ws"]
    outs = [mask, eos, status]
    if kind == "mask":
        grid.mask(cfg, pool, B, mask[0], eos[0], status[0], ws)
    elif kind == "step":
        grid.mask(cfg, pool, B, mask[0], eos[0], status[0], ws)
        G.apply(mask[0], st["logits"][0])
        outs.append(st["logits"])
    elif kind == "decode":
        cfg.copy_(st["cfg0"])
        pool.copy_(st["pool0"])
        grid.stack_hash(cfg, pool, B, out=st["hash"])
        for k in range(case["steps"]):
            grid.mask(cfg, pool, B, mask[k], eos[k], status[k], ws)
            G.apply(mask[k], st["logits"][k])
            grid.accept_inplace(cfg, pool, st["tokens"][k], B, CAP, stack_hash=st["hash"], status=st["acc"][k])
        outs += [st["logits"], st["acc"], cfg, pool, st["hash"]]
    elif kind == "cached":
        grid.clear_cache(st["cache"])
        for k in range(2):
            grid.mask(cfg, pool, B, mask[k], eos[k], status[k], ws, cache=st["cache"], stack_hash=st["hash"])
    elif kind == "warm":
        grid.clear_ci_cache(st["cache"])
        for k in range(2):
            grid.mask_warm(cfg, pool, B, st["cache"], G.grid.CI_LOOKUP | G.grid.CI_INSERT, mask[k], eos[k], status[k],
                           ws)
    return outs


def work(case):
    """Each mask call reads the vocabulary's spellings (4 bytes a token on
    average) and the rows' configurations once and writes every row's mask; a
    fill reads the mask and writes the logits it forbids (nearly all of them);
    an advance reads and writes one configuration and its stack per row."""
    V, B, kind = case["V"], case["B"], case["kind"]
    words = (V + 31) // 32
    row = 32 + 2 * max(16, 2 * case["depth"])
    one_mask = 4 * V + B * (row + 4 * words + 5)
    fill = B * (4 * words + V * (2 if case["dtype"] == "bf16" else 4))
    step = B * (2 * row + 8)
    total = {"mask": one_mask, "step": one_mask + fill, "accept": step, "cached": 2 * one_mask, "warm": 2 * one_mask,
             "decode": case["steps"] * (one_mask + fill + step), "span": one_mask + B * 4 * case["steps"]}[kind]
    return {"bytes": total, "flops": 0}


def tolerance(case):
    return "exact"


def exact(case, seed):
    # no output is a rounded number: bits and states have no 64-bit value to be near to
    return None
