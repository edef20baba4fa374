"""The calls whose speed on the GPU counts: what a user of this library has it do.

Every case is one prefill of an attention layer (or of a packed batch of
prompts) through a public entry point of ``paper_2505_11254_amd.binding``:

  delta      Delta Attention prefill (sink + window base), fixed length or packed
             with cu_seqlens
  noalloc    the same through the allocation-free entry point (serving loops)
  variant    a step-5 correction variant (recompute, interpolation, EMA, filter)
  lists      Delta Attention over key-block lists
  sparse     the sparse base alone (sink + window)
  dense      dense causal attention for every row (the quadratic baseline)

Inputs are bf16, the library's one data type: unit normal queries, keys and
values, keys with a mean offset per kv head as trained models show.  ``kept``
says who owns the output and the workspace: the caller, laid out once per shape
as a serving loop does, or each call (a first try at the API).
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2505_11254_amd import binding, blocklists

DEV = "cuda"
MODES = {"recompute": 1, "interp": 2, "ema": 3, "filter": 4}
PARAMS = {"recompute": (0.0, 0.0, 0.0), "interp": (0.0, 0.0, 0.0), "ema": (0.5, 0.0, 0.0),
          "filter": (0.2, 5e-2, 3.5e-3)}


def _case(kind, lens, Hq, Hkv, d, window=0, n_sink=0, gamma=0, kept=True, packed=False, **more):
    return dict(kind=kind, lens=",".join(str(n) for n in lens), Hq=Hq, Hkv=Hkv, d=d, window=window,
                n_sink=n_sink, gamma=gamma, kept=kept, packed=packed, **more)


def _lens(case):
    return [int(x) for x in case["lens"].split(",")]


def listed():
    def named(name, c):
        c["name"] = name
        return c

    llama = dict(Hq=32, Hkv=8, d=128, window=2048, n_sink=64, gamma=64)
    return [
        # The smallest call, as a unit test or a first try makes it: one short head, nothing kept.
        named("tiny_1k_d64", _case("delta", [1024], 1, 1, 64, 128, 4, 16, kept=False)),
        # An everyday prompt of a few thousand tokens, of no round length, in an 8B-shaped layer.
        named("prompt_4k", _case("delta", [4021], **llama)),
        # The 8B-shaped layer at the lengths of the method's latency study.
        named("llama8b_32k", _case("delta", [32768], **llama)),
        named("llama8b_131k", _case("delta", [131072], **llama)),
        named("llama8b_1m", _case("delta", [1048576], **llama)),
        # A packed batch of long documents, GQA 8, wide window, dense anchors.
        named("ragged_b4_gqa8", _case("delta", [16384, 40000, 65536, 131072], 64, 8, 128, 4096, 128,
                                      32, packed=True)),
        # A serving step: short prompts of mixed lengths packed together, no allocation allowed.
        named("serve_noalloc_b8", _case("noalloc", [777, 64, 2500, 1000, 3071, 1, 513, 1800],
                                        packed=True, **llama)),
        # GQA 3 and a stride that no power of two is a multiple of.
        named("gqa3_gamma48_20k", _case("delta", [20011], 24, 8, 128, 1024, 16, 48)),
        # A smoothing correction (moving average over the rows) at a usual long-prompt length.
        named("variant_ema_64k", _case("variant", [65536], mode="ema", **llama)),
        # The correction over another sparse base: columns, band and diagonals as key-block lists.
        named("lists_vslash_64k", _case("lists", [65536], 32, 8, 128, 0, 0, 64, layout="vslash",
                                        block_q=64)),
        # The sparse base alone, multi-head attention with small heads, two odd-sized prompts.
        named("sparse_mha_d64", _case("sparse", [30011, 8190], 16, 16, 64, 1024, 16, packed=True)),
        # The quadratic baseline that the method is compared with.
        named("dense_16k", _case("dense", [16384], 32, 8, 128)),
    ]


def _log_int(rng, lo, hi):
    n = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    return max(lo, min(hi, n))


def draw(rng):
    while True:
        kind = rng.choice(["delta", "delta", "delta", "noalloc", "variant", "variant", "lists",
                           "sparse", "dense"])
        packed = rng.random() < 0.4
        top = {"noalloc": 24576, "dense": 49152, "lists": 131072}.get(kind, 262144)
        n = _log_int(rng, 300, top)
        if rng.random() < 0.4:
            n = max(256, n // 256 * 256)
        lens = [n]
        if packed:
            lens = [max(1, int(n * rng.uniform(0.02, 1.0))) for _ in range(rng.randint(2, 6))]
        G = rng.choice([1, 2, 3, 4, 4, 4, 5, 8])
        Hkv = rng.choice([2, 4, 8, 8])
        d = rng.choice([64, 128, 128])
        gamma = rng.choice([8, 16, 32, 64, 64, 64, 128, 256, 7, 48, 100])
        window = rng.choice([64, 256, 512, 1000, 1024, 2048, 2048, 4096])
        n_sink = rng.choice([0, 1, 4, 16, 64, 64, 128])
        kept = rng.random() < 0.75
        more = {}
        if kind == "variant":
            more["mode"] = rng.choice(["recompute", "interp", "ema", "filter"])
        if kind == "lists":
            more["layout"] = rng.choice(["vslash", "topk", "star"])
            slab = 256 // max(h for h in (1, 2, 4, 8) if G % h == 0)
            more["block_q"] = rng.choice([b for b in (64, 128, 256) if b >= slab])
            window = n_sink = 0
        if kind == "sparse":
            gamma = 0
        if kind == "dense":
            gamma = window = n_sink = 0
        case = _case(kind, lens, G * Hkv, Hkv, d, window, n_sink, gamma, kept, packed, **more)
        if kind == "noalloc":  # the static scratch holds a bounded problem (one key chunk at least)
            rows = max(lens) // gamma + gamma
            if len(lens) * G * Hkv * rows * (2 * d + 2) * 4 > binding_scratch_bytes() * 3 // 4:
                continue
        if _flops(case) < 1.2e14 and _partials(case) < 16e9:
            return case


def binding_scratch_bytes():
    return 256 << 20  # DA_NOALLOC_SCRATCH_BYTES of include/delta_attn.h


def _partials(case):
    """A bound on the workspace of the strided rows, in bytes."""
    if not case["gamma"]:
        return 0
    lens = _lens(case)
    rows = max(lens) // case["gamma"] + case["gamma"]
    return len(lens) * case["Hq"] * rows * (case["d"] + 2) * 4 * 2


# ---- inputs ----

def _inputs(case, seed):
    T = sum(_lens(case))
    Hq, Hkv, d = case["Hq"], case["Hkv"], case["d"]
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 8 + 3)
    offset = torch.randn((Hkv, d), generator=g, device=DEV) * 0.5

    def normal(H, add=None):
        x = torch.empty((T, H, d), dtype=torch.bfloat16, device=DEV)
        for t0 in range(0, T, 65536):
            y = torch.randn((min(65536, T - t0), H, d), generator=g, device=DEV)
            x[t0:t0 + y.shape[0]].copy_(y if add is None else y + add)
        return x

    return normal(Hq), normal(Hkv, offset), normal(Hkv)


def _lists(case, seed):
    lens, Hkv, bq = _lens(case), case["Hkv"], case["block_q"]
    if case["layout"] == "vslash":  # about 1980 keys a row
        return blocklists.vertical_slash(lens, Hkv, block_q=bq, n_vertical=8, n_local=24, seed=seed)
    if case["layout"] == "topk":    # about 2140
        return blocklists.block_topk(lens, Hkv, block_q=bq, k=33, seed=seed)
    return blocklists.star(lens, Hkv, block_q=bq, anchor=2048, context=4096)  # about 4090


def prepare(case, seed):
    """Q, K and V in HBM, the batch's offsets and lists, and where the caller keeps
    them, the output and the workspace."""
    lens = _lens(case)
    q, k, v = _inputs(case, seed)
    kw = {}
    if case["packed"]:
        cu = [0]
        for n in lens:
            cu.append(cu[-1] + n)
        kw.update(cu_seqlens=torch.tensor(cu, dtype=torch.int32, device=DEV), max_seqlen=max(lens))
    kind = case["kind"]
    if kind in ("delta", "noalloc", "variant", "sparse"):
        kw.update(window=case["window"], n_sink=case["n_sink"])
    if kind in ("delta", "noalloc", "variant", "lists"):
        kw.update(gamma=case["gamma"])
    if kind == "variant":
        kw.update(mode=MODES[case["mode"]], params=PARAMS[case["mode"]])
    if kind == "lists":
        ptr, idx = _lists(case, seed).to(DEV)
        kw.update(block_q=case["block_q"], block_ptr=ptr, block_idx=idx)
    if case["kept"]:
        kw.update(out=torch.empty_like(q))
        sizes = (len(lens), max(lens), case["Hq"], case["Hkv"], case["d"], case["gamma"])
        if kind == "variant":
            n = int(binding.load_library().da_workspace_bytes_correction(*sizes, kw["mode"]))
        elif kind in ("delta", "lists"):
            n = binding.workspace_bytes(*sizes)
        else:
            n = 0
        if n:
            kw.update(workspace=torch.empty(n, dtype=torch.uint8, device=DEV))
    fn = {"delta": binding.delta_attn_prefill, "noalloc": binding.delta_attn_prefill_noalloc,
          "variant": binding.delta_attn_prefill_correction,
          "lists": binding.delta_attn_prefill_blocksparse, "sparse": binding.sparse_attn_prefill,
          "dense": binding.dense_causal_attn_prefill}[kind]
    return fn, (q, k, v), kw


def run(state):
    fn, qkv, kw = state
    return fn(*qkv, **kw)


# ---- what a pass cannot do without ----

def _pairs(case):
    """(row, key) pairs of one query head, summed over the batch: the sparse rows,
    plus the dense rows at the anchors whose key set is not already whole and at
    the tail rows."""
    kind, w, s, gamma = case["kind"], case["window"], case["n_sink"], case["gamma"]
    lens = _lens(case)
    tot = 0
    if kind == "lists":  # keys a row sees on average in each layout, plus half its own block
        mean = {"vslash": 1980, "topk": 2140, "star": 4090}[case["layout"]]
        for L in lens:
            i = np.arange(L, dtype=np.int64)
            tot += int(np.minimum(i + 1, mean).sum())
    for L in lens:
        i = np.arange(L, dtype=np.int64)
        if kind == "dense":
            tot += int((i + 1).sum())
        elif kind != "lists":
            tot += int((np.minimum(i + 1, w) + np.minimum(np.maximum(i + 1 - w, 0), s)).sum())
        if gamma:
            a = np.arange(0, L // gamma * gamma, gamma, dtype=np.int64)
            if kind != "lists":
                a = a[a >= w + s]
            tot += int((a + 1).sum()) + int((np.arange(L // gamma * gamma, L, dtype=np.int64) + 1).sum())
    return tot


def _flops(case):
    return 4.0 * case["d"] * case["Hq"] * _pairs(case)


def work(case):
    T = sum(_lens(case))
    return {"bytes": 2.0 * T * case["d"] * (2 * case["Hq"] + 2 * case["Hkv"]),
            "flops": _flops(case)}


def tolerance(case):
    # bf16 outputs (half an ulp: 0.0011-0.0020 of the value), weights rounded to bf16 for P V, and
    # sparse rows rounded to bf16 before the correction in one of the two schedules.  Measured
    # against `exact` over the listed cases and 24 drawn ones: rel 0.0019-0.0029; max 0.01-0.09 (the
    # long tensors, whose first rows average few keys and stand far above the tensor's rms).
    return {"rel": 1e-2, "max": 0.3}


# ---- 64-bit reference, plain torch ----

def _softmax_rows(q, k, v, mask):
    """q [Hkv, G*R, d], k/v [Hkv, K, d], mask [Hkv or 1, R, K] -> [Hkv, G*R, d]."""
    Hkv, GR, d = q.shape
    R = mask.shape[1]
    s = torch.bmm(q, k.transpose(1, 2).contiguous()).view(Hkv, GR // R, R, -1)
    s.mul_(1.0 / math.sqrt(d)).masked_fill_(~mask[:, None], -math.inf)
    s.sub_(s.amax(-1, keepdim=True)).exp_()
    s.div_(s.sum(-1, keepdim=True))
    return torch.bmm(s.view(Hkv, GR, -1), v)


def _group(q, pos, Hkv):
    """Rows `pos` of q [L, Hq, d] as float64 [Hkv, G*R, d] (head outer, row inner)."""
    x = q[pos].double()
    R, Hq, d = x.shape
    return x.permute(1, 0, 2).reshape(Hkv, Hq // Hkv * R, d)


def _ungroup(o, R):
    Hkv, GR, d = o.shape
    return o.view(Hkv * GR // R, R, d).permute(1, 0, 2)  # [R, Hq, d]


def _kv(x, idx):
    return x[idx].double().permute(1, 0, 2).contiguous()  # [Hkv, K, d]


def _dense_rows(q, k, v, pos):
    """Dense causal rows at the ascending positions `pos`."""
    Hkv, Hq = k.shape[1], q.shape[1]
    out = torch.empty((len(pos), Hq, q.shape[2]), dtype=torch.float64, device=DEV)
    i = 0
    while i < len(pos):
        r = 256
        while r > 1 and r * Hq * (int(pos[min(i + r, len(pos)) - 1]) + 1) > (1 << 28):
            r //= 2
        p = pos[i:i + r]
        keys = torch.arange(int(p[-1]) + 1, device=DEV)
        o = _softmax_rows(_group(q, p, Hkv), _kv(k, keys), _kv(v, keys), (keys <= p[:, None])[None])
        out[i:i + len(p)] = _ungroup(o, len(p))
        i += r
    return out


def _sparse_rows(case, q, k, v, blocks):
    """The sparse base for every row of one sequence."""
    L, Hq, d = q.shape
    Hkv, w, s = k.shape[1], case["window"], case["n_sink"]
    out = torch.empty((L, Hq, d), dtype=torch.float64, device=DEV)
    step = case["block_q"] if blocks is not None else 512
    for r0 in range(0, L, step):
        p = torch.arange(r0, min(L, r0 + step), device=DEV)
        R, hi = len(p), int(p[-1])
        if blocks is None:
            ns = min(s, hi + 1)
            keys = torch.cat([torch.arange(ns, device=DEV),
                              torch.arange(max(ns, r0 - w + 1), hi + 1, device=DEV)])
            mask = ((keys <= p[:, None]) & ((keys < s) | (p[:, None] - keys < w)))[None]
            o = _softmax_rows(_group(q, p, Hkv), _kv(k, keys), _kv(v, keys), mask)
        else:
            tiles = [blocks(g, r0 // step) for g in range(Hkv)]
            m = max(len(t) for t in tiles)
            own = np.arange(r0, hi + 1)
            idx = np.full((Hkv, m * 64 + len(own)), -1, dtype=np.int64)
            for g, t in enumerate(tiles):
                idx[g, :len(t) * 64] = (t[:, None].astype(np.int64) * 64 + np.arange(64)).reshape(-1)
                idx[g, m * 64:] = own
            idx = torch.from_numpy(idx).to(DEV)
            heads = torch.arange(Hkv, device=DEV)[:, None]
            at = idx.clamp(min=0)
            mask = (idx[:, None] >= 0) & (idx[:, None] <= p[None, :, None])
            o = _softmax_rows(_group(q, p, Hkv), k[at, heads].double(), v[at, heads].double(), mask)
        out[r0:r0 + R] = _ungroup(o, R)
    return out


def _corrected(case, sp, dn, L):
    """Algorithm 1's last step on one sequence: sp [L, Hq, d] (overwritten), dn the
    dense rows at the anchors and then at the tail rows."""
    gamma = case["gamma"]
    nA = L // gamma
    if nA:
        whole = sp[:nA * gamma].view(nA, gamma, *sp.shape[1:])
        delta = dn[:nA] - whole[:, 0]
        mode = case.get("mode", "delta")
        if mode == "recompute":
            whole[:, 0] += delta
        elif mode == "interp":
            nxt = torch.cat([delta[1:], delta[-1:]])
            b = (torch.arange(gamma, device=DEV, dtype=torch.float64) / max(gamma - 1, 1))[None, :, None, None]
            whole += (1 - b) * delta[:, None] + b * nxt[:, None]
        elif mode == "ema":
            wgt = PARAMS["ema"][0]
            decay = (1.0 - wgt) ** torch.arange(1, gamma + 1, device=DEV, dtype=torch.float64)
            e = delta[0].clone()
            for i in range(nA):
                rows = decay[:, None, None] * e + (1 - decay)[:, None, None] * delta[i]
                whole[i] += rows
                e = rows[-1].clone()
        elif mode == "filter":
            g0, g1, g2 = PARAMS["filter"]
            x, y, z = delta[0].clone(), torch.zeros_like(delta[0]), torch.zeros_like(delta[0])
            whole[0] += x
            for i in range(1, nA):
                px, py, pz = x + y + 0.5 * z, y + z, z
                r = delta[i] - px
                x, y, z = px + g0 * r, py + g1 * r, pz + g2 * r
                whole[i] += x
        else:
            whole += delta[:, None]
    sp[nA * gamma:] = dn[nA:]
    return sp


def exact(case, seed):
    if _flops(case) > 5e13:
        return None
    q, k, v = _inputs(case, seed)
    lists = _lists(case, seed) if case["kind"] == "lists" else None
    out = torch.empty(q.shape, dtype=torch.float64, device=DEV)
    t0 = 0
    for b, L in enumerate(_lens(case)):
        qs, ks, vs = q[t0:t0 + L], k[t0:t0 + L], v[t0:t0 + L]
        if case["kind"] == "dense":
            out[t0:t0 + L] = _dense_rows(qs, ks, vs, torch.arange(L, device=DEV))
        else:
            blocks = None if lists is None else (lambda g, qb, b=b: lists.tiles(b, g, qb))
            sp = _sparse_rows(case, qs, ks, vs, blocks)
            gamma = case["gamma"]
            if gamma:
                nA = L // gamma
                pos = torch.cat([torch.arange(nA, device=DEV) * gamma,
                                 torch.arange(nA * gamma, L, device=DEV)])
                sp = _corrected(case, sp, _dense_rows(qs, ks, vs, pos), L)
            out[t0:t0 + L] = sp
        t0 += L
    return out
