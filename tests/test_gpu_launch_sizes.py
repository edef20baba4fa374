"""Both workgroup sizes of the attention kernels (eight wavefronts, and the four
of small launches, short key sets and d = 64) on the same rows: bitwise equal
to each other where one call can take either, and against the oracle."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
from sampling import assert_parity, gather_rows, least_workspace, sample_rows, to_oracle_bits

pytestmark = pytest.mark.gpu

DEV = "cuda"
# with this max_seqlen the grid is past every small-launch rule, whatever the lengths
# are: d = 128 takes eight wavefronts unless the rows have few keys
LONG = 1 << 18


def B():
    from paper_2505_11254_amd import binding
    return binding


def make(lens, Hq, Hkv, d, seed):
    from paper_2505_11254_amd.inputs import random_qkv
    return random_qkv(lens, Hq, Hkv, d, seed, device="cpu")


# ragged lengths around a wavefront's 32 rows, the slabs of both sizes and a key tile
LENS = [(1, 31, 33, 0, 63, 65, 127, 129, 255, 257, 700), (2500,)]


@pytest.mark.parametrize("Hq,Hkv", [(2, 2), (4, 2), (6, 2), (4, 1), (8, 1)])
@pytest.mark.parametrize("lens", LENS, ids=["ragged", "one"])
def test_small_and_large_launches_agree_bitwise(lens, Hq, Hkv):
    """More keys per row than the short key sets that take half-size workgroups in every
    launch, fewer than the longest sequence has."""
    q, k, v, cu = (x.to(DEV) for x in make(lens, Hq, Hkv, 128, seed=Hq + len(lens)))
    kw = dict(cu_seqlens=cu)
    base = dict(window=1700, n_sink=3)
    for fn, more, which in ((B().sparse_attn_prefill, base, "base_waves"),
                            (B().dense_causal_attn_prefill, {}, "dense_waves")):
        for n, waves in ((max(lens), 4), (LONG, 8)):
            assert B().launch_workgroups(len(lens), n, Hq, Hkv, 128, 1, packed=True, **base)[which] == waves
        small = fn(q, k, v, max_seqlen=max(lens), **kw, **more)
        large = fn(q, k, v, max_seqlen=LONG, **kw, **more)
        torch.cuda.synchronize()
        assert torch.equal(small, large), fn.__name__


@pytest.mark.parametrize("Hq,Hkv,window,gamma", [(2, 1, 700, 2), (4, 1, 700, 16), (4, 1, 700, 64), (8, 1, 700, 32),
                                                 (2, 2, 1700, 2), (2, 2, 1700, 64), (6, 2, 1700, 128)])
def test_fused_delta_agrees_bitwise_at_both_sizes(Hq, Hkv, window, gamma):
    """The staged dense rows of open anchors and the fused store, in workgroups of both
    sizes.  The least workspace gives the small launch the one key chunk that these
    lengths fill of the large launch's."""
    lens, d = (2500, 129, 31, 0, 1000), 128
    q, k, v, cu = (x.to(DEV) for x in make(lens, Hq, Hkv, d, seed=gamma + Hq))
    kw = dict(window=window, n_sink=3, gamma=gamma, cu_seqlens=cu)
    sizes = lambda n: (len(lens), n, Hq, Hkv, d, gamma)
    assert B().fused_supported(Hq, Hkv, gamma)
    for n, waves in ((max(lens), 4), (LONG, 8)):
        got = B().launch_workgroups(*sizes(n), window=window, n_sink=3, packed=True)
        assert got["sparse_waves"] == waves and not got["together"], got
    assert B().launch_plan(*sizes(LONG))["chunk_keys"] >= max(lens)
    ws = torch.empty(least_workspace(*sizes(max(lens))), dtype=torch.uint8, device=DEV)
    small = B().delta_attn_prefill(q, k, v, max_seqlen=max(lens), workspace=ws, **kw)
    large = B().delta_attn_prefill(q, k, v, max_seqlen=LONG, **kw)
    torch.cuda.synchronize()
    assert torch.equal(small, large)


# (lens, Hq, Hkv, d, window, n_sink, gamma, max_seqlen, sparse wavefronts): fused slabs
# of half-size workgroups with one, two and four heads, gammas that only a full-size slab
# holds (256 at one head), many and few staged dense rows, odd gammas (unfused); with
# open anchors in every case
DELTA = [
    ((300, 1, 515), 1, 1, 64, 40, 3, 256, None, 8),
    ((700,), 2, 2, 64, 64, 4, 128, None, 4),
    ((900, 33), 8, 1, 64, 100, 5, 32, None, 4),
    ((700,), 4, 1, 64, 50, 0, 2, None, 4),
    ((515,), 5, 1, 64, 60, 1, 48, None, 4),
    ((700,), 4, 1, 128, 50, 0, 2, None, 4),
    ((1500,), 4, 1, 128, 700, 0, 2, LONG, 8),
    ((600, 129), 4, 1, 128, 64, 4, 64, None, 4),
    ((1500, 129), 4, 1, 128, 700, 4, 64, LONG, 8),
    ((515, 64), 3, 1, 128, 64, 4, 256, None, 8),
    ((2500, 64), 3, 1, 128, 1700, 4, 256, LONG, 8),
    ((515,), 2, 1, 128, 60, 1, 7, None, 4),
]


@pytest.mark.parametrize("case", DELTA, ids=[f"L{c[0]}-H{c[1]}/{c[2]}-d{c[3]}-w{c[4]}-g{c[6]}"
                                             f"{'-long' if c[7] else ''}" for c in DELTA])
def test_delta_matches_oracle_at_both_sizes(case):
    lens, Hq, Hkv, d, w, s, gamma, max_seqlen, waves = case
    assert max(lens) // gamma * gamma - gamma >= w + s  # (the last anchor's Delta)
    assert B().launch_workgroups(len(lens), max_seqlen or max(lens), Hq, Hkv, d, gamma, window=w,
                                 n_sink=s, packed=True)["sparse_waves"] == waves
    q, k, v, cu = make(lens, Hq, Hkv, d, seed=sum(lens) + d)
    out = B().delta_attn_prefill(q.to(DEV), k.to(DEV), v.to(DEV), window=w, n_sink=s, gamma=gamma,
                                 cu_seqlens=cu.to(DEV), max_seqlen=max_seqlen or max(lens))
    torch.cuda.synchronize()
    ref = oracle.delta_attention(*(to_oracle_bits(x) for x in (q, k, v)),
                                 cu.numpy().astype(np.int64), window=w, n_sink=s, gamma=gamma)
    assert_parity(out, ref, "delta path")


# (lens, Hq, Hkv, d, window, n_sink, gamma, wavefronts of both parts): the unfused schedule's
# sparse and strided rows in one launch, for both workgroup sizes and head sizes; a
# packed batch, numbers of strided workgroups that are no multiple of 8
SHARED = [
    ((32768,), 32, 8, 128, 2048, 64, 64, 8),
    ((4000, 1777, 31), 7, 7, 128, 2048, 16, 7, 8),
    ((515,), 2, 1, 128, 60, 1, 7, 4),
    ((700, 33), 3, 1, 128, 60, 1, 48, 4),
    ((515, 1, 449), 5, 1, 64, 60, 1, 48, 4),
    ((3000,), 8, 1, 64, 300, 1, 64, 4),
]


@pytest.mark.parametrize("case", SHARED, ids=[f"L{c[0]}-H{c[1]}/{c[2]}-d{c[3]}-g{c[6]}" for c in SHARED])
def test_one_launch_of_both_row_sets_equals_two(case):
    """The unfused schedule in one call, whose sparse and strided rows share a launch,
    against its steps in calls of their own (two launches): bitwise equal.  A smoothing
    correction takes the same launch; both against the oracle, the longest on sampled rows."""
    lens, Hq, Hkv, d, w, s, gamma, waves = case
    N, nb, packed = max(lens), len(lens), len(lens) > 1
    b = B()
    got = b.launch_workgroups(nb, N, Hq, Hkv, d, gamma, window=w, n_sink=s, mode=3, packed=packed)
    assert (got["sparse_waves"], got["rows_waves"], got["together"]) == (waves, waves, 1)
    q, k, v, cu = make(lens, Hq, Hkv, d, seed=N + Hq)
    qd, kd, vd, cud = (x.to(DEV) for x in (q, k, v, cu))
    kw = dict(window=w, n_sink=s, gamma=gamma)
    kw.update(dict(cu_seqlens=cud, max_seqlen=N) if packed else dict(B=1))

    def steps(*groups):
        ws = torch.full((b.workspace_bytes(nb, N, Hq, Hkv, d, gamma) // 4,), float("nan"), device=DEV)
        out = torch.full_like(qd, float("nan"))
        for bits in groups:
            b.delta_attn_prefill_steps(qd, kd, vd, out, ws, bits, **kw)
        torch.cuda.synchronize()
        return out

    one = steps(b.STEP_ALL)
    assert torch.equal(one, steps(b.STEP_SPARSE, b.STEP_DENSE_ROWS, b.STEP_CORRECT))
    assert torch.equal(one, steps(b.STEP_SPARSE | b.STEP_DENSE_ROWS, b.STEP_CORRECT))
    bits, cun = [to_oracle_bits(x) for x in (q, k, v)], cu.numpy().astype(np.int64)
    # (a short window leaves outputs of O(1): two bf16 roundings on top of the parity bound)
    slack = lambda ref: 2 * np.abs(ref) * 2.0 ** -8
    if N > 8192:
        rows = sample_rows(lens, Hq, w, s, gamma, n_random=64, seed=3)
        ref = oracle.delta_attention_rows(*bits, cun, rows=rows, window=w, n_sink=s, gamma=gamma)
        assert_parity(gather_rows(one, cun, rows), ref, "unfused schedule", slack=slack(ref))
        return
    ref = oracle.delta_attention(*bits, cun, window=w, n_sink=s, gamma=gamma)
    assert_parity(one, ref, "unfused schedule", slack=slack(ref))
    ema = b.delta_attn_prefill_correction(qd, kd, vd, mode=3, params=(0.5, 0.0, 0.0), **kw)
    torch.cuda.synchronize()
    ref = oracle.delta_attention_variant(*bits, cun, window=w, n_sink=s, gamma=gamma, mode=3,
                                         params=(0.5, 0.0, 0.0))
    assert_parity(ema, ref, "moving average", slack=slack(ref))


# one key chunk (448 keys) and the first sizes past it, one workgroup and many;
# chunks of the shortest and of in-between lengths; a batch, whose chunks are shorter
CHUNKS = [((n,), h, 1, d) for d in (64, 128) for n, h in ((1, 8), (448, 8), (449, 16), (1024, 1), (1025, 1))] + \
         [((2600,), 8, 8, 64), ((4021,), 2, 1, 128), ((1, 800, 1300), 4, 2, 128)]


@pytest.mark.parametrize("lens,Hq,Hkv,d", CHUNKS, ids=[f"L{c[0]}-H{c[1]}/{c[2]}-d{c[3]}" for c in CHUNKS])
def test_key_chunks_match_oracle_and_the_steps(lens, Hq, Hkv, d):
    """The whole call (which skips the merge of a single chunk) equals its steps
    one at a time bitwise, and the oracle."""
    w, s, gamma = 40, 3, 32
    q, k, v, cu = make(lens, Hq, Hkv, d, seed=sum(lens) + Hq)
    qd, kd, vd, cud = (x.to(DEV) for x in (q, k, v, cu))
    kw = dict(window=w, n_sink=s, gamma=gamma, cu_seqlens=cud, max_seqlen=max(lens))
    out = B().delta_attn_prefill(qd, kd, vd, **kw)
    ws = torch.empty(B().workspace_bytes(len(lens), max(lens), Hq, Hkv, d, gamma),
                     dtype=torch.uint8, device=DEV)
    by_steps = torch.empty_like(qd)
    for st in (B().STEP_DENSE_ROWS, B().STEP_CORRECT, B().STEP_SPARSE):
        B().delta_attn_prefill_steps(qd, kd, vd, by_steps, ws, st | B().STEP_FUSED, **kw)
    torch.cuda.synchronize()
    assert torch.equal(out, by_steps)
    ref = oracle.delta_attention(*(to_oracle_bits(x) for x in (q, k, v)),
                                 cu.numpy().astype(np.int64), window=w, n_sink=s, gamma=gamma)
    assert_parity(out, ref, "delta path")


@pytest.mark.parametrize("mode,params", [(2, (0.0, 0.0, 0.0)), (3, (0.05, 0.0, 0.0)), (3, (1.0, 0.0, 0.0)),
                                         (4, (0.2, 5e-2, 3.5e-3)), (4, (0.05, 1.25e-4, 2.08e-5))])
def test_recurrences_over_segment_edges_match_oracle(mode, params):
    """The scan cuts a sequence's anchors into 64 segments: none, one and two
    anchors, one per segment and around it, and several per segment with a
    short last one (the last filter setting is the unstable one)."""
    lens, gamma = (0, 1, 2, 4, 126, 128, 130, 133, 1900), 2
    q, k, v, cu = make(lens, 2, 1, 64, seed=mode)
    out = B().delta_attn_prefill_correction(
        *(x.to(DEV) for x in (q, k, v)), window=9, n_sink=1, gamma=gamma, mode=mode,
        params=params, cu_seqlens=cu.to(DEV), max_seqlen=max(lens))
    torch.cuda.synchronize()
    ref = oracle.delta_attention_variant(*(to_oracle_bits(x) for x in (q, k, v)),
                                         cu.numpy().astype(np.int64), window=9, n_sink=1,
                                         gamma=gamma, mode=mode, params=params)
    # (a window of 9 keys leaves outputs of O(1): their bf16 rounding, twice in this
    # schedule, comes on top of the parity bound)
    err = np.abs(out.float().cpu().numpy().astype(np.float64) - ref)
    assert (err <= 2e-2 + 2 * np.abs(ref) * 2.0 ** -8).all(), err.max()
    assert err.mean() <= 2e-3 + np.abs(ref).mean() * 2.0 ** -8


@pytest.mark.parametrize("Hkv", [1, 2, 3, 4, 5, 8, 10, 12, 16])
@pytest.mark.parametrize("G", [1, 2, 3, 4, 5, 8])
def test_block_order_covers_every_head_and_row(Hkv, G):
    """Each kv head's group in a call of its own (another number of head groups,
    so another block order) gives the same bits, for all three kernels (at most
    448 keys: one key chunk whatever the heads are)."""
    lens, d, window, n_sink, gamma = (430, 1, 137), 64 if G % 2 else 128, 30, 2, 32
    q, k, v, cu = (x.to(DEV) for x in make(lens, Hkv * G, Hkv, d, seed=Hkv * 10 + G))
    kw = dict(cu_seqlens=cu, max_seqlen=max(lens))

    def all_three(q, k, v):
        return (B().sparse_attn_prefill(q, k, v, window=window, n_sink=n_sink, **kw),
                B().dense_causal_attn_prefill(q, k, v, **kw),
                B().delta_attn_prefill(q, k, v, window=window, n_sink=n_sink, gamma=gamma, **kw))

    whole = all_three(q, k, v)
    for h in range(Hkv):
        one = all_three(q[:, h * G:(h + 1) * G].contiguous(), k[:, h:h + 1].contiguous(),
                        v[:, h:h + 1].contiguous())
        torch.cuda.synchronize()
        for name, x, y in zip(("sparse", "dense", "delta"), whole, one):
            assert torch.equal(x[:, h * G:(h + 1) * G], y), (name, h)


@pytest.mark.parametrize("N,Hq,Hkv,d,gamma", [(4021, 8, 2, 128, 64), (3000, 4, 4, 64, 48), (900, 16, 4, 128, 32)])
def test_a_smaller_workspace_splits_the_keys_coarser(N, Hq, Hkv, d, gamma):
    """Less than da_workspace_bytes, down to what chunks of at least 2560 keys
    need, is taken (within rounding of the full split); less than that is refused."""
    q, k, v, _ = make((N,), Hq, Hkv, d, seed=N)
    least = least_workspace(1, N, Hq, Hkv, d, gamma)
    full = B().workspace_bytes(1, N, Hq, Hkv, d, gamma)
    assert full > least
    qd, kd, vd = (x.to(DEV) for x in (q, k, v))
    kw = dict(window=64, n_sink=4, gamma=gamma)
    ref = oracle.delta_attention(*(to_oracle_bits(x) for x in (q, k, v)), None, **kw)
    for size in (least, (least + full) // 2 // 16 * 16, full):
        ws = torch.empty(size, dtype=torch.uint8, device=DEV)
        out = B().delta_attn_prefill(qd, kd, vd, workspace=ws, **kw)
        torch.cuda.synchronize()
        assert_parity(out, ref, f"workspace of {size}")
    with pytest.raises(RuntimeError, match="DA_ERR_WORKSPACE"):
        B().delta_attn_prefill(qd, kd, vd, workspace=ws[:least - 256].clone(), **kw)
