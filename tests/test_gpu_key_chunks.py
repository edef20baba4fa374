"""The split of the strided rows' key axis: what a finer one may change, and what
the workspace and the steps of one pass have to do with it."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
from sampling import assert_parity, gather_rows, least_workspace, sample_rows, to_oracle_bits

pytestmark = pytest.mark.gpu

DEV = "cuda"


def B():
    from paper_2505_11254_amd import binding
    return binding


def make(lens, Hq, Hkv, d, seed):
    from paper_2505_11254_amd.inputs import random_qkv
    return random_qkv(lens, Hq, Hkv, d, seed, device="cpu")


@pytest.mark.parametrize("N,d,window,gamma", [(2500, 128, 1024, 64), (2500, 64, 1024, 32), (4021, 128, 2048, 64)])
def test_a_finer_key_split_costs_no_precision(N, d, window, gamma):
    """Corrected rows against the 64-bit oracle, long key chunks and the 16 that the
    launch takes.  Where every weight rounds alike the two errors differ by the rare
    roundings that a last bit of the exponent's argument turns (under 1 %); with a
    reference of its own per chunk, 16 chunks of 2500 tokens read 21 % more."""
    Hq, Hkv, n_sink = 8, 2, 64
    q, k, v, _ = make((N,), Hq, Hkv, d, seed=N + d)
    qd, kd, vd = (x.to(DEV) for x in (q, k, v))
    kw = dict(window=window, n_sink=n_sink, gamma=gamma)
    ref = oracle.delta_attention(*(to_oracle_bits(x) for x in (q, k, v)), None, **kw)
    pos = np.arange(N)
    rows = (pos - pos % gamma >= window + n_sink) & (pos % gamma != 0) & (pos < N // gamma * gamma)
    full = B().workspace_bytes(1, N, Hq, Hkv, d, gamma)
    least = least_workspace(1, N, Hq, Hkv, d, gamma)
    assert full > 3 * least
    err = []
    for size in (least, full):
        ws = torch.empty(size, dtype=torch.uint8, device=DEV)
        out = B().delta_attn_prefill(qd, kd, vd, workspace=ws, **kw).float().cpu().numpy()
        err.append(np.linalg.norm(out[rows] - ref[rows]) / np.linalg.norm(ref[rows]))
    print("rel error: long chunks %.6f, finer %.6f" % tuple(err))
    assert err[1] <= 1.02 * err[0]


@pytest.mark.parametrize("N,Hq,Hkv,d", [(300, 8, 2, 128), (320, 1, 1, 64), (40, 4, 4, 64)])
@pytest.mark.parametrize("first", ["whole", "all steps", "both steps"])
def test_the_merge_alone_follows_any_call_that_ran_the_strided_rows(N, Hq, Hkv, d, first):
    """One key chunk: the call that needs no merge leaves what a merge on its own
    reads, and what the sparse step on its own reads."""
    q, k, v, _ = (x.to(DEV) for x in make((N,), Hq, Hkv, d, seed=N))
    kw = dict(window=40, n_sink=3, gamma=32)
    b = B()
    assert b.launch_plan(1, N, Hq, Hkv, d, 32)["key_chunks"] == 1
    want = b.delta_attn_prefill(q, k, v, **kw)
    ws = torch.full((b.workspace_bytes(1, N, Hq, Hkv, d, 32) // 4,), float("nan"), device=DEV)
    out = torch.full_like(q, float("nan"))
    step = lambda bits: b.delta_attn_prefill_steps(q, k, v, out, ws, bits | b.STEP_FUSED, **kw)
    if first == "whole":
        b.delta_attn_prefill(q, k, v, out=out, workspace=ws, **kw)
    else:
        step(b.STEP_ALL if first == "all steps" else b.STEP_DENSE_ROWS | b.STEP_CORRECT)
    for again in (b.STEP_SPARSE, b.STEP_CORRECT, b.STEP_SPARSE):
        out.fill_(float("nan")) if again == b.STEP_SPARSE else None
        step(again)
        if again == b.STEP_SPARSE:
            torch.cuda.synchronize()
            assert torch.equal(out, want)


@pytest.mark.parametrize("fused", [True, False])
def test_steps_agree_on_the_layout_whatever_smaller_workspace_each_is_given(fused):
    """Strided rows and merge in calls of their own, on one buffer, told of different
    sizes below the full one: one layout, that of the long chunks."""
    N, Hq, Hkv, d, gamma = 6000, 4, 2, 128, 64
    b = B()
    q, k, v, _ = (x.to(DEV) for x in make((N,), Hq, Hkv, d, seed=N))
    kw = dict(window=100, n_sink=3, gamma=gamma)
    full, least = b.workspace_bytes(1, N, Hq, Hkv, d, gamma), least_workspace(1, N, Hq, Hkv, d, gamma)
    middle = (least + full) // 512 * 256
    ws = torch.empty(full, dtype=torch.uint8, device=DEV)
    F = b.STEP_FUSED if fused else 0

    def run(out, size, bits):
        b.delta_attn_prefill_steps(q, k, v, out, ws[:size], bits | F, **kw)
        torch.cuda.synchronize()

    want = torch.empty_like(q)
    run(want, least, b.STEP_ALL)
    order = [b.STEP_DENSE_ROWS, b.STEP_CORRECT, b.STEP_SPARSE] if fused else \
            [b.STEP_SPARSE, b.STEP_DENSE_ROWS, b.STEP_CORRECT]
    for sizes in ((least, middle, full - 256), (full - 256, least, middle), (middle, full - 256, least)):
        ws.fill_(255)
        out = torch.empty_like(q)
        for bits, size in zip(order, sizes):
            run(out, size, bits)
        assert torch.equal(out, want), sizes
    whole = torch.empty_like(q)
    run(whole, full, b.STEP_ALL)
    for bits in order:
        run(out, full, bits)
    assert torch.equal(out, whole)


@pytest.mark.parametrize("N,Hq,Hkv,d,gamma,chunks", [(14000, 64, 8, 64, 4, 6), (16500, 32, 8, 128, 8, 7)])
def test_merge_of_many_rows_matches_the_oracle(N, Hq, Hkv, d, gamma, chunks):
    """Five to eight key chunks and more rows than the merge takes eight at a time:
    sampled rows, and every anchor row (the merged dense row) against the dense kernel."""
    b = B()
    assert b.launch_plan(1, N, Hq, Hkv, d, gamma)["key_chunks"] == chunks
    assert Hq * (N // gamma) * (d // 4) >= 1 << 21
    q, k, v, cu = make((N,), Hq, Hkv, d, seed=N)
    kw = dict(window=300, n_sink=5, gamma=gamma)
    qd, kd, vd = (x.to(DEV) for x in (q, k, v))
    out = b.delta_attn_prefill(qd, kd, vd, **kw)
    dense = b.dense_causal_attn_prefill(qd, kd, vd)
    a = torch.arange(0, N // gamma * gamma, gamma, device=DEV)
    # (outputs below 1/8 past the first rows: half a bf16 ulp each, and weights in bf16)
    diff = (out[a] - dense[a]).float().abs()
    assert float((diff - 2.0 ** -7 * dense[a].float().abs()).max()) <= 4e-3
    rows = sample_rows((N,), Hq, 300, 5, gamma, n_random=48, seed=2)
    ref = oracle.delta_attention_rows(*(to_oracle_bits(x) for x in (q, k, v)), cu.numpy().astype(np.int64),
                                      rows=rows, **kw)
    assert_parity(gather_rows(out, [0, N], rows), ref, "delta path")
