"""The recurrences of the smoothing corrections where they leave the usual range."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
from sampling import to_oracle_bits

pytestmark = pytest.mark.gpu

DEV = "cuda"


def B():
    from paper_2505_11254_amd import binding
    return binding


def make(lens, Hq, Hkv, d, seed):
    from paper_2505_11254_amd.inputs import random_qkv
    return [x.to(DEV) for x in random_qkv(lens, Hq, Hkv, d, seed, device="cpu")]


# gains whose closed loop grows by 1.362 (20000 anchors: 1e42 over a 64th of them),
# 19 and 2e5 per anchor
@pytest.mark.parametrize("N,d,params,window", [
    (20000, 64, (0.1, 1.0, 1.0), 2048), (20000, 64, (0.1, 1.0, 1.0), 20000),
    (2100, 128, (20.0, 0.0, 0.0), 900), (2100, 64, (20.0, 0.0, 0.0), 4096),
    (300, 64, (2e5, 1.0, 1.0), 200), (60, 64, (2e5, 1.0, 1.0), 40)])
def test_a_diverging_filter_keeps_the_rows_before_its_first_delta(N, d, params, window):
    """Anchors whose key set is whole have a Delta of exactly zero, and so has the
    filter until the first other anchor: their rows stay the sparse rows bit for bit,
    and the rows that follow are finite until the filter itself is not."""
    n_sink = 1
    q, k, v, _ = make((N,), 1, 1, d, seed=N + d)
    out = B().delta_attn_prefill_correction(q, k, v, window=window, n_sink=n_sink, gamma=1,
                                            mode=B().CORR_ABG, params=params)
    sparse = B().sparse_attn_prefill(q, k, v, window=window, n_sink=n_sink)
    torch.cuda.synchronize()
    cover = min(N, window + n_sink)
    assert torch.equal(out[:cover], sparse[:cover])
    assert torch.isfinite(out[:cover + 6].float()).all()


@pytest.mark.parametrize("mode,params", [(3, (0.3, 0.0, 0.0)), (4, (0.2, 5e-2, 3.5e-3))])
def test_more_channels_than_one_launch_takes(mode, params):
    """32768 sequences of 32 heads: 2^32 threads of the scan, more than one dispatch
    holds.  Any part of the batch gives the same bits by itself."""
    nb, L, Hq, d = 32768, 4, 32, 64
    g = torch.Generator(device=DEV)
    g.manual_seed(mode)
    rand = lambda H: torch.randn((nb * L, H, d), generator=g, device=DEV, dtype=torch.bfloat16)
    q, k, v = rand(Hq), rand(1), rand(1)
    kw = dict(window=1, n_sink=0, gamma=2, mode=mode, params=params)
    out = B().delta_attn_prefill_correction(q, k, v, B=nb, **kw)
    for b0 in (0, 8191, 16383, nb - 16):
        part = slice(b0 * L, (b0 + 16) * L)
        some = B().delta_attn_prefill_correction(*(x[part].contiguous() for x in (q, k, v)), B=16, **kw)
        torch.cuda.synchronize()
        assert torch.equal(out[part], some), b0


# (lens, heads, gamma): channels (64 per sequence and head) around the lines between
# one thread per channel and segments: 64 anchors, a 64th of the channels, 32768 channels;
# a number of channels that is no multiple of a workgroup's 256
@pytest.mark.parametrize("lens,Hq,gamma", [((128,), 1, 2), ((130,), 1, 2), ((258,), 128, 2), ((256, 7), 64, 2),
                                           ((170, 9, 0, 64, 131, 66, 140, 1), 64, 1)])
@pytest.mark.parametrize("mode,params", [(3, (0.3, 0.0, 0.0)), (4, (0.2, 5e-2, 3.5e-3))])
def test_scans_in_order_and_in_segments_match_the_oracle(lens, Hq, gamma, mode, params):
    from paper_2505_11254_amd.inputs import random_qkv
    q, k, v, cu = random_qkv(lens, Hq, 1, 64, seed=len(lens) + Hq, device="cpu")
    kw = dict(window=9, n_sink=1, gamma=gamma, mode=mode, params=params)
    out = B().delta_attn_prefill_correction(*(x.to(DEV) for x in (q, k, v)), cu_seqlens=cu.to(DEV),
                                            max_seqlen=max(lens), **kw)
    torch.cuda.synchronize()
    ref = oracle.delta_attention_variant(*(to_oracle_bits(x) for x in (q, k, v)), cu.numpy().astype(np.int64), **kw)
    # (a window of 9 keys leaves outputs of O(1): their bf16 rounding, twice in this
    # schedule, comes on top of the parity bound)
    err = np.abs(out.float().cpu().numpy().astype(np.float64) - ref)
    assert (err <= 2e-2 + 2 * np.abs(ref) * 2.0 ** -8).all(), err.max()
    assert err.mean() <= 2e-3 + np.abs(ref).mean() * 2.0 ** -8
