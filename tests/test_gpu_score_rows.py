"""Scoring with 16 queries a workgroup: probabilities and on-the-fly salience against the oracle at key counts around
the edges of its five row lengths and of a key block, at query counts around one and two tiles, with and without a
scoring bias, and at batches on both sides of the number of workgroups up to which it is taken."""
import re
from dataclasses import replace

import numpy as np
import pytest
import torch

import oracle as O
from helpers import device_layer, layer_cfg, oracle_weights, to64
from paper_2604_09244_amd import binding as mv
from paper_2604_09244_amd import workloads as W

pytestmark = pytest.mark.gpu

# bf16 queries and keys (relative error 2^-9 each) put about 2^-8 of a logit's magnitude on it: a few percent
# of a probability at logits of a few units (as in test_gpu_layer.py)
RTOL, ATOL = 6e-2, 2e-5


@pytest.mark.parametrize("dh,H", [(64, 4), (128, 2)])
@pytest.mark.parametrize("S,nq,B", [(18, 17, 1), (33, 1, 2), (130, 16, 1), (256, 33, 1), (257, 15, 3), (640, 31, 1),
                                    (641, 17, 2), (1024, 64, 1), (1025, 16, 1), (300, 17, 32), (300, 17, 33),
                                    (300, 17, 64), (300, 17, 65), (300, 16, 65), (256, 17, 65)])
def test_scoring_rows(dh, H, S, nq, B):
    wl = replace(W.WORKLOADS["tiny"], D=H * dh, H=H, dh=dh, F=256, n2=(S - nq) // 2, n3=S - nq - (S - nq) // 2, nt=nq,
                 B=B, L=1, p=0, seed=S + nq + dh)
    ctx = mv.Context(B, S, wl.D, H, wl.F, nq)
    w_cpu = W.layer_weights(wl, 0)
    packed, ws = device_layer(ctx, wl, w_cpu)
    x, pos = W.hidden_states(wl)
    kb = W.scoring_bias(wl) if B % 2 else None
    xd, pd, kd = x.cuda(), pos.cuda(), None if kb is None else kb.cuda()
    probs = to64(ctx.score_only(layer_cfg(wl), ws, xd, pd, nq, kd))
    y, full = ctx.prefill_layer(layer_cfg(wl), ws, xd, pd, n_query_tail=nq, key_bias=kd)
    _, sal = ctx.prefill_layer_salience(layer_cfg(wl), ws, xd, pd, nq, S - nq, key_bias=kd)
    full, sal = to64(full), to64(sal)
    wo = oracle_weights(w_cpu)
    for b in sorted({0, B - 1}):
        ref = O.score_only(to64(x[b]), pos[b].numpy(), wo, H, nq, wl.rms_eps, wl.rope_base,
                           None if kb is None else kb[b].numpy())
        for got in (probs[b], full[b]):
            assert np.all(np.abs(got - ref) <= RTOL * np.abs(ref) + ATOL), np.abs(got - ref).max()
            assert np.allclose(got.sum(-1), 1.0, atol=1e-4)
    # the salience of the same call's probabilities: fp32 sums of at most 256 terms each way (256 * 2^-24 = 1.5e-5)
    mean = full[:, :, :, :S - nq].sum((1, 2)) / (H * nq)
    assert np.all(np.abs(sal - mean) <= 1.6e-5 * mean), np.max(np.abs(sal - mean) / mean)
    ctx.close()


@pytest.mark.parametrize("dh,H", [(64, 4), (128, 2)])
@pytest.mark.parametrize("S,nq,B", [(1027, 33, 1), (2047, 17, 2), (2049, 16, 1), (2559, 32, 1), (2688, 33, 3), (2689, 17, 1)])
def test_long_scoring_rows(dh, H, S, nq, B):
    """Around the last key block of the longest rows that 16 queries a workgroup take, and just beyond them."""
    test_scoring_rows(dh, H, S, nq, B)


@pytest.mark.parametrize("dh,H", [(64, 4), (128, 2)])
@pytest.mark.parametrize("S,nq,B", [(17, 16, 3), (80, 33, 2), (112, 16, 1), (127, 17, 2), (128, 1, 2), (128, 64, 1), (129, 16, 2)])
def test_short_scoring_rows(dh, H, S, nq, B):
    """Up to 128 keys a wave has one block of them and no second one to fetch."""
    test_scoring_rows(dh, H, S, nq, B)
    wl = replace(W.WORKLOADS["tiny"], D=H * dh, H=H, dh=dh, F=256, n2=S - nq, n3=0, nt=nq, B=B, L=1, p=0)
    ctx = mv.Context(B, S, wl.D, H, wl.F, nq)
    packed, ws = device_layer(ctx, wl, W.layer_weights(wl, 0))
    x, pos = W.hidden_states(wl, device="cuda")
    torch.cuda.synchronize()
    with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CUDA]) as prof:
        ctx.score_only(layer_cfg(wl), ws, x, pos, nq)
        torch.cuda.synchronize()
    (blocks,) = [int(m.group(1)) for e in prof.events() for m in [re.search(r"rows16_kernel<\d+, 8, (\d+)", e.name)] if m]
    assert blocks == (1 if S <= 128 else 2)
    ctx.close()


@pytest.mark.parametrize("dh,H", [(64, 4), (128, 2)])
@pytest.mark.parametrize("S,nq,B", [(2689, 33, 3), (2720, 64, 2)])
def test_two_passes_over_the_keys(dh, H, S, nq, B):
    """Beyond 2688 keys, with several samples and tiles of 32 queries (the offsets of both)."""
    test_scoring_rows(dh, H, S, nq, B)
    wl = replace(W.WORKLOADS["tiny"], D=H * dh, H=H, dh=dh, F=256, n2=S - nq, n3=0, nt=nq, B=B, L=1, p=0)
    ctx = mv.Context(B, S, wl.D, H, wl.F, nq)
    packed, ws = device_layer(ctx, wl, W.layer_weights(wl, 0))
    x, pos = W.hidden_states(wl, device="cuda")
    torch.cuda.synchronize()
    with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CUDA]) as prof:
        ctx.score_only(layer_cfg(wl), ws, x, pos, nq)
        ctx.prefill_layer_salience(layer_cfg(wl), ws, x, pos, nq, S - nq)
        torch.cuda.synchronize()
    names = [e.name for e in prof.events() if "mvla::score_probs" in e.name]
    assert len(names) == 2 and all("score_probs_kernel<" in n for n in names), names
    ctx.close()
