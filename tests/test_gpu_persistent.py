"""The persistent projection kernel (tile configuration 4) with more tiles than compute units, so that
its stream of loads crosses tile borders: one, three, four, five and eleven slabs a tile, heads of 64 and
128, V^T stored by whole groups of eight tokens (S % 8 == 0) and token by token (S odd), row and column
counts that end inside a tile, the last round whole, cut into quarters and cut along K (the last two run
on other configurations, in a second launch).  Against the oracle layer on the first and the last sample."""
from dataclasses import replace

import pytest
import torch

import oracle as O
from helpers import (EPI_DOWN, EPI_GATEUP, EPI_OUT, EPI_QKV, assert_layer_close, check_layer, device_layer,
                     layer_cfg, oracle_weights, projection_launches, to64)
from paper_2604_09244_amd import binding as mv
from paper_2604_09244_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,H,F,B,S", [(256, 4, 704, 16, 1605), (256, 2, 320, 17, 1520),
                                       (192, 3, 704, 8, 1601), (1024, 8, 64, 13, 1290), (256, 4, 64, 3000, 9)])
def test_persistent_projections(D, H, F, B, S):
    wl = replace(W.WORKLOADS["tiny"], D=D, H=H, dh=D // H, F=F, n2=S // 2, n3=S - S // 2, nt=0, B=B, seed=D + S)
    ctx = mv.Context(B, S, D, H, F, 0)
    w_cpu = W.layer_weights(wl, 0)
    packed, struct = device_layer(ctx, wl, w_cpu)
    ow = oracle_weights(w_cpu)
    x, pos = W.hidden_states(wl, device="cuda")
    refs = {b: O.decoder_layer(to64(x[b]), pos[b].cpu().numpy(), ow, H, wl.rms_eps, wl.rope_base)[0]
            for b in (0, B - 1)}
    for split_pct in (0, 101):
        for N, K, epi in [(3 * D, D, 0), (D, D, 1), (D, F, 2), (2 * F, D, 3)]:
            ctx.set_gemm_choice(B * S, N, K, epi, 4, split_pct)
        y = ctx.prefill_layer(layer_cfg(wl), struct, x, pos)
        again = ctx.prefill_layer(layer_cfg(wl), struct, x, pos)
        torch.cuda.synchronize()
        for b, ref in refs.items():
            assert_layer_close(y[b], ref, f"D={D} F={F} S={S} split {split_pct} sample {b}", D)
        assert torch.equal(y, again)
    ctx.close()


# Sizes at which the last round is predicted to be faster along K than in quarters: a little over a quarter,
# a half or three quarters of a round of tiles, and a contraction long enough.
@pytest.mark.parametrize("D,H,F,B,S,split", [(6144, 48, 3072, 8, 511, {EPI_QKV, EPI_OUT, EPI_GATEUP}),
                                             (1024, 8, 11008, 16, 1290, {EPI_DOWN})])
def test_last_round_along_k(D, H, F, B, S, split):
    """The second launch of a projection takes over the tiles of the first's last round: same numbering,
    partial sums and arrival counters of its own."""
    wl = replace(W.WORKLOADS["tiny"], D=D, H=H, dh=D // H, F=F, n2=S // 2, n3=S - S // 2, nt=0, B=B, seed=D + S)
    ctx = mv.Context(B, S, D, H, F, 0)
    w_cpu = W.layer_weights(wl, 0)
    packed, struct = device_layer(ctx, wl, w_cpu)
    ow = oracle_weights(w_cpu)
    x, pos = W.hidden_states(wl, device="cuda")
    for N, K, epi in [(3 * D, D, EPI_QKV), (D, D, EPI_OUT), (D, F, EPI_DOWN), (2 * F, D, EPI_GATEUP)]:
        if epi in split:
            ctx.set_gemm_choice(B * S, N, K, epi, 4, 101)
    y = ctx.prefill_layer(layer_cfg(wl), struct, x, pos)
    again = torch.empty_like(y)
    ran = projection_launches(lambda: ctx.prefill_layer(layer_cfg(wl), struct, x, pos, again))
    for epi in split:
        assert [c for e, c in ran if e == epi] == [4, 0], ran
    for b in (0, B - 1):
        check_layer(y[b], to64(x[b]), pos[b].cpu().numpy(), ow, wl, f"D={D} F={F} B={B} S={S} sample {b}")
    assert torch.equal(y, again)
    ctx.close()
