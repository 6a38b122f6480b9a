"""The small whole-tile projection kernels (64x64, 64x128, 128x64, 128x128 on four waves, 128x192), which
only the choice by size uses: layers with rows and columns that end inside a tile, one to 44 slabs, heads of
64 and 128, V^T stored in whole groups of eight tokens and token by token, every configuration with every
epilogue and every configuration of the paired projections among them (by the names of the kernels that ran).
Against the oracle at the stated bar."""
from dataclasses import replace

import pytest
import torch

import oracle as O
from helpers import (EPI_DOWN, EPI_GATEUP, EPI_OUT, EPI_QKV, assert_layer_close, device_layer, layer_cfg,
                     oracle_weights, projection_launches, to64)
from paper_2604_09244_amd import binding as mv
from paper_2604_09244_amd import workloads as W
from test_gpu_layer import PROBS_ATOL, PROBS_RTOL

pytestmark = pytest.mark.gpu
EPI_QKV_ROPE = 0


@pytest.mark.parametrize("D,H,F", [(256, 4, 1024), (256, 2, 192), (192, 3, 64), (1024, 8, 2816), (1024, 16, 704)])
@pytest.mark.parametrize("B,S", [(1, 1), (1, 65), (3, 79), (2, 136), (4, 435)])
def test_small_tiles(D, H, F, B, S):
    wl = replace(W.WORKLOADS["tiny"], D=D, H=H, dh=D // H, F=F, n2=S // 2, n3=S - S // 2, nt=0, B=B, seed=D + S)
    ctx = mv.Context(B, S, D, H, F, 0)
    w_cpu = W.layer_weights(wl, 0)
    packed, struct = device_layer(ctx, wl, w_cpu)
    ow = oracle_weights(w_cpu)
    x, pos = W.hidden_states(wl, device="cuda")
    y = ctx.prefill_layer(layer_cfg(wl), struct, x, pos)
    again = ctx.prefill_layer(layer_cfg(wl), struct, x, pos)
    torch.cuda.synchronize()
    for b in range(B):
        ref = O.decoder_layer(to64(x[b]), pos[b].cpu().numpy(), ow, H, wl.rms_eps, wl.rope_base)[0]
        assert_layer_close(y[b], ref, f"D={D} F={F} B={B} S={S} sample {b}", D)
    assert torch.equal(y, again)
    ctx.close()


@pytest.mark.parametrize("D,H", [(256, 4), (192, 3), (1024, 8)])
@pytest.mark.parametrize("B,S,nt", [(1, 9, 1), (1, 66, 33), (3, 201, 7), (2, 520, 65)])
def test_paired_projections(D, H, B, S, nt):
    """Scoring pass with the key and the query projection in one launch, and (a choice recorded) in two:
    both against the oracle at the bar of the layer's own scoring rows."""
    wl = replace(W.WORKLOADS["tiny"], D=D, H=H, dh=D // H, F=64, n2=(S - nt) // 2, n3=S - nt - (S - nt) // 2,
                 nt=nt, B=B, seed=D + S)
    w_cpu = W.layer_weights(wl, 0)
    ow = oracle_weights(w_cpu)
    x, pos = W.hidden_states(wl, device="cuda")
    for paired in (True, False):
        ctx = mv.Context(B, S, D, H, 64, nt)
        packed, struct = device_layer(ctx, wl, w_cpu)
        if not paired:
            ctx.set_gemm_choice(B * S, D, D, EPI_QKV_ROPE, 3, 0)
        ctx.profile_enable(None)
        probs = ctx.score_only(layer_cfg(wl), struct, x, pos, nt)
        launches = [name for name, _, _ in ctx.profile_read()]
        ctx.profile_enable([])
        again = ctx.score_only(layer_cfg(wl), struct, x, pos, nt)
        torch.cuda.synchronize()
        assert launches.count("gemm_qkv") == (1 if paired else 2), launches
        assert torch.equal(probs, again)
        for b in range(B):
            ref = O.score_only(to64(x[b]), pos[b].cpu().numpy(), ow, H, nt, wl.rms_eps, wl.rope_base)
            assert (abs(to64(probs[b]) - ref) <= PROBS_RTOL * abs(ref) + PROBS_ATOL).all(), f"sample {b}"
        ctx.close()


# configurations 7 .. 11 with each of the four epilogues, at sizes where the prediction picks them
@pytest.mark.parametrize("D,H,F,B,S,expect", [
    (64, 1, 64, 1, 33, {EPI_QKV: 8, EPI_OUT: 8, EPI_DOWN: 10, EPI_GATEUP: 8}),
    (128, 1, 64, 1, 33, {EPI_QKV: 10}),
    (64, 1, 2816, 1, 130, {EPI_DOWN: 8, EPI_GATEUP: 10}),
    (448, 7, 2816, 1, 130, {EPI_GATEUP: 11}),
    (576, 9, 320, 3, 201, {EPI_QKV: 11}),
    (576, 9, 64, 3, 399, {EPI_QKV: 7}),
    (256, 2, 2816, 3, 299, {EPI_GATEUP: 7}),
    (256, 2, 2112, 3, 259, {EPI_GATEUP: 9}),
    (384, 3, 192, 3, 901, {EPI_QKV: 9, EPI_OUT: 10}),
    (768, 6, 192, 3, 1001, {EPI_OUT: 9, EPI_DOWN: 9}),
    (896, 7, 1600, 3, 401, {EPI_OUT: 11, EPI_DOWN: 11}),
    (896, 7, 192, 3, 1667, {EPI_OUT: 7, EPI_DOWN: 7})])
def test_every_small_tile_with_every_epilogue(D, H, F, B, S, expect):
    wl = replace(W.WORKLOADS["tiny"], D=D, H=H, dh=D // H, F=F, n2=S // 2, n3=S - S // 2, nt=0, B=B, seed=D + S)
    ctx = mv.Context(B, S, D, H, F, 0)
    w_cpu = W.layer_weights(wl, 0)
    packed, struct = device_layer(ctx, wl, w_cpu)
    ow = oracle_weights(w_cpu)
    x, pos = W.hidden_states(wl, device="cuda")
    y = ctx.prefill_layer(layer_cfg(wl), struct, x, pos)
    again = torch.empty_like(y)
    ran = projection_launches(lambda: ctx.prefill_layer(layer_cfg(wl), struct, x, pos, again))
    assert len(ran) == 4 and expect.items() <= dict(ran).items(), ran
    for b in (0, B - 1):
        ref = O.decoder_layer(to64(x[b]), pos[b].cpu().numpy(), ow, H, wl.rms_eps, wl.rope_base)[0]
        assert_layer_close(y[b], ref, f"D={D} F={F} B={B} S={S} sample {b}", D)
    assert torch.equal(y, again)
    ctx.close()


@pytest.mark.parametrize("D,H,B,S,nt,config", [(640, 5, 15, 622, 33, 1), (640, 5, 14, 430, 33, 5), (64, 1, 1, 33, 33, 8),
                                               (1024, 8, 15, 75, 64, 9), (128, 1, 1, 33, 33, 10), (1024, 16, 16, 33, 33, 11)])
def test_every_configuration_of_the_paired_projections(D, H, B, S, nt, config):
    wl = replace(W.WORKLOADS["tiny"], D=D, H=H, dh=D // H, F=64, n2=(S - nt) // 2, n3=S - nt - (S - nt) // 2,
                 nt=nt, B=B, seed=D + S)
    w_cpu = W.layer_weights(wl, 0)
    ow = oracle_weights(w_cpu)
    x, pos = W.hidden_states(wl, device="cuda")
    ctx = mv.Context(B, S, D, H, 64, nt)
    packed, struct = device_layer(ctx, wl, w_cpu)
    probs = ctx.score_only(layer_cfg(wl), struct, x, pos, nt)
    again = torch.empty_like(probs)
    ran = projection_launches(lambda: ctx.score_only(layer_cfg(wl), struct, x, pos, nt, None, again))
    assert ran == [(EPI_QKV, config)], ran
    assert torch.equal(probs, again)
    for b in (0, B - 1):
        ref = O.score_only(to64(x[b]), pos[b].cpu().numpy(), ow, H, nt, wl.rms_eps, wl.rope_base)
        assert (abs(to64(probs[b]) - ref) <= PROBS_RTOL * abs(ref) + PROBS_ATOL).all(), f"sample {b}"
    ctx.close()


@pytest.mark.parametrize("D,H,norms", [(64, 1, 1), (320, 5, 1), (384, 3, 1), (448, 7, 2)])
@pytest.mark.parametrize("B,S", [(1, 1), (1, 63), (2, 33)])
def test_rows_normalised_by_the_projection(D, H, norms, B, S):
    """Gate/up rows of up to 384 values: one to six slabs, rows that end inside the tile, and the first length beyond."""
    wl = replace(W.WORKLOADS["tiny"], D=D, H=H, dh=D // H, F=192, n2=S // 2, n3=S - S // 2, nt=0, B=B, seed=D + S)
    ctx = mv.Context(B, S, D, H, 192, 0)
    w_cpu = W.layer_weights(wl, 0)
    packed, struct = device_layer(ctx, wl, w_cpu)
    x, pos = W.hidden_states(wl, device="cuda")
    y = ctx.prefill_layer(layer_cfg(wl), struct, x, pos)
    torch.cuda.synchronize()
    with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CUDA]) as prof:
        ctx.prefill_layer(layer_cfg(wl), struct, x, pos)
        torch.cuda.synchronize()
    assert sum("rmsnorm" in e.name for e in prof.events()) == norms
    for b in range(B):
        ref = O.decoder_layer(to64(x[b]), pos[b].cpu().numpy(), oracle_weights(w_cpu), H, wl.rms_eps, wl.rope_base)[0]
        assert_layer_close(y[b], ref, f"D={D} B={B} S={S} sample {b}", D)
    ctx.close()
