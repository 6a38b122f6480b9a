"""The projection tiles that are fitted to the row count (configurations 12 to 23 of the choice by size): every one of
them with every epilogue that the prediction gives it at these sizes (by the names of the kernels that ran), rows
and columns that end inside a tile, heads of 64 and 128, tile widths that heads of 64 divide and the q/k/v borders
fall between, V^T token by token and in whole groups of eight.  Against the oracle layer."""
import re
from dataclasses import replace

import pytest
import torch

from helpers import EPI_DOWN, EPI_GATEUP, EPI_OUT, EPI_QKV, check_layer, device_layer, layer_cfg, oracle_weights, to64
from paper_2604_09244_amd import binding as mv
from paper_2604_09244_amd import workloads as W

pytestmark = pytest.mark.gpu
SHAPES = {12: (160, 128), 13: (192, 128), 14: (160, 192), 15: (256, 128), 16: (128, 256), 17: (192, 192), 18: (160, 256),
          19: (224, 192), 20: (192, 256), 21: (288, 192), 22: (224, 256), 23: (320, 192)}


def fitted_launches(fn):
    """{epilogue: (rows, columns) of the tile} of the fitted kernels that fn launched."""
    torch.cuda.synchronize()
    with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CUDA]) as prof:
        fn()
        torch.cuda.synchronize()
    names = [re.search(r"fitted_tile_kernel<(\d+), (\d+), 64, 2, 2, \d, (\d)>", e.name) for e in prof.events()]
    return {int(m.group(3)): (int(m.group(1)), int(m.group(2))) for m in names if m}


@pytest.mark.parametrize("D,H,F,B,S,expect", [
    (1280, 20, 1600, 11, 291, {EPI_QKV: 20, EPI_OUT: 12, EPI_DOWN: 12, EPI_GATEUP: 19}),
    (1344, 21, 1600, 11, 339, {EPI_QKV: 23, EPI_OUT: 13, EPI_DOWN: 13, EPI_GATEUP: 21}),
    (1024, 16, 1600, 11, 563, {EPI_QKV: 18, EPI_OUT: 16, EPI_DOWN: 16, EPI_GATEUP: 18}),
    (1152, 9, 1600, 11, 611, {EPI_QKV: 15, EPI_OUT: 15, EPI_DOWN: 15, EPI_GATEUP: 20}),
    (1024, 16, 1600, 11, 771, {EPI_QKV: 22, EPI_OUT: 18, EPI_DOWN: 18, EPI_GATEUP: 22}),
    (1280, 20, 2816, 11, 99, {EPI_QKV: 12, EPI_GATEUP: 14}),
    (1536, 24, 1600, 11, 120, {EPI_QKV: 13, EPI_GATEUP: 12}),
    (1024, 16, 1600, 11, 227, {EPI_QKV: 16, EPI_GATEUP: 15}),
    (1344, 21, 1600, 11, 451, {EPI_QKV: 19, EPI_OUT: 16, EPI_DOWN: 14, EPI_GATEUP: 16}),
    (1152, 18, 1600, 11, 243, {EPI_QKV: 17, EPI_GATEUP: 17}),
    (1152, 18, 704, 11, 744, {EPI_QKV: 23, EPI_OUT: 19, EPI_GATEUP: 13}),
    (1152, 18, 64, 11, 163, {EPI_QKV: 14}),
    (1152, 18, 1600, 11, 659, {EPI_OUT: 17, EPI_DOWN: 17, EPI_GATEUP: 20}),
    (1280, 20, 1600, 11, 744, {EPI_OUT: 20, EPI_DOWN: 20, EPI_GATEUP: 21}),
    (1536, 24, 1600, 11, 755, {EPI_OUT: 22, EPI_DOWN: 22, EPI_GATEUP: 21}),
    (1152, 18, 64, 11, 595, {EPI_OUT: 14}),
    (1792, 28, 4160, 7, 227, {EPI_QKV: 18, EPI_GATEUP: 23}),
    (1152, 18, 2816, 11, 744, {EPI_QKV: 23, EPI_OUT: 19, EPI_DOWN: 19}),
    (1344, 21, 1600, 11, 900, {EPI_OUT: 21}),
    (4096, 32, 1024, 8, 394, {EPI_OUT: 21}),
    (1152, 18, 2816, 11, 1205, {EPI_OUT: 23, EPI_DOWN: 23}),
    (1344, 21, 2816, 11, 739, {EPI_OUT: 13, EPI_DOWN: 21})])
def test_fitted_tiles(D, H, F, B, S, expect):
    wl = replace(W.WORKLOADS["tiny"], D=D, H=H, dh=D // H, F=F, n2=S // 2, n3=S - S // 2, nt=0, B=B, seed=D + S)
    ctx = mv.Context(B, S, D, H, F, 0)
    w_cpu = W.layer_weights(wl, 0)
    packed, struct = device_layer(ctx, wl, w_cpu)
    ow = oracle_weights(w_cpu)
    x, pos = W.hidden_states(wl, device="cuda")
    y = ctx.prefill_layer(layer_cfg(wl), struct, x, pos)
    again = torch.empty_like(y)
    ran = fitted_launches(lambda: ctx.prefill_layer(layer_cfg(wl), struct, x, pos, again))
    assert {e: SHAPES[c] for e, c in expect.items()}.items() <= ran.items(), ran
    assert torch.equal(y, again)
    for b in (0, B - 1):
        check_layer(y[b], to64(x[b]), pos[b].cpu().numpy(), ow, wl, f"D={D} F={F} B={B} S={S} sample {b}")
    ctx.close()
