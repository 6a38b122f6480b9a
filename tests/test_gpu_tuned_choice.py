"""Set-up measurement at row counts where the choice by size takes a tile that cannot be recorded by its own index: the
measurement may keep that choice, launches then run its kernel, and the record can be replayed by hand."""
import re
from dataclasses import replace

import pytest
import torch

from helpers import EPI_GATEUP, EPI_QKV, device_layer, layer_cfg
from paper_2604_09244_amd import binding as mv
from paper_2604_09244_amd import workloads as W

pytestmark = pytest.mark.gpu
BY_SIZE = 7


def _fitted_epilogues(fn):
    torch.cuda.synchronize()
    with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CUDA]) as prof:
        fn()
        torch.cuda.synchronize()
    names = [re.search(r"fitted_tile_kernel<\d+, \d+, 64, 2, 2, \d, (\d)>", e.name) for e in prof.events()]
    return {int(m.group(1)) for m in names if m}


# gate/up on the best recordable configuration and on the fitted tile: 76 and 58 us, 158 and 136 us
@pytest.mark.parametrize("B,S", [(1, 288), (4, 237)])
def test_measurement_keeps_the_choice_by_size_where_it_is_faster(B, S):
    wl = replace(W.WORKLOADS["single_view"], n2=S // 2, n3=S - S // 2, nt=0, B=B)
    M, N, K = B * S, 2 * wl.F, wl.D
    ctx = mv.Context(B, S, wl.D, wl.H, wl.F, 1)
    packed, ws = device_layer(ctx, wl, W.layer_weights(wl, 0))
    x, pos = W.hidden_states(wl, device="cuda")
    cfg = layer_cfg(wl)
    y = torch.empty_like(x)
    assert EPI_GATEUP in _fitted_epilogues(lambda: ctx.prefill_layer(cfg, ws, x, pos, y))
    ctx.tune_layers(cfg, [ws], B, S)
    assert ctx.tuned_choice(M, N, K, EPI_GATEUP) == (BY_SIZE, 0)
    assert EPI_GATEUP in _fitted_epilogues(lambda: ctx.prefill_layer(cfg, ws, x, pos, y))
    ctx.close()


def test_measurement_where_no_recordable_tile_holds_whole_heads():
    """Five heads of 64: none of the recordable tile widths divides a q/k/v section."""
    wl = replace(W.WORKLOADS["tiny"], D=320, H=5, dh=64, F=256, n2=50, n3=50, nt=0)
    ctx = mv.Context(1, 100, wl.D, wl.H, wl.F, 1)
    packed, ws = device_layer(ctx, wl, W.layer_weights(wl, 0))
    x, pos = W.hidden_states(wl, device="cuda")
    y = ctx.prefill_layer(layer_cfg(wl), ws, x, pos).clone()
    ctx.tune_layers(layer_cfg(wl), [ws], 1, 100)
    assert ctx.tuned_choice(100, 3 * wl.D, wl.D, EPI_QKV) == (BY_SIZE, 0)
    again = ctx.prefill_layer(layer_cfg(wl), ws, x, pos)
    # (another order of fp32 sums in the other projections: a bf16 rounding step, a little more next to zero)
    assert torch.all((again.float() - y.float()).abs() <= 2.0 ** -7 * y.float().abs() + 4e-3 * y.float().std())
    ctx.close()


def test_choice_by_size_recorded_by_hand():
    wl = W.WORKLOADS["single_view"]
    ctx = mv.Context(wl.B, wl.S, wl.D, wl.H, wl.F, wl.nt)
    packed, ws = device_layer(ctx, wl, W.layer_weights(wl, 0))
    x, pos = W.hidden_states(wl, device="cuda")
    cfg, M = layer_cfg(wl), wl.B * wl.S
    shapes = [(3 * wl.D, wl.D, 0), (wl.D, wl.D, 1), (wl.D, wl.F, 2), (2 * wl.F, wl.D, 3), (wl.D, wl.D, EPI_QKV)]
    y, probs = ctx.prefill_layer(cfg, ws, x, pos), ctx.score_only(cfg, ws, x, pos, wl.nt)
    for N, K, epi in shapes:
        ctx.set_gemm_choice(M, N, K, epi, BY_SIZE, 50)
        assert ctx.tuned_choice(M, N, K, epi) == (BY_SIZE, 50)
        with pytest.raises(RuntimeError):
            ctx.set_gemm_choice(M, N, K, epi, BY_SIZE + 1, 50)
    assert torch.equal(ctx.prefill_layer(cfg, ws, x, pos), y)
    ctx.profile_enable(None)
    again = ctx.score_only(cfg, ws, x, pos, wl.nt)
    launches = [name for name, _, _ in ctx.profile_read()]
    assert torch.equal(again, probs) and launches.count("gemm_qkv") == 1, launches     # (key and query in one launch)
    ctx.close()


@pytest.mark.parametrize("S", [80, 400])
def test_measurement_counts_the_norm_that_a_choice_needs(S):
    """Gate/up rows of up to 384 values: the choice by size normalises them itself, any other needs the norm's launch, and
    is timed with it.  Whatever is kept, the layer's output is the same but for the order of fp32 sums."""
    wl = replace(W.WORKLOADS["tiny"], n2=S // 2, n3=S - S // 2, nt=0)
    ctx = mv.Context(1, S, wl.D, wl.H, wl.F, 1)
    packed, ws = device_layer(ctx, wl, W.layer_weights(wl, 0))
    x, pos = W.hidden_states(wl, device="cuda")
    cfg = layer_cfg(wl)
    y = ctx.prefill_layer(cfg, ws, x, pos).clone()
    torch.cuda.synchronize()
    with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CUDA]) as prof:
        ctx.tune_layers(cfg, [ws], 1, S)
        torch.cuda.synchronize()
    names = [e.name for e in sorted(prof.events(), key=lambda e: e.time_range.start) if "mvla::" in e.name]
    gateup = [i for i, n in enumerate(names) if re.search(r"(gemm_kernel|tile_kernel)<.*, 3>", n)]
    own = [i for i in gateup if "small_tile_kernel<64, 64," in names[i]]
    assert own and len(own) < len(gateup)
    for i in gateup:
        assert ("rmsnorm" in names[i - 1]) == (i not in own), (names[i - 1], names[i])
    again = ctx.prefill_layer(cfg, ws, x, pos)
    assert torch.all((again.float() - y.float()).abs() <= 2.0 ** -7 * y.float().abs() + 4e-3 * y.float().std())
    ctx.close()
