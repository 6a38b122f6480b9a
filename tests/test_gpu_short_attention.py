"""Attention of short launches (32 queries a workgroup, key tiles dealt out to its waves): a layer against the
oracle at sequence lengths around the edges of the tiles, of the number of waves and of the two lengths at which the
dispatch's limit changes, and at batches on both sides of that limit, for both head dimensions."""
from dataclasses import replace

import pytest
import torch

from helpers import check_layer, device_layer, layer_cfg, oracle_weights, to64
from paper_2604_09244_amd import binding as mv
from paper_2604_09244_amd import workloads as W

pytestmark = pytest.mark.gpu


def _attention_kernels(fn):
    torch.cuda.synchronize()
    with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CUDA]) as prof:
        fn()
        torch.cuda.synchronize()
    return [e.name for e in prof.events() if "attention_kernel" in e.name]


@pytest.mark.parametrize("dh", [64, 128])
@pytest.mark.parametrize("S,limit", [(65, 256), (96, 256), (127, 256), (129, 256), (161, 256), (192, 256), (193, 512),
                                     (257, 512), (511, 512), (512, 0), (545, 0)])
def test_layer_with_short_attention(dh, S, limit):
    limit = limit or (1024 if dh == 64 else 512)
    H = 4
    most = limit // (H * ((S + 31) // 32))       # samples up to which the launch is a short one
    wl = replace(W.WORKLOADS["tiny"], D=H * dh, H=H, dh=dh, F=256, n2=S // 2, n3=S - S // 2, nt=0, B=most + 1, L=1, p=0,
                 seed=S + dh)
    ctx = mv.Context(wl.B, S, wl.D, H, wl.F, 1)
    w_cpu = W.layer_weights(wl, 0)
    packed, ws = device_layer(ctx, wl, w_cpu)
    x, pos = W.hidden_states(wl)
    wo, cfg = oracle_weights(w_cpu), layer_cfg(wl)
    for B in (most, most + 1):
        xb, pb = x[:B].contiguous().cuda(), pos[:B].contiguous().cuda()
        y = ctx.prefill_layer(cfg, ws, xb, pb)
        names = _attention_kernels(lambda: ctx.prefill_layer(cfg, ws, xb, pb, y))
        assert len(names) == 1 and ("short_attention" in names[0]) == (B <= most), names
        for b in {0, B - 1}:
            check_layer(y[b], to64(x[b]), pos[b].numpy(), wo, wl, f"dh={dh} B={B} b={b} S={S}")
    ctx.close()


@pytest.mark.parametrize("dh,H,S", [(128, 4, 1024), (128, 4, 1025), (128, 4, 1344), (128, 4, 2047), (128, 4, 4096),
                                    (128, 1, 8191), (64, 4, 1024), (64, 4, 1344), (64, 4, 2047), (64, 2, 4097),
                                    (64, 1, 8191)])
def test_long_sequences_with_few_heads(dh, H, S):
    """Up to 64 key tiles a wave: its one stage of LDS is written and read again for each."""
    wl = replace(W.WORKLOADS["tiny"], D=H * dh, H=H, dh=dh, F=256, n2=S // 2, n3=S - S // 2, nt=0, B=1, L=1, p=0,
                 seed=S + dh)
    ctx = mv.Context(1, S, wl.D, H, wl.F, 1)
    w_cpu = W.layer_weights(wl, 0)
    packed, ws = device_layer(ctx, wl, w_cpu)
    x, pos = W.hidden_states(wl)
    xd, pd = x.cuda(), pos.cuda()
    y = ctx.prefill_layer(layer_cfg(wl), ws, xd, pd)
    again = torch.empty_like(y)
    names = _attention_kernels(lambda: ctx.prefill_layer(layer_cfg(wl), ws, xd, pd, again))
    assert len(names) == 1 and "short_attention" in names[0], names
    assert torch.equal(y, again)
    check_layer(y[0], to64(x[0]), pos[0].numpy(), oracle_weights(w_cpu), wl, f"dh={dh} H={H} S={S}")
    ctx.close()


def test_up_to_one_tile_stays_with_the_long_kernel():
    wl = replace(W.WORKLOADS["tiny"], n2=32, n3=32, nt=0, seed=5)
    ctx = mv.Context(1, 64, wl.D, wl.H, wl.F, 1)
    packed, ws = device_layer(ctx, wl, W.layer_weights(wl, 0))
    x, pos = (t.cuda() for t in W.hidden_states(wl))
    names = _attention_kernels(lambda: ctx.prefill_layer(layer_cfg(wl), ws, x, pos))
    assert len(names) == 1 and "short_attention" not in names[0], names
    ctx.close()


@pytest.mark.parametrize("dh,H,S,limit", [(128, 4, 544, 544), (128, 8, 703, 703), (128, 4, 900, 704), (128, 4, 1400, 912),
                                          (64, 4, 639, 1024), (64, 4, 640, 1280)])
def test_limit_of_long_chains(dh, H, S, limit):
    """The last batch that takes short chains and the first that does not, where the limit grows with the length."""
    most = limit // (H * ((S + 31) // 32))
    wl = replace(W.WORKLOADS["tiny"], D=H * dh, H=H, dh=dh, F=256, n2=S // 2, n3=S - S // 2, nt=0, B=most + 1, L=1, p=0,
                 seed=S + dh)
    ctx = mv.Context(wl.B, S, wl.D, H, wl.F, 1)
    w_cpu = W.layer_weights(wl, 0)
    packed, ws = device_layer(ctx, wl, w_cpu)
    x, pos = W.hidden_states(wl)
    for B in (most, most + 1):
        xb, pb = x[:B].contiguous().cuda(), pos[:B].contiguous().cuda()
        y = ctx.prefill_layer(layer_cfg(wl), ws, xb, pb)
        names = _attention_kernels(lambda: ctx.prefill_layer(layer_cfg(wl), ws, xb, pb, y))
        assert len(names) == 1 and ("short_attention" in names[0]) == (B <= most), names
        check_layer(y[B - 1], to64(x[B - 1]), pos[B - 1].numpy(), oracle_weights(w_cpu), wl, f"dh={dh} B={B} S={S}")
    ctx.close()


@pytest.mark.parametrize("dh,H,B,S,short", [
    (128, 32, 1, 543, True), (128, 32, 1, 545, True), (128, 32, 1, 600, True), (128, 32, 1, 703, True),
    (128, 32, 1, 705, True), (128, 32, 1, 1024, True), (128, 32, 1, 1025, False), (128, 11, 3, 600, False),
    (128, 8, 4, 672, True), (128, 8, 4, 673, False), (128, 4, 7, 800, True), (128, 4, 7, 801, False),
    (128, 2, 16, 543, True), (128, 2, 16, 545, False), (128, 1, 30, 544, True), (128, 1, 32, 544, False),
    (128, 1, 16, 1408, True), (128, 1, 16, 1409, False), (64, 1, 24, 1696, True), (64, 1, 24, 1697, False),
    (64, 1, 25, 1280, True), (64, 1, 25, 1281, False)])
def test_limit_counts_tiles_and_samples(dh, H, B, S, short):
    """Lengths of one number of tiles go the same way, and the limit falls with the number of samples."""
    wl = replace(W.WORKLOADS["tiny"], D=H * dh, H=H, dh=dh, F=64, n2=S // 2, n3=S - S // 2, nt=0, B=B, L=1, p=0, seed=S + dh)
    ctx = mv.Context(B, S, wl.D, H, wl.F, 1)
    w_cpu = W.layer_weights(wl, 0)
    packed, ws = device_layer(ctx, wl, w_cpu)
    x, pos = W.hidden_states(wl)
    xd, pd = x.cuda(), pos.cuda()
    y = ctx.prefill_layer(layer_cfg(wl), ws, xd, pd)
    names = _attention_kernels(lambda: ctx.prefill_layer(layer_cfg(wl), ws, xd, pd, y))
    assert len(names) == 1 and ("short_attention" in names[0]) == short, names
    if H <= 4:
        check_layer(y[B - 1], to64(x[B - 1]), pos[B - 1].numpy(), oracle_weights(w_cpu), wl, f"dh={dh} H={H} B={B} S={S}")
    ctx.close()
