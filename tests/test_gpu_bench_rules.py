"""The rules by which bench.py counts bytes against the kernels that run: queries a workgroup of the scoring kernel, and
whether the gather writes the next norm."""
from dataclasses import replace

import pytest
import torch

import bench
from helpers import device_layer, layer_cfg
from paper_2604_09244_amd import binding as mv
from paper_2604_09244_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,S,nq", [(1, 144, 17), (33, 256, 64), (32, 256, 64), (8, 544, 32), (32, 544, 32), (33, 544, 32),
                                    (65, 544, 16), (1, 1024, 64), (1, 1025, 16)])
@pytest.mark.parametrize("sums", [True, False])
def test_score_tile(B, S, nq, sums):
    wl = replace(W.WORKLOADS["tiny"], D=256, H=4, dh=64, F=256, n2=S - nq - 8, n3=8, nt=nq, B=B, L=1, p=0)
    ctx = mv.Context(B, S, wl.D, wl.H, wl.F, nq)
    packed, ws = device_layer(ctx, wl, W.layer_weights(wl, 0))
    x, pos = W.hidden_states(wl, device="cuda")

    def layer():
        if sums:
            ctx.prefill_layer_salience(layer_cfg(wl), ws, x, pos, nq, S - nq)
        else:
            ctx.prefill_layer(layer_cfg(wl), ws, x, pos, n_query_tail=nq)

    layer()
    torch.cuda.synchronize()
    with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CUDA]) as prof:
        layer()
        torch.cuda.synchronize()
    names = [e.name for e in prof.events() if "score_probs" in e.name]
    assert len(names) == 1
    assert ("rows16" in names[0]) == (bench.score_tile(B, wl.H, S, nq, sums) == 16), names
    ctx.close()


@pytest.mark.parametrize("B,S,nq", [(17, 2048, 64), (17, 2049, 64), (17, 2688, 64), (17, 2689, 64), (1, 2689, 16)])
@pytest.mark.parametrize("sums", [True, False])
def test_score_tile_of_many_workgroups(B, S, nq, sums):
    """Two lines that a number of workgroups up to one per compute unit does not show: what 32 queries keep in registers
    (2048 keys), and what 16 do (2688)."""
    test_score_tile(B, S, nq, sums)


@pytest.mark.parametrize("D,K", [(256, 33), (4096, 1021), (4096, 1022)])
def test_gather_writes_norm(D, K):
    wl = replace(W.WORKLOADS["tiny"], D=D, H=D // 128, dh=128, F=64, n2=600, n3=500, nt=3, B=1, L=1, p=0)
    ctx = mv.Context(1, wl.S, D, wl.H, 64, wl.nt)
    plan = mv.PrefillPlan(ctx, layer_cfg(wl), [mv.pack_layer(W.layer_weights(wl, 0, device="cuda"))], 1, wl.n2, wl.n3,
                          wl.nt, K, 0)
    x, pos = W.hidden_states(wl, device="cuda")
    ctx.profile_enable(None)
    plan.run(x, pos)
    norms = [name for name, _, _ in ctx.profile_read()].count("rmsnorm")     # (one is the scoring pass's)
    assert norms == (1 if bench.gather_writes_norm(K + wl.nt, D) else 2)
    ctx.close()
