"""The gather of the kept tokens with the first kept layer's norm in the same launch, at row lengths around
every workgroup size of the norm (one, two and four waves, one to four chunks a thread), ragged row counts, and
beyond the size up to which the two are one launch: a whole prefill against the same steps as separate
calls, bit for bit."""
from dataclasses import replace

import pytest
import torch

from helpers import layer_cfg
from paper_2604_09244_amd import binding as mv
from paper_2604_09244_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,H", [(64, 1), (512, 4), (576, 9), (1024, 16), (1088, 17), (2048, 16), (2112, 33), (4096, 32),
                                 (4160, 65)])
@pytest.mark.parametrize("p,options", [(0, {}), (1, {}), (1, {"on_the_fly": True}), (1, {"fused_prune": False})])
def test_gather_with_the_next_norm(D, H, p, options):
    B, n2, n3, nt, K = (2, 37, 45, 9, 33)
    wl = replace(W.WORKLOADS["tiny"], D=D, H=H, dh=D // H, F=256, n2=n2, n3=n3, nt=nt, B=B, L=p + 1, p=p, seed=D)
    ctx = mv.Context(B, wl.S, D, H, 256, nt)
    packed = [mv.pack_layer(W.layer_weights(wl, l, device="cuda")) for l in range(wl.L)]
    plan = mv.PrefillPlan(ctx, layer_cfg(wl), packed, B, n2, n3, nt, K, p)
    x, pos = W.hidden_states(wl, device="cuda")
    ctx.profile_enable(None)
    y = plan.run(x, pos, None, **options).clone()
    names = [name for name, _, _ in ctx.profile_read()]
    ctx.profile_enable([])
    h = ctx.prefill_layer(layer_cfg(wl), plan.structs[0], x, pos) if p else x
    hk, pk = ctx.compact(h, pos, plan.prune["kept_idx"])
    ref = ctx.prefill_layer(layer_cfg(wl), plan.structs[p], hk, pk)
    assert torch.equal(plan.prune["pos"], pk) and torch.equal(plan.h_kept[0], hk) and torch.equal(y, ref)
    assert names.count("compact") == 1 and names.count("rmsnorm") == 1, names
    ctx.close()


def test_long_gather_keeps_its_own_launch():
    wl = replace(W.WORKLOADS["tiny"], D=4096, H=32, dh=128, F=64, n2=600, n3=500, nt=3, B=1, L=1, p=0, seed=9)
    ctx = mv.Context(1, wl.S, wl.D, wl.H, 64, wl.nt)
    packed = [mv.pack_layer(W.layer_weights(wl, 0, device="cuda"))]
    x, pos = W.hidden_states(wl, device="cuda")
    for K, norms in ((1021, 1), (1022, 2)):          # 1024 rows of 4096 values are the limit
        plan = mv.PrefillPlan(ctx, layer_cfg(wl), packed, 1, wl.n2, wl.n3, wl.nt, K, 0)
        ctx.profile_enable(None)
        y = plan.run(x, pos).clone()
        names = [name for name, _, _ in ctx.profile_read()]
        ctx.profile_enable([])
        assert names.count("rmsnorm") == norms, (K, names)
        hk, pk = ctx.compact(x, pos, plan.prune["kept_idx"])
        assert torch.equal(plan.h_kept[0], hk)
        assert torch.equal(y, ctx.prefill_layer(layer_cfg(wl), plan.structs[0], hk, pk))
    ctx.close()
