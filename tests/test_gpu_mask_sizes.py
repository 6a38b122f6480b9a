"""Mask generation and index scan at the sizes where the workgroup changes: patch counts on both sides of every sorted
variant's limit, scores with wide exponents, negative, tied and constant ones, one and two assignments only; flag counts
on both sides of every index variant's limit.  Bit-exact against the oracle."""
from dataclasses import replace

import numpy as np
import pytest
import torch

import oracle as O
from paper_2604_09244_amd import binding as mv
from paper_2604_09244_amd import workloads as W

pytestmark = pytest.mark.gpu


def _scores(kind, B, P, seed):
    wl = replace(W.WORKLOADS["single_view"], n2=P, n3=P, seed=seed)
    if kind == "constant":
        return torch.full((B, 2 * P), 0.375)
    s = W.synthetic_salience(wl, B=B, **({"levels": 8} if kind == "ties" else {}))
    if kind == "wide":           # (differences of 2^40 between scores of a sample)
        e = torch.from_numpy(np.random.default_rng(seed).integers(-20, 21, size=(B, 2 * P)))
        s = torch.ldexp(s, e.to(s.dtype))
    if kind == "negative":
        s = s - s.mean()
    return s.to(torch.float32)


@pytest.mark.parametrize("P", [2, 63, 64, 65, 128, 129, 255, 256, 257, 512, 513, 1024, 1025, 2048, 2049, 4096, 4097, 8192, 8193])
@pytest.mark.parametrize("kind", ["heavy", "ties", "constant", "wide", "negative"])
def test_candidate_masks_at_every_size(P, kind):
    B = 2
    ctx = mv.Context(B, 8, 64, 4, 64, 8)
    x_hat = W.synthetic_indicators(W.WORKLOADS["single_view"], B=B, n_patch=P, seed=P)
    sal, u = _scores(kind, B, P, P + 1), W.uniform_draws(replace(W.WORKLOADS["single_view"], n2=P), B=B, step=P)
    for kw in (dict(), dict(max_iter=1), dict(max_iter=2)):
        rules = mv.MaskRules.default(**{{"max_iter": "kmeans_max_iter"}.get(k, k): v for k, v in kw.items()})
        m2, m3, sem, klen = ctx.candidate_masks(x_hat.cuda(), sal.cuda(), u.cuda(), 5, rules)
        ref = O.candidate_masks(x_hat.numpy(), O.patch_score(sal.numpy(), P), u.numpy(), **kw)
        if kind not in ("ties", "constant"):
            assert np.all(ref["kmeans_margin"] > 1e-12)
        assert np.array_equal(sem.cpu().numpy(), ref["sem"])
        assert np.array_equal(m2.cpu().numpy(), ref["mask2d"]) and np.array_equal(m3.cpu().numpy(), ref["mask3d"])
        assert np.array_equal(klen.cpu().numpy(), ref["mask2d"].sum(1).astype(np.int64) + ref["mask3d"].sum(1) + 5)
    ctx.close()


def _labels(score, max_iter):
    """Lloyd's iteration as the header states it, on scores that may be infinite or NaN: a patch changes centre only
    for a smaller distance, NaN is left out of the range."""
    x = score.astype(np.float64)
    lo, hi = np.fmin.reduce(x, initial=np.inf), np.fmax.reduce(x, initial=-np.inf)
    c, label = [lo, 0.5 * (lo + hi), hi], None
    for _ in range(max_iter):
        d = [np.abs(x - v) for v in c]
        one = d[1] < d[0]
        new = np.where(d[2] < np.where(one, d[1], d[0]), 2, one.astype(np.int64))
        if label is not None and np.array_equal(new, label):
            break
        label = new
        c = [x[label == j].sum() / (label == j).sum() if (label == j).any() else c[j] for j in range(3)]
    return label


@pytest.mark.parametrize("P", [2, 64, 65, 256, 257, 512, 1024, 2048, 4096, 8192, 8193])
@pytest.mark.parametrize("values", [(-np.inf,), (np.inf,), (-np.inf, np.inf), (np.nan,), (-np.inf, np.nan)])
@np.errstate(invalid="ignore")
def test_labels_of_scores_that_are_not_finite(P, values):
    """The header calls them invalid input; the labels are the same on both sides of the largest sorted variant."""
    ctx = mv.Context(2, 8, 64, 4, 64, 8)
    x_hat = W.synthetic_indicators(W.WORKLOADS["single_view"], B=2, n_patch=P, seed=P)
    u = W.uniform_draws(replace(W.WORKLOADS["single_view"], n2=P), B=2, step=P)
    sal = _scores("heavy", 2, P, P + 3)
    for i, v in enumerate(values):
        sal[0, (P // 2 + i) % P] = v             # (the second sample stays finite)
    for n in (1, 2, 32):
        sem = ctx.candidate_masks(x_hat.cuda(), sal.cuda(), u.cuda(), 5, mv.MaskRules.default(kmeans_max_iter=n))[2]
        for b in range(2):
            assert np.array_equal(sem[b].cpu().numpy(), _labels(O.patch_score(sal.numpy(), P)[b], n)), (n, b)
    ctx.close()


@pytest.mark.parametrize("P", [1, 32, 33, 127, 128, 129, 255, 256, 257, 511, 1023, 1024, 1025, 4095, 4096, 4097, 16384])
def test_mask_indices_at_every_size(P):
    ctx = mv.Context(3, 8, 64, 4, 64, 8)
    r = np.random.default_rng(P)
    m2, m3 = ((r.uniform(size=(3, P)) < q).astype(np.uint8) * v for q, v in ((0.45, 1), (0.3, 255)))
    m2[1], m3[1], m2[2], m3[2] = 0, 0, 1, 1
    ref = O.mask_indices((m2 != 0).astype(np.uint8), (m3 != 0).astype(np.uint8), 4)
    for S_pad in (2 * P + 4, max(P // 2, 1)):           # (a short row takes what fits)
        got = ctx.mask_indices(torch.from_numpy(m2).cuda(), torch.from_numpy(m3).cuda(), 4, S_pad).cpu().numpy()
        for b in range(3):
            n = min(len(ref[b]), S_pad)
            assert np.array_equal(got[b, :n], ref[b][:n]) and np.all(got[b, n:] == 2 * P + 3)
    ctx.close()
