"""Selection and fused pruning at the sizes where their kernels change path: segments of one wave
(ranked directly), segments around the four- / sixteen-wave limit, keys that agree in all but their
last bits (one histogram of single key values), thresholds that take one to four histograms, the fused step with few and many rows and columns.  Selection is compared with the oracle exactly; the fused step with the
four single calls exactly (same order of additions, same selection)."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2604_09244_amd import binding as mv

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = mv.Context(4, 32768 + 8, 64, 4, 64, 160)
    yield c
    c.close()


def _scores(kind, shape, r):
    if kind == "lognormal":
        return r.lognormal(size=shape).astype(np.float32)
    if kind == "last bits":        # 1 + i * 2^-23 for few i: thousands of equal keys per value
        return (1.0 + r.integers(0, 5, size=shape) * 2.0 ** -23).astype(np.float32)
    if kind == "all equal":
        return np.full(shape, 0.25, np.float32)
    # both signs over the whole exponent range, and both zeros
    s = (np.sign(r.normal(size=shape)) * np.exp(r.uniform(-80, 80, size=shape))).astype(np.float32)
    return np.where(r.uniform(size=shape) < 0.2, np.float32(-0.0), s).astype(np.float32)


@pytest.mark.parametrize("kind", ["lognormal", "last bits", "all equal", "wide"])
@pytest.mark.parametrize("n2,n3", [(1, 0), (64, 64), (64, 65), (65, 1), (2048, 2047), (2049, 63), (16384, 16384)])
def test_select_paths(ctx, n2, n3, kind):
    r = np.random.default_rng(n2 * 31 + n3)
    B, n = 2, n2 + n3
    s = _scores(kind, (B, n), r)
    for K in sorted({0, 1, n // 7, n // 2, n - 1, n}):
        k2 = r.integers(max(0, K - n3), min(n2, K) + 1, size=B)
        k2k3 = np.stack([k2, K - k2], 1).astype(np.int32)
        got = ctx.select_topk(torch.from_numpy(s).cuda(), torch.from_numpy(k2k3).cuda(), n2, n3, 3, K)
        assert np.array_equal(got.cpu().numpy(), O.select_topk(s, k2k3, n2, n3, 3)), (n2, n3, kind, K)


def _rounds(s, k):
    """Histograms that the search for the k-th largest score takes: 1024 bins over the keys' range, then over
    the bin that holds the threshold, until it holds at most 64 keys or is one key value."""
    u = s.view(np.uint32).astype(np.int64)
    keys = np.where(u >> 31, 0xFFFFFFFF - u, u + 0x80000000)
    lo, hi, n = int(keys.min()), int(keys.max()), 0
    t = int(np.sort(keys)[len(keys) - k])
    while True:
        n += 1
        shift = max(0, (hi - lo).bit_length() - 10)
        b = (t - lo) >> shift
        lo, hi = lo + (b << shift), min(hi, lo + ((b + 1) << shift) - 1)
        if shift == 0 or np.sum((keys >= lo) & (keys <= hi)) <= 64:
            return n


@pytest.mark.parametrize("n", [1200, 5000])          # four waves, sixteen
def test_select_takes_every_number_of_histograms(ctx, n):
    """Scores between two outliers, crowded around 1 in ever narrower bands: most of a bin's keys lie in
    one bin of the next histogram."""
    r = np.random.default_rng(n)
    bands = np.concatenate([r.integers(0, w, size=n // 6) for w in (4, 4, 1 << 9, 1 << 17)]).astype(np.uint32)
    s = np.concatenate([[-3e38, 3e38], r.uniform(2, 1e30, size=n - 2 - len(bands))]).astype(np.float32)
    s = r.permutation(np.concatenate([s, (bands + np.uint32(0x3F800000)).view(np.float32)]))
    took = set()
    for k in [1, 2, n // 6, n // 3, n // 2, *range(n // 3 + 20, n, n // 37), n - 1]:
        took.add(_rounds(s, k))
        k2k3 = np.array([[k, 0]], np.int32)
        got = ctx.select_topk(torch.from_numpy(s[None]).cuda(), torch.from_numpy(k2k3).cuda(), n, 0, 0, k)
        assert np.array_equal(got.cpu().numpy(), O.select_topk(s[None], k2k3, n, 0, 0)), k
    assert took == {1, 2, 3, 4}, took


# H * Nq rows x columns: up to 128 rows are one split, more are several
@pytest.mark.parametrize("H,Nq,n2,n3,nt", [(4, 16, 64, 64, 16), (4, 16, 64, 65, 16), (4, 32, 32, 32, 32), (4, 33, 30, 30, 33),
                                           (4, 32, 64, 65, 32), (1, 8, 512, 512, 8), (1, 7, 513, 512, 7),
                                           (4, 8, 256, 256, 32), (2, 8, 3, 700, 9), (4, 160, 300, 700, 160)])
def test_fused_step_equals_single_calls(ctx, H, Nq, n2, n3, nt):
    B, D, S = 3, 64, n2 + n3 + nt
    g = torch.Generator().manual_seed(H * 1000 + S)
    p = torch.rand(B, H, Nq, S, generator=g) ** 4
    p = (p / p.sum(-1, keepdim=True)).cuda()
    h = torch.randn(B, S, D, generator=g).to(torch.bfloat16).cuda()
    pos = torch.arange(S, dtype=torch.int32).repeat(B, 1).cuda()
    K = (n2 + n3) * 2 // 5
    o = ctx.prune_step(p, h, pos, n2, n3, nt, K)
    sal = ctx.salience(p, n2 + n3)
    k2k3 = ctx.modality_budget(sal, n2, n3, K)
    kept = ctx.select_topk(sal, k2k3, n2, n3, nt, K)
    hk, pk = ctx.compact(h, pos, kept)
    ref = O.salience(p.cpu().numpy().astype(np.float64), n2 + n3)
    # a column sum of H*Nq fp32 values: at most (H*Nq) * 2^-24 relative, far less in groups of 16
    assert np.max(np.abs(sal.cpu().numpy() - ref) / ref) < H * Nq * 2.0 ** -24
    for a, b in ((o["sal"], sal), (o["k2k3"], k2k3), (o["kept_idx"], kept), (o["h"], hk), (o["pos"], pk)):
        assert torch.equal(a, b)


@pytest.mark.parametrize("B,H,Nq,P,nt", [(4, 32, 32, 256, 32), (2, 32, 33, 20, 4), (1, 4, 256, 17, 3), (3, 4, 257, 16, 0),
                                         (2, 4, 260, 18, 2), (1, 1, 1, 1, 0), (2, 3, 5, 50, 1)])
def test_decompose_paths(ctx, B, H, Nq, P, nt):
    """Per-patch indicators with rows kept in registers (up to 1024) and read twice, aligned and not,
    patches that end inside a workgroup."""
    S = 2 * P + nt
    g = torch.Generator().manual_seed(B * 1000 + P)
    p = torch.rand(B, H, Nq, S, generator=g) ** 4
    p = (p / p.sum(-1, keepdim=True)).contiguous()
    m2, m3 = ctx.modality_decompose(p.cuda(), P)
    r2, r3 = O.modality_decompose(p.numpy().astype(np.float64), P)
    # sums of H*Nq fp32 values in groups of at most 16 a thread: well inside 1e-5 relative
    for got, ref in ((m2, r2), (m3, r3)):
        assert np.max(np.abs(got.cpu().numpy() - ref)) <= 1e-5 * max(1.0, float(np.max(ref)))


@pytest.mark.parametrize("P,nt", [(20, 4), (21, 2)])       # 16 bytes a lane, and 4
@pytest.mark.parametrize("R", [1, 15, 16, 17, 255, 256, 257, 511, 512, 513, 1023, 1025])
def test_decompose_row_limits(R, P, nt):
    """Row counts around the limits of the workgroup sizes, a row of one value among them."""
    B, S = 2, 2 * P + nt
    g = torch.Generator().manual_seed(R * 100 + P)
    p = torch.rand(B, 1, R, S, generator=g) ** 4
    p = (p / p.sum(-1, keepdim=True)).contiguous()
    ctx = mv.Context(B, S, 64, 1, 64, R)
    m2, m3 = ctx.modality_decompose(p.cuda(), P)
    r2, r3 = O.modality_decompose(p.numpy().astype(np.float64), P)
    # sums of R fp32 values, at most 64 a thread: inside 1e-5 relative
    for got, ref in ((m2, r2), (m3, r3)):
        assert np.max(np.abs(got.cpu().numpy() - ref)) <= 1e-5 * max(1.0, float(np.max(ref)))
    ctx.close()


@pytest.mark.parametrize("R,P", [(5, 20), (300, 20), (300, 21), (900, 20), (900, 21)])
def test_decompose_overflowed_coefficient(R, P):
    """<a2,a3>/<a2,a2> beyond fp32: every row's rest is infinite and so is the share.  Rows that a thread
    keeps room for and that do not exist must not turn it into NaN."""
    ctx = mv.Context(1, 2 * P, 64, 1, 64, R)
    p = torch.empty(1, 1, R, 2 * P, device="cuda")
    p[..., :P], p[..., P:] = 1e-19, 1e21               # squares 1e-38, coefficient 1e40, products finite
    m2, m3 = ctx.modality_decompose(p, P)
    assert (m2 < 1e-30).all() and torch.isposinf(m3).all(), (m2, m3)
    ctx.close()
