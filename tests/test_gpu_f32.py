"""GPU parity of the fp32 path at the edges of its tiles: 32-key tiles, 4 per
pass, 128 groups staged at a time by the assignment, 64 by the attention, 16
rows per batch and 64 indices per window of the ordered sums."""
import numpy as np
import pytest
import torch

from paper_2306_01926_amd import ga, inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    ga.lib()
    return torch.device("cuda:0")


def f64(t):
    return inputs.as_float64(t)


def assert_groups(got, ref):
    bel, cnt, cen = (x.cpu().numpy() for x in got)
    assert np.array_equal(bel, ref["belong"]), f"{(bel != ref['belong']).sum()} assignments differ"
    assert np.array_equal(cnt, ref["count"]), "counts differ"
    assert np.array_equal(cen.view(np.uint32), ref["centroid"].view(np.uint32)), "centroids differ"


CASES = [
    # B, H, n, N, iters, widen: the certification bound (65536: every key takes the exact decision)
    (1, 1, 1, 1, 1, None),
    (1, 2, 33, 33, 3, None),        # N = n, one ragged tile and block
    (1, 1, 127, 32, 2, None),       # just below a pass
    (1, 1, 700, 128, 3, None),      # exactly one staged chunk
    (2, 1, 700, 129, 3, None),      # a second chunk of one group
    (1, 1, 1300, 1024, 2, None),    # largest N
    (1, 1, 4000, 3, 3, None),       # groups of more than a thousand members
    (4, 8, 4000, 40, 2, None),      # several passes per workgroup
    (1, 2, 900, 200, 2, "65536"),
    (1, 1, 333, 20, 3, "65536"),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(map(str, c)))
def test_cluster_f32_bit_exact(oracle_mod, dev, case, monkeypatch):
    B, H, n, N, iters, widen = case
    if widen:
        monkeypatch.setenv("GA_CERT_WIDEN", widen)
    print(f"\n[case] cluster f32 {case}", flush=True)
    _, K, _ = inputs.make_qkv(B, H, n, 64, "f32", 70 + n + N, max(4, N // 2), 0.05, 0.3)
    got = ga.cluster(K.to(dev), N, iters)
    torch.cuda.synchronize()
    assert_groups(got, oracle_mod.cluster(f64(K), N, iters, "f32"))


def test_cluster_f32_ties_and_scales(oracle_mod, dev):
    """Exact ties (repeated keys and a repeated initial centroid: the lowest
    index wins) and keys near 1e18 and 1e-18, where fp32 scores stay normal but
    |r|^2 does not bound them from below."""
    print("\n[case] cluster f32, ties and scales", flush=True)
    rng = np.random.default_rng(4)
    K = np.repeat(rng.standard_normal((1, 3, 50, 64)).astype(np.float32), 8, axis=2)
    K[0, 1] *= np.float32(1e18)
    K[0, 2] *= np.float32(1e-18)
    init = np.ascontiguousarray(K[:, :, 5:405:8][:, :, :40])
    init[:, :, 20:30] = init[:, :, 0:10]
    Kt, it = torch.from_numpy(K), torch.from_numpy(init)
    got = ga.cluster(Kt.to(dev), 40, 3, init=it.to(dev))
    torch.cuda.synchronize()
    assert_groups(got, oracle_mod.cluster(f64(Kt), 40, 3, "f32", init=init))


def launched(f):
    ga.timing_enable(True)
    try:
        r = f()
        torch.cuda.synchronize()
    finally:
        ga.timing_enable(False)
        names = ga.timing_collect()
    return r, names


@pytest.mark.parametrize("B,H,n,N,sort", [(4, 8, 2000, 499, False), (4, 8, 2003, 500, True), (2, 4, 4500, 1000, True),
                                          (1, 1, 5000, 700, False)])
def test_aggregate_f32_order(oracle_mod, dev, B, H, n, N, sort):
    """The value sums on both sides of the rule that sorts the keys first: groups
    of none to hundreds of members added in ascending order, values whose sums
    depend on it, entries outside [0, N) ignored."""
    print(f"\n[case] aggregate f32 {B} {H} {n} {N}", flush=True)
    rng = np.random.default_rng(n)
    V = (rng.standard_normal((B, H, n, 64)) * 2.0 ** rng.integers(-30, 30, (B, H, n, 64))).astype(np.float32)
    belong = (N * rng.random((B, H, n)) ** 3).astype(np.int32)
    belong[rng.random((B, H, n)) < 0.3] = 7
    belong[0, 0, ::97], belong[-1, -1, 1::89] = -1, N
    vs, names = launched(lambda: ga.aggregate(torch.from_numpy(V).to(dev), torch.from_numpy(belong).to(dev), N))
    ref, _ = oracle_mod.aggregate(V.astype(np.float64), belong, N)
    assert np.array_equal(vs.cpu().numpy().view(np.uint32), ref.astype(np.float32).view(np.uint32))
    assert ("bucket" in names) == sort, sorted(names)


def test_forward_f32_sorted(oracle_mod, dev):
    """A forward whose updates sort the keys and whose value sums take the last
    round's order; groups that end empty keep their centroid."""
    print("\n[case] forward f32, sorted sums", flush=True)
    B, H, n, N, iters = 8, 8, 1000, 512, 2
    Q, K, V = inputs.make_qkv(B, H, n, 64, "f32", 9, 100, 0.05, 0.3)
    K[:, :, 1::2] = K[:, :, ::2]
    (O, *got), names = launched(lambda: ga.forward(Q.to(dev), K.to(dev), V.to(dev), N, iters, 0.125,
                                                   return_groups=True))
    assert names["bucket"][0] == iters, names
    ref = oracle_mod.forward(f64(Q), f64(K), f64(V), N, iters, 0.125, "f32")
    assert_groups(got, ref)
    assert (ref["count"] == 0).any()
    # 1e-4 per row: the documented bound of the fp32 attention
    err = np.linalg.norm(O.cpu().numpy() - ref["O"], axis=-1)
    assert (err <= 1e-4 * np.linalg.norm(ref["O"], axis=-1)).all()


ATTEND = [
    # B, H, n, N, scale
    (1, 1, 1, 1, 0.125),
    (1, 2, 97, 31, 0.125),
    (1, 1, 129, 64, -0.4),      # one staged chunk
    (1, 1, 200, 65, 0.125),     # a second chunk of one group
    (1, 1, 1100, 1000, 1.0),
    (4, 8, 4000, 40, 0.125),    # several passes per workgroup
]


@pytest.mark.parametrize("case", ATTEND, ids=lambda c: "-".join(map(str, c)))
def test_attend_f32_edges(oracle_mod, dev, case):
    """Error bound in units of u = 2^-24: a score is off by at most 66 u S (64
    products and the scaling, S = |scale| max|q| max|r|), which moves numerator
    and denominator by that share each; the exponential, the sums over the
    groups and the division add N + 16.  Relative to the largest value mean.
    The last block of groups is empty where there is more than one, and an
    empty group's rows may hold anything (here NaN)."""
    B, H, n, N, scale = case
    print(f"\n[case] attend f32 {case}", flush=True)
    rng = np.random.default_rng(n + N)
    Q, _, V = inputs.make_qkv(B, H, n, 64, "f32", 12, 8, 0.1, 0.1)
    live = max(1, (N - 1) // 32 * 32)
    belong = rng.integers(0, live, size=(B, H, n)).astype(np.int32)
    count = np.stack([[np.bincount(belong[b, h], minlength=N) for h in range(H)] for b in range(B)]).astype(np.int32)
    centroid = (0.3 * rng.standard_normal((B, H, N, 64))).astype(np.float32)
    vsum = oracle_mod.aggregate(f64(V), belong, N)[0].astype(np.float32)
    ref = oracle_mod.attend(f64(Q), centroid, count, vsum, N, scale, "f32")
    centroid[count == 0] = np.nan
    vsum[count == 0] = np.nan
    O = ga.attend(Q.to(dev), torch.from_numpy(centroid).to(dev), torch.from_numpy(count).to(dev),
                  torch.from_numpy(vsum).to(dev), N, scale)
    torch.cuda.synchronize()
    S = abs(scale) * np.linalg.norm(f64(Q), axis=-1).max() * np.nanmax(np.linalg.norm(centroid, axis=-1))
    mean = np.nanmax(np.linalg.norm(vsum / np.maximum(count, 1)[..., None], axis=-1))
    err = np.linalg.norm(O.cpu().numpy() - ref, axis=-1)
    assert err.max() <= 2.0**-24 * (2 * 66 * S + N + 16) * mean, (err.max(), S, mean)
