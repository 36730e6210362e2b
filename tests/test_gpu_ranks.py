"""GPU parity of the one-launch grouping around the changes of its rank count:
one rank per slice (nothing exchanged) up to 1024 keys (1536 where two ranks are
the alternative), at most 8 below 3584 keys, else up to 16."""
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


CASES = [
    # B, H, n, N, iters, one rank (no reset launch)
    (1, 1, 5, 5, 2, True),         # one tile, seven waves without one
    (1, 2, 257, 16, 4, True),      # nine tiles: one wave has two
    (1, 3, 1024, 128, 4, True),    # four tiles per wave
    (1, 3, 1025, 128, 4, False),   # 5 ranks
    (13, 8, 1536, 40, 3, True),    # 104 slices, where two ranks are the alternative
    (13, 8, 1537, 40, 3, False),   # 2 ranks, 4 tiles in one wave and 3 in the others
    (10, 8, 1100, 50, 3, False),   # 3 ranks
    (1, 2, 3583, 64, 3, False),    # 8 ranks
    (1, 2, 3584, 64, 3, False),    # 14 ranks
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(map(str, c)))
def test_forward_around_rank_changes(oracle_mod, dev, case):
    B, H, n, N, iters, one = case
    print(f"\n[case] ranks {case}", flush=True)
    Q, K, V = inputs.make_qkv(B, H, n, 64, "bf16", 11 * n + N, max(4, N), 0.05, 0.3)
    ga.timing_enable(True)
    try:
        O, bel, cnt, cen = ga.forward(Q.to(dev), K.to(dev), V.to(dev), N, iters, 0.125, return_groups=True)
        torch.cuda.synchronize()
        ga.workspace_check(Q.to(dev), N)
    finally:
        ga.timing_enable(False)
        names = ga.timing_collect()
    assert ("lloyd_reset" not in names) == one and "lloyd" in names, sorted(names)
    ref = oracle_mod.forward(*(inputs.as_float64(t) for t in (Q, K, V)), N, iters, 0.125, "bf16")
    assert np.array_equal(bel.cpu().numpy(), ref["belong"])
    assert np.array_equal(cnt.cpu().numpy(), ref["count"])
    assert np.array_equal(cen.cpu().numpy().view(np.uint32), ref["centroid"].view(np.uint32))
    # 2e-2 per row: the documented bound of the bf16 attention
    err = np.linalg.norm(O.float().cpu().numpy() - ref["O"], axis=-1)
    assert (err <= 2e-2 * np.linalg.norm(ref["O"], axis=-1)).all()


def test_one_rank_special_rounds(oracle_mod, dev, monkeypatch):
    """One rank: a fixed point before the last round, and every key through
    the exact decision with a caller's init."""
    print("\n[case] one rank: fixed point, exact decisions", flush=True)
    _, K, _ = inputs.make_qkv(1, 3, 900, 64, "bf16", 79, 32, 0.01, 0.01)
    init = K[:, :, :32].float().contiguous()
    for widen in ("1", "65536"):
        monkeypatch.setenv("GA_CERT_WIDEN", widen)
        for ini in (None, init):
            bel, cnt, cen = ga.cluster(K.to(dev), 32, 12, init=None if ini is None else ini.to(dev))
            torch.cuda.synchronize()
            ref = oracle_mod.cluster(inputs.as_float64(K), 32, 12, "bf16", init=None if ini is None else ini.numpy())
            assert np.array_equal(bel.cpu().numpy(), ref["belong"])
            assert np.array_equal(cnt.cpu().numpy(), ref["count"])
            assert np.array_equal(cen.cpu().numpy().view(np.uint32), ref["centroid"].view(np.uint32))


REPEATS = [
    # B, H, n, N, iters: one rank, one rank of four blocks, four ranks, sixteen, and a launch per round
    (1, 3, 600, 50, 4), (1, 2, 1000, 128, 4), (1, 2, 1800, 100, 3), (1, 1, 8000, 128, 3), (1, 2, 900, 200, 3),
]


@pytest.mark.parametrize("case", REPEATS, ids=lambda c: "-".join(map(str, c)))
@pytest.mark.parametrize("form", ["tail", "equal", "pairs", "init"])
def test_repeated_representatives(oracle_mod, dev, case, form):
    """Series whose strided keys repeat (zero padding, one value throughout, pairs)
    and given centroids that do: exact ties, which the group of lowest index wins."""
    B, H, n, N, iters = case
    print(f"\n[case] repeats {case} {form}", flush=True)
    _, K, _ = inputs.make_qkv(B, H, n, 64, "bf16", n + N, N, 0.05, 0.3)
    init = None
    if form == "tail":
        K[:, :, n - n // 3:] = 0
    elif form == "equal":
        K[:] = K[:, :, 3:4].clone()
    elif form == "pairs":
        K[:, :, n // 2:] = K[:, :, :n - n // 2].clone()
    else:
        at = np.random.default_rng(N).integers(0, N // 3, N)
        init = np.ascontiguousarray(inputs.as_float64(K)[:, :, at].astype(np.float32))
    got = ga.cluster(K.to(dev), N, iters, init=None if init is None else torch.from_numpy(init).to(dev))
    torch.cuda.synchronize()
    ref = oracle_mod.cluster(inputs.as_float64(K), N, iters, "bf16", init=init)
    for x, what in zip(got, ("belong", "count", "centroid")):
        assert np.array_equal(x.cpu().numpy().view(np.uint32), ref[what].view(np.uint32)), what


def test_padding_costs_no_multiple(dev):
    """Zero-padded series on one rank: a tenth of the keys zero takes 1.3 times the
    time without padding, and 5 to 6 times where every key near the repeated zero
    representatives takes the exact decision.  The bound lies between."""
    print("\n[case] cost of padding", flush=True)
    _, K, _ = inputs.make_qkv(2, 4, 1000, 64, "bf16", 3, 64, 0.05, 0.3)
    padded = K.clone()
    padded[:, :, 900:] = 0

    def time(x):
        ts = []
        for _ in range(20):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(10):
                ga.cluster(x, 64, 5)
            b.record()
            b.synchronize()
            ts.append(a.elapsed_time(b))
        return sorted(ts)[len(ts) // 2]

    K, padded = K.to(dev), padded.to(dev)
    time(K)
    assert time(padded) < 3 * time(K)
