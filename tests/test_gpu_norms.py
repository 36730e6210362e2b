"""The canonical |r|^2 (an fp64 chain over the features in order) where no other
order of summation gives the same bits: representatives whose components span
more than 16 binades, so that the squares added by eight lanes are not exact and
the chain itself has to run."""
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


def wide_rows(rng, shape):
    """bf16 rows whose components lie within 2^-22 and 1."""
    x = rng.choice([-1.0, 1.0], shape) * (1.0 + rng.integers(0, 128, shape) / 128.0)
    return (x * 2.0 ** -rng.integers(0, 23, shape)).astype(np.float32)


def chain(r):
    """|r|^2 of the rows: each square is exact in fp64, so an addition in order is the fma chain."""
    acc = np.zeros(r.shape[:-1])
    for c in range(64):
        acc = acc + r[..., c] * r[..., c]
    return acc


def eight_lanes(r):
    part = np.zeros((*r.shape[:-1], 8))
    for e in range(8):
        part = part + r.reshape(*r.shape[:-1], 8, 8)[..., e] ** 2
    part = part[..., 0::2] + part[..., 1::2]
    part = part[..., 0::2] + part[..., 1::2]
    return part[..., 0] + part[..., 1]


@pytest.mark.parametrize("N,init", [(100, False), (129, False), (500, False), (600, False), (200, True), (300, True)])
@pytest.mark.parametrize("rounds", [False, True])
def test_initial_norms(oracle_mod, dev, N, init, rounds, monkeypatch):
    """Every representative of a slice is a permutation of one row, so all are
    equally long but for the rounding of the chain, which alone decides the
    group of a zero key."""
    if rounds:
        monkeypatch.setenv("GA_GROUPING", "rounds")
    B, H, n = 2, 16, 2 * N
    print(f"\n[case] initial norms {N} {init} {rounds}", flush=True)
    rng = np.random.default_rng(N)
    row = wide_rows(rng, (B, H, 1, 64))
    reps = np.ascontiguousarray(rng.permuted(np.broadcast_to(row, (B, H, N, 64)), axis=-1))
    assert (chain(reps.astype(np.float64)).argmin(-1) != eight_lanes(reps.astype(np.float64)).argmin(-1)).any()
    K = np.zeros((B, H, n, 64), np.float32)
    if not init:
        K[:, :, ::2] = reps  # the strided keys
    Kt = inputs.to_storage(K, "bf16")
    assert np.array_equal(inputs.as_float64(Kt), K)
    bel, cnt, _ = ga.cluster(Kt.to(dev), N, 1, init=torch.from_numpy(reps).to(dev) if init else None)
    ref = oracle_mod.cluster(inputs.as_float64(Kt), N, 1, "bf16", init=reps if init else None)
    assert np.array_equal(bel.cpu().numpy(), ref["belong"])
    assert np.array_equal(cnt.cpu().numpy(), ref["count"])


@pytest.mark.parametrize("n,N,iters", [(700, 100, 1), (700, 100, 4), (1500, 130, 1), (1500, 130, 4), (9000, 40, 1),
                                       (9000, 300, 2), (2500, 1000, 3)])
def test_updated_norms(dev, n, N, iters, monkeypatch):
    """The |r|^2 that the updates leave for the next round, found in the workspace:
    the first round's (from partitions, whole or in parts) and those of groups that
    later rounds' moved keys touched."""
    monkeypatch.setenv("GA_GROUPING", "rounds")
    print(f"\n[case] updated norms {n} {N} {iters}", flush=True)
    rng = np.random.default_rng(n + N)
    centre = wide_rows(rng, (max(4, N // 3), 64))
    K = centre[rng.integers(0, len(centre), n)] * (1.0 + 0.2 * rng.standard_normal((n, 64)))
    Kt = inputs.to_storage(K[None, None].astype(np.float32), "bf16").to(dev)
    ws = torch.zeros(ga.workspace_bytes(ga.shape_of(Kt), N), dtype=torch.uint8, device=dev)
    _, _, cen = ga.cluster(Kt, N, iters, ws=ws)
    rep = cen.to(torch.bfloat16).double().cpu().numpy()[0, 0]
    assert (chain(rep) != eight_lanes(rep)).any()
    at = ws.cpu().numpy().tobytes().find(chain(rep).tobytes())
    assert at >= 0 and at % 256 == 0
