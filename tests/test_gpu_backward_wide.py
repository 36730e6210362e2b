"""GPU parity of the backward's query kernel for more than 128 groups: the
softmax shift found in the first, a middle or the last block, blocks without a
member, and the wave counts of its launch."""
import hashlib

import numpy as np
import pytest
import torch

from paper_2306_01926_amd import ga, inputs

pytestmark = pytest.mark.gpu
TOL = 2e-2  # the documented bound of the gradient, per slice

CASES = [
    # B, H, n, N, scale, empty groups, growth of the centroids from block to block
    (1, 1, 130, 129, 0.125, (0, 0), 1.0),    # one group in the last block, two keys in the last tile
    (1, 2, 500, 160, 0.5, (0, 40), 1.6),     # the first block and part of the second empty, shifts grow
    (1, 1, 500, 224, 0.5, (180, 224), 0.6),  # the last block empty, shifts fall
    (1, 1, 33000, 130, 0.125, (3, 9), 1.0),  # five tiles for four waves
    (30, 10, 600, 130, -0.2, (0, 32), 1.2),  # more slices than compute units
    (30, 10, 1250, 130, 0.2, (0, 32), 1.0),  # and two workgroups of 20 tiles for each
    (20, 7, 650, 222, 0.125, (3, 9), 1.0),   # 21 tiles for eight waves
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(map(str, c[:4])))
def test_backward_wide(oracle_mod, case):
    B, H, n, N, scale, (e0, e1), grow = case
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    print(f"\n[case] backward {case}", flush=True)
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(n + N)
    Q, _, V = inputs.make_qkv(B, H, n, 64, "bf16", 5, 8, 0.1, 0.1)
    dO = inputs.to_storage(rng.standard_normal((B, H, n, 64), dtype=np.float32), "bf16")
    live = np.array([g for g in range(N) if not e0 <= g < e1], np.int32)
    belong = live[rng.integers(0, len(live), size=(B, H, n))]
    count = np.stack([[np.bincount(belong[b, h], minlength=N) for h in range(H)] for b in range(B)]).astype(np.int32)
    centroid = 0.2 * rng.standard_normal((B, H, N, 64)) * grow ** (np.arange(N) // 32)[:, None]
    centroid = centroid.astype(np.float32)
    vsum = oracle_mod.aggregate(inputs.as_float64(V), belong, N)[0].astype(np.float32)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)  # noqa: E731
    got = [ga.backward(Q.to(dev), dO.to(dev), t(belong), t(centroid), t(count), t(vsum), N, scale) for _ in range(2)]
    torch.cuda.synchronize()
    assert all(torch.equal(x, y) for x, y in zip(*got)), "repeated calls differ"
    ref = oracle_mod.backward(inputs.as_float64(Q), inputs.as_float64(dO), belong, centroid, count, vsum, N, scale,
                              "bf16")
    for X, R, what in zip(got[0], ref, ("dQ", "dK", "dV")):
        err = np.abs(X.float().cpu().numpy() - R).max(axis=(2, 3))
        assert (err <= TOL * np.abs(R).max(axis=(2, 3))).all(), (what, (err / np.abs(R).max(axis=(2, 3))).max())


# B, H, n, N, scale and SHA-256 (16 digits) of dQ, dK, dV: the softmax shift is the
# largest score of all blocks before any weight is summed, every sum in
# ascending blocks and registers
BITS = [
    (1, 2, 333, 160, 0.125, "4cf53323e96d982e", "534f9dee9680a689", "f4c65e4a38c4d6e4"),
    (2, 1, 500, 161, -0.5, "d8be9c19852ab2e0", "78d1a6b419d4f7e4", "71689d51fe19e8e8"),
    (1, 3, 700, 200, 0.125, "0370d56236e6ef1b", "89ad5e83d63882d9", "f0e281a33138a3e1"),
    (1, 1, 1000, 256, 0.3, "dc9e8d94c32ce383", "3bea71e2d6f9410c", "13aec6e5aca4f122"),
]


def uniform(shape, seed):
    """Reproducible values in (-1, 1) from integer arithmetic alone."""
    x = (np.arange(np.prod(shape), dtype=np.uint64) + np.uint64(seed << 32)) * np.uint64(0x9E3779B97F4A7C15)
    x ^= x >> np.uint64(32)
    x *= np.uint64(0xD6E8FEB86659FD93)
    x ^= x >> np.uint64(32)
    return ((x >> np.uint64(40)).astype(np.float64) * 2.0**-23 - 1.0).astype(np.float32).reshape(shape)


def digests(case):
    B, H, n, N, scale = case[:5]
    dev = torch.device("cuda:0")
    Q, dO, V = (inputs.to_storage(2 * uniform((B, H, n, 64), s), "bf16") for s in range(3))
    belong = ((np.arange(B * H * n, dtype=np.int64) * 7919 >> 3) % (N - 2)).astype(np.int32).reshape(B, H, n)
    count = np.stack([[np.bincount(belong[b, h], minlength=N) for h in range(H)] for b in range(B)]).astype(np.int32)
    centroid = uniform((B, H, N, 64), 3)
    vsum = np.zeros((B, H, N, 64))
    Vd = inputs.as_float64(V)
    for b in range(B):
        for h in range(H):
            np.add.at(vsum[b, h], belong[b, h], Vd[b, h])
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)  # noqa: E731
    got = ga.backward(Q.to(dev), dO.to(dev), t(belong), t(centroid), t(count), t(vsum.astype(np.float32)), N, scale)
    return [hashlib.sha256(x.view(torch.int16).cpu().numpy().tobytes()).hexdigest()[:16] for x in got]


@pytest.mark.parametrize("case", BITS, ids=lambda c: "-".join(map(str, c[:4])))
def test_backward_wide_bits(case):
    print(f"\n[case] backward bits {case[:5]}", flush=True)
    assert digests(case) == list(case[5:])
