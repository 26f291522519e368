"""The backward walk over stored rows in two parts (csrc/adj_coop.hip, k_adj_duo) at the edges of
its chunks of symbols (16 steps), of its rule and of the emission partial, with weights, an
impossible and an empty sequence: bit for bit the counts of the checkpointed kernels, and the
FP64 oracle's.

Tolerance against the oracle.  A step of either recursion rounds at most 30 times (24 matrix
products of 4 terms in a row at 96 states, the emission product, the scale and its sum), each
below 2^-24, over at most 70 steps: 1.3e-4 of each sequence's counts, hence of their sums."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_1310_3322_amd import hmm, workloads

pytestmark = pytest.mark.gpu

TOL = 1.3e-4
EDGES = [0, 1, 2, 3, 4, 13, 14, 15, 16, 17, 18, 19, 30, 31, 32, 33, 34, 35, 47, 48, 49, 50, 62, 63, 64, 65, 66, 70]


@pytest.fixture(scope="module", autouse=True)
def _lib():
    hmm.load_library()
    yield


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("N,M,S,K", [(64, 7, 29, 1), (49, 30, 120, 3), (64, 300, 200, 3), (60, 511, 200, 2), (64, 515, 200, 2),
                                     (64, 519, 60, 2), (64, 40, 9000, 3), (65, 12, 120, 3), (96, 200, 200, 3), (81, 300, 90, 9),
                                     (96, 312, 90, 1), (90, 330, 90, 1), (96, 20, 9000, 8)])
def test_stored_walk(N, M, S, K):
    print(f"[case] stored walk N={N} M={M} S={S} K={K}", flush=True)
    rng = np.random.default_rng([101, N, M, S])
    lengths = np.array(EDGES + [int(x) for x in rng.integers(1, 71 if S < 1000 else 7, size=S - len(EDGES))], np.int32)
    w = workloads.random_lengths_workload(rng, K=K, N=N, M=M, lengths=rng.permutation(lengths), all_pairs=False, conc=0.5)
    weight = rng.uniform(0.25, 1.75, size=S).astype(np.float32)
    for s in range(0, S, 3):  # many slots of a tile on one symbol
        w.symbols[w.offsets[s]:w.offsets[s] + w.lengths[s]] = 3
    w.B[0, :, 4] = 0.0            # impossible in model 0: such a sequence takes no part
    w.B[0] /= w.B[0].sum(axis=1, keepdims=True)
    w.symbols[w.symbols == 4] = 0
    dead = int(np.flatnonzero((w.owner == 0) & (w.lengths >= 13))[0])
    w.symbols[w.offsets[dead] + 7] = 4
    B = w.B.astype(np.float32)
    p = hmm.Problem(dev(w.pi), dev(w.A), dev(B), dev(w.symbols), dev(w.offsets), dev(w.lengths), dev(w.owner),
                    max_len=70, total_symbols=w.total_symbols)
    out = []
    for rows in (p.total_symbols, 0):
        ll, counts, _ = hmm.forward_backward_grad(p, dev(weight), ws=p.grad_workspace(rows))
        out.append([x.cpu().numpy() for x in (ll, *counts)])
    for name, x, y in zip(("ll", "pi", "A", "B"), *out):
        assert np.array_equal(x.view(np.int32), y.view(np.int32)), name
    ref = O.counts(w.pi, w.A, B, w.symbols, w.offsets, w.lengths, w.owner, weight)[1:]
    for name, g, r in zip(("pi", "A", "B"), out[0][1:], ref):
        for k in range(K):
            assert np.linalg.norm(g[k] - r[k]) <= TOL * np.linalg.norm(r[k]), (name, k)
