"""Products on the bf16 matrix cores by three-way splits (csrc/split3.cuh): the kernels
that use them against the FP64 oracle at the edges of their tiles, and on emission
probabilities far below one, where the unscaled vectors and their pieces are small.

Tolerance.  A product of N terms in six partial products has a relative error below
(N / 32 + 8) 2^-24 + 3 2^-26 (one FP32 rounding per matrix instruction and per final
sum, and the three partial products left out), the emission product and the sum add
(N / 16 + 4) 2^-24: at most 48 2^-24 = 3e-6 per step at 256 states.  The logarithm of
the likelihood takes the sum of those, and a step adds at least ln 2 to its magnitude
for the symbols below (their probabilities stay under a half), so the relative error is
below 3e-6 / ln 2 < 5e-6."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_1310_3322_amd import hmm, workloads

pytestmark = pytest.mark.gpu

LL_TOL = 5e-6
CHUNK_EDGES = [1, 2, 3, 30, 31, 32, 33, 34, 63, 64, 65, 66, 97]


@pytest.fixture(scope="module", autouse=True)
def _lib():
    hmm.load_library()
    yield
    hmm.select_kernel(hmm.KERNEL_AUTO)


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def problem(w, own):
    return hmm.Problem(dev(w.pi), dev(w.A), dev(w.B), dev(w.symbols), dev(w.offsets), dev(w.lengths),
                       dev(w.owner) if own else None, max_len=max(w.max_len, 1), total_symbols=w.total_symbols)


def rel(gpu, ref):
    ref = np.asarray(ref, np.float64)
    return float(np.max(np.abs(gpu.cpu().numpy().astype(np.float64) - ref) / np.maximum(np.abs(ref), 1.0)))


@pytest.mark.parametrize("N", [49, 64, 65, 96, 97, 128, 129, 160, 161, 192, 193, 224, 225, 255, 256])
def test_cooperative_forward_state_counts(N):
    print(f"[case] split forward N={N}", flush=True)
    rng = np.random.default_rng([71, N])
    lengths = np.array(CHUNK_EDGES + [int(x) for x in rng.integers(1, 140, size=24)], np.int32)
    w = workloads.random_lengths_workload(rng, K=3, N=N, M=37, lengths=lengths, all_pairs=False, conc=0.3)
    hmm.select_kernel(hmm.KERNEL_COOP)
    for own in (True, False):
        ll = hmm.forward_loglik(problem(w, own))
        ref = O.forward(w.pi, w.A, w.B, w.symbols, w.offsets, w.lengths, w.owner if own else None)
        assert rel(ll, ref) <= LL_TOL, own


@pytest.mark.parametrize("N", [64, 144, 256])
@pytest.mark.parametrize("small", [1e-12, 1e-25])
def test_cooperative_forward_small_emissions(N, small):
    """Every third symbol has probability `small` in every state (one in ten of them zero
    in most states), so that steps scale the sum by 2^-40 and 2^-83."""
    print(f"[case] split forward N={N} small={small}", flush=True)
    rng = np.random.default_rng([73, N])
    lengths = rng.integers(40, 90, size=33).astype(np.int32)
    w = workloads.random_lengths_workload(rng, K=2, N=N, M=12, lengths=lengths, all_pairs=False)
    w.B[:, :, 0] = (small * (0.5 + rng.random((2, N)))).astype(np.float32)
    w.B[:, N // 4:, 1] = 0.0
    w.symbols[::3] = 0
    w.symbols[1::30] = 1
    hmm.select_kernel(hmm.KERNEL_COOP)
    ll = hmm.forward_loglik(problem(w, True))
    ref = O.forward(w.pi, w.A, w.B, w.symbols, w.offsets, w.lengths, w.owner)
    assert np.isfinite(ref).all() and rel(ll, ref) <= LL_TOL
