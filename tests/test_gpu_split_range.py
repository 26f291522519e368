"""The cooperative forward (csrc/fwd_coop.hip) where its vectors or its transition rows are near
the smallest FP32 numbers: emission probabilities down to 1e-38, and a state some 2^-120 below the
others that alone can emit the next symbol.  Split into bf16 pieces at their place, such values
lose their lower pieces.

Tolerance.  With every one of the N terms of a product, the three partial products left out and
the N / 16 + 4 additions and the emission product of a step truncated, a step's relative error is
below (N + N / 16 + 8) 2^-23 = 3.4e-5 at 256 states, and every third step below adds at
least ln 1e30 = 69 to the magnitude of the log-likelihood: 3 * 3.4e-5 / 69 = 1.5e-6 of it, and
the rounding of the result."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_1310_3322_amd import hmm, workloads

pytestmark = pytest.mark.gpu

LL_TOL = 1.6e-6


@pytest.fixture(scope="module", autouse=True)
def _lib():
    hmm.load_library()
    hmm.select_kernel(hmm.KERNEL_COOP)
    yield
    hmm.select_kernel(hmm.KERNEL_AUTO)


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def check(w):
    for own in (True, False):
        p = hmm.Problem(dev(w.pi), dev(w.A), dev(w.B), dev(w.symbols), dev(w.offsets), dev(w.lengths),
                        dev(w.owner) if own else None, max_len=w.max_len, total_symbols=w.total_symbols)
        ll = hmm.forward_loglik(p).cpu().numpy().astype(np.float64)
        ref = O.forward(w.pi, w.A, w.B, w.symbols, w.offsets, w.lengths, w.owner if own else None)
        assert np.isfinite(ref).all() and np.isfinite(ll).all(), own
        err = float(np.max(np.abs(ll - ref) / np.maximum(np.abs(ref), 1.0)))
        print(f"  own={own} error {err:.2e}", flush=True)
        assert err <= LL_TOL, own


@pytest.mark.parametrize("N", [64, 100, 144, 200, 256])
@pytest.mark.parametrize("small", [1e-30, 1e-33, 1e-35, 1e-37, 1e-38])
def test_smallest_emissions(N, small):
    """Every third symbol has a probability around `small` in every state."""
    print(f"[case] split range N={N} small={small}", flush=True)
    rng = np.random.default_rng([107, N])
    lengths = (3 * rng.integers(1, 30, size=33)).astype(np.int32)
    w = workloads.random_lengths_workload(rng, K=2, N=N, M=12, lengths=lengths, all_pairs=False)
    w.B[:, :, 0] = (small * (0.5 + rng.random((2, N)))).astype(np.float32)
    for o, n in zip(w.offsets, w.lengths):
        w.symbols[o:o + n] = np.where(np.arange(n) % 3 == 1, 0, 1 + w.symbols[o:o + n] % 11)
    check(w)


@pytest.mark.parametrize("N", [64, 100, 144, 200, 256])
@pytest.mark.parametrize("row", [False, True])
def test_lone_survivor(N, row):
    """A state that every third step is the only one with the symbol: reached by transitions of
    2^-120 (row), or with that probability of the symbol before."""
    print(f"[case] lone survivor N={N} row={row}", flush=True)
    rng = np.random.default_rng([109, N, row])
    lengths = (3 * rng.integers(1, 30, size=33)).astype(np.int32)
    w = workloads.random_lengths_workload(rng, K=2, N=N, M=12, lengths=lengths, all_pairs=False)
    tiny = np.float32(2.0 ** -120)
    lone = N - 3
    w.B[:, :, 0] = 0.0
    w.B[:, lone, 0] = 0.4  # symbol 0: the lone state alone
    if row:
        w.A[:, :, lone] = tiny * (0.5 + rng.random((2, N))).astype(np.float32)
        w.pi[:, lone] = 0.0
    else:
        w.A[:, :, lone] *= np.float32(0.5)
        w.A[:, :lone, lone] = 0.0
        w.A[:, lone + 1:, lone] = 0.0
        w.A[:, lone, lone] = 0.5        # the lone state's mass comes from itself
        w.B[:, lone, 1] = tiny * np.float32(1.3)  # symbol 1: all but never in it
        w.pi[:, lone] = 0.3
    for o, n in zip(w.offsets, w.lengths):
        pattern = np.array([2, 3, 0] if row else [2, 1, 0])
        w.symbols[o:o + n] = pattern[np.arange(n) % 3]
    check(w)
