"""All-pairs tiles of 32 sequences split over the XCDs (csrc/fwd_mfma32.hip) with more tiles per
slice than its waves take by rank, so that the rest come from the slice's queue, also where a slice
of the grid is no multiple of the models (workgroups per model then differ by one): every entry of
the table against the oracle, and bit for bit as without the split.

Tolerance.  At most 6 steps of at most 36 roundings of 2^-24 each: 1.3e-5 of the likelihood, hence an
absolute error of the log-likelihood below 1.4e-5 (and as much of a larger one)."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_1310_3322_amd import hmm, workloads

pytestmark = pytest.mark.gpu

TOL = 1.4e-5


@pytest.fixture(scope="module", autouse=True)
def _lib():
    hmm.load_library()
    hmm.select_kernel(hmm.KERNEL_AUTO)
    yield
    hmm.tune_clear()


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


# workgroups of a 256-unit device after the cap and the rounding to the models, and per slice:
# 504 and 63 for 12, 24 and 56 models, 512 and 64 for 8, 256 and 32 for 4
@pytest.mark.parametrize("K,N,S,cap", [(12, 20, 13001, 2), (12, 50, 13000, 2), (24, 32, 9000, 2), (56, 20, 5003, 2),
                                       (8, 20, 20001, 2), (4, 50, 20000, 1)])
def test_slices_with_queue(K, N, S, cap):
    print(f"[case] tile slices K={K} N={N} S={S} cap={cap}", flush=True)
    rng = np.random.default_rng([127, K, N, S])
    w = workloads.random_lengths_workload(rng, K=K, N=N, M=11, lengths=rng.integers(1, 7, size=S).astype(np.int32),
                                          all_pairs=True)
    p = hmm.Problem(dev(w.pi), dev(w.A), dev(w.B), dev(w.symbols), dev(w.offsets), dev(w.lengths), None, max_len=6,
                    total_symbols=w.total_symbols)
    key = hmm.tune_key(p.bank, p.batch, hmm.OP_FORWARD)
    out = []
    for flags in (0, hmm.TUNE_XCD_OFF):
        hmm.tune_set(key, hmm.KERNEL_TILE32, cap, flags)
        table = torch.full((S, K), float("nan"), device="cuda")
        out.append(hmm.forward_loglik(p, out=table).clone())
    assert torch.equal(out[0].view(torch.int32), out[1].view(torch.int32))
    ref = O.forward(w.pi, w.A, w.B, w.symbols, w.offsets, w.lengths, None)
    got = out[0].cpu().numpy().astype(np.float64)
    assert np.all(np.abs(got - ref) <= TOL * np.maximum(np.abs(ref), 1.0))
