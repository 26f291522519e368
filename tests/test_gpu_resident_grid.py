"""Tile forwards whose grid the LDS bounds (csrc/kernels.h, ranked_per_cu): emission tables at the
edge of what four, three and two workgroups per CU leave each, with few and with many models: every
sequence is scored once.

Tolerance.  At most 6 steps of at most 20 roundings of 2^-24 each: 7.2e-6 of the likelihood, hence an
absolute error of the log-likelihood below 1e-5 (and as much of a larger one)."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_1310_3322_amd import hmm, workloads

pytestmark = pytest.mark.gpu

TOL = 1e-5


@pytest.mark.parametrize("K,N,M,S,kernel", [(12, 16, 287, 3000, hmm.KERNEL_TILE16), (12, 16, 288, 3000, hmm.KERNEL_TILE16),
                                            (12, 16, 300, 3000, hmm.KERNEL_TILE16), (600, 6, 300, 300, hmm.KERNEL_TILE16),
                                            (300, 9, 300, 500, hmm.KERNEL_TILE16), (12, 30, 318, 2000, hmm.KERNEL_TILE16),
                                            (12, 20, 344, 4000, hmm.KERNEL_TILE32), (12, 20, 347, 4000, hmm.KERNEL_TILE32),
                                            (600, 20, 347, 300, hmm.KERNEL_TILE32)])
def test_every_tile_once(K, N, M, S, kernel):
    print(f"[case] resident grid K={K} N={N} M={M} S={S} kernel={kernel}", flush=True)
    rng = np.random.default_rng([137, K, N, M])
    w = workloads.random_lengths_workload(rng, K=K, N=N, M=M, lengths=rng.integers(1, 7, size=S), all_pairs=True)
    p = hmm.Problem(*(torch.from_numpy(np.ascontiguousarray(a)).cuda()
                      for a in (w.pi, w.A, w.B, w.symbols, w.offsets, w.lengths)), None, max_len=6,
                    total_symbols=w.total_symbols)
    hmm.load_library()
    hmm.select_kernel(kernel)
    try:
        out = torch.full((S, K), float("nan"), device="cuda")
        got = hmm.forward_loglik(p, out=out).cpu().numpy().astype(np.float64)
    finally:
        hmm.select_kernel(hmm.KERNEL_AUTO)
    ref = O.forward(w.pi, w.A, w.B, w.symbols, w.offsets, w.lengths, None)
    assert np.all(np.abs(got - ref) <= TOL * np.maximum(np.abs(ref), 1.0))
