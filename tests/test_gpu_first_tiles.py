"""Tiles taken by a workgroup's rank (csrc/kernels.h, first_rank) and from the queue: every
sequence is scored once whatever the numbers of tiles, models and workgroups, also where one
model has all the sequences.

Tolerance.  At most 6 steps of at most 16 roundings of 2^-24 each: 6e-6 of the likelihood,
hence an absolute error of the log-likelihood below 1e-5 (and as much of a larger one)."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_1310_3322_amd import hmm, workloads

pytestmark = pytest.mark.gpu

TOL = 1e-5
# sequences around one, two and three turns of 256 workgroups of 4 tiles of 16 (over all
# models), with a ragged end, and models beyond the workgroups
SHAPES = [(3, 5, 1), (3, 5, 5000), (1, 7, 16384), (1, 7, 16385), (3, 16, 17000), (5, 9, 33000), (2, 4, 50001),
          (7, 20, 35000), (2, 33, 17000), (2, 50, 17000), (300, 4, 700), (1100, 3, 60)]


@pytest.fixture(scope="module", autouse=True)
def _lib():
    hmm.load_library()
    yield
    hmm.select_kernel(hmm.KERNEL_AUTO)


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("K,N,S", SHAPES)
@pytest.mark.parametrize("mode", ["own", "skewed", "all"])
def test_every_tile_once(K, N, S, mode):
    if mode == "all":
        S = max(1, S // K)
    print(f"[case] first tiles K={K} N={N} S={S} {mode}", flush=True)
    rng = np.random.default_rng([89, K, N, S])
    w = workloads.random_lengths_workload(rng, K=K, N=N, M=11, lengths=rng.integers(1, 7, size=S), all_pairs=mode == "all")
    owner = np.full_like(w.owner, K // 2) if mode == "skewed" else w.owner
    own = None if mode == "all" else owner
    p = hmm.Problem(dev(w.pi), dev(w.A), dev(w.B), dev(w.symbols), dev(w.offsets), dev(w.lengths),
                    None if own is None else dev(own), max_len=6, total_symbols=w.total_symbols)
    ref = O.forward(w.pi, w.A, w.B, w.symbols, w.offsets, w.lengths, own)
    for kernel in [hmm.KERNEL_TILE16] + ([hmm.KERNEL_TILE32] if N in (20, 50) else []):  # 32 and 64 padded states
        hmm.select_kernel(kernel)
        out = torch.full((S,) if own is not None else (S, K), float("nan"), device="cuda")
        got = hmm.forward_loglik(p, out=out).cpu().numpy().astype(np.float64)
        assert np.all(np.abs(got - ref) <= TOL * np.maximum(np.abs(ref), 1.0)), kernel
