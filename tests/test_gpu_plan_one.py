"""The plan of a small batch in one launch (csrc/planner.hip, k_plan_one): the work list against
a stable sort at the limits of its rule (16, 8 or 4 waves of at most 1024 sequences, at most
32768 entries of the count matrix), one past them, and with invalid entries; and its tables,
through the log-likelihoods of the general way's kernels.  Integer work: bit-exact."""
import numpy as np
import pytest
import torch

from paper_1310_3322_amd import hmm, workloads
from test_gpu_plan import run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K,max_len,S", [(1, 1, 1), (1, 9, 63), (1, 9, 64), (1, 9, 65), (3, 40, 1000), (8, 255, 16383),
                                         (8, 255, 16384), (8, 255, 16385), (8, 256, 8192), (16, 255, 8193),
                                         (16, 256, 4095), (32, 255, 4096), (32, 255, 4097), (32, 256, 4096),
                                         (1, 2047, 5000), (1, 4095, 5000), (1, 8191, 3000), (200, 10, 777)])
def test_order_at_the_limits(K, max_len, S):
    print(f"[case] plan in one launch K={K} max_len={max_len} S={S}", flush=True)
    rng = np.random.default_rng([97, K, max_len, S])
    lengths = rng.integers(0, max_len + 1, size=S).astype(np.int32)
    lengths[rng.random(S) < 0.3] = min(3, max_len)  # many in one bin
    w = workloads.random_lengths_workload(rng, K=K, N=3, M=5, lengths=np.minimum(lengths, 12), all_pairs=False)
    owner = rng.integers(0, K, size=S).astype(np.int32)
    total = int(lengths.astype(np.int64).sum()) + 1
    w.symbols = np.zeros(total, np.int32)
    w.offsets[:] = np.concatenate(([0], np.cumsum(lengths[:-1].astype(np.int64))))
    if S > 60:
        lengths[5], lengths[7], w.offsets[17] = -1, 1 << 20, -8
        if K > 1:  # (one model: one group, whose plan does not read the owners)
            owner[11], owner[13] = K, -3
    for own in (True, False):
        run(w, hmm.OP_FORWARD, own, max_len=max_len, lengths=lengths, owner=owner)


@pytest.mark.parametrize("K,N,M,S", [(1, 1, 1, 40), (5, 16, 33, 300), (3, 31, 200, 300), (2, 40, 1000, 200),
                                     (9, 64, 300, 100), (2, 100, 1024, 50)])
def test_tables_agree_with_the_general_way(K, N, M, S):
    """A batch and the same one with sequences of length 0 appended until it takes the general
    way: the same kernels on the same tables give the same bits."""
    rng = np.random.default_rng([98, K, N, M])
    w = workloads.random_lengths_workload(rng, K=K, N=N, M=M, lengths=rng.integers(1, 60, size=S), all_pairs=True)

    def dev(a):
        return torch.from_numpy(np.ascontiguousarray(a)).cuda()

    more = 17000
    big_off = np.concatenate((w.offsets, np.zeros(more, np.int64)))
    big_len = np.concatenate((w.lengths, np.zeros(more, np.int32)))
    hmm.select_kernel(hmm.KERNEL_TILE16 if N <= 64 else hmm.KERNEL_COOP)
    try:
        out = [hmm.forward_loglik(hmm.Problem(dev(w.pi), dev(w.A), dev(w.B), dev(w.symbols), dev(o), dev(n), None, max_len=60,
                                              total_symbols=w.total_symbols)).cpu().numpy()[:S]
               for o, n in ((w.offsets, w.lengths), (big_off, big_len))]
    finally:
        hmm.select_kernel(hmm.KERNEL_AUTO)
    assert np.isfinite(out[0]).all() and np.array_equal(out[0].view(np.int32), out[1].view(np.int32))
