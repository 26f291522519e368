"""Recognition on the cooperative forward (csrc/fwd_coop.hip) computes in FP32, like the gradient's
forward: the table's entries are the bits of the gradient call's log-likelihoods, and labels are
the oracle's wherever its two best models are further apart than the measured rounding, also
in a bank with two models that all but agree."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_1310_3322_amd import hmm, workloads
from test_gpu_parity import label_parity

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _lib():
    hmm.load_library()
    yield
    hmm.select_kernel(hmm.KERNEL_AUTO)


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("N", [49, 64, 65, 100, 160, 192, 224, 256])
def test_table_and_labels(N):
    print(f"[case] recognition table N={N}", flush=True)
    rng = np.random.default_rng([113, N])
    w = workloads.random_lengths_workload(rng, K=4, N=N, M=33, lengths=rng.integers(0, 120, size=700).astype(np.int32),
                                          all_pairs=False, conc=0.5)
    for x in (w.pi, w.A, w.B):  # model 1: model 0 but for the last bits
        x[1] = x[0] * (1 + 2.0 ** -22 * rng.integers(-1, 2, size=x[0].shape)).astype(np.float32)
    p = hmm.Problem(dev(w.pi), dev(w.A), dev(w.B), dev(w.symbols), dev(w.offsets), dev(w.lengths), dev(w.owner),
                    max_len=w.max_len, total_symbols=w.total_symbols)
    hmm.select_kernel(hmm.KERNEL_COOP)
    table = torch.empty((w.S, 4), dtype=torch.float32, device="cuda")
    labels = hmm.classify(p, loglik=table).cpu().numpy()
    every = hmm.Problem(p.pi, p.A, p.B, p.symbols, p.offsets, p.lengths, None, max_len=w.max_len,
                        total_symbols=w.total_symbols)
    assert torch.equal(hmm.forward_loglik(every).view(torch.int32), table.view(torch.int32))
    hmm.select_kernel(hmm.KERNEL_AUTO)
    own = hmm.forward_backward_grad(p)[0].cpu().numpy()
    got = table.cpu().numpy()
    assert np.array_equal(got[np.arange(w.S), w.owner].view(np.int32), own.view(np.int32))
    ref = O.forward(w.pi, w.A, w.B, w.symbols, w.offsets, w.lengths, None)
    label_parity(labels, got, ref, f"N={N}", max_near_tie_share=1.0)
    far = [0, 2, 3]  # without the twin
    label_parity(O.classify(np.ascontiguousarray(got[:, far])), got[:, far], ref[:, far], f"N={N}, no twin", 0.05)
