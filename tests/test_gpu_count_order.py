"""Emission counts of a 16-sequence tile up to 48 states (csrc/adj_mfma.hip): slots that share a
symbol are added in slot order whatever the number of steps per chunk, so a model's counts are the
same bits beside few other tiles (chunks of four steps at 16 states) and beside many (chunks
of two)."""
import numpy as np
import pytest
import torch

from paper_1310_3322_amd import hmm, workloads

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("N,M", [(3, 2), (8, 6), (16, 1), (16, 40), (24, 3), (48, 5)])
def test_counts_do_not_depend_on_the_chunks(N, M):
    print(f"[case] count order N={N} M={M}", flush=True)
    rng = np.random.default_rng([131, N, M])
    lengths = rng.integers(1, 90, size=14).astype(np.int32)
    lengths = np.concatenate((lengths, np.full(18, 61, np.int32)))  # two tiles of model 0, one of equal lengths
    few, many = len(lengths), 12000
    w = workloads.random_lengths_workload(rng, K=2, N=N, M=M, lengths=np.concatenate((lengths, np.full(many, 2, np.int32))),
                                          all_pairs=False, conc=0.5)
    owner = np.concatenate((np.zeros(few, np.int32), np.ones(many, np.int32)))
    weight = rng.uniform(0.25, 1.75, size=few + many).astype(np.float32)
    got = []
    for S in (few, few + many):
        p = hmm.Problem(dev(w.pi), dev(w.A), dev(w.B), dev(w.symbols), dev(w.offsets[:S]), dev(w.lengths[:S]),
                        dev(owner[:S]), max_len=90, total_symbols=w.total_symbols)
        ll, (_, _, n_B), _ = hmm.forward_backward_grad(p, dev(weight[:S]))
        got.append((ll[:few].clone(), n_B[0].clone()))
    assert float(got[0][1].sum()) > 0.0
    for a, b in zip(*got):
        assert torch.equal(a.view(torch.int32), b.view(torch.int32))
