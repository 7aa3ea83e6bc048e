"""Assignment and update with codebooks of more than 256 entries, alone and in stacks whose
layers differ in size and codebook: every index and best distance equals the oracle's fp32
decision, counts are exact and the distortion is the oracle's sum (1e-9: fp64 sums of the same
fp32 distances in another order, at most 2^17 terms of relative rounding 2^-53 each)."""
import numpy as np
import pytest
import torch

import oracle
import synth

pytestmark = pytest.mark.gpu

kq = pytest.importorskip("paper_2003_05148_amd")
DEV = torch.device("cuda:0")


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


def host(t):
    torch.cuda.synchronize()
    return t.cpu().numpy()


def layer(n, k, seed):
    X = synth.laplace_layer(max(1, n // 64), 64, seed)
    X = np.ascontiguousarray(np.resize(X, (n, 9)) if X.shape[0] < n else X[:n])
    return X, synth.random_codebook_state(X, k, seed + 1)


STACKS = [
    # small and large codebooks side by side, small and large layers (paper's layerwise sizes)
    [(192, 60), (4096, 128), (8192, 1008), (32768, 1088), (65536, 640)],
    [(4096, 1203), (4096, 609), (16384, 2974), (20000, 6987)],
    # ragged: fewer kernels than a unit, one kernel, k > n, one entry
    [(63, 300), (1, 257), (1000, 1), (4097, 257), (130, 513)],
]


@pytest.mark.parametrize("shape", STACKS)
def test_stack_of_mixed_codebooks(shape):
    layers = [layer(n, k, 100 + 7 * i) for i, (n, k) in enumerate(shape)]
    st = kq.Stack([dev(X) for X, _ in layers], [dev(C) for _, C in layers], iters=1, best_d=True)
    kq.kq_assign_stack(st)
    kq.kq_update_stack(st, dist_slot=1, distortion_from_assign=True)
    for i, (X, C) in enumerate(layers):
        a = oracle.assign(X, C)
        assert np.array_equal(host(st.idx[i]), a["idx"]), shape[i]
        assert np.array_equal(host(st.best_d[i]), a["d32"]), shape[i]
        assert np.array_equal(host(st.counts[i]), np.bincount(a["idx"], minlength=C.shape[0])), shape[i]
        J = float(a["d32"].astype(np.float64).sum())
        assert abs(float(host(st.distortion[i])[0]) - J) <= 1e-9 * J, shape[i]
        assert abs(float(host(st.distortion[i])[1]) - J) <= 1e-9 * J, shape[i]
