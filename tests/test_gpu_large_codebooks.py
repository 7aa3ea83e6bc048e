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


def best_us(f, reps=5):
    f()
    torch.cuda.synchronize()
    best = np.inf
    for _ in range(reps):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        f()
        b.record()
        b.synchronize()
        best = min(best, 1e3 * a.elapsed_time(b))
    return best


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


# sizes at the edges of the kernels' variants: 1024 | 1025 entries (three bf16 terms | one fp16
# term), 1920 | 1921 (fp32 rows in LDS | in memory), 2048 | 2049 (segments of 256 | 512 entries),
# 4864 | 4865 (resident | streamed), a last segment of one tile or one entry, and kernel counts
# with several waves per unit and one wave per unit (more units per wave: the next test)
EDGES = [(1000, 1024), (1000, 1025), (64 * 300, 1025), (1000, 1920), (1000, 1921), (700, 2048), (700, 2049),
         (64 * 300 + 1, 2049), (500, 2561), (500, 4864), (500, 4865), (64 * 260, 4865), (300, 9217)]


def laplace(n, seed):
    return np.random.default_rng(seed).laplace(0.0, 0.05, (n, 9)).astype(np.float32)


def check_assign(X, C, tag):
    a = oracle.assign(X, C)
    idx, bd, J = kq.kq_assign(dev(X), dev(C))
    bad = np.nonzero(host(idx) != a["idx"])[0]
    assert bad.size == 0, (tag, bad.size, bad[:4], host(idx)[bad[:4]], a["idx"][bad[:4]])
    assert np.array_equal(host(bd).view(np.uint32), a["d32"].view(np.uint32)), tag
    Jr = float(a["d32"].astype(np.float64).sum())
    assert not np.isfinite(Jr) or abs(float(host(J)[0]) - Jr) <= 1e-9 * abs(Jr), tag


@pytest.mark.parametrize("n,k", EDGES)
def test_assign_at_the_edges_of_the_variants(n, k):
    X = laplace(n, n + k)
    check_assign(X, synth.random_codebook_state(X, k, k), (n, k))


@pytest.mark.parametrize("n,k", [(64 * 256 * 13 + 5, 1500), (64 * 256 * 13 + 5, 2303), (64 * 256 * 13 + 5, 4865),
                                 (64 * 256 * 30 + 63, 4096), (64 * 256 * 97 + 1, 4865), (64 * 256 * 97 + 1, 9217)])
def test_assign_of_many_units_per_workgroup(n, k):
    """More than 12 units for a workgroup's 12 waves (the next unit handed out, its kernels loaded ahead; a
    streaming wave's later units), and more than the 96 that streaming waves keep (the codebook streams
    again).  The kernels repeat a block of 4099, so the oracle decides that block only."""
    X = laplace(4099, n + k)
    C = synth.random_codebook_state(X, k, k)
    a = oracle.assign(X, C)
    i = torch.arange(n, device=DEV) % 4099
    idx, bd, J = kq.kq_assign(dev(X)[i], dev(C))
    assert torch.equal(idx, dev(a["idx"]).to(torch.int32)[i])
    assert torch.equal(bd, dev(a["d32"])[i])
    Jr = float(a["d32"].astype(np.float64)[np.arange(n) % 4099].sum())
    assert abs(float(host(J)[0]) - Jr) <= 1e-9 * Jr


@pytest.mark.parametrize("n,k", [(4096, 60), (5000, 256), (20000, 512), (64 * 300 + 5, 1024)])
def test_the_two_assignments_agree(n, k):
    """A codebook of at most 1024 entries beside a larger one goes through the larger one's kernel: the
    same indices and distances as alone, bit for bit, near ties among them."""
    X, C = layer(n, k, 300 + k)
    C[k // 2:k // 2 + 8] = np.nextafter(C[:8], np.float32(np.inf))
    Y, D = layer(700, 1100, 5)
    st = kq.Stack([dev(X), dev(Y)], [dev(C), dev(D)], best_d=True)
    kq.kq_assign_stack(st)
    idx, bd, _ = kq.kq_assign(dev(X), dev(C))
    assert torch.equal(st.idx[0], idx) and torch.equal(st.best_d[0], bd)


@pytest.mark.parametrize("k", [1500, 3000, 5000])
def test_assign_near_ties_and_scales(k):
    """What the fp16 screening cannot tell apart: copied entries, entries one unit in the last
    place from each other, a codebook whose entries span many magnitudes, kernels far larger and
    far smaller than the codebook, exact hits."""
    rng = np.random.default_rng(k)
    X = laplace(1200, k)
    C = X[rng.integers(0, 1200, k)].copy()                      # copies and exact hits
    C[::3] = np.nextafter(C[::3], np.float32(np.inf))
    check_assign(X, C, "copies")
    C = synth.random_codebook_state(X, k, k) * (10.0 ** rng.uniform(-12, 6, (k, 1))).astype(np.float32)
    check_assign(X, C, "spread codebook")
    Y = X * (10.0 ** rng.uniform(-20, 12, (1200, 1))).astype(np.float32)
    check_assign(Y, synth.random_codebook_state(X, k, k), "spread kernels")
    for s in (1e-30, 1e-18, 1e9, 1e17):
        check_assign(X * np.float32(s), synth.random_codebook_state(X, k, k) * np.float32(s), f"scale {s}")


@pytest.mark.parametrize("k", [1500, 5000])
def test_assign_extreme_values(k):
    rng = np.random.default_rng(k)
    X = laplace(300, k)
    C = synth.random_codebook_state(X, k, k)
    for name, v in [("huge entry", 3e38), ("infinite entry", np.inf), ("zero codebook", None)]:
        D = C.copy()
        if v is None:
            D[:] = 0
        else:
            D[rng.integers(0, k, 5)] = v
        check_assign(X, D, name)
    Z = X.copy()
    Z[::7] = 0
    Z[3] = 1e-45
    check_assign(Z, C, "zero kernels")
    Z[5] = 3e38
    check_assign(Z, C, "huge kernel")


@pytest.mark.parametrize("k", [1500, 3000, 5000])
def test_assign_with_far_entries(k):
    """A few entries whose size would take the scale from the others: their exponents just below and
    above where entries count as far, and at the ends of the range, kernels that lie at them, next to
    them and midway, entries of zeros, and far entries only in one wave's part of the codebook."""
    rng = np.random.default_rng(k)
    X = laplace(1500, k)
    C = synth.random_codebook_state(X, k, k)
    top = float(2.0 ** np.floor(np.log2(np.abs(C).max())))
    for name, sizes in [("edge", top * 2.0 ** np.arange(10, 16)), ("one step", [top * 4096 * 1.99, top * 8192 * 1.01]),
                        ("huge", [1e10, 1e30, 3e38]), ("not finite", [np.inf, np.nan, 1e20]), ("tiny others", [1e25])]:
        D, Y = C.copy(), X.copy()
        if name == "tiny others":
            D[:, :], Y = D * np.float32(1e-25), Y * np.float32(1e-25)
        at = rng.integers(0, 64, len(sizes)) + 64 * rng.integers(0, 3)
        for j, v in zip(at, sizes):
            D[j] = np.float32(v) * rng.choice([-1.0, 1.0], 9).astype(np.float32)
            if np.isfinite(v):
                rows = rng.integers(0, 1500, 12)
                Y[rows[:4]] = D[j] * np.float32(0.4)
                Y[rows[4:8]] = D[j] * np.float32(0.6)
                Y[rows[8:]] = D[j]
        D[k // 2:k // 2 + 300] = 0
        check_assign(Y, D, (k, name))


@pytest.mark.parametrize("k", [1500, 4096])
def test_assign_with_one_far_entry_takes_no_longer(k):
    """(with the scale from the largest entry, whatever its size, up to ten times as long)"""
    g = torch.Generator(device=DEV)
    g.manual_seed(k)
    X = torch.randn(131072, 9, device=DEV, generator=g)
    C = X[:k].clone()
    plain = best_us(lambda: kq.kq_assign(X, C))
    for v in (1e3, 1e4, 1e30, float("inf"), float("nan")):
        D = C.clone()
        D[k // 2] = v
        us = best_us(lambda: kq.kq_assign(X, D))
        assert us <= 1.6 * plain, (v, us, plain)
    S = X * torch.exp(2 * torch.randn(131072, 1, device=DEV, generator=g))   # kernels of all sizes
    us = best_us(lambda: kq.kq_assign(S, S[:k].clone()))
    assert us <= 1.6 * plain, (us, plain)


@pytest.mark.parametrize("bits", [2, 6])
def test_wide_codebooks_share_their_launches(bits):
    """Codebooks of at least 16384 scalars of several sizes, some weights zero: together (the
    queried workspace), one after another (a workspace for the largest alone) and in one workgroup
    each give the same codes and levels; more of them than one sequence of launches takes."""
    rng = np.random.default_rng(bits)
    ks = [1821, 3000, 1900, 100, 4096] + [1830 + i for i in range(14)]
    Cs = [dev(rng.laplace(0, 0.03, (k, 9)).astype(np.float32)) for k in ks]
    ws = [dev(rng.integers(0, 50, k).astype(np.int32)) for k in ks]
    one = kq.kq_quantize_codebook_stack(Cs, ws, bits, wide=False)
    together = kq.kq_quantize_codebook_stack(Cs, ws, bits)
    arr = (kq.KqCbqLayer * 1)(kq.KqCbqLayer(Cs[4].data_ptr(), 4096, None, None, None, None))
    least = kq.lib.kq_quantize_codebook_stack_workspace_bytes(arr, 1, bits)
    alone = kq.kq_quantize_codebook_stack(Cs, ws, bits, workspace=torch.empty(least, dtype=torch.uint8, device=DEV))
    for a, b, c in zip(one, together, alone):
        for x, y, z in zip(a, b, c):
            assert torch.equal(x.view(torch.uint8), y.view(torch.uint8))
            assert torch.equal(x.view(torch.uint8), z.view(torch.uint8))


# one launch updates layers of at most 16384 kernels and 4096 entries, with about 2048 kernels to 16
# entries at most; beyond, the general path
SMALL_UPDATES = [[(2048, 16)], [(2049, 16)], [(2048, 1)], [(16384, 128)], [(16384, 127)], [(1, 1)], [(16384, 300)], [(16385, 300)], [(16384, 4096)], [(4096, 4097)], [(8191, 1000), (100, 17), (700, 513)]]


@pytest.mark.parametrize("shape", SMALL_UPDATES)
def test_update_of_small_layers(shape):
    """Counts, means and distortion after an assignment, through the stack calls and through a fit
    (bit for bit the separate update's), with entries that have no kernels."""
    layers = [layer(n, k, 40 + i) for i, (n, k) in enumerate(shape)]
    st = kq.Stack([dev(X) for X, _ in layers], [dev(C) for _, C in layers], iters=2)
    kq.kq_assign_stack(st, distortion=False)
    before = [c.clone() for c in st.C]
    kq.kq_update_stack(st, dist_slot=1, distortion_from_assign=True)
    for i, (X, C) in enumerate(layers):
        idx = host(st.idx[i])
        assert np.array_equal(idx, oracle.assign(X, C)["idx"])
        Cn, z, _ = kq.kq_update(st.X[i], st.idx[i], before[i])       # sums by the general path
        assert torch.equal(st.counts[i], z) and torch.equal(st.C[i], Cn), shape[i]
        oC, oz = oracle.update(X, idx, C)
        assert np.array_equal(host(st.counts[i]), oz)
        err = np.abs(host(st.C[i]).astype(np.float64) - oC).max(axis=1)
        assert (err <= 1e-5 * np.maximum(np.abs(oC).max(axis=1), 1e-300)).all(), shape[i]
        if C.shape[0] <= X.shape[0]:
            gC, gi, gz, gJ = kq.kq_fit_layer(st.X[i], dev(C), 2)
            D = dev(C)
            for _ in range(2):
                a = kq.kq_assign(st.X[i], D)[0]
                D = kq.kq_update(st.X[i], a, D)[0]
            a, _, J = kq.kq_assign(st.X[i], D)
            assert torch.equal(gC, D) and torch.equal(gi, a) and torch.equal(gJ[-1:], J), shape[i]
            assert np.array_equal(host(gz), np.bincount(host(a), minlength=C.shape[0]))


@pytest.mark.parametrize("k", [64, 200, 800, 1500, 3000, 5000])
def test_rescans_of_any_number_of_kernels(k):
    """Units of 64 kernels of which 0 to 64 are copies of an entry that the codebook holds twice: the
    screening cannot settle those, and the lower index wins whether they are rescored by four or alone."""
    rng = np.random.default_rng(k)
    counts = [0, 1, 2, 3, 4, 5, 7, 8, 9, 63, 64, 30]
    X = laplace(64 * len(counts) - 5, k)
    C = synth.random_codebook_state(X, k, k)
    pairs = rng.permutation(k)[:40].reshape(20, 2)
    C[pairs[:, 1]] = C[pairs[:, 0]]
    for u, c in enumerate(counts):
        rows = 64 * u + rng.permutation(64 if u + 1 < len(counts) else 59)[:c]
        X[rows] = C[pairs[rng.integers(0, 20, c), 0]]
    check_assign(X, C, k)


def test_assign_of_near_ties_by_four():
    """Kernels around an offset of ten times their deviation: nearly all are rescored over the whole
    codebook (one by one thirteen times as long as without the offset, by four five times)."""
    k = 4096
    g = torch.Generator(device=DEV)
    g.manual_seed(k)
    X = torch.randn(131072, 9, device=DEV, generator=g)
    plain = best_us(lambda: kq.kq_assign(X, X[:k].clone()))
    Y = X + 10.0
    C = Y[:k].clone()
    us = best_us(lambda: kq.kq_assign(Y, C))
    assert us <= 8.0 * plain, (us, plain)


# members of one workgroup's entries at the edge where a frequent entry is added in registers (3072)
@pytest.mark.parametrize("n,k,share", [(3071, 200, 1.0), (3072, 200, 1.0), (3073, 200, 1.0), (16384, 300, 0.99), (16384, 300, 0.4),
                                       (16384, 300, 0.2), (12289, 4096, 0.9), (16000, 130, 0.7), (16384, 1024, 1.0)])
def test_update_of_small_layers_with_a_frequent_entry(n, k, share):
    """The one-launch update against the general one, bit for bit, with indices of which one entry has
    a large share, at both ends of its workgroup's entries and with another frequent one beside it."""
    X, C = layer(n, k, n + k)
    st = kq.Stack([dev(X)], [dev(C)], iters=2)
    rng = np.random.default_rng(k)
    for entry in (0, 15 if k > 15 else k - 1, k - 1):
        idx = rng.integers(0, k, n).astype(np.int32)
        frequent = rng.random(n) < share
        idx[frequent] = entry
        idx[frequent & (rng.random(n) < 0.2)] = max(entry - 1, 0)
        kq.kq_assign_stack(st)
        st.idx[0].copy_(dev(idx))
        st.set_codebooks([dev(C)])
        Cn, z, _ = kq.kq_update(st.X[0], st.idx[0], dev(C))
        for counts_only in (False, True):
            kq.kq_update_stack(st, distortion_from_assign=True, counts_only=counts_only)
            assert np.array_equal(host(st.counts[0]), np.bincount(idx, minlength=k)) and torch.equal(st.counts[0], z)
            assert np.array_equal(host(st.C[0]).view(np.uint32), host(Cn).view(np.uint32)), entry


def test_fit_of_a_small_layer_with_many_zero_kernels():
    """(with an atomic per member and value: three times as long as without zeros)"""
    X, C = layer(16384, 256, 7)
    Z = X.copy()
    Z[np.random.default_rng(1).random(16384) < 0.9] = 0
    C[0] = 0
    X, Z, C = dev(X), dev(Z), dev(C)
    plain, zeros = best_us(lambda: kq.kq_fit_layer(X, C, 20)), best_us(lambda: kq.kq_fit_layer(Z, C, 20))
    assert zeros <= 2.2 * plain, (zeros, plain)


def test_fits_of_mixed_small_layers():
    """A layer with many kernels and few entries beside one that takes the one-launch update: as long as
    both alone at most (the first in that launch too: half as long again as both)."""
    made = [layer(16384, 16, 1), layer(4096, 300, 2)]
    st = kq.Stack([dev(X) for X, _ in made], [dev(C) for _, C in made], iters=20)

    def both():
        st.set_codebooks(start)
        kq.kq_fit_stack(st, 20)

    start = [c.clone() for c in st.C]
    alone = [best_us(lambda i=i: kq.kq_fit_layer(st.X[i], start[i], 20)) for i in range(2)]
    together = best_us(both)
    assert together <= sum(alone), (together, alone)
    for i in range(2):
        C, idx, z, _ = kq.kq_fit_layer(st.X[i], start[i], 20)
        assert torch.equal(C, st.C[i]) and torch.equal(idx, st.idx[i]) and torch.equal(z, st.counts[i])


# runs of few units: one to six per workgroup, several waves per unit, and k at the edges
@pytest.mark.parametrize("n,k", [(64, 300), (100, 257), (4096, 600), (64 * 256 * 2, 700), (64 * 256 * 3 + 5, 1024),
                                 (64 * 256 * 7, 300), (1, 1024)])
def test_assign_several_waves_per_unit(n, k):
    X = laplace(n, n + k)
    check_assign(X, synth.random_codebook_state(X, k, k), (n, k))
    C = X[np.random.default_rng(n).integers(0, n, k)].copy()       # copies: exact ties
    check_assign(X, C, (n, k, "copies"))


# (the last three: chunks of several tiles of 4096 indices, the last tile ragged)
@pytest.mark.parametrize("n,k", [(4095, 769), (4097, 1537), (8193, 7679), (40001, 2305), (262145, 4096), (300001, 7679),
                                 (1048577, 2000)])
def test_update_over_several_ranges(n, k):
    """The listed sums (no distortion asked for) and the sums in the order of the rows are the same
    integers: codebooks and counts bit for bit, with indices to ignore, an entry that holds every
    other kernel and entries without any."""
    X, C = layer(n, k, 70 + k)
    idx = synth.random_indices(n, k, 71)
    idx[::2] = k - 1
    idx[1:40:4], idx[3:40:4] = -1, k
    idx[idx == 5] = 6
    rows = kq.kq_update(dev(X), dev(idx), dev(C))
    listed = kq.kq_update(dev(X), dev(idx), dev(C), with_distortion=False)
    want = np.bincount(idx[(idx >= 0) & (idx < k)], minlength=k)
    assert np.array_equal(host(listed[1]), want) and np.array_equal(host(rows[1]), want)
    assert np.array_equal(host(listed[0]).view(np.uint32), host(rows[0]).view(np.uint32))
    assert np.array_equal(host(listed[0])[want == 0], C[want == 0])


def test_update_finish_of_many_entries():
    """Three large codebooks finished in one launch (96 entries a workgroup) and one by one (16)."""
    sizes = [(8193, 7679), (9000, 5000), (18001, 6001)]
    made = [layer(n, k, 80 + i) for i, (n, k) in enumerate(sizes)]
    st = kq.Stack([dev(X) for X, _ in made], [dev(C) for _, C in made])
    for i, (n, k) in enumerate(sizes):
        st.idx[i].copy_(dev(synth.random_indices(n, k, 90 + i)))
    alone = [kq.kq_update(st.X[i], st.idx[i], st.C[i], with_distortion=False)[:2] for i in range(3)]
    kq.kq_update_stack(st)
    for i in range(3):
        assert np.array_equal(host(st.counts[i]), host(alone[i][1]))
        assert np.array_equal(host(st.C[i]).view(np.uint32), host(alone[i][0]).view(np.uint32))


@pytest.mark.parametrize("k", [456, 910, 911, 1366, 1820, 1821])
def test_quantize_codebook_exact_rounds_of_larger_codebooks(k):
    """6-bit weighted k-means of 4104 to 16389 scalars, bit for bit the oracle's: around the sizes
    held with a weight per scalar (8192) and with a weight per entry (16384), zero and huge weights,
    few distinct values (equal levels), a value too small for the exact rounds."""
    rng = np.random.default_rng(k)
    laplace = rng.laplace(0, 0.03, (k, 9)).astype(np.float32)
    laplace[np.abs(laplace) < 1e-6] = 0.0
    w = rng.integers(0, 300, k)
    w[::5] = 0
    tiny = laplace.copy()
    tiny[k // 2, 4] = np.float32(1e-12)
    cases = [(laplace, w), (laplace, rng.integers(1, (1 << 31) - 1, k)), (tiny, w),
             (rng.choice(np.float32([-1, 0.5, 3]), (k, 9)), rng.integers(1, 9, k))]
    for i, (C, w) in enumerate(cases):
        codes, levels, C_hat = kq.kq_quantize_codebook(dev(C), dev(w.astype(np.int32)), 6, kq.KQ_CBQ_WKMEANS, 30)
        oc, ol, oh, _ = oracle.cbq_wkmeans(C, w, 6, 30)
        assert np.array_equal(host(codes), oc), i
        assert np.array_equal(host(levels).view(np.uint32), ol.view(np.uint32)), i
        assert np.array_equal(host(C_hat).view(np.uint32), oh.view(np.uint32)), i
