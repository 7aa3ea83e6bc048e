"""GPU parity of the large-set scalar quantizer (the fully-connected layers, end of
Sec. 3.2) through the C ABI.  Every step is exact or correctly rounded, so codes,
levels, dequantised values and the number of rounds are bit-exact against the oracle
and against the single-workgroup codebook quantizer with unit weights; at the full
VGG-16 fc6 size (too large for the oracle) the result is checked by properties that fix
it: every level is the correctly rounded mean of its scalars, every sampled code is the
nearest level, and a run that stopped early is a fixed point."""
import math

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


def data(kind, m, seed):
    rng = np.random.default_rng(seed)
    if kind == "normal":
        return (rng.standard_normal(m) * 0.01).astype(np.float32)
    if kind == "heavy":
        v = rng.laplace(0.0, 0.003, m)
        v[rng.choice(m, max(1, m // 500), replace=False)] *= 40.0
        return v.astype(np.float32)
    if kind == "constant":
        return np.full(m, -0.375, np.float32)
    if kind == "integers":                     # exact ties and midpoints between levels
        return rng.integers(-40, 41, m).astype(np.float32)
    if kind == "outliers":                      # a few far values: many thresholds share a bucket
        v = 1.0 + rng.standard_normal(m) * 0.01  # (no tiny values, so thresholds are allowed)
        v[rng.choice(m, min(m, 8), replace=False)] = rng.choice([-500.0, 500.0], min(m, 8))
        return v.astype(np.float32)
    if kind == "pruned":                        # one value (a zero of either sign) nearly everywhere
        v = rng.standard_normal(m).astype(np.float32)
        v[rng.random(m) < 0.995] = 0.0
        v[::97] *= -1.0
        return v
    if kind == "floor":                         # the most frequent value is the smallest
        return np.maximum(rng.standard_normal(m), 0.5).astype(np.float32)
    if kind == "spikes":                        # two frequent values, one of them far out, and a spread
        v = (rng.standard_normal(m) * 0.1).astype(np.float32)
        v[rng.random(m) < 0.4] = 0.05
        v[rng.random(m) < 0.1] = 7.0
        return v
    if kind == "tiny":                          # subnormal and zero values among normal ones
        v = (rng.standard_normal(m) * 1e-3).astype(np.float32)
        v[::7] = np.float32(3e-42)
        v[::11] = 0.0
        return v
    raise ValueError(kind)


def check(v, bits, iters, tag):
    oc, ol, ov, orr = oracle.quantize_scalars(v, bits, iters)
    for search in ("auto", "thresholds"):   # the exact search below 3 * 2^20, and the threshold path
        codes, levels, v_hat, rounds = kq.kq_quantize_scalars(dev(v), bits, iters, search=search)
        assert np.array_equal(host(codes), oc), (tag, search)
        assert np.array_equal(host(levels).view(np.uint32), ol.view(np.uint32)), (tag, search)
        assert np.array_equal(host(v_hat).view(np.uint32), ov.view(np.uint32)), (tag, search)
        assert int(host(rounds)[0]) == orr, (tag, search)


@pytest.mark.parametrize("m", [1, 2, 9, 1000, 65537])
@pytest.mark.parametrize("kind", ["normal", "heavy", "integers", "tiny", "outliers"])
def test_fc_quantizer_bit_exact(m, kind):
    check(data(kind, m, m + len(kind)), 6, 30, f"{kind} m={m}")


@pytest.mark.parametrize("bits,iters", [(1, 30), (2, 5), (6, 0), (6, 1), (8, 30)])
def test_fc_quantizer_widths_and_rounds(bits, iters):
    check(data("heavy", 30001, bits * 100 + iters), bits, iters, f"bits={bits} iters={iters}")
    check(data("constant", 500, 1), bits, iters, "constant")


def test_fc_quantizer_equals_codebook_quantizer_with_unit_weights():
    v = data("normal", 9 * 900, 5)
    a = kq.kq_quantize_scalars(dev(v), 6, 30)
    C = dev(v.reshape(-1, 9))
    w = torch.ones(900, dtype=torch.int32, device=DEV)
    codes, levels, C_hat = kq.kq_quantize_codebook(C, w, 6, kq.KQ_CBQ_WKMEANS, 30)
    assert torch.equal(a[0], codes.reshape(-1)) and torch.equal(a[1], levels)
    assert torch.equal(a[2], C_hat.reshape(-1))


def test_fc_quantizer_full_size_fc6_properties():
    """VGG-16 fc6 (4096 x 25088 = 102,760,448 scalars, N(0, sqrt(2/25088)))."""
    m = 4096 * 25088
    g = torch.Generator(device=DEV)
    g.manual_seed(6)
    v = torch.randn(m, device=DEV, generator=g) * math.sqrt(2.0 / 25088)
    codes, levels, v_hat, rounds = kq.kq_quantize_scalars(v, 6, 30)
    c, L, r = host(codes), host(levels), int(host(rounds)[0])
    x = host(v)
    assert 1 <= r <= 30
    # the last codes are always computed against the final levels: nearest, lowest on ties
    rows = np.random.default_rng(3).choice(m, 20000, replace=False)
    near = np.argmin(np.abs(x[rows].astype(np.float64)[:, None] - L.astype(np.float64)[None, :]), axis=1)
    assert np.array_equal(c[rows], near)
    assert np.array_equal(host(v_hat)[rows], L[c[rows]])
    if r < 30:  # stopped early: a fixed point, every level the correctly rounded mean of its scalars
        for q in np.linspace(0, 63, 9).astype(int):
            mem = x[c == q].astype(np.float64)
            if mem.size:
                assert L[q] == np.float32(math.fsum(mem.tolist()) / mem.size), q


# Where v_hat goes decides who takes a large set: its own tensor gives room for the partitioned copy,
# none ("absent") or v itself ("in place") leaves the coding launches, whose threshold form serves
# sets from 3 * 2^20 scalars on
def quantize_to(v, bits, iters, where, **kw):
    if where == "own":
        return kq.kq_quantize_scalars(v, bits, iters, **kw)
    if where == "absent":
        c, l, _, r = kq.kq_quantize_scalars(v, bits, iters, want_v_hat=False, **kw)
        return c, l, l[c.long()], r
    w = v.clone()
    return kq.kq_quantize_scalars(w, bits, iters, v_hat=w, **kw)


def same_as_exact(v, bits, iters, where, tag, **kw):
    a = quantize_to(v, bits, iters, where, **kw)
    b = kq.kq_quantize_scalars(v, bits, iters, search="exact")
    for x, y, name in zip(a, b, ["codes", "levels", "v_hat", "rounds"]):
        assert torch.equal(x.view(torch.uint8), y.view(torch.uint8)), (tag, where, name)


@pytest.mark.parametrize("where", ["own", "absent", "in place"])
@pytest.mark.parametrize("kind", ["normal", "integers", "tiny", "outliers"])
def test_fc_threshold_path_equals_the_exact_search(kind, where):
    """From 3 * 2^20 scalars on, codes come from per-level thresholds (a bucket table over
    the data range, fp32 comparisons), on the set partitioned by value or in the coding launches; with
    KQ_F_EXACT_SEARCH every code comes from the exact fp64 search.  They agree bit for bit, also on
    integer data (exact midpoints between levels), on data whose tiny values make fp64 distances inexact
    and on data with a few far values, where most thresholds fall into one bucket and are compared one by
    one."""
    m = 9 * 932068                                            # 8,388,612 >= 3 * 2^20
    same_as_exact(dev(data(kind, m, 77)), 6, 30, where, kind)


@pytest.mark.parametrize("where", ["absent", "in place"])
@pytest.mark.parametrize("bits", [1, 2, 3, 4, 5, 7, 8])
def test_fc_threshold_coding_launches_of_other_widths(bits, where):
    """(several steps of the grid, the last one ragged, and a set that begins off a 16-byte boundary)"""
    v = dev(data("heavy", 4 * (512 * 1024 + 7) * 2 + 1, bits))
    same_as_exact(v, bits, 6, where, bits)
    same_as_exact(v[1:], bits, 6, where, bits)


def test_fc_narrow_codes_of_a_large_set_with_v_hat():
    """1 and 2 bits are never partitioned: thresholds in the coding launches, v_hat given."""
    v = dev(data("heavy", 4 * (512 * 1024 + 7) * 2 + 3, 1))
    for bits in (1, 2):
        same_as_exact(v, bits, 30, "own", bits)


@pytest.mark.parametrize("bits", [1, 2, 3, 6])
@pytest.mark.parametrize("m", [64, 5001])
def test_fc_thresholds_with_values_far_below_the_levels(m, bits):
    """Values down to the smallest subnormal between levels that lie symmetrically around zero:
    their fp64 distances to both levels round to the same number, and the tie goes to the
    lower level; the thresholds (and the exact search) must code them alike."""
    rng = np.random.default_rng(m + bits)
    v = rng.choice([-0.5, -0.25, 0.25, 0.5], m).astype(np.float32)
    tiny = rng.random(m) < 0.4
    e = rng.uniform(-45.0, -9.0, int(tiny.sum()))
    v[tiny] = (rng.choice([-1.0, 1.0], e.size) * 10.0 ** e).astype(np.float32)
    v[:4] = [0.0, -0.0, 1e-45, -1e-45]
    check(v, bits, 30, f"m={m} bits={bits}")
    check(np.concatenate([v, -v]), bits, 30, f"symmetric m={m} bits={bits}")


@pytest.mark.parametrize("where", ["own", "absent", "in place"])
@pytest.mark.parametrize("groups", [1, 5, 63, 65, 129, 600, 512 * 1024 + 7, 2 * 512 * 1024 + 7])
def test_fc_threshold_rounds_with_a_partial_last_wave(groups, where):
    """Sets whose last wave holds fewer than 64 groups of four scalars, with many codes changing
    there: every change must move its level's sums (the count of a wave's queued changes has to
    agree in all its lanes, also in those past the end).  The larger ones take one and two whole steps
    of the coding launches' grid before (with a v_hat of their own they are partitioned instead)."""
    m = 4 * groups
    v = data("heavy", m, groups)
    v[-min(m, 256):] = np.random.default_rng(1).uniform(-0.02, 0.02, min(m, 256)).astype(np.float32)
    vd = dev(v)
    for iters in (1, 2, 3, 30):
        same_as_exact(vd, 6, iters, where, (groups, iters), search="thresholds")


@pytest.mark.parametrize("kind", ["symmetric", "late", "integers", "constant", "two", "heavy", "outliers", "tiny",
                                  "pruned", "floor", "spikes"])
@pytest.mark.parametrize("bits", [6, 8])
def test_fc_partitioned_rounds(kind, bits):
    """Rounds on the set partitioned by value (thresholds asked for, v_hat given): against the
    oracle at sizes with a ragged last tile; values far below the others
    ("symmetric", "late"; the rounds that go over to full scans have tests of their own below); a
    frequent value; few distinct values (buckets of one value, empty
    buckets); values at every scale."""
    m = 70001
    rng = np.random.default_rng(bits)
    if kind == "symmetric":
        v = rng.choice([-1.0, -1e-30, 1e-30, 1.0], m).astype(np.float32)
    elif kind == "late":
        v = (rng.standard_normal(m) * 0.1).astype(np.float32)
        v[::2] = (rng.choice([-1.0, 1.0], v[::2].size) * 10.0 ** rng.uniform(-40, -25, v[::2].size)).astype(np.float32)
        v = np.concatenate([v, -v])[:m]
    elif kind == "two":
        v = rng.choice([0.25, 0.75], m).astype(np.float32)
    else:
        v = data(kind, m, 3)
    for iters in (0, 2, 30):
        oc, ol, ov, orr = oracle.quantize_scalars(v, bits, iters)
        for u in (dev(v), dev(np.concatenate([[np.float32(0)], v]))[1:]):   # aligned to 16 bytes, and not
            codes, levels, v_hat, rounds = kq.kq_quantize_scalars(u, bits, iters, search="thresholds")
            assert np.array_equal(host(levels).view(np.uint32), ol.view(np.uint32)), (kind, bits, iters)
            assert np.array_equal(host(codes), oc), (kind, bits, iters)
            assert np.array_equal(host(v_hat).view(np.uint32), ov.view(np.uint32)), (kind, bits, iters)
            assert int(host(rounds)[0]) == orr, (kind, bits, iters)


def test_fc_without_and_in_place_of_v_hat():
    """Without v_hat there is no room for the partitioned copy, in place it would overwrite the
    set: both take the coding launches, with the same codes and levels."""
    m = 9 * 100003
    v = dev(data("normal", m, 8))
    a = kq.kq_quantize_scalars(v, 6, 30)
    b = kq.kq_quantize_scalars(v, 6, 30, want_v_hat=False)
    w = v.clone()
    c = kq.kq_quantize_scalars(w, 6, 30, v_hat=w)
    for x, y in ((a, b), (a, c)):
        assert torch.equal(x[0], y[0]) and torch.equal(x[1], y[1]) and torch.equal(x[3], y[3])
    assert torch.equal(a[2], w)


@pytest.mark.parametrize("bits", [3, 4, 5, 7])
@pytest.mark.parametrize("kind", ["normal", "heavy", "integers", "tiny"])
def test_fc_partitioned_rounds_of_other_widths(kind, bits):
    v = dev(data(kind, 786432 + 5, bits))                     # partitioned without being asked for
    for iters in (3, 30):
        a = kq.kq_quantize_scalars(v, bits, iters)
        b = kq.kq_quantize_scalars(v, bits, iters, search="exact")
        for x, y, name in zip(a, b, ["codes", "levels", "v_hat", "rounds"]):
            assert torch.equal(x.view(torch.uint8), y.view(torch.uint8)), (kind, bits, iters, name)


def best_us(f, reps=5):
    f()
    torch.cuda.synchronize()
    best = math.inf
    for _ in range(reps):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        f()
        b.record()
        b.synchronize()
        best = min(best, 1e3 * a.elapsed_time(b))
    return best


@pytest.mark.parametrize("kind", ["pruned", "floor", "spikes"])
def test_fc_partitioned_rounds_with_a_frequent_value(kind):
    """A value that holds much of the set has a bucket of its own, which no round reads: the same
    codes and levels as the exact search, and the rounds do not take longer than it (with the value's
    neighbours in its bucket, four times as long)."""
    v = dev(data(kind, 4 * 1024 * 1024 + 3, 5))
    a = kq.kq_quantize_scalars(v, 6, 30)
    b = kq.kq_quantize_scalars(v, 6, 30, search="exact")
    for x, y, name in zip(a, b, ["codes", "levels", "v_hat", "rounds"]):
        assert torch.equal(x.view(torch.uint8), y.view(torch.uint8)), (kind, name)
    auto = best_us(lambda: kq.kq_quantize_scalars(v, 6, 30, *a))
    exact = best_us(lambda: kq.kq_quantize_scalars(v, 6, 30, *b, search="exact"))
    assert auto <= 1.5 * exact, (kind, auto, exact)


def close_levels(m, bits, late=False):
    """Half of the values near 1e-16 of the others: the two middle levels, which start the same way off
    zero, end closer than thresholds allow (2^-50 of the largest magnitude) while the outer ones still
    move.  From the first update on, or `late`: from the second, once they have lost the values near
    the edge of their first range.  The set is its own mirror image (m even), so that the middle levels
    stay the same way off zero."""
    rng = np.random.default_rng(bits)
    n = 1 << bits
    m //= 2
    v = rng.uniform(-1.0, 1.0, m) * (n - 1) / n
    v = np.where(np.abs(v) < 4.0 / n, np.sign(v) * 4.5 / n, v)
    tiny = rng.random(m) < 0.5
    v[tiny] = rng.choice([-1.0, 1.0], int(tiny.sum())) * rng.uniform(5e-17, 3e-16, int(tiny.sum()))
    if late:
        edge = rng.random(m) < 0.1
        v[edge] = rng.choice([-2.1, -1.9, 1.9, 2.1], int(edge.sum())) / n
    v[0] = (n - 1) / n                          # the first levels: odd multiples of 1 / n
    return np.concatenate([v, -v]).astype(np.float32)


def first_close_update(v, bits, iters):
    """The first update after which two levels are too close for thresholds, by the oracle."""
    apart = 2.0 ** -50 * float(np.abs(v).max())
    for it in range(1, iters + 1):
        gap = np.diff(oracle.quantize_scalars(v, bits, it)[1].astype(np.float64))
        if (gap[gap != 0] < apart).any():
            return it
    return None


@pytest.mark.parametrize("bits", [3, 4, 5, 6, 7, 8])
@pytest.mark.parametrize("late", [False, True])
def test_fc_full_scan_rounds_move_what_changed(bits, late):
    """Rounds after the thresholds were given up: the first full scan forms the sums, the later ones
    move the changes; ending with, one after and several after the first such update."""
    v = close_levels(131072 + 78, bits, late)
    first = first_close_update(v, bits, 4)
    assert first == (2 if late else 1)                       # (the fallback is what runs)
    for iters in (first, first + 1, first + 7):
        oc, ol, ov, orr = oracle.quantize_scalars(v, bits, iters)
        codes, levels, v_hat, rounds = kq.kq_quantize_scalars(dev(v), bits, iters, search="thresholds")
        assert np.array_equal(host(levels).view(np.uint32), ol.view(np.uint32)), iters
        assert np.array_equal(host(codes), oc), iters
        assert np.array_equal(host(v_hat).view(np.uint32), ov.view(np.uint32)), iters
        assert int(host(rounds)[0]) == orr, iters


def test_fc_full_scan_rounds_take_no_longer_than_the_exact_search():
    """(by a scan of all levels and whole sums in every round several times as long)"""
    v = dev(close_levels(8_000_010, 6))
    a = kq.kq_quantize_scalars(v, 6, 30)
    b = kq.kq_quantize_scalars(v, 6, 30, search="exact")
    gap = np.diff(host(a[1]).astype(np.float64))
    assert 0 < gap[gap > 0].min() < 2.0 ** -50 and int(host(a[3])[0]) > 10   # (the fallback is what runs)
    for x, y, name in zip(a, b, ["codes", "levels", "v_hat", "rounds"]):
        assert torch.equal(x.view(torch.uint8), y.view(torch.uint8)), name
    auto = best_us(lambda: kq.kq_quantize_scalars(v, 6, 30, *a), 3)
    exact = best_us(lambda: kq.kq_quantize_scalars(v, 6, 30, *b, search="exact"), 3)
    assert auto <= 2.0 * exact, (auto, exact)


@pytest.mark.parametrize("m,iters", [(1_000_003, 0), (1_000_003, 1), (1_000_003, 5), (4_096_000, 1), (4_096_000, 2)])
def test_fc_few_rounds_do_not_pay_for_a_partition(m, iters):
    """(partitioned, twice as long at one round)"""
    v = dev(data("normal", m, iters))
    a = kq.kq_quantize_scalars(v, 6, iters)
    b = kq.kq_quantize_scalars(v, 6, iters, search="exact")
    for x, y, name in zip(a, b, ["codes", "levels", "v_hat", "rounds"]):
        assert torch.equal(x.view(torch.uint8), y.view(torch.uint8)), name
    auto = best_us(lambda: kq.kq_quantize_scalars(v, 6, iters, *a))
    exact = best_us(lambda: kq.kq_quantize_scalars(v, 6, iters, *b, search="exact"))
    assert auto <= 1.5 * exact, (auto, exact)
