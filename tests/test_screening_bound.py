"""The error bound of the fp16 screening product of codebooks of more than 1024 entries, on the CPU:
the operands as the kernel forms them (scaled by powers of two, rounded to fp16, values below its
smallest normal lost, the norm in three parts with weights u, 2^-11 u, 2^-22 u), summed in fp64, against
the score |c|^2 - 2 x . c.  The sums' own roundings have a term of their own in the kernel's bound."""
import numpy as np
import pytest


def fp16(v):
    return np.where(np.abs(v) < 2.0 ** -14, 0.0, v.astype(np.float16).astype(np.float64))


@pytest.mark.parametrize("seed", range(12))
def test_screened_scores_stay_within_the_bound(seed):
    rng = np.random.default_rng(seed)
    n = 2000
    for _ in range(20):
        c = rng.standard_normal((n, 9)) * 2.0 ** rng.uniform(rng.uniform(-20, 0), 0, (n, 1))
        c = np.clip(c, -1.99, 1.99).astype(np.float32)
        c[0, 0] = 1.5                                            # the codebook's exponent is 0
        x = rng.standard_normal((n, 9)) * 2.0 ** (rng.uniform(-20, 40) + rng.uniform(-3, 3, (n, 1)))
        x = x.astype(np.float32)
        a = 12
        b = 12 - np.maximum(np.floor(np.log2(np.abs(x).max(1))), 0)
        cs = c.astype(np.float64) * 2.0 ** a
        nn = np.zeros(n, np.float32)
        for d in range(9):
            nn = (cs[:, d] * cs[:, d] + nn.astype(np.float64)).astype(np.float32)
        v = nn.astype(np.float64) * 2.0 ** -14
        n0 = fp16(v)
        t = (v - n0) * 2.0 ** 11
        n1 = fp16(t)
        n2 = fp16((t - n1) * 2.0 ** 11)
        w = fp16(-2.0 * cs)
        assert max(np.abs(m).max() for m in (w, n0, n1, n2)) <= 65504
        u = 2.0 ** (14 + b - a)
        s = (w * fp16(x.astype(np.float64) * 2.0 ** b[:, None])).sum(1)
        s = (s + n0 * fp16(u) + n1 * fp16(u * 2.0 ** -11) + n2 * fp16(u * 2.0 ** -22)) * 2.0 ** (-a - b)
        c, x = c.astype(np.float64), x.astype(np.float64)
        score = (c * c).sum(1) - 2.0 * (c * x).sum(1)
        X, C = np.sqrt((x * x).sum(1)), np.sqrt((c * c).sum(1))
        A, B = 2.0 ** (-14 - a), 2.0 ** (-14 - b)
        bound = ((2.0 ** -10 + 2.0 ** -22) * 2 * X * C + 1.01 * (6 * B * C + 3 * A * X) + 2.0 ** (-22 - 2 * a)
                 + 9 * 2.0 ** -24 * (2 * X * C + C * C) + 2.0 ** -29 * X * X)
        assert (np.abs(s - score) <= bound).all()
