"""The (-2 2 0) polynomial as a shifted product and a rest (n_shift, n_rest): the
identity in integers, and the rest inside 2^53 over every patch that shares a shift."""
import numpy as np
import pytest

C = 0.14644660940672624          # (1 - 1/sqrt 2)/2


def rest(s, d, a):
    S, D = (s + 1) ** 2, d ** 2
    q, r = divmod((S - D) ** 2 + 6 * S - 2 * D - 7, 8)
    assert r == 0
    return q - a * (S - D + 1) + a * a


def shift(s, d):
    return int(C * max(0, (s + 1) ** 2 - d ** 2))


def test_identity():
    rng = np.random.default_rng(1)
    for _ in range(2000):
        l1, l2 = sorted(int(x) for x in rng.integers(0, 16385, 2))
        s, d = l1 + l2, l2 - l1
        l3 = d + 2 * int(rng.integers(0, l1 + 1))
        a, b, c = (x * (x + 1) for x in (l1, l2, l3))
        u = a + b - c
        k = shift(s, d) + int(rng.integers(-1000, 1000))
        S, D = (s + 1) ** 2, d * d
        assert (c - S + 1 + k) * (c - D + 2 - k) + rest(s, d, k) == u * (u - 2) - 2 * a * b


@pytest.mark.parametrize("lmax", [8001, 16384])
def test_rest_is_exact_over_tiles_and_strip_items(lmax):
    worst = 0
    for par in (0, 1):                                    # tiles of 64 x 64 halved (s, d)
        for S0 in range(0, lmax + 1, 64):
            for D0 in range(0, min(S0 + 63, lmax - par - S0) + 1, 64):
                a = shift(2 * S0 + 64 + par, 2 * D0 + 64 + par)
                for S in (S0, S0 + 32, S0 + 63):
                    for D in (D0, D0 + 32, D0 + 63):
                        if D <= S and S + D + par <= lmax:
                            worst = max(worst, abs(rest(2 * S + par, 2 * D + par, a)))
    for d in range(0, lmax + 1, 61):                      # items of 256 rows, aligned to the diagonal's last row
        for A in range(lmax - d + 1 - 256, -256, -256):
            a = shift(2 * max(A + 128, 0) + d, d)
            for l1 in (max(A, 0), max(A + 128, 0), A + 255):
                worst = max(worst, abs(rest(2 * l1 + d, d, a)))
    assert worst < 2 ** 52
