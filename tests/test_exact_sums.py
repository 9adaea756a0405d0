"""The exact (high, low) sums of products of csrc/fp64_mod.hpp, step by step on
the CPU: with whole-number operands, float(a * b + c) is the correctly rounded
fma(a, b, c).  Every sum is compared with the integer sum, at the largest
operands the kernels' bounds allow and at random ones."""
import random

import pytest

PRIMES = [8193 * 2 + 15, (1 << 20) - 3, 1099511480321, (1 << 47) + 5, 140737488355213, 281474976694273, (1 << 48) - 59]


def fma(a, b, c):
    return float(int(a) * int(b) + int(c))


def offset(q, x):
    b = q.bit_length()
    e = max(2 * b + x, 52)
    kappa = int(6755399441055744.0 / float(q))
    return float(kappa * q) * 2.0 ** (e - 52)


def mac(a, b, hi, lo):
    h = fma(a, b, hi)
    t = hi - h
    assert int(t) == int(hi) - int(h)              # exact
    e = fma(a, b, t)
    assert int(e) == int(a) * int(b) + int(t)      # exact
    s = lo + e
    assert int(s) == int(lo) + int(e) and abs(s) < 2 ** 53
    return h, s


def fold(hi, lo, q):
    qinv = 1.0 / float(q)
    k = float(round(hi * qinv))
    r = fma(-k, q, hi)
    assert int(r) == int(hi) - int(k) * q          # exact
    s = r + lo
    assert int(s) == int(r) + int(lo) and abs(s) < 2 ** 53
    return s


def reduce(x, q):
    k = float(round(x * (1.0 / float(q))))
    r = fma(-k, q, x)
    assert int(r) == int(x) - int(k) * q and 2 * abs(r) <= q + 1
    return r


@pytest.mark.parametrize("q", PRIMES)
@pytest.mark.parametrize("extreme", [1, -1, 0])
def test_sums_stay_exact(q, extreme):
    g = random.Random(q + extreme)
    B = 1 << q.bit_length()
    half = (q - 1) // 2

    def val(m):
        return float(extreme * m) if extreme else float(g.randint(-m, m))

    for terms in (1, 8, 9, 40):
        cin3, cin2, cout = offset(q, 3), offset(q, 2), offset(q, 6)
        assert int(cout) % q == 0 and int(cin2) % q == 0 and int(cin3) % q == 0
        hi, lo, exact, cnt = cout, 0.0, 0, 0
        for i in range(terms):
            # four digits: its own limb below q, three centred; keys centred; P c0 in the sum or added to its fold
            inside = i % 2 == 0
            digits = [val(q)] + [val(half) for _ in range(3)]
            keys = [float(abs(int(val(half)))) for _ in range(4)]
            h, l, u_exact = (cin3 if inside else cin2), 0.0, 0
            for d, k in zip(digits, keys):
                h, l = mac(d, k, h, l)
                u_exact += int(d) * int(k)
            c0, p = val(q), float(half)
            if inside:
                h, l = mac(c0, p, h, l)
                u_exact += int(c0) * int(p)
            else:
                c0 = val(half)
                l += c0
                u_exact += int(c0)
            u = fold(h, l, q)
            assert (int(u) - u_exact) % q == 0 and abs(u) < 3 * B
            pt = float(abs(int(val(q))))
            hi, lo = mac(pt, u, hi, lo)
            exact += int(pt) * u_exact
            cnt += 1
            # nine terms in the first group (the kernels count diagonal 0 among eight), eight after
            if cnt == (9 if i < 9 else 8):
                lo = reduce(fold(hi, lo, q), q)
                hi, cnt = cout, 0
        assert (int(reduce(fold(hi, lo, q), q)) - exact) % q == 0


def test_long_sums_of_centred_products():
    """the encrypted-matrix kernel's sums: plaintexts below q times ciphertext residues below q, eight at a time"""
    for q in PRIMES:
        c = offset(q, 5)
        hi, lo, exact = c, 0.0, 0
        for i in range(32):
            a, b = float(q), float(q if i % 3 else -q)
            hi, lo = mac(a, b, hi, lo)
            exact += int(a) * int(b)
            if i % 8 == 7:
                lo = reduce(fold(hi, lo, q), q)
                hi = c
        assert (int(reduce(fold(hi, lo, q), q)) - exact) % q == 0
