"""The FP64 form of the copy function A_j = floor((N S_j + U) / S): wherever its
value is more than the slack away from an integer it has to give the integer
rule's floor and comparisons (csrc/afun.hpp decides the rest in 128 bits).

The device's operations are repeated here one by one, fused multiply-adds rounded
once from exact rationals.
"""
import random
from fractions import Fraction

import pytest

SLACK = 2.0 ** -18


def fma(a, b, c):
    return float(Fraction(a) * Fraction(b) + Fraction(c))  # CPython rounds correctly


def u64_to_f64(v):
    return fma(float(v >> 32), 2.0 ** 32, float(v & 0xFFFFFFFF))


def check(n, S, U, Sj):
    inv = 1.0 / u64_to_f64(S)
    nS, uS = float(n) * inv, u64_to_f64(U) * inv
    est = fma(u64_to_f64(Sj), nS, uS)
    a = int(est)
    fr = est - a
    exact = (n * Sj + U) // S
    if abs(fr - 0.5) < 0.5 - SLACK:
        assert a == exact, (n, S, U, Sj)
        return 1
    # left to the integers: the estimate is off by one at most
    assert abs(a - exact) <= 1, (n, S, U, Sj)
    return 0


@pytest.mark.parametrize("n", [1, 2, 3, 1000, 4097, (1 << 20) - 1, 1 << 24, (1 << 31) - 1])
def test_fp64_copies_agree_with_the_integer_rule(n):
    rnd = random.Random(n)
    k = 63 - n.bit_length()  # S stays below 2^63
    settled = 0
    for trial in range(3000):
        top = 1 << rnd.randint(1, k)
        S = rnd.randint(top, min(n * top, (1 << 63) - 1))
        U = rnd.choice([0, S - 1, rnd.randrange(S)])
        Sj = rnd.choice([0, S, rnd.randint(0, S), S // 2, S - 1])
        settled += check(n, S, U, Sj)
        # next to a whole quotient: N S_j + U just below, at and above a S
        a = rnd.randint(0, n)
        for d in (-2, -1, 0, 1, 2):
            sj = (a * S - U) // n + d
            if 0 <= sj <= S:
                settled += check(n, S, U, sj)
    assert settled > 0 or n < 3


@pytest.mark.parametrize("n", [1, 7, 4096, (1 << 31) - 1])
def test_equal_weights_are_whole_quotients(n):
    q = 1 << (62 - n.bit_length())
    for j in sorted({0, 1, n // 3, n // 2, n - 1, n}):
        for U in (0, q - 1, n * q - 1):
            check(n, n * q, U, j * q)
