"""The copy function and the merge path's test as csrc/afun.hpp has them, compiled for
the host, against whole numbers: the FP64 form, its slack and the 128-bit products
that decide next to a whole quotient."""
import ctypes as C
import os
import random
import subprocess
from fractions import Fraction

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1905_10252_amd", "csrc")


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    from paper_1905_10252_amd import build
    if not os.path.exists(build.HIPCC):
        pytest.skip("no hipcc")
    so = str(tmp_path_factory.mktemp("afun") / "afun.so")
    subprocess.check_call([build.HIPCC, "-x", "hip", "--offload-host-only", "-O2", "-std=c++17",
                           "-fPIC", "-shared", "-ffp-contract=off", "-I", CSRC,
                           os.path.join(HERE, "afun_host.hip"), "-o", so])
    L = C.CDLL(so)
    n, q = C.c_longlong, C.c_ulonglong
    L.afun_slack.restype = C.c_double
    L.afun_estimate.argtypes, L.afun_estimate.restype = [n, q, q, q], C.c_double
    L.afun_copies.argtypes, L.afun_copies.restype = [n, q, q, q], C.c_uint
    L.afun_before.argtypes, L.afun_before.restype = [n, q, q, q, n, n], C.c_int
    return L


def prefixes(rnd, n, S, U, slack):
    """Prefix values with quotients everywhere, next to whole numbers, and just inside and
    outside the slack around them."""
    out = [0, S, S - 1, S // 2, rnd.randint(0, S)]
    for _ in range(4):
        a = rnd.randint(0, n)
        for off in (0, slack, -slack, slack / 2, 2 * slack):
            at = int((Fraction(a) + Fraction(off)) * S - U) // n
            out += [at + d for d in (-1, 0, 1)]
    return [s for s in out if 0 <= s <= S]


@pytest.mark.parametrize("n", [1, 2, 3, 1000, 4097, (1 << 20) - 1, 1 << 24, 123456789,
                               (1 << 31) - 1])
def test_copies_and_merge_test(lib, n):
    rnd = random.Random(n)
    slack = lib.afun_slack()
    K = min(52, 61 - (n - 1).bit_length())  # fixed-point bits; the largest weight is 2^K
    inside = outside = 0
    for _ in range(300):
        S = rnd.choice([1 << K, n << K, rnd.randint(1 << K, n << K)])
        U = rnd.choice([0, S - 1, rnd.randrange(S)])
        for sj in prefixes(rnd, n, S, U, slack):
            quot = Fraction(n * sj + U, S)
            exact = n * sj + U
            a = exact // S
            if abs(quot - round(quot)) > Fraction(slack):
                outside += 1
            else:
                inside += 1
            assert abs(Fraction(lib.afun_estimate(n, S, U, sj)) - quot) < Fraction(slack) / 2
            assert lib.afun_copies(n, S, U, sj) == a, (n, S, U, sj)
            j = rnd.choice([0, n - 1, rnd.randrange(n)])
            for c in (a - 1, a, a + 1, a + 2, 0, 2 * n - j):
                want = c > 0 and exact < c * S
                if c + j >= 0:
                    assert lib.afun_before(n, S, U, sj, j, c + j) == want, (n, S, U, sj, j, c)
    assert outside > 100 and inside > 100
