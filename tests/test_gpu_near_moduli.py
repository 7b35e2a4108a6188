"""GPU parity for moduli near a multiple of 2^32 (he_internal.h): their points are signed and never reduced inside a transform.  Fullest where the
modulus and its low word are at the ends of what the rules take, so the checks of every form of the passes (test_gpu_modulus_classes) run there:
below and above the line of the inverse passes, at the top of the forward ones, in the range above 2^59 that is centred first, low words on
both sides of the bound, and moduli of little more than 20 bits."""
import pytest

from he_inputs.params import is_prime
from test_gpu_modulus_classes import check_batches, check_large_launches, check_single_calls

pytestmark = pytest.mark.gpu

INVERSE, WORD = (1 << 63) // 550, 1 << 27


def near_primes(kind, two_n, count):
    """primes = 1 mod two_n, half of them with the low word at each end of its range"""
    first, step, word = {
        "inverse below": (INVERSE >> 32, -1, WORD), "inverse above": ((INVERSE >> 32) + 2, 1, WORD), "forward top": (1 << 26, -1, WORD),
        "centred top": ((1 << 27) + (1 << 18) - 1, -1, WORD >> 1), "centred": (1 << 27, 1, WORD >> 1), "words beyond": (1 << 21, 1, 2 * WORD),
    }.get(kind, (0, 0, 0))
    out, k = [], first
    if kind == "small":
        c = 1 + two_n * ((1 << 20) // two_n + 1)
        while len(out) < count:
            if is_prime(c):
                out.append(c)
            c += two_n
        return out
    while len(out) < count:
        for sign in (1, -1):                             # down from the end of the range of low words, up from the other
            end = (k << 32) + sign * (word - 1)
            c = end - (end - 1) % two_n + (two_n if sign < 0 else 0)
            found = 0
            while found < 1 and len(out) < count and abs(c - (k << 32)) < word:
                if is_prime(c) and c not in out:
                    out.append(c)
                    found += 1
                c -= sign * two_n
        k += step
    return out


KINDS = ["inverse below", "inverse above", "forward top", "centred top", "centred", "words beyond", "small"]


@pytest.mark.parametrize("logN", [13, 16, 17])
@pytest.mark.parametrize("kind", KINDS)
def test_single_calls(kind, logN):
    check_single_calls(logN, near_primes(kind, 2 << logN, 6))


@pytest.mark.parametrize("kind", KINDS[:5])
@pytest.mark.parametrize("logN,counts", [(16, (133, 130, 129)), (16, (5,) * 13), (17, (5,) * 7)])
def test_large_launches(kind, logN, counts):
    check_large_launches(logN, counts, near_primes(kind, 2 << logN, len(counts)))


@pytest.mark.parametrize("kind", KINDS)
def test_batches(kind):
    check_batches(13, near_primes(kind, 2 << 13, 9))
