"""The sizes that the workspace queries return, without a GPU: a query reads the ring degree, the prime counts and the digit
width of its context, and whether the column conversion's tables are there, so a block of memory that starts with those words
stands in for one, with every pointer behind them null or (operands) none of them."""
import ctypes as C

import pytest

# logN, ciphertext primes, special primes, digits, operands
SETS = [(16, 24, 8, 3), (16, 24, 4, 6), (15, 12, 4, 3), (9, 25, 1, 25), (12, 3, 1, 3), (17, 24, 8, 3),
        (16, 24, 8, 3, True), (16, 24, 4, 6, True), (15, 12, 4, 3, True)]


def context(logN, nq, np_, dnum, operands=False):
    words = (C.c_uint32 * 65536)()
    if operands:
        words[:] = [1] * 65536
    words[:7] = [logN, 1 << logN, nq, np_, dnum, -(-nq // dnum), nq + np_]
    return words


def query(name, ctx, *args):
    from paper_2302_02407_amd import binding
    v = C.c_uint64()
    assert getattr(binding.load(), name)(C.addressof(ctx), *args, C.byref(v)) == 0
    return v.value


@pytest.mark.parametrize("prm", SETS)
def test_a_batch_fits_what_a_larger_one_reserved(prm):
    """Fewer ciphertexts, fewer steps (or steps of zero, which need no key switch) never need more."""
    ctx = context(*prm)
    for level in range(prm[1]):
        for hoisted in (0, 1):
            q = [[query("he_ws_query_rotate_batch", ctx, level, n, s, hoisted) for s in range(1, 5)] for n in range(1, 36)]
            for n in range(35):
                for s in range(4):
                    assert n == 0 or q[n - 1][s] <= q[n][s], (level, hoisted, n + 1, s + 1)
                    assert s == 0 or q[n][s - 1] <= q[n][s], (level, hoisted, n + 1, s + 1)


@pytest.mark.parametrize("prm", SETS)
def test_the_hoisted_sum_of_a_block_leaves_room_for_its_square(prm):
    """Both forms of a block relinearise a group's squares with one launch set; the hoisted one does not get by with less than
    the stepwise one, whose rotate-and-sum has that same shape."""
    from paper_2302_02407_amd.binding import BlockPlan
    ctx, slots = context(*prm), 1 << (prm[0] - 1)
    for level in range(3, prm[1]):
        for group in (1, 4, 8, 9, 16, 24):
            need = []
            for hoisted in (0, 1):
                plan = BlockPlan(2, 8, slots // 16, 1, 3, 1, 2 * group, level, group, 0, hoisted)
                need.append(query("he_ws_query_ca_ra_block", ctx, C.byref(plan)))
            assert need[0] <= need[1], (level, group)


@pytest.mark.parametrize("prm", SETS)
def test_nothing_is_reserved_that_no_launch_uses(prm):
    """One key switch holds its digits and, in one place, either the limbs it raises or those of its ModDown; accumulators over the
    raised basis only where they are stored: more than 8 digits."""
    logN, nq, k, dnum = prm[:4]
    ctx, N, alpha = context(*prm), 1 << logN, -(-nq // dnum)
    for level in range(nq):
        L1, beta = level + 1, -(-(level + 1) // alpha)
        down = 2 * k + 2 * L1 + (2 * (L1 + k) if beta > 8 else 0)
        assert query("he_ws_query_rotate_batch", ctx, level, 1, 1, 0) == (beta * (L1 + k) + max(L1, down)) * N * 8, level


def test_the_benchmarks_batch_of_rotations():
    """240 rotations of 16 ciphertexts at the top level: sixteen sources' digits and sixteen jobs' ModDown at most."""
    assert query("he_ws_query_rotate_batch", context(16, 24, 8, 3, True), 23, 16, 15, 0) <= 16 * (3 * 32 + 2 * 8 + 2 * 24) << 19


def test_a_chain_without_special_primes_is_refused():
    """The calls refuse it and so do their queries."""
    from paper_2302_02407_amd import binding
    ctx, v, lib = context(12, 8, 0, 4), C.c_uint64(), binding.load()
    plans = {"he_ws_query_conv2d": binding.ConvPlan(2, 8, 128, 1, 3, 2, 4), "he_ws_query_raconv": binding.RaConvPlan(2, 32, 1, 3, 4),
             "he_ws_query_ca_ra_block": binding.BlockPlan(2, 8, 128, 1, 3, 1, 2, 4)}
    for name, plan in plans.items():
        assert getattr(lib, name)(C.addressof(ctx), C.byref(plan), C.byref(v)) == -1, name
    assert lib.he_ws_query_rotate_batch(C.addressof(ctx), 4, 3, 2, 0, C.byref(v)) == -1
    assert lib.he_ws_query_rotate_batch(C.addressof(ctx), 4, 0, 2, 0, C.byref(v)) == 0 and v.value == 0
