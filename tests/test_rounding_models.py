"""Pins of the kernel-rounding models in tests/rounding_models.py (CPU only)."""
import numpy as np
import pytest

import tmac_workloads as wl
from oracle import tmac_oracle as orc
import rounding_models as rm

# ---------------------------------------------- narrow running sums (fp16) ----

def test_narrow_sum_is_exact_on_small_integers_and_bounded_on_gaussian_data():
    """fp16 pairwise sums of eight table entries (the batched kernel's aggregation, Section 3.3 /
    Section 4 "fast aggregation" read for fp16 tables): exact whenever every partial sum is an
    integer below 2048 (then the route must equal the definition bit for bit), and on Gaussian
    activations an error of a few 1e-4, between the error of fp16 tables alone and the 2e-3 bar."""
    rng = np.random.default_rng(77)
    N, M, K, G, b = 2, 24, 512, 128, 4
    q = rng.integers(0, 16, size=(M, K), dtype=np.uint8)
    ones = np.ones((M, K // G), np.float16)
    zer = np.zeros((M, K // G), np.float16)
    ai = rng.integers(-30, 31, size=(N, K)).astype(np.float16)      # |entry| <= 120, |sum of 8| <= 960
    exact = (ai.astype(np.int64) @ q.astype(np.int64).T).astype(np.float64)
    assert np.array_equal(rm.lut_mpgemm_narrow(ai, q, b, ones, zer, G), exact)
    p = wl.make_grouped(5, 40, 4, 96, 5120, 4, 128)
    ref = orc.mpgemm_definition(p.act, p.q, p.scales, p.zeros, p.group)
    e_tab = orc.rel_frobenius(orc.lut_mpgemm(p.act, p.q, 4, p.scales, p.zeros, p.group, table_dtype=np.float16), ref)
    e_nar = orc.rel_frobenius(rm.lut_mpgemm_narrow(p.act, p.q, 4, p.scales, p.zeros, p.group), ref)
    assert 5e-5 < e_tab < e_nar < 8e-4
    # sums of two entries only: closer to the tables' own error
    e_2 = orc.rel_frobenius(rm.lut_mpgemm_narrow(p.act, p.q, 4, p.scales, p.zeros, p.group, tables_per_sum=2), ref)
    assert e_tab < e_2 < e_nar


# ------------------------------------------------ tables built by fp16 additions ----

def test_fp16_tree_tables_worked_example_and_special_cases():
    """Tables built with fp16 additions, pair sums first.  Worked by hand for a = (2048, 1, 1, 0),
    where fp16 has a spacing of 2 above 2048: +a0+a1 = 2049 is a tie and goes to the even 2048,
    +a2+a3 = 1, and 2048 + 1 is a tie again -> 2048, whereas the exact sum 2050 is representable;
    with -a1 every partial sum is exact.  The negated index mirrors exactly; one addition (g = 2)
    equals the once-rounded exact sum; small integers are exact at every g."""
    a = np.array([[2048, 1, 1, 0]], dtype=np.float16)
    t = rm.precompute_lut_fp16_tree(a, 4)[0, 0].astype(np.float64)
    once = orc.precompute_lut(a, 4, dtype=np.float16)[0, 0].astype(np.float64)
    assert t[15] == 2048.0 and once[15] == 2050.0
    assert t[0] == -2048.0 and once[0] == -2050.0
    assert t[0b1101] == 2048.0 == once[0b1101]          # 2048 - 1 = 2047, + 1 = 2048: no rounding anywhere
    assert t[0b0111] == 2048.0 and once[0b0111] == 2050.0   # a3 = 0: its sign does not matter
    rng = np.random.default_rng(91)
    A = (rng.standard_normal((3, 64)) * 50).astype(np.float16)
    for g in (2, 4, 8):
        T = rm.precompute_lut_fp16_tree(A, g)
        assert T.dtype == np.float16 and T.shape == (3, 64 // g, 1 << g)
        assert np.array_equal(T.astype(np.float64), -T[..., ::-1].astype(np.float64))
        exact = orc.precompute_lut(A, g)
        # each of the g - 1 additions is off by at most half a spacing of its result, and no partial
        # sum exceeds sum |a_j|
        top = np.abs(A.astype(np.float64)).reshape(3, -1, g).sum(-1).astype(np.float16)
        bound = 0.5 * (g - 1) * np.spacing(top).astype(np.float64)
        assert np.all(np.abs(T.astype(np.float64) - exact) <= bound[..., None])
    assert np.array_equal(rm.precompute_lut_fp16_tree(A, 2).view(np.uint16),
                          orc.precompute_lut(A, 2, dtype=np.float16).view(np.uint16))
    Ai = rng.integers(-100, 101, size=(2, 32)).astype(np.float16)
    for g in (2, 4, 8):
        assert np.array_equal(rm.precompute_lut_fp16_tree(Ai, g).astype(np.float64), orc.precompute_lut(Ai, g))


def test_fp16_tree_tables_route_error():
    """End to end the extra roundings of the partial sums cost little: on Gaussian activations the
    route with tree-built tables errs more than the once-rounded tables and stays far inside the
    2e-3 bar."""
    p = wl.make_grouped(5, 41, 2, 96, 5120, 4, 128)
    ref = orc.mpgemm_definition(p.act, p.q, p.scales, p.zeros, p.group)
    e_once = orc.rel_frobenius(orc.lut_mpgemm(p.act, p.q, 4, p.scales, p.zeros, p.group, table_dtype=np.float16), ref)
    e_tree = orc.rel_frobenius(rm.lut_mpgemm_fp16_tree(p.act, p.q, 4, p.scales, p.zeros, p.group), ref)
    print(f"fp16 tables: once-rounded {e_once:.2e}, built by fp16 additions {e_tree:.2e}")
    assert 5e-5 < e_once < e_tree < 6e-4


def test_fp16_routes_keep_their_error_on_heavy_tailed_activations():
    """The roundings of the fp16 routes (tables built by fp16 additions, narrow chunk sums) scale with
    the entries themselves: outlier channels 50 or 300 times the rest, Student-t tails or an all-positive
    offset leave the relative error where it is on Gaussian data, a fifth of the 2e-3 bar."""
    rng = np.random.default_rng(95)
    M, K, G, b = 32, 2048, 128, 4
    q = rng.integers(0, 16, size=(M, K), dtype=np.uint8)
    s = rng.uniform(0.01, 0.1, size=(M, K // G)).astype(np.float16)
    z = rng.uniform(0, 15, size=(M, K // G)).astype(np.float16)
    base = rng.standard_normal((2, K))
    cases = {
        "gauss": base,
        "1% x50": base * np.where(rng.random((2, K)) < 0.01, 50.0, 1.0),
        "0.2% x300": base * np.where(rng.random((2, K)) < 0.002, 300.0, 1.0),
        "student t3": rng.standard_t(3, size=(2, K)),
        "positive": np.abs(base) + 3.0,
    }
    for name, a in cases.items():
        a = a.astype(np.float16)
        ref = orc.mpgemm_definition(a, q, s, z, group=G)
        e_tree = orc.rel_frobenius(rm.lut_mpgemm_fp16_tree(a, q, b, s, z, group=G), ref)
        e_narrow = orc.rel_frobenius(rm.lut_mpgemm_narrow(a, q, b, s, z, G), ref)
        assert e_tree < 5e-4 and e_narrow < 7e-4, (name, e_tree, e_narrow)


# ------------------------------------------------ fixed-point tables of large calls ----

def unequal_groups(rng, N, M, K, bits, group, ratio):
    """Activations whose size changes from group to group by up to `ratio` and scales that undo it: every
    group weighs the same in the result.  Returns (act, q, scales, zeros)."""
    nq = K // group
    size = ratio ** rng.uniform(-0.5, 0.5, size=nq)
    act = (rng.standard_normal((N, K)) * np.repeat(size, group)).astype(np.float16)
    s = (rng.uniform(0.01, 0.1, size=(M, nq)) / size).astype(np.float16)
    z = rng.uniform(0, 2 ** bits - 1, size=(M, nq)).astype(np.float16)
    return act, rng.integers(0, 1 << bits, size=(M, K), dtype=np.uint8), s, z


def test_fixed_point_tables_err_less_than_fp16_sums():
    """One unit per activation row and quantisation group (of at most 128 k): closer to the product than fp16
    chunk sums for every group size, also with group sizes and scales that undo each other and with outlier
    channels, which one unit for several groups would not be (2e-3 and more)."""
    rng = np.random.default_rng(96)
    M, K = 48, 2048
    for bits, group in ((2, 32), (4, 32), (4, 64), (3, 128), (4, 512), (2, 2048)):
        for ratio in (1.0, 30.0, 1000.0):
            act, q, s, z = unequal_groups(rng, 4, M, K, bits, group, ratio)
            act[2:] *= np.where(rng.random(K) < 0.002, 30, 1).astype(np.float16)
            ref = orc.mpgemm_definition(act, q, s, z, group)
            fixed = orc.rel_frobenius(rm.lut_mpgemm_fixed(act, q, bits, s, z, group), ref)
            narrow = orc.rel_frobenius(rm.lut_mpgemm_narrow(act, q, bits, s, z, group), ref)
            assert fixed < narrow and fixed < 4e-4, (bits, group, ratio, fixed, narrow)


def coarse_activations(rng, kind, N, K):
    """Activations with few significant bits, or with sums that fp16 holds as they are."""
    sign = rng.choice([-1.0, 1.0], size=(N, K))
    normal = rng.standard_normal((N, K))
    if kind.startswith("mantissa"):
        m, e = np.frexp(normal)
        bits = int(kind[8:])
        return np.ldexp(np.round(m * 2 ** bits), e - bits).astype(np.float16)
    return {"+-10": lambda: rng.integers(-10, 11, size=(N, K)), "+-127": lambda: rng.integers(-127, 128, size=(N, K)),
            "quarters": lambda: rng.integers(-40, 41, size=(N, K)) / 4,
            "subnormal": lambda: rng.integers(-500, 501, size=(N, K)) * 2.0 ** -24,
            "1e-6": lambda: normal * 1e-6, "2^0..7": lambda: sign * 2.0 ** rng.integers(0, 8, size=(N, K)),
            "2^-12..12": lambda: sign * 2.0 ** rng.integers(-12, 13, size=(N, K)),
            "sparse": lambda: normal * (rng.random((N, K)) < 0.01), "relu": lambda: np.maximum(normal, 0),
            "ones": lambda: np.ones((N, K))}[kind]().astype(np.float16)


@pytest.mark.parametrize("kind,exact", [("+-10", True), ("+-127", True), ("quarters", True), ("subnormal", True), ("1e-6", True),
                                        ("2^0..7", True), ("ones", True), ("2^-12..12", False), ("sparse", False),
                                        ("relu", False), ("mantissa3", False), ("mantissa4", False), ("mantissa8", False)])
def test_fixed_point_tables_are_no_further_off_on_activations_with_few_bits(kind, exact):
    """Where the entries of a unit are multiples of a power of two that is a unit too, they are held as they are: whole
    numbers, fractions of a power of two and subnormal numbers keep the exact sums that fp16 gives them, and none of
    these kinds is further from the product than with fp16 sums (the next test has one that is)."""
    rng = np.random.default_rng(97)
    N, M, K = 3, 40, 2048
    for bits, group in ((2, 32), (4, 128), (3, 96), (4, 2048)):
        K_ = K // group * group
        act = coarse_activations(rng, kind, N, K_)
        q = rng.integers(0, 1 << bits, size=(M, K_), dtype=np.uint8)
        s = rng.uniform(0.01, 0.1, size=(M, K_ // group)).astype(np.float16)
        z = rng.uniform(0, 2 ** bits - 1, size=(M, K_ // group)).astype(np.float16)
        ref = orc.mpgemm_definition(act, q, s, z, group)
        fixed = orc.rel_frobenius(rm.lut_mpgemm_fixed(act, q, bits, s, z, group), ref)
        narrow = orc.rel_frobenius(rm.lut_mpgemm_narrow(act, q, bits, s, z, group), ref)
        assert fixed <= max(narrow, 1e-12), (kind, bits, group, fixed, narrow)
        assert not exact or fixed <= 1e-12, (kind, bits, group, fixed)


@pytest.mark.parametrize("big", [300, 3000, 30000])
def test_a_large_number_alone_in_its_chunk_costs_the_rest_of_its_group(big):
    """The kind of activations whose fixed-point tables are further off than fp16 sums: one large whole number in an otherwise
    empty chunk of each group.  fp16 adds that chunk exactly; in fixed point the group's other entries take its unit, big / 32700,
    and each is off by at most half of it: 24 entries of a plane add up to about sqrt(24 / 12) units, 4e-5 of what the large number
    gives, and 1e-4 is allowed."""
    rng = np.random.default_rng(98)
    N, M, K, group = 3, 40, 2048, 128
    act = rng.standard_normal((N, K)).reshape(N, K // group, group)
    act[:, :, :32] = 0
    act[:, :, 5] = big
    act = act.reshape(N, K).astype(np.float16)
    for bits in (2, 4):
        q = rng.integers(0, 1 << bits, size=(M, K), dtype=np.uint8)
        s = rng.uniform(0.01, 0.1, size=(M, K // group)).astype(np.float16)
        z = rng.uniform(0, 2 ** bits - 1, size=(M, K // group)).astype(np.float16)
        ref = orc.mpgemm_definition(act, q, s, z, group)
        fixed = orc.rel_frobenius(rm.lut_mpgemm_fixed(act, q, bits, s, z, group), ref)
        narrow = orc.rel_frobenius(rm.lut_mpgemm_narrow(act, q, bits, s, z, group), ref)
        assert narrow < fixed <= 1e-4, (big, bits, narrow, fixed)
