"""Arithmetic identities the HIP quantiser relies on, checked on the CPU with numpy (no GPU, no
library code: the kernel's instruction sequence is re-enacted with exact intermediate types)."""
import numpy as np
import pytest

f32, f64, ld = np.float32, np.float64, np.longdouble


def correction_step_quotient(num, S):
    """q0 = fl(num * r), rem = num - S * q0 (exact in a fused multiply-add), q = fl(q0 + rem * r)
    with r = fl(1 / S): the sequence the kernel uses instead of a division per element."""
    r = (f32(1) / S).astype(f32)
    q0 = (num * r).astype(f32)
    rem = num.astype(f64) - S.astype(f64) * q0.astype(f64)          # 24 x 24-bit product: exact in fp64
    assert np.array_equal(rem, rem.astype(f32).astype(f64))          # and the remainder fits fp32
    return (q0.astype(ld) + rem.astype(ld) * r.astype(ld)).astype(f32)   # one rounding to fp32


def fp16_values(rng, n, lo=0):
    return rng.integers(lo, 0x7C00, n, dtype=np.uint16).view(np.float16).astype(f32)


@pytest.mark.skipif(np.finfo(ld).nmant < 63, reason="needs an extended-precision long double")
@pytest.mark.parametrize("kind", ["asym_numerators", "sym_numerators", "group_like", "ties"])
def test_reciprocal_correction_step_equals_ieee_division(kind):
    """Code formula of Section "Quantization Scheme" (Eq. asym_quant): the quotient (x - Z) / S is
    an fp32 division.  The kernel's three-instruction replacement must give the identical fp32
    value for every numerator the quantiser can meet (differences of fp16 values, fp16 values)
    and every fp16 scale, including quotients that sit on or beside k + 0.5."""
    rng = np.random.default_rng({"asym_numerators": 1, "sym_numerators": 2, "group_like": 3, "ties": 4}[kind])
    n = 3_000_000
    S = fp16_values(rng, n, lo=1)                                    # every positive finite fp16, subnormals too
    if kind == "asym_numerators":
        num = (fp16_values(rng, n) - fp16_values(rng, n)).astype(f32)
    elif kind == "sym_numerators":
        num = fp16_values(rng, n) * rng.choice(f32([-1, 1]), n)
    elif kind == "group_like":
        lo = rng.standard_normal(n).astype(np.float16).astype(f32)
        hi = lo + np.abs(rng.standard_normal(n)).astype(np.float16).astype(f32)
        S = ((hi - lo) / f32(3)).astype(np.float16).astype(f32)
        S[S == 0] = f32(2.0 ** -24)
        x = (lo + (hi - lo) * rng.random(n).astype(f32)).astype(np.float16).astype(f32)
        num = (x - lo).astype(f32)
    else:
        k = rng.integers(-8, 8, n).astype(f32)
        S = fp16_values(rng, n, lo=0x0400) * f32(2.0 ** -4)             # keep (k + 0.5) S and its neighbours finite in fp16
        mid = ((k + f32(0.5)) * S).astype(f32)                        # exact: few bits times 11 bits
        step = np.spacing(np.abs(mid).astype(np.float16)).astype(f32)
        num = (mid + rng.integers(-2, 3, n).astype(f32) * step).astype(f32)
    with np.errstate(all="ignore"):
        want = (num / S).astype(f32)
        got = correction_step_quotient(num, S)
    ok = np.isfinite(want)
    assert ok.mean() > 0.9
    assert np.array_equal(want[ok], got[ok])
    if kind == "ties":
        frac = np.abs(want - np.trunc(want))
        assert (frac[ok] == 0.5).mean() > 0.1                        # the exact ties are really in the sample


def numerators_and_scales(kind, n):
    """What a lane that holds a whole group meets: (x - min) or x, and the group's scale; also the exact ties
    (k + 1/2) S and their fp32 neighbours."""
    rng = np.random.default_rng({"asym": 11, "sym": 12, "ties": 13, "beside_ties": 14, "denormal_scale": 15}[kind])
    S = fp16_values(rng, n, lo=0x0400)
    if kind == "denormal_scale":
        S = rng.integers(1, 0x400, n, dtype=np.uint16).view(np.float16).astype(f32)
    if kind in ("ties", "beside_ties"):
        k = rng.integers(-9, 17, n).astype(f32)
        num = ((k + f32(0.5)) * S).astype(f32)                        # exact: at most 16 bits
        if kind == "beside_ties":
            num = np.nextafter(num, rng.choice(f32([-np.inf, np.inf]), n))
        return num, S
    lo = (rng.standard_normal(n) * np.exp2(rng.integers(-10, 8, n))).astype(np.float16).astype(f32)
    with np.errstate(over="ignore"):                                  # (infinite ones are left out below)
        x = (lo + S * (rng.random(n) * 16).astype(f32)).astype(np.float16).astype(f32)
        return ((S * (rng.random(n) * 18 - 9)).astype(np.float16).astype(f32) if kind == "sym" else (x - lo).astype(f32)), S


@pytest.mark.skipif(np.finfo(ld).nmant < 63, reason="needs an extended-precision long double")
@pytest.mark.parametrize("kind", ["asym", "sym", "ties", "beside_ties", "denormal_scale"])
def test_two_piece_reciprocal_gives_the_code_of_ieee_division(kind):
    """A lane that holds a whole group forms its codes as rint(fma(num, r_hi, fl(num r_lo))) with r_hi = fl(1 / S) and
    r_lo = fl((1 - S r_hi) r_hi): the same integer as rint(fl(num / S)) for every quotient that a code can come from."""
    num, S = numerators_and_scales(kind, 2_000_000)
    with np.errstate(all="ignore"):
        hi = (f32(1) / S).astype(f32)
        rem = f64(1) - S.astype(f64) * hi.astype(f64)                # 11 x 24 bits: exact in fp64
        assert np.array_equal(rem, rem.astype(f32).astype(f64))       # and what the fused multiply-add leaves fits fp32
        lo = (rem.astype(f32) * hi).astype(f32)
        tail = (num * lo).astype(f32)
        quotient = (num.astype(ld) * hi.astype(ld) + tail.astype(ld)).astype(f32)      # one rounding
        want = (num / S).astype(f32)
    ok = np.isfinite(num) & np.isfinite(S) & (np.abs(want) <= 64)
    assert ok.mean() > 0.8
    assert np.array_equal(np.rint(quotient[ok]), np.rint(want[ok]))
    if kind == "ties":
        assert (np.abs(want[ok] - np.trunc(want[ok])) == 0.5).all()


@pytest.mark.skipif(np.finfo(ld).nmant < 63, reason="needs an extended-precision long double")
def test_ternary_codes():
    """2-bit symmetric codes (S = max |x|, so |x| <= S): x r + 1.5 2^23 with r = fl(fl(1 / S) (1 - 2^-20)) leaves
    rint(x / S) in its low bits for every positive fp16 S: the tie S / 2 and its neighbours on both sides, S itself, small
    and random values, and every value where S is a denormal."""
    rng = np.random.default_rng(21)
    bits = np.arange(1, 0x7C00, dtype=np.uint16)
    S = bits.view(np.float16).astype(f32)

    def check(x, S):
        x, S = x.astype(f32), S.astype(f32)
        r = ((f32(1) / S).astype(f32) * f32(1 - 2.0 ** -20)).astype(f32)
        t = (x.astype(ld) * r.astype(ld) + ld(12582912.0)).astype(f32)
        code = t - f32(12582912.0)
        want = np.rint((x / S).astype(f32))
        assert np.array_equal(code, want)
        assert np.array_equal(t.view(np.uint32) - np.uint32(0x4B400000), want.astype(np.int32).view(np.uint32))

    half = (S / 2).astype(np.float16)
    for step in range(-3, 4):
        x = (half.view(np.uint16).astype(np.int32) + step).clip(0, bits).astype(np.uint16).view(np.float16)
        check(x, S)
        check(-x, S)
    check(S, S)
    check(-S, S)
    check(np.zeros_like(S), S)
    for _ in range(20):
        check((rng.integers(0, bits.astype(np.int64) + 1).astype(np.uint16)).view(np.float16), S)
    for s in range(1, 0x400, 7):
        x = np.arange(0, s + 1, dtype=np.uint16).view(np.float16)
        check(x, np.full(x.shape, S[s - 1]))


@pytest.mark.parametrize("bits,bias", [(2, 0), (2, 2), (3, 0), (3, 4), (4, 0), (4, 8)])
def test_fields_collected_in_fp32(bits, bias):
    """Sixteen bits of fields at a time are summed as c 2^(b i) in fp32 (3 bits: low parts and high bits apart, the high bit
    taken off the low sum): every partial sum is an integer below 2^24, so the result is the packed field word."""
    rng = np.random.default_rng(bits)
    low_bits = 2 if bits == 3 else bits
    per = 16 // low_bits
    field = rng.integers(0, 1 << bits, (200_000, 16))
    c = (field - bias).astype(f32)
    low = np.full((field.shape[0], 16 // per), f32(sum(bias << (low_bits * i) for i in range(per))))
    high = np.zeros(field.shape[0], dtype=f32)
    for i in range(16):
        low[:, i // per] += c[:, i] * f32(1 << (low_bits * (i % per)))
        if bits == 3:
            h = np.clip(c[:, i] + f32(bias - 3), f32(0), f32(1))
            low[:, i // per] += h * f32(-4 * (1 << (low_bits * (i % per))))
            high += h * f32(1 << i)
    want_low = np.zeros(low.shape, dtype=np.int64)
    for i in range(16):
        want_low[:, i // per] |= (field[:, i] & ((1 << low_bits) - 1)) << (low_bits * (i % per))
    assert np.array_equal(low.astype(np.int64), want_low)
    if bits == 3:
        assert np.array_equal(high.astype(np.int64), ((field >> 2) << np.arange(16)).sum(axis=1))


def test_zero_scale_gives_code_zero_without_a_select():
    """A group whose scale is 0 gets r = 0 instead of 1 / 0: every quotient is then exactly 0."""
    num = f32([0.0, 1.5, -3.0, 65504.0])
    S, r = f32(0), f32(0)
    q0 = num * r
    rem = num - S * q0
    assert np.array_equal(q0 + rem * r, np.zeros(4, dtype=f32))


@pytest.mark.skipif(np.finfo(ld).nmant < 63, reason="needs an extended-precision long double")
def test_reciprocal_of_a_scale_from_any_start_within_an_ulp():
    """r0 is the instruction's 1 / S, within one ulp; e = fl(1 - S r0), r = fl(e r0 + r0) is the correctly rounded 1 / S from
    every such start, for every positive finite fp16 S."""
    S = np.arange(1, 0x7C00, dtype=np.uint16).view(np.float16).astype(f32)
    want = (f32(1) / S).astype(f32)
    for ulps in (-1, 0, 1):
        r0 = (want.view(np.int32) + ulps).view(f32)
        e = (ld(1) - S.astype(ld) * r0.astype(ld)).astype(f32)
        got = (e.astype(ld) * r0.astype(ld) + r0.astype(ld)).astype(f32)
        assert np.array_equal(got, want)


@pytest.mark.skipif(np.finfo(ld).nmant < 63, reason="needs an extended-precision long double")
@pytest.mark.parametrize("den", [3, 7, 15])
def test_scale_quotient_equals_ieee_division(den):
    """Scales: x / (2^b - 1) and x / (2^(b-1) - 1) by the correction step with r = fl(1 / den), for every fp16 magnitude and for
    differences of fp16 values."""
    rng = np.random.default_rng(den)
    every = np.arange(0, 0x7C00, dtype=np.uint16).view(np.float16).astype(f32)
    ranges = np.abs(fp16_values(rng, 3_000_000) - fp16_values(rng, 3_000_000) * rng.choice(f32([-1, 1]), 3_000_000)).astype(f32)
    x = np.concatenate([every, ranges])
    assert np.array_equal(correction_step_quotient(x, np.full_like(x, f32(den))), (x / f32(den)).astype(f32))


def test_distances_of_a_symmetric_two_bit_group():
    """min(|x|, S - |x|) in fp16 is |x - S code| with S = max |x|, exactly, for every fp16 x up to S."""
    rng = np.random.default_rng(31)
    S = np.concatenate([np.arange(1, 0x7C00, dtype=np.uint16), rng.integers(1, 0x7C00, 2_000_000).astype(np.uint16)])
    x = (rng.integers(0, S.astype(np.int64) + 1)).astype(np.uint16)
    half = (S.view(np.float16).astype(f32) / 2).astype(np.float16).view(np.uint16)
    for pick in (x, S, np.minimum(half, S), np.minimum(half + 1, S), half - (half > 0)):
        a, s = pick.astype(np.uint16).view(np.float16), S.view(np.float16)
        code = np.rint((a.astype(f32) / s.astype(f32)).astype(f32))
        want = np.abs(a.astype(f64) - s.astype(f64) * code)
        assert np.array_equal(np.minimum(a, (s - a).astype(np.float16)).astype(f64), want)


@pytest.mark.parametrize("bits", [2, 3, 4])
@pytest.mark.parametrize("G", [32, 64])
def test_bound_of_the_short_error_sum(bits, G):
    """sum |(x - mn) - S code| against sum |x - (S code + mn)|, every operation rounded to fp32: they differ by less than the bound
    2.1 G u sum + 4.4 G u max |x| below which the kernel takes the comparison again, on groups whose values span many binades."""
    rng = np.random.default_rng(bits * G)
    n, u, top = 30_000, 2.0 ** -24, (1 << bits) - 1
    x = (rng.standard_normal((n, G)) * np.exp2(rng.integers(-12, 3, (n, G)) * (rng.random((n, 1)) < 0.5))).astype(np.float16)
    x[:2000] += np.float16(1000)
    x[2000:4000] = np.abs(x[2000:4000])
    x = x.astype(f32)
    mn, mx = x.min(1, keepdims=True), x.max(1, keepdims=True)
    S = ((mx - mn) / f32(top)).astype(np.float16).astype(f32)
    num = (x - mn).astype(f32)
    with np.errstate(all="ignore"):
        c = np.rint(np.where(S == 0, f32(0), num / S)).astype(f32).clip(0, top)
    fma = lambda a, b, d: (a.astype(f64) * b.astype(f64) + d.astype(f64)).astype(f32)  # noqa: E731  (11 x 4 bits: the sum is exact in fp64)
    exact, short = np.zeros(n, f32), np.zeros(n, f32)
    for i in range(G):
        exact = exact + np.abs(x[:, i] - fma(S[:, 0], c[:, i], mn[:, 0]))
        short = short + np.abs(fma(-S[:, 0], c[:, i], num[:, i]))
    bound = 2.1 * G * u * short + 4.4 * G * u * np.abs(x).max(1)
    assert (np.abs(exact.astype(f64) - short) <= 0.5 * bound).all()          # (the bound is a worst case: half of it is never reached here)
    assert (exact != short).any()
