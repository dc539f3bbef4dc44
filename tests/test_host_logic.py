"""CPU checks of arithmetic shortcuts that the HIP kernels take, restated in numpy from their description
and compared with the oracle's exact definition over many more cases than a GPU test can afford.

The quantizer kernel does not divide: it multiplies by a reciprocal and applies one fused-remainder correction.  That rounding
this fp32 quotient to a format's grid (nearest, ties to the even code, saturating) gives what rounding the exact |w|/scale
gives, ties included, and that the quotient of a zero keeps its sign, is an argument about fp32 arithmetic; here it is tested.
The rounding itself, which the kernel leaves to the chip's conversions (3 bits: to comparisons), is only stated here;
tests/test_gpu_pack_rounding.py holds the kernel's codes against the oracle's.
"""
import subprocess

import numpy as np
import pytest

# (mantissa bits, exponent of the lowest normal binade, bits of the magnitude code)
GRID = {"fp6": (2, -2, 5), "fp5": (2, 0, 4), "fp4": (1, 0, 3), "fp3": (0, 0, 2)}


def _oracle(width):
    from oracle import fp6_oracle, fpx_oracle

    return fp6_oracle if width == "fp6" else fpx_oracle.BY_PREFIX[width]


def _kernel_ratio(w_bits, s_bits):
    """w / scale as the kernel forms it, float32 (fma via fp64: both factors have 24 bits at most)."""
    a = w_bits.astype(np.uint16).view(np.float16).astype(np.float32)
    s = s_bits.astype(np.uint16).view(np.float16).astype(np.float32)
    with np.errstate(divide="ignore"):
        inv = np.where(s == 0, np.float32(0), np.float32(1) / s).astype(np.float32)
    q = (a * inv).astype(np.float32)
    rem = (q.astype(np.float64) * s.astype(np.float64) + -a.astype(np.float64)).astype(np.float32)         # fma(q, s, -w)
    return (-rem.astype(np.float64) * inv.astype(np.float64) + q.astype(np.float64)).astype(np.float32)    # fma(-rem, inv, q)


def _codes(width, w_bits, s_bits):
    """Codes of w at the given scales: the kernel's quotient on the format's grid."""
    w_bits, s_bits = np.broadcast_arrays(w_bits, s_bits)
    m, e_min, bits = GRID[width]
    ratio = _kernel_ratio(np.ascontiguousarray(w_bits), np.ascontiguousarray(s_bits))
    r = np.abs(ratio).astype(np.float64)
    e = np.floor(np.log2(np.maximum(r, 2.0 ** e_min)))
    code = np.where(r < 2.0 ** e_min, r * 2.0 ** (m - e_min), (e - e_min) * 2.0 ** m + r * 2.0 ** (m - e))  # in units of the code
    code = np.minimum(np.rint(code), 2 ** bits - 1).astype(np.uint32)
    return (np.signbit(ratio).astype(np.uint32) << bits) | code


def _oracle_codes(oracle, w_bits, s_bits):
    w_bits, s_bits = np.broadcast_arrays(w_bits, s_bits)
    out = np.empty(w_bits.shape, dtype=np.uint32)
    it = np.nditer([w_bits, s_bits, out], op_flags=[["readonly"], ["readonly"], ["writeonly"]])
    for w, s, o in it:
        o[...] = oracle.quantize_one(int(w), int(s))
    return out


@pytest.mark.parametrize("width", list(GRID))
def test_quantizer_shortcut_random(width):
    rng = np.random.default_rng(0)
    s_bits = np.concatenate([rng.integers(1, 0x7BFF, 300), rng.integers(0x1800, 0x2400, 300), [0, 1, 2, 0x3FF, 0x400, 0x3C00]]).astype(np.uint16)
    w_bits = rng.integers(0, 0x10000, (s_bits.size, 60)).astype(np.uint16)
    w_bits = np.where((w_bits & 0x7C00) == 0x7C00, np.uint16(0x1234), w_bits)     # finite only
    w_bits[:, :2] = [0, 0x8000]                                                   # a zero keeps its sign
    assert np.array_equal(_codes(width, w_bits, s_bits[:, None]), _oracle_codes(_oracle(width), w_bits, s_bits[:, None]))


@pytest.mark.parametrize("width", list(GRID))
def test_quantizer_shortcut_on_exact_ties(width):
    """Every (scale, midpoint) pair whose product is an fp16: |w| = midpoint * scale exactly."""
    oracle, magnitudes = _oracle(width), 2 ** GRID[width][2]
    grid = oracle.decode_table()[:magnitudes]
    mids = (grid[:-1] + grid[1:]) / 2
    s_bits = np.arange(1, 0x7BFF, 7, dtype=np.uint16)
    s = s_bits.view(np.float16).astype(np.float64)
    with np.errstate(over="ignore"):
        prod = mids[None, :] * s[:, None]
        h = prod.astype(np.float16)
    exact = (h.astype(np.float64) == prod) & np.isfinite(h.astype(np.float64))
    rows, cols = np.nonzero(exact)
    assert rows.size > 350 * mids.size
    w_bits = h.view(np.uint16)[rows, cols]
    sb = s_bits[rows]
    got = _codes(width, w_bits, sb)
    # ties go to the even code: midpoint j sits between codes j and j+1
    want = np.where(cols % 2 == 0, cols, cols + 1).astype(np.uint32)
    assert np.array_equal(got, want)
    # neighbours of the ties (one fp16 ulp either side) against the oracle, on a sample
    idx = np.random.default_rng(1).choice(rows.size, 3000 if rows.size > 3000 else rows.size, replace=False)
    for d in (-1, 1):
        wb = (w_bits[idx].astype(np.int32) + d).clip(0, 0x7BFF).astype(np.uint16)
        assert np.array_equal(_codes(width, wb, sb[idx]), _oracle_codes(oracle, wb, sb[idx]))
    # and the oracle agrees on the ties themselves (sample)
    assert np.array_equal(_oracle_codes(oracle, w_bits[idx], sb[idx]), want[idx])


def test_block_order_is_a_bijection_that_fills_the_xcds_evenly(tmp_path):
    """The block kernel's own map from block ids to output pieces, evaluated by the compiler: every piece once, no XCD
    with more rounds of 32 blocks than an eighth of them (rounded up) takes or with 1/8 more of them, for even and uneven
    numbers of units and short last groups."""
    from paper_2401_14112_amd import build

    (tmp_path / "order.hip").write_text("""
#include "linear_block.hpp"
template <int UNITS, int NB> struct Order {
    static constexpr bool covers() {
        const int chunk = fp6::pieces_per_xcd(UNITS, NB);
        const int even = (UNITS * NB + 7) / 8;
        if (chunk < even || 8 * chunk > 9 * even || (chunk + 31) / 32 > (even + 31) / 32) return false;
        bool seen[UNITS * NB] = {};
        int found = 0;
        for (int id = 0; id < 8 * chunk; ++id) {
            const fp6::BlockPiece p = fp6::piece_of_block(id, UNITS, NB, chunk);
            if (p.unit == UNITS) continue;
            if (p.unit < 0 || p.unit > UNITS || p.n_block < 0 || p.n_block >= NB || seen[p.n_block * UNITS + p.unit]) return false;
            seen[p.n_block * UNITS + p.unit] = true;
            ++found;
        }
        return found == UNITS * NB;
    }
};
template <int... UNITS> constexpr bool all() {
    return ((Order<UNITS, 1>::covers() && Order<UNITS, 2>::covers() && Order<UNITS, 3>::covers() && Order<UNITS, 11>::covers()
             && Order<UNITS, 16>::covers()) && ...);
}
static_assert(all<1, 2, 7, 8, 9, 19, 20, 25, 50, 63, 64, 65, 72, 76, 84, 100, 128, 224, 257>(), "a piece is missed or dealt twice");
// an eighth of the units with all their token blocks, one round and several; evenly dealt pieces
static_assert(fp6::pieces_per_xcd(50, 2) == 14 && fp6::pieces_per_xcd(100, 4) == 52, "whole units");
static_assert(fp6::pieces_per_xcd(20, 11) == 28 && fp6::pieces_per_xcd(9, 3) == 4, "pieces");
""")
    subprocess.run([build.hipcc(), "--offload-arch=gfx950", "-std=c++17", "--cuda-host-only", "-fsyntax-only", "-w",
                    "-fconstexpr-steps=100000000", "-I", str(build.CSRC), str(tmp_path / "order.hip")], check=True)
