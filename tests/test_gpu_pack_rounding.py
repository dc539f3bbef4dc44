"""The quantizer's rounding, bit for bit: every fp16 magnitude that can occur under a row maximum, for 512 maxima of all binades
(subnormal scales and scales that round to zero among them), hence every exact tie, the values next to it and the smallest ratios under
these scales; and rows with infinities and NaN."""
import numpy as np
import pytest
import torch

from launch_plans import BITS
from packed_rows import row_tiles_of

pytestmark = pytest.mark.gpu

COLUMNS = 32768  # more than there are finite magnitudes (31744)
TILE = {"fp6": (3072, 256), "fp5": (2560, 256), "fp4": (2048, 256), "fp3": (3072, 512)}


@pytest.fixture(scope="module")
def pkg():
    import paper_2401_14112_amd as p

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    p.load_library()
    return p


def _oracle(fmt):
    from oracle import fp6_oracle, fpx_oracle

    return fp6_oracle if fmt == "fp6" else fpx_oracle.BY_PREFIX[fmt]


def _maxima():
    """Bits of 512 row maxima: the smallest ones (scales of 0 and of a few subnormal steps), both ends of each binade, random ones."""
    rng = np.random.default_rng(512)
    edges = [(e << 10) + m for e in range(31) for m in (0, 1, 0x3FF)]
    some = np.concatenate([np.arange(1, 60), edges, rng.choice(0x7C00, 512, replace=False)])
    _, first = np.unique(some, return_index=True)
    some = some[np.sort(first)]
    return some[some > 0][:512]


def _sweep(maxima):
    """One row per maximum: all magnitudes up to it, ascending, signs alternating; then the magnitudes from below the maximum down
    to zero with the other sign, as far as the row reaches."""
    column = np.arange(COLUMNS)[None, :]
    top = maxima[:, None].astype(np.int64)
    up = column <= top
    magnitude = np.where(up, column, np.maximum(2 * top - column, 0))
    negative = (column % 2 == 1) ^ ~up
    return (magnitude | (negative.astype(np.int64) << 15)).astype(np.uint16).view(np.float16)


@pytest.mark.parametrize("rows,one_launch", [(512, True), (256, False)])
@pytest.mark.parametrize("fmt", ["fp6", "fp5", "fp4", "fp3"])
def test_every_magnitude_under_a_maximum(pkg, fmt, rows, one_launch):
    print("quantize_pack, all magnitudes: %s, %d rows" % (fmt, rows), flush=True)
    maxima = _maxima()
    assert maxima.size == 512
    W = _sweep(maxima if rows == 512 else maxima[1::2])
    parts = pkg.load_library().fp6_tuning_pack_parts(BITS[fmt], rows, COLUMNS)
    assert parts == (COLUMNS // 1024 if one_launch and fmt != "fp3" else 0)  # 3 bits: this size takes two launches
    packed, scales = getattr(pkg, fmt + "_quantize_pack")(torch.from_numpy(W).cuda())
    ref_packed, ref_scales = _oracle(fmt).quantize_pack(W)
    assert np.array_equal(scales.cpu().numpy().view(np.uint16), np.asarray(ref_scales).view(np.uint16))
    assert np.array_equal(packed.cpu().numpy(), np.asarray(ref_packed).reshape(-1))


SPECIAL = np.array([0x7C00, 0xFC00, 0x7E00, 0xFE00, 0x7C01, 0xFFFF], dtype=np.uint16).view(np.float16)  # +-Inf, NaN of both signs


def _all_largest(W):
    """Finite rows whose codes are the largest magnitude with the signs of W."""
    return np.where(W.view(np.uint16) >> 15, np.float16(-1), np.float16(1)).astype(np.float16)


@pytest.mark.parametrize("M,K,parts", [(48, 1024, 1), (48, 2048, 0), (4096, 4096, 4)])
@pytest.mark.parametrize("fmt", ["fp6", "fp5", "fp4", "fp3"])
def test_rows_with_infinities_and_nan(pkg, fmt, M, K, parts):
    """Not weights, but one answer: the largest magnitude with the sign of each weight of that row; rows beside it are untouched."""
    print("quantize_pack with Inf and NaN: %s M=%d K=%d" % (fmt, M, K), flush=True)
    if fmt == "fp3" and parts > 1:
        M, K, parts = 17200, 15616, 16
    assert pkg.load_library().fp6_tuning_pack_parts(BITS[fmt], M, K) == parts
    rng = np.random.default_rng(K)
    W = rng.normal(0, 0.02, (48, K)).astype(np.float16)
    clean = W.copy()
    for i, special in enumerate(SPECIAL):  # alone in a row, in every part of it, and all of them in one
        W[5 * i, (K - 1) * i // (SPECIAL.size - 1)] = special
        W[40, 7 * i + K // 2] = special
    bad = [5 * i for i in range(SPECIAL.size)] + [40]
    clean[bad] = _all_largest(W[bad])
    whole = torch.zeros((M, K), dtype=torch.float16, device="cuda")
    tiles = [0, 1, M // 16 - 1]
    for k, t in enumerate(tiles):
        whole[16 * t:16 * t + 16] = torch.from_numpy(W[16 * k:16 * k + 16]).cuda()
    packed, scales = getattr(pkg, fmt + "_quantize_pack")(whole)
    ref_packed, ref_scales = _oracle(fmt).quantize_pack(clean)
    tile_bytes, tile_cols = TILE[fmt]
    assert np.array_equal(row_tiles_of(packed, M, K, tiles, tile_bytes, tile_cols), np.asarray(ref_packed).reshape(-1))
    got = np.concatenate([scales[16 * t:16 * t + 16].cpu().numpy() for t in tiles])
    good = np.setdiff1d(np.arange(48), bad)
    assert np.array_equal(got[good].view(np.uint16), np.asarray(ref_scales)[good].view(np.uint16))
    assert not np.isfinite(got[bad]).any()


def test_groups_with_infinities_and_nan(pkg):
    """Group scales: only the group that has them answers so, the other group of the same tile and row keeps its codes and scale."""
    from oracle import fp6g_oracle

    M, K = 32, 512
    rng = np.random.default_rng(128)
    W = rng.normal(0, 0.02, (M, K)).astype(np.float16)
    clean = W.copy()
    bad = []
    for i, special in enumerate(SPECIAL):
        row, group = 5 * i, i % (K // 128)
        W[row, 128 * group + 17 * i] = special
        bad.append((row, group))
        clean[row, 128 * group:128 * group + 128] = _all_largest(W[row:row + 1, 128 * group:128 * group + 128])
    packed, scales = pkg.fp6g_quantize_pack(torch.from_numpy(W).cuda())
    ref_packed, ref_scales = fp6g_oracle.quantize_pack(clean, 128)
    assert np.array_equal(packed.cpu().numpy(), np.asarray(ref_packed).reshape(-1))
    got, want = scales.cpu().numpy().reshape(M, -1), np.asarray(ref_scales).reshape(M, -1)
    kept = np.ones(got.shape, dtype=bool)
    for row, group in bad:
        kept[row, group] = False
        assert not np.isfinite(got[row, group])
    assert np.array_equal(got[kept].view(np.uint16), want[kept].view(np.uint16))
