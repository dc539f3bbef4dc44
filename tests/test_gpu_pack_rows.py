"""fp6/fp5/fp4/fp3_quantize_pack where one launch reads W once: no exchange (up to 1024 columns), the parts of a row tile agreeing on
its maxima (large matrices), last parts with one k-tile, uneven numbers of row tiles, output buffers full of other bytes.

Codes and scales have one right value: sampled row tiles are compared bit for bit with the oracle's for those rows alone.
"""
import numpy as np
import pytest
import torch

from launch_plans import BITS
from packed_rows import row_tiles_of

pytestmark = pytest.mark.gpu

TILE = {"fp6": (3072, 256), "fp5": (2560, 256), "fp4": (2048, 256), "fp3": (3072, 512)}
SHAPES = [(16, 256), (48, 768), (4112, 1024), (4096, 4096), (1040, 16640), (416, 40960), (52432, 1280)]
# (the last of 3 bits: an odd number of k-tiles, so that the last part ends with half a tile)
CASES = [(f, M, K) for f in ("fp6", "fp5", "fp4") for M, K in SHAPES] + [("fp3", 16, 256), ("fp3", 48, 768), ("fp3", 4112, 1024), ("fp3", 16400, 16384),
                                                                         ("fp3", 17200, 15616)]


@pytest.fixture(scope="module")
def pkg():
    import paper_2401_14112_amd as p

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    p.load_library()
    return p


def _oracle(fmt):
    from oracle import fp6_oracle, fpx_oracle

    return fp6_oracle if fmt == "fp6" else fpx_oracle.BY_PREFIX[fmt]


def _parts(pkg, fmt, M, K):
    return pkg.load_library().fp6_tuning_pack_parts(BITS[fmt], M, K)


def _matrix(M, K, tiles):
    g = torch.Generator(device="cuda")
    g.manual_seed(M + K)
    W = torch.empty((M, K), dtype=torch.float16, device="cuda").normal_(0, 0.02, generator=g)
    for t in tiles:  # rows that differ in where their maximum lies, and rows without one
        W[16 * t, :] = 0
        W[16 * t + 1, :] = -0.0
        W[16 * t + 2, :] = 6e-8  # the scale rounds to zero
        W[16 * t + 3, 0] = 3.0
        W[16 * t + 4, K - 1] = -5.0
        W[16 * t + 5, K // 2] = 65504.0
    return W


@pytest.mark.parametrize("fmt,M,K", CASES)
def test_one_pass_quantize_pack(pkg, fmt, M, K):
    print("quantize_pack %s M=%d K=%d" % (fmt, M, K), flush=True)
    assert _parts(pkg, fmt, M, K) == -(-K // 1024)
    tiles = sorted({0, M // 32, M // 16 - 1})
    W = _matrix(M, K, tiles)
    tile_bytes, tile_cols = TILE[fmt]
    packed = torch.full((-(-K // tile_cols) * (M // 16) * tile_bytes,), 0xFF, dtype=torch.uint8, device="cuda")
    scales = torch.full((M,), float("nan"), dtype=torch.float16, device="cuda")
    rows = np.concatenate([np.arange(16 * t, 16 * t + 16) for t in tiles])
    ref_packed, ref_scales = _oracle(fmt).quantize_pack(W[torch.from_numpy(rows).cuda()].cpu().numpy())
    first = None
    for _ in range(2):
        getattr(pkg, fmt + "_quantize_pack")(W, packed=packed, scales=scales)
        got = row_tiles_of(packed, M, K, tiles, tile_bytes, tile_cols)
        assert np.array_equal(got, np.asarray(ref_packed).reshape(-1))
        assert np.array_equal(scales.cpu().numpy()[rows].view(np.uint16), np.asarray(ref_scales).view(np.uint16))
        assert first is None or torch.equal(first, packed)
        first = packed.clone()


@pytest.mark.parametrize("polls", [0, 1])
@pytest.mark.parametrize("fmt,M,K", [(f, M, K) for f, M, K in CASES if K > 1024])
def test_parts_that_do_not_wait(pkg, fmt, M, K, polls):
    """A part that has not seen the others arrive reads its rows itself and answers for the parts that come later: the same bytes and
    scales, the first tile (where the exchange took place) included."""
    print("quantize_pack, %d polls, %s M=%d K=%d" % (polls, fmt, M, K), flush=True)
    lib = pkg.load_library()
    assert _parts(pkg, fmt, M, K) > 1
    tiles = sorted({0, M // 32, M // 16 - 1})
    W = _matrix(M, K, tiles)
    want, want_scales = getattr(pkg, fmt + "_quantize_pack")(W)
    tile_bytes, tile_cols = TILE[fmt]
    rows = np.concatenate([np.arange(16 * t, 16 * t + 16) for t in tiles])
    ref_packed, ref_scales = _oracle(fmt).quantize_pack(W[torch.from_numpy(rows).cuda()].cpu().numpy())
    packed, scales = torch.full_like(want, 0xFF), torch.full_like(want_scales, float("nan"))
    lib.fp6_tuning_set_pack_polls(polls)
    try:
        for _ in range(2):
            getattr(pkg, fmt + "_quantize_pack")(W, packed=packed, scales=scales)
            torch.cuda.synchronize()
            assert torch.equal(packed, want) and torch.equal(scales.view(torch.int16), want_scales.view(torch.int16))
    finally:
        lib.fp6_tuning_set_pack_polls(-1)
    assert np.array_equal(row_tiles_of(packed, M, K, tiles, tile_bytes, tile_cols), np.asarray(ref_packed).reshape(-1))
    assert np.array_equal(scales.cpu().numpy()[rows].view(np.uint16), np.asarray(ref_scales).view(np.uint16))


@pytest.mark.parametrize("fmt", ["fp6", "fp4"])
def test_one_pass_in_a_graph(pkg, fmt):
    """The exchange is cleared by a launch of the graph: replays on new weights, other work between, give the bytes of eager calls."""
    print("quantize_pack %s in a graph" % fmt, flush=True)
    M, K = 4096, 4096
    assert _parts(pkg, fmt, M, K) > 1
    call = getattr(pkg, fmt + "_quantize_pack")
    W = torch.empty((M, K), dtype=torch.float16, device="cuda")
    packed, scales = call(W.fill_(1.0))
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call(W, packed=packed, scales=scales)
    for seed in range(4):
        W.normal_(0, 0.01 + seed, generator=torch.Generator(device="cuda").manual_seed(seed))
        want, want_scales = call(W)
        packed.fill_(0xA5)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(packed, want) and torch.equal(scales, want_scales), seed


def test_one_pass_on_two_streams(pkg):
    """Parts of two matrices wait for their row tiles on the chip together."""
    print("quantize_pack on two streams", flush=True)
    sizes = {"fp6": (4096, 16640), "fp5": (8192, 8192)}
    jobs = []
    for fmt, (M, K) in sizes.items():
        W = torch.empty((M, K), dtype=torch.float16, device="cuda").normal_(0, 0.02, generator=torch.Generator(device="cuda").manual_seed(M))
        call = getattr(pkg, fmt + "_quantize_pack")
        assert _parts(pkg, fmt, M, K) > 1
        want = call(W)
        jobs.append((call, W, want, [t.clone().fill_(1) for t in want], torch.cuda.Stream()))
    torch.cuda.synchronize()
    for _ in range(6):
        for call, W, _, out, stream in jobs:
            with torch.cuda.stream(stream):
                call(W, packed=out[0], scales=out[1])
    torch.cuda.synchronize()
    for _, _, want, out, _ in jobs:
        assert torch.equal(out[0], want[0]) and torch.equal(out[1], want[1])
