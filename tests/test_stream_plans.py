"""The streaming kernel's plans (CPU only): what a call asks its caller for depends on the shape, not on the block chosen."""
import random

from launch_plans import BITS, STREAM, plan, workspace_bytes

REFUSED = 3  # FP6_ERR_WORKSPACE
REGION = 4096


def _slices(width, M, N, K):
    """k slices and token tiles of blocks of eight (four) row tiles, which the workspace is sized for."""
    row_tiles, cols = M // 16, 512 if width == "fp3" else 256
    k_tiles = -(-K // cols)
    most = k_tiles // 2 if k_tiles >= 4 else 1
    best = None
    for waves in ([4] if width == "fp16" and N > 32 else [4, 8] if N <= 16 else [8]):
        rb = -(-row_tiles // waves)
        s = max(1, min(256 // rb, most, 64))
        key = (rb * s <= 256, rb * s if rb * s <= 256 else -rb * s, s)
        best = max(best, key) if best else key
    return best[2], 1 if N <= 16 else 2 if N <= 32 else 4


def test_what_a_call_asks_for():
    import paper_2401_14112_amd as pkg

    lib = pkg.load_library()
    rng = random.Random(2)
    without = with_slices = 0
    for _ in range(3000):
        width = rng.choice(list(BITS))
        M, K = 16 * round(2 ** rng.uniform(0, 11.8)), 256 * round(2 ** rng.uniform(0, 6.8))
        N = rng.randint(1, 1 << rng.randint(0, 6))
        s, tiles = _slices(width, M, N, K)
        most = REGION + s * (M // 16) * tiles * 1024 if s > 1 else 0
        p = plan(lib, width, M, N, K)
        assert p.kernel == STREAM and p.block_tokens >= N and p.split_k <= s * tiles
        # the k slices of the plan, or those of blocks of eight row tiles where it has none; the most of the formats that share a query
        sharing = (width,) if width in ("fp3", "fp16") else ("fp6", "fp5", "fp4", "fp6g")
        asked = {}
        for w in sharing:
            q = plan(lib, w, M, N, K)
            asked[w] = q.partial_offset + q.partial_bytes if q.split_k > 1 else most
        assert workspace_bytes(lib, width, M, N, K) == max(asked.values()), (width, M, N, K)
        assert s == 1 or plan(lib, width, M, N, K, workspace_bytes=asked[width] - 1) == REFUSED
        # what was enough for eight row tiles is enough, and without any the call runs where those took no slices
        assert plan(lib, width, M, N, K, workspace_bytes=most) != REFUSED, (width, M, N, K)
        assert (plan(lib, width, M, N, K, workspace_bytes=0) == REFUSED) == (s > 1), (width, M, N, K)
        with_slices += p.split_k > 1
        without += p.split_k == 1 and s > 1
    assert with_slices > 300 and without > 300


def test_group_scales_take_every_block_of_six_bits():
    """Nothing but the LDS, the same for both, says which blocks exist."""
    import paper_2401_14112_amd as pkg

    lib = pkg.load_library()
    for N in (1, 2, 3, 8, 9, 16, 17, 32, 33, 48, 49, 64):
        blocks = {w: {plan(lib, w, M, N, K).block_rows for M in range(256, 16384, 496) for K in (512, 1024, 2048, 4096, 8192, 22016)}
                  for w in ("fp6", "fp6g")}
        assert blocks["fp6"] == blocks["fp6g"], N
    assert plan(lib, "fp6g", 8192, 16, 2048).block_rows == 32


def test_fp16_ties_go_to_the_fuller_chip():
    """Two blocks at the memory's rate have one estimate: 43 row blocks of eight row tiles x 3 slices, or 85 of four x 3."""
    import paper_2401_14112_amd as pkg

    p = plan(pkg.load_library(), "fp16", 5424, 9, 20992)
    assert (p.block_rows, p.split_k) == (64, 3)


def test_six_row_tiles_with_four_token_tiles_take_slices():
    """Without k slices eight are faster (18608 x 22272, N = 57)."""
    import paper_2401_14112_amd as pkg

    lib = pkg.load_library()
    rng = random.Random(6)
    six = 0
    for _ in range(4000):
        width, M = rng.choice(["fp6", "fp5", "fp4", "fp3", "fp6g"]), 16 * round(3584 ** rng.random())
        p = plan(lib, width, M, rng.randint(49, 64), 256 * round(112 ** rng.random()))
        assert p.block_rows != 96 or p.split_k > 1 or (width == "fp6g" and M > 16384)
        six += p.block_rows == 96
    assert six > 100 and plan(lib, "fp5", 18608, 57, 22272).block_rows == 128
