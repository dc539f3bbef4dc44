"""Where the launches of a call keep their split-K state (CPU only: the plans are host arithmetic).  Every launch counts
arrivals in the counters that the launches before it left at zero, so no launch may keep partial sums where another one
that uses the workspace, in the same call or a later one, counts."""
import random

import pytest

from launch_plans import BITS, BLOCK, STREAM, TILED, k_groups, partials, plan, workspace_bytes


@pytest.fixture(scope="module")
def lib():
    import paper_2401_14112_amd as pkg

    return pkg.load_library()


def _launches(lib, width, M, N, K):
    first = plan(lib, width, M, N, K)
    assert first.first_token == 0
    last = plan(lib, width, M, N, K, N - 1)
    assert last.first_token + last.tokens == N and last.tokens <= first.tokens
    return [first, last]


def _check(lib, shapes):
    """All launches of all calls in `shapes` on one workspace of the largest size queried."""
    launches = []
    for width, M, N, K in shapes:
        need = workspace_bytes(lib, width, M, N, K)
        for p in _launches(lib, width, M, N, K):
            assert (p.partial_bytes == 0) == (p.counter_bytes == 0) == (p.split_k == 1)
            if p.split_k > 1:
                assert p.partial_offset + p.partial_bytes <= need, (width, M, N, K)
                assert p.partial_offset % 16 == 0
                assert p.counter_bytes <= lib.fp6_workspace_zero_bytes(M, N, K)
                launches.append(((width, M, N, K), p))
    for a, p in launches:
        for b, q in launches:
            assert q.counter_bytes <= p.partial_offset, "counters of %s lie in the partial sums of %s" % (b, a)
    return launches


@pytest.mark.parametrize("width,M,N,K", [
    # X beyond 2 GiB: a full chunk and a shorter last one with different blocks and more counters ...
    ("fp16", 128, 33088, 49152), ("fp6g", 384, 12864, 139264),
    # ... or fewer, so that the last launch of one call could write where the first of the next one counts
    ("fp16", 2048, 1200, 1 << 20), ("fp6", 16, 400, (1 << 23) - 256), ("fp6g", 1024, 6000, 1 << 18)])
def test_launches_of_a_chunked_call(lib, width, M, N, K):
    a, b = _launches(lib, width, M, N, K)
    assert a.first_token != b.first_token, "the case is meant to be cut into chunks"
    assert _check(lib, [(width, M, N, K)])


@pytest.mark.parametrize("N", [1, 16, 17, 33, 64, 65, 100, 200, 512])
def test_formats_share_the_workspace_of_a_shape(lib, N):
    assert _check(lib, [(w, 8192, N, 8192) for w in BITS])


def test_any_calls_share_a_workspace(lib):
    rng = random.Random(0)
    for _ in range(200):
        shapes = []
        for _ in range(6):
            M, K = 16 * rng.randint(1, 1 << rng.randint(0, 11)), 256 * rng.randint(1, 1 << rng.randint(0, 7))
            shapes.append((rng.choice(list(BITS)), M, rng.randint(1, 1 << rng.randint(0, 12)), K))
        _check(lib, shapes)


@pytest.mark.parametrize("split", [2, 5, 16])
def test_forced_split_factors_on_one_shape(lib, split):
    lib.fp6_tuning_set_split_k(split)
    try:
        for M, N, K in [(8192, 16, 8192), (28672, 200, 4096), (57344, 700, 4096), (128, 33088, 49152)]:
            assert _check(lib, [(w, M, N, K) for w in BITS])
    finally:
        lib.fp6_tuning_set_split_k(0)


REFUSED = 3  # FP6_ERR_WORKSPACE


@pytest.mark.parametrize("width,M,N,K", [("fp16", 8192, 512, 22016), ("fp16", 8288, 68, 2048), ("fp6g", 4096, 640, 8192),
                                         ("fp6g", 16640, 100, 4096)])
def test_calls_whose_small_blocks_fill_the_chip_need_no_workspace(lib, width, M, N, K):
    """More than 128 blocks of 128 x 128 (128 x 64) outputs: no k slices needed, though the best plan has some."""
    queried = workspace_bytes(lib, width, M, N, K)
    best = plan(lib, width, M, N, K, workspace_bytes=queried)
    assert best.split_k > 1
    assert plan(lib, width, M, N, K, workspace_bytes=0).split_k == 1
    for have in range(0, queried, queried // 7):
        p = plan(lib, width, M, N, K, workspace_bytes=have)
        assert p.split_k == 1 or p.partial_offset + p.partial_bytes <= have


def test_smaller_workspaces_are_refused_otherwise(lib):
    rng = random.Random(1)
    refused = 0
    for _ in range(400):
        width = rng.choice(list(BITS))
        M, K = 16 * rng.randint(1, 1 << rng.randint(0, 11)), 256 * rng.randint(8, 64)
        N = rng.randint(1, 1 << rng.randint(0, 10))
        best = plan(lib, width, M, N, K)
        if best.split_k == 1:
            continue
        need = best.partial_offset + best.partial_bytes
        assert plan(lib, width, M, N, K, workspace_bytes=need).split_k == best.split_k
        less = plan(lib, width, M, N, K, workspace_bytes=need - 16)
        tokens = 64 if N <= 128 and (M + 255) // 256 < 64 else 128
        blocks = (M + 127) // 128 * ((N + tokens - 1) // tokens)
        if N <= 64 or width not in ("fp6g", "fp16"):
            assert less == REFUSED, (width, M, N, K)
            refused += 1
        elif blocks <= 128:
            assert plan(lib, width, M, N, K, workspace_bytes=0) == REFUSED, (width, M, N, K)
            refused += 1
        if less != REFUSED:
            assert less.split_k == 1 or less.partial_offset + less.partial_bytes <= need - 16
    assert refused > 50


# {rows, tokens}: figures by which the block of fp16_linear was chosen before they were measured anew, ns per run of 32 columns
FP16_ACCEPTED = {(256, 256): 924.0, (256, 128): 632.0, (128, 128): 333.0, (128, 64): 228.0}


def _fp16_accepted(M, N, K):
    """Partial sums of the block with the least estimated time by those figures."""
    best = None
    for (rows, tokens), ns in FP16_ACCEPTED.items():
        tiles, k_tiles = -(-M // rows) * -(-N // tokens), K // 256
        s = max(1, min(256 // tiles, k_tiles // 4 if k_tiles >= 8 else 1, 16))
        partials = s * tiles * rows * tokens * 4 if s > 1 else 0
        cost = -(-tiles * s // 256) * (8.0 * -(-k_tiles // s) * ns + 8000.0)
        if s > 1:
            cost += s * rows * tokens * 4.0 / 50.0 + partials * 1.5e-4
        if best is None or cost < best[0]:
            best = cost, partials
    return best[1]


def test_fp16_calls_that_ran_still_run(lib):
    """What a call of fp16_linear asks for at least does not move with the figures that choose its block."""
    rng = random.Random(4)
    shapes = [(5328, 352, 3328), (784, 1656, 2048), (2224, 646, 2816)]
    while len(shapes) < 6000:
        M, K = 16 * round(2 ** rng.uniform(4, 11.8)), 256 * round(2 ** rng.uniform(1, 6.8))
        shapes.append((M, round(2 ** rng.uniform(6.1, 12)), K))
    smaller = without = 0
    for M, N, K in shapes:
        partials = _fp16_accepted(M, N, K)
        have = 4096 + partials if partials else 0
        p = plan(lib, "fp16", M, N, K, workspace_bytes=have)
        assert p != REFUSED, (M, N, K, have)
        assert p.split_k == 1 or p.partial_offset + p.partial_bytes <= have
        more = have < workspace_bytes(lib, "fp16", M, N, K)
        smaller += more and have > 0
        without += more and have == 0
    assert smaller > 10 and without > 3


@pytest.mark.parametrize("width,K,groups", [("fp6", 8192, 1), ("fp6", 98304, 1), ("fp5", 65536, 1), ("fp5", 98304, 2), ("fp4", 32768, 1),
                                            ("fp4", 49152, 2), ("fp3", 65536, 2), ("fp6g", 65536, 1), ("fp6g", 98304, 2)])
def test_tiled_counters_are_one_per_wave(lib, width, K, groups):
    """One arrival counter per wave that the launch has, 128 bytes apart where there are few."""
    M, N = 128, 80
    p = plan(lib, width, M, N, K)
    assert (p.kernel, p.block_rows, p.block_tokens) == (TILED, 128, 64) and p.split_k > 1
    assert k_groups(lib, width, M, N, K) == groups
    assert p.counter_bytes == 2 * 4 * groups * 128


def _tiled_partials(M, N, K):
    """Partial sums of the tiled kernel's plan for weights with a scale per row."""
    rows, tokens = (128, 64) if N <= 128 and -(-M // 256) < 64 else (256, 128)
    n_blocks, k_tiles = -(-N // tokens), K // 256
    s = max(1, min(256 // (-(-M // rows) * n_blocks), k_tiles // 4 if k_tiles >= 8 else 1, 16))
    return s * (M // 16) * n_blocks * (tokens // 16) * 1024 if s > 1 else 0


def test_blocks_in_place_of_tiled_ones_ask_for_what_those_did(lib):
    """The 128 x 128 block takes calls from the tiled kernel: size query, acceptance and refusal are those of the tiled plan, and what
    is launched stays within them."""
    rng = random.Random(7)
    sliced = whole = 0
    for _ in range(4000):
        width = rng.choice(["fp6", "fp5", "fp4", "fp3"])
        M, K = 16 * round(2 ** rng.uniform(0, 11.8)), 256 * round(2 ** rng.uniform(0, 6.8))
        N = round(2 ** rng.uniform(6.1, 12))
        p = plan(lib, width, M, N, K)
        if (p.kernel, p.block_rows, p.block_tokens) != (BLOCK, 128, 128):
            continue
        partials, need = _tiled_partials(M, N, K), workspace_bytes(lib, width, M, N, K)
        own = p.split_k * -(-M // 128) * -(-N // 128) * 128 * 128 * 4 if p.split_k > 1 else 0
        assert own <= partials, (width, M, N, K)
        if not partials:
            assert p.split_k == 1 and plan(lib, width, M, N, K, workspace_bytes=0) != REFUSED
            whole += 1
            continue
        sliced += 1
        assert plan(lib, width, M, N, K, workspace_bytes=need) != REFUSED, (width, M, N, K)
        if p.split_k == 1:  # no counters in use that would say where the partial sums begin
            assert plan(lib, width, M, N, K, workspace_bytes=partials - 16) == REFUSED, (width, M, N, K)
            continue
        least = p.partial_offset + partials
        assert p.counter_bytes <= p.partial_offset and least <= need, (width, M, N, K)
        assert plan(lib, width, M, N, K, workspace_bytes=least).split_k == p.split_k
        assert plan(lib, width, M, N, K, workspace_bytes=least - 16) == REFUSED, (width, M, N, K)
    assert sliced > 50 and whole > 50


@pytest.mark.parametrize("width,M,N,K", [("fp3", 16, 309, 22016), ("fp3", 16, 847, 14080), ("fp4", 16, 694, 8448), ("fp5", 32, 183, 14592), ("fp6", 32, 183, 23552)])
def test_few_rows_keep_their_k_slices(lib, width, M, N, K):
    """The partial sums of few rows are small, and the 128 x 128 block, held to them, would take a third of the tiled kernel's slices or less."""
    assert plan(lib, width, M, N, K).kernel == TILED


def test_partial_sums_used_and_required(lib):
    """What a launch writes, from its block and k slices, lies within what the call asks for; with that much it runs, with less it is
    refused or takes another plan."""
    rng = random.Random(11)
    more_than_used = untouched = 0
    for _ in range(4000):
        width = rng.choice(list(BITS))
        M, K = 16 * round(2 ** rng.uniform(0, 11.8)), 256 * round(2 ** rng.uniform(0, 6.8))
        N = round(2 ** rng.uniform(0, 12))
        p, (used, required) = plan(lib, width, M, N, K), partials(lib, width, M, N, K)
        rows = M if p.kernel != BLOCK else -(-M // p.block_rows) * p.block_rows  # the block kernel keeps whole blocks
        tokens = p.block_tokens if p.kernel == STREAM else -(-N // p.block_tokens) * p.block_tokens
        assert used == (p.split_k * rows * tokens * 4 if p.split_k > 1 else 0), (width, M, N, K)
        assert used <= required <= workspace_bytes(lib, width, M, N, K)
        assert p.partial_bytes == (required if p.split_k > 1 else 0)
        more_than_used += 0 < used < required
        untouched += used == 0 < required
        if required == 0:
            assert partials(lib, width, M, N, K, workspace_bytes=0) == (0, 0)
            continue
        least = p.partial_offset + required
        assert partials(lib, width, M, N, K, workspace_bytes=least) == (used, required)
        less = plan(lib, width, M, N, K, workspace_bytes=least - 16)
        assert less == REFUSED or (less.kernel, less.block_rows, less.block_tokens, less.split_k) != (p.kernel, p.block_rows, p.block_tokens,
                                                                                                    p.split_k), (width, M, N, K)
        assert less == REFUSED or width in ("fp16", "fp6g")
    assert more_than_used > 50 and untouched > 50
