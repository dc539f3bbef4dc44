"""The streaming kernel's blocks: row tiles, groups of k-tiles and staged tokens, at the sizes where each can go wrong (token
counts at the edges of what is staged, groups with fewer k-tiles than others or none, a padded last tile of 3-bit weights, row
tiles that do not fill a block), and every block that a plan takes, with k slices and without."""
import importlib
import random

import numpy as np
import pytest
import torch

import workloads
from gpu_checks import check_linear
from launch_plans import STREAM, k_groups, plan

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pkg():
    import paper_2401_14112_amd as p

    p.load_library()
    return p


def _oracle(width):
    from oracle import fp6_oracle, fpx_oracle
    if width in ("fp6", "fp16"):
        return fp6_oracle
    return fpx_oracle.BY_PREFIX[width] if width in fpx_oracle.BY_PREFIX else importlib.import_module("oracle.%s_oracle" % width)


# (M, K): one k-tile; nine for two to eight groups; five, eight groups (packed weights, up to 16 tokens), a last row block with few row
# tiles; three; 31 in k slices; two, more row blocks than CUs
SIZES = [(32, 256), (144, 2304), (2192, 1280), (4112, 768), (400, 7936), (6160, 512)]


@pytest.mark.parametrize("N", [1, 2, 3, 8, 9, 16, 17, 33, 48, 49, 64])
@pytest.mark.parametrize("width", ["fp6", "fp6g", "fp5", "fp4", "fp3", "fp16"])
def test_blocks(pkg, width, N):
    lib = pkg.load_library()
    o = _oracle(width)
    group = (128,) if width == "fp6g" else ()
    rows = set()
    for M, K in SIZES:
        p = plan(lib, width, M, N, K)
        assert p.kernel == STREAM
        rows.add((p.block_rows, p.split_k > 1))
        print("%s M=%d K=%d N=%d: %d rows, %d slices" % (width, M, K, N, p.block_rows, p.split_k), flush=True)
        W, X = workloads.make_weights(M, K, 3 * M + N), workloads.make_activations(N, K, M + N)
        if width == "fp16":
            runs = [pkg.fp16_linear(W.cuda(), X.cuda()) for _ in range(2)]
            Y_ref = o.linear_f16(W.numpy(), X.numpy())
        else:
            packed, scales = o.quantize_pack(W.numpy(), *group)
            device = (torch.from_numpy(packed).cuda(), torch.from_numpy(scales).cuda())
            runs = [getattr(pkg, width + "_linear")(*device, X.cuda(), M, K, *group) for _ in range(2)]
            Y_ref = o.linear(packed, scales, X.numpy(), M, K, *group)
        assert torch.equal(runs[0].view(torch.int16), runs[1].view(torch.int16))
        check_linear(runs[0].cpu().numpy(), Y_ref, "%s M=%d K=%d N=%d" % (width, M, K, N))
    assert len(rows) > 1, "the sizes are meant to reach several blocks"


def _blocks_taken(lib, width, N):
    """{(row tiles, k groups, has k slices): (M, K)} over the plan's choices, each at the smallest layer drawn for it; where one has a
    last row block that is not full, at the smallest of those."""
    rng = random.Random(N)
    taken = {}
    for _ in range(20000):
        M, K = 16 * round(3584 ** rng.random()), 256 * round(112 ** rng.random())
        p = plan(lib, width, M, N, K)
        key = (p.block_rows // 16, k_groups(lib, width, M, N, K), p.split_k > 1)
        size = (M % p.block_rows == 0, M * K)
        if key not in taken or size < taken[key][0]:
            taken[key] = size, M, K
    return {key: (M, K) for key, (_, M, K) in taken.items()}


def _blocks(width, N):
    """(row tiles, k groups) of the blocks that there are for a token count."""
    if width == "fp16":
        return {(8, 1), (4, 1), (4, 2), (1, 4)} if N <= 16 else {(8, 1), (6, 1), (2, 2)} if N <= 32 else {(4, 1), (6, 1)}
    if width == "fp3":  # twice the columns per k-tile: fewer groups fit the LDS
        return ({(8, 1), (4, 2), (2, 4), (1, 8)} if N <= 8 else {(8, 1), (4, 2), (2, 4)} if N <= 16 else
                {(8, 1), (6, 1), (4, 2)} if N <= 32 else {(8, 1), (6, 1)})
    return ({(8, 1), (4, 2), (2, 4), (1, 8)} if N <= 16 else {(8, 1), (6, 1), (4, 2), (2, 4)} if N <= 32 else
            {(8, 1), (6, 1), (4, 2)})


@pytest.mark.parametrize("N", [2, 8, 15, 17, 33, 64])
@pytest.mark.parametrize("width", ["fp6", "fp6g", "fp5", "fp4", "fp3", "fp16"])
def test_every_block_with_and_without_slices(pkg, width, N):
    """Against fp32 products with the code values (fp6g, fp16: with the fp16 weights)."""
    lib = pkg.load_library()
    taken = _blocks_taken(lib, width, N)
    missing = {(rows, groups, slices) for rows, groups in _blocks(width, N) for slices in (False, True)} - set(taken)
    # with four token tiles (3 bits: with two as well) six row tiles take k slices, of fp16 weights none, of group scales both
    assert missing == ({(6, 1, width == "fp16")} if N > 48 and width != "fp6g" or N == 17 and width == "fp3" else set()), missing
    assert {key[:2] for key in taken} == _blocks(width, N)
    for (rows, groups, slices), (M, K) in sorted(taken.items()):
        print("%s M=%d K=%d N=%d: %d row tiles x %d groups%s" % (width, M, K, N, rows, groups, ", slices" if slices else ""), flush=True)
        W, X = workloads.make_weights(M, K, M + N, device="cuda"), workloads.make_activations(N, K, K + N, device="cuda")
        if width == "fp16":
            runs = [pkg.fp16_linear(W, X) for _ in range(2)]
            ref = X.float() @ W.float().t()
        else:
            packed, scales = getattr(pkg, width + "_quantize_pack")(W)
            runs = [getattr(pkg, width + "_linear")(packed, scales, X, M, K) for _ in range(2)]
            if width == "fp6g":
                ref = X.float() @ pkg.fp6g_unpack(packed, scales, M, K).float().t()
            else:
                ref = X.float() @ getattr(pkg, width + "_unpack")(packed, torch.ones_like(scales), M, K).float().t() * scales.float()
        assert torch.equal(runs[0].view(torch.int16), runs[1].view(torch.int16))
        check_linear(runs[0].cpu().numpy(), ref.cpu().numpy().astype(np.float64), "%s M=%d K=%d N=%d" % (width, M, K, N))


@pytest.mark.parametrize("width,M,K,N,slices", [("fp16", 1504, 2304, 6, 2), ("fp16", 1088, 2816, 2, 3), ("fp6g", 64, 4352, 16, 4), ("fp5", 96, 5120, 11, 5),
                                                ("fp6", 112, 6400, 9, 6), ("fp16", 64, 14848, 5, 7), ("fp16", 112, 17152, 2, 8), ("fp16", 128, 9216, 4, 9),
                                                ("fp16", 96, 21760, 6, 10), ("fp6", 176, 21248, 10, 11), ("fp16", 304, 13312, 2, 13)])
def test_slice_counts_of_one_token_tile(pkg, width, M, K, N, slices):
    """Whole and last batches of the other slices' partial tiles, the own one first, between and last: any wave may be the last to
    arrive, and the bits may not depend on which."""
    print("slices %s M=%d K=%d N=%d: %d" % (width, M, K, N, slices), flush=True)
    assert plan(pkg.load_library(), width, M, N, K).split_k == slices
    W, X = workloads.make_weights(M, K, M + N, device="cuda"), workloads.make_activations(N, K, K + N, device="cuda")
    if width == "fp16":
        call, ref = (lambda: pkg.fp16_linear(W, X)), X.float() @ W.float().t()
    else:
        packed, scales = getattr(pkg, width + "_quantize_pack")(W)
        call = lambda: getattr(pkg, width + "_linear")(packed, scales, X, M, K)
        if width == "fp6g":
            ref = X.float() @ pkg.fp6g_unpack(packed, scales, M, K).float().t()
        else:
            ref = X.float() @ getattr(pkg, width + "_unpack")(packed, torch.ones_like(scales), M, K).float().t() * scales.float()
    first = call()
    for _ in range(20):
        assert torch.equal(call().view(torch.int16), first.view(torch.int16))
    check_linear(first.cpu().numpy(), ref.cpu().numpy().astype(np.float64), "%s M=%d K=%d N=%d" % (width, M, K, N))


@pytest.mark.parametrize("width", ["fp6", "fp6g", "fp5", "fp4", "fp3", "fp16"])
@pytest.mark.parametrize("M,K,N", [(32, 256, 2), (144, 2304, 7), (2192, 1280, 16), (400, 7936, 33)])
def test_tokens_stay_apart(pkg, width, M, K, N):
    """A token of infinities and NaN changes no other token's bits (the padding of a tile, and what a lane without a token
    of its own reads, are multiplied too)."""
    print("tokens apart %s M=%d K=%d N=%d" % (width, M, K, N), flush=True)
    W, X = workloads.make_weights(M, K, 5, device="cuda"), workloads.make_activations(N, K, 6, device="cuda")
    weights = (W,) if width == "fp16" else getattr(pkg, width + "_quantize_pack")(W)
    call = (lambda x: pkg.fp16_linear(W, x)) if width == "fp16" else (lambda x: getattr(pkg, width + "_linear")(*weights, x, M, K))
    clean = call(X)
    for bad in range(N):
        poisoned = X.clone()
        poisoned[bad, 0::2], poisoned[bad, 1::2] = float("inf"), float("nan")
        out = call(poisoned)
        others = [n for n in range(N) if n != bad]
        assert torch.equal(out[others].view(torch.int16), clean[others].view(torch.int16)), bad
        assert torch.isnan(out[bad].float()).all()


def test_fused_steps_of_a_grouped_block(pkg):
    M, K, N = 4096, 1024, 5
    o = _oracle("fp6")
    assert plan(pkg.load_library(), "fp6", M, N, K).block_rows < 128
    W, X = workloads.make_weights(M, K, 9), workloads.make_activations(N, K, 10)
    bias = (workloads.make_activations(1, M, 11)[0] * 0.02 * np.sqrt(K)).to(torch.float16)
    R = workloads.make_activations(N, M // 2, 12)
    packed, scales = o.quantize_pack(W.numpy())
    Y = pkg.fp6_linear_fused(torch.from_numpy(packed).cuda(), torch.from_numpy(scales).cuda(), X.cuda(), M, K,
                             bias=bias.cuda(), residual=R.cuda(), gated=True)
    Y_ref = o.linear_fused(packed, scales, X.numpy(), M, K, bias=bias.numpy(), residual=R.numpy(), gated=True)
    check_linear(Y.cpu().numpy(), Y_ref, "fused grouped block")
