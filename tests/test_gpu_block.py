"""The block kernel (prompt-sized N: fp16 weights, group scales, large products) against the CPU oracle, with its
blocks pinned so that small inputs reach them: fewer rows and tokens than a block, one more than a block, row counts
that end inside a 16-row tile pair, one k-tile, k-tile counts that the slices and the k groups divide unevenly, more
look-ahead stages than the slice has.  Column bound and regression threshold of gpu_checks."""
import importlib

import numpy as np
import pytest
import torch

import workloads
from gpu_checks import check_linear
from launch_plans import BLOCK, TILED, plan

pytestmark = pytest.mark.gpu

# (format, block) pairs that the block kernel serves
SHAPES = [(f, (256, 256)) for f in ("fp6", "fp5", "fp4", "fp3", "fp16")] + [
    ("fp6g", (256, 128)), ("fp6g", (128, 128)), ("fp16", (256, 128)), ("fp16", (128, 128)), ("fp16", (128, 64))]
# M, K, N, forced split-K factor
SIZES = [(16, 256, 65, 0), (272, 768, 66, 1), (528, 2816, 129, 2), (240, 4352, 257, 3), (1040, 512, 300, 1)]


@pytest.fixture(scope="module")
def pkg():
    import paper_2401_14112_amd as p

    p.load_library()
    return p


def _oracle(width):
    from oracle import fp6_oracle

    fp6_oracle.build()
    if width in ("fp6", "fp16"):
        return fp6_oracle
    from oracle import fpx_oracle

    return fpx_oracle.BY_PREFIX[width] if width in fpx_oracle.BY_PREFIX else importlib.import_module("oracle.%s_oracle" % width)


@pytest.mark.parametrize("M,K,N,split", SIZES)
@pytest.mark.parametrize("width,block", SHAPES)
def test_block_shapes(pkg, width, block, M, K, N, split):
    print("block %s %dx%d M=%d K=%d N=%d split=%d" % (width, *block, M, K, N, split), flush=True)
    o = _oracle(width)
    W, X = workloads.make_weights(M, K, 3 * M + N), workloads.make_activations(N, K, M + N)
    group = (128,) if width == "fp6g" else ()
    if width != "fp16":
        packed, scales = o.quantize_pack(W.numpy(), *group)
        device = (torch.from_numpy(packed).cuda(), torch.from_numpy(scales).cuda())
    pkg.fp6_tuning_set_tile(*block)
    pkg.fp6_tuning_set_split_k(split)
    try:
        if width == "fp16":
            runs = [pkg.fp16_linear(W.cuda(), X.cuda()) for _ in range(2)]
        else:
            runs = [getattr(pkg, width + "_linear")(*device, X.cuda(), M, K, *group) for _ in range(2)]
        torch.cuda.synchronize()
    finally:
        pkg.fp6_tuning_set_tile(0, 0)
        pkg.fp6_tuning_set_split_k(0)
    assert torch.equal(runs[0].view(torch.int16), runs[1].view(torch.int16))
    Y_ref = o.linear_f16(W.numpy(), X.numpy()) if width == "fp16" else o.linear(packed, scales, X.numpy(), M, K, *group)
    check_linear(runs[0].cpu().numpy(), Y_ref, "%s %dx%d M=%d K=%d N=%d split=%d" % (width, *block, M, K, N, split))


@pytest.mark.parametrize("split", [1, 2])
@pytest.mark.parametrize("width,block", [("fp6", (256, 256)), ("fp4", (256, 256)), ("fp6g", (256, 128)), ("fp6g", (128, 128))])
def test_block_fused_steps(pkg, width, block, split):
    M, K, N = 288, 2304, 131
    print("block fused %s %dx%d split=%d" % (width, *block, split), flush=True)
    from oracle import fp6_oracle, fpx_oracle
    o = _oracle(width)
    group = (128,) if width == "fp6g" else ()
    W, X = workloads.make_weights(M, K, 5), workloads.make_activations(N, K, 6)
    amp = 0.02 * np.sqrt(K)   # bias and residual of the size of the products
    bias = (workloads.make_activations(1, M, 7)[0] * amp).to(torch.float16)
    R = (workloads.make_activations(N, M // 2, 8) * amp).to(torch.float16)
    packed, scales = o.quantize_pack(W.numpy(), *group)
    pkg.fp6_tuning_set_tile(*block)
    pkg.fp6_tuning_set_split_k(split)
    try:
        Y = getattr(pkg, width + "_linear_fused")(torch.from_numpy(packed).cuda(), torch.from_numpy(scales).cuda(), X.cuda(),
                                                  M, K, *group, bias=bias.cuda(), residual=R.cuda(), gated=True)
        torch.cuda.synchronize()
    finally:
        pkg.fp6_tuning_set_tile(0, 0)
        pkg.fp6_tuning_set_split_k(0)
    # the steps in 64 bits on the oracle's plain layer
    z = o.linear(packed, scales, X.numpy(), M, K, *group) + bias.numpy().astype(np.float64)
    gate, up = z[:, 0::2], z[:, 1::2]
    Y_ref = gate / (1.0 + np.exp(-gate)) * up + R.numpy().astype(np.float64)
    check_linear(Y.cpu().numpy(), Y_ref, "fused %s %dx%d" % (width, *block))


@pytest.mark.parametrize("width,block,M,K,N", [("fp16", (128, 64), 9616, 256, 130), ("fp6", (256, 256), 5104, 512, 1300),
                                               ("fp6g", (256, 128), 18448, 256, 200)])
def test_block_order_over_several_groups(pkg, width, block, M, K, N):
    """More than eight units per XCD, or numbers of them that eight does not divide: 76 x 3, 20 x 6 and 73 x 2 pieces."""
    print("order %s M=%d K=%d N=%d" % (width, M, K, N), flush=True)
    W, X = workloads.make_weights(M, K, 1, device="cuda"), workloads.make_activations(N, K, 2, device="cuda")
    weights = (W,) if width == "fp16" else getattr(pkg, width + "_quantize_pack")(W)
    dense = W if width == "fp16" else getattr(pkg, width + "_unpack")(*weights, M, K)
    out = torch.full((N, M), float("nan"), dtype=torch.float16, device="cuda")
    pkg.fp6_tuning_set_tile(*block)
    pkg.fp6_tuning_set_split_k(1)
    try:
        p = plan(pkg.load_library(), width, M, N, K)
        assert (p.kernel, p.block_rows, p.block_tokens) == (BLOCK, *block)
        if width == "fp16":
            pkg.fp16_linear(W, X, out=out)
        else:
            getattr(pkg, width + "_linear")(*weights, X, M, K, out=out)
    finally:
        pkg.fp6_tuning_set_tile(0, 0)
        pkg.fp6_tuning_set_split_k(0)
    check_linear(out.cpu().numpy(), (X.float() @ dense.float().t()).cpu().numpy().astype(np.float64), "order %s" % width)


def test_plan_reaches_the_block_kernel_unforced(pkg):
    """6-bit weights: the automatic plan's largest block against the other kernel on the same call."""
    M, K, N = 4096, 512, 3100      # 16 x 13 tiles of 256 x 256 (the last one ragged) against 16 x 25 of 256 x 128
    p = plan(pkg.load_library(), "fp6", M, N, K)
    assert (p.kernel, p.block_rows, p.block_tokens) == (BLOCK, 256, 256)
    print("automatic plan M=%d K=%d N=%d" % (M, K, N), flush=True)
    W = workloads.make_weights(M, K, 1, device="cuda")
    X = workloads.make_activations(N, K, 2, device="cuda")
    packed, scales = pkg.fp6_quantize_pack(W)
    auto = pkg.fp6_linear(packed, scales, X, M, K)
    pkg.fp6_tuning_set_tile(256, 128)
    try:
        assert plan(pkg.load_library(), "fp6", M, N, K).kernel == TILED
        other = pkg.fp6_linear(packed, scales, X, M, K)
    finally:
        pkg.fp6_tuning_set_tile(0, 0)
    ref = (X.float() @ pkg.fp6_unpack(packed, scales, M, K).float().t()).cpu().numpy().astype(np.float64)
    # both against fp32 products of the de-quantized weights (rounded to fp16 once: another 2^-11)
    check_linear(auto.cpu().numpy(), ref, "automatic")
    check_linear(other.cpu().numpy(), ref, "256x128")


@pytest.mark.parametrize("M,K,N,kernel,split", [
    (560, 512, 385, TILED, 1), (528, 1280, 130, TILED, 1), (528, 1536, 130, BLOCK, 1),            # up to 128 blocks
    (4112, 512, 513, TILED, 1), (4112, 1024, 513, BLOCK, 1),                                        # more of them
    (9232, 512, 385, BLOCK, 1),                                                                    # two rounds of the tiled kernel
    (560, 2048, 150, TILED, 2), (16, 6656, 129, TILED, 6), (2064, 3584, 385, BLOCK, 3),            # k slices
    (16, 16384, 129, TILED, 16), (16, 20480, 129, BLOCK, 16), (20464, 3072, 118, TILED, 1)])
def test_group_scales_with_few_k_tiles_per_block(pkg, M, K, N, kernel, split):
    """Either side of the rule that gives short blocks to the tiled kernel, as the automatic plan chooses."""
    print("group scales M=%d K=%d N=%d" % (M, K, N), flush=True)
    p = plan(pkg.load_library(), "fp6g", M, N, K)
    assert (p.kernel, p.split_k) == (kernel, split)
    W, X = workloads.make_weights(M, K, 1, device="cuda"), workloads.make_activations(N, K, 2, device="cuda")
    weights = pkg.fp6g_quantize_pack(W)
    outs = [pkg.fp6g_linear(*weights, X, M, K) for _ in range(2)]
    assert torch.equal(outs[0].view(torch.int16), outs[1].view(torch.int16))
    dense = pkg.fp6g_unpack(*weights, M, K)
    check_linear(outs[0].cpu().numpy(), (X.float() @ dense.float().t()).cpu().numpy().astype(np.float64), "group scales")
