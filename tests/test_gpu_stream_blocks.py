"""The streaming kernel's blocks: row tiles, groups of k-tiles and staged tokens, at the sizes where each can go wrong (token
counts at the edges of what is staged, fewer k-tiles than groups, a padded last tile of 3-bit weights, row tiles that do not
fill a block, blocks with k slices)."""
import importlib

import numpy as np
import pytest
import torch

import workloads
from gpu_checks import check_linear
from launch_plans import STREAM, plan

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


# (M, K): one k-tile for eight groups; an odd number of them; a last row block with one row tile; with and without k slices
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
