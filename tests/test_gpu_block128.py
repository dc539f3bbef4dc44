"""The block kernel's 128 x 128 block with weights of a scale per row (6, 5, 4 and 3 bits), as the plan picks it: ragged last row and
token blocks, one row tile, one and two k-tiles, odd numbers of k-tiles (half a 3-bit tile at the end), with k slices and without, on a workspace of the
queried size, and the steps after the sum."""
import pytest
import torch

import workloads
from gpu_checks import check_linear
from launch_plans import BLOCK, plan, workspace_bytes

pytestmark = pytest.mark.gpu

# M, K, N, k slices
SHAPES = [(16, 256, 129, 1), (272, 256, 300, 1), (144, 512, 130, 1), (1040, 512, 257, 1), (16, 2048, 200, 1), (144, 2048, 130, 1), (272, 2304, 129, 1), (1040, 1024, 257, 1), (2064, 768, 129, 1), (656, 4352, 140, 3),
          (1024, 4096, 256, 4), (1152, 8192, 193, 8)]
NARROW = ["fp5", "fp4", "fp3"]


def _packed(width, M, K):
    from oracle import fp6_oracle, fpx_oracle

    o = fp6_oracle if width == "fp6" else fpx_oracle.BY_PREFIX[width]
    packed, scales = o.quantize_pack(workloads.make_weights(M, K, M + K).numpy())
    return o, packed, scales, (torch.from_numpy(packed).cuda(), torch.from_numpy(scales).cuda())


@pytest.mark.parametrize("M,K,N,split", SHAPES)
@pytest.mark.parametrize("width", ["fp6"] + NARROW)
def test_block_of_128_rows(width, M, K, N, split):
    import paper_2401_14112_amd as pkg

    print("128 x 128 block %s M=%d K=%d N=%d" % (width, M, K, N), flush=True)
    lib = pkg.load_library()
    p = plan(lib, width, M, N, K)
    assert (p.kernel, p.block_rows, p.block_tokens, p.split_k) == (BLOCK, 128, 128, split)
    o, packed, scales, device = _packed(width, M, K)
    X = workloads.make_activations(N, K, K + N)
    nbytes = workspace_bytes(lib, width, M, N, K)
    guard = 4096
    store = torch.full((nbytes + guard,), 0x5A, dtype=torch.uint8, device="cuda")
    workspace = store[:nbytes] if nbytes else None
    if nbytes:
        workspace.zero_()
    runs = [getattr(pkg, width + "_linear")(*device, X.cuda(), M, K, workspace=workspace) for _ in range(2)]
    torch.cuda.synchronize()
    assert bool((store[nbytes:] == 0x5A).all())
    assert torch.equal(runs[0].view(torch.int16), runs[1].view(torch.int16))
    check_linear(runs[0].cpu().numpy(), o.linear(packed, scales, X.numpy(), M, K), "%s %d x %d, N = %d" % (width, M, K, N))


@pytest.mark.parametrize("gated", [False, True])
@pytest.mark.parametrize("M,K,N", [(272, 2304, 129), (656, 4352, 140)])
@pytest.mark.parametrize("width,bits", [("fp6", 6), ("fp4", 4)])
def test_steps_after_the_sum(width, bits, M, K, N, gated):
    import paper_2401_14112_amd as pkg
    from oracle import fp6_oracle

    print("128 x 128 block, steps %s M=%d K=%d N=%d gated=%d" % (width, M, K, N, gated), flush=True)
    assert plan(pkg.load_library(), width, M, N, K).block_rows == 128
    _, packed, scales, device = _packed(width, M, K)
    X = workloads.make_activations(N, K, K + N)
    g = torch.Generator().manual_seed(M)
    bias = (0.5 * torch.randn(M, generator=g)).half()
    residual = torch.randn(N, M // 2 if gated else M, generator=g).half()
    want = fp6_oracle.linear_fused(packed, scales, X.numpy(), M, K, bias=bias.numpy(), residual=residual.numpy(), gated=gated, bits=bits)
    out = residual.cuda()
    got = getattr(pkg, width + "_linear_fused")(*device, X.cuda(), M, K, bias=bias.cuda(), residual=out, gated=gated, out=out)
    check_linear(got.cpu().numpy(), want, "%s gated=%d" % (width, gated))
