"""The tiled kernel's 128 x 64 block with one and with two groups of k-tiles, which meet in LDS: at either side of the lengths at which
the second group comes in, odd and even numbers of k-tiles, a ragged last row block and token block."""
import importlib

import pytest
import torch

import workloads
from gpu_checks import check_linear
from launch_plans import TILED, k_groups, plan

pytestmark = pytest.mark.gpu


# k-tiles of a slice from which a format takes two groups
TWO_GROUPS_FROM = {"fp6": None, "fp6g": 20, "fp5": 20, "fp4": 12, "fp3": 12}


@pytest.mark.parametrize("split", [1, 2])
@pytest.mark.parametrize("M,K,N", [(32, 256, 65), (144, 2816, 100), (272, 3328, 128), (128, 9472, 77), (144, 10752, 66)])
@pytest.mark.parametrize("width", ["fp6", "fp6g", "fp5", "fp4", "fp3"])
def test_two_k_groups(width, M, K, N, split):
    import paper_2401_14112_amd as pkg
    from oracle import fp6_oracle, fpx_oracle

    o = fp6_oracle if width == "fp6" else fpx_oracle.BY_PREFIX.get(width) or importlib.import_module("oracle.%s_oracle" % width)
    group = (128,) if width == "fp6g" else ()
    print("two k groups %s M=%d K=%d N=%d split=%d" % (width, M, K, N, split), flush=True)
    W, X = workloads.make_weights(M, K, M + N), workloads.make_activations(N, K, K + N)
    packed, scales = o.quantize_pack(W.numpy(), *group)
    device = (torch.from_numpy(packed).cuda(), torch.from_numpy(scales).cuda())
    pkg.fp6_tuning_set_tile(128, 64)
    pkg.fp6_tuning_set_split_k(split)
    try:
        p = plan(pkg.load_library(), width, M, N, K)
        assert (p.kernel, p.block_rows, p.block_tokens) == (TILED, 128, 64)
        start = TWO_GROUPS_FROM[width]
        assert k_groups(pkg.load_library(), width, M, N, K) == (2 if start and K // 256 // p.split_k >= start else 1)
        runs = [getattr(pkg, width + "_linear")(*device, X.cuda(), M, K, *group) for _ in range(2)]
        torch.cuda.synchronize()
    finally:
        pkg.fp6_tuning_set_tile(0, 0)
        pkg.fp6_tuning_set_split_k(0)
    assert torch.equal(runs[0].view(torch.int16), runs[1].view(torch.int16))
    check_linear(runs[0].cpu().numpy(), o.linear(packed, scales, X.numpy(), M, K, *group), "%s %d" % (width, split))


def test_rows_stay_apart():
    """An odd number of k-tiles: the second group multiplies one tile past the end by zero activations.  A row whose neighbour has
    infinite group scales keeps its bits (the tile past the end of a row is the next row's first)."""
    import paper_2401_14112_amd as pkg

    M, K, N = 144, 5376, 80
    print("rows apart M=%d K=%d N=%d" % (M, K, N), flush=True)
    pkg.fp6_tuning_set_tile(128, 64)
    pkg.fp6_tuning_set_split_k(1)
    try:
        lib = pkg.load_library()
        assert plan(lib, "fp6g", M, N, K).kernel == TILED and k_groups(lib, "fp6g", M, N, K) == 2
        packed, scales = pkg.fp6g_quantize_pack(workloads.make_weights(M, K, 1, device="cuda"))
        X = workloads.make_activations(N, K, 2, device="cuda")
        clean = pkg.fp6g_linear(packed, scales, X, M, K)
        bad = torch.arange(0, M, 3)
        poisoned = scales.clone()
        poisoned[bad.cuda()] = float("inf")
        out = pkg.fp6g_linear(packed, poisoned, X, M, K)
    finally:
        pkg.fp6_tuning_set_tile(0, 0)
        pkg.fp6_tuning_set_split_k(0)
    good = torch.ones(M, dtype=torch.bool)
    good[bad] = False
    assert torch.equal(out.cpu()[:, good].view(torch.int16), clean.cpu()[:, good].view(torch.int16))
    assert not torch.isfinite(out.cpu()[:, bad].float()).any()
