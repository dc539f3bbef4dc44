"""What the library would launch for a call (host arithmetic of the loaded library, no GPU)."""
import ctypes

STREAM, TILED, BLOCK = 0, 1, 2
BITS = {"fp6": 6, "fp5": 5, "fp4": 4, "fp3": 3, "fp6g": -6, "fp16": 16}


class LaunchPlan(ctypes.Structure):
    _fields_ = [("kernel", ctypes.c_int), ("block_rows", ctypes.c_int), ("block_tokens", ctypes.c_int), ("split_k", ctypes.c_int),
                ("first_token", ctypes.c_int64), ("tokens", ctypes.c_int64), ("counter_bytes", ctypes.c_size_t),
                ("partial_offset", ctypes.c_size_t), ("partial_bytes", ctypes.c_size_t)]


def plan(lib, width, M, N, K, token=0, workspace_bytes=2 ** 64 - 1):
    """The plan, or the status of a refusal."""
    p = LaunchPlan()
    status = lib.fp6_tuning_plan(BITS[width], M, N, K, token, workspace_bytes, ctypes.byref(p))
    return p if status == 0 else status


def k_groups(lib, width, M, N, K, token=0, workspace_bytes=2 ** 64 - 1):
    """Groups of k-tiles of a workgroup of the same launch; 0: refused."""
    return lib.fp6_tuning_plan_k_groups(BITS[width], M, N, K, token, workspace_bytes)


def partials(lib, width, M, N, K, token=0, workspace_bytes=2 ** 64 - 1):
    """Bytes of partial sums that the same launch writes, and that the call asks for; or the status of a refusal."""
    used, required = ctypes.c_size_t(), ctypes.c_size_t()
    status = lib.fp6_tuning_plan_partials(BITS[width], M, N, K, token, workspace_bytes, ctypes.byref(used), ctypes.byref(required))
    return (used.value, required.value) if status == 0 else status


def workspace_bytes(lib, width, M, N, K):
    name = "fp6" if width == "fp6g" else width
    return getattr(lib, name + "_linear_workspace_bytes")(M, N, K)
