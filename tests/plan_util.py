"""What the library's size rules give a call, from the debug build's host-only hooks (no GPU needed; 256 compute units
are assumed where there is none)."""
import ctypes as C
import os

from paper_2606_19004_amd import ditstep

LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2606_19004_amd", "libditstep_debug.so")
OPS = ("patch", "qkv", "out", "mlp_up", "mlp_down")
_lib = None


def debug_lib():
    global _lib
    if _lib is None:
        _lib = C.CDLL(LIB)
        _lib.dit_debug_gemm_plan.argtypes = [C.POINTER(ditstep.BlockConfig), C.c_int32, C.c_int32, C.c_int32, C.c_void_p]
        _lib.dit_debug_reward_check_in_launch.argtypes = [C.c_int32, C.c_int32]
    return _lib


def reward_check_in_launch(groups, n):
    return bool(debug_lib().dit_debug_reward_check_in_launch(groups, n))


def gemm_plan(cfg, batch, op, latent_dim=64):
    """(tile rows, tile columns, columns of a second launch's tiles or 0, workgroups that share a tile's K, LDS stages of
    a ring kernel or 0)"""
    out = (C.c_int32 * 5)()
    assert debug_lib().dit_debug_gemm_plan(C.byref(cfg), batch, latent_dim, OPS.index(op), out) == 0
    return tuple(out)
