"""The library's host-side choice of a search, through its C++ symbols (no GPU needed)."""
import ctypes
import functools

import torch

CUS = 256                                                   # compute units: one workgroup of the walk on each


class WalkPlan(ctypes.Structure):
    """struct WalkPlan of csrc/ttf_internal.h."""
    _fields_ = [("ok", ctypes.c_bool), ("patch", ctypes.c_bool)] + [
        (n, ctypes.c_int) for n in ("nk", "lines", "lsegs", "ysegs", "groups", "nf")] + [("tiles", ctypes.c_double)]


def params(B, F, H, W, C, dtype, r=1):
    from paper_2605_07355_amd import binding
    return binding._Params(B, F, H, W, C, binding.TTF_F32 if dtype == torch.float32 else binding.TTF_BF16, r, 0.7, 0, 0)


@functools.lru_cache(None)
def _symbol(name, restype, *argtypes):
    import paper_2605_07355_amd as ttf
    f = getattr(ttf.load_library(), name)
    f.restype, f.argtypes = restype, list(argtypes)
    return f


def walk_plan(p, frames, sums):
    """How the walk deals `frames` frames a clip to workgroups."""
    f = _symbol("_ZN3ttf9walk_planERK10ttf_paramsib", WalkPlan, ctypes.c_void_p, ctypes.c_int, ctypes.c_bool)
    return f(ctypes.addressof(p), frames, sums)


def units(p, plan):
    return p.B * plan.nk * plan.groups * plan.lsegs * plan.ysegs


def search_walks(p, segment=False):
    f = _symbol("_ZN3ttf12search_walksERK10ttf_paramsb", ctypes.c_bool, ctypes.c_void_p, ctypes.c_bool)
    return f(ctypes.addressof(p), segment)


def matrix_cores(p, segment=False):
    """Whether a search that does not walk runs on the matrix cores."""
    f = _symbol("_ZN3ttf13use_mfma_pathERK10ttf_paramsbb", ctypes.c_bool, ctypes.c_void_p, ctypes.c_bool, ctypes.c_bool)
    return f(ctypes.addressof(p), True, segment)


def search_guesses(p, mode):
    """How many clips have to have a clear guess for any to be taken; -1: anchors are not guessed."""
    f = _symbol("_ZN3ttf14search_guessesERK10ttf_paramsi", ctypes.c_int, ctypes.c_void_p, ctypes.c_int)
    return f(ctypes.addressof(p), mode)


def kept_share(p, walks, mfma):
    """Share of the input that the frame sums leave in the caches for the search."""
    f = _symbol("_ZN3ttf10kept_shareERK10ttf_paramsbb", ctypes.c_double, ctypes.c_void_p, ctypes.c_bool, ctypes.c_bool)
    return f(ctypes.addressof(p), walks, mfma)
