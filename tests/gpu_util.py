"""Helpers for the GPU parity tests: numpy <-> device tensors and error metrics."""
import ctypes

import numpy as np
import torch

from paper_2503_08640_amd import binding, synth

MAX_ABS_TOL = 2e-2    # bf16 inputs vs the fp64 oracle
MEAN_ABS_TOL = 2e-3


def to_dev(x: np.ndarray) -> torch.Tensor:
    """fp32 array or bf16 bit patterns -> device tensor of the same values."""
    if x.dtype == np.uint16:
        return torch.from_numpy(x.view(np.int16)).cuda().view(torch.bfloat16)
    return torch.from_numpy(np.ascontiguousarray(x, dtype=np.float32)).cuda()


def to_f64(t: torch.Tensor) -> np.ndarray:
    return t.detach().float().cpu().numpy().astype(np.float64)


def two_waves(layout, classes, cuts=False):
    """Whether a head_dim 64 launch over `layout` runs two waves to a SIMD with `classes` workers per head block
    (the library's own C++ rule)."""
    rule = binding.lib()._Z16dbsa_crowd_worthPK11dbsa_layoutlb
    rule.restype, rule.argtypes = ctypes.c_bool, [ctypes.c_void_p, ctypes.c_int64, ctypes.c_bool]
    return bool(rule(layout.handle, classes, cuts))


def errors(got: np.ndarray, want: np.ndarray):
    d = np.abs(got - want)
    return float(d.max()), float(d.mean())


def assert_close(got, want, what="", max_tol=MAX_ABS_TOL, mean_tol=MEAN_ABS_TOL):
    assert np.all(np.isfinite(got)), f"{what}: non-finite output"
    mx, mean = errors(got, want)
    print(f"[parity] {what}: max-abs {mx:.3e} mean-abs {mean:.3e}", flush=True)
    assert mx <= max_tol and mean <= mean_tol, f"{what}: max-abs {mx:.3e} mean-abs {mean:.3e}"


def pool_f64(pc):
    return synth.as_f64(pc.q), synth.as_f64(pc.k), synth.as_f64(pc.v)
