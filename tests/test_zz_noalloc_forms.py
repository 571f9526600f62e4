"""kp_phi_combo_noalloc against kp_phi_combo where the kernel depends on the
form and the grid: the forms without block steps run another kernel above 2^18
elements, and both entry points have to choose alike.  And the capacity at the
edge: what is accepted does not move with the size of internal records.
Runs with the no-alloc tests at the end (one static array per GPU)."""
import ctypes

import numpy as np
import pytest
import torch

import workloads as W
from paper_2410_14917_amd import _lib

pytestmark = pytest.mark.gpu


def _call(fn, h, pr, m_max, out):
    op = pr.op
    kop = _lib.KpOp(op.kind, op.nx, op.ny, 0, op.dx, op.dy, op.nu, op.nu2, op.ax, op.ay,
                    op.react, op.brus_a, op.brus_b, None, None)
    B = torch.as_tensor(np.ascontiguousarray(pr.B[:, :pr.p + 1].T), device="cuda")
    info = _lib.KpInfo()
    rc = fn(h, ctypes.byref(kop), ctypes.c_void_p(B.data_ptr()), pr.p, op.n, pr.h, 1e-8, m_max,
            ctypes.c_void_p(out.data_ptr()), ctypes.byref(info))
    torch.cuda.synchronize()
    return rc, info.as_dict()


def _both(nx, ny, p, m, **cfg):
    lib = _lib.load()
    c = _lib.KpConfig(stream=ctypes.c_void_p(torch.cuda.current_stream().cuda_stream),
                      fixed_m=m, fixed_substeps=1, **cfg)
    h = ctypes.c_void_p()
    assert lib.kp_create(ctypes.byref(h), ctypes.byref(c)) == 0
    try:
        pr = W.random_problem(211, kind=W.OP_ADR, nx=nx, ny=ny, p=p, h=0.02, nu=0.02 / nx)
        outs, res = [], []
        for fn in (lib.kp_phi_combo, lib.kp_phi_combo_noalloc):
            y = torch.full((pr.op.n,), float("nan"), dtype=torch.float64, device="cuda")
            res.append(_call(fn, h, pr, m, y))
            outs.append(y)
        return outs, res
    finally:
        lib.kp_destroy(h)


@pytest.mark.parametrize("nx,ny", [(512, 512), (600, 500)])
@pytest.mark.parametrize("cfg", [{"orth": _lib.KP_ORTH_H_CWY}, {"orth": _lib.KP_ORTH_H_NCWY},
                                 {"fallback_delta": 1e-3}, {}],
                         ids=["h-cwy", "h-ncwy", "h-gsmgs-delta", "h-gsmgs"])
def test_noalloc_runs_the_kernel_of_the_allocating_call(nx, ny, cfg):
    print(f"noalloc: {nx}x{ny} {cfg}", flush=True)
    (ya, yb), ((ra, ia), (rb, ib)) = _both(nx, ny, 1, 20, **cfg)
    assert ra == 0 and rb == 0 and ia["status"] == 0
    assert ib == ia and torch.equal(ya, yb)


def test_noalloc_capacity_at_its_edge():
    """413 x 737 with m_max = 24 takes KP_NOALLOC_BYTES - 768 as the header
    counts it; 413 x 739 takes more than all."""
    (ya, yb), ((ra, ia), (rb, ib)) = _both(413, 737, 1, 24)
    assert ra == 0 and rb == 0 and ib == ia and torch.equal(ya, yb)
    _, ((ra, _), (rb, _)) = _both(413, 739, 1, 24)
    assert ra == 0 and rb == _lib.KP_ETOOLARGE
