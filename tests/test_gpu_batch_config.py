"""The batched call's kept workspace across configurations: kp_set_config
between two batched calls of the same shapes changes what the workspace has to
hold (block steps take a second buffer of halo rows; a fallback threshold above
1e-4 switches them off)."""
import ctypes

import numpy as np
import pytest
import torch

import workloads as W
import paper_2410_14917_amd as kp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("first,second", [(1e-3, 0.0), (0.0, 1e-3)])
def test_batched_call_after_a_configuration_change(first, second):
    """The second call gives the bits of a fresh context."""
    print(f"batch config: fallback_delta {first} then {second}", flush=True)
    grids = [(W.OP_ADR, 96, 40), (W.OP_ALLEN_CAHN, 61, 37), (W.OP_BRUSSELATOR, 40, 33)]
    probs = [W.random_problem(900 + i, kind=k, nx=nx, ny=ny, p=2, h=0.02, nu=0.01)
             for i, (k, nx, ny) in enumerate(grids)]
    ops = [kp.Operator.from_host(q.op) for q in probs]
    Bs = [torch.as_tensor(np.ascontiguousarray(q.B[:, :3].T), device="cuda") for q in probs]
    hs = [q.h for q in probs]

    def call(ctx):
        return [y.clone() for y in ctx.phi_combo_batched(ops, Bs, hs, tol=1e-8, m_max=32)]

    with kp.Context(fallback_delta=first) as ctx:
        call(ctx)
        torch.cuda.synchronize()
        ctx.cfg.fallback_delta = second
        assert ctx.lib.kp_set_config(ctx.h, ctypes.byref(ctx.cfg)) == 0
        got = call(ctx)
    with kp.Context(fallback_delta=second) as ctx:
        want = call(ctx)
    for y, y1 in zip(got, want):
        assert torch.equal(y, y1)
