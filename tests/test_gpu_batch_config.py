"""The batched call's kept workspace across configurations: kp_set_config
between two batched calls of the same shapes changes what the workspace has to
hold (block steps take a second buffer of halo rows; a fallback threshold above
1e-4 switches them off)."""
import ctypes

import numpy as np
import pytest
import torch

import workloads as W
from oracle import krylov
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


@pytest.mark.parametrize("grids", [
    [(W.OP_ADR, 7, 3), (W.OP_ADR, 45, 33), (W.OP_ALLEN_CAHN, 301, 210), (W.OP_BRUSSELATOR, 64, 41),
     (W.OP_ADR, 600, 450)],
    [(W.OP_BRUSSELATOR, 64, 41), (W.OP_BRUSSELATOR, 33, 150)]], ids=["mixed", "two-plane"])
@pytest.mark.parametrize("cfg,tform", [({"orth": "h-cwy"}, "cwy"), ({"orth": "h-ncwy"}, "ncwy"),
                                       ({"fallback_delta": 1e-3}, "gsmgs"), ({}, "gsmgs")],
                         ids=["h-cwy", "h-ncwy", "h-gsmgs-delta", "h-gsmgs"])
def test_batched_forms_with_and_without_block_steps(cfg, tform, grids):
    """Single steps (k_run's phases, or the block kernel's where every problem has
    two planes) and block steps: one workgroup, teams, odd rows, two species;
    against the oracle, and the same bits from a graph replay."""
    print(f"batch forms: {cfg}", flush=True)
    probs = [W.random_problem(920 + i, kind=k, nx=nx, ny=ny, p=2, h=0.02, nu=0.02 / nx)
             for i, (k, nx, ny) in enumerate(grids)]
    ops = [kp.Operator.from_host(q.op) for q in probs]
    Bs = [torch.as_tensor(np.ascontiguousarray(q.B[:, :3].T), device="cuda") for q in probs]
    m = 13
    with kp.Context(fixed_m=m, fixed_substeps=2, **cfg) as ctx:
        ys, infos = ctx.phi_combo_batched(ops, Bs, [q.h for q in probs], m_max=m, info=True)
        ys = [y.clone() for y in ys]
        again = ctx.phi_combo_batched(ops, Bs, [q.h for q in probs], m_max=m)
    delta = cfg.get("fallback_delta", 1e-10)
    for q, y, y2, inf in zip(probs, ys, again, infos):
        ref, rinfo = krylov.phi_combo(q.op, q.B, q.h, 2, fixed_m=m, fixed_substeps=2, m_max=m,
                                      orth="hybrid", tform=tform, delta=delta)
        assert inf["status"] == 0 and inf["arnoldi_steps"] == rinfo.arnoldi_steps
        assert np.linalg.norm(y.cpu().numpy() - ref) <= 1e-10 * np.linalg.norm(ref)
        assert torch.equal(y, y2)


def test_calibration_is_a_fit_of_the_present_kernels(tmp_path, monkeypatch):
    """The model is fitted (none of the built-in constants comes back), and a
    cached fit of the kernels before block steps is not taken."""
    dev = torch.cuda.get_device_properties(0)
    cache = tmp_path / "autotune.txt"
    old = f"{dev.gcnArchName}/cu{dev.multi_processor_count}/lib{kp._lib.load().kp_version()}"
    cache.write_text(f"{old} 1.9e10 1e-7 0 7e-6 9e-5\n")
    monkeypatch.setenv("KP_AUTOTUNE_CACHE", str(cache))
    with kp.Context() as ctx:
        src, md = ctx.calibrate()
    print(src, md, flush=True)
    assert src == "measured" and len(cache.read_text().splitlines()) == 2
    assert abs(md["bw_wg_Bps"] / (19.5e9 / 0.45) - 1) > 1e-9
    assert abs(md["t_expm64_s"] / (0.45 * 2.6e-4) - 1) > 1e-9
    assert md["t_step_s"] >= 1e-7 and md["t_team_s"] >= 0.0 and md["t_log_s"] >= 0.0
    # (streaming: 256 workgroups at 10 to 200 GB/s of two-pass bytes each)
    assert 1e10 < md["bw_wg_Bps"] < 2e11
