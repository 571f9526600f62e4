"""kp_phi_combo under stream capture with a workspace from an earlier, larger
call: the finer partitions of the float64 forms must not need more workspace
for a smaller grid (growing it is refused under capture, and frees what the
graphs of earlier calls use)."""
import numpy as np
import pytest
import torch

import paper_2410_14917_amd as kp

pytestmark = pytest.mark.gpu


def _problem(nx, ny, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    op = kp.Operator(kp.KP_OP_ADR, nx, ny, nu=1e-4, ax=1.0, ay=0.5)
    return op, torch.randn(3, nx * ny, generator=g, device="cuda", dtype=torch.float64)


# (form, grid of the first call, grids captured after it)
CASES = [
    ("h-gsmgs", (300, 300), [(256, 256), (64, 64), (97, 61)]),   # tagged exchange after flags
    ("h-gsmgs", (1024, 600), [(512, 512), (1000, 30)]),
    ("h-cwy", (600, 600), [(512, 512), (256, 256)]),             # k_run first, then the block kernel
    ("iocgs", (700, 700), [(300, 300), (64, 2000)]),
    ("mgs", (200, 200), [(64, 64)]),
]


@pytest.mark.parametrize("orth,first,then", CASES, ids=lambda c: str(c).replace(" ", ""))
def test_smaller_calls_are_captured_in_the_workspace_of_a_larger_one(orth, first, then):
    m, h = 12, 0.01
    s = torch.cuda.Stream()
    with torch.cuda.stream(s), kp.Context(orth=orth, fixed_m=m, fixed_substeps=1) as ctx:
        op, B = _problem(*first, 1)
        y0 = ctx.phi_combo(op, B, h, m_max=m)
        s.synchronize()
        graphs = []
        for i, (nx, ny) in enumerate(then):
            print(f"capture: {orth} {nx}x{ny} after {first}", flush=True)
            o, b = _problem(nx, ny, 2 + i)
            y = torch.empty(nx * ny, device="cuda", dtype=torch.float64)
            s.synchronize()
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g, stream=s):
                ctx.phi_combo(o, b, h, m_max=m, out=y)
            graphs.append((g, o, b, y))
        eager = [ctx.phi_combo(o, b, h, m_max=m) for _, o, b, _ in graphs]
        s.synchronize()
        for rep in range(3):
            for (g, _, _, y), e in zip(graphs, eager):
                y.zero_()
                g.replay()
                s.synchronize()
                assert torch.equal(y, e), f"replay {rep}"
            # eager work between the replays, the first grid again among it
            assert torch.equal(ctx.phi_combo(op, B, h, m_max=m), y0)
            float(torch.randn(1 << 16, device="cuda").sum())
    assert np.isfinite(y0.cpu().numpy()).all()
