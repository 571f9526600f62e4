"""Block steps (up to three Arnoldi steps per reduction, float64 H-GSMGS) on the
partitions where their kernels can go wrong: one and two element pairs per
thread at the edges of their tiles, one and two tiles on chip, the leader's own
gather (up to 16 partial rows) and the two-hop one, the block's vectors on chip
or in memory, halo rows in LDS or not, two planes, Krylov dimensions of every
remainder modulo three, and the points where a block has to stop early.

Tolerances: the block's Hessenberg matrix has the single steps' error to a small
factor (its later vectors cost one more cancellation each, 12 at most on a
diffusion operator), so the Arnoldi bounds of the single steps hold: 1e-12 for
H and for the loss of orthogonality at m <= 30, 1e-10 for results."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import arnoldi, krylov, phi
import paper_2410_14917_amd as kp

pytestmark = pytest.mark.gpu


def rel(a, b):
    return np.linalg.norm(np.asarray(a) - np.asarray(b)) / np.linalg.norm(b)


# (kind, nx, ny, p, rows per workgroup: 0 automatic)
GRIDS = [
    (W.OP_ADR, 64, 34, 3, 2),           # 17 workgroups: two-hop gather, 128 elements each
    (W.OP_ADR, 64, 34, 3, 3),           # 12: the leader's gather, a ragged last one
    (W.OP_ADR, 64, 32, 2, 2),           # 16, the most it takes
    (W.OP_ALLEN_CAHN, 1024, 20, 1, 1),  # 1024 elements: the largest one-pair tile
    (W.OP_ALLEN_CAHN, 1026, 20, 1, 1),  # 1026: the smallest two-pair tile
    (W.OP_ADR, 512, 40, 2, 4),          # 2048: one full two-pair tile
    (W.OP_ADR, 514, 40, 2, 4),          # 2056: the second tile's first pairs
    (W.OP_ADR, 512, 40, 2, 8),          # 4096: the largest region on chip
    (W.OP_ADR, 512, 40, 2, 9),          # 4608: two tiles, nothing on chip
    (W.OP_ADR, 333, 36, 2, 4),          # odd rows: padding element, pair alignment
    (W.OP_ADR, 2050, 18, 2, 1),         # rows too wide for the on-chip path
    (W.OP_ADR, 4100, 18, 1, 1),         # rows too wide for the LDS halo copy
    (W.OP_BRUSSELATOR, 130, 36, 2, 2),  # two planes, one-pair tiles, 18 workgroups
    (W.OP_BRUSSELATOR, 2049, 6, 1, 2),  # two planes, wide odd rows, halo rows from memory
    (W.OP_ADR, 7, 3, 8, 0),             # one workgroup, every tail entry
    (W.OP_ADR, 256, 34, 2, 2),          # the widest rows of the tagged exchange
    (W.OP_ADR, 258, 34, 2, 2),          # one pair wider: flags
    (W.OP_ALLEN_CAHN, 97, 2, 1, 1),     # one row per workgroup is both halo rows
    (W.OP_ADR, 63, 2, 8, 2),            # one workgroup, its own neighbour
]


@pytest.mark.parametrize("grid", GRIDS, ids=lambda g: f"{g[0]}-{g[1]}x{g[2]}-r{g[4]}")
@pytest.mark.parametrize("m", [14, 15, 16])
def test_block_steps_match_single_reduction_oracle(grid, m):
    kind, nx, ny, p, rows = grid
    print(f"block: kind={kind} {nx}x{ny} p={p} rows={rows} m={m}", flush=True)
    pr = W.random_problem(41 + nx, kind=kind, nx=nx, ny=ny, p=p, h=0.02, with_diag=True,
                          nu=0.02 / max(nx, ny), react=0.1)
    op = kp.Operator.from_host(pr.op)
    B = torch.as_tensor(np.ascontiguousarray(pr.B[:, :p + 1].T), device="cuda")
    with kp.Context(rows_per_wg=rows) as ctx:
        ctx.arnoldi_begin(op, B, m)
        ctx.arnoldi_step(m)
        r = ctx.arnoldi_read()
    mu = krylov.balance_scale(pr.B, p)
    mgs = arnoldi.MGSArnoldi(lambda x: krylov.aug_apply(pr.op, pr.B, p, mu, x),
                             krylov.start_vector(pr.B, p, mu), m)
    mgs.extend(m)
    assert r["j"] == m and not r["breakdown"] and r["n_fallback"] == 0
    assert rel(r["H"][:m + 1, :m], mgs.H[:m + 1, :m]) <= 1e-12
    assert np.linalg.norm(np.eye(m + 1) - r["V"].T @ r["V"], 2) <= 1e-12
    with kp.Context(rows_per_wg=rows, fixed_m=m, fixed_substeps=2) as ctx:
        y, info = ctx.phi_combo(op, B, pr.h, m_max=m, info=True)
        y2 = ctx.phi_combo(op, B, pr.h, m_max=m)
    ref, _ = krylov.phi_combo(pr.op, pr.B, pr.h, p, fixed_m=m, fixed_substeps=2, m_max=m)
    assert info["status"] == 0 and info["arnoldi_steps"] == 2 * m
    assert rel(y.cpu().numpy(), ref) <= 1e-10
    assert torch.equal(y, y2)


@pytest.mark.parametrize("m", [1, 2, 3, 4, 5])
def test_block_steps_of_the_shortest_processes(m):
    pr = W.random_problem(43, nx=40, ny=36, p=1, h=1e-3, nu=1e-3)
    op = kp.Operator.from_host(pr.op)
    B = torch.as_tensor(np.ascontiguousarray(pr.B.T), device="cuda")
    with kp.Context(fixed_m=m, fixed_substeps=3) as ctx:
        y, info = ctx.phi_combo(op, B, pr.h, m_max=m, info=True)
    ref, _ = krylov.phi_combo(pr.op, pr.B, pr.h, 1, fixed_m=m, fixed_substeps=3, m_max=m)
    assert info["arnoldi_steps"] == 3 * m and rel(y.cpu().numpy(), ref) <= 1e-10


@pytest.mark.parametrize("nval", [1, 2, 3, 4, 5, 6])
@pytest.mark.parametrize("p", [0, 1])
def test_block_stops_at_an_invariant_subspace(nval, p):
    """A diagonal operator with nval values: the process ends at nval + p
    columns, in the first or in a later vector of a block."""
    d = np.linspace(-3.0, 1.0, nval)
    nx, ny = 70, 40
    diag = d[np.random.default_rng(5).integers(0, nval, nx * ny)]
    op_h = W.Operator(kind=W.OP_ADR, nx=nx, ny=ny, field0=diag)
    Bh = np.random.default_rng(6).standard_normal((op_h.n, p + 1))
    op = kp.Operator.from_host(op_h)
    B = torch.as_tensor(np.ascontiguousarray(Bh.T), device="cuda")
    with kp.Context() as ctx:
        y, info = ctx.phi_combo(op, B, 0.3, tol=1e-10, m_max=20, info=True)
    assert info["status"] == 0 and info["breakdowns"] >= 1 and info["m_last"] == nval + p
    assert rel(y.cpu().numpy(), phi.phi_combo_diag(diag, Bh, 0.3, p)) <= 1e-12


def test_nearly_scalar_operator_takes_single_steps():
    """A = -50 I + (small): every vector lies almost in the span of the ones
    before, the guard keeps single steps, with the oracle's result."""
    rng = np.random.default_rng(8)
    op_h = W.Operator(kind=W.OP_ADR, nx=60, ny=50, nu=1e-6, react=-50.0,
                      field0=0.1 * rng.standard_normal(3000))
    Bh = rng.standard_normal((op_h.n, 3))
    op = kp.Operator.from_host(op_h)
    B = torch.as_tensor(np.ascontiguousarray(Bh.T), device="cuda")
    with kp.Context(fixed_m=9, fixed_substeps=2) as ctx:
        y, info = ctx.phi_combo(op, B, 0.05, m_max=9, info=True)
    ref, _ = krylov.phi_combo(op_h, Bh, 0.05, 2, fixed_m=9, fixed_substeps=2, m_max=9)
    assert info["status"] == 0 and info["arnoldi_steps"] == 18
    assert rel(y.cpu().numpy(), ref) <= 1e-10


# (kind, nx, ny, p, rows per workgroup: 0 automatic)
IOCGS_GRIDS = [
    (W.OP_ADR, 512, 40, 2, 8),          # 4096 elements: the largest tile on chip
    (W.OP_ALLEN_CAHN, 2048, 18, 1, 2),  # the widest rows on chip
    (W.OP_ADR, 2050, 18, 2, 1),         # wider: through memory
    (W.OP_ADR, 1025, 20, 1, 4),         # 4100 elements: through memory
    (W.OP_ADR, 333, 36, 3, 4),          # odd rows: padding element
    (W.OP_ADR, 333, 35, 3, 2),          # odd size: the last workgroup's padding element
    (W.OP_ALLEN_CAHN, 98, 2, 1, 1),     # one row per workgroup is both halo rows
    (W.OP_ADR, 7, 3, 8, 0),             # one workgroup, every tail entry
    (W.OP_ADR, 63, 61, 0, 0),           # spread, no augmentation
]


@pytest.mark.parametrize("grid", IOCGS_GRIDS, ids=lambda g: f"{g[0]}-{g[1]}x{g[2]}-r{g[4]}")
def test_iocgs_on_chip_matches_oracle(grid):
    """ioCGS with its window on chip at the edges of that path, paused and
    resumed (the resumed launch reloads), and over two substeps; the bounds are
    those of the orthogonalization tests."""
    kind, nx, ny, p, rows = grid
    m = 15
    print(f"iocgs: kind={kind} {nx}x{ny} p={p} rows={rows}", flush=True)
    pr = W.random_problem(51 + nx, kind=kind, nx=nx, ny=ny, p=p, h=0.02, with_diag=True,
                          nu=0.02 / max(nx, ny), react=0.1)
    op = kp.Operator.from_host(pr.op)
    B = torch.as_tensor(np.ascontiguousarray(pr.B[:, :p + 1].T), device="cuda")
    with kp.Context(orth="iocgs", rows_per_wg=rows) as ctx:
        ctx.arnoldi_begin(op, B, m)
        ctx.arnoldi_step(4)
        ctx.arnoldi_step(m - 4)
        r = ctx.arnoldi_read()
    mu = krylov.balance_scale(pr.B, p)
    iop = arnoldi.IOPArnoldi(lambda x: krylov.aug_apply(pr.op, pr.B, p, mu, x),
                             krylov.start_vector(pr.B, p, mu), m, window=2)
    iop.extend(m)
    assert r["j"] == m and not r["breakdown"]
    assert rel(r["H"][:m + 1, :m], iop.H[:m + 1, :m]) <= 1e-11
    assert rel(r["V"], iop.V[:, :m + 1]) <= 1e-10
    with kp.Context(orth="iocgs", rows_per_wg=rows, fixed_m=m, fixed_substeps=2) as ctx:
        y, info = ctx.phi_combo(op, B, pr.h, m_max=m, info=True)
        y2 = ctx.phi_combo(op, B, pr.h, m_max=m)
    ref, _ = krylov.phi_combo(pr.op, pr.B, pr.h, p, fixed_m=m, fixed_substeps=2, m_max=m, orth="iop")
    assert info["status"] == 0 and info["arnoldi_steps"] == 2 * m
    assert rel(y.cpu().numpy(), ref) <= 1e-10
    assert torch.equal(y, y2)


@pytest.mark.parametrize("nx,ny", [(512, 512), (512, 513), (513, 514)])
@pytest.mark.parametrize("orth", ["h-cwy", "h-ncwy"])
def test_single_steps_on_both_sides_of_the_kernel_choice(nx, ny, orth):
    """The forms without block steps: the largest grid of the block kernel, and
    the next ones, against the oracle's modified Gram-Schmidt."""
    print(f"singles: {orth} {nx}x{ny}", flush=True)
    m = 7
    pr = W.random_problem(61, kind=W.OP_ADR, nx=nx, ny=ny, p=1, h=0.02, nu=0.02 / nx, with_diag=True)
    op = kp.Operator.from_host(pr.op)
    B = torch.as_tensor(np.ascontiguousarray(pr.B[:, :2].T), device="cuda")
    with kp.Context(orth=orth, fixed_m=m, fixed_substeps=1) as ctx:
        y, info = ctx.phi_combo(op, B, pr.h, m_max=m, info=True)
    ref, _ = krylov.phi_combo(pr.op, pr.B, pr.h, 1, fixed_m=m, fixed_substeps=1, m_max=m)
    assert info["status"] == 0 and info["arnoldi_steps"] == m
    assert rel(y.cpu().numpy(), ref) <= 1e-10
