"""The time-blocked D2Q9 kernels at the sizes where their tiling changes:
steps per launch and region by lattice size, tiles cut by the lattice's edge,
periodic axes shorter than a region, step counts that are no multiple of a
launch, taped segments, loss frames and recompute.  Against the FP64 oracle
from a random equilibrium state (velocity relative L2 <= 1e-5, loss 1e-4,
gradients 1e-3: a dozen FP32 steps), and bit for bit between groupings of the
same steps."""
import numpy as np
import pytest

import oracle as O
from paper_2310_00810_amd import geometry as G
from tests.test_gpu_lbm import _inlet, rel_l2, solver_for

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

P, W, X, A, V = O.BC_PRESSURE, O.BC_WALL, O.BC_PERIODIC, O.BC_ABB, O.BC_VELOCITY


def _lattice(nx, ny, bcx, bcy, mrt=None):
    rng = np.random.default_rng(nx * 1000 + ny)
    solid = (rng.random((1, ny, nx)) < 0.25).astype(np.uint8) if min(nx, ny) < 20 else \
        G.boolean_disks(nx, ny, (2.0, 5.0), 0.75, seed=nx + ny)[None]
    solid[:, :, :2] = solid[:, :, -2:] = 0
    return O.Lattice(9, nx, ny, 1, (bcx, bcy, O.BC_PERIODIC), solid, mrt=mrt)


def _start(lat, seed):
    rng = np.random.default_rng(seed)
    drho = (0.01 * rng.standard_normal(lat.shape)).astype(np.float32)
    u = (0.01 * rng.standard_normal(lat.shape + (3,))).astype(np.float32)
    u[..., 2] = 0
    return drho * lat.fluid(), u * lat.fluid()[..., None]


def _init(s, drho, u):
    s.set_initial(torch.from_numpy(np.ascontiguousarray(drho)).reshape(-1).cuda(),
                  torch.from_numpy(np.ascontiguousarray(u[..., :2])).reshape(-1, 2).cuda())


CASES = [
    (9, 5, P, W, 1, None),             # smaller than a region, one step
    (18, 2, P, X, 9, None),            # one tile exactly, periodic rows wrap several times in a region
    (19, 3, X, X, 8, None),            # one node over in both axes, periodic both
    (37, 23, W, W, 15, None),
    (150, 91, A, W, 13, None),         # 6 steps per launch
    (233, 160, V, X, 12, O.MRT_RATES),  # 5
    (401, 301, P, W, 11, None),        # 4
    (655, 317, P, W, 11, None),        # the large region, 3 adjoint steps
    (1027, 401, V, X, 8, O.MRT_RATES),  # single-step adjoint
]


@pytest.mark.parametrize("nx,ny,bcx,bcy,T,mrt", CASES)
def test_block_steps_and_gradients_match_oracle(nx, ny, bcx, bcy, T, mrt):
    lat = _lattice(nx, ny, bcx, bcy, mrt)
    drho, u = _start(lat, 3)
    rng = np.random.default_rng(4)
    tgt = (1e-2 * rng.standard_normal(lat.shape + (3,))).astype(np.float32)
    tgt[..., 2] = 0
    frames = 2 if T > 9 and lat.nx < 500 else 1
    if frames > 1:
        tgt = np.stack([tgt, 0.5 * tgt])
    tau, d = 0.8, float(np.float32(0.05 if bcx == V else 0.004))
    s = solver_for(lat, T, tape=True, K=5, target=tgt, frames=frames, stride=3)
    _init(s, drho, u)
    loss = s.forward(tau, d, 0.0, record_tape=True)
    _, ug = s.macro()
    s.adjoint()
    g = s.grad()
    f0 = O.init_eq(lat, 1.0 + drho.astype(np.float64), u.astype(np.float64))
    # the kernels start from a post-collision state; an equilibrium is both
    ref = O.grad(lat, tau, _inlet(lat, d), 1.0, f0, T, tgt.astype(np.float64), K=5, frames=frames, stride=3)
    _, uo = O.macro(lat, O.run(lat, tau, _inlet(lat, d), 1.0, f0, T))
    fl = lat.fluid()
    assert rel_l2(ug.cpu().numpy().reshape(lat.shape + (2,))[fl], uo[..., :2][fl]) <= 1e-5
    assert abs(loss[0] - ref["loss"]) <= 1e-4 * ref["loss"]
    scale = abs(ref["dtau"]) + abs(ref["drho_in"].sum()) + abs(ref["drho_out"].sum())
    for got, want in ((g["dtau"][0], ref["dtau"]), (g["drho_in"][0], ref["drho_in"].sum()),
                      (g["drho_out"][0], ref["drho_out"].sum())):
        assert abs(got - want) <= 1e-3 * max(abs(want), 0.1 * scale)


@pytest.mark.parametrize("nx,ny", [(18, 2), (150, 91), (401, 301), (655, 317)])
def test_block_grouping_is_bitwise(nx, ny):
    """Checkpoints, kept segments and the untaped forward group the same steps
    differently into launches; states and gradients stay the same bits."""
    lat = _lattice(nx, ny, P, W)
    drho, u = _start(lat, 5)
    T, out = 17, []
    for K, R in ((17, 1), (1, 1), (4, 1), (6, 2), (9, 2)):
        s = solver_for(lat, T, tape=True, K=K, resident=R, target=np.zeros(lat.shape + (3,), np.float32))
        _init(s, drho, u)
        loss = s.forward(0.7, 0.003, 0.0, record_tape=True)
        s.adjoint()
        g = s.grad()
        adj = s.get_populations("adjoint").cpu().numpy()
        s.forward(0.7, 0.003, 0.0, want_loss=False)
        out.append((loss, g["dtau"], g["drho_in"], g["drho_out"], adj, s.get_populations().cpu().numpy()))
    for o in out[1:]:
        for a, b in zip(o, out[0]):
            assert np.array_equal(a, b)


def test_block_residual_steps_match_single_forward():
    """run_to_residual groups its steps with the check interval: the same
    state as a forward pass of as many steps."""
    lat = _lattice(150, 91, P, W)
    s = solver_for(lat, 36)
    s.forward(0.8, 0.004, 0.0, want_loss=False)
    ref, um = s.get_populations(), s.macro(mean2=True)[1]
    for check in (4, 6, 12, 18, 36):
        s.set_initial(None, None)
        n, _ = s.run_to_residual(0.8, 0.004, 0.0, tol=1e-12, max_steps=36, check_every=check)
        assert n == 36
        assert torch.equal(s.get_populations(), ref) and torch.equal(s.macro(mean2=True)[1], um)


def _solver(lattice, insts, bc, T, **kw):
    from paper_2310_00810_amd.lbm import Solver
    return Solver(lattice, insts, bc=bc, steps=T, tape=True, **kw)


def _gradient(s, drho, u, tau, din):
    s.set_initial(torch.from_numpy(drho).cuda().reshape(-1), torch.from_numpy(u).cuda().reshape(-1, s.D))
    loss = s.forward(tau, din, 0.0, record_tape=True)
    s.adjoint()
    g = s.grad()
    return loss, g["drho_in"], g["dtau"], g["drho_out"], s.get_populations("adjoint").cpu().numpy()


def _batch_equals_single(lattice, nxyz, n, bc, T, frames, collision, spread=0.1):
    """The gradients of a batch against those of its first and last instance alone, bit for bit."""
    from paper_2310_00810_amd.lbm import Instance
    nx, ny, nz = nxyz
    D, sh = (2 if lattice == 9 else 3), (nz, ny, nx)
    rng = np.random.default_rng(17)
    solid = (rng.random((n,) + sh) < 0.1).astype(np.uint8)
    solid[..., 0] = solid[..., -1] = 0
    drho = (0.01 * rng.standard_normal((n,) + sh, dtype=np.float32)).astype(np.float32)
    u = (0.02 * rng.standard_normal((n,) + sh + (D,), dtype=np.float32)).astype(np.float32)
    tgt = (0.02 * rng.standard_normal((n, frames) + sh + (D,), dtype=np.float32)).astype(np.float32)
    insts = [Instance(nx, ny, nz, solid=solid[b], target_u=tgt[b]) for b in range(n)]
    tau = 0.7 + 0.02 * np.arange(n)
    din = (0.05 if bc[0] == "velocity" else 0.006) * (1 + spread * np.arange(n))
    kw = dict(ckpt_interval=5, collision=collision, loss_frames=frames, loss_stride=2)
    all_ = _gradient(_solver(lattice, insts, bc, T, **kw), drho, u, tau, din)
    k = lattice * nx * ny * nz
    for b in (0, n - 1):
        one = _gradient(_solver(lattice, [insts[b]], bc, T, **kw), drho[b], u[b], tau[b], din[b])
        for x, y in zip(all_[:4], one[:4]):
            assert np.array_equal(x[b:b + 1], y)
        assert np.array_equal(all_[4][b * k:(b + 1) * k], one[4])


@pytest.mark.parametrize("collision", ["bgk", "mrt"])
@pytest.mark.parametrize("frames", [1, 3])
@pytest.mark.parametrize("bcx", ["pressure", "abb", "velocity", "wall", "periodic"])
def test_single_step_and_blocked_adjoint_are_the_same_bits(bcx, frames, collision):
    """462 000 nodes take single adjoint steps, one instance of them the time-blocked ones."""
    _batch_equals_single(9, (300, 220, 1), 7, (bcx, "wall", "periodic"), 13, frames, collision)


@pytest.mark.parametrize("frames", [1, 2])
@pytest.mark.parametrize("bcx", ["pressure", "abb", "velocity"])
def test_d3q19_states_beyond_the_cache_are_the_same_bits(bcx, frames):
    """Two states of 2.1 M nodes exceed the Infinity Cache (streaming kernels), those of one instance do not."""
    _batch_equals_single(19, (96, 64, 68), 5, (bcx, "wall", "periodic"), 5, frames, "bgk")


@pytest.mark.parametrize("bcx,bcy,collision", [("pressure", "wall", "bgk"), ("abb", "periodic", "mrt"),
                                               ("velocity", "wall", "mrt"), ("periodic", "periodic", "bgk")])
def test_thin_lattices_step_singly_with_the_same_bits(bcx, bcy, collision):
    """60 lattices of 3 x 700 take single steps (a tile would own 24 nodes), one of them time-blocked ones."""
    _batch_equals_single(9, (3, 700, 1), 60, (bcx, bcy, "periodic"), 13, 3, collision, spread=0.005)
