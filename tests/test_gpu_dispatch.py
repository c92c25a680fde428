"""Parity with the oracle at the edges of the kernels' dispatch rules: every axis length's own transform
kernels, and tiles holding more particles than one dealing chunk."""

import numpy as np
import pytest

from gpu_common import EPS, banner, max_rel, np64, oracle_species, periodic_pos_err, put, rounded

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import centering as ocent  # noqa: E402
from oracle import particles as opart  # noqa: E402
from oracle import step as ostep  # noqa: E402
from paper_2106_12919_amd import autograd as pag  # noqa: E402
from paper_2106_12919_amd import inputs  # noqa: E402
from paper_2106_12919_amd import lib as piclib  # noqa: E402

LENGTHS = sorted(2 ** a * 3 ** b for a in range(1, 11) for b in range(7) if 8 <= 2 ** a * 3 ** b <= 1024)


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("axis", [0, 1, 2])
def test_field_solve_at_every_axis_length(dtype, axis):
    """Each accepted length on x, y and z (the z transform takes other stages than the strided ones)."""
    for n in LENGTHS:
        shape = tuple(n if a == axis else (8, 18, 12)[a] for a in range(3))
        banner(f"psatd_push_fields dtype={dtype} shape={shape}")
        p = ostep.Params(shape, (1.0, 1.0, 1.0), 0.5, 1, 8, 16)
        ctx = piclib.Context(shape, (1.0, 1.0, 1.0), 0.5, 1, 8, 16, dtype)
        f = piclib.Fields(shape, dtype)
        src = rounded(inputs.random_grid(shape, seed=n, count=11), dtype)
        put(f.E_stag, src[0:3])
        put(f.B_stag, src[3:6])
        put(f.J_stag, src[6:9])
        put([f.rho_old, f.rho_new], src[9:11])
        piclib.psatd_push_fields(ctx.ctx, f)
        piclib.pic_sync(ctx.ctx)
        E, B = ostep.push_fields(src[0:3], src[3:6], src[6:9], src[9], src[10], p)
        # log2(N) eps per transform (Higham), two transforms around the 11-term update, margin 10
        tol = 10 * 2 * np.log2(np.prod(shape)) * EPS[dtype] * 3
        for d in range(3):
            assert max_rel(np64(f.E_stag[d]), E[d]) <= tol, (shape, "E", d)
            assert max_rel(np64(f.B_stag[d]), B[d]) <= tol, (shape, "B", d)
        ctx.close()


def steps_against_oracle(shape, ppc, order, center, dtype, nsteps, flags=0, seed=31):
    """One call of ``nsteps`` cycles against as many oracle steps: fields, sources and every particle."""
    wl = inputs.small(shape, ppc=ppc, shape_order=order, center_order=center, dtype=dtype, u_th=0.2,
                      field_amp=0.02, seed=seed)
    base = 2.0 ** np.floor(np.log2(wl.electrons.w[0]))
    wl.electrons.w = base * (1.0 + np.arange(wl.electrons.n) * 2.0 ** -23)  # identities, exact in FP32
    ctx = piclib.Context.for_workload(wl, flags=flags)
    f = ctx.fields_from_workload(wl)
    el = piclib.Species.from_host(wl.electrons, shape, dtype)
    ions = piclib.Species.from_host(wl.ions, shape, dtype)
    ctx.init_charge(f, el, ions)
    p = ostep.Params(shape, wl.spacing, wl.dt, order, center, wl.psatd_order)
    osp = oracle_species(el, shape, wl.spacing)
    rho_static = ostep.deposit_rho([oracle_species(ions, shape, wl.spacing)], p)
    state = {"E_stag": rounded(wl.E, dtype), "B_stag": rounded(wl.B, dtype),
             "rho_old": ostep.deposit_rho([osp], p, rho_static)}
    piclib.pic_step(ctx.ctx, f, [el], nsteps)
    piclib.pic_sync(ctx.ctx)
    for n in range(nsteps):
        if n == nsteps - 1:
            E_nod, B_nod = ostep.center_fields_s2n(state["E_stag"], state["B_stag"], p)
        out = ostep.step(state, [osp], p, rho_static)
    J_stag = ostep.center_current_n2s(out["J_nod"], p)
    tol = 1e-10 if dtype == "f64" else 2e-4  # the tolerances of the other several-step parity tests
    for d in range(3):
        for got, ref in ((f.E_stag, state["E_stag"]), (f.B_stag, state["B_stag"]), (f.E_nod, E_nod),
                         (f.B_nod, B_nod), (f.J_nod, out["J_nod"]), (f.J_stag, J_stag)):
            assert max_rel(np64(got[d]), ref[d]) <= tol, d
    assert max_rel(np64(f.rho_old), state["rho_old"]) <= tol
    gi, oi = np.argsort(np64(el.w)), np.argsort(osp["w"])
    tol_p = 1e-11 if dtype == "f64" else 4e-5
    assert periodic_pos_err(el.positions(shape, wl.spacing)[gi], osp["pos"][oi], p.lengths) <= tol_p
    assert np.max(np.abs(np.stack([np64(x) for x in el.u], axis=1)[gi] - osp["u"][oi])) <= tol_p
    ctx.close()


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("shape,ppc", [((16, 8, 16), 5), ((12, 18, 24), 3)])
def test_several_chunks_per_tile(dtype, shape, ppc):
    """Cubic tiles of more particles than one dealing chunk (1024 FP32, 512 FP64), whole and ragged tiles:
    the gather follows the order the deposition published, chunk by chunk."""
    banner(f"pic_step 4 steps, several chunks per tile dtype={dtype} shape={shape} ppc={ppc}")
    steps_against_oracle(shape, ppc, 3, 8, dtype, 4)


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("shape,ppc,order", [((12, 12, 12), 24, 1), ((18, 18, 18), 12, 3), ((12, 8, 18), 16, 3)])
def test_split_ragged_tiles(dtype, shape, ppc, order):
    """Tiles in several parts on grids with partial tiles, with tiles of fewer particles than one part among them."""
    banner(f"pic_step 3 steps, split ragged tiles dtype={dtype} shape={shape} ppc={ppc} order={order}")
    steps_against_oracle(shape, ppc, order, 8, dtype, 3)


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("shape", [(48, 48, 64), (16, 16, 16)])
def test_chunks_spread_over_heavy_tiles(dtype, shape):
    """pic_deposit of particles in cell order, cubic: tiles just below, at and above the size from which a chunk
    takes particles from all over its tile, as whole tiles and split in parts."""
    banner(f"pic_deposit heavy tiles dtype={dtype} shape={shape}")
    rng = np.random.default_rng(17)
    sizes = {(0, 0, 0): 16383, (1, 0, 1): 16384, (1, 1, 1): 20001, (0, 1, 1): 17 * 1024}
    cells = []
    for t, n in sizes.items():
        l = rng.integers(0, 8, (n, 3)) + 8 * np.array(t)
        cells.append((l[:, 0] * shape[1] + l[:, 1]) * shape[2] + l[:, 2])
    cell = np.sort(np.concatenate(cells)).astype(np.int32)
    n, td = cell.size, torch.float32 if dtype == "f32" else torch.float64
    dev = lambda a: torch.tensor(a, dtype=td, device="cuda")  # noqa: E731
    off = [dev(rng.random(n) * 0.999) for _ in range(3)]
    u = [dev(m + 0.1 * rng.standard_normal(n)) for m in (0.5, -0.4, 0.3)]
    sp = piclib.Species(torch.tensor(cell, device="cuda"), off, u, None, -1.0, 1.0, w_const=0.5)
    ctx = piclib.Context(shape, (1.0, 1.0, 1.0), 0.5, 3, 8, 16, dtype)
    f = piclib.Fields(shape, dtype)
    piclib.pic_deposit(ctx.ctx, [sp], f, piclib.PIC_DEP_RHO_AND_J)
    piclib.pic_sync(ctx.ctx)
    p = ostep.Params(shape, (1.0, 1.0, 1.0), 0.5, 3, 8, 16)
    ijk = np.stack(np.unravel_index(cell, shape), axis=1)
    pos = ijk + np.stack([np64(x) for x in off], axis=1)
    uu = np.stack([np64(x) for x in u])
    v = uu / np.sqrt(1.0 + np.sum(uu * uu, axis=0))
    rho = opart.deposit([np.full(n, -0.5)], pos, shape, (1.0, 1.0, 1.0), 3)[0]
    half = opart.wrap(pos - 0.5 * 0.5 * v.T, p.lengths)
    J = opart.deposit(list(-0.5 * v), half, shape, (1.0, 1.0, 1.0), 3)
    # A node sums at most 64 cells of about 40 particles (2600 contributions), each rounded to half a unit.  FP32:
    # a unit is at most 2^-29 of 0.3 times the tile's 20001 charges, 1.1e-5 charges; a full node holds about 32.
    # FP64: at most 2^-46 charges.  The contributions themselves are good to about 64 eps.
    tol = {"f32": 2600 / 2 * 1.1e-5 / 32, "f64": 2600 / 2 * 2.0 ** -46 / 32}[dtype] + 64 * EPS[dtype]
    assert max_rel(np64(f.rho_new), rho) <= tol
    for d in range(3):
        assert max_rel(np64(f.J_nod[d]), J[d]) <= tol
    ctx.close()


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("shape,order", [((24, 36, 54), 3), ((18, 32, 48), 1)])
def test_centering_in_the_transforms_of_any_length(dtype, shape, order):
    """Calls of several steps centre inside the transforms on every grid; here axes with factors of 9."""
    banner(f"pic_step 3 steps, centering in the transforms dtype={dtype} shape={shape} order={order}")
    steps_against_oracle(shape, 1, order, 8, dtype, 3)


@pytest.mark.parametrize("order", ["grouped", "scattered"])
@pytest.mark.parametrize("shape", [(16, 16, 24), (72, 72, 128), (192, 324, 256), (256, 256, 288)])
def test_tile_sort_tables(shape, order):
    """The counting sort's tables: few buckets (small workgroups), more than 1024, the most the indexed table
    holds, and the hashed table (more than 32768 buckets), with grouped and with scattered particles, some of
    them outside the grid.  Every valid particle deposits its charge once, wherever it lies in the arrays."""
    banner(f"pic_deposit over the sort's tables shape={shape} order={order}")
    N, n = int(np.prod(shape)), 70000
    gen = torch.Generator(device="cuda")
    gen.manual_seed(9)
    cell = torch.randint(0, N, (n,), generator=gen, device="cuda", dtype=torch.int32)
    if order == "grouped":
        cell = cell.sort().values
    bad = torch.arange(0, n, 997, device="cuda")
    cell[bad] = -1
    half = torch.full((n,), 0.5, device="cuda", dtype=torch.float64)
    ctx = piclib.Context(shape, (1.0, 1.0, 1.0), 0.5, 1, 4, 16, "f64")
    f = piclib.Fields(shape, "f64")
    sp = piclib.Species(cell, [half] * 3, [torch.zeros_like(half)] * 3, None, 1.0, 1.0, w_const=8.0)
    for _ in range(2):  # the second call counts into what the first left
        piclib.pic_deposit(ctx.ctx, [sp], f, piclib.PIC_DEP_RHO_ONLY)
    # an offset of 1/2 gives every one of the eight nodes of the cell the charge 8 / 8 = 1
    c = cell[cell >= 0].long()
    i, j, k = c // (shape[1] * shape[2]), (c // shape[2]) % shape[1], c % shape[2]
    ref = torch.zeros(N, device="cuda", dtype=torch.float64)
    one = torch.ones(c.numel(), device="cuda", dtype=torch.float64)
    for a in range(8):
        q = (((i + a // 4) % shape[0]) * shape[1] + (j + a // 2 % 2) % shape[1]) * shape[2] + (k + a % 2) % shape[2]
        ref.index_add_(0, q, one)
    assert torch.equal(f.rho_new.reshape(-1), ref)
    with pytest.raises(RuntimeError, match="out-of-range"):
        piclib.pic_sync(ctx.ctx)
    ctx.close()


@pytest.mark.parametrize("n", [4095, 4096 * 3 + 1, 1300000])
def test_tile_sort_hashed_in_stretches(n):
    """The hashed table with stretches of grouped and of scattered particles in turn: workgroups that place
    their particles themselves beside ones that leave it to the kernel after them, more particles than that
    kernel takes in one walk."""
    shape = (256, 256, 288)
    banner(f"pic_deposit, particles in stretches of either order n={n}")
    N = int(np.prod(shape))
    gen = torch.Generator(device="cuda")
    gen.manual_seed(11)
    cell = torch.randint(0, N, (n,), generator=gen, device="cuda", dtype=torch.int32)
    stretch = torch.arange(n, device="cuda") // 5000
    cell = torch.where(stretch % 2 == 0, cell.sort().values, cell)
    half = torch.full((n,), 0.5, device="cuda", dtype=torch.float64)
    ctx = piclib.Context(shape, (1.0, 1.0, 1.0), 0.5, 1, 4, 16, "f64")
    f = piclib.Fields(shape, "f64")
    sp = piclib.Species(cell, [half] * 3, [torch.zeros_like(half)] * 3, None, 1.0, 1.0, w_const=8.0)
    c = cell.long()
    i, j, k = c // (shape[1] * shape[2]), (c // shape[2]) % shape[1], c % shape[2]
    ref = torch.zeros(N, device="cuda", dtype=torch.float64)
    one = torch.ones(n, device="cuda", dtype=torch.float64)
    for a in range(8):
        q = (((i + a // 4) % shape[0]) * shape[1] + (j + a // 2 % 2) % shape[1]) * shape[2] + (k + a % 2) % shape[2]
        ref.index_add_(0, q, one)
    for _ in range(2):
        piclib.pic_deposit(ctx.ctx, [sp], f, piclib.PIC_DEP_RHO_ONLY)
        assert torch.equal(f.rho_new.reshape(-1), ref)
    ctx.close()


# every workgroup and tile shape of the fused x pass, and the first lengths past its last one
FUSED = [("f32", (8, 288, 384)), ("f32", (96, 96, 96)), ("f32", (108, 96, 96)), ("f32", (216, 64, 64)),
         ("f32", (432, 48, 48)), ("f32", (768, 36, 36)), ("f32", (864, 32, 36)),
         ("f64", (8, 216, 256)), ("f64", (54, 96, 96)), ("f64", (108, 64, 72)), ("f64", (216, 48, 48)),
         ("f64", (512, 32, 32)), ("f64", (576, 32, 32))]


@pytest.mark.parametrize("dtype,shape,nodal", [(*c, False) for c in FUSED] + [("f32", (108, 96, 96), True),
                                                                              ("f64", (216, 48, 48), True)])
def test_field_solve_fused_along_x(dtype, shape, nodal):
    """psatd_push_fields on grids large enough for the x pass, update and inverse x pass in one kernel."""
    banner(f"psatd_push_fields fused along x dtype={dtype} shape={shape} nodal={nodal}")
    p = ostep.Params(shape, (1.0, 1.0, 1.0), 0.5, 1, 8, 16, nodal=nodal)
    ctx = piclib.Context(shape, (1.0, 1.0, 1.0), 0.5, 1, 8, 16, dtype,
                         flags=piclib.PIC_NODAL_SOLVER if nodal else 0)
    f = piclib.Fields(shape, dtype)
    src = rounded(inputs.random_grid(shape, seed=3, count=11), dtype)
    put(f.E_stag, src[0:3])
    put(f.B_stag, src[3:6])
    put(f.J_stag, src[6:9])
    put([f.rho_old, f.rho_new], src[9:11])
    piclib.psatd_push_fields(ctx.ctx, f)
    piclib.pic_sync(ctx.ctx)
    E, B = ostep.push_fields(src[0:3], src[3:6], src[6:9], src[9], src[10], p)
    tol = 10 * 2 * np.log2(np.prod(shape)) * EPS[dtype] * 3
    for d in range(3):
        assert max_rel(np64(f.E_stag[d]), E[d]) <= tol, ("E", d)
        assert max_rel(np64(f.B_stag[d]), B[d]) <= tol, ("B", d)
    ctx.close()


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("shape,ppc,order", [((16, 16, 16), 7, 1), ((16, 16, 16), 5, 3), ((12, 18, 24), 6, 1),
                                             ((8, 8, 16), 9, 3)])
@pytest.mark.parametrize("flags", [0, piclib.PIC_KEEP_ORDER])
def test_few_tiles_in_parts(dtype, shape, ppc, order, flags):
    """Grids of few tiles: each tile is deposited and gathered in parts by several workgroups, the last part
    of a tile holding fewer chunks than the others or none; grouped and in the caller's order."""
    banner(f"pic_step 3 steps, few tiles dtype={dtype} shape={shape} ppc={ppc} order={order} flags={flags}")
    steps_against_oracle(shape, ppc, order, 8, dtype, 3, flags=flags)


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("shape,order", [((8, 12, 18), 2), ((16, 8, 54), 8), ((24, 36, 32), 16), ((32, 36, 1024), 32)])
def test_centerings_in_one_launch(dtype, shape, order):
    """Small grids: the three components in one launch.  Rows and lines that do not fill a workgroup, and lines
    whose rows are over the batch's LDS (FP64, 1024: separate launches), every direction against the oracle."""
    banner(f"centerings in one launch dtype={dtype} shape={shape} order={order}")
    ctx = piclib.Context(shape, (1.0, 1.0, 1.0), 0.5, 1, order, 8, dtype)
    src = rounded(inputs.random_grid(shape, seed=5, count=3), dtype)
    x = torch.tensor(np.stack(src), device="cuda", dtype=torch.float32 if dtype == "f32" else torch.float64)
    tol = 10 * 2 * order * EPS[dtype]  # two axes of a sum of ``order`` terms, margin 10
    names = {piclib.PIC_J: ostep.J_NAMES, piclib.PIC_E: ostep.E_NAMES, piclib.PIC_B: ostep.B_NAMES}
    for direction, centre in ((piclib.PIC_S2N, ocent.s2n), (piclib.PIC_N2S, ocent.n2s)):
        for what in names:
            got = pag._center(ctx, direction, what, x)
            for d in range(3):
                ref = centre(names[what][d], src[d], order // 2)
                assert max_rel(np64(got[d]), ref) <= tol, (direction, what, d)
    ctx.close()


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("shape,order", [((24, 24, 24), 1), ((24, 32, 24), 3), ((16, 24, 32), 3), ((8, 24, 24), 1),
                                         ((36, 24, 54), 3)])
def test_particles_leaving_tiles(dtype, shape, order):
    """The neighbour tile and the faces of a tile's box from the box indices (three or more whole tiles along
    every axis), on one and two tiles along an axis and on ragged ones, where it comes from the cells."""
    banner(f"pic_step 4 steps, particles leaving tiles dtype={dtype} shape={shape} order={order}")
    steps_against_oracle(shape, 2, order, 8, dtype, 4)


def test_field_solve_fused_along_x_rounds_as_the_separate_kernels():
    """The fused x pass forms the same differences before it adds them as the separate update: the same axis
    lengths with x and y exchanged, once along a length that the fused kernel is built for and once along one
    that it is not, have the same rounding errors.  One more rounding of E or B per mode raises their RMS by
    0.4 to 0.6%; that of 3.5 M points and three components is known to 0.02%; the bound is 0.2%."""
    err = {}
    for shape in ((96, 1024, 36), (1024, 96, 36)):
        banner(f"rounding errors of psatd_push_fields FP32 shape={shape}")
        p = ostep.Params(shape, (1.0, 1.0, 1.0), 0.5, 1, 8, 16)
        ctx = piclib.Context(shape, (1.0, 1.0, 1.0), 0.5, 1, 8, 16, "f32")
        f = piclib.Fields(shape, "f32")
        rng = np.random.default_rng(17)
        src = rounded([rng.standard_normal(shape) for _ in range(11)], "f32")
        put(f.E_stag, src[0:3])
        put(f.B_stag, src[3:6])
        put(f.J_stag, src[6:9])
        put([f.rho_old, f.rho_new], src[9:11])
        piclib.psatd_push_fields(ctx.ctx, f)
        piclib.pic_sync(ctx.ctx)
        E, B = ostep.push_fields(src[0:3], src[3:6], src[6:9], src[9], src[10], p)
        err[shape] = [np.sqrt(sum(np.mean((np64(g[d]) - r[d]) ** 2) for d in range(3)))
                      for g, r in ((f.E_stag, E), (f.B_stag, B))]
        ctx.close()
    fused, separate = err.values()
    assert fused[0] <= 1.002 * separate[0], ("E", fused, separate)
    assert fused[1] <= 1.002 * separate[1], ("B", fused, separate)


# both sides of the sizes from which the fused x pass is taken, per group of lengths, and lengths without it
FUSED_FROM = [("f32", (192, 36, 128)), ("f32", (192, 48, 128)), ("f32", (768, 24, 64)), ("f32", (162, 54, 144)),
              ("f32", (162, 64, 162)), ("f32", (486, 128, 144)), ("f32", (648, 64, 96)), ("f64", (16, 128, 216)),
              ("f64", (72, 48, 144)), ("f64", (128, 64, 72)), ("f64", (162, 108, 192)), ("f64", (144, 162, 162)),
              ("f64", (108, 216, 288)), ("f64", (12, 192, 256)), ("f64", (486, 32, 48))]


@pytest.mark.parametrize("dtype,shape", FUSED_FROM)
def test_field_solve_around_the_fused_sizes(dtype, shape):
    """psatd_push_fields on both sides of the rule that chooses the fused x pass."""
    test_field_solve_fused_along_x(dtype, shape, False)


@pytest.mark.parametrize("order", [3, 1])
@pytest.mark.parametrize("dtype,ppc", [("f32", 3), ("f64", 1)])
def test_several_chunks_in_whole_unsplit_tiles(monkeypatch, dtype, ppc, order):
    """Whole tiles, three along every axis, each by one workgroup, some of them of several dealing chunks and
    some empty: neighbour bases, faces gathered over the chunks, neighbours from the box indices and (cubic)
    the published order together, as in the dense tiles of a beam.  The particles of the middle third of x
    move to the first third, so that the average tile stays under two chunks (not split)."""
    shape = (24, 24, 24)
    banner(f"pic_step 4 steps, several chunks in whole tiles dtype={dtype} ppc={ppc} order={order}")
    small = inputs.small

    def crowded(*args, **kw):
        wl = small(*args, **kw)
        wl.electrons.cell = wl.electrons.cell.copy()
        wl.electrons.cell[:, 0] -= 8 * (wl.electrons.cell[:, 0] // 8 == 1)
        return wl

    monkeypatch.setattr(inputs, "small", crowded)
    steps_against_oracle(shape, ppc, order, 8, dtype, 4)
