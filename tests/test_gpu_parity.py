"""GPU parity: the HIP library (through the C ABI) against the FP64 oracle on
the same seeded float32 inputs.

Tolerances (the contract of the library):
  plain FP32 path:  relative energy error <= 1e-6, relative RMS force error <= 1e-5;
  BF16X3 path:      relative RMS force error <= 1e-3, relative energy error <= 1e-3
                    (the form's force budget; random charges reach ~1e-4 in energy).
The GPU evaluates the far part on a grid, so its error against the oracle's
exact image sums also contains the spreading discretisation (about 2e-6 in
force at the default 10^3 stencil with sigma_s = 0.9 h, under 1e-4 at the
BF16X3 default 6^3 with 0.74 h).
"""
import math

import numpy as np
import pytest

import oracle
from gpu_util import compare, gpu_eval, log, oracle_eval, oracle_params, rel_rms

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_1911_01377_amd import (USERIES_BF16X3, USERIES_C0, USERIES_C1, USERIES_C2_B2,  # noqa: E402
                                  USERIES_TABLE1_ROW1, USERIES_TABLE1_ROW2, USERIES_TABLE1_ROW3,
                                  synth)


@pytest.fixture(scope="module", autouse=True)
def need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def test_random_cube_512_plain():
    xyz, q, box = synth.random_cube(512, 24.0, seed=1377)
    compare("random512/plain", xyz, q, box, 9.0, (32, 32, 32), 1e-6, 1e-5)


def test_random_cube_512_bf16x3():
    xyz, q, box = synth.random_cube(512, 24.0, seed=1377)
    compare("random512/bf16x3", xyz, q, box, 9.0, (32, 32, 32), 1e-3, 1e-3,
            precision=USERIES_BF16X3)


@pytest.mark.parametrize("n_mol", [300, 517])
def test_small_water_ragged_grid(n_mol):
    L = (n_mol / synth.WATER_DENSITY) ** (1 / 3)
    xyz, q, box = synth.water_box(n_mol=n_mol, L=L, seed=50 + n_mol)
    g = int(np.ceil(L))
    compare("water%d/plain" % n_mol, xyz, q, box, min(9.0, 0.45 * L), (g, g, g), 1e-6, 1e-5)


def test_small_water_bf16x3():
    n_mol = 700
    L = (n_mol / synth.WATER_DENSITY) ** (1 / 3)
    xyz, q, box = synth.water_box(n_mol=n_mol, L=L, seed=3)
    g = int(np.ceil(L))
    compare("water700/bf16x3", xyz, q, box, 9.0, (g, g, g), 1e-3, 1e-3,
            precision=USERIES_BF16X3)


@pytest.mark.parametrize("P,ratio", [(6, 0.9), (8, 0.9), (4, 0.83)])
def test_stencil_widths(P, ratio):
    """Non-default spreading stencils through the plain path: P = 6 and 8 take
    the gather kernel's 4^3 bricks (P > 5) and larger halos; every width sizes
    the gather kernel's LDS.  P >= 5 at sigma_s = 0.9 h meets the plain
    contract; the 8^3 stencil at 0.83 h (about 2e-5 in force on water) is held
    to 1e-4."""
    n_mol = 500
    L = (n_mol / synth.WATER_DENSITY) ** (1 / 3)
    xyz, q, box = synth.water_box(n_mol=n_mol, L=L, seed=61)
    g = int(np.ceil(L))
    tol = (1e-6, 1e-5) if P >= 5 else (1e-4, 1e-4)
    compare("water500/plain/P%d" % P, xyz, q, box, min(9.0, 0.45 * L), (g, g, g), tol[0], tol[1],
            stencil_half=P, sigma_s_over_h=ratio)


@pytest.mark.parametrize("form,n_mol,grid", [
    ("plain", 137, (16, 17, 18)), ("plain", 137, (18, 16, 17)), ("plain", 137, (17, 23, 24)),
    ("plain", 137, (15, 23, 24)), ("plain", 73, (10, 11, 12)), ("plain", 73, (13, 10, 14)),
    ("bf16x3", 73, (12, 13, 14)), ("bf16x3", 73, (14, 12, 13)), ("bf16x3", 73, (15, 16, 17))])
def test_stencil_and_brick_about_as_wide_as_the_grid(form, n_mol, grid):
    """Axes of about brick + stencil points (8 + 2P - 1: 17 plain, 13 BF16X3),
    where a charge's stencil can meet a spreading brick from both sides of the
    periodic boundary, and bricks cut to 1 to 7 points."""
    L = (n_mol / synth.WATER_DENSITY) ** (1 / 3)
    xyz, q, box = synth.water_box(n_mol=n_mol, L=L, seed=17)
    tol = (1e-6, 1e-5) if form == "plain" else (1e-3, 1e-3)
    compare("water%d/%s/%s" % (n_mol, form, grid), xyz, q, box, 0.45 * L, grid, tol[0], tol[1],
            precision=USERIES_BF16X3 if form == "bf16x3" else 0)


@pytest.mark.parametrize("n_mol,seed", [(73, 17), (20, 3), (3, 1)])
def test_clusters_longer_than_half_the_cell(n_mol, seed):
    """A few waters in cells of 8.4 to 13 A: a sparse column's clusters can
    extend over more than half the cell along z (the pair kernel's bounding
    box of the i-cluster)."""
    L = max(8.4, (n_mol / synth.WATER_DENSITY) ** (1 / 3))
    xyz, q, box = synth.water_box(n_mol=n_mol, L=L, seed=seed)
    compare("water%d/sparse" % n_mol, xyz, q, box, 0.45 * L, (16, 16, 16), 1e-6, 1e-5,
            e_scale="parts")


def test_orthorhombic_box_and_grid():
    rng = np.random.default_rng(4)
    box = (20.0, 23.5, 27.0)
    n = 700
    xyz = (rng.uniform(0, 1, (n, 3)) * box).astype(np.float32)
    q = synth._quantise(rng.uniform(-1, 1, n))
    q[-1] = -np.sum(q[:-1])
    compare("ortho700/plain", xyz, q.astype(np.float32), box, 8.0, (20, 24, 30), 1e-6, 1e-5)


@pytest.mark.parametrize("box", [(22.37, 22.8, 22.63), (22.53, 23.03, 21.39),
                                 (22.87, 21.65, 22.87), (23.83, 22.61, 23.31)])
def test_near_energy_with_the_axes_in_any_order(box):
    """300 waters in cells whose near energy, with the axes' units relative to
    x formed from units already rounded to FP32, differs by 1.3e-7 to 1.5e-7
    between the three orders of the axes.  With each such factor rounded once
    they agree to 1.5e-8 (both from the factors put into an FP64 pair sum);
    the FP32 polynomial coefficients, whose unit is the x axis's, and the sum's
    own rounding add to either."""
    L = (300 / synth.WATER_DENSITY) ** (1 / 3)
    xyz, q, _ = synth.water_box(n_mol=300, L=L, seed=77)
    e = []
    for ax in ([0, 1, 2], [1, 2, 0], [2, 0, 1]):
        cell = tuple(box[a] for a in ax)
        parts, _, _ = gpu_eval(np.ascontiguousarray(xyz[:, ax]), q, cell, 9.0, (28, 28, 28))
        e.append(parts[0])
    spread = (max(e) - min(e)) / abs(e[0])
    log("case axes %s: near energies %s, spread %.2e" % (box, e, spread))
    assert spread <= 5e-8


@pytest.mark.parametrize("form", ["plain", "bf16x3"])
def test_small_charges_in_a_non_cubic_cell(form):
    """Charges 2^-50 times as large give forces 2^-100 and energies 2^-100 times
    as large: scaling by a power of two rounds nothing while every term of the
    sums stays a normal FP32 number (1e-6: those of the spread that do not)."""
    rng = np.random.default_rng(4)
    box, n = (20.0, 23.5, 27.0), 700
    xyz = (rng.uniform(0, 1, (n, 3)) * box).astype(np.float32)
    q = rng.choice([-1.0, 1.0], n).astype(np.float32)
    kw = dict(precision=USERIES_BF16X3) if form == "bf16x3" else {}
    p0, f0, _ = gpu_eval(xyz, q, box, 8.0, (20, 24, 30), **kw)
    p1, f1, _ = gpu_eval(xyz, q * np.float32(2.0 ** -50), box, 8.0, (20, 24, 30), **kw)
    df, de = rel_rms(f1 * 2.0 ** 100, f0), abs(p1[4] * 2.0 ** 100 / p0[4] - 1.0)
    log("case small charges/%s: dF=%.2e dE=%.2e" % (form, df, de))
    assert df <= 1e-6 and de <= 1e-6


def test_tall_box_long_columns():
    # a 16 x 16 x 96 A water cell (six z-replicas of a 16 A water box): 9
    # columns of ~270 charges, so the column sort takes more than one charge
    # per thread
    x1, q1, box1 = synth.water_box(n_mol=137, L=16.0, seed=29)
    L = box1[0]
    xyz = np.concatenate([x1 + np.array([0.0, 0.0, k * L], np.float32) for k in range(6)])
    q = np.concatenate([q1] * 6)
    box = (L, L, 6 * L)
    _, _, _, _, info = compare("tallwater/plain", xyz.astype(np.float32), q, box, 0.45 * L,
                               (16, 16, 96), 1e-6, 1e-5)
    assert len(q) / (info["ncell"][0] * info["ncell"][1]) > 256


def test_one_dense_column_global_ranking():
    """2,000 random charges in a 3 x 3 A wire along z of a 20 x 20 x 64 A cell:
    the 4 x 4 columns are 5 A wide, so one column holds every charge, more
    than the 1,024 that the column sort ranks in LDS (it ranks them from
    global memory), and the other fifteen are empty."""
    xyz, q, _ = synth.random_box(2000, (3.0, 3.0, 64.0), seed=43)
    xyz = (xyz + np.array([0.5, 0.5, 0.0], np.float32)).astype(np.float32)
    box = (20.0, 20.0, 64.0)
    _, _, _, _, info = compare("wire2000/plain", xyz, q, box, 9.0, (20, 20, 64), 1e-6, 1e-5,
                               e_scale="parts")
    assert tuple(info["ncell"][:2]) == (4, 4), info["ncell"]


@pytest.mark.parametrize("n", [1024, 1025])
def test_column_at_the_lds_sort_limit(n):
    """The wire of the test above with 1,024 charges, the most a column sorts
    in LDS, and with one more."""
    xyz, q, _ = synth.random_box(n, (3.0, 3.0, 64.0), seed=n)
    xyz = (xyz + np.array([0.5, 0.5, 0.0], np.float32)).astype(np.float32)
    compare("wire%d/plain" % n, xyz, q, (20.0, 20.0, 64.0), 9.0, (20, 20, 64), 1e-6, 1e-5,
            e_scale="parts")


def test_dense_column_among_many_blocks():
    """262,500 random charges in a 140 A cube and 1,500 more in a 3 x 3 A wire
    along z: a column of more than 1,024 charges, ranked from global memory,
    among 1,032 blocks of 256 input charges.  Forces on 64 sampled charges of the wire."""
    x1, q1, _ = synth.random_box(262500, (140.0, 140.0, 140.0), seed=81)
    x2, q2, _ = synth.random_box(1500, (3.0, 3.0, 140.0), seed=82)
    xyz = np.concatenate([x1, x2 + np.array([0.3, 0.3, 0.0], np.float32)]).astype(np.float32)
    q, box, rc = np.concatenate([q1, q2]), (140.0, 140.0, 140.0), 9.0
    order = np.random.default_rng(83).permutation(len(q))
    xyz, q = xyz[order], q[order]
    _, gf, info = gpu_eval(xyz, q, box, rc, (128, 128, 128))
    idx = np.nonzero(order >= 262500)[0][:64]
    fo = oracle.forces_subset(xyz.astype(np.float64), q.astype(np.float64), box,
                              oracle_params(info, rc), idx)
    df = rel_rms(gf[idx], fo)
    log("case dense column among many blocks/plain: dF(64 sampled)=%.2e" % df)
    assert df <= 1e-5


def kernel_us(xyz, q, box, rc, grid, kernel, reps=5, **kw):
    """Time of one kernel of an evaluation: the mean of `reps`, best of five."""
    from paper_1911_01377_amd import Plan
    plan = Plan(box, rc, grid, **kw)
    x, qq = torch.from_numpy(xyz).cuda(), torch.from_numpy(q).cuda()
    best = math.inf
    for _ in range(5):
        plan.eval(x, qq)
        torch.cuda.synchronize()
        plan.timing(True)
        for _ in range(reps):
            plan.eval(x, qq)
        torch.cuda.synchronize()
        ms = {name: total / max(count, 1) for name, total, count in plan.timing()}
        plan.timing(False)
        best = min(best, 1e3 * ms[kernel])
    plan.close()
    return best


def wire(n, seed):
    """n charges +-1 in a 3 x 3 A wire along z of a 20 x 20 x 64 A cell (one
    column holds them all), no two at the same z, in increasing z."""
    rng = np.random.default_rng(seed)
    xyz = np.empty((n, 3), np.float32)
    xyz[:, :2] = rng.uniform(0.5, 3.5, (n, 2))
    xyz[:, 2] = (np.arange(n) + rng.uniform(0.0, 0.5, n)) * (64.0 / n)
    return xyz, rng.choice([-1.0, 1.0], n).astype(np.float32), (20.0, 20.0, 64.0)


@pytest.mark.parametrize("n", [1025, 2048, 2049, 4100])
def test_long_column_in_any_input_order(n):
    """A column longer than the LDS sort, its charges in z order (few input
    blocks per stretch of it) and shuffled: it sorts to the same sequence, so
    the forces are the same bits."""
    xyz, q, box = wire(n, n)
    order = np.random.default_rng(n).permutation(n)
    _, f0, _ = gpu_eval(xyz, q, box, 9.0, (20, 20, 64))
    _, f1, _ = gpu_eval(xyz[order], q[order], box, 9.0, (20, 20, 64))
    assert np.array_equal(f0[order], f1)


@pytest.mark.parametrize("n", [1100, 2000])
def test_long_column_uses_all_threads(n):
    """Sorting a column of 1,100 or 2,000 charges, which lie in 5 or 8 blocks
    of 256 input charges, takes at most 100 times as long as one of 1,000 in
    LDS.  (Four to eight charges per thread against n keys from global memory
    are 35 to 100 times, one thread per input block was 1,600 to 3,000.)"""
    short = kernel_us(*wire(1000, 1), 9.0, (20, 20, 64), "colbuild")
    long = kernel_us(*wire(n, 2), 9.0, (20, 20, 64), "colbuild")
    log("case wire%d: colbuild %.1f us, 1,000 charges %.1f us" % (n, long, short))
    assert long <= 100.0 * short


def layers(n, nz, seed):
    """n charges +-1 in a 3 x 3 A footprint of a 20 x 20 x 64 A cell (one
    column), at nz values of z."""
    rng = np.random.default_rng(seed)
    xyz = np.empty((n, 3), np.float32)
    xyz[:, :2] = rng.uniform(0.5, 3.5, (n, 2))
    xyz[:, 2] = 30.0 + 1.5 * rng.permutation(np.arange(n) % nz)
    return xyz, rng.choice([-1.0, 1.0], n).astype(np.float32), (20.0, 20.0, 64.0)


@pytest.mark.parametrize("nz", [1, 7, 9])
@pytest.mark.parametrize("n", [5, 256, 257, 512, 513, 1024])
def test_layers_in_one_column(n, nz):
    """A column whose charges share 1 to 9 values of z: 1 and 7 leave more than
    an eighth of it in one sort bucket (ranked against the whole column, 1, 2
    or 4 charges per thread), 9 do not.  The order is by (z, input index)
    either way, so the forces are those of the same charges given in that
    order, bit for bit."""
    xyz, q, box = layers(n, nz, 10 * n + nz)
    order = np.argsort(xyz[:, 2], kind="stable")
    _, f0, _ = gpu_eval(xyz, q, box, 9.0, (20, 20, 64))
    _, f1, _ = gpu_eval(xyz[order], q[order], box, 9.0, (20, 20, 64))
    assert np.array_equal(f0[order], f1)


@pytest.mark.parametrize("n,factor", [(256, 2.0), (1024, 6.0)])
def test_one_layer_sorts_in_time(n, factor):
    """A column whose charges all share one z: 256 keys per thread take at
    most twice the time of distinct z, and 1,024 for four charges per thread
    at most 6 times.  (Ranked one key at a time within the bucket they took
    2.3 and 17 times.)"""
    box, grid = (20.0, 20.0, 64.0), (20, 20, 64)
    xyz, q, _ = layers(n, 1, 1)
    tied = kernel_us(xyz, q, box, 9.0, grid, "colbuild", reps=50)
    apart = kernel_us(*wire(n, 2), 9.0, grid, "colbuild", reps=50)
    log("case layer%d: colbuild %.1f us, distinct z %.1f us" % (n, tied, apart))
    assert tied <= factor * apart


@pytest.mark.parametrize("gz", [20, 128])
def test_columns_of_tied_z(gz):
    """A 10 x 10 x 10 lattice of alternating unit charges, jittered in x and y
    only and in shuffled input order: each column's charges share ten values
    of z, so its sort buckets hold ties that the input index orders."""
    rng = np.random.default_rng(gz)
    ijk = np.stack(np.meshgrid(*[np.arange(10)] * 3, indexing="ij"), -1).reshape(-1, 3)
    xyz = (ijk + 0.5) * 2.0
    xyz[:, :2] += rng.uniform(-0.4, 0.4, (1000, 2))
    order = rng.permutation(1000)
    q = (1.0 - 2.0 * (ijk.sum(1) % 2)).astype(np.float32)[order]
    compare("ties1000/plain", xyz.astype(np.float32)[order], q, (20.0, 20.0, 20.0), 9.0,
            (20, 20, gz), 1e-6, 1e-5, e_scale="parts")


def test_many_columns_global_binning():
    """A flat 256 x 256 x 19 A cell of 200,000 random charges: 69 x 69
    columns, more than the 4096 whose counts the binning kernels keep in LDS,
    so the column counts, the slot counters and the offsets (scan kernel) take
    their global-memory paths.  The oracle's full O(n^2) sum is out of reach
    at this size: forces on 128 sampled charges are compared (each an O(n)
    oracle sum), and the force sum must vanish up to rounding.  The x-y grid
    spacing is 2 A (0.95 A in z)."""
    xyz, q, box = synth.random_box(200000, (256.0, 256.0, 19.0), seed=31)
    rc, grid = 9.0, (128, 128, 20)
    log("case manycols/plain: n=%d box=%s rc=%g grid=%s" % (len(q), box, rc, grid))
    _, gf, info = gpu_eval(xyz, q, box, rc, grid)
    ncol = info["ncell"][0] * info["ncell"][1]
    assert ncol > 4096, info["ncell"]
    idx = np.random.default_rng(3).choice(len(q), 128, replace=False)
    fo = oracle.forces_subset(xyz.astype(np.float64), q.astype(np.float64), box,
                              oracle_params(info, rc), idx)
    df = rel_rms(gf[idx], fo)
    rms = float(np.sqrt(np.mean(np.sum(gf ** 2, axis=1))))
    mag = np.sqrt(np.sum(fo ** 2, axis=1))
    da = float((np.sqrt(np.sum((gf[idx] - fo) ** 2, axis=1)) / np.maximum(mag, rms)).max())
    fsum = float(np.linalg.norm(gf.sum(axis=0)))
    log("   columns %s, dF(128 sampled)=%.2e, max|dF_i|/max(|F_i|,rms)=%.2e, |sum F|=%.3e (rms %.3e)"
        % (info["ncell"], df, da, fsum, rms))
    assert df <= 1e-5
    assert da <= 1e-4
    assert fsum <= 1e-3 * math.sqrt(len(q)) * rms


def test_more_than_64_columns_under_a_brick():
    """A jittered 32^3 lattice of alternating unit charges in an 18 A cell on a
    14^3 grid (BF16X3): 15 x 15 columns, so a gather brick overlaps 81 of them
    (the ranges are held 64 at a time) and a spreading brick's window all 225.
    Forces on 128 sampled charges."""
    rng = np.random.default_rng(71)
    ijk = np.stack(np.meshgrid(*[np.arange(32)] * 3, indexing="ij"), -1).reshape(-1, 3)
    xyz = ((ijk + 0.5) * (18.0 / 32) + rng.uniform(-0.1, 0.1, ijk.shape)).astype(np.float32)
    q = (1.0 - 2.0 * (ijk.sum(1) % 2)).astype(np.float32)
    box, rc = (18.0, 18.0, 18.0), 4.7
    _, gf, info = gpu_eval(xyz, q, box, rc, (14, 14, 14), precision=USERIES_BF16X3)
    assert tuple(info["ncell"][:2]) == (15, 15), info["ncell"]
    idx = rng.choice(len(q), 128, replace=False)
    fo = oracle.forces_subset(xyz.astype(np.float64), q.astype(np.float64), box,
                              oracle_params(info, rc), idx)
    df = rel_rms(gf[idx], fo)
    log("case columns under a brick/bf16x3: dF(128 sampled)=%.2e" % df)
    assert df <= 1e-3


@pytest.mark.parametrize("grid", [(90, 91, 64), (91, 90, 30), (96, 86, 31), (91, 90, 110)])
def test_wide_z_convolution(grid):
    """BF16X3 grids of 8,190 to 8,256 (x, y) columns: 512 groups of 16 and
    more, from which conv_z takes two groups per block, ragged last ones among
    them; padded z lengths of 32, 64 and 128 (4, 2 and 1 term groups).  Against
    a grid below the line (44 x 44) on the same cell: the forces agree to the
    sum of the grids' own errors (1e-3 each)."""
    xyz, q, box = synth.water_box(n_mol=1094, L=32.0, seed=12)
    _, f, _ = gpu_eval(xyz, q, box, 9.0, grid, precision=USERIES_BF16X3)
    _, f0, _ = gpu_eval(xyz, q, box, 9.0, (44, 44, grid[2]), precision=USERIES_BF16X3)
    assert rel_rms(f, f0) <= 2e-3


@pytest.mark.parametrize("nx,nz", [(8, 8), (9, 8)])
def test_gather_on_either_side_of_512_bricks(nx, nz):
    """512 bricks (16 wavefronts per gather block at P = 5) and 576 (8), on a
    32 A cell of water, against a 48^3 grid (216 bricks): the forces agree to
    the sum of the grids' own errors (1e-5 each)."""
    xyz, q, box = synth.water_box(n_mol=1094, L=32.0, seed=9)
    _, f, _ = gpu_eval(xyz, q, box, 9.0, (8 * nx, 64, 8 * nz))
    _, f0, _ = gpu_eval(xyz, q, box, 9.0, (48, 48, 48))
    assert rel_rms(f, f0) <= 2e-5


FORMS = [(0, (1e-6, 1e-5)), (USERIES_BF16X3, (1e-3, 1e-3))]


def _form(precision):
    return "bf16x3" if precision else "plain"


@pytest.mark.parametrize("precision,tol", FORMS)
def test_many_candidates_per_cluster(precision, tol):
    """3,000 random charges in a 20 A cube (0.375 per A^3) with r_c = 9.5 A:
    every cluster has 2,400 to 3,000 candidates (a host count with the
    kernel's column and z-window rules), more than the 2,048 whose ranges
    the pair kernel looks up in its table, so every block takes the range
    search instead."""
    xyz, q, box = synth.random_box(3000, (20.0, 20.0, 20.0), seed=47)
    compare("dense3000/" + _form(precision), xyz, q, box, 9.5, (20, 20, 20), tol[0], tol[1],
            e_scale="parts", precision=precision)


@pytest.mark.parametrize("precision,tol", FORMS)
def test_terms_staged_in_chunks(precision, tol):
    """N = 4 on grids of 128 z points: a z-convolution block stages the columns
    of at most 2 terms at once (20 KiB of LDS), so it runs over two chunks of
    terms, in both forms.  A 32 A water box (32 x 32 x 128 grid) is held to
    the form's tolerances.  The second chunk's terms (16 and 32 A wide) must
    be in the result: for 2000 random charges in a 32 A cube, whose far energy
    they move by about 1%, the far energy lies within a fifth of the gap
    between the oracle's 4-term value and its value from the first 2 terms."""
    xyz, q, box = synth.water_box(None, 32.0, seed=23)
    _, _, _, _, info = compare("chunks/%s" % _form(precision), xyz, q, box, 8.0, (32, 32, 128),
                               tol[0], tol[1], n_terms=4, precision=precision)
    assert info["n_terms"] == 4 and info["n_terms_grid"] == 4
    xyz, q, box = synth.random_cube(2000, 32.0, seed=5)
    gp, _, info = gpu_eval(xyz, q, box, 8.0, (48, 48, 128), n_terms=4, precision=precision)
    x64, q64 = xyz.astype(np.float64), q.astype(np.float64)
    far4, _ = oracle.eval_far(x64, q64, box, oracle_params(info, 8.0))
    far2, _ = oracle.eval_far(x64, q64, box, oracle_params(dict(info, n_terms=2), 8.0))
    log("   random2000 far energy: gpu %.9f, oracle 4 terms %.9f, first 2 only %.9f"
        % (gp[1], far4, far2))
    assert abs(gp[1] - far4) < 0.2 * abs(far4 - far2)


@pytest.mark.parametrize("precision,tol", FORMS)
def test_terms_wider_than_the_box_are_skipped(precision, tol):
    """N = 8 in a 30 A water box: terms 4..7 (64 to 515 A wide) have every
    non-zero Fourier mode below 2^-60 of their k = 0 mode, so the grid
    evaluates terms 0..3 only; the oracle sums all eight.  Evaluated on the
    grid, those terms' nearly constant values would only add FP32 rounding
    (about 5e-6 of the far energy at N = 8)."""
    xyz, q, box = synth.water_box(None, 30.0, seed=24)
    _, _, _, _, info = compare("wide/%s" % _form(precision), xyz, q, box, 8.0, (32, 32, 32),
                               tol[0], tol[1], n_terms=8, precision=precision)
    assert info["n_terms"] == 8 and info["n_terms_grid"] == 4


@pytest.mark.parametrize("k", range(6))
@pytest.mark.parametrize("precision,tol", FORMS)
def test_random_water_configurations(k, precision, tol):
    """Seeded random water boxes: 200-1,200 molecules (L = 18-33 A), a grid
    spacing drawn per axis from [0.75, 0.95] A (grids of any length, not
    multiples of the tile sizes), r_c = min(9, 0.45 L), the default series."""
    rng = np.random.default_rng(1000 + k)
    n_mol = int(rng.integers(200, 1201))
    L = (n_mol / synth.WATER_DENSITY) ** (1 / 3)
    xyz, q, box = synth.water_box(n_mol=n_mol, L=L, seed=2000 + k)
    grid = tuple(int(np.ceil(L / rng.uniform(0.75, 0.95))) for _ in range(3))
    compare("randwater%d/%s" % (k, _form(precision)), xyz, q, box, min(9.0, 0.45 * L), grid,
            tol[0], tol[1], precision=precision)


@pytest.mark.parametrize("precision,tol", FORMS)
def test_non_neutral_and_single_charge(precision, tol):
    """A net charge Q: the far part sums only k != 0 (eqs. 4, 9, 10), so any
    uniform offset of the grid potential (left by the spreading weights' sums
    and the FP32 rounding of the widest terms) must not reach the energy, where
    it would enter as Q x offset / 2.  Held to the form's neutral-input
    tolerances, together with a single charge (the simple-cubic Wigner
    lattice)."""
    rng = np.random.default_rng(8)
    L = 18.0
    xyz = rng.uniform(0, L, (200, 3)).astype(np.float32)
    q = (rng.uniform(-1, 1, 200) + 0.05).astype(np.float32)
    f = _form(precision)
    compare("nonneutral200/" + f, xyz, q, (L, L, L), 8.0, (24, 24, 24), tol[0], tol[1],
            precision=precision)
    q2 = (rng.uniform(-1, 1, 300) + 0.3).astype(np.float32)
    xyz2 = rng.uniform(0, 22.0, (300, 3)).astype(np.float32)
    compare("nonneutral300/" + f, xyz2, q2, (22.0, 22.0, 22.0), 9.0, (22, 22, 22), tol[0], tol[1],
            precision=precision)
    compare("single/" + f, np.array([[1.0, 2.0, 3.0]], np.float32), np.array([1.0], np.float32),
            (L, L, L), 8.0, (24, 24, 24), tol[0], tol[1], precision=precision)


def test_empty_input():
    log("case empty")
    parts, f, _ = gpu_eval(np.zeros((0, 3), np.float32), np.zeros(0, np.float32),
                           (20.0, 20.0, 20.0), 8.0, (20, 20, 20))
    assert np.all(parts == 0.0) and f.shape == (0, 3)


def test_images_and_permutation():
    xyz, q, box = synth.random_cube(300, 21.0, seed=12)
    # positions on a 2^-12 A lattice, so that adding whole box lengths is exact in float32
    xyz = (np.round(xyz.astype(np.float64) * 4096) / 4096).astype(np.float32)
    log("case images/permutation")
    p0, f0, _ = gpu_eval(xyz, q, box, 9.0, (24, 24, 24))
    shift = np.array([21.0, -42.0, 63.0], np.float32)
    p1, f1, _ = gpu_eval(xyz + shift, q, box, 9.0, (24, 24, 24))
    assert abs(p1[4] - p0[4]) <= 1e-9 * abs(p0[4])
    assert np.max(np.abs(f1 - f0)) <= 1e-6 * np.max(np.abs(f0))
    perm = np.random.default_rng(1).permutation(len(q))
    p2, f2, _ = gpu_eval(xyz[perm], q[perm], box, 9.0, (24, 24, 24))
    assert abs(p2[4] - p0[4]) <= 1e-7 * abs(p0[4])
    assert rel_rms(f2, f0[perm]) <= 1e-6


def test_repeat_is_bitwise_identical():
    import torch as T
    from paper_1911_01377_amd import Plan
    log("case determinism")
    xyz, q, box = synth.water_box(n_mol=800, L=(800 / synth.WATER_DENSITY) ** (1 / 3), seed=9)
    plan = Plan(box, 9.0, (29, 29, 29))
    x = T.from_numpy(xyz).cuda()
    qq = T.from_numpy(q).cuda()
    e1, f1, _ = plan.eval(x, qq)
    e1, f1 = e1.clone(), f1.clone()
    for _ in range(3):
        e2, f2, _ = plan.eval(x, qq)
    T.cuda.synchronize()
    assert T.equal(e1, e2) and T.equal(f1, f2)
    plan.close()


def test_near_and_far_parts_separately():
    """The near energy matches the oracle's pair sum; the far energy its image sums."""
    xyz, q, box = synth.random_cube(400, 22.0, seed=31)
    log("case parts")
    gp, gf, info = gpu_eval(xyz, q, box, 9.0, (30, 30, 30))
    op, of = oracle_eval(xyz, q, box, info, 9.0)
    # the total of random charges is a small difference of much larger parts,
    # so the parts are measured against the sum of their magnitudes
    scale = abs(op["near"]) + abs(op["far"]) + abs(op["total"])
    log("   near %.3e far %.3e (x scale)" % (abs(gp[0] - op["near"]) / scale,
                                            abs(gp[1] - op["far"]) / scale))
    assert abs(gp[0] - op["near"]) <= 1e-6 * scale
    assert abs(gp[1] - op["far"]) <= 1e-6 * scale
    assert abs(gp[2] - op["self"]) <= 1e-12 * op["self"]


def test_graph_replay_matches_eager():
    """One evaluation captured in a HIP graph (as the benchmark times it):
    every replay, with eager evaluations between them, gives the eager result
    bitwise."""
    from paper_1911_01377_amd import Plan
    xyz, q, box = synth.water_box(n_mol=400, L=(400 / synth.WATER_DENSITY) ** (1 / 3), seed=71)
    g = int(np.ceil(box[0]))
    log("case graph replay: n=%d grid=%d" % (len(q), g))
    dev = torch.device("cuda:0")
    x = torch.from_numpy(xyz).to(dev)
    qq = torch.from_numpy(q).to(dev)
    for prec in (0, USERIES_BF16X3):
        plan = Plan(box, min(9.0, 0.45 * box[0]), (g, g, g), precision=prec)
        e_ref, f_ref, _ = plan.eval(x, qq)
        torch.cuda.synchronize()
        e_ref, f_ref = e_ref.clone(), f_ref.clone()
        forces = torch.empty_like(f_ref)
        energy = torch.empty_like(e_ref)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            plan.eval(x, qq, forces, energy)
        for rep in range(4):
            forces.zero_()
            energy.zero_()
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(forces, f_ref) and torch.equal(energy, e_ref), (prec, rep)
            e2, f2, _ = plan.eval(x, qq)       # eager work between replays
            torch.cuda.synchronize()
            assert torch.equal(f2, f_ref) and torch.equal(e2, e_ref)
        plan.close()


CONSTRUCTIONS = [(USERIES_C0, "C0"), (USERIES_C2_B2, "C2b2"), (USERIES_TABLE1_ROW1, "T1r1"),
                 (USERIES_TABLE1_ROW2, "T1r2"), (USERIES_TABLE1_ROW3, "T1r3")]


@pytest.mark.parametrize("construction,name", CONSTRUCTIONS)
@pytest.mark.parametrize("precision,tol", FORMS)
def test_every_construction(construction, name, precision, tol):
    """Every construction the plan accepts, through the same kernels, at the
    form's tolerances: C0 (eqs. 19-21), the C2 series of eq. 28 with Table 2's
    b = 2 parameters, and the three C2 points of the C1 construction in
    Table 1 (b = 1.63, 1.32, 1.22: sigma = r_c / r0 down to 1.6 A, N up to
    15 terms, and the narrowest Gaussians evaluated exactly in the near part).
    A water box and a box of random charges each; the oracle takes the plan's
    (b, sigma, w0, s0, N).

    The grid spacing follows the narrowest far Gaussian s_0 = sigma s0: at most
    1 A and at most s_0 / 2.  Spreading, convolution and gathering represent
    s_0 through Gaussians narrower still (sigma_s and the on-grid kernel), so
    a grid much coarser than s_0 / 2 loses the far part's accuracy (Table 1
    row 3 at r_c = 9 A has s_0 = 1.6 A: the FP64 discrete scheme misses the
    exact far energy by 8e-6 of the total at h = 0.61 s_0 and by 4e-8 at
    0.50 s_0)."""
    from paper_1911_01377_amd import _native
    _, r0, _, s0 = _native.useries_solve_construction(construction, 2.0)
    s_min = 9.0 / r0 * s0
    n_mol = 600
    L = (n_mol / synth.WATER_DENSITY) ** (1 / 3)
    xyz, q, box = synth.water_box(n_mol=n_mol, L=L, seed=300 + construction)
    g = int(np.ceil(L / min(1.0, 0.5 * s_min)))
    f = _form(precision)
    _, _, _, _, info = compare("water600/%s/%s" % (name, f), xyz, q, box, 9.0, (g, g, g),
                               tol[0], tol[1], construction=construction, precision=precision)
    if construction in (USERIES_TABLE1_ROW2, USERIES_TABLE1_ROW3) and not precision:
        assert info["near_exact"] > 0
    # random charges: the total energy is a small difference of the parts
    # (random512 with Table 1 row 2: near 3.9, far 30.8, self 36.3, total
    # -1.6), so the energy is held relative to the parts' magnitudes; with N = 10
    # terms the FP32 far part errs by about 2.5e-7 of itself, and the BF16X3
    # form's 6^3 stencil truncates its Gaussians at 4 sigma_s (2.7e-4 of the
    # far part)
    xyz, q, box = synth.random_cube(512, 24.0, seed=400 + construction)
    g = max(32, int(np.ceil(24.0 / (0.5 * s_min))))
    compare("random512/%s/%s" % (name, f), xyz, q, box, 9.0, (g, g, g), tol[0], tol[1],
            e_scale="parts", construction=construction, precision=precision)


@pytest.mark.parametrize("construction,degree,ne", [
    (USERIES_TABLE1_ROW3, 4, 8), (USERIES_TABLE1_ROW3, 5, 7), (USERIES_TABLE1_ROW3, 6, 6),
    (USERIES_TABLE1_ROW3, 8, 4), (USERIES_TABLE1_ROW3, 9, 3), (USERIES_TABLE1_ROW1, 5, 2),
    (USERIES_TABLE1_ROW1, 7, 1)])
def test_counts_of_exact_gaussians(construction, degree, ne):
    """Polynomial degrees that leave 1 to 8 exact Gaussians to the pair
    kernel, which is compiled for 1, 2, 3, 5 and 8 of them (others rounded
    up), in a cubic and a non-cubic cell, at the plain tolerances.  (Row 3
    stays at degrees up to 9: its monomial coefficients of degree 11 and
    above are too large for FP32 at 1e-5 in force.)"""
    L = (300 / synth.WATER_DENSITY) ** (1 / 3)
    xyz, q, box = synth.water_box(n_mol=300, L=L, seed=77)
    for b in (box, (box[0], box[1] * 1.05, box[2])):
        _, _, _, _, info = compare("water300/exact%d/degree%d" % (ne, degree), xyz, q, b, 9.0,
                                   (28, 28, 28), 1e-6, 1e-5, construction=construction,
                                   poly_degree=degree)
        assert info["near_exact"] == ne


def test_c1_at_other_bases():
    """The C1 construction solved on the host for b other than 2 (the
    smallest root of eq. 26 with w0 from eq. 25): b = 1.5 and 3."""
    n_mol = 500
    L = (n_mol / synth.WATER_DENSITY) ** (1 / 3)
    xyz, q, box = synth.water_box(n_mol=n_mol, L=L, seed=77)
    g = int(np.ceil(L))
    for b in (1.5, 3.0):
        compare("water500/C1/b%.1f" % b, xyz, q, box, min(9.0, 0.45 * L), (g, g, g), 1e-6, 1e-5,
                construction=USERIES_C1, b=b)


@pytest.mark.parametrize("precision,tol", FORMS)
def test_dispersion_kernel_alpha6(precision, tol):
    """The 1/r^6 series (App. A, C1 construction for 1/r^6 at b = 2) through
    the same kernels: positive coefficients (no neutrality; the far terms keep
    their k = 0 components), a water box with one coefficient per site kind
    and random coefficients in a cube; against the oracle's 1/r^6 series with
    the plan's parameters."""
    f = _form(precision)
    n_mol = 600
    L = (n_mol / synth.WATER_DENSITY) ** (1 / 3)
    xyz, _, box = synth.water_box(n_mol=n_mol, L=L, seed=66)
    c = np.tile(np.array([1.0, 0.25, 0.25], np.float32), n_mol)
    g = int(np.ceil(L))
    _, _, _, _, info = compare("water600/r^-6/" + f, xyz, c, box, 9.0, (g, g, g), tol[0], tol[1],
                               alpha=6, precision=precision)
    assert info["n_terms"] >= 2
    rng = np.random.default_rng(67)
    xyz = rng.uniform(0, 22.0, (700, 3)).astype(np.float32)
    c = rng.uniform(0.2, 1.5, 700).astype(np.float32)
    compare("random700/r^-6/" + f, xyz, c, (22.0, 22.0, 22.0), 8.5, (24, 24, 24), tol[0], tol[1],
            alpha=6, precision=precision)


@pytest.mark.parametrize("precision,tol", FORMS)
def test_repulsion_kernel_alpha12(precision, tol):
    """The 1/r^12 series (App. A, C1 construction for 1/r^12 at b = 2,
    mellin factor 3840) through the same kernels: a water box with one
    coefficient per site kind (close intramolecular pairs dominate) and random
    positive coefficients in a cube; against the oracle's 1/r^12 series with
    the plan's parameters."""
    f = _form(precision)
    n_mol = 600
    L = (n_mol / synth.WATER_DENSITY) ** (1 / 3)
    xyz, _, box = synth.water_box(n_mol=n_mol, L=L, seed=68)
    c = np.tile(np.array([1.0, 0.1, 0.1], np.float32), n_mol)
    g = int(np.ceil(L))
    _, _, _, _, info = compare("water600/r^-12/" + f, xyz, c, box, 9.0, (g, g, g), tol[0], tol[1],
                               alpha=12, precision=precision)
    assert info["n_terms"] >= 1
    rng = np.random.default_rng(69)
    xyz = rng.uniform(0, 22.0, (700, 3)).astype(np.float32)
    c = rng.uniform(0.2, 1.5, 700).astype(np.float32)
    compare("random700/r^-12/" + f, xyz, c, (22.0, 22.0, 22.0), 8.5, (24, 24, 24), tol[0], tol[1],
            alpha=12, precision=precision)


@pytest.mark.parametrize("alpha", [6, 12])
def test_power_kernels_in_a_non_cubic_cell(alpha):
    """1/r^6 and 1/r^12 (App. A) in a 22 x 24 x 26 A cell: the three axes
    have different fixed-point scales, so the pair kernel scales each
    distance component to A with its own hi/lo scale pair (the cubic path
    keeps them in units); random positive coefficients, both forms, against
    the oracle."""
    rng = np.random.default_rng(70 + alpha)
    box = (22.0, 24.0, 26.0)
    xyz = (rng.uniform(0, 1, (900, 3)) * np.array(box)).astype(np.float32)
    c = rng.uniform(0.2, 1.5, 900).astype(np.float32)
    for precision, tol in FORMS:
        compare("noncubic900/r^-%d/%s" % (alpha, _form(precision)), xyz, c, box, 9.0, (24, 24, 27),
                tol[0], tol[1], alpha=alpha, precision=precision)


def test_repulsion_lattice_forces_vanish():
    """Identical coefficients on a simple-cubic lattice (64 sites, spacing
    2 A): the 1/r^12 forces vanish by symmetry and the energy matches the
    oracle's."""
    g = np.arange(8) * 2.0
    xyz = np.stack(np.meshgrid(g, g, g, indexing="ij"), -1).reshape(-1, 3).astype(np.float32)
    c = np.ones(len(xyz), np.float32)
    box = (16.0, 16.0, 16.0)
    log("case sc512/r^-12")
    gp, gf, info = gpu_eval(xyz, c, box, 7.9, (16, 16, 16), alpha=12)
    op, of = oracle_eval(xyz, c, box, info, 7.9, alpha=12)
    de = abs(gp[4] - op["total"]) / abs(op["total"])
    fpair = 12.0 / 2.0 ** 13
    log("   E_gpu=%.12g E_oracle=%.12g dE=%.2e max|F_gpu|=%.2e max|F_oracle|=%.2e (pair %.2e)"
        % (gp[4], op["total"], de, np.max(np.abs(gf)), np.max(np.abs(of)), fpair))
    assert de <= 1e-6
    assert np.max(np.abs(of)) < 1e-12 * fpair
    assert np.max(np.abs(gf)) < 1e-5 * fpair


def test_dispersion_lattice_forces_vanish():
    """Identical coefficients on a simple-cubic lattice (64 sites, spacing
    4 A): the 1/r^6 forces vanish by symmetry and the energy matches the
    oracle's."""
    g = np.arange(4) * 4.0
    xyz = np.stack(np.meshgrid(g, g, g, indexing="ij"), -1).reshape(-1, 3).astype(np.float32)
    c = np.ones(len(xyz), np.float32)
    box = (16.0, 16.0, 16.0)
    log("case sc64/r^-6")
    gp, gf, info = gpu_eval(xyz, c, box, 7.9, (16, 16, 16), alpha=6)
    op, of = oracle_eval(xyz, c, box, info, 7.9, alpha=6)
    de = abs(gp[4] - op["total"]) / abs(op["total"])
    # a typical pair force at the lattice spacing, for scale
    fpair = 6.0 / 4.0 ** 7
    log("   E_gpu=%.12g E_oracle=%.12g dE=%.2e max|F_gpu|=%.2e max|F_oracle|=%.2e (pair %.2e)"
        % (gp[4], op["total"], de, np.max(np.abs(gf)), np.max(np.abs(of)), fpair))
    assert de <= 1e-6
    assert np.max(np.abs(of)) < 1e-12 * fpair
    assert np.max(np.abs(gf)) < 1e-5 * fpair


@pytest.mark.parametrize("precision,tol", FORMS)
def test_spectral_wide_terms(precision, tol):
    """The widest far terms applied together in spectral form (a low-rank form
    of their circulants: the real Fourier modes each needs down to 1e-9 of its
    first mode), against the oracle's exact image sums: a 30 A water box at
    b = 2 (N = 3, the two widest spectral), the same with N = 8 terms, and
    Table 1 row 3 (N = 15, the eight widest spectral).  The spectral and
    dense forms of one plan agree to the truncation (1e-9) plus FP32
    rounding."""
    f = _form(precision)
    xyz, q, box = synth.water_box(None, 30.0, seed=24)
    for nt in (0, 8):
        _, gf, _, of, info = compare("wide30/spectral/N%d/%s" % (nt, f), xyz, q, box, 9.0,
                                     (30, 30, 30), tol[0], tol[1], n_terms=nt, spectral=1,
                                     precision=precision)
        assert info["n_terms_spectral"] >= 2, info
        assert info["n_terms_grid"] - info["n_terms_spectral"] >= 1
        gd, fd, infod = gpu_eval(xyz, q, box, 9.0, (30, 30, 30), n_terms=nt, spectral=0,
                                 precision=precision)
        log("   spectral %d of %d grid terms, ranks %s; vs the dense form: dF=%.2e"
            % (info["n_terms_spectral"], info["n_terms_grid"], info["spectral_rank"],
               rel_rms(gf, fd)))
        assert rel_rms(gf, fd) < (2e-6 if not precision else 1e-4)
    n_mol = 600
    L = (n_mol / synth.WATER_DENSITY) ** (1 / 3)
    xyz, q, box = synth.water_box(n_mol=n_mol, L=L, seed=313)
    _, _, _, _, info = compare("water600/T1r3/spectral/" + f, xyz, q, box, 9.0, (33, 33, 33),
                               tol[0], tol[1], construction=USERIES_TABLE1_ROW3, spectral=1,
                               precision=precision)
    assert info["n_terms_spectral"] >= 2, info
