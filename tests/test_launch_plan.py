"""The launches that the library plans for a push (rad_debug_plan: host only, no GPU needed)."""
import ctypes

import numpy as np
import pytest

from paper_1802_03972_amd import _lib
from workloads import block_log_omegas

DP = ctypes.POINTER(ctypes.c_double)
CUS = 256
FIXED, FLEXIBLE, MATRIX = 0, 1, 2


def plan(n_dir, n_omega, n, kind="uniform", shape="cic", tile=None, omega_max=1e19, shape_len=1e-7, cus=CUS):
    th = np.linspace(-0.02, 0.02, n_dir)
    dirs = np.ascontiguousarray(np.stack([th, np.zeros(n_dir), np.sqrt(1.0 - th ** 2)], axis=1))
    om = {"uniform": None, "log": np.geomspace(1e15, omega_max, n_omega),
          "blocks": block_log_omegas(1e15, omega_max, n_omega)}[kind]
    d = _lib.GridDesc(n_dir, dirs.ctypes.data_as(DP), 0.0, omega_max / max(1, n_omega - 1), n_omega, _lib.SHAPES[shape],
                      shape_len, 5e-17, 0, 0, None if om is None else om.ctypes.data_as(DP))
    out = (_lib.DebugLaunch * 64)()
    count = ctypes.c_int32()
    t = None if tile is None else ctypes.byref(_lib.Tile(*tile))
    _lib.check(_lib.lib().rad_debug_plan(ctypes.byref(d), t, cus, n, out, len(out), ctypes.byref(count)))
    assert count.value <= len(out)
    return out[:count.value]


@pytest.mark.parametrize("kind", ["uniform", "log", "blocks"])
@pytest.mark.parametrize("n_dir", [1, 2, 3, 5, 7, 8, 9, 11, 13, 15])
def test_flexible_lds(n_dir, kind):
    """The flexible build's LDS: its table of weights is read 16 bytes at a time, so it starts on
    16 bytes for odd chunks of an odd number of directions too; a chunk fits the staging arrays, and two
    workgroups fit a CU's 160 KB."""
    odd = 0
    for n_omega in [16, 100, 241, 300, 529, 540, 600, 700, 800, 1000, 1024]:
        for n in [1, 37, 333, 1000, 5003, 27 * 512, 50001, 200003]:
            for l in plan(n_dir, n_omega, n, kind):
                if l.kernel != FLEXIBLE:
                    continue
                odd += l.chunk * n_dir % 2
                assert l.weights_at % 16 == 0, (n_omega, n, l.chunk)
                assert l.chunk <= 128 and 2 * l.lds_bytes <= 160 * 1024
    if n_dir in (7, 9, 11, 13, 15):      # the odd chunks that this is about
        assert odd > 0


TILE = (16, 32, 4, 3)


@pytest.mark.parametrize("shape", ["point", "gauss", "cic"])
@pytest.mark.parametrize("n_dir,n_omega", [(1, 1000), (8, 256), (36, 100), (64, 1024), (128, 300)])
def test_a_set_tile_takes_the_whole_grid(n_dir, n_omega, shape):
    """A launch shape that the caller sets is the one that every push runs, for all frequencies, also
    on grids that would otherwise go to the matrix cores in part or in whole."""
    for n in [1000, 200000]:
        for l in plan(n_dir, n_omega, n, shape=shape, tile=TILE):
            assert l.kernel != MATRIX and (l.k0, l.n_omega) == (0, n_omega)
            assert tuple(getattr(l.tile, k) for k, _ in _lib.Tile._fields_) == TILE
    free = plan(n_dir, n_omega, 200000, shape=shape)
    assert any(l.kernel == MATRIX for l in free) == (shape != "cic")


def test_a_gaussian_in_two_parts_covers_every_frequency():
    """More than four frequencies before the constant: the general kernel takes whole blocks of 16."""
    parts = plan(16, 600, 1000, shape="gauss", omega_max=2e18)
    assert [l.kernel for l in parts][-1] == MATRIX and len(parts) == 2
    assert parts[0].k0 == 0 and parts[0].n_omega == parts[1].k0 and parts[1].k0 % 16 == 0
    assert parts[1].k0 + parts[1].n_omega == 600


@pytest.mark.parametrize("kind", ["uniform", "log", "blocks"])
@pytest.mark.parametrize("n_dir,n_omega", [(1, 1000), (3, 100), (5, 800), (7, 1024), (11, 300), (11, 529), (15, 540), (15, 1000),
                                           (16, 64), (37, 100), (128, 256)])
def test_small_pushes_do_not_split_to_single_particles(n_dir, n_omega, kind):
    """Each split writes a whole partial tile that the fold reads: at least 8 particles each once there
    are 32 splits, and all particles are in one of them."""
    for n in [1, 2, 15, 31, 32, 33, 64, 255, 256, 257, 600, 1500, 4000, 4097, 50000]:
        for l in plan(n_dir, n_omega, n, kind):
            assert (l.splits - 1) * l.per_split < n <= l.splits * l.per_split
            assert l.splits <= 32 or l.per_split >= 8, (n, l.splits, l.per_split)


# tiles (directions, waves) that were measured 1.03 to 1.77 times slower than the best on these grids
@pytest.mark.parametrize("n_dir,n_omega,kind,shape,slow", [
    (128, 96, "uniform", "cic", (64, 6)), (128, 300, "uniform", "cic", (32, 5)), (64, 786, "uniform", "cic", (32, 5)),
    (56, 440, "log", "cic", (32, 5)), (32, 267, "blocks", "cic", (32, 5)), (64, 784, "uniform", "cic3d", (32, 5)),
    (64, 830, "log", "cic", (64, 6)), (20, 418, "uniform", "cic3d", (32, 5))])
def test_default_tiles(n_dir, n_omega, kind, shape, slow):
    l, = plan(n_dir, n_omega, 1000000, kind, shape)
    assert l.kernel == FIXED
    assert (l.tile.dir_per_wave, l.tile.waves) != slow


@pytest.mark.parametrize("shape", ["cic", "cic3d"])
@pytest.mark.parametrize("n_dir,n_omega", [(16, 64), (37, 100), (44, 34), (128, 256), (88, 200), (64, 123)])
def test_small_pushes_fill_the_chip(n_dir, n_omega, shape):
    """Splits of fewer than 32 particles: never more of them than the tile asks for, and never so few
    that half of the chip's compute units stand idle where splits of 8 particles would fill them."""
    for n in [300, 1000, 1024, 5003, 9660, 16000, 32769]:
        l, = plan(n_dir, n_omega, n, shape=shape)
        tiles = -(-n_dir // l.tile.dir_per_wave) * -(-n_omega // (64 // l.tile.dir_per_wave * 16 * l.tile.waves))
        assert l.splits * tiles <= CUS * l.tile.wg_per_cu
        most = min(-(-n // 8), CUS * l.tile.wg_per_cu // tiles)
        assert l.per_split > 32 or l.splits * tiles >= min(CUS // 2, most * tiles), (n, l.splits, l.per_split)


@pytest.mark.parametrize("kind,shape", [("log", "cic"), ("uniform", "cic3d"), ("log", "cic3d")])
def test_default_tiles_of_the_other_kernels(kind, shape):
    """Of the kernels that three waves of share a SIMD, five to eight waves of a workgroup cost the
    same, so no tile of five to seven is taken where it needs as many workgroups as one of eight."""
    for n_dir in [16, 20, 37, 64, 100, 128]:
        for n_omega in [80, 150, 272, 300, 440, 580, 786, 1000]:
            l, = plan(n_dir, n_omega, 1000000, kind, shape)
            per = (64 // l.tile.dir_per_wave) * 16
            assert l.tile.waves <= 4 or -(-n_omega // (per * l.tile.waves)) == -(-n_omega // (per * 8)), (n_dir, n_omega)
