"""The committed profile of the matrix-core kernel describes the committed kernel, and the bench's
roofline of that kernel is made of bounds that it can reach (no GPU needed)."""
import bench
from paper_1802_03972_amd.build import MATRIX_FILES, source_sha256
from tests.test_profiles import machine_lines


def test_matrix_profile_matches_sources():
    vals = machine_lines(bench.MATRIX_PROFILE)
    assert vals["kernel_source_sha256"] == source_sha256(MATRIX_FILES)
    got = bench.profile_values(bench.MATRIX_PROFILE, bench.MATRIX_TILE, MATRIX_FILES)
    # a wave of 64 lanes takes 6 matrix instructions of 32 x 32 x 16 for each 16 particles x 256 frequencies
    assert abs(got["mfma_instructions_per_update"] - 6 * 64 / (16 * 256)) < 1e-3
    assert 1.0 < got["valu_instructions_per_update"] < 4.0


def test_matrix_roofline_fractions():
    """At the profiled rate (1.2e13 updates/s) both fractions are below one."""
    r = bench.matrix_roofline(1.2e13 * 5e-3, 5.0)
    assert r["bound"] == "matrix" and 0.1 < r["frac"] < 1.0
    assert r["valu"]["bound"] == "valu issue" and 0.1 < r["valu"]["frac"] < 1.0
