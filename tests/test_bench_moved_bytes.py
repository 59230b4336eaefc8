"""The bytes and operations that the benchmark's rates divide by
(bench.moved_bytes_per_point, bench.sphere_issued_flops): the fields that the
passes store (nine FMT spectra on the z side of the y passes, seven on the x
side) and the operations of the folded sphere columns."""
import pytest

import bench

MIXED, FP64 = 1, 0


def test_pass_tables_three_species():
    got = bench.moved_bytes_per_point(3, MIXED)
    assert got == {"z_fwd_rho": 36, "y_fwd_rho": 24, "x_fwd_weights": 40, "y_inv_n": 64, "z_deriv": 72,
                   "y_fwd_dphi": 64, "x_back_pairs": 52, "y_inv_mu": 24, "z_inv_final": 60}
    assert sum(got.values()) == 436
    assert sum(bench.moved_bytes_per_point(3, FP64).values()) == 800


@pytest.mark.parametrize("S", [1, 3, 4])
@pytest.mark.parametrize("precision,c", [(MIXED, 4), (FP64, 8)])
def test_one_field_less_than_the_yardstick(S, precision, c):
    moved, yard = bench.moved_bytes_per_point(S, precision), bench.pass_bytes_per_point(S, precision)
    assert sum(yard.values()) - sum(moved.values()) == 8 * c
    assert sum(bench.moved_bytes_per_point(S, precision, slot=False).values()) == sum(moved.values()) - 8 * S


def test_kernels_store_as_many_fields():
    """The slots and counts in the kernels' header are those of the byte model."""
    import os
    import re
    src = open(os.path.join(bench.ROOT, "paper_1407_0674_amd", "csrc", "pnp_kernels.hpp")).read()
    assert int(re.search(r"constexpr int kBackFields = (\d+);", src).group(1)) == 7
    x, stride = (int(re.search(rf"{k} = (\d+)", src).group(1)) for k in ("kSlotX", "kVecStride"))
    assert x + 2 + stride == 9  # the slots below n_2v,z, which has no spectrum


def test_sphere_operations_of_a_small_rule():
    # r = 1/2, order 2: four nodes at (+-a, 0, +-b) (theta 0 and pi), a = sin, b = |cos| of
    # phi = pi (1 - 1/sqrt 3) / 2, half a cell off the axes in x and z at most: offsets
    # -1, 0, 1 in x and z, 0 in y; columns dz = 0 and |dz| = 1 with dx = 0 and +-1 each
    fold = (8 + 2) / 8  # planes read per output
    assert bench.sphere_issued_flops(0.5, 2, 8, fp32=False) == pytest.approx((2 + 6) + (4 + 9) + 2 * fold)
    assert bench.sphere_issued_flops(0.5, 2, 8) == pytest.approx((2 + 6) + (4 + 11) + 5 * fold)


@pytest.mark.parametrize("r,k,cubic", [(1.5, 8, False), (3.0, 8, False), (2.2, 6, True)])
def test_sphere_operations_below_the_unfolded_count(r, k, cubic):
    unfolded = 8.0 * bench.sphere_stencil_size(r, k, cubic)
    assert 0.2 * unfolded < bench.sphere_issued_flops(r, k, 8, cubic) < unfolded
    # thinner columns share the folding among fewer outputs
    assert bench.sphere_issued_flops(r, k, 2, cubic) > bench.sphere_issued_flops(r, k, 8, cubic)
