"""The profile summariser's reading of kernel names (no GPU needed)."""

import pytest

import bench

NAMES = [
    ("void hu::k_cols_bin<128, 1, 0, true, true>(hu::BinArgs)", "cols_bin", "2D 128^2"),
    ("void hu::k_cols_bin<96, 0, 0, true, false>(hu::BinArgs)", "cols_bin", "3D 96^3"),
    ("void hu::k_cols_filter<64, 3, 0, 0, 0, false>(hu::FilterArgs)", "cols_filter", "3D 64^3"),
    ("void hu::k_cols<256, true, 0, 0>(hu::ColsArgs)", "cols_y_inv", "3D 256^3"),
    ("void hu::k_rows_r2c<512, 0, true, 0>(hu::RowsArgs)", "rows_r2c_noise", "2D 1024^2"),
    ("void hu::k_rows_c2r<64, true, false, 0, 0>(hu::RowsZArgs)", "rows_c2r_thresh", "3D 128^3"),
    ("void hu::k_plane_inv<64, 128, true>(hu::RowsZArgs)", "plane_inv_thresh", "3D 128^3"),
    ("void hu::k_field_lds<64, 128, true>(hu::SmallArgs)", "field_lds", "2D 128^2"),
    ("void hu::k_amp<2, true>(hu::AmpArgs)", "amp", None),
    ("hu::k_finalize(hu::FinalizeArgs)", "finalize", None),
    ("void at::native::vectorized_elementwise_kernel<4>()", None, None),
]


@pytest.mark.parametrize("name,family,shape", NAMES)
def test_family_and_shape_class(name, family, shape):
    assert bench.kernel_family(name) == family
    assert bench.kernel_shape_class(name) == shape


def test_the_binning_kernel_has_the_arguments_that_the_names_are_read_by():
    # k_cols_bin<length, width, radix, exchange, angular>
    import os
    import re
    src = open(os.path.join(bench.ROOT, "paper_2509_08675_amd", "csrc", "hu_bin.hip")).read()
    args = re.search(r"template <([^>]*)>\s*__global__", src).group(1)
    assert [a.split()[-1] for a in args.split(",")] == ["L", "V", "RV", "SPLIT", "ANG"]
