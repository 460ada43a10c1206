"""Kernel names of a profile and the launch classes that their traffic is counted with."""
import re

import pytest

from paper_2010_14501_amd import profsum

ANON = "void monet::(anonymous namespace)::"


@pytest.mark.parametrize("name, label", [
    (ANON + "conv_tile_kernel<0, 2, 4, 1, 0, 1>(monet::(anonymous namespace)::TileArgs)", "conv_fwd"),
    (ANON + "conv_tile_kernel<2, 2, 4, 1, 3, 1>(monet::(anonymous namespace)::TileArgs)", "conv_wgrad_winograd"),
    (ANON + "rows32::conv_short_kernel<0>(monet::(anonymous namespace)::TileArgs)", "conv_fwd"),
    (ANON + "rows64::conv_short_kernel<1>(monet::(anonymous namespace)::TileArgs)", "conv_dgrad"),
    (ANON + "rows32::conv_short_kernel<2>(monet::(anonymous namespace)::TileArgs)", "conv_wgrad"),
    (ANON + "stem7_fwd_kernel(float const*, float const*, float*, monet::(anonymous namespace)::Stem7Geom)", "conv_fwd"),
    (ANON + "stem_fwd_kernel<7, 7, 2>(float const*, float const*, float*, monet::(anonymous namespace)::StemGeom)", "conv_fwd"),
    (ANON + "stem7_wgrad_kernel<7, 7, 2>(float const*, float const*, float*, monet::(anonymous namespace)::StemGeom)", "conv_wgrad"),
    (ANON + "pw_wgrad_kernel<true, 2>(float const*, float const*, float*, long)", "conv_wgrad"),
    (ANON + "wino4_vertical_kernel(monet::(anonymous namespace)::VerticalArgs)", "conv_wgrad_winograd"),
    (ANON + "wino4_wgrad_kernel(monet::(anonymous namespace)::WgradArgs)", "conv_wgrad_winograd"),
    (ANON + "wino4_pieces_kernel<true, 0>(monet::(anonymous namespace)::PiecesArgs)", "conv_dgrad_winograd"),
    ("void monet::bn_bwd_small<false, 1>(float const*, void const*, float const*)", "bn_bwd"),
])
def test_kernels_are_counted_with_their_launch_class(name, label):
    kernel = profsum.short(name)
    assert [labels[0] for labels, patterns in profsum.GROUPS if any(re.search(p, kernel) for p in patterns)] == [label], kernel
