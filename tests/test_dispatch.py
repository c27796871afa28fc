"""Layers on which a rule once chose the slower kernel.  Each with the pass, what it has to run on and both times (us); on the CPU, as
descriptors name their kernels without a device."""
import pytest

import paper_1810_02272_amd as conv
from parity_cases import P

CASES = {
    # the launch that clears dx belongs to either kernel's time
    "zero_fill_counts_on_both_sides": [
        (P(12, 125, 56, 56, 27, 1, 7, 3, 3), "f32", "bwd_data", "corr_m", (18.6, 23.0)),
    ],
    # doubles: one launch against the tiles as they are planned, not as the rules would have them (95.6 and 28.5 us)
    "doubles_are_planned_before_they_are_compared": [
        (P(127, 2, 12, 12, 324, 3, 3, 1, 1, 1, 0), "f64", "bwd_data", "corr64_16x64x16[es](S=8,", (52.6, 77.9)),
        (P(9, 54, 19, 24, 91, 8, 8, 4, 4, 0, 1), "f64", "fwd", "corr64_16x64x16[es](S=12,", (19.3, 27.6)),
    ],
    # below 0.7 GFLOP the tiled kernels' time is modelled in their own range: packing and reducing are most of such a pass
    "small_passes_are_modelled_in_their_range": [
        (P(64, 20, 12, 12, 50, 5, 5), "f32", "bwd_data", "corrsmall_32x16x4[w3]", (19.5, 23.7)),
        (P(64, 20, 12, 12, 50, 5, 5), "f32", "fwd", "corrsmall_32x16x4[w0]", (7.0, 14.0)),
        (P(32, 249, 3, 3, 206, 3, 3, 2, 2), "f32", "fwd", "corr_m16_16x64x16", (11.6, 18.7)),
        (P(16, 142, 6, 6, 147, 6, 6, 1, 1, 1, 0), "f32", "fwd", "corr_m32_32x128x16", (23.1, 33.3)),
    ],
    # nothing but the modelled time keeps a size on the tiled kernels: short reductions, few columns, thin rows, few places
    "no_size_is_kept_for_the_tests": [
        (P(64, 1, 28, 28, 20, 5, 5), "f32", "fwd", "corrsmall", (8.0, 8.6)),
        (P(2, 6, 6, 6, 343, 5, 5, 2, 2, 1, 2), "f32", "fwd", "corrsmall", (5.0, 10.4)),
        (P(6, 256, 1, 1, 1, 3, 3, 1, 1, 1, 1), "f32", "bwd_data", "corrsmall", (3.7, 8.3)),
        (P(8, 2, 12, 12, 2, 6, 6, 1, 1, 2, 2), "f32", "fwd", "corrsmall", (4.2, 9.6)),
        (P(21, 4, 1, 25, 1, 3, 7, 1, 1, 1, 2), "f32", "bwd_data", "corrsmall", (3.8, 7.4)),
        (P(4, 47, 3, 3, 3, 3, 3), "f32", "bwd_filter", "smallwgrad", (3.5, 6.2)),
        (P(2, 4, 4, 4, 153, 3, 7, 3, 3, 1, 3), "f64", "fwd", "corrsmall64", (4.2, 9.6)),
        (P(45, 24, 8, 8, 2, 1, 1), "f64", "bwd_data", "corrsmall64", (3.5, 7.4)),
        (P(12, 177, 3, 3, 2, 2, 2), "f64", "bwd_filter", "smallwgrad64", (3.4, 5.7)),
        (P(12, 378, 5, 5, 3, 5, 5, 3, 3, 1, 1), "f64", "bwd_filter", "wgrad64", (5.3, 7.7)),
        (P(5, 88, 3, 3, 39, 11, 11, 1, 1, 5, 5), "f64", "bwd_filter", "wgrad64", (10.5, 15.3)),
    ],
}


@pytest.mark.parametrize("rule", list(CASES))
def test_the_faster_kernel_is_chosen(rule):
    for pd, base, which, prefix, times in CASES[rule]:
        d = conv.conv_desc_create(conv.ConvParams(**pd))
        names = conv.conv_desc_kernel_names(d) if base == "f32" else conv.conv_desc_kernel_names_f64(d)
        got = dict(kv.split("=", 1) for kv in names.split(";"))[which]
        assert got.startswith(prefix), (pd, base, which, got, "should take %.1f us, not %.1f" % times)


def test_one_launch_asks_for_no_partial_sums():
    """Its passes touch no workspace: what is asked for must not hold the slices of a plan that does not run (689 KB and 1.4 MB)."""
    d = conv.conv_desc_create(conv.ConvParams(**P(3, 40, 23, 15, 127, 1, 1, 3, 3)))
    assert all("small" in v for v in conv.conv_desc_kernel_names(d).split(";")[:3])
    assert 0 < conv.conv_desc_workspace_bytes(d) <= 64 << 10 and 0 < conv.conv_desc_workspace_bytes_f64(d) <= 128 << 10
