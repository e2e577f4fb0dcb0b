"""Calls whose binning emits entries and sorts them (imported by test modules): the
recording runtime names their kernels (test_launch_routes.py) and the GPU runs them
(test_gpu_sorted_binning.py).  name: (view sizes, same camera, n3, n4, tile, batched,
pair capacity, kernels)."""
CALLS = {
    # 6,600 super-tiles: two radix passes; 540,000 depth-ordered entries: 2,110 count workgroups
    "scanned counts": ([(2100, 1600)] * 2, False, 200_000, 70_000, 8, 1, 1 << 24,
                       ("k_coarse_top", "k_coarse_down", "k_radix_downsweep", "k_ranges")),
    "one view": ([(2100, 1600)], False, 200_000, 70_000, 8, 0, 1 << 24,
                 ("k_coarse_down_direct", "k_radix_downsweep", "k_ranges")),
    "shared static": ([(2100, 1600)] * 3, True, 14_000, 6_000, 8, 1, 1 << 24,
                      ("k_coarse_down_direct", "k_radix_downsweep", "k_ranges")),
    # 1,900 super-tiles in one 11-bit pass, whose digit runs are the lists' ranges: the
    # capacity is too small for the ranked binning's histograms
    "single pass": ([(1600, 1200)], False, 36_000, 24_000, 8, 0, 16 * 40_000,
                    ("k_coarse_down_direct", "k_radix_downsweep")),
    # and in one call with a view of two 6-bit passes, the histogram sized for the wider digit
    "digit widths": ([(2100, 1600), (1600, 1200)], False, 36_000, 24_000, 8, 0, 16 * 40_000,
                     ("k_coarse_down_direct", "k_radix_downsweep", "k_ranges")),
}
