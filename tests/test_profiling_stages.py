"""Host logic of the traffic summary: the kernels that make up one execution of
a step stage are added up, and those of other work are left out."""

from paper_2003_03931_amd import profiling


def _rows(*names):
    return [(i + 1, n, float(10 ** (i % 3))) for i, n in enumerate(names)]


def _sum(rows, *at):
    return sum(rows[i][2] for i in at)


def test_large_coarse_solve_is_five_sweeps():
    r = _rows("k_coarse_deposit<16, 512, 1>", "k_fft<512, 0, 0>", "k_fft<512, 1, 0>", "k_fft<512, 2, 2>",
              "k_fft<512, 1, 1>", "k_fft<512, 0, 1>", "k_deposit_zm<32, 4, 512, 2, false, unsigned int, 100, 3072>")
    assert profiling.stage_mean(r, "coarse_fft_green") == _sum(r, 1, 2, 3, 4, 5)


def test_small_coarse_solve_is_three_sweeps_and_the_spectrum_none_of_it():
    r = _rows("k_fft_xy<64, false, false>", "k_fft<64, 2, 2>", "k_fft_xy<64, true, true>",
              "k_deposit<16, true, unsigned int, 216, 4096>", "k_fft<256, 0, 0>", "k_fft<256, 1, 0>",
              "k_fft<256, 2, 0>", "k_power_bins")
    assert profiling.stage_mean(r, "coarse_fft_green") == _sum(r, 0, 1, 2)


def test_scan_holds_the_cell_statistics_and_not_the_sort():
    r = _rows("k_digit_hist", "k_tile_sums", "k_tile_scan<true>", "k_digit_scatter<true>", "k_cell_stats",
              "k_scatter_compressed", "k_gather<0, 2, false, false, 4>", "k_cell_stats", "k_tile_sums",
              "k_tile_scan<true>", "k_tile_scan<false>", "k_decide", "k_compact_brick<4>")
    assert profiling.stage_mean(r, "scan_counts") == _sum(r, 7, 8, 9, 10, 11)


def test_mean_over_executions():
    r = _rows("k_vc_mean", "k_vc_sigma", "k_vc_encode", "k_vc_mean", "k_vc_sigma", "k_vc_encode", "k_r2c_plane_w<160, 0>",
              "k_zconv_half<160, 0>", "k_r2c_plane_w<160, 0>")
    assert profiling.stage_mean(r, "velocity_encode") == _sum(r, 0, 1, 2, 3, 4, 5) / 2
    assert profiling.stage_mean(r, "fine_r2c_xy") == _sum(r, 6, 8) / 2
    assert profiling.stage_mean(r, "pp_force") is None
