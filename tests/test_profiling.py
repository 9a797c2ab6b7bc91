"""The counter summaries of paper_2512_08478_amd.profiling."""
from paper_2512_08478_amd import profiling


def test_calibration_is_the_copys_not_a_larger_fills():
    """A 256 MiB copy calibrates the counters, also where the process fills a
    1 GiB buffer too (with the fill's reading, written bytes came out a quarter
    of what they are)."""
    copy, fill = 256 * 1024.0, 1024 * 1024.0
    disp = {"1": ("elementwise_kernel<copy>", 1, copy), "2": ("k_raster<32, 16>", 1, 5e6),
            "3": ("vectorized_elementwise_kernel<FillFunctor>", 1, fill),
            "4": ("vectorized_elementwise_kernel<Mul>", 1, 1000.0)}
    assert profiling._calibration(disp, 256)[0] == 1.0
    disp["1"] = (disp["1"][0], 1, copy / 2)  # a counter of half the bytes
    assert profiling._calibration(disp, 256)[0] == 2.0
