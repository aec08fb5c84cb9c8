"""bench.py's split of a hoisted rotation's time names the kernel classes that ran, and all of them."""
import bench


def test_split_lists_what_ran():
    prof = {"ntt_fwd_lo": {"ms": 2.0, "launches": 16, "bytes": 8e9, "ops": 1.0}, "ntt_fwd_hi": {"ms": 1.0, "launches": 9, "bytes": 3e9, "ops": 1.0}}
    s = bench.rotation_split(prof, 64)
    assert s["us_per_rotation"] == {"ntt_fwd_lo": 31.25, "ntt_fwd_hi": 15.625}
    assert s["GBs"] == {"ntt_fwd_lo": 4000.0, "ntt_fwd_hi": 3000.0}
    assert s["launches"] == {"ntt_fwd_lo": 16, "ntt_fwd_hi": 9}
