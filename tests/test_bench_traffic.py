"""bench.py's HBM bytes per screened round from profiler counters: the rounds
are counted right whichever way they were screened (synthetic counter files)."""
import csv
import os

import pytest

import bench

SCREEN = "void iso::(anonymous namespace)::k_screen_pairs<1, %s, %d, false>(iso::ScreenArgs, HIP_vector_type<int, 2u> const*)"
RECHECK = "void iso::(anonymous namespace)::k_recheck_rows<false>(float const*)"
FINAL = "void iso::(anonymous namespace)::k_fr_recheck<false>(float const*)"
PLAIN = [SCREEN % ("false", 0), SCREEN % ("true", 0)]
SAMPLE = [SCREEN % ("true", 0)] * 4
LIST = [SCREEN % ("false", 1), SCREEN % ("true", 1), SCREEN % ("false", 1)]
END = [SCREEN % ("false", 2), FINAL]

# name: (dispatches, screened rounds)
CASES = {
    "lists-from-the-first-round": (SAMPLE + LIST + [RECHECK, RECHECK] + END, 2),
    "lists-from-the-second-round": (PLAIN + PLAIN + [RECHECK] + LIST + [RECHECK, RECHECK] + END, 3),
    "sample-without-lists": (SAMPLE + PLAIN + [RECHECK] + LIST + [RECHECK] + END, 3),
    "every-round-screened": ((PLAIN + [RECHECK]) * 5, 5),
    "two-calls": ((SAMPLE + LIST + [RECHECK, RECHECK] + END) * 2, 4),
}


@pytest.mark.parametrize("name", list(CASES))
def test_rounds_of_a_traffic_report(tmp_path, name):
    dispatches, rounds = CASES[name]
    mib = 64
    for counter in ("FETCH_SIZE", "WRITE_SIZE"):
        d = tmp_path / counter / "host"
        os.makedirs(d)
        with open(d / "run_counter_collection.csv", "w", newline="") as f:
            w = csv.writer(f)
            w.writerow(["Dispatch_Id", "Kernel_Name", "Counter_Name", "Counter_Value"])
            w.writerow([1, "__amd_rocclr_copyBuffer", counter, mib * 1024])
            for q, kernel in enumerate(dispatches):
                w.writerow([2 + q, kernel, counter, 100 if "k_screen" in kernel else 7])
    rec = bench.traffic_report(str(tmp_path / "FETCH_SIZE"), str(tmp_path / "WRITE_SIZE"), "bf16", mib)
    screens = sum("k_screen" in k for k in dispatches)
    assert rec["launches"] == rounds
    assert rec["fetch_bytes_per_launch"] == pytest.approx(screens * 100 * 1024 / rounds)
