"""Index arithmetic of the device code, evaluated by the compiler on the host: no GPU, nothing is run."""
import subprocess

from paper_2603_27156_amd import build

PROGRAM = r"""
#include "gsr_internal.h"
#include "gsr_device.h"

// every lane of every round of the edges [e_a, e_b) loads an entry of an array that holds max(e_b, 1) of them; in a range
// that is not empty, one of the range, and every edge is the own edge of exactly one lane
template <int ROUND>
constexpr bool sound(int e_a, int e_b) {
    int eb = e_a;
    do {                               // (the first round is asked for whether there is one or not)
        const int steps = gsr::run_steps<ROUND>(eb, e_b);
        if (steps < 1 || steps > 16 || steps % ROUND) return false;
        int own = 0;
        for (int lane = 0; lane < 64; ++lane) {
            const int e = gsr::run_entry(eb, e_b, steps, lane);
            if (e < 0 || e >= (e_b > 0 ? e_b : 1)) return false;
            if (e_b > e_a && e < e_a) return false;
            const int place = eb + (lane >> 4) * steps + (lane & 15);
            if ((lane & 15) < steps && place < e_b) {
                if (e != place) return false;
                ++own;
            }
        }
        if (own != (e_b - eb < 64 ? e_b - eb : 64)) return false;
        eb += 64;
    } while (eb < e_b);
    return true;
}
template <int ROUND>
constexpr bool all_sound() {
    for (int e_a : {0, 1, 63, 1000})
        for (int len = 0; len <= 130; ++len)
            if (!sound<ROUND>(e_a, e_a + len)) return false;
    return true;
}
static_assert(all_sound<4>() && all_sound<8>(), "a lane of a round loads outside the arrays");
"""


def test_lanes_of_a_round_load_existing_entries_also_in_an_empty_range(tmp_path):
    src = tmp_path / "indexing.hip"
    src.write_text(PROGRAM)
    out = subprocess.run([build._hipcc(), *build.HIPCC_FLAGS, "-fconstexpr-steps=100000000", "--offload-host-only", "-fsyntax-only", str(src)],
                         capture_output=True, text=True)
    assert out.returncode == 0, out.stderr[-2000:]
