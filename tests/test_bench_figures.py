"""The counter figures that bench.py reports beside its times are those of the
summarised profiles, and every form's kernel has its own: bytes per launch are
the calibrated reads and writes of profiles/bns1e4_hbm_counters.md, VALU
instructions those of profiles/bns1e4_flop_counters.md (both written to three
digits and more: 0.5 %)."""
import os
import re

import bench

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ROWS = {
    "items_kernel<tidal,rot>": ("`items_kernel` FP64", "bns1e4 plan", "`items_kernel` FP64, bns1e4"),
    "items_kernel<tidal,rot,mixed>": ("`items_kernel` mixed", "bns1e4 plan", "`items_kernel` mixed, bns1e4"),
    "items_kernel<tidal,rot,parts>": ("`items_kernel` FP64", "bns1e4 plain", "`items_kernel`, plain form of bns1e4"),
    "waveform_kernel<rot,tidal>": ("`waveform_kernel` FP64", "bns1e4 strain", None),
    "waveform_kernel<rot,tidal,mixed>": ("`waveform_kernel` mixed", "bns1e4 strain", None),
    "waveform_deriv_kernel<rot,tidal>": ("`waveform_deriv_kernel`", "first 10^3", None),
}


def _rows(name):
    with open(os.path.join(ROOT, "profiles", name)) as f:
        return [[c.strip() for c in line.strip().strip("|").split("|")] for line in f if line.startswith("|")]


def test_traffic_and_instructions_are_the_profiles():
    hbm, flops = _rows("bns1e4_hbm_counters.md"), _rows("bns1e4_flop_counters.md")
    assert set(bench.MEASURED_TRAFFIC) == set(ROWS)
    for key, (kernel, workload, counters) in ROWS.items():
        r = [r for r in hbm if r[0] == kernel and r[1].startswith(workload)]
        assert len(r) == 1, key
        want = 1e6 * (float(r[0][2]) + float(r[0][3]))
        assert abs(bench.MEASURED_TRAFFIC[key] / want - 1.0) < 5e-3, (key, want)
        if counters:
            v = [r for r in flops if r[0] == counters]
            assert len(v) == 1 and abs(bench.MEASURED_VALU_INSTS[key] / float(v[0][1]) - 1.0) < 5e-3, key
    assert set(bench.MEASURED_VALU_INSTS) <= set(ROWS)


def test_the_plain_form_names_the_kernel_it_runs():
    with open(os.path.join(ROOT, "bench.py")) as f:
        src = f.read()
    cand = dict(re.findall(r'\("(plain_fp64|batched_fp64|batched_mixed)", \w+, "([^"]+)"', src))
    assert cand == {"plain_fp64": "items_kernel<tidal,rot,parts>", "batched_fp64": "items_kernel<tidal,rot>",
                    "batched_mixed": "items_kernel<tidal,rot,mixed>"}
    assert "fisher_kernel" not in src
