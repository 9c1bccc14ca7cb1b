"""The bench's roofline entries of the ILU(0) sweeps: the bytes of a whole sweep
over the time of all its launches, whatever the number of phases, and not
counted by the prolongations of single solves, which are one more than the
sweeps in a solve that converges inside a cycle."""
import pytest

import bench


@pytest.mark.parametrize("phases", [1, 2])
@pytest.mark.parametrize("name,whole", [("ilu_lower", "ilu_sum"), ("bilu_upper", "bprolong")])
def test_sweep_entry_counts_whole_sweeps(name, whole, phases):
    sweeps, ms = 30, 6.0
    stats = {name: (ms, phases * sweeps), whole: (1.0, sweeps), "prolong": (1.0, sweeps + 1)}
    e = bench.hbm_entry(name, stats, 1e9, "none")
    assert e["achieved"] == pytest.approx(sweeps * 1e9 / (ms * 1e-3) / 1e9)
