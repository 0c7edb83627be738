"""The shipped cache of launch choices: an entry spells out the choices its
search found best, also where they are the library's defaults, so that the
parity tests of the full workloads run what a graph runs."""
import pytest

from paper_2507_00528_amd import nep, tune


@pytest.mark.parametrize("workload", ["c2", "c3", "c4", "l8"])
def test_entry_holds_the_choices_in_full(workload):
    (e,) = [v for v in tune.load_cache().values() if v["workload"] == workload]
    assert set(tune.SPACE) - {"cell_min_atoms"} <= set(e["tuning"]) <= set(tune.SPACE)
    assert all(e["tuning"][k] in tune.SPACE[k] for k in e["tuning"])
    nep.tuning_struct(e["tuning"])
    best = min(r["ms"] for r in e["measurements"] if r["ms"] is not None)
    assert e["ms"] <= best * 1.01 / 0.99      # within the gain a choice has to bring
