"""Calls at the edges of what the entry points take."""
import numpy as np
import pytest

from paper_2112_03804_amd import instances as I

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _game(d):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2112_03804_amd import pmx
    return pmx.Game(d)


# entries past a row's hands are ignored on input and written as 0 on output:
# a plan loaded with anything there leaves no trace in the averages
@pytest.mark.parametrize("steps", [1, 3, 40])
@pytest.mark.parametrize("kind", ["rm+", "dcfr"])
def test_padding_of_a_loaded_plan(kind, steps):
    descs = [I.river_config(seed=4, n_keep=(33, 21), max_raises=1), I.small_river(0)]
    clean, dirty = _game(descs), _game(descs)
    for g in (clean, dirty):
        g.solver_set_params(kind)
        g.solver_step(5)
    torch.cuda.synchronize()
    pads = []
    for p in range(2):
        pad = np.ones(clean.elems[p], bool)
        for L in (l[p] for l in clean.layouts):
            rows = pad[L["vec_offset"]:L["vec_offset"] + L["n_seq"] * L["stride"]].reshape(L["n_seq"], L["stride"])
            rows[:, :L["n_hands"]] = False
        assert pad.any()
        pads.append(pad)
        st = clean.solver_get_state(p)
        for g, fill in ((clean, 0.0), (dirty, np.nan)):
            plan = st["plan"].copy()
            plan[pad] = fill
            g.solver_set_state(p, regret=st["regret"], plan=plan, avg_sum=st["avg_sum"], t=5, wsum=st["wsum"])
    for g in (clean, dirty):
        g.solver_step(steps)
    torch.cuda.synchronize()
    for p in range(2):
        a, b = clean.get_average_strategy(p), dirty.get_average_strategy(p)
        assert (a[pads[p]] == 0).all() and np.array_equal(a, b)
        s, t = clean.solver_get_state(p), dirty.solver_get_state(p)
        for k in ("regret", "plan", "avg_sum"):
            assert np.array_equal(s[k][~pads[p]], t[k][~pads[p]]), (p, k)
    assert np.array_equal(clean.saddle_gap()[0], dirty.saddle_gap()[0])
