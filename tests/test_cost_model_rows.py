"""The committed cost model was fitted to the planner's present work features: the
features stored with its measured builds are what the planner computes now, and its
coefficients are the fit of its rows (no GPU)."""
import json
import os

import numpy as np
import pytest

import paper_2102_02989_amd as P
import synth
from paper_2102_02989_amd import fit_cost_model

MODEL = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2102_02989_amd", "data",
                     "cost_model.json")
MAKERS = {"C1": synth.config1, "C2": synth.config2, "C3": synth.config3, "C5": synth.config5,
          "tiny 2x2x2": lambda: synth.tiny_problem(kmesh=(2, 2, 2), omega=0.5, diffuse=False)}


@pytest.mark.parametrize("workload,most", [("C1", 17), ("tiny 2x2x2", 17), ("C2", 4), ("C3", 2), ("C5", 2)])
def test_rows_have_the_present_features(workload, most):
    rows = [r for r in json.load(open(MODEL))["rows"] if r["workload"] == workload]
    assert rows
    p = MAKERS[workload]()
    for r in rows[::max(1, len(rows) // most)][:most]:
        f = P.plan_features(p.cell, p.basis, p.aux, p.kmesh, r["omega"], p.thresh, p.g_thr, alpha_cut=r["alpha_cut"])
        assert np.allclose(f, r["features"], rtol=1e-9), (workload, r["omega"], r["alpha_cut"])


@pytest.mark.parametrize("form", ["fp64", "fp32"])
def test_coefficients_are_the_fit_of_the_rows(form):
    m = json.load(open(MODEL))
    coef, worst = fit_cost_model.fit(m["rows"], form)
    F = np.array([r["features"] for r in m["rows"]])
    assert np.allclose(F @ coef, F @ np.array(m[f"coef_{form}"]), rtol=1e-6)
    assert worst == pytest.approx(m[f"max_rel_err_{form}"], rel=1e-6)
