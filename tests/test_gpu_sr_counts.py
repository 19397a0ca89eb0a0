"""The short range's work counters: every contraction that a lane performs is
counted, so none stands for more than the 12 lattice vectors that a lane holds, and
the terms do not depend on how the items are split over waves and lanes."""
import os

import numpy as np
import pytest

import oracle
import synth
from gpu_util import run_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kmesh,omega", [((1, 1, 1), 0.3), ((1, 3, 2), 0.5)])
def test_contractions_are_counted(kmesh, omega, tmp_path, monkeypatch):
    p = synth.tiny_problem(kmesh=kmesh, omega=omega, seed=11, diffuse=False)
    terms = {}
    for split in (1e3, 1.0, 0.02):
        print("case SR counts", kmesh, omega, split, flush=True)
        f = str(tmp_path / f"counts_{split}")
        monkeypatch.setitem(os.environ, "RSGDF_COUNTS_FILE", f)
        _, st = run_gpu(p, parts=oracle.PART_SR, sr_split=np.full(24, split, np.float32))
        monkeypatch.delitem(os.environ, "RSGDF_COUNTS_FILE")
        c = np.loadtxt(f)  # aux, pair, l_P, l_a, l_b, terms, contractions, shell terms, R_c
        nt, nc = c[:, 5], c[:, 6]
        print(f"  terms {nt.sum():.0f}, contractions {nc.sum():.0f}, most terms of one {(nt / np.maximum(nc, 1)).max():.1f}",
              flush=True)
        assert nt.sum() == st["n_sr_terms"] > 0
        assert np.all(nc <= nt) and np.all(nt <= 12 * nc)
        terms[split] = nt.tolist()
    assert terms[1e3] == terms[1.0] == terms[0.02]
