"""The short range with many lattice vectors per unit (small omega), where a lane's
list takes several passes and the lanes of a unit share it: parity with the oracle, and
the work counters.  Every contraction that is performed is counted: a lane contracts
at most the 64 vectors that its list holds, and in the classes with the most components
((d|dd), (f|dp), (f|dd)) the lanes of a unit are added up first, so that their
contractions stand for many terms.  The terms do not depend on how the items are split."""
import os

import numpy as np
import pytest

import oracle
import synth
from gpu_util import run_gpu

pytestmark = pytest.mark.gpu


def _counted(p, split, tmp_path, monkeypatch, thresh=None):
    f = str(tmp_path / "counts")
    monkeypatch.setitem(os.environ, "RSGDF_COUNTS_FILE", f)
    got, st = run_gpu(p, thresh=thresh, parts=oracle.PART_SR, sr_split=np.full(24, split, np.float32))
    monkeypatch.delitem(os.environ, "RSGDF_COUNTS_FILE")
    c = np.loadtxt(f)  # aux, pair, l_P, l_a, l_b, terms, contractions, shell terms, R_c
    wide = (c[:, 2:5].sum(1) >= 6) & (c[:, 3] == 2) & (c[:, 4] >= 1)
    nt, nc = c[:, 5], c[:, 6]
    print(f"  terms {nt.sum():.0f}, contractions {nc.sum():.0f}, most terms of one {(nt / np.maximum(nc, 1)).max():.1f}, "
          f"wide classes {nt[wide].sum() / max(nc[wide].sum(), 1):.1f}", flush=True)
    assert nt.sum() == st["n_sr_terms"] > 0
    assert np.all(nc <= nt) and np.all(nt[~wide] <= 64 * nc[~wide]) and np.all(nt <= 64 * 64 * nc)
    return got, nt, nc, wide


@pytest.mark.parametrize("kmesh,omega", [((1, 1, 1), 0.3), ((1, 3, 2), 0.5)])
def test_contractions_are_counted(kmesh, omega, tmp_path, monkeypatch):
    p = synth.tiny_problem(kmesh=kmesh, omega=omega, seed=11, diffuse=False)
    terms = {}
    for split in (1e3, 1.0, 0.02):
        print("case SR counts", kmesh, omega, split, flush=True)
        terms[split] = _counted(p, split, tmp_path, monkeypatch)[1].tolist()
    assert terms[1e3] == terms[1.0] == terms[0.02]


def _parity(p, got, aux, pairs):
    ref = oracle.j3c(p, parts=oracle.PART_SR, aux_shells=aux, pairs=pairs)
    ao, ax = p.basis.offsets(), p.aux.offsets()
    err = 0.0
    for P in aux:
        for a, b in pairs:
            blk = np.s_[:, ax[P]:ax[P + 1], ao[a]:ao[a + 1], ao[b]:ao[b + 1]]
            assert np.abs(ref[blk]).max() > 0.0
            err = max(err, float(np.abs(got[blk] - ref[blk]).max()))
    print(f"  max err {err:.3e} (max |V| {np.abs(ref).max():.3e})", flush=True)
    assert err <= 1e-8


@pytest.mark.parametrize("kmesh,split", [((1, 1, 1), 1e3), ((2, 1, 1), 1.0)])
def test_lanes_of_a_unit_are_added_up(kmesh, split, tmp_path, monkeypatch):
    """Aux d and f with d-d and d-p pairs; about 1000 vectors per image."""
    p = synth.tiny_problem(kmesh=kmesh, omega=0.17, seed=11, diffuse=False)
    print("case SR wide classes", kmesh, split, flush=True)
    got, nt, nc, wide = _counted(p, split, tmp_path, monkeypatch, thresh=1e-12)
    _parity(p, got, [2, 4], [(3, 3), (3, 1)])
    assert wide.any() and nt[wide].sum() > 64 * nc[wide].sum()


def test_several_passes(tmp_path, monkeypatch):
    """Some 1400 vectors per (image, cell) near the centre: more than the lanes' lists hold."""
    p = synth.tiny_problem(kmesh=(2, 2, 2), omega=0.1, seed=11, diffuse=False)
    print("case SR several passes", flush=True)
    got, _, _, _ = _counted(p, 1e3, tmp_path, monkeypatch, thresh=1e-12)
    _parity(p, got, [0, 1], [(0, 0), (1, 0), (1, 1)])
