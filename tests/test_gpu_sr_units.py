"""GPU parity of the one-unit-per-lane short-range kernel against the oracle,
short-range part only, at the shapes where its lane layout can go wrong:
pair images of one BvK class over several batches (Gamma), whole runs of
several classes in one batch (4x4x1), a mesh that does not divide the wave
(1x3x2, 5x1x1), work split over cells and images in the ways the planner can
choose (a class that ends where the queue of images does), more primitive triples than one chunk of constants holds and
contracted auxiliary shells (their exponent factors enter per primitive, the
pure numbers once at the store), up to f on d-d pairs.  Screened at 1e-12, so that
the FP64 1e-8 au bar checks the lane layout and not the screening."""
import sys

import numpy as np
import pytest

import oracle
import synth
from gpu_util import run_gpu

pytestmark = pytest.mark.gpu
TOL = 1e-8


def _contracted(p, nprim, seed):
    """The same shells with nprim primitives each in the auxiliary basis."""
    rng = np.random.default_rng(seed)
    b = synth.configs._ShellList()
    for at, l in zip(p.aux.shell_atom, p.aux.shell_l):
        b.add(int(at), int(l), np.exp(rng.uniform(np.log(0.3), np.log(6.0), nprim)), rng.normal(size=nprim))
    p.aux = b.basis()
    return p


@pytest.mark.parametrize("kmesh,omega,nprim,split", [
    ((1, 1, 1), 0.4, 1, 1.0), ((4, 4, 1), 0.7, 1, 1.0), ((1, 3, 2), 0.6, 3, 1.0), ((5, 1, 1), 0.9, 1, 1.0),
    ((2, 1, 1), 0.8, 13, 1.0), ((1, 3, 2), 0.5, 1, 1e3), ((1, 3, 2), 0.5, 1, 8.0), ((1, 3, 2), 0.5, 1, 0.02)])
def test_sr_units(kmesh, omega, nprim, split):
    p = synth.tiny_problem(kmesh=kmesh, omega=omega, seed=11, diffuse=False)
    if nprim > 1:
        p = _contracted(p, nprim, 5)
    print("case SR units", kmesh, omega, nprim, split, flush=True)
    got, st = run_gpu(p, thresh=1e-12, parts=oracle.PART_SR, sr_split=np.full(24, split, np.float32))
    ref = oracle.j3c(p, parts=oracle.PART_SR)
    err = float(np.abs(got - ref).max())
    print(f"  max err {err:.3e} (max |V| {np.abs(ref).max():.3e}), terms {st['n_sr_terms']}", flush=True)
    sys.stdout.flush()
    assert err <= TOL
