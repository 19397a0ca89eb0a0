"""The short range's work counters do not depend on how its items are split over
waves, lanes and passes: terms, and contractions counted once per (pair image, BvK
cell, primitive triple) with a lattice vector, whichever lane of the unit has it."""
import numpy as np
import pytest

import oracle
import synth
from gpu_util import run_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kmesh,omega", [((1, 1, 1), 0.3), ((1, 3, 2), 0.5)])
def test_counts_do_not_depend_on_the_split(kmesh, omega):
    p = synth.tiny_problem(kmesh=kmesh, omega=omega, seed=11, diffuse=False)
    got = {}
    for split in (1e3, 1.0, 0.02):
        print("case SR counts", kmesh, omega, split, flush=True)
        _, st = run_gpu(p, parts=oracle.PART_SR, sr_split=np.full(24, split, np.float32))
        got[split] = (st["n_sr_terms"], st["n_sr_shell_terms"], st["sr_flops"])
    print("  ", got, flush=True)
    assert got[1e3] == got[1.0] == got[0.02]
    assert got[1.0][2] > 0
