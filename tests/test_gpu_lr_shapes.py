"""GPU parity of the long-range part where the pair transforms change the way
they deal out a class's q vectors: fewer q than lanes (the lanes share the
terms), one block and a bit of it, many blocks, in each contraction form; and
where the k2 phases change theirs: few elements (narrow passes), more k-pairs in
a class than one pass takes (3x3x3).  Reference: the oracle's
long-range part for some k-pairs.  Bars as elsewhere: 1e-8 au in FP64, 1e-6 in
the reduced forms."""
import numpy as np
import pytest

import oracle
import synth
from gpu_util import run_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kmesh,omega,kpairs,forms", [
    ((1, 1, 1), 0.2, [0], (0,)), ((2, 1, 1), 0.25, [0, 1, 2], (0, 1)), ((1, 2, 1), 0.45, [0, 1], (0, 2)),
    ((2, 2, 2), 2.65, [4, 35], (0, 1, 2)), ((3, 3, 3), 0.6, [0, 100, 377], (0, 1, 2))])
def test_lr_shapes(kmesh, omega, kpairs, forms):
    p = synth.tiny_problem(kmesh=kmesh, omega=omega, seed=3, diffuse=False)
    ref = oracle.j3c(p, parts=oracle.PART_LR, kpairs=kpairs)[kpairs]
    for f in forms:
        print("case LR shapes", kmesh, omega, f, flush=True)
        got, st = run_gpu(p, parts=oracle.PART_LR, lr_precision=f)
        err = float(np.abs(got[kpairs] - ref).max())
        print(f"  max err {err:.3e} (max |V| {np.abs(ref).max():.3e}), q {st['n_g_total']}", flush=True)
        assert err <= (1e-8 if f == 0 else 1e-6)
