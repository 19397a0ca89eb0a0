"""GPU parity of the long-range part with the pair transforms at every width that the
launch rule gives them: 1, 2, 4 and 8 q per lane (s-s), 1, 2 and 4 (p-s), 1 and 2 (up to
l_a + l_b = 3), d-d plain and with the terms shared by four waves; and at each with one q
less than, as many as, and one more than fill the last block.  A cell of four atoms with
24 s, 8 p and 4 d shells on a 3x3x3 mesh; omega sets the q count of the class whose k-pair
is compared.  Reference: the oracle's long-range part of selected AO pairs, two of each
angular class.  Bar: 1e-8 au."""
import ctypes
import math

import numpy as np
import pytest

import lanes_util
import oracle
import synth
from gpu_util import run_gpu

pytestmark = pytest.mark.gpu

SRC = """
#include "lanes.h"
extern "C" void shape(long nx, int nq, int la, int lb, int *out) {
  const rsgdf::PairFtShape s = rsgdf::pairft_shape(nx, nq, rsgdf::pairft_qpl(la, lb));
  out[0] = s.qp, out[1] = s.nql, out[2] = s.waves;
}
"""
GROUPS = [(0, 0), (1, 0), (1, 1), (2, 0), (2, 1), (2, 2)]
# omega, k12 class, its q count, the s-s width and where the count lies in a block of 64 width
CASES = [(0.2058, 3, 64, 1, 0), (0.2088, 3, 65, 1, 1), (0.26, 15, 127, 1, -1), (0.262, 15, 128, 1, 0),
         (0.2624, 15, 129, 2, 1), (0.331, 10, 255, 2, -1), (0.3316, 10, 256, 2, 0), (0.3322, 10, 257, 4, 1),
         (0.4202, 13, 511, 4, -1), (0.4207, 13, 512, 4, 0), (0.421, 13, 513, 8, 1), (0.5304, 9, 1023, 8, -1),
         (0.5304, 15, 1024, 8, 0), (0.625, 1, 1663, 8, None), (0.6255, 16, 1664, 8, None),
         (0.6245, 14, 1665, 8, None)]


def _problem(omega):
    rng = np.random.default_rng(7)
    lat = np.array([[7.1, 0.0, 0.0], [0.9, 6.6, 0.0], [0.4, 1.1, 7.4]])
    frac = np.array([[0.05, 0.1, 0.02], [0.55, 0.48, 0.1], [0.1, 0.6, 0.52], [0.57, 0.05, 0.6]])
    ao, ax = synth.configs._ShellList(), synth.configs._ShellList()
    for a in range(4):
        for e in np.exp(np.linspace(math.log(0.25), math.log(6.0), 6)):
            ao.add(a, 0, [e * rng.uniform(0.95, 1.05)], [1.0])
        for e in (0.35, 1.4):
            ao.add(a, 1, [e * rng.uniform(0.95, 1.05)], [1.0])
        ao.add(a, 2, [0.8 * rng.uniform(0.95, 1.05)], [1.0])
    for a in (0, 2):
        ax.add(a, 0, [0.9 + 0.2 * a], [1.0])
        ax.add(a, 1, [0.7 + 0.1 * a], [1.0])
    return synth.Problem("widths", synth.Cell(lat, frac @ lat), ao.basis(), ax.basis(), (3, 3, 3), omega)


def _nq(p, c):
    lat, n = p.cell.lattice, p.kmesh
    rec = 2.0 * np.pi * np.linalg.inv(lat).T
    w = [int(np.sqrt(-4.0 * p.omega ** 2 * np.log(p.g_thr)) * np.linalg.norm(lat[d]) / (2.0 * np.pi)) + 3
         for d in range(3)]
    G = np.array(np.meshgrid(*[np.arange(-x, x + 1) for x in w], indexing="ij")).reshape(3, -1).T
    q = (G + np.array(np.unravel_index(c, n)) / np.array(n)) @ rec
    q2 = (q * q).sum(1)
    return int(((q2 > 1e-20) & (np.exp(-q2 / (4.0 * p.omega ** 2)) >= p.g_thr)).sum())


def _shapes(lanes, p, nq):
    n = [int((p.basis.shell_l == l).sum()) for l in range(3)]
    out, got = (ctypes.c_int * 3)(), {}
    for la, lb in GROUPS:
        npair = n[la] * (n[la] + 1) // 2 if la == lb else n[la] * n[lb]
        lanes.shape(ctypes.c_long(npair * 27), nq, la, lb, out)
        got[la, lb] = tuple(out)
    return got


@pytest.fixture(scope="module")
def lanes(tmp_path_factory):
    return lanes_util.build(tmp_path_factory.mktemp("widths"), SRC)


def test_cases_cover_the_widths(lanes):
    seen = set()
    for omega, c, nq, width, at in CASES:
        p = _problem(omega)
        assert _nq(p, c) == nq
        s = _shapes(lanes, p, nq)
        assert s[0, 0] == (width, 0, 1) and (at is None or (nq - at) % (64 * width) == 0)
        seen |= {(k, v[0] if v[1] == 0 else "sliced") for k, v in s.items()}
    want = {((0, 0), w) for w in (1, 2, 4, 8)} | {((1, 0), w) for w in (1, 2, 4)}
    want |= {(g, w) for g in ((1, 1), (2, 0), (2, 1)) for w in (1, 2)} | {((2, 2), 1), ((2, 2), "sliced")}
    assert want <= seen


@pytest.mark.parametrize("omega,c,nq,width,at", CASES)
def test_lr_widths(omega, c, nq, width, at):
    p = _problem(omega)
    print("case pair-transform widths", omega, c, nq, flush=True)
    kp = [t for t, (k1, k2) in enumerate(oracle.kpair_list(p.kmesh))
          if np.ravel_multi_index(tuple((np.array(np.unravel_index(k2, p.kmesh)) - np.unravel_index(k1, p.kmesh)) % 3),
                                  p.kmesh) == c][:1]
    s, pp, d = ([i for i in range(p.basis.nshell) if p.basis.shell_l[i] == l] for l in range(3))
    pairs = [(s[0], s[7]), (s[5], s[5]), (pp[0], s[9]), (pp[5], s[3]), (pp[1], pp[6]), (pp[2], pp[2]), (d[0], s[20]),
             (d[3], s[1]), (d[1], pp[7]), (d[2], pp[0]), (d[2], d[3]), (d[0], d[0])]
    got, st = run_gpu(p, parts=oracle.PART_LR)
    ref = oracle.j3c(p, parts=oracle.PART_LR, kpairs=kp, pairs=pairs)
    off = p.basis.offsets()
    err = 0.0
    for a, b in pairs:
        blk = np.s_[kp[0], :, off[a]:off[a + 1], off[b]:off[b + 1]]
        assert np.abs(ref[blk]).max() > 0.0
        err = max(err, float(np.abs(got[blk] - ref[blk]).max()))
    print(f"  max err {err:.3e} (max |V| {np.abs(ref).max():.3e})", flush=True)
    assert err <= 1e-8
