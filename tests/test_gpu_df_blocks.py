"""The density-fitting solve at the edges of its 64-column blocks and 16-column
strips (one block, exactly one, one column more, several, a ragged last one),
on random Hermitian positive definite metrics against torch's solve of the same
systems in FP64.  Bar: a backward-stable solve of each has a forward error of a
few units of cond(J) eps |d|, so |d_gpu - d_ref| <= 1e-13 cond(J) max|d|."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("naux,kmesh", [(1, (1, 1, 1)), (15, (2, 1, 1)), (64, (1, 1, 1)), (65, (1, 2, 1)),
                                        (130, (3, 1, 1)), (257, (1, 1, 1))])
def test_df_solve_blocks(naux, kmesh):
    import torch

    import paper_2102_02989_amd as P
    print("case DF blocks", naux, kmesh, flush=True)
    g = torch.Generator().manual_seed(naux)
    nk = kmesh[0] * kmesh[1] * kmesh[2]
    nao = 3

    def r(*s):
        return torch.complex(torch.randn(*s, dtype=torch.float64, generator=g),
                             torch.randn(*s, dtype=torch.float64, generator=g))
    A = r(nk, naux, naux)
    J = torch.stack([a @ a.conj().T.contiguous() + 0.1 * torch.eye(naux, dtype=torch.float64) for a in A])
    V = r(P.nkpairs(kmesh), naux, nao, nao)
    d = P.df_solve(kmesh, J.cuda(), V.cuda()).cpu()
    t = 0
    for k1 in range(nk):
        for k2 in range(k1, nk):
            j1 = (k1 // (kmesh[1] * kmesh[2]), k1 // kmesh[2] % kmesh[1], k1 % kmesh[2])
            j2 = (k2 // (kmesh[1] * kmesh[2]), k2 // kmesh[2] % kmesh[1], k2 % kmesh[2])
            c = [(b - a) % n for a, b, n in zip(j1, j2, kmesh)]
            m = J[(c[0] * kmesh[1] + c[1]) * kmesh[2] + c[2]]
            ref = torch.linalg.solve(m, V[t].reshape(naux, -1)).reshape(V[t].shape)
            err = float((d[t] - ref).abs().max())
            assert err <= 1e-13 * float(torch.linalg.cond(m)) * max(float(ref.abs().max()), 1.0)
            t += 1
