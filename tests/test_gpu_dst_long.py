"""The sine-transform solver's longest 3D lines (N = 1024 and 2048: several
wavefronts a pair, every axis kernel) on rough data, where every coefficient up
to the highest is alive, against dense sine matrices in FP64.  Tolerance:
2e-13 for the six transforms (a few eps log2 N each), and for the reference
six products of length m, m eps each by the general bound: 6 x 1023 x 1.1e-16
= 7e-13; 1e-12 asked, in the 2-norm."""
import math

import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


def _along_all(x, s):
    m = s.shape[0]
    for _ in range(3):  # the last axis, then rotated to the front
        x = (x.reshape(-1, m) @ s).reshape(m, m, m).movedim(-1, 0).contiguous()
    return x


@pytest.mark.parametrize("L", [9, 10])
def test_rough_data(L):
    from paper_1208_4247_amd.solver import DstSolver

    print("dst 3d", L, flush=True)
    n, m = 1 << L, (1 << L) - 1
    g = torch.Generator(device="cuda").manual_seed(890 + L)
    f = torch.rand((m,) * 3, dtype=torch.float64, device="cuda", generator=g).mul_(2.0).sub_(1.0)
    f[0, 0, 0] += 3.0  # the corners are live
    f[-1, -1, -1] -= 2.0
    solver = DstSolver(3, L)
    u = torch.full_like(f, float("nan"))
    solver.solve(u, f)

    k = torch.arange(1, n, device="cuda")
    s = torch.sin((torch.outer(k, k) % (2 * n)).double() * (math.pi / n)) * math.sqrt(2.0 / n)
    lam = (2.0 * n * torch.sin(k.double() * (math.pi / (2 * n)))) ** 2
    x = _along_all(f, s)
    for a in range(m):  # a plane at a time
        x[a].div_(lam[a] + lam[:, None] + lam[None, :])
    want = _along_all(x, s)
    err = float(torch.linalg.vector_norm(u - want) / torch.linalg.vector_norm(want))
    print("relative error %.2e" % err, flush=True)
    assert err <= 1e-12
