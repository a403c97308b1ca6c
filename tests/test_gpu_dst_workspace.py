"""The workspace of the sine-transform solver is scratch: plans used in turn may
share it and the caller may write it between solves, with the same bits."""
import ctypes

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1208_4247_amd import workloads as wl  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shapes", [((2, 5), (2, 7)), ((3, 4), (2, 6)), ((2, 12), (3, 7)),
                                    ((2, 1), (3, 3))])
def test_plans_share_one_workspace(shapes):
    from paper_1208_4247_amd import capi
    from paper_1208_4247_amd.solver import DstSolver, _ptr, _stream

    L = capi.lib()
    sizes = []
    for d, lv in shapes:
        n = ctypes.c_size_t(0)
        assert L.gmg_dst_setup(d, lv, None, ctypes.byref(n), _stream(), None) == 0
        sizes.append(n.value)
    ws = torch.zeros(max(sizes), dtype=torch.uint8, device="cuda")
    plans, fs, want = [], [], []
    for (d, lv), n in zip(shapes, sizes):
        h = ctypes.c_void_p()
        assert L.gmg_dst_setup(d, lv, _ptr(ws), ctypes.byref(ctypes.c_size_t(n)), _stream(),
                               ctypes.byref(h)) == 0
        plans.append(h)
        fs.append(torch.from_numpy(wl.rhs_uniform(d, (1 << lv) - 1, seed=820 + lv)).cuda())
        own = DstSolver(d, lv)
        u = torch.empty_like(fs[-1])
        own.solve(u, fs[-1])
        want.append(u.cpu().numpy())
    for _ in range(2):
        for h, f, w in zip(plans, fs, want):
            u = torch.empty_like(f)
            assert L.gmg_dst_solve(h, _ptr(u), _ptr(f)) == 0
            assert np.array_equal(u.cpu().numpy(), w)
            ws.fill_(255)  # NaN where it is read as numbers
    for h in plans:
        assert L.gmg_dst_destroy(h) == 0
