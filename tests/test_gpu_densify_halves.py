"""The densification step's two halves (counts, then outputs of exact size) against the single call with
its largest capacity, and both against the oracle, at every SH degree and around a block of Gaussians."""
import ctypes

import numpy as np
import pytest

from oracle import densify as OD
from tests.test_gpu_densify import _random_densify_inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,deg", [(1, 0), (255, 1), (256, 2), (257, 3), (70_001, 0), (70_001, 1), (70_001, 2), (70_001, 3)])
def test_halves_match_the_single_call(n, deg):
    import torch
    from paper_2410_20686_amd import _odgs as B
    from paper_2410_20686_amd.densify import DensifyStats, densify
    k3 = 3 * (deg + 1) ** 2
    arrs = list(_random_densify_inputs(n, 90 + deg, 37.5))
    arrs[4] = np.ascontiguousarray(arrs[4][:k3])
    T = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in arrs]
    params, noise = tuple(T[:5]), T[8]
    stats = DensifyStats(n)
    for t, a in zip((stats.grad_sum, stats.tau_sum, stats.count), T[5:8]):
        t.copy_(a)
    new, src, counts = densify(params, stats, noise, 37.5, deg)
    cap = 2 * n + 3
    out = [torch.full((r, cap), -7.0, device="cuda") for r in (3, 3, 4, 1, k3)]
    osrc = torch.full((cap,), -7, dtype=torch.int32, device="cuda")
    oc = torch.empty(4, dtype=torch.int64, device="cuda")
    wsb = B.odgs_densify_workspace_bytes(n)
    ws = torch.empty(wsb, dtype=torch.uint8, device="cuda")
    p = lambda t: ctypes.c_void_p(t.data_ptr())
    B.odgs_densify(n, deg, *map(p, params), p(stats.grad_sum), p(stats.tau_sum), p(stats.count), p(noise),
                   B.DensifyParams(37.5, 1e-3, 0.005, 0.0), cap, *map(p, out), p(osrc), p(oc), p(ws), wsb,
                   ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    m = sum(counts)
    assert tuple(oc.tolist()) == counts and src.shape == (m,)
    for a, b in zip((*new, src), (*out, osrc)):
        a, b = a.reshape(-1, m).cpu().numpy(), b.reshape(-1, cap).cpu().numpy()
        np.testing.assert_array_equal(a, b[:, :m])
        assert (b[:, m:] == -7).all()  # entries past the total are left untouched
    ref = OD.densify(*arrs, extent=37.5)
    assert counts == ref["counts"]
    np.testing.assert_array_equal(src.cpu().numpy(), ref["src"])
    np.testing.assert_array_equal(new[4].cpu().numpy(), ref["sh"])
    np.testing.assert_array_equal(new[1].cpu().numpy(), ref["scales"])
