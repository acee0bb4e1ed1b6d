"""The Adam update's four-element form (arrays 16-byte aligned) against its one-element form (arrays at
odd words of a buffer), bit for bit, at sizes around four elements and around a block, every SH degree."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,deg", [(0, 0), (1, 0), (2, 1), (3, 2), (5, 3), (341, 0), (1023, 1), (1024, 2), (1025, 3), (10_007, 3)])
def test_aligned_and_unaligned_arrays_agree(n, deg):
    import torch
    from paper_2410_20686_amd import _odgs as B
    sizes = (3 * n, 3 * n, 4 * n, n, 3 * (deg + 1) ** 2 * n)
    lr = torch.tensor([1.6e-4, 5e-3, 1e-3, 5e-2, 2.5e-3, 1.25e-4], device="cuda")
    hyper = B.AdamHyper(0.9, 0.999, 1e-15)
    out = []
    for shift in (0, 1):
        rng = np.random.default_rng(17 + n)
        keep, sets = [], []
        for kind in ("raw", "act", "grad", "m", "v"):
            arrays = []
            for s in sizes:
                x = rng.standard_normal(s).astype(np.float32)
                x = np.abs(x) if kind == "v" else (1.0 / (1.0 + np.exp(-x)) if kind == "act" else x)
                buf = torch.zeros(s + shift + 4, device="cuda")
                buf[shift:shift + s] = torch.from_numpy(x.astype(np.float32)).cuda()
                arrays.append(buf[shift:shift + s])
                assert s == 0 or arrays[-1].data_ptr() % 16 == 4 * shift
                keep.append(buf)
            sets.append((arrays, B.ParamPtrs(*[a.data_ptr() if a.numel() else None for a in arrays])))
        step = torch.full((1,), 3, dtype=torch.int32, device="cuda")
        for _ in range(2):
            B.odgs_adam_step(n, deg, *[p for _, p in sets], ctypes.c_void_p(lr.data_ptr()), ctypes.c_void_p(step.data_ptr()),
                             hyper, ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
        assert int(step.cpu()) == 5
        for b, s in zip(keep, sizes * 5):  # nothing past an array's end
            assert (b[shift + s:] == 0).all() and (b[:shift] == 0).all()
        out.append([a.cpu().numpy() for arrays, _ in sets for a in arrays])
    for a, b in zip(*out):
        np.testing.assert_array_equal(a, b)


def test_more_elements_than_a_launch_has_threads():
    """73M Gaussians at SH degree 3 in unaligned arrays: 4.3e9 elements.  The five kinds of array share their
    memory, which the update then leaves holding the activated values; every array is one constant, so
    its elements agree with those of a small update."""
    import torch
    from paper_2410_20686_amd import _odgs as B
    lr = torch.tensor([1.6e-4, 5e-3, 1e-3, 5e-2, 2.5e-3, 1.25e-4], device="cuda")

    def update(n):
        sizes = (3 * n, 3 * n, 4 * n, n, 48 * n)
        buf = torch.full((sum(sizes) + 1,), 0.25, device="cuda")
        at = np.cumsum((1,) + sizes)
        p = B.ParamPtrs(*[buf[int(k):].data_ptr() for k in at[:5]])
        step = torch.zeros(1, dtype=torch.int32, device="cuda")
        B.odgs_adam_step(n, 3, p, p, p, p, p, ctypes.c_void_p(lr.data_ptr()), ctypes.c_void_p(step.data_ptr()),
                         B.AdamHyper(0.9, 0.999, 1e-15), ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
        parts = [buf[int(a):int(b)] for a, b in zip(at[:4], at[1:5])]
        parts += [buf[int(at[4]):int(at[4]) + 3 * n], buf[int(at[4]) + 3 * n:]]  # the two SH rates
        lo_hi = [(float(x.min()), float(x.max())) for x in parts]
        assert float(buf[0]) == 0.25 and int(step) == 1
        return lo_hi

    small = update(5)
    assert all(a == b for a, b in small) and len({a for a, _ in small}) == 6
    if torch.cuda.mem_get_info()[0] < 24 << 30:
        pytest.skip("needs 17 GB of device memory")
    assert update(73_000_000) == small
    torch.cuda.empty_cache()
