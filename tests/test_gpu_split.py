"""The stencil on four threads per site (launches of few sites, several right-hand sides)
against the one-thread-per-site kernels: the same operations in the same order, so the
results are equal bit for bit.  A tile with nb = 0 selects one thread per site.

Lattices: one wavefront not filled (2^4), t-slices that are no multiple of 64 sites, groups
across slices (plain order), and eight or more 64-site groups a slice (slab order)."""
import pytest
import torch

from gpu_common import Case, to_dev, to_dev16
from paper_2407_08092_amd import api
from paper_2407_08092_amd._lib import DDQ_BF16, DDQ_F16, DDQ_F32, DDQ_F64

pytestmark = pytest.mark.gpu

N = 3
DTYPES = [torch.complex128, torch.complex64, torch.float16, torch.bfloat16]


def dev(v, dtype):
    return to_dev16(v, dtype) if dtype in (torch.float16, torch.bfloat16) else to_dev(v, dtype)


@pytest.mark.parametrize("link12", [False, True])
@pytest.mark.parametrize("dims", [(2, 2, 2, 2), (4, 6, 8, 10), (12, 10, 6, 2), (18, 8, 8, 4)])
def test_split_equals_one_thread_per_site(dims, link12):
    c = Case(dims, 0.5, 1.0, -0.1, 811)
    U = torch.from_numpy(c.U).cuda()
    got = []
    for tile in (False, True):
        lat = api.create_lattice(dims)
        api.set_gauge(lat, U, store=(DDQ_F64, DDQ_F32, DDQ_F16, DDQ_BF16), link12=link12)
        api.set_clover(lat, 1.0, -0.1)
        if tile:
            api.set_multi_rhs_tile(lat, N, 0)
        out = []
        for dtype in DTYPES:
            x, b = dev(c.vec(812, N), dtype), dev(c.vec(813, N), dtype)
            out.append(api.apply_schur(lat, x))
            if dtype.is_complex:
                out.append(api.apply_schur(lat, x, dagger=True))
            out.append(api.richardson_smooth(lat, x.clone(), b, 2, 0.15))
        full = torch.stack([torch.from_numpy(c.full(820 + r)).cuda() for r in range(N)])
        xe = to_dev(c.vec(814, N))
        out += [api.oe_prepare(lat, full), api.oe_reconstruct(lat, xe, full)]
        got.append(out)
    for a, b in zip(*got):
        assert torch.equal(a, b)


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("dims", [(4, 6, 8, 10), (18, 8, 8, 4)])
def test_right_hand_sides_are_independent(dims, dtype):
    # three right-hand sides in one launch and each alone; an in-place sweep reads every row of
    # x before any of them is written
    c = Case(dims, 0.5, 1.0, -0.1, 821)
    lat = api.create_lattice(dims)
    api.set_gauge(lat, torch.from_numpy(c.U).cuda(), store=(DDQ_F64, DDQ_F32, DDQ_F16, DDQ_BF16))
    api.set_clover(lat, 1.0, -0.1)
    x, b = dev(c.vec(822, N), dtype), dev(c.vec(823, N), dtype)
    y, z = api.apply_schur(lat, x), api.richardson_smooth(lat, x.clone(), b, 3, 0.15)
    for r in range(N):
        assert torch.equal(api.apply_schur(lat, x[r].contiguous()), y[r])
        assert torch.equal(api.richardson_smooth(lat, x[r].clone(), b[r].contiguous(), 3, 0.15), z[r])
