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


def random_lattice(dims, link12=False):
    """Links that are no SU(3) elements, which the kernels do not ask for: quick at any size."""
    lat = api.create_lattice(dims)
    gen = torch.Generator(device="cuda").manual_seed(831)
    U = torch.rand(lat.full_shape[:4] + (4, 3, 3, 2), generator=gen, dtype=torch.float64, device="cuda") - 0.5
    api.set_gauge(lat, torch.view_as_complex(U), store=(DDQ_F64, DDQ_F32, DDQ_F16, DDQ_BF16), link12=link12)
    api.set_clover(lat, 0.5, 0.25)
    return lat


def random_vectors(lat, n, dtype, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    vh = lat.dims[0] * lat.dims[1] * lat.dims[2] * lat.dims[3] // 2
    shape = {torch.complex128: (12, vh, 2), torch.complex64: (6, vh, 2, 2)}.get(dtype, (3, vh, 4, 2))
    v = torch.randn((n,) + shape, generator=gen, dtype=torch.float64, device="cuda")
    return torch.view_as_complex(v.to(torch.float64 if dtype == torch.complex128 else torch.float32)) if dtype.is_complex else v.to(dtype)


# One right-hand side, on both sides of every line of the size rules and in every cache policy, in
# one launch and in ranges of t-slices, against launches of two, which take four threads a site
# (16 bits: one, two vectors a thread).  Sites of a parity / what one takes:
#   5,760: four threads a site, nine groups of 64 sites a slice in a row (two vectors: slab order);
#   44,000: one thread a site but for FP32 sweeps; 69,696: FP32 four threads again, 16 bits one;
#   216,000: FP32 sweeps stream links and results; 405,000: FP32 one thread, vectors kept;
#   629,440: FP64 streams; 1,207,184: FP32 streams
@pytest.mark.parametrize("dims, dtypes", [
    ((18, 8, 8, 10), DTYPES),
    ((20, 22, 10, 20), (torch.complex128, torch.complex64)),
    ((22, 22, 18, 16), DTYPES),
    ((30, 30, 30, 16), (torch.complex128, torch.complex64)),
    ((30, 30, 30, 30), (torch.complex64, torch.float16)),
    ((34, 34, 34, 32), (torch.complex128,)),
    ((38, 38, 38, 44), (torch.complex64,)),
])
def test_one_right_hand_side_on_either_kernel(dims, dtypes):
    for link12 in (False, True):
        lat = random_lattice(dims, link12)
        for dtype in dtypes if not link12 else [d for d in dtypes if d == torch.complex64]:
            x, b = random_vectors(lat, 2, dtype, 832), random_vectors(lat, 2, dtype, 833)
            for c32 in (False, True) if not dtype.is_complex else (False,):
                api.set_h16_clover(lat, c32)
                y, z = api.apply_schur(lat, x), api.richardson_smooth(lat, x.clone(), b, 2, 0.15)
                yd = api.apply_schur(lat, x, dagger=True) if dtype.is_complex else None
                for r in range(2):
                    for chunks in (1, 3):
                        api.set_sweep_chunks(lat, chunks)
                        assert torch.equal(api.apply_schur(lat, x[r].contiguous()), y[r])
                        assert torch.equal(api.richardson_smooth(lat, x[r].clone(), b[r].contiguous(), 2, 0.15), z[r])
                        if yd is not None:
                            assert torch.equal(api.apply_schur(lat, x[r].contiguous(), dagger=True), yd[r])
                    api.set_sweep_chunks(lat, 0)
        api.destroy_lattice(lat)


def dense(v, blocks):
    """Dense clover blocks [V/2, 2, 6, 6] on a parity vector [12, V/2], on the CPU."""
    s = v.cpu().T.reshape(-1, 2, 6, 1)
    return (blocks.cpu() @ s).reshape(-1, 12).T.contiguous().cuda()


@pytest.mark.parametrize("n", [1, 3])
@pytest.mark.parametrize("dims", [(4, 6, 8, 10), (12, 10, 6, 2), (18, 8, 8, 4), (16, 16, 16, 22)])
def test_eq2_against_the_full_operator(dims, n):
    """oe_prepare, oe_reconstruct and the FP32 form of b~_e that M_nu starts from, against D on
    vectors of one parity and the exported clover blocks: sums of some 30 products in FP64, 2e-14
    relative; the FP32 form is exactly the rounded one, times omega in FP32."""
    c = Case(dims, 0.5, 1.0, -0.1, 841)
    a_oo_inv = api.get_clover(c.lat)[1]
    gen = torch.Generator(device="cuda").manual_seed(842)
    b, x = (torch.view_as_complex(torch.randn((n,) + c.lat.full_shape + (2,), generator=gen, dtype=torch.float64, device="cuda"))
            for _ in range(2))
    xe = torch.stack([api.pack_parity(c.lat, v, 0) for v in x])
    bt, full = api.oe_prepare(c.lat, b), api.oe_reconstruct(c.lat, xe, b)
    omega = 0.15
    z = api.oe_smoother(c.lat, b, 1, omega, prec=DDQ_F32)
    for r in range(n):
        be, bo = api.pack_parity(c.lat, b[r], 0), api.pack_parity(c.lat, b[r], 1)
        odd = api.unpack_parity(c.lat, dense(bo, a_oo_inv), 1, torch.zeros_like(b[r]))
        ref = be - api.pack_parity(c.lat, api.apply_dirac(c.lat, odd), 0)
        assert ((bt[r] - ref).norm() / ref.norm()).item() < 2e-14
        even = api.unpack_parity(c.lat, xe[r].contiguous(), 0, torch.zeros_like(b[r]))
        ref = dense(bo - api.pack_parity(c.lat, api.apply_dirac(c.lat, even), 1), a_oo_inv)
        xo = api.pack_parity(c.lat, full[r].contiguous(), 1)
        assert ((xo - ref).norm() / ref.norm()).item() < 2e-14
        assert torch.equal(api.pack_parity(c.lat, full[r].contiguous(), 0), xe[r])
        b32 = torch.view_as_real(bt[r]).to(torch.float32)
        assert torch.equal(torch.view_as_real(api.pack_parity(c.lat, z[r].contiguous(), 0)), (b32 * torch.tensor(omega, dtype=torch.float32)).to(torch.float64))
