"""Bits of the stencil's results in the precisions below 64 bits.  A kernel may be replaced or its
work split differently, but a caller's numbers stay: an FP16 result is rounded once, by the
multiply-add that forms it, and the third row of a 12-real link is rebuilt with one fixed set of
multiply-adds, whichever kernel takes the launch.

tests/golden/stencil_bits.json holds SHA-256 digests of the outputs of the one-thread-per-site
kernels.  Links, vectors and couplings are integers over powers of two, so the inputs are
the same on every machine; the links are no SU(3) elements, which the kernels do not ask for."""
import hashlib
import json
import math
import os

import numpy as np
import pytest
import torch

from paper_2407_08092_amd import api
from paper_2407_08092_amd._lib import DDQ_BF16, DDQ_F16, DDQ_F32, DDQ_F64

pytestmark = pytest.mark.gpu

GOLDEN = os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden", "stencil_bits.json")
DTYPES = {"f32": torch.complex64, "f16": torch.float16, "bf16": torch.bfloat16}
# launches below and above the sizes where the kernels change over
CASES = [(dims, n) for dims in ((4, 6, 8, 10), (18, 8, 8, 4)) for n in (1, 2, 3)] + [((16, 16, 16, 34), 1), ((16, 16, 16, 34), 2)]


def lattice(dims, link12):
    rng = np.random.default_rng(77)
    q = rng.integers(-2**22, 2**22, size=dims[::-1] + (4, 3, 3, 2)).astype(np.float64) / 2**23
    lat = api.create_lattice(dims)
    U = torch.view_as_complex(torch.from_numpy(q)).cuda()
    api.set_gauge(lat, U, store=(DDQ_F64, DDQ_F32, DDQ_F16, DDQ_BF16), link12=link12)
    api.set_clover(lat, 0.5, 0.25)
    return lat


def vectors(dims, n, dtype, seed):
    vh = math.prod(dims) // 2
    rng = np.random.default_rng(seed)
    shape = ((n,) if n > 1 else ()) + ((6, vh, 2, 2) if dtype == torch.complex64 else (3, vh, 4, 2))
    v = torch.from_numpy(rng.integers(-128, 129, size=shape).astype(np.float32) / 64)
    return torch.view_as_complex(v).cuda() if dtype == torch.complex64 else v.to(dtype).cuda()


def digest(t):
    r = torch.view_as_real(t) if t.is_complex() else t
    assert torch.isfinite(r).all()
    return hashlib.sha256(r.contiguous().view(torch.uint8).cpu().numpy().tobytes()).hexdigest()[:32]


def outputs(dims, n):
    """Digest of every form of the apply and of three sweeps on n right-hand sides."""
    out = {}
    for link12 in (False, True):
        lat = lattice(dims, link12)
        for prec, dtype in DTYPES.items():
            if prec != "f32" and link12:
                continue  # 16-bit links are 12-real already
            x, b = vectors(dims, n, dtype, 78), vectors(dims, n, dtype, 79)
            for c32 in (False,) if prec == "f32" else (False, True):
                if prec != "f32":
                    api.set_h16_clover(lat, c32)
                key = prec + ("_l12" if link12 else "") + ("_c32" if c32 else "")
                out[key + "_apply"] = digest(api.apply_schur(lat, x))
                if prec == "f32":
                    out[key + "_dagger"] = digest(api.apply_schur(lat, x, dagger=True))
                out[key + "_sweeps"] = digest(api.richardson_smooth(lat, x.clone(), b, 3, 0.15625))
    return out


def name(dims, n):
    return "x".join(map(str, dims)) + f"_n{n}"


@pytest.mark.parametrize("dims, n", CASES)
def test_results_keep_their_bits(dims, n):
    want = json.load(open(GOLDEN))[name(dims, n)]
    got = outputs(dims, n)
    assert got.keys() == want.keys()
    assert [k for k in got if got[k] != want[k]] == []
