"""Which launches and copies a call makes, and with which arguments, without a GPU: the library runs
in a process of its own on a stand-in for the HIP runtime (fake_hip.cpp) that executes nothing."""
import ctypes as C
import json
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
DEVICE, HOST, UNREGISTERED, MANAGED = 2, 1, 0, 3  # hipMemoryType
U = 0x7F0000000000


class Event(C.Structure):
    _fields_ = [("kind", C.c_int), ("name", C.c_char_p), ("ptr", C.c_void_p), ("grid", C.c_uint64), ("block", C.c_uint64)]


def events(fake):
    n = C.c_int()
    e = fake.fake_events(C.byref(n))
    return [dict(kind=e[k].kind, name=e[k].name.decode(), ptr=e[k].ptr, grid=e[k].grid, block=e[k].block) for k in range(n.value)]


def lattice(L, dims):
    h = C.c_void_p()
    assert L.ddq_create_lattice((C.c_int * 4)(*dims), 1, None, C.byref(h)) == 0, L.ddq_last_error()
    return h


def gauge_source(fake, L, error, type_, device, ptr, on_device):
    """ddq_set_gauge with links of these pointer attributes: its copies and launches."""
    h = lattice(L, (4, 4, 4, 4))
    fake.fake_pointer(error, type_, device)
    events(fake)
    assert L.ddq_set_gauge(h, C.c_void_p(ptr), on_device, 1) == 0, L.ddq_last_error()
    return events(fake)


def applies(fake, L, dims, nrhs, prec):
    """The stencil launches of one apply on nrhs right-hand sides."""
    h = lattice(L, dims)
    fake.fake_pointer(0, DEVICE, 0)
    assert L.ddq_set_gauge(h, C.c_void_p(U), 1, 1 | 2) == 0, L.ddq_last_error()
    assert L.ddq_set_clover(h, 1.0, 0.1) == 0, L.ddq_last_error()
    assert L.ddq_reserve(h, nrhs, 0, 0) == 0, L.ddq_last_error()
    events(fake)
    assert L.ddq_apply_schur(h, prec, nrhs, C.c_void_p(U), C.c_void_p(2 * U), 0) == 0, L.ddq_last_error()
    return [e for e in events(fake) if e["kind"] == 1]


def clover_twice(fake, L):
    """What ddq_set_clover enqueues and waits for after the clover build, on a new lattice and again."""
    h = lattice(L, (4, 4, 4, 4))
    fake.fake_pointer(0, DEVICE, 0)
    out = []
    for _ in range(2):
        assert L.ddq_set_gauge(h, C.c_void_p(U), 1, 1 | 2) == 0, L.ddq_last_error()
        events(fake)
        assert L.ddq_set_clover(h, 1.0, 0.1) == 0, L.ddq_last_error()
        e = events(fake)
        build = max(k for k, v in enumerate(e) if "k_clover_build" in v["name"])
        out.append([v["name"] for v in e[build + 1:]])
    return out


def main(fake_path, call, args):
    fake = C.CDLL(fake_path, mode=C.RTLD_GLOBAL)
    fake.fake_events.restype = C.POINTER(Event)
    sys.path.insert(0, os.path.dirname(HERE))
    from paper_2407_08092_amd import _lib

    print(json.dumps(globals()[call](fake, _lib.lib(), *args)))


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("fake") / "libfake_hip.so")
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", os.path.join(HERE, "fake_hip.cpp"), "-o", so, "-ldl"], check=True)

    def go(call, *args):
        r = subprocess.run([sys.executable, __file__, so, call, json.dumps(args)], capture_output=True, text=True, timeout=120)
        assert r.returncode == 0, r.stdout + r.stderr
        return json.loads(r.stdout.splitlines()[-1])

    return go


@pytest.mark.parametrize("error, type_, device, ptr, in_place", [
    (0, DEVICE, 0, U, True),
    (0, DEVICE, 0, U + 8, False),      # off the loads' alignment
    (0, DEVICE, 1, U, False),          # another GPU's memory: a copy works where a kernel's load may not
    (0, HOST, 0, U, False),
    (0, MANAGED, 0, U, False),
    (0, UNREGISTERED, 0, U, False),
    (1, DEVICE, 0, U, False),          # an address the runtime does not know
])
def test_links_are_read_in_place_only_from_the_lattices_gpu(run, error, type_, device, ptr, in_place):
    ev = run("gauge_source", error, type_, device, ptr, 1)
    pack = [e for e in ev if "k_pack_gauge" in e["name"]]
    assert len(pack) == 1
    assert (pack[0]["ptr"] == ptr) == in_place
    assert [e["ptr"] for e in ev if e["kind"] == 0] == ([] if in_place else [ptr])


# 2 x 2 x 258 x 256: the slab order's padding doubles the workgroups (4096 right-hand sides: 52 GB
# a vector in FP32)
@pytest.mark.parametrize("dims, nrhs, split", [((48, 48, 48, 96), 2, True), ((2, 2, 258, 256), 2, True), ((2, 2, 258, 256), 4096, False)])
def test_a_launch_stays_below_the_limit_of_threads(run, dims, nrhs, split):
    ev = run("applies", list(dims), nrhs, 1)
    assert len(ev) == 2
    for e in ev:
        assert e["grid"] * e["block"] < 2**32
        assert ("hop_split_kernel" in e["name"]) == split


def test_a_new_lattices_clover_leaves_no_batch_to_retire(run):
    assert run("clover_twice") == [["wait", "memset", "wait"], ["wait", "wait"]]


if __name__ == "__main__":
    main(sys.argv[1], sys.argv[2], json.loads(sys.argv[3]))
