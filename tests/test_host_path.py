"""The library's host path on a HIP runtime without a device (fake_hip.cpp,
whose functions take the runtime's place in a child process): what is refused,
what a launch may ask for and in which order things are given back.  No kernel
runs."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2304_05735_amd", "libromap.so")
pytestmark = pytest.mark.skipif(not os.path.exists(LIB), reason="libromap.so not built")

PRELUDE = """
import ctypes, sys, types
torch = types.ModuleType("torch")  # the binding only tells its tensors from arrays
torch.Tensor = type("Tensor", (), {})
sys.modules["torch"] = torch
fake = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
for f in ("fake_launches", "fake_graph_launches", "fake_busy_graphs_destroyed", "fake_max_record_slots",
          "fake_threads"):
    getattr(fake, f).restype = ctypes.c_int64
import numpy as np
import paper_2304_05735_amd as pk
L = pk.lib()
here = ctypes.c_void_p(4096)  # a device address that nothing reads

def code(call):
    try:
        call()
    except pk.RomapError as e:
        return e.code
    return 0

def context(n=1, half=0.4, log2T=0, **kw):
    g = pk.Context(pk.default_config(**{"samples_per_ray": 32, "rays_per_step": 64, "autotune": 0,
                                        "log2_table_size": 12, "n_levels": 4, "max_res": 64, **kw}))
    ids = [g.add_object(k + 1, [0, 0, 0], 0.0, [half] * 3, log2T) for k in range(n)]
    mask = np.repeat(np.arange(n, dtype=np.int32) + 1, 2)[None].repeat(2, 0)
    T = np.eye(4)[:3]
    T[2, 3] = -2.0
    cam = dict(T_wc=T, fx=50.0, fy=50.0, cx=n, cy=1.0, W=2 * n, H=2)
    g.add_keyframe(cam, np.zeros((2, 2 * n, 3), np.uint8), mask)
    return g, ids, cam

def forward(g, i, n):
    g._check(L.romap_field_forward(g.h, i, None, here, n, here, here, here))

def backward(g, i, n):
    g._check(L.romap_field_backward(g.h, i, None, here, n, here, here, here, here))
"""


@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("fake") / "libfake_hip.so")
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__",
                    "-I", os.path.join(rocm, "include"),
                    "-I", os.path.join(ROOT, "paper_2304_05735_amd", "csrc"),
                    os.path.join(ROOT, "tests", "fake_hip.cpp"), "-o", so], check=True)

    def run(body):
        r = subprocess.run([sys.executable, "-c", PRELUDE + body, so], cwd=ROOT, capture_output=True,
                           text=True, timeout=300)
        assert r.returncode == 0, (r.returncode, r.stdout[-2000:], r.stderr[-4000:])
    return run


def test_no_call_that_uses_context_scratch_joins_a_capture(fake):
    """A replay would read work tables and scratch that later calls overwrite or
    free.  Refused also where the call's tables are in place already, nothing is
    launched, and the call works again once the capture is over."""
    fake("""
g, (i,), cam = context(use_graph=0)
ga, (ia,), _ = context(autotune=1)
noalloc = lambda: g._check(L.romap_field_forward_noalloc(g.h, i, None, here, 64, here, here, here))
calls = [lambda: forward(g, i, 64), lambda: backward(g, i, 64), lambda: g.train(1, [i], stats=False),
         lambda: g.train(1, [i]), lambda: g.loss_and_grad([i]), lambda: g.render(i, cam),
         lambda: g.debug_rays(i, 64), noalloc, lambda: ga.train(1, [ia], stats=False)]
for k, call in enumerate(calls):
    assert code(call) == 0 and code(call) == 0, k
    fake.fake_capture(1)
    n = fake.fake_launches()
    assert code(call) == pk.ROMAP_E_STATE, (k, code(call))
    assert fake.fake_launches() == n, k
    # wrong arguments are still told as such, and calls without work are none
    assert code(lambda: forward(g, 7, 64)) == pk.ROMAP_E_NOT_FOUND
    assert code(lambda: g.train(1, [i], [0])) == pk.ROMAP_E_INVALID_ARG
    assert code(lambda: g.train(0, [i])) == 0
    fake.fake_capture(0)
    assert code(call) == 0 and fake.fake_launches() > n, k
""")


@pytest.mark.parametrize("base,log2T", [(252, 24), (160, 24), (16, 19)])
def test_record_slots_fit_their_index(fake, base, log2T):
    """A record's slot within its level is a 32-bit number, also for the most
    samples that one object takes (2^27: 8 records each, and a dense level's
    bins twice that)."""
    fake(f"""
g, (i,), cam = context(n_levels=1, base_res={base}, max_res=1024, log2_table_size={log2T},
                       samples_per_ray=128)
backward(g, i, 1 << 20)
print(fake.fake_max_record_slots())
assert (1 << 30) <= fake.fake_max_record_slots() < (1 << 31)
""")


def test_step_graph_is_destroyed_after_its_last_launch(fake):
    """Calls without stats do not wait, so the graph that another step count,
    another set of rays or a buffer's growth replaces may still run."""
    fake("""
g, ids, cam = context(n=2, use_graph=2)
g.train(8, ids, stats=False)
assert fake.fake_graph_launches() == 2
g.train(2, ids, stats=False)               # a graph of one step takes its place
g.train(8, ids, [40, 30], stats=False)
backward(g, ids[0], 5000)                  # buffers grow
g.train(8, ids, stats=False)
for k in range(2, 18):
    g.add_object(k + 1, [0, 0, 0], 0.0, [0.4] * 3)   # the object table grows
g.train(8, ids, stats=False)
for k in range(70):
    g.add_keyframe(cam, np.zeros((2, 4, 3), np.uint8), np.zeros((2, 4), np.int32))
g.train(8, ids, stats=False)
assert fake.fake_graph_launches() == 2 + 2 + 2 + 2 + 2 + 2
g.close()
assert fake.fake_busy_graphs_destroyed() == 0, fake.fake_busy_graphs_destroyed()
""")


def test_launches_stay_below_the_grid_limit(fake):
    """The runtime takes fewer than 2^32 work-items to a launch: densities at
    2^32 - 64 points, and live masks of 2^32 samples."""
    fake("""
g, (i,), cam = context()
n = (1 << 32) - 64
g._check(L.romap_query_density(g.h, i, here, n, here, 1))
assert fake.fake_threads(b"k_query_density") >= 4 * n
g, ids, cam = context(n=32, n_levels=1, samples_per_ray=128, streams=1, use_graph=0)
for i in ids:
    g.set_occupancy(i, np.full(32768, 255, np.uint8))
g.train(1, ids, [1 << 20] * 32, stats=False)
assert fake.fake_threads(b"k_live") > 0
""")


def test_render_after_a_failed_host_allocation(fake):
    fake("""
g, (i,), cam = context()
fake.fake_fail_host_malloc(1)
assert code(lambda: g.render(i, cam)) == pk.ROMAP_E_OUT_OF_MEMORY
assert code(lambda: g.render(i, cam)) == 0 and code(lambda: g.render(i, cam)) == 0
""")
