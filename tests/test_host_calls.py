"""The host side of the C ABI without a GPU: libnbody.so runs against a
stand-in for the HIP runtime (hip_stub.c) that logs the kernels instead of
running them, in a process of its own.

* ``nbody_force_noalloc`` with an output on top of an input: the evaluation
  may store no output while another workgroup still fetches its sources from
  that memory, so it writes partial sums, also for a single split, and the
  split sums write the outputs when it is done.  Calls without overlap keep
  the single launch, calls without the potential pack their sources first.
* ``nbody_energy`` and the start-up with clusters of mixed sizes: the launch
  shape of the largest must not leave the small ones' lanes without particles,
  nor the large ones in a few long workgroups.
* a context's pinned words: kept for the next context only if the wait for the
  context's own work succeeded, and only while the runtime knows them.
"""
import json
import os
import re
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
LIB = os.path.join(os.path.dirname(HERE), "paper_1207_2367_amd", "libnbody.so")

PRELUDE = """
import ctypes as C, json, sys
stub = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)   # its symbols come before the runtime's
lib = C.CDLL(sys.argv[2])
vp, i64 = C.c_void_p, C.c_int64
stub.stub_name.restype, stub.stub_part.restype = C.c_char_p, vp
def var(name):
    return C.c_int.in_dll(stub, name)
def log():
    q = [(stub.stub_name(k).decode(), stub.stub_gx(k), stub.stub_gy(k), stub.stub_part(k) is not None)
         for k in range(var("stub_launches").value)]
    var("stub_launches").value = 0
    return q
"""


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("stub") / "hip_stub.so")
    subprocess.check_call(["gcc", "-O1", "-Wall", "-shared", "-fPIC", "-o", so,
                           os.path.join(HERE, "hip_stub.c")])

    def run(code):
        r = subprocess.run([sys.executable, "-c", PRELUDE + code, so, LIB], capture_output=True,
                           text=True, timeout=120)
        assert r.returncode == 0, r.stderr
        return json.loads(r.stdout)
    return run


NOALLOC = """
f = lib.nbody_force_noalloc
f.argtypes = [i64, vp, vp, vp, vp, C.c_double, C.c_int32, i64] + [vp] * 6
B = 1 << 32   # addresses far apart; nothing is read or written
def call(n, na, prec, over):
    mass, pos, vel, acc, idx, a, j, s, p = (vp((k + 2) * B).value for k in range(9))
    if over == "acc":
        a = acc
    elif over == "acc tail":        # only the last particle's row
        a = acc + 24 * (n - 1)
    elif over == "vel":
        s = vel
    elif over == "pos end":         # an output that ends inside the first row
        j = pos - 24 * na + 8
    elif over == "mass":
        p = mass
    elif over == "beside":          # right behind and right before: no overlap
        a, j = acc + 24 * n, acc - 24 * na
    elif over == "no pot":
        a, p = acc, None
    rc = f(n, mass, pos, vel, acc, 1e-4, prec, na, idx, a, j, s, p, None)
    return rc, log()
out = []
for n, na in ((64, 64), (256, 256), (511, 511), (1000, 1000), (1000, 3), (300000, 200000)):
    for prec in (0, 2):
        for over in ("", "beside", "acc", "acc tail", "vel", "pos end", "mass", "no pot"):
            out.append((n, na, over, *call(n, na, prec, over)))
print(json.dumps(out))
"""


def test_noalloc_outputs_on_inputs(host):
    single = 0
    for n, na, over, rc, launches in host(NOALLOC):
        what = (n, na, over, launches)
        assert rc == 0, what
        names = [q[0] for q in launches]
        if over == "no pot":
            assert "pack_arrays" in names[0] and "force_kernel" in names[1], what
            continue
        assert "force_kernel" in names[0], what
        splits, staged = launches[0][2], launches[0][3]
        if over in ("", "beside"):
            assert staged == (splits > 1), what
            single += splits == 1
        else:
            assert staged, what
        assert len(names) == 1 + staged and all("reduce_split" in q for q in names[1:]), what
    assert single >= 10   # sizes that the rule evaluates in one split are among them


CONTEXT = """
class Config(C.Structure):
    _fields_ = [("eta", C.c_double), ("eta_init", C.c_double), ("dt_min", C.c_double), ("dt_max", C.c_double),
                ("precision", C.c_int32), ("n_clusters", C.c_int32), ("cluster_offsets", C.POINTER(i64)),
                ("stream", vp), ("validate", C.c_int32), ("skip_startup", C.c_int32)]
lib.nbody_workspace_bytes.restype = C.c_size_t
lib.nbody_workspace_bytes.argtypes = [i64, vp]
lib.nbody_init.argtypes = [vp, i64, vp, vp, vp, C.c_double, vp, vp, C.c_size_t]
lib.nbody_free.argtypes = [vp]
lib.nbody_free.restype = None
def context(sizes, want=0, startup=False):
    global launches
    cfg = Config()
    lib.nbody_default_config(C.byref(cfg))
    cfg.skip_startup = not startup
    off = [0]
    for k in sizes:
        off.append(off[-1] + k)
    n = off[-1]
    cfg.cluster_offsets = (i64 * len(off))(*off)
    cfg.n_clusters = len(sizes)
    size = lib.nbody_workspace_bytes(n, C.byref(cfg))
    ws = C.create_string_buffer(size + 256)
    base = (C.addressof(ws) + 255) // 256 * 256
    rows = [(C.c_double * (n * k))() for k in (1, 3, 3)]
    ctx = vp()
    rc = lib.nbody_init(C.byref(ctx), n, *rows, 1e-4, C.byref(cfg), base, size)
    assert rc == want, rc
    launches = log()
    return ctx, ws
"""

ENERGY = CONTEXT + """
lib.nbody_energy.argtypes = [vp, vp, vp, vp]
out = []
for sizes in ([32767], [65536], [100003], [40000] + [100] * 900, [65536] + [256] * 300, [40000, 40000],
              [65536, 30000, 30000, 30000]):
    ctx, ws = context(sizes)
    assert lib.nbody_energy(ctx, None, None, None) == 0
    out.append((sizes, [q for q in log() if "energy_kernel" in q[0]]))
    lib.nbody_free(ctx)
print(json.dumps(out))
"""


def test_energy_shape_of_mixed_clusters(host):
    for sizes, launches in host(ENERGY):
        (name, gx, gy, _), = launches
        per_lane = int(re.search(r"energy_kernelIL[ib]\dELi(\d)E", name).group(1))
        what = (sizes[:2], len(sizes), gx, gy, per_lane)
        # particle slots of the workgroups, at most an eighth above one
        # particle per lane (and one idle workgroup per cluster in the grid)
        slots = sum(-(-k // (256 * per_lane)) * 256 * per_lane for k in sizes)
        assert slots <= 1.125 * sum(-(-k // 256) * 256 for k in sizes), what
        # the largest cluster's windows spread over the chip
        assert max(sizes) // (256 * per_lane) * gy >= 2048, what
        if min(sizes) >= 40000:
            assert per_lane == 2, what


STARTUP = CONTEXT + """
out = []
for sizes in ([4096], [40000], [4096] + [256] * 500, [16384] + [2048] * 100, [1000] + [33] * 50, [256] * 3000,
              [2000] + [60] * 300):
    ctx, ws = context(sizes, startup=True)
    out.append((sizes, [q for q in launches if "startup_kernel" in q[0]]))
    lib.nbody_free(ctx)
print(json.dumps(out))
"""


def test_startup_shape_of_mixed_clusters(host):
    for sizes, launches in host(STARTUP):
        assert len(launches) == 2
        for name, gx, gy, _ in launches:
            lpi, ipt = (int(q) for q in re.search(r"startup_kernelILi\dELi(\d+)ELi(\d)E", name).groups())
            ib = 256 // lpi * ipt
            blocks = [(-(-k // ib), -(-k // 256)) for k in sizes]     # workgroups, tiles each
            what = (sizes[:2], len(sizes), lpi, ipt, gy)
            # pair slots that hold no particle: at most an eighth more than with one per lane
            assert sum(b * ib * t for b, t in blocks) <= 1.125 * sum(256 * t * t for _, t in blocks), what
            # no walk is longer than half of a compute unit's share of the units,
            # unless twice the splits' partial sums exceed the split buffer
            n = sum(sizes)
            longest = max(t for _, t in blocks) / gy
            assert (longest <= max(1, sum(b * t for b, t in blocks) / 512) or
                    12 * gy * n > 10 * max(2 * n, 1 << 20)), what


BLOCKS = CONTEXT + """
out = []
def state(what):
    out.append((what, var("stub_mallocs").value, var("stub_frees").value))
EDEVICE, DEAD = -2, 709
a, ws = context([64])
lib.nbody_free(a)
b, ws = context([64])
state("kept")
var("stub_sync_rc").value = DEAD             # the stream is gone: no wait is possible
lib.nbody_free(b)
var("stub_sync_rc").value = 0
c, ws = context([64])
state("not kept after a failed wait")
var("stub_sync_rc").value = DEAD
context([64], EDEVICE)
var("stub_sync_rc").value = 0
state("freed by a failed init")
lib.nbody_free(c)
C.c_void_p.in_dll(stub, "stub_block").value = None   # a device reset: old blocks are unknown
var("stub_mapped_rc").value = 1
d, ws = context([64])
state("forgotten after a reset")
e, ws = context([64, 64])
lib.nbody_free(d)
lib.nbody_free(e)
state("two at once")
print(json.dumps(out))
"""


def test_pinned_words_of_closed_contexts(host):
    assert host(BLOCKS) == [["kept", 1, 0], ["not kept after a failed wait", 2, 1],
                            ["freed by a failed init", 3, 2], ["forgotten after a reset", 4, 2],
                            ["two at once", 5, 2]]
