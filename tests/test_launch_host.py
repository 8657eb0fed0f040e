"""What the library asks of the HIP runtime, recorded on the CPU: a stand-in for the runtime's entry points takes the
launches (function, grid, dynamic LDS, current device) and the calls that raise a function's LDS limit.  Nothing is
dereferenced on the way to a launch, so the device addresses are made up."""
import ctypes as C
import json
import os
import subprocess
import sys
import textwrap

import pytest

from paper_2605_19561_amd import build

STUB = r"""
#include <hip/hip_runtime.h>
#include <cstdio>
#include <cstdlib>
#include <cstring>
static int device = 0;
static FILE *events = nullptr;
static thread_local struct { dim3 g, b; size_t lds; hipStream_t s; } config;
extern "C" {
void stub_open(const char *path) { events = fopen(path, "w"); }
void stub_close() { fclose(events); }
void stub_device(int d) { device = d; }
hipError_t hipGetDevice(int *d) { *d = device; return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600 *p, int) {
  memset(p, 0, sizeof *p);
  strcpy(p->gcnArchName, "gfx950");
  return hipSuccess;
}
hipError_t hipMalloc(void **p, size_t n) { return posix_memalign(p, 256, n) ? hipErrorOutOfMemory : hipSuccess; }
hipError_t hipFree(void *p) { free(p); return hipSuccess; }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) { memcpy(d, s, n); return hipSuccess; }
hipError_t hipFuncSetAttribute(const void *f, hipFuncAttribute, int v) {
  fprintf(events, "{\"raise\": %zu, \"bytes\": %d, \"device\": %d}\n", (size_t)f, v, device);
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void *f, dim3 g, dim3, void **, size_t lds, hipStream_t) {
  fprintf(events, "{\"launch\": %zu, \"grid\": [%u, %u], \"lds\": %zu, \"device\": %d}\n", (size_t)f, g.x, g.y, lds, device);
  return hipSuccess;
}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, hipStream_t s) { config = {g, b, lds, s}; return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *lds, hipStream_t *s) {
  *g = config.g; *b = config.b; *lds = config.lds; *s = config.s;
  return hipSuccess;
}
}
"""

# the child loads the stand-in globally before the library, so that the library's calls bind to it
CHILD = """
import array
import ctypes as C, sys
stub = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)
L = C.CDLL(sys.argv[2])
stub.stub_open(sys.argv[3].encode())
vp, i64, sz = C.c_void_p, C.c_int64, C.c_size_t
for name in ("torq_block_gram_workspace_bytes", "torq_linear_workspace_bytes_n", "mxfp4_gemm_workspace_bytes"):
    getattr(L, name).restype = sz
P, BIG = vp(1 << 20), sz(1 << 40)
def gram(fn, M, d, G, ws=BIG):
    return fn(P, i64(M), d, G, P, P, ws, None)
def gemm(M, N, d):
    return L.mxfp4_gemm_ws(P, P, P, P, P, i64(M), i64(N), d, P, BIG, None)
def on(device):
    stub.stub_device(device)
adr = lambda a: vp(a.buffer_info()[0])
def identity(n):
    I = array.array("f", [0.0]) * (n * n)
    for i in range(n): I[i * n + i] = 1.0
    return I
def rotation(d, G):
    I, J, r = identity(G), identity(32), vp()
    assert L.torq_rotation_create(C.byref(r), d, G, adr(I), adr(J)) == 0
    return r
def butterfly(d, G):
    T, J, r = array.array("f", [0.5]) * (G * G), identity(32), vp()
    assert L.torq_rotation_create_butterfly(C.byref(r), d, G, adr(T), adr(J)) == 0
    return r
"""


@pytest.fixture(scope="module")
def stub(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("stub")
    src, lib = str(tmp / "stub.cpp"), str(tmp / "libstub.so")
    open(src, "w").write(STUB)
    subprocess.run(["g++", "-shared", "-fPIC", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", src, "-o", lib], check=True)
    return lib


@pytest.fixture
def record(stub, tmp_path):
    def run(body):
        if not os.path.exists(build.LIB):
            build.build()
        events = str(tmp_path / "events")
        code = CHILD + textwrap.dedent(body) + "\nstub.stub_close()\n"
        subprocess.run([sys.executable, "-c", code, stub, build.LIB, events], check=True, timeout=120)
        return [json.loads(line) for line in open(events)]
    return run


LDS_CALLS = {
    "gram": "assert gram(L.torq_block_gram, 65536, 4096, 128) == 0",
    "positions": "assert gram(L.torq_block_gram_positions, 4096, 4096, 128) == 0",
    "tiled": "assert gemm(2048, 14336, 4096) == 0",
    "streaming": "assert gemm(33, 15616, 15872) == 0",
    "one_launch": """
        r = rotation(28672, 128)
        assert L.torq_linear_single_launch_probe(r, P, P, P, P, i64(64), i64(4096), P, BIG, 1, 0, None) == 0
        """,
}


@pytest.mark.parametrize("name", sorted(LDS_CALLS))
def test_lds_limit_is_raised_on_every_device(record, name):
    # 64 KB is what a launch may ask for without; the limit belongs to a function on ONE device
    call = textwrap.dedent(LDS_CALLS[name])
    events = record("for device in (0, 1, 0):\n    on(device)\n" + textwrap.indent(call, "    "))
    limit, checked = {}, 0
    for e in events:
        if "raise" in e:
            limit[e["raise"], e["device"]] = e["bytes"]
        elif e["lds"] > 64 * 1024:
            checked += 1
            assert limit.get((e["launch"], e["device"]), 0) >= e["lds"], e
    assert checked >= 3, "this call is meant to need more than 64 KB of LDS"
    assert len([e for e in events if "raise" in e]) == len(limit), "once for each function and device"


@pytest.mark.parametrize("G", range(16, 257, 16))
def test_block_gram_reads_its_input_in_one_launch(record, G):
    # one pass over the input and one reduction, whatever the number of tiles
    events = record(f"""
        for M in (1, 4096, 70000):
            assert gram(L.torq_block_gram, M, 32 * {G}, {G}) == 0
            assert gram(L.torq_block_gram_positions, M, 32 * {G}, {G}) == 0
        """)
    assert len([e for e in events if "launch" in e]) == 3 * 2 * 2


@pytest.mark.parametrize("G", range(16, 257, 16))
def test_block_gram_takes_workspaces_of_earlier_sizes(record, G):
    # what the query has returned before: 512 square fp32 results and 16 in double; 32 slices of 32 positions of the
    # tiles of one launch.  Neither may be refused, and no launch may write past it
    nt = G // 16
    tiles = nt * (nt + 1) // 2
    launches = -(-tiles // (36 if nt < 14 else 28))
    sizes = [512 * G * G * 4 + 16 * G * G * 8, 32 * 32 * -(-tiles // launches) * 1024]
    events = record(f"""
        query, least = L.torq_block_gram_workspace_bytes({G}), 2176 * {G} * {G} if {G} <= 128 else 23 << 20
        least = min(query, least)
        for size in {sizes} + [query, least]:
            for fn in (L.torq_block_gram, L.torq_block_gram_positions):
                assert gram(fn, 70000, 32 * {G}, {G}, sz(size)) == 0, size
        for fn in (L.torq_block_gram, L.torq_block_gram_positions):
            assert gram(fn, 70000, 32 * {G}, {G}, sz(least - 1)) == -3
        """)
    launched = [e for e in events if "launch" in e]
    for size, e in zip(sizes, launched[0::4]):
        assert e["grid"][0] * tiles * 1024 <= size


@pytest.mark.parametrize("what,G", [("gram", 32), ("gram", 80), ("gram", 128), ("dense", 80), ("dense", 96), ("dense", 112),
                                    ("dense", 128), ("butterfly", 32), ("butterfly", 64), ("butterfly", 128), ("butterfly", 256)])
def test_inputs_are_read_past_the_cache_from_240_mib_on(record, what, G):
    # a form of its own, where the cache cannot hold the input; below that a program may find it there
    rows = [m * 2 ** 20 // (64 * G) for m in (96, 110, 128, 180, 240)] + [240 * 2 ** 20 // (64 * G) + 1, 2 ** 30 // (64 * G)]
    make = {"gram": f"r = None; call = lambda M: gram(L.torq_block_gram, M, {32 * G}, {G})",
            "dense": f"r = rotation({32 * G}, {G})", "butterfly": f"r = butterfly({32 * G}, {G})"}[what]
    events = record(f"""
        {make}
        if r: call = lambda M: L.torq_rotate_quantize(r, P, i64(M), P, P, None)
        for M in {rows}:
            assert call(M) == 0
        """)
    reads = [e["launch"] for e in events if "launch" in e][:: 2 if what == "gram" else 1]
    assert len(reads) == 7 and len(set(reads[:5])) == 1 and len(set(reads[5:])) == 1 and reads[0] != reads[5]


@pytest.mark.parametrize("what,G", [("rotation", 80), ("rotation", 128), ("butterfly", 32), ("butterfly", 128)])
def test_linear_reads_its_input_past_the_cache_from_96_mib_on(record, what, G):
    # the codes and the output come right behind: the line is lower than for the rotation alone
    rows = [96 * 2 ** 20 // (64 * G) + i for i in (0, 1)]
    events = record(f"""
        r = {what}({32 * G}, {G})
        for M in {rows}:
            assert L.torq_linear(r, P, P, P, P, i64(M), i64(4096), P, BIG, None) == 0
            assert L.torq_rotate_quantize(r, P, i64(M), P, P, None) == 0
        assert L.torq_rotate_quantize(r, P, i64({3 * rows[0]}), P, P, None) == 0
        """)
    launches = [e["launch"] for e in events if "launch" in e]
    plain, once = launches[0], launches[-1]
    assert plain != once and launches.count(plain) == 3 and launches.count(once) == 2
