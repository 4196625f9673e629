"""Dynamic LDS of every launch, on the host alone: the library runs against a HIP runtime of a few lines that launches nothing and
writes down what it was asked for."""
import json
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

RUNTIME = r"""
#include <cstddef>
#include <cstdint>
#include <cstdio>
#include <map>
#include <string>
struct dim3 { uint32_t x, y, z; };
static dim3 grid_, block_;
static size_t lds_;
static void* stream_;
static std::map<const void*, std::string>& names() { static std::map<const void*, std::string> m; return m; }
static std::map<const void*, int> allowed;
static FILE* out() { static FILE* f = fopen(LOG, "w"); return f; }
extern "C" {
void** __hipRegisterFatBinary(const void*) { static void* h; return &h; }
void __hipRegisterFunction(void**, const void* f, char*, const char* name, unsigned, void*, void*, void*, void*, int*) { names()[f] = name; }
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipUnregisterFatBinary(void**) {}
int __hipPushCallConfiguration(dim3 g, dim3 b, size_t l, void* s) { grid_ = g; block_ = b; lds_ = l; stream_ = s; return 0; }
int __hipPopCallConfiguration(dim3* g, dim3* b, size_t* l, void** s) { *g = grid_; *b = block_; *l = lds_; *s = stream_; return 0; }
int hipFuncSetAttribute(const void* f, int, int v) { allowed[f] = v; return 0; }
int hipLaunchKernel(const void* f, dim3, dim3, void**, size_t lds, void*) {
    fprintf(out(), "%zu %d %s\n", lds, allowed.count(f) ? allowed[f] : 65536, names()[f].c_str());
    fflush(out());
    return 0;
}
int hipGetLastError() { return 0; }
int hipMemcpyAsync(void*, const void*, size_t, int, void*) { return 0; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) { *n = 2; return 0; }
}
"""

# arguments: the recording runtime, then a list of [channels, taps]; a greedy iteration, a module step and a MoDL step of each network
CALLS = r"""
import ctypes as C, json, sys
C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)
from paper_2207_08393_amd import binding as gb, synth
L = gb.lib()
geom = gb.make_geom(synth.Geom(2, 1, 2, 6, 1, 64, 96))
p = lambda i: i << 40
ok = lambda rc: rc == 0 or sys.exit(gb.strerror(rc))
for chans, taps in json.loads(sys.argv[2]):
    prox = gb.make_prox(synth.chain_prox(chans, [tuple(t) for t in taps]))
    ws, saved = gb.gleam_workspace_bytes(geom, prox)
    ok(L.gleam_greedy_iteration(C.byref(geom), C.byref(prox), 1, p(1), p(2), p(3), p(4), C.c_float(1), p(5), p(6), p(7), C.byref(gb.make_adam(1e-3)), 1,
                                p(8), p(9), p(10), p(11), p(12), p(13), saved, p(14), ws, None))
    ok(L.gleam_module_fwd(C.byref(geom), C.byref(prox), p(1), p(2), p(3), p(4), C.c_float(1), p(5), p(8), p(9), p(11), p(13), saved, p(14), ws, None))
    ok(L.gleam_module_bwd(C.byref(geom), C.byref(prox), p(5), p(13), saved, p(12), p(14), ws, None))
    ws, saved = gb.gleam_modl_workspace_bytes(geom, prox)
    ok(L.gleam_modl_module_fwd(C.byref(geom), C.byref(prox), p(1), p(2), p(3), p(4), C.c_float(1), 2, p(5), p(8), p(9), p(11), p(13), saved, p(14), ws, None))
    ok(L.gleam_modl_module_bwd(C.byref(geom), C.byref(prox), p(2), p(3), C.c_float(1), 2, p(5), p(13), saved, p(12), p(14), ws, None))
"""

KS, KT = (1, 1, 3, 3), (3, 1, 1, 1)


# the two forms of the covering weight gradient, one behind the other; temporal layers whose weights take more than 64 KB of LDS: two
# blocks of output channels by four chunks, one by eight
@pytest.mark.parametrize("nets,kernels", [([([2, 100, 100, 2], [KS] * 3), ([2, 100, 68, 2], [KS] * 3)], ["wgrad_cover_kernel<3>", "wgrad_cover_kernel<2>"]),
                                          ([([2, 64, 64, 2], [KS, KT, KS]), ([2, 128, 32, 2], [KS, KT, KS])],
                                           ["conv_time_split_kernel<4, false>", "conv_time_split_kernel<4, true>", "conv_time_split_kernel<8, false>"])],
                         ids=["cover", "time"])
def test_launches_beyond_64_kb_of_lds_are_allowed_it(nets, kernels, tmp_path):
    source, runtime, log = tmp_path / "runtime.cpp", tmp_path / "runtime.so", tmp_path / "launches"
    source.write_text(RUNTIME)
    subprocess.run(["g++", "-shared", "-fPIC", "-O1", f'-DLOG="{log}"', str(source), "-o", str(runtime)], check=True)
    subprocess.run([sys.executable, "-c", CALLS, str(runtime), json.dumps(nets)], check=True, cwd=ROOT)
    launches = [line.split(" ", 2) for line in log.read_text().splitlines()]
    names = subprocess.run(["c++filt"], input="\n".join(n for _, _, n in launches), capture_output=True, text=True, check=True).stdout.splitlines()
    beyond = {n: (int(lds), int(may)) for n, (lds, may, _) in zip(names, launches) if int(lds) > 65536}
    for k in kernels:
        assert any(k in n for n in beyond), (k, beyond)
    assert all(lds <= may for lds, may in beyond.values()), beyond
