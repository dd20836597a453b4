"""Setting parameters when an allocation fails (no GPU): the library on a stand-in for the HIP runtime, defined by a small
host program, whose n-th allocation fails.  Whichever it is, the call says so, the net has no parameters after it (a pass is
refused, not run on what was allocated before the failure), the next call succeeds, and nothing is left at the end."""
import os
import subprocess

from paper_1302_1690_amd import mpcnn

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <dlfcn.h>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <set>
#include <vector>
#include "mpcnn.h"
struct dim3_like { unsigned x, y, z; };
namespace {
int until_failure = -1, calls = 0;
std::set<void*> held;
int error = 0, last = 0;
int take(void** p, size_t n)
{
    ++calls;
    if (until_failure == 0) { until_failure = -1; return last = 2; }
    if (until_failure > 0) --until_failure;
    *p = calloc(1, n ? n : 1);
    held.insert(*p);
    return 0;
}
int give(void* p)
{
    if (p && !held.erase(p)) error = 1;
    free(p);
    return 0;
}
char image[1 << 24];   // the library's own array on the device
}
#define FAKE extern "C" __attribute__((visibility("default"), used)) int
FAKE hipMalloc(void** p, size_t n) { return take(p, n); }
FAKE hipHostMalloc(void** p, size_t n, unsigned) { return take(p, n); }
FAKE hipFree(void* p) { return give(p); }
FAKE hipHostFree(void* p) { return give(p); }
FAKE hipGetDevice(int* d) { *d = 0; return 0; }
FAKE hipSetDevice(int) { return 0; }
FAKE hipMemset(void* p, int v, size_t n) { memset(p, v, n); return 0; }
FAKE hipMemcpy(void* d, const void* s, size_t n, int) { memcpy(d, s, n); return 0; }
FAKE hipDeviceSynchronize() { return 0; }
FAKE hipStreamSynchronize(void*) { return 0; }
FAKE hipFuncSetAttribute(const void*, int, int) { return 0; }
FAKE hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) { *n = 2; return 0; }
FAKE hipGetSymbolAddress(void** p, const void*) { *p = image; return 0; }
FAKE hipGetLastError() { const int e = last; last = 0; return e; }
FAKE __hipPushCallConfiguration(dim3_like, dim3_like, size_t, void*) { return 0; }
FAKE __hipPopCallConfiguration(void*, void*, size_t*, void*) { return 0; }
int launches = 0;
FAKE hipLaunchKernel(const void*, dim3_like, dim3_like, void**, size_t, void*) { ++launches; return 0; }

template <typename F> F* sym(void* lib, const char* name) { return reinterpret_cast<F*>(dlsym(lib, name)); }

int main(int, char** argv)
{
    void* lib = dlopen(argv[1], RTLD_NOW);
    if (!lib) { printf("%s\n", dlerror()); return 2; }
    auto create = sym<decltype(mpcnn_net_create)>(lib, "mpcnn_net_create");
    auto destroy = sym<decltype(mpcnn_net_destroy)>(lib, "mpcnn_net_destroy");
    auto count = sym<decltype(mpcnn_param_count)>(lib, "mpcnn_param_count");
    auto set = sym<decltype(mpcnn_set_params)>(lib, "mpcnn_set_params");
    auto get = sym<decltype(mpcnn_get_params)>(lib, "mpcnn_get_params");
    auto need = sym<decltype(mpcnn_workspace_bytes)>(lib, "mpcnn_workspace_bytes");
    auto forward = sym<decltype(mpcnn_seg_forward)>(lib, "mpcnn_seg_forward");
    const mpcnn_layer_desc layers[] = {{MPCNN_C, 16, 3, 0}, {MPCNN_MP, 0, 2, 0}, {MPCNN_C, 16, 2, 0}, {MPCNN_FC, 250, 0, 0}, {MPCNN_FC, 2, 0, 0}};
    for (int bf16 = 0; bf16 < 2; ++bf16)
        for (int fail = -1; fail < 8; ++fail) {
            mpcnn_net* net = nullptr;
            if (create(layers, 5, 1, 6, bf16 ? MPCNN_BF16 : MPCNN_F32, &net) != MPCNN_OK) return 3;
            const size_t n = count(net);
            std::vector<float> p(n), q(n);
            std::vector<char> image(4 * 20 * 20 + 16), probs(1 << 16);
            const size_t bytes = need(net, 1, 20, 20, 0);
            void* ws = aligned_alloc(256, (bytes + 255) / 256 * 256);
            float* img = reinterpret_cast<float*>((reinterpret_cast<size_t>(image.data()) + 15) & ~size_t(15));
            until_failure = fail; calls = 0;
            const mpcnn_status first = set(net, p.data(), n);
            const bool failed = fail >= 0 && calls > fail;
            if (failed != (first != MPCNN_OK)) { printf("allocation %d of %d: status %d\n", fail, calls, (int)first); return 4; }
            if (failed) {
                launches = 0;
                if (forward(net, img, 1, 20, 20, reinterpret_cast<float*>(probs.data()), ws, bytes, nullptr) == MPCNN_OK || launches) {
                    printf("allocation %d failed and a pass ran\n", fail); return 5;
                }
                if (get(net, q.data(), n) == MPCNN_OK) { printf("allocation %d failed and parameters were read\n", fail); return 6; }
                until_failure = -1;
                if (set(net, p.data(), n) != MPCNN_OK) { printf("allocation %d failed once, and again\n", fail); return 7; }
            }
            until_failure = -1;
            if (forward(net, img, 1, 20, 20, reinterpret_cast<float*>(probs.data()), ws, bytes, nullptr) != MPCNN_OK) return 8;
            destroy(net);
            free(ws);
            if (error || !held.empty()) { printf("allocation %d: %zu left, %d freed twice\n", fail, held.size(), error); return 9; }
            if (fail < 0) printf("%d allocations\n", calls);
        }
    printf("done\n");
    return 0;
}
"""


def test_set_params_when_an_allocation_fails(tmp_path):
    src = tmp_path / "fake.cpp"
    src.write_text(PROGRAM)
    exe = tmp_path / "fake"
    subprocess.run(["g++", "-std=c++17", "-O1", "-rdynamic", "-I", os.path.join(ROOT, "include"), str(src), "-o", str(exe), "-ldl"],
                   check=True)
    r = subprocess.run([str(exe), mpcnn.LIB_PATH], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.endswith("done\n"), (r.returncode, r.stdout, r.stderr)
    assert "4 allocations" in r.stdout and "5 allocations" in r.stdout, r.stdout   # (one more with bf16 storage)
