"""Host build of the wavefront kernels for logic checks without a GPU.

``rt_stream.hip``, ``rt_cascade.hip`` and, for its geometry, ``rt_deep.hip`` of
``paper_2203_02293_amd/csrc`` are compiled for the host whole, launchers included.  Each
launch runs its workgroups one after another, every GPU thread a fiber of one OS thread:
a fiber runs until it meets a barrier of the workgroup or of its wavefront (shuffles,
votes and ``wave_sync`` are wavefront barriers), so runs are deterministic, and a barrier
that some thread does not reach is an error.  Dynamic LDS is a host buffer, poisoned, with
an inaccessible page right after its last byte; a launch that asks for more of it than
the kernel was set up for is an error, as it is on the GPU.  Where lanes of a wavefront
rely on running in lockstep (LOCKSTEP) the build adds a barrier of those lanes.  Device intrinsics take their host
branch, so results differ from the GPU's in the last bits only.  Test infrastructure:
only the tests use it.
"""
import os
import pathlib
import re
import subprocess

ROOT = pathlib.Path(__file__).resolve().parents[2]
CSRC = ROOT / "paper_2203_02293_amd" / "csrc"
# one folder per process: parallel test workers each build their own copy
OUT = pathlib.Path("/tmp") / f"rt_host_emu_{os.getpid()}"

EMU = r'''// generated by tests/host_emu/wave_build.py -- do not edit
#pragma once
#include <algorithm>
#include <cstring>
#include <functional>
#include <map>
#include <vector>
#include <sys/mman.h>
#include <ucontext.h>
#include <unistd.h>
#include "rt_internal.hpp"
#include "rt_math.hpp"
#include "rt_physics.hpp"
using std::min; using std::max;

struct EmuIdx { int x, y, z; };
inline EmuIdx emu_block, emu_grid;
inline int emu_tid, emu_W;
inline double *emu_smem;
inline hipError_t emu_err = hipSuccess;

// Bytes ending right before an inaccessible page, every double a NaN.
struct EmuLds {
    void *map = nullptr;
    size_t len = 0;
    double *p = nullptr;
    explicit EmuLds(size_t bytes) {
        const size_t pg = (size_t)sysconf(_SC_PAGESIZE), body = (bytes + pg - 1) / pg * pg;
        len = body + pg;
        map = mmap(nullptr, len, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS, -1, 0);
        mprotect((char *)map + body, pg, PROT_NONE);
        std::memset(map, 0xFF, body);
        p = (double *)((char *)map + body - (bytes + 15) / 16 * 16);
    }
    ~EmuLds() { munmap(map, len); }
};

// A fiber waits for the `width` threads of its aligned group (0: the workgroup).
struct EmuFiber {
    ucontext_t ctx;
    int width = -1;   // -1: runnable
    bool done = false;
};
constexpr size_t kEmuStack = 256 * 1024;
inline std::vector<EmuFiber> emu_fib;
inline ucontext_t emu_main;
inline const std::function<void()> *emu_body;
inline double emu_x[1024];
inline void emu_wait(int width)
{
    EmuFiber &f = emu_fib[emu_tid];
    f.width = width;
    swapcontext(&f.ctx, &emu_main);
}
inline void emu_entry()
{
    (*emu_body)();
    emu_fib[emu_tid].done = true;
    swapcontext(&emu_fib[emu_tid].ctx, &emu_main);
}
// one workgroup of W threads; false: a barrier that not all threads reach
inline bool emu_workgroup(int W, const std::function<void()> &body)
{
    static char *stacks = (char *)mmap(nullptr, 1024 * kEmuStack, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
    emu_fib.assign(W, EmuFiber());
    emu_body = &body;
    emu_W = W;
    for (int t = 0; t < W; ++t) {
        getcontext(&emu_fib[t].ctx);
        emu_fib[t].ctx.uc_stack.ss_sp = stacks + t * kEmuStack;
        emu_fib[t].ctx.uc_stack.ss_size = kEmuStack;
        emu_fib[t].ctx.uc_link = nullptr;
        makecontext(&emu_fib[t].ctx, emu_entry, 0);
    }
    for (;;) {
        bool ran = false;
        for (int t = 0; t < W; ++t)
            if (!emu_fib[t].done && emu_fib[t].width < 0) {
                emu_tid = t;
                ran = true;
                swapcontext(&emu_main, &emu_fib[t].ctx);
            }
        bool left = false;
        for (int t = 0; t < W; ++t) {
            if (emu_fib[t].done || emu_fib[t].width < 0) continue;
            left = true;
            const int w = emu_fib[t].width, n = w ? w : W, t0 = t / n * n;
            bool all = true;
            for (int u = t0; u < min(t0 + n, W); ++u) all = all && (emu_fib[u].done || emu_fib[u].width == w);
            if (!all) continue;
            ran = true;
            for (int u = t0; u < min(t0 + n, W); ++u) emu_fib[u].width = -1;
        }
        if (!left) {
            bool done = true;
            for (int t = 0; t < W; ++t) done = done && emu_fib[t].done;
            if (done) return true;
        }
        if (!ran) return false;
    }
}
inline void emu_wave_sync() { emu_wait(64); }
inline void emu_lanes_sync(int n) { emu_wait(n); }
inline void emu_sync() { emu_wait(0); }
inline double emu_shfl_xor(double v, int m)
{
    emu_x[emu_tid] = v;
    emu_wait(64);
    const double o = emu_x[emu_tid ^ m];
    emu_wait(64);
    return o;
}
inline bool emu_wave_any(bool c)
{
    emu_x[emu_tid] = c;
    emu_wait(64);
    bool any = false;
    for (int t = emu_tid & ~63; t < (emu_tid & ~63) + 64; ++t) any = any || emu_x[t] != 0.0;
    emu_wait(64);
    return any;
}
inline uint32_t emu_atomic_or(uint32_t *p, uint32_t v) { const uint32_t o = *p; *p |= v; return o; }
inline int emu_lo(double v) { return (int)(uint32_t)__builtin_bit_cast(uint64_t, v); }
inline int emu_hi(double v) { return (int)(__builtin_bit_cast(uint64_t, v) >> 32); }
inline double emu_hilo(int h, int l) { return __builtin_bit_cast(double, (uint64_t)(uint32_t)h << 32 | (uint32_t)l); }
inline int emu_f2i(float v) { return __builtin_bit_cast(int, v); }
inline float emu_i2f(int v) { return __builtin_bit_cast(float, v); }
inline int emu_frexp_exp(double v) { int e; (void)frexp(v, &e); return e; }

// the dynamic LDS each kernel was set up for (64 KiB without a call), and what its launches ask for
inline std::map<const void *, size_t> emu_limit, emu_asked;
inline hipError_t emu_set_lds(const void *f, int bytes) { emu_limit[f] = (size_t)bytes; return hipSuccess; }
inline bool emu_dry = false;   // launches check their LDS and run nothing
template <class F>
void emu_launch(const void *kernel, F f, dim3 grid, dim3 block, size_t lds)
{
    const size_t limit = emu_limit.count(kernel) ? emu_limit[kernel] : 65536;
    emu_asked[kernel] = max(emu_asked[kernel], lds);
    if (lds > limit) emu_err = hipErrorInvalidValue;
    if (emu_err != hipSuccess || emu_dry) return;
    emu_grid = {(int)grid.x, (int)grid.y, (int)grid.z};
    const std::function<void()> body = f;
    for (unsigned z = 0; z < grid.z; ++z)
        for (unsigned y = 0; y < grid.y; ++y)
            for (unsigned x = 0; x < grid.x; ++x) {
                EmuLds smem(lds > 0 ? lds : 8);
                emu_smem = smem.p;
                emu_block = {(int)x, (int)y, (int)z};
                if (!emu_workgroup((int)block.x, body)) {
                    emu_err = hipErrorLaunchFailure;
                    return;
                }
            }
}
inline hipError_t emu_last_error() { const hipError_t e = emu_err; emu_err = hipSuccess; return e; }
#define EMU_LAUNCH(k, grid, block, lds, stream, ...) \
    emu_launch((const void *)(k), [=]() { (k)(__VA_ARGS__); }, dim3(grid), dim3(block), (size_t)(lds))
'''

MAIN = r'''
#include "emu.hpp"
using namespace rtk;
static void setup(const DeviceLimits &dev)
{
    (void)prepare_stream_kernels(dev);
    (void)prepare_cascade_kernels(dev);
}
extern "C" void emu_stream_geometry(int C, int N, int NB, int NG, int mixed, int ncu, int lds, long long *o)
{
    const Geometry g = stream_geometry(C, N, NB, NG, mixed != 0, DeviceLimits{ncu, (size_t)lds});
    o[0] = g.K; o[1] = g.PC; o[2] = g.CH; o[3] = g.threads; o[4] = g.blocks; o[5] = (long long)g.lds;
    o[6] = (long long)g.scratch;
}
extern "C" int emu_stream_solve(const SolveArgs *a, int mixed, int ncu, int lds)
{
    const DeviceLimits dev{ncu, (size_t)lds};
    setup(dev);
    const Geometry g = stream_geometry(a->C, a->N, a->NB, a->NG, mixed != 0, dev);
    return g.threads == 0 ? -1 : (int)launch_stream(*a, g, mixed ? 1 : 0, nullptr);
}
// n requests as one batch (all in one shape class: the first's threads, segmented or not)
extern "C" int emu_stream_batch(const SolveArgs *reqs, int n, int mixed, int ncu, int lds, int dry)
{
    const DeviceLimits dev{ncu, (size_t)lds};
    setup(dev);
    std::vector<SolveArgs> a(reqs, reqs + n);
    std::vector<int> first(n);
    Geometry gb{};
    int blocks = 0, layers = 0;
    for (int r = 0; r < n; ++r) {
        const Geometry g = stream_geometry(a[r].C, a[r].N, a[r].NB, a[r].NG, mixed != 0, dev);
        if (g.threads == 0) return -1;
        if (r == 0) gb = g;
        if (g.threads != gb.threads || (g.PC > 1) != (gb.PC > 1)) return -2;
        a[r].K = g.K; a[r].PC = g.PC; a[r].CH = g.CH; a[r].L = g.lanes;
        gb.lds = max(gb.lds, g.lds);
        first[r] = blocks;
        blocks += g.blocks;
        layers = max(layers, a[r].N);
    }
    emu_dry = dry != 0;
    const int e = (int)BATCH;
    emu_dry = false;
    return e;
}
extern "C" int emu_cascade_solve(const SolveArgs *a, int mixed, int ncu, int lds)
{
    const DeviceLimits dev{ncu, (size_t)lds};
    setup(dev);
    const Geometry g = deep_geometry(a->C, a->N, a->NB, dev);
    if (g.threads == 0 || !cascade_fits(g, a->C, a->N, a->NB, a->NG, a->sub != 0, dev)) return -1;
    return (int)launch_cascade(*a, g, mixed ? 1 : 0, nullptr);
}
extern "C" long long emu_deep_scratch(int C, int N, int NB, int ncu, int lds)
{
    return (long long)deep_geometry(C, N, NB, DeviceLimits{ncu, (size_t)lds}).scratch;
}
'''
# places where lanes of a wavefront rely on running in lockstep, and what stands for it here
LOCKSTEP = [("auto step = [&](int q, int k) {", "emu_lanes_sync(NBp);"),   # padding lanes: the same records again
            ("auto edges = [&](double T, int from, int n, bool check) {", "emu_wave_sync();"),   # rows read before
            ("constexpr int RD = MIXED ? 4 : 8;", "emu_wave_sync();")]         # rows in place of the edges
BATCH = ("launch_stream_batch(a.data(), first.data(), n, blocks, layers, gb, a[0].NB, mixed ? 1 : 0, a[0].in_f32, nullptr)")


def _transform(s: str) -> str:
    s = re.sub(r"__launch_bounds__\((?:[^()]|\((?:[^()]|\([^()]*\))*\))*\)\s*", "", s)
    s = re.sub(r"asm volatile\([^;]*;", "(void)0;", s)
    s = re.sub(r"(void wave_sync\(\)\n\{\n)[^}]*\}", r"\1    emu_wave_sync();\n}", s)
    s = re.sub(r"extern __shared__ double (\w+)\[\];", r"double *\1 = emu_smem;", s)
    s = re.sub(r"return hipMemcpyToSymbol\([^;]*;", "memcpy(planck_values, host, sizeof host);\n    return hipSuccess;", s)
    for old, new in (("static __device__ __attribute__((aligned(16)))", "static"), ("__global__ ", ""),
                     ("__shared__ ", "static "), ("threadIdx.x", "emu_tid"), ("blockIdx.", "emu_block."),
                     ("gridDim.", "emu_grid."), ("blockDim.x", "emu_W"), ("__syncthreads()", "emu_sync()"),
                     ("atomicOr(", "emu_atomic_or("), ("hipLaunchKernelGGL(", "EMU_LAUNCH("),
                     ("hipGetLastError()", "emu_last_error()"), ("wave_any(", "emu_wave_any("),
                     ("__shfl_xor(", "emu_shfl_xor("), ("__double2loint(", "emu_lo("), ("__double2hiint(", "emu_hi("),
                     ("__hiloint2double(", "emu_hilo("), ("__float_as_int(", "emu_f2i("), ("__int_as_float(", "emu_i2f("),
                     ("__builtin_amdgcn_frexp_exp(", "emu_frexp_exp("), ("__host__ __device__ __forceinline__", "inline"),
                     ("__device__ __forceinline__", "inline"), ("__host__ __device__ inline", "inline"),
                     ("__host__ __device__ constexpr", "constexpr"), ('#include "rt_wave.hpp"', ""),
                     ('#include "rt_internal.hpp"', '#include "emu.hpp"')):
        s = s.replace(old, new)
    s = re.sub(r"hipFuncSetAttribute\(([^;]*?),\s*hipFuncAttributeMaxDynamicSharedMemorySize,", r"emu_set_lds(\1,", s)
    for before, sync in LOCKSTEP:
        s = s.replace(before, before + "\n" + sync if before.endswith("{") else sync + "\n" + before)
    return s


def build() -> pathlib.Path:
    """Generate and compile the host build; returns the shared library."""
    OUT.mkdir(exist_ok=True)
    (OUT / "emu.hpp").write_text(EMU)
    (OUT / "rt_lanes.hpp").write_text(_transform((CSRC / "rt_lanes.hpp").read_text()))
    srcs = []
    for name in ("rt_stream", "rt_cascade", "rt_deep"):
        s = _transform((CSRC / f"{name}.hip").read_text())
        srcs.append(OUT / f"{name}_wave.cpp")
        srcs[-1].write_text('#include "emu.hpp"\n' + s)
    srcs.append(OUT / "wave_main.cpp")
    srcs[-1].write_text(MAIN.replace("BATCH", BATCH))
    lib = OUT / "librt_wave_emu.so"
    cmd = ["hipcc", "-O1", "-std=c++20", "-fPIC", "-shared", f"-I{OUT}", f"-I{ROOT / 'include'}", f"-I{CSRC}",
           *map(str, srcs), "-o", str(lib)]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("host build failed:\n" + r.stderr[-5000:])
    return lib
