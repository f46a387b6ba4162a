// host_runtime.cpp -- HIP calls and kernel launchers for running the library's
// host side (corr_runtime.cpp, corr_autotune.cpp) on the CPU, in tests.
//
// Device memory is host memory.  The launchers compute nothing: those that add
// a push to a per-step group's sums record which push they add (its number and
// its first sample, a float), those that copy a push to its row copy it, and
// a write past an allocation is counted and not made.  Any launcher can be told
// to fail once, as it does where the runtime refuses the launch.
#include <hip/hip_runtime.h>

#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

#include "../paper_2503_07526_amd/csrc/corr_kernels.h"

using namespace corr;

namespace {

std::map<char *, size_t> allocations;
std::map<std::string, int> calls, failing; // failing: calls left before the one that fails
struct Added {
    int64_t push;
    float value;
};
std::map<int64_t, std::vector<Added>> added; // by the group's channel count
std::map<int64_t, std::vector<int64_t>> folded; // by channel count: block * 1e6 + tile group, in order
int out_of_range = 0;

hipError_t launched(const char *name)
{
    calls[name] += 1;
    auto f = failing.find(name);
    if (f == failing.end() || f->second-- > 0) return hipSuccess;
    failing.erase(f);
    return hipErrorLaunchFailure;
}

bool inside(const void *p, int64_t bytes)
{
    char *c = static_cast<char *>(const_cast<void *>(p));
    auto it = allocations.upper_bound(c);
    if (it == allocations.begin()) return false;
    --it;
    return c + bytes <= it->first + it->second;
}

void copy_row(const KeepRow &k)
{
    if (k.bytes <= 0) return;
    if (inside(k.dst, k.bytes))
        memcpy(k.dst, k.src, (size_t)k.bytes);
    else
        ++out_of_range;
}

void add(const GroupArgs &g, int64_t before, const void *sample)
{
    added[g.n_ch].push_back({before + 1, *static_cast<const float *>(sample)});
}

hipError_t push_one(const char *name, const GroupArgs &g, StepRef step)
{
    const hipError_t e = launched(name);
    if (e == hipSuccess) add(g, step.count, g.samples);
    return e;
}

// The tile groups that a fold launch covers, and their block.
void fold(const DeferredArgs &a)
{
    int64_t q = a.fixed_block, j0, j1;
    if (a.fixed_group == -2) {
        j0 = a.tile_first / a.tiles_per_group;
        j1 = (a.tile_end + a.tiles_per_group - 1) / a.tiles_per_group;
    } else {
        const int64_t s = a.step.count + 1;
        q = s / a.g.defer_t;
        j0 = s % a.g.defer_t;
        j1 = j0 + 1;
    }
    for (int64_t j = j0; j < j1; ++j) folded[a.g.n_ch].push_back(q * 1000000 + j);
}

} // namespace

extern "C" {

void stub_reset()
{
    calls.clear();
    failing.clear();
    added.clear();
    folded.clear();
    out_of_range = 0;
}
void stub_fail(const char *name, int after) { failing[name] = after; }
int stub_calls(const char *name) { return calls[name]; }
int stub_out_of_range() { return out_of_range; }
int64_t stub_allocated()
{
    int64_t n = 0;
    for (const auto &a : allocations) n += (int64_t)a.second;
    return n;
}
int stub_added(int64_t n_ch, int64_t *push, float *value, int cap)
{
    const auto &v = added[n_ch];
    for (int i = 0; i < (int)v.size() && i < cap; ++i) {
        push[i] = v[(size_t)i].push;
        value[i] = v[(size_t)i].value;
    }
    return (int)v.size();
}

int stub_folded(int64_t n_ch, int64_t *out, int cap)
{
    const auto &v = folded[n_ch];
    for (int i = 0; i < (int)v.size() && i < cap; ++i) out[i] = v[(size_t)i];
    return (int)v.size();
}

// ------------------------------------------------------------------ HIP
hipError_t hipMalloc(void **p, size_t bytes)
{
    *p = calloc(1, bytes ? bytes : 1);
    allocations[static_cast<char *>(*p)] = bytes;
    return hipSuccess;
}
hipError_t hipFree(void *p)
{
    allocations.erase(static_cast<char *>(p));
    free(p);
    return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t bytes, unsigned) { return hipMalloc(p, bytes); }
hipError_t hipHostFree(void *p) { return hipFree(p); }
hipError_t hipMemGetInfo(size_t *f, size_t *t)
{
    *f = *t = (size_t)1 << 34;
    return hipSuccess;
}
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind)
{
    memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t)
{
    memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemsetAsync(void *d, int v, size_t n, hipStream_t)
{
    memset(d, v, n);
    return hipSuccess;
}
hipError_t hipGetSymbolAddress(void **p, const void *s)
{
    *p = const_cast<void *>(s);
    return hipSuccess;
}
hipError_t hipGetDevice(int *d)
{
    *d = 0;
    return hipSuccess;
}
hipError_t hipGetDeviceCount(int *n)
{
    *n = 1;
    return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int)
{
    *v = 256;
    return hipSuccess;
}
hipError_t hipGetDeviceProperties(hipDeviceProp_t *, int) { return hipErrorInvalidDevice; }
hipError_t hipGetLastError() { return launched("last_error"); }
const char *hipGetErrorString(hipError_t) { return "refused"; }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned)
{
    *s = reinterpret_cast<hipStream_t>(malloc(1));
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s)
{
    free(s);
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return launched("synchronize"); }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *g)
{
    *g = nullptr;
    return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t *x, hipGraph_t, hipGraphNode_t *, char *, size_t)
{
    *x = nullptr;
    return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *e)
{
    *e = nullptr;
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned)
{
    *e = nullptr;
    return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t)
{
    *ms = 0.f;
    return hipSuccess;
}

} // extern "C"

// ------------------------------------------------------------- launchers
namespace corr {

bool multi_supported(int, int p, int m, bool) { return m == 2 && (p == 16 || p == 24 || p == 32); }
bool deferred_supported(int kind, int p, int m) { return kind <= K_F32_F32 && p == 16 && m == 2; }
bool window_deferred_supported(int) { return true; }
int window_lags_per_block(int p) { return (p + kWindowT - 1) / kWindowT; }
bool window_folds_share_launch(const GroupArgs &, const GroupArgs &) { return false; }
int rhok_mfma_cols() { return 16; }
int rhok_mfma_max_nmax() { return 15; }
int rhok_mfma_chunks(int, int) { return 1; }
int rhok_mfma_blocks_per_cu(int, int, int) { return 1; }
hipError_t rhok_mfma_prepare(int, int, int) { return hipSuccess; }
int momentum_blocks(int64_t) { return 1; }
int64_t deferred_readout_rows(const GroupArgs &g) { return g.n_tiles * (int64_t)g.tw / 64; }
int64_t deferred_readout_group_rows() { return 1024; }
int64_t deferred_readout_groups(const GroupArgs &g) { return (deferred_readout_rows(g) + 1023) / 1024; }

hipError_t launch_keep_rows(KeepArgs &a, hipStream_t)
{
    const hipError_t e = launched("keep_rows");
    for (int i = 0; e == hipSuccess && i < a.n; ++i) copy_row(a.row[i]);
    return e;
}
hipError_t launch_multi_push(const GroupArgs &g, StepRef step, const void *rows, int64_t stride, int n, hipStream_t)
{
    if (n < 1 || n > kMultiT) return hipErrorInvalidValue;
    const hipError_t e = launched("multi_push");
    for (int r = 0; e == hipSuccess && r < n; ++r)
        add(g, step.count + r, static_cast<const char *>(rows) + r * stride);
    return e;
}
hipError_t launch_push_batched(const PushArgs &a, int, int, int, int, hipStream_t)
{
    const hipError_t e = launched("push_batched");
    for (int i = 0; e == hipSuccess && i < a.n_groups; ++i) add(a.g[i], a.step.count, a.g[i].samples);
    return e;
}
hipError_t launch_push_group(const GroupArgs &g, StepRef step, int, int, int, hipStream_t)
{
    return push_one("push_group", g, step);
}
hipError_t launch_push_split(const GroupArgs &g, StepRef step, int, int, int, int, hipStream_t)
{
    return push_one("push_split", g, step);
}
hipError_t launch_push_window(const GroupArgs &g, StepRef step, int, int, int, int, hipStream_t)
{
    return push_one("push_window", g, step);
}
hipError_t launch_window_fold(const GroupArgs &, StepRef, hipStream_t) { return launched("window_fold"); }
hipError_t launch_window_fold2(const GroupArgs &, const GroupArgs &, StepRef, hipStream_t)
{
    return launched("window_fold2");
}
hipError_t launch_rhok(const RhokArgs &, hipStream_t) { return launched("producer"); }
hipError_t launch_rhok_mfma(const RhokMfmaArgs &, const KeepRow &rider, hipStream_t)
{
    const hipError_t e = launched("producer");
    if (e == hipSuccess) copy_row(rider);
    return e;
}
hipError_t launch_momentum(const MomentumArgs &, const KeepRow &rider, hipStream_t)
{
    const hipError_t e = launched("producer");
    if (e == hipSuccess) copy_row(rider);
    return e;
}
hipError_t launch_stage(const GroupArgs &, StepRef, hipStream_t) { return launched("stage"); }
hipError_t launch_stage_rows(const GroupArgs &, StepRef, int64_t, int, hipStream_t) { return launched("stage"); }
hipError_t launch_flush_fold(const DeferredArgs &a, hipStream_t)
{
    const hipError_t e = launched("fold");
    if (e == hipSuccess) fold(a);
    return e;
}
hipError_t launch_history_fold(const DeferredArgs &a, hipStream_t)
{
    const hipError_t e = launched("history_fold");
    if (e == hipSuccess) fold(a);
    return e;
}
hipError_t launch_push_end(const PushEndArgs &, hipStream_t) { return launched("push_end"); }
hipError_t launch_reduce(const ReduceArgs &, hipStream_t) { return launched("reduce"); }
hipError_t launch_gather(const ReduceArgs &, hipStream_t) { return launched("gather"); }
hipError_t launch_deferred_readout_pass(const DeferredArgs &, double *, hipStream_t) { return launched("readout"); }
hipError_t launch_deferred_readout_final(const DeferredArgs &, const double *, double *, hipStream_t)
{
    return launched("readout");
}

} // namespace corr
