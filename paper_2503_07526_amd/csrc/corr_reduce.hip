// corr_reduce.hip -- readout support (Algorithm 2): per-(level, lag) sums of
// the accumulators over a channel range, in double precision, in a fixed
// order (block partials, then partials in block order), plus a gather of the
// accumulators of a channel slice.  A compensated accumulator is read as
// value - compensation, evaluated in double; a one-level window in the
// block-deferred form adds the products of its pending pushes.
#include <hip/hip_runtime.h>

#include "corr_kernels.h"

namespace corr {

// n consecutive (new, lagged) value pairs of a ring of p0 slots in order, eight
// loaded ahead of their products (one pair after the other the sums of 1536
// complex channels at p = 4096 took 113 us instead of 58).
template <typename S, typename F>
__device__ __forceinline__ void pending_products(const S *ring, int tw, int p0, int sx, int sy, int n, F &&add)
{
    constexpr int U = 8;
    for (int i = 0; i < n; i += U) {
        S x[U], y[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            x[u] = ring[(size_t)sx * tw]; // (past n: read, not used)
            y[u] = ring[(size_t)sy * tw];
            sx = sx + 1 == p0 ? 0 : sx + 1;
            sy = sy + 1 == p0 ? 0 : sy + 1;
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (i + u < n) add(x[u], y[u]);
    }
}

// Products of the pushes that a one-level window in the block-deferred form
// (corr_window.hip) has staged but not yet folded into lag L = e: its lag
// block j = L / wlpb has folded every block q with kWindowT q + j <= S, so the
// pushes after f = kWindowT floor((S - j) / kWindowT) are pending.  Summed in
// double in push order; pushes s <= L have no lagged value and add nothing.
__device__ double2 window_pending(const ReduceArgs &a, int e, int64_t c)
{
    const int L = e;
    const int j = L / a.wlpb;
    const int64_t S = a.n_push;
    const int64_t f = S >= j ? ((S - j) / kWindowT) * kWindowT : 0;
    const int64_t s1 = f + 1 > (int64_t)L + 1 ? f + 1 : (int64_t)L + 1;
    if (s1 > S) return make_double2(0.0, 0.0);
    const int64_t tile = c / a.tw;
    const int64_t lane = c - tile * a.tw;
    const char *tb = a.state + tile * a.tile_bytes;
    const int p0 = a.p0;
    int sx = (int)((s1 - 1) % p0);
    int sy = (int)((s1 - L - 1) % p0);
    double re = 0.0, im = 0.0;
    if (a.kind >= K_CF32_F64) {
        const float2 *ring = reinterpret_cast<const float2 *>(tb) + lane;
        pending_products(ring, a.tw, p0, sx, sy, (int)(S - s1 + 1), [&](float2 x, float2 y) {
            re += (double)x.x * (double)y.x + (double)x.y * (double)y.y;
            im += (double)x.y * (double)y.x - (double)x.x * (double)y.y;
        });
    } else {
        const float *ring = reinterpret_cast<const float *>(tb) + lane;
        pending_products(ring, a.tw, p0, sx, sy, (int)(S - s1 + 1),
                         [&](float x, float y) { re += (double)x * (double)y; });
    }
    return make_double2(re, im);
}

// Where entry e's accumulators lie inside a tile, and its count.
struct EntryRow {
    int64_t hi, lo, count;
};

__device__ __forceinline__ EntryRow entry_row(const ReduceArgs &a, int e)
{
    int k = 0;
    while (k + 1 < a.n_levels && e >= a.level_e[k + 1]) ++k;
    const int j = e - a.level_e[k];
    EntryRow r;
    r.hi = (k == 0 ? a.acc0 : a.lvl0_bytes + (int64_t)(k - 1) * a.lvlk_bytes + a.acck) + j * a.row_bytes;
    r.lo = r.hi + (k == 0 ? a.lo0 : a.lok);
    r.count = a.level_n[k] - (k == 0 ? 0 : a.lag0) - j;
    return r;
}

__device__ __forceinline__ double2 stored_acc(const ReduceArgs &a, const EntryRow &r, int64_t c)
{
    const int64_t tile = c / a.tw;
    const int64_t lane = c - tile * a.tw;
    const char *tb = a.state + tile * a.tile_bytes;
    switch (a.kind) {
    case K_F32_F64:
    case K_F64_F64:
        return make_double2(reinterpret_cast<const double *>(tb + r.hi)[lane], 0.0);
    case K_F32_KAHAN: {
        const float h = reinterpret_cast<const float *>(tb + r.hi)[lane];
        const float l = reinterpret_cast<const float *>(tb + r.lo)[lane];
        return make_double2((double)h - (double)l, 0.0);
    }
    case K_F32_F32:
        return make_double2((double)reinterpret_cast<const float *>(tb + r.hi)[lane], 0.0);
    case K_CF32_F64:
    case K_CF64_F64:
        return reinterpret_cast<const double2 *>(tb + r.hi)[lane];
    case K_CF32_KAHAN: {
        const float2 h = reinterpret_cast<const float2 *>(tb + r.hi)[lane];
        const float2 l = reinterpret_cast<const float2 *>(tb + r.lo)[lane];
        return make_double2((double)h.x - (double)l.x, (double)h.y - (double)l.y);
    }
    default: {
        const float2 h = reinterpret_cast<const float2 *>(tb + r.hi)[lane];
        return make_double2((double)h.x, (double)h.y);
    }
    }
}

__device__ __forceinline__ double2 read_acc(const ReduceArgs &a, int e, const EntryRow &r, int64_t c)
{
    double2 v = stored_acc(a, r, c);
    if (a.wlpb > 0) {
        const double2 w = window_pending(a, e, c);
        v.x += w.x;
        v.y += w.y;
    }
    return v;
}

constexpr int kRedThreads = 256;

__global__ __launch_bounds__(kRedThreads) void reduce_partial_kernel(ReduceArgs a)
{
    __shared__ double sr[kRedThreads];
    __shared__ double si[kRedThreads];
    const int e = blockIdx.y;
    const int64_t n = a.ch_end - a.ch_begin;
    const int64_t per = (n + a.blocks_per_entry - 1) / a.blocks_per_entry;
    const int64_t b0 = a.ch_begin + (int64_t)blockIdx.x * per;
    int64_t b1 = b0 + per;
    if (b1 > a.ch_end) b1 = a.ch_end;
    double ar = 0.0, ai = 0.0;
    const EntryRow row = entry_row(a, e);
    for (int64_t c = b0 + threadIdx.x; c < b1; c += kRedThreads) {
        const double2 v = read_acc(a, e, row, c);
        ar += v.x;
        ai += v.y;
    }
    sr[threadIdx.x] = ar;
    si[threadIdx.x] = ai;
    __syncthreads();
    for (int w = kRedThreads / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) {
            sr[threadIdx.x] += sr[threadIdx.x + w];
            si[threadIdx.x] += si[threadIdx.x + w];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        double *dst = a.partial + ((size_t)e * a.blocks_per_entry + blockIdx.x) * 2;
        dst[0] = sr[0];
        dst[1] = si[0];
    }
}

__global__ void reduce_final_kernel(ReduceArgs a)
{
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= a.n_entries) return;
    double r = 0.0, i = 0.0;
    for (int b = 0; b < a.blocks_per_entry; ++b) {
        r += a.partial[((size_t)e * a.blocks_per_entry + b) * 2 + 0];
        i += a.partial[((size_t)e * a.blocks_per_entry + b) * 2 + 1];
    }
    a.out[2 * e + 0] = r;
    a.out[2 * e + 1] = i;
}

// Correlation functions of the channels [ch_begin, ch_end) as the caller takes
// them, out[(c - ch_begin) * n_entries + e] (complex: re, im): the division by
// the count is done here, and the result copied straight into the caller's
// array (the division by the host, on zero-filled copies, and the binding's
// complex arithmetic made a readout of a slice of 6144 channels and 59 entries
// take 1.7 ms; now 0.7, nearly all of it the copy into fresh host pages).
__global__ void gather_kernel(ReduceArgs a)
{
    const int64_t n = (a.ch_end - a.ch_begin) * a.n_entries;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        const int64_t c = a.ch_begin + i / a.n_entries;
        const int e = (int)(i % a.n_entries);
        const EntryRow row = entry_row(a, e);
        const double2 v = read_acc(a, e, row, c);
        const double den = (double)row.count;
        if (a.cplx)
            reinterpret_cast<double2 *>(a.out)[i] = make_double2(v.x / den * a.norm, v.y / den * a.norm);
        else
            a.out[i] = v.x / den * a.norm;
    }
}

hipError_t launch_reduce(const ReduceArgs &a, hipStream_t st)
{
    dim3 grid((unsigned)a.blocks_per_entry, (unsigned)a.n_entries);
    hipLaunchKernelGGL(reduce_partial_kernel, grid, dim3(kRedThreads), 0, st, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(reduce_final_kernel, dim3((unsigned)((a.n_entries + 63) / 64)), dim3(64), 0,
                       st, a);
    return hipGetLastError();
}

hipError_t launch_gather(const ReduceArgs &a, hipStream_t st)
{
    const int64_t n = (a.ch_end - a.ch_begin) * a.n_entries;
    int64_t blocks = (n + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    if (blocks < 1) blocks = 1;
    hipLaunchKernelGGL(gather_kernel, dim3((unsigned)blocks), dim3(256), 0, st, a);
    return hipGetLastError();
}

} // namespace corr
