// corr_multi.hip -- several pushes of a per-step group in one pass.
//
// A per-step push reads and writes every accumulator row that it adds to, and
// a push of a small group is one short chain of memory latencies.  Algorithm
// 1's sums of a lag take one product per push, in push order, so r pushes can
// be added with the accumulators (and their compensations) kept in registers
// in between: the same operations on the same values in the same order, and so
// the same bits, with each accumulator row read and written once per r pushes.
//
// The pushes' samples wait in rows outside the state (kMultiT at most); a pass
// adds them level by level.  A block holds 32 consecutive channels, eight
// threads to a channel, which share the lags of a level evenly.  The values of
// a level (the p - 1 old ones its lags reach back to, then its new ones) lie
// in LDS, one row of 32 channels each, so a thread reads the newest value and
// the one entering its window of lags once per push and keeps the rest of the
// window in registers.  After a level's sums the block forms the next level's
// values from these rows.  The ring and accumulator rows of the next level are
// loaded while a level is summed.
//
// Memory-bound for large groups (64 pushes move about 5 KB per pair channel of
// p = 32 and 10 levels instead of 64 KB: 99999 channels 126 us a pass, against
// 64 pushes of 15 us), a chain of about log2(64) short levels for small ones
// (300 complex channels, p = 32: 31 us against 64 x 6; nine double ones, p = 16
// and 20 levels: 13 us against 64 x 4).
#include <hip/hip_runtime.h>

#include "corr_keep.h"
#include "corr_kernels.h"
#include "corr_sums.h"

namespace corr {

namespace {

constexpr int kMultiCh = 32;      // channels of a block
constexpr int kMultiParts = 8;    // threads of a channel
constexpr int kMultiThreads = kMultiCh * kMultiParts;

// (member by member, so that arrays of them stay in registers: copied whole, a
// level's complex doubles went through 112 to 176 bytes of scratch a thread, and
// 64 pushes of 150000 channels at p = 32 took 682 us instead of 346, one push
// 145 instead of 65; 76 by the per-step kernel)
template <typename T> __device__ __forceinline__ void put(T &to, const T &v) { to = v; }
__device__ __forceinline__ void put(double2 &to, const double2 &v)
{
    to.x = v.x;
    to.y = v.y;
}

// A level's rows of a thread, loaded ahead: its share of the P - 1 old values
// (rows part, part + 8, ..), the newest old x value (pairs) and the accumulators of
// its lags.
template <int K, int P> struct LevelRegs {
    using S = typename KT<K>::S;
    using A = typename KT<K>::A;
    static constexpr int NOLD = (P - 1 + kMultiParts - 1) / kMultiParts;
    static constexpr int NL = P / kMultiParts; // lags of a thread: NL at level 0, NLK above
    S old[NOLD], xold;
    A h[NL], c[NL];
    __device__ __forceinline__ void take(const LevelRegs &o)
    {
#pragma unroll
        for (int i = 0; i < NOLD; ++i) put(old[i], o.old[i]);
        put(xold, o.xold);
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            put(h[i], o.h[i]);
            put(c[i], o.c[i]);
        }
    }
};

template <int K, int P, bool PAIR> struct Level {
    using S = typename KT<K>::S;
    using A = typename KT<K>::A;
    S *ring;   // lagged values (pairs: the x ring P rows later)
    A *hi, *lo;
    int lag0, nl, per; // first lag, lags, lags of a thread
    __device__ __forceinline__ Level(const GroupArgs &g, char *tb, int k)
    {
        constexpr int rings = PAIR ? 2 : 1;
        char *base = k == 0 ? tb : tb + g.lvl0_bytes + (int64_t)(k - 1) * g.lvlk_bytes;
        lag0 = k == 0 ? 0 : P / 2;
        nl = P - lag0;
        per = (nl + kMultiParts - 1) / kMultiParts;
        ring = reinterpret_cast<S *>(base);
        hi = reinterpret_cast<A *>(ring + (size_t)rings * P * g.tw);
        lo = hi + (size_t)nl * g.tw;
    }
};

template <int K, int P, bool PAIR, int NL>
__device__ __forceinline__ void load_level(LevelRegs<K, P> &r, const Level<K, P, PAIR> &lv, int64_t f,
                                           int part, int tw, int off)
{
    const int s0 = (int)(f % P); // slot of value f + 1
#pragma unroll
    for (int i = 0; i < LevelRegs<K, P>::NOLD; ++i) {
        const int row = part + i * kMultiParts; // value f - (P - 2) + row
        int slot = s0 - (P - 1) + row;
        if (slot < 0) slot += P;
        if (row < P - 1) r.old[i] = lv.ring[(size_t)slot * tw + off];
    }
    if constexpr (PAIR) {
        if (part == 0) r.xold = lv.ring[(size_t)(P + (s0 == 0 ? P - 1 : s0 - 1)) * tw + off];
    }
#pragma unroll
    for (int i = 0; i < NL; ++i) {
        const int l = part * NL + i;
        if (l < lv.nl) {
            r.h[i] = lv.hi[(size_t)l * tw + off];
            if constexpr (KT<K>::NP == 2) r.c[i] = lv.lo[(size_t)l * tw + off];
        }
    }
}

// Add the n new values of a level (values f + 1 .. f + n) to the sums of the
// thread's NL lags.
template <int K, int P, bool PAIR, int NL>
__device__ __forceinline__ void add_level(LevelRegs<K, P> &r, const Level<K, P, PAIR> &lv, int64_t f,
                                          int n, int part, int ch, int tw, int off,
                                          const typename KT<K>::S *yb, const typename KT<K>::S *xb)
{
    using S = typename KT<K>::S;
    const int l0 = part * NL;
    if (l0 >= lv.nl) return;
    const int L0 = lv.lag0 + l0;
    const S *ent = yb + (P - 1 - L0) * kMultiCh + ch; // value f + 1 - L0
    const S *nw = PAIR ? xb + kMultiCh + ch : yb + (P - 1) * kMultiCh + ch;
    S w[NL]; // w[i] = value f + 1 + s - (L0 + i)
#pragma unroll
    for (int i = 0; i < NL - 1; ++i) w[i] = ent[L0 + i + 1 < P ? -(i + 1) * kMultiCh : 0];
    const bool early = f < P; // the first lags of a series have no value to look back to
    auto step = [&](int s, bool check) {
        const S e = ent[s * kMultiCh], x = nw[s * kMultiCh];
#pragma unroll
        for (int i = NL - 1; i >= 1; --i) w[i] = w[i - 1];
        w[0] = e;
#pragma unroll
        for (int i = 0; i < NL; ++i)
            if (l0 + i < lv.nl && (!check || L0 + i <= f + s)) Acc<K>::add(r.h[i], r.c[i], x, w[i]);
    };
    if (early) {
        for (int s = 0; s < n; ++s) step(s, true);
    } else {
#pragma unroll 4
        for (int s = 0; s < n; ++s) step(s, false);
    }
#pragma unroll
    for (int i = 0; i < NL; ++i)
        if (l0 + i < lv.nl) {
            lv.hi[(size_t)(l0 + i) * tw + off] = r.h[i];
            if constexpr (KT<K>::NP == 2) lv.lo[(size_t)(l0 + i) * tw + off] = r.c[i];
        }
}

// Waves per SIMD the registers are held to: five blocks a CU for single real
// sums (99999 pairs at p = 32: 126 us against 146 with four, and 144 with six,
// which spill); the wider types, whose registers would not fit, are left alone.
template <int K> constexpr int kMultiWaves = sizeof(typename KT<K>::A) == 4 ? 5 : 1;

template <int K, int P, bool PAIR>
__global__ __launch_bounds__(kMultiThreads) __attribute__((amdgpu_waves_per_eu(kMultiWaves<K>))) void multi_push_kernel(GroupArgs g, StepRef step,
                                                                    const char *rows, int64_t stride, int n_rows)
{
    using S = typename KT<K>::S;
    constexpr int NL0 = P / kMultiParts, NLK = (P / 2 + kMultiParts - 1) / kMultiParts;
    static_assert(P % kMultiParts == 0, "level 0 shares its lags evenly");
    __shared__ S yb[(P - 1 + kMultiT) * kMultiCh];
    __shared__ S xb[PAIR ? (1 + kMultiT) * kMultiCh : 1];
    const int ch = (int)threadIdx.x & (kMultiCh - 1), part = (int)threadIdx.x / kMultiCh;
    const int64_t c0 = (int64_t)blockIdx.x * kMultiCh;
    const int tw = g.tw;
    const int64_t tile = c0 / tw;
    const int off = (int)(c0 - tile * tw) + ch;
    const bool valid = c0 + ch < g.n_ch; // (the state's padded tail takes zeros)
    char *tb = g.state + tile * g.tile_bytes;
    int64_t f = pushes_before(step);
    int n = n_rows;

    LevelRegs<K, P> r;
    Level<K, P, PAIR> lv(g, tb, 0);
    load_level<K, P, PAIR, NL0>(r, lv, f, part, tw, off);
    for (int s = part; s < n; s += kMultiParts) {
        const S *row = reinterpret_cast<const S *>(rows + (int64_t)s * stride);
        S x = valid ? row[c0 + ch] : szero<S>();
        if constexpr (PAIR) {
            xb[(1 + s) * kMultiCh + ch] = x;
            x = valid ? row[g.n_ch + c0 + ch] : szero<S>();
        }
        yb[(P - 1 + s) * kMultiCh + ch] = x;
    }
    for (int k = 0;; ++k) {
        // the level's old rows beside its new ones
#pragma unroll
        for (int i = 0; i < LevelRegs<K, P>::NOLD; ++i) {
            const int row = part + i * kMultiParts;
            if (row < P - 1) yb[row * kMultiCh + ch] = r.old[i];
        }
        if constexpr (PAIR) {
            if (part == 0) xb[ch] = r.xold;
        }
        __syncthreads();
        const int64_t f1 = f >> 1;
        const int n1 = k + 1 < g.levels ? (int)(((f + n) >> 1) - f1) : 0;
        Level<K, P, PAIR> lv1(g, tb, k + 1);
        LevelRegs<K, P> r1;
        if (n1 > 0) load_level<K, P, PAIR, NLK>(r1, lv1, f1, part, tw, off);
        if (k == 0)
            add_level<K, P, PAIR, NL0>(r, lv, f, n, part, ch, tw, off, yb, xb);
        else
            add_level<K, P, PAIR, NLK>(r, lv, f, n, part, ch, tw, off, yb, xb);
        // ring slots of the last P new values (the earlier ones would be overwritten)
        for (int s = (n > P ? n - P : 0) + part; s < n; s += kMultiParts) {
            const int slot = (int)((f + s) % P);
            lv.ring[(size_t)slot * tw + off] = yb[(P - 1 + s) * kMultiCh + ch];
            if constexpr (PAIR) lv.ring[(size_t)(P + slot) * tw + off] = xb[(1 + s) * kMultiCh + ch];
        }
        if (n1 == 0) return;
        // the next level's values: means of the pairs (2 j - odd, 2 j + 1 - odd)
        // of new values (index -1: the newest old one)
        constexpr int NM = (kMultiT / 2 + kMultiParts - 1) / kMultiParts;
        const int odd = (int)(f & 1);
        S my[NM], mx[NM];
#pragma unroll
        for (int i = 0; i < NM; ++i) {
            const int j = part + i * kMultiParts;
            if (j < n1) {
                const S *p = yb + (P - 1 + 2 * j - odd) * kMultiCh + ch;
                my[i] = sdiv(sadd(p[0], p[kMultiCh]), 2);
                if constexpr (PAIR) {
                    const S *px = xb + (1 + 2 * j - odd) * kMultiCh + ch;
                    mx[i] = sdiv(sadd(px[0], px[kMultiCh]), 2);
                }
            }
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < NM; ++i) {
            const int j = part + i * kMultiParts;
            if (j < n1) {
                yb[(P - 1 + j) * kMultiCh + ch] = my[i];
                if constexpr (PAIR) xb[(1 + j) * kMultiCh + ch] = mx[i];
            }
        }
        r.take(r1);
        lv = lv1;
        f = f1;
        n = n1;
    }
}

template <int K, int P, bool PAIR>
hipError_t launch_multi_kp(const GroupArgs &g, StepRef step, const void *rows, int64_t stride, int n,
                           hipStream_t st)
{
    const int64_t blocks = (g.n_ch + kMultiCh - 1) / kMultiCh;
    hipLaunchKernelGGL((multi_push_kernel<K, P, PAIR>), dim3((unsigned)blocks), dim3(kMultiThreads), 0, st,
                       g, step, static_cast<const char *>(rows), stride, n);
    return hipGetLastError();
}

template <int K, bool PAIR>
hipError_t launch_multi_k(const GroupArgs &g, StepRef step, const void *rows, int64_t stride, int n,
                          hipStream_t st)
{
    switch (g.p) {
    case 16: return launch_multi_kp<K, 16, PAIR>(g, step, rows, stride, n, st);
    case 24: return launch_multi_kp<K, 24, PAIR>(g, step, rows, stride, n, st);
    case 32: return launch_multi_kp<K, 32, PAIR>(g, step, rows, stride, n, st);
    default: return hipErrorInvalidValue;
    }
}

template <bool PAIR>
hipError_t launch_multi_pair(const GroupArgs &g, StepRef step, const void *rows, int64_t stride, int n,
                             hipStream_t st)
{
    switch (g.kind) {
    case K_F32_F64: return launch_multi_k<K_F32_F64, PAIR>(g, step, rows, stride, n, st);
    case K_F32_KAHAN: return launch_multi_k<K_F32_KAHAN, PAIR>(g, step, rows, stride, n, st);
    case K_F32_F32: return launch_multi_k<K_F32_F32, PAIR>(g, step, rows, stride, n, st);
    case K_F64_F64: return launch_multi_k<K_F64_F64, PAIR>(g, step, rows, stride, n, st);
    case K_CF32_F64: return launch_multi_k<K_CF32_F64, PAIR>(g, step, rows, stride, n, st);
    case K_CF32_KAHAN: return launch_multi_k<K_CF32_KAHAN, PAIR>(g, step, rows, stride, n, st);
    case K_CF32_F32: return launch_multi_k<K_CF32_F32, PAIR>(g, step, rows, stride, n, st);
    default:
        if constexpr (!PAIR) return launch_multi_k<K_CF64_F64, false>(g, step, rows, stride, n, st);
        return hipErrorInvalidValue; // the rows of complex double pairs exceed a block's LDS
    }
}

// One group, or several (blockIdx.y: the group).  The push of a small group is
// mostly the host's launch, and that grows with the argument: 2.8 us for one
// row, 3.4 for the room of eight.
__global__ __launch_bounds__(256) void keep_row_kernel(KeepRow k)
{
    keep_row(k, (int64_t)blockIdx.x * blockDim.x + threadIdx.x, (int64_t)gridDim.x * blockDim.x);
}
__global__ __launch_bounds__(256) void keep_rows_kernel(KeepArgs a)
{
    keep_row(a.row[blockIdx.y], (int64_t)blockIdx.x * blockDim.x + threadIdx.x, (int64_t)gridDim.x * blockDim.x);
}

} // namespace

// m = 2 is built in (a level's values are means of two), and a kernel is built
// for each point count, so that a thread's share of the lags (P / 8) is held in
// registers: 16 and 32, which the library's workloads use, and 24 between them
// (15 kernels a count).  64 pushes of 150000 float pairs, pass / push by push: p =
// 16 118 / 1044 us, 24 165 / 1451, 32 184 / 1852.  Other counts, for which nothing
// has been measured, keep the per-step push.
bool multi_supported(int kind, int p, int m, bool pair)
{
    return m == 2 && (p == 16 || p == 24 || p == 32) && !(pair && kind == K_CF64_F64);
}

hipError_t launch_multi_push(const GroupArgs &g, StepRef step, const void *rows, int64_t stride, int n,
                             hipStream_t st)
{
    if (n < 1 || n > kMultiT || g.deferred || !multi_supported(g.kind, g.p, g.m, g.pair != 0))
        return hipErrorInvalidValue;
    return g.pair ? launch_multi_pair<true>(g, step, rows, stride, n, st)
                  : launch_multi_pair<false>(g, step, rows, stride, n, st);
}

hipError_t launch_keep_rows(KeepArgs &a, hipStream_t st)
{
    if (a.n < 1 || a.n > kMaxGroups) return hipErrorInvalidValue;
    int64_t most = 0;
    for (int i = 0; i < a.n; ++i) {
        KeepRow &k = a.row[i];
        k.wide = keep_wide(k);
        most = k.bytes > most ? k.bytes : most;
    }
    int64_t blocks = (most / 16 + 255) / 256;
    blocks = blocks < 1 ? 1 : blocks > 2048 ? 2048 : blocks;
    if (a.n == 1)
        hipLaunchKernelGGL(keep_row_kernel, dim3((unsigned)blocks), dim3(256), 0, st, a.row[0]);
    else
        hipLaunchKernelGGL(keep_rows_kernel, dim3((unsigned)blocks, (unsigned)a.n), dim3(256), 0, st, a);
    return hipGetLastError();
}

} // namespace corr
