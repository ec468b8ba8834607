// Wavefront and block primitives shared by the kernel translation units:
// decoupled look-back (Merrill & Garland 2016) status words and the look-back
// itself, wave reductions, block-wide exclusive scans (gfx950: 64-wide
// wavefronts, blocks of up to 1024 threads) and the exact fixed-point
// accumulation of FP64 terms used by the estimators.
#pragma once

#include "fq_kernels.h"

namespace fq {

// ---------------------------------------------------------------------------
// decoupled look-back status words: [epoch:24 | flag:2 | value:38]
// ---------------------------------------------------------------------------
constexpr unsigned long long ST_AGG = 1ull, ST_INC = 2ull;
constexpr int ST_VBITS = 38;
constexpr unsigned long long ST_VMASK = (1ull << ST_VBITS) - 1;

__device__ __forceinline__ uint32_t epoch_of(uint32_t t, uint32_t use) { return ((t << 4) | use) & 0xFFFFFFu; }

__device__ __forceinline__ unsigned long long st_pack(uint32_t epoch, unsigned long long flag, long long v)
{
    return ((unsigned long long)epoch << 40) | (flag << ST_VBITS) | ((unsigned long long)v & ST_VMASK);
}

__device__ __forceinline__ void st_store(unsigned long long *p, unsigned long long v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned long long st_load(unsigned long long *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ int lane_id() { return __lane_id(); }
__device__ __forceinline__ uint64_t lanemask_lt() { return (1ull << lane_id()) - 1ull; }

// Whether an error bit is set, the same answer for every wave of the block. The
// blocks of a launch set bits while others of it start: waves that each looked
// for themselves could disagree, and the rest of a block would go on without
// the wave that keeps its loop counts, splits or sums. Called once by every
// thread, after the kernel has read its sizes, which then are on their way
// together with the bits (one after the other cost the eight-site ring 1.4 us
// of 92 an iteration).
__device__ __forceinline__ bool block_stops(const Ctl *c)
{
    __shared__ uint32_t s_err;
    if (threadIdx.x == 0) s_err = c->err;
    __syncthreads();
    return s_err != 0;
}

template <typename T>
__device__ __forceinline__ T wave_sum(T v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

__device__ __forceinline__ double wave_max(double v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
    return v;
}

// Decoupled look-back, run by one whole wavefront: publishes this tile's
// aggregate, then inspects the 64 preceding tiles at a time until it meets an
// inclusive prefix, publishes its own inclusive prefix and returns the
// exclusive one (to every lane). It waits only on tiles with smaller tickets,
// which are resident and never wait on this tile, so every wait ends.
static __device__ long long lookback(unsigned long long *st, long long tile, uint32_t epoch, long long agg)
{
    const int lane = lane_id();
    if (lane == 0) st_store(st + tile, st_pack(epoch, tile == 0 ? ST_INC : ST_AGG, agg));
    if (tile == 0) return 0;
    long long excl = 0;
    long long j = tile - 1;
    for (;;) {
        const long long idx = j - lane;
        unsigned long long sw = 0;
        if (idx >= 0) sw = st_load(st + idx);
        const uint32_t e = (uint32_t)(sw >> 40);
        const unsigned long long f = (sw >> ST_VBITS) & 3ull;
        const bool valid = idx >= 0 && e == epoch && f != 0;
        const uint64_t inc = __ballot(valid && f == ST_INC);
        const uint64_t bad = __ballot(idx >= 0 && !valid);
        // lanes that count: up to and including the nearest inclusive prefix
        const uint64_t need = inc ? ((inc & (~inc + 1)) << 1) - 1 : ~0ull;
        if (bad & need) {
            __builtin_amdgcn_s_sleep(1);
            continue;
        }
        const long long v = (((need >> lane) & 1ull) && valid) ? (long long)(sw & ST_VMASK) : 0;
        excl += wave_sum<long long>(v);
        if (inc) break;
        j -= 64;
    }
    if (lane == 0) st_store(st + tile, st_pack(epoch, ST_INC, excl + agg));
    return excl;
}

// exclusive block scan of one value per thread (blockDim = 256)
template <typename T>
__device__ T block_excl_scan(T v, T &total, T *lds /* 8 entries */)
{
    const int lane = lane_id(), wid = threadIdx.x >> 6;
    T x = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const T y = __shfl_up(x, o, 64);
        if (lane >= o) x += y;
    }
    if (lane == 63) lds[wid] = x;
    __syncthreads();
    T base = 0, tot = 0;
    const int nw = blockDim.x >> 6;
    for (int w = 0; w < nw; ++w) {
        if (w < wid) base += lds[w];
        tot += lds[w];
    }
    total = tot;
    __syncthreads();
    return base + x - v;
}

// two exclusive block scans at once (one pair of barriers)
static __device__ void block_excl_scan2(long long v, long long u, long long &ex_v, long long &ex_u, long long &tot_v,
                                 long long &tot_u, long long *lds /* 16 entries */)
{
    const int lane = lane_id(), wid = threadIdx.x >> 6;
    long long x = v, y = u;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const long long a = __shfl_up(x, o, 64), b = __shfl_up(y, o, 64);
        if (lane >= o) {
            x += a;
            y += b;
        }
    }
    if (lane == 63) {
        lds[wid] = x;
        lds[8 + wid] = y;
    }
    __syncthreads();
    long long bv = 0, bu = 0, tv = 0, tu = 0;
    const int nw = blockDim.x >> 6;
    for (int w = 0; w < nw; ++w) {
        if (w < wid) {
            bv += lds[w];
            bu += lds[8 + w];
        }
        tv += lds[w];
        tu += lds[8 + w];
    }
    tot_v = tv;
    tot_u = tu;
    ex_v = bv + x - v;
    ex_u = bu + y - u;
    __syncthreads();
}

// Exact fixed-point accumulation of one FP64 term: |x| 2^64 truncated toward
// zero, split into four 32-bit limbs added with the sign of x (int64 limb
// sums are exact and order independent).
__device__ __forceinline__ void add_limbs4(long long &a0, long long &a1, long long &a2, long long &a3, double x)
{
    if (x == 0.0) return;
    const bool neg = x < 0.0;
    const uint64_t bits = (uint64_t)__double_as_longlong(fabs(x));
    const int ex = (int)((bits >> 52) & 0x7FF);
    const uint64_t mant = (bits & ((1ull << 52) - 1)) | (ex ? (1ull << 52) : 0ull);
    const int sh = (ex ? ex : 1) - 1075 + 64;  // |x| * 2^64 = mant * 2^sh
    uint64_t lo = 0, hi = 0;
    if (sh >= 64) {
        hi = mant << (sh - 64);
    } else if (sh > 0) {
        lo = mant << sh;
        hi = mant >> (64 - sh);
    } else if (sh == 0) {
        lo = mant;
    } else if (sh > -64) {
        lo = mant >> (-sh);
    }
    const long long l0 = (long long)(lo & 0xFFFFFFFFull), l1 = (long long)(lo >> 32);
    const long long l2 = (long long)(hi & 0xFFFFFFFFull), l3 = (long long)(hi >> 32);
    a0 += neg ? -l0 : l0;
    a1 += neg ? -l1 : l1;
    a2 += neg ? -l2 : l2;
    a3 += neg ? -l3 : l3;
}

// ---------------------------------------------------------------------------
// estimator fields of a block's table in LDS (replicas below acc_rows(R); the
// others are added to global memory directly)
// ---------------------------------------------------------------------------
enum { F_NW = 0, F_NOCC, F_N0, F_NSPAWN, F_NUNIQ, F_FLIPS, F_REJU, F_DEATH, F_SPAWN, F_REJ, F_L0, F_L1, F_L2, F_L3 };

__device__ __forceinline__ void acc_table_clear(long long *tab, int rl)
{
    for (int i = threadIdx.x; i < rl * EST_FIELDS; i += blockDim.x) tab[i] = 0;
}

__device__ __forceinline__ void acc_add(long long *tab, int rl, EstAcc *g, int rep, int f, long long v)
{
    if (rep < rl)
        atomicAdd((unsigned long long *)&tab[rep * EST_FIELDS + f], (unsigned long long)v);
    else
        atomicAdd((unsigned long long *)(&g[rep].nw + f), (unsigned long long)v);
}

// Time-step search maxima, per replica, into the replica's estimator record
// of the iteration: KD = false the largest |H_ji| / p_gen (as its bits), true
// the largest K_ii (as an order-preserving key). A thread keeps the running
// maximum of one replica and hands it over when it moves to another replica
// and at the end of the kernel; there the wave reduces first when its holders
// share one replica (the lists are sorted by replica, so they nearly always do).
template <bool KD>
__device__ __forceinline__ void ts_put(const Work &w, int rep, double v)
{
    if constexpr (KD)
        atomicMax(&w.acc[rep].kd_key, ordered_key(v));
    else
        atomicMax(&w.acc[rep].rs_bits, (unsigned long long)__double_as_longlong(v));
}

template <bool KD>
__device__ void ts_finish(const Work &w, double v, int rep, bool has)
{
    const uint64_t act = __ballot(has);
    if (!act) return;
    const int leader = __ffsll((unsigned long long)act) - 1;
    const int r0 = __shfl(rep, leader, 64);
    if (__ballot(has && rep != r0) == 0) {
        const double m = wave_max(has ? v : -INFINITY);
        if (lane_id() == leader) ts_put<KD>(w, r0, m);
    } else if (has) {
        ts_put<KD>(w, rep, v);
    }
}

// The diagonal element death uses, relative to H_00: K_ii for a determinant;
// for a pair (i, j) of the density-matrix methods (Sec. 2.3) (K_ii + K_jj) / 2
// (DMQMC, the symmetrised Bloch equation) or K_jj - K_ii (IP-DMQMC, with H^0
// the diagonal part of H).
template <int KIND, int W>
__device__ double entry_kdiag(const Work &w, const DevSys &sy, const uint64_t (&key)[W])
{
    if constexpr (is_pair(KIND)) {
        constexpr int BK = base_kind(KIND), WH = W / 2;
        uint64_t a[WH], b[WH];
#pragma unroll
        for (int x = 0; x < WH; ++x) {
            a[x] = key[x];
            b[x] = key[WH + x];
        }
        const double ki = diag_element<BK, WH>(sy, a) - sy.H00;
        const double kj = diag_element<BK, WH>(sy, b) - sy.H00;
        return w.dm == 1 ? (ki + kj) * 0.5 : kj - ki;
    } else {
        return diag_element<KIND, W>(sy, key) - sy.H00;
    }
}

// End of an iteration, by one block of END_T threads per replica: folds the
// partials of the reduction and the merge into the accumulators, one wave per
// field, then records them in the history ring.
constexpr int END_T = 512;
static __device__ void end_replica(const Work &w, int r, int nb_red, int nb_mrg)
{
    const int lane = threadIdx.x & 63;
    if (r < acc_rows(w.R)) {
        for (int f = threadIdx.x >> 6; f < EST_FIELDS; f += END_T / 64) {
            const long long *pr = w.part_red + (size_t)(r * EST_FIELDS + f) * PART_MAX_BLOCKS;
            const long long *pm = w.part_mrg + (size_t)(r * EST_FIELDS + f) * PART_MAX_BLOCKS;
            // sixteen loads in flight (one after another they took 14 of the 19 us
            // of this step at 1024 partials)
            long long sum = 0;
            for (int b = lane; b < nb_red || b < nb_mrg; b += 8 * 64) {
                long long x[8], y[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    x[u] = b + 64 * u < nb_red ? pr[b + 64 * u] : 0;
                    y[u] = b + 64 * u < nb_mrg ? pm[b + 64 * u] : 0;
                }
#pragma unroll
                for (int u = 0; u < 8; ++u) sum += x[u] + y[u];
            }
            sum = wave_sum<long long>(sum);
            if (lane == 0) (&w.acc[r].nw)[f] += sum;
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        const uint32_t t = w.ctl->t;
        EstAcc a = w.acc[r];
        a.t = t;
        w.hist[(size_t)(t % (uint32_t)w.hist_len) * w.R + r] = a;
    }
}

// calls fn<KIND, W> for the kernel kind and key width of a context
#define FQ_DISPATCH(fn, ...)                                                                  \
    switch (kind * 16 + w.W) {                                                               \
    case K_HUBBARD * 16 + 1: fn<K_HUBBARD, 1>(__VA_ARGS__); break;                           \
    case K_UEG * 16 + 1: fn<K_UEG, 1>(__VA_ARGS__); break;                                   \
    case K_UEG * 16 + 2: fn<K_UEG, 2>(__VA_ARGS__); break;                                   \
    case K_UEG * 16 + 4: fn<K_UEG, 4>(__VA_ARGS__); break;                                   \
    case K_UEG * 16 + 8: fn<K_UEG, 8>(__VA_ARGS__); break;                                   \
    case K_MOLECULAR * 16 + 1: fn<K_MOLECULAR, 1>(__VA_ARGS__); break;                       \
    case K_MOLECULAR * 16 + 2: fn<K_MOLECULAR, 2>(__VA_ARGS__); break;                       \
    case (K_HUBBARD | K_PAIR) * 16 + 2: fn<K_HUBBARD | K_PAIR, 2>(__VA_ARGS__); break;       \
    case (K_UEG | K_PAIR) * 16 + 2: fn<K_UEG | K_PAIR, 2>(__VA_ARGS__); break;               \
    case (K_MOLECULAR | K_PAIR) * 16 + 2: fn<K_MOLECULAR | K_PAIR, 2>(__VA_ARGS__); break;   \
    default: return hipErrorInvalidValue;                                                    \
    }

}  // namespace fq
