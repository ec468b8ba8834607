// One FCIQMC projector iteration (paper Sec. 2.1 eq. fciqmc, Sec. 2.4 spawning /
// death / annihilation, appendix "Parallelization": sorted main list, spawned list
// sorted and merged into it) enqueued on a stream, its radix passes, the
// deterministic projection and the set-up kernels, for gfx950: 64-wide
// wavefronts, LDS-staged tiles, grids that read their problem sizes from device
// memory and a onesweep LSD radix sort (Adinets & Merrill 2022) with decoupled
// look-back (Merrill & Garland 2016).
#include "fq_kernels.h"
#include "fq_scan.h"

#include <algorithm>

namespace fq {

// ---------------------------------------------------------------------------
// iteration epilogue of CCMC (its pair sum comes after the merge's last launch;
// the other methods end there)
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(END_T) void k_end(Work w, int nb_red, int nb_mrg)
{
    if (w.ctl->err) return;
    end_replica(w, blockIdx.x, nb_red, nb_mrg);
}

// ---------------------------------------------------------------------------
// attempt scan (set-up only; iterations get the prefix from the merge):
// att_off = exclusive prefix of natt over the main list
// ---------------------------------------------------------------------------
constexpr int SCAN_T = 256, SCAN_I = 8, SCAN_TILE = SCAN_T * SCAN_I;

__global__ __launch_bounds__(SCAN_T) void k_scan_attempts(Work w)
{
    Ctl *c = w.ctl;
    if (c->err) return;
    const long long n = c->n_main;
    const long long ntiles = (n + SCAN_TILE - 1) / SCAN_TILE;
    const uint32_t epoch = epoch_of(c->t, 8);
    __shared__ long long s_tile, s_base;
    __shared__ long long s_red[8];
    for (;;) {
        if (threadIdx.x == 0) s_tile = atomicAdd(&c->tickets[TK_SCAN], 1u);
        __syncthreads();
        const long long tile = s_tile;
        if (tile >= ntiles) break;
        const long long base = tile * SCAN_TILE + (long long)threadIdx.x * SCAN_I;
        long long v[SCAN_I];
        long long sum = 0;
#pragma unroll
        for (int i = 0; i < SCAN_I; ++i) {
            v[i] = (base + i < n) ? (long long)w.cur.natt[base + i] : 0;
            sum += v[i];
        }
        long long tot;
        const long long ex = block_excl_scan<long long>(sum, tot, s_red);
        if (threadIdx.x < 64) {
            const long long lb_ = lookback(w.st_scan, tile, epoch, tot);
            if (threadIdx.x == 0) s_base = lb_;
        }
        __syncthreads();
        long long run = s_base + ex;
#pragma unroll
        for (int i = 0; i < SCAN_I; ++i) {
            if (base + i < n) w.att_off[base + i] = run;
            run += v[i];
        }
        if (tile == ntiles - 1 && threadIdx.x == 0) {
            w.att_off[n] = s_base + tot;
            c->n_att_new = s_base + tot;
        }
        __syncthreads();
    }
    if (n == 0 && blockIdx.x == 0 && threadIdx.x == 0) {
        w.att_off[0] = 0;
        c->n_att_new = 0;
    }
}

// ---------------------------------------------------------------------------
// onesweep LSD radix passes of (sort key, index) pairs over the top digits of
// 8 bits (Work::sort_p of them)
// ---------------------------------------------------------------------------
// Tiles of 256 threads x OS_I keys: 2048 (8 per thread), 3072 (12: three
// blocks fit a compute unit's LDS) or 4096 (16), chosen per context
constexpr int OS_T = 256, OS_WAVES = OS_T / 64;
static_assert(SORT_TILE_MIN == 8 * OS_T, "the status words are sized for the smallest sort tile");

// predecessors a digit's look-back reads per round trip after the first (an
// instrumented copy measured ~12 round trips per walk at four; eight made
// each pass slower, the wider reads costing more than the shorter walks)
constexpr int SORT_LB = 4;

template <int OS_I>
__global__ __launch_bounds__(OS_T) void k_sort_pass(Work w, int pass, const uint64_t *kin, const uint32_t *iin,
                                                    uint64_t *kout, uint32_t *iout)
{
    constexpr int OS_TILE = OS_T * OS_I;
    Ctl *c = w.ctl;
    if (c->err) return;
    __shared__ uint64_t lk[OS_TILE];
    __shared__ uint32_t li[OS_TILE];
    __shared__ uint32_t wh[OS_WAVES][256];
    __shared__ uint32_t gofs[256];     // global digit start (from the histogram)
    __shared__ uint32_t lofs[256];     // digit start inside the tile
    __shared__ long long gbase[256];   // tile's first output per digit
    __shared__ uint32_t s_tile;
    __shared__ uint32_t s_red[8];
    const long long n = (long long)min(c->n_spawn, (unsigned long long)w.spawn_cap);
    const long long ntiles = (n + OS_TILE - 1) / OS_TILE;
    const uint32_t epoch = epoch_of(c->t, (uint32_t)pass);
    const int shift = 8 * pass;
    const int lane = lane_id(), wid = threadIdx.x >> 6;
    {
        // global exclusive digit offsets of this pass
        const uint32_t v = c->hist[pass][threadIdx.x];
        uint32_t tot;
        gofs[threadIdx.x] = block_excl_scan<uint32_t>(v, tot, s_red);
    }
    for (;;) {
        if (threadIdx.x == 0) s_tile = atomicAdd(&c->tickets[TK_SORT + pass], 1u);
        __syncthreads();
        const long long tile = s_tile;
        if (tile >= ntiles) break;
        const long long tbase = tile * OS_TILE;
        const int tcount = (int)min((long long)OS_TILE, n - tbase);
        for (int i = threadIdx.x; i < OS_WAVES * 256; i += OS_T) (&wh[0][0])[i] = 0;
        __syncthreads();
        uint64_t kk[OS_I];
        uint32_t ix[OS_I];
        uint32_t rk[OS_I];
        // warp-striped sub-tile: element e = tbase + wid*64*OS_I + i*64 + lane
#pragma unroll
        for (int i = 0; i < OS_I; ++i) {
            const int le = wid * 64 * OS_I + i * 64 + lane;
            const long long e = tbase + le;
            const bool valid = le < tcount;
            kk[i] = valid ? kin[e] : 0;
            ix[i] = valid ? (iin ? iin[e] : (uint32_t)e) : 0;
            const uint32_t d = (uint32_t)(kk[i] >> shift) & 255u;
            uint64_t peers = __ballot(valid);
#pragma unroll
            for (int b = 0; b < 8; ++b) {
                const uint64_t m = __ballot((d >> b) & 1u);
                peers &= ((d >> b) & 1u) ? m : ~m;
            }
            uint32_t r = 0;
            if (valid) r = wh[wid][d] + (uint32_t)__popcll(peers & lanemask_lt());
            __builtin_amdgcn_wave_barrier();
            if (valid && lane == __ffsll((unsigned long long)peers) - 1) wh[wid][d] += (uint32_t)__popcll(peers);
            __builtin_amdgcn_wave_barrier();
            rk[i] = r;
        }
        __syncthreads();
        {
            const int d = threadIdx.x;
            uint32_t run = 0;
#pragma unroll
            for (int q = 0; q < OS_WAVES; ++q) {
                const uint32_t x = wh[q][d];
                wh[q][d] = run;
                run += x;
            }
            uint32_t tot;
            const uint32_t lo = block_excl_scan<uint32_t>(run, tot, s_red);
            lofs[d] = lo;
            gbase[d] = run;  // temporarily the tile count
        }
        __syncthreads();
        {
            const int d = threadIdx.x;
            const long long cnt = gbase[d];
            unsigned long long *st = w.st_sort + (size_t)tile * 256 + d;
            long long excl = 0;
            if (tile == 0) {
                st_store(st, st_pack(epoch, ST_INC, cnt));
            } else {
                st_store(st, st_pack(epoch, ST_AGG, cnt));
                long long j = tile - 1;
                int width = 1;  // the immediate predecessor first, then SORT_LB per round trip
                for (;;) {
                    unsigned long long s4[SORT_LB];
#pragma unroll
                    for (int u = 0; u < SORT_LB; ++u)
                        s4[u] = (u < width && j - u >= 0) ? st_load(w.st_sort + (size_t)(j - u) * 256 + d) : 0ull;
                    bool done = false, stop = false;
                    int used = 0;
                    long long add = 0;
#pragma unroll
                    for (int u = 0; u < SORT_LB; ++u) {
                        if (done || stop || u >= width) continue;
                        const unsigned long long s = s4[u];
                        const uint32_t e = (uint32_t)(s >> 40);
                        const unsigned long long f = (s >> ST_VBITS) & 3ull;
                        if (j - u < 0 || e != epoch || f == 0) {
                            stop = true;
                            continue;
                        }
                        add += (long long)(s & ST_VMASK);
                        ++used;
                        if (f == ST_INC) done = true;
                    }
                    excl += add;
                    j -= used;
                    if (done) break;
                    if (used == 0) __builtin_amdgcn_s_sleep(1);
                    width = SORT_LB;
                }
                st_store(st, st_pack(epoch, ST_INC, excl + cnt));
            }
            gbase[d] = (long long)gofs[d] + excl;
        }
        __syncthreads();
        // scatter into LDS in digit order (stable)
#pragma unroll
        for (int i = 0; i < OS_I; ++i) {
            const int le = wid * 64 * OS_I + i * 64 + lane;
            if (le < tcount) {
                const uint32_t d = (uint32_t)(kk[i] >> shift) & 255u;
                const uint32_t pos = lofs[d] + wh[wid][d] + rk[i];
                lk[pos] = kk[i];
                li[pos] = ix[i];
            }
        }
        __syncthreads();
        for (int p = threadIdx.x; p < tcount; p += OS_T) {
            const uint64_t k = lk[p];
            const uint32_t d = (uint32_t)(k >> shift) & 255u;
            const long long o = gbase[d] + (p - (long long)lofs[d]);
            kout[o] = k;
            iout[o] = li[p];
        }
        __syncthreads();
    }
}

// The value sum_k a_k 2^(32k - 64) of four limb sums, rounded once to the
// nearest FP64 value (ties to even).
__device__ double limbs_to_double(long long a0, long long a1, long long a2, long long a3)
{
    // signed 128-bit total as (hi, lo), two's complement
    uint64_t lo = 0, hi = 0;
    auto add_shifted = [&](long long v, int s) {
        // v * 2^s, s in {0, 32, 64, 96}, sign-extended to 128 bits
        const uint64_t ext = v < 0 ? ~0ull : 0ull;
        uint64_t vlo, vhi;
        if (s == 0) { vlo = (uint64_t)v; vhi = ext; }
        else if (s < 64) { vlo = (uint64_t)v << s; vhi = (ext << s) | ((uint64_t)v >> (64 - s)); }
        else if (s == 64) { vlo = 0; vhi = (uint64_t)v; }
        else { vlo = 0; vhi = (uint64_t)v << (s - 64); }
        const uint64_t nlo = lo + vlo;
        hi = hi + vhi + (nlo < lo ? 1ull : 0ull);
        lo = nlo;
    };
    add_shifted(a0, 0);
    add_shifted(a1, 32);
    add_shifted(a2, 64);
    add_shifted(a3, 96);
    if ((hi | lo) == 0) return 0.0;
    const bool neg = (long long)hi < 0;
    if (neg) {
        lo = ~lo + 1ull;
        hi = ~hi + (lo == 0 ? 1ull : 0ull);
    }
    // leading bit position of the magnitude
    const int msb = hi ? 127 - __clzll(hi) : 63 - __clzll(lo);
    double r;
    if (msb < 53) {
        r = (double)lo;  // exact
    } else {
        const int shift = msb - 52;  // bits below the 53-bit mantissa
        uint64_t m, rem_hi_bit, rem_rest;
        // m = magnitude >> shift; the dropped bits decide the rounding
        if (shift >= 64) {
            m = hi >> (shift - 64);
            const int rs = shift - 64;  // dropped bits of hi below m, then all of lo
            const uint64_t dh = rs ? (hi & ((1ull << rs) - 1)) : 0ull;
            rem_hi_bit = rs ? (dh >> (rs - 1)) & 1ull : (lo >> 63);
            rem_rest = rs ? ((dh & ((1ull << (rs - 1)) - 1)) | lo) : (lo & ~(1ull << 63));
        } else {
            m = (lo >> shift) | (shift ? hi << (64 - shift) : 0ull);
            const uint64_t dl = lo & ((1ull << shift) - 1);  // shift >= 1 here
            rem_hi_bit = (dl >> (shift - 1)) & 1ull;
            rem_rest = dl & ((1ull << (shift - 1)) - 1);
        }
        if (rem_hi_bit && (rem_rest || (m & 1ull))) m += 1;
        r = ldexp((double)m, shift);  // m <= 2^53: exact
    }
    r = r * 0x1p-64;
    return neg ? -r : r;
}

// ---------------------------------------------------------------------------
// deterministic projection (Sec. 2.1 semi-stochastic): y = K_DD n_D, summed
// exactly in fixed point and rounded once (FP64 mode), or as BF16 x3 products
// with FP32 accumulation (split mode); then n_D += SR(-dtau (y - S n_D))
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint16_t bf16_rn(float f)
{
    uint32_t u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}
__device__ __forceinline__ float bf16_f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

__global__ void k_det_gather(Work w)
{
    const Ctl *c = w.ctl;
    if (c->err || !c->ss_active) return;
    const int n = w.ds.n, np = w.ds.npad;
    const int nd = n * w.R;
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < nd; i += gridDim.x * blockDim.x)
        w.ds.c[i] = (double)w.cur.pop[w.ds.pos[i]];
    if (w.ds.precision == 1) {
        // BF16 hi/lo split of the amplitudes (zero padded to npad)
        const int tot = np * w.R;
        for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < tot; i += gridDim.x * blockDim.x) {
            const int r = i / np, j = i % np;
            const float cf = j < n ? (float)w.cur.pop[w.ds.pos[r * n + j]] : 0.0f;
            const uint16_t hi = bf16_rn(cf);
            w.ds.Chi[i] = hi;
            w.ds.Clo[i] = bf16_rn(cf - bf16_f(hi));
        }
    }
}

// rounded increment of a deterministic entry: n += SR(-dtau (y - S n))
__device__ __forceinline__ void det_update(const Work &w, const Ctl *c, int rep, long long row, double y, double nv)
{
    const RepParams &rp = w.rep[rep];
    const double delta = (-rp.tau) * (y - w.shift[rep] * nv);
    const U4 r = draw(TAG_SEMISTOCH, 0, c->t, w.ds.h64[row], rp.k0, rp.k1);
    const double u = u53(r.x, r.y);
    if (!(fabs(delta) < 0x1p40)) atomicOr(&((Ctl *)c)->err, ERR_OVERFLOW);
    const long long k = delta >= 0.0 ? sround(delta, u) : -sround(-delta, u);
    w.ds.y[row] = y;
    w.ds.delta[row] = k;
}

// mode 0: the FP64 projection of the iteration. mode 1 (split precision, every
// check_period iterations): FP64 reference y and the error of the split result
// relative to sum_j |K_ij||c_j|, maximised into the replica's estimators.
__global__ __launch_bounds__(256) void k_det_project_fp64(Work w, int mode)
{
    const Ctl *c = w.ctl;
    if (c->err || !c->ss_active) return;
    if (mode == 1 && (w.ds.precision != 1 || w.ds.check_period <= 0 || c->t % (uint32_t)w.ds.check_period != 0))
        return;
    const int n = w.ds.n;
    const int lane = lane_id();
    const long long rows = (long long)n * w.R;
    for (long long job = (long long)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6); job < rows;
         job += (long long)gridDim.x * (blockDim.x >> 6)) {
        // shared space: the replicas of one row of K_DD are consecutive jobs
        // (the row is read once from memory)
        const int rep = w.ds.shared ? (int)(job % w.R) : (int)(job / n);
        const int d = w.ds.shared ? (int)(job / w.R) : (int)(job % n);
        const long long row = (long long)rep * n + d;
        const double *K = w.ds.K + ((size_t)(w.ds.shared ? 0 : rep) * n + d) * n;
        const double *cv = w.ds.c + (size_t)rep * n;
        // y = sum_j K_ij n_j, exact in fixed point (2^-64), rounded once: the
        // order of the terms over lanes and the wave reduction does not matter.
        // A term x, truncated at 2^-64, is h 2^-20 + l 2^-64 with whole numbers
        // h = trunc(x 2^20) and l: their FP64 sums are exact up to 2^53, so a lane
        // of k <= 512 terms below 2^33 / k (2^28 for the 32 terms of a row of
        // 2000) adds them in FP64; beyond that the wave takes the limbs. 8 x 2000
        // rows of 2000: 87 us by limbs alone, 48 now.
        long long a0 = 0, a1 = 0, a2 = 0, a3 = 0;
        double pabs = 0.0, sh = 0.0, sl = 0.0, big = 0.0;
        bool odd = false;  // a NaN: the limbs decide
#pragma unroll 4
        for (int j = lane; j < n; j += 64) {
            const double x = K[j] * cv[j];
            const double a = x * 0x1p20, h = trunc(a);
            sh = sh + h;
            sl = sl + trunc((a - h) * 0x1p44);
            big = fmax(big, fabs(a));
            odd = odd || a != a;
            if (mode == 1) pabs = pabs + fabs(K[j]) * fabs(cv[j]);
        }
        if (n / 64 >= 512 || __any(odd || !(big * (double)(n / 64 + 1) < 0x1p53))) {
            for (int j = lane; j < n; j += 64) add_limbs4(a0, a1, a2, a3, K[j] * cv[j]);
            a0 = wave_sum<long long>(a0);
            a1 = wave_sum<long long>(a1);
            a2 = wave_sum<long long>(a2);
            a3 = wave_sum<long long>(a3);
        } else {
            // h 2^44 = (h >> 20) 2^64 + (h mod 2^20) 2^12 2^32
            const long long h = wave_sum<long long>((long long)sh);
            a0 = wave_sum<long long>((long long)sl);
            a1 = (h & ((1ll << 20) - 1)) << 12;
            a2 = h >> 20;
        }
        if (mode == 1) pabs = wave_sum<double>(pabs);
        if (lane == 0) {
            const double part = limbs_to_double(a0, a1, a2, a3);
            if (mode == 0) {
                det_update(w, c, rep, row, part, cv[d]);
            } else {
                w.ds.yref[row] = part;
                const double e = pabs > 0.0 ? fabs(w.ds.y[row] - part) / pabs : 0.0;
                atomicMax((unsigned long long *)&w.acc[rep].ss_err, (unsigned long long)__double_as_longlong(e));
            }
        }
    }
}

// Split-precision projection on MFMA: y = K c with K and c split into BF16
// hi + lo planes, y = K_hi c_hi + K_hi c_lo + K_lo c_hi accumulated in FP32
// (the "bf16x3" scheme) with v_mfma_f32_16x16x32_bf16. A block computes 16
// rows of up to 16 replicas (one K_DD shared by all) or of one replica (its
// amplitudes in column 0 of the 16 x 16 B tile).
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));

constexpr int DP_WAVES = 8;  // waves per block of the split projection (split over k)

__global__ __launch_bounds__(64 * DP_WAVES) void k_det_project_split(Work w)
{
    // One block per job (16 rows x up to 16 columns of Y = K C); its waves
    // take interleaved 32-wide steps of the k range (gfx950's 16x16x32 BF16
    // MFMA: each lane holds 8 consecutive k of its row of A and of its column
    // of B, loaded with the same k order so the dot products pair correctly)
    // and their FP32 partial tiles are summed in LDS in wave order. Shared
    // space: the columns are 16 replicas, one K_DD for all. Otherwise: one
    // replica per job, in column 0.
    const Ctl *c = w.ctl;
    const bool ss = c->ss_active != 0 && w.ds.precision == 1;
    if (block_stops(c) || !ss) return;
    __shared__ float s_part[DP_WAVES][64][4];
    const int n = w.ds.n, np = w.ds.npad;
    const int lane = lane_id(), wv = threadIdx.x >> 6;
    const int tiles = np / 16;
    const bool shared = w.ds.shared != 0;
    const int cblocks = shared ? (w.R + 15) / 16 : w.R;
    const long long jobs = (long long)tiles * cblocks;
    for (long long job = blockIdx.x; job < jobs; job += gridDim.x) {
        const int rt = (int)(job / cblocks), cb = (int)(job % cblocks);
        const int arow = rt * 16 + (lane & 15);
        const int kq = 8 * (lane >> 4);
        // this lane's column of B (and of the result): a replica
        const int rep = shared ? cb * 16 + (lane & 15) : cb;
        const bool bval = shared ? rep < w.R : (lane & 15) == 0;
        const size_t kmat = shared ? 0 : (size_t)cb;
        const uint16_t *kh = w.ds.Khi + (kmat * np + arow) * np + kq;
        const uint16_t *kl = w.ds.Klo + (kmat * np + arow) * np + kq;
        const uint16_t *ch = w.ds.Chi + (size_t)(bval ? rep : 0) * np + kq;
        const uint16_t *cl = w.ds.Clo + (size_t)(bval ? rep : 0) * np + kq;
        f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
        const bf16x8_t zero = {};
        for (int kk = 32 * wv; kk < np; kk += 32 * DP_WAVES) {
            const bf16x8_t ah = *(const bf16x8_t *)(kh + kk);
            const bf16x8_t al = *(const bf16x8_t *)(kl + kk);
            bf16x8_t bh = zero, bl = zero;
            if (bval) {
                bh = *(const bf16x8_t *)(ch + kk);
                bl = *(const bf16x8_t *)(cl + kk);
            }
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, bh, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, bl, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(al, bh, acc, 0, 0, 0);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) s_part[wv][lane][i] = acc[i];
        __syncthreads();
        // lane holds rows 4 (lane / 16) + i of column lane % 16
        if (wv == 0 && bval) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                float y = s_part[0][lane][i];
                for (int q = 1; q < DP_WAVES; ++q) y = y + s_part[q][lane][i];
                const int d = rt * 16 + 4 * (lane >> 4) + i;
                if (d < n) {
                    const long long row = (long long)rep * n + d;
                    det_update(w, c, rep, row, (double)y, w.ds.c[row]);
                }
            }
        }
        __syncthreads();
    }
}

// BF16 hi/lo planes of K_DD (zero padded to npad), once per deterministic space
__global__ void k_split_planes(Work w)
{
    const int n = w.ds.n, np = w.ds.npad;
    const long long tot = (long long)w.ds.nk * np * np;
    for (long long x = (long long)blockIdx.x * blockDim.x + threadIdx.x; x < tot; x += (long long)gridDim.x * blockDim.x) {
        const int r = (int)(x / ((long long)np * np));
        const int i = (int)((x / np) % np), j = (int)(x % np);
        float k = 0.0f;
        if (i < n && j < n) k = (float)w.ds.K[((size_t)r * n + i) * n + j];
        const uint16_t hi = bf16_rn(k);
        w.ds.Khi[x] = hi;
        w.ds.Klo[x] = bf16_rn(k - bf16_f(hi));
    }
}

}  // namespace fq

// ---------------------------------------------------------------------------
// set-up kernels: H_00 per system, K_ii - H_00 and attempt counts of a list,
// K_DD of a deterministic space
// ---------------------------------------------------------------------------
namespace fq {

template <int KIND, int W>
__global__ void k_h00(DevSys *sys, int n_sys)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n_sys) return;
    uint64_t ref[W];
#pragma unroll
    for (int q = 0; q < W; ++q) ref[q] = sys[i].ref[q];
    sys[i].H00 = diag_element<KIND, W>(sys[i], ref);
}

template <int KIND, int W>
__global__ void k_kdiag(Work w, MainList L, long long n)
{
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x) {
        uint64_t key[W];
#pragma unroll
        for (int q = 0; q < W; ++q) key[q] = L.key[(size_t)q * w.main_cap + i];
        const int rep = (int)skey_rep(L.skey[i], w.rb);
        const RepParams rp = w.rep[rep];
        const DevSys &sy = w.sys[rp.sys];
        L.kdiag[i] = entry_kdiag<KIND, W>(w, sy, key);
        const int32_t p = L.pop[i];
        const long long ap = p < 0 ? -(long long)p : (long long)p;
        L.natt[i] = (int32_t)((w.dm == 1 ? 2 : 1) * (rp.bits == 0 ? ap : ((ap + (1ll << rp.bits) - 1) >> rp.bits)));
    }
}

// K[rep][d][e] = <D_d|H|D_e> - H_00 delta_de for D keys given in D order
template <int KIND, int W>
__global__ void k_build_kdd(Work w, const uint64_t *dkeys /* [W][R*n] */, double *K)
{
    const int n = w.ds.n;
    const int nd = n * w.R;
    const long long tot = (long long)w.ds.nk * n * n;  // shared space: replica 0's keys (the same for all)
    for (long long x = (long long)blockIdx.x * blockDim.x + threadIdx.x; x < tot; x += (long long)gridDim.x * blockDim.x) {
        const int rep = (int)(x / ((long long)n * n));
        const int d = (int)((x / n) % n), e = (int)(x % n);
        uint64_t a[W], b[W];
#pragma unroll
        for (int q = 0; q < W; ++q) {
            a[q] = dkeys[(size_t)q * nd + (size_t)rep * n + d];
            b[q] = dkeys[(size_t)q * nd + (size_t)rep * n + e];
        }
        const DevSys &sy = w.sys[w.rep[rep].sys];
        double v;
        if (d == e)
            v = diag_element<KIND, W>(sy, a) - sy.H00;
        else
            v = hij<KIND, W>(sy, a, b);
        K[x] = v;
    }
}

// ---------------------------------------------------------------------------
// launchers used by the host library
// ---------------------------------------------------------------------------
template <int KIND, int W>
static void setup_kind(int what, const Work &w, DevSys *sys, int n_sys, MainList L, long long n, const uint64_t *dk,
                       double *K, hipStream_t s)
{
    // H_00 of the reference determinant (for pairs: of one half)
    if (what == 0) k_h00<base_kind(KIND), is_pair(KIND) ? W / 2 : W><<<(n_sys + 63) / 64, 64, 0, s>>>(sys, n_sys);
    if (what == 1) {
        if (n > 0) k_kdiag<KIND, W><<<(int)std::min<long long>((n + 255) / 256, 4096), 256, 0, s>>>(w, L, n);
        Work w2 = w;
        w2.cur = L;
        k_scan_attempts<<<256, SCAN_T, 0, s>>>(w2);
    }
    if constexpr (!is_pair(KIND)) {
        if (what == 2) {
            k_build_kdd<KIND, W><<<2048, 256, 0, s>>>(w, dk, K);
            if (w.ds.precision == 1) k_split_planes<<<2048, 256, 0, s>>>(w);
        }
    }
}

hipError_t enqueue_iteration(const Work &w, int kind, const Grids &g, hipStream_t s, hipEvent_t *ev)
{
    // ev (optional): N_KERNEL_SLOTS + 1 events, one before the first launch and
    // one after every launch of the iteration
    int e = 0;
    auto rec = [&]() {
        if (ev) (void)hipEventRecord(ev[e++], s);
    };
    hipError_t he;
    rec();
    rec();  // (the iteration begins in the attempt partition)
    if ((he = enqueue_spawn(0, kind, w, g, s)) != hipSuccess) return he;
    rec();
    if ((he = enqueue_spawn(1, kind, w, g, s)) != hipSuccess) return he;
    rec();
    if (w.ccmc_trunc > 0) (void)enqueue_ccmc(0, kind, w, g, s);
    rec();
    // (the digit histograms come with the spawned records)
    rec();
    // the top digits of the sort key, lowest first; the collapse orders the rest
    uint64_t *K[2] = {w.sp.skey, w.sp.skey2};
    uint32_t *I[2] = {w.sp.idx, w.sp.idx2};
    for (int p = 8 - w.sort_p, q = 0; p < 8; ++p, ++q) {
        const uint64_t *ki = K[q & 1];
        const uint32_t *ii = q == 0 ? nullptr : I[q & 1];
        if (g.sort_i == 8)
            k_sort_pass<8><<<g.sort, OS_T, 0, s>>>(w, p, ki, ii, K[(q + 1) & 1], I[(q + 1) & 1]);
        else if (g.sort_i == 16)
            k_sort_pass<16><<<g.sort, OS_T, 0, s>>>(w, p, ki, ii, K[(q + 1) & 1], I[(q + 1) & 1]);
        else
            k_sort_pass<12><<<g.sort, OS_T, 0, s>>>(w, p, ki, ii, K[(q + 1) & 1], I[(q + 1) & 1]);
        rec();
    }
    for (int q = w.sort_p; q < 8; ++q) rec();  // unused timing slots
    if ((he = enqueue_collapse(w, g, w.sort_p, s)) != hipSuccess) return he;
    rec();
    rec();
    rec();
    if (g.ss) k_det_gather<<<g.det, 256, 0, s>>>(w);
    rec();
    if (g.ss && w.ds.precision == 1)
        k_det_project_split<<<g.det, 64 * DP_WAVES, 0, s>>>(w);
    else if (g.ss)
        k_det_project_fp64<<<g.det, 256, 0, s>>>(w, 0);
    rec();
    if (g.ss && w.ds.precision == 1 && w.ds.check_period > 0) k_det_project_fp64<<<g.det, 256, 0, s>>>(w, 1);
    rec();
    rec();  // (a merge block finds its own splits)
    if ((he = enqueue_merge(0, kind, w, g, s)) != hipSuccess) return he;
    if ((he = enqueue_merge(1, kind, w, g, s)) != hipSuccess) return he;
    rec();
    if ((he = enqueue_merge(2, kind, w, g, s)) != hipSuccess) return he;
    rec();
    if (w.ccmc_trunc > 0) (void)enqueue_ccmc(1, kind, w, g, s);
    rec();
    if (w.ccmc_trunc > 0) k_end<<<w.R, END_T, 0, s>>>(w, g.reduce, g.merge);
    rec();
    return hipGetLastError();
}

hipError_t enqueue_setup(int what, int kind, const Work &w, DevSys *sys, int n_sys, MainList L, long long n,
                         const uint64_t *dk, double *K, hipStream_t s)
{
    FQ_DISPATCH(setup_kind, what, w, sys, n_sys, L, n, dk, K, s)
    return hipGetLastError();
}

int occupancy_blocks(int which)
{
    int nb = 1;
    hipError_t e = hipSuccess;
    switch (which) {
    case 0: e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_sort_pass<12>, OS_T, 0); break;
    case 1: return merge_occupancy(false);
    case 2: return collapse_occupancy();
    case 3: e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_scan_attempts, SCAN_T, 0); break;
    case 4: return spawn_occupancy();
    case 5: return merge_occupancy(true);
    default: break;
    }
    if (e != hipSuccess) nb = 1;  // a persistent grid of one block per CU still covers every tile
    return nb < 1 ? 1 : nb;
}

}  // namespace fq
