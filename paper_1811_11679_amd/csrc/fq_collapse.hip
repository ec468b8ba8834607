// Segmented reduction of the spawned list (paper Sec. 2.4 annihilation: combine
// walkers on the same determinant). The radix passes before it have ordered
// the list by the top 8 * passes bits of the sort key only; this kernel
// finishes the order inside each group of equal top bits and writes one entry
// per distinct determinant: the int64 sum of its amplitudes and the OR of its
// initiator flags, in (sort key, key) order. A tile writes its entries at the
// places of its records: no tile waits for another's count (a look-back for
// dense output took two thirds of the kernel), and the places left over hold
// copies of the tile's last determinant marked UNIQ_FILLER, which keep the
// list sorted and which the merge drops.
//
// A tile owns the groups that start in its CL_SPAN records, so no segment
// crosses a tile. Its records (up to CL_CAP) are gathered into LDS once. In
// the plans the host chooses groups hold a few records, or many of one
// determinant: a group of one sort key needs no order, a small mixed one is
// ranked by counting, and only a tile with a large mixed group goes through a
// bitonic network (registers, lane exchanges, and LDS for the two strides that
// cross waves). The network sorts one 64-bit word, the sort key with its low
// bits replaced by the record's place. Keys that agree in the other bits and
// records on one sort key with different determinants (hash collisions) are
// put in full order by a rare last step.
//
// Bound: the gathers of the records (8W + 8 bytes at random). The one to four
// radix passes and this kernel replace eight passes, a reduction, its
// collision fix-up and a repeated reduction: each launch costs about 4.5 us in
// a replayed graph however little it does, and each pass a trip over the list.
#include "fq_kernels.h"
#include "fq_scan.h"

#include <type_traits>

namespace fq {

constexpr int CL_T = 256, CL_I = 4;
constexpr int CL_CAP = CL_T * CL_I;  // records of a window
// A tile's window of CL_CAP records holds the groups that start in its first
// CL_SPAN; groups of up to CL_CAP - CL_SPAN + 1 records always fit.
constexpr int CL_SPAN = 768;
constexpr uint64_t CL_LOW = CL_CAP - 1;
// largest mixed group ranked by counting: a record then reads as many sort
// keys from LDS as its group holds; the network costs a tile about 20 us
constexpr int CL_COUNT = 128;
constexpr int CL_MAX_KEYS = 64;  // determinants on one sort key; more cannot be hash collisions
static_assert((CL_CAP & (CL_CAP - 1)) == 0, "the place of a record is a bit field of the sorted word");

template <int W>
__device__ __forceinline__ void rec_key(const Work &w, uint32_t j, uint64_t (&k)[W])
{
#pragma unroll
    for (int q = 0; q < W; ++q) k[q] = w.sp.rec[(size_t)j * (W + 1) + q];
}

__device__ __forceinline__ void cas_up(uint64_t &a, uint64_t &b, bool up)
{
    const bool sw = (a > b) == up;
    const uint64_t x = sw ? b : a, y = sw ? a : b;
    a = x;
    b = y;
}

// bitonic sort of CL_CAP words, ascending: element CL_I t + r in register r of
// thread t. The two loops stay loops: unrolled, the masks of the 55 stages spill.
__device__ __forceinline__ void block_sort(uint64_t (&v)[CL_I], uint64_t *lds)
{
    static_assert(CL_I == 4, "the first runs are written out for four words per thread");
    const int t = threadIdx.x;
    cas_up(v[0], v[1], true);
    cas_up(v[2], v[3], false);
#pragma unroll 1
    for (int kt = 1; kt <= CL_T; kt <<= 1) {  // runs of CL_I kt elements, kt threads
        const bool up = (t & kt) == 0;
        int x = kt >> 1;
#pragma unroll 1
        for (; x >= 64; x >>= 1) {
            // partner in another wave
            __syncthreads();
#pragma unroll
            for (int r = 0; r < CL_I; ++r) lds[r * CL_T + t] = v[r];
            __syncthreads();
            const int p = t ^ x;
            const bool keep_small = ((t & x) == 0) == up;
#pragma unroll
            for (int r = 0; r < CL_I; ++r) {
                const uint64_t o = lds[r * CL_T + p];
                v[r] = ((v[r] < o) == keep_small) ? v[r] : o;
            }
        }
#pragma unroll 1
        for (; x >= 1; x >>= 1) {
            const bool keep_small = ((t & x) == 0) == up;
#pragma unroll
            for (int r = 0; r < CL_I; ++r) {
                const uint64_t o = (uint64_t)__shfl_xor((unsigned long long)v[r], x, 64);
                v[r] = ((v[r] < o) == keep_small) ? v[r] : o;
            }
        }
        cas_up(v[0], v[2], up);
        cas_up(v[1], v[3], up);
        cas_up(v[0], v[1], up);
        cas_up(v[2], v[3], up);
    }
}

// end of the group of prefix p that holds every record before lo: the block
// probes 256 places at once
__device__ long long group_end(const uint64_t *skey, long long lo, long long hi, uint64_t p, int sh)
{
    while (lo < hi) {
        const long long step = (hi - lo + CL_T - 1) / CL_T;
        const long long e = lo + threadIdx.x * step;
        const int cnt = __syncthreads_count(e < hi && (skey[e] >> sh) == p);  // they come first
        if (cnt == 0 || step == 1) return lo + cnt;
        hi = min(hi, lo + cnt * step);
        lo += (cnt - 1) * step + 1;
    }
    return lo;
}

// f(place, sort key) for a thread's share of the places [lo, hi), U keys in flight
template <int U, typename F>
__device__ __forceinline__ void scan_keys(const uint64_t *skey, long long lo, long long hi, F &&f)
{
    for (long long e = lo + threadIdx.x; e < hi; e += U * CL_T) {
        uint64_t x[U];
#pragma unroll
        for (int u = 0; u < U; ++u) x[u] = skey[U == 1 ? e : min(e + u * CL_T, hi - 1)];
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (U == 1 || e + u * CL_T < hi) f(e + u * CL_T, x[u]);
    }
}

// Sum and count (initiators above bit 32) of this thread's records of sort key k and
// the determinant det, U in flight; true if it met another determinant on that key.
template <int W, int U>
__device__ __forceinline__ bool group_sum(const uint64_t *rec, const uint64_t *skey, const uint32_t *idx, long long lo,
                                          long long hi, uint64_t k, const uint64_t (&det)[W], long long &sum, long long &cnt)
{
    sum = cnt = 0;
    bool mixed = false;
    for (long long e = lo + threadIdx.x; e < hi; e += U * CL_T) {
        uint64_t x[U], r[U][W + 1];
        uint32_t j[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const long long at = U == 1 ? e : min(e + u * CL_T, hi - 1);
            x[u] = skey[at];
            j[u] = idx[at];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (U == 1 && x[u] != k) continue;
#pragma unroll
            for (int q = 0; q <= W; ++q) r[u][q] = rec[(size_t)j[u] * (W + 1) + q];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (e + u * CL_T >= hi || x[u] != k) continue;
            bool here = true;
#pragma unroll
            for (int q = 0; q < W; ++q) here = here && r[u][q] == det[q];
            if (!here) {
                mixed = true;
                continue;
            }
            sum += (int32_t)(uint32_t)r[u][W];
            cnt += 1ll + ((uint32_t)(r[u][W] >> 32) ? 1ll << 32 : 0ll);
        }
    }
    return mixed;
}

// skey, idx: the list as the passes left it; spare: the other index buffer,
// free here (places of an oversized tile's selected records)
// HEAVY, for lists with many records per determinant (the host's rule): a block
// keeps several keys and records of an oversized group in flight. All records of a
// determinant fall to one block, so their latency is what such a list waits for
// (3.6e6 records on 12 determinants: 1530 -> 950 us, 3.2e7 on 4900: 2700 -> 1710);
// in the other kernel the registers for it would spill those of the windows' path,
// which made every case 2 to 9% slower.
template <int W, bool HEAVY>
__global__ __launch_bounds__(CL_T, 4) void k_collapse(Work w, const uint64_t *skey, const uint32_t *idx, uint32_t *spare,
                                                   int passes)
{
    Ctl *c = w.ctl;
    extern __shared__ __align__(16) unsigned char dyn_lds[];
    long long *tab = (long long *)dyn_lds;  // estimator table, acc_rows(R) rows
    const int rl = acc_rows(w.R);
    acc_table_clear(tab, rl);
    constexpr int UK = HEAVY ? 8 : 1, UR = !HEAVY ? 1 : W <= 2 ? 8 : W == 4 ? 4 : 2;
    constexpr bool STAGE = W <= 2;          // the window's keys in LDS; longer ones are gathered again for the output
    __shared__ uint64_t s_x[CL_CAP + 1];    // sort keys of the window, then prefix sums at the heads
    __shared__ uint64_t s_key[STAGE ? W : 1][STAGE ? CL_CAP : 1];
    __shared__ int32_t s_am[CL_CAP];
    __shared__ uint16_t s_ord[CL_CAP];      // sorted position -> place, then segment -> place of its head
    __shared__ uint16_t s_fl[CL_CAP + 1];   // initiator contributions before a segment
    __shared__ uint8_t s_ini[CL_CAP];
    __shared__ uint8_t s_mix[CL_CAP];       // by a group's first place: it holds several sort keys
    __shared__ int s_gs[CL_T / 64];
    __shared__ int s_first, s_end, s_coll, s_cnt, s_swap, s_big;
    __shared__ uint64_t s_lastk[W + 1];     // the tile's last determinant: key, then sort key
    __shared__ long long s_red[16];
    __shared__ int s_bits[65];              // records of a group by their highest difference from its lowest key
    const long long n = (long long)min(c->n_spawn, (unsigned long long)w.spawn_cap);
    const long long ntiles = (n + CL_SPAN - 1) / CL_SPAN;
    const int sh = 64 - 8 * passes;
    const int tid = threadIdx.x;
    if (block_stops(c)) return;
    long long a_n = 0, a_sum = 0, a_uniq = 0;  // this thread's estimator sums of replica a_rep
    int a_rep = -1;
    auto acc_flush = [&]() {
        if (a_rep >= 0) {
            if (a_n) acc_add(tab, rl, w.acc, a_rep, F_NSPAWN, a_n);
            if (a_sum) acc_add(tab, rl, w.acc, a_rep, F_SPAWN, a_sum);
            if (a_uniq) acc_add(tab, rl, w.acc, a_rep, F_NUNIQ, a_uniq);
        }
        a_n = a_sum = a_uniq = 0;
    };
    auto acc_put = [&](int rep, long long nrec, long long sum, long long nseg) {
        if (rep != a_rep) {
            acc_flush();
            a_rep = rep;
        }
        a_n += nrec;
        a_sum += sum;
        a_uniq += nseg;
    };
    for (long long tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        __syncthreads();
        if (tid == 0) {
            s_first = CL_CAP;
            s_end = -1;
        }
        __syncthreads();
        const long long tb = tile * CL_SPAN;
        // the window's sort keys, and where the tile's groups begin and end
        uint64_t sk[CL_I];
        int first = CL_CAP, end = CL_CAP;
#pragma unroll
        for (int r = 0; r < CL_I; ++r) {
            const int l = r * CL_T + tid;
            const long long e = tb + l;
            sk[r] = e < n ? skey[e] : ~0ull;
            if (e < n) {
                const bool start = e == 0 || (skey[e - 1] >> sh) != (sk[r] >> sh);
                if (start && l < CL_SPAN) first = min(first, l);
                if (start && l >= CL_SPAN) end = min(end, l);
            }
        }
        if (first < CL_CAP) atomicMin(&s_first, first);
        if (end < CL_CAP) atomicMax(&s_end, CL_CAP - end);  // the smallest end, as a maximum
        __syncthreads();
        const int l0 = s_first;
        bool over = false;
        long long g0 = tb + l0, g1;  // the tile's records
        if (l0 >= CL_SPAN) {
            continue;  // inside a group that an earlier tile owns
        } else if (s_end >= 0) {
            g1 = tb + CL_CAP - s_end;
        } else if (n <= tb + CL_CAP) {
            g1 = n;
        } else {
            // the last group runs past the window
            over = true;
            g1 = group_end(skey, tb + CL_SPAN, n, skey[tb + CL_SPAN - 1] >> sh, sh);
        }
        // An oversized tile goes through its records in windows: whole groups
        // while they fit; a group that does not fit and holds one sort key is
        // summed as it is; any other is cut into ranges [wl, wu] of sort keys whose
        // records are picked out of it: from the lowest key left to the last that
        // agrees with it above the highest bit with which they fit a window, or
        // that key alone, summed as it is, if its own records do not. (Three trips
        // over the group a range. Ranges found by halving took some 200 trips for
        // two keys: the seven-site ring at 1e6 records on 1225 determinants, 11
        // pairs of which share a group, 1280 us an iteration, 344 now.)
        long long written = 0, gc = g0, ge = g1;
        bool sub = false;
        uint64_t wl = 0, wu = 0, wend = 0;
        for (;;) {
            int m = (int)(g1 - g0);
            bool hot = false, picked = false;
            long long base = g0;  // place q is record base + q (not picked)
            if (over) {
                if (!sub) {
                    if (gc >= g1) break;
                    __syncthreads();
                    if (tid == 0) s_end = 0;
                    __syncthreads();
                    int stop = 0;
#pragma unroll
                    for (int r = 0; r < CL_I; ++r) {
                        const int l = r * CL_T + tid;
                        const long long e = gc + l;
                        sk[r] = e < g1 ? skey[e] : ~0ull;
                        // the group of record e ends here
                        if (e < g1 && (e + 1 == g1 || (skey[e + 1] >> sh) != (sk[r] >> sh))) stop = max(stop, l + 1);
                    }
                    if (stop) atomicMax(&s_end, stop);
                    __syncthreads();
                    m = s_end;
                    base = gc;
                    if (m > 0) {
                        gc += m;  // (base stays)
                    } else {
                        const uint64_t p = skey[gc] >> sh;
                        ge = group_end(skey, gc, g1, p, sh);
                        wl = skey[gc];
                        bool same = true;
                        scan_keys<UK>(skey, gc, ge, [&](long long, uint64_t x) { same = same && x == wl; });
                        __syncthreads();
                        if (tid == 0) s_cnt = 0;
                        __syncthreads();
                        if (!same) s_cnt = 1;
                        __syncthreads();
                        sub = true;
                        if (s_cnt) {
                            wl = p << sh;
                            wend = wl | ((1ull << sh) - 1);
                            continue;
                        }
                        hot = true;
                        wu = wend = wl;
                    }
                } else {
                    // the group's next sort key at or above wl, and its records
                    // by the highest bit in which they differ from that key
                    uint64_t next = ~0ull;
                    bool any = false;
                    scan_keys<UK>(skey, gc, ge, [&](long long, uint64_t x) {
                        any = any || x >= wl;
                        if (x >= wl && x < next) next = x;
                    });
#pragma unroll
                    for (int o = 32; o > 0; o >>= 1) {
                        const uint64_t x = (uint64_t)__shfl_xor((unsigned long long)next, o, 64);
                        next = x < next ? x : next;
                    }
                    __syncthreads();
                    if (tid == 0) s_cnt = 0;
                    if (tid <= 64) s_bits[tid] = 0;
                    if (lane_id() == 0) s_red[tid >> 6] = (long long)next;
                    __syncthreads();
                    if (any) s_cnt = 1;
                    __syncthreads();
                    if (s_cnt == 0) {
                        sub = false;
                        gc = ge;
                        continue;
                    }
                    wl = (uint64_t)s_red[0];
                    for (int q = 1; q < CL_T / 64; ++q) wl = min(wl, (uint64_t)s_red[q]);
                    int equal = 0;
                    scan_keys<UK>(skey, gc, ge, [&](long long, uint64_t x) {
                        if (x == wl)
                            ++equal;
                        else if (x > wl)
                            atomicAdd(&s_bits[64 - __clzll((long long)(x ^ wl))], 1);
                    });
                    if (equal) atomicAdd(&s_bits[0], equal);
                    __syncthreads();
                    m = s_bits[0];
                    hot = m > CL_CAP;
                    wu = wl;
                    for (int b = 1; b <= sh && !hot && m + s_bits[b] <= CL_CAP; ++b) {
                        m += s_bits[b];
                        wu = wl | ((1ull << b) - 1);
                    }
                    if (!hot) {
                        picked = true;
                        __syncthreads();
                        if (tid == 0) s_cnt = 0;
                        __syncthreads();
                        scan_keys<UK>(skey, gc, ge, [&](long long e, uint64_t x) {
                            if (x >= wl && x <= wu) spare[gc + atomicAdd(&s_cnt, 1)] = (uint32_t)(e - gc);
                        });
                        __syncthreads();
#pragma unroll
                        for (int r = 0; r < CL_I; ++r) {
                            const int l = r * CL_T + tid;
                            sk[r] = l < m ? skey[gc + spare[gc + l]] : ~0ull;
                        }
                    }
                }
            }
            // place q of the window -> record of the list
            auto place = [&](int q) -> long long { return picked ? gc + spare[gc + q] : base + q; };
            auto place_key = [&](int q, uint64_t (&k)[W]) {
                if constexpr (STAGE) {
#pragma unroll
                    for (int x = 0; x < W; ++x) k[x] = s_key[x][q];
                } else {
                    rec_key<W>(w, idx[place(q)], k);
                }
            };
            if (hot) {
                // More records than a window on one sort key. Nearly always one
                // determinant: every key is compared with one of them.
                __syncthreads();
                if (tid == 0) s_cnt = 0x7FFFFFFF;
                __syncthreads();
                for (long long e = gc + tid; e < ge; e += CL_T)
                    if (skey[e] == wl) {
                        atomicMin(&s_cnt, (int)(e - gc));
                        break;
                    }
                __syncthreads();
                uint64_t prev[W];
                rec_key<W>(w, idx[gc + s_cnt], prev);
                bool mixed = false;
                bool one = true;  // the first round: the key just read
                for (int d = 0;; ++d) {
                    long long sum, cnt;
                    if (group_sum<W, UR>(w.sp.rec, skey, idx, gc, ge, wl, prev, sum, cnt)) mixed = true;
                    long long es, ec, ts, tc;
                    block_excl_scan2(sum, cnt, es, ec, ts, tc, s_red);
                    if (one) {
                        if (tid == 0) s_coll = 0;
                        __syncthreads();
                        if (mixed) s_coll = 1;
                        __syncthreads();
                        mixed = s_coll != 0;
                    }
                    if (!one || !mixed) {
                        if (tid == 0) {
                            const long long o = g0 + written;
                            w.u.skey[o] = wl;
                            s_lastk[W] = wl;
#pragma unroll
                            for (int q = 0; q < W; ++q) {
                                w.u.key[(size_t)q * w.spawn_cap + o] = prev[q];
                                s_lastk[q] = prev[q];
                            }
                            w.u.sum[o] = ts;
                            w.u.flag[o] = (tc >> 32) ? UNIQ_INITIATOR : 0u;
                            acc_put((int)skey_rep(wl, w.rb), tc & 0xFFFFFFFFll, ts, 1);
                        }
                        ++written;
                    }
                    if (!mixed) break;
                    // several: one after another, the smallest key above the last one
                    // (only the first CL_MIN threads keep minima: they fit s_x)
                    constexpr int CL_MIN = CL_CAP / W < CL_T ? CL_CAP / W : CL_T;
                    uint64_t(*s_k)[W] = (uint64_t(*)[W])s_x;
                    bool have = false;
                    uint64_t best[W];
#pragma unroll
                    for (int q = 0; q < W; ++q) best[q] = ~0ull;
                    for (long long e = gc + tid; e < ge && tid < CL_MIN; e += CL_MIN) {
                        if (skey[e] != wl) continue;
                        uint64_t k[W];
                        rec_key<W>(w, idx[e], k);
                        if (!one && key_cmp<W>(k, prev) <= 0) continue;
                        if (!have || key_cmp<W>(k, best) < 0) {
#pragma unroll
                            for (int q = 0; q < W; ++q) best[q] = k[q];
                            have = true;
                        }
                    }
                    one = false;
                    __syncthreads();
                    if (tid == 0) s_cnt = 0;
                    __syncthreads();
                    if (tid < CL_MIN) {
#pragma unroll
                        for (int q = 0; q < W; ++q) s_k[tid][q] = best[q];
                    }
                    if (have) s_cnt = 1;
                    __syncthreads();
                    if (s_cnt == 0) break;
                    if (d == CL_MAX_KEYS) {
                        if (tid == 0) atomicOr(&c->err, ERR_COLLISION);
                        break;
                    }
                    for (int o = CL_MIN / 2; o > 0; o >>= 1) {
                        if (tid < o && key_cmp<W>(s_k[tid + o], s_k[tid]) < 0) {
#pragma unroll
                            for (int q = 0; q < W; ++q) s_k[tid][q] = s_k[tid + o][q];
                        }
                        __syncthreads();
                    }
#pragma unroll
                    for (int q = 0; q < W; ++q) prev[q] = s_k[0][q];
                    __syncthreads();
                }
                __syncthreads();
            } else if (m > 0) {
                if (tid == 0) {
                    s_coll = 0;
                    s_big = 0;
                }
                // sort keys and records of the window, by place
#pragma unroll
                for (int r = 0; r < CL_I; ++r) {
                    const int l = r * CL_T + tid;
                    const int q = over ? l : l - l0;
                    if (q < 0 || q >= m) continue;
                    const uint64_t *rec = w.sp.rec + (size_t)idx[place(q)] * (W + 1);
                    const uint64_t ai = rec[W];
                    if constexpr (STAGE) {
#pragma unroll
                        for (int x = 0; x < W; ++x) s_key[x][q] = rec[x];
                    }
                    s_x[q] = sk[r];
                    s_am[q] = (int32_t)(uint32_t)ai;
                    s_ini[q] = (uint32_t)(ai >> 32) ? 1 : 0;
                    s_mix[q] = 0;
                }
                __syncthreads();
                // each thread's run of places: where their groups start, and
                // which groups hold several sort keys
                int gs[CL_I];
                {
                    int lastp = -1;
                    bool diff[CL_I];
#pragma unroll
                    for (int r = 0; r < CL_I; ++r) {
                        const int q = tid * CL_I + r;
                        gs[r] = -1;
                        diff[r] = false;
                        if (q >= m) continue;
                        bool start = q == 0;
                        if (!start) {
                            const uint64_t a = s_x[q - 1], b = s_x[q];
                            start = !picked && (a >> sh) != (b >> sh);
                            diff[r] = a != b;
                        }
                        if (start) lastp = q;
                        gs[r] = lastp;
                        diff[r] = diff[r] && !start;
                    }
                    int x = lastp;
#pragma unroll
                    for (int o = 1; o < 64; o <<= 1) {
                        const int y = __shfl_up(x, o, 64);
                        if (lane_id() >= o) x = max(x, y);
                    }
                    if (lane_id() == 63) s_gs[tid >> 6] = x;
                    int before = __shfl_up(x, 1, 64);
                    if (lane_id() == 0) before = -1;
                    __syncthreads();
                    for (int q = 0; q < (tid >> 6); ++q) before = max(before, s_gs[q]);
#pragma unroll
                    for (int r = 0; r < CL_I; ++r) {
                        if (gs[r] < 0) gs[r] = before;
                        if (diff[r]) s_mix[gs[r]] = 1;
                    }
                }
                __syncthreads();
#pragma unroll
                for (int r = 0; r < CL_I; ++r) {
                    const int q = tid * CL_I + r;
                    if (q < m && q - gs[r] >= CL_COUNT && s_mix[gs[r]]) s_big = 1;
                }
                __syncthreads();
                if (!s_big) {
#pragma unroll
                    for (int r = 0; r < CL_I; ++r) {
                        const int q = tid * CL_I + r;
                        if (q >= m) continue;
                        int pos = q;
                        if (s_mix[gs[r]]) {
                            const uint64_t my = s_x[q];
                            pos = gs[r];
                            for (int j = gs[r]; j < m; ++j) {
                                const uint64_t o = s_x[j];
                                if (!picked && (o >> sh) != (my >> sh)) break;
                                pos += (o < my || (o == my && j < q)) ? 1 : 0;
                            }
                        }
                        s_ord[pos] = (uint16_t)q;
                    }
                } else {
                    uint64_t v[CL_I];
#pragma unroll
                    for (int r = 0; r < CL_I; ++r) {
                        const int q = tid * CL_I + r;
                        v[r] = q < m ? (s_x[q] & ~CL_LOW) | (uint64_t)q : ~0ull;
                    }
                    block_sort(v, s_x);
                    __syncthreads();
#pragma unroll
                    for (int r = 0; r < CL_I; ++r) {
                        const int q = tid * CL_I + r;
                        if (q >= m) continue;
                        s_ord[q] = (uint16_t)(v[r] & CL_LOW);
                        s_x[q] = skey[place(q)];
                    }
                }
                __syncthreads();
                // neighbours on one sort key are on one determinant, and the order
                // is final, but for collisions and the network's low bits
                {
                    bool bad = false;
#pragma unroll
                    for (int r = 0; r < CL_I; ++r) {
                        const int p = tid * CL_I + r;
                        if (p == 0 || p >= m) continue;
                        const int a = s_ord[p - 1], b = s_ord[p];
                        const uint64_t sa = s_x[a], sb = s_x[b];
                        if (sa < sb) continue;
                        if (sa > sb) {
                            bad = true;
                        } else {
                            uint64_t ka[W], kb[W];
                            place_key(a, ka);
                            place_key(b, kb);
                            bad = bad || !key_eq<W>(ka, kb);
                        }
                    }
                    if (bad) s_coll = 1;
                }
                __syncthreads();
                const bool coll = s_coll != 0;
                if (coll) {
                    // order by (sort key, key): neighbours swapped until none is out of order
                    auto after = [&](int a, int b) -> bool {
                        const uint64_t sa = s_x[a], sb = s_x[b];
                        if (sa != sb) return sa > sb;
                        uint64_t ka[W], kb[W];
                        place_key(a, ka);
                        place_key(b, kb);
                        return key_cmp<W>(ka, kb) > 0;
                    };
                    for (bool again = true; again;) {
                        __syncthreads();
                        if (tid == 0) s_swap = 0;
                        __syncthreads();
                        for (int ph = 0; ph < 2; ++ph) {
                            for (int p = 2 * tid + ph; p + 1 < m; p += 2 * CL_T) {
                                const uint16_t a = s_ord[p], b = s_ord[p + 1];
                                if (after(a, b)) {
                                    s_ord[p] = b;
                                    s_ord[p + 1] = a;
                                    s_swap = 1;
                                }
                            }
                            __syncthreads();
                        }
                        again = s_swap != 0;
                    }
                    // determinants on one sort key
                    for (int p = tid; p < m; p += CL_T) {
                        const uint64_t s0 = s_x[s_ord[p]];
                        if (p > 0 && s_x[s_ord[p - 1]] == s0) continue;
                        int d = 1;
                        uint64_t k0[W];
                        place_key(s_ord[p], k0);
                        for (int x = p + 1; x < m && s_x[s_ord[x]] == s0; ++x) {
                            uint64_t k[W];
                            place_key(s_ord[x], k);
                            if (!key_eq<W>(k, k0)) {
                                ++d;
#pragma unroll
                                for (int q = 0; q < W; ++q) k0[q] = k[q];
                            }
                        }
                        if (d > CL_MAX_KEYS) atomicOr(&c->err, ERR_COLLISION);
                    }
                    __syncthreads();
                }
                // heads, amplitudes and flags of this thread's run of positions
                uint32_t heads = 0;
                int nh = 0, nf = 0;
                int32_t am[CL_I];
                uint16_t pl[CL_I];
                uint32_t fl = 0;
                long long sum = 0;
#pragma unroll
                for (int r = 0; r < CL_I; ++r) {
                    const int p = tid * CL_I + r;
                    am[r] = 0;
                    pl[r] = 0;
                    if (p >= m) continue;
                    const int b = s_ord[p];
                    pl[r] = (uint16_t)b;
                    bool head = p == 0;
                    if (!head) {
                        const int a = s_ord[p - 1];
                        head = s_x[a] != s_x[b];
                        if (coll && !head) {
                            uint64_t ka[W], kb[W];
                            place_key(a, ka);
                            place_key(b, kb);
                            head = !key_eq<W>(ka, kb);
                        }
                    }
                    if (head) {
                        heads |= 1u << r;
                        ++nh;
                    }
                    am[r] = s_am[b];
                    sum += am[r];
                    if (s_ini[b]) {
                        fl |= 1u << r;
                        ++nf;
                    }
                    if (w.R > 1) acc_put((int)skey_rep(s_x[b], w.rb), 1, am[r], head ? 1 : 0);
                }
                long long es, eh, ts, th;
                block_excl_scan2(sum, ((long long)nf << 32) | nh, es, eh, ts, th, s_red);
                const int nseg = (int)(th & 0xFFFFFFFFll);
                // sums and flag counts before each segment, and its head's place
                // (every thread has read the sort keys and places it needs)
                {
                    int seg = (int)(eh & 0xFFFFFFFFll), f = (int)(eh >> 32);
                    long long run = es;
#pragma unroll
                    for (int r = 0; r < CL_I; ++r) {
                        if ((heads >> r) & 1u) {
                            s_x[seg] = (uint64_t)run;
                            s_fl[seg] = (uint16_t)f;
                            s_ord[seg] = pl[r];
                            ++seg;
                        }
                        run += am[r];
                        f += (fl >> r) & 1u;
                    }
                    if (tid == 0) {
                        s_x[nseg] = (uint64_t)ts;
                        s_fl[nseg] = (uint16_t)(th >> 32);
                    }
                }
                __syncthreads();
                const long long ob = g0 + written;
                for (int q = tid; q < nseg; q += CL_T) {
                    const int l = s_ord[q];
                    uint64_t k[W];
                    place_key(l, k);
                    const long long o = ob + q;
                    const uint64_t ks = skey[place(l)];
                    w.u.skey[o] = ks;
#pragma unroll
                    for (int x = 0; x < W; ++x) w.u.key[(size_t)x * w.spawn_cap + o] = k[x];
                    if (q == nseg - 1) {
                        s_lastk[W] = ks;
#pragma unroll
                        for (int x = 0; x < W; ++x) s_lastk[x] = k[x];
                    }
                    w.u.sum[o] = (long long)(s_x[q + 1] - s_x[q]);
                    w.u.flag[o] = s_fl[q + 1] != s_fl[q] ? UNIQ_INITIATOR : 0u;
                }
                if (w.R == 1 && tid == 0) acc_put(0, m, ts, nseg);
                written += nseg;
            }
            if (!over) break;
            if (sub) {
                if (wu >= wend) {
                    sub = false;
                    gc = ge;
                } else {
                    wl = wu + 1;
                }
            }
        }
        // the rest of the tile's room: copies of its last determinant, marked
        __syncthreads();
        for (long long o = g0 + written + tid; o < g1; o += CL_T) {
            w.u.skey[o] = s_lastk[W];
#pragma unroll
            for (int x = 0; x < W; ++x) w.u.key[(size_t)x * w.spawn_cap + o] = s_lastk[x];
            w.u.flag[o] = UNIQ_FILLER;
        }
    }
    acc_flush();
    __syncthreads();
    for (int i = tid; i < rl * EST_FIELDS; i += CL_T) w.part_red[(size_t)i * PART_MAX_BLOCKS + blockIdx.x] = tab[i];
}

hipError_t enqueue_collapse(const Work &w, const Grids &g, int passes, hipStream_t s)
{
    const uint64_t *sk = passes & 1 ? w.sp.skey2 : w.sp.skey;
    const uint32_t *ix = passes & 1 ? w.sp.idx2 : w.sp.idx;
    uint32_t *spare = passes & 1 ? w.sp.idx : w.sp.idx2;
    const int accb = acc_rows(w.R) * EST_FIELDS * 8;
    auto launch = [&](auto width) {
        constexpr int W = decltype(width)::value;
        if (g.heavy)
            k_collapse<W, true><<<g.reduce, CL_T, accb, s>>>(w, sk, ix, spare, passes);
        else
            k_collapse<W, false><<<g.reduce, CL_T, accb, s>>>(w, sk, ix, spare, passes);
    };
    switch (w.W) {
    case 1: launch(std::integral_constant<int, 1>()); break;
    case 2: launch(std::integral_constant<int, 2>()); break;
    case 4: launch(std::integral_constant<int, 4>()); break;
    case 8: launch(std::integral_constant<int, 8>()); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

int collapse_occupancy()
{
    int nb = 1;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_collapse<2, false>, CL_T, 0) != hipSuccess) nb = 1;
    return nb < 1 ? 1 : nb;
}

}  // namespace fq
