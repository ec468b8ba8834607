// Annihilation merge (paper Sec. 2.4, appendix "Parallelization") fused with
// death and the initiator rule, and the diagonal elements of new determinants,
// for gfx950.
#include "fq_kernels.h"
#include "fq_scan.h"

namespace fq {

// ---------------------------------------------------------------------------
// estimator accumulation. A thread sums its values in registers for one
// replica at a time; when it moves on to another replica (and at the end of
// the kernel) the values go to the block's table in LDS (replicas below
// acc_rows(R); others are added to global memory directly). At the end each
// block stores its table as one row of partials with plain stores and the
// iteration epilogue folds the rows. The accumulators are a few addresses
// that every block would otherwise hit with device-scope atomics.
// ---------------------------------------------------------------------------
struct MergeAcc {
    enum { NW, NOCC, FLIPS, DEATH, REJU, REJ, N };
    long long v[N];
    int rep;
    static __device__ __forceinline__ int field(int i)
    {
        return i == NW ? F_NW : i == NOCC ? F_NOCC : i == FLIPS ? F_FLIPS : i == DEATH ? F_DEATH : i == REJU ? F_REJU : F_REJ;
    }
    __device__ void clear()
    {
#pragma unroll
        for (int i = 0; i < N; ++i) v[i] = 0;
    }
    // the thread's values to the block table, lane by lane
    __device__ void spill(long long *tab, int rl, EstAcc *g)
    {
        if (rep < 0) return;
#pragma unroll
        for (int i = 0; i < N; ++i)
            if (v[i]) acc_add(tab, rl, g, rep, field(i), v[i]);
        clear();
    }
    __device__ __forceinline__ void use(int r, long long *tab, int rl, EstAcc *g)
    {
        if (r == rep) return;
        spill(tab, rl, g);
        rep = r;
    }
    // end of a kernel (all threads): reduced over the wave when its active
    // lanes hold one replica
    __device__ void finish(long long *tab, int rl, EstAcc *g)
    {
        const bool active = rep >= 0;
        const uint64_t act = __ballot(active);
        if (!act) return;
        const int leader = __ffsll((unsigned long long)act) - 1;
        const int rep0 = __shfl(rep, leader, 64);
        if (__ballot(active && rep != rep0) == 0) {
#pragma unroll
            for (int i = 0; i < N; ++i) {
                const long long sv = wave_sum<long long>(active ? v[i] : 0);
                if (lane_id() == leader && sv != 0) acc_add(tab, rl, g, rep0, field(i), sv);
            }
        } else {
            spill(tab, rl, g);
        }
        clear();
    }
};

// Reference population (or trace) and exact terms of the projected energy of
// one slot per lane, added at once: few entries have one, so they take no
// registers between tiles. All lanes of the wave call it.
__device__ void acc_terms(long long *tab, int rl, EstAcc *g, int rep, int32_t n0, bool term, double x)
{
    long long l0 = 0, l1 = 0, l2 = 0, l3 = 0;
    if (term) add_limbs4(l0, l1, l2, l3, x);
    const uint64_t act = __ballot(n0 != 0 || term);
    const int leader = __ffsll((unsigned long long)act) - 1;
    const int rep0 = __shfl(rep, leader, 64);
    const bool mine = n0 != 0 || term;
    if (__popcll(act) > 4 && __ballot(mine && rep != rep0) == 0) {
        l0 = wave_sum<long long>(l0);
        l1 = wave_sum<long long>(l1);
        l2 = wave_sum<long long>(l2);
        l3 = wave_sum<long long>(l3);
        const long long n = wave_sum<long long>((long long)n0);
        if (lane_id() == leader) {
            if (n) acc_add(tab, rl, g, rep0, F_N0, n);
            if (l0) acc_add(tab, rl, g, rep0, F_L0, l0);
            if (l1) acc_add(tab, rl, g, rep0, F_L1, l1);
            if (l2) acc_add(tab, rl, g, rep0, F_L2, l2);
            if (l3) acc_add(tab, rl, g, rep0, F_L3, l3);
        }
    } else if (mine) {
        if (n0) acc_add(tab, rl, g, rep, F_N0, n0);
        if (l0) acc_add(tab, rl, g, rep, F_L0, l0);
        if (l1) acc_add(tab, rl, g, rep, F_L1, l1);
        if (l2) acc_add(tab, rl, g, rep, F_L2, l2);
        if (l3) acc_add(tab, rl, g, rep, F_L3, l3);
    }
}

// ---------------------------------------------------------------------------
// annihilation merge (Sec. 2.4; appendix "Parallelization"): merge-path merge
// of the distinct spawned determinants into the sorted main list, fused with
// death/cloning of existing entries, the deterministic-space update, the
// initiator rule for new determinants (Sec. 2.1), removal of empty entries,
// the estimators of the new list (tutorial appendix) and the attempt counts of
// the next iteration. Ties in the merge order put the main entry first.
//
// Two kernels. k_merge decides: for each merge position the new population
// and the slot it comes from, and how many entries each tile keeps. k_move
// writes the kept entries at their places. A block takes a run of neighbouring
// tiles, so a block's place in the output is a sum over the runs before it,
// read when k_move starts; no tile waits for another. (One kernel with a
// decoupled look-back moved 65 bytes per entry instead of 101 but took 2890 us
// for 6e7 entries: its time fitted 8.6 ns per tile + 2310 us, a tile being held
// up by every tile in flight before it, and wider look-back reads made it
// slower, 3650 us. Now k_merge 1480 us, 2.2 TB/s and 44% of it vector ALU, the
// rest the latency of loads, bisection and rounding; k_move 1160 us, 4.1 TB/s.)
// ---------------------------------------------------------------------------
// MI: merge positions per thread and tile, 1, 2 or 4 for keys of up to two
// words (chosen per context), 2 for longer keys
template <int W, int MI>
struct MergeCfg {
    static constexpr int T = 256;
    static constexpr int TILE = T * MI;
    static constexpr int WPE = MI >= 4 || W > 2 ? 4 : (MI == 2 ? 5 : 6);  // waves per SIMD
};
static_assert(MergeCfg<1, 1>::TILE >= MERGE_TILE_MIN && MergeCfg<8, 2>::TILE >= MERGE_TILE_MIN,
              "the splits and totals of the merge are sized for MERGE_TILE_MIN-position tiles");

template <int W>
__device__ __forceinline__ void load_key(const uint64_t *base, long long cap, long long i, uint64_t (&k)[W])
{
#pragma unroll
    for (int q = 0; q < W; ++q) k[q] = base[(size_t)q * cap + i];
}

// sort key of main entry i (see stored_skey)
template <int W>
__device__ __forceinline__ uint64_t main_skey(const Work &w, long long i)
{
    if (stored_skey(w.rb != 0, W)) return w.cur.skey[i];
    uint64_t k[W];
    load_key<W>(w.cur.key, w.main_cap, i, k);
    return hash64<W>(k);
}

// main[i] <= uniq[j] in (sort key, key) order (global memory)
template <int W>
__device__ __forceinline__ bool le_ab(const Work &w, long long i, uint64_t si, long long j, uint64_t sj)
{
    if (si != sj) return si < sj;
    uint64_t a[W], b[W];
    load_key<W>(w.cur.key, w.main_cap, i, a);
    load_key<W>(w.u.key, w.spawn_cap, j, b);
    return key_cmp<W>(a, b) <= 0;
}

// Split of merge diagonal d: how many main entries come before it. Without a
// replica field the sort keys are hashes, spread evenly, so the split is looked
// for within a few standard deviations of its expected place first.
struct SplitRange {
    long long lo, hi, a, b;
    __device__ SplitRange(const Work &w, long long d, long long na, long long nb)
    {
        lo = max(0ll, d - nb);
        hi = min(d, na);
        a = lo;
        b = hi;
        if (w.rb == 0 && hi - lo > 4096) {
            const double g = (double)d * ((double)na / (double)(na + nb)), s = 4.0 * sqrt((double)hi);
            a = min(max(lo, (long long)(g - s)), hi);
            b = max(min(hi, (long long)(g + s)), lo);
        }
    }
};

template <int W>
__device__ __forceinline__ bool split_after(const Work &w, long long d, long long i)
{
    const long long j = d - 1 - i;
    return le_ab<W>(w, i, main_skey<W>(w, i), j, w.u.skey[j]);
}

// by one thread
template <int W>
__device__ long long split_thread(const Work &w, long long d, long long na, long long nb)
{
    SplitRange r(w, d, na, nb);
    long long lo = r.lo, hi = r.hi;
    if (r.a > lo) {
        if (split_after<W>(w, d, r.a - 1)) lo = r.a; else hi = r.a - 1;
    }
    if (r.b < hi && r.b >= lo) {
        if (split_after<W>(w, d, r.b)) lo = r.b + 1; else hi = r.b;
    }
    while (lo < hi) {
        const long long mid = (lo + hi) >> 1;
        if (split_after<W>(w, d, mid)) lo = mid + 1; else hi = mid;
    }
    return lo;
}

// by a wavefront, 64 places at once
template <int W>
__device__ long long split_wave(const Work &w, long long d, long long na, long long nb)
{
    SplitRange r(w, d, na, nb);
    const int lane = lane_id();
    long long lo = r.lo, hi = r.hi;
    if (r.a > lo || r.b < hi) {
        const bool in = lane == 0 ? r.a > lo : lane == 1 && r.b < hi;
        const uint64_t yes = __ballot(in && split_after<W>(w, d, lane == 0 ? r.a - 1 : r.b));
        if (r.a > lo) {
            if (yes & 1) lo = r.a; else hi = r.a - 1;
        }
        if (r.b < hi && r.b >= lo) {
            if (yes & 2) lo = r.b + 1; else hi = r.b;
        }
    }
    while (lo < hi) {
        const long long step = (hi - lo + 63) >> 6;
        const long long p = lo + lane * step;
        const int cnt = __popcll(__ballot(p < hi && split_after<W>(w, d, p)));  // they come first
        if (cnt == 0) return lo;
        hi = min(hi, lo + cnt * step);
        lo += (cnt - 1) * step + 1;
    }
    return lo;
}

// spawning attempts of an entry holding p units: |p| for integer walkers,
// ceil(|p| 2^-b) for fixed point, times mult (2 for DMQMC pairs: that many
// at each end); 2^28 or more does not fit the counter's attempt field
constexpr long long MAX_ATTEMPTS = 1ll << 28;
__device__ __forceinline__ long long attempts_of(long long p, int bits, int mult)
{
    const long long ap = p < 0 ? -p : p;
    return mult * (bits == 0 ? ap : (ap + (1ll << bits) - 1) >> bits);
}

// a tile's totals in one word: kept entries above MT_SHIFT, attempts below
// (fewer than 2^28 each for at most 1024 entries)
constexpr int MT_SHIFT = 44;
constexpr long long MT_MASK = (1ll << MT_SHIFT) - 1;
// place of a merge position's entry: slot of its tile, and whether it is kept
constexpr uint32_t MS_KEEP = 0x8000u;

template <int KIND, int W, bool MULTI, int MI>
__global__ __launch_bounds__((MergeCfg<W, MI>::T), (MergeCfg<W, MI>::WPE)) void k_merge(Work w)
{
    Ctl *c = w.ctl;
    constexpr int MG_T = MergeCfg<W, MI>::T, TILE = MergeCfg<W, MI>::TILE;
    __shared__ uint64_t s_sk[TILE];            // sort keys by slot
    constexpr int CHUNK = 64;                  // tiles whose splits are found at once
    __shared__ long long s_split[CHUNK + 1];
    __shared__ uint64_t s_pa_sk, s_pa_key[W];  // main entry before the tile
    __shared__ uint64_t s_nb_sk, s_nb_key[W];  // spawned entry after the tile
    __shared__ long long s_nb_sum;
    __shared__ int s_pa_ok, s_nb_ok;
    __shared__ long long s_red[MG_T / 64];
    const long long na = c->n_main, nb = (long long)min(c->n_spawn, (unsigned long long)w.spawn_cap);
    const long long ntiles = (na + nb + TILE - 1) / TILE;
    const long long run = (ntiles + gridDim.x - 1) / gridDim.x;  // tiles of a block
    const long long t0 = min((long long)blockIdx.x * run, ntiles), t1 = min(t0 + run, ntiles);
    const uint32_t t = c->t;
    const bool ss = c->ss_active != 0;
    const int tid = threadIdx.x;
    if (block_stops(c)) return;
    extern __shared__ __align__(16) unsigned char dyn_lds[];
    long long *tab = (long long *)dyn_lds;  // estimator table, acc_rows(R) rows
    const int rl = acc_rows(w.R);
    acc_table_clear(tab, rl);
    MergeAcc acc;
    acc.clear();
    acc.rep = -1;
    // time-step search: the largest K_ii of the entries this thread's death steps act on
    const bool ts = w.tau_search != 0;
    double kd_max = -INFINITY;
    int kd_rep = 0;
    long long run_cnt = 0, run_att = 0;  // thread 0: of the block's tiles
    for (long long tile = t0; tile < t1; ++tile) {
        const int at = (int)((tile - t0) % CHUNK);
        if (at == 0) {
            // the splits of the next tiles: a wavefront each while they are few
            const int n = (int)min((long long)CHUNK, t1 - tile) + 1;
            __syncthreads();
            if (n <= 8) {
                for (int q = tid >> 6; q < n; q += MG_T / 64) {
                    const long long i = split_wave<W>(w, min((tile + q) * TILE, na + nb), na, nb);
                    if (lane_id() == 0) s_split[q] = i;
                }
            } else if (tid < n) {
                s_split[tid] = split_thread<W>(w, min((tile + tid) * TILE, na + nb), na, nb);
            }
            __syncthreads();
            for (int q = tid; q < n; q += MG_T) w.mpart[tile + q] = s_split[q];
        }
        const long long d0 = tile * TILE, d1 = min(d0 + TILE, na + nb);
        const long long i0 = s_split[at], i1 = s_split[at + 1];
        const long long j0 = d0 - i0, j1 = d1 - i1;
        const int la = (int)(i1 - i0), lb = (int)(j1 - j0);
        // slot it * MG_T + tid: main entries in [0, la), spawned ones in [la, la + lb)
        uint64_t key[MI][W], sk[MI];
        int32_t pop[MI], dsl[MI];  // main: population, slot in the deterministic space; spawned: -, flags
        long long val[MI];         // main: the bits of K_ii - H_00; spawned: the sum
#pragma unroll
        for (int it = 0; it < MI; ++it) {
            const int q = it * MG_T + tid;
            pop[it] = 0;
            dsl[it] = -1;
            if (q < la) {
                const long long g = i0 + q;
                load_key<W>(w.cur.key, w.main_cap, g, key[it]);
                pop[it] = w.cur.pop[g];
                val[it] = __double_as_longlong(w.cur.kdiag[g]);
                if (ss) dsl[it] = w.cur.dslot[g];
                sk[it] = stored_skey(MULTI, W) ? w.cur.skey[g] : hash64<W>(key[it]);
                s_sk[q] = sk[it];
            } else if (q < la + lb) {
                const long long g = j0 + (q - la);
                sk[it] = w.u.skey[g];
                load_key<W>(w.u.key, w.spawn_cap, g, key[it]);
                val[it] = w.u.sum[g];
                dsl[it] = (int32_t)w.u.flag[g];
                s_sk[q] = sk[it];
            }
        }
        if (tid == 0) {
            s_pa_ok = i0 > 0;
            if (i0 > 0) {
                uint64_t k[W];
                load_key<W>(w.cur.key, w.main_cap, i0 - 1, k);
#pragma unroll
                for (int x = 0; x < W; ++x) s_pa_key[x] = k[x];
                s_pa_sk = stored_skey(MULTI, W) ? w.cur.skey[i0 - 1] : hash64<W>(k);
            }
        } else if (tid == 64) {
            s_nb_ok = j1 < nb;
            if (j1 < nb) {
                s_nb_sk = w.u.skey[j1];
#pragma unroll
                for (int x = 0; x < W; ++x) s_nb_key[x] = w.u.key[(size_t)x * w.spawn_cap + j1];
                s_nb_sum = w.u.sum[j1];
            }
        }
        __syncthreads();
        long long loc = 0;
#pragma unroll
        for (int it = 0; it < MI; ++it) {
            const int q = it * MG_T + tid;
            bool kept = false;
            int rep = 0;
            if (q < la) {
                const uint64_t x = sk[it];
                rep = MULTI ? (int)skey_rep(x, w.rb) : 0;
                const RepParams &rp = w.rep[rep];
                acc.use(rep, tab, rl, w.acc);
                // spawned entries before it, and the one on the same determinant
                int j = 0, hi = lb;
                while (j < hi) {
                    const int mid = (j + hi) >> 1;
                    if (s_sk[la + mid] < x) j = mid + 1; else hi = mid;
                }
                long long add = 0;
                while (j < lb && s_sk[la + j] == x) {
                    uint64_t kb[W];
                    load_key<W>(w.u.key, w.spawn_cap, j0 + j, kb);
                    const int r = key_cmp<W>(kb, key[it]);
                    if (r == 0) add = w.u.sum[j0 + j];
                    if (r >= 0) break;
                    ++j;
                }
                if (j == lb && s_nb_ok && s_nb_sk == x) {
                    bool e = true;
#pragma unroll
                    for (int y = 0; y < W; ++y) e = e && s_nb_key[y] == key[it][y];
                    if (e) add = s_nb_sum;
                }
                const int32_t n0 = pop[it];
                long long v;
                if (ss && dsl[it] >= 0) {
                    v = (long long)n0 + w.ds.delta[(size_t)rep * w.ds.n + dsl[it]];
                } else if (n0 != 0) {
                    const double kd = __longlong_as_double(val[it]);
                    if (ts) {
                        if (MULTI && rep != kd_rep) {
                            if (kd_max > -INFINITY) ts_put<true>(w, kd_rep, kd_max);
                            kd_max = -INFINITY;
                            kd_rep = rep;
                        }
                        kd_max = fmax(kd_max, kd);
                    }
                    const double an = (double)(n0 < 0 ? -(long long)n0 : (long long)n0);
                    const double mm = (rp.tau * (kd - w.shift[rep])) * an;
                    const uint64_t h = MULTI ? hash64<W>(key[it]) : x;
                    const U4 r = draw(TAG_DEATH, 0, t, h, rp.k0, rp.k1);
                    const double u = u53(r.x, r.y);
                    if (!(fabs(mm) < 0x1p40)) atomicOr(&c->err, ERR_OVERFLOW);
                    const long long k = mm >= 0.0 ? sround(mm, u) : -sround(-mm, u);
                    const long long sg = n0 > 0 ? 1 : -1;
                    v = (long long)n0 - sg * k;
                    if ((v > 0 && n0 < 0) || (v < 0 && n0 > 0)) acc.v[MergeAcc::FLIPS] += 1;
                } else {
                    v = 0;
                }
                acc.v[MergeAcc::DEATH] += v;
                v += add;
                if (v > 2147483647ll || v < -2147483647ll) atomicOr(&c->err, ERR_OVERFLOW);
                pop[it] = (int32_t)v;
                kept = v != 0 || dsl[it] >= 0;
                w.mpop[d0 + q + j] = (int32_t)v;
                w.msrc[d0 + q + j] = (uint16_t)((uint32_t)q | (kept ? MS_KEEP : 0u));
            } else if (q < la + lb) {
                const uint64_t x = sk[it];
                // main entries up to it; is the last of them the same determinant
                int i = 0, hi = la;
                while (i < hi) {
                    const int mid = (i + hi) >> 1;
                    if (s_sk[mid] <= x) i = mid + 1; else hi = mid;
                }
                bool matched = false;
                while (i > 0 && s_sk[i - 1] == x) {
                    uint64_t ka[W];
                    load_key<W>(w.cur.key, w.main_cap, i0 + i - 1, ka);
                    const int r = key_cmp<W>(ka, key[it]);
                    matched = r == 0;  // that entry's thread added the sum
                    if (r <= 0) break;
                    --i;
                }
                if (i == 0 && s_pa_ok && s_pa_sk == x) {
                    matched = true;
#pragma unroll
                    for (int y = 0; y < W; ++y) matched = matched && s_pa_key[y] == key[it][y];
                }
                const uint32_t fl = (uint32_t)dsl[it];
                if (!matched && !(fl & UNIQ_FILLER)) {
                    const long long sum = val[it];
                    rep = MULTI ? (int)skey_rep(x, w.rb) : 0;
                    const RepParams &rp = w.rep[rep];
                    acc.use(rep, tab, rl, w.acc);
                    if ((!rp.initiator || fl) && sum != 0) {
                        if (sum > 2147483647ll || sum < -2147483647ll) atomicOr(&c->err, ERR_OVERFLOW);
                        kept = true;
                        pop[it] = (int32_t)sum;
                    } else {
                        acc.v[MergeAcc::REJU] += sum < 0 ? -sum : sum;
                        acc.v[MergeAcc::REJ] += sum;
                    }
                }
                w.mpop[d0 + (q - la + i)] = pop[it];
                w.msrc[d0 + (q - la + i)] = (uint16_t)((uint32_t)q | (kept ? MS_KEEP : 0u));
            }
            // estimators and next iteration's attempts of a kept entry
            bool n0_term = false, term = false;
            double e = 0.0;
            const int32_t p = pop[it];
            if (kept) {
                const DevSys &sy = w.sys[w.rep[rep].sys];
                const long long natt = attempts_of(p, w.rep[rep].bits, w.dm == 1 ? 2 : 1);
                if (natt >= MAX_ATTEMPTS) atomicOr(&c->err, ERR_ATTEMPTS);
                loc += (1ll << MT_SHIFT) + natt;
                acc.v[MergeAcc::NW] += p < 0 ? -(long long)p : (long long)p;
                acc.v[MergeAcc::NOCC] += 1;
                if constexpr (is_pair(KIND)) {
                    // density matrix (Sec. 2.3): the trace sum_i rho_ii and
                    // Tr(rho H) = sum rho_ij H_ji over pairs at most doubly excited
                    constexpr int BK = base_kind(KIND), WH = W / 2;
                    uint64_t a[WH], b[WH];
                    int nd = 0;
#pragma unroll
                    for (int y = 0; y < WH; ++y) {
                        a[y] = key[it][y];
                        b[y] = key[it][WH + y];
                        nd += __popcll(a[y] ^ b[y]);
                    }
                    n0_term = nd == 0;
                    term = nd == 0 || nd == 2 || nd == 4;
                    if (nd == 0)
                        e = diag_element<BK, WH>(sy, a) * (double)p;
                    else if (term)
                        e = hij<BK, WH>(sy, b, a) * (double)p;
                } else {
                    const uint64_t(&ref)[W] = *(const uint64_t(*)[W])sy.ref;
                    int nd = 0;
#pragma unroll
                    for (int y = 0; y < W; ++y) nd += __popcll(key[it][y] ^ ref[y]);
                    n0_term = nd == 0;
                    term = nd == 2 || nd == 4;
                    if (term) e = hij<KIND, W>(sy, ref, key[it]) * (double)p;
                }
            }
            if (__any(n0_term || term)) acc_terms(tab, rl, w.acc, rep, n0_term ? p : 0, term, e);
        }
        loc = wave_sum<long long>(loc);
        if (lane_id() == 0) s_red[tid >> 6] = loc;
        __syncthreads();  // (also: the tile's sort keys have been read)
        if (tid == 0) {
            long long tot = 0;
#pragma unroll
            for (int q = 0; q < MG_T / 64; ++q) tot += s_red[q];
            w.mtile[tile] = tot;
            run_cnt += tot >> MT_SHIFT;
            run_att += tot & MT_MASK;
        }
    }
    if (tid == 0) {
        w.mrun[2 * blockIdx.x] = run_cnt;
        w.mrun[2 * blockIdx.x + 1] = run_att;
    }
    acc.finish(tab, rl, w.acc);
    __syncthreads();
    for (int i = tid; i < rl * EST_FIELDS; i += MG_T) w.part_mrg[(size_t)i * PART_MAX_BLOCKS + blockIdx.x] = tab[i];
    if (ts) ts_finish<true>(w, kd_max, kd_rep, kd_max > -INFINITY);
}

// Writes the entries k_merge has kept: merge position by merge position, each
// from its slot of the old list or of the spawned one. runs: blocks k_merge
// had. Bound: HBM; 6 bytes per position and 8W + 12 per entry read, 8W + 21
// written (one instance, no deterministic space).
constexpr int MV_T = 256;
template <int W, bool MULTI, int MI>
__global__ __launch_bounds__(MV_T) void k_move(Work w, int runs)
{
    Ctl *c = w.ctl;
    constexpr int TILE = MergeCfg<W, MI>::TILE, WAVES = MV_T / 64;
    static_assert(TILE == MV_T * MI, "a thread takes MI positions");
    __shared__ long long s_w[WAVES];
    __shared__ long long s_red[16];
    const int tid = threadIdx.x, lane = lane_id(), wid = tid >> 6;
    const bool ss = c->ss_active != 0;
    const long long na = c->n_main, nb = (long long)min(c->n_spawn, (unsigned long long)w.spawn_cap);
    const long long ntiles = (na + nb + TILE - 1) / TILE;
    const long long run = (ntiles + runs - 1) / runs, per = (ntiles + gridDim.x - 1) / gridDim.x;
    const long long t0 = min((long long)blockIdx.x * per, ntiles), t1 = min(t0 + per, ntiles);
    if (block_stops(c)) return;
    if (ntiles == 0 && blockIdx.x == 0 && tid == 0) {
        c->n_main_new = 0;
        w.att_off[0] = 0;
        c->n_att_new = 0;
    }
    if (t0 >= t1) return;
    // entries kept and attempts before this block's first tile
    long long base, abase;
    {
        long long n = 0, a = 0, xn, xa;
        const long long r0 = t0 / run;
        for (long long q = tid; q < r0; q += MV_T) {
            n += w.mrun[2 * q];
            a += w.mrun[2 * q + 1];
        }
        for (long long q = r0 * run + tid; q < t0; q += MV_T) {
            n += w.mtile[q] >> MT_SHIFT;
            a += w.mtile[q] & MT_MASK;
        }
        block_excl_scan2(n, a, xn, xa, base, abase, s_red);
    }
    for (long long tile = t0; tile < t1; ++tile) {
        const long long d0 = tile * TILE, d1 = min(d0 + TILE, na + nb);
        const long long i0 = w.mpart[tile], i1 = w.mpart[tile + 1];
        const long long j0 = d0 - i0;
        const int la = (int)(i1 - i0);
        // position wid * 64 MI + it * 64 + lane of the tile
        uint32_t src[MI];
        int32_t p[MI];
        long long x[MI];  // kept and attempts of the wave's positions up to this one
        long long sum = 0;
#pragma unroll
        for (int it = 0; it < MI; ++it) {
            const long long d = d0 + wid * 64 * MI + it * 64 + lane;
            src[it] = d < d1 ? w.msrc[d] : 0u;
            p[it] = d < d1 ? w.mpop[d] : 0;
        }
        uint64_t sk[MI];
#pragma unroll
        for (int it = 0; it < MI; ++it) {
            long long v = 0;
            sk[it] = 0;
            if (src[it] & MS_KEEP) {
                const int q = (int)(src[it] & (MS_KEEP - 1));
                if constexpr (stored_skey(MULTI, W)) sk[it] = q < la ? w.cur.skey[i0 + q] : w.u.skey[j0 + q - la];
                const int rep = MULTI ? (int)skey_rep(sk[it], w.rb) : 0;
                v = (1ll << MT_SHIFT) + attempts_of(p[it], w.rep[rep].bits, w.dm == 1 ? 2 : 1);
            }
            x[it] = v;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const long long y = __shfl_up(x[it], o, 64);
                if (lane >= o) x[it] += y;
            }
            const long long tot = __shfl(x[it], 63, 64);
            x[it] += sum - v;
            sum += tot;
        }
        __syncthreads();
        if (lane == 0) s_w[wid] = sum;
        __syncthreads();
        long long before = 0, total = 0;
#pragma unroll
        for (int q = 0; q < WAVES; ++q) {
            if (q < wid) before += s_w[q];
            total += s_w[q];
        }
        const long long tot = total >> MT_SHIFT, atot = total & MT_MASK;
        const bool fits = base + tot <= w.main_cap;
        if (!fits) {
            if (tid == 0) atomicOr(&c->err, ERR_MAIN_CAP);
        } else {
#pragma unroll
            for (int it = 0; it < MI; ++it) {
                if (!(src[it] & MS_KEEP)) continue;
                const int q = (int)(src[it] & (MS_KEEP - 1));
                const bool old = q < la;
                const long long g = old ? i0 + q : j0 + (q - la);
                const long long e = before + x[it];
                const long long o = base + (e >> MT_SHIFT);
                uint64_t key[W];
                if (old)
                    load_key<W>(w.cur.key, w.main_cap, g, key);
                else
                    load_key<W>(w.u.key, w.spawn_cap, g, key);
                // K_jj - H_00 of a new determinant is filled in by k_new_diag
                const double kd = old ? w.cur.kdiag[g] : __longlong_as_double(0x7FF8000000000000ll);
                if constexpr (stored_skey(MULTI, W)) w.nxt.skey[o] = sk[it];
#pragma unroll
                for (int y = 0; y < W; ++y) w.nxt.key[(size_t)y * w.main_cap + o] = key[y];
                w.nxt.pop[o] = p[it];
                w.nxt.kdiag[o] = kd;
                w.newdet[o] = old ? 0 : 1;
                w.att_off[o] = abase + (e & MT_MASK);
                if (ss) {
                    const int rep = MULTI ? (int)skey_rep(sk[it], w.rb) : 0;
                    const int32_t ds = old ? w.cur.dslot[g] : -1;
                    w.nxt.dslot[o] = ds;
                    if (ds >= 0) w.ds.pos[(size_t)rep * w.ds.n + ds] = (int32_t)o;
                }
            }
        }
        base += tot;
        abase += atot;
        if (tile == ntiles - 1 && tid == 0) {
            c->n_main_new = base;
            if (fits) w.att_off[base] = abase;
            c->n_att_new = abase;
        }
    }
}

// K_jj - H_00 of the determinants the merge has just created (marked NaN).
// Each block scans a chunk of the new list, queues the marked entries in LDS
// and evaluates them one per thread, so no lane idles on unmarked entries;
// for a single replica the diagonal's tables are read from LDS.
// New determinants are a few per cent of the list: a chunk must hold enough of
// them to fill the block's waves and to pay for its tables, and there must be
// enough chunks for the compute units: 4, 8, 16 or 32 flags per thread by the
// host's rule (Grids::diag_chunk).
constexpr int ND_T = DIAG_T;

// Diagonal of the electron gas on a large basis (its exchange table does not
// fit LDS). A thread lists its electrons, alpha and beta, as bytes in LDS; the
// exchange of a pair is v(|n_p - n_q|^2), the distance one dot product of bytes:
// pa = (n_p, 1), pb = (-2 n_q, |n_q|^2), |n_p - n_q|^2 = pa . pb + |n_p|^2. The
// terms are subtracted in the order of diag_ueg: rows P ascending (both spins),
// Q > P of the same spin ascending. Bound: LDS reads (12 bytes a pair at
// random). 54 electrons, 251
// plane waves, 4.4e6 determinants: 353 -> 118 us; 123 plane waves 35 -> 21 us.
struct DiagLists {
    const double *eps, *vtab;
    const int32_t *pa, *pb;
    uint32_t *word;  // this thread's list: four electrons a word, ND_T words apart
    int na, nb;

    template <int W>
    __device__ double operator()(const uint64_t (&key)[W]) const
    {
        const int wa = (na + 3) >> 2;
        unsigned char *byte = (unsigned char *)word;
        double e = 0.0;
        int ia = 0, ib = 0;
        for_bits<W>(key, [&](int P) {
            e = e + eps[P >> 1];
            const int k = (P & 1) ? 4 * wa + ib : ia;
            byte[(size_t)(k >> 2) * (4 * ND_T) + (k & 3)] = (unsigned char)(P >> 1);
            if (P & 1) ++ib; else ++ia;
        });
        auto at = [&](int k) -> int { return byte[(size_t)(k >> 2) * (4 * ND_T) + (k & 3)]; };
        ia = ib = 0;
        int ca = na > 0 ? at(0) : 0, cb = nb > 0 ? at(4 * wa) : 0;
        for (int r = 0; r < na + nb; ++r) {
            const bool alpha = ib >= nb || (ia < na && ca <= cb);  // 2a < 2b + 1
            const int p = alpha ? ca : cb, k = alpha ? ia : ib, n = alpha ? na : nb;
            const int w0 = alpha ? 0 : wa, wn = (n + 3) >> 2;
            const int32_t vp = pa[p], np = pb[p] >> 24;
            for (int w = (k + 1) >> 2; w < wn; ++w) {
                const uint32_t q4 = word[(w0 + w) * ND_T];
                double v[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int i = 4 * w + j;
                    const bool in = i > k && i < n;
                    const int q = in ? (int)((q4 >> (8 * j)) & 255u) : p;
                    v[j] = vtab[__builtin_amdgcn_sdot4(vp, pb[q], np, false)];
                    v[j] = in ? v[j] : 0.0;
                }
#pragma unroll
                for (int j = 0; j < 4; ++j) e = e - v[j];
            }
            if (alpha) {
                ++ia;
                ca = ia < na ? at(ia) : 0;
            } else {
                ++ib;
                cb = ib < nb ? at(4 * wa + ib) : 0;
            }
        }
        return e;
    }
};

// The blocks beyond nd_blocks end the iteration, one replica each: the merge is
// the last kernel that adds to the accumulators.
template <int KIND, int W>
__global__ __launch_bounds__(ND_T) void k_new_diag(Work w, int nd_blocks, int per, int nb_red, int nb_mrg)
{
    const Ctl *c = w.ctl;
    if (c->err) return;
    static_assert(ND_T == END_T, "the blocks that end the iteration have the size of the others");
    if ((int)blockIdx.x >= nd_blocks) {
        end_replica(w, (int)blockIdx.x - nd_blocks, nb_red, nb_mrg);
        return;
    }
    extern __shared__ __align__(16) unsigned char dyn_lds[];
    uint16_t *s_q = (uint16_t *)(dyn_lds + w.lds_diag + w.lds_list);  // offsets of the chunk's new determinants
    __shared__ int s_n;
    const long long n = c->n_main_new;
    const DevSys &s0 = w.sys[w.rep[0].sys];
    // the host stages tables only when every replica has the same system
    const bool local = w.lds_diag > 0 && (KIND == K_UEG || KIND == K_MOLECULAR);
    UegTables lu = s0.u;
    const double *lhd = s0.hd, *lJ = s0.Jt, *lK = s0.Kt;
    DiagLists lists{};
    constexpr bool LISTS = KIND == K_UEG && W > 2;
    if (local) {
        double *t0 = (double *)dyn_lds;
        const int m = s0.n_spatial;
        if (KIND == K_UEG) {
            if (8 * (m + m * m) <= ND_LDS_MAX) {
                // kinetic energies and the exchange table v(|n_p - n_q|^2)
                double *t1 = t0 + m;
                for (int i = threadIdx.x; i < m; i += ND_T) t0[i] = lu.eps[i];
                for (int i = threadIdx.x; i < m * m; i += ND_T) t1[i] = lu.vx[i];
                lu.eps = t0;
                lu.vx = t1;
            } else {
                // large bases: kinetic energies, v by |dn|^2 and the packed momenta
                const int nv = s0.vlen;
                double *t1 = t0 + m;
                int32_t *t2 = (int32_t *)(t1 + nv);
                for (int i = threadIdx.x; i < m; i += ND_T) t0[i] = lu.eps[i];
                for (int i = threadIdx.x; i < nv; i += ND_T) t1[i] = lu.vtab[i];
                for (int i = threadIdx.x; i < m; i += ND_T) t2[i] = lu.npk[i];
                lu.eps = t0;
                lu.vtab = t1;
                lu.npk = t2;
                lu.vx = nullptr;
                if (LISTS && w.lds_list > 0) {
                    int32_t *pa = t2 + m, *pb = pa + m;
                    for (int i = threadIdx.x; i < m; i += ND_T) {
                        const int32_t n = s0.u.npk[i];
                        const int x = pk_comp(n, 0), y = pk_comp(n, 1), z = pk_comp(n, 2);
                        pa[i] = (x & 255) | (y & 255) << 8 | (z & 255) << 16 | 1 << 24;
                        pb[i] = (-2 * x & 255) | (-2 * y & 255) << 8 | (-2 * z & 255) << 16 | (x * x + y * y + z * z) << 24;
                    }
                    lists.eps = t0;
                    lists.vtab = t1;
                    lists.pa = pa;
                    lists.pb = pb;
                    lists.word = (uint32_t *)(dyn_lds + w.lds_diag) + threadIdx.x;
                    lists.na = s0.na;
                    lists.nb = s0.nb;
                }
            }
        } else {
            double *t1 = t0 + m, *t2 = t1 + m * m;
            for (int i = threadIdx.x; i < m; i += ND_T) t0[i] = lhd[i];
            for (int i = threadIdx.x; i < m * m; i += ND_T) {
                t1[i] = lJ[i];
                t2[i] = lK[i];
            }
            lhd = t0;
            lJ = t1;
            lK = t2;
        }
    }
    const int chunk = ND_T * per;
    for (long long base = (long long)blockIdx.x * chunk; base < n; base += (long long)nd_blocks * chunk) {
        if (threadIdx.x == 0) s_n = 0;
        __syncthreads();
        // the merge's new-determinant flags, 4 to 32 of a thread in one or two loads
        {
            const int q0 = threadIdx.x * per;
            const long long i0 = base + q0;
            if (i0 + per <= n) {
                uint32_t fw[8] = {0, 0, 0, 0, 0, 0, 0, 0};
                if (per >= 16) {
                    const uint4 f = *(const uint4 *)(w.newdet + i0);
                    fw[0] = f.x, fw[1] = f.y, fw[2] = f.z, fw[3] = f.w;
                    if (per == 32) {
                        const uint4 g = *(const uint4 *)(w.newdet + i0 + 16);
                        fw[4] = g.x, fw[5] = g.y, fw[6] = g.z, fw[7] = g.w;
                    }
                } else {
                    fw[0] = *(const uint32_t *)(w.newdet + i0);
                    if (per == 8) fw[1] = *(const uint32_t *)(w.newdet + i0 + 4);
                }
#pragma unroll
                for (int b = 0; b < 32; ++b)
                    if ((fw[b >> 2] >> (8 * (b & 3))) & 0xFFu) s_q[atomicAdd(&s_n, 1)] = (uint16_t)(q0 + b);
            } else {
                for (int b = 0; b < per && i0 + b < n; ++b)
                    if (w.newdet[i0 + b]) s_q[atomicAdd(&s_n, 1)] = (uint16_t)(q0 + b);
            }
        }
        __syncthreads();
        for (int q = threadIdx.x; q < s_n; q += ND_T) {
            const long long i = base + s_q[q];
            uint64_t key[W];
#pragma unroll
            for (int x = 0; x < W; ++x) key[x] = w.nxt.key[(size_t)x * w.main_cap + i];
            if (local) {
                double e;
                if constexpr (KIND == K_UEG) {
                    bool listed = false;
                    if constexpr (LISTS) {
                        // (an imported determinant may hold other numbers of electrons)
                        int ca = 0, cb = 0;
#pragma unroll
                        for (int x = 0; x < W; ++x) {
                            ca += __popcll(key[x] & 0x5555555555555555ull);
                            cb += __popcll(key[x] & 0xAAAAAAAAAAAAAAAAull);
                        }
                        listed = w.lds_list > 0 && ca == s0.na && cb == s0.nb;
                        if (listed) e = lists(key);
                    }
                    if (!listed) e = diag_ueg<W>(lu, key);
                } else {
                    const int m = s0.n_spatial;
                    e = 0.0;
                    for_bits<W>(key, [&](int P) { e = e + lhd[P >> 1]; });
                    for_pairs<W>(key, [&](int P, int Q) {
                        const int p = P >> 1, q = Q >> 1;
                        const double x = lJ[p * m + q];
                        const double y = ((P & 1) == (Q & 1)) ? lK[p * m + q] : 0.0;
                        e = e + (x - y);
                    });
                }
                w.nxt.kdiag[i] = e - s0.H00;
            } else {
                const int rep = w.rb ? (int)skey_rep(w.nxt.skey[i], w.rb) : 0;
                const DevSys &sy = w.sys[w.rep[rep].sys];
                w.nxt.kdiag[i] = entry_kdiag<KIND, W>(w, sy, key);
            }
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
template <int KIND, int W, int MI>
static void launch_merge(int part, const Work &w, const Grids &g, hipStream_t s)
{
    const int accb = acc_rows(w.R) * EST_FIELDS * 8;
    if (part == 0 && w.R > 1)
        k_merge<KIND, W, true, MI><<<g.merge, MergeCfg<W, MI>::T, accb, s>>>(w);
    else if (part == 0)
        k_merge<KIND, W, false, MI><<<g.merge, MergeCfg<W, MI>::T, accb, s>>>(w);
    else if (w.R > 1)
        k_move<W, true, MI><<<g.move, MV_T, 0, s>>>(w, g.merge);
    else
        k_move<W, false, MI><<<g.move, MV_T, 0, s>>>(w, g.merge);
}

template <int KIND, int W>
static void launch_merge_kind(int part, const Work &w, const Grids &g, hipStream_t s)
{
    if (part == 2) {
        const int ends = w.ccmc_trunc > 0 ? 0 : w.R;  // CCMC ends after its pair sum
        const int per = g.diag_chunk / ND_T, lds = w.lds_diag + w.lds_list + 2 * g.diag_chunk;
        k_new_diag<KIND, W><<<g.newdiag + ends, ND_T, lds, s>>>(w, g.newdiag, per, g.reduce, g.merge);
        return;
    }
    const int mi = W <= 2 ? g.merge_i : 2;
    if (mi == 1)
        launch_merge<KIND, W, W <= 2 ? 1 : 2>(part, w, g, s);
    else if (mi == 4)
        launch_merge<KIND, W, W <= 2 ? 4 : 2>(part, w, g, s);
    else
        launch_merge<KIND, W, 2>(part, w, g, s);
}

hipError_t enqueue_merge(int part, int kind, const Work &w, const Grids &g, hipStream_t s)
{
    FQ_DISPATCH(launch_merge_kind, part, w, g, s)
    return hipGetLastError();
}

int merge_occupancy(bool wide)
{
    int nb = 1;
    const hipError_t e =
        wide ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_merge<K_UEG, 8, false, 2>, MergeCfg<8, 2>::T, 0)
             : hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_merge<K_UEG, 2, false, 4>, MergeCfg<2, 4>::T, 0);
    if (e != hipSuccess) nb = 1;
    return nb < 1 ? 1 : nb;
}

}  // namespace fq
