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
struct LocalAcc {
    long long v[EST_FIELDS];
    int rep;
    __device__ void clear()
    {
#pragma unroll
        for (int i = 0; i < EST_FIELDS; ++i) v[i] = 0;
    }
};

// the thread's values to the block table, lane by lane
__device__ __forceinline__ void acc_spill(LocalAcc &a, long long *tab, int rl, EstAcc *g)
{
    if (a.rep < 0) return;
#pragma unroll
    for (int f = 0; f < EST_FIELDS; ++f)
        if (a.v[f]) acc_add(tab, rl, g, a.rep, f, a.v[f]);
    a.clear();
}

__device__ __forceinline__ void acc_switch(LocalAcc &acc, int rep, long long *tab, int rl, EstAcc *g)
{
    if (rep == acc.rep) return;
    acc_spill(acc, tab, rl, g);
    acc.rep = rep;
}

// end of a kernel (all threads): reduce over the wave when its active lanes
// hold one replica, then store the block's table as partial row blockIdx.x
__device__ void acc_finish(LocalAcc &a, bool active, long long *tab, int rl, EstAcc *g, long long *part)
{
    const uint64_t act = __ballot(active);
    if (act) {
        const int leader = __ffsll((unsigned long long)act) - 1;
        const int rep0 = __shfl(a.rep, leader, 64);
        const bool uniform = __ballot(active && a.rep != rep0) == 0;
        if (uniform) {
#pragma unroll
            for (int f = 0; f < EST_FIELDS; ++f) {
                const long long sv = wave_sum<long long>(active ? a.v[f] : 0);
                if (lane_id() == leader && sv != 0) acc_add(tab, rl, g, rep0, f, sv);
            }
        } else if (active) {
            acc_spill(a, tab, rl, g);
        }
    }
    a.clear();
    __syncthreads();
    // partials are laid out [replica][field][block] so that the fold reads
    // each (replica, field) as one contiguous run
    for (int i = threadIdx.x; i < rl * EST_FIELDS; i += blockDim.x) part[(size_t)i * PART_MAX_BLOCKS + blockIdx.x] = tab[i];
}

// ---------------------------------------------------------------------------
// annihilation merge (Sec. 2.4; appendix "Parallelization"): merge-path merge
// of the distinct spawned determinants into the sorted main list, fused with
// death/cloning of existing entries, the deterministic-space update, the
// initiator rule for new determinants (Sec. 2.1), removal of empty entries,
// the estimators of the new list (tutorial appendix) and the attempt counts of
// the next iteration. Ties in the merge order put the main entry first.
//
// A tile's slices of both lists are staged in LDS with coalesced loads (main
// entries in slots [0, la), spawned ones in [la, la + lb)); every thread
// merges its run of positions from LDS, writes each result into the source
// slot, and the kept entries leave in merge order with coalesced stores.
// ---------------------------------------------------------------------------
// Keys of up to two words: 512 threads of two positions each, whose tile's
// dependent phases (ticket, partition, staging, look-back) are shorter than
// with 256 threads of four; two such blocks fit a compute unit's registers
// and LDS. Longer keys: 256 threads of two positions (their LDS slice is
// larger, and three such blocks per compute unit measured faster).
// MI: merge positions per thread and tile, 1, 2 or 4 for keys of up to two
// words (chosen per context), 2 for longer keys
template <int W, int MI>
struct MergeCfg {
    static constexpr int T = W <= 2 ? 512 : 256;
    static constexpr int I = MI;
    static constexpr int TILE = T * I;
};
static_assert(MergeCfg<1, 1>::TILE == 512 && MergeCfg<8, 2>::TILE == 512,
              "the merge partition and status arrays are sized for 512-position tiles");

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

template <int W, int MI>
__global__ void k_merge_partition(Work w)
{
    const Ctl *c = w.ctl;
    if (c->err) return;
    constexpr int TILE = MergeCfg<W, MI>::TILE;
    const long long na = c->n_main, nb = (long long)min(c->n_spawn, (unsigned long long)w.spawn_cap);
    const long long ntiles = (na + nb + TILE - 1) / TILE;
    for (long long tile = (long long)blockIdx.x * blockDim.x + threadIdx.x; tile <= ntiles;
         tile += (long long)gridDim.x * blockDim.x) {
        const long long d = min(tile * TILE, na + nb);
        long long lo = max(0ll, d - nb), hi = min(d, na);
        while (lo < hi) {
            const long long mid = (lo + hi) >> 1;
            const long long j = d - 1 - mid;
            if (le_ab<W>(w, mid, main_skey<W>(w, mid), j, w.u.skey[j])) lo = mid + 1; else hi = mid;
        }
        w.mpart[tile] = lo;
    }
}


__device__ __forceinline__ void add_limbs(long long (&v)[EST_FIELDS], double x)
{
    add_limbs4(v[F_L0], v[F_L1], v[F_L2], v[F_L3], x);
}

// spawning attempts of an entry holding p units: |p| for integer walkers,
// ceil(|p| 2^-b) for fixed point, times mult (2 for DMQMC pairs: that many
// at each end); 2^28 or more does not fit the counter's attempt field
__device__ __forceinline__ long long attempts_of(long long p, int bits, int mult, Ctl *c)
{
    const long long ap = p < 0 ? -p : p;
    const long long n = mult * (bits == 0 ? ap : (ap + (1ll << bits) - 1) >> bits);
    if (n >= (1ll << 28)) atomicOr(&c->err, ERR_ATTEMPTS);
    return n;
}

template <int KIND, int W, bool MULTI, int MI>
__global__ __launch_bounds__((MergeCfg<W, MI>::T)) void k_merge(Work w)
{
    Ctl *c = w.ctl;
    if (c->err) return;
    constexpr int MG_T = MergeCfg<W, MI>::T, TILE = MergeCfg<W, MI>::TILE;
    __shared__ uint64_t s_sk[TILE];
    __shared__ uint64_t s_key[W][TILE];
    __shared__ long long s_val[TILE];   // main: population, then the new one; spawned: sum
    __shared__ double s_kd[TILE];       // K_ii - H_00
    __shared__ int32_t s_meta[TILE];    // main: dslot; spawned: initiator flag, then dslot (-1)
    __shared__ uint16_t s_src[TILE];    // merge position -> slot
    __shared__ uint16_t s_dst[TILE];    // merge position -> rank among kept
    __shared__ uint8_t s_keep[TILE];
    __shared__ uint64_t s_pa_sk, s_pa_key[W];  // main entry before the tile
    __shared__ uint64_t s_nb_sk, s_nb_key[W];  // spawned entry after the tile
    __shared__ long long s_nb_sum;
    __shared__ int s_pa_ok, s_nb_ok;
    __shared__ long long s_tile, s_base, s_abase;
    __shared__ long long s_red[16];
    const long long na = c->n_main, nb = (long long)min(c->n_spawn, (unsigned long long)w.spawn_cap);
    const long long ntiles = (na + nb + TILE - 1) / TILE;
    const uint32_t t = c->t;
    const uint32_t epoch = epoch_of(t, 11), epoch_att = epoch_of(t, 13);
    const bool ss = c->ss_active != 0;
    extern __shared__ __align__(16) unsigned char dyn_lds[];
    long long *tab = (long long *)dyn_lds;  // estimator table, acc_rows(R) rows
    const int rl = acc_rows(w.R);
    acc_table_clear(tab, rl);
    LocalAcc acc;
    acc.clear();
    acc.rep = -1;
    bool any = false;
    // time-step search: the largest K_ii of the entries this thread's death steps act on
    const bool ts = w.tau_search != 0;
    double kd_max = -INFINITY;
    int kd_rep = 0;
    for (;;) {
        if (threadIdx.x == 0) s_tile = atomicAdd(&c->tickets[TK_MERGE], 1u);
        __syncthreads();
        const long long tile = s_tile;
        if (tile >= ntiles) break;
        const long long d0 = tile * TILE, d1 = min(d0 + TILE, na + nb);
        const long long i0 = w.mpart[tile], i1 = w.mpart[tile + 1];
        const long long j0 = d0 - i0, j1 = d1 - i1;
        const int la = (int)(i1 - i0), lb = (int)(j1 - j0);
        for (int q = threadIdx.x; q < la; q += MG_T) {
            const long long g = i0 + q;
            uint64_t k[W];
#pragma unroll
            for (int x = 0; x < W; ++x) {
                k[x] = w.cur.key[(size_t)x * w.main_cap + g];
                s_key[x][q] = k[x];
            }
            s_sk[q] = stored_skey(MULTI, W) ? w.cur.skey[g] : hash64<W>(k);
            s_val[q] = w.cur.pop[g];
            s_kd[q] = w.cur.kdiag[g];
            s_meta[q] = ss ? w.cur.dslot[g] : -1;
        }
        for (int q = threadIdx.x; q < lb; q += MG_T) {
            const long long g = j0 + q;
            s_sk[la + q] = w.u.skey[g];
#pragma unroll
            for (int x = 0; x < W; ++x) s_key[x][la + q] = w.u.key[(size_t)x * w.spawn_cap + g];
            s_val[la + q] = w.u.sum[g];
            s_meta[la + q] = (int32_t)w.u.flag[g];
        }
        if (threadIdx.x == 0) {
            s_pa_ok = i0 > 0;
            if (i0 > 0) {
#pragma unroll
                for (int x = 0; x < W; ++x) s_pa_key[x] = w.cur.key[(size_t)x * w.main_cap + i0 - 1];
                s_pa_sk = stored_skey(MULTI, W) ? w.cur.skey[i0 - 1] : hash64<W>(s_pa_key);
            }
            s_nb_ok = j1 < nb;
            if (j1 < nb) {
                s_nb_sk = w.u.skey[j1];
#pragma unroll
                for (int x = 0; x < W; ++x) s_nb_key[x] = w.u.key[(size_t)x * w.spawn_cap + j1];
                s_nb_sum = w.u.sum[j1];
            }
        }
        __syncthreads();
        auto le = [&](int a, int b) -> bool {  // A slot a <= B slot la + b
            const uint64_t sa = s_sk[a], sb = s_sk[la + b];
            if (sa != sb) return sa < sb;
            int r = 0;
#pragma unroll
            for (int x = W - 1; x >= 0; --x)
                if (r == 0) r = s_key[x][a] < s_key[x][la + b] ? -1 : (s_key[x][a] > s_key[x][la + b] ? 1 : 0);
            return r <= 0;
        };
        auto eq_slots = [&](int p, int q) -> bool {
            bool e = s_sk[p] == s_sk[q];
#pragma unroll
            for (int x = 0; x < W; ++x) e = e && s_key[x][p] == s_key[x][q];
            return e;
        };
        const int dl = min((int)threadIdx.x * MI, la + lb);
        int lo = max(0, dl - lb), hi = min(dl, la);
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (le(mid, dl - 1 - mid)) lo = mid + 1; else hi = mid;
        }
        int ia = lo, jb = dl - lo;
        const int steps = min(MI, la + lb - dl);
        for (int st = 0; st < steps; ++st) {
            const int m = dl + st;
            bool takeA;
            if (ia >= la) takeA = false;
            else if (jb >= lb) takeA = true;
            else takeA = le(ia, jb);
            if (takeA) {
                const int a = ia++;
                const uint64_t sk = s_sk[a];
                const int32_t n0 = (int32_t)s_val[a];
                const int32_t dsl = s_meta[a];
                const int rep = MULTI ? (int)skey_rep(sk, w.rb) : 0;
                acc_switch(acc, rep, tab, rl, w.acc);
                any = true;
                // matching spawned determinant: the next unconsumed one
                long long add = 0;
                if (jb < lb) {
                    if (eq_slots(a, la + jb)) add = s_val[la + jb];
                } else if (s_nb_ok && s_nb_sk == sk) {
                    bool e = true;
#pragma unroll
                    for (int x = 0; x < W; ++x) e = e && s_nb_key[x] == s_key[x][a];
                    if (e) add = s_nb_sum;
                }
                long long v;
                if (ss && dsl >= 0) {
                    v = (long long)n0 + w.ds.delta[(size_t)rep * w.ds.n + dsl];
                } else if (n0 != 0) {
                    const RepParams &rp = w.rep[rep];
                    if (ts) {
                        if (MULTI && rep != kd_rep) {
                            if (kd_max > -INFINITY) ts_put<true>(w, kd_rep, kd_max);
                            kd_max = -INFINITY;
                            kd_rep = rep;
                        }
                        kd_max = fmax(kd_max, s_kd[a]);
                    }
                    const double an = (double)(n0 < 0 ? -(long long)n0 : (long long)n0);
                    const double mm = (rp.tau * (s_kd[a] - w.shift[rep])) * an;
                    uint64_t h = sk;
                    if constexpr (MULTI) {
                        uint64_t key[W];
#pragma unroll
                        for (int x = 0; x < W; ++x) key[x] = s_key[x][a];
                        h = hash64<W>(key);
                    }
                    const U4 r = draw(TAG_DEATH, 0, t, h, rp.k0, rp.k1);
                    const double u = u53(r.x, r.y);
                    if (!(fabs(mm) < 0x1p40)) atomicOr(&c->err, ERR_OVERFLOW);
                    const long long k = mm >= 0.0 ? sround(mm, u) : -sround(-mm, u);
                    const long long sg = n0 > 0 ? 1 : -1;
                    v = (long long)n0 - sg * k;
                    if ((v > 0 && n0 < 0) || (v < 0 && n0 > 0)) acc.v[F_FLIPS] += 1;
                } else {
                    v = 0;
                }
                acc.v[F_DEATH] += v;
                v += add;
                if (v > 2147483647ll || v < -2147483647ll) atomicOr(&c->err, ERR_OVERFLOW);
                s_val[a] = v;
                s_src[m] = (uint16_t)a;
                s_keep[m] = (v != 0 || dsl >= 0) ? 1 : 0;
            } else {
                const int b = jb++;
                const int slot = la + b;
                // matched with the preceding main entry: that entry's thread added it
                bool matched;
                if (ia > 0) {
                    matched = eq_slots(ia - 1, slot);
                } else {
                    matched = s_pa_ok && s_pa_sk == s_sk[slot];
#pragma unroll
                    for (int x = 0; x < W; ++x) matched = matched && s_pa_key[x] == s_key[x][slot];
                }
                s_src[m] = (uint16_t)slot;
                s_keep[m] = 0;
                if (!matched && !(s_meta[slot] & (int32_t)UNIQ_FILLER)) {
                    const long long sum = s_val[slot];
                    const int32_t fl = s_meta[slot];
                    const int rep = MULTI ? (int)skey_rep(s_sk[slot], w.rb) : 0;
                    const RepParams &rp = w.rep[rep];
                    acc_switch(acc, rep, tab, rl, w.acc);
                    any = true;
                    const bool accept = (!rp.initiator || fl) && sum != 0;
                    if (accept) {
                        if (sum > 2147483647ll || sum < -2147483647ll) atomicOr(&c->err, ERR_OVERFLOW);
                        // K_jj - H_00 is filled in by k_new_diag (off the merge's critical path)
                        s_kd[slot] = __longlong_as_double(0x7FF8000000000000ll);
                        s_meta[slot] = -1;
                        s_keep[m] = 1;
                    } else {
                        acc.v[F_REJU] += sum < 0 ? -sum : sum;
                        acc.v[F_REJ] += sum;
                    }
                }
            }
        }
        // ranks of the kept entries in merge order, and their spawning attempts
        // for the next iteration (the attempt prefix replaces a separate scan)
        int cnt = 0;
        long long asum = 0;
        for (int st = 0; st < steps; ++st) {
            const int m = dl + st;
            if (!s_keep[m]) continue;
            ++cnt;
            const int slot = s_src[m];
            const int rep = MULTI ? (int)skey_rep(s_sk[slot], w.rb) : 0;
            asum += attempts_of(s_val[slot], w.rep[rep].bits, w.dm == 1 ? 2 : 1, c);
        }
        long long tot, atot, ex, aex;
        block_excl_scan2((long long)cnt, asum, ex, aex, tot, atot, s_red);
        if (threadIdx.x < 64) {
            const long long lb_ = lookback(w.st_merge, tile, epoch, tot);
            if (threadIdx.x == 0) s_base = lb_;
        } else if (threadIdx.x < 128) {
            const long long lb_ = lookback(w.st_att, tile, epoch_att, atot);
            if (threadIdx.x == 64) s_abase = lb_;
        }
        {
            int r = (int)ex;
            for (int st = 0; st < steps; ++st)
                if (s_keep[dl + st]) s_dst[dl + st] = (uint16_t)r++;
        }
        __syncthreads();
        if (s_base + tot <= w.main_cap) {
            long long ar = s_abase + aex;
            for (int st = 0; st < steps; ++st) {
                const int m = dl + st;
                if (!s_keep[m]) continue;
                const int slot = s_src[m];
                const int rep = MULTI ? (int)skey_rep(s_sk[slot], w.rb) : 0;
                w.att_off[s_base + s_dst[m]] = ar;
                ar += attempts_of(s_val[slot], w.rep[rep].bits, w.dm == 1 ? 2 : 1, c);
            }
        }
        const long long obase = s_base;
        if (obase + tot > w.main_cap) {
            if (threadIdx.x == 0) atomicOr(&c->err, ERR_MAIN_CAP);
        } else {
            for (int m = threadIdx.x; m < la + lb; m += MG_T) {
                if (!s_keep[m]) continue;
                const long long o = obase + s_dst[m];
                const int slot = s_src[m];
                const uint64_t sk = s_sk[slot];
                const int rep = MULTI ? (int)skey_rep(sk, w.rb) : 0;
                const RepParams &rp = w.rep[rep];
                const DevSys &sy = w.sys[rp.sys];
                const int32_t p = (int32_t)s_val[slot];
                const int32_t ds = s_meta[slot];
                if (stored_skey(MULTI, W)) w.nxt.skey[o] = sk;
                uint64_t key[W];
#pragma unroll
                for (int x = 0; x < W; ++x) {
                    key[x] = s_key[x][slot];
                    w.nxt.key[(size_t)x * w.main_cap + o] = key[x];
                }
                w.nxt.pop[o] = p;
                w.nxt.kdiag[o] = s_kd[slot];
                w.newdet[o] = slot >= la ? 1 : 0;
                if (ss) w.nxt.dslot[o] = ds;
                if (ds >= 0) w.ds.pos[(size_t)rep * w.ds.n + ds] = (int32_t)o;
                const long long ap = p < 0 ? -(long long)p : (long long)p;
                acc_switch(acc, rep, tab, rl, w.acc);
                any = true;
                acc.v[F_NW] += ap;
                acc.v[F_NOCC] += 1;
                if constexpr (is_pair(KIND)) {
                    // density matrix (Sec. 2.3): the trace sum_i rho_ii and
                    // Tr(rho H) = sum rho_ij H_ji over pairs at most doubly excited
                    constexpr int BK = base_kind(KIND), WH = W / 2;
                    uint64_t a[WH], b[WH];
                    int nd = 0;
#pragma unroll
                    for (int x = 0; x < WH; ++x) {
                        a[x] = key[x];
                        b[x] = key[WH + x];
                        nd += __popcll(a[x] ^ b[x]);
                    }
                    if (nd == 0) {
                        acc.v[F_N0] += p;
                        add_limbs(acc.v, diag_element<BK, WH>(sy, a) * (double)p);
                    } else if (nd == 2 || nd == 4) {
                        add_limbs(acc.v, hij<BK, WH>(sy, b, a) * (double)p);
                    }
                } else {
                    const uint64_t(&ref)[W] = *(const uint64_t(*)[W])sy.ref;
                    int nd = 0;
#pragma unroll
                    for (int x = 0; x < W; ++x) nd += __popcll(key[x] ^ ref[x]);
                    if (nd == 0) {
                        acc.v[F_N0] += p;
                    } else if (nd == 2 || nd == 4) {
                        const double hv = hij<KIND, W>(sy, ref, key);
                        add_limbs(acc.v, hv * (double)p);
                    }
                }
            }
        }
        if (tile == ntiles - 1 && threadIdx.x == 0) {
            c->n_main_new = obase + tot;
            if (obase + tot <= w.main_cap) w.att_off[obase + tot] = s_abase + atot;
            c->n_att_new = s_abase + atot;
        }
        __syncthreads();
    }
    acc_finish(acc, any && acc.rep >= 0, tab, rl, w.acc, w.part_mrg);
    if (ts) ts_finish<true>(w, kd_max, kd_rep, kd_max > -INFINITY);
    if (blockIdx.x == 0 && threadIdx.x == 0 && ntiles == 0) {
        c->n_main_new = 0;
        w.att_off[0] = 0;
        c->n_att_new = 0;
    }
}

// K_jj - H_00 of the determinants the merge has just created (marked NaN).
// Each block scans a chunk of the new list, queues the marked entries in LDS
// and evaluates them one per thread, so no lane idles on unmarked entries;
// for a single replica the diagonal's tables are read from LDS.
// Chunks of 16384 flags: new determinants are a few per cent of the list, and
// a chunk must hold enough of them to fill the block's waves (at 4096 flags a
// 256-thread block had about one partial wave of work per chunk)
constexpr int ND_T = 512, ND_CHUNK = 16384;
static_assert(ND_CHUNK == ND_T * 32, "each thread scans 32 new-determinant flags");

template <int KIND, int W>
__global__ __launch_bounds__(ND_T) void k_new_diag(Work w)
{
    const Ctl *c = w.ctl;
    if (c->err) return;
    extern __shared__ __align__(16) unsigned char dyn_lds[];
    __shared__ uint16_t s_q[ND_CHUNK];  // offsets of the chunk's new determinants
    __shared__ int s_n;
    const long long n = c->n_main_new;
    const DevSys &s0 = w.sys[w.rep[0].sys];
    // the host stages tables only when every replica has the same system
    const bool local = w.lds_diag > 0 && (KIND == K_UEG || KIND == K_MOLECULAR);
    UegTables lu = s0.u;
    const double *lhd = s0.hd, *lJ = s0.Jt, *lK = s0.Kt;
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
    for (long long base = (long long)blockIdx.x * ND_CHUNK; base < n; base += (long long)gridDim.x * ND_CHUNK) {
        if (threadIdx.x == 0) s_n = 0;
        __syncthreads();
        // the merge's new-determinant flags, 32 per thread in two 16-byte loads
        {
            const int q0 = threadIdx.x * 32;
            const long long i0 = base + q0;
            if (i0 + 32 <= n) {
                const uint4 f0 = *(const uint4 *)(w.newdet + i0);
                const uint4 f1 = *(const uint4 *)(w.newdet + i0 + 16);
                const uint32_t fw[8] = {f0.x, f0.y, f0.z, f0.w, f1.x, f1.y, f1.z, f1.w};
#pragma unroll
                for (int b = 0; b < 32; ++b)
                    if ((fw[b >> 2] >> (8 * (b & 3))) & 0xFFu) s_q[atomicAdd(&s_n, 1)] = (uint16_t)(q0 + b);
            } else {
                for (int b = 0; b < 32 && i0 + b < n; ++b)
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
                    e = diag_ueg<W>(lu, key);
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
    if (part == 0)
        k_merge_partition<W, MI><<<g.part, 256, 0, s>>>(w);
    else if (w.R > 1)
        k_merge<KIND, W, true, MI><<<g.merge, MergeCfg<W, MI>::T, accb, s>>>(w);
    else
        k_merge<KIND, W, false, MI><<<g.merge, MergeCfg<W, MI>::T, accb, s>>>(w);
}

template <int KIND, int W>
static void launch_merge_kind(int part, const Work &w, const Grids &g, hipStream_t s)
{
    if (part == 2) {
        k_new_diag<KIND, W><<<g.newdiag, ND_T, w.lds_diag, s>>>(w);
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
             : hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_merge<K_UEG, 2, false, 2>, MergeCfg<2, 2>::T, 0);
    if (e != hipSuccess) nb = 1;
    return nb < 1 ? 1 : nb;
}

}  // namespace fq
