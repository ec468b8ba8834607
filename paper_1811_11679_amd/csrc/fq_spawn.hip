// Spawning kernels of the FCIQMC iteration (paper Sec. 2.4 "spawning", heat-bath
// sampling Sec. 2.1) for gfx950.
#include "fq_kernels.h"
#include "fq_scan.h"

namespace fq {

// ---------------------------------------------------------------------------
// spawning (Sec. 2.4): one thread per attempt, parents found through the
// attempt prefix (load balanced: a heavily populated determinant spreads its
// attempts over many threads and tiles). A tile of consecutive attempts, SP_I for
// each of its threads, finds its spawn count, reserves that many records with one atomic on the
// spawn counter and writes them contiguously. The records of different tiles
// land in completion order: the radix sort and the segmented sums downstream
// make the result independent of it (equal keys are summed as exact
// integers), and a tile never waits on another.
// ---------------------------------------------------------------------------


__device__ __forceinline__ long long upper_bound_ll(const long long *a, long long lo, long long hi, long long x)
{
    while (lo < hi) {
        const long long mid = (lo + hi) >> 1;
        if (a[mid] <= x) lo = mid + 1; else hi = mid;
    }
    return lo;
}

// Also the iteration's beginning: block 0 advances the counters and clears
// what the iteration accumulates. The other blocks read only the counts of the
// list the last iteration wrote, which it leaves alone.
__global__ __launch_bounds__(256) void k_spawn_partition(Work w, int span_len)
{
    Ctl *c = w.ctl;
    if (c->err) return;
    const long long total = c->n_att_new, n = c->n_main_new;
    const long long nspans = (total + span_len - 1) / span_len;
    if (blockIdx.x == 0) {
        if (threadIdx.x == 0) {
            c->t += 1;
            c->n_main = n;
            c->n_spawn = 0;
            c->n_att = total;
            c->ccmc_n0 = 0;
            c->ccmc_nex = 0;
            c->n_single = 0;
        }
        for (int i = threadIdx.x; i < TK_COUNT; i += blockDim.x) c->tickets[i] = 0;
        for (int i = threadIdx.x; i < w.sort_p * 256; i += blockDim.x) c->hist[7 - (i >> 8)][i & 255] = 0;
        for (int i = threadIdx.x; i < w.R * (int)(sizeof(EstAcc) / 8); i += blockDim.x) ((long long *)w.acc)[i] = 0;
    }
    if (total > w.att_cap) {
        if (blockIdx.x == 0 && threadIdx.x == 0) atomicOr(&c->err, ERR_SPAWN_CAP);
        return;
    }
    for (long long s = (long long)blockIdx.x * blockDim.x + threadIdx.x; s <= nspans;
         s += (long long)gridDim.x * blockDim.x) {
        if (s == nspans) {
            w.span_lo[s] = n > 0 ? n - 1 : 0;
        } else {
            w.span_lo[s] = upper_bound_ll(w.att_off, 0, n + 1, s * span_len) - 1;
        }
    }
}

// MULTI = false: a single replica (rb = 0), so the replica index is 0, its
// parameters are uniform over the grid and a determinant's hash is its sort key.
// LT (single-replica electron gas): the generator's small tables are staged in
// LDS; a compile-time choice, so that their loads are LDS loads.
// SUMS (heat-bath, with LT): the pair weights of a determinant are summed from
// registers (PairSums).
//
// LDS per block: the attempt offsets of the tile's parents and the first
// SP_STAGE spawn records (written out coalesced); records beyond that, rare at
// the spawn rates of the method, go to global memory directly.
constexpr int SP_STAGE = 256;
template <int KIND, int W, bool MULTI, bool LT, int SP_I, bool SUMS = false>
__global__ __launch_bounds__(SP_T) void k_spawn(Work w)
{
    Ctl *c = w.ctl;
    constexpr int SPAN = SP_T * SP_I;
    constexpr int LCAP = SPAN + 2;
    __shared__ long long s_off[LCAP];
    __shared__ uint32_t s_cnt[SP_I][SP_T / 64];
    __shared__ long long s_tile, s_base;
    __shared__ uint32_t s_rrep[MULTI ? SP_STAGE : 1];  // replica of a staged record
    __shared__ uint64_t s_rkey[W][SP_STAGE];
    __shared__ int32_t s_ramp[SP_STAGE];
    __shared__ uint8_t s_rinit[SP_STAGE];
    __shared__ uint32_t s_hist[SORT_P_MAX][256];  // digits of the block's sort keys, for the radix passes
    for (int i = threadIdx.x; i < w.sort_p * 256; i += SP_T) (&s_hist[0][0])[i] = 0;
    const long long total = c->n_att;
    const long long nspans = (total + SPAN - 1) / SPAN;
    const uint32_t t = c->t;
    const bool ss = c->ss_active != 0;
    if (block_stops(c) || total > w.att_cap) return;
    // a plan has up to twice the blocks its tiles need: the others stage no tables
    // (2 electrons in 30 orbitals, 2e5 walkers: 124 us an iteration with, 103 without)
    if (blockIdx.x >= nspans) return;
    const int lane = lane_id(), wid = threadIdx.x >> 6;
    // time-step search: the largest |H_ji| / p_gen of this thread's attempts
    // of replica rs_rep
    const bool ts = w.tau_search != 0;
    double rs_max = 0.0;
    int rs_rep = 0;
    extern __shared__ __align__(16) unsigned char dyn_lds[];
    UegTables lu = w.sys[w.rep[0].sys].u;
    const double *hb_tri = nullptr;  // heat-bath pair weights staged in LDS (LT, molecular)
    if constexpr (LT && KIND == K_MOLECULAR) {
        const DevSys &sy0 = w.sys[w.rep[0].sys];
        const int nso = sy0.n_so, ntri = nso * (nso - 1) / 2;
        double *tt = (double *)dyn_lds;
        for (int x = threadIdx.x; x < ntri; x += SP_T) {
            // x -> (P, Q), P < Q, row by row
            int P = 0, rem = x;
            while (rem >= nso - 1 - P) {
                rem -= nso - 1 - P;
                ++P;
            }
            tt[x] = sy0.hb_S[P * nso + P + 1 + rem];
        }
        if (threadIdx.x == 0) tt[ntri] = 0.0;  // the weight of no pair
        hb_tri = tt;
    }
    if constexpr (LT && KIND == K_UEG) {
        const int M = lu.M, nv = w.sys[w.rep[0].sys].vlen, ng = lu.gdim * lu.gdim * lu.gdim;
        int32_t *tn = (int32_t *)dyn_lds;
        double *tv = (double *)(dyn_lds + ((4 * M + 15) & ~15));
        int16_t *tg = (int16_t *)((unsigned char *)tv + ((8 * nv + 15) & ~15));
        for (int i = threadIdx.x; i < M; i += SP_T) tn[i] = lu.npk[i];
        for (int i = threadIdx.x; i < nv; i += SP_T) tv[i] = lu.vtab[i];
        for (int i = threadIdx.x; i < ng; i += SP_T) tg[i] = lu.grid[i];
        lu.npk = tn;
        lu.vtab = tv;
        lu.grid = tg;
        lu.vx = nullptr;
    }
    for (;;) {
        if (threadIdx.x == 0) s_tile = atomicAdd(&c->tickets[TK_SPAWN], 1u);
        __syncthreads();
        const long long span = s_tile;
        if (span >= nspans) break;
        const long long lo = w.span_lo[span];
        const long long hi = w.span_lo[span + 1];  // parent of the next tile's first attempt
        const long long len = hi - lo + 2;
        const bool staged = len <= LCAP;
        if (staged)
            for (long long i = threadIdx.x; i < len; i += SP_T) s_off[i] = w.att_off[lo + i];
        __syncthreads();
        bool has[SP_I];
        uint64_t child[SP_I][W];
        int32_t amp[SP_I];
        uint8_t init[SP_I];
        uint32_t rep[SP_I];
        // phase 1: the parent of each attempt (blocked: thread t takes attempts
        // SP_I t to SP_I t + SP_I - 1 of the tile; one search finds the first
        // parent, later attempts advance from it), its first attempt and its
        // attempt count
        long long pi[SP_I], pa0[SP_I], pnat[SP_I];
        {
            long long ip = -1;
#pragma unroll
            for (int it = 0; it < SP_I; ++it) {
                pi[it] = -1;
                pa0[it] = 0;
                pnat[it] = 1;
                const long long a = span * SPAN + (long long)threadIdx.x * SP_I + it;
                if (a < total) {
                    long long i;
                    if (staged) {
                        if (ip < 0) {
                            int l = 0, h = (int)len;
                            while (l < h) {
                                const int m = (l + h) >> 1;
                                if (s_off[m] <= a) l = m + 1; else h = m;
                            }
                            ip = lo + l - 1;
                        } else {
                            while (s_off[ip - lo + 1] <= a) ++ip;
                        }
                        i = ip;
                    } else {
                        i = upper_bound_ll(w.att_off, lo, hi + 2, a) - 1;
                    }
                    pi[it] = i;
                    pa0[it] = staged ? s_off[i - lo] : w.att_off[i];
                    pnat[it] = (staged ? s_off[i - lo + 1] : w.att_off[i + 1]) - pa0[it];
                }
            }
        }
        // phase 2 (short keys): every parent load of the thread in flight at once
        constexpr bool PF = W <= 2;
        uint64_t pkey[PF ? SP_I : 1][W];
        int32_t pn0[PF ? SP_I : 1], pdsl[PF ? SP_I : 1];
        uint64_t ppsk[PF ? SP_I : 1];
        if constexpr (PF) {
#pragma unroll
            for (int it = 0; it < SP_I; ++it) {
                const long long i = pi[it] < 0 ? 0 : pi[it];
#pragma unroll
                for (int q = 0; q < W; ++q) pkey[it][q] = w.cur.key[(size_t)q * w.main_cap + i];
                pn0[it] = w.cur.pop[i];
                pdsl[it] = ss ? w.cur.dslot[i] : -1;  // read only with the deterministic space active
                ppsk[it] = stored_skey(MULTI, W) ? w.cur.skey[i] : 0;
            }
        }
        // phase 3: excitation, matrix element, amplitude
#pragma unroll
        for (int it = 0; it < SP_I; ++it) {
            has[it] = false;
            amp[it] = 0;
            init[it] = 0;
            rep[it] = 0;
#pragma unroll
            for (int q = 0; q < W; ++q) child[it][q] = 0;
            if (pi[it] >= 0) {
                const long long i = pi[it];
                const long long nat = pnat[it];
                const long long k = span * SPAN + (long long)threadIdx.x * SP_I + it - pa0[it];
                uint64_t key[W];
                int32_t n0, dsl;
                uint64_t psk;
                if constexpr (PF) {
#pragma unroll
                    for (int q = 0; q < W; ++q) key[q] = pkey[it][q];
                    n0 = pn0[it];
                    dsl = pdsl[it];
                    psk = ppsk[it];
                } else {
#pragma unroll
                    for (int q = 0; q < W; ++q) key[q] = w.cur.key[(size_t)q * w.main_cap + i];
                    n0 = w.cur.pop[i];
                    dsl = ss ? w.cur.dslot[i] : -1;
                    psk = stored_skey(MULTI, W) ? w.cur.skey[i] : 0;
                }
                rep[it] = MULTI ? skey_rep(psk, w.rb) : 0u;
                const RepParams &rp = w.rep[MULTI ? rep[it] : 0u];
                // tables are staged only when all replicas share one system
                const DevSys &sy = w.sys[LT ? w.rep[0].sys : rp.sys];
                const uint64_t h = (!MULTI && W > 2) ? psk : hash64<W>(key);
                const long long an = n0 < 0 ? -(long long)n0 : (long long)n0;
                const bool pin_d = ss && dsl >= 0;
                // the determinant the generator acts on: the entry itself, or for
                // a pair (Sec. 2.3) the bra (even attempts of DMQMC) or the ket
                // (odd attempts of DMQMC; every attempt of IP-DMQMC)
                constexpr int BK = base_kind(KIND), WG = is_pair(KIND) ? W / 2 : W;
                int side = 0;
                long long nat_s = nat;  // attempts per end
                if constexpr (is_pair(KIND)) {
                    side = w.dm == 1 ? (int)(k & 1) : 1;
                    if (w.dm == 1) nat_s = nat >> 1;
                    init[it] = 1;  // no initiator rule on pairs
                } else {
                    init[it] = (uint8_t)(an > rp.thr || key_eq<W>(key, *(const uint64_t(*)[W])sy.ref) || pin_d);
                }
                uint64_t gdet[WG], gchild[WG];
#pragma unroll
                for (int q = 0; q < WG; ++q) {
                    gdet[q] = key[side * WG + q];
                    gchild[q] = 0;
                }
                const U4 r0 = draw(TAG_SELECT, (uint32_t)k, t, h, rp.k0, rp.k1);
                double pgen = 0.0, hv = 0.0;
                bool ok;
                if constexpr (BK == K_HUBBARD)
                    ok = gen_hubbard<WG>(sy, gdet, r0.x, gchild, pgen, hv);
                else if constexpr (BK == K_UEG)
                    ok = gen_ueg<WG>(LT ? lu : sy.u, gdet, r0.x, r0.y, gchild, pgen, hv);
                else
                    ok = gen_heatbath<WG, SUMS>(sy, rp.p_single, gdet, r0, (uint32_t)k, t, h, rp.k0, rp.k1, gchild, pgen,
                                                hv, hb_tri);
#pragma unroll
                for (int q = 0; q < W; ++q) child[it][q] = key[q];
#pragma unroll
                for (int q = 0; q < WG; ++q) child[it][side * WG + q] = gchild[q];
                if (ok && hv != 0.0) {
                    bool skip = false;
                    if constexpr (!is_pair(KIND)) {
                        // CCMC: amplitudes exist only up to the truncation level
                        if (w.ccmc_trunc > 0) {
                            int d = 0;
#pragma unroll
                            for (int q = 0; q < W; ++q) d += __popcll(child[it][q] ^ sy.ref[q]);
                            skip = (d >> 1) > w.ccmc_trunc;
                        }
                    }
                    if (!skip && pin_d) {
                        // discard spawns that stay inside the deterministic space
                        const uint64_t cs = make_skey(hash64<W>(child[it]) & w.hmask, rep[it], w.rb);
                        const int nd = w.ds.n * w.R;
                        int l = 0, hh = nd;
                        while (l < hh) {
                            const int m = (l + hh) >> 1;
                            const uint64_t sk = w.ds.skey_sorted[m];
                            bool less = sk < cs;
                            if (sk == cs) {
                                uint64_t dk[W];
#pragma unroll
                                for (int q = 0; q < W; ++q) dk[q] = w.ds.key_sorted[(size_t)q * nd + m];
                                less = key_cmp<W>(dk, child[it]) < 0;
                            }
                            if (less) l = m + 1; else hh = m;
                        }
                        if (l < nd && w.ds.skey_sorted[l] == cs) {
                            uint64_t dk[W];
#pragma unroll
                            for (int q = 0; q < W; ++q) dk[q] = w.ds.key_sorted[(size_t)q * nd + l];
                            skip = key_eq<W>(dk, child[it]);
                        }
                    }
                    if (!skip) {
                        const double ah = fabs(hv);
                        if (ts) {
                            if (MULTI && (int)rep[it] != rs_rep) {
                                if (rs_max > 0.0) ts_put<false>(w, rs_rep, rs_max);
                                rs_max = 0.0;
                                rs_rep = (int)rep[it];
                            }
                            rs_max = fmax(rs_max, ah / pgen);
                        }
                        // DMQMC: the symmetrised Bloch equation's dbeta / 2 at each end
                        const double tau_s = (is_pair(KIND) && w.dm == 1) ? rp.tau * 0.5 : rp.tau;
                        double m;
                        if (rp.bits == 0)
                            m = (tau_s * ah) / pgen;
                        else if (nat_s == 1)
                            m = ((tau_s * ah) / pgen) * (double)an;  // x / 1.0 is x
                        else
                            m = (((tau_s * ah) / pgen) * (double)an) / (double)nat_s;
                        // the Hubbard and electron-gas generators leave the last two
                        // words of the selection block unused: they give the
                        // rounding uniform; heat-bath uses a block of its own
                        double u;
                        if constexpr (BK == K_MOLECULAR) {
                            const U4 rr = draw(TAG_SPAWN_ROUND, (uint32_t)k, t, h, rp.k0, rp.k1);
                            u = u53(rr.x, rr.y);
                        } else {
                            u = u53(r0.z, r0.w);
                        }
                        long long kk = 0;
                        if (!(m < 0x1p31)) {
                            atomicOr(&c->err, ERR_OVERFLOW);
                        } else {
                            if (rp.bits != 0 && m < (double)rp.cu)
                                kk = (u * (double)rp.cu < m) ? rp.cu : 0;
                            else
                                kk = sround(m, u);
                            if (kk > 2147483647ll) {
                                atomicOr(&c->err, ERR_OVERFLOW);
                                kk = 0;
                            }
                        }
                        if (kk != 0) {
                            const int sh = hv > 0.0 ? 1 : -1;
                            const int sn = n0 > 0 ? 1 : -1;
                            amp[it] = (int32_t)(-(long long)(sh * sn) * kk);
                            has[it] = true;
                        }
                    }
                }
            }
            const uint64_t m = __ballot(has[it]);
            if (lane == 0) s_cnt[it][wid] = (uint32_t)__popcll(m);
        }
        __syncthreads();
        // offsets in attempt order: slab it, wave wid, lane
        uint32_t tot = 0, before[SP_I];
#pragma unroll
        for (int it = 0; it < SP_I; ++it)
#pragma unroll
            for (int q = 0; q < SP_T / 64; ++q) {
                if (q == wid) before[it] = tot;
                tot += s_cnt[it][q];
            }
        // the tile's output range, reserved with one atomic: records land in
        // tile completion order, which the sort and the segmented sums make
        // irrelevant (equal keys are summed as exact integers)
        if (threadIdx.x == 0) s_base = (long long)atomicAdd(&c->n_spawn, (unsigned long long)tot);
        // staged records get their sort key (a hash of the child) in the dense
        // output loop below, not in the divergent per-attempt code
        uint32_t rk[SP_I];
#pragma unroll
        for (int it = 0; it < SP_I; ++it) {
            const uint64_t m = __ballot(has[it]);
            rk[it] = before[it] + (uint32_t)__popcll(m & lanemask_lt());
            if (has[it]) {
                const uint32_t r = rk[it];
                if (r < SP_STAGE) {
                    if constexpr (MULTI) s_rrep[r] = rep[it];
#pragma unroll
                    for (int q = 0; q < W; ++q) s_rkey[q][r] = child[it][q];
                    s_ramp[r] = amp[it];
                    s_rinit[r] = init[it];
                }
            }
        }
        __syncthreads();
        const long long base = s_base;
        if (base + tot > w.spawn_cap) {
            if (threadIdx.x == 0) atomicOr(&c->err, ERR_SPAWN_CAP);
        } else {
            const uint32_t ns = tot < SP_STAGE ? tot : SP_STAGE;
            for (uint32_t p = threadIdx.x; p < ns; p += SP_T) {
                const long long o = base + p;
                uint64_t key[W];
#pragma unroll
                for (int q = 0; q < W; ++q) key[q] = s_rkey[q][p];
                const uint64_t sk = make_skey(hash64<W>(key) & w.hmask, MULTI ? s_rrep[p] : 0u, w.rb);
                w.sp.skey[o] = sk;
                for (int q = 0; q < w.sort_p; ++q) atomicAdd(&s_hist[q][(sk >> (56 - 8 * q)) & 255], 1u);
                uint64_t *rec = w.sp.rec + (size_t)o * (W + 1);
#pragma unroll
                for (int q = 0; q < W; ++q) rec[q] = key[q];
                rec[W] = (uint64_t)(uint32_t)s_ramp[p] | ((uint64_t)s_rinit[p] << 32);
            }
#pragma unroll
            for (int it = 0; it < SP_I; ++it)
                if (has[it] && rk[it] >= SP_STAGE) {
                    const long long o = base + rk[it];
                    const uint64_t sk = make_skey(hash64<W>(child[it]) & w.hmask, rep[it], w.rb);
                    w.sp.skey[o] = sk;
                    for (int q = 0; q < w.sort_p; ++q) atomicAdd(&s_hist[q][(sk >> (56 - 8 * q)) & 255], 1u);
                    uint64_t *rec = w.sp.rec + (size_t)o * (W + 1);
#pragma unroll
                    for (int q = 0; q < W; ++q) rec[q] = child[it][q];
                    rec[W] = (uint64_t)(uint32_t)amp[it] | ((uint64_t)init[it] << 32);
                }
        }
        __syncthreads();
    }
    if (ts) ts_finish<false>(w, rs_max, rs_rep, rs_max > 0.0);
    for (int i = threadIdx.x; i < w.sort_p * 256; i += SP_T) {
        const uint32_t v = (&s_hist[0][0])[i];
        if (v) atomicAdd(&c->hist[7 - (i >> 8)][i & 255], v);
    }
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
// spawning, SI attempts per thread: LDS-staged generator tables when the
// host staged them, the multi-replica kernel for several instances
template <int KIND, int W, int SI>
static void launch_spawn(const Work &w, const Grids &g, hipStream_t s)
{
    constexpr bool TAB = KIND == K_UEG || KIND == K_MOLECULAR, PAIRS = KIND == K_MOLECULAR;
    if (PAIRS && g.pair_sums && w.R > 1)
        k_spawn<KIND, W, true, TAB, SI, PAIRS><<<g.spawn, SP_T, g.spawn_lds, s>>>(w);
    else if (PAIRS && g.pair_sums)
        k_spawn<KIND, W, false, TAB, SI, PAIRS><<<g.spawn, SP_T, g.spawn_lds, s>>>(w);
    else if (w.R > 1 && TAB && w.lds_tables > 0)
        k_spawn<KIND, W, true, TAB, SI><<<g.spawn, SP_T, g.spawn_lds, s>>>(w);
    else if (w.R > 1)
        k_spawn<KIND, W, true, false, SI><<<g.spawn, SP_T, 0, s>>>(w);
    else if (TAB && w.lds_tables > 0)
        k_spawn<KIND, W, false, TAB, SI><<<g.spawn, SP_T, g.spawn_lds, s>>>(w);
    else
        k_spawn<KIND, W, false, false, SI><<<g.spawn, SP_T, 0, s>>>(w);
}

template <int KIND, int W>
static void launch_spawn_kind(int part, const Work &w, const Grids &g, hipStream_t s)
{
    constexpr bool VAR = W <= 2 && !is_pair(KIND);
    const int si = spawn_items(is_pair(KIND), W, g.spawn_i);  // the partition and the spawn must agree on it
    if (part == 0) {
        k_spawn_partition<<<g.part, 256, 0, s>>>(w, SP_T * si);
        return;
    }
    if (si == 2)
        launch_spawn<KIND, W, VAR ? 2 : (W <= 2 ? 4 : 2)>(w, g, s);
    else if (si == 8)
        launch_spawn<KIND, W, VAR ? 8 : (W <= 2 ? 4 : 2)>(w, g, s);
    else
        launch_spawn<KIND, W, W <= 2 ? 4 : 2>(w, g, s);
}

hipError_t enqueue_spawn(int part, int kind, const Work &w, const Grids &g, hipStream_t s)
{
    FQ_DISPATCH(launch_spawn_kind, part, w, g, s)
    return hipGetLastError();
}

int spawn_occupancy()
{
    int nb = 1;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_spawn<K_UEG, 2, false, true, 4>, SP_T, 8192) != hipSuccess) nb = 1;
    return nb < 1 ? 1 : nb;
}

}  // namespace fq
