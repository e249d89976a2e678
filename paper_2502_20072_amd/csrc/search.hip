// Exhaustive l0 search on gfx950: every D-tuple of the S features is scored
// by the SSE of its least-squares fit (intercept per task), and the k best
// by (SSE, lexicographic rank) are kept.
//
// The paper factorises each tuple's n x (D+1) descriptor matrix with
// Householder QR, one GPU thread per tuple.  Here the fits come from the
// correlation matrices G_t, b_t, c_t that the Gram step precomputed: for a
// tuple T = (P, k) with prefix P,
//     w = R_P^{-1} G[P,k],  d = 1 - |w|^2,  zeta = b_k - w.z_P,
//     SSE_t(T) = p_P - zeta^2 / d       (p_P = c_t - |z_P|^2 = SSE_t(P)),
// with R_P the Cholesky factor of G[P,P] and z_P = R_P^{-1} b_P.  d is the
// pivot of k (1 - R^2 of x_k on the intercept and P), which is also the
// rank test.  For a single task the comparison SSE <= theta needs no
// division: zeta^2 >= (p_P - theta) d.
//
// D = 2 with one task, D = 3 and D = 4 with one task run kernels of their own
// (search2_kernel; search3_kernel and search4_kernel, which bound several
// tuples by the fit on a superset); search_kernel serves the rest.
//
// Work decomposition of search_kernel.  A tuple is (P', j, k): a sub-prefix P' of D-2
// indices, the (D-1)-th index j and the last index k.  A work item is a
// block of 64 consecutive j values together with a group of sub-prefixes
// (SUBP of them for one task, one when lanes are split over tasks).  The
// workgroup builds the Cholesky row of every (P', j) pair of the item in
// parallel (one thread each) into LDS; then each wave sweeps chunks of 64
// consecutive k (one per lane), keeps the k-dependent part of the
// sub-prefix solve in registers, and for every j loads one G[j][k] that
// serves all sub-prefixes of the item.  Items are dealt round-robin in order
// of increasing j, i.e. largest first; sub-prefix
// groups are addressed by colexicographic rank (combinatorial number
// system), so item -> (j-block, sub-prefixes) is a bisection, not a table.
//
// Top-k.  Each wave keeps a sorted list of the KP best (SSE, rank) pairs in
// LDS; insertions happen only for tuples that pass the current bound, which
// is the minimum of a pre-pass bound theta0 (see pre_*), the wave's own
// KP-th entry and a device-wide bound that full lists publish with an
// atomic min.  Any list's KP-th entry bounds the global KP-th best, so the
// filter never drops a tuple of the global top-KP.  A merge kernel gathers
// the entries under the final bound, and every survivor is re-scored from F
// itself (explicit residuals in FP64), which fixes the reported SSE to the
// accuracy of a direct least-squares fit, before the final ordering.
#include <math.h>

#include <type_traits>

#include "common.h"
#include "kernels.h"

namespace sl0 {

constexpr int MAXD = SISSO_MAX_D;
constexpr double INF = __builtin_huge_val();
constexpr double THETA_SLACK = 1e-9;  // relative slack of the filter bound
constexpr double THETA_SLACK_F32 = 1e-5;  // FP32 solve form: absolute slack, in units of sum_t c_t
constexpr int SEARCH_JG = 8;  // G rows per prefetch group (two groups in flight)

__device__ inline bool key_less(double s1, uint64_t r1, double s2, uint64_t r2) {
    return s1 < s2 || (s1 == s2 && r1 < r2);
}

__device__ inline double theta_load(const unsigned long long *p) {
    unsigned long long b = __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return __longlong_as_double((long long)b);
}

__device__ inline void theta_publish(unsigned long long *p, double v) {
    // non-negative doubles order like their bit patterns
    if (v >= 0.0 && v < INF) atomicMin(p, (unsigned long long)__double_as_longlong(v));
}

// Values every lane holds identically (read from LDS or a uniform address)
// are moved to scalar registers, so address arithmetic on them stays scalar.
__device__ inline int64_t uni(int64_t v) {
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)(uint64_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)((uint64_t)v >> 32));
    return (int64_t)(((uint64_t)hi << 32) | lo);
}
__device__ inline uint64_t uni(uint64_t v) { return (uint64_t)uni((int64_t)v); }
__device__ inline double uni(double v) { return __longlong_as_double(uni((int64_t)__double_as_longlong(v))); }

// Lane permutation inside rows of 16 lanes (DPP), for both halves of a double.
template <int CTRL>
__device__ inline double dpp_f64(double v) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)b, CTRL, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xF, 0xF, true);
    return __longlong_as_double((long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo));
}

// the same lane permutation for the FP32 form's sums
template <int CTRL>
__device__ inline float dpp_r(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, true));
}
template <int CTRL>
__device__ inline double dpp_r(double v) { return dpp_f64<CTRL>(v); }
__device__ inline float rcp_r(float d) {
    const float r = __builtin_amdgcn_rcpf(d);
    return fmaf(r, fmaf(-d, r, 1.0f), r);
}
__device__ inline double rcp_r(double d) {
    const double r = __builtin_amdgcn_rcp(d);
    return fma(r, fma(-d, r, 1.0), r);
}
// pivot ratio at or below which the solve of type R calls a tuple rank
// deficient: FP32 resolves 1 - |w|^2 only to a few units of 2^-23
template <typename R>
__device__ constexpr R rank_eps_r() { return sizeof(R) == 8 ? (R)RANK_EPS : (R)RANK_EPS_F32; }

__device__ inline int next_pow2_dev(int x) {
    int p = 1;
    while (p < x) p <<= 1;
    return p;
}

__device__ inline double Gat(const Ctx &c, int64_t i, int64_t k, int t) {
    return c.G[gidx(i, k, c.Gnt, c.TP, t)];
}

// ----------------------------------------------------------------- helpers
// Normal-equation SSE of one sorted tuple summed over tasks, from the
// correlation matrices (Cholesky in increasing index order).  +inf when a
// pivot is <= RANK_EPS in some task.  Used by the threshold pre-pass.  All
// entries a task needs are loaded before any arithmetic, so the loads of one
// call overlap instead of forming a chain.
// SSE of one task from its tuple's correlation block g (lower triangle,
// sorted-index order), b and c = |y_c|^2; clears ok on a pivot <= RANK_EPS.
template <int D>
__device__ inline double ne_sse_core(const double (&g)[D][D], const double (&bv)[D], double cyy, bool &ok) {
    double L[D][D], z[D];
    double p = cyy;
#pragma unroll
    for (int m = 0; m < D; ++m) {
#pragma unroll
        for (int j = 0; j < m; ++j) {
            double s = g[m][j];
#pragma unroll
            for (int l = 0; l < j; ++l) s -= L[m][l] * L[j][l];
            L[m][j] = s / L[j][j];
        }
        double d = g[m][m];
#pragma unroll
        for (int l = 0; l < m; ++l) d -= L[m][l] * L[m][l];
        ok &= d > RANK_EPS;
        L[m][m] = sqrt(fmax(d, RANK_EPS));
        double zm = bv[m];
#pragma unroll
        for (int l = 0; l < m; ++l) zm -= L[m][l] * z[l];
        z[m] = zm / L[m][m];
        p -= z[m] * z[m];
    }
    return p;
}

template <int D>
__device__ double ne_sse_t(const Ctx &c, const int32_t *tup) {
    double total = 0.0;
    bool ok = true;
    for (int t = 0; t < c.T; ++t) {
        double g[D][D], bv[D];
#pragma unroll
        for (int m = 0; m < D; ++m) {
#pragma unroll
            for (int j = 0; j <= m; ++j) g[m][j] = Gat(c, tup[m], tup[j], t);
            bv[m] = c.bhat[(int64_t)tup[m] * c.TP + t];
        }
        total += ne_sse_core<D>(g, bv, c.cyy[t], ok);
    }
    return ok ? total : INF;
}

__device__ double ne_sse(const Ctx &c, int D, const int32_t *tup) {
    switch (D) {
        case 1: return ne_sse_t<1>(c, tup);
        case 2: return ne_sse_t<2>(c, tup);
        case 3: return ne_sse_t<3>(c, tup);
        default: return ne_sse_t<4>(c, tup);
    }
}

// Sorted per-wave list in LDS: entries e = lane + 64 m, m < KP/64.
// A wave's sorted list is written to global memory only up to its first
// empty (+inf) entry, which is written too as a terminator: readers stop
// there, so the (usually empty) tail of KP entries costs no traffic.
__device__ inline void list_store(double *__restrict__ ds, uint64_t *__restrict__ dr, const double *Ls,
                                  const uint64_t *Lr, int KP) {
    const int lane = threadIdx.x & 63;
    int nv = 0;
    for (int m = 0; m < KP; m += 64) nv += __popcll(__ballot(Ls[m + lane] < INF));
    for (int m = lane; m < KP && m <= nv; m += 64) {
        ds[m] = Ls[m];
        dr[m] = Lr[m];
    }
}

// Reads a list written by list_store into LDS (entries past the terminator
// are +inf).
__device__ inline void list_load(double *Ls, uint64_t *Lr, const double *__restrict__ ss,
                                 const uint64_t *__restrict__ sr, int KP) {
    const int lane = threadIdx.x & 63;
    bool end = false;
    for (int m = 0; m < KP; m += 64) {
        // the live entries are the prefix before the terminator; what lies
        // after it in the same chunk is stale and is not read as an entry
        const double v = end ? INF : ss[m + lane];
        const unsigned long long b = __ballot(v < INF);
        const int nlive = end ? 0 : (b == ~0ull ? 64 : __builtin_ctzll(~b));
        const bool live = lane < nlive;
        Ls[m + lane] = live ? v : INF;
        Lr[m + lane] = live ? sr[m + lane] : ~0ull;
        end = end || nlive < 64;
    }
}

__device__ void list_insert(double *Ls, uint64_t *Lr, int KP, double s, uint64_t r) {
    const int lane = threadIdx.x & 63;
    const int nper = KP >> 6;
    int pos = 0;
    for (int m = 0; m < nper; ++m) {
        const int e = lane + 64 * m;
        pos += __popcll(__ballot(key_less(Ls[e], Lr[e], s, r)));
    }
    if (pos >= KP) return;
    if (Ls[pos] == s && Lr[pos] == r) return;  // the same tuple, offered twice (list search)
    // shift the entries above pos up by one, highest chunk of 64 first: a
    // chunk is read whole before it is written, and its lowest lane reads the
    // top entry of the chunk below before that chunk is written (few live
    // registers, whatever the list length)
    for (int m = nper - 1; m >= 0 && 64 * m + 63 > pos; --m) {
        const int e = lane + 64 * m;
        const bool mv = e > pos;
        double vs = 0.0;
        uint64_t vr = 0;
        if (mv) {
            vs = Ls[e - 1];
            vr = Lr[e - 1];
        }
        __atomic_signal_fence(__ATOMIC_SEQ_CST);
        __builtin_amdgcn_wave_barrier();
        if (mv) {
            Ls[e] = vs;
            Lr[e] = vr;
        }
        __atomic_signal_fence(__ATOMIC_SEQ_CST);
        __builtin_amdgcn_wave_barrier();
    }
    if (lane == 0) {
        Ls[pos] = s;
        Lr[pos] = r;
    }
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    __builtin_amdgcn_wave_barrier();
}

// Inserts the entries of the lanes in take (distinct keys, none in the list)
// into the wave's list; offered counts them.  One by one an insertion costs
// a pass over the list; from LIST_BULK on all are merged in one: an entry's
// new place is its rank among the new ones plus the number of old ones before
// it, and an old one moves up by the number of new ones before it (64 entries
// into 128: about 3 us against 45).
constexpr int LIST_BULK = 4;
__device__ void list_insert_lanes(double *Ls, uint64_t *Lr, int KP, bool take, uint64_t key, double sse,
                                  unsigned &offered) {
    const int lane = threadIdx.x & 63;
    unsigned long long m = __ballot(take);
    const int n = __popcll(m);
    if (!n) return;
    offered += (unsigned)n;
    if (n < LIST_BULK) {
        while (m) {
            const int src = __ffsll((long long)m) - 1;
            m &= m - 1;
            list_insert(Ls, Lr, KP, __shfl(sse, src), (uint64_t)__shfl((long long)key, src));
        }
        return;
    }
    // new entries of the lanes in m before (s, r)
    auto before = [&](double s, uint64_t r) {
        int c = 0;
        for (unsigned long long q = m; q; q &= q - 1) {
            const int src = __ffsll((long long)q) - 1;
            const double bs = uni(__shfl(sse, src));
            const uint64_t br = uni((uint64_t)__shfl((long long)key, src));
            c += key_less(bs, br, s, r);
        }
        return c;
    };
    // old entries before this lane's (the list is sorted)
    int at = 0;
    for (int step = KP >> 1; step; step >>= 1)
        if (key_less(Ls[at + step - 1], Lr[at + step - 1], sse, key)) at += step;
    if (at == KP - 1 && key_less(Ls[at], Lr[at], sse, key)) ++at;
    at += before(sse, key);
    // old entries move up, the highest chunk first
    for (int x = KP - 64; x >= 0; x -= 64) {
        const int e = x + lane;
        const double vs = Ls[e];
        const uint64_t vr = Lr[e];
        const int to = e + before(vs, vr);
        __atomic_signal_fence(__ATOMIC_SEQ_CST);
        __builtin_amdgcn_wave_barrier();
        if (to != e && to < KP) {
            Ls[to] = vs;
            Lr[to] = vr;
        }
        __atomic_signal_fence(__ATOMIC_SEQ_CST);
        __builtin_amdgcn_wave_barrier();
    }
    if (take && at < KP) {
        Ls[at] = sse;
        Lr[at] = key;
    }
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    __builtin_amdgcn_wave_barrier();
}

// Sorts a wave's LDS list of KP (power of two) entries by (SSE, key).
__device__ void wave_sort_list(double *Ls, uint64_t *Lr, int KP) {
    const int lane = threadIdx.x & 63;
    for (int k = 2; k <= KP; k <<= 1)
        for (int j = k >> 1; j > 0; j >>= 1) {
            for (int i = lane; i < KP; i += 64) {
                const int ixj = i ^ j;
                if (ixj > i) {
                    const bool up = (i & k) == 0;
                    const double a = Ls[i], b = Ls[ixj];
                    const uint64_t ra = Lr[i], rb = Lr[ixj];
                    if (key_less(b, rb, a, ra) == up) {
                        Ls[i] = b;
                        Ls[ixj] = a;
                        Lr[i] = rb;
                        Lr[ixj] = ra;
                    }
                }
            }
            __atomic_signal_fence(__ATOMIC_SEQ_CST);
            __builtin_amdgcn_wave_barrier();
        }
}

// Drops the later copies of equal entries of a sorted, full list (one tuple
// reached from several prefixes); the places behind the others are empty.
__device__ void wave_drop_copies(double *Ls, uint64_t *Lr, int KP) {
    const int lane = threadIdx.x & 63;
    int n = 0;
    double ps = INF;  // the entry before the chunk
    uint64_t pr = ~0ull;
    for (int m = 0; m < KP; m += 64) {
        const double v = Ls[m + lane];
        const uint64_t r = Lr[m + lane];
        double vb = __shfl_up(v, 1);
        uint64_t rb = (uint64_t)__shfl_up((long long)r, 1);
        if (lane == 0) {
            vb = ps;
            rb = pr;
        }
        ps = __shfl(v, 63);
        pr = (uint64_t)__shfl((long long)r, 63);
        const bool keep = v < INF && !(v == vb && r == rb);
        const unsigned long long b = __ballot(keep);
        __atomic_signal_fence(__ATOMIC_SEQ_CST);
        __builtin_amdgcn_wave_barrier();
        Ls[m + lane] = INF;
        Lr[m + lane] = ~0ull;
        __atomic_signal_fence(__ATOMIC_SEQ_CST);
        __builtin_amdgcn_wave_barrier();
        if (keep) {
            const int to = n + __popcll(b & ((1ull << lane) - 1ull));
            Ls[to] = v;
            Lr[to] = r;
        }
        __atomic_signal_fence(__ATOMIC_SEQ_CST);
        __builtin_amdgcn_wave_barrier();
        n += __popcll(b);
    }
}

// ------------------------------------------------------------ init kernel
// Resets the per-search device state and tabulates the cumulative number
// of work items per j-block: block jb covers j in [JB*jb, N_jb) with
// N_jb = min(JB*(jb+1), S-1); its sub-prefixes are the q-combinations of
// {0..N_jb-2}, grouped R at a time.
__device__ void s3_tile_table(const Ctx &c);

__device__ void s4_tile_table(const Ctx &c);

// s3: 0 = work-item table of the general kernel, 2 = none (D = 2, one task), 4 =
// the D = 4 record-table items, other = the D = 3 record-table items
__device__ void search_init_body(const Ctx &c, int64_t e, bool leader, int D, int R, int JB, int s3) {
    if (e < (int64_t)(SISSO_MAX_D + 1) * (c.S + 1)) {
        const int r = (int)(e / (c.S + 1));
        const int64_t n = e % (c.S + 1);
        c.btab[e] = binom(n, r);
    }
    if (leader) {
        *c.work_counter = 0;
        *c.cand_counter = 0;
        *c.theta_bits = (unsigned long long)__double_as_longlong(INF);
        *c.merge_count = 0;
        c.flags[FLAG_BATCHQ] = 0;
        c.flags[FLAG_NLISTS] = 0;
        c.stats[1] = 0;
        if (s3 == 2) {
            const int64_t q = (c.S + 63) / 64;
            c.stats[1] = (uint64_t)(q * (q + 1) / 2);
            return;
        }
        if (s3 == 4) {
            s4_tile_table(c);
            return;
        }
        if (s3) {
            s3_tile_table(c);
            return;
        }
        const int q = D - 2;
        const int64_t nblk = (c.S - 1 + JB - 1) / JB;
        uint64_t acc = 0;
        c.cum[0] = 0;
        for (int64_t b = 0; b < nblk; ++b) {
            int64_t N = JB * (b + 1);
            if (N > c.S - 1) N = c.S - 1;
            // C(N - 1, q) in closed form (q = D - 2 <= 2)
            const uint64_t m1 = (uint64_t)(N - 1);
            const uint64_t nsub = q == 0 ? 1 : q == 1 ? m1 : (m1 * (m1 - 1)) / 2;
            acc += (nsub + R - 1) / R;
            c.cum[b + 1] = acc;
        }
    }
}

__global__ void search_init_kernel(Ctx c, int D, int R, int JB, int s3) {
    search_init_body(c, (int64_t)blockIdx.x * blockDim.x + threadIdx.x, threadIdx.x == 0 && blockIdx.x == 0, D, R,
                     JB, s3);
}

// ----------------------------------------------------- threshold pre-pass
// The search starts from an upper bound theta0 of the KP-th best SSE, so
// that almost no tuple reaches the exact path.  It is built from a small,
// structured set of real tuples: the best (D-1)-subsets of the PRE_M most
// relevant features, each extended by every feature, then (D - 2 more
// rounds) the (D-1)-subsets of the best tuples found so far, extended again.
// The tuples of all rounds are distinct, so the KP-th smallest SSE of the
// pool bounds the KP-th best of the search.  Any set of real tuples gives a
// valid bound, so the selections may be heuristic: block-wide histogram
// thresholds for the first prefixes, a histogram of the pool for the bound.
constexpr int PRE_WG = 1024;      // threads of the pre-pass workgroups
constexpr int PRE_SORT = 4096;    // largest sorted candidate set
constexpr int PRE_KEEP = PRE_SORT / PRE_WG;  // candidates a thread keeps when S > PRE_SORT


// Fill key/id[0..N) with the candidates v(x) for x in [0, n): directly when
// n <= PRE_SORT, else each thread keeps its PRE_KEEP smallest.  Returns N.
template <class F>
__device__ int gather_candidates(double *key, int *id, int64_t n, F v) {
    const int tid = threadIdx.x;
    if (n <= PRE_SORT) {
        const int N = next_pow2_dev((int)n);
        for (int x = tid; x < N; x += PRE_WG) {
            key[x] = x < n ? v(x) : INF;
            id[x] = x;
        }
        return N;
    }
    double kv[PRE_KEEP];
    int ki[PRE_KEEP];
#pragma unroll
    for (int m = 0; m < PRE_KEEP; ++m) {
        kv[m] = INF;
        ki[m] = 0x7fffffff;
    }
    for (int64_t x = tid; x < n; x += PRE_WG) {
        double cv = v(x);
        int ci = (int)x;
#pragma unroll
        for (int m = 0; m < PRE_KEEP; ++m) {
            const bool less = cv < kv[m] || (cv == kv[m] && ci < ki[m]);
            const double tv = kv[m];
            const int ti = ki[m];
            kv[m] = less ? cv : tv;
            ki[m] = less ? ci : ti;
            cv = less ? tv : cv;
            ci = less ? ti : ci;
        }
    }
#pragma unroll
    for (int m = 0; m < PRE_KEEP; ++m) {
        key[tid * PRE_KEEP + m] = kv[m];
        id[tid * PRE_KEEP + m] = ki[m];
    }
    return PRE_SORT;
}

// Selections of the pre-pass without sorting: a histogram of 1024 bins over
// the order keys of the candidate values (IEEE doubles mapped to integers so
// that integer order = value order) finds, in a few barrier steps, a
// threshold t such that at least L candidates are <= t and t lies within one
// bin of the L-th smallest value.
constexpr int SEL_NB = PRE_WG;  // one histogram bin per thread
struct SelScratch {
    unsigned long long mn, mx;
    unsigned cnt;
    unsigned hist[SEL_NB];
    unsigned wsum[PRE_WG / 64];
    double res;
    int npick;
};

__device__ inline uint64_t okey(double v) {
    const uint64_t u = (uint64_t)__double_as_longlong(v);
    return (u >> 63) ? ~u : (u | 0x8000000000000000ull);
}
__device__ inline double okey_inv(uint64_t t) {
    const uint64_t u = (t >> 63) ? (t & 0x7fffffffffffffffull) : ~t;
    return __longlong_as_double((long long)u);
}

// Block-wide inclusive prefix sum of one value per thread (PRE_WG threads).
__device__ inline unsigned block_scan(unsigned v, unsigned *wsum) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    unsigned incl = v;
    for (int o = 1; o < 64; o <<= 1) {
        const unsigned y = __shfl_up(incl, o);
        if (lane >= o) incl += y;
    }
    if (lane == 63) wsum[wave] = incl;
    __syncthreads();
    unsigned base = 0;
    for (int w = 0; w < wave; ++w) base += wsum[w];
    __syncthreads();
    return incl + base;
}

// Threshold over key[0..n) (smaller is better, INF = not a candidate): a
// value t, equal to a bin's upper edge or to the largest candidate, with at
// least L candidates <= t; INF when fewer than L candidates exist.  Called
// by all PRE_WG threads.
__device__ double block_threshold(const double *key, int n, int L, SelScratch &sc) {
    const int tid = threadIdx.x;
    if (tid == 0) {
        sc.mn = ~0ull;
        sc.mx = 0;
        sc.cnt = 0;
    }
    sc.hist[tid] = 0;
    __syncthreads();
    unsigned long long mn = ~0ull, mx = 0;
    unsigned cnt = 0;
    for (int x = tid; x < n; x += PRE_WG) {
        const double v = key[x];
        if (v < INF) {
            const uint64_t u = okey(v);
            mn = u < mn ? u : mn;
            mx = u > mx ? u : mx;
            ++cnt;
        }
    }
    for (int o = 32; o >= 1; o >>= 1) {
        const unsigned long long a = (unsigned long long)__shfl_xor((long long)mn, o);
        const unsigned long long b = (unsigned long long)__shfl_xor((long long)mx, o);
        mn = a < mn ? a : mn;
        mx = b > mx ? b : mx;
        cnt += __shfl_xor(cnt, o);
    }
    if ((tid & 63) == 0) {
        atomicMin(&sc.mn, mn);
        atomicMax(&sc.mx, mx);
        atomicAdd(&sc.cnt, cnt);
    }
    __syncthreads();
    if (L < 1 || sc.cnt < (unsigned)L) return INF;
    const uint64_t lo = sc.mn, hi = sc.mx, span = hi - lo;
    int sh = 0;
    while ((span >> sh) >= (uint64_t)SEL_NB) ++sh;
    for (int x = tid; x < n; x += PRE_WG) {
        const double v = key[x];
        if (v < INF) atomicAdd(&sc.hist[(okey(v) - lo) >> sh], 1u);
    }
    __syncthreads();
    const unsigned h = sc.hist[tid];
    const unsigned incl = block_scan(h, sc.wsum);
    if (incl >= (unsigned)L && incl - h < (unsigned)L) {
        // the bin holding the L-th smallest: every candidate of bins <= tid is
        // <= its upper edge (the last occupied bin's edge is the maximum)
        const uint64_t top = span >> sh;
        const uint64_t edge = (uint64_t)tid + 1 > top ? hi : lo + (((uint64_t)tid + 1) << sh) - 1;
        sc.res = okey_inv(edge);
    }
    __syncthreads();
    return sc.res;
}

// The first (by position) up to M positions x < n with key[x] <= t, into
// out[]; returns how many.  Called by all PRE_WG threads.
__device__ int block_pick_first(const double *key, int n, double t, int M, int *out, SelScratch &sc) {
    int taken = 0;
    for (int base = 0; base < n && taken < M; base += PRE_WG) {
        const int x = base + (int)threadIdx.x;
        const bool f = x < n && key[x] < INF && key[x] <= t;
        const unsigned incl = block_scan(f ? 1u : 0u, sc.wsum);
        const int pos = taken + (int)incl - (f ? 1 : 0);
        if (f && pos < M) out[pos] = x;
        if (threadIdx.x == PRE_WG - 1) sc.npick = taken + (int)incl;
        __syncthreads();
        taken = sc.npick < M ? sc.npick : M;
        __syncthreads();
    }
    return taken;
}

// pre_select: relevance of feature j = sum over tasks of b_tj^2 (its D=1
// explained sum of squares); the PRE_M most relevant full-rank features;
// every (D-1)-subset of them scored; the PRE_Q best subsets become the first
// round's prefixes (D = 2: the PRE_Q most relevant features).  Resets the
// pre-pass state.
template <int D>
__device__ void pre_select_body(const Ctx &c) {
    __shared__ double key[PRE_SORT];
    __shared__ int id[PRE_SORT];
    __shared__ int pick[PRE_M > PRE_Q ? PRE_M : PRE_Q];
    __shared__ int sel[PRE_M];
    __shared__ SelScratch sc;
    const int tid = threadIdx.x;
    constexpr int q = D - 1;
    constexpr int NM = q > 1 ? PRE_M : PRE_Q;
    PreState &ps = *c.pre;
    if (tid == 0) ps.theta0 = INF;
    if (tid < PRE_R) {
        ps.count[tid] = 0;
        ps.done[tid] = 0;
    }
    if (tid < PRE_R * PRE_Q) ps.best[tid / PRE_Q][tid % PRE_Q] = ~0ull;
    for (int b = tid; b < PRE_BINS; b += PRE_WG) ps.hist[b] = 0;
    // 1. the NM most relevant full-rank features (up to the last histogram
    //    bin), in increasing index order
    const int N = gather_candidates(key, id, c.S, [&](int64_t j) {
        double r = 0.0;
        bool ok = true;
        for (int t = 0; t < c.T; ++t) {
            ok &= Gat(c, j, j, t) == 1.0;
            const double b = c.bhat[j * c.TP + t];
            r += b * b;
        }
        return ok ? -r : INF;
    });
    __syncthreads();
    double th = block_threshold(key, N, NM, sc);
    if (!(th < INF)) th = __DBL_MAX__;  // fewer than NM full-rank features: take them all
    const int M = block_pick_first(key, N, th, NM, pick, sc);
    // increasing feature index (positions are indices unless S > PRE_SORT)
    if (tid < M) {
        const int f = id[pick[tid]];
        int r = 0;
        for (int b2 = 0; b2 < M; ++b2) r += id[pick[b2]] < f;
        sel[r] = f;
    }
    __syncthreads();
    if (M < q) return;
    if constexpr (q == 1) {
        if (tid < M) ps.prefix[0][tid][0] = sel[tid];
        if (tid == 0) ps.count[0] = M;
        return;
    }
    // 2. score every q-subset of the selection (<= C(16, 3) = 560 of them)
    const int nsub = (int)binom(M, q);
    for (int e = tid; e < nsub; e += PRE_WG) {
        int32_t loc[MAXD], tup[MAXD];
        colex_unrank_small((uint64_t)e, q, M, loc);
        for (int m = 0; m < q; ++m) tup[m] = sel[loc[m]];
        key[e] = ne_sse_t<(D > 1 ? D - 1 : 1)>(c, tup);
    }
    __syncthreads();
    // 3. PRE_Q of the best subsets (the first in subset order at or below
    //    the threshold of the PRE_Q-th best)
    double th2 = block_threshold(key, nsub, PRE_Q, sc);
    if (!(th2 < INF)) th2 = __DBL_MAX__;
    const int Q = block_pick_first(key, nsub, th2, PRE_Q, pick, sc);
    if (tid < Q) {
        int32_t loc[MAXD];
        colex_unrank_small((uint64_t)pick[tid], q, M, loc);
        for (int m = 0; m < q; ++m) ps.prefix[0][tid][m] = sel[loc[m]];
    }
    if (tid == 0) ps.count[0] = Q;
}

template <int D>
__global__ __launch_bounds__(PRE_WG) void pre_select_kernel(Ctx c) {
    pre_select_body<D>(c);
}

// Bins of the pool histogram: 64 per factor of two (the top six mantissa
// bits), the total sum of squares c 64 bins below the top; SSEs below
// c 2^-30 share bin 0.  pool_edge(b) is the smallest value above bin b.
constexpr int PRE_SHIFT = 46;
__device__ inline int64_t pool_base(double ctot) {
    const int64_t b = (__double_as_longlong(ctot) >> PRE_SHIFT) - (PRE_BINS - 64);
    return b > 0 ? b : 0;
}
__device__ inline int pool_bin(double s, int64_t base) {
    if (!(s > 0.0)) return 0;
    const int64_t b = (__double_as_longlong(s) >> PRE_SHIFT) - base;
    return b < 0 ? 0 : b < PRE_BINS ? (int)b : PRE_BINS - 1;
}
__device__ inline double pool_edge(int b, int64_t base) {
    return b < PRE_BINS - 1 ? __longlong_as_double((base + b + 1) << PRE_SHIFT) : INF;
}

// pre_extend, round r: the workgroups of row qq score every tuple
// prefix_qq + {k} that no earlier prefix of this or a previous round reaches
// (so all tuples of the pool are distinct) and that lies in the searched
// rank range, and add them to the pool's histogram; the last workgroup of
// the round sets theta0 to the upper edge of the bin that holds the pool's
// KP-th smallest (within 1/64 of it), and, unless the round is the last,
// takes the next prefixes: the (D-1)-subsets of each prefix's best tuple,
// best tuple first, that have not been prefixes yet.  Bound: one pass of
// gathered G loads per round, spread over S / 256 workgroups per prefix.
// With one round and the largest of the prefixes' own L-th best as the bound
// theta0 was 1.7 to 8.8 times the true KP-th best on the benchmark's tree
// columns, and the tuples between the two went through the exact path one by
// one; the pooled bound is 1.0 to 1.25 times it after D - 1 rounds.
constexpr int PRE_XT = 256;      // threads per workgroup
constexpr int PRE_XBLOCKS = 64;  // most workgroups per prefix
template <int D>
__global__ __launch_bounds__(PRE_XT) void pre_extend_kernel(Ctx c, int ranged, uint64_t r0, uint64_t r1, int round,
                                                            int rounds) {
    constexpr int q = D - 1;
    constexpr int BPT = PRE_BINS / PRE_XT;  // bins per thread
    __shared__ unsigned h[PRE_BINS];
    __shared__ unsigned wsum[PRE_XT / 64];
    __shared__ unsigned long long wbest[PRE_XT / 64];
    __shared__ int exk[PRE_R * PRE_Q];
    __shared__ int s_last;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    PreState &ps = *c.pre;
    const int qq = blockIdx.y, Q = ps.count[round];
    double ctot = 0.0;
    for (int t = 0; t < c.T; ++t) ctot += c.cyy[t];
    const int64_t base = pool_base(ctot);
    // this thread's BPT consecutive bins of h: the count before them
    auto scan = [&](const unsigned (&v)[BPT]) {
        unsigned own = 0;
#pragma unroll
        for (int b = 0; b < BPT; ++b) own += v[b];
        unsigned incl = own;
        for (int o = 1; o < 64; o <<= 1) {
            const unsigned y = __shfl_up(incl, o);
            if (lane >= o) incl += y;
        }
        if (lane == 63) wsum[wave] = incl;
        __syncthreads();
        unsigned before = incl - own;
        for (int w = 0; w < wave; ++w) before += wsum[w];
        return before;
    };
    if (qq < Q) {
        int32_t P[q];
#pragma unroll
        for (int m = 0; m < q; ++m) P[m] = ps.prefix[round][qq][m];
        // an earlier prefix is part of P + {k} for one k at most: its only
        // index outside P (-1: none or several)
        if (tid < PRE_R * PRE_Q) {
            const int orr = tid / PRE_Q, oq = tid % PRE_Q;
            int out = -1, n = 0;
            if ((orr < round && oq < ps.count[orr]) || (orr == round && oq < qq)) {
#pragma unroll
                for (int m = 0; m < q; ++m) {
                    const int32_t v = ps.prefix[orr][oq][m];
                    bool in = false;
#pragma unroll
                    for (int l = 0; l < q; ++l) in |= P[l] == v;
                    if (!in) {
                        out = v;
                        ++n;
                    }
                }
            }
            exk[tid] = n == 1 ? out : -1;
        }
        for (int b = tid; b < PRE_BINS; b += PRE_XT) h[b] = 0;
        __syncthreads();
        const int nex = round * PRE_Q + qq;
        unsigned long long best = ~0ull;
        for (int64_t k = (int64_t)blockIdx.x * PRE_XT + tid; k < c.S; k += (int64_t)gridDim.x * PRE_XT) {
            bool skip = false;
#pragma unroll
            for (int m = 0; m < q; ++m) skip |= P[m] == k;
            for (int o = 0; o < nex; ++o) skip |= exk[o] == k;
            if (skip) continue;
            int32_t tup[MAXD];
            int n = 0;
            bool placed = false;
#pragma unroll
            for (int m = 0; m < q; ++m) {
                if (!placed && k < P[m]) {
                    tup[n++] = (int32_t)k;
                    placed = true;
                }
                tup[n++] = P[m];
            }
            if (!placed) tup[n++] = (int32_t)k;
            if (ranged) {
                const uint64_t rk = lex_rank(BinomTab{c.btab, c.S}, c.S, D, tup);
                if (rk < r0 || rk >= r1) continue;
            }
            const double s = ne_sse_t<D>(c, tup);
            if (!(s < INF)) continue;
            atomicAdd(&h[pool_bin(s, base)], 1u);
            const unsigned long long pk =
                ((unsigned long long)__float_as_uint((float)fmax(s, 0.0)) << 32) | (unsigned long long)(uint32_t)k;
            best = pk < best ? pk : best;
        }
        for (int o = 32; o >= 1; o >>= 1) {
            const unsigned long long y = (unsigned long long)__shfl_xor((long long)best, o);
            best = y < best ? y : best;
        }
        if (lane == 0) wbest[wave] = best;
        __syncthreads();
        if (tid == 0) {
            for (int w = 1; w < PRE_XT / 64; ++w) best = wbest[w] < best ? wbest[w] : best;
            if (best != ~0ull) atomicMin(&ps.best[round][qq], best);
        }
        // bins past the workgroup's own KP smallest cannot hold the pool's KP-th
        unsigned v[BPT];
#pragma unroll
        for (int b = 0; b < BPT; ++b) v[b] = h[tid * BPT + b];
        unsigned before = scan(v);
#pragma unroll
        for (int b = 0; b < BPT; ++b) {
            if (v[b] && before < (unsigned)c.KP) atomicAdd(&ps.hist[tid * BPT + b], v[b]);
            before += v[b];
        }
    }
    __threadfence();
    __syncthreads();
    if (tid == 0) s_last = atomicAdd(&ps.done[round], 1u) == gridDim.x * gridDim.y - 1u;
    __syncthreads();
    if (!s_last) return;
    __threadfence();
    {
        unsigned v[BPT];
#pragma unroll
        for (int b = 0; b < BPT; ++b)
            v[b] = __hip_atomic_load(&ps.hist[tid * BPT + b], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        unsigned before = scan(v);
#pragma unroll
        for (int b = 0; b < BPT; ++b) {
            if (before < (unsigned)c.KP && before + v[b] >= (unsigned)c.KP) ps.theta0 = pool_edge(tid * BPT + b, base);
            before += v[b];
        }
    }
    if (round + 1 >= rounds || wave != 0) return;
    // the next prefixes, one candidate per lane: lane i drops index i % D of
    // the tuple of rank i / D among the prefixes' best
    unsigned long long bp = ~0ull;
    if (lane < Q) bp = __hip_atomic_load(&ps.best[round][lane], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    int src = -1;
    for (int x = 0; x < PRE_Q; ++x) {
        const unsigned long long bx = (unsigned long long)__shfl((long long)bp, x);
        int rx = 0;
        for (int y = 0; y < PRE_Q; ++y) {
            const unsigned long long by = (unsigned long long)__shfl((long long)bp, y);
            rx += by < bx || (by == bx && y < x);
        }
        if (rx == lane / D) src = x;
    }
    const bool have = lane < PRE_Q * D && src >= 0;
    const unsigned long long bs = (unsigned long long)__shfl((long long)bp, have ? src : 0);
    bool take = have && bs != ~0ull;
    int32_t sub[q];
    if (take) {
        const int32_t k = (int32_t)(uint32_t)bs;
        int32_t tup[D];
#pragma unroll
        for (int m = 0; m < q; ++m) tup[m] = ps.prefix[round][src][m];
        tup[q] = k;
#pragma unroll
        for (int m = q; m > 0; --m)
            if (tup[m] < tup[m - 1]) {
                const int32_t x = tup[m];
                tup[m] = tup[m - 1];
                tup[m - 1] = x;
            }
        const int drop = lane % D;
#pragma unroll
        for (int m = 0; m < q; ++m) sub[m] = m < drop ? tup[m] : tup[m + 1];
    }
    const uint64_t key = take ? pack_tuple(sub, q) : ~0ull;
    for (int r = 0; r <= round; ++r)
        for (int o = 0; o < ps.count[r]; ++o) take = take && key != pack_tuple(ps.prefix[r][o], q);
    for (int x = 0; x < PRE_Q * D; ++x) {
        const uint64_t kx = (uint64_t)__shfl((long long)key, x);
        if (x < lane) take = take && kx != key;
    }
    const unsigned long long m = __ballot(take);
    const int at = __popcll(m & ((1ull << lane) - 1ull));
    if (take && at < PRE_Q)
#pragma unroll
        for (int x = 0; x < q; ++x) ps.prefix[round + 1][at][x] = sub[x];
    if (lane == 0) ps.count[round + 1] = __popcll(m) < PRE_Q ? __popcll(m) : PRE_Q;
}

template <class CtxT>
__device__ double theta0_of(const CtxT &c) { return c.pre->theta0; }

// --------------------------------------------------------- search kernel
constexpr int MT_RECS = 512;  // records per work item with many tasks (JB * TP)

struct SearchArgs {
    int D, TL, JB, R, KP, ranged;
    uint64_t r0, r1;
};


// LDS record of the Cholesky row of prefix (P', j) for one task:
//   v[0..q-1] = R_{P'}^{-1} G[P', j],  alpha = 1/d_j,  zs = z_j / s_j,
//   pi = p - theta_f (single task) ,  p = SSE of the prefix (P', j)
// z_j = (b_j - v.z') / s_j, s_j = sqrt(d_j), d_j = 1 - |v|^2.
// An invalid record has p = pi = NaN, which fails every comparison.

// k-dependent part of each sub-prefix solve for last index kc:
//   w' = R_{P'}^{-1} G[P', kc],  d' = 1 - |w'|^2,  zeta' = b_kc - w'.z'
// (sub-prefix factors read from LDS).  One set per sub-prefix (one task) or
// for the lane's task (many tasks).
template <int D, int NR, bool MT, typename R>
__device__ inline void hoist_k(const Ctx &c, const R *subf, const int32_t *sub, int64_t kc, int myt,
                               R (&wq)[NR][(D - 2) > 0 ? (D - 2) : 1], R (&dq)[NR], R (&zq)[NR]) {
    constexpr int q = D - 2;
    constexpr int QA = q > 0 ? q : 1;
    constexpr int SUBW = QA * QA + QA + 2;
#pragma unroll
    for (int r = 0; r < NR; ++r) {
        const int sid = MT ? myt : r;
        const R *f = subf + sid * SUBW;
        const int tt = MT ? myt : 0;
        R g[QA];
#pragma unroll
        for (int m = 0; m < q; ++m) {
            const int32_t pm = sub[(MT ? 0 : r) * QA + m];
            g[m] = (pm >= 0 && tt < c.T) ? (R)Gat(c, pm, kc, tt) : (R)0;
        }
        R dd = (tt < c.T) ? (R)Gat(c, kc, kc, tt) : (R)1;
        R zz = (tt < c.T) ? (R)c.bhat[kc * c.TP + tt] : (R)0;
#pragma unroll
        for (int m = 0; m < q; ++m) {
            R s = 0;
#pragma unroll
            for (int l = 0; l <= m; ++l) s += f[m * QA + l] * g[l];
            wq[r][m] = s;
            dd -= s * s;
            zz -= s * f[QA * QA + m];
        }
        dq[r] = dd;
        zq[r] = zz;
    }
}

// Rare path of the sweep: at least one lane passed the filter for (P', j, k).
// Recomputes the tuple terms exactly as the fast loop does, takes the SSE
// with a true division, applies the rank test and the current bound, and
// inserts the survivors into the wave's list.  Kept out of line so the fast
// loop's registers are not shaped by it.  Returns the wave's published bound.
template <int D, int NR, bool MT, typename R>
__device__ inline double slow_path(const Ctx &c, const SearchArgs &a, double *Ls, uint64_t *Lr,
                                         const R *recs, const R *subf, const int32_t *sub,
                                         const unsigned long long *smask, int64_t j, int jj, int64_t k,
                                         bool kin, bool flagged, int myt, int TL, double theta_f,
                                         double theta_pub, unsigned &offered) {
    constexpr int q = D - 2;
    constexpr int QA = q > 0 ? q : 1;
    constexpr int RECW = q + 4;
    const int KP = a.KP;
    const int lane = threadIdx.x & 63;
    const int64_t kc = kin ? k : c.S - 1;
    R wq[NR][QA], dq[NR], zq[NR];
    hoist_k<D, NR, MT, R>(c, subf, sub, kc, myt, wq, dq, zq);
    const bool lane_ok = kin && (k > j) && (MT || flagged);
    for (int r = 0; r < NR; ++r) {
        if (!MT && !((smask[r] >> jj) & 1ull)) continue;
        const R *rr = MT ? recs + (jj * TL + myt) * RECW : recs + (jj * NR + r) * RECW;
        const R g = (R)Gat(c, j, kc, MT ? myt : 0);
        R u = g;
        for (int x = 0; x < q; ++x) u = fma(-rr[x], wq[r][x], u);
        const R d = fma(-rr[q], u * u, dq[r]);
        const R z = fma(-rr[q + 1], u, zq[r]);
        double es;
        bool pass;
        if (MT) {
            R ex = 0;
            if (myt < c.T) ex = (d > rank_eps_r<R>()) ? rr[q + 3] - z * z / d : (R)INF;
            for (int o = 1; o < TL; o <<= 1) ex += __shfl_xor(ex, o);
            es = (double)ex;
            pass = (myt == 0);
        } else {
            es = (d > rank_eps_r<R>()) ? (double)(rr[q + 3] - z * z / d) : INF;
            pass = true;
        }
        const double thc = fmin(theta_f, Ls[KP - 1]);
        bool take = pass && lane_ok && (es <= thc);
        uint64_t rk = 0;
        if (take) {
            int32_t tup[MAXD];
            for (int m = 0; m < q; ++m) tup[m] = sub[(MT ? 0 : r) * QA + m];
            tup[q] = (int32_t)j;
            tup[q + 1] = (int32_t)k;
            rk = pack_tuple(tup, D);
            if (a.ranged) {
                const uint64_t lr = lex_rank(BinomTab{c.btab, c.S}, c.S, D, tup);
                if (lr < a.r0 || lr >= a.r1) take = false;
            }
        }
        list_insert_lanes(Ls, Lr, KP, take, rk, es, offered);
    }
    const double tw = Ls[KP - 1];
    if (tw < theta_pub) {
        theta_pub = tw;
        if (lane == 0) theta_publish(c.theta_bits, tw);
    }
    return theta_pub;
}

template <int D, bool MT, typename R>
__global__ __launch_bounds__(256) void search_kernel(Ctx c, SearchArgs a) {
    constexpr int q = D - 2;
    constexpr int QA = q > 0 ? q : 1;               // array extent
    constexpr int RECW = q + 4;                      // values per record
    constexpr int SUBW = QA * QA + QA + 2;           // Linv (QA x QA), z', p', valid
    constexpr int NR = MT ? 1 : SUBP;                // sub-prefixes per item

    extern __shared__ double smem[];
    const int KP = a.KP;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform (kept in an SGPR)

    // LDS carve: per-wave lists, records [256][RECW], sub-prefix factors
    double *Ls = smem + (size_t)wave * KP * 2;
    uint64_t *Lr = reinterpret_cast<uint64_t *>(Ls + KP);
    R *recs = reinterpret_cast<R *>(smem + (size_t)SEARCH_WAVES * KP * 2);
    R *subf = recs + (MT ? a.JB * a.TL : SEARCH_WG) * RECW;  // [64][SUBW] (per r, or per task)
    __shared__ int32_t s_sub[SUBP][QA];                // sub-prefix indices per r
    __shared__ int s_iq[SUBP];                         // last sub-prefix index (or -1)
    __shared__ unsigned long long s_mask[SUBP > 64 ? SUBP : 64];  // record validity per r (ST) / per jj (MT)
    __shared__ uint64_t s_item;
    __shared__ double s_theta;
    __shared__ unsigned long long s_qmask[SEARCH_WAVES][JBLK];
    __shared__ int s_qj[SEARCH_WAVES][JBLK];

    for (int m = lane; m < KP; m += 64) {
        Ls[m] = INF;
        Lr[m] = ~0ull;
    }
    double theta_pub = INF;  // last value this wave published
    unsigned offered = 0;    // tuples offered to the list (diagnostics; one atomic per wave)
    const double theta0 = theta0_of(c);
    // the FP32 form's filter bound is widened by an absolute margin (a
    // multiple of the FP32 rounding of SSEs of size up to c)
    double ctot = 0.0;
    if (sizeof(R) < 8)
        for (int t = 0; t < c.T; ++t) ctot += c.cyy[t];
    const double abs_slack = sizeof(R) < 8 ? THETA_SLACK_F32 * ctot : 0.0;

    const int TL = MT ? a.TL : 1;         // lanes per last index
    const int KL = 64 / TL;               // last indices per wave chunk
    const int JB = a.JB;                  // j values per item

    const uint64_t nitems = uni(c.cum[(c.S - 1 + JB - 1) / JB]);
    if (blockIdx.x == 0 && tid == 0) c.stats[1] = nitems;
    const double *__restrict__ Gbase = c.G;
    // items are dealt round-robin over the workgroups (largest first): a
    // shared counter would serialise on one address
    for (uint64_t next = blockIdx.x;; next += gridDim.x) {
        if (tid == 0) {
            s_item = next;
            const double ts = theta_load(c.theta_bits);
            s_theta = fmin(ts, theta0);
        }
        __syncthreads();
        const uint64_t item = uni(s_item);
        if (item >= nitems) break;
        const double theta_item = uni(s_theta);
        const double theta_f = theta_item < INF ? theta_item * (1.0 + THETA_SLACK) + abs_slack : INF;
        const R theta_r = (R)theta_f;

        // item -> (j-block, sub-prefix group) by bisection on the cumulative table
        int64_t lo = 0, hi = (c.S - 1 + JB - 1) / JB - 1;
        while (lo < hi) {
            const int64_t mid = (lo + hi + 1) / 2;
            if (c.cum[mid] <= item) lo = mid; else hi = mid - 1;
        }
        const int64_t jb = uni(lo);
        const uint64_t grp = uni(item - c.cum[jb]);
        int64_t Nj = JB * (jb + 1);
        if (Nj > c.S - 1) Nj = c.S - 1;
        const int64_t j0 = JB * jb;
        const uint64_t nsub = q > 0 ? binom(Nj - 1, q) : 1;

        // ---- records: thread -> (r, jj) for one task, (jj, t) for many (then
        //      JB * TL records, several per thread)
        for (int rid = tid; rid < (MT ? JB * TL : SEARCH_WG); rid += SEARCH_WG) {
            int r, jj, t;
            if (MT) {
                r = 0;
                jj = rid / TL;
                t = rid % TL;
            } else {
                r = tid >> 6;
                jj = tid & 63;
                t = 0;
            }
            const uint64_t sr = grp * NR + r;
            const bool rvalid = (r < NR) && (sr < nsub) && (jj < JB);
            int32_t P[QA];
            if (rvalid) {
                if (q > 0) colex_unrank_small(sr, q, Nj - 1, P);
            }
            // sub-prefix factorisation (normalised: unit diagonal)
            R Li[QA][QA], zp[QA], pp = 0;
            bool pvalid = rvalid && t < c.T;
            if (pvalid) {
                pp = (R)c.cyy[t];
                R Lf[QA][QA];
                for (int m = 0; m < q; ++m) {
                    for (int jx = 0; jx < m; ++jx) {
                        R s = (R)Gat(c, P[m], P[jx], t);
                        for (int l = 0; l < jx; ++l) s -= Lf[m][l] * Lf[jx][l];
                        Lf[m][jx] = s / Lf[jx][jx];
                    }
                    R d = (R)Gat(c, P[m], P[m], t);
                    for (int l = 0; l < m; ++l) d -= Lf[m][l] * Lf[m][l];
                    if (!(d > rank_eps_r<R>())) pvalid = false;
                    Lf[m][m] = sqrt(fmax(d, (R)0));
                }
                if (pvalid) {
                    // Li = Lf^{-1} (lower), z' = Li b_P', p' = c - |z'|^2
                    for (int m = 0; m < q; ++m) {
                        for (int jx = 0; jx <= m; ++jx) {
                            R s = (m == jx) ? (R)1 : (R)0;
                            for (int l = jx; l < m; ++l) s -= Lf[m][l] * Li[l][jx];
                            Li[m][jx] = s / Lf[m][m];
                        }
                        for (int jx = m + 1; jx < QA; ++jx) Li[m][jx] = 0;
                    }
                    for (int m = 0; m < q; ++m) {
                        R s = 0;
                        for (int l = 0; l <= m; ++l) s += Li[m][l] * (R)c.bhat[(int64_t)P[l] * c.TP + t];
                        zp[m] = s;
                        pp -= s * s;
                    }
                }
            }
            // publish the sub-prefix (one writer per r / per task)
            const int sid = MT ? t : r;
            const bool writer = MT ? (jj == 0 && t < 64) : (jj == 0 && r < NR);
            if (writer) {
                R *f = subf + sid * SUBW;
                for (int m = 0; m < QA; ++m)
                    for (int l = 0; l < QA; ++l) f[m * QA + l] = (pvalid && m < q) ? Li[m][l] : (R)0;
                for (int m = 0; m < QA; ++m) f[QA * QA + m] = (pvalid && m < q) ? zp[m] : (R)0;
                f[QA * QA + QA] = pvalid ? pp : (R)0;
                f[QA * QA + QA + 1] = pvalid ? (R)1 : (R)0;
                if (!MT) {
                    for (int m = 0; m < QA; ++m) s_sub[r][m] = (rvalid && m < q) ? P[m] : -1;
                    s_iq[r] = (rvalid && q > 0) ? P[q - 1] : (rvalid ? -1 : 1 << 30);
                } else if (t == 0) {
                    for (int m = 0; m < QA; ++m) s_sub[0][m] = (rvalid && m < q) ? P[m] : -1;
                    s_iq[0] = (rvalid && q > 0) ? P[q - 1] : (rvalid ? -1 : 1 << 30);
                }
            }
            // record of (P', j)
            const int64_t j = j0 + jj;
            const int iq = (q > 0 && rvalid) ? P[q - 1] : -1;
            bool jvalid = rvalid && (j > iq) && (j < Nj);
            R rec[RECW];
            for (int m = 0; m < RECW; ++m) rec[m] = 0;
            bool ok = false;
            if (jvalid && t < c.T && pvalid) {
                R v[QA];
                R d = (R)Gat(c, j, j, t);
                for (int m = 0; m < q; ++m) {
                    R s = 0;
                    for (int l = 0; l <= m; ++l) s += Li[m][l] * (R)Gat(c, P[l], j, t);
                    v[m] = s;
                    d -= s * s;
                }
                if (d > rank_eps_r<R>()) {
                    const R sj = sqrt(d);
                    R zn = (R)c.bhat[j * c.TP + t];
                    for (int m = 0; m < q; ++m) zn -= v[m] * zp[m];
                    zn /= sj;
                    const R p = pp - zn * zn;
                    for (int m = 0; m < q; ++m) rec[m] = v[m];
                    rec[q] = (R)1 / d;
                    rec[q + 1] = zn / sj;
                    rec[q + 2] = p - theta_r;
                    rec[q + 3] = p;
                    ok = true;
                }
            } else if (MT && jvalid && t >= c.T) {
                ok = true;  // padding task: contributes exactly zero
            }
            if (!ok) {
                rec[q + 2] = (R)__builtin_nan("");
                rec[q + 3] = (R)__builtin_nan("");
            }
            const int slot = MT ? (jj * TL + t) : (jj * NR + r);
            if (MT ? (jj < JB) : true) {
                R *dst = recs + slot * RECW;
                for (int m = 0; m < RECW; ++m) dst[m] = rec[m];
            }
            // validity masks: ST per r over jj; MT per jj over all tasks
            if (!MT) {
                const unsigned long long bal = __ballot(ok);
                if (lane == 0) s_mask[r] = bal;
            }
        }
        if (MT) {
            if (tid < 64) s_mask[tid] = 0;
        }
        __syncthreads();
        if (MT) {
            // a j is live if every real task has a valid record
            if (tid < JB) {
                bool all = true;
                for (int t = 0; t < c.T; ++t) {
                    const R *rr = recs + (tid * TL + t) * RECW;
                    all &= !__builtin_isnan(rr[q + 3]);
                }
                s_mask[tid] = all ? 1ull : 0ull;
            }
            __syncthreads();
        }

        // ---- sweep the last index k in chunks of KL per wave
        const int64_t jhi = (j0 + JB < Nj ? j0 + JB : Nj) - 1;  // largest j of the block
        const int64_t kstart = j0;  // chunks are aligned to KL, which divides the tile width
        const int tl = MT ? (lane % TL) : 0;
        const int kl = MT ? (lane / TL) : lane;
        const int myt = tl;
        unsigned long long *qmask = s_qmask[wave];
        int *qj = s_qj[wave];
        for (int64_t kb = kstart + (int64_t)wave * KL; kb < c.S; kb += (int64_t)SEARCH_WAVES * KL) {
            const int64_t k = kb + kl;
            const bool kin = k < c.S;
            const int64_t kc = kin ? k : c.S - 1;
            R wq[NR][QA], dq[NR], zq[NR];
            hoist_k<D, NR, MT, R>(c, subf, &s_sub[0][0], kc, myt, wq, dq, zq);
            const bool check = (kb <= jhi) || (kb + KL > c.S);
            // G rows of the tile (j-block, k-chunk): a uniform pointer to row j0
            // plus 32-bit row and lane offsets (one task: TP = 1).  Rows are
            // clamped to the block's last row, which lies inside the tile; lanes
            // past S read the tile's zero padding.
            const int TPk = MT ? c.TP : 1;
            const int rs = GT * TPk;
            const int ko = (int)(k & (GT - 1)) * TPk + myt;
            const int nrow = (int)(jhi - j0);            // last row of the block, < 64
            const int kr = (int)(k - j0);                // lane's k relative to j0 (> row means k > j)
            const double *__restrict__ gp =
                Gbase + ((((j0 >> 6) * c.Gnt + (kb >> 6)) << 12) + ((j0 & (GT - 1)) << 6)) * TPk;
            int nq = 0;  // steps of this chunk where some lane passed the filter
            // the j sweep, versioned on whether lanes need the k > j / k < S masks
            auto sweep = [&](auto checkc) {
                constexpr bool CHECK = decltype(checkc)::value;
                // records of one step: (P', j) for every sub-prefix (one task)
                typedef R RecSet[NR][q + 3];
                auto load_rv = [&](RecSet &rv, int jj) {
                    const R *rj = recs + jj * (NR * RECW);
#pragma unroll
                    for (int r = 0; r < NR; ++r)
#pragma unroll
                        for (int x = 0; x < q + 3; ++x) rv[r][x] = rj[r * RECW + x];
                };
                auto body = [&](int jj, R g, bool live, const RecSet &rvs) {
                    unsigned long long m = 0;
                    if (MT) {
                        // a j whose record is invalid in some task has p = NaN
                        // there, so its task sum fails the comparison
                        const R *rr = recs + (jj * TL + myt) * RECW;
                        R rv[q + 4];
#pragma unroll
                        for (int x = 0; x < q + 4; ++x) rv[x] = rr[x];
                        __asm__ volatile("" ::: "memory");
                        R u = g;
#pragma unroll
                        for (int x = 0; x < q; ++x) u = fma(-rv[x], wq[0][x], u);
                        const R d = fma(-rv[q], u * u, dq[0]);
                        const R z = fma(-rv[q + 1], u, zq[0]);
                        // p - z^2/d with a reciprocal refined by one Newton step
                        R sum = fma(-(z * z), rcp_r(d), rv[q + 3]);
                        for (int o = 1; o < TL; o <<= 1) sum += __shfl_xor(sum, o);
                        m = __ballot(sum <= theta_r && tl == 0);
                    } else {
#pragma unroll
                        for (int r = 0; r < NR; ++r) {
                            R u = g;
#pragma unroll
                            for (int x = 0; x < q; ++x) u = fma(-rvs[r][x], wq[r][x], u);
                            const R d = fma(-rvs[r][q], u * u, dq[r]);
                            const R z = fma(-rvs[r][q + 1], u, zq[r]);
                            m |= __ballot(z * z >= rvs[r][q + 2] * d);
                        }
                    }
                    if (CHECK) m &= __ballot(kin && kr > jj);
                    m = live ? m : 0ull;
                    if (m) {
                        if (lane == 0) {
                            qmask[nq] = m;
                            qj[nq] = jj;
                        }
                        ++nq;
                    }
                };
                // rows are fetched a group of JG ahead into the other of two
                // register sets, so JG loads per wave are in flight while a
                // group is scored
                constexpr int JG = SEARCH_JG;
                R ga[JG], gb[JG];
                // a uniform 64-bit base plus a 32-bit byte offset per load
                // (uniform row part + per-lane column part)
                const char *__restrict__ gpc = reinterpret_cast<const char *>(gp);
                const uint32_t ko8 = (uint32_t)ko * 8u;
                auto fetch = [&](R (&dst)[JG], int jg) {
#pragma unroll
                    for (int x = 0; x < JG; ++x) {
                        const int jr = jg + x < nrow ? jg + x : nrow;
                        const uint32_t ro = (uint32_t)(jr * rs) * 8u;
                        dst[x] = (R)*reinterpret_cast<const double *>(gpc + (ro + ko8));
                    }
                };
                // every fetched row is scored (rows past the block repeat its
                // last row and are masked out), so no load is left pending on
                // a skipped path
                auto score = [&](const R (&src)[JG], int jg) {
                    if (MT) {
                        // many tasks: the task terms of all JG rows first (independent
                        // chains), then their sums over the TL task lanes of each last
                        // index, all rows at once (row-local DPP steps; wider groups
                        // by lane shuffles)
                        R sm[JG];
#pragma unroll
                        for (int x = 0; x < JG; ++x) {
                            const int jj = jg + x <= nrow ? jg + x : nrow;
                            const R *rr = recs + (jj * TL + myt) * RECW;
                            R u = src[x];
#pragma unroll
                            for (int xx = 0; xx < q; ++xx) u = fma(-rr[xx], wq[0][xx], u);
                            const R d = fma(-rr[q], u * u, dq[0]);
                            const R z = fma(-rr[q + 1], u, zq[0]);
                            sm[x] = fma(-(z * z), rcp_r(d), rr[q + 3]);
                        }
                        if (TL >= 2) {
#pragma unroll
                            for (int x = 0; x < JG; ++x) sm[x] += dpp_r<0xB1>(sm[x]);  // lane ^ 1
                        }
                        if (TL >= 4) {
#pragma unroll
                            for (int x = 0; x < JG; ++x) sm[x] += dpp_r<0x4E>(sm[x]);  // lane ^ 2
                        }
                        if (TL >= 8) {
#pragma unroll
                            for (int x = 0; x < JG; ++x) sm[x] += dpp_r<0x141>(sm[x]);  // mirror in 8
                        }
                        if (TL >= 16) {
#pragma unroll
                            for (int x = 0; x < JG; ++x) sm[x] += dpp_r<0x140>(sm[x]);  // mirror in 16
                        }
                        if (TL >= 32) {
#pragma unroll
                            for (int x = 0; x < JG; ++x) sm[x] += __shfl_xor(sm[x], 16);
                        }
                        if (TL >= 64) {
#pragma unroll
                            for (int x = 0; x < JG; ++x) sm[x] += __shfl_xor(sm[x], 32);
                        }
#pragma unroll
                        for (int x = 0; x < JG; ++x) {
                            const int jj = jg + x <= nrow ? jg + x : nrow;
                            unsigned long long m = __ballot(sm[x] <= theta_r && tl == 0);
                            if (CHECK) m &= __ballot(kin && kr > jj);
                            m = (jg + x <= nrow) ? m : 0ull;
                            if (m) {
                                if (lane == 0) {
                                    qmask[nq] = m;
                                    qj[nq] = jj;
                                }
                                ++nq;
                            }
                        }
                        return;
                    }
#pragma unroll
                    for (int x = 0; x < JG; ++x) {
                        const int jj = jg + x <= nrow ? jg + x : nrow;
                        RecSet rv;
                        // all record reads of the step are issued before any use
                        load_rv(rv, jj);
                        __asm__ volatile("" ::: "memory");
                        body(jj, src[x], jg + x <= nrow, rv);
                    }
                };
                // drain the loads of the chunk set-up first, so that only the
                // row prefetches are outstanding when the sweep loop starts
                // (vmcnt(0); expcnt and lgkmcnt not waited on)
                __builtin_amdgcn_s_waitcnt(0x0F70);
                // one exit at the bottom: every path into the loop head has the
                // same loads outstanding, so the head needs no full drain
                fetch(ga, 0);
                for (int jg = 0;; jg += 2 * JG) {
                    fetch(gb, jg + JG);
                    score(ga, jg);
                    fetch(ga, jg + 2 * JG);
                    score(gb, jg + JG);
                    if (jg + 2 * JG > nrow) break;
                }
            };
            if (check) sweep(std::true_type{});
            else sweep(std::false_type{});
            // exact scoring of the queued steps (rare)
            for (int e = 0; e < nq; ++e) {
                const int jj = qj[e];
                const unsigned long long lm = qmask[e];
                theta_pub = slow_path<D, NR, MT, R>(c, a, Ls, Lr, recs, subf, &s_sub[0][0], s_mask, j0 + jj, jj, k,
                                                 kin, (lm >> lane) & 1ull, myt, TL, theta_f, theta_pub, offered);
            }
        }
        __syncthreads();
    }
    if (lane == 0 && offered) atomicAdd(c.cand_counter, offered);
    // write this wave's list
    const int64_t gw = (int64_t)blockIdx.x * SEARCH_WAVES + wave;
    list_store(c.list_sse + gw * KP, c.list_rank + gw * KP, Ls, Lr, KP);
}

// ---------------------------------------------- D = 3: record-table sweep
// Per search two tables of Cholesky rows are built (rec3_kernel): one row per
// pair (i1, j), and one per (group of four consecutive i1, column) for the
// group and the column together.  A tuple's SSE is at least that of any
// superset, so the sweep first tests, per (group, j, k), the fit on all six
// features {the group, j, k}: a product with four terms and 5 FP64
// instructions for four tuples, against 28 for testing the four one by one.
// Only where that bound is at or below the threshold are the group's tuples
// tested themselves.  (Bound on k: on operator-tree columns 0.1 to 1 in 1000 of the
// six-feature fits pass.)
//
// The bound's unit of work is (group, BU rows j from j0, BU columns k from j0
// + BU c) (bound_unit); an item is a run of groups over one block of G, which
// a workgroup holds in LDS while its waves take the groups in turn.  Per
// tuple, the arithmetic of the group's own test is that of search_kernel's
// single-task path: u = g - v w', d = d' - alpha u^2, zeta = zeta' - zs u, pass
// iff zeta^2 >= (p - theta) d; the group's bound is the same with four v and
// w'.  s3_group tests whole rows of a unit: lanes run over k, so a record is
// the same for every lane and is read with scalar loads; it enters the FP64
// instructions as a scalar operand, at no LDS or vector-memory cost.
constexpr int S3_NR = 4;              // i1 per group
constexpr int BU = 64;                // rows and columns of a unit (a tile of G)
constexpr int BU_WGS = 1024;  // workgroups of the bound kernels: four per CU (LDS)
constexpr int S3_LANES = 32;          // flagged (row, column) pairs of a unit taken one per lane, one task
constexpr int S3_LANES_MT = 128;      //   the same, several tasks; with more, the flagged rows are swept whole
constexpr int S3_JR = BU;
constexpr int S3_JG = 2;  // G rows per prefetch group (two groups in flight)
constexpr int S3_XCDS = 8;            // XCDs of the chip

// Rows of the record table: group g (i1 = S3_NR g .. S3_NR g + 3) holds rows
// j = S3_NR g + 1 .. S - 2, starting at row s3_rowoff(S, g).
__host__ __device__ inline int64_t s3_rowoff(int64_t S, int64_t g) {
    // sum over g' < g of (S - 2 - S3_NR g')
    return g * (S - 2) - (int64_t)S3_NR * (g * (g - 1) / 2);
}
__host__ __device__ inline int64_t s3_rows(int64_t S) {
    const int64_t ng = (S - 3) / S3_NR + 1;  // groups with at least one row (S >= 3)
    return s3_rowoff(S, ng);
}

// record of (i1, j), i1 = S3_NR g + r, in row R = s3_rowoff(S, g) + j - S3_NR g - 1:
//   rec[(R S3_NR + r) 4 + {0, 1, 2, 3}] = {v, 1/d_j, z_j / s_j, p}
// with v = G[i1][j], d_j = 1 - v^2, s_j = sqrt(d_j), z_j = (b_j - v b_i1) / s_j,
// p = c - b_i1^2 - z_j^2 (the SSE of the pair); p = NaN (fails every
// comparison) unless i1 < j, column i1 is live and d_j > RANK_EPS.
// Group tables: group g's own factor (correlations of its live columns, in
// index order, G = R^T R) projects any column x onto the group's span, v = R^-T
// G[g, x].  Columns x = 4 g .. S - 1, field by field (columns consecutive):
//   v0..v3, alpha = 1/d, zs = e/d, p, d, e with e = b_x - v.z, d = 1 - |v|^2,
//   z = R^-T b_g, p = c - |z|^2 - e^2/d (the SSE of the group and x).
// A tuple's j reads alpha, zs, p, its k reads d and e.  p = 0 marks a j whose
// group or column is too close to dependent for the bound (it always passes), p
// = S3_NEVER one without a tuple (a constant column), d = S3_NEVER a constant
// k.  A column of the group itself leaves the group alone (v = 0, alpha = 0).
//
// The bound is compared with a slack, S3_SLACK on d and S3_SLACK c on theta,
// so it has to be known to that.  A factor of K columns is the exact one of a G
// changed by at most (K + 1) 2^-53 per entry (Cholesky's backward error; as
// much again is allowed for the explicit inverse), which changes d, zeta /
// sqrt(c) and p / c of the pair (j, k) by at most
//   e = 2 K (K + 1) 2^-53 |R^-1|^2 (1 + 1 / sqrt(d_j))^2
// (|.| the Frobenius norm, d_j the pivot of j).  With a = S3_SLACK - e and P =
// (p - theta) / c, a fit at or below theta has zeta^2 >= P d c, and it passes if
// (sqrt(P d) - e)^2 >= (P - a) (d - a), which holds for e <= S3_SLACK / 2.
// bound_tau gives the smallest d_j with that.  (Pivots above S3_TAU alone are
// not enough: in a group of columns each close to the span of the ones before
// it |R^-1|^2 reaches 1e15, and the fit came out up to c too high.)
constexpr double S3_TAU = 1e-5;       // smallest pivot of a group
constexpr double S3_SLACK = 1e-6;
constexpr double S3_ESLACK = 1e-13;   // slack above the rounding of the test itself, times c
constexpr double S3_NEVER = 1e300;
// smallest pivot of a column j that is tried with a group of K columns, norm = |R^-1|^2 (above 1: none)
template <int K>
__device__ inline double bound_tau(double norm) {
    const double t = sqrt(S3_SLACK / (4.0 * K * (K + 1) * 0x1p-53 * norm)) - 1.0;
    return t >= 1.0 ? fmax(S3_TAU, 1.0 / (t * t)) : 2.0;
}
// fields of a table over K features
enum { BF_AL, BF_ZS, BF_P, BF_D, BF_E, BF_N };  // after the K entries of v
constexpr int S3_FIELDS = S3_NR + BF_N;
// columns of the groups before g (S - 4 g' each)
__host__ __device__ inline int64_t s3g_off(int64_t S, int64_t g) { return g * S - (int64_t)S3_NR * (g * (g - 1) / 2); }
int64_t s3_group_doubles(int64_t S) { return S >= 3 ? s3g_off(S, (S - 3) / S3_NR + 1) * S3_FIELDS : 0; }

__device__ void s3_group_record(const Ctx &c, int64_t g, int64_t x) {
    const int64_t S = c.S, nt = c.Gnt;
    const int64_t j = S3_NR * g + x;
    if (g > (S - 3) / S3_NR || j > S - 1) return;
    const int ts = c.tstar[0], TP = c.TP;
    const double *__restrict__ G1 = c.G1;
    // the group's factor (the same for every thread of the group)
    double Li[S3_NR][S3_NR], L[S3_NR][S3_NR], z[S3_NR], pg = c.cyy[ts], norm = 0.0;
    bool bad = false;
#pragma unroll
    for (int m = 0; m < S3_NR; ++m) {
        const int64_t i = S3_NR * g + m;
        const bool live = i < S && G1[gidx(i, i, nt, 1, 0)] > 0.5;
        double d = 1.0;
#pragma unroll
        for (int l = 0; l < m; ++l) {
            double s = live ? G1[gidx(S3_NR * g + l, i, nt, 1, 0)] : 0.0;
#pragma unroll
            for (int q = 0; q < l; ++q) s -= L[m][q] * L[l][q];
            L[m][l] = s * Li[l][l];
            d -= L[m][l] * L[m][l];
        }
        bad |= live && !(d > S3_TAU);
        Li[m][m] = live && d > S3_TAU ? 1.0 / sqrt(d) : 0.0;
        double zz = 0.0;
#pragma unroll
        for (int l = 0; l < m; ++l) {
            double s = 0.0;
#pragma unroll
            for (int q = l; q < m; ++q) s += L[m][q] * Li[q][l];
            Li[m][l] = -Li[m][m] * s;
            norm += Li[m][l] * Li[m][l];
            zz += Li[m][l] * c.bhat[(S3_NR * g + l < S ? S3_NR * g + l : 0) * TP + ts];
        }
        norm += Li[m][m] * Li[m][m];
        if (live) zz += Li[m][m] * c.bhat[i * TP + ts];
        z[m] = zz;
        pg -= zz * zz;
    }
    const double tau = bound_tau<S3_NR>(norm);
    bad |= tau > 1.0;
    double v[S3_NR] = {0.0, 0.0, 0.0, 0.0}, al = 0.0, zs = 0.0, p = pg, d = 0.0, e = 0.0;
    if (!(G1[gidx(j, j, nt, 1, 0)] > 0.5)) {
        p = d = S3_NEVER;
    } else if (bad) {
        p = 0.0;
    } else if (j >= S3_NR * (g + 1)) {
        d = 1.0;
        e = c.bhat[j * TP + ts];
#pragma unroll
        for (int m = 0; m < S3_NR; ++m) {
            double s = 0.0;
#pragma unroll
            for (int l = 0; l <= m; ++l) s += Li[m][l] * G1[gidx(S3_NR * g + l, j, nt, 1, 0)];
            v[m] = s;
            d -= s * s;
            e -= s * z[m];
        }
        if (d > tau) {
            al = 1.0 / d;
            zs = e * al;
            p = pg - e * zs;
        } else {
            p = 0.0;
        }
    }
    const int64_t len = S - S3_NR * g;
    double *o = c.recg + s3g_off(S, g) * S3_FIELDS + x;
#pragma unroll
    for (int m = 0; m < S3_NR; ++m) o[m * len] = v[m];
    o += S3_NR * len;
    o[BF_AL * len] = al;
    o[BF_ZS * len] = zs;
    o[BF_P * len] = p;
    o[BF_D * len] = d;
    o[BF_E * len] = e;
}

// (its grid also does the per-search initialisation of search_init_kernel)
// Grid: x over (j, r) of one group, y over groups (blockIdx.y = g); z = 1
// builds the group records, x over j.
// Launched with PRE_WG threads per workgroup and one workgroup column more
// than the records need: workgroup (last, 0) runs the pre-pass selection
// (independent of the table and of the initialisation, which leaves the
// pre-pass count to it), beside the record workgroups.
__global__ __launch_bounds__(PRE_WG) void rec3_kernel(Ctx c, double *__restrict__ rec) {
    const int64_t ex = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t g = blockIdx.y;
    if (blockIdx.z == 1) {
        s3_group_record(c, g, ex);
        return;
    }
    search_init_body(c, g * (int64_t)gridDim.x * blockDim.x + ex, ex == 0 && g == 0, 3, SUBP, JBLK, 1);
    if (blockIdx.x == gridDim.x - 1 && g == 0) {
        pre_select_body<3>(c);
        return;
    }
    const int64_t S = c.S;
    const int r = (int)(ex % S3_NR);
    const int64_t j = S3_NR * g + 1 + ex / S3_NR;
    if (g > (S - 3) / S3_NR || j > S - 2) return;
    const int64_t i1 = S3_NR * g + r;
    const int64_t e = (s3_rowoff(S, g) + j - S3_NR * g - 1) * S3_NR + r;
    // the filter task's pair (i1, j) (the only task when T = 1)
    const int ts = c.tstar[0];
    const double *G1 = c.G1;
    const int64_t nt = c.Gnt;
    double v = 0.0, al = 0.0, zs = 0.0, p = __builtin_nan("");
    if (i1 < j && G1[gidx(i1, i1, nt, 1, 0)] > RANK_EPS) {
        const double zp = c.bhat[i1 * c.TP + ts];
        const double pp = c.cyy[ts] - zp * zp;
        const double g = G1[gidx(i1, j, nt, 1, 0)];
        const double d = G1[gidx(j, j, nt, 1, 0)] - g * g;
        if (d > RANK_EPS) {
            const double sj = sqrt(d);
            const double zn = (c.bhat[j * c.TP + ts] - g * zp) / sj;
            v = g;
            al = 1.0 / d;
            zs = zn / sj;
            p = pp - zn * zn;
        }
    }
    double *o = rec + e * 4;
    o[0] = v;
    o[1] = al;
    o[2] = zs;
    o[3] = p;
}

// Row blocks jb: j in [BU jb, BU jb + BU), j <= S - 2; each has the column
// chunks from its own on (k >= j0).  The bases of class q (a base is a group, D
// = 4 a pair of groups) are those whose first row lies in row block q; class
// q's units are its bases times the s3_class_units(S, q) blocks of G.  Items
// are numbered by class, then by run of bases, then by block of G, so that the
// items at work at one time read few bases' tables, and these from L2.
__host__ __device__ inline int64_t s3_nblocks(int64_t S) { return S >= 3 ? (S - 2) / BU + 1 : 0; }
// blocks of G in the first r row blocks of class q
__host__ __device__ inline int64_t s3_class_below(int64_t S, int64_t q, int64_t r) {
    return r * ((S + BU - 1) / BU - q) - r * (r - 1) / 2;
}
__host__ __device__ inline int64_t s3_class_units(int64_t S, int64_t q) {
    return s3_class_below(S, q, s3_nblocks(S) - q);
}
// groups with a first row 4 g + 1 below row block q's end
__host__ __device__ inline int64_t s3_groups_to(int64_t S, int64_t q) {
    int64_t jmax = q * BU + BU - 1;
    if (jmax > S - 2) jmax = S - 2;
    return q >= 0 && jmax >= 1 ? (jmax - 1) / S3_NR + 1 : 0;
}
// bases below class q (pairs: of groups g1 <= g2)
struct S3Groups {
    static __host__ __device__ int64_t below(int64_t S, int64_t q) { return s3_groups_to(S, q - 1); }
};

// Bases per item: a block of G (32 KB) is read once per run, and the runs
// have to fill the chip: 16 from 8192 units on (4 a wave), down to one a wave.
__host__ __device__ inline int bound_run(uint64_t units) { return units <= 4096 ? 4 : units <= 8192 ? 8 : 16; }
template <class B>
__host__ __device__ inline uint64_t bound_units(int64_t S) {
    uint64_t acc = 0;
    for (int64_t q = 0; q < s3_nblocks(S); ++q)
        acc += (uint64_t)((B::below(S, q + 1) - B::below(S, q)) * s3_class_units(S, q));
    return acc;
}
// all items; cum[q] = items of the classes before q
template <class B>
__host__ __device__ inline uint64_t bound_items(int64_t S, int run, uint64_t *cum) {
    uint64_t acc = 0;
    if (cum) cum[0] = 0;
    for (int64_t q = 0; q < s3_nblocks(S); ++q) {
        const int64_t nb = B::below(S, q + 1) - B::below(S, q);
        acc += (uint64_t)((nb + run - 1) / run * s3_class_units(S, q));
        if (cum) cum[q + 1] = acc;
    }
    return acc;
}
__device__ void s3_tile_table(const Ctx &c) {
    c.stats[1] = bound_items<S3Groups>(c.S, bound_run(bound_units<S3Groups>(c.S)), c.cum);
}
uint64_t s3_items_host(int64_t S) { return bound_items<S3Groups>(S, bound_run(bound_units<S3Groups>(S)), nullptr); }

constexpr int S3_WPE = 4;  // waves per SIMD the register budget is sized for
// Several tasks, D = 3: tuples that pass the filter task's own test are
// buffered in LDS (key, filter-task SSE), and mt_flush takes up to 64 of them,
// one per lane: the second largest task's SSE is added (a tighter lower
// bound), and the survivors are scored over every task, 64 / LT tuples at a
// time with LT lanes each (lane q LT + l sums the tasks t = l mod LT of tuple
// q, then a butterfly sum and rank flag), and inserted into the wave's list.
constexpr int MT_BUF = 128;  // buffered tuples per wave (a flush takes 64)

__device__ __forceinline__ unsigned mt_flush(const Ctx &c, double *Ls, uint64_t *Lr, int KP, const uint64_t *bk,
                                             const double *be, int cnt, double theta_f) {
    const int lane = threadIdx.x & 63;
    const int TP = c.TP, t2 = c.tstar[1];
    auto task_sse = [&](const int32_t (&tq)[3], int t, bool &ok) {
        double gm[3][3], bv[3];
#pragma unroll
        for (int m2 = 0; m2 < 3; ++m2) {
#pragma unroll
            for (int j2 = 0; j2 <= m2; ++j2) gm[m2][j2] = Gat(c, tq[m2], tq[j2], t);
            bv[m2] = c.bhat[(int64_t)tq[m2] * TP + t];
        }
        return ne_sse_core<3>(gm, bv, c.cyy[t], ok);
    };
    bool take = lane < cnt;
    const uint64_t key = take ? bk[lane] : 0;
    int32_t tup[3] = {0, 1, 2};
    if (take) {
        unpack_tuple(key, 3, tup);
        if (t2 >= 0) {
            bool ok2 = true;
            const double e2 = task_sse(tup, t2, ok2);
            take = ok2 && be[lane] + e2 <= theta_f;
        }
    }
    const int LT = TP < 64 ? TP : 64;
    const int R = 64 / LT, slot = lane / LT;
    unsigned offered = 0;
    unsigned long long m = __ballot(take);
    while (m) {
        int src = -1;
        for (int q = 0; q < R; ++q) {
            const int sb = m ? __ffsll((long long)m) - 1 : -1;
            if (slot == q) src = sb;
            m &= m - 1;
        }
        const uint64_t kq = (uint64_t)__shfl((long long)key, src < 0 ? 0 : src);
        double part = 0.0;
        bool okp = true;
        if (src >= 0) {
            int32_t tq[3];
            unpack_tuple(kq, 3, tq);
            for (int t = lane % LT; t < c.T; t += LT) part += task_sse(tq, t, okp);
        }
        for (int o = 1; o < LT; o <<= 1) {
            part += __shfl_xor(part, o);
            okp = __shfl_xor((int)okp, o) != 0 && okp;
        }
        const double esv = okp ? part : INF;
        for (int q = 0; q < R; ++q) {
            if (__shfl(src, q * LT) < 0) break;
            const double v2 = __shfl(esv, q * LT);
            const uint64_t k2 = (uint64_t)__shfl((long long)kq, q * LT);
            if (v2 <= fmin(theta_f, Ls[KP - 1])) {
                ++offered;
                list_insert(Ls, Lr, KP, v2, k2);
            }
        }
    }
    return offered;
}

// a wave's buffer of tuples that passed the filter task (several tasks)
struct MtBuf {
    uint64_t *key;
    double *sse;
    int n;
};

// Appends the tuples of the lanes in take to the buffer and flushes it from 64 on.
__device__ __forceinline__ void mt_append(const Ctx &c, double *Ls, uint64_t *Lr, int KP, MtBuf &mb, bool take,
                                          uint64_t key, double sse, double theta_f, unsigned &offered) {
    const int lane = threadIdx.x & 63;
    const unsigned long long m = __ballot(take);
    if (!m) return;
    if (take) {
        const int at = mb.n + __popcll(m & ((1ull << lane) - 1ull));
        mb.key[at] = key;
        mb.sse[at] = sse;
    }
    mb.n += __popcll(m);
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    __builtin_amdgcn_wave_barrier();
    if (mb.n < 64) return;
    offered += mt_flush(c, Ls, Lr, KP, mb.key, mb.sse, 64, theta_f);
    // keep the rest (fewer than 64) at the front
    const int rest = mb.n - 64;
    uint64_t kx = 0;
    double ex = 0.0;
    if (lane < rest) {
        kx = mb.key[64 + lane];
        ex = mb.sse[64 + lane];
    }
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    __builtin_amdgcn_wave_barrier();
    if (lane < rest) {
        mb.key[lane] = kx;
        mb.sse[lane] = ex;
    }
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    __builtin_amdgcn_wave_barrier();
    mb.n = rest;
}

// Tables that a launch only reads, in the constant address space: where the
// address is uniform the loads are scalar, also in a kernel that stores.
typedef const __attribute__((address_space(4))) double CDouble;
typedef const __attribute__((address_space(4))) char CChar;
__device__ inline CDouble *cptr(const double *p) { return (CDouble *)(uintptr_t)p; }

// Where a unit lies: its rows j0 .. jhi, column chunk kcx, from column kb.
struct S3Tile {
    int64_t j0, jhi, kb, kcx;
};

// The rows jlo .. jhi of a unit for one group: the unit's k-dependent terms, the
// tuples' own test over the rows, exact scoring of the flagged steps into the
// wave's list (one task) or buffer (several tasks), and the publication of the
// wave's bound.
// CtxT: Ctx (a kernel argument) or a Ctx in the constant address space (a
// copy in device memory, read by the batched kernel): both let the compiler
// read the fields with scalar loads into scalar registers.
template <bool MT, class CtxT>
__device__ __forceinline__ void s3_group(const CtxT &c, const SearchArgs &a, const double *__restrict__ rec,
                                         const S3Tile &tl, int64_t g, int64_t jlo, int64_t jhi, double *Ls,
                                         uint64_t *Lr, double theta0, double &theta_pub, unsigned &offered,
                                         MtBuf &mb, unsigned long long *s_qw, int *s_qjw) {
    const int KP = a.KP;
    const int lane = threadIdx.x & 63;
    const int64_t S = c.S;
    const int64_t nt = c.Gnt;
    const double *__restrict__ Gb = c.G1;
    const int TP = c.TP;
    const int ts = c.tstar[0];
    const double *__restrict__ inv_st = c.inv_s + (int64_t)ts * S;
    {
        const int64_t kcx = tl.kcx;
        const int64_t j0 = tl.j0;
        const int nrow = (int)(jhi - jlo);  // steps 0..nrow
        const int64_t kb = tl.kb;
        const int64_t k0 = kb + lane;
        const bool kv0 = k0 < S;
        // columns read for lanes past S: any valid one (never passes)
        const int64_t kk0 = kv0 ? k0 : S - 1;
        const bool diag = kcx == 0;            // k <= j only in chunk 0

        double th = fmin(theta0, theta_load(c.theta_bits));
        th = fmin(th, Ls[KP - 1]);
        const double theta_f = th < INF ? th * (1.0 + THETA_SLACK) : INF;

        // k-dependent part of each i1's solve
        double w[S3_NR], dq[S3_NR], zq[S3_NR];
        {
            // G[k][k] is 1 for a live column and 0 for a constant one; the
            // contiguous 1/|x - mean| row says which (0 = constant)
            const double gd0 = inv_st[kk0] > 0.0 ? 1.0 : 0.0;
            const double b0 = c.bhat[kk0 * TP + ts];
#pragma unroll
            for (int r = 0; r < S3_NR; ++r) {
                int64_t i1 = S3_NR * g + r;
                if (i1 > S - 1) i1 = S - 1;
                const double zp = c.bhat[i1 * TP + ts];
                const double wv = Gb[gidx(i1, kk0, nt, 1, 0)];
                w[r] = wv;
                // a lane past S or on a constant column never passes
                dq[r] = (kv0 && gd0 > RANK_EPS) ? fma(-wv, wv, gd0) : __builtin_nan("");
                zq[r] = fma(-wv, zp, b0);
            }
        }
        // G[j][k] for the block's rows: j >> 6 is the same for the whole block
        // (S3_JR divides 64), so one uniform tile-row base plus 32-bit per-lane
        // byte offsets (column part + row j & 63) address every step
        const char *__restrict__ gtile =
            reinterpret_cast<const char *>(Gb + (((j0 >> 6) * nt) << 12));
        const uint32_t voff0 = (uint32_t)((((kk0 >> 6) << 12) + (kk0 & 63) + ((jlo & 63) << 6)) * 8);
        // records of row jlo + x are 128 bytes at recj + 128 x (uniform)
        CChar *recj = (CChar *)(cptr(rec) + (size_t)(s3_rowoff(S, g) + jlo - S3_NR * g - 1) * (S3_NR * 4));
        int nq = 0;
        auto sweep = [&](auto diagc) {
            constexpr bool DIAG = decltype(diagc)::value;
            constexpr int JG = S3_JG;
            double ga[JG], gb[JG];  // g(j, k)
            auto fetch = [&](double (&dst)[JG], int jg) {
#pragma unroll
                for (int x = 0; x < JG; ++x) {
                    const uint32_t jr = (uint32_t)(jg + x < nrow ? jg + x : nrow);
                    dst[x] = *reinterpret_cast<const double *>(gtile + (voff0 + jr * 512u));
                }
            };
            // records of one step are two halves of 64 bytes (i1 = 4g, 4g+1 and
            // 4g+2, 4g+3); each half is loaded while the other is scored.  Scalar
            // loads may return out of order, so the half in flight is waited for
            // (lgkmcnt(0)) before the next one is issued.
            auto load_half = [&](double (&rv)[8], int jr, int h) {
                CDouble *rp = (CDouble *)(recj + (size_t)jr * 128 + h * 64);
#pragma unroll
                for (int e = 0; e < 8; ++e) rv[e] = rp[e];
            };
            auto score_half = [&](const double (&rv)[8], const double gv, int h, unsigned long long &m0) {
#pragma unroll
                for (int rr = 0; rr < 2; ++rr) {
                    const int r = 2 * h + rr;
                    const double pi = rv[4 * rr + 3] - theta_f;
                    const double u = fma(-rv[4 * rr], w[r], gv);
                    const double d = fma(-rv[4 * rr + 1], u * u, dq[r]);
                    const double z = fma(-rv[4 * rr + 2], u, zq[r]);
                    m0 |= __ballot(z * z >= pi * d);
                }
            };
            double ra[8], rb[8];
            load_half(ra, 0, 0);
            auto score = [&](const double (&src)[JG], int jg) {
#pragma unroll
                for (int x = 0; x < JG; ++x) {
                    const int jr = jg + x;
                    const int jc = jr <= nrow ? jr : nrow;
                    unsigned long long m0 = 0;
                    __builtin_amdgcn_s_waitcnt(0xC07F);
                    load_half(rb, jc, 1);
                    __builtin_amdgcn_sched_barrier(0);
                    score_half(ra, src[x], 0, m0);
                    __builtin_amdgcn_s_waitcnt(0xC07F);
                    load_half(ra, jr + 1 <= nrow ? jr + 1 : nrow, 0);
                    __builtin_amdgcn_sched_barrier(0);
                    score_half(rb, src[x], 1, m0);
                    if (DIAG) m0 &= __ballot(k0 > jlo + jr);
                    if (jr > nrow) m0 = 0;
                    if (m0) {
                        if (lane == 0) {
                            s_qw[nq] = m0;
                            s_qjw[nq] = jr;
                        }
                        ++nq;
                    }
                }
            };
            __builtin_amdgcn_s_waitcnt(0x0F70);
            fetch(ga, 0);
            for (int jg = 0;; jg += 2 * JG) {
                fetch(gb, jg + JG);
                score(ga, jg);
                fetch(ga, jg + 2 * JG);
                score(gb, jg + JG);
                if (jg + 2 * JG > nrow) break;
            }
        };
        if (diag) sweep(std::true_type{});
        else sweep(std::false_type{});
        __atomic_signal_fence(__ATOMIC_SEQ_CST);
        __builtin_amdgcn_wave_barrier();

        // exact scoring of the flagged steps (rare): the same terms, a true
        // division, the rank test and the current bound
        for (int e = 0; e < nq; ++e) {
            const int jr = s_qjw[e];
            const int64_t j = jlo + jr;
            const unsigned long long fm = s_qw[e];
            CDouble *rp = (CDouble *)(recj + (size_t)jr * 128);
            const double gg = *reinterpret_cast<const double *>(gtile + (voff0 + (uint32_t)jr * 512u));
            // r is wave-uniform here: pick the k-data by selects, so the
            // arrays stay in registers (an indexed read would move them to
            // scratch memory, stored on every unit)
            auto pick = [&](const double (&arr)[S3_NR], int r) {
                double v = arr[0];
#pragma unroll
                for (int q = 1; q < S3_NR; ++q)
                    if (q == r) v = arr[q];
                return v;
            };
            for (int r = 0; r < S3_NR; ++r) {
                const double v = rp[4 * r], al = rp[4 * r + 1], zs = rp[4 * r + 2], p = rp[4 * r + 3];
                const double u = fma(-v, pick(w, r), gg);
                const double d = fma(-al, u * u, pick(dq, r));
                const double z = fma(-zs, u, pick(zq, r));
                const int32_t tup[3] = {(int32_t)(S3_NR * g + r), (int32_t)j, (int32_t)k0};
                // the step's flag covers all four i1 of the group: this i1's own
                // terms decide (NaN records: i1 >= j or a rank deficient pair)
                const double es = (d > RANK_EPS) ? p - (z * z) / d : INF;
                bool take =
                    ((fm >> lane) & 1ull) && kv0 && k0 > j && es <= (MT ? theta_f : fmin(theta_f, Ls[KP - 1]));
                if (take && a.ranged) {
                    const uint64_t lr = lex_rank(BinomTab{c.btab, c.S}, c.S, 3, tup);
                    if (lr < a.r0 || lr >= a.r1) take = false;
                }
                const uint64_t rk = take ? pack_tuple(tup, 3) : 0;
                if constexpr (MT) mt_append(c, Ls, Lr, KP, mb, take, rk, es, theta_f, offered);
                else list_insert_lanes(Ls, Lr, KP, take, rk, es, offered);
            }
        }
        const double tw = Ls[KP - 1];
        if (tw < theta_pub) {
            theta_pub = tw;
            if (lane == 0) theta_publish(c.theta_bits, tw);
        }
    }
}

// 64 candidates, one per lane: (group g, row j, column k) whose bound passed.
// Each lane tests the group's four tuples (the terms of s3_group, the same
// arithmetic).
template <bool MT, class CtxT>
__device__ __forceinline__ void s3_candidates(const CtxT &c, const SearchArgs &a, const double *__restrict__ rec,
                                              bool have, uint64_t key, double *Ls, uint64_t *Lr, double theta0,
                                              double &theta_pub, unsigned &offered, MtBuf &mb) {
    const int KP = a.KP;
    const int64_t S = c.S, nt = c.Gnt;
    const int TP = c.TP, ts = c.tstar[0];
    const double *__restrict__ G1 = c.G1;
    const int64_t g = have ? (int64_t)(key >> 44) : 0, j = have ? (int64_t)((key >> 22) & 0x3FFFFF) : 1;
    const int64_t k = have ? (int64_t)(key & 0x3FFFFF) : 2;
    double th = fmin(theta0, theta_load(c.theta_bits));
    th = fmin(th, Ls[KP - 1]);
    const double theta_f = th < INF ? th * (1.0 + THETA_SLACK) : INF;
    const double gg = G1[gidx(j, k, nt, 1, 0)];
    const double gd = c.inv_s[(int64_t)ts * S + k] > 0.0 ? 1.0 : 0.0;
    const double bk = c.bhat[k * TP + ts];
    const double *__restrict__ rp = rec + (s3_rowoff(S, g) + j - S3_NR * g - 1) * (S3_NR * 4);
    double es[S3_NR];
#pragma unroll
    for (int r = 0; r < S3_NR; ++r) {
        int64_t i1 = S3_NR * g + r;
        i1 = i1 < S ? i1 : S - 1;  // past S: the record is NaN
        const double v = rp[4 * r], al = rp[4 * r + 1], zs = rp[4 * r + 2], p = rp[4 * r + 3];
        const double w = G1[gidx(i1, k, nt, 1, 0)], zp = c.bhat[i1 * TP + ts];
        const double dq = gd > RANK_EPS ? fma(-w, w, gd) : __builtin_nan("");
        const double zq = fma(-w, zp, bk);
        const double u = fma(-v, w, gg);
        const double d = fma(-al, u * u, dq);
        const double z = fma(-zs, u, zq);
        es[r] = (d > RANK_EPS) ? p - (z * z) / d : INF;
    }
#pragma unroll
    for (int r = 0; r < S3_NR; ++r) {
        const int32_t tup[3] = {(int32_t)(S3_NR * g + r), (int32_t)j, (int32_t)k};
        bool take = have && es[r] <= (MT ? theta_f : fmin(theta_f, Ls[KP - 1]));
        if (take && a.ranged) {
            const uint64_t lr = lex_rank(BinomTab{c.btab, c.S}, c.S, 3, tup);
            if (lr < a.r0 || lr >= a.r1) take = false;
        }
        const uint64_t rk = pack_tuple(tup, 3);
        if constexpr (MT) mt_append(c, Ls, Lr, KP, mb, take, rk, es[r], theta_f, offered);
        else list_insert_lanes(Ls, Lr, KP, take, rk, es[r], offered);
    }
    const double tw = Ls[KP - 1];
    if (tw < theta_pub) {
        theta_pub = tw;
        if ((threadIdx.x & 63) == 0) theta_publish(c.theta_bits, tw);
    }
}

// Where the bound does not help (a wave's units pass it in succession for more
// pairs than are taken one by one) a wave leaves it out for the next 1, 3, ..
// 31 units, so a problem whose fits all reach the threshold pays a few per cent.
struct S3Skip {
    int left = 0, fails = 0;
    __device__ bool skip() {
        if (left == 0) return false;
        --left;
        return true;
    }
    __device__ void result(bool failed) {
        fails = failed ? (fails < 6 ? fails + 1 : 6) : 0;
        left = fails < 2 ? 0 : (1 << (fails - 1)) - 1;
    }
};

// item t: its block of G and its bases b0 .. b1 - 1
template <class B>
__device__ __forceinline__ void bound_locate(int64_t S, const uint64_t *__restrict__ cum, uint64_t t, int run,
                                             S3Tile &tl, int64_t &b0, int64_t &b1) {
    int64_t q = 0, hi = s3_nblocks(S) - 1;
    while (q < hi) {
        const int64_t mid = (q + hi + 1) >> 1;
        if (cum[mid] <= t) q = mid; else hi = mid - 1;
    }
    const uint32_t nu = (uint32_t)s3_class_units(S, q), rem = (uint32_t)(t - cum[q]);
    const uint32_t u = rem % nu;
    b0 = B::below(S, q) + (int64_t)(rem / nu) * run;
    b1 = b0 + run < B::below(S, q + 1) ? b0 + run : B::below(S, q + 1);
    // u = s3_class_below(S, q, r) + column chunk
    const float m = (float)((S + BU - 1) / BU - q) + 0.5f;
    int64_t r = (int64_t)(m - sqrtf(fmaxf(m * m - 2.0f * (float)u, 0.0f)));
    while (s3_class_below(S, q, r) > (int64_t)u) --r;
    while (s3_class_below(S, q, r + 1) <= (int64_t)u) ++r;
    r = uni(r);
    tl.kcx = (int64_t)u - s3_class_below(S, q, r);
    tl.j0 = (q + r) * BU;
    tl.jhi = (tl.j0 + BU - 1 < S - 2) ? tl.j0 + BU - 1 : S - 2;
    tl.kb = tl.j0 + tl.kcx * BU;
}

// A unit's G (one tile, 32 KB) to LDS by the workgroup.  Odd rows are turned by
// 16 columns: a wave's read of four rows by sixteen columns then covers every
// bank once per pass.
__device__ __forceinline__ void bound_load(double *__restrict__ s_g, const double *__restrict__ G1, int64_t nt,
                                           const S3Tile &tl) {
    const double2 *__restrict__ src =
        reinterpret_cast<const double2 *>(G1 + (((tl.j0 >> 6) * nt + (tl.kb >> 6)) << 12));
#pragma unroll
    for (int it = 0; it < BU * BU / 2 / 256; ++it) {
        const int e = (int)threadIdx.x + 256 * it, row = e >> 5, c = 2 * (e & 31);
        *reinterpret_cast<double2 *>(s_g + row * BU + (c ^ ((row & 1) << 4))) = src[e];
    }
}

// The bound of one unit for one base of K = 4 NK features (its table: columns
// from x0, len of them; its rows with a tuple from j0 + lo).  A pair (j, k)
// passes unless
//   x = zeta^2 - (p - theta) d < -eps, as a polynomial in u = g - v.w:
//   q + u (A u - 2 zeta' zs), A = zs^2 + (p - theta) alpha, q = zeta'^2 - (p - theta) d'
// (eps a slack above the rounding of the terms, which cancel): a NaN passes,
// and so does any pair when p is at or below theta.
// u is a matrix product (rows x K by K x columns, G the addend), so it runs in
// 16 x 16 blocks on the FP64 matrix cores; the rest is 4 FMAs and a comparison
// per (j, k).  (The matrix cores multiply FP64 at the vector units' rate; what
// the blocks save is the rows' operands: read by scalar loads, 96 bytes a row
// and wave, they held a vector form of this loop at 530 us for n = 2000, S =
// 600, D = 4 (422 here) and at 56 us for S = 1000, D = 3 (45).)
// Operands of v_mfma_f64_16x16x4f64: A[i][f] in lane i + 16 f, B[f][c] in lane
// c + 16 f, D[i][c] in lane c + 16 (i % 4), register i / 4.
// Passing pairs: `lanes` of them; lane e = 16 rb + 4 cb + i returns those of
// the 16 x 16 block (rb, cb)'s rows 4 i .. 4 i + 3 in m, bit 16 h + c for row 16
// rb + 4 i + h and column 16 cb + c.
typedef double double4_t __attribute__((ext_vector_type(4)));
template <int NK>
__device__ __forceinline__ void bound_unit(const double *__restrict__ s_g, int64_t S, const S3Tile &tl,
                                           const double *__restrict__ tab, int64_t x0, int64_t len, int lo,
                                           double theta_s, double neg, double (*par)[BU],
                                           unsigned long long &mine, int &lanes) {
    constexpr int K = 4 * NK;
    const int lane = threadIdx.x & 63, col = lane & 15, h = lane >> 4;
    const int nrow = (int)(tl.jhi - tl.j0) + 1;
    bool some = false;
    mine = 0;
    // field f of column x (a table has less than 4 GB: 32-bit offsets)
    const uint32_t ln = (uint32_t)len;
    auto at = [&](uint32_t f, uint32_t x) {
        return *reinterpret_cast<const double *>(reinterpret_cast<const char *>(tab) + (f * ln + x) * 8u);
    };
    auto colx = [&](int x) {  // column j0 or kb + .., kept inside the table
        const int y = x < (int)S ? x : (int)S - 1;
        return (uint32_t)(y > (int)x0 ? y - (int)x0 : 0);
    };
    // the rows' terms (a lane per row)
    {
        const uint32_t j = colx((int)tl.j0 + lane);
        const double al = at(K + BF_AL, j), zs = at(K + BF_ZS, j);
        const double pi = fmax(at(K + BF_P, j) - theta_s, 0.0);
        par[0][lane] = fma(pi, al, zs * zs);
        par[1][lane] = zs;
        par[2][lane] = pi;
    }
    // the columns' terms
    const int ncb = S - tl.kb >= BU ? 4 : (int)((S - tl.kb + 15) >> 4);
    double w[4][NK], dq[4], z2[4], zz[4];  // z2 = -2 zeta', zz = zeta'^2
#pragma unroll
    for (int cb = 0; cb < 4; ++cb) {
        const uint32_t k = colx((int)tl.kb + 16 * cb + col);
#pragma unroll
        for (int s = 0; s < NK; ++s) w[cb][s] = at(4 * s + h, k);
        const double e = at(K + BF_E, k);
        dq[cb] = at(K + BF_D, k) - S3_SLACK;
        z2[cb] = -2.0 * e;
        zz[cb] = e * e;
    }
    const bool diag = tl.kcx == 0;
    auto rowv = [&](double (&v)[NK], int rb) {
        const uint32_t j = colx((int)tl.j0 + 16 * rb + col);
#pragma unroll
        for (int s = 0; s < NK; ++s) v[s] = -at(4 * s + h, j);
    };
    double v[NK], vn[NK];
    const int rb0 = lo >> 4;
    rowv(vn, rb0);
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    __builtin_amdgcn_wave_barrier();
#pragma unroll 1
    for (int rb = rb0; rb < 4 && 16 * rb < nrow; ++rb) {
#pragma unroll
        for (int s = 0; s < NK; ++s) v[s] = vn[s];
        rowv(vn, rb < 3 ? rb + 1 : 3);
        double A[4], zs[4], pi[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            A[i] = par[0][16 * rb + 4 * i + h];
            zs[i] = par[1][16 * rb + 4 * i + h];
            pi[i] = par[2][16 * rb + 4 * i + h];
        }
        const double *__restrict__ grow = s_g + (16 * rb + h) * BU + col;
        // two blocks at a time (their products and tests overlap), but those
        // past S or all below the diagonal
#pragma unroll
        for (int cp = 0; cp < 4; cp += 2) {
            if (cp >= ncb || (diag && cp + 1 < rb)) continue;
            double4_t u[2];
            unsigned long long m[2][4], any = 0;
#pragma unroll
            for (int e = 0; e < 2; ++e)
#pragma unroll
                for (int i = 0; i < 4; ++i) u[e][i] = grow[4 * i * BU + 16 * ((cp + e) ^ (h & 1))];
#pragma unroll
            for (int s = 0; s < NK; ++s)
#pragma unroll
                for (int e = 0; e < 2; ++e)
                    u[e] = __builtin_amdgcn_mfma_f64_16x16x4f64(v[s], w[cp + e][s], u[e], 0, 0, 0);
#pragma unroll
            for (int e = 0; e < 2; ++e)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const double x = fma(u[e][i], fma(A[i], u[e][i], zs[i] * z2[cp + e]),
                                         fma(-pi[i], dq[cp + e], zz[cp + e]));
                    m[e][i] = __ballot(!(x < neg));
                    any |= m[e][i];
                }
            if (any) {
                some = true;
                unsigned long long f = 0;
#pragma unroll
                for (int e = 0; e < 2; ++e)
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        if ((lane & 7) == 4 * e + i) f = m[e][i];
                if ((lane >> 3) == 2 * rb + (cp >> 1)) mine = f;
            }
        }
    }
    lanes = 0;
    if (some) {
        // those with a tuple: lo <= row < nrow, column < S, k > j
        const int x = 16 * (lane >> 4) + 4 * (lane & 3), c0 = 16 * ((lane >> 2) & 3);
        const int64_t left = S - tl.kb - c0;  // columns of the block
        const unsigned cols = left >= 16 ? 0xffffu : left > 0 ? (1u << left) - 1u : 0u;
        unsigned long long ok = 0;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int first = diag ? x + r - c0 + 1 : 0;  // first column with k > j
            const unsigned f = first >= 16 ? 0u : first > 0 ? cols & (0xffffu << first) : cols;
            if (x + r >= lo && x + r < nrow) ok |= (unsigned long long)(f & 0xffffu) << (16 * r);
        }
        mine &= ok;
        int n = __popcll(mine);
        for (int o = 1; o < 64; o <<= 1) n += __shfl_xor(n, o);
        lanes = __builtin_amdgcn_readfirstlane(n);
    }
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    __builtin_amdgcn_wave_barrier();
}

// Calls put(place, row, column) for every passing pair: places count from 0.
template <class Put>
__device__ __forceinline__ void bound_each(unsigned long long mine, Put put) {
    const int lane = threadIdx.x & 63;
    const int n = __popcll(mine);
    int at = n;
    for (int o = 1; o < 64; o <<= 1) {
        const int y = __shfl_up(at, o);
        if (lane >= o) at += y;
    }
    at -= n;
    while (mine) {
        const int b = __builtin_ctzll(mine);
        mine &= mine - 1;
        put(at++, 16 * (lane >> 4) + 4 * (lane & 3) + (b >> 4), 16 * ((lane >> 2) & 3) + (b & 15));
    }
}
// bit x: some pair of row x passes
__device__ __forceinline__ unsigned long long bound_rows(unsigned long long mine) {
    const int lane = threadIdx.x & 63;
    unsigned f = 0;
#pragma unroll
    for (int r = 0; r < 4; ++r)
        if ((mine >> (16 * r)) & 0xffffull) f |= 1u << r;
    unsigned long long rows = (unsigned long long)f << (16 * (lane >> 4) + 4 * (lane & 3));
    for (int o = 1; o < 64; o <<= 1) rows |= (unsigned long long)__shfl_xor((long long)rows, o);
    return uni((uint64_t)rows);
}

// Group g's bound over a unit (threshold th): the pairs that pass, as
// bound_unit returns them.  Without a bound (th infinite, or left out) all
// rows with a tuple are set in rows, and lanes is more than any limit; else
// rows is set when there are more than limit.
template <class CtxT>
__device__ __forceinline__ void s3_bound(const CtxT &c, const double *__restrict__ recg, const double *__restrict__ s_g,
                                         const S3Tile &tl, int64_t g, double th, S3Skip &skip, int limit,
                                         double (*par)[BU], unsigned long long &mine,
                                         unsigned long long &rows, int &lanes) {
    const int64_t S = c.S;
    const int64_t first = S3_NR * g + 1;  // the group's first row
    const int lo = first > tl.j0 ? (int)(first - tl.j0) : 0, n = (int)(tl.jhi - tl.j0);
    if (!skip.skip() && th < INF) {
        const double ctot = c.cyy[c.tstar[0]];
        bound_unit<1>(s_g, S, tl, recg + s3g_off(S, g) * S3_FIELDS, S3_NR * g, S - S3_NR * g, lo,
                      th * (1.0 + THETA_SLACK) + S3_SLACK * ctot, -S3_ESLACK * ctot, par, mine, lanes);
        skip.result(lanes > limit);
        rows = lanes > limit ? bound_rows(mine) : 0;
    } else {
        rows = (~0ull >> (63 - n)) & (~0ull << lo);
        lanes = 1 << 30;
    }
}

__device__ inline uint64_t s3_cand(int64_t g, int64_t j, int64_t k) {
    return ((uint64_t)g << 44) | ((uint64_t)j << 22) | (uint64_t)k;
}

// The bound pass of the single search.  What it flags goes to the workgroup's
// own segments of two pools (no shared counter: same-address atomics
// serialise): the (group, row, column) candidates of a unit one by one while
// there are at most `limit`, else the unit's flagged rows, eight to an item.
// The groups of the best features are flagged on most rows, so the pools are
// scored by a kernel of their own, spread evenly: scored where they were found
// they left a few waves running long after the rest (n = 2000, S = 1000: 145
// us against 105 without the bound; the two kernels take 43 and 22).  Vector
// instructions and the matrix cores take 0.54 to 0.58 of the CUs' busy cycles
// here; the rest waits for tables and blocks of G, and the CUs are idle for 0.4
// to 0.45 of the kernel, at its start and as its waves end.
__device__ inline uint64_t s3_row_item(int64_t octet, int64_t g, int64_t kcx, unsigned mask) {
    return ((uint64_t)octet << 42) | ((uint64_t)g << 22) | ((uint64_t)kcx << 8) | mask;
}
// Items t0 .. t1 - 1 are dealt to the workgroups in turn (their costs are
// nearly equal; a shared counter would serialise on one address), XCD-aware:
// workgroup b runs on XCD b mod 8, and each round's items go to the XCDs in
// eight runs, whose G and tables meet in one L2.
__device__ inline uint64_t bound_first(uint64_t t0) {
    const uint64_t b = blockIdx.x, n = gridDim.x;
    return t0 + (n % S3_XCDS == 0 ? b % S3_XCDS * (n / S3_XCDS) + b / S3_XCDS : b);
}
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(S3_WPE))) void search3_kernel(
    Ctx c, const double *__restrict__ recg, const uint64_t *__restrict__ cum, uint64_t t0, uint64_t t1,
    uint32_t wg_units, int limit, int run, int glo, int ghi) {
    __shared__ double s_g[BU * BU];
    __shared__ double s_par[SEARCH_WAVES][3][BU];
    __shared__ unsigned s_n[2];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    uint64_t *__restrict__ cands = c.s3_cands + (size_t)blockIdx.x * wg_units * limit;
    uint64_t *__restrict__ items = c.s3_rows + (size_t)blockIdx.x * wg_units * (BU / 8);
    if (threadIdx.x < 2) s_n[threadIdx.x] = 0;
    const int64_t S = c.S;
    const double th = fmin(theta0_of(c), theta_load(c.theta_bits));
    S3Skip skip;
    for (uint64_t t = bound_first(t0); t < t1; t += gridDim.x) {
        S3Tile tl;
        int64_t b0, b1;
        bound_locate<S3Groups>(S, cum, t, run, tl, b0, b1);
        b0 = b0 > glo ? b0 : glo;
        b1 = b1 <= ghi ? b1 : (int64_t)ghi + 1;
        if (b0 >= b1) continue;
        __syncthreads();  // the waves have left the previous item's G
        bound_load(s_g, c.G1, c.Gnt, tl);
        __syncthreads();
        for (int64_t g = b0 + wave; g < b1; g += SEARCH_WAVES) {
            unsigned long long mine = 0, rows;
            int lanes;
            s3_bound<Ctx>(c, recg, s_g, tl, g, th, skip, limit, s_par[wave], mine, rows, lanes);
            if (!lanes) continue;
            if (lanes > limit) {
                const unsigned m = lane < 8 ? (unsigned)(rows >> (8 * lane)) & 0xffu : 0u;  // rows 8 lane ..
                const unsigned long long b = __ballot(m != 0);
                unsigned at = 0;
                if (lane == 0) at = atomicAdd(&s_n[1], (unsigned)__popcll(b));
                at = (unsigned)__shfl((int)at, 0);
                if (m)
                    items[at + __popcll(b & ((1ull << lane) - 1ull))] = s3_row_item((tl.j0 >> 3) + lane, g, tl.kcx, m);
                continue;
            }
            unsigned at = 0;
            if (lane == 0) at = atomicAdd(&s_n[0], (unsigned)lanes);
            at = (unsigned)__shfl((int)at, 0);
            bound_each(mine, [&](int p, int x, int k) { cands[at + p] = s3_cand(g, tl.j0 + x, tl.kb + k); });
        }
    }
    __syncthreads();
    if (threadIdx.x < 2) c.s3_count[2 * blockIdx.x + threadIdx.x] = s_n[threadIdx.x];
}

// A large search runs in passes of S3_PASS units (bound, then scoring), which
// bounds the pools (0.7 GB with one task, 2.3 GB with several; S = 5000 is one
// pass).  Units that the segments hold: each workgroup takes at most one item
// more than its share.
constexpr uint64_t S3_PASS = 1ull << 21;
static size_t pool_units(uint64_t items, int run, uint64_t pass) {
    return (size_t)(((items < pass / run ? items : pass / run) + BU_WGS) * run);
}
size_t s3_pool_units(int64_t S) { return pool_units(s3_items_host(S), bound_run(bound_units<S3Groups>(S)), S3_PASS); }
int s3_lanes(int T) { return T > 1 ? S3_LANES_MT : S3_LANES; }

// first[p][s] = items of pool p in the segments before s, first[p][nseg] = all
// of them (workgroup-wide, 256 threads; ends with a barrier)
__device__ void pool_scan(const uint32_t *__restrict__ count, uint32_t nseg, uint64_t *const (&first)[2],
                          unsigned long long (*s_w)[SEARCH_WAVES]) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // thread i owns segments i per .. (i + 1) per - 1
    const uint32_t per = (nseg + 255) / 256;
    unsigned long long own[2] = {0, 0}, incl[2];
    for (uint32_t x = 0; x < per; ++x) {
        const uint32_t s = tid * per + x;
        if (s < nseg)
            for (int p = 0; p < 2; ++p) own[p] += count[2 * s + p];
    }
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        incl[p] = own[p];
        for (int o = 1; o < 64; o <<= 1) {
            const unsigned long long y = (unsigned long long)__shfl_up((long long)incl[p], o);
            if (lane >= o) incl[p] += y;
        }
        if (lane == 63) s_w[p][wave] = incl[p];
    }
    __syncthreads();
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        unsigned long long at = incl[p] - own[p];
        for (int w = 0; w < wave; ++w) at += s_w[p][w];
        for (uint32_t x = 0; x < per; ++x) {
            const uint32_t s = tid * per + x;
            if (s >= nseg) break;
            first[p][s] = at;
            at += count[2 * s + p];
        }
        if (tid == 255) first[p][nseg] = at;
    }
    __syncthreads();
}
__device__ inline uint32_t pool_segment(const uint64_t *first, uint32_t nseg, uint64_t e) {
    uint32_t lo = 0, hi = nseg - 1;
    while (lo < hi) {
        const uint32_t mid = (lo + hi + 1) >> 1;
        if (first[mid] <= e) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// Scores the pools: the candidates 64 at a time, one per lane, and the row
// items in equal contiguous runs, one run per wave (consecutive items of one
// group, row block and column chunk are swept together).  Every workgroup
// scans the segments' counts itself (a scan kernel in between cost 7 us).
// resume: the waves' lists of the previous pass are carried on.
template <bool MT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void s3_eval_kernel(
    Ctx c, SearchArgs a, const double *__restrict__ rec, uint32_t nseg, uint32_t wg_units, int limit, int resume) {
    extern __shared__ double smem[];
    __shared__ unsigned long long s_q[SEARCH_WAVES][S3_JR];
    __shared__ int s_qj[SEARCH_WAVES][S3_JR];
    __shared__ uint64_t s_bk[MT ? SEARCH_WAVES : 1][MT ? MT_BUF : 1];
    __shared__ double s_be[MT ? SEARCH_WAVES : 1][MT ? MT_BUF : 1];
    __shared__ unsigned long long s_w[2][SEARCH_WAVES];
    const int KP = a.KP;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    double *Ls = smem + (size_t)wave * KP * 2;
    uint64_t *Lr = reinterpret_cast<uint64_t *>(Ls + KP);
    // first[p][s]: items of pool p in the segments before s
    uint64_t *first[2];
    first[0] = reinterpret_cast<uint64_t *>(smem + (size_t)SEARCH_WAVES * KP * 2);
    first[1] = first[0] + nseg + 1;
    const int64_t gw = (int64_t)blockIdx.x * SEARCH_WAVES + wave;
    const uint64_t nw = (uint64_t)gridDim.x * SEARCH_WAVES;
    if (resume) {
        list_load(Ls, Lr, c.list_sse + gw * KP, c.list_rank + gw * KP, KP);
    } else {
        for (int m = lane; m < KP; m += 64) {
            Ls[m] = INF;
            Lr[m] = ~0ull;
        }
    }
    pool_scan(c.s3_count, nseg, first, s_w);
    // the segment of item e of pool p
    auto segment = [&](int p, uint64_t e) { return pool_segment(first[p], nseg, e); };
    const uint64_t ncand = uni(first[0][nseg]), nitem = uni(first[1][nseg]);
    const double theta0 = theta0_of(c);
    double theta_pub = INF;
    unsigned offered = 0;
    MtBuf mb{s_bk[MT ? wave : 0], s_be[MT ? wave : 0], 0};
    // the last waves take the first candidates: the first ones get the items
    // (several tasks: as few at a time as leave every wave some, see below)
    const uint64_t fair = (ncand + nw - 1) / nw;
    const uint32_t per = MT && fair < 64 ? (uint32_t)(fair ? fair : 1) : 64u;
    for (uint64_t b = nw - 1 - (uint64_t)gw; b * per < ncand; b += nw) {
        const uint64_t e = b * per + lane;
        const bool in = lane < (int)per && e < ncand;
        uint64_t key = 0;
        if (in) {
            const uint32_t s = segment(0, e);
            key = c.s3_cands[(size_t)s * wg_units * limit + (e - first[0][s])];
        }
        s3_candidates<MT, Ctx>(c, a, rec, in, key, Ls, Lr, theta0, theta_pub, offered, mb);
    }
    auto place = [](uint64_t it, S3Tile &tl) {
        tl.kcx = (int64_t)((it >> 8) & 0x3FFF);
        tl.j0 = (int64_t)(it >> 42) * 8 / S3_JR * S3_JR;
        tl.kb = tl.j0 + tl.kcx * BU;
        return (int64_t)((it >> 22) & 0xFFFFF);  // the group
    };
    if constexpr (MT) {
        // a tuple that passes the filter task costs a solve per task, mostly one
        // tuple after another in the wave that found it: the items' rows are
        // dealt out in turn, 8 at a time while that leaves a wave four shares,
        // else 4, 2 or 1.  (In runs of whole items a few waves went on long after
        // the rest: 40 tasks of 12 rows, S = 60: the call 2375 us, now 577; 8 tasks
        // of 60, S = 500, a noise target: 4625, now 3375.)
        const uint64_t nrow = nitem * 8;
        int R = 8;
        while (R > 1 && nrow < (uint64_t)R * 4 * nw) R >>= 1;
        for (uint64_t q = (uint64_t)gw * R; q < nrow; q += nw * R) {
            const uint64_t e = q >> 3;
            const uint32_t s = pool_segment(first[1], nseg, e);
            const uint64_t it = uni(c.s3_rows[(size_t)s * wg_units * (BU / 8) + (e - first[1][s])]);
            const unsigned m = ((unsigned)it & 0xffu) & (((1u << R) - 1u) << (q & 7));
            if (!m) continue;
            S3Tile tl;
            const int64_t g = place(it, tl);
            const int64_t j = tl.j0 + 8 * (int64_t)((it >> 42) & 7);
            s3_group<MT, Ctx>(c, a, rec, tl, g, j + __builtin_ctz(m), j + 31 - __builtin_clz(m), Ls, Lr, theta0,
                              theta_pub, offered, mb, s_q[wave], s_qj[wave]);
        }
        if (mb.n > 0) {
            const double th = fmin(theta0, theta_load(c.theta_bits));
            const double theta_f = th < INF ? th * (1.0 + THETA_SLACK) : INF;
            offered += mt_flush(c, Ls, Lr, KP, mb.key, mb.sse, mb.n, theta_f);
        }
    } else {
        const uint64_t run = (nitem + nw - 1) / nw;
        uint64_t e = uni((uint64_t)((uint64_t)gw * run));
        const uint64_t e1 = uni((uint64_t)(e + run < nitem ? e + run : nitem));
        if (e < e1) {
            uint32_t s = segment(1, e);
            auto item = [&]() {
                while (first[1][s + 1] <= e) ++s;
                return uni(c.s3_rows[(size_t)s * wg_units * (BU / 8) + (e - first[1][s])]);
            };
            constexpr uint64_t OCTET = 7ull << 42;  // the rows' place in their block
            uint64_t it = item();
            for (;;) {
                S3Tile tl;
                const int64_t g = place(it, tl);
                const uint64_t same = (it & ~OCTET) >> 8;  // group, column chunk, row block
                unsigned long long rows = 0;
                bool more = true;
                for (;;) {
                    rows |= (unsigned long long)(it & 0xff) << (8 * ((it >> 42) & 7));
                    if (++e >= e1) {
                        more = false;
                        break;
                    }
                    it = item();
                    if ((it & ~OCTET) >> 8 != same) break;
                }
                const int x0 = __builtin_ctzll(rows), x1 = 63 - __builtin_clzll(rows);
                s3_group<MT, Ctx>(c, a, rec, tl, g, tl.j0 + x0, tl.j0 + x1, Ls, Lr, theta0, theta_pub, offered, mb,
                                  s_q[wave], s_qj[wave]);
                if (!more) break;
            }
        }
    }
    if (lane == 0 && offered) atomicAdd(c.cand_counter, offered);
    list_store(c.list_sse + gw * KP, c.list_rank + gw * KP, Ls, Lr, KP);
}

// ---------------------------------------- batched D = 3 search (one task)
constexpr int S3B_WPE = 3;  // waves per SIMD of the batched kernel (its per-problem state)
// Several independent one-task problems searched by one launch: the record
// tables and pre-pass bounds of every problem are built first (each problem
// on its own), then the workgroups of one persistent grid pull entries from a
// device queue -- entry = a run of S3B_RUN consecutive items of one problem,
// problems ordered by decreasing item count, so the largest start first and
// the small ones fill the tail.  A wave keeps one list per problem it works
// on: when its next entry belongs to another problem it writes the list to
// that problem's next free list slot (a wave never returns to a problem, as
// entries are taken in queue order) and starts an empty one.  Each problem's
// merge then reads the lists its waves wrote; the rest is the one-problem
// path, so the results equal those of separate searches bitwise.
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(S3B_WPE))) void search3_batch_kernel(
    BatchSearchArgs b) {
    extern __shared__ double smem[];
    __shared__ double s_g[BU * BU];
    __shared__ double s_par[SEARCH_WAVES][3][BU];
    __shared__ unsigned long long s_q[SEARCH_WAVES][BU];
    __shared__ int s_qj[SEARCH_WAVES][BU];
    __shared__ uint64_t s_k[SEARCH_WAVES][S3_LANES];
    __shared__ uint32_t s_it;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    double *Ls = smem + (size_t)wave * b.KPmax * 2;
    uint64_t *Lr = reinterpret_cast<uint64_t *>(Ls + b.KPmax);
    uint32_t *queue = b.ctx[0]->flags + FLAG_BATCHQ;
    const uint32_t nitems = b.item_end[b.P - 1];
    int cur = -1;
    S3Skip skip;
    MtBuf mb{nullptr, nullptr, 0};
    const Ctx *cur_ctx = nullptr;
    double theta0 = INF, theta_pub = INF;
    unsigned offered = 0;
    int run = 0;
    SearchArgs a{};
    a.D = 3;
    auto flush = [&](const Ctx &c) {
        uint32_t slot = 0;
        if (lane == 0) slot = atomicAdd(c.flags + FLAG_NLISTS, 1u);
        slot = (uint32_t)__shfl((int)slot, 0);
        if (lane == 0 && offered) atomicAdd(c.cand_counter, offered);
        if (slot < (uint32_t)c.nwaves)
            list_store(c.list_sse + (int64_t)slot * a.KP, c.list_rank + (int64_t)slot * a.KP, Ls, Lr, a.KP);
    };
    uint32_t nxt = 0;  // thread 0: the entry after this one (taken ahead)
    if (threadIdx.x == 0) nxt = atomicAdd(queue, 1u);
    for (;;) {
        __syncthreads();
        if (threadIdx.x == 0) s_it = nxt;
        __syncthreads();
        const uint32_t it = (uint32_t)__builtin_amdgcn_readfirstlane((int)s_it);
        if (it >= nitems) break;
        if (threadIdx.x == 0) nxt = atomicAdd(queue, 1u);
        typedef const __attribute__((address_space(4))) uint32_t CU32;
        typedef const __attribute__((address_space(4))) uint64_t CU64;
        CU32 *ie = (CU32 *)(uintptr_t)b.item_end;
        int p = 0;
        while (ie[p] <= it) ++p;
        p = __builtin_amdgcn_readfirstlane(p);
        const uint32_t first = p ? ie[p - 1] : 0u;
        const Ctx *cp = (const Ctx *)(uintptr_t)((CU64 *)(uintptr_t)b.ctx)[p];
        typedef const __attribute__((address_space(4))) Ctx CCtx;
        CCtx &c = *(CCtx *)(uintptr_t)cp;
        const int64_t S = c.S;
        if (p != cur) {
            if (cur >= 0) flush(*cur_ctx);
            cur_ctx = cp;
            cur = p;
            a.KP = c.KP;
            for (int m = lane; m < a.KP; m += 64) {
                Ls[m] = INF;
                Lr[m] = ~0ull;
            }
            __atomic_signal_fence(__ATOMIC_SEQ_CST);
            __builtin_amdgcn_wave_barrier();
            theta0 = theta0_of(c);
            theta_pub = INF;
            offered = 0;
            skip = S3Skip{};
            run = bound_run(bound_units<S3Groups>(S));
        }
        const uint64_t n = c.cum[s3_nblocks(S)];
        const uint64_t t0 = (uint64_t)(it - first) * S3B_RUN;
        const uint64_t t1 = t0 + S3B_RUN < n ? t0 + S3B_RUN : n;
        for (uint64_t t = t0; t < t1; ++t) {
            S3Tile tl;
            int64_t b0, b1;
            bound_locate<S3Groups>(S, c.cum, t, run, tl, b0, b1);
            __syncthreads();
            bound_load(s_g, c.G1, c.Gnt, tl);
            __syncthreads();
            for (int64_t g = b0 + wave; g < b1; g += SEARCH_WAVES) {
                unsigned long long mine = 0, rows;
                int lanes;
                s3_bound<CCtx>(c, c.recg, s_g, tl, g, fmin(fmin(theta0, theta_load(c.theta_bits)), Ls[a.KP - 1]), skip,
                               S3_LANES, s_par[wave], mine, rows, lanes);
                if (!lanes) continue;
                if (lanes > S3_LANES) {
                    const int x0 = __builtin_ctzll(rows), x1 = 63 - __builtin_clzll(rows);
                    s3_group<false, CCtx>(c, a, c.rec3, tl, g, tl.j0 + x0, tl.j0 + x1, Ls, Lr, theta0, theta_pub,
                                          offered, mb, s_q[wave], s_qj[wave]);
                    continue;
                }
                // at most S3_LANES candidates: one per lane
                const int cnt = lanes;
                bound_each(mine, [&](int p, int x, int k) { s_k[wave][p] = s3_cand(g, tl.j0 + x, tl.kb + k); });
                __atomic_signal_fence(__ATOMIC_SEQ_CST);
                __builtin_amdgcn_wave_barrier();
                const uint64_t key = lane < cnt ? s_k[wave][lane] : 0;
                s3_candidates<false, CCtx>(c, a, c.rec3, lane < cnt, key, Ls, Lr, theta0, theta_pub, offered, mb);
                __atomic_signal_fence(__ATOMIC_SEQ_CST);
                __builtin_amdgcn_wave_barrier();
            }
        }
    }
    if (cur >= 0) flush(*cur_ctx);
}

// ------------------------------------------- D = 4, one task: record table
// The D = 3 design one level up, with a larger superset.  The indices are cut
// into groups of four; per pair of groups (g1 <= g2) and j the Cholesky row of
// j against the pair's eight columns is built once per search (rec4_kernel).
// The sweep tests, per (pair, j, k), the fit on all ten features {g1, g2, j,
// k}: a product with eight terms and 5 FP64 instructions for sixteen tuples i1
// in g1, i2 in g2, against 144 for testing the tuples one by one.  A tuple's
// SSE is at least that of any superset, so only where that bound is at or
// below the threshold are the sixteen tuples tested themselves (2 in 1000
// ten-feature fits on operator-tree columns, n = 2000, S = 600; three in four
// of those are rows in the span of their pair, whose bound is not tried).
// Units and items are those of D = 3, over pairs; what a unit flags goes to
// its workgroup's segments of two pools, which s4_eval_kernel scores: the
// candidates (g1, g2, j, k) one per lane while there are at most S4_LANES of
// them, else (also without a threshold) the whole unit, in items of one i2 and
// S4_DR rows.  n = 2000, S = 600: tables 47 us, bound 420 us, scoring 170 us,
// against 0.5 ms for a table of all triples and 5.3 ms for the tuples' own
// tests.  The bound is limited by FP64 issue: vector instructions (at four
// cycles each) and the matrix cores take 0.65 of the CUs' busy cycles, which are
// 0.86 of the kernel's; tables and blocks of G take the rest.
constexpr int S4_WPE = 4;  // waves per SIMD the register budget is sized for
constexpr int S4_NR = 4;              // indices per group
constexpr int S4_DR = 16;             // rows of a dense item (of a unit taken whole)
constexpr int S4_ITEMS = S4_NR * S3_JR / S4_DR;  // dense items of a unit
constexpr int S4_FIELDS = 2 * S4_NR + BF_N;
constexpr int S4_FAC = 48;            // doubles per factor: R^-1 (36), z (8), SSE of the pair, bound_tau
// A large search runs in passes of S4_PASS units (bound, then scoring), which
// bounds the candidate pool at 1.1 GB.
constexpr uint64_t S4_PASS = 1ull << 18;

// groups with a tuple (i2 in the group, j = i2 + 1 <= S - 2)
__host__ __device__ inline int64_t s4_groups(int64_t S) { return S >= 4 ? (S - 3) / S4_NR + 1 : 0; }
__host__ __device__ inline int64_t s4_pairs_below(int64_t g) { return g * (g + 1) / 2; }  // pairs with g2 < g
// columns of the pairs before (g1, g2), S - 4 g2 each (x = 4 g2 .. S - 1):
// sum over g < g2 of (g + 1) (S - 4 g), and g1 (S - 4 g2) more
__host__ __device__ inline int64_t s4_off(int64_t S, int64_t g1, int64_t g2) {
    return S * s4_pairs_below(g2) - S4_NR * ((g2 - 1) * g2 * (g2 + 1) / 3) + g1 * (S - S4_NR * g2);
}
struct S4Pairs {
    static __host__ __device__ int64_t below(int64_t S, int64_t q) { return s4_pairs_below(s3_groups_to(S, q - 1)); }
};
__device__ inline void s4_pair(int64_t p, int64_t &g1, int64_t &g2) {
    g2 = (int64_t)((sqrt(8.0 * (double)p + 1.0) - 1.0) * 0.5);
    while (s4_pairs_below(g2) > p) --g2;
    while (s4_pairs_below(g2 + 1) <= p) ++g2;
    g1 = p - s4_pairs_below(g2);
}

int64_t s4_doubles_host(int64_t S) { return S >= 4 ? s4_off(S, 0, s4_groups(S)) * S4_FIELDS : 0; }
int64_t s4_pairs_host(int64_t S) { return s4_pairs_below(s4_groups(S)); }
__device__ void s4_tile_table(const Ctx &c) {
    c.stats[1] = bound_items<S4Pairs>(c.S, bound_run(bound_units<S4Pairs>(c.S)), c.cum);
}
uint64_t s4_items_host(int64_t S) { return bound_items<S4Pairs>(S, bound_run(bound_units<S4Pairs>(S)), nullptr); }
size_t s4_pool_units(int64_t S) { return pool_units(s4_items_host(S), bound_run(bound_units<S4Pairs>(S)), S4_PASS); }

// The factor of pair e = (g1, g2): of its live columns in index order, G =
// R^T R, {R^-1 by rows, z = R^-T b, c - |z|^2, and the smallest pivot of a j
// that is tried with it (above 1: none)}.  The columns past S, the constant ones and, with
// g1 = g2, the second four have zero rows.
__device__ void s4_factor(const Ctx &c, int64_t e) {
    int64_t g1, g2;
    s4_pair(e, g1, g2);
    const int64_t S = c.S, nt = c.Gnt;
    const double *__restrict__ G1 = c.G1;
    constexpr int N = 2 * S4_NR;
    int64_t id[N];
    bool live[N];
#pragma unroll
    for (int m = 0; m < N; ++m) {
        const int64_t i = S4_NR * (m < S4_NR ? g1 : g2) + m % S4_NR;
        id[m] = i < S ? i : S - 1;
        live[m] = i < S && c.inv_s[id[m]] > 0.0 && (m < S4_NR || g1 != g2);
    }
    double L[N][N], Li[N][N], pg = c.cyy[0], norm = 0.0;
    bool bad = false;
    double *f = c.fac4 + e * S4_FAC;
#pragma unroll
    for (int m = 0; m < N; ++m) {
        double d = 1.0;
#pragma unroll
        for (int l = 0; l < m; ++l) {
            double s = live[m] ? G1[gidx(id[l], id[m], nt, 1, 0)] : 0.0;
#pragma unroll
            for (int q = 0; q < l; ++q) s -= L[m][q] * L[l][q];
            L[m][l] = s * Li[l][l];
            d -= L[m][l] * L[m][l];
        }
        bad |= live[m] && !(d > S3_TAU);
        Li[m][m] = live[m] && d > S3_TAU ? 1.0 / sqrt(d) : 0.0;
        double zz = Li[m][m] * c.bhat[id[m]];
#pragma unroll
        for (int l = 0; l < m; ++l) {
            double s = 0.0;
#pragma unroll
            for (int q = l; q < m; ++q) s += L[m][q] * Li[q][l];
            Li[m][l] = -Li[m][m] * s;
            zz += Li[m][l] * c.bhat[id[l]];
        }
#pragma unroll
        for (int l = 0; l <= m; ++l) {
            f[m * (m + 1) / 2 + l] = Li[m][l];
            norm += Li[m][l] * Li[m][l];
        }
        f[36 + m] = zz;
        pg -= zz * zz;
    }
    f[44] = pg;
    f[45] = bad ? 2.0 : bound_tau<N>(norm);
    f[46] = f[47] = 0.0;
}

__global__ __launch_bounds__(64) void s4_init_kernel(Ctx c) {
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    search_init_body(c, e, e == 0, 4, SUBP, JBLK, 4);
    if (e < s4_pairs_below(s4_groups(c.S))) s4_factor(c, e);
}

// One workgroup per pair, a thread per column.  Bound by the writes: 240 MB in
// 50 us at S = 600.
__global__ __launch_bounds__(256) void rec4_kernel(Ctx c) {
    const int64_t S = c.S, nt = c.Gnt;
    int64_t g1, g2;
    s4_pair(blockIdx.x, g1, g2);
    g1 = uni(g1);
    g2 = uni(g2);
    const double *__restrict__ G1 = c.G1;
    CDouble *f = cptr(c.fac4) + (s4_pairs_below(g2) + g1) * S4_FAC;
    constexpr int N = 2 * S4_NR;
    const int64_t x0 = S4_NR * g2, len = S - x0;
    for (int64_t j = x0 + threadIdx.x; j < S; j += 256) {
        double x[N], v[N], al = 0.0, zs = 0.0, p = f[44], d = 0.0, e = 0.0;
#pragma unroll
        for (int m = 0; m < N; ++m) {
            const int64_t i = S4_NR * (m < S4_NR ? g1 : g2) + m % S4_NR;
            x[m] = G1[gidx(i < S ? i : S - 1, j, nt, 1, 0)];
            v[m] = 0.0;
        }
        if (!(c.inv_s[j] > 0.0)) {
            p = d = S3_NEVER;
        } else if (f[45] > 1.0) {
            p = 0.0;
        } else if (j >= S4_NR * (g2 + 1)) {  // (a column of g2 itself leaves the pair alone)
            d = 1.0;
            e = c.bhat[j];
#pragma unroll
            for (int m = 0; m < N; ++m) {
                double s = 0.0;
#pragma unroll
                for (int l = 0; l <= m; ++l) s += f[m * (m + 1) / 2 + l] * x[l];
                v[m] = s;
                d -= s * s;
                e -= s * f[36 + m];
            }
            if (d > f[45]) {
                al = 1.0 / d;
                zs = e * al;
                p = p - e * zs;
            } else {
                p = 0.0;
            }
        }
        double *o = c.rec4 + s4_off(S, g1, g2) * S4_FIELDS + (j - x0);
#pragma unroll
        for (int m = 0; m < N; ++m) o[m * len] = v[m];
        o += N * len;
        o[BF_AL * len] = al;
        o[BF_ZS * len] = zs;
        o[BF_P * len] = p;
        o[BF_D * len] = d;
        o[BF_E * len] = e;
    }
}

__device__ inline uint64_t s4_cand(int64_t g1, int64_t g2, int64_t j, int64_t k) {
    return ((uint64_t)g1 << 48) | ((uint64_t)g2 << 32) | ((uint64_t)j << 16) | (uint64_t)k;
}

__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(S4_WPE))) void search4_kernel(
    Ctx c, const double *__restrict__ rec, const double *__restrict__ fac, const uint64_t *__restrict__ cum,
    uint64_t t0, uint64_t t1, uint32_t wg_units, int run, int glo, int ghi) {
    __shared__ double s_g[BU * BU];
    __shared__ double s_par[SEARCH_WAVES][3][BU];
    __shared__ unsigned s_n[2];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    uint64_t *__restrict__ cands = c.s3_cands + (size_t)blockIdx.x * wg_units * S4_LANES;
    uint64_t *__restrict__ items = c.s3_rows + (size_t)blockIdx.x * wg_units * S4_ITEMS;
    if (threadIdx.x < 2) s_n[threadIdx.x] = 0;
    const int64_t S = c.S;
    const double th = fmin(theta0_of(c), theta_load(c.theta_bits)), ctot = c.cyy[0];
    const double theta_s = th * (1.0 + THETA_SLACK) + S3_SLACK * ctot, neg = -S3_ESLACK * ctot;
    S3Skip skip;
    for (uint64_t t = bound_first(t0); t < t1; t += gridDim.x) {
        S3Tile tl;
        int64_t b0, b1, g1, g2;
        bound_locate<S4Pairs>(S, cum, t, run, tl, b0, b1);
        s4_pair(b0, g1, g2);
        g1 = uni(g1) + wave;
        g2 = uni(g2);
        __syncthreads();  // the waves have left the previous item's G
        bound_load(s_g, c.G1, c.Gnt, tl);
        __syncthreads();
        for (int64_t b = b0 + wave; b < b1; b += SEARCH_WAVES, g1 += SEARCH_WAVES) {
            while (g1 > g2) g1 -= ++g2;
            if (g1 < glo || g1 > ghi) continue;
            unsigned long long mine = 0;
            int lanes = 1 << 30;
            if (!skip.skip() && th < INF && cptr(fac)[b * S4_FAC + 45] <= 1.0) {
                const int lo = S4_NR * g2 + 1 > tl.j0 ? (int)(S4_NR * g2 + 1 - tl.j0) : 0;
                bound_unit<2>(s_g, S, tl, rec + s4_off(S, g1, g2) * S4_FIELDS, S4_NR * g2, S - S4_NR * g2, lo, theta_s,
                              neg, s_par[wave], mine, lanes);
                skip.result(lanes > S4_LANES);
            }
            if (lanes > S4_LANES) {
                // the whole unit, an item per i2 and S4_DR rows with a tuple in it
                const int64_t i2 = S4_NR * g2 + lane % S4_NR, jr = tl.j0 + lane / S4_NR * S4_DR;
                const bool in = lane < S4_ITEMS && i2 > S4_NR * g1 && jr <= tl.jhi && i2 < jr + S4_DR - 1 &&
                                i2 < tl.jhi && c.inv_s[i2 < S ? i2 : S - 1] > 0.0;
                const unsigned long long m = __ballot(in);
                unsigned at = 0;
                if (lane == 0) at = atomicAdd(&s_n[1], (unsigned)__popcll(m));
                at = (unsigned)__shfl((int)at, 0);
                // (group g1, i2, first row / S4_DR, column chunk)
                if (in)
                    items[at + __popcll(m & ((1ull << lane) - 1ull))] = s4_cand(g1, i2, jr / S4_DR, tl.kcx);
                continue;
            }
            if (!lanes) continue;
            unsigned at = 0;
            if (lane == 0) at = atomicAdd(&s_n[0], (unsigned)lanes);
            at = (unsigned)__shfl((int)at, 0);
            bound_each(mine, [&](int p, int x, int k) { cands[at + p] = s4_cand(g1, g2, tl.j0 + x, tl.kb + k); });
        }
    }
    __syncthreads();
    if (threadIdx.x < 2) c.s3_count[2 * blockIdx.x + threadIdx.x] = s_n[threadIdx.x];
}

// The terms of the pair (i1, i2) in a tuple's solve: r = G[i1][i2], 1/s with
// s^2 = 1 - r^2 (0: rank deficient), z0 = b_i1, z1 = (b_i2 - r z0) / s; and
// the row of a column x against the pair: x0 = G[i1][x], x1 = (G[i2][x] - r x0) / s.
struct S4Pair {
    double r, is, z0, z1;
    __device__ S4Pair(double rr, double b1, double b2, bool valid) : r(rr), z0(b1) {
        const double s2 = 1.0 - rr * rr;
        is = valid && s2 > RANK_EPS ? 1.0 / sqrt(s2) : 0.0;
        z1 = (b2 - rr * b1) * is;
    }
};

// A tuple's record {v0, v1, 1/d_j, z_j / s_j, p} (as a D = 3 record, against
// the pair); p = NaN (fails every comparison) where the triple is rank
// deficient.
__device__ inline void s4_record(const S4Pair &q, double g1j, double g2j, double bj, double ctot, double (&o)[5]) {
    const double a0 = g1j, a1 = (g2j - q.r * g1j) * q.is;
    const double d = 1.0 - a0 * a0 - a1 * a1;
    const bool ok = q.is > 0.0 && d > RANK_EPS;
    const double id = ok ? 1.0 / d : 0.0;
    const double ee = bj - a0 * q.z0 - a1 * q.z1;
    o[0] = a0;
    o[1] = a1;
    o[2] = id;
    o[3] = ee * id;
    o[4] = ok ? ctot - q.z0 * q.z0 - q.z1 * q.z1 - ee * o[3] : __builtin_nan("");
}

// 64 candidates, one per lane: (group g1, group g2, j, k) whose bound passed.
// Each lane scores the sixteen tuples.
__device__ __forceinline__ void s4_candidates(const Ctx &c, const SearchArgs &a, bool have, uint64_t key, double *Ls,
                                              uint64_t *Lr, double theta0, double &theta_pub, unsigned &offered) {
    const int KP = a.KP;
    const int64_t S = c.S, nt = c.Gnt;
    const double *__restrict__ G1 = c.G1;
    const double ctot = c.cyy[0];
    const int64_t g1 = have ? (int64_t)(key >> 48) : 0, g2 = have ? (int64_t)((key >> 32) & 0xFFFF) : 0;
    const int64_t j = have ? (int64_t)((key >> 16) & 0xFFFF) : 2, k = have ? (int64_t)(key & 0xFFFF) : 3;
    double th = fmin(theta0, theta_load(c.theta_bits));
    th = fmin(th, Ls[KP - 1]);
    const double theta_f = th < INF ? th * (1.0 + THETA_SLACK) : INF;
    const double gjk = G1[gidx(j, k, nt, 1, 0)], bj = c.bhat[j], bk = c.bhat[k];
    have = have && c.inv_s[j] > 0.0 && c.inv_s[k] > 0.0;
    double gj[S4_NR], gk[S4_NR], b1[S4_NR];
    bool lv[S4_NR];
#pragma unroll
    for (int r = 0; r < S4_NR; ++r) {
        const int64_t i = S4_NR * g1 + r < S ? S4_NR * g1 + r : S - 1;
        gj[r] = G1[gidx(i, j, nt, 1, 0)];
        gk[r] = G1[gidx(i, k, nt, 1, 0)];
        b1[r] = c.bhat[i];
        lv[r] = c.inv_s[i] > 0.0;
    }
    for (int y = 0; y < S4_NR; ++y) {
        const int64_t i2 = S4_NR * g2 + y, ii = i2 < S ? i2 : S - 1;
        const bool in2 = have && i2 < j && c.inv_s[ii] > 0.0;
        const double g2j = G1[gidx(ii, j, nt, 1, 0)], g2k = G1[gidx(ii, k, nt, 1, 0)], b2 = c.bhat[ii];
        double es[S4_NR];
        bool any = false;
#pragma unroll
        for (int r = 0; r < S4_NR; ++r) {
            const int64_t i1 = S4_NR * g1 + r < S ? S4_NR * g1 + r : S - 1;
            const S4Pair q(G1[gidx(i1, ii, nt, 1, 0)], b1[r], b2, in2 && S4_NR * g1 + r < i2 && lv[r]);
            double o[5];
            s4_record(q, gj[r], g2j, bj, ctot, o);
            const double w1 = (g2k - q.r * gk[r]) * q.is;
            const double u = fma(-o[1], w1, fma(-o[0], gk[r], gjk));
            const double d = fma(-o[2], u * u, 1.0 - gk[r] * gk[r] - w1 * w1);
            const double z = fma(-o[3], u, bk - gk[r] * q.z0 - w1 * q.z1);
            es[r] = (d > RANK_EPS) ? o[4] - z * z / d : INF;
            any |= es[r] <= theta_f;
        }
        if (!__ballot(any)) continue;
#pragma unroll
        for (int r = 0; r < S4_NR; ++r) {
            const int32_t tup[4] = {(int32_t)(S4_NR * g1 + r), (int32_t)i2, (int32_t)j, (int32_t)k};
            bool take = es[r] <= fmin(theta_f, Ls[KP - 1]);
            if (take && a.ranged) {
                const uint64_t lr = lex_rank(BinomTab{c.btab, c.S}, c.S, 4, tup);
                if (lr < a.r0 || lr >= a.r1) take = false;
            }
            list_insert_lanes(Ls, Lr, KP, take, pack_tuple(tup, 4), es[r], offered);
        }
    }
    const double tw = Ls[KP - 1];
    if (tw < theta_pub) {
        theta_pub = tw;
        if ((threadIdx.x & 63) == 0) theta_publish(c.theta_bits, tw);
    }
}

// A dense item: all tuples of S4_DR rows of a unit with second index i2 and
// first index in group g1.  The rows' records are built in LDS and read by all
// lanes at one address.
__device__ __forceinline__ void s4_dense(const Ctx &c, const SearchArgs &a, uint64_t item, double *Ls, uint64_t *Lr,
                                         double theta0, double &theta_pub, unsigned &offered,
                                         double (*s_r)[S4_NR][6], unsigned long long *s_q) {
    const int KP = a.KP;
    const int lane = threadIdx.x & 63;
    const int64_t S = c.S, nt = c.Gnt;
    const int64_t g1 = (int64_t)(item >> 48), i2 = (int64_t)((item >> 32) & 0xFFFF);
    const int64_t jr = (int64_t)((item >> 16) & 0xFFFF) * S4_DR, kcx = (int64_t)(item & 0xFFFF);
    const double *__restrict__ Gb = c.G1;
    const double *__restrict__ inv_s = c.inv_s;
    const double ctot = c.cyy[0];
    const int64_t k = jr / BU * BU + kcx * BU + lane, kk = k < S ? k : S - 1;
    // k-dependent part of each pair's solve
    double w0[S4_NR], w1[S4_NR], dq[S4_NR], zq[S4_NR];
    {
        const bool lk = k < S && inv_s[kk] > 0.0;
        const double bk = c.bhat[kk], x2 = Gb[gidx(i2, kk, nt, 1, 0)];
#pragma unroll
        for (int r = 0; r < S4_NR; ++r) {
            const bool pin = S4_NR * g1 + r < i2;
            const int64_t i1 = pin ? S4_NR * g1 + r : i2;  // a void pair reads valid memory and never passes
            const S4Pair q(Gb[gidx(i1, i2, nt, 1, 0)], c.bhat[i1], c.bhat[i2], pin && inv_s[i1] > 0.0);
            const double a0 = Gb[gidx(i1, kk, nt, 1, 0)], c0 = (x2 - q.r * a0) * q.is;
            w0[r] = a0;
            w1[r] = c0;
            // a lane past S, a constant column or a void pair never passes
            dq[r] = q.is > 0.0 && lk ? 1.0 - a0 * a0 - c0 * c0 : __builtin_nan("");
            zq[r] = bk - a0 * q.z0 - c0 * q.z1;
        }
    }
    {
        const int64_t jhi = jr + S4_DR - 1 < S - 2 ? jr + S4_DR - 1 : S - 2;
        const int64_t jlo = jr > i2 + 1 ? jr : i2 + 1;
        const int nr = (int)(jhi - jlo + 1);
        double th = fmin(theta0, theta_load(c.theta_bits));
        th = fmin(th, Ls[KP - 1]);
        const double theta_f = th < INF ? th * (1.0 + THETA_SLACK) : INF;
        __atomic_signal_fence(__ATOMIC_SEQ_CST);
        __builtin_amdgcn_wave_barrier();
        for (int e = lane; e < S4_DR * S4_NR; e += 64) {
            const int x = e % S4_DR, r = e / S4_DR;
            const int64_t j = x < nr ? jlo + x : jlo + nr - 1;
            const bool pin = S4_NR * g1 + r < i2;
            const int64_t i1 = pin ? S4_NR * g1 + r : i2;
            const S4Pair q(Gb[gidx(i1, i2, nt, 1, 0)], c.bhat[i1], c.bhat[i2],
                           pin && inv_s[i1] > 0.0 && inv_s[j] > 0.0);
            double o[5];
            s4_record(q, Gb[gidx(i1, j, nt, 1, 0)], Gb[gidx(i2, j, nt, 1, 0)], c.bhat[j], ctot, o);
#pragma unroll
            for (int z = 0; z < 5; ++z) s_r[x][r][z] = o[z];
        }
        __atomic_signal_fence(__ATOMIC_SEQ_CST);
        __builtin_amdgcn_wave_barrier();
        unsigned rows = 0;
        for (int x = 0; x < nr; ++x) {
            const int64_t j = jlo + x;
            const double gx = Gb[gidx(j, kk, nt, 1, 0)];
            unsigned long long m = 0;
#pragma unroll
            for (int r = 0; r < S4_NR; ++r) {
                const double v0 = s_r[x][r][0], v1 = s_r[x][r][1], al = s_r[x][r][2], zs = s_r[x][r][3];
                const double pi = s_r[x][r][4] - theta_f;
                const double u = fma(-v1, w1[r], fma(-v0, w0[r], gx));
                const double d = fma(-al, u * u, dq[r]);
                const double z = fma(-zs, u, zq[r]);
                m |= __ballot(z * z >= pi * d);
            }
            m &= __ballot(k > j);
            if (m) {
                if (lane == 0) s_q[x] = m;
                rows |= 1u << x;
            }
        }
        __atomic_signal_fence(__ATOMIC_SEQ_CST);
        __builtin_amdgcn_wave_barrier();
        // exact scoring of the flagged rows: the same terms, a true division,
        // the rank test and the current bound
        auto pick = [&](const double (&arr)[S4_NR], int r) {
            double v = arr[0];
#pragma unroll
            for (int q = 1; q < S4_NR; ++q)
                if (q == r) v = arr[q];
            return v;
        };
        while (rows) {
            const int x = __builtin_ctz(rows);
            rows &= rows - 1;
            const int64_t j = jlo + x;
            const unsigned long long fm = s_q[x];
            const double gx = Gb[gidx(j, kk, nt, 1, 0)];
            for (int r = 0; r < S4_NR; ++r) {
                const double v0 = s_r[x][r][0], v1 = s_r[x][r][1], al = s_r[x][r][2], zs = s_r[x][r][3];
                const double p = s_r[x][r][4];
                const double u = fma(-v1, pick(w1, r), fma(-v0, pick(w0, r), gx));
                const double d = fma(-al, u * u, pick(dq, r));
                const double z = fma(-zs, u, pick(zq, r));
                const int32_t tup[4] = {(int32_t)(S4_NR * g1 + r), (int32_t)i2, (int32_t)j, (int32_t)k};
                const double es = (d > RANK_EPS) ? p - z * z / d : INF;
                bool take = ((fm >> lane) & 1ull) && k < S && es <= fmin(theta_f, Ls[KP - 1]);
                if (take && a.ranged) {
                    const uint64_t lr = lex_rank(BinomTab{c.btab, c.S}, c.S, 4, tup);
                    if (lr < a.r0 || lr >= a.r1) take = false;
                }
                list_insert_lanes(Ls, Lr, KP, take, take ? pack_tuple(tup, 4) : 0, es, offered);
            }
        }
        const double tw = Ls[KP - 1];
        if (tw < theta_pub) {
            theta_pub = tw;
            if (lane == 0) theta_publish(c.theta_bits, tw);
        }
    }
}

// Scores the pools, as s3_eval_kernel does.
constexpr int S4E_WPE = 3;
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(S4E_WPE))) void s4_eval_kernel(Ctx c, SearchArgs a, uint32_t nseg, uint32_t wg_units, int resume) {
    extern __shared__ double smem[];
    __shared__ double s_r[SEARCH_WAVES][S4_DR][S4_NR][6];
    __shared__ unsigned long long s_q[SEARCH_WAVES][S4_DR];
    __shared__ unsigned long long s_w[2][SEARCH_WAVES];
    const int KP = a.KP;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    double *Ls = smem + (size_t)wave * KP * 2;
    uint64_t *Lr = reinterpret_cast<uint64_t *>(Ls + KP);
    uint64_t *first[2];
    first[0] = reinterpret_cast<uint64_t *>(smem + (size_t)SEARCH_WAVES * KP * 2);
    first[1] = first[0] + nseg + 1;
    const int64_t gw = (int64_t)blockIdx.x * SEARCH_WAVES + wave;
    const uint64_t nw = (uint64_t)gridDim.x * SEARCH_WAVES;
    if (resume) {
        list_load(Ls, Lr, c.list_sse + gw * KP, c.list_rank + gw * KP, KP);
    } else {
        for (int m = lane; m < KP; m += 64) {
            Ls[m] = INF;
            Lr[m] = ~0ull;
        }
    }
    pool_scan(c.s3_count, nseg, first, s_w);
    const uint64_t ncand = uni(first[0][nseg]), nitem = uni(first[1][nseg]);
    const double theta0 = theta0_of(c);
    double theta_pub = INF;
    unsigned offered = 0;
    // the last waves take the first candidates: the first ones get the items
    for (uint64_t b = nw - 1 - (uint64_t)gw; b * 64 < ncand; b += nw) {
        const uint64_t e = b * 64 + lane;
        const bool in = e < ncand;
        uint64_t key = 0;
        if (in) {
            const uint32_t s = pool_segment(first[0], nseg, e);
            key = c.s3_cands[(size_t)s * wg_units * S4_LANES + (e - first[0][s])];
        }
        s4_candidates(c, a, in, key, Ls, Lr, theta0, theta_pub, offered);
    }
    // the items round-robin: consecutive ones lie on different waves
    for (uint64_t e = (uint64_t)gw; e < nitem; e += nw) {
        const uint32_t s = pool_segment(first[1], nseg, e);
        const uint64_t it = uni(c.s3_rows[(size_t)s * wg_units * S4_ITEMS + (e - first[1][s])]);
        s4_dense(c, a, it, Ls, Lr, theta0, theta_pub, offered, s_r[wave], s_q[wave]);
    }
    if (lane == 0 && offered) atomicAdd(c.cand_counter, offered);
    list_store(c.list_sse + gw * KP, c.list_rank + gw * KP, Ls, Lr, KP);
}

// ------------------------------------------------------- D = 2, one task
// A tuple (j, k) costs one element of G and six FP64 instructions: z = b_k -
// g b_j, d = 1 - g^2, pass iff z^2 >= (p_j - theta) d, p_j = c - b_j^2 (the
// arithmetic of search_kernel).  A workgroup takes one 64 x 64 tile of G at a
// time, a wave 16 of its rows, a lane a column: the upper triangle is read
// once, in whole lines, 8 KB in flight a wave.  Bound by HBM once G leaves
// the caches (10 GB at S = 50,000: 2570 us, now 1890), by latency below (S = 200:
// 42 us, now 13; S = 4096: 171, now 21): search_kernel has S / 64 work items at
// D = 2, each a row
// block against all columns, and a quarter of its registers in use.
constexpr int S2_ROWS = 16;
__global__ __launch_bounds__(256) void search2_kernel(Ctx c, SearchArgs a, int64_t ntiles) {
    extern __shared__ double smem[];
    const int KP = a.KP;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    double *Ls = smem + (size_t)wave * KP * 2;
    uint64_t *Lr = reinterpret_cast<uint64_t *>(Ls + KP);
    for (int m = lane; m < KP; m += 64) {
        Ls[m] = INF;
        Lr[m] = ~0ull;
    }
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    __builtin_amdgcn_wave_barrier();
    const int64_t S = c.S, nt = c.Gnt;
    const double theta0 = theta0_of(c), ctot = c.cyy[0];
    double theta_pub = INF;
    unsigned offered = 0;
    for (int64_t t = blockIdx.x; t < ntiles; t += gridDim.x) {
        int64_t ta, tb;  // tile (ta, tb), ta <= tb
        s4_pair(t, ta, tb);
        ta = uni(ta);
        tb = uni(tb);
        const int64_t j0 = ta * 64 + wave * S2_ROWS, k = tb * 64 + lane;
        if (j0 >= S) continue;
        const double *__restrict__ G = c.G + ((ta * nt + tb) << 12) + wave * S2_ROWS * 64 + lane;
        double g[S2_ROWS];
#pragma unroll
        for (int x = 0; x < S2_ROWS; ++x) g[x] = G[x * 64];
        const int64_t kk = k < S ? k : S - 1;
        const bool kv = k < S && c.inv_s[kk] > 0.0;
        const double bk = c.bhat[kk];
        const double th = fmin(fmin(theta0, theta_load(c.theta_bits)), Ls[KP - 1]);
        const double theta_f = th < INF ? th * (1.0 + THETA_SLACK) : INF;
#pragma unroll
        for (int x = 0; x < S2_ROWS; ++x) {
            const int64_t j = j0 + x, jj = j < S ? j : S - 1;
            const double bj = cptr(c.bhat)[jj];
            const bool jv = j < S && cptr(c.inv_s)[jj] > 0.0;
            const double p = ctot - bj * bj;
            const double d = 1.0 - g[x] * g[x], z = fma(-bj, g[x], bk);
            if (!__ballot(jv && kv && k > j && z * z >= (p - theta_f) * d)) continue;
            const int32_t tup[2] = {(int32_t)j, (int32_t)k};
            const double es = (d > RANK_EPS) ? p - (z * z) / d : INF;
            bool take = jv && kv && k > j && z * z >= (p - theta_f) * d && es <= fmin(theta_f, Ls[KP - 1]);
            if (take && a.ranged) {
                const uint64_t lr = lex_rank(BinomTab{c.btab, c.S}, c.S, 2, tup);
                if (lr < a.r0 || lr >= a.r1) take = false;
            }
            list_insert_lanes(Ls, Lr, KP, take, take ? pack_tuple(tup, 2) : 0, es, offered);
        }
        const double tw = Ls[KP - 1];
        if (tw < theta_pub) {
            theta_pub = tw;
            if (lane == 0) theta_publish(c.theta_bits, tw);
        }
    }
    if (lane == 0 && offered) atomicAdd(c.cand_counter, offered);
    const int64_t gw = (int64_t)blockIdx.x * SEARCH_WAVES + wave;
    list_store(c.list_sse + gw * KP, c.list_rank + gw * KP, Ls, Lr, KP);
}

// D = 1: every feature is a tuple; SSE = sum_t (c_t - b_t^2) over full-rank columns.
__global__ __launch_bounds__(256) void search_d1_kernel(Ctx c, SearchArgs a) {
    extern __shared__ double smem[];
    const int KP = a.KP;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    double *Ls = smem + (size_t)wave * KP * 2;
    uint64_t *Lr = reinterpret_cast<uint64_t *>(Ls + KP);
    for (int m = lane; m < KP; m += 64) {
        Ls[m] = INF;
        Lr[m] = ~0ull;
    }
    const int64_t gw = (int64_t)blockIdx.x * SEARCH_WAVES + wave;
    const int64_t nw = (int64_t)gridDim.x * SEARCH_WAVES;
    for (int64_t kb = gw * 64; kb < c.S; kb += nw * 64) {
        const int64_t k = kb + lane;
        double s = INF;
        if (k < c.S) {
            s = 0.0;
            for (int t = 0; t < c.T; ++t) {
                if (!(Gat(c, k, k, t) == 1.0)) {
                    s = INF;
                    break;
                }
                const double b = c.bhat[k * c.TP + t];
                s += c.cyy[t] - b * b;
            }
            if (a.ranged && ((uint64_t)k < a.r0 || (uint64_t)k >= a.r1)) s = INF;
        }
        unsigned offered = 0;
        list_insert_lanes(Ls, Lr, KP, s < INF && s <= Ls[KP - 1], (uint64_t)k, s, offered);
    }
    list_store(c.list_sse + gw * KP, c.list_rank + gw * KP, Ls, Lr, KP);
}

// ------------------------------------------------- prefix-list evaluation
// Exact evaluation driven by a list of (D-1)-prefixes: every tuple P + {k}
// (k not in P) is scored by ne_sse on its sorted indices, so a tuple reached
// from several prefixes of the list gets bitwise the same SSE and key.

// Sorted tuple P + {k} (P sorted, k not in P); returns false if k is in P.
template <int M>
__device__ inline bool extend_sorted(const int32_t *P, int32_t k, int32_t *tup) {
    int n = 0;
    bool placed = false, dup = false;
#pragma unroll
    for (int m = 0; m < M; ++m) {
        dup |= P[m] == k;
        if (!placed && k < P[m]) {
            tup[n++] = k;
            placed = true;
        }
        tup[n++] = P[m];
    }
    if (!placed) tup[n] = k;
    return !dup;
}

// Reads prefix p (M indices) and checks it: strictly increasing, in [0, S).
template <int M>
__device__ inline bool load_prefix(const Ctx &c, const int32_t *pre, int64_t p, int32_t *P) {
    bool ok = true;
#pragma unroll
    for (int m = 0; m < M; ++m) {
        P[m] = pre[p * M + m];
        ok &= P[m] >= 0 && P[m] < c.S && (m == 0 || P[m] > P[m - 1]);
    }
    return ok;
}

// best[p] = min over k not in P of SSE(P + {k}); +inf if no extension is
// full rank, NaN for a malformed prefix.  One wavefront per prefix.
template <int M>
__global__ __launch_bounds__(256) void prefix_best_kernel(Ctx c, const int32_t *__restrict__ pre, int64_t n,
                                                          double *__restrict__ best) {
    const int lane = threadIdx.x & 63;
    const int64_t nw = (int64_t)gridDim.x * 4;
    for (int64_t p = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); p < n; p += nw) {
        int32_t P[M];
        const bool ok = load_prefix<M>(c, pre, p, P);
        double mn = INF;
        if (ok)
            for (int64_t k = lane; k < c.S; k += 64) {
                int32_t tup[M + 1];
                if (extend_sorted<M>(P, (int32_t)k, tup)) mn = fmin(mn, ne_sse_t<M + 1>(c, tup));
            }
        for (int o = 32; o >= 1; o >>= 1) mn = fmin(mn, __shfl_xor(mn, o));
        if (lane == 0) best[p] = ok ? mn : __builtin_nan("");
    }
}

// Initialisation of a prefix-list search: the per-search state, and an empty
// pool without a bound.
__global__ __launch_bounds__(256) void list_init_kernel(Ctx c) {
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    search_init_body(c, e, e == 0, 2, 1, JBLK, 0);
    if (e < PRE_BINS) c.pre->hist[e] = 0;
    if (e == 0) {
        c.pre->done[0] = 0;
        c.pre->theta0 = INF;
    }
}

// One task: an upper bound of the KP-th best SSE over the list's extensions,
// from the pool of tuples P + {k} with k behind P's last index, P among the
// first LIST_POOL rows and not a repeat of an earlier one (so the pool's
// tuples are distinct).  A tuple counts if the product of its pivots clears
// RANK_EPS (a pivot is at most 1, so that is the full-rank test in any order
// of the columns), at its incremental SSE plus the slack of list_search_kernel's
// filter.  Without the bound every wave filled a list of its own first: at 895
// prefixes, S = 600 the search took 198 us and the merge of its lists 267 us.
constexpr int LIST_POOL = 4096;
template <int M>
__global__ __launch_bounds__(256) void list_pool_kernel(Ctx c, const int32_t *__restrict__ pre, int64_t n) {
    constexpr int BPT = PRE_BINS / 256;
    __shared__ unsigned h[PRE_BINS];
    __shared__ unsigned wsum[4];
    __shared__ int s_last;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t p = (int64_t)blockIdx.x * 4 + wave;
    const int64_t base = pool_base(c.cyy[0]);
    for (int b = tid; b < PRE_BINS; b += 256) h[b] = 0;
    __syncthreads();
    int32_t P[M];
    if (p < n && load_prefix<M>(c, pre, p, P)) {
        bool fresh = true;
        for (int64_t o = lane; o < p; o += 64) {
            bool same = true;
#pragma unroll
            for (int m = 0; m < M; ++m) same &= pre[o * M + m] == P[m];
            fresh &= !same;
        }
        double L[M][M], z[M], pp = c.cyy[0], det = 1.0;
#pragma unroll
        for (int a = 0; a < M; ++a) {
#pragma unroll
            for (int b2 = 0; b2 < a; ++b2) {
                double v = Gat(c, P[a], P[b2], 0);
#pragma unroll
                for (int l = 0; l < b2; ++l) v -= L[a][l] * L[b2][l];
                L[a][b2] = v / L[b2][b2];
            }
            double d = Gat(c, P[a], P[a], 0);
#pragma unroll
            for (int l = 0; l < a; ++l) d -= L[a][l] * L[a][l];
            det *= d;
            L[a][a] = sqrt(fmax(d, RANK_EPS));
            double zz = c.bhat[(int64_t)P[a] * c.TP];
#pragma unroll
            for (int l = 0; l < a; ++l) zz -= L[a][l] * z[l];
            z[a] = zz / L[a][a];
            pp -= z[a] * z[a];
        }
        if (!__any(!fresh) && det > 10.0 * RANK_EPS)
            for (int64_t k = P[M - 1] + 1 + lane; k < c.S; k += 64) {
                double w[M], d = Gat(c, k, k, 0), zeta = c.bhat[k * c.TP];
#pragma unroll
                for (int a = 0; a < M; ++a) {
                    double v = Gat(c, P[a], k, 0);
#pragma unroll
                    for (int l = 0; l < a; ++l) v -= L[a][l] * w[l];
                    w[a] = v / L[a][a];
                    d -= w[a] * w[a];
                    zeta -= w[a] * z[a];
                }
                if (!(det * d > 10.0 * RANK_EPS)) continue;
                const double s = fmax(pp - zeta * zeta / d, 0.0) * (1.0 + 1e-8) + 1e-12 * c.cyy[0];
                atomicAdd(&h[pool_bin(s, base)], 1u);
            }
    }
    __syncthreads();
    auto scan = [&](const unsigned (&v)[BPT]) {
        unsigned own = 0;
#pragma unroll
        for (int b = 0; b < BPT; ++b) own += v[b];
        unsigned incl = own;
        for (int o = 1; o < 64; o <<= 1) {
            const unsigned y = __shfl_up(incl, o);
            if (lane >= o) incl += y;
        }
        if (lane == 63) wsum[wave] = incl;
        __syncthreads();
        unsigned before = incl - own;
        for (int w = 0; w < wave; ++w) before += wsum[w];
        return before;
    };
    // bins past the workgroup's own KP smallest cannot hold the pool's KP-th
    unsigned v[BPT];
#pragma unroll
    for (int b = 0; b < BPT; ++b) v[b] = h[tid * BPT + b];
    unsigned before = scan(v);
#pragma unroll
    for (int b = 0; b < BPT; ++b) {
        if (v[b] && before < (unsigned)c.KP) atomicAdd(&c.pre->hist[tid * BPT + b], v[b]);
        before += v[b];
    }
    __threadfence();
    __syncthreads();
    if (tid == 0) s_last = atomicAdd(&c.pre->done[0], 1u) == gridDim.x - 1u;
    __syncthreads();
    if (!s_last) return;
    __threadfence();
#pragma unroll
    for (int b = 0; b < BPT; ++b)
        v[b] = __hip_atomic_load(&c.pre->hist[tid * BPT + b], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    before = scan(v);
#pragma unroll
    for (int b = 0; b < BPT; ++b) {
        if (before < (unsigned)c.KP && before + v[b] >= (unsigned)c.KP) c.pre->theta0 = pool_edge(tid * BPT + b, base);
        before += v[b];
    }
}

// Top-k candidates over the extensions of a prefix list: persistent waves
// take prefixes in turn, lanes run over k, and each wave keeps its sorted
// list as in the exhaustive search (bound: own KP-th entry and the
// device-wide bound).  The lists feed the same merge, re-score and final
// ordering (merge removes tuples that several prefixes produced).
// (M = 3: registers for three waves per SIMD, n = 60,000: 577 us at two, 521 at three)
template <int M>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(M == 3 ? 3 : 1))) void list_search_kernel(
    Ctx c, const int32_t *__restrict__ pre, int64_t n) {
    extern __shared__ double smem[];
    const int KP = c.KP;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    double *Ls = smem + (size_t)wave * KP * 2;
    uint64_t *Lr = reinterpret_cast<uint64_t *>(Ls + KP);
    for (int m = lane; m < KP; m += 64) {
        Ls[m] = INF;
        Lr[m] = ~0ull;
    }
    double theta_pub = INF;
    int fill = 0;  // entries appended (KP: the list is sorted)
    unsigned offered = 0;  // tuples offered to the list (diagnostics; one atomic per wave)
    const int64_t gw = (int64_t)blockIdx.x * SEARCH_WAVES + wave;
    const int64_t nw = (int64_t)gridDim.x * SEARCH_WAVES;
    for (int64_t p = gw; p < n; p += nw) {
        int32_t P[M];
        if (!load_prefix<M>(c, pre, p, P)) continue;
        // one task: the prefix's own factor (uniform) turns each extension
        // into an incremental filter (w = L^-1 G[P,k], d = G[k,k] - |w|^2,
        // SSE ~ p - zeta^2 / d); only extensions that pass it (or whose pivot
        // is too small to judge) are scored canonically
        double L[M][M], z[M], pp = 0.0;
        double gP[M][M], bP[M];  // the prefix's own correlation block and b (one task)
        bool pok = false;
        if (c.T == 1) {
            pp = c.cyy[0];
            pok = true;
#pragma unroll
            for (int a = 0; a < M; ++a) {
                bP[a] = c.bhat[(int64_t)P[a] * c.TP];
#pragma unroll
                for (int b2 = 0; b2 <= a; ++b2) gP[a][b2] = Gat(c, P[a], P[b2], 0);
            }
#pragma unroll
            for (int a = 0; a < M; ++a) {
#pragma unroll
                for (int b2 = 0; b2 < a; ++b2) {
                    double v = gP[a][b2];
#pragma unroll
                    for (int l = 0; l < b2; ++l) v -= L[a][l] * L[b2][l];
                    L[a][b2] = v / L[b2][b2];
                }
                double d = gP[a][a];
#pragma unroll
                for (int l = 0; l < a; ++l) d -= L[a][l] * L[a][l];
                pok &= d > RANK_EPS;
                L[a][a] = sqrt(fmax(d, RANK_EPS));
                double zz = bP[a];
#pragma unroll
                for (int l = 0; l < a; ++l) zz -= L[a][l] * z[l];
                z[a] = zz / L[a][a];
                pp -= z[a] * z[a];
            }
        }
        // the device-wide bound is read once per prefix (a memory round trip)
        const double th_dev = fmin(theta_load(c.theta_bits), theta0_of(c));
        for (int64_t kb = 0; kb < c.S; kb += 64) {
            const int64_t k = kb + lane;
            double sse = INF;
            uint64_t key = ~0ull;
            int32_t tup[M + 1];
            const double th = fmin(Ls[KP - 1], th_dev);
            bool score = k < c.S && extend_sorted<M>(P, (int32_t)k, tup);
            if (score && c.T == 1) {
                const int64_t kc = k;
                double gk[M];
#pragma unroll
                for (int a = 0; a < M; ++a) gk[a] = Gat(c, P[a], kc, 0);
                const double gkk = Gat(c, kc, kc, 0), bk = c.bhat[kc * c.TP];
                if (pok) {
                    double w[M], ww = 0.0, wz = 0.0;
#pragma unroll
                    for (int a = 0; a < M; ++a) {
                        double v = gk[a];
#pragma unroll
                        for (int l = 0; l < a; ++l) v -= L[a][l] * w[l];
                        w[a] = v / L[a][a];
                        ww += w[a] * w[a];
                        wz += w[a] * z[a];
                    }
                    const double d = gkk - ww;
                    const double zeta = bk - wz;
                    const double inc = d > 1e3 * RANK_EPS ? pp - zeta * zeta / d : -INF;
                    score = inc <= (th < INF ? th * (1.0 + 1e-8) + 1e-12 * c.cyy[0] : INF);
                }
                // (a tiny pivot in the prefix's own order says nothing certain about
                // the tuple's sorted order: such extensions are scored canonically)
                if (score) {
                    // canonical: the tuple's block in sorted-index order, from the
                    // values already loaded (G is bitwise symmetric)
                    int pos = 0;
#pragma unroll
                    for (int a = 0; a < M; ++a) pos += P[a] < kc;
                    // pos differs across lanes: the prefix values are picked by
                    // selects over constant indexes, so gP, bP and gk stay in
                    // registers (an indexed read would put them in scratch memory)
                    // (each candidate passes through an empty asm, so the
                    // compiler cannot fold the selects back into an indexed load)
                    auto opaque = [](double x) {
                        __asm__ volatile("" : "+v"(x));
                        return x;
                    };
                    auto pick1 = [&](const double (&arr)[M], int a) {
                        double r = opaque(arr[0]);
#pragma unroll
                        for (int q = 1; q < M; ++q) r = a == q ? opaque(arr[q]) : r;
                        return r;
                    };
                    auto pickg = [&](int a, int b) {  // b <= a (lower triangle)
                        double r = opaque(gP[0][0]);
#pragma unroll
                        for (int q = 1; q < M; ++q)
#pragma unroll
                            for (int q2 = 0; q2 <= q; ++q2) r = (a == q && b == q2) ? opaque(gP[q][q2]) : r;
                        return r;
                    };
                    double g4[M + 1][M + 1], b4[M + 1];
#pragma unroll
                    for (int u = 0; u <= M; ++u) {
                        const int au = u < pos ? u : u - 1;  // prefix slot of tuple slot u (u != pos)
                        b4[u] = u == pos ? bk : pick1(bP, au);
#pragma unroll
                        for (int v2 = 0; v2 <= u; ++v2) {
                            const int av = v2 < pos ? v2 : v2 - 1;
                            double val;
                            if (u == pos && v2 == pos) val = gkk;
                            else if (u == pos) val = pick1(gk, av);
                            else if (v2 == pos) val = pick1(gk, au);
                            else val = pickg(au, av);
                            g4[u][v2] = val;
                        }
                    }
                    bool ok = true;
                    const double v = ne_sse_core<M + 1>(g4, b4, c.cyy[0], ok);
                    sse = ok ? v : INF;
                    key = pack_tuple(tup, M + 1);
                }
            } else if (score) {
                sse = ne_sse_t<M + 1>(c, tup);
                key = pack_tuple(tup, M + 1);
            }
            unsigned long long m = __ballot(sse < INF && sse <= th);
            offered += (unsigned)__popcll(m);
            if (fill < KP && m) {
                // the list is not full: append (one slot per passing lane), and
                // sort once it is and drop the copies of a tuple, so that a full
                // list holds KP tuples and its last entry bounds the KP-th best;
                // from there on the entries are inserted
                const int rank = __popcll(m & ((1ull << lane) - 1ull));
                const int nfit = min(__popcll(m), KP - fill);
                const bool mine = ((m >> lane) & 1ull) && rank < nfit;
                if (mine) {
                    Ls[fill + rank] = sse;
                    Lr[fill + rank] = key;
                }
                __atomic_signal_fence(__ATOMIC_SEQ_CST);
                __builtin_amdgcn_wave_barrier();
                m &= ~__ballot(mine);
                fill += nfit;
                if (fill == KP) {
                    wave_sort_list(Ls, Lr, KP);
                    wave_drop_copies(Ls, Lr, KP);
                }
            }
            while (m) {
                const int src = __ffsll((long long)m) - 1;
                m &= m - 1;
                list_insert(Ls, Lr, KP, __shfl(sse, src), (uint64_t)__shfl((long long)key, src));
            }
            const double tw = Ls[KP - 1];
            if (tw < theta_pub) {
                theta_pub = tw;
                if (lane == 0) theta_publish(c.theta_bits, tw);
            }
        }
    }
    if (fill < KP) wave_sort_list(Ls, Lr, KP);  // unused slots hold +inf and sort last
    if (lane == 0 && offered) atomicAdd(c.cand_counter, offered);
    list_store(c.list_sse + gw * KP, c.list_rank + gw * KP, Ls, Lr, KP);
}

// Per-prefix features for the learned proposal (FP32, PROP_NF per prefix),
// dimension-agnostic so that a model trained on one prefix length applies
// to another: with r_i^2 = b_i^2 / c (squared correlation with y) and the
// prefix's own fit R^2 = 1 - SSE(P) / c (sums over tasks):
//   R^2, max r_i^2, min r_i^2, mean r_i^2, max |G_ij|, mean |G_ij|,
//   R^2 - max r_i^2 (gain over the best single feature), 1 / M.
// One thread per prefix.
template <int M>
__device__ void prefix_features(const Ctx &c, const int32_t *P, float *o) {
    double ctot = 0.0;
    for (int t = 0; t < c.T; ++t) ctot += c.cyy[t];
    const double ic = ctot > 0.0 ? 1.0 / ctot : 0.0;
    double r2max = 0.0, r2min = INF, r2sum = 0.0, gmax = 0.0, gsum = 0.0;
#pragma unroll
    for (int m = 0; m < M; ++m) {
        double e = 0.0;
        for (int t = 0; t < c.T; ++t) {
            const double b = c.bhat[(int64_t)P[m] * c.TP + t];
            e += b * b;
        }
        e *= ic;
        r2max = fmax(r2max, e);
        r2min = fmin(r2min, e);
        r2sum += e;
#pragma unroll
        for (int l = 0; l < m; ++l) {
            double g = 0.0;
            for (int t = 0; t < c.T; ++t) g = fmax(g, fabs(Gat(c, P[m], P[l], t)));
            gmax = fmax(gmax, g);
            gsum += g;
        }
    }
    const double sse = ne_sse_t<M>(c, P);
    const double R2 = sse < INF ? 1.0 - sse * ic : 0.0;
    o[0] = (float)R2;
    o[1] = (float)r2max;
    o[2] = (float)r2min;
    o[3] = (float)(r2sum / M);
    o[4] = (float)gmax;
    o[5] = (float)(M > 1 ? gsum / (M * (M - 1) / 2) : 0.0);
    o[6] = (float)(R2 - r2max);
    o[7] = (float)(1.0 / M);
}

// Features of the prefixes of a list (one thread each).
template <int M>
__global__ __launch_bounds__(256) void prefix_features_kernel(Ctx c, const int32_t *__restrict__ pre, int64_t n,
                                                              float *__restrict__ out) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    int32_t P[M];
    float *o = out + p * PROP_NF;
    if (!load_prefix<M>(c, pre, p, P)) {
        for (int f = 0; f < PROP_NF; ++f) o[f] = __builtin_nanf("");
        return;
    }
    prefix_features<M>(c, P, o);
}

// Features of the M-subsets of {0..S-1} with colexicographic ranks
// r0 .. r0 + n - 1 (no prefix array needed for a full sweep).
template <int M>
__global__ __launch_bounds__(256) void prefix_features_range_kernel(Ctx c, uint64_t r0, int64_t n,
                                                                    float *__restrict__ out) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    int32_t P[M];
    colex_unrank_small(r0 + (uint64_t)p, M, c.S, P);
    prefix_features<M>(c, P, out + p * PROP_NF);
}

// ----------------------------------------------------------------- merge
// One workgroup: gather every list entry at or below the final bound, then
// select the KP smallest (SSE, rank) keys with bitonic sorts in LDS, a
// running top-KP carried across chunks when there are many.
constexpr int MERGE_THREADS = 1024;
constexpr int MERGE_CAP = 2048;
// Most candidates of a prefix-list search that are ranked by counting (others:
// MERGE_THREADS): copies have to be found first, and from here on a sort, after
// which they are neighbours, is faster (n = 500, S = 400, D = 4, 128 rows, noise,
// 900 candidates: the call 216 us, now 174; S = 60, 400 rows: 334, now 204).
constexpr int MERGE_RANK_LIST = 256;

__device__ void bitonic_sort_lds(double *ks, uint64_t *kr, int N) {
    for (int k = 2; k <= N; k <<= 1) {
        for (int j = k >> 1; j > 0; j >>= 1) {
            for (int i = threadIdx.x; i < N; i += blockDim.x) {
                const int ixj = i ^ j;
                if (ixj > i) {
                    const bool up = (i & k) == 0;
                    const double a = ks[i], b = ks[ixj];
                    const uint64_t ra = kr[i], rb = kr[ixj];
                    const bool gt = key_less(b, rb, a, ra);
                    if (gt == up) {
                        ks[i] = b;
                        ks[ixj] = a;
                        kr[i] = rb;
                        kr[ixj] = ra;
                    }
                }
            }
            __syncthreads();
        }
    }
}

// merge_compact: one wave per list.  Lists are sorted ascending, so the
// entries at or below the bound are a prefix; its length is a ballot count
// and the prefix is appended to the candidate array at an atomically
// reserved offset.  The candidate set does not depend on the append order,
// and keys are unique, so the selection below is deterministic.
__device__ inline double merge_bound(const Ctx &c, int use_pre) {
    double bound = theta_load(c.theta_bits);
    if (use_pre) bound = fmin(bound, theta0_of(c));
    return bound < INF ? bound * (1.0 + THETA_SLACK) : INF;
}

// nl_dev (may be null): the number of lists written, read on the device (at
// most nlists; the batched search writes a variable number per problem)
__global__ __launch_bounds__(MERGE_THREADS) void merge_compact_kernel(Ctx c, int nlists, int KP, int use_pre,
                                                                      const uint32_t *nl_dev) {
    const int lane = threadIdx.x & 63;
    const int64_t l = (int64_t)blockIdx.x * (MERGE_THREADS / 64) + (threadIdx.x >> 6);
    const int64_t nl = nl_dev ? (int64_t)min(*nl_dev, (uint32_t)nlists) : (int64_t)nlists;
    if (l >= nl) return;
    const double bound = merge_bound(c, use_pre);
    const double *ls = c.list_sse + l * KP;
    const uint64_t *lr = c.list_rank + l * KP;
    // sorted: the entries at or below the bound are a prefix, which ends at
    // the list's terminator at the latest
    int n = 0;
    for (int m = 0; m < KP; m += 64) {
        const double v = ls[m + lane];
        const unsigned long long b = __ballot(v < INF && v <= bound);
        if (b != ~0ull) {
            n += __builtin_ctzll(~b);  // the prefix before the first entry that fails
            break;
        }
        n += 64;
    }
    if (n == 0) return;
    unsigned base = 0;
    if (lane == 0) base = atomicAdd(c.merge_count, (unsigned)n);
    base = __shfl(base, 0);
    for (int e = lane; e < n; e += 64) {
        c.cand_sse[base + e] = ls[e];
        c.cand_rank[base + e] = lr[e];
    }
}

// Takes the later copies of equal (SSE, key) pairs out of the N sorted entries and
// closes the gaps; the places behind the others are empty.  (A prefix-list
// search can offer one tuple from several prefixes, always with bitwise the
// same SSE, so copies are adjacent after a sort.)
__device__ void drop_adjacent_duplicates(double *ks, uint64_t *kr, int N) {
    static_assert(MERGE_CAP == 2 * MERGE_THREADS, "a thread takes two entries");
    __shared__ int s_kept[MERGE_THREADS / 64];
    const int tid = threadIdx.x, lane = tid & 63, e = 2 * tid;
    double v[2] = {INF, INF};
    uint64_t r[2] = {~0ull, ~0ull};
    bool keep[2] = {false, false};
    if (e < N) {
        for (int u = 0; u < 2; ++u) {
            v[u] = ks[e + u];
            r[u] = kr[e + u];
        }
        keep[0] = v[0] < INF && !(e > 0 && v[0] == ks[e - 1] && r[0] == kr[e - 1]);
        keep[1] = v[1] < INF && !(v[1] == v[0] && r[1] == r[0]);
    }
    const bool copy = (v[0] < INF && !keep[0]) || (v[1] < INF && !keep[1]);
    if (!__syncthreads_or(copy)) return;
    const int mine = keep[0] + keep[1];
    int to = mine;  // entries kept up to this thread's
    for (int o = 1; o < 64; o <<= 1) {
        const int below = __shfl_up(to, o);
        if (lane >= o) to += below;
    }
    if (lane == 63) s_kept[tid >> 6] = to;
    __syncthreads();
    to -= mine;
    int kept = 0;
    for (int w = 0; w < MERGE_THREADS / 64; ++w) {
        if (w < (tid >> 6)) to += s_kept[w];
        kept += s_kept[w];
    }
    for (int u = 0; u < 2; ++u)
        if (keep[u]) {
            ks[to] = v[u];
            kr[to++] = r[u];
        }
    for (int i = kept + tid; i < N; i += MERGE_THREADS) {
        ks[i] = INF;
        kr[i] = ~0ull;
    }
    __syncthreads();
}

// merge_select: one workgroup selects the KP smallest (SSE, key) pairs of
// the candidates with bitonic sorts in LDS, carrying a running top-KP across
// fills of the buffer when there are many.
template <bool dedupe>  // copies of a tuple among the candidates (prefix lists)
__global__ __launch_bounds__(MERGE_THREADS) void merge_select_kernel(Ctx c, int KP, int use_pre, int nlists,
                                                                     const uint32_t *nl_dev) {
    __shared__ double ks[MERGE_CAP];
    __shared__ uint64_t kr[MERGE_CAP];
    __shared__ int fill;
    const int tid = threadIdx.x;
    const int64_t total = *c.merge_count;
    if (tid == 0) {
        const double th0 = use_pre ? theta0_of(c) : INF;
        c.stats[0] = *c.cand_counter;
        c.stats[2] = (uint64_t)__double_as_longlong(th0);
        c.stats[3] = (uint64_t)__double_as_longlong(theta_load(c.theta_bits));
    }
    // Few candidates (the usual case once the pre-pass bound is tight): the
    // KP smallest by rank counting, with no sort.  Once the later copies of a
    // tuple are empty (dedupe; otherwise there are none) the keys are distinct,
    // so the ranks (candidates ordered before each one) are too,
    // and writing candidate x at position rank(x) < KP gives the sorted
    // prefix the sorting path below returns (the candidates are finite:
    // merge_compact appends only entries below INF); positions past the
    // candidates are empty (INF, ~0) as there.
    if (total <= (dedupe ? MERGE_RANK_LIST : MERGE_THREADS)) {
        const int n = (int)total;
        bool mine = tid < n;
        if (mine) {
            ks[tid] = c.cand_sse[tid];
            kr[tid] = c.cand_rank[tid];
        }
        __syncthreads();
        int kept = n;
        if (dedupe) {
            if (mine) {
                const double v = ks[tid];
                const uint64_t r = kr[tid];
                int copy = 0;
#pragma unroll 8
                for (int i = 0; i < tid; ++i) copy |= (int)((ks[i] == v) & (kr[i] == r));
                mine = !copy;
            }
            kept = __syncthreads_count(mine);
            if (tid < n && !mine) {
                ks[tid] = INF;
                kr[tid] = ~0ull;
            }
            __syncthreads();
        }
        if (mine) {
            const double v = ks[tid];
            const uint64_t r = kr[tid];
            // (SSE, key) order written without short-circuit evaluation, so
            // that the eight steps' LDS reads are all in flight together
            auto before = [&](int i) {
                const double a = ks[i];
                const uint64_t b = kr[i];
                return (int)((a < v) | ((a == v) & (b < r)));
            };
            int rank = 0, i = 0;
            for (; i + 8 <= n; i += 8) {
#pragma unroll
                for (int u = 0; u < 8; ++u) rank += before(i + u);
            }
            for (; i < n; ++i) rank += before(i);
            if (rank < KP) {
                c.merged_sse[rank] = v;
                c.merged_rank[rank] = r;
            }
        }
        for (int i = kept + tid; i < KP; i += MERGE_THREADS) {
            c.merged_sse[i] = INF;
            c.merged_rank[i] = ~0ull;
        }
        return;
    }
    auto clear_from = [&](int at) {
        for (int i = at + tid; i < MERGE_CAP; i += MERGE_THREADS) {
            ks[i] = INF;
            kr[i] = ~0ull;
        }
    };
    auto pow2_at_least = [&](int64_t need) {
        int N = 2 * KP;
        while (N < need) N <<= 1;
        return N;
    };
    clear_from(0);
    __syncthreads();
    const int chunk = MERGE_CAP - KP;
    // Many candidates: every list is sorted, so the KP-th smallest of the
    // lists' first entries bounds the KP-th smallest candidate (those KP
    // lists each hold an entry at or below it); only candidates at or below
    // that cut can be selected.  Not with dedupe: there one tuple can head
    // several lists, and KP first entries need not be KP tuples.
    double cut = INF;
    const int64_t nl = nl_dev ? (int64_t)min(*nl_dev, (uint32_t)nlists) : (int64_t)nlists;
    if (!dedupe && total > chunk && nl >= KP) {
        for (int64_t base = 0; base < nl; base += chunk) {
            const int64_t here = nl - base < chunk ? nl - base : chunk;
            const int N = pow2_at_least(KP + here);
            for (int i = tid; i < N - KP; i += MERGE_THREADS) {
                ks[KP + i] = i < here ? c.list_sse[(base + i) * KP] : INF;
                kr[KP + i] = 0;
            }
            __syncthreads();
            bitonic_sort_lds(ks, kr, N);
        }
        cut = ks[KP - 1];
        __syncthreads();
        clear_from(0);
        if (tid == 0) fill = 0;
        __syncthreads();
    } else if (tid == 0) {
        fill = 0;
    }
    __syncthreads();
    // the candidates at or below the cut are appended behind the KP kept in
    // front; the buffer is sorted (the KP smallest kept) before it could
    // overflow.  Append order does not matter: the sort is by (SSE, key).
    auto sort_keep = [&]() {
        const int N = pow2_at_least(KP + fill);
        bitonic_sort_lds(ks, kr, N);
        if (dedupe) drop_adjacent_duplicates(ks, kr, N);
        clear_from(KP);
        if (tid == 0) fill = 0;
        __syncthreads();
    };
    for (int64_t e = 0; e < total; e += MERGE_THREADS) {
        // sort only when this batch could overflow the buffer
        const int64_t batch = total - e < MERGE_THREADS ? total - e : MERGE_THREADS;
        if (fill + batch > chunk) sort_keep();
        const int64_t i = e + tid;
        if (i < total) {
            const double v = c.cand_sse[i];
            if (v <= cut) {
                const int at = atomicAdd(&fill, 1);
                ks[KP + at] = v;
                kr[KP + at] = c.cand_rank[i];
            }
        }
        __syncthreads();
    }
    sort_keep();
    for (int i = tid; i < KP; i += MERGE_THREADS) {
        c.merged_sse[i] = ks[i];
        c.merged_rank[i] = kr[i];
    }
}

// --------------------------------------------------------------- rescore
// One workgroup per candidate: for each task, the (D x D) normal equations
// of the centred columns are accumulated straight from F in a fixed order,
// solved by Cholesky (pivot-ratio rank test), and the SSE is taken as the
// squared norm of the explicit residual y_c - X_c beta.
template <int D>
__global__ __launch_bounds__(256) void rescore_kernel(Ctx c) {
    constexpr int NACC = D * (D + 1) / 2 + D;
    __shared__ double red[NACC][4];
    __shared__ double s_beta[D];
    __shared__ int s_ok;
    const int cand = blockIdx.x;
    const int tid = threadIdx.x;
    const int W = D + 1;
    double *coef = c.resc_coef + (int64_t)cand * c.T * (c.D_max + 1);
    if (!(c.merged_sse[cand] < INF)) {
        if (tid == 0) c.resc_sse[cand] = INF;
        for (int i = tid; i < c.T * (c.D_max + 1); i += 256) coef[i] = __builtin_nan("");
        return;
    }
    int32_t tup[MAXD];
    unpack_tuple(c.merged_rank[cand], D, tup);
    if (c.T > 1) {
        // several tasks: wave w takes tasks w, w + 4, ... on its own (wave
        // sums, the small solve repeated in every lane), then the four wave
        // totals are added in a fixed order
        __shared__ double wtot[4];
        __shared__ int wok[4];
        const int lane = tid & 63, wave = tid >> 6;
        double tw = 0.0;
        bool okw = true;
        for (int t = wave; t < c.T; t += 4) {
            const int64_t r0 = c.off_dev[t], r1 = c.off_dev[t + 1];
            const double ym = c.ybar[t];
            double mu[D];
#pragma unroll
            for (int m = 0; m < D; ++m) mu[m] = c.mu[(int64_t)t * c.S + tup[m]];
            double acc[NACC];
#pragma unroll
            for (int i = 0; i < NACC; ++i) acc[i] = 0.0;
            for (int64_t i = r0 + lane; i < r1; i += 64) {
                double x[D];
#pragma unroll
                for (int m = 0; m < D; ++m) x[m] = c.F[(int64_t)tup[m] * c.n_total + i] - mu[m];
                const double yc = c.y[i] - ym;
                int e = 0;
#pragma unroll
                for (int m = 0; m < D; ++m)
#pragma unroll
                    for (int l = 0; l <= m; ++l) acc[e++] += x[m] * x[l];
#pragma unroll
                for (int m = 0; m < D; ++m) acc[e++] += x[m] * yc;
            }
#pragma unroll
            for (int i = 0; i < NACC; ++i)
                for (int o = 32; o > 0; o >>= 1) acc[i] += __shfl_xor(acc[i], o);
            double M[D][D], v[D], L[D][D], z[D], bt[D];
            int e = 0;
#pragma unroll
            for (int m = 0; m < D; ++m)
#pragma unroll
                for (int l = 0; l <= m; ++l) {
                    M[m][l] = acc[e];
                    M[l][m] = acc[e];
                    ++e;
                }
#pragma unroll
            for (int m = 0; m < D; ++m) v[m] = acc[e++];
            bool ok = true;
#pragma unroll
            for (int m = 0; m < D; ++m) {
#pragma unroll
                for (int jx = 0; jx < m; ++jx) {
                    double sm = M[m][jx];
#pragma unroll
                    for (int l = 0; l < jx; ++l) sm -= L[m][l] * L[jx][l];
                    L[m][jx] = sm / L[jx][jx];
                }
                double d = M[m][m];
#pragma unroll
                for (int l = 0; l < m; ++l) d -= L[m][l] * L[m][l];
                ok = ok && (M[m][m] > 0.0) && (d > RANK_EPS * M[m][m]);
                L[m][m] = ok ? sqrt(d) : 1.0;
            }
#pragma unroll
            for (int m = 0; m < D; ++m) {
                double sm = v[m];
#pragma unroll
                for (int l = 0; l < m; ++l) sm -= L[m][l] * z[l];
                z[m] = sm / L[m][m];
            }
#pragma unroll
            for (int m = D - 1; m >= 0; --m) {
                double sm = z[m];
#pragma unroll
                for (int l = m + 1; l < D; ++l) sm -= L[l][m] * bt[l];
                bt[m] = sm / L[m][m];
            }
            okw = okw && ok;
            double ss = 0.0;
            for (int64_t i = r0 + lane; i < r1; i += 64) {
                double er = c.y[i] - ym;
#pragma unroll
                for (int m = 0; m < D; ++m) er -= bt[m] * (c.F[(int64_t)tup[m] * c.n_total + i] - mu[m]);
                ss += er * er;
            }
            for (int o = 32; o > 0; o >>= 1) ss += __shfl_xor(ss, o);
            tw += ss;
            if (lane == 0) {
                double alpha = ym;
#pragma unroll
                for (int m = 0; m < D; ++m) alpha -= bt[m] * mu[m];
                coef[t * (c.D_max + 1)] = alpha;
#pragma unroll
                for (int m = 0; m < D; ++m) coef[t * (c.D_max + 1) + 1 + m] = bt[m];
            }
        }
        if (lane == 0) {
            wtot[wave] = tw;
            wok[wave] = okw ? 1 : 0;
        }
        __syncthreads();
        if (tid == 0) {
            const bool all = wok[0] && wok[1] && wok[2] && wok[3];
            c.resc_sse[cand] = all ? ((wtot[0] + wtot[1]) + wtot[2]) + wtot[3] : INF;
        }
        return;
    }
    double total = 0.0;
    bool valid = true;
    for (int t = 0; t < c.T; ++t) {
        const int64_t r0 = c.off_dev[t], r1 = c.off_dev[t + 1];
        const double ym = c.ybar[t];
        double mu[D];
        for (int m = 0; m < D; ++m) mu[m] = c.mu[(int64_t)t * c.S + tup[m]];
        double acc[NACC];
        for (int i = 0; i < NACC; ++i) acc[i] = 0.0;
#pragma unroll 4
        for (int64_t i = r0 + tid; i < r1; i += 256) {
            double x[D];
            for (int m = 0; m < D; ++m) x[m] = c.F[(int64_t)tup[m] * c.n_total + i] - mu[m];
            const double yc = c.y[i] - ym;
            int e = 0;
            for (int m = 0; m < D; ++m)
                for (int l = 0; l <= m; ++l) acc[e++] += x[m] * x[l];
            for (int m = 0; m < D; ++m) acc[e++] += x[m] * yc;
        }
        constexpr int nacc = NACC;
        // wave butterflies, then the 4 wave sums in a fixed order
        for (int i = 0; i < nacc; ++i) {
            double v = acc[i];
            for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
            if ((tid & 63) == 0) red[i][tid >> 6] = v;
        }
        __syncthreads();
        if (tid < nacc) red[tid][0] = ((red[tid][0] + red[tid][1]) + red[tid][2]) + red[tid][3];
        __syncthreads();
        if (tid == 0) {
            // fully unrolled (D is fixed), so the small matrices stay in registers
            double M[D][D], v[D], L[D][D], z[D], bt[D];
            int e = 0;
#pragma unroll
            for (int m = 0; m < D; ++m)
#pragma unroll
                for (int l = 0; l <= m; ++l) {
                    M[m][l] = red[e][0];
                    M[l][m] = red[e][0];
                    ++e;
                }
#pragma unroll
            for (int m = 0; m < D; ++m) v[m] = red[e++][0];
            // Cholesky; once a pivot fails the rest is computed on a unit
            // pivot and discarded
            bool ok = true;
#pragma unroll
            for (int m = 0; m < D; ++m) {
#pragma unroll
                for (int jx = 0; jx < m; ++jx) {
                    double s = M[m][jx];
#pragma unroll
                    for (int l = 0; l < jx; ++l) s -= L[m][l] * L[jx][l];
                    L[m][jx] = s / L[jx][jx];
                }
                double d = M[m][m];
#pragma unroll
                for (int l = 0; l < m; ++l) d -= L[m][l] * L[m][l];
                ok = ok && (M[m][m] > 0.0) && (d > RANK_EPS * M[m][m]);
                L[m][m] = ok ? sqrt(d) : 1.0;
            }
            if (ok) {
#pragma unroll
                for (int m = 0; m < D; ++m) {
                    double s = v[m];
#pragma unroll
                    for (int l = 0; l < m; ++l) s -= L[m][l] * z[l];
                    z[m] = s / L[m][m];
                }
#pragma unroll
                for (int m = D - 1; m >= 0; --m) {
                    double s = z[m];
#pragma unroll
                    for (int l = m + 1; l < D; ++l) s -= L[l][m] * bt[l];
                    bt[m] = s / L[m][m];
                }
#pragma unroll
                for (int m = 0; m < D; ++m) s_beta[m] = bt[m];
            }
            s_ok = ok;
        }
        __syncthreads();
        if (!s_ok) {
            valid = false;
            __syncthreads();
            break;
        }
        double beta[D];
        for (int m = 0; m < D; ++m) beta[m] = s_beta[m];
        double ss = 0.0;
#pragma unroll 4
        for (int64_t i = r0 + tid; i < r1; i += 256) {
            double e = c.y[i] - ym;
            for (int m = 0; m < D; ++m) e -= beta[m] * (c.F[(int64_t)tup[m] * c.n_total + i] - mu[m]);
            ss += e * e;
        }
        for (int o = 32; o > 0; o >>= 1) ss += __shfl_xor(ss, o);
        if ((tid & 63) == 0) red[0][tid >> 6] = ss;
        __syncthreads();
        if (tid == 0) {
            total += ((red[0][0] + red[0][1]) + red[0][2]) + red[0][3];
            double alpha = ym;
            for (int m = 0; m < D; ++m) alpha -= beta[m] * mu[m];
            coef[t * (c.D_max + 1)] = alpha;
            for (int m = 0; m < D; ++m) coef[t * (c.D_max + 1) + 1 + m] = beta[m];
        }
        __syncthreads();
    }
    if (tid == 0) c.resc_sse[cand] = valid ? total : INF;
    (void)W;
}

// ----------------------------------------------------------------- final
// Order the re-scored candidates by (SSE, rank) (rank by counting; invalid
// ones last in candidate order) and write the k best.  The KP keys are staged
// in LDS once, so each thread's count runs over LDS.
template <int D>
__global__ __launch_bounds__(1024) void final_kernel(Ctx c, int k, int KP) {
    // status words travel with the results (one readout transfer)
    if (threadIdx.x < 4) c.res_flags[threadIdx.x] = c.flags[threadIdx.x];
    __shared__ double fs[KP_MAX];
    __shared__ uint64_t fr[KP_MAX];
    __shared__ double ferr[1024 / 64];
    for (int i = threadIdx.x; i < KP; i += blockDim.x) {
        const double si = c.resc_sse[i];
        fs[i] = si < INF ? si : INF;
        fr[i] = c.merged_rank[i];
    }
    __syncthreads();
    double err = 0.0;  // largest relative gap between the ranked and the exact SSE of a result
    // rank by counting: FIN_SPLIT neighbouring lanes share one candidate and
    // count over interleaved slices of the others (short LDS chains), then
    // add their counts with shuffles
    constexpr int FIN_SPLIT = 8;
    for (int i0 = 0; i0 < KP; i0 += 1024 / FIN_SPLIT) {
        const int i = i0 + (int)(threadIdx.x / FIN_SPLIT);
        const int part = (int)(threadIdx.x % FIN_SPLIT);
        const bool have = i < KP;
        const double si = have ? fs[i] : INF;
        const uint64_t ri = have ? fr[i] : 0;
        const bool vi = si < INF;
        int pos = 0;
        if (have) {
#pragma unroll 4
            for (int j = part; j < KP; j += FIN_SPLIT) {
                const double sj = fs[j];
                const bool vj = sj < INF;
                bool before;
                if (vi && vj) before = key_less(sj, fr[j], si, ri);
                else if (vj) before = true;
                else if (vi) before = false;
                else before = j < i;
                pos += before;
            }
        }
        for (int o = 1; o < FIN_SPLIT; o <<= 1) pos += __shfl_xor(pos, o);
        if (have && part == 0 && pos < k) {
            if (vi) {
                const double a = c.merged_sse[i];
                err = fmax(err, si > 0.0 ? fabs(a - si) / si : fabs(a - si));
            }
            c.res_sse[pos] = vi ? si : INF;
            int32_t tup[MAXD];
            if (vi) unpack_tuple(ri, D, tup);
            for (int m = 0; m < D; ++m) c.res_idx[pos * D + m] = vi ? tup[m] : -1;
            for (int t = 0; t < c.T; ++t)
                for (int m = 0; m <= D; ++m)
                    c.res_coef[((int64_t)pos * c.T + t) * (D + 1) + m] =
                        vi ? c.resc_coef[((int64_t)i * c.T + t) * (c.D_max + 1) + m] : __builtin_nan("");
        }
    }
    for (int o = 32; o >= 1; o >>= 1) err = fmax(err, __shfl_xor(err, o));
    if ((threadIdx.x & 63) == 0) ferr[threadIdx.x >> 6] = err;
    __syncthreads();
    if (threadIdx.x == 0) {
        double e = 0.0;
        for (int w = 0; w < (int)(blockDim.x >> 6); ++w) e = fmax(e, ferr[w]);
        c.err_bits[1] = (unsigned long long)__double_as_longlong(e);
    }
}

// -------------------------------------------------------------- launcher
// the small per-search kernels are compiled per D (short code, no runtime
// dimension loops)
static void launch_rescore_final(const Ctx &c, int D, int k, hipStream_t st) {
    phase_begin(c, SISSO_PHASE_RESCORE, st);
    switch (D) {
        case 1: hipLaunchKernelGGL((rescore_kernel<1>), dim3(c.KP), dim3(256), 0, st, c); break;
        case 2: hipLaunchKernelGGL((rescore_kernel<2>), dim3(c.KP), dim3(256), 0, st, c); break;
        case 3: hipLaunchKernelGGL((rescore_kernel<3>), dim3(c.KP), dim3(256), 0, st, c); break;
        default: hipLaunchKernelGGL((rescore_kernel<4>), dim3(c.KP), dim3(256), 0, st, c); break;
    }
    phase_end(c, SISSO_PHASE_RESCORE, st);
    phase_begin(c, SISSO_PHASE_FINAL, st);
    switch (D) {
        case 1: hipLaunchKernelGGL((final_kernel<1>), dim3(1), dim3(1024), 0, st, c, k, c.KP); break;
        case 2: hipLaunchKernelGGL((final_kernel<2>), dim3(1), dim3(1024), 0, st, c, k, c.KP); break;
        case 3: hipLaunchKernelGGL((final_kernel<3>), dim3(1), dim3(1024), 0, st, c, k, c.KP); break;
        default: hipLaunchKernelGGL((final_kernel<4>), dim3(1), dim3(1024), 0, st, c, k, c.KP); break;
    }
    phase_end(c, SISSO_PHASE_FINAL, st);
}

template <int D>
static void launch_prepass(const Ctx &c, const SearchCall &sc, hipStream_t st, bool select = true) {
    if (select) hipLaunchKernelGGL((pre_select_kernel<D>), dim3(1), dim3(PRE_WG), 0, st, c);
    const int64_t nb = (c.S + PRE_XT - 1) / PRE_XT;
    const dim3 grid((unsigned)(nb < PRE_XBLOCKS ? nb : PRE_XBLOCKS), PRE_Q);
    constexpr int rounds = D - 1;
    for (int r = 0; r < rounds; ++r)
        hipLaunchKernelGGL((pre_extend_kernel<D>), grid, dim3(PRE_XT), 0, st, c, sc.ranged, sc.r0, sc.r1, r, rounds);
}

template <int D, bool MT>
static void launch_one(const Ctx &c, const SearchArgs &a, size_t lds, hipStream_t st) {
    if (c.fp32)
        hipLaunchKernelGGL((search_kernel<D, MT, float>), dim3(c.search_wgs), dim3(SEARCH_WG), lds, st, c, a);
    else
        hipLaunchKernelGGL((search_kernel<D, MT, double>), dim3(c.search_wgs), dim3(SEARCH_WG), lds, st, c, a);
}

static void launch_merge(const Ctx &c, int nlists, int use_pre, hipStream_t st, int dedupe = 0,
                         const uint32_t *nl_dev = nullptr) {
    const int per = MERGE_THREADS / 64;
    hipLaunchKernelGGL(merge_compact_kernel, dim3((nlists + per - 1) / per), dim3(MERGE_THREADS), 0, st, c, nlists,
                       c.KP, use_pre, nl_dev);
    hipLaunchKernelGGL(dedupe ? merge_select_kernel<true> : merge_select_kernel<false>, dim3(1), dim3(MERGE_THREADS),
                       0, st, c, c.KP, use_pre, nlists, nl_dev);
}

// The one-task D = 3 record-table path applies (it also needs the table in
// the workspace and fewer than 2^31 items).
bool s3_batchable(const Ctx &c, int D) {
    return D == 3 && c.T == 1 && !c.fp32 && c.rec3 != nullptr && s3_items_host(c.S) < (1ull << 31);
}

// record table + initialisation + pre-pass selection (one launch), then the
// pre-pass extension: everything before the sweep of the one-task D = 3 path
static void s3_prologue(const Ctx &c, const SearchCall &sc, hipStream_t st) {
    const unsigned init_blocks = (unsigned)(((SISSO_MAX_D + 1) * (c.S + 1) + 255) / 256);
    const int64_t ngr = (c.S - 3) / S3_NR + 1;
    int64_t bx = ((c.S - 2) * S3_NR + PRE_WG - 1) / PRE_WG;
    const int64_t ninit = (int64_t)init_blocks * 256;
    if (bx * PRE_WG * ngr < ninit) bx = (ninit / ngr + PRE_WG - 1) / PRE_WG + 1;
    // one more column: its first workgroup runs the pre-pass selection
    hipLaunchKernelGGL(rec3_kernel, dim3((unsigned)(bx + 1), (unsigned)ngr, 2), dim3(PRE_WG), 0, st, c, c.rec3);
    launch_prepass<3>(c, sc, st, false);
}

int launch_batch_prologue(const Ctx &c, const SearchCall &sc, hipStream_t st) {
    s3_prologue(c, sc, st);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_batch_search3(const BatchSearchArgs &b, int wgs, hipStream_t st) {
    // one resident round: S3B_WPE waves on each of the 4 SIMDs of 256 CUs
    if (wgs <= 0 || wgs > S3B_WPE * 256) wgs = S3B_WPE * 256;
    const size_t lds = (size_t)SEARCH_WAVES * b.KPmax * 2 * sizeof(double);
    hipLaunchKernelGGL(search3_batch_kernel, dim3((unsigned)wgs), dim3(SEARCH_WG), lds, st, b);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_batch_epilogue(const Ctx &c, const SearchCall &sc, hipStream_t st) {
    launch_merge(c, c.nwaves, 1, st, 0, c.flags + FLAG_NLISTS);
    launch_rescore_final(c, 3, sc.k, st);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

// first index of the D-tuple with lexicographic rank r
static int64_t first_index(int64_t S, int D, uint64_t r) {
    int64_t i = 0;
    for (; i < S - D; ++i) {
        const uint64_t n = binom(S - 1 - i, D - 1);  // tuples that start with i
        if (r < n) break;
        r -= n;
    }
    return i;
}

int launch_search(const Ctx &c, const SearchCall &sc, hipStream_t st) {
    const int D = sc.D;
    const bool MT = c.T > 1;
    SearchArgs a{};
    a.D = D;
    a.KP = c.KP;
    a.ranged = sc.ranged;
    a.r0 = sc.r0;
    a.r1 = sc.r1;
    a.TL = MT ? c.TP : 1;
    // many tasks: JB * TP <= MT_RECS records of the item in LDS (JB <= 64)
    a.JB = MT ? (64 < MT_RECS / c.TP ? 64 : MT_RECS / c.TP) : JBLK;
    a.R = MT ? 1 : SUBP;
    const int q = D - 2;
    const int RECW = q + 4;
    const int QA = q > 0 ? q : 1;
    const int SUBW = QA * QA + QA + 2;
    const size_t lds_lists = (size_t)SEARCH_WAVES * c.KP * 2 * sizeof(double);
    const unsigned init_blocks = (unsigned)(((SISSO_MAX_D + 1) * (c.S + 1) + 255) / 256);

    if (D == 1) {
        int wgs = (int)((c.S + SEARCH_WG - 1) / SEARCH_WG);
        if (wgs > c.search_wgs) wgs = c.search_wgs;
        phase_begin(c, SISSO_PHASE_PREPASS, st);
        hipLaunchKernelGGL(search_init_kernel, dim3(init_blocks), dim3(256), 0, st, c, 2, 1, JBLK, 0);
        phase_end(c, SISSO_PHASE_PREPASS, st);
        phase_begin(c, SISSO_PHASE_SEARCH, st);
        hipLaunchKernelGGL(search_d1_kernel, dim3(wgs), dim3(SEARCH_WG), lds_lists, st, c, a);
        phase_end(c, SISSO_PHASE_SEARCH, st);
        phase_begin(c, SISSO_PHASE_MERGE, st);
        launch_merge(c, wgs * SEARCH_WAVES, 0, st);
        phase_end(c, SISSO_PHASE_MERGE, st);
    } else {
        phase_begin(c, SISSO_PHASE_PREPASS, st);
        // one task, D = 3: record table + sweep of the units
        // D = 3: the record-table sweep, on the filter task's matrix when
        // there are several tasks
        const bool s3 = D == 3 && !c.fp32 && c.rec3 != nullptr && s3_items_host(c.S) < (1ull << 31);
        // one task, D = 4: the record table of group pairs (sized at create
        // only while it stays within S4_TABLE_MAX)
        const bool s4 = D == 4 && !MT && !c.fp32 && c.rec4 != nullptr;
        const bool s2 = D == 2 && !MT && !c.fp32;
        const int64_t ntiles2 = ((c.S + 63) / 64) * ((c.S + 63) / 64 + 1) / 2;
        const int wgs = s2 && ntiles2 < c.search_wgs ? (int)ntiles2 : c.search_wgs;
        if (s4) {
            const int64_t nt = std::max((int64_t)(SISSO_MAX_D + 1) * (c.S + 1), s4_pairs_below(s4_groups(c.S)));
            hipLaunchKernelGGL(s4_init_kernel, dim3((unsigned)((nt + 63) / 64)), dim3(64), 0, st, c);
        } else if (s3) {
            // record table + initialisation in one launch (its grid covers the binomial table)
            // x: the rows of one group (j, r); y: groups; the grid also covers
            // the binomial table of the initialisation
            const int64_t ngr = (c.S - 3) / S3_NR + 1;
            int64_t bx = ((c.S - 2) * S3_NR + PRE_WG - 1) / PRE_WG;
            const int64_t ninit = (int64_t)init_blocks * 256;
            if (bx * PRE_WG * ngr < ninit) bx = (ninit / ngr + PRE_WG - 1) / PRE_WG + 1;
            // one more column: its first workgroup runs the pre-pass selection
            hipLaunchKernelGGL(rec3_kernel, dim3((unsigned)(bx + 1), (unsigned)ngr, 2), dim3(PRE_WG), 0, st, c, c.rec3);
        } else {
            hipLaunchKernelGGL(search_init_kernel, dim3(init_blocks), dim3(256), 0, st, c, D, a.R, a.JB,
                               s2 ? 2 : 0);
        }
        switch (D) {
            case 2: launch_prepass<2>(c, sc, st); break;
            case 3: launch_prepass<3>(c, sc, st, !s3); break;
            default: launch_prepass<4>(c, sc, st); break;
        }
        if (s4) {
            // the record table (part of the set-up, like rec3 above)
            const int64_t nitem = s4_pairs_below(s4_groups(c.S));
            hipLaunchKernelGGL(rec4_kernel, dim3((unsigned)nitem), dim3(SEARCH_WG), 0, st, c);
        }
        phase_end(c, SISSO_PHASE_PREPASS, st);
        phase_begin(c, SISSO_PHASE_SEARCH, st);
        const size_t nrec = MT ? (size_t)a.JB * c.TP : (size_t)SEARCH_WG;
        const size_t lds = lds_lists + nrec * RECW * sizeof(double) + (size_t)64 * SUBW * sizeof(double);
        // groups of first indices with a rank in the range
        int glo = 0, ghi = INT32_MAX;
        if (sc.ranged && (s3 || s4)) {
            glo = (int)(first_index(c.S, D, sc.r0) / S3_NR);
            ghi = (int)(first_index(c.S, D, sc.r1 > sc.r0 ? sc.r1 - 1 : sc.r0) / S3_NR);
        }
        if (s2) {
            hipLaunchKernelGGL(search2_kernel, dim3(wgs), dim3(SEARCH_WG), lds_lists, st, c, a, ntiles2);
        } else if (s4) {
            const int run = bound_run(bound_units<S4Pairs>(c.S));
            const uint64_t n = s4_items_host(c.S), pass = S4_PASS / run;
            const uint32_t nseg = (uint32_t)(c.search_wgs < BU_WGS ? c.search_wgs : BU_WGS);
            const size_t lds4 = lds_lists + (size_t)2 * (nseg + 1) * sizeof(uint64_t);
            for (uint64_t t0 = 0; t0 < n; t0 += pass) {
                const uint64_t t1 = t0 + pass < n ? t0 + pass : n;
                const uint32_t wu = (uint32_t)((t1 - t0 + nseg - 1) / nseg * run);
                hipLaunchKernelGGL(search4_kernel, dim3(nseg), dim3(SEARCH_WG), 0, st, c, (const double *)c.rec4,
                                   (const double *)c.fac4, (const uint64_t *)c.cum, t0, t1, wu, run, glo, ghi);
                hipLaunchKernelGGL(s4_eval_kernel, dim3(c.search_wgs), dim3(SEARCH_WG), lds4, st, c, a, nseg, wu,
                                   t0 > 0);
            }
        } else if (s3) {
            const int run = bound_run(bound_units<S3Groups>(c.S));
            const uint64_t n = s3_items_host(c.S), pass = S3_PASS / run;
            const uint32_t nseg = (uint32_t)(c.search_wgs < BU_WGS ? c.search_wgs : BU_WGS);
            const int limit = s3_lanes(c.T);
            const size_t lds3 = lds_lists + (size_t)2 * (nseg + 1) * sizeof(uint64_t);
            for (uint64_t t0 = 0; t0 < n; t0 += pass) {
                const uint64_t t1 = t0 + pass < n ? t0 + pass : n;
                const uint32_t wu = (uint32_t)((t1 - t0 + nseg - 1) / nseg * run);
                hipLaunchKernelGGL(search3_kernel, dim3(nseg), dim3(SEARCH_WG), 0, st, c, (const double *)c.recg,
                                   (const uint64_t *)c.cum, t0, t1, wu, limit, run, glo, ghi);
                if (MT)
                    hipLaunchKernelGGL(s3_eval_kernel<true>, dim3(c.search_wgs), dim3(SEARCH_WG), lds3, st, c, a,
                                       (const double *)c.rec3, nseg, wu, limit, t0 > 0);
                else
                    hipLaunchKernelGGL(s3_eval_kernel<false>, dim3(c.search_wgs), dim3(SEARCH_WG), lds3, st, c, a,
                                       (const double *)c.rec3, nseg, wu, limit, t0 > 0);
            }
        }
        else switch (D) {
            // (one task, D = 2 comes here in the FP32 solve form only)
            case 2:
                if (MT) launch_one<2, true>(c, a, lds, st);
                else hipLaunchKernelGGL((search_kernel<2, false, float>), dim3(c.search_wgs), dim3(SEARCH_WG), lds, st, c, a);
                break;
            // (D = 3 too: 2^31 items of the record-table sweep are some 150,000
            // features, whose table is larger than the card's memory)
            case 3:
                if (!c.fp32) return -1;
                if (MT) hipLaunchKernelGGL((search_kernel<3, true, float>), dim3(c.search_wgs), dim3(SEARCH_WG), lds, st, c, a);
                else hipLaunchKernelGGL((search_kernel<3, false, float>), dim3(c.search_wgs), dim3(SEARCH_WG), lds, st, c, a);
                break;
            case 4: MT ? launch_one<4, true>(c, a, lds, st) : launch_one<4, false>(c, a, lds, st); break;
            default: return -1;
        }
        phase_end(c, SISSO_PHASE_SEARCH, st);
        phase_begin(c, SISSO_PHASE_MERGE, st);
        launch_merge(c, wgs * SEARCH_WAVES, 1, st);
        phase_end(c, SISSO_PHASE_MERGE, st);
    }
    launch_rescore_final(c, D, sc.k, st);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}


int launch_prefix_best(const Ctx &c, int M, const int32_t *pre, int64_t n, double *best, hipStream_t st) {
    const unsigned wgs = (unsigned)(n < 4096 ? (n + 3) / 4 : 1024);
    switch (M) {
        case 1: hipLaunchKernelGGL((prefix_best_kernel<1>), dim3(wgs), dim3(256), 0, st, c, pre, n, best); break;
        case 2: hipLaunchKernelGGL((prefix_best_kernel<2>), dim3(wgs), dim3(256), 0, st, c, pre, n, best); break;
        case 3: hipLaunchKernelGGL((prefix_best_kernel<3>), dim3(wgs), dim3(256), 0, st, c, pre, n, best); break;
        default: return -1;
    }
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

// Training target of a prefix from its best extension's SSE:
// -log10(best / sum_t |y_t - mean|^2), the fraction clamped to [1e-12, 1];
// a prefix with no full-rank extension (best = +inf) or a malformed row
// (NaN) gets 0 (fraction 1).
__global__ void prefix_target_kernel(const double *__restrict__ cyy, int T, const double *__restrict__ best,
                                     int64_t n, float *__restrict__ target) {
    double ctot = 0.0;
    for (int t = 0; t < T; ++t) ctot += cyy[t];
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const double b = best[i];
        double frac = b / ctot;
        frac = frac < 1e-12 ? 1e-12 : (frac > 1.0 ? 1.0 : frac);
        if (!(b <= 1.7976931348623157e308)) frac = 1.0;  // +inf or NaN
        target[i] = (float)(-log10(frac));
    }
}

int launch_prefix_target(const Ctx &c, const double *best, int64_t n, float *target, hipStream_t st) {
    const unsigned blocks = (unsigned)(n < 262144 ? (n + 255) / 256 : 1024);
    hipLaunchKernelGGL(prefix_target_kernel, dim3(blocks), dim3(256), 0, st, c.cyy, c.T, best, n, target);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

// Every extension of each listed prefix: thread (p, t) writes the sorted
// (M + 1)-tuple P + {j}, j the t-th index of {0..S-1} not in P (walking the
// sorted prefix: each member at or below the running index pushes it up by
// one).  A malformed prefix row gives rows of -1.
template <int M>
__global__ __launch_bounds__(256) void prefix_extend_kernel(int64_t S, const int32_t *__restrict__ pre, int64_t n,
                                                            int32_t *__restrict__ out) {
    const int64_t w = S - M;
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n * w) return;
    const int64_t p = e / w, t = e - p * w;
    int32_t P[M];
    bool ok = true;
    for (int q = 0; q < M; ++q) {
        P[q] = pre[p * M + q];
        ok &= P[q] >= 0 && P[q] < S && (q == 0 || P[q] > P[q - 1]);
    }
    int32_t *o = out + e * (M + 1);
    if (!ok) {
        for (int q = 0; q <= M; ++q) o[q] = -1;
        return;
    }
    int64_t j = t;
    for (int q = 0; q < M; ++q) j += P[q] <= j ? 1 : 0;
    int q = 0, x = 0;
    for (; q < M && P[q] < j; ++q) o[x++] = P[q];
    o[x++] = (int32_t)j;
    for (; q < M; ++q) o[x++] = P[q];
}

int launch_prefix_extend(const Ctx &c, int M, const int32_t *pre, int64_t n, int32_t *out, hipStream_t st) {
    const int64_t tot = n * (c.S - M);
    const unsigned blocks = (unsigned)((tot + 255) / 256);
    switch (M) {
        case 1: hipLaunchKernelGGL((prefix_extend_kernel<1>), dim3(blocks), dim3(256), 0, st, c.S, pre, n, out); break;
        case 2: hipLaunchKernelGGL((prefix_extend_kernel<2>), dim3(blocks), dim3(256), 0, st, c.S, pre, n, out); break;
        case 3: hipLaunchKernelGGL((prefix_extend_kernel<3>), dim3(blocks), dim3(256), 0, st, c.S, pre, n, out); break;
        default: return -1;
    }
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_prefix_features(const Ctx &c, int M, const int32_t *pre, int64_t n, float *out, hipStream_t st) {
    const unsigned blocks = (unsigned)((n + 255) / 256);
    switch (M) {
        case 1: hipLaunchKernelGGL((prefix_features_kernel<1>), dim3(blocks), dim3(256), 0, st, c, pre, n, out); break;
        case 2: hipLaunchKernelGGL((prefix_features_kernel<2>), dim3(blocks), dim3(256), 0, st, c, pre, n, out); break;
        case 3: hipLaunchKernelGGL((prefix_features_kernel<3>), dim3(blocks), dim3(256), 0, st, c, pre, n, out); break;
        case 4: hipLaunchKernelGGL((prefix_features_kernel<4>), dim3(blocks), dim3(256), 0, st, c, pre, n, out); break;
        default: return -1;
    }
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_prefix_features_range(const Ctx &c, int M, uint64_t r0, int64_t n, float *out, hipStream_t st) {
    const unsigned blocks = (unsigned)((n + 255) / 256);
    switch (M) {
        case 1: hipLaunchKernelGGL((prefix_features_range_kernel<1>), dim3(blocks), dim3(256), 0, st, c, r0, n, out); break;
        case 2: hipLaunchKernelGGL((prefix_features_range_kernel<2>), dim3(blocks), dim3(256), 0, st, c, r0, n, out); break;
        case 3: hipLaunchKernelGGL((prefix_features_range_kernel<3>), dim3(blocks), dim3(256), 0, st, c, r0, n, out); break;
        default: return -1;
    }
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_list_search(const Ctx &c, int D, int k, const int32_t *pre, int64_t n, hipStream_t st) {
    const unsigned init_blocks = (unsigned)(((SISSO_MAX_D + 1) * (c.S + 1) + 255) / 256);
    phase_begin(c, SISSO_PHASE_PREPASS, st);
    hipLaunchKernelGGL(list_init_kernel, dim3(init_blocks > PRE_BINS / 256 ? init_blocks : PRE_BINS / 256), dim3(256),
                       0, st, c);
    // (one row: a single wave's list, which the merge takes as it is; with the
    // pool 177 us, without 161)
    if (c.T == 1 && n > 1) {
        const int64_t np = n < LIST_POOL ? n : LIST_POOL;
        const dim3 grid((unsigned)((np + 3) / 4));
        switch (D - 1) {
            case 1: hipLaunchKernelGGL((list_pool_kernel<1>), grid, dim3(256), 0, st, c, pre, np); break;
            case 2: hipLaunchKernelGGL((list_pool_kernel<2>), grid, dim3(256), 0, st, c, pre, np); break;
            case 3: hipLaunchKernelGGL((list_pool_kernel<3>), grid, dim3(256), 0, st, c, pre, np); break;
            default: return -1;
        }
    }
    phase_end(c, SISSO_PHASE_PREPASS, st);
    int64_t wgs = (n + SEARCH_WAVES - 1) / SEARCH_WAVES;
    if (wgs > c.search_wgs) wgs = c.search_wgs;
    if (wgs < 1) wgs = 1;
    const size_t lds = (size_t)SEARCH_WAVES * c.KP * 2 * sizeof(double);
    phase_begin(c, SISSO_PHASE_SEARCH, st);
    switch (D - 1) {
        case 1: hipLaunchKernelGGL((list_search_kernel<1>), dim3((unsigned)wgs), dim3(SEARCH_WG), lds, st, c, pre, n); break;
        case 2: hipLaunchKernelGGL((list_search_kernel<2>), dim3((unsigned)wgs), dim3(SEARCH_WG), lds, st, c, pre, n); break;
        case 3: hipLaunchKernelGGL((list_search_kernel<3>), dim3((unsigned)wgs), dim3(SEARCH_WG), lds, st, c, pre, n); break;
        default: return -1;
    }
    phase_end(c, SISSO_PHASE_SEARCH, st);
    phase_begin(c, SISSO_PHASE_MERGE, st);
    launch_merge(c, (int)wgs * SEARCH_WAVES, 1, st, 1);
    phase_end(c, SISSO_PHASE_MERGE, st);
    launch_rescore_final(c, D, k, st);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

}  // namespace sl0
