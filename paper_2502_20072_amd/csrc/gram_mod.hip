// The FP64 Gram on the integer matrix cores: exact integer products in
// residue arithmetic.
//
// Every centred column of a task is scaled by a power of two to a norm in
// (2^57, 2^58] and rounded to integers a (at most half a unit per value,
// 2^-58 of the column's norm), so that the centred cross product of two
// columns is, up to that rounding, an integer C with |C| <= 2^116
// (Cauchy-Schwarz) times a power of two.  C is computed exactly: modulo each
// of GM_NP pairwise coprime moduli p <= 256 (product M > 2^117) the
// columns' residues are signed bytes, their products accumulate exactly in
// the 32-bit accumulators of the INT8 matrix instructions, and the Chinese
// remainder theorem gives C back from the GM_NP residues (residue number
// systems for dense products: Ozaki, Uchino and Imamura 2025, "Ozaki Scheme
// II").  The only roundings are that of the scaled values and that of the
// result: as a rule an entry's error does not grow with the number of samples.
//
// The rounding of the values is absolute: a value keeps as many bits as it
// lies above 2^-58 of its column's norm (some 50 bits of a typical value at n =
// 50,000, 38 of one that is 2^-20 of the norm).  An entry's error is relative to
// the diagonal: rms about 2^-58 of it (independent roundings), at most sqrt(n)
// 2^-57 (the roundings as a vector against the other column, twice), plus the
// entry's own rounding.  The solves on the matrix round at 2^-53 of the diagonal.
// Measured against 64 bits the entries are closer than those of FP64 products on
// columns without large spikes (rms 4e-18 against 1.4e-17 at n = 50,000), and
// further off on columns that a few values dominate, whose other entries are
// tiny (n = 2000, unit noise with spikes of 1e8: rms 3e-18 of the diagonal against
// 6e-24, which is 3e-10 of an entry against 5e-16).
//
// Why this and not the FP64 matrix instructions: those sustain 36 to 50
// TFLOP/s here (one instruction is 2048 products and takes 64 cycles at
// best); GM_NP INT8 products per FP64 product at the INT8 rate are cheaper,
// and the bytes of all residues are 1.9 times those of F.  (Tasks of few rows
// take the FP64 products nevertheless: gram_f64.)  One modulus fewer would leave
// 2^-54 of the norm per value, more than the FP64 products' rounding on
// uncorrelated columns (3e-17 against 1e-17 of the diagonal).
#include "common.h"
#include "kernels.h"

namespace sl0 {

typedef int int4_t __attribute__((ext_vector_type(4)));

// ------------------------------------------------------------ the moduli
// The largest pairwise coprime moduli up to 256 (residues are taken in
// [-p/2, p/2], signed bytes; modulo 256 the byte wraps by itself).
struct ModTables {
    double p[GM_NP], ip[GM_NP];    // modulus, reciprocal
    double c30[GM_NP];             // 2^30 mod p, in (-p/2, p/2]
    double wh[GM_NP], wl[GM_NP];   // CRT weight q/p, q = (M/p)^-1 mod p, in (-1/2, 1/2]:
                                   // a multiple of 2^-42 and the rest
    double M;                      // product of the moduli
};
constexpr int GM_MODULI[GM_NP] = {256, 255, 253, 251, 247, 241, 239, 233, 229, 227, 223, 217, 211, 199, 197};

constexpr ModTables make_tables() {
    ModTables t{};
    unsigned __int128 M = 1;
    for (int l = 0; l < GM_NP; ++l) M *= (unsigned)GM_MODULI[l];
    t.M = (double)M;
    for (int l = 0; l < GM_NP; ++l) {
        const int p = GM_MODULI[l];
        t.p[l] = p;
        t.ip[l] = 1.0 / p;
        const int c30 = (1 << 30) % p;
        t.c30[l] = 2 * c30 > p ? c30 - p : c30;
        int rest = 1;  // M / p mod p
        for (int m = 0; m < GM_NP; ++m)
            if (m != l) rest = rest * (GM_MODULI[m] % p) % p;
        int q = 1;
        while (rest * q % p != 1) ++q;
        if (2 * q > p) q -= p;
        // q / p = wh + wl, wh = floor(q 2^42 / p) / 2^42
        const long long num = (long long)q * (1ll << 42);
        long long h = num / p;
        if (num % p < 0) --h;
        t.wh[l] = (double)h / (double)(1ll << 42);
        t.wl[l] = (double)(num - h * p) / (double)p / (double)(1ll << 42);
    }
    return t;
}
__constant__ constexpr ModTables GM_T = make_tables();

// Exponent e of a column's integer scale 2^e from inv_s = 1 / norm > 0:
// norm 2^e in (2^57, 2^58].
__device__ inline int mod_exp(double inv) { return 58 + ilogb(inv); }

// C (a double, rounded once) from the residues r[l] of C modulo the moduli:
// C / M = frac(sum_l r_l q_l / p_l).  The sum of r_l wh_l is exact (|r| <=
// 128, multiples of 2^-42, below 2^10), its integer part is dropped exactly,
// and the sum of r_l wl_l is below 2^-32 with an error below 2^-85.
__device__ inline void crt_add(double r, int l, double &hi, double &lo) {
    hi = fma(r, GM_T.wh[l], hi);
    lo = fma(r, GM_T.wl[l], lo);
}
__device__ inline double crt_value(double hi, double lo) { return ((hi - rint(hi)) + lo) * GM_T.M; }

// ------------------------------------------------------------- residues
// One workgroup per (feature, GM_RB padded samples): each thread takes four
// consecutive samples of the padded axis, on which every task starts at a
// multiple of GM_BK (kb[t]) and is zero-padded, and writes one dword of
// residues per modulus.  Bound by HBM: 8 bytes read and GM_NP written per
// sample, about 110 VALU instructions.
constexpr int GM_RB = 1024;
__global__ __launch_bounds__(256) void residue_kernel(const double *__restrict__ F, int64_t n_total, int64_t S,
                                                      const int64_t *__restrict__ off,
                                                      const int64_t *__restrict__ kb, int T,
                                                      const double *__restrict__ mu,
                                                      const double *__restrict__ inv_s, int64_t c0, int64_t kc,
                                                      int64_t nseg, uint8_t *__restrict__ res) {
    const int64_t j = blockIdx.x / nseg;
    const int64_t kl = (blockIdx.x % nseg) * GM_RB + threadIdx.x * 4;  // within the chunk
    if (kl >= kc) return;
    const int64_t k = c0 + kl;
    int t = 0;
    while (t + 1 < T && kb[t + 1] <= k) ++t;
    const int64_t row = off[t] + (k - kb[t]), r1 = off[t + 1];
    const double m = mu[(int64_t)t * S + j], inv = inv_s[(int64_t)t * S + j];
    const double sc = inv > 0.0 ? ldexp(1.0, mod_exp(inv)) : 0.0;
    double a[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) a[i] = row + i < r1 ? F[j * n_total + row + i] : m;
#pragma unroll
    for (int i = 0; i < 4; ++i) a[i] = inv > 0.0 ? rint((a[i] - m) * sc) : 0.0;
    // a = ah 2^30 + al, |ah| <= 2^28, |al| <= 2^29, so that ah c30 + al stays
    // exact and far from the quotient's rounding
    double ah[4], al[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        ah[i] = rint(a[i] * 0x1p-30);
        al[i] = fma(ah[i], -0x1p30, a[i]);
    }
    uint8_t *o = res + j * kc + kl;
#pragma unroll
    for (int l = 0; l < GM_NP; ++l) {
        uint32_t w = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const double v = fma(ah[i], GM_T.c30[l], al[i]);
            const int r = (int)fma(-rint(v * GM_T.ip[l]), GM_T.p[l], v);
            w |= ((uint32_t)r & 0xffu) << (8 * i);
        }
        *reinterpret_cast<uint32_t *>(o + (int64_t)l * S * kc) = w;
    }
}

// ---------------------------------------------------------- INT8 products
// One workgroup per (task, modulus, TM x TM tile pair bi <= bj): the product
// of two panels of residues over the chunk's samples of the task, reduced
// modulo p to a byte per entry.  A chunk that does not start the task adds
// the residue already there.  Where the tiles are few, ns workgroups share the
// samples of a product, each with a plane of its own (the finishing pass adds
// them): 4 tasks of 30,000 rows, S = 40: 756 us, now 119.
//
// Tiles.  WM x WN waves; a wave owns (16 MB) columns gj times (16 NB) rows
// gi of G as MB x NB blocks of v_mfma_i32_16x16x64_i8 (A[i][k] in lane
// i + 16 (k / 16), byte k % 16; B likewise; D[i][j] in lane j + 16 (i / 4),
// register i % 4).  The A operand holds the columns gj in the order that
// leaves each lane 4 MB consecutive ones of one row: block m, row i is
// column 4 MB (i / 4) + 4 m + i % 4, so a lane's results are stored 16
// bytes at a time.
// K-steps of BK samples go global -> registers -> LDS, double-buffered in LDS
// and loaded PD steps ahead, one barrier per step (the loads are
// unconditional, clamped to the last step, so that none is waited for
// early).  The 16-byte pieces of an LDS row are permuted by the row
// (XOR) so that the 16 rows of a fragment read fall on distinct banks: rows
// i % 16 for B, and for A rows that differ in bits 0, 1 and log2(4 MB) and up.
// SPLIT: ns workgroups share a product's samples, a plane each.
template <int TM, int WM, int WN, int BK, int PD, int WPE, bool SPLIT>
__global__ __launch_bounds__(64 * WM * WN) __attribute__((amdgpu_waves_per_eu(WPE, WPE))) void gram_mod_kernel(
    const uint8_t *__restrict__ res, int64_t S, int64_t kc, int64_t c0, const int64_t *__restrict__ kb,
    const int32_t *__restrict__ torder, int T, int ntile, int ns, uint8_t *__restrict__ planes) {
    constexpr int NT = 64 * WM * WN;          // threads
    constexpr int MB = TM / (16 * WM);        // 16-column blocks per wave
    constexpr int NB = TM / (16 * WN);        // 16-row blocks per wave
    constexpr int PC = BK / 16;               // 16-byte pieces of a row
    constexpr int PPT = TM * PC / NT;         // pieces per thread and operand
    constexpr int SHA = MB == 8 ? 5 : 4;      // log2(4 MB)
    static_assert(MB == 4 || MB == 8, "A rows are permuted for 4 or 8 blocks");
    static_assert(BK == 64 || BK == 128, "piece permutations");
    __shared__ __attribute__((aligned(16))) uint8_t As[2][TM * BK];
    __shared__ __attribute__((aligned(16))) uint8_t Bs[2][TM * BK];
    // address of piece c of row r: sixteen 16-byte slots cover the banks, a row
    // takes PC of them, and a 16-byte read serves lanes 0-3, 12-15, 20-23,
    // 24-27 (and so on) together: rows 0-3 and 12-15 of one piece with rows
    // 4-11 of the next
    auto perm4 = [](int x) { return ((x & 1) << 1) ^ ((x >> 1) * 3); };
    auto slot_a = [=](int r, int c) {
        const int f = BK == 128 ? ((r >> 1) & 1) | (((r >> SHA) & 3) << 1) : perm4((r >> SHA) & 3);
        return r * BK + 16 * (c ^ f);
    };
    auto slot_b = [=](int r, int c) {
        const int f = BK == 128 ? (r >> 1) & 7 : perm4((r >> 2) & 3);
        return r * BK + 16 * (c ^ f);
    };

    const uint32_t npair = (uint32_t)((int64_t)ntile * (ntile + 1) / 2);
    const uint32_t nblk = npair * GM_NP * (uint32_t)(SPLIT ? ns : 1);  // workgroups of a task
    uint32_t b = blockIdx.x;
    int t;
    {
        // workgroup b runs on XCD b mod 8: of every task each XCD takes a
        // contiguous range, i.e. neighbouring tiles of one or two moduli, whose
        // panels its L2 holds (dealt one by one, 16 tasks at S = 1500 missed
        // L2 on 37 % of the reads and were bound by them)
        const uint32_t q = (nblk + 7) / 8;
        t = torder[b / (8 * q)];              // tasks by decreasing row count
        b %= 8 * q;
        b = (b % 8) * q + b / 8;
        if (b >= nblk) return;
    }
    const int split = SPLIT ? (int)(b / (npair * GM_NP)) : 0;
    const int l = (int)(SPLIT ? b / npair % GM_NP : b / npair);
    const uint32_t pair = b % npair;
    int bi, bj;
    gm_tile_pair(pair, ntile, bi, bj);

    // the task's samples inside the chunk [c0, c0 + kc), and this workgroup's
    int64_t k0 = kb[t] > c0 ? kb[t] - c0 : 0;
    const int64_t k1 = kb[t + 1] - c0 < kc ? kb[t + 1] - c0 : kc;
    if (k0 >= k1) return;
    const bool first = kb[t] >= c0;
    int steps = (int)((k1 - k0) / BK);
    auto plane = [&] { return planes + ((((int64_t)split * T + t) * npair + pair) * GM_NP + l) * (TM * TM); };
    if constexpr (SPLIT) {
        const uint32_t all = (uint32_t)steps;  // (at most GM_KC_MAX / BK)
        const int s0 = (int)(all * (uint32_t)split / (uint32_t)ns);
        steps = (int)(all * (uint32_t)(split + 1) / (uint32_t)ns) - s0;
        k0 += (int64_t)s0 * BK;
        if (steps == 0) {  // (a task with fewer steps than parts)
            if (first)
                for (int e = threadIdx.x; e < TM * TM / 16; e += NT)
                    reinterpret_cast<int4_t *>(plane())[e] = (int4_t){0, 0, 0, 0};
            return;
        }
    }

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wj = (wave % WM) * 16 * MB, wi = (wave / WM) * 16 * NB;

    const uint8_t *base = res + (int64_t)l * S * kc + k0;
    const uint8_t *pa[PPT], *pb[PPT];
    int la[PPT], lb[PPT];
#pragma unroll
    for (int x = 0; x < PPT; ++x) {
        const int e = tid + NT * x, row = e / PC, cpc = e % PC;
        int64_t fj = (int64_t)bj * TM + row, fi = (int64_t)bi * TM + row;
        fj = fj < S ? fj : S - 1;             // entries past S are not read back
        fi = fi < S ? fi : S - 1;
        pa[x] = base + fj * kc + 16 * cpc;
        pb[x] = base + fi * kc + 16 * cpc;
        la[x] = slot_a(row, cpc);
        lb[x] = slot_b(row, cpc);
    }
    // fragment addresses: piece 4 h + lane / 16 of the row (K half h)
    int fa[MB], fb[NB];
#pragma unroll
    for (int m = 0; m < MB; ++m) {
        const int i = lane & 15, row = wj + ((i >> 2) << SHA) + 4 * m + (i & 3);
        fa[m] = slot_a(row, lane >> 4);
    }
#pragma unroll
    for (int n = 0; n < NB; ++n) {
        fb[n] = slot_b(wi + 16 * n + (lane & 15), lane >> 4);
    }

    int4_t acc[MB][NB];
#pragma unroll
    for (int m = 0; m < MB; ++m)
#pragma unroll
        for (int n = 0; n < NB; ++n) acc[m][n] = (int4_t){0, 0, 0, 0};
    int4_t ra[PD][PPT], rb[PD][PPT];
    auto load = [&](int s, int4_t (&qa)[PPT], int4_t (&qb)[PPT]) {
        const int64_t o = (int64_t)(s < steps ? s : steps - 1) * BK;
#pragma unroll
        for (int x = 0; x < PPT; ++x) {
            qa[x] = *reinterpret_cast<const int4_t *>(pa[x] + o);
            qb[x] = *reinterpret_cast<const int4_t *>(pb[x] + o);
        }
    };
    auto store = [&](int buf, const int4_t (&qa)[PPT], const int4_t (&qb)[PPT]) {
#pragma unroll
        for (int x = 0; x < PPT; ++x) {
            *reinterpret_cast<int4_t *>(&As[buf][la[x]]) = qa[x];
            *reinterpret_cast<int4_t *>(&Bs[buf][lb[x]]) = qb[x];
        }
    };
#pragma unroll
    for (int d = 0; d < PD; ++d) load(d, ra[d], rb[d]);
    // nothing outstanding at the loop's entry: the compiler's waits inside it
    // are then those of the steady state
    __builtin_amdgcn_s_waitcnt(0x0F70);
    store(0, ra[0], rb[0]);
    __syncthreads();
    auto multiply = [&](int buf) {
#pragma unroll
        for (int h = 0; h < BK / 64; ++h) {
            int4_t av[MB], bv[NB];
            // half h: piece 4 h + lane / 16, i.e. bit 2 of the piece (bit 6 of the address) flipped
#pragma unroll
            for (int m = 0; m < MB; ++m) av[m] = *reinterpret_cast<const int4_t *>(&As[buf][fa[m] ^ (64 * h)]);
#pragma unroll
            for (int n = 0; n < NB; ++n) bv[n] = *reinterpret_cast<const int4_t *>(&Bs[buf][fb[n] ^ (64 * h)]);
#pragma unroll
            for (int m = 0; m < MB; ++m)
#pragma unroll
                for (int n = 0; n < NB; ++n)
                    acc[m][n] = __builtin_amdgcn_mfma_i32_16x16x64_i8(av[m], bv[n], acc[m][n], 0, 0, 0);
        }
    };
    // step s: slot s mod PD is free (its step is in LDS), slot (s + 1) mod PD
    // holds the next one
    for (int s = 0;;) {
        bool done = false;
#pragma unroll
        for (int d = 0; d < (PD > 1 ? PD : 1); ++d) {
            if (done) continue;
            load(s + PD, ra[d], rb[d]);
            __builtin_amdgcn_sched_barrier(0);  // the loads first: they have PD steps to arrive
            multiply(s & 1);
            store((s + 1) & 1, ra[(d + 1) % PD], rb[(d + 1) % PD]);
            __syncthreads();
            done = ++s >= steps;
        }
        if (done) break;
    }

    // residues of the sums: a lane holds row wi + 16 n + lane % 16, columns
    // wj + 4 MB (lane / 16) + 0 .. 4 MB - 1
    const double p = GM_T.p[l], ip = GM_T.ip[l];
    uint8_t *o0 = plane() + (wi + (lane & 15)) * TM + wj + 4 * MB * (lane >> 4);
    if (!first) {
#pragma unroll
        for (int n = 0; n < NB; ++n)
#pragma unroll
            for (int m = 0; m < MB; ++m) {
                const uint32_t w = *reinterpret_cast<const uint32_t *>(o0 + 16 * n * TM + 4 * m);
#pragma unroll
                for (int r = 0; r < 4; ++r) acc[m][n][r] += (int)(int8_t)(w >> (8 * r));
            }
    }
#pragma unroll
    for (int n = 0; n < NB; ++n)
#pragma unroll
        for (int m4 = 0; m4 < MB / 4; ++m4) {
            int4_t w;
#pragma unroll
            for (int x = 0; x < 4; ++x) {
                uint32_t v = 0;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const double a = (double)acc[4 * m4 + x][n][r];
                    const int rr = (int)fma(-rint(a * ip), p, a);
                    v |= ((uint32_t)rr & 0xffu) << (8 * r);
                }
                w[x] = (int)v;
            }
            *reinterpret_cast<int4_t *>(o0 + 16 * n * TM + 16 * m4) = w;
        }
}

// ------------------------------------------------------------------ finish
// Correlations from the residue planes, into the tiled layout.  G_ij =
// C_ij f_i f_j with f = inv_s 2^-e (the scale 2^e of the integers undone
// exactly); C is an exact integer, so C_ij = C_ji and the matrix is bitwise
// symmetric.  The diagonal is 1 for a live column and 0 for a constant one;
// padding rows, columns and tasks are zero.  A non-finite column's mean is
// not finite either and carries over to its row and column.
__device__ inline double mod_scale(double inv) { return inv > 0.0 ? ldexp(inv, -mod_exp(inv)) : 0.0; }

// Four consecutive entries; SPLIT: ns parts, `part` bytes apart, are added first.
template <bool SPLIT>
__device__ inline void crt_read(const uint8_t *src, int64_t stride, int ns, int64_t part, double (&v)[4]) {
    uint32_t w[GM_NP];
#pragma unroll
    for (int l = 0; l < GM_NP; ++l) w[l] = *reinterpret_cast<const uint32_t *>(src + l * stride);
    if constexpr (!SPLIT) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            double hi = 0.0, lo = 0.0;
#pragma unroll
            for (int l = 0; l < GM_NP; ++l) crt_add((double)(int)(int8_t)(w[l] >> (8 * e)), l, hi, lo);
            v[e] = crt_value(hi, lo);
        }
        return;
    }
    double hi[4] = {0.0, 0.0, 0.0, 0.0}, lo[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int l = 0; l < GM_NP; ++l) {
        int r[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) r[e] = (int)(int8_t)(w[l] >> (8 * e));
        for (int q = 1; q < ns; ++q) {
            const uint32_t x = *reinterpret_cast<const uint32_t *>(src + q * part + l * stride);
#pragma unroll
            for (int e = 0; e < 4; ++e) r[e] += (int)(int8_t)(x >> (8 * e));
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const double a = (double)r[e];
            crt_add(fma(-rint(a * GM_T.ip[l]), GM_T.p[l], a), l, hi[e], lo[e]);
        }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = crt_value(hi[e], lo[e]);
}

// One task per workgroup: a band of GM_FIN rows of a 64 x 64 tile pair (ti <=
// tk), four consecutive entries per thread.  The values pass through LDS, so
// that tile (ti, tk) is written row by row and its mirror in runs of GM_FIN
// entries.  Bound by HBM: GM_NP / 2 bytes read and 8 written per matrix entry;
// bands rather than whole tiles keep a small matrix from leaving CUs idle
// (S = 200: 12.7 us with whole tiles).
// (with several tasks the filter task's tiles also go to G1, bitwise the same)
constexpr int GM_FIN = 16;
template <bool SPLIT>
__global__ __launch_bounds__(256) void gram_mod_finish_kernel(const uint8_t *__restrict__ planes, int64_t S, int T,
                                                              int TP, int tm, int ntile, int ns,
                                                              const double *__restrict__ mu,
                                                              const double *__restrict__ inv_s,
                                                              double *__restrict__ G, int64_t nt,
                                                              double *__restrict__ G1,
                                                              const int32_t *__restrict__ tstar) {
    __shared__ double tile[GM_FIN][GT + 1];
    constexpr int NB = GT / GM_FIN;
    static_assert(GM_FIN * GT == 4 * 256, "four entries per thread");
    const int64_t npair64 = nt * (nt + 1) / 2;
    const int band = (int)(blockIdx.x % NB);
    const int64_t pb = blockIdx.x / NB;
    const int t = (int)(pb / npair64);
    int ti, tk;
    gm_tile_pair(pb - t * npair64, (int)nt, ti, tk);
    const int per = tm / GT;  // 64-wide tiles per plane tile
    const int bi = ti / per, bj = tk / per;
    const int64_t npair = (int64_t)ntile * (ntile + 1) / 2;
    const int li = threadIdx.x >> 4, lk = (threadIdx.x & 15) * 4;  // band row, first of four columns
    const uint8_t *src = planes + ((int64_t)t * npair + gm_pair_index(bi, bj, ntile)) * GM_NP * tm * tm +
                         (int64_t)((ti % per) * GT + GM_FIN * band + li) * tm + (tk % per) * GT + lk;
    const double *ist = inv_s + (int64_t)t * S, *mt = mu + (int64_t)t * S;
    const int64_t i = (int64_t)ti * GT + GM_FIN * band + li;
    const double fi = i < S ? mod_scale(ist[i]) : 0.0, mi = i < S ? mt[i] : 0.0;
    double v[4];
    crt_read<SPLIT>(src, (int64_t)tm * tm, ns, (int64_t)T * npair * GM_NP * tm * tm, v);
#pragma unroll
    for (int x = 0; x < 4; ++x) {
        const int64_t k = (int64_t)tk * GT + lk + x;
        double g = 0.0;
        if (i < S && k < S)
            g = i == k ? (fi > 0.0 ? 1.0 : 0.0) : v[x] * (fi * mod_scale(ist[k])) + 0.0 * (mi + mt[k]);
        tile[li][lk + x] = g;
    }
    __syncthreads();
    const bool one = G1 != nullptr && t == *tstar;
    const int64_t o0 = (((int64_t)ti * nt + tk) << 12) + GM_FIN * GT * band;
    const int64_t o1 = (((int64_t)tk * nt + ti) << 12) + GM_FIN * band;
#pragma unroll
    for (int x = 0; x < 4; ++x) {
        const int e = threadIdx.x + 256 * x;
        const double g = tile[e >> 6][e & 63];
        G[(o0 + e) * TP + t] = g;
        if (one) G1[o0 + e] = g;
        if (t == T - 1)
            for (int tp = T; tp < TP; ++tp) G[(o0 + e) * TP + tp] = 0.0;
    }
    if (ti == tk) return;
#pragma unroll
    for (int x = 0; x < 4; ++x) {
        const int e = threadIdx.x + 256 * x;
        const int r = e / GM_FIN, cc = e % GM_FIN;
        const double g = tile[cc][r];
        const int64_t at = o1 + (r << 6) + cc;
        G[at * TP + t] = g;
        if (one) G1[at] = g;
        if (t == T - 1)
            for (int tp = T; tp < TP; ++tp) G[at * TP + tp] = 0.0;
    }
}

// Several tasks (TP <= 16): one workgroup per (tile pair, band of GM_FR rows)
// takes every task, so that the TP task values of an entry (task fastest in
// G) are written together.  The band is held in LDS for all tasks
// ([task][row][column], one padding double per task), then written row by
// row to tile (ti, tk) and column by column to tile (tk, ti).
constexpr int GM_FR = 4;
template <bool SPLIT>
__global__ __launch_bounds__(256) void gram_mod_finish_tasks_kernel(const uint8_t *__restrict__ planes, int64_t S,
                                                                    int T, int TP, int tm, int ntile, int ns,
                                                                    const double *__restrict__ mu,
                                                                    const double *__restrict__ inv_s,
                                                                    double *__restrict__ G, int64_t nt,
                                                                    double *__restrict__ G1,
                                                                    const int32_t *__restrict__ tstar) {
    extern __shared__ double val[];  // [TP][GM_FR * 64 + 1]
    constexpr int NB = GT / GM_FR, VS = GM_FR * GT + 1, QR = GT / 4;
    const int band = (int)(blockIdx.x % NB);
    int ti, tk;
    gm_tile_pair(blockIdx.x / NB, (int)nt, ti, tk);
    const int per = tm / GT, bi = ti / per, bj = tk / per;
    const int64_t npair = (int64_t)ntile * (ntile + 1) / 2;
    const uint8_t *src0 = planes + gm_pair_index(bi, bj, ntile) * GM_NP * tm * tm +
                          (int64_t)((ti % per) * GT + GM_FR * band) * tm + (tk % per) * GT;
    const int ts = G1 != nullptr ? *tstar : -1;
    for (int x = threadIdx.x; x < TP * GM_FR * QR; x += 256) {
        const int t = x / (GM_FR * QR), r = x / QR % GM_FR, q = x % QR;
        double v[4] = {0.0, 0.0, 0.0, 0.0};
        if (t < T) {
            const double *ist = inv_s + (int64_t)t * S, *mt = mu + (int64_t)t * S;
            const int64_t i = (int64_t)ti * GT + GM_FR * band + r;
            const double fi = i < S ? mod_scale(ist[i]) : 0.0, mi = i < S ? mt[i] : 0.0;
            crt_read<SPLIT>(src0 + (int64_t)t * npair * GM_NP * tm * tm + (int64_t)r * tm + 4 * q, (int64_t)tm * tm, ns,
                     (int64_t)T * npair * GM_NP * tm * tm, v);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int64_t k = (int64_t)tk * GT + 4 * q + e;
                double g = 0.0;
                if (i < S && k < S)
                    g = i == k ? (fi > 0.0 ? 1.0 : 0.0) : v[e] * (fi * mod_scale(ist[k])) + 0.0 * (mi + mt[k]);
                v[e] = g;
            }
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) val[t * VS + r * GT + 4 * q + e] = v[e];
    }
    __syncthreads();
    const int64_t o0 = ((int64_t)ti * nt + tk) << 12, o1 = ((int64_t)tk * nt + ti) << 12;
    for (int x = threadIdx.x; x < GM_FR * GT * TP; x += 256) {
        const int t = x % TP, e = x / TP;
        const double v = val[t * VS + e];
        G[(o0 + GM_FR * GT * band + e) * TP + t] = v;
        if (t == ts) G1[o0 + GM_FR * GT * band + e] = v;
    }
    if (ti == tk) return;
    for (int x = threadIdx.x; x < GT * GM_FR * TP; x += 256) {
        const int t = x % TP, y = x / TP;
        const int r = y % GM_FR, lk = y / GM_FR;
        const double v = val[t * VS + r * GT + lk];
        G[(o1 + (lk << 6) + GM_FR * band + r) * TP + t] = v;
        if (t == ts) G1[o1 + (lk << 6) + GM_FR * band + r] = v;
    }
}

// ---------------------------------------------------------------- launcher
int launch_gram_mod(const Ctx &c, hipStream_t st) {
    const int tm = c.gm_tile;
    const int ntile = (int)((c.S + tm - 1) / tm);
    const int64_t npair = (int64_t)ntile * (ntile + 1) / 2;
    const unsigned blocks = (unsigned)((npair * GM_NP * c.gm_ns + 7) / 8 * 8 * c.T);
    for (int64_t c0 = 0; c0 < c.gm_kpad; c0 += c.gm_kc) {
        const int64_t kc = c.gm_kpad - c0 < c.gm_kc ? c.gm_kpad - c0 : c.gm_kc;
        const int64_t nseg = (kc + GM_RB - 1) / GM_RB;
        hipLaunchKernelGGL(residue_kernel, dim3((unsigned)(c.S * nseg)), dim3(256), 0, st, c.F, c.n_total, c.S,
                           c.off_dev, c.gm_kb, c.T, c.mu, c.inv_s, c0, kc, nseg, c.gm_res);
        const auto wide = c.gm_ns > 1 ? gram_mod_kernel<256, 2, 4, GM_BK, 1, 2, true>
                                      : gram_mod_kernel<256, 2, 4, GM_BK, 1, 2, false>;
        const auto narrow = c.gm_ns > 1 ? gram_mod_kernel<128, 2, 2, GM_BK_S, 2, 3, true>
                                        : gram_mod_kernel<128, 2, 2, GM_BK_S, 2, 3, false>;
        hipLaunchKernelGGL(tm == 256 ? wide : narrow, dim3(blocks), dim3(tm == 256 ? 512 : 256), 0, st, c.gm_res, c.S, kc,
                           c0, c.gm_kb, c.torder, c.T, ntile, c.gm_ns, (uint8_t *)c.part);
    }
    const int64_t npair64 = c.Gnt * (c.Gnt + 1) / 2;
    double *G1 = c.G1 != c.G ? c.G1 : nullptr;
    const auto *planes = (const uint8_t *)c.part;
    if (c.T > 1 && c.TP <= 16)
        hipLaunchKernelGGL(c.gm_ns > 1 ? gram_mod_finish_tasks_kernel<true> : gram_mod_finish_tasks_kernel<false>,
                           dim3((unsigned)(npair64 * (GT / GM_FR))), dim3(256),
                           (size_t)c.TP * (GM_FR * GT + 1) * sizeof(double), st, planes, c.S, c.T, c.TP, tm, ntile,
                           c.gm_ns, c.mu, c.inv_s, c.G, c.Gnt, G1, c.tstar);
    else
        hipLaunchKernelGGL(c.gm_ns > 1 ? gram_mod_finish_kernel<true> : gram_mod_finish_kernel<false>,
                           dim3((unsigned)(npair64 * c.T * (GT / GM_FIN))), dim3(256), 0, st, planes, c.S, c.T, c.TP,
                           tm, ntile, c.gm_ns, c.mu, c.inv_s, c.G, c.Gnt, G1, c.tstar);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

}  // namespace sl0
