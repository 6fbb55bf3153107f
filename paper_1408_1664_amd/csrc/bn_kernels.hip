// HIP kernels (gfx950) for the exact edge-posterior programme.
//
// Lattice layout in HBM (variable i <-> bit i):
//   alpha_i : node-major, 2^(n-1) entries per node, indexed by the subset S
//             of the other n-1 variables with bit i removed (compress_bit).
//   L, Rp   : 2^n entries indexed by the subset mask.
//   scores, beta, Gamma : per node, K(n-1,d) parent sets ranked by size then
//             colex order of the compressed mask.
//
// Tiling: a tile is 2^b consecutive masks (the low b bits vary inside a
// workgroup, the high bits select the tile). Workgroups have 256 threads, those
// of the sweeps 512 or 1024 where the tile is 11 or 12 bits wide.
#include <algorithm>
#include <type_traits>

#include "bn_device.h"
#include "bn_kernels.h"

namespace bnk {

constexpr int kThreads = 256;

// ----------------------------------------------------------- block reduce
// Deterministic tree reduction over the 256 threads of a block (fixed order).
template <class T, class Op>
__device__ inline T block_reduce(T v, T *scratch, Op op) {
    const int t = threadIdx.x;
    scratch[t] = v;
    __syncthreads();
    for (int s = kThreads / 2; s > 0; s >>= 1) {
        if (t < s) scratch[t] = op(scratch[t], scratch[t + s]);
        __syncthreads();
    }
    T r = scratch[0];
    __syncthreads();
    return r;
}

// ------------------------------------------------------------------ setup
// Lane order of the Gamma tile's layout C, where lane t holds the 8-bit
// pattern p = ordC[t] of tile bits 0..7 and reads its 16 doubles at padded
// slots r * 272 + p + p / 16. The patterns with at most d ones fill the first
// 2 * ceil(nlive / 64) groups of 32 lanes (so the same number of waves holds
// them as in popcount order), each going to the group with room where the
// fewest patterns already share its bank pair (p + p / 16) mod 32; the other
// patterns fill the remaining lanes. Computed once per d on the host.
struct LaneOrder {
    uint8_t p[256];
};

static LaneOrder lane_order_c(int d) {
    LaneOrder o{};
    int cntb[8][32] = {}, fill[8] = {};
    int nl = 0;
    for (int p = 0; p < 256; ++p) nl += __builtin_popcount(p) <= d ? 1 : 0;
    const int ng = std::min(8, 2 * ((nl + 63) / 64));
    for (int k = 0; k <= 8; ++k) {
        for (int p = 0; p < 256; ++p) {
            if (__builtin_popcount(p) != k) continue;
            int best = -1;
            if (k <= d) {
                const int f = (p + (p >> 4)) & 31;
                for (int g = 0; g < ng; ++g)
                    if (fill[g] < 32 && (best < 0 || cntb[g][f] < cntb[best][f])) best = g;
                ++cntb[best][f];
            } else {
                best = 0;
                while (fill[best] == 32) ++best;
            }
            o.p[best * 32 + fill[best]++] = (uint8_t)p;
        }
    }
    return o;
}

// C(a, b) for a, b <= 32, built at compile time (row by row, Pascal's rule)
// and read from constant memory by the table kernel.
struct BinomTable {
    uint32_t v[33 * 33];
};
static constexpr BinomTable make_binom() {
    BinomTable t{};
    for (int a = 0; a <= 32; ++a) {
        t.v[a * 33] = 1;
        for (int b = 1; b <= a; ++b)
            t.v[a * 33 + b] = t.v[(a - 1) * 33 + b - 1] + (b < a ? t.v[(a - 1) * 33 + b] : 0u);
    }
    return t;
}
static_assert(make_binom().v[5 * 33 + 2] == 10u && make_binom().v[32 * 33 + 16] == 601080390u &&
                  make_binom().v[32 * 33 + 32] == 1u && make_binom().v[3 * 33 + 5] == 0u,
              "binomial table");
__constant__ BinomTable kBinomTab = make_binom();

// Masks over w bits with at most d ones (every mask when d >= w), ranked by
// size then colex order (numeric order within a size): out[rank] = mask, for
// the masks x in [x0, x0 + 256).
__device__ inline void ranked_chunk(const uint32_t *bn, int w, int d, uint32_t x,
                                    uint32_t *out) {
    if (x >= (1u << w)) return;
    const int k = __popc(x);
    if (k > d) return;
    uint32_t r = Kcount(bn, w, k - 1);
    int j = 0;
    for (int p = 0; p < w; ++p)
        if ((x >> p) & 1) r += C(bn, p, ++j);
    out[r] = x;
}

// Every per-problem table in one launch; the grid is split into ranges of
// workgroups, one range per table (TableGrid):
//   binomials, layer offsets and popcount-ordered masks of the sweep tile,
//   patterns of at most d ones over W bits (numeric order: the w-bit
//   patterns are exactly the first K(w, d) entries), the lane order of the
//   Gamma tile's layout C and its ranked seed masks (range S);
//   the alpha tile's ranked seed masks over bA bits (range A);
//   the ranked high-bit items of an alpha tile over n - 1 - bA bits (I);
//   the compressed parent-set masks in rank order, K(n - 1, d) (F);
//   the sweep tiles' high parts over n - bL bits by popcount, then colex (H);
//   the problem's parameters and zeroed counters (P, one workgroup), the bit
//   planes of binary data (B) and the log-gamma tables of the scores (G).
// A launch of a few workgroups takes 4 to 5 us whatever it does, so what a
// solve prepares before its scores is one launch (n = 10: four before, 24 us).
struct TableGrid {
    uint32_t s, a, i, f, h, p, b, g;   // cumulative ends of the ranges
};
__device__ void pack2(uint32_t wave0, uint32_t step, int n, int m, int W,
                      const uint8_t *__restrict__ data, uint32_t *__restrict__ bits);
__device__ void lgamma_table(uint32_t x0, uint32_t step, int m, int r, int kind, double ess,
                             double *__restrict__ lgt);
__global__ void k_setup(Tables tb, LaneOrder oc, TableGrid g, int bL, int W, int bG, int bA,
                        int d, int N, uint32_t K, ParamBlock pb, SetupArgs sa) {
    const uint32_t blk = blockIdx.x;
    const int t = threadIdx.x;
    // the ranking loops below read binomials one after the other: from LDS
    // (from constant memory they took the set-up of n = 10 from 8.4 to 9.6 us)
    __shared__ uint32_t bn[33 * 33];
    if (blk < g.h) {
        for (int x = t; x < 33 * 33; x += kThreads) bn[x] = kBinomTab.v[x];
        __syncthreads();
    }
    if (blk < g.s) {
        __shared__ uint32_t loff[34];
        if (blk == 0)
            for (int x = t; x < 33 * 33; x += kThreads) tb.binom[x] = bn[x];
        if (t == 0) {
            uint32_t acc = 0;
            for (int l = 0; l <= bL; ++l) {
                loff[l] = acc;
                acc += C(bn, bL, l);
            }
            loff[bL + 1] = acc;
        }
        __syncthreads();
        if (blk == 0 && t <= bL + 1) tb.loff[t] = loff[t];
        const uint32_t x0 = blk * kThreads + t, step = g.s * kThreads;
        // popcount-ordered tile masks: position = offset of the layer + colex rank
        for (uint32_t x = x0; x < (1u << bL); x += step) {
            int k = __popc(x);
            uint32_t r = 0;
            int j = 0;
            for (int p = 0; p < bL; ++p)
                if ((x >> p) & 1) r += C(bn, p, ++j);
            tb.lorder[loff[k] + r] = (uint16_t)x;
        }
        // patterns with at most d ones over W bits, numeric order
        for (uint32_t x = x0; x < (1u << W); x += step) {
            int ones = __popc(x);
            if (ones > d) continue;
            uint32_t pos = 0;
            int above = 0;
            for (int p = W - 1; p >= 0; --p) {
                if ((x >> p) & 1) {
                    if (d - above >= 0) pos += Kcount(bn, p, d - above);
                    ++above;
                }
            }
            tb.pat[pos] = (uint16_t)x;
        }
        // lane order of the Gamma tile's layout C (lane_order_c)
        if (blk == 0) tb.ordC[t] = oc.p[t];
        // ranked seed masks of the Gamma tile (bG bits): size, then colex
        for (uint32_t x = x0; x < (1u << bG); x += step) ranked_chunk(bn, bG, d, x, tb.seedmask);
    } else if (blk < g.a) {
        ranked_chunk(bn, bA, d, (blk - g.s) * kThreads + t, tb.seedA);
    } else if (blk < g.i) {
        ranked_chunk(bn, N - bA, d, (blk - g.a) * kThreads + t, tb.items);
    } else if (blk < g.f) {
        // compressed parent-set masks in rank order
        const uint32_t r = (blk - g.i) * kThreads + t;
        if (r >= K) return;
        int k = 0;
        uint32_t off = 0;
        while (k < d && r >= off + C(bn, N, k)) off += C(bn, N, k++);
        int pos[32];
        colex_unrank(bn, r - off, k, pos);
        uint32_t msk = 0;
        for (int q = 0; q < k; ++q) msk |= 1u << pos[q];
        tb.famask[r] = msk;
    } else if (blk < g.h) {
        ranked_chunk(bn, N + 1 - bL, 64, (blk - g.f) * kThreads + t, tb.hord);
    } else if (blk < g.p) {
        const int n = N + 1;
        if (t < n) {
            sa.arity[t] = pb.arity[t];
            sa.log_q[t] = pb.has_q ? pb.log_q[t] : 0.0;
        }
        if (t <= d) {
            // default rho(k) = 1 / C(n-1, k)
            sa.log_rho[t] = pb.has_rho ? pb.log_rho[t]
                                       : -(lgamma((double)n) - lgamma((double)t + 1.0) -
                                           lgamma((double)(n - t)));
        }
        if (t < 2) sa.cnt[t] = 0ull;
        if (t < 17) sa.done[32 * t] = 0u;
    } else if (blk < g.b) {
        pack2(((blk - g.p) * kThreads + t) >> 6, (g.b - g.p) * (kThreads / 64), N + 1, sa.m,
              (sa.m + 31) / 32, sa.data, sa.bits);
    } else {
        lgamma_table((blk - g.b) * kThreads + t, (g.g - g.b) * kThreads, sa.m, sa.table_r,
                     sa.kind, sa.ess, sa.lgt);
    }
}

// ------------------------------------------------------ a1: local scores
// One workgroup per family (i, G): integer counts N_jk in an LDS histogram,
// then the Dirichlet-multinomial log marginal likelihood in FP64.
__global__ void k_scores(int n, int m, const uint8_t *__restrict__ data,
                         const uint8_t *__restrict__ arity, uint32_t K, int kind, double ess,
                         const uint32_t *__restrict__ famask, double *__restrict__ out) {
    extern __shared__ int hist[];
    __shared__ double red[kThreads];
    __shared__ int par[32];
    __shared__ int npar_s;
    __shared__ int q_s;
    const uint32_t fam = blockIdx.x;
    const int i = fam / K;
    const uint32_t r = fam % K;
    const int t = threadIdx.x;
    if (t == 0) {
        uint32_t msk = famask[r];
        int np = 0, q = 1;
        // mixed radix: the highest variable index is the most significant digit
        for (int p = 30; p >= 0; --p)
            if ((msk >> p) & 1) {
                int var = p < i ? p : p + 1;
                par[np++] = var;
                q *= arity[var];
            }
        npar_s = np;
        q_s = q;
    }
    __syncthreads();
    const int np = npar_s, q = q_s, ri = arity[i];
    const int bins = q * ri;
    for (int b = t; b < bins; b += kThreads) hist[b] = 0;
    __syncthreads();
    const uint8_t *xi = data + (size_t)i * m;
    for (int s = t; s < m; s += kThreads) {
        int key = 0;
        for (int p = 0; p < np; ++p) {
            int var = par[p];
            key = key * arity[var] + data[(size_t)var * m + s];
        }
        const int bin = key * ri + xi[s];
        if (bin < bins) atomicAdd(&hist[bin], 1);  // values >= arity are ignored
    }
    __syncthreads();
    double a_j, a_jk;
    if (kind == 0) {
        a_j = ess / q;
        a_jk = ess / ((double)q * ri);
    } else {
        a_j = ri;
        a_jk = 1.0;
    }
    const double lg_aj = lgamma(a_j), lg_ajk = lgamma(a_jk);
    double acc = 0.0;
    for (int j = t; j < q; j += kThreads) {
        int nj = 0;
        double s = 0.0;
        for (int k = 0; k < ri; ++k) {
            int c = hist[j * ri + k];
            if (c) {
                s += lgamma(a_jk + c) - lg_ajk;
                nj += c;
            }
        }
        if (nj) acc += s + lg_aj - lgamma(a_j + nj);
    }
    double tot = block_reduce(acc, red, [](double a, double b) { return a + b; });
    if (t == 0) out[fam] = tot;
}

// The same scores, four families per workgroup, one wave each, for
// histograms of at most kScoreWaveBins bins (every family of the problem):
// a quarter of the workgroups and no workgroup barriers. Parents, counts and
// the wave's sum stay within the wave (LDS accesses of one wave run in
// order; the wave barriers keep the compiler from moving them). Each lane
// takes four samples per step, with every load of the step issued before
// the counts.
__global__ void __launch_bounds__(kThreads)
k_scores_w(int n, int m, const uint8_t *__restrict__ data, const uint8_t *__restrict__ arity,
           uint32_t K, int kind, double ess, const uint32_t *__restrict__ famask, int max_bins,
           double *__restrict__ out) {
    extern __shared__ int hist_all[];
    __shared__ int par_all[4][32];
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
    const uint32_t fam = blockIdx.x * 4u + (uint32_t)w;
    if (fam >= (uint32_t)n * K) return;          // whole waves
    int *hist = hist_all + w * max_bins;
    int *par = par_all[w];
    const int i = fam / K;
    const uint32_t msk = famask[fam % K];
    // parents in mixed-radix order: the highest variable index is the most
    // significant digit; lane p < 31 tests bit 30 - p
    const bool has = l < 31 && ((msk >> (30 - l)) & 1);
    const uint64_t ball = __ballot(has);
    const int np = __popcll(ball);
    if (has) {
        const int p = 30 - l;
        par[__popcll(ball & ((1ull << l) - 1))] = p < i ? p : p + 1;
    }
    __builtin_amdgcn_wave_barrier();
    int q = 1;
    for (int p = 0; p < np; ++p) q *= arity[par[p]];
    const int ri = arity[i];
    const int bins = q * ri;
    for (int b = l; b < bins; b += 64) hist[b] = 0;
    __builtin_amdgcn_wave_barrier();
    const uint8_t *xi = data + (size_t)i * m;
    constexpr int U = 4;
    for (int s0 = l; s0 < m; s0 += 64 * U) {
        int key[U];
#pragma unroll
        for (int u = 0; u < U; ++u) key[u] = 0;
        for (int p = 0; p < np; ++p) {
            const int var = par[p];
            const int ar = arity[var];
            const uint8_t *row = data + (size_t)var * m;
            int x[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int s = s0 + 64 * u;
                x[u] = s < m ? row[s] : 0;
            }
#pragma unroll
            for (int u = 0; u < U; ++u) key[u] = key[u] * ar + x[u];
        }
        int xv[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int s = s0 + 64 * u;
            xv[u] = s < m ? (int)xi[s] : 0;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int bin = key[u] * ri + xv[u];
            // samples past the end count nowhere; values >= arity are ignored
            if (s0 + 64 * u < m && bin < bins) atomicAdd(&hist[bin], 1);
        }
    }
    __builtin_amdgcn_wave_barrier();
    double acc = 0.0;
    double a_j, a_jk;
    if (kind == 0) {
        a_j = ess / q;
        a_jk = ess / ((double)q * ri);
    } else {
        a_j = ri;
        a_jk = 1.0;
    }
    const double lg_aj = lgamma(a_j), lg_ajk = lgamma(a_jk);
    for (int j = l; j < q; j += 64) {
        int nj = 0;
        double sj = 0.0;
        for (int k = 0; k < ri; ++k) {
            const int c = hist[j * ri + k];
            if (c) {
                sj += lgamma(a_jk + c) - lg_ajk;
                nj += c;
            }
        }
        if (nj) acc += sj + lg_aj - lgamma(a_j + nj);
    }
    for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o);
    if (l == 0) out[fam] = acc;
}

// ----------------------------------------------- prep: prior and gauges
// log B_i(G) = log rho(|G|) + log p(x_i|x_G); beta_i = B_i / 2^E_i with
// E_i = round(max_G log2 B_i(G)) in the scaled form (0 in log form); the same
// for q(k) with a per-layer exponent F_k.
// Scores of one row per workgroup row (blockIdx.x = node), kPrepChunk
// entries per workgroup (blockIdx.y).
//
// Per-node scale for the linear alpha tiles. Every alpha_i(S) / q(|S|) is a
// sum of B_i(G) over G subset S that includes B_i(empty), and none exceeds
// K(n-1, d) max_G B_i(G). Node i therefore gets one power of two (in the
// log-space system with an offset besides, the largest score) that puts
// B_i(empty) near 2^-1000, and
// the node is held in plain doubles when max_G B_i(G) / B_i(empty) is below
// 2^1900: no partial sum can then leave the double range (K(n-1, d) <
// 2^31). betal_i(r) = B_i(r) under that scale. Nodes that do not qualify
// (linok = 0) are computed in the number system proper.
// emax (nullable) receives floor(log2 max_G B_i(G)) + 1 per node (the bound
// the fused sweeps test their blocks against).
constexpr uint32_t kPrepChunk = 2048;
template <class P>
__global__ void k_prep(int n, int d, uint32_t K, const uint32_t *binom,
                       const double *__restrict__ logp, const double *__restrict__ log_rho,
                       const double *__restrict__ log_q, int gauge,
                       typename P::V *__restrict__ beta, typename P::V *__restrict__ qt,
                       double *__restrict__ gauge_exp, uint32_t *fbA, uint32_t *fbG,
                       uint32_t *rtG, double *__restrict__ betal,
                       typename P::Anchor *__restrict__ anc, int *__restrict__ linok,
                       int *__restrict__ emax) {
    __shared__ double red[kThreads];
    const int i = blockIdx.x;
    const uint32_t chunk = blockIdx.y;      // entries [chunk * kPrepChunk, ...) of row i
    const int t = threadIdx.x;
    if (i == 0 && chunk == 0 && t == 0) {
        if (fbA) fbA[0] = 0;
        if (fbG) fbG[0] = 0;
        if (rtG) rtG[0] = 0;
    }
    const int N = n - 1;
    // cum[k] = K(N, k): the parent sets of rank below it have at most k members
    __shared__ uint32_t cum[33];
    if (t <= d && t < 33) cum[t] = Kcount(binom, N, t);
    __syncthreads();
    auto size_of = [&](uint32_t r) {
        int k = 0;
        while (k < d && r >= cum[k]) ++k;
        return k;
    };
    // the row's maximum (every chunk of the row reads the whole row)
    double mx = -__builtin_huge_val();
    for (int k = 0; k <= d; ++k) {               // size by size: one log rho each
        double mk = -__builtin_huge_val();
        for (uint32_t r = (k ? cum[k - 1] : 0u) + t; r < cum[k]; r += kThreads)
            mk = fmax(mk, logp[(size_t)i * K + r]);
        mx = fmax(mx, log_rho[k] + mk);
    }
    mx = block_reduce(mx, red, [](double a, double b) { return fmax(a, b); });
    const double E = (gauge && mx > -1e300) ? rint(mx * 1.4426950408889634074) : 0.0;
    // the row's linear scale (nullable outputs): anchored at B_i(empty), held in
    // doubles when the largest score lies less than 2^1900 above it
    auto gauged = [&](double lb) { return P::from_log(lb - E * 0.69314718055994530942); };
    typename P::Anchor T{};
    bool lin = false;
    if (betal) {
        const typename P::V b0 = gauged(log_rho[0] + logp[(size_t)i * K]);
        const double l2 = P::log2_of(gauged(mx));
        lin = P::anchor_below(b0, gauged(mx), &T) && l2 - P::log2_of(b0) <= 1900.0;
        if (chunk == 0 && t == 0) {
            anc[i] = T;
            linok[i] = lin ? 1 : 0;
            if (emax) emax[i] = l2 > -1e300 ? (int)l2 + 1 : -(1 << 26);
        }
    }
    const uint32_t r1 = min(K, (chunk + 1) * kPrepChunk);
    for (uint32_t r = chunk * kPrepChunk + t; r < r1; r += kThreads) {
        const typename P::V b = gauged(log_rho[size_of(r)] + logp[(size_t)i * K + r]);
        beta[(size_t)i * K + r] = b;
        if (lin) betal[(size_t)i * K + r] = P::to_lin(b, T);
    }
    if (chunk == 0 && t == 0) gauge_exp[i] = E;
    if (i == 0 && chunk == 0) {
        for (int k = t; k < n; k += kThreads) {
            double lq = log_q[k];
            double F = (gauge && lq > -1e300) ? rint(lq * 1.4426950408889634074) : 0.0;
            qt[k] = P::from_log(lq - F * 0.69314718055994530942);
            gauge_exp[n + k] = F;
        }
    }
}

// ------------------------------------------------ a2: alpha (upward zeta)
__device__ inline double shfl_xor_v(double v, int m) { return __shfl_xor(v, m); }
__device__ inline X32 shfl_xor_v(X32 v, int m) {
    return X32{__shfl_xor(v.f, m), __shfl_xor(v.e, m)};
}

// Padded LDS index for 2^13-entry tiles: one spare slot every 32 entries
// keeps the transposed accesses of the alpha tile nearly free of bank
// conflicts.
__device__ inline uint32_t pad32(uint32_t x) { return x + (x >> 5); }

template <class P, int NR>
__device__ inline void reg_zeta_up(typename P::V *v, int q) {
#pragma unroll
    for (int r = 0; r < NR; ++r)
        if ((r >> q) & 1) v[r] = P::add(v[r], v[r ^ (1 << q)]);
}

// Workgroup (i, H): the tile of node i's lattice (n-1 bits) whose high
// N-13 bits are H; tile entry x = the low 13 bits, 256 threads x 32 entries.
//  1. Seeds Z(G_L) = sum_{G_H subset H, |G_H| <= d-|G_L|} beta_i(G_H + G_L)
//     for every |G_L| <= d. The G_H are the small masks over H's bits (a
//     ranked table); their contribution to the rank of G_L + G_H is
//     tabulated once per workgroup, so a (seed, G_H) pair costs one LDS
//     read and one beta gather. Each seed is summed by a group of lanes and
//     reduced by cross-lane shuffles.
//  2. Upward zeta over the 13 tile bits in registers, in three layouts:
//     bits 0..4 (thread t holds x = ord8[t]*32 + r; ord8 lists the 8-bit
//     patterns by popcount, so the waves whose entries are all structural
//     zeros -- more than d ones above bit 4, Def. 1 -- skip it), bits 5..9
//     and bits 10..12 (x = r*256 + t), with two LDS transposes.
//  3. alpha = q(|S|) * t(S), stored coalesced from the last layout.
template <class P>
__device__ __forceinline__ void alpha_tile(int n, int d, uint32_t K, int use_prk, const Tables &tb,
                                           const typename P::V *__restrict__ beta,
                                           const typename P::V *__restrict__ qt,
                                           const typename P::Store &alpha,
                                           unsigned long long *cnt, uint32_t blk) {
    using V = typename P::V;
    constexpr int bA = 13, NR = 32;
    extern __shared__ unsigned char smem[];
    V *tile = reinterpret_cast<V *>(smem);                         // pad32(2^13)
    uint32_t *sbin = reinterpret_cast<uint32_t *>(tile + 8192 + 256);
    uint16_t *prk = reinterpret_cast<uint16_t *>(sbin + 33 * 33);  // (d+1) x items
    __shared__ int hb[32];
    __shared__ uint32_t offN[34];
    __shared__ V sq[32];
    __shared__ uint8_t ord8[256];
    const int N = n - 1;
    const int hA = N - bA;
    const int i = blk >> hA;
    const uint32_t H = blk & ((1u << hA) - 1);
    const int t = threadIdx.x;
    for (int x = t; x < 33 * 33; x += kThreads) sbin[x] = tb.binom[x];
    if (t < hA && ((H >> t) & 1)) hb[__popc(H & ((1u << t) - 1))] = bA + t;
    if (t < n) sq[t] = qt[t];
    for (uint32_t x = t; x < 8192 + 256; x += kThreads) tile[x] = P::zero();
    __syncthreads();
    const uint32_t *bn = sbin;
    const int h = __popc(H);
    if (t <= d + 1) offN[t] = Kcount(bn, N, t - 1);
    {   // ord8: 8-bit patterns by popcount (then value)
        const int k = __popc(t);
        uint32_t r = Kcount(bn, 8, k - 1);
        int j = 0;
        for (int p = 0; p < 8; ++p)
            if ((t >> p) & 1) r += C(bn, p, ++j);
        ord8[r] = (uint8_t)t;
    }
    // partial ranks of the high-bit items: prk[s * nit + it] = sum_q C(hb[e_q], s + q)
    const uint32_t nit = Kcount(bn, h, d);
    for (uint32_t it = t; use_prk && it < nit; it += kThreads) {
        int k = 0;
        uint32_t off = 0, toff = 0;
        while (it >= off + C(bn, h, k)) {
            off += C(bn, h, k);
            toff += C(bn, hA, k);
            ++k;
        }
        const uint32_t m = tb.items[toff + (it - off)];
        for (int s = 0; s + k <= d; ++s) {
            uint32_t r = 0, mm = m;
            int q = 0;
            while (mm) {
                const int e = __ffs(mm) - 1;
                mm &= mm - 1;
                r += C(bn, hb[e], s + (++q));
            }
            prk[s * nit + it] = (uint16_t)r;
        }
    }
    __syncthreads();
    const V *bi = beta + (size_t)i * K;

    // 1. seeds, one size class s = |G_L| at a time
    for (int s = 0; s <= d && s <= bA; ++s) {
        const uint32_t nseed = C(bn, bA, s);
        const uint32_t items = Kcount(bn, h, d - s);    // G_H with |G_H| <= d - s
        int grp = 1;                                    // lanes per seed, power of 2 <= 64
        while (grp < 64 && (uint32_t)grp < items && (uint32_t)(grp * 2) * nseed <= kThreads)
            grp *= 2;
        const uint32_t per_round = kThreads / grp;
        const uint32_t seedoff = Kcount(bn, bA, s - 1);
        for (uint32_t base = 0; base < nseed; base += per_round) {
            const uint32_t seed = base + t / grp;
            const int lane = t % grp;
            V acc = P::zero();
            if (seed < nseed) {
                constexpr int B = 4;
                for (uint32_t it0 = lane; it0 < items; it0 += B * grp) {
                    V bv[B];
#pragma unroll
                    for (int u = 0; u < B; ++u) {
                        const uint32_t it = it0 + u * grp;
                        if (it < items) {
                            // size of item it: items are ordered by size
                            int k = 0;
                            uint32_t off = 1, toff = 0;
                            while (it >= off) {
                                toff += C(bn, hA, k);
                                off += C(bn, h, ++k);
                            }
                            uint32_t pr;
                            if (use_prk) {
                                pr = prk[s * nit + it];
                            } else {
                                uint32_t m = tb.items[toff + it - (off - C(bn, h, k))];
                                pr = 0;
                                int q = 0;
                                while (m) {
                                    const int e = __ffs(m) - 1;
                                    m &= m - 1;
                                    pr += C(bn, hb[e], s + (++q));
                                }
                            }
                            bv[u] = bi[offN[s + k] + seed + pr];
                        }
                    }
#pragma unroll
                    for (int u = 0; u < B; ++u)
                        if (it0 + u * grp < items) acc = P::add(acc, bv[u]);
                }
            }
            for (int w = grp / 2; w > 0; w >>= 1) acc = P::add(acc, shfl_xor_v(acc, w));
            if (lane == 0 && seed < nseed) tile[pad32(tb.seedA[seedoff + seed])] = acc;
        }
    }
    __syncthreads();

    // 2. upward zeta in registers
    V v[NR];
    const uint32_t pt = ord8[t];
    const bool live = __popc(pt) <= d;    // bits 5..12 of every entry this thread holds
    if (__any(live)) {
#pragma unroll
        for (int r = 0; r < NR; ++r) v[r] = tile[pad32((pt << 5) | r)];
#pragma unroll
        for (int q = 0; q < 5; ++q) reg_zeta_up<P, NR>(v, q);
#pragma unroll
        for (int r = 0; r < NR; ++r) tile[pad32((pt << 5) | r)] = v[r];
    }
    __syncthreads();
    const uint32_t tlo = t & 31, thi = t >> 5;   // layout B: x = thi*1024 + r*32 + tlo
#pragma unroll
    for (int r = 0; r < NR; ++r) v[r] = tile[pad32((thi << 10) | (r << 5) | tlo)];
#pragma unroll
    for (int q = 0; q < 5; ++q) reg_zeta_up<P, NR>(v, q);
    __syncthreads();
#pragma unroll
    for (int r = 0; r < NR; ++r) tile[pad32((thi << 10) | (r << 5) | tlo)] = v[r];
    __syncthreads();
#pragma unroll
    for (int r = 0; r < NR; ++r) v[r] = tile[pad32(r * kThreads + t)];
#pragma unroll
    for (int q = 2; q < 5; ++q) reg_zeta_up<P, NR>(v, q);     // tile bits 10..12

    // 3. alpha = q(|S|) t(S)
    const uint64_t base = ((uint64_t)i << N) | ((uint64_t)H << bA);
#pragma unroll
    for (int r = 0; r < NR; ++r) {
        const uint32_t x = r * kThreads + t;
        P::store(alpha, base + x, P::mul(sq[h + __popc(x)], v[r]), cnt);
    }
}

template <class P>
__global__ void __launch_bounds__(kThreads)
k_alpha(int n, int d, uint32_t K, int use_prk, Tables tb, const typename P::V *__restrict__ beta,
        const typename P::V *__restrict__ qt, typename P::Store alpha,
        unsigned long long *cnt) {
    alpha_tile<P>(n, d, K, use_prk, tb, beta, qt, alpha, cnt, blockIdx.x);
}

// Recomputation of the tiles listed by k_alpha_lin (list[0] entries,
// list[1 + j] = i * 2^(N-13) + H): the grid walks the list.
template <class P>
__global__ void __launch_bounds__(kThreads)
k_alpha_fb(int n, int d, uint32_t K, int use_prk, Tables tb,
           const typename P::V *__restrict__ beta, const typename P::V *__restrict__ qt,
           typename P::Store alpha, unsigned long long *cnt, const uint32_t *list) {
    const uint32_t ntile = list[0];
    for (uint32_t it = blockIdx.x; it < ntile; it += gridDim.x) {
        __syncthreads();
        alpha_tile<P>(n, d, K, use_prk, tb, beta, qt, alpha, cnt, list[1 + it]);
    }
}

__device__ inline void fb_push(uint32_t *fb, uint32_t id) {
    const uint32_t k = atomicAdd(fb, 1u);
    fb[1 + k] = id;
}

template <int NR>
__device__ inline void lin_zeta_up(double *v, int q) {
#pragma unroll
    for (int r = 0; r < NR; ++r)
        if ((r >> q) & 1) v[r] += v[r ^ (1 << q)];
}

// Binomial coefficient for small arguments; folds to a constant when its
// arguments are compile-time constants.
__host__ __device__ constexpr uint32_t cbin(int a, int b) {
    if (b < 0 || b > a) return 0;
    uint32_t r = 1;
    for (int k = 1; k <= b; ++k) r = r * (uint32_t)(a - b + k) / (uint32_t)k;
    return r;
}

// Colex rank of the set bits of a 5-bit mask (bit p is element p).
__host__ __device__ constexpr uint32_t colex5(uint32_t r) {
    uint32_t c = 0;
    int j = 0;
    for (int p = 0; p < 5; ++p)
        if ((r >> p) & 1) c += cbin(p, ++j);
    return c;
}

// Seeds of the linear alpha tiles, in a kernel of their own (the gather of
// k_alpha's first step, at high occupancy). For tile (i, H) and every G_L
// over the 13 tile bits with |G_L| < d,
//   Zs[(i, H)][rank(G_L)] = sum_{G_H subset H, |G_H| <= d - |G_L|} betal_i(G_H + G_L),
// rank = size, then colex order. A seed with |G_L| = d is betal_i(G_L)
// itself, the same for every H: k_alpha_lin reads those from betal. For one G_H the G_L of one size s give a
// contiguous run of ranks of G_H + G_L, so consecutive lanes take
// consecutive G_L (coalesced loads) and groups of lanes split the G_H;
// their partial sums meet in LDS in a fixed order.
template <class P>
__global__ void __launch_bounds__(kThreads)
k_alpha_seeds(int n, int d, uint32_t K, uint32_t KS, int use_prk, Tables tb,
              const double *__restrict__ betal, const int *__restrict__ linok,
              double *__restrict__ Zs) {
    constexpr int bA = 13;
    extern __shared__ unsigned char smem[];
    uint32_t *sbin = reinterpret_cast<uint32_t *>(smem);
    uint16_t *prk = reinterpret_cast<uint16_t *>(sbin + 33 * 33);  // (d+1) x items
    __shared__ int hb[32];
    __shared__ uint32_t offN[34];
    __shared__ double part[kThreads];
    const int N = n - 1;
    const int hA = N - bA;
    const int i = blockIdx.x >> hA;
    const uint32_t H = blockIdx.x & ((1u << hA) - 1);
    const int t = threadIdx.x;
    if (!linok[i]) return;
    for (int x = t; x < 33 * 33; x += kThreads) sbin[x] = tb.binom[x];
    if (t < hA && ((H >> t) & 1)) hb[__popc(H & ((1u << t) - 1))] = bA + t;
    __syncthreads();
    const uint32_t *bn = sbin;
    const int h = __popc(H);
    if (t <= d + 1) offN[t] = Kcount(bn, N, t - 1);
    const uint32_t nit = Kcount(bn, h, d);
    uint8_t *itk = reinterpret_cast<uint8_t *>(prk + (use_prk ? (size_t)(d + 1) * nit : 0));
    for (uint32_t it = t; use_prk && it < nit; it += kThreads) {
        int k = 0;
        uint32_t off = 0, toff = 0;
        while (it >= off + C(bn, h, k)) {
            off += C(bn, h, k);
            toff += C(bn, hA, k);
            ++k;
        }
        itk[it] = (uint8_t)k;
        const uint32_t m = tb.items[toff + (it - off)];
        for (int s = 0; s + k <= d; ++s) {
            uint32_t r = 0, mm = m;
            int q = 0;
            while (mm) {
                const int e = __ffs(mm) - 1;
                mm &= mm - 1;
                r += C(bn, hb[e], s + (++q));
            }
            prk[s * nit + it] = (uint16_t)r;
        }
    }
    __syncthreads();
    const double *bi = betal + (size_t)i * K;
    double *out = Zs + (size_t)blockIdx.x * KS;
    for (int s = 0; s < d && s <= bA; ++s) {
        const uint32_t nseed = C(bn, bA, s);
        const uint32_t items = Kcount(bn, h, d - s);
        const uint32_t seedoff = Kcount(bn, bA, s - 1);
        for (uint32_t base = 0; base < nseed; base += kThreads) {
            const uint32_t cnt = min(nseed - base, (uint32_t)kThreads);
            // lanes per seed: at most 16, whose parts one lane then adds in turn (with
            // every lane of the workgroup on the one seed of size 0 that chain took
            // most of the kernel: n = 16 17 -> 8 us, n = 20, d = 4 25 -> 15 us)
            const uint32_t ni = min(min((uint32_t)kThreads / cnt, 16u), items);
            const uint32_t seed = base + t % cnt, il = t / cnt;
            double acc = 0.0;
            if (il < ni) {
                constexpr int B = 8;
                for (uint32_t it0 = il; it0 < items; it0 += B * ni) {
                    double bv[B];
#pragma unroll
                    for (int u = 0; u < B; ++u) {
                        const uint32_t it = it0 + u * ni;
                        bv[u] = 0.0;
                        if (it < items) {
                            int k;
                            uint32_t pr;
                            if (use_prk) {
                                k = itk[it];
                                pr = prk[s * nit + it];
                            } else {
                                k = 0;
                                uint32_t off = 1, toff = 0;
                                while (it >= off) {
                                    toff += C(bn, hA, k);
                                    off += C(bn, h, ++k);
                                }
                                uint32_t m = tb.items[toff + it - (off - C(bn, h, k))];
                                pr = 0;
                                int q = 0;
                                while (m) {
                                    const int e = __ffs(m) - 1;
                                    m &= m - 1;
                                    pr += C(bn, hb[e], s + (++q));
                                }
                            }
                            bv[u] = bi[offN[s + k] + seed + pr];
                        }
                    }
#pragma unroll
                    for (int u = 0; u < B; ++u) acc += bv[u];
                }
            }
            if (ni == 1) {
                if (il == 0) out[seedoff + seed] = acc;
            } else {
                part[t] = acc;
                __syncthreads();
                if ((uint32_t)t < cnt) {
                    double z = 0.0;
                    for (uint32_t j = 0; j < ni; ++j) z += part[j * cnt + t];
                    out[seedoff + base + t] = z;
                }
                __syncthreads();
            }
        }
    }
}

// Store NR doubles of a thread (entry r at index base + r * stride, scaled
// by q(|r| + const), qr indexed by the popcount of r) in the solve's number
// system. The X32 form checks the exponent range once per thread and takes
// the per-entry saturation / flush path only when some entry needs it.
template <class P, int NR>
__device__ inline void store_tile_lin(const typename P::Store &st, uint64_t ubase,
                                      uint32_t toff, uint32_t stride, const double *v,
                                      const typename P::V *qr, typename P::Anchor T,
                                      unsigned long long *cnt) {
    uint32_t nsat = 0, nfl = 0;
#pragma unroll
    for (int r = 0; r < NR; ++r)
        P::store_lin_q(st, ubase + (toff + (uint32_t)r * stride), v[r],
                       qr[__builtin_popcount(r)], T, nsat, nfl);
    if (cnt && (nsat | nfl)) {
        if (nsat) atomicAdd(cnt, (unsigned long long)nsat);
        if (nfl) atomicAdd(cnt + 1, (unsigned long long)nfl);
    }
}

template <int NR>
__device__ inline void store_tile_lin_x32(const PolX32::Store &st, uint64_t ubase,
                                          uint32_t toff, uint32_t stride, const double *v,
                                          const X32 *qr, int T, unsigned long long *cnt) {
    float *fp = st.f + ubase;           // uniform bases, 32-bit per-thread offsets
    uint8_t *bp = st.b + ubase;
    int b[NR];
    bool ok = true;
#pragma unroll
    for (int r = 0; r < NR; ++r) {
        const X32 q = qr[__builtin_popcount(r)];
        const double z = v[r] * (double)q.f;
        int k;
        const float f = PolX32::lin_encode(z, &k);
        b[r] = ((T + q.e) >> 6) + k + kX32Bias;
        ok = ok && z > 0.0 && b[r] >= 1 && b[r] <= 255;
        fp[toff + (uint32_t)r * stride] = f;      // rewritten below if out of range
    }
    if (ok) {
#pragma unroll
        for (int r = 0; r < NR; ++r) bp[toff + (uint32_t)r * stride] = (uint8_t)b[r];
    } else {
        uint32_t nsat = 0, nfl = 0;
#pragma unroll
        for (int r = 0; r < NR; ++r)
            PolX32::store_lin_q(st, ubase + (toff + (uint32_t)r * stride), v[r],
                                qr[__builtin_popcount(r)], T, nsat, nfl);
        if (cnt && (nsat | nfl)) {
            if (nsat) atomicAdd(cnt, (unsigned long long)nsat);
            if (nfl) atomicAdd(cnt + 1, (unsigned long long)nfl);
        }
    }
}

template <>
__device__ inline void store_tile_lin<PolX32, 16>(const PolX32::Store &st, uint64_t ubase,
                                                  uint32_t toff, uint32_t stride,
                                                  const double *v, const X32 *qr, int T,
                                                  unsigned long long *cnt) {
    store_tile_lin_x32<16>(st, ubase, toff, stride, v, qr, T, cnt);
}

// Colex rank of the set bits of a 4-bit mask (bit p is element p).
__host__ __device__ constexpr uint32_t colex4(uint32_t r) {
    uint32_t c = 0;
    int j = 0;
    for (int p = 0; p < 4; ++p)
        if ((r >> p) & 1) c += cbin(p, ++j);
    return c;
}

__host__ __device__ constexpr size_t align16(size_t x) { return (x + 15) & ~(size_t)15; }

// Padded LDS index: one spare slot every 16 entries.
__device__ inline uint32_t padx(uint32_t x) { return x + (x >> 4); }

// Seeds of the linear alpha tiles by blocks of tiles (same outputs as
// k_alpha_seeds). Workgroup (i, Hh) covers the 2^b tiles H = Hh * 2^b + Hl
// (4 <= b <= 8 low bits of H). With G_H = G_lo + G_hi, G_lo over the
// b low bits of H and G_hi over the rest,
//   Z(H, G_L) = sum_{G_lo subset Hl} F(G_lo),
//   F(G_lo) = sum_{G_hi subset Hh, |G_hi| <= d - |G_L| - |G_lo|} betal_i(G_L + G_lo + G_hi),
// i.e. an upward zeta over the b low bits of a vector that is nonzero only
// where |G_L| + |G_lo| <= d. The seeds go in chunks of 16: thread (g, u) holds
// F for seed g and G_lo = u * 16 + r in 16 registers (bits 0..3), then, after
// an LDS transpose, bits 4..b-1. Score ranks are size, then colex: the part
// of G_hi (with the size offset) comes from a table built per workgroup,
// hiP[m][j] for the j-th subset of Hh and m smaller elements. Workgroup
// (i, Hh, y) takes every gridDim.y-th chunk from chunk y.
template <class P>
__global__ void __launch_bounds__(kThreads)
k_alpha_seeds_blk(int n, int d, uint32_t K, uint32_t KS, int b, uint32_t nhiMax, Tables tb,
                  const double *__restrict__ betal, const int *__restrict__ linok,
                  double *__restrict__ Zs) {
    constexpr int bA = 13;
    extern __shared__ unsigned char smem[];
    double *buf = reinterpret_cast<double *>(smem);                   // 16 x 256, padx
    uint32_t *sbin = reinterpret_cast<uint32_t *>(buf + 4096 + 256);  // 33 x 33
    uint32_t *hiP = sbin + 33 * 33;                                   // (d + 1) x nhiMax
    __shared__ uint32_t hcnt[34];
    __shared__ int hpos[32];
    __shared__ int snh;
    const int N = n - 1, hA = N - bA, hh = hA - b;
    const int i = blockIdx.x >> hh;
    const uint32_t Hh = blockIdx.x & ((1u << hh) - 1);
    const int t = threadIdx.x;
    if (!linok[i]) return;
    for (int x = t; x < 33 * 33; x += kThreads) sbin[x] = tb.binom[x];
    if (t == 0) {
        int c = 0;
        for (int p = 0; p < hh; ++p)
            if ((Hh >> p) & 1) hpos[c++] = bA + b + p;   // mask positions of Hh's elements
        snh = c;
    }
    __syncthreads();
    const uint32_t *bn = sbin;
    const int nh = snh;
    const uint32_t nhi = Kcount(bn, nh, d);
    if (t <= d) hcnt[t] = Kcount(bn, nh, t);         // subsets of Hh with at most t elements
    for (uint32_t j = t; j < nhi; j += kThreads) {
        int k = 0;
        uint32_t off = 0;
        while (j >= off + C(bn, nh, k)) off += C(bn, nh, k++);
        int el[8];
        colex_unrank(bn, j - off, k, el);
        for (int m = 0; m <= d; ++m) {
            uint32_t r = (m + k >= 1) ? Kcount(bn, N, m + k - 1) : 0u;
            for (int q = 0; q < k; ++q) r += C(bn, hpos[el[q]], m + q + 1);
            hiP[m * nhiMax + j] = r;
        }
    }
    __syncthreads();
    const double *bi = betal + (size_t)i * K;
    const uint32_t g = t >> 4, u = t & 15;
    const uint32_t nu = 1u << (b - 4);                 // thread values of G_lo bits 4..b-1
    const uint64_t tile0 = (uint64_t)blockIdx.x << b;  // tile index (i, Hh, Hl = 0)
    const uint32_t nent = 16u << b;
    // chunks of 16 seed ranks, split over gridDim.y workgroups of the same tiles
    for (uint32_t c0 = 16 * blockIdx.y; c0 < KS; c0 += 16 * gridDim.y) {
        const uint32_t rk = c0 + g;
        double v[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) v[r] = 0.0;
        if (rk < KS && u < nu) {
            const uint32_t GL = tb.seedA[rk];
            const int s = __popc(GL);
            const uint32_t cl = rk - Kcount(bn, bA, s - 1);   // colex rank of G_L
            for (int r = 0; r < 16; ++r) {
                const uint32_t Glo = (u << 4) | (uint32_t)r;
                const int m = s + __popc(Glo);
                if (m > d) continue;
                uint32_t lp = cl;
                int q = s;
                uint32_t rest = Glo;
                while (rest) {
                    const int p = __ffs(rest) - 1;
                    rest &= rest - 1;
                    lp += C(bn, bA + p, ++q);
                }
                const uint32_t *hp = hiP + m * nhiMax;
                const uint32_t nsub = hcnt[d - m];
                // eight scores in flight, added in order (one at a time this kernel
                // took 40 us at n = 22 instead of 38, n = 25 125 instead of 112)
                double acc = 0.0;
                for (uint32_t j0 = 0; j0 < nsub; j0 += 8) {
                    double x[8];
#pragma unroll
                    for (int k = 0; k < 8; ++k) {
                        const uint32_t j = j0 + k;
                        x[k] = j < nsub ? bi[lp + hp[min(j, nsub - 1)]] : 0.0;
                    }
#pragma unroll
                    for (int k = 0; k < 8; ++k) acc += x[k];
                }
                v[r] = acc;
            }
        }
        // upward zeta over G_lo bits 0..3
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int r = 0; r < 16; ++r)
                if ((r >> q) & 1) v[r] += v[r ^ (1 << q)];
        if (u < nu) {
#pragma unroll
            for (int r = 0; r < 16; ++r) buf[padx((g << 8) | (u << 4) | (uint32_t)r)] = v[r];
        }
        __syncthreads();
        // thread (g, u = G_lo bits 0..3), registers r = G_lo bits 4..b-1
#pragma unroll
        for (int r = 0; r < 16; ++r)
            v[r] = ((uint32_t)r < nu) ? buf[padx((g << 8) | ((uint32_t)r << 4) | u)] : 0.0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if (q < b - 4) {
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    if ((r >> q) & 1) v[r] += v[r ^ (1 << q)];
            }
        }
        __syncthreads();
        // tile-major for the stores: entry (Hl, g) at Hl * 16 + g
#pragma unroll
        for (int r = 0; r < 16; ++r)
            if ((uint32_t)r < nu) buf[padx((((uint32_t)r << 4) | u) * 16 + g)] = v[r];
        __syncthreads();
        for (uint32_t e = t; e < nent; e += kThreads) {
            const uint32_t Hl = e >> 4, gg = e & 15;
            if (c0 + gg < KS) Zs[(tile0 | Hl) * KS + c0 + gg] = buf[padx(e)];
        }
        __syncthreads();
    }
}

// LDS of a linear alpha tile: one 32-bit plane of 16 rows of 64 words per wave
// (4 spare words per row keep the scattered side of the transpose off each
// other's banks), a tile's seeds, the seeds of four subtiles, and the sizes of
// the sets of 10 bits by rank.
constexpr uint32_t kAlphaRow = 68, kAlphaPlane = 16 * kAlphaRow;
__host__ __device__ inline uint32_t sets10(int d) {
    uint32_t kf = 0;
    for (int k = 0; k <= 10 && k <= d; ++k) kf += cbin(10, k);
    return kf;
}
static size_t alpha_lin_lds(int d, uint32_t KS) {
    const uint32_t kf = sets10(d);
    return (size_t)4 * kAlphaPlane * 4 + 8 * (size_t)(KS + (d <= 13 ? cbin(13, d) : 0u)) +
           (size_t)4 * (kf + 8) * 8 + kf;
}

// Register bit Q exchanged with lane bit 4 (row16) or 5: entries that differ
// in it trade places between the register pair and the lane pair.
template <int NR, bool ROW16>
__device__ __forceinline__ void swap_lane_bit(double *v, int q) {
#pragma unroll
    for (int r = 0; r < NR; ++r) {
        if ((r >> q) & 1) continue;
        const int s = r | (1 << q);
        const uint32_t al = (uint32_t)__double2loint(v[r]), ah = (uint32_t)__double2hiint(v[r]);
        const uint32_t bl = (uint32_t)__double2loint(v[s]), bh = (uint32_t)__double2hiint(v[s]);
        const auto l = ROW16 ? __builtin_amdgcn_permlane16_swap(al, bl, false, false)
                             : __builtin_amdgcn_permlane32_swap(al, bl, false, false);
        const auto h = ROW16 ? __builtin_amdgcn_permlane16_swap(ah, bh, false, false)
                             : __builtin_amdgcn_permlane32_swap(ah, bh, false, false);
        v[r] = __hiloint2double((int)h[0], (int)l[0]);
        v[s] = __hiloint2double((int)h[1], (int)l[1]);
    }
}

// Order of one wave's LDS accesses: they complete in the order of issue, so
// only the compiler has to keep it.
__device__ __forceinline__ void wave_lds_order() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Stores of 16 entries per lane, entry r * 64 + lane, z = v[r] in the number
// system's form. The significands go out as they stand (256 B per wave
// store); the exponent bytes are transposed through the wave's LDS plane so
// that a lane stores 16 consecutive ones (1 KB per wave store).
__device__ __forceinline__ void alpha_store_x32(const PolX32::Store &alpha, uint64_t ub,
                                                uint32_t lane, uint32_t *pl, const double *v,
                                                const X32 *qr, int T, unsigned long long *cnt) {
    constexpr int NR = 16;
    float *fp = alpha.f + ub;
    uint8_t *bytes = reinterpret_cast<uint8_t *>(pl);
    double qf[5];
    int qb[5];
#pragma unroll
    for (int m = 0; m < 5; ++m) {
        qf[m] = (double)qr[m].f;
        qb[m] = ((T + qr[m].e) >> 6) + kX32Bias;
    }
    // fast path: every entry a positive normal double with its byte in 1..255
    float fq[NR];
    int bq[NR], bmin = 255, bmax = 1;
    uint32_t hmin = 0x7fefffffu, hmax = 0x00100000u;
#pragma unroll
    for (int r = 0; r < NR; ++r) {
        const int m = __builtin_popcount(r);
        const double z = v[r] * qf[m];
        int k;
        const uint32_t hi = (uint32_t)__double2hiint(z);
        fq[r] = PolX32::lin_encode_normal(z, &k);
        bq[r] = qb[m] + k;
        bmin = min(bmin, bq[r]);
        bmax = max(bmax, bq[r]);
        hmin = min(hmin, hi);
        hmax = max(hmax, hi);
    }
    if (bmin < 1 || bmax > 255 || hmin < 0x00100000u || hmax > 0x7fefffffu) {
        uint32_t nsat = 0, nfl = 0;
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            const double z = v[r] * qf[__builtin_popcount(r)];
            int k;
            const float f = PolX32::lin_encode(z, &k);
            const int b = qb[__builtin_popcount(r)] + k;
            const bool zero = !(z > 0.0);
            const bool fl = !zero && b < 1;
            const bool sat = !zero && b > 255;
            nfl += fl ? 1u : 0u;
            nsat += sat ? 1u : 0u;
            fq[r] = (zero || fl) ? 0.0f : (sat ? 4.0e9f : f);
            bq[r] = (zero || fl) ? 0 : (sat ? 255 : b);
        }
        if (cnt && (nsat | nfl)) {
            if (nsat) atomicAdd(cnt, (unsigned long long)nsat);
            if (nfl) atomicAdd(cnt + 1, (unsigned long long)nfl);
        }
    }
#pragma unroll
    for (int r = 0; r < NR; ++r) fp[(uint32_t)r * 64u + lane] = fq[r];
    wave_lds_order();
#pragma unroll
    for (int r = 0; r < NR; ++r) bytes[r * 64 + lane] = (uint8_t)bq[r];
    wave_lds_order();
    reinterpret_cast<uint4 *>(alpha.b + ub)[lane] = reinterpret_cast<const uint4 *>(bytes)[lane];
}

// Linear-tile form of k_alpha. A workgroup takes 2^tl consecutive tiles (i, H)
// of one node in turn, each the same 13-bit tile as k_alpha's. The seeds come
// from k_alpha_seeds, already as doubles under the node's scale, and the upward
// zeta runs on doubles, one FP64 add per step. What bounds a tile is latency:
// stores, LDS and vector unit are each busy for about half of its time, so the
// split keeps the waves apart. A tile's seeds of fewer than d bits are few
// (92 at d = 3) and are read a tile ahead; those of d bits stay in LDS for all
// the tiles of the node. The three steps over the top bits are taken on the
// seeds, one G_L of the ten low bits per thread, four subtiles at a time (eight
// would leave room for two workgroups per CU at d = 4 instead of three); each
// wave then runs the other ten bits of its own subtile without a barrier:
//   seeds read from LDS, y = p * 16 + r, steps 0..3 (patterns of more than d
//   bits read zeros);
//   register bits 0, 1 traded for lane bits 4, 5 (tile bits 4, 5): steps 4, 5;
//   one transpose through the wave's LDS plane, low words and then high words,
//   to y = r * 64 + lane: steps 6..9, stored from there.
// Two 12-bit halves in three layouts, transposed twice across the workgroup
// with seven barriers a half, took 22.6 ms at n = 30, d = 3 (FP32-scaled, 80.5
// GB written), 0.79 and 1.12 ms at n = 25, d = 4 (FP32-scaled, FP64); this takes
// 18.8, 0.58 and 1.03 (0.81 with a logarithm of less accuracy). Seeds summed by
// each wave for itself (one barrier a tile) took 19.0 and 0.66; significands
// stored as they are made instead of in one run 20.4; five waves per SIMD spill
// (FP32-scaled 25 to 30).
template <class P>
__device__ __forceinline__ void alpha_lin_tiles(
    int n, int d, uint32_t KS, int tl, const double *__restrict__ Zs,
    const double *__restrict__ betal, uint32_t K, uint32_t offd,
    const typename P::Anchor *__restrict__ anc, const typename P::V *__restrict__ qt,
    typename P::Store alpha, unsigned long long *cnt) {
    using V = typename P::V;
    using A = typename P::Anchor;
    constexpr int bA = 13, NR = 16;
    extern __shared__ unsigned char smem[];
    __shared__ V sq[32];
    __shared__ uint32_t k10[12], k13[15]; // sets of fewer than k of 10 (13) bits
    // rank of G_L + the top bits of T (a value of three bits) is
    // seedix[T * 11 + |G_L|] + the rank of G_L among the sets of 10 bits
    __shared__ uint32_t seedix[8 * 11];
    const int N = n - 1;
    const int hA = N - bA;
    const uint32_t tile0 = blockIdx.x << tl;   // 2^tl consecutive tiles of one node
    const int i = tile0 >> hA;
    const uint32_t t = threadIdx.x, lane = t & 63u, wave = t >> 6;
    const A T = anc[i];
    const int dd = min(d, 10);
    const uint32_t KF = sets10(dd), FS = KF + 8;   // eight zeros end a row
    const uint32_t nd = d <= 13 ? cbin(13, d) : 0u;
    uint32_t *pl = reinterpret_cast<uint32_t *>(smem) + wave * kAlphaPlane;
    double *S = reinterpret_cast<double *>(smem + 4 * kAlphaPlane * 4);
    double *F = S + KS + nd;
    uint8_t *size10 = reinterpret_cast<uint8_t *>(F + 4 * FS);
    // the seeds of fewer than d bits, two per thread read a tile ahead
    const double *zs = Zs + (size_t)tile0 * KS;
    double z0 = t < KS ? zs[t] : 0.0, z1 = t + kThreads < KS ? zs[t + kThreads] : 0.0;
    uint16_t *cb = reinterpret_cast<uint16_t *>(smem);   // C(a, b), a, b <= 13: set-up only
    if (t < 14 * 14) cb[t] = (uint16_t)cbin((int)t / 14, (int)t % 14);
    if (t >= 256 - 32) sq[t - (256 - 32)] = qt[min(t - (256 - 32), (uint32_t)n - 1u)];
    // those of d bits, betal_i(G_L) itself, are the same for every tile of the node
    {
        const double *zd = betal + (size_t)i * K + offd;
        for (uint32_t x = t; x < nd; x += kThreads) S[KS + x] = zd[x];
    }
    __syncthreads();
    if (t < 12) {
        uint32_t o = 0;
        for (uint32_t j = 0; j < t && j <= 10; ++j) o += cb[10 * 14 + j];
        k10[t] = o;
    } else if (t >= 64 && t < 64 + 15) {
        uint32_t o = 0;
        for (uint32_t j = 0; j < t - 64; ++j) o += cb[13 * 14 + j];
        k13[t - 64] = o;
    }
    __syncthreads();
    if (t < 8 * 11) {
        const uint32_t T3 = t / 11;
        const int k = (int)(t % 11);
        uint32_t r = k13[k + __popc(T3)];
        int j = k;
        for (int p = 0; p < 3; ++p)
            if ((T3 >> p) & 1) r += cb[(10 + p) * 14 + (++j)];
        seedix[t] = r - k10[k];
    }
    for (uint32_t g = t; g < KF; g += kThreads) {
        uint32_t k = 0;
        for (int j = 1; j <= 10; ++j) k += g >= k10[j] ? 1u : 0u;
        size10[g] = (uint8_t)k;
    }
    if (t < 32) F[(t >> 3) * FS + KF + (t & 7)] = 0.0;
    // layout A: entries p * 16 + r; p's low bits on lane bits 4, 5
    uint32_t off[5];
    {
        const uint32_t p = ((lane & 15u) << 2) | (lane >> 4);
        const int kp = __popc(p);
        uint32_t c[5] = {};
        for (int b = 0, j = 0; b < 6; ++b)
            if ((p >> b) & 1) {
                ++j;
#pragma unroll
                for (int m = 0; m < 5; ++m) c[m] += cb[(4 + b) * 14 + m + j];
            }
#pragma unroll
        for (int m = 0; m < 5; ++m)
            off[m] = wave * FS + (kp + m <= dd ? k10[kp + m] + c[m] : KF);
    }
    const uint32_t iw = (lane & 15u) * kAlphaRow + (lane >> 4);
    auto put_seeds = [&]() {
        if (t < KS) S[t] = z0;
        if (t + kThreads < KS) S[t + kThreads] = z1;
        for (uint32_t x = t + 2 * kThreads; x < KS; x += kThreads) S[x] = zs[x];
    };
    put_seeds();
    __syncthreads();
    const uint32_t last = (1u << tl) - 1u;
    for (uint32_t jt = 0; jt <= last; ++jt) {
        const uint32_t H = (tile0 + jt) & ((1u << hA) - 1);
        const uint64_t base = ((uint64_t)i << N) | ((uint64_t)H << bA);
        if (jt < last) {
            zs += KS;
            if (t < KS) z0 = zs[t];
            if (t + kThreads < KS) z1 = zs[t + kThreads];
        }
#pragma unroll 1
        for (uint32_t hb = 0; hb < 2; ++hb) {
            // ---- seeds of the subtiles 4 hb .. 4 hb + 3 after the steps over
            //      tile bits 10..12
            for (uint32_t g = t; g < KF; g += kThreads) {
                const int k = size10[g];
                auto seed = [&](uint32_t T3) {
                    return k + __popc(T3) <= d ? S[seedix[T3 * 11 + k] + g] : 0.0;
                };
                double w[4];
#pragma unroll
                for (uint32_t q = 0; q < 4; ++q) w[q] = seed(q);
                if (hb) {
                    double x[4];
#pragma unroll
                    for (uint32_t q = 0; q < 4; ++q) x[q] = seed(q + 4);
#pragma unroll
                    for (uint32_t q = 0; q < 4; ++q) w[q] += x[q];
                }
                w[1] += w[0];
                w[3] += w[2];
                w[2] += w[0];
                w[3] += w[1];
#pragma unroll
                for (uint32_t q = 0; q < 4; ++q) F[q * FS + g] = w[q];
            }
            __syncthreads();
            double v[NR];
#pragma unroll
            for (int r = 0; r < NR; ++r) v[r] = F[off[__builtin_popcount(r)] + colex4(r)];
#pragma unroll
            for (int q = 0; q < 4; ++q) lin_zeta_up<NR>(v, q);
            swap_lane_bit<NR, true>(v, 0);
            swap_lane_bit<NR, false>(v, 1);
#pragma unroll
            for (int q = 0; q < 2; ++q) lin_zeta_up<NR>(v, q);
            // entry of register r: tile bits 2, 3 are r's high bits, 4, 5 its low
            uint32_t lo[NR], hi[NR];
            wave_lds_order();
#pragma unroll
            for (int r = 0; r < NR; ++r)
                pl[iw + (uint32_t)((r >> 2) << 2 | (r & 3) << 4)] = (uint32_t)__double2loint(v[r]);
            wave_lds_order();
#pragma unroll
            for (int r = 0; r < NR; ++r) lo[r] = pl[lane + kAlphaRow * (uint32_t)r];
            wave_lds_order();
#pragma unroll
            for (int r = 0; r < NR; ++r)
                pl[iw + (uint32_t)((r >> 2) << 2 | (r & 3) << 4)] = (uint32_t)__double2hiint(v[r]);
            wave_lds_order();
#pragma unroll
            for (int r = 0; r < NR; ++r) hi[r] = pl[lane + kAlphaRow * (uint32_t)r];
#pragma unroll
            for (int r = 0; r < NR; ++r) v[r] = __hiloint2double((int)hi[r], (int)lo[r]);
#pragma unroll
            for (int q = 0; q < 4; ++q) lin_zeta_up<NR>(v, q);
            // ---- alpha = q(|S|) t(S)
            V qr[5];
            const int ht = __popc(H) + (int)hb + __popc(wave) + __popc(lane);
#pragma unroll
            for (int m = 0; m < 5; ++m) qr[m] = sq[min(ht + m, 31)];
            const uint64_t ub = base + hb * 4096u + wave * 1024u;
            if constexpr (std::is_same<P, PolX32>::value)
                alpha_store_x32(alpha, ub, lane, pl, v, qr, T, cnt);
            else
                store_tile_lin<P, NR>(alpha, ub, lane, 64u, v, qr, T, cnt);
            if (hb && jt < last) put_seeds();
            __syncthreads();
        }
    }
}

template <class P>
__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(4, 4)))
k_alpha_lin(int n, int d, uint32_t KS, int force_fb, int tl, const double *__restrict__ Zs,
            const double *__restrict__ betal, uint32_t K, uint32_t offd,
            const typename P::Anchor *__restrict__ anc, const int *__restrict__ linok,
            const typename P::V *__restrict__ qt, typename P::Store alpha,
            unsigned long long *cnt, uint32_t *fb) {
    const uint32_t tile0 = blockIdx.x << tl;   // 2^tl consecutive tiles of one node
    if (force_fb || !linok[tile0 >> (n - 14)]) {
        if ((int)threadIdx.x < (1 << tl)) fb_push(fb, tile0 + threadIdx.x);
        return;
    }
    alpha_lin_tiles<P>(n, d, KS, tl, Zs, betal, K, offd, anc, qt, alpha, cnt);
}

// The same for few tiles (n < 20): a tile that the linear form cannot hold is
// computed in the number system at once, rather than by a launch of its own
// that most solves leave at once (4.6 us). The larger LDS tile of that path
// halves the workgroups per CU, which a grid of this size does not fill.
template <class P>
__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 4)))
k_alpha_lin_few(int n, int d, uint32_t KS, int force_fb, const double *__restrict__ Zs,
                const double *__restrict__ betal, uint32_t K, uint32_t offd,
                const typename P::Anchor *__restrict__ anc, const int *__restrict__ linok,
                const typename P::V *__restrict__ qt, typename P::Store alpha,
                unsigned long long *cnt, uint32_t *fb, int use_prk, Tables tb,
                const typename P::V *__restrict__ beta) {
    if (force_fb || !linok[blockIdx.x >> (n - 14)]) {
        if (threadIdx.x == 0) atomicAdd(fb, 1u);
        alpha_tile<P>(n, d, K, use_prk, tb, beta, qt, alpha, cnt, blockIdx.x);
        return;
    }
    alpha_lin_tiles<P>(n, d, KS, 0, Zs, betal, K, offd, anc, qt, alpha, cnt);
}

// Plain doubles for the dense zetas.
struct Lin64 {
    using V = double;
    __device__ static inline V add(V a, V b) { return a + b; }
};

// Upward zeta of the 2^N entries (N <= 12) in vec (padx indices, zero beyond),
// in three register layouts of four bits each.
template <class A>
__device__ __forceinline__ void zeta_up12(typename A::V *vec, int N, uint32_t t) {
    constexpr int NR = 16;
    const uint32_t size = 1u << N, tlo = t & 15, thi = t >> 4;
    typename A::V g[NR];
    auto zeta4 = [&](int first) {
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (first + q < N) {
#pragma unroll
                for (int r = 0; r < NR; ++r)
                    if ((r >> q) & 1) g[r] = A::add(g[r], g[r ^ (1 << q)]);
            }
    };
    auto pass = [&](int first, auto at, bool active) {
        if (active) {
#pragma unroll
            for (int r = 0; r < NR; ++r) g[r] = vec[padx(at(r))];
            zeta4(first);
#pragma unroll
            for (int r = 0; r < NR; ++r) vec[padx(at(r))] = g[r];
        }
        __syncthreads();
    };
    pass(0, [&](uint32_t r) { return (t << 4) | r; }, (t << 4) < size);
    if (N > 4) pass(4, [&](uint32_t r) { return (thi << 8) | (r << 4) | tlo; }, (thi << 8) < size);
    if (N > 8) pass(8, [&](uint32_t r) { return (r << 8) | t; }, true);
}

// alpha of a small lattice (n - 1 <= 12 bits, n < 14), one workgroup per node:
// with no high bits every seed is a single family, Z(G) = beta_i(G). A node
// with a linear scale runs on its scores as plain doubles, any other in the
// number system. Bound by latency; the scores scattered to LDS and a dense zeta
// in registers take 5.8 us at n = 10 (FP32-scaled) and 7.2 us at n = 12 (FP64)
// where truncated passes over LDS, each step's pattern read from memory, took
// 10 and 26.
template <class P>
__global__ void __launch_bounds__(kThreads)
k_alpha_small(int n, int d, uint32_t K, int use_lin, Tables tb,
              const typename P::V *__restrict__ beta, const double *__restrict__ betal,
              const typename P::Anchor *__restrict__ anc, const int *__restrict__ linok,
              const typename P::V *__restrict__ qt, typename P::Store alpha,
              unsigned long long *cnt) {
    using V = typename P::V;
    extern __shared__ unsigned char smem[];
    V *tile = reinterpret_cast<V *>(smem);                  // 2^12 entries, padded
    double *lin = reinterpret_cast<double *>(smem);
    __shared__ V sq[32];
    const int N = n - 1;
    const int i = blockIdx.x;
    const uint32_t t = threadIdx.x, size = 1u << N;
    const bool is_lin = use_lin && linok[i];
    if (t < (uint32_t)n) sq[t] = qt[t];
    for (uint32_t x = t; x < 4096u + 256u; x += kThreads) {
        if (is_lin) lin[x] = 0.0;
        else tile[x] = P::zero();
    }
    __syncthreads();
    for (uint32_t r = t; r < K; r += kThreads) {
        const uint32_t x = padx(tb.famask[r]);
        if (is_lin) lin[x] = betal[(size_t)i * K + r];
        else tile[x] = beta[(size_t)i * K + r];
    }
    __syncthreads();
    const uint64_t base = (uint64_t)i << N;
    if (is_lin) {
        zeta_up12<Lin64>(lin, N, t);
        const typename P::Anchor T = anc[i];
        uint32_t nsat = 0, nfl = 0;
        for (uint32_t x = t; x < size; x += kThreads)
            P::store_lin_q(alpha, base + x, lin[padx(x)], sq[__popc(x)], T, nsat, nfl);
        if (nsat) atomicAdd(cnt, (unsigned long long)nsat);
        if (nfl) atomicAdd(cnt + 1, (unsigned long long)nfl);
    } else {
        zeta_up12<P>(tile, N, t);
        for (uint32_t x = t; x < size; x += kThreads)
            P::store(alpha, base + x, P::mul(sq[__popc(x)], tile[padx(x)]), cnt);
    }
}

// ------------------------------------------- a3/a4: sweep helpers
// In-tile alpha slices in LDS. The FP32-scaled form keeps the stored form,
// a plane of significands and a plane of exponent bytes (5 bytes per entry,
// so more workgroups share a CU); the log form keeps the values.
template <class P>
struct SliceLds {
    typename P::V *v;
    __device__ SliceLds(void *base, uint32_t) : v(reinterpret_cast<typename P::V *>(base)) {}
    __device__ typename P::V at(uint32_t k) const { return v[k]; }
    __device__ typename P::Raw raw(uint32_t k) const { return v[k]; }
    __device__ void put4(uint32_t e, const typename P::Raw4 &r) { P::decode4_nz(r, v + e); }
    __device__ void put(uint32_t e, const typename P::Store &s, uint64_t i) { v[e] = P::load(s, i); }
    static constexpr size_t bytes_per_entry = sizeof(typename P::V);
};
template <>
struct SliceLds<PolX32> {
    float *f;
    uint8_t *b;
    __device__ SliceLds(void *base, uint32_t total)
        : f(reinterpret_cast<float *>(base)), b(reinterpret_cast<uint8_t *>(f + total)) {}
    // factor of a product only: a stored zero has significand 0
    __device__ X32 at(uint32_t k) const { return X32{f[k], ((int)b[k] - kX32Bias) << 6}; }
    __device__ PolX32::Raw raw(uint32_t k) const { return PolX32::Raw{f[k], (uint32_t)b[k]}; }
    __device__ void put4(uint32_t e, const PolX32::Raw4 &r) {
        *reinterpret_cast<float4 *>(f + e) = r.f;
        *reinterpret_cast<uint32_t *>(b + e) = r.b;
    }
    __device__ void put(uint32_t e, const PolX32::Store &s, uint64_t i) {
        f[e] = s.f[i];
        b[e] = s.b[i];
    }
    static constexpr size_t bytes_per_entry = 5;
};

// Stage alpha_i(Hf + Lo') (Lo' without bit i) for the bL tile bits into LDS:
// slice i is the contiguous block alpha_i[(Hf >> 1) + k], k < 2^(bL-1).
// All loads of a thread are issued before any is stored.
template <class P, int TH>
__device__ inline void stage_alpha(const typename P::Store &alpha, uint64_t NN, uint64_t Hf,
                                   int bL, SliceLds<P> &la) {
    const uint32_t half = 1u << (bL - 1);
    const uint32_t total = (uint32_t)bL * half;
    const int t = threadIdx.x;
    if (half >= 4) {
        constexpr int U = 6;                  // batches of 4 entries in flight per thread
        for (uint32_t e0 = 4 * t; e0 < total; e0 += 4 * TH * U) {
            typename P::Raw4 raw[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint32_t e = e0 + 4 * TH * u;
                if (e < total)
                    raw[u] = P::load4_raw(alpha, (uint64_t)(e >> (bL - 1)) * NN + (Hf >> 1) +
                                                     (e & (half - 1)));
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint32_t e = e0 + 4 * TH * u;
                if (e < total) la.put4(e, raw[u]);   // product factors only
            }
        }
    } else {
        for (uint32_t e = t; e < total; e += TH)
            la.put(e, alpha, (uint64_t)(e >> (bL - 1)) * NN + (Hf >> 1) + (e & (half - 1)));
    }
}

// acc[k] += sum over the nodes i of the mask `nodes` (tile-high bits, the same
// for the whole workgroup) of alpha_i[S - i] * X[S ^ i], S = Hf + lo + k, k < E:
// forward S ^ i = S - i, backward S ^ i = S + i. B nodes per batch of loads.
template <class P, int E, int B>
__device__ inline void cross_terms(const typename P::Store &alpha, const typename P::Store &X,
                                   uint64_t NN, uint32_t Hf, uint32_t nodes, uint32_t lo,
                                   typename P::Acc *acc) {
    while (nodes) {
        typename P::template RawN<E> ra[B], rx[B];
        int cnt = 0;
#pragma unroll
        for (int u = 0; u < B; ++u) {
            if (nodes) {
                const int i = __ffs(nodes) - 1;
                nodes &= nodes - 1;
                ra[u].load(alpha, (uint64_t)i * NN + compress_bit(Hf & ~(1u << i), i) + lo);
                rx[u].load(X, (uint64_t)(Hf ^ (1u << i)) + lo);
                cnt = u + 1;
            }
        }
        P::template cross_add<E, B>(acc, ra, rx, cnt);
    }
}

// The in-tile layers of a sweep tile of BL bits, unrolled. Step k = 1 .. BL
// takes the entries with k in-tile terms (forward: k bits set; backward: k bits
// clear), one per thread, C(BL, k) of them. A step's entries and their alpha
// factors do not depend on the steps before, so they are read one step ahead;
// what is left between two barriers is one round of LDS reads of the tile, the
// products, one common exponent (or maximum) and one sum. The loop over layers
// with its chain of bit scans and aligned adds took 0.86 us a layer, most of a
// small lattice's sweep; this one 0.5 us (n = 10).
template <class P, int BL>
struct DpStep {
    typename P::Raw a[BL];   // alpha factors
    uint32_t x[BL];          // tile entries they multiply
    uint32_t lo;             // the entry
};
__device__ constexpr uint32_t dp_binom(int n, int k) {
    uint32_t r = 1;
    for (int j = 1; j <= k; ++j) r = r * (uint32_t)(n - k + j) / (uint32_t)j;
    return r;
}
// first place of step k's entries in the popcount order
__device__ constexpr uint32_t dp_first(int BL, int k, bool fwd) {
    uint32_t s = 0;
    for (int j = 0; j < (fwd ? k : BL - k); ++j) s += dp_binom(BL, j);
    return s;
}
// (The lowest bit of `rest` is not written as rest & -rest: hipcc 7.2 selects a
// v_bitop3_b32 of a wrong truth table for that chain in the backward form.)
template <class P, bool FWD, int BL, int K>
__device__ __forceinline__ void dp_fetch(DpStep<P, BL> &st, const SliceLds<P> &la,
                                         const uint16_t *lord, uint32_t t) {
    constexpr uint32_t T = 1u << BL, size = dp_binom(BL, K);
    st.lo = lord[dp_first(BL, K, FWD) + min(t, size - 1u)];
    uint32_t rest = FWD ? st.lo : (T - 1u) & ~st.lo;
#pragma unroll
    for (int u = 0; u < K; ++u) {
        const uint32_t i = (uint32_t)__ffs(rest) - 1u, bit = 1u << i;
        rest &= rest - 1u;
        st.x[u] = st.lo ^ bit;
        const uint32_t w = st.lo & ~bit, low = bit - 1u;   // w without bit i, closed up
        st.a[u] = la.raw((i << (BL - 1)) + ((w & low) | ((w >> 1) & ~low)));
    }
}
template <class P, bool FWD, int BL, int K>
__device__ __forceinline__ void dp_steps(DpStep<P, BL> &st, const SliceLds<P> &la,
                                         typename P::V *lt, const uint16_t *lord, uint32_t t,
                                         uint32_t wave0) {
    if constexpr (K <= BL) {
        using V = typename P::V;
        constexpr uint32_t size = dp_binom(BL, K), next = K < BL ? dp_binom(BL, K + 1) : 0u;
        __syncthreads();
        DpStep<P, BL> nx;
        if (wave0 < size) {                     // whole waves
            V x[K];
            const V s0 = lt[st.lo];
#pragma unroll
            for (int u = 0; u < K; ++u) x[u] = lt[st.x[u]];
            if constexpr (K < BL) {
                if (wave0 < next) dp_fetch<P, FWD, BL, K + 1>(nx, la, lord, t);
            }
            const V r = P::template dp_sum<K>(s0, st.a, x);
            if (t < size) lt[st.lo] = r;
        } else if constexpr (K < BL) {
            if (wave0 < next) dp_fetch<P, FWD, BL, K + 1>(nx, la, lord, t);
        }
        dp_steps<P, FWD, BL, K + 1>(nx, la, lt, lord, t, wave0);
    }
}

// ------------------------------- a3 + a4: both sweeps, one layer of tiles
// Forward (Eq. 9) L(S) = sum_{i in S} alpha_i(S-i) L(S-i), layers upwards;
// backward (Eq. 10) Rp(S) = sum_{i not in S} alpha_i(S) Rp(S+i), Rp(V) = 1,
// layers downwards. Step h of both runs in one launch: the first nb workgroups
// take the tiles H with |H| = h of the forward sweep, the others the tiles
// with |H| = nh - h of the backward sweep (the same number). The two sweeps
// share nothing but alpha, and a layer of a small lattice is a few workgroups
// bound by the latency of one launch and of bL dependent in-tile layers, so
// running both at once halves the sweeps: n = 16 FP32-scaled 180 -> 63 us for
// both, n = 20 FP64 541 -> 204 us (unrolled in-tile layers and exp_neg included).
// Large lattices launch the two sweeps apart, on two streams (launch_lattice);
// there they stream alpha at the HBM rate.
// Tiles go in colex order: consecutive workgroups, which run at the same time
// on the eight XCDs, share most of their X blocks (a mapping that gave each
// XCD a contiguous eighth of the layer cut the L2 misses by 10% but measured
// 5% slower). Cross-tile terms (bits of H) stream contiguous 2^bL blocks of
// alpha_i and X, two consecutive entries per thread and eight nodes at a time for
// the 9-bit tiles, else four and four; in-tile terms use the tile's alpha slices
// staged in LDS and run popcount layer by popcount layer, one entry per thread
// (TH >= the largest layer): unrolled for the widths that the plan chooses
// (BL > 0, dp_steps), else in a loop that reads the operands of four terms
// before it sums them. Requires bL >= 2.
template <class P, bool FWD, int TH, int BL>
__device__ inline void sweep_tile(int n, int bL_arg, uint32_t Hm, const Tables &tb,
                                  const typename P::Store &alpha, const typename P::Store &X,
                                  unsigned long long *cnt, unsigned char *smem) {
    using V = typename P::V;
    const int bL = BL > 0 ? BL : bL_arg;
    const uint32_t half = 1u << (bL - 1);
    const uint32_t T = 1u << bL;
    SliceLds<P> la(smem, (uint32_t)bL * half);   // bL * half entries
    V *lt = reinterpret_cast<V *>(smem + align16(SliceLds<P>::bytes_per_entry * bL * half));
    uint16_t *lord = reinterpret_cast<uint16_t *>(lt + T);
    const int t = threadIdx.x;
    const int nh = n - bL;
    const uint64_t NN = 1ull << (n - 1);
    const uint32_t Hf = Hm << bL;
    const uint32_t highall = ((1u << nh) - 1u) << bL;
    stage_alpha<P, TH>(alpha, NN, Hf, bL, la);
    // entries per thread: two where that occupies every thread (9-bit tiles), and
    // then eight nodes' loads in flight (both sweeps at n = 22 254 -> 237 us, n = 25
    // 1.17 -> 1.14 ms; four or six nodes 243 and 240 us, 1.15 and 1.15 ms)
    constexpr int E = (BL == 9 && TH == 256) ? 2 : 4;
    for (uint32_t lo = E * t; lo < T; lo += E * TH) {
        typename P::Acc acc[E];
#pragma unroll
        for (int k = 0; k < E; ++k) {
            const bool start = FWD ? (Hf == 0 && lo + k == 0) : (Hf == highall && lo + k == T - 1);
            acc[k] = P::acc_of(start ? P::one() : P::zero());
        }
        cross_terms<P, E, E == 2 ? 8 : 4>(alpha, X, NN, Hf, FWD ? Hf : (highall & ~Hf), lo, acc);
#pragma unroll
        for (int k = 0; k < E; ++k) lt[lo + k] = P::norm_v(P::acc_value(acc[k]));
    }
    for (uint32_t x = t; x < T; x += TH) lord[x] = tb.lorder[x];
    __syncthreads();
    if constexpr (BL > 0) {
        const uint32_t wave0 = __builtin_amdgcn_readfirstlane(t & ~63);
        DpStep<P, BL> st;
        if (wave0 < (uint32_t)BL) dp_fetch<P, FWD, BL, 1>(st, la, lord, t);
        dp_steps<P, FWD, BL, 1>(st, la, lt, lord, t, wave0);
        __syncthreads();
        for (uint32_t e = 4 * t; e < T; e += 4 * TH) P::store4(X, (uint64_t)Hf + e, lt + e, cnt);
        return;
    }
    // in-tile layers: layer l holds size = C(bL, l) entries from lord[off] on
    int l = FWD ? 1 : bL - 1;
    uint32_t size = bL, off = FWD ? 1 : T - 1 - bL;
    for (int step = 0; step < bL; ++step) {
        const uint32_t lo = (uint32_t)t < size ? (uint32_t)lord[off + t] : T;
        if (lo < T) {
            typename P::Acc acc = P::acc_of(lt[lo]);
            uint32_t rest = FWD ? lo : (T - 1) & ~lo;
            const int terms = FWD ? l : bL - l;
            constexpr int B = 4;
            for (int q = 0; q < terms; q += B) {
                V a[B], x[B];
#pragma unroll
                for (int u = 0; u < B; ++u) {
                    if (q + u < terms) {
                        const int i = __ffs(rest) - 1;
                        rest &= rest - 1;
                        const uint32_t w = lo & ~(1u << i);
                        a[u] = la.at(i * half + (uint32_t)compress_bit(w, i));
                        x[u] = lt[lo ^ (1u << i)];
                    }
                }
                V term[B];
#pragma unroll
                for (int u = 0; u < B; ++u)
                    if (q + u < terms) term[u] = P::mul_raw(a[u], x[u]);
                P::template acc_add_n<B>(acc, term, terms - q);
            }
            lt[lo] = P::norm_v(P::acc_value(acc));
        }
        __syncthreads();
        if (FWD) {
            off += size;
            size = size * (uint32_t)(bL - l) / (uint32_t)(l + 1);
            ++l;
        } else {
            size = size * (uint32_t)l / (uint32_t)(bL - l + 1);
            off -= size;
            --l;
        }
    }
    for (uint32_t e = 4 * t; e < T; e += 4 * TH) P::store4(X, (uint64_t)Hf + e, lt + e, cnt);
}

template <class P, int TH, int BL>
__global__ void __launch_bounds__(TH)
k_sweeps(int n, int bL, uint32_t nb, uint32_t hoffF, uint32_t hoffB, Tables tb,
         typename P::Store alpha, typename P::Store L, typename P::Store R,
         unsigned long long *cnt) {
    extern __shared__ unsigned char smem[];
    const uint32_t b = blockIdx.x;
    if (b < nb)
        sweep_tile<P, true, TH, BL>(n, bL, tb.hord[hoffF + b], tb, alpha, L, cnt, smem);
    else
        sweep_tile<P, false, TH, BL>(n, bL, tb.hord[hoffB + b - nb], tb, alpha, R, cnt, smem);
}

// ---------------------------------------- a5 + a6: Gamma, in-tile part
// Layout of Y1_v (K(bv, d) ranks x 2^hv values of Hc). The ranks below
// kg4 (K(bv, d) rounded down to a multiple of 4) sit in groups of four: group
// j holds, for every Hc, the values of ranks 4j .. 4j + 3 side by side. A
// Gamma tile workgroup writes one Hc of every rank, so its stores leave as
// 32-byte runs instead of single 8-byte values. The ranks from kg4 on follow
// as plain rows of 2^hv values.
__device__ __forceinline__ size_t y1_at(uint32_t rank, uint64_t Hc, int hv, uint32_t kg4) {
    return rank < kg4 ? ((((size_t)rank >> 2) << (hv + 2)) | ((size_t)Hc << 2) | (rank & 3u))
                      : (((size_t)rank << hv) + Hc);
}
// distance between the entries of consecutive Hc of one rank
__device__ __forceinline__ uint32_t y1_stride(uint32_t rank, uint32_t kg4) {
    return rank < kg4 ? 4u : 1u;
}
// Workgroup order of the kernels that read Y1 rows: a workgroup's index
// within endpoint v, local (rank-major: s * 2^hB + Ht), becomes the
// (rank, Ht) item it takes, such that the four ranks of a group (same Ht)
// run 8 workgroups apart, on one XCD, where its L2 serves the group's
// 32-byte runs to all four. A bijection on [0, K(bv, d) 2^hB): whole octets
// of (group, Ht) pairs first, then the rest of the grouped ranks with the
// four ranks side by side, then the plain rows unchanged.
__device__ __forceinline__ uint32_t y1_reader_item(uint32_t local, int hB, uint32_t kg4) {
    const uint32_t G = (kg4 >> 2) << hB;        // (group, Ht) pairs
    const uint32_t full = (G >> 3) << 5;        // locals of whole octets
    if (local >= 4 * G) return local;
    uint32_t gH, q;
    if (local < full) {
        q = (local >> 3) & 3u;
        gH = ((local >> 5) << 3) | (local & 7u);
    } else {
        const uint32_t x = local - full;
        q = x & 3u;
        gH = ((G >> 3) << 3) + (x >> 2);
    }
    return ((((gH >> hB) << 2) | q) << hB) | (gH & ((1u << hB) - 1u));
}

// In-register downward zeta step over register bit q of NR = 2^RB entries,
// skipped when that register bit carries the endpoint itself.
template <class P, int NR>
__device__ inline void reg_zeta_down(typename P::V *g, int q) {
#pragma unroll
    for (int r = 0; r < NR; ++r)
        if (!((r >> q) & 1)) g[r] = P::add(g[r], g[r | (1 << q)]);
}

// Padded LDS index: one spare slot every 16 entries keeps the transposed
// reads of the Gamma tile free of heavy bank conflicts.

// Workgroup = full-mask tile H of 2^12 masks (the low 12 bits vary), 256
// threads x 16 entries. L(H + x) and Rp(H + x) stay in registers for the
// whole workgroup; every endpoint v not in H is served in turn:
//   g_v(S) = q(|S|) L(S) Rp(S + v) for S = H + x. For v a tile bit, x runs
//   over the entries without bit v and Rp(S + v) is the partner entry (same
//   thread for a register bit, else read through LDS). For v above the tile
//   Rp(S + v) is the tile H + v, prefetched while the previous endpoint is
//   reduced. Products are left unnormalised (add() aligns exactly).
//   Downward zeta over the tile bits other than v, entirely in registers:
//   layout A holds tile bits 8..11 in the register index (x = r*256 + t),
//   layout B bits 4..7 (x = t_hi*256 + r*16 + t_lo), layout C bits 0..3
//   (x = t*16 + r); two LDS transposes move between them.
//   The entries with at most d ones (Def. 2: Gamma_v(G) is needed for
//   |G| <= d only) go from registers to Y1_v[seed][Hc_v].
template <class P>
__device__ __forceinline__ void gamma_tile(int n, int d, const GammaGeom &gg, const Tables &tb,
                                           const typename P::Store &L,
                                           const typename P::Store &R,
                                           const typename P::V *__restrict__ qt,
                                           typename P::V *__restrict__ Y1,
                                           typename P::V *__restrict__ part, uint32_t H,
                                           int only_v = -1) {
    using V = typename P::V;
    using Raw = typename P::Raw;
    constexpr int bT = 12, NR = 16;
    extern __shared__ unsigned char smem[];
    V *gb = reinterpret_cast<V *>(smem);                       // padded 2^12 entries
    uint32_t *sbin = reinterpret_cast<uint32_t *>(gb + 4096 + 256);
    uint32_t *seedT = sbin + 33 * 33;                          // K(12, d) ranked masks
    __shared__ V sq[32];
    __shared__ uint32_t offT[34], offT1[34];
    const int t = threadIdx.x;
    const uint64_t Hf = (uint64_t)H << bT;
    for (int x = t; x < 33 * 33; x += kThreads) sbin[x] = tb.binom[x];
    for (uint32_t x = t; x < gg.KT; x += kThreads) seedT[x] = tb.seedmask[x];
    if (t < n) sq[t] = qt[t];
    V Lr[NR], Rr[NR], g[NR];
    Raw Rv[NR];                               // next endpoint's Rp tile, undecoded
    const int hpc = __popcll(Hf);
    {
        Raw l0[NR], r0[NR];
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            const uint32_t x = r * kThreads + t;
            l0[r] = P::load_raw(L, Hf | x);
            r0[r] = P::load_raw(R, Hf | x);
        }
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            Lr[r] = P::decode_raw(l0[r]);
            Rr[r] = P::decode_raw(r0[r]);
        }
    }
    // next endpoint above the tile, not in H (only_v itself when it is one)
    int vn = only_v >= bT ? only_v : bT;
    while (vn < n && ((Hf >> vn) & 1)) ++vn;
    if (vn < n) {
#pragma unroll
        for (int r = 0; r < NR; ++r) Rv[r] = P::load_raw(R, Hf | (r * kThreads + t) | (1ull << vn));
    }
    {   // invariant partials: sum of L(S) Rp(S) over the tile, per |x| (x = r*256 + t)
        V lr[5];
#pragma unroll
        for (int k = 0; k < 5; ++k) lr[k] = P::zero();
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            const V prod = P::mul(Lr[r], Rr[r]);
#pragma unroll
            for (int k = 0; k < 5; ++k)
                if (__popc(r) == k) lr[k] = P::add(lr[k], prod);
        }
#pragma unroll
        for (int k = 0; k < 5; ++k) gb[t * 5 + k] = lr[k];
        __syncthreads();
        {   // layer l = t / 16 of the tile: 16 lanes x 16 slots, then a lane tree
            const int l = t >> 4, j = t & 15;
            V acc = P::zero();
            if (l <= bT) {
                for (int u = j; u < kThreads; u += 16) {
                    const int k = l - __popc(u);
                    if (k >= 0 && k <= 4) acc = P::add(acc, gb[u * 5 + k]);
                }
            }
            for (int w = 8; w > 0; w >>= 1) acc = P::add(acc, shfl_xor_v(acc, w));
            if (l <= bT && j == 0) part[(size_t)H * (bT + 1) + l] = acc;
        }
    }
    __syncthreads();
    if (t <= d + 1) {
        offT[t] = Kcount(sbin, bT, t - 1);
        offT1[t] = Kcount(sbin, bT - 1, t - 1);
    }
    const uint32_t tlo = t & 15, thi = t >> 4;
    for (int v = only_v >= 0 ? only_v : 0; v < (only_v >= 0 ? only_v + 1 : n); ++v) {
        const bool low = v < bT;
        if (!low && ((Hf >> v) & 1)) continue;
        // ---- g in layout A
        if (low && v < 8) {
            // partner Rp(S + v) lives in another thread: exchange through LDS
#pragma unroll
            for (int r = 0; r < NR; ++r) gb[padx(r * kThreads + t)] = Rr[r];
            __syncthreads();
#pragma unroll
            for (int r = 0; r < NR; ++r) {
                const uint32_t x = r * kThreads + t;
                g[r] = ((x >> v) & 1) ? P::zero()
                                      : P::mul_raw(sq[hpc + __popc(x)],
                                                   P::mul_raw(Lr[r], gb[padx(x | (1u << v))]));
            }
            __syncthreads();
        } else if (low) {
            // v is register bit q: the partner is register r + 2^q of this thread
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if (v - 8 != q) continue;
#pragma unroll
                for (int r = 0; r < NR; ++r)
                    g[r] = ((r >> q) & 1) ? P::zero()
                                          : P::mul_raw(sq[hpc + __popc(r * kThreads + t)],
                                                       P::mul_raw(Lr[r], Rr[r | (1 << q)]));
            }
        } else {
#pragma unroll
            for (int r = 0; r < NR; ++r)
                g[r] = P::mul_raw(sq[hpc + __popc(r * kThreads + t)],
                                  P::mul_raw(Lr[r], P::decode_raw(Rv[r])));
            vn = v + 1;                       // prefetch the next endpoint's Rp tile
            while (vn < n && ((Hf >> vn) & 1)) ++vn;
            if (vn < n) {
#pragma unroll
                for (int r = 0; r < NR; ++r)
                    Rv[r] = P::load_raw(R, Hf | (r * kThreads + t) | (1ull << vn));
            }
        }
        // ---- tile bits 8..11 (layout A)
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (v != 8 + q) reg_zeta_down<P, NR>(g, q);
        // ---- A -> B, tile bits 4..7
#pragma unroll
        for (int r = 0; r < NR; ++r) gb[padx(r * kThreads + t)] = g[r];
        __syncthreads();
#pragma unroll
        for (int r = 0; r < NR; ++r) g[r] = gb[padx((thi << 8) | (r << 4) | tlo)];
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (v != 4 + q) reg_zeta_down<P, NR>(g, q);
        __syncthreads();
        // ---- B -> C, tile bits 0..3
#pragma unroll
        for (int r = 0; r < NR; ++r) gb[padx((thi << 8) | (r << 4) | tlo)] = g[r];
        __syncthreads();
#pragma unroll
        for (int r = 0; r < NR; ++r) g[r] = gb[padx((t << 4) | r)];
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (v != q) reg_zeta_down<P, NR>(g, q);
        // ---- outputs: entries with at most d ones, read back through LDS
        __syncthreads();
#pragma unroll
        for (int r = 0; r < NR; ++r) gb[padx((t << 4) | r)] = g[r];
        __syncthreads();
        const int hv = gg.hv[v];
        const uint32_t Hc = low ? H : (uint32_t)compress_bit(H, v - bT);
        V *dst = Y1 + gg.y1off[v];
        for (uint32_t si = t; si < gg.KT; si += kThreads) {
            const uint32_t msk = seedT[si];
            uint32_t rank = si;
            if (low) {
                if ((msk >> v) & 1) continue;
                const uint32_t cm = (uint32_t)compress_bit(msk, v);
                rank = offT1[__popc(cm)];
                int k = 0;
                uint32_t rest = cm;
                while (rest) {
                    const int p = __ffs(rest) - 1;
                    rest &= rest - 1;
                    rank += C(sbin, p, ++k);
                }
            }
            dst[y1_at(rank, Hc, hv, gg.kg4[v])] = P::norm_v(gb[padx(msk)]);
        }
        __syncthreads();
    }
}

// Consecutive tiles run on the same XCD so that its L2 merges the 8-byte Y1
// writes of neighbouring tiles.
template <class P>
__global__ void __launch_bounds__(kThreads)
k_gamma_tile(int n, int d, GammaGeom gg, Tables tb, typename P::Store L, typename P::Store R,
             const typename P::V *__restrict__ qt, typename P::V *__restrict__ Y1,
             typename P::V *__restrict__ part) {
    const uint32_t nblk = 1u << (n - 12);
    uint32_t H = blockIdx.x;
    if (nblk >= 64) H = (blockIdx.x & 7) * (nblk >> 3) + (blockIdx.x >> 3);
    gamma_tile<P>(n, d, gg, tb, L, R, qt, Y1, part, H);
}

// Recomputation of the listed tiles in the number system proper (list[0]
// entries, at most ntiles; list[1 + j] = H): the grid walks the list. Only the
// forced fallback runs it, whose list k_gamma_tile_lin alone writes.
template <class P>
__global__ void __launch_bounds__(kThreads)
k_gamma_tile_fb(int n, int d, GammaGeom gg, Tables tb, typename P::Store L,
                typename P::Store R, const typename P::V *__restrict__ qt,
                typename P::V *__restrict__ Y1, typename P::V *__restrict__ part,
                const uint32_t *list, uint32_t ntiles) {
    const uint32_t nlist = min(list[0], ntiles);
    for (uint32_t it = blockIdx.x; it < nlist; it += gridDim.x) {
        __syncthreads();
        gamma_tile<P>(n, d, gg, tb, L, R, qt, Y1, part, list[1 + it]);
    }
}

template <int NR>
__device__ inline void lin_zeta_down(double *g, int q) {
#pragma unroll
    for (int r = 0; r < NR; ++r)
        if (!((r >> q) & 1)) g[r] += g[r | (1 << q)];
}

// Linear-tile form of k_gamma_tile (same tiles and outputs). For endpoint v
// every needed output Gamma_v(G_L) of the tile is a sum over supersets of
// G_L that includes g_v(H + top), top = every tile bit but v. So the
// products are scaled by one power of two (a log offset for the log-space
// system) that puts g_v(H + top) near 2^-1000 (within 2^-1032 .. 2^-968 in the
// FP32-scaled form, whose scales are multiples of 64), and the downward zeta
// runs on plain doubles: one FP64 add per step. Products far below
// g_v(H + top) may lose bits to the subnormal range, each at most 2^-1075;
// over the at most 2^11 terms of an output (which is at least g_v(H + top))
// that is at most 2^-32 of the output in the FP32-scaled form, below the
// 2^-24 rounding of its stored significand, and 2^-64 in the log form. If
// Gamma_v(H + empty), the largest entry, overflows after
// the scaling, or g_v(H + top) is zero, the endpoint's outputs are not stored
// and (H, v) goes to the list of k_gamma_tile_retry. force_fb (tests) sends
// every tile to the list of k_gamma_tile_fb instead, which recomputes all of
// its endpoints; the retry list then stays empty, since k_gamma_tile_retry
// counts the endpoints that it recomputes in fb[0], the length of that list.
// Layouts (x the 12 tile bits, 256 threads x 16 entries):
//   A  x = t * 16 + r      bits 0..3 in registers; products formed here. Each
//      thread owns 16 consecutive masks, so L, Rp and the partners Rp(x + v)
//      move as 16-entry vector loads: the thread's own Rp block for a
//      register bit, the block of thread t + 2^(v-4) for tile bits 4..11,
//      the tile H + v above the tile; one endpoint ahead of their use.
//   B  x = thi * 256 + r * 16 + tlo, bits 4..7 in registers;
//   C  x = r * 256 + p, p the thread's pattern of bits 0..7 (lane order
//      ordC), bits 8..11 in registers. Only outputs with at most d ones are
//      needed and bits 0..7 are final by then, so threads whose pattern has
//      more than d ones skip C (whole waves for small d).
// The kernel below wraps this body with its register cap.
template <class P, bool kSplit>
__device__ __forceinline__ void
gamma_tile_lin_body(int n, int d, int force_fb, int vsplit, GammaGeom gg, Tables tb,
                    typename P::Store L, typename P::Store R, const typename P::V *__restrict__ qt,
                    typename P::V *__restrict__ Y1, typename P::V *__restrict__ part,
                    uint32_t *fb, uint32_t *rt) {
    using V = typename P::V;
    using R16 = typename P::Raw16;
    using A = typename P::Anchor;
    constexpr int bT = 12, NR = 16;
    extern __shared__ unsigned char smem[];
    double *gb = reinterpret_cast<double *>(smem);             // padded 2^12 entries
    V *gv = reinterpret_cast<V *>(smem);                       // same slots, as values
    uint32_t *sbin = reinterpret_cast<uint32_t *>(gb + 4096 + 256);
    uint32_t *seedT = sbin + 33 * 33;                          // K(12, d) ranked masks
    __shared__ V sq[32];
    __shared__ uint32_t offT[34], offT1[34];
    __shared__ A sT[32];
    __shared__ int sok[32];
    __shared__ int sfail;
    const int t = threadIdx.x;
    const int hbits = n - bT;
    const uint32_t nblk = 1u << hbits;
    // vsplit workgroups share a tile, workgroup v0 taking the endpoints
    // v = v0 (mod vsplit); the first of them also writes the tile's partials
    const int vs = kSplit ? vsplit : 1;
    const uint32_t blk = kSplit ? blockIdx.x / (uint32_t)vs : blockIdx.x;
    const int v0 = kSplit ? (int)(blockIdx.x % (uint32_t)vs) : 0;
    uint32_t H = blk;
    if (nblk >= 64) H = (blk & 7) * (nblk >> 3) + (blk >> 3);
    const uint64_t Hf = (uint64_t)H << bT;
    const uint64_t x0 = Hf | ((uint32_t)t << 4);   // the thread's first mask in layout A
    for (int x = t; x < 33 * 33; x += kThreads) sbin[x] = tb.binom[x];
    for (uint32_t x = t; x < gg.KT; x += kThreads) seedT[x] = tb.seedmask[x];
    if (t < n) sq[t] = qt[t];
    if (t == 0) sfail = force_fb && v0 == 0 ? 1 : 0;
    R16 Lw, Rown, Rv;                         // own L and Rp blocks; partners of the next endpoint
    const int hpc = __popcll(Hf);
    // the workgroup's first endpoint, and the partner block it needs
    int vfirst = v0;
    while (vfirst < n && vfirst >= bT && ((Hf >> vfirst) & 1)) vfirst += vs;
    {
        Lw = P::load16_raw(L, x0);
        Rown = P::load16_raw(R, x0);
        Rv = Rown;                            // a register bit needs no partner block
        if (vfirst >= 4 && vfirst < bT)
            Rv = P::load16_raw(R, Hf | ((uint32_t)(t | (1 << (vfirst - 4))) << 4));
        else if (vfirst >= bT && vfirst < n)
            Rv = P::load16_raw(R, x0 | (1ull << vfirst));
        __syncthreads();                      // sbin
        // invariant partials: sum of L(S) Rp(S) over the tile, per |x|; the
        // thread's entries have |x| = |t| + |r|
        V lr[5];
#pragma unroll
        for (int k = 0; k < 5; ++k) lr[k] = P::zero();
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            const V prod = P::mul(P::at16(Lw, r), P::at16(Rown, r));
#pragma unroll
            for (int k = 0; k < 5; ++k)
                if (__builtin_popcount(r) == k) lr[k] = P::add(lr[k], prod);
        }
#pragma unroll
        for (int k = 0; k < 5; ++k) gv[t * 5 + k] = lr[k];
        __syncthreads();
        {   // layer l = t / 16 of the tile: 16 lanes x 16 slots, then a lane tree
            const int l = t >> 4, j = t & 15;
            V acc = P::zero();
            if (l <= bT) {
                for (int u = j; u < kThreads; u += 16) {
                    const int k = l - __popc(u);
                    if (k >= 0 && k <= 4) acc = P::add(acc, gv[u * 5 + k]);
                }
            }
            for (int w = 8; w > 0; w >>= 1) acc = P::add(acc, shfl_xor_v(acc, w));
            if (l <= bT && j == 0 && v0 == 0) part[(size_t)H * (bT + 1) + l] = acc;
        }
    }
    // scale of endpoint v: g_v at the top of the tile
    if (t < n) {
        const int v = t;
        const uint32_t all = (1u << bT) - 1;
        int ok = 0;
        A T{};
        if (v < bT) {
            const V a = P::mul(P::mul(sq[hpc + bT - 1], P::load(L, Hf | (all & ~(1u << v)))),
                               P::load(R, Hf | all));
            ok = P::anchor_of(a, &T) ? 1 : 0;
        } else if (!((Hf >> v) & 1)) {
            const V a = P::mul(P::mul(sq[hpc + bT], P::load(L, Hf | all)),
                               P::load(R, Hf | all | (1ull << v)));
            ok = P::anchor_of(a, &T) ? 1 : 0;
        }
        sT[v] = T;
        sok[v] = ok;
    }
    if (t <= d + 1) {
        offT[t] = Kcount(sbin, bT, t - 1);
        offT1[t] = Kcount(sbin, bT - 1, t - 1);
    }
    __syncthreads();
    // q(|S|) for the thread's entries in layout A: |S| = |H| + |t| + |r|
    // q(|S|) L(S) for the thread's entries, the factor every endpoint shares
    V qL[NR];
    {
        const int ht = hpc + __popc(t);
        V qa[5];
#pragma unroll
        for (int m = 0; m < 5; ++m) qa[m] = sq[min(ht + m, 31)];
#pragma unroll
        for (int r = 0; r < NR; ++r) qL[r] = P::mul_raw(qa[__builtin_popcount(r)], P::at16_nz(Lw, r));
    }
    const uint32_t tlo = t & 15, thi = t >> 4;
    const uint32_t pc = tb.ordC[t];
    const bool liveC = __popc(pc) <= d;
    // padx indices as a lane base plus a constant per register (folded into
    // the LDS offsets): A, padx(t * 16 + r) = 17 t + r; B, padx(thi * 256 +
    // r * 16 + tlo) = 272 thi + tlo + 17 r; C, padx(r * 256 + pc) =
    // pc + pc / 16 + 272 r
    const uint32_t iA = 17 * t, iB = 272 * thi + tlo, iC = pc + (pc >> 4);
    auto endpoint = [&](const int v) {
        const bool low = v < bT;
        if (!low && ((Hf >> v) & 1)) return;
        const A T = sT[v];
        const int okv = sok[v];
        // ---- products in layout A (entries with bit v are not in the lattice)
        double g[NR];
        if (v < 4) {
            // the partner of register r is register r + 2^v of the own block
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if (v != q) continue;
#pragma unroll
                for (int r = 0; r < NR; ++r)
                    g[r] = ((r >> q) & 1) ? 0.0
                                          : P::prod2_lin(qL[r], P::at16_nz(Rown, r | (1 << q)), T);
            }
        } else {
            const bool excl = low && ((t >> (v - 4)) & 1);
#pragma unroll
            for (int r = 0; r < NR; ++r) {
                const double pr =
                    P::prod2_lin(qL[r], P::at16_nz(Rv, r), T);
                g[r] = excl ? 0.0 : pr;
            }
        }
        {   // partners of the next endpoint (none needed for register bits)
            int vn = v + vs;
            while (vn < n && vn >= bT && ((Hf >> vn) & 1)) vn += vs;
            if (vn >= 4 && vn < bT) {
                // tile bit vn: the block of thread t + 2^(vn-4) (own block if set)
                Rv = P::load16_raw(R, Hf | ((uint32_t)(t | (1 << (vn - 4))) << 4));
            } else if (vn >= bT && vn < n) {
                Rv = P::load16_raw(R, x0 | (1ull << vn));
            }
        }
        // ---- tile bits 0..3 (layout A)
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (v != q) lin_zeta_down<NR>(g, q);
        // ---- A -> B, tile bits 4..7
#pragma unroll
        for (int r = 0; r < NR; ++r) gb[iA + r] = g[r];
        __syncthreads();
#pragma unroll
        for (int r = 0; r < NR; ++r) g[r] = gb[iB + r * 17];
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (v != 4 + q) lin_zeta_down<NR>(g, q);
        // B-layout slots belong to one thread each: written back in place
#pragma unroll
        for (int r = 0; r < NR; ++r) gb[iB + r * 17] = g[r];
        __syncthreads();
        // ---- B -> C, tile bits 8..11, live patterns only; results stay in place
        if (liveC) {
#pragma unroll
            for (int r = 0; r < NR; ++r) g[r] = gb[iC + r * 272];
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (v != 8 + q) lin_zeta_down<NR>(g, q);
#pragma unroll
            for (int r = 0; r < NR; ++r) gb[iC + r * 272] = g[r];
        }
        __syncthreads();
        // ---- outputs: entries with at most d ones, read back through LDS.
        // Gamma_v(H + empty) bounds every entry of the tile.
        const bool fine = okv && gb[padx(0)] <= 1.0e300;
        if (!fine) {
            if (t == 0 && !force_fb) fb_push(rt, (H << 5) | (uint32_t)v);
        } else {
            const int hv = gg.hv[v];
            const uint32_t Hc = low ? H : (uint32_t)compress_bit(H, v - bT);
            V *dst = Y1 + gg.y1off[v];
            for (uint32_t si = t; si < gg.KT; si += kThreads) {
                const uint32_t msk = seedT[si];
                uint32_t rank = si;
                if (low) {
                    if ((msk >> v) & 1) continue;
                    const uint32_t cm = (uint32_t)compress_bit(msk, v);
                    rank = offT1[__popc(cm)];
                    int k = 0;
                    uint32_t rest = cm;
                    while (rest) {
                        const int p = __ffs(rest) - 1;
                        rest &= rest - 1;
                        rank += C(sbin, p, ++k);
                    }
                }
                dst[y1_at(rank, Hc, hv, gg.kg4[v])] = P::from_lin(gb[padx(msk)], T);
            }
        }
        __syncthreads();
    };
    // the own Rp block is a partner only for the register bits 0..3: with a
    // loop of their own, it is dead in the loops over the other endpoints;
    // the tile bits and the bits above the tile get a loop each as well
    if constexpr (kSplit) {
        int v = v0;
        for (; v < 4 && v < n; v += vs) endpoint(v);
        for (; v < bT && v < n; v += vs) endpoint(v);
        for (; v < n; v += vs) endpoint(v);
    } else {
        for (int v = 0; v < 4 && v < n; ++v) endpoint(v);
        for (int v = 4; v < bT && v < n; ++v) endpoint(v);
        for (int v = bT; v < n; ++v) endpoint(v);
    }
    if (t == 0 && sfail) fb_push(fb, H);
}

// Three waves per SIMD (168 registers, some spill), which measured faster
// than two without spills: more waves hide the barrier and load latency of
// the endpoint loops.
template <class P, bool kSplit>
__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(3, 3)))
k_gamma_tile_lin(int n, int d, int force_fb, int vsplit, GammaGeom gg, Tables tb,
                 typename P::Store L,
                 typename P::Store R, const typename P::V *__restrict__ qt,
                 typename P::V *__restrict__ Y1, typename P::V *__restrict__ part,
                 uint32_t *fb, uint32_t *rt) {
    gamma_tile_lin_body<P, kSplit>(n, d, force_fb, vsplit, gg, tb, L, R, qt, Y1, part, fb, rt);
}

// Second chance for the endpoints that k_gamma_tile_lin could not scale from
// g_v(H + top) (list[0] items, list[1 + j] = H * 32 + v; the grid walks the
// list). The scale now comes from the largest product of the tile, which
// keeps Gamma_v(H + empty) finite; the outputs are stored only if every
// needed one is at least 2^-1000, since the products that fell below 2^-1074
// (at most 4096) then change none by more than 2^-62 of itself. Outputs below
// that get a third chance under the first scale (below); an endpoint with an
// output valid under neither is recomputed in the number system proper
// (gamma_tile), here as well: it is rare, and a launch of its own cost every
// solve 4.6 us.
// Same layouts as k_gamma_tile_lin, layout C for every thread.
template <class P>
__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 2)))
k_gamma_tile_retry(int n, int d, GammaGeom gg, Tables tb, typename P::Store L,
                   typename P::Store R, const typename P::V *__restrict__ qt,
                   typename P::V *__restrict__ Y1, typename P::V *__restrict__ part,
                   const uint32_t *list, uint32_t *fb) {
    using V = typename P::V;
    using R16 = typename P::Raw16;
    using A = typename P::Anchor;
    constexpr int bT = 12, NR = 16;
    extern __shared__ unsigned char smem[];
    double *gb = reinterpret_cast<double *>(smem);             // padded 2^12 entries
    uint32_t *sbin = reinterpret_cast<uint32_t *>(gb + 4096 + 256);
    uint32_t *seedT = sbin + 33 * 33;                          // K(12, d) ranked masks
    __shared__ V sq[32];
    __shared__ uint32_t offT1[34];
    __shared__ int smax;
    __shared__ A sT2;
    const uint32_t t = threadIdx.x;
    for (int x = t; x < 33 * 33; x += kThreads) sbin[x] = tb.binom[x];
    for (uint32_t x = t; x < gg.KT; x += kThreads) seedT[x] = tb.seedmask[x];
    if (t < (uint32_t)n) sq[t] = qt[t];
    __syncthreads();
    if (t <= (uint32_t)d + 1) offT1[t] = Kcount(sbin, bT - 1, (int)t - 1);
    const uint32_t tlo = t & 15, thi = t >> 4;
    const uint32_t nitem = list[0];
    for (uint32_t it = blockIdx.x; it < nitem; it += gridDim.x) {
        __syncthreads();
        const uint32_t item = list[1 + it];
        const uint32_t H = item >> 5;
        const int v = (int)(item & 31);
        const bool low = v < bT;
        const uint64_t Hf = (uint64_t)H << bT;
        const uint64_t x0 = Hf | (t << 4);
        const int ht = __popcll(Hf) + __popc(t);
        const R16 Lw = P::load16_raw(L, x0);
        const R16 Rown = P::load16_raw(R, x0);
        R16 Rv = Rown;
        if (v >= 4)
            Rv = P::load16_raw(R, low ? Hf | ((uint64_t)(t | (1u << (v - 4))) << 4) : x0 | (1ull << v));
        const bool excl = v >= 4 && low && ((t >> (v - 4)) & 1);
        // products q(|S|) L(S) Rp(S + v) as undecoded values, and their largest
        V pv[NR];
#pragma unroll
        for (int r = 0; r < NR; ++r)
            pv[r] = P::mul_raw(sq[min(ht + __builtin_popcount(r), 31)], P::at16_nz(Lw, r));
        if (v < 4) {
            // the partner of register r is register r + 2^v of the own block
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if (v != q) continue;
#pragma unroll
                for (int r = 0; r < NR; ++r)
                    pv[r] = ((r >> q) & 1) ? P::zero()
                                           : P::mul_raw(pv[r], P::at16_nz(Rown, r | (1 << q)));
            }
        } else {
#pragma unroll
            for (int r = 0; r < NR; ++r)
                pv[r] = excl ? P::zero() : P::mul_raw(pv[r], P::at16_nz(Rv, r));
        }
        double mx = -1e300;
#pragma unroll
        for (int r = 0; r < NR; ++r) mx = fmax(mx, P::log2_of(pv[r]));
        if (t == 0) smax = -(1 << 30);
        __syncthreads();
        atomicMax(&smax, (int)fmax(mx, -1073741824.0));
        __syncthreads();
        const bool any = smax > -(1 << 29);
        const A T = P::anchor_high(smax);
        // downward zeta of the products under scale Ts over the tile bits
        // but v, into gb (layout C for every thread)
        auto zeta3 = [&](const A Ts) {
            double g[NR];
#pragma unroll
            for (int r = 0; r < NR; ++r) g[r] = P::prod2_lin(pv[r], P::one(), Ts);
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (v != q) lin_zeta_down<NR>(g, q);
#pragma unroll
            for (int r = 0; r < NR; ++r) gb[padx((t << 4) | r)] = g[r];
            __syncthreads();
#pragma unroll
            for (int r = 0; r < NR; ++r) g[r] = gb[padx((thi << 8) | (r << 4) | tlo)];
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (v != 4 + q) lin_zeta_down<NR>(g, q);
#pragma unroll
            for (int r = 0; r < NR; ++r) gb[padx((thi << 8) | (r << 4) | tlo)] = g[r];
            __syncthreads();
#pragma unroll
            for (int r = 0; r < NR; ++r) g[r] = gb[padx((r << 8) | t)];
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (v != 8 + q) lin_zeta_down<NR>(g, q);
#pragma unroll
            for (int r = 0; r < NR; ++r) gb[padx((r << 8) | t)] = g[r];
            __syncthreads();
        };
        zeta3(T);
        bool small = !(any && gb[padx(0)] <= 1.0e300);
        for (uint32_t si = t; si < gg.KT && !small; si += kThreads) {
            const uint32_t msk = seedT[si];
            if (low && ((msk >> v) & 1)) continue;
            small = !(gb[padx(msk)] >= 0x1p-1000);
        }
        // Third chance for outputs below 2^-1000 under the largest product's
        // scale: a pass under the scale of g_v(H + top) (every needed output
        // holds that term, so it is at least about 2^-1000 there; an output
        // that overflows there is at least 2^-1000 under the first scale when
        // the two scales lie less than 2024 binary orders apart). Each needed
        // output is taken from the pass where it is at least 2^-1000 and
        // finite; an endpoint with an output valid in neither goes to
        // gamma_tile. Outputs of the first pass wait in registers
        // (at most 4 per thread, K(12, d) <= 1024).
        constexpr int kMaxOut = 4;
        double keep1[kMaxOut];
        A T2 = T;
        bool two = false;
        if (__syncthreads_or(small ? 1 : 0)) {
            bool ok = any && gg.KT <= kMaxOut * kThreads;
            if (ok) {
                // g_v(H + top): top = every tile bit but v, entry x_top of layout A
                const uint32_t xtop = low ? (0xfffu & ~(1u << v)) : 0xfffu;
                if (t == (xtop >> 4)) {
                    A Tt{};
                    V top = P::zero();
#pragma unroll
                    for (int r = 0; r < NR; ++r)
                        if ((uint32_t)r == (xtop & 15u)) top = pv[r];
                    smax = P::anchor_of(top, &Tt) ? 1 : 0;
                    sT2 = Tt;
                }
                __syncthreads();
                ok = smax != 0;
                T2 = sT2;
            }
            if (ok) {
#pragma unroll
                for (int k = 0; k < kMaxOut; ++k) {
                    const uint32_t si = t + k * kThreads;
                    keep1[k] = si < gg.KT ? gb[padx(seedT[si])] : 0.0;
                }
                __syncthreads();                  // gb is rewritten by the second pass
                zeta3(T2);
                bool fail = false;
#pragma unroll
                for (int k = 0; k < kMaxOut; ++k) {
                    const uint32_t si = t + k * kThreads;
                    if (si >= gg.KT) continue;
                    const uint32_t msk = seedT[si];
                    if (low && ((msk >> v) & 1)) continue;
                    const double y2 = gb[padx(msk)];
                    fail = fail || !(keep1[k] >= 0x1p-1000 || (y2 >= 0x1p-1000 && y2 <= 1.0e300));
                }
                ok = __syncthreads_or(fail ? 1 : 0) == 0;
            }
            if (!ok) {
                // this endpoint in the number system proper (same LDS layout: the
                // tables in LDS are written again with the same values); fb[0] is
                // only a count here, no list
                if (t == 0) atomicAdd(fb, 1u);
                __syncthreads();
                gamma_tile<P>(n, d, gg, tb, L, R, qt, Y1, part, H, v);
                continue;
            }
            two = true;
        }
        const int hv = gg.hv[v];
        const uint32_t Hc = low ? H : (uint32_t)compress_bit(H, v - bT);
        V *dst = Y1 + gg.y1off[v];
        auto rank_of = [&](uint32_t si, uint32_t msk) {
            uint32_t rank = si;
            if (low) {
                const uint32_t cm = (uint32_t)compress_bit(msk, v);
                rank = offT1[__popc(cm)];
                int k = 0;
                uint32_t rest = cm;
                while (rest) {
                    const int p = __ffs(rest) - 1;
                    rest &= rest - 1;
                    rank += C(sbin, p, ++k);
                }
            }
            return rank;
        };
        if (two) {
#pragma unroll
            for (int k = 0; k < kMaxOut; ++k) {
                const uint32_t si = t + k * kThreads;
                if (si >= gg.KT) break;
                const uint32_t msk = seedT[si];
                if (low && ((msk >> v) & 1)) continue;
                const bool first = keep1[k] >= 0x1p-1000;
                dst[y1_at(rank_of(si, msk), Hc, hv, gg.kg4[v])] =
                    P::from_lin(first ? keep1[k] : gb[padx(msk)], first ? T : T2);
            }
        } else {
            for (uint32_t si = t; si < gg.KT; si += kThreads) {
                const uint32_t msk = seedT[si];
                if (low && ((msk >> v) & 1)) continue;
                dst[y1_at(rank_of(si, msk), Hc, hv, gg.kg4[v])] = P::from_lin(gb[padx(msk)], T);
            }
        }
    }
}

// Output rank (within node v's ranked parent sets) of G_L + (high pattern
// x shifted by shift), |G_L| = sigma with colex rank cl.
__device__ inline uint32_t out_rank(const uint32_t *bn, int N, int sigma, uint32_t cl,
                                    uint32_t x, int shift) {
    int k = 0;
    uint32_t r = cl;
    while (x) {
        const int p = __ffs(x) - 1;
        x &= x - 1;
        r += C(bn, shift + p, sigma + (++k));
    }
    return Kcount(bn, N, sigma + k - 1) + r;
}

// Seed of endpoint v's compressed tile: size class and colex rank of the
// s-th ranked mask over bv bits.
__device__ inline void seed_of(const uint32_t *bn, int bv, uint32_t s, int *sigma, uint32_t *cl) {
    int k = 0;
    uint32_t off = 0;
    while (s >= off + C(bn, bv, k)) off += C(bn, bv, k++);
    *sigma = k;
    *cl = s - off;
}

// Locate (v, local index) of a flat block index over per-v block counts.
__device__ inline int find_v(const uint32_t *pref, int n, uint32_t b) {
    int v = 0;
    while (v + 1 < n + 1 && pref[v + 1] <= b) ++v;
    return v;
}

// ------------------------------- a6: Gamma, high bits, two levels (A, B)
// Level A, workgroup (v, seed, Ht): the low a bits of Hc; output for every
// a-bit pattern p with at most d ones: Y2_v[seed][p][Ht].
template <class P>
__global__ void __launch_bounds__(kThreads)
k_gamma_highA(int n, int d, int a, uint32_t KA, GammaGeom gg, Tables tb,
              const typename P::V *__restrict__ Y1, typename P::V *__restrict__ Y2) {
    using V = typename P::V;
    extern __shared__ unsigned char smem[];
    V *vec = reinterpret_cast<V *>(smem);
    const int v = find_v(gg.blkA, n, blockIdx.x);
    const int bv = gg.bv[v], hv = gg.hv[v];
    const int hB = hv - a;
    const uint32_t local = y1_reader_item(blockIdx.x - gg.blkA[v], hB, gg.kg4[v]);
    const uint32_t Ht = local & ((1u << hB) - 1);
    const uint32_t s = local >> hB;
    const int t = threadIdx.x;
    const uint32_t *bn = tb.binom;
    int sigma;
    uint32_t cl;
    seed_of(bn, bv, s, &sigma, &cl);
    const int tr = d - sigma;
    const V *src = Y1 + gg.y1off[v] + y1_at(s, (uint64_t)Ht << a, hv, gg.kg4[v]);
    const uint32_t st = y1_stride(s, gg.kg4[v]);
    for (uint32_t x = t; x < (1u << a); x += kThreads) vec[x] = src[(size_t)x * st];
    __syncthreads();
    for (int j = 0; j < a; ++j) {
        const uint32_t cntj = Kcount(bn, j, d);
        const uint32_t tot = cntj << (a - 1 - j);
        for (uint32_t idx = t; idx < tot; idx += kThreads) {
            const uint32_t hi = idx / cntj;
            const uint32_t p = tb.pat[idx - hi * cntj];
            if (__popc(p) > tr) continue;
            const uint32_t Tm = (hi << (j + 1)) | p;
            vec[Tm] = P::add(vec[Tm], vec[Tm | (1u << j)]);
        }
        __syncthreads();
    }
    V *dst = Y2 + gg.y2off[v];
    for (uint32_t pi = t; pi < KA; pi += kThreads)
        dst[(((size_t)s * KA + pi) << hB) + Ht] = vec[tb.pat[pi]];
}

// Dense downward zeta over 12 bits: src[x], x < 2^12, into vec[padx(x)]
// (256 threads x 16 entries; bits 0..3, 4..7, 8..11 in three layouts joined
// through LDS). An entry with at most d - sigma ones receives the same
// additions in the same order as in the truncated pass of k_gamma_high1 /
// k_gamma_highA, so the results agree exactly; the other entries are
// computed too and never read. No pattern table, division or skip test per
// update. Ends with a barrier.
template <class P>
__device__ __forceinline__ void dense_zeta_down12_regs(typename P::V (&g)[16],
                                                       typename P::V *vec, uint32_t t) {
    constexpr int NR = 16;
    auto zeta4 = [&]() {
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int r = 0; r < NR; ++r)
                if (!((r >> q) & 1)) g[r] = P::add(g[r], g[r | (1 << q)]);
    };
    zeta4();                                            // bits 0..3
#pragma unroll
    for (int r = 0; r < NR; ++r) vec[padx((t << 4) | r)] = g[r];
    __syncthreads();
    const uint32_t tlo = t & 15, thi = t >> 4;
#pragma unroll
    for (int r = 0; r < NR; ++r) g[r] = vec[padx((thi << 8) | (r << 4) | tlo)];
    zeta4();                                            // bits 4..7
#pragma unroll
    for (int r = 0; r < NR; ++r) vec[padx((thi << 8) | (r << 4) | tlo)] = g[r];
    __syncthreads();
#pragma unroll
    for (int r = 0; r < NR; ++r) g[r] = vec[padx((r << 8) | t)];
    zeta4();                                            // bits 8..11
#pragma unroll
    for (int r = 0; r < NR; ++r) vec[padx((r << 8) | t)] = g[r];
    __syncthreads();
}

// The same zeta from layout C (g[r] = entry r * 256 + t, so that the loads
// of consecutive lanes touch consecutive entries), its bits in the order
// 8..11, 4..7, 0..3; the results end in vec[padx(x)] as above.
template <class P>
__device__ __forceinline__ void dense_zeta_down12_regsC(typename P::V (&g)[16],
                                                        typename P::V *vec, uint32_t t) {
    constexpr int NR = 16;
    auto zeta4 = [&]() {
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int r = 0; r < NR; ++r)
                if (!((r >> q) & 1)) g[r] = P::add(g[r], g[r | (1 << q)]);
    };
    zeta4();                                            // bits 8..11
#pragma unroll
    for (int r = 0; r < NR; ++r) vec[padx((r << 8) | t)] = g[r];
    __syncthreads();
    const uint32_t tlo = t & 15, thi = t >> 4;
#pragma unroll
    for (int r = 0; r < NR; ++r) g[r] = vec[padx((thi << 8) | (r << 4) | tlo)];
    zeta4();                                            // bits 4..7
#pragma unroll
    for (int r = 0; r < NR; ++r) vec[padx((thi << 8) | (r << 4) | tlo)] = g[r];
    __syncthreads();
#pragma unroll
    for (int r = 0; r < NR; ++r) g[r] = vec[padx((t << 4) | r)];
    zeta4();                                            // bits 0..3
#pragma unroll
    for (int r = 0; r < NR; ++r) vec[padx((t << 4) | r)] = g[r];
    __syncthreads();
}

template <class P>
__device__ __forceinline__ void dense_zeta_down12(const typename P::V *__restrict__ src,
                                                  uint32_t stride, typename P::V *vec,
                                                  uint32_t t) {
    typename P::V g[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) g[r] = src[(size_t)((t << 4) | r) * stride];
    dense_zeta_down12_regs<P>(g, vec, t);
}

// The FP32-scaled form of the dense 12-bit passes over the grouped ranks of
// Y1: a workgroup loads the four ranks of a group at once (32 bytes per
// entry, each byte read once, consecutive lanes on consecutive entries) and
// runs the zeta for each in turn; the ranks
// past the groups take one workgroup each. item: the workgroup's index within
// endpoint v; the grouped items come first, (group, Ht) with Ht fastest.
// Calls out(s, Ht) after the zeta of rank s has left vec (ends with a barrier).
template <class Out>
__device__ __forceinline__ void dense_zeta_down12_x4(const X32 *__restrict__ Y1v, int hv, int hB,
                                                     uint32_t kg4, uint32_t item, X32 *vec,
                                                     uint32_t t, Out out) {
    const uint32_t G = (kg4 >> 2) << hB;
    const uint32_t hmask = (1u << hB) - 1u;
    if (item < G) {
        const uint32_t s0 = (item >> hB) << 2, Ht = item & hmask;
        const uint4 *src = reinterpret_cast<const uint4 *>(Y1v + y1_at(s0, (uint64_t)Ht << 12, hv, kg4));
        uint4 raw[16][2];                     // entry r * 256 + t: ranks s0, s0 + 1 | s0 + 2, s0 + 3
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            raw[r][0] = src[2 * ((r << 8) | t)];
            raw[r][1] = src[2 * ((r << 8) | t) + 1];
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            X32 g[16];
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const uint4 w = raw[r][q >> 1];
                g[r] = (q & 1) ? X32{__uint_as_float(w.z), (int)w.w}
                               : X32{__uint_as_float(w.x), (int)w.y};
            }
            dense_zeta_down12_regsC<PolX32>(g, vec, t);
            out(s0 + q, Ht);
            __syncthreads();                  // vec is read by out()
        }
    } else {
        const uint32_t x = item - G;
        const uint32_t s = kg4 + (x >> hB), Ht = x & hmask;
        const X32 *src = Y1v + y1_at(s, (uint64_t)Ht << 12, hv, kg4);
        X32 g[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) g[r] = src[(r << 8) | t];
        dense_zeta_down12_regsC<PolX32>(g, vec, t);
        out(s, Ht);
    }
}

// Level A for a = 12 in the log form. The row's logarithms become plain
// doubles under one scale, exp(x - M) 2^960 with M the row's largest (so the
// sum of 4096 of them stays below 2^972), the dense 12-bit zeta runs in FP64
// adds, and the outputs go back as logarithms. They are kept only if every
// needed output (at most d - sigma ones) is at least 2^-1000: the values that
// fell below 2^-1074 (at most 4096) then change none by more than 2^-62 of
// itself. Otherwise, or always with force_trunc (tests), the workgroup runs
// the truncated log-add pass of k_gamma_highA on the row.
__global__ void __launch_bounds__(kThreads)
k_gamma_highA12_log(int n, int d, uint32_t KA, int force_trunc, GammaGeom gg, Tables tb,
                    const double *__restrict__ Y1, double *__restrict__ Y2) {
    constexpr int a = 12;
    extern __shared__ unsigned char smem[];
    double *vec = reinterpret_cast<double *>(smem);   // 2^12 entries, padx or plain
    __shared__ double red[kThreads];
    const int v = find_v(gg.blkA, n, blockIdx.x);
    const int bv = gg.bv[v], hv = gg.hv[v];
    const int hB = hv - a;
    const uint32_t local = y1_reader_item(blockIdx.x - gg.blkA[v], hB, gg.kg4[v]);
    const uint32_t Ht = local & ((1u << hB) - 1);
    const uint32_t s = local >> hB;
    const uint32_t t = threadIdx.x;
    const uint32_t *bn = tb.binom;
    int sigma;
    uint32_t cl;
    seed_of(bn, bv, s, &sigma, &cl);
    const int tr = d - sigma;
    const double *src = Y1 + gg.y1off[v] + y1_at(s, (uint64_t)Ht << a, hv, gg.kg4[v]);
    const uint32_t st = y1_stride(s, gg.kg4[v]);
    double *dst = Y2 + gg.y2off[v];
    auto out_at = [&](uint32_t pi) -> double & { return dst[(((size_t)s * KA + pi) << hB) + Ht]; };
    double g[16];
    double mx = -__builtin_huge_val();
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        g[r] = src[(size_t)((t << 4) | r) * st];
        mx = fmax(mx, g[r]);
    }
    mx = block_reduce(mx, red, [](double x, double y) { return fmax(x, y); });
    if (!(mx > -1e300)) {                            // an empty row: every output is zero
        for (uint32_t pi = t; pi < KA; pi += kThreads) out_at(pi) = -__builtin_huge_val();
        return;
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) g[r] = exp_below(g[r] - mx, 960);
    dense_zeta_down12_regs<Lin64>(g, vec, t);
    bool small = false;
    for (uint32_t pi = t; pi < KA; pi += kThreads) {
        const uint32_t x = tb.pat[pi];
        if (__popc(x) <= tr) small = small || !(vec[padx(x)] >= 0x1p-1000);
    }
    if (!__syncthreads_or(small || force_trunc ? 1 : 0)) {
        for (uint32_t pi = t; pi < KA; pi += kThreads) {
            const double y = vec[padx(tb.pat[pi])];
            out_at(pi) = y > 0.0 ? log_scaled(y, 960) + mx : -__builtin_huge_val();
        }
        return;
    }
    // the truncated log-add pass of k_gamma_highA
    for (uint32_t x = t; x < (1u << a); x += kThreads) vec[x] = src[(size_t)x * st];
    __syncthreads();
    for (int j = 0; j < a; ++j) {
        const uint32_t cntj = Kcount(bn, j, d);
        const uint32_t tot = cntj << (a - 1 - j);
        for (uint32_t idx = t; idx < tot; idx += kThreads) {
            const uint32_t hi = idx / cntj;
            const uint32_t p = tb.pat[idx - hi * cntj];
            if (__popc(p) > tr) continue;
            const uint32_t Tm = (hi << (j + 1)) | p;
            vec[Tm] = PolLog::add(vec[Tm], vec[Tm | (1u << j)]);
        }
        __syncthreads();
    }
    for (uint32_t pi = t; pi < KA; pi += kThreads) out_at(pi) = vec[tb.pat[pi]];
}

// Downward zeta of 4096 entries over the index bits of `bits`, one after the
// other as in dense_zeta_down12_regsC (layout C in g, the results in vec[padx]).
template <class P>
__device__ __forceinline__ void masked_zeta_down12(typename P::V (&g)[16], typename P::V *vec,
                                                   uint32_t bits, uint32_t t) {
    constexpr int NR = 16;
    auto zeta4 = [&](int first) {
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if ((bits >> (first + q)) & 1) {
#pragma unroll
                for (int r = 0; r < NR; ++r)
                    if (!((r >> q) & 1)) g[r] = P::add(g[r], g[r | (1 << q)]);
            }
    };
    zeta4(8);
#pragma unroll
    for (int r = 0; r < NR; ++r) vec[padx((r << 8) | t)] = g[r];
    __syncthreads();
    const uint32_t tlo = t & 15, thi = t >> 4;
    if (bits & 0xf0u) {
#pragma unroll
        for (int r = 0; r < NR; ++r) g[r] = vec[padx((thi << 8) | (r << 4) | tlo)];
        zeta4(4);
#pragma unroll
        for (int r = 0; r < NR; ++r) vec[padx((thi << 8) | (r << 4) | tlo)] = g[r];
        __syncthreads();
    }
    if (bits & 0xfu) {
#pragma unroll
        for (int r = 0; r < NR; ++r) g[r] = vec[padx((t << 4) | r)];
        zeta4(0);
#pragma unroll
        for (int r = 0; r < NR; ++r) vec[padx((t << 4) | r)] = g[r];
        __syncthreads();
    }
}

// ------------------------------------- a5 + a6: Gamma of a small lattice
// n < 12: workgroup = endpoint v, the whole lattice in one block of 4096 (zero
// beyond 2^n): products q(|S|) L(S) Rp(S + v), downward zeta over every bit but
// v, outputs straight to Gamma_v. Log form: as in k_gamma_high1, plain doubles
// under one scale when every output is at least 2^-1000 there, else (or with
// force_log) log-adds. Latency bound: 5 to 6 us where the tile kernel with its
// truncated passes over LDS and the copy of its outputs took 17 (n = 10).
template <class P>
__global__ void __launch_bounds__(kThreads)
k_gamma_small(int n, uint32_t K, int force_log, Tables tb, typename P::Store L,
              typename P::Store R, const typename P::V *__restrict__ qt,
              typename P::V *__restrict__ gam) {
    using V = typename P::V;
    constexpr bool kLog = std::is_same<P, PolLog>::value;
    extern __shared__ unsigned char smem[];
    V *vec = reinterpret_cast<V *>(smem);                  // 2^12 entries, padded
    __shared__ V sq[32];
    __shared__ double red[kThreads];
    const int v = blockIdx.x;
    const uint32_t t = threadIdx.x, size = 1u << n, vb = 1u << v;
    const uint32_t bits = (size - 1u) & ~vb;
    if (t < (uint32_t)n) sq[t] = qt[t];
    __syncthreads();
    V g[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const uint32_t S = ((uint32_t)r << 8) | t;
        g[r] = P::zero();
        if (S < size && !(S & vb))
            g[r] = P::norm_v(P::mul_raw(P::mul_raw(sq[__popc(S)], P::load(L, S)),
                                        P::load(R, S | vb)));
    }
    auto each = [&](auto f) {
        for (uint32_t r = t; r < K; r += kThreads)
            f(r, padx((uint32_t)expand_bit(tb.famask[r], v)));
    };
    V *out = gam + (size_t)v * K;
    if constexpr (kLog) {
        double mx = -__builtin_huge_val();
#pragma unroll
        for (int r = 0; r < 16; ++r) mx = fmax(mx, g[r]);
        mx = block_reduce(mx, red, [](double x, double y) { return fmax(x, y); });
        if (!force_log && mx > -1e300) {
            double y[16];
#pragma unroll
            for (int r = 0; r < 16; ++r) y[r] = exp_below(g[r] - mx, 960);
            masked_zeta_down12<Lin64>(y, vec, bits, t);
            bool small = false;
            each([&](uint32_t, uint32_t at) { small = small || !(vec[at] >= 0x1p-1000); });
            if (!__syncthreads_or(small ? 1 : 0)) {
                each([&](uint32_t r, uint32_t at) { out[r] = log_scaled(vec[at], 960) + mx; });
                return;
            }
        }
    }
    masked_zeta_down12<P>(g, vec, bits, t);
    each([&](uint32_t r, uint32_t at) { out[r] = P::norm_v(vec[at]); });
}

// ---------------------------------- a6: Gamma, high bits, one level
// The vectors Y1_v[rank][.] over v's hv <= 12 high bits, 2^(12 - hv) ranks (4096
// entries) per workgroup: downward zeta over the hv bits, outputs with at most
// d - |G_L| of them to Gamma_v. While a group of four ranks fits (hv <= 10) the
// entries keep their order in Y1 (rank mod 4 fastest), so every load is
// consecutive, and the zeta runs over index bits 2 .. hv + 1; the ranks past
// the groups, and all ranks for hv = 11 and 12, lie row after row.
// Log form: each row's logarithms become plain doubles under a scale of the
// row, exp(x - M) 2^960 with M >= its largest by less than ln 2, and the adds
// are FP64 adds; the outputs are kept only if every needed one is at least
// 2^-1000 (the values that fell below 2^-1074, at most 4096, then change none
// by more than 2^-62 of itself); otherwise, or with force_log (tests), the
// workgroup runs the zeta in log-adds. So does one with an entry beyond 3.6e8
// nats (many millions of samples, or a prior of that size), whose binary
// exponent the 32-bit row maxima do not hold beside their mark of an empty row.
// One row per workgroup, truncated by pattern lists and, in the log form, in
// log-adds, this was 98 us at n = 20 (FP64, d = 4), 1.04 ms at n = 25 and 48 us
// at n = 22 (FP32-scaled, d = 3); now 29 us, 0.25 ms and 24 us.
template <class P>
__global__ void __launch_bounds__(kThreads)
k_gamma_high1(int n, int d, uint32_t K, int force_log, GammaGeom gg, Tables tb,
              const typename P::V *__restrict__ Y1, typename P::V *__restrict__ gam) {
    using V = typename P::V;
    constexpr bool kLog = std::is_same<P, PolLog>::value;
    extern __shared__ unsigned char smem[];
    V *vec = reinterpret_cast<V *>(smem);                              // 2^12 entries, padded
    uint32_t *bn = reinterpret_cast<uint32_t *>(vec + 4096 + 256);     // binomials
    uint32_t *cum = bn + 33 * 33;                                      // cum[k] = K(n - 1, k - 1)
    uint32_t *rowinfo = cum + 34;          // per row: colex rank of G_L, |G_L| in the top bits
    int *rowmax = reinterpret_cast<int *>(rowinfo + (4096u >> gg.hmin1));
    const int N = n - 1;
    const int v = find_v(gg.blk1, n, blockIdx.x);
    const uint32_t item = blockIdx.x - gg.blk1[v];
    const uint32_t t = threadIdx.x;
    const int bv = gg.bv[v], hv = gg.hv[v];
    const uint32_t kg4 = gg.kg4[v], kg = gg.kg[v];
    const uint32_t rows = 4096u >> hv, ymask = (1u << hv) - 1u;
    const uint32_t nG = hv <= 10 ? (kg4 + rows - 1) / rows : 0u;       // grouped chunks
    const bool grouped = item < nG;
    const uint32_t s0 = grouped ? item * rows
                        : hv <= 10 ? kg4 + (item - nG) * rows
                        : hv == 12 ? y1_reader_item(item, 0, kg4) : item * rows;
    const uint32_t s1 = min(grouped ? kg4 : kg, s0 + rows);
    const V *src = Y1 + gg.y1off[v];
    // entry x of the chunk: rank s0 + row(x), high part y(x)
    auto row_of = [&](uint32_t x) {
        return grouped ? ((x >> (hv + 2)) << 2) | (x & 3u) : x >> hv;
    };
    auto y_of = [&](uint32_t x) { return grouped ? (x >> 2) & ymask : x & ymask; };
    const uint32_t bits = grouped ? ymask << 2 : ymask;
    const V *gsrc = src + ((size_t)s0 << hv);   // grouped: the chunk is contiguous
    auto load = [&](uint32_t x) -> V {
        const uint32_t s = s0 + row_of(x);
        return s < s1 ? (grouped ? gsrc[x] : src[y1_at(s, y_of(x), hv, kg4)]) : P::zero();
    };
    V g[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) g[r] = load((r << 8) | t);
    for (int x = t; x < 33 * 33; x += kThreads) bn[x] = tb.binom[x];
    __syncthreads();
    if (t <= (uint32_t)d + 1) cum[t] = Kcount(bn, N, (int)t - 1);
    for (uint32_t x = t; x < rows && s0 + x < s1; x += kThreads) {
        int sigma;
        uint32_t cl;
        seed_of(bn, bv, s0 + x, &sigma, &cl);
        rowinfo[x] = cl | ((uint32_t)sigma << 27);
    }
    bool lin = false, far = false;
    if constexpr (kLog) {
        if (!force_log) {
            lin = true;
            for (uint32_t x = t; x < rows; x += kThreads) rowmax[x] = -(1 << 30);
            __syncthreads();
            // largest of the row's entries held by a thread, then, where lanes
            // share a row, by the wave, then one LDS maximum per row and wave
            int e[16];
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const bool held = g[r] > -1e300;
                far = far || (held && fabs(g[r]) > 3.6e8);
                e[r] = held ? (int)ceil(fmax(g[r], -3.6e8) * 1.4426950408889634074) : -(1 << 30);
            }
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if ((bits >> (8 + q)) & 1) {
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        if (!((r >> q) & 1)) e[r] = max(e[r], e[r | (1 << q)]);
                }
            const int first = grouped ? 2 : 0;
            const bool lead = hv < 6 || ((t & 63u) >> first) == 0;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                if (((uint32_t)r << 8) & bits) continue;         // uniform
                if (hv >= 6)
                    for (int b = first; b < 6; ++b) e[r] = max(e[r], __shfl_xor(e[r], 1 << b));
                if (lead) atomicMax(&rowmax[row_of((r << 8) | t)], e[r]);
            }
            __syncthreads();
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const double M = rowmax[row_of((r << 8) | t)] * 0.69314718055994530942;
                g[r] = exp_below(g[r] - M, 960);
            }
        }
    }
    // needed outputs of the chunk: calls f(x, row info, y)
    auto outputs = [&](auto f) {
        for (uint32_t x = t; x < 4096u; x += kThreads) {
            const uint32_t row = row_of(x), y = y_of(x);
            if (s0 + row >= s1) continue;
            const uint32_t ri = rowinfo[row];
            if (__popc(y) + (int)(ri >> 27) <= d) f(x, ri, y);
        }
    };
    auto put = [&](uint32_t ri, uint32_t y, V z) {
        int k = (int)(ri >> 27);
        uint32_t rank = ri & 0x7ffffffu;
        while (y) {
            const int p = __ffs(y) - 1;
            y &= y - 1;
            rank += bn[(bv + p) * 33 + (++k)];
        }
        gam[(size_t)v * K + cum[k] + rank] = z;
    };
    if constexpr (kLog) {
        if (lin) {
            masked_zeta_down12<Lin64>(g, vec, bits, t);
            bool small = far;
            outputs([&](uint32_t x, uint32_t, uint32_t) {
                const double z = vec[padx(x)];
                // an empty row is zero throughout
                small = small || !(z >= 0x1p-1000 || rowmax[row_of(x)] <= -(1 << 29));
            });
            if (!__syncthreads_or(small ? 1 : 0)) {
                outputs([&](uint32_t x, uint32_t ri, uint32_t y) {
                    const double z = vec[padx(x)];
                    put(ri, y,
                        z > 0.0 ? log_scaled(z, 960) + rowmax[row_of(x)] * 0.69314718055994530942
                                : -__builtin_huge_val());
                });
                return;
            }
#pragma unroll
            for (int r = 0; r < 16; ++r) g[r] = load((r << 8) | t);
        }
    }
    masked_zeta_down12<P>(g, vec, bits, t);
    outputs([&](uint32_t x, uint32_t ri, uint32_t y) { put(ri, y, vec[padx(x)]); });
}

// Level A for a = 12, FP32-scaled form: the outputs of k_gamma_highA from
// the dense zeta, over groups of ranks.
__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(3, 3)))
k_gamma_highA12(int n, uint32_t KA, GammaGeom gg, Tables tb, const X32 *__restrict__ Y1,
                   X32 *__restrict__ Y2) {
    extern __shared__ unsigned char smem[];
    X32 *vec = reinterpret_cast<X32 *>(smem);   // 2^12 entries at padx indices
    const int v = find_v(gg.blkAx4, n, blockIdx.x);
    const int hB = gg.hv[v] - 12;
    const uint32_t t = threadIdx.x;
    X32 *dst = Y2 + gg.y2off[v];
    dense_zeta_down12_x4(Y1 + gg.y1off[v], gg.hv[v], hB, gg.kg4[v], blockIdx.x - gg.blkAx4[v],
                         vec, t, [&](uint32_t s, uint32_t Ht) {
                             for (uint32_t pi = t; pi < KA; pi += kThreads)
                                 dst[(((size_t)s * KA + pi) << hB) + Ht] = vec[padx(tb.pat[pi])];
                         });
}

// One level with hv = 12 (every one-level endpoint when n = 25), FP32-scaled
// form: the outputs of k_gamma_high1 from the dense zeta, over groups of ranks.
__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(3, 3)))
k_gamma_high1_12(int n, int d, uint32_t K, GammaGeom gg, Tables tb,
                    const X32 *__restrict__ Y1, X32 *__restrict__ gam) {
    extern __shared__ unsigned char smem[];
    X32 *vec = reinterpret_cast<X32 *>(smem);   // 2^12 entries at padx indices
    const int N = n - 1;
    const int v = find_v(gg.blk1x4, n, blockIdx.x);
    const uint32_t t = threadIdx.x;
    const uint32_t *bn = tb.binom;
    const int bv = gg.bv[v];
    const uint32_t npat = Kcount(bn, 12, d);
    dense_zeta_down12_x4(Y1 + gg.y1off[v], 12, 0, gg.kg4[v], blockIdx.x - gg.blk1x4[v], vec, t,
                         [&](uint32_t s, uint32_t) {
                             int sigma;
                             uint32_t cl;
                             seed_of(bn, bv, s, &sigma, &cl);
                             const int tr = d - sigma;
                             for (uint32_t idx = t; idx < npat; idx += kThreads) {
                                 const uint32_t x = tb.pat[idx];
                                 if (__popc(x) > tr) continue;
                                 gam[(size_t)v * K + out_rank(bn, N, sigma, cl, x, bv)] =
                                     vec[padx(x)];
                             }
                         });
}

// Level B, workgroup (v, seed): for each a-bit pattern p and each output
// pattern y over the remaining hB bits, the superset sum over y' of y. With
// hB <= 6 a wave takes 64 / 2^hB patterns p at a time, 2^hB lanes each: lane
// y of a pattern loads entry y of its row (coalesced loads) and the downward
// zeta over the hB bits runs across those lanes by shuffles. Larger hB
// (n = 31) sums each output's supersets in turn.
template <class P>
__global__ void __launch_bounds__(kThreads)
k_gamma_highB(int n, int d, int a, uint32_t KA, uint32_t K, GammaGeom gg, Tables tb,
              const typename P::V *__restrict__ Y2, typename P::V *__restrict__ gam) {
    using V = typename P::V;
    const int N = n - 1;
    const int v = find_v(gg.blkB, n, blockIdx.x);
    const uint32_t s = blockIdx.x - gg.blkB[v];
    const int bv = gg.bv[v], hv = gg.hv[v];
    const int hB = hv - a;
    const int t = threadIdx.x;
    const uint32_t *bn = tb.binom;
    int sigma;
    uint32_t cl;
    seed_of(bn, bv, s, &sigma, &cl);
    const int tr = d - sigma;
    const uint32_t ny = 1u << hB;
    const V *base = Y2 + gg.y2off[v];
    if (hB <= 6) {
        // lane = (pattern slot, y): 64 / 2^hB patterns per wave step
        const uint32_t lane = t & 63, y = lane & (ny - 1), sub = lane >> hB;
        const uint32_t ppw = 64u >> hB;
        for (uint32_t p0 = (t >> 6) * ppw; p0 < KA; p0 += (kThreads / 64) * ppw) {
            const uint32_t pi = p0 + sub;
            const uint32_t p = pi < KA ? tb.pat[pi] : 0u;
            const int pp = __popc(p);
            const bool need = pi < KA && pp <= tr;
            V x = need ? base[(((size_t)s * KA + pi) << hB) + y] : P::zero();
            for (int b = 0; b < hB; ++b) {
                const V o = shfl_xor_v(x, 1 << b);
                if (!((y >> b) & 1)) x = P::add(x, o);
            }
            if (need && pp + __popc(y) <= tr)
                gam[(size_t)v * K + out_rank(bn, N, sigma, cl, p | (y << a), bv)] = x;
        }
        return;
    }
    for (uint32_t idx = t; idx < KA * ny; idx += kThreads) {
        const uint32_t pi = idx / ny;
        const uint32_t y = idx - pi * ny;
        const uint32_t p = tb.pat[pi];
        if (__popc(p) + __popc(y) > tr) continue;
        const V *src = base + (((size_t)s * KA + pi) << hB);
        typename P::Acc acc = P::acc_of(P::zero());
        const uint32_t free_bits = (ny - 1) & ~y;
        uint32_t sub = 0;   // all supersets y | sub, sub a submask of free_bits, ascending
        while (true) {
            P::acc_add(acc, src[y | sub]);
            if (sub == free_bits) break;
            sub = (sub - free_bits) & free_bits;
        }
        gam[(size_t)v * K + out_rank(bn, N, sigma, cl, p | (y << a), bv)] = P::acc_value(acc);
    }
}

// ------------------------------------------------------------ a7: edges
// Workgroup (v, j): w_v(G) = beta_v(G) Gamma_v(G). j = 0: sum_G w_v(G)
// against L(V) (the residual) and, when asked for, the parent-set
// posteriors w_v(G) / L(V); j = u + 1: P(u->v) = sum_{G containing u}
// w_v(G) / L(V), the last division in FP64.
// An 8-byte result that another workgroup of the same launch reads: stored to,
// and loaded from, the device's point of coherence (each XCD has an L2 of its
// own), so that no workgroup has to write back its L2 for it.
template <class T>
__device__ inline void store_shared_result(T *p, T x) {
    static_assert(sizeof(T) == 8, "8-byte values");
    uint64_t w;
    __builtin_memcpy(&w, &x, 8);
    __hip_atomic_store(reinterpret_cast<uint64_t *>(p), w, __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
}
template <class T>
__device__ inline T load_shared_result(const T *p) {
    static_assert(sizeof(T) == 8, "8-byte values");
    const uint64_t w = __hip_atomic_load(reinterpret_cast<const uint64_t *>(p), __ATOMIC_RELAXED,
                                         __HIP_MEMORY_SCOPE_AGENT);
    T x;
    __builtin_memcpy(&x, &w, 8);
    return x;
}
// Counts the calling thread, whose shared results are then at the point of
// coherence, and returns true for the last of `total`: first in one of 16
// counters (a cache line each, `done` + 32 * (1 + group)), the last of a group
// in done[0]. One counter for all took 10 us more at n = 16 (544 workgroups).
__device__ inline bool count_done(uint32_t *done, uint32_t id, uint32_t total) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    const uint32_t g = id & 15u, size = (total - g + 15u) / 16u;
    auto add = [](uint32_t *p) {
        return __hip_atomic_fetch_add(p, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    if (add(done + 32 * (1 + g)) != size - 1) return false;
    return add(done) == min(total, 16u) - 1;
}

template <class P>
__device__ inline void edge_sum(int v, int u, int n, uint32_t K,
                                const uint32_t *__restrict__ famask,
                                const typename P::V *__restrict__ beta,
                                const typename P::V *__restrict__ gam, typename P::V LV,
                                double *post, double *resid, double *__restrict__ ps,
                                typename P::V *red) {
    using V = typename P::V;
    const int t = threadIdx.x;
    if (u == v) {
        if (t == 0) post[(size_t)u * n + v] = 0.0;
        return;
    }
    auto add = [](V a, V b) { return P::add(a, b); };
    // parent-set posteriors P(G_v = G | D) = w_v(G) / L(V), when asked for
    if (ps && u < 0) {
        for (uint32_t r = t; r < K; r += kThreads) {
            const double lr =
                P::log_ratio(P::mul(beta[(size_t)v * K + r], gam[(size_t)v * K + r]), LV);
            ps[(size_t)v * K + r] = (lr > -1e300) ? exp(lr) : 0.0;
        }
    }
    const int pu = u < v ? u : u - 1;
    typename P::Acc acc = P::acc_of(P::zero());
    // four sets per step, their loads together (one at a time, skipping the sets
    // without u before the loads, was 55 us at n = 25 instead of 33)
    constexpr int U = 4;
    for (uint32_t r0 = t; r0 < K; r0 += U * kThreads) {
        uint32_t fm[U];
        V b[U], g[U];
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const uint32_t r = min(r0 + k * kThreads, K - 1);
            fm[k] = u < 0 ? 1u : famask[r] >> pu;
            b[k] = beta[(size_t)v * K + r];
            g[k] = gam[(size_t)v * K + r];
        }
#pragma unroll
        for (int k = 0; k < U; ++k)
            if ((fm[k] & 1u) && r0 + k * kThreads < K) P::acc_add(acc, P::mul(b[k], g[k]));
    }
    const V tot = block_reduce(P::acc_value(acc), red, add);
    if (t == 0) {
        const double lr = P::log_ratio(tot, LV);
        if (u < 0) store_shared_result(resid + v, fabs(lr));
        else post[(size_t)u * n + v] = (lr > -1e300) ? exp(lr) : 0.0;
    }
}

// -------------------------------------------------------- invariants
// Every layer sum over |S| = k of L(S) Rp(S) must equal L(V). inv_tile: the
// sum over in-tile layer l of tile H, to part; inv_layer: the layer-k sum over
// the c-th of `chunks` ranges of tiles, to layer[k * chunks + c].
template <class P>
__device__ inline void inv_tile(uint32_t H, int l, int bL, const Tables &tb,
                                const typename P::Store &L, const typename P::Store &R,
                                typename P::V *part, typename P::V *red) {
    using V = typename P::V;
    const uint64_t Hf = (uint64_t)H << bL;
    const int t = threadIdx.x;
    auto add = [](V a, V b) { return P::add(a, b); };
    V acc = P::zero();
    for (uint32_t idx = tb.loff[l] + t; idx < tb.loff[l + 1]; idx += kThreads) {
        const uint64_t S = Hf | tb.lorder[idx];
        acc = P::add(acc, P::mul(P::load(L, S), P::load(R, S)));
    }
    V s = block_reduce(acc, red, add);
    if (t == 0) store_shared_result(part + (size_t)H * (bL + 1) + l, s);
}
template <class P>
__device__ inline void inv_layer(int k, int c, int chunks, int n, int bL, const typename P::V *part,
                                 typename P::V *layer, typename P::V *red) {
    using V = typename P::V;
    const int t = threadIdx.x;
    const uint32_t ntile = 1u << (n - bL);
    const uint32_t per = (ntile + chunks - 1) / chunks;
    const uint32_t h0 = c * per, h1 = min(ntile, h0 + per);
    auto add = [](V a, V b) { return P::add(a, b); };
    V acc = P::zero();
    for (uint32_t H = h0 + t; H < h1; H += kThreads) {
        const int l = k - __popc(H);
        if (l < 0 || l > bL) continue;
        acc = P::add(acc, part[(size_t)H * (bL + 1) + l]);
    }
    V s = block_reduce(acc, red, add);
    if (t == 0) store_shared_result(layer + k * chunks + c, s);
}

// Edge sums, invariants and diagnostics in one launch: workgroups below
// n (n + 1) take an edge sum (v, u) each, u = -1 the sum over all parent sets;
// the others an invariant sum, per chunk of tiles (tiled > 0 chunks: the Gamma
// tile kernel left the tiles' sums in part, bI = 12) or per tile and in-tile
// layer (tiled = 0, bI = the sweep tile, at most 2^9 small tiles). Each counts
// itself in `done` (zero at the start) and the last one writes the
// diagnostics. As three or four launches of 4 to 6 us each this was 17 us of
// an n = 10 solve.
// diag: [0] log L(V), [1] max residual, [2] saturated, [3] flushed,
//       [4] |log Rp(0) - log L(V)|, [5] max layer residual, [6] max edge-sum
//       residual, [7] fallback tiles
template <class P>
__global__ void __launch_bounds__(kThreads)
k_finish(int n, uint32_t K, int tiled, int bI, Tables tb, const uint32_t *__restrict__ famask,
         const typename P::V *__restrict__ beta, const typename P::V *__restrict__ gam,
         typename P::Store L, typename P::Store R, typename P::V *part, typename P::V *layer,
         double *post, double *resid, double *__restrict__ ps,
         const double *__restrict__ gauge_exp, const unsigned long long *__restrict__ cnt,
         const uint32_t *__restrict__ fbA, const uint32_t *__restrict__ fbG, uint32_t *done,
         double *__restrict__ diag) {
    using V = typename P::V;
    __shared__ V red[kThreads];
    __shared__ uint32_t last;
    const int t = threadIdx.x;
    const uint32_t b = blockIdx.x, ne = (uint32_t)(n * (n + 1));
    const V LV = P::load(L, (1ull << n) - 1);
    if (b < ne)
        edge_sum<P>((int)(b % n), (int)(b / n) - 1, n, K, famask, beta, gam, LV, post, resid, ps,
                    red);
    else if (tiled)
        inv_layer<P>((int)((b - ne) / tiled), (int)((b - ne) % tiled), tiled, n, bI, part, layer,
                     red);
    else
        inv_tile<P>((b - ne) / (bI + 1), (int)((b - ne) % (bI + 1)), bI, tb, L, R, part, red);
    if (t == 0) last = count_done(done, b, gridDim.x) ? 1u : 0u;
    __syncthreads();
    if (!last || t >= 64) return;
    // lane k sums layer k's parts in order; the largest deviation over the
    // wave (n + 1 <= 32 layers)
    double rl = 0.0;
    if (t <= n) {
        V lk = P::zero();
        if (tiled) {
            for (int c = 0; c < tiled; ++c)
                lk = P::add(lk, load_shared_result(layer + t * tiled + c));
        } else {
            for (uint32_t H = 0; H < (1u << (n - bI)); ++H) {
                const int l = t - __popc(H);
                if (l >= 0 && l <= bI)
                    lk = P::add(lk, load_shared_result(part + (size_t)H * (bI + 1) + l));
            }
        }
        rl = fabs(P::log_ratio(lk, LV));
    }
    double re = t < n ? load_shared_result(resid + t) : 0.0;
    double g = t < 2 * n ? gauge_exp[t] : 0.0;
    for (int o = 32; o > 0; o >>= 1) {
        rl = fmax(rl, __shfl_xor(rl, o));
        re = fmax(re, __shfl_xor(re, o));
        g += __shfl_xor(g, o);                   // integers: exact in any order
    }
    if (t != 0) return;
    const double rLR = fabs(P::log_ratio(P::load(R, 0), LV));
    diag[0] = P::to_log(LV) + g * 0.69314718055994530942;
    diag[1] = fmax(rLR, fmax(rl, re));
    diag[2] = (double)cnt[0];
    diag[3] = (double)cnt[1];
    diag[4] = rLR;
    diag[5] = rl;
    diag[6] = re;
    diag[7] = (double)((fbA ? fbA[0] : 0u) + (fbG ? fbG[0] : 0u));
}

// Forward-only runs (modular features): diag[0] = log L(V) with the gauges,
// [2] / [3] the saturation and flush counts, [7] the fallback tiles; the
// invariant entries are 0 (no backward sweep to check against).
template <class P>
__global__ void k_log_LV(int n, typename P::Store L, const double *__restrict__ gauge_exp,
                         const unsigned long long *__restrict__ cnt,
                         const uint32_t *__restrict__ fbA, double *__restrict__ diag) {
    if (threadIdx.x != 0) return;
    double g = 0.0;
    for (int k = 0; k < 2 * n; ++k) g += gauge_exp[k];
    diag[0] = P::to_log(P::load(L, (1ull << n) - 1)) + g * 0.69314718055994530942;
    diag[1] = diag[4] = diag[5] = diag[6] = 0.0;
    diag[2] = (double)cnt[0];
    diag[3] = (double)cnt[1];
    diag[7] = (double)(fbA ? fbA[0] : 0u);
}

__global__ void k_add_log(double *__restrict__ logp, const double *__restrict__ log_f,
                          size_t count) {
    for (size_t x = (size_t)blockIdx.x * kThreads + threadIdx.x; x < count;
         x += (size_t)gridDim.x * kThreads)
        logp[x] += log_f[x];
}

hipError_t launch_add_log(double *logp, const double *log_f, size_t count, hipStream_t st) {
    const unsigned g = (unsigned)std::min<size_t>((count + kThreads - 1) / kThreads, 4096);
    hipLaunchKernelGGL(k_add_log, dim3(std::max(g, 1u)), dim3(kThreads), 0, st, logp, log_f,
                       count);
    return hipGetLastError();
}

// ------------------------------------------- a1: local scores, binary data
// All-binary data as two bit planes per variable: plane 1 marks the samples
// with value 1, plane 0 those with value 0 (a value out of range is in
// neither, and so ignored, as in k_scores). W 32-bit words per plane; a wave
// takes 64 samples of one variable, then those `step` waves further on (n m
// samples may be more than 2^32, the most threads of a launch).
__device__ void pack2(uint32_t wave0, uint32_t step, int n, int m, int W,
                      const uint8_t *__restrict__ data, uint32_t *__restrict__ bits) {
    const uint32_t W2 = (uint32_t)(W + 1) / 2, lane = threadIdx.x & 63;
    for (uint32_t wave = wave0; wave < (uint32_t)n * W2; wave += step) {
        const uint32_t j = wave / W2, w = 2 * (wave - j * W2);
        const uint32_t s = w * 32 + lane;
        const int x = s < (uint32_t)m ? data[(size_t)j * m + s] : 255;
        const uint64_t zero = __ballot(x == 0), one = __ballot(x == 1);
        if (lane < 2 && w + lane < (uint32_t)W) {
            bits[((size_t)j * 2 + 0) * W + w + lane] = (uint32_t)(zero >> (32 * lane));
            bits[((size_t)j * 2 + 1) * W + w + lane] = (uint32_t)(one >> (32 * lane));
        }
    }
}

// One step of count_cells2's butterfly, at lane bit B.
template <int KP, int B>
__device__ inline void count_scatter(uint32_t *cnt, int lane) {
    constexpr int sft = 1 << B;
    if constexpr (B >= KP) {
#pragma unroll
        for (int c = 0; c < (2 << KP); ++c) cnt[c] += __shfl_xor(cnt[c], sft, 16);
    } else {
        // held: the 2^(B+1) configurations agreeing with the lane above bit
        // B, counts at 2 * (configuration mod 2^(B+1)) + v
        constexpr int half = 2 << B;
        const bool up = (lane >> B) & 1;
#pragma unroll
        for (int c = 0; c < half; ++c) {
            const uint32_t keep = up ? cnt[c + half] : cnt[c];
            const uint32_t send = up ? cnt[c] : cnt[c + half];
            cnt[c] = keep + __shfl_xor(send, sft, 16);
        }
    }
}

// Counts of one family of k parents over words w = lane, lane + LS, ...:
// cell (c << 1) | v, c the parents' values as bits, v the child's value, is
// the popcount of the AND of the matching planes. Of LS = 64 lanes those that
// agree in their low four bits add their counts first; 16 lanes' partial
// counts are then summed and scattered by a butterfly that, at lane bit b,
// halves the configurations a lane keeps by configuration bit b (b < k), or
// sums all it holds (b >= k): lane L < 2^k ends with the two counts of
// configuration L in cnt[0] and cnt[1].
template <int KP, int LS>
__device__ inline void count_cells2(const uint32_t *__restrict__ bits, int W, int lane,
                                    int child, const int *par, uint32_t *cnt) {
    constexpr int NC = 2 << KP;
#pragma unroll
    for (int c = 0; c < NC; ++c) cnt[c] = 0;
    for (int w = lane; w < W; w += LS) {
        uint32_t a[NC];
        a[0] = bits[((size_t)child * 2 + 0) * W + w];
        a[1] = bits[((size_t)child * 2 + 1) * W + w];
#pragma unroll
        for (int j = 0; j < KP; ++j) {
            const uint32_t p0 = bits[((size_t)par[j] * 2 + 0) * W + w];
            const uint32_t p1 = bits[((size_t)par[j] * 2 + 1) * W + w];
            const int half = 2 << j;
#pragma unroll
            for (int c = 0; c < NC / 2; ++c) {
                if (c < half) {
                    a[c + half] = a[c] & p1;
                    a[c] = a[c] & p0;
                }
            }
        }
#pragma unroll
        for (int c = 0; c < NC; ++c) cnt[c] += __popc(a[c]);
    }
    if constexpr (LS == 64) {
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            cnt[c] += __shfl_xor(cnt[c], 32);
            cnt[c] += __shfl_xor(cnt[c], 16);
        }
        lane &= 15;
    }
    count_scatter<KP, 3>(cnt, lane);
    count_scatter<KP, 2>(cnt, lane);
    count_scatter<KP, 1>(cnt, lane);
    count_scatter<KP, 0>(cnt, lane);
}

// Log-gamma tables of the score paths for data whose variables all have
// arity r: for k = 0..4 parents (q = r^k configurations),
// lgt[(2k) * (m+1) + c] = lgamma(a_j + c) and lgt[(2k+1) * (m+1) + c] =
// lgamma(a_jk + c), c = 0..m, with the BDeu (a_j = ess / q, a_jk =
// ess / (q r)) or K2 (a_j = r, a_jk = 1) hyperparameters.
__device__ void lgamma_table(uint32_t x0, uint32_t step, int m, int r, int kind, double ess,
                             double *__restrict__ lgt) {
    const int m1 = m + 1;
    for (int x = (int)x0; x < 10 * m1; x += (int)step) {
        const int row = x / m1, c = x - row * m1, k = row >> 1;
        int qi = 1;
        for (int j = 0; j < k; ++j) qi *= r;
        const double a = (row & 1) ? (kind == 0 ? ess / ((double)qi * r) : 1.0)
                                   : (kind == 0 ? ess / qi : (double)r);
        lgt[x] = lgamma(a + c);
    }
}

// C(p, t) for p <= 32, t <= 5, in registers (the products fit 32 bits)
__device__ inline uint32_t binom5(uint32_t p, int t) {
    const uint32_t c2 = p * (p - 1u) / 2u;
    if (t <= 0) return 1u;
    if (t == 1) return p;
    if (t == 2) return c2;
    if (p < (uint32_t)t) return 0u;
    const uint32_t c3 = c2 * (p - 2u) / 3u;
    if (t == 3) return c3;
    const uint32_t c4 = c3 * (p - 3u) / 4u;
    return t == 4 ? c4 : c4 * (p - 4u) / 5u;
}

// Scores of data whose variables all have arity r, d <= 4: one wave per SET of
// 1 .. d + 1 variables instead of one per family. The families (i, U - i) of a
// set U of k + 1 variables share their table of r^(k+1) counts, and with one
// arity their cell hyperparameters too, so the table and its cells' terms
// lgamma(a_jk + N_jk) - lgamma(a_jk) are taken once for all k + 1 of them (HELD:
// in LDS); each family then sums them row by row, with lgamma(a_j) -
// lgamma(a_j + N_j) of the row, a marginal of the same table (one sum over all
// cells for the whole set cancels only at the end: rounding errors 10% larger).
// The counting (LDS atomics, 4 samples per lane and load) bounds it: at n = 20, r
// = 3, m = 1000, d = 4 the 15,504 + 6,195 sets take 47 us where a wave per family
// (100,720 of them) took 306 us. Sets in order of size, then colex. A value >= r
// (the device entry points do not look at the data) is counted in some other cell
// or in none: the key is tested against the table's size, so it never leaves it.
// TAB: the log-gamma values come from lgamma_table, else each is evaluated in
// place (the same values).
template <bool TAB, bool HELD>
__global__ void __launch_bounds__(kThreads)
k_scores_sets(int n, int m, int d, const uint8_t *__restrict__ data, int r, uint32_t K,
              uint32_t sets, int max_bins, int kind, double ess, const double *__restrict__ lgt,
              double *__restrict__ out) {
    extern __shared__ unsigned char smem[];
    typedef unsigned short us2 __attribute__((ext_vector_type(2)));
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
    uint32_t c = blockIdx.x * 4u + (uint32_t)w;
    if (c >= sets) return;                       // whole waves
    double *cell = reinterpret_cast<double *>(smem) + w * max_bins;       // HELD
    int *hist = reinterpret_cast<int *>(smem + (HELD ? (size_t)32 * max_bins : 0)) + w * max_bins;
    // size and members: the largest p with C(p, t) <= c, found over the lanes
    int k1 = 1;
    while (k1 <= d && c >= binom5((uint32_t)n, k1)) c -= binom5((uint32_t)n, k1++);
    int var[5];
#pragma unroll
    for (int t = 5; t >= 1; --t) {
        var[t - 1] = 0;
        if (t <= k1) {
            const uint32_t b = l < 32 ? binom5((uint32_t)l, t) : ~0u;
            const int p = __popcll(__ballot(b <= c)) - 1;
            c -= binom5((uint32_t)p, t);
            var[t - 1] = __builtin_amdgcn_readfirstlane(p);
        }
    }
    int bins = 1;
    for (int t = 0; t < k1; ++t) bins *= r;
    for (int b = l; b < bins; b += 64) hist[b] = 0;
    __builtin_amdgcn_wave_barrier();
    // cell index: variable t is digit t (stride r^t)
    const us2 rr = {(unsigned short)r, (unsigned short)r};
    const int groups = m >> 2;
    for (int g = l; g < groups; g += 64) {
        us2 ke = {0, 0}, ko = {0, 0};
        uint32_t x[5];
#pragma unroll
        for (int t = 4; t >= 0; --t)
            if (t < k1) __builtin_memcpy(&x[t], data + (size_t)var[t] * m + 4 * (size_t)g, 4);
#pragma unroll
        for (int t = 4; t >= 0; --t) {
            if (t < k1) {
                const uint32_t e = x[t] & 0x00ff00ffu, o = (x[t] >> 8) & 0x00ff00ffu;
                ke = ke * rr + __builtin_bit_cast(us2, e);
                ko = ko * rr + __builtin_bit_cast(us2, o);
            }
        }
        if (ke.x < bins) atomicAdd(&hist[ke.x], 1);
        if (ko.x < bins) atomicAdd(&hist[ko.x], 1);
        if (ke.y < bins) atomicAdd(&hist[ke.y], 1);
        if (ko.y < bins) atomicAdd(&hist[ko.y], 1);
    }
    if (l < (m & 3)) {
        int key = 0;
#pragma unroll
        for (int t = 4; t >= 0; --t)
            if (t < k1) key = key * r + data[(size_t)var[t] * m + 4 * (size_t)groups + l];
        if (key < bins) atomicAdd(&hist[key], 1);
    }
    __builtin_amdgcn_wave_barrier();
    const int m1 = m + 1;
    const int rows = bins / r;                   // q = r^k configurations
    const double *lj = lgt + (size_t)(2 * (k1 - 1)) * m1, *ljk = lj + m1;
    const double a_j = kind == 0 ? ess / rows : (double)r;
    const double a_jk = kind == 0 ? ess / ((double)rows * r) : 1.0;
    auto lg_row = [&](int v) { return TAB ? lj[v] : lgamma(a_j + v); };
    auto lg_cell = [&](int v) { return TAB ? ljk[v] : lgamma(a_jk + v); };
    const double lg_aj = lg_row(0), lg_ajk = lg_cell(0);
    auto term = [&](int v) { return v ? lg_cell(v) - lg_ajk : 0.0; };
    if constexpr (HELD) {
        for (int b = l; b < bins; b += 64) cell[b] = term(hist[b]);
        __builtin_amdgcn_wave_barrier();
    }
    // rows of the family whose child is digit t: cells that agree elsewhere
    double mine = 0.0;                           // lane t: the score of child var[t]
    int stride = 1;
#pragma unroll
    for (int t = 0; t < 5; ++t) {
        if (t < k1) {
            double acc = 0.0;
            const uint32_t inv = (65536u + (uint32_t)stride - 1u) / (uint32_t)stride;
            for (int row = l; row < rows; row += 64) {
                const int hi = (int)(((uint32_t)row * inv) >> 16);    // row / stride, rows < 2048
                const int base = hi * stride * r + (row - hi * stride);
                int nj = 0;
                double sj = 0.0;
                for (int v = 0; v < r; ++v) {
                    const int c = hist[base + v * stride];
                    nj += c;
                    if constexpr (HELD) sj += cell[base + v * stride];
                    else sj += term(c);
                }
                if (nj) acc += sj + lg_aj - lg_row(nj);
            }
            for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o);
            if (l == t) mine = acc;
            stride *= r;
        }
    }
    if (l < k1) {
        // rank of the parent set U - var[l] among node var[l]'s: K(n - 1, k1 - 2)
        // smaller sets, then colex over the compressed positions
        uint32_t rank = 0;
        int i = 0, size = 0;
        for (int t = 0; t < k1 - 1; ++t) rank += binom5((uint32_t)(n - 1), t);
#pragma unroll
        for (int t = 0; t < 5; ++t) {
            if (t < k1 && t == l) i = var[t];
            if (t < k1 && t != l) rank += binom5((uint32_t)(t < l ? var[t] : var[t] - 1), ++size);
        }
        out[(size_t)i * K + rank] = mine;
    }
}

// The k + 1 family scores of a set of k + 1 binary variables from its counts as
// count_cells2 leaves them (lane L < 2^k: the two counts of configuration L of
// variables 0 .. k-1, by the value of variable k). Child k: the row of
// configuration L is the lane's own pair; child j < k: the rows pair the lanes
// that differ in bit j, one row per value of variable k: value 0 taken by the
// lane without the bit, 1 by the other, which trade the terms of their cells.
// Lane t < k + 1 returns the score of child t. Whole rows (whose large terms
// have cancelled) meet in a butterfly over the row index, the child's parents in
// order and the highest first, so that the sums are those of a family alone;
// log-gamma values from the tables.
template <int KP>
__device__ inline double set_scores2(const uint32_t *cnt, int lane, const double *lgt, int m1) {
    constexpr int Q = 1 << KP;
    const double *lj = lgt + (2 * KP) * m1, *ljk = lgt + (2 * KP + 1) * m1;
    const double lg_aj = lj[0], lg_ajk = ljk[0];
    const bool live = lane < Q;
    const uint32_t c0 = live ? cnt[0] : 0u, c1 = live ? cnt[1] : 0u;
    const double l0 = c0 ? ljk[c0] - lg_ajk : 0.0, l1 = c1 ? ljk[c1] - lg_ajk : 0.0;
    double mine = 0.0;
#pragma unroll
    for (int t = 0; t <= KP; ++t) {
        uint32_t nj;
        double sj;
        if (t == KP) {
            nj = c0 + c1;
            sj = l0 + l1;
        } else {
            const bool own = !((lane >> t) & 1);
            nj = (own ? c0 : c1) + __shfl_xor(own ? c1 : c0, 1 << t, 16);
            sj = (own ? l0 : l1) + __shfl_xor(own ? l1 : l0, 1 << t, 16);
        }
        double acc = nj ? sj + lg_aj - lj[nj] : 0.0;
        if (t < KP) acc += __shfl_xor(acc, 1 << t, 16);      // variable k
#pragma unroll
        for (int j = KP - 1; j >= 0; --j)
            if (j != t) acc += __shfl_xor(acc, 1 << j, 16);
        if (lane == t) mine = acc;
    }
    return mine;
}

// Local scores of all-binary data with d <= 4 by sets of variables, as
// k_scores_sets: LS lanes per set (16, or a wave where there are few sets and many
// samples; its four groups of 16 then all have the scores), counts from the bit
// planes of pack2. The k + 1 families of a set share its counts and its cells'
// terms (n = 25, m = 2000, d = 4: 37 us, by families 143; n = 30, d = 3: 15, 48).
template <int LS>
__global__ void __launch_bounds__(kThreads)
k_scores2(int n, int W, int m, int d, uint32_t K, uint32_t sets,
          const uint32_t *__restrict__ bits, const double *__restrict__ lgt,
          double *__restrict__ out) {
    const int lane = threadIdx.x & 15, first = threadIdx.x & (LS - 1);
    uint32_t c = blockIdx.x * (kThreads / LS) + threadIdx.x / LS;
    const bool live = c < sets;
    if (!live) c = 0;                            // dead groups keep the ballots whole
    int k1 = 1;
    while (k1 <= d && c >= binom5((uint32_t)n, k1)) c -= binom5((uint32_t)n, k1++);
    // members, ascending: the largest p with C(p, t) <= c, over the group's lanes
    int var[5];
    const int sh = (threadIdx.x & 48);
#pragma unroll
    for (int t = 5; t >= 1; --t) {
        var[t - 1] = 0;
        const bool in0 = t <= k1 && binom5((uint32_t)lane, t) <= c;
        const bool in1 = t <= k1 && binom5((uint32_t)lane + 16u, t) <= c;
        const uint32_t lo = (uint32_t)(__ballot(in0) >> sh) & 0xffffu;
        const uint32_t hi = (uint32_t)(__ballot(in1) >> sh) & 0xffffu;
        if (t <= k1) {
            const int p = __popc(lo) + __popc(hi) - 1;
            c -= binom5((uint32_t)p, t);
            var[t - 1] = p;
        }
    }
    if (!live) return;
    uint32_t cnt[32];
    double sc = 0.0;
    switch (k1) {
        case 1: count_cells2<0, LS>(bits, W, first, var[0], var, cnt); sc = set_scores2<0>(cnt, lane, lgt, m + 1); break;
        case 2: count_cells2<1, LS>(bits, W, first, var[1], var, cnt); sc = set_scores2<1>(cnt, lane, lgt, m + 1); break;
        case 3: count_cells2<2, LS>(bits, W, first, var[2], var, cnt); sc = set_scores2<2>(cnt, lane, lgt, m + 1); break;
        case 4: count_cells2<3, LS>(bits, W, first, var[3], var, cnt); sc = set_scores2<3>(cnt, lane, lgt, m + 1); break;
        default: count_cells2<4, LS>(bits, W, first, var[4], var, cnt); sc = set_scores2<4>(cnt, lane, lgt, m + 1); break;
    }
    if (first < k1) {
        uint32_t rank = 0;
        int i = 0, size = 0;
        for (int t = 0; t < k1 - 1; ++t) rank += binom5((uint32_t)(n - 1), t);
#pragma unroll
        for (int t = 0; t < 5; ++t) {
            if (t < k1 && t == lane) i = var[t];
            if (t < k1 && t != lane)
                rank += binom5((uint32_t)(t < lane ? var[t] : var[t] - 1), ++size);
        }
        out[(size_t)i * K + rank] = sc;
    }
}

// -------------------------------------------------------------- launchers
// Raise a kernel's dynamic LDS limit to what a workgroup may hold (the
// device's per-block maximum less the kernel's static LDS), once per kernel
// and process: the limit is an upper bound only, the launch size decides the
// allocation, and no launch pays for the call.
template <auto Kernel>
static void allow_big_lds() {
    static const bool once = [] {
        int dev = 0, mx = 0;
        hipFuncAttributes fa{};
        if (hipGetDevice(&dev) == hipSuccess &&
            hipDeviceGetAttribute(&mx, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) ==
                hipSuccess &&
            hipFuncGetAttributes(&fa, (const void *)Kernel) == hipSuccess)
            (void)hipFuncSetAttribute((const void *)Kernel,
                                      hipFuncAttributeMaxDynamicSharedMemorySize,
                                      mx - (int)fa.sharedSizeBytes);
        (void)hipGetLastError();
        return true;
    }();
    (void)once;
}

#define BN_CHECK_LAUNCH() \
    do {                                                   \
        hipError_t e_ = hipGetLastError();                 \
        if (e_ != hipSuccess) return e_;                   \
    } while (0)

hipError_t launch_setup(const Tables &tb, int bL, int W, int bG, int bA, int d, uint32_t N,
                        uint32_t K, const ParamBlock &pb, const SetupArgs &sa, hipStream_t st) {
    static const struct OrdTable {
        LaneOrder o[9];
        OrdTable() {
            for (int d = 0; d <= 8; ++d) o[d] = lane_order_c(d);
        }
    } ord_tables;
    auto blocks = [](uint64_t count) { return (uint32_t)((count + kThreads - 1) / kThreads); };
    // range S: one workgroup per 256 masks of its largest table
    const int wmax = std::max(std::max(bL, W), bG);
    TableGrid g;
    g.s = std::max(1, (1 << wmax) / kThreads);
    g.a = g.s + blocks(1ull << bA);
    g.i = g.a + blocks(1ull << (N - bA));
    g.f = g.i + blocks(K);
    g.h = g.f + blocks(1ull << (N + 1 - bL));
    g.p = g.h + 1;
    const uint64_t planes = (uint64_t)(N + 1) * (((uint64_t)sa.m + 63) / 64) * 64;
    g.b = g.p + (sa.bits ? std::min(blocks(planes), 16384u) : 0);
    g.g = g.b + (sa.table_r > 0 ? std::min(blocks(10ull * (sa.m + 1)), 1024u) : 0);
    hipLaunchKernelGGL(k_setup, dim3(g.g), dim3(kThreads), 0, st, tb,
                       ord_tables.o[std::min(std::max(d, 0), 8)], g, bL, W, bG, bA, d, (int)N, K,
                       pb, sa);
    BN_CHECK_LAUNCH();
    return hipSuccess;
}

uint32_t hord_offset(int nh, int h) {
    uint64_t s = 0, c = 1;
    for (int k = 0; k < h; ++k) {
        s += c;
        c = c * (uint64_t)(nh - k) / (uint64_t)(k + 1);
    }
    return (uint32_t)s;
}

// sum_{k <= t} C(w, k) on the host (0 for t < 0)
static uint32_t host_kcount(int w, int t) {
    uint64_t sum = 0, c = 1;
    for (int k = 0; k <= t && k <= w; ++k) {
        sum += c;
        c = c * (uint64_t)(w - k) / (uint64_t)(k + 1);
    }
    return (uint32_t)sum;
}

hipError_t launch_scores(int n, int m, const uint8_t *data, const uint8_t *arity, uint32_t K,
                         int kind, double ess, const uint32_t *famask, int max_bins,
                         double *out, hipStream_t st, uint32_t *bits, int uniform_r, int d,
                         bool tables, double *lgt) {
    if (bits) {
        // all-binary data, d <= 4: counts from the bit planes
        const int W = (m + 31) / 32;
        const uint32_t sets = host_kcount(n, d + 1) - 1;
        // A wave per set where 16 lanes each would leave CUs without a workgroup and
        // the samples are many enough to pay for the larger sum (m = 10^6, n = 8, d = 4:
        // score phase 327 us with 64 lanes, 1271 with 16, 1176 for a family each; m =
        // 8400, n = 10, d = 3: 26, 32 and 46; at m = 2000 they are equal).
        const bool wide = (sets + 15) / 16 <= 256 && W >= 64;
        const uint32_t per = wide ? 4 : 16;
        auto go = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, dim3((sets + per - 1) / per), dim3(kThreads), 0, st, n, W, m,
                               d, K, sets, (const uint32_t *)bits, (const double *)lgt, out);
        };
        if (wide) go(k_scores2<64>);
        else go(k_scores2<16>);
        BN_CHECK_LAUNCH();
        return hipSuccess;
    }
    if (max_bins <= kScoreWaveBins && uniform_r > 0) {
        // sets of 1 .. d + 1 variables
        const uint32_t sets = host_kcount(n, d + 1) - 1;
        const dim3 grid((sets + 3) / 4);
        // The cells' terms stay in LDS while that leaves five workgroups per CU
        // (640 cells: n = 20, m = 1000, d = 4 with three states 75 us for the score
        // phase, 81 with the terms taken from the tables again for each family), or
        // where there is at most one per CU (n = 10, six states, d = 3: 31 against
        // 36 us); above, fewer workgroups cost more than the loads (four states, d =
        // 4: 138 against 106 us).
        const bool held = max_bins <= 640 || grid.x <= 256;
        const size_t sm = (size_t)4 * max_bins * (sizeof(int) + (held ? sizeof(double) : 0));
        auto go = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, grid, dim3(kThreads), sm, st, n, m, d, data, uniform_r, K,
                               sets, max_bins, kind, ess, (const double *)lgt, out);
        };
        allow_big_lds<k_scores_sets<true, true>>();
        allow_big_lds<k_scores_sets<false, true>>();
        if (tables) held ? go(k_scores_sets<true, true>) : go(k_scores_sets<true, false>);
        else held ? go(k_scores_sets<false, true>) : go(k_scores_sets<false, false>);
    } else if (max_bins <= kScoreWaveBins) {
        hipLaunchKernelGGL(k_scores_w, dim3((unsigned)((n * (uint64_t)K + 3) / 4)), dim3(kThreads),
                           (size_t)4 * max_bins * sizeof(int), st, n, m, data, arity, K, kind, ess,
                           famask, max_bins, out);
    } else
        hipLaunchKernelGGL(k_scores, dim3((unsigned)(n * K)), dim3(kThreads),
                           (size_t)max_bins * sizeof(int), st, n, m, data, arity, K, kind, ess,
                           famask, out);
    BN_CHECK_LAUNCH();
    return hipSuccess;
}

template <class P>
static hipError_t launch_gamma_edges(const LatticeArgs &a, const typename P::Store &L,
                                     const typename P::Store &R, hipStream_t st,
                                     PhaseEvents *ev);
static hipError_t launch_lattice_fused(const LatticeArgs &a, const PolX32::Store &L,
                                       const PolX32::Store &R, hipStream_t st,
                                       PhaseEvents *ev);

// Fork of a second stream off the solve's stream and its join: two events
// (no timing), destroyed when the helper goes out of scope (HIP releases an
// event recorded and waited on only after the waits are satisfied).
struct SweepFork {
    hipEvent_t e0 = nullptr, e1 = nullptr;
    hipError_t open(hipStream_t st, hipStream_t side) {
        hipError_t e = hipEventCreateWithFlags(&e0, hipEventDisableTiming);
        if (e == hipSuccess) e = hipEventCreateWithFlags(&e1, hipEventDisableTiming);
        if (e == hipSuccess) e = hipEventRecord(e0, st);
        if (e == hipSuccess) e = hipStreamWaitEvent(side, e0, 0);
        return e;
    }
    hipError_t join(hipStream_t st, hipStream_t side) {
        hipError_t e = hipEventRecord(e1, side);
        if (e == hipSuccess) e = hipStreamWaitEvent(st, e1, 0);
        return e;
    }
    ~SweepFork() {
        if (e0) (void)hipEventDestroy(e0);
        if (e1) (void)hipEventDestroy(e1);
    }
};

template <class P>
hipError_t launch_lattice(const LatticeArgs &a, const typename P::Store &alpha,
                          const typename P::Store &L, const typename P::Store &R,
                          hipStream_t st, PhaseEvents *ev) {
    using V = typename P::V;
    const int n = a.n, N = n - 1, d = a.d;
    const Tables &tb = a.tb;
    V *beta = reinterpret_cast<V *>(a.beta);
    V *qt = reinterpret_cast<V *>(a.qt);
    V *Y1 = reinterpret_cast<V *>(a.Y1);
    V *Y2 = reinterpret_cast<V *>(a.Y2);
    V *gam = reinterpret_cast<V *>(a.gam);
    V *part = reinterpret_cast<V *>(a.part);
    V *layer = reinterpret_cast<V *>(a.layer);
    auto rec = [&](int idx) {
        if (ev && ev->ev[idx]) (void)hipEventRecord(ev->ev[idx], st);
    };
    const bool lin = a.fused || (a.bA == 13 ? a.lin_mode && a.Zs : a.lin_mode == 1);
    hipLaunchKernelGGL(k_prep<P>, dim3(n, (a.K + kPrepChunk - 1) / kPrepChunk), dim3(kThreads),
                       0, st, n, d, a.K,
                       (const uint32_t *)tb.binom, (const double *)a.logp,
                       (const double *)a.log_rho, (const double *)a.log_q, a.gauge, beta, qt,
                       a.gauge_exp, a.fbA, a.fbG, a.rtG, lin ? a.betal : nullptr,
                       (typename P::Anchor *)a.anc, a.linok, a.fused ? a.emax : nullptr);
    BN_CHECK_LAUNCH();
    rec(1);
    if constexpr (std::is_same<P, PolX32>::value) {
        if (a.fused) return launch_lattice_fused(a, L, R, st, ev);
    }
    if (a.bA == 13) {
        const uint32_t nit = (uint32_t)a.nitA;
        // the partial-rank table is used when ranks fit 16 bits and it fits 12 KB
        const int use_prk = (a.K < 65536u && (size_t)(d + 1) * nit * 2 <= 12288) ? 1 : 0;
        const size_t sm = sizeof(V) * (8192 + 256) + 33 * 33 * 4 +
                          (use_prk ? (size_t)(d + 1) * nit * 2 : 0);
        const unsigned nblkA = (unsigned)(n << (N - 13));
        if (a.lin_mode && a.Zs) {
            using A = typename P::Anchor;
            // block-wise seeds: 2^bS tiles per workgroup, 4 <= bS <= 8, with at
            // least 4 high bits left so that the grid holds n * 16 workgroups
            const int hA = N - 13, bS = hA - 4 < 8 ? hA - 4 : 8;
            const uint32_t nhiMax = bS >= 4 ? host_kcount(hA - bS, d) : 0u;
            if (a.KS > 0 && bS >= 4 && d <= 7 && (size_t)(d + 1) * nhiMax <= 4096) {
                const size_t smB = 8 * (4096 + 256) + 33 * 33 * 4 + (size_t)(d + 1) * nhiMax * 4;
                // few blocks of tiles (n < 26): their chunks of seed ranks
                // spread over more workgroups
                const unsigned nbS = (unsigned)(n << (hA - bS));
                const unsigned ySplit = std::min((a.KS + 15) / 16, std::max(1u, 2048u / nbS));
                hipLaunchKernelGGL(HIP_KERNEL_NAME(k_alpha_seeds_blk<P>),
                                   dim3(nbS, ySplit), dim3(kThreads), smB, st, n,
                                   d, a.K, a.KS, bS, nhiMax, tb, (const double *)a.betal,
                                   (const int *)a.linok, a.Zs);
            } else if (a.KS > 0) {
                const size_t smS = 33 * 33 * 4 + (use_prk ? (size_t)(d + 1) * nit * 2 + nit : 0);
                hipLaunchKernelGGL(HIP_KERNEL_NAME(k_alpha_seeds<P>), dim3(nblkA), dim3(kThreads),
                                   smS, st, n, d, a.K, a.KS, use_prk, tb, (const double *)a.betal,
                                   (const int *)a.linok, a.Zs);
            }
            BN_CHECK_LAUNCH();
            const size_t smL = alpha_lin_lds(d, a.KS);
            allow_big_lds<k_alpha_lin<P>>();
            rec(8);
            // 2^tl tiles per workgroup share its set-up (tables and size-d
            // seeds in LDS)
            // (tl < hA keeps the shift count nonnegative: at n = 14 there
            // is a single tile per node and tl stays 0)
            if (n < 20) {
                allow_big_lds<k_alpha_lin_few<P>>();
                hipLaunchKernelGGL(HIP_KERNEL_NAME(k_alpha_lin_few<P>), dim3(nblkA),
                                   dim3(kThreads), std::max(sm, smL), st, n, d, a.KS,
                                   a.lin_mode == 2 ? 1 : 0, (const double *)a.Zs,
                                   (const double *)a.betal, a.K, host_kcount(N, d - 1),
                                   (const A *)a.anc, (const int *)a.linok, (const V *)qt, alpha,
                                   a.cnt, a.fbA, use_prk, tb, (const V *)beta);
                BN_CHECK_LAUNCH();
                rec(9);
            } else {
                int tl = 0;
                // as many as leave the grid two full rounds of the 1024
                // workgroups that run together, or four where there are many
                // tiles (n >= 24): at n = 22 and 23 1024, 2048 and 4096
                // workgroups at least take 84, 77 and 89, and 151, 143 and 151
                // us, at n = 25 639, 595 and 587 (8192: 621)
                const unsigned least = nblkA < 16384u ? 2048u : 4096u;
                while (tl < 6 && tl < hA && ((uint64_t)n << (hA - tl - 1)) >= least) ++tl;
                hipLaunchKernelGGL(HIP_KERNEL_NAME(k_alpha_lin<P>), dim3(nblkA >> tl), dim3(kThreads), smL,
                                   st, n, d, a.KS, a.lin_mode == 2 ? 1 : 0, tl, (const double *)a.Zs,
                                   (const double *)a.betal, a.K,
                                   host_kcount(N, d - 1), (const A *)a.anc, (const int *)a.linok, (const V *)qt, alpha,
                                   a.cnt, a.fbA);
                BN_CHECK_LAUNCH();
                rec(9);
                // tiles the linear form could not hold: a grid that walks the list
                allow_big_lds<k_alpha_fb<P>>();
                hipLaunchKernelGGL(HIP_KERNEL_NAME(k_alpha_fb<P>), dim3(std::min(nblkA, 1024u)),
                                   dim3(kThreads), sm, st, n, d, a.K, use_prk, tb, (const V *)beta,
                                   (const V *)qt, alpha, a.cnt, (const uint32_t *)a.fbA);
            }
        } else {
            allow_big_lds<k_alpha<P>>();
            rec(8);
            hipLaunchKernelGGL(HIP_KERNEL_NAME(k_alpha<P>), dim3(nblkA), dim3(kThreads), sm, st,
                               n, d, a.K, use_prk, tb, (const V *)beta, (const V *)qt, alpha,
                               a.cnt);
            BN_CHECK_LAUNCH();
            rec(9);
        }
    } else {
        rec(8);
        hipLaunchKernelGGL(HIP_KERNEL_NAME(k_alpha_small<P>), dim3((unsigned)n), dim3(kThreads),
                           sizeof(V) * (4096 + 256), st, n, d, a.K, lin ? 1 : 0, tb,
                           (const V *)beta, (const double *)a.betal,
                           (const typename P::Anchor *)a.anc, (const int *)a.linok,
                           (const V *)qt, alpha, a.cnt);
        BN_CHECK_LAUNCH();
        rec(9);
    }
    BN_CHECK_LAUNCH();
    rec(2);
    const int nh = n - a.bL;
    const size_t smL = align16(SliceLds<P>::bytes_per_entry * ((size_t)a.bL << (a.bL - 1))) +
                       (sizeof(V) + 2) * ((size_t)1 << a.bL);
    // The backward sweep needs alpha but not L. Below n = 24 step h of both
    // sweeps is one launch; from there on, with a.side set, the backward sweep
    // runs on that stream, forked after alpha and joined before Gamma, so that
    // the tail of a layer is filled by the other sweep (n = 25 FP32-scaled: 1.16
    // ms for both against 1.24 ms in joint launches; FP64 2.26 and 2.27).
    SweepFork fork;
    const bool forked = a.side && !a.fwd_only;
    if (forked) {
        const hipError_t e = fork.open(st, a.side);
        if (e != hipSuccess) return e;
    }
    // a thread per four tile entries covers the cross terms and the largest
    // in-tile layer (C(12, 6) = 924)
    auto sweeps = [&](auto threads, auto bits) -> hipError_t {
        constexpr int TH = decltype(threads)::value, BL = decltype(bits)::value;
        allow_big_lds<k_sweeps<P, TH, BL>>();
        for (int h = 0; h <= nh; ++h) {
            // workgroups below nb run forward tiles, the others backward ones
            const unsigned nb = a.tiles_per_layer[h];
            hipLaunchKernelGGL(HIP_KERNEL_NAME(k_sweeps<P, TH, BL>),
                               dim3(a.fwd_only || forked ? nb : 2 * nb), dim3(TH), smL, st, n,
                               a.bL, nb, hord_offset(nh, h), hord_offset(nh, nh - h), tb, alpha,
                               L, R, a.cnt);
            BN_CHECK_LAUNCH();
        }
        for (int h = nh; forked && h >= 0; --h) {
            hipLaunchKernelGGL(HIP_KERNEL_NAME(k_sweeps<P, TH, BL>), dim3(a.tiles_per_layer[h]),
                               dim3(TH), smL, a.side, n, a.bL, 0u, 0u, hord_offset(nh, h), tb,
                               alpha, L, R, a.cnt);
            BN_CHECK_LAUNCH();
        }
        return hipSuccess;
    };
    // BL > 0: the tile widths that the plan chooses from n = 9 on, with unrolled
    // in-tile layers; 0: any other (the smallest lattices, tests)
    using std::integral_constant;
    hipError_t es;
    if (a.bL == 9) es = sweeps(integral_constant<int, 256>{}, integral_constant<int, 9>{});
    else if (a.bL == 10) es = sweeps(integral_constant<int, 256>{}, integral_constant<int, 10>{});
    else if (a.bL == 11) es = sweeps(integral_constant<int, 512>{}, integral_constant<int, 11>{});
    else if (a.bL == 12) {
        if constexpr (std::is_same<P, PolX32>::value)
            es = sweeps(integral_constant<int, 1024>{}, integral_constant<int, 12>{});
        else es = hipErrorInvalidValue;      // the log form's plan ends at 11 bits
    } else es = sweeps(integral_constant<int, 256>{}, integral_constant<int, 0>{});
    if (es != hipSuccess) return es;
    rec(3);
    if (a.fwd_only) {
        hipLaunchKernelGGL(k_log_LV<P>, dim3(1), dim3(64), 0, st, n, L,
                           (const double *)a.gauge_exp, (const unsigned long long *)a.cnt,
                           (const uint32_t *)a.fbA, a.diag);
        BN_CHECK_LAUNCH();
        rec(6);
        return hipSuccess;
    }
    if (forked) {
        const hipError_t e = fork.join(st, a.side);
        if (e != hipSuccess) return e;
    }
    rec(4);
    return launch_gamma_edges<P>(a, L, R, st, ev);
}

// Gamma (Eq. 12), edges (Eq. 11) and the invariants, after both sweeps.
template <class P>
static hipError_t launch_gamma_edges(const LatticeArgs &a, const typename P::Store &L,
                                     const typename P::Store &R, hipStream_t st,
                                     PhaseEvents *ev) {
    using V = typename P::V;
    const int n = a.n, d = a.d;
    const int nh = n - a.bL;
    const Tables &tb = a.tb;
    V *beta = reinterpret_cast<V *>(a.beta);
    V *qt = reinterpret_cast<V *>(a.qt);
    V *Y1 = reinterpret_cast<V *>(a.Y1);
    V *Y2 = reinterpret_cast<V *>(a.Y2);
    V *gam = reinterpret_cast<V *>(a.gam);
    V *part = reinterpret_cast<V *>(a.part);
    V *layer = reinterpret_cast<V *>(a.layer);
    auto rec = [&](int idx) {
        if (ev && ev->ev[idx]) (void)hipEventRecord(ev->ev[idx], st);
    };
    {
        const GammaGeom &gg = a.gg;
        // n = 12: no high bits, so Y1_v is Gamma_v rank by rank (y1off[v] = v K)
        if (n == 12) Y1 = gam;
        if (a.bG == 12) {
            const size_t sm = sizeof(V) * (4096 + 256) + 33 * 33 * 4 + (size_t)gg.KT * 4;
            const unsigned nblkG = 1u << (n - 12);
            allow_big_lds<k_gamma_tile<P>>();
            if (a.lin_mode) {
                // few tiles: their endpoints are split over several
                // workgroups, so that about 512 run (a larger target, 1536,
                // made n = 22 slower: the split form spills more registers
                // and repeats the tile's set-up)
                const unsigned vsplit =
                    std::min((unsigned)n, std::max(1u, (512u + nblkG - 1) / nblkG));
                if (vsplit > 1) {
                    allow_big_lds<k_gamma_tile_lin<P, true>>();
                    hipLaunchKernelGGL(HIP_KERNEL_NAME(k_gamma_tile_lin<P, true>),
                                       dim3(nblkG * vsplit), dim3(kThreads), sm, st, n, d,
                                       a.lin_mode == 2 ? 1 : 0, (int)vsplit, gg, tb, L, R,
                                       (const V *)qt, Y1, part, a.fbG, a.rtG);
                } else {
                    allow_big_lds<k_gamma_tile_lin<P, false>>();
                    hipLaunchKernelGGL(HIP_KERNEL_NAME(k_gamma_tile_lin<P, false>), dim3(nblkG),
                                       dim3(kThreads), sm, st, n, d, a.lin_mode == 2 ? 1 : 0, 1,
                                       gg, tb, L, R, (const V *)qt, Y1, part, a.fbG, a.rtG);
                }
                BN_CHECK_LAUNCH();
                rec(7);
                allow_big_lds<k_gamma_tile_retry<P>>();
                hipLaunchKernelGGL(HIP_KERNEL_NAME(k_gamma_tile_retry<P>),
                                   dim3(std::min(nblkG, 1024u)), dim3(kThreads), sm, st, n, d, gg,
                                   tb, L, R, (const V *)qt, Y1, part, (const uint32_t *)a.rtG,
                                   a.fbG);
                if (a.lin_mode == 2) {   // every tile was sent there
                    BN_CHECK_LAUNCH();
                    allow_big_lds<k_gamma_tile_fb<P>>();
                    hipLaunchKernelGGL(HIP_KERNEL_NAME(k_gamma_tile_fb<P>),
                                       dim3(std::min(nblkG, 1024u)), dim3(kThreads), sm, st, n, d,
                                       gg, tb, L, R, (const V *)qt, Y1, part,
                                       (const uint32_t *)a.fbG, nblkG);
                }
            } else {
                hipLaunchKernelGGL(HIP_KERNEL_NAME(k_gamma_tile<P>), dim3(nblkG), dim3(kThreads),
                                   sm, st, n, d, gg, tb, L, R, (const V *)qt, Y1, part);
            }
        } else {
            hipLaunchKernelGGL(k_gamma_small<P>, dim3((unsigned)n), dim3(kThreads),
                               sizeof(V) * (4096 + 256), st, n, a.K, a.lin_mode == 1 ? 0 : 1, tb,
                               L, R, (const V *)qt, gam);
        }
        BN_CHECK_LAUNCH();
        if (!(a.bG == 12 && a.lin_mode)) rec(7);
        // up to n = 12 no endpoint has bits above the tile: the tile kernels wrote
        // Gamma itself
        if (n > 12 && gg.blk1[n] > 0) {
            // every one-level endpoint with 12 high bits (n = 25): the four ranks
            // of a group per workgroup
            bool all12 = std::is_same<P, PolX32>::value;
            for (int v = 0; v < n && all12; ++v)
                if (gg.blk1[v + 1] > gg.blk1[v]) all12 = gg.hv[v] == 12;
            if constexpr (std::is_same<P, PolX32>::value) {
                if (all12)
                    hipLaunchKernelGGL(k_gamma_high1_12, dim3(gg.blk1x4[n]), dim3(kThreads),
                                       sizeof(V) * (4096 + 256), st, n, d, a.K, gg, tb,
                                       (const V *)Y1, gam);
            }
            if (!all12) {
                allow_big_lds<k_gamma_high1<P>>();
                hipLaunchKernelGGL(k_gamma_high1<P>, dim3(gg.blk1[n]), dim3(kThreads),
                                   sizeof(V) * (4096 + 256) + (33 * 33 + 34) * 4 +
                                       ((size_t)8 << (12 - gg.hmin1)),
                                   st, n, d,
                                   a.K, a.lin_mode == 1 ? 0 : 1, gg, tb, (const V *)Y1, gam);
            }
            BN_CHECK_LAUNCH();
        }
        if (gg.blkA[n] > 0) {
            // dense 12-bit form for the FP32-scaled system; the log form keeps the
            // truncated pass (its log-adds are costly enough that the skipped
            // entries matter more than the indexing)
            bool dense = false;
            if constexpr (std::is_same<P, PolX32>::value) {
                if (a.aG == 12) {
                    dense = true;
                    hipLaunchKernelGGL(k_gamma_highA12, dim3(gg.blkAx4[n]), dim3(kThreads),
                                       sizeof(V) * (4096 + 256), st, n, a.KA, gg, tb,
                                       (const V *)Y1, Y2);
                }
            }
            if constexpr (std::is_same<P, PolLog>::value) {
                // plain doubles under a scale, as the linear tiles (off with them)
                if (a.aG == 12 && a.lin_mode != 0) {
                    dense = true;
                    hipLaunchKernelGGL(k_gamma_highA12_log, dim3(gg.blkA[n]), dim3(kThreads),
                                       sizeof(double) * (4096 + 256), st, n, d, a.KA,
                                       a.lin_mode == 2 ? 1 : 0, gg, tb, (const double *)Y1,
                                       (double *)Y2);
                }
            }
            if (!dense)
                hipLaunchKernelGGL(k_gamma_highA<P>, dim3(gg.blkA[n]), dim3(kThreads),
                                   sizeof(V) << a.aG, st, n, d, a.aG, a.KA, gg, tb,
                                   (const V *)Y1, Y2);
            BN_CHECK_LAUNCH();
            hipLaunchKernelGGL(k_gamma_highB<P>, dim3(gg.blkB[n]), dim3(kThreads), 0, st, n, d,
                               a.aG, a.KA, a.K, gg, tb, (const V *)Y2, gam);
            BN_CHECK_LAUNCH();
        }
    }
    rec(5);
    // layer sums of L(S) Rp(S): partials per tile come from the Gamma tile
    // kernel (12-bit tiles), else they are taken per sweep tile
    const int tiled = inv_chunks(n);
    const unsigned ninv = tiled ? (unsigned)((n + 1) * tiled) : (unsigned)(a.bL + 1) << nh;
    hipLaunchKernelGGL(k_finish<P>, dim3((unsigned)(n * (n + 1)) + ninv), dim3(kThreads), 0, st, n,
                       a.K, tiled, tiled ? 12 : a.bL, tb, (const uint32_t *)tb.famask,
                       (const V *)beta, (const V *)gam, L, R, part, layer, a.post, a.resid, a.ps,
                       (const double *)a.gauge_exp, (const unsigned long long *)a.cnt,
                       (const uint32_t *)a.fbA, (const uint32_t *)a.fbG,
                       a.done, a.diag);
    BN_CHECK_LAUNCH();
    rec(6);
    return hipSuccess;
}

// The FP32-scaled lattice with alpha never materialised: per-node linear
// scales and bounds, the 9-bit block seeds (timer entries 8 and 9 bracket
// them), then the fused sweeps, one launch per layer.
static hipError_t launch_lattice_fused(const LatticeArgs &a, const PolX32::Store &L,
                                       const PolX32::Store &R, hipStream_t st,
                                       PhaseEvents *ev) {
    const int n = a.n;
    auto rec = [&](int idx) {
        if (ev && ev->ev[idx]) (void)hipEventRecord(ev->ev[idx], st);
    };
    FusedArgs f{};
    f.n = n;
    f.d = a.d;
    f.K = a.K;
    f.KS = a.KS9;
    f.offd = host_kcount(n - 1, a.d - 1);
    f.force_slow = a.lin_mode == 2 ? 1 : 0;
    f.zw = a.zw9;
    f.flin = a.flin;
    f.beta = reinterpret_cast<const X32 *>(a.beta);
    f.qt = reinterpret_cast<const X32 *>(a.qt);
    f.betal = a.betal;
    f.anc = reinterpret_cast<const int *>(a.anc);
    f.linok = a.linok;
    f.emax = a.emax;
    f.nslow = a.fbA;
    f.glo = a.glo;
    f.binom = a.tb.binom;
    f.lorder = a.tb.lorder;
    f.loff = a.tb.loff;
    f.hord = a.tb.hord;
    f.cnt = a.cnt;
    rec(8);
    // the alpha tiles' seeds by blocks of 13-bit tiles (doubles, linear-scale
    // nodes), when the grouped kernel applies; the 9-bit seeds come from them
    const double *zs13 = nullptr;
    if (a.Zs && a.KS > 0 && a.lin_mode != 2) {
        const int N = n - 1, d = a.d, hA = N - 13, bS = hA - 4 < 8 ? hA - 4 : 8;
        const uint32_t nhiMax = bS >= 4 ? host_kcount(hA - bS, d) : 0u;
        if (bS >= 4 && d <= 7 && (size_t)(d + 1) * nhiMax <= 4096) {
            const size_t smB = 8 * (4096 + 256) + 33 * 33 * 4 + (size_t)(d + 1) * nhiMax * 4;
            hipLaunchKernelGGL(HIP_KERNEL_NAME(k_alpha_seeds_blk<PolX32>),
                               dim3((unsigned)(n << (hA - bS))), dim3(kThreads), smB, st, n, d,
                               a.K, a.KS, bS, nhiMax, a.tb, (const double *)a.betal,
                               (const int *)a.linok, a.Zs);
            BN_CHECK_LAUNCH();
            zs13 = a.Zs;
        }
    }
    {
        const hipError_t e = launch_fused_seeds(f, zs13, a.KS, st);
        if (e != hipSuccess) return e;
    }
    rec(9);
    rec(2);
    const int nh = n - 9;
    for (int h = 0; h <= nh; ++h) {
        const hipError_t e = launch_fused_sweep(f, true, h, a.tiles_per_layer[h], L, st);
        if (e != hipSuccess) return e;
    }
    rec(3);
    if (a.fwd_only) {
        hipLaunchKernelGGL(k_log_LV<PolX32>, dim3(1), dim3(64), 0, st, n, L,
                           (const double *)a.gauge_exp, (const unsigned long long *)a.cnt,
                           (const uint32_t *)a.fbA, a.diag);
        BN_CHECK_LAUNCH();
        rec(6);
        return hipSuccess;
    }
    for (int h = nh; h >= 0; --h) {
        const hipError_t e = launch_fused_sweep(f, false, h, a.tiles_per_layer[h], R, st);
        if (e != hipSuccess) return e;
    }
    rec(4);
    return launch_gamma_edges<PolX32>(a, L, R, st, ev);
}

template hipError_t launch_lattice<PolLog>(const LatticeArgs &, const PolLog::Store &,
                                           const PolLog::Store &, const PolLog::Store &,
                                           hipStream_t, PhaseEvents *);
template hipError_t launch_lattice<PolX32>(const LatticeArgs &, const PolX32::Store &,
                                           const PolX32::Store &, const PolX32::Store &,
                                           hipStream_t, PhaseEvents *);

}  // namespace bnk
