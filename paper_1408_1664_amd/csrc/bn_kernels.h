// Declarations shared by the kernel file and the host solver.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "bn_device.h"

namespace bnk {

// Device tables generated by k_setup inside the workspace.
struct Tables {
    uint32_t *binom;     // 33 x 33 binomial coefficients
    uint16_t *lorder;    // 2^bL tile masks, by popcount then value
    uint32_t *loff;      // bL + 2 layer offsets into lorder
    uint16_t *pat;       // masks over W bits with <= d ones, numeric order
    uint32_t *seedmask;  // K(bG, d) Gamma-tile seed masks, by size then colex
    uint32_t *famask;    // K(n-1, d) compressed parent-set masks in rank order
    uint32_t *seedA;     // K(bA, d) alpha-tile seed masks, by size then colex
    uint32_t *items;     // K(n-1-bA, d) masks over the alpha tile's high bits,
                         // by size then colex
    uint8_t *ordC;       // 256 lanes of the Gamma tile's layout C (lane_order_c)
    uint32_t *hord;      // 2^(n-bL) masks over the sweep tiles' high bits, by
                         // popcount then colex: tile t of layer h has the high
                         // part hord[sum_{k<h} C(n-bL, k) + t]
};

// Per-endpoint geometry of the Gamma reduction. Endpoint v's lattice has
// n-1 bits; its tile holds bv = bT-1 (v a tile bit) or bT (v above the tile)
// low bits and hv = n-1-bv high bits. Y1_v holds K(bv,d) x 2^hv values.
struct GammaGeom {
    int bv[32], hv[32];
    uint64_t y1off[32], y2off[32];
    uint32_t blk1[33], blkA[33], blkB[33];  // prefix sums of per-v block counts
    uint32_t kg4[32];  // K(bv, d) rounded down to a multiple of 4: Y1_v's grouped ranks
    // prefix sums of per-v block counts of the dense 12-bit passes, which take
    // the four ranks of a group per workgroup (then one rank of the rest)
    uint32_t blk1x4[33], blkAx4[33];
    uint32_t KT;      // K(bT, d): ranked seed masks over the tile bits
    uint32_t kg[32];  // K(bv, d): ranks of Y1_v
    int hmin1;        // smallest hv among one-level endpoints
};

struct LatticeArgs {
    int n, d;
    uint32_t K;          // parent sets per node
    int bA, bL, bG, aG;  // tile bits: alpha, sweeps, Gamma tile, Gamma level A
    uint32_t KG, KA;     // K(bG, d), K(aG, d)
    uint32_t nitA;       // K(n-1-bA, d): high-bit items of an alpha tile
    int gauge;           // 1: per-node / per-layer power-of-two gauges
    Tables tb;
    const double *logp, *log_rho, *log_q;
    void *beta, *qt, *Y1, *Y2, *gam, *part, *layer;
    double *gauge_exp;   // 2n exponents (E_i, then F_k)
    double *post, *resid, *diag;
    unsigned long long *cnt;
    uint32_t *done;      // workgroup counters of k_finish, zero before a solve
    const uint32_t *tiles_per_layer;  // host array: C(n - bL, h)
    GammaGeom gg;
    // Linear tiles (k_alpha_lin, k_gamma_tile_lin) with fallback lists
    // ([0] = count, then tile ids) for the tiles recomputed by k_alpha /
    // k_gamma_tile. lin_mode: 0 off, 1 on, 2 on with every tile sent to
    // the fallback (tests).
    int lin_mode;
    uint32_t *fbA, *fbG;
    uint32_t *rtG;       // Gamma endpoints for a second scale ([0] = count, then H * 32 + v)
    double *betal;       // n x K: B_i under its node's linear scale
    void *anc;           // n per-node scales (the number system's Anchor type)
    int *linok;          // n flags: node held in plain doubles
    double *Zs;          // alpha-tile seeds in doubles (null: no linear alpha tiles)
    double *ps;          // n x K parent-set posteriors, or null
    uint32_t KS;         // K(13, d - 1): seeds per alpha tile (sizes below d)
    int fwd_only;        // 1: stop after the forward sweep, diag[0] = log L(V)
    hipStream_t side;    // non-null: the backward sweep runs on this stream, forked
                         // after alpha and joined before Gamma
    // alpha never materialised (FP32-scaled form, 9-bit sweep tiles): the
    // sweeps rebuild alpha from the seeds of 9-bit blocks
    int fused;
    uint32_t KS9;        // K(9, d - 1): stored seeds per block
    void *zw9;           // seeds, 8 bytes each
    int *emax;           // per node: floor(log2 max_G B_i(G)) + 1
    int *flin;           // per node: held in plain doubles by the fused sweeps
    uint32_t *glo;       // 512 entries: where a block entry's seed sits (fused sweeps)
};

// The fused sweeps of the FP32-scaled form (alpha never materialised;
// bn_fused.hip).
struct FusedArgs {
    int n, d;
    uint32_t K;            // parent sets per node
    uint32_t KS;           // stored seeds per 9-bit block, K(9, d - 1)
    uint32_t offd;         // K(n - 1, d - 1): rank of the first size-d parent set
    int force_slow;        // every seed and block in the number system (tests)
    void *zw;              // seeds [node][block][rank], 8 bytes: a double under the
                           // node's fused scale (flin) or an X32
    int *flin;             // per-node flags: the node runs in plain doubles
    const X32 *beta;       // n x K gauged scores
    const X32 *qt;         // q(k), gauged
    const double *betal;   // scores under each node's linear scale (linok nodes)
    const int *anc;        // per-node linear scales (multiples of 64)
    const int *linok;      // per-node flags: held in plain doubles
    const int *emax;       // per node: floor(log2 max_G B_i(G)) + 1
    uint32_t *nslow;       // blocks run in the number system (fallback count)
    uint32_t *glo;         // 512 entries: a block entry's slot among its block's seeds
    const uint32_t *binom;
    const uint16_t *lorder;
    const uint32_t *loff;
    const uint32_t *hord;  // sweep tiles' high parts (Tables::hord)
    unsigned long long *cnt;
};
// Node flags and the 9-bit block seeds; zs13 (KS13 doubles per 13-bit tile,
// the alpha tiles' seeds) or null.
hipError_t launch_fused_seeds(const FusedArgs &f, const double *zs13, uint32_t KS13,
                              hipStream_t st);
hipError_t launch_fused_sweep(const FusedArgs &f, bool forward, int h, unsigned tiles,
                              PolX32::Store X, hipStream_t st);
size_t fused_sweep_lds(int d);

// Optional events recorded between phases: [0] start, [1] after scores and
// prior/gauges, [2] after alpha, [3] after the forward sweep, [4] after the
// backward sweep, [5] after Gamma, [6] after edges and diagnostics, [7] after
// the Gamma in-tile kernel alone, [8] and [9] around the alpha tile kernel.
// Null entries are skipped.
struct PhaseEvents {
    hipEvent_t ev[10];
};

// Parameters passed by value to the set-up kernel (host arrays are consumed at
// launch, so no caller pointer is kept).
struct ParamBlock {
    uint8_t arity[32];
    double log_rho[33];
    double log_q[32];
    int has_rho, has_q;
};
// What the set-up kernel prepares besides the tables: the parameters in the
// workspace, zeroed counters (cnt: 2, done: 17 of a cache line each), and for the scores the bit planes of binary
// data (bits, or null) and the log-gamma tables of arity table_r (0: none).
struct SetupArgs {
    uint8_t *arity;
    double *log_rho, *log_q;
    unsigned long long *cnt;
    uint32_t *done;
    const uint8_t *data;
    int m, kind, table_r;
    double ess;
    uint32_t *bits;
    double *lgt;
};
// Ranges of Gamma tiles that the layer sums of L(S) Rp(S) are taken over: at
// most 32, about 256 tiles each; 0 where the sweep tiles serve (n < 12).
inline int inv_chunks(int n) {
    return n < 12 ? 0 : n < 20 ? 1 : n < 25 ? 1 << (n - 20) : 32;
}
hipError_t launch_setup(const Tables &tb, int bL, int W, int bG, int bA, int d, uint32_t N,
                        uint32_t K, const ParamBlock &pb, const SetupArgs &sa, hipStream_t st);
// sum_{k < h} C(nh, k): the first entry of layer h in Tables::hord
uint32_t hord_offset(int nh, int h);
// logp[x] += log_f[x], x < count (scores times a modular feature's factors)
hipError_t launch_add_log(double *logp, const double *log_f, size_t count, hipStream_t st);
// Local scores of every family (Eq. 3). bits non-null: all-binary data with
// d <= 4, counted from the bit planes there; uniform_r > 0: every variable
// has arity uniform_r and d <= 4, so all families of a set of variables are
// scored together, with log-gamma values from tables (`tables`) or evaluated
// in place; lgt: the tables, 10 (m + 1) doubles.
// Planes and tables are those of launch_setup.
constexpr int kScoreWaveBins = 2048;   // cells of a wave's table in the score kernels
hipError_t launch_scores(int n, int m, const uint8_t *data, const uint8_t *arity, uint32_t K,
                         int kind, double ess, const uint32_t *famask, int max_bins,
                         double *out, hipStream_t st, uint32_t *bits, int uniform_r, int d,
                         bool tables, double *lgt);
template <class P>
hipError_t launch_lattice(const LatticeArgs &a, const typename P::Store &alpha,
                          const typename P::Store &L, const typename P::Store &R,
                          hipStream_t st, PhaseEvents *ev);

}  // namespace bnk
