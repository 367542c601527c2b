// Refit of the cost model on measured programs (Algorithm 1: the top-K states are measured and
// the cost model is trained on (S^, P); Section 6.1 and Appendix A.1: XGBoost with Ansor's
// settings).  One boosting round of histogram-based gradient boosting under the pack-sum squared
// error 1/2 sum_p w_p (s_p - y_p)^2, s_p = base + the sum of program p's statement margins; the
// gain, leaf weight and learned missing direction follow Chen and Guestrin (KDD'16, Sections 3
// and 3.4).
//
//   k_gb_bin        bin of feature f of row r = number of cut points <= x (upper bound), 255 for NaN,
//                   stored in 8-feature groups: byte ((f / 8) ld + r) 8 + f % 8, so that a
//                   workgroup of one group reads its rows' 8 bytes from one contiguous plane
//   k_gb_start      per program: s_p (fp64, statements in order), g_p = w_p (s_p - y_p), h_p = w_p,
//                   per-block maxima of |g|, |h|; other workgroups clear the tree and node arrays
//   k_gb_row_q      the fixed-point exponents: |v 2^e| <= 2^(62 - ceil(log2 N)), so sums of N rows
//                   of 64-bit integers are exact, and no result depends on summation order; each
//                   statement row's integer gradient and hessian
//   per depth d < max_depth (rows kept grouped by node in `order`, the root in row order):
//     k_gb_segments (before d = 1, some large sets) bins and gradient pairs as lines of a row
//     k_gb_hist     workgroup = (chunk of a node's rows, 8 features): a [2][8][256] int64 histogram
//                   in LDS (ds_add of integers; the lanes of one add instruction are spread over the
//                   8 features, so at most 8 meet on one bin; the bin of 0.0 is the total minus the
//                   others).  Only one child of a kept parent is built, the smaller; a node of one
//                   chunk without a kept parent is evaluated at once, the others store partials
//     k_gb_split    workgroup = (node, feature): partials summed, or the parent's histogram minus the
//                   sibling's partials; the node's histogram kept if it has more than keep_rows rows;
//                   split evaluation
//     k_gb_part     workgroup = chunk of a node's rows: the node's best split over the features, then
//                   its rows moved to the children's ranges, or the leaf's weight added to their
//                   margins
//
// What bounds it, on 2.12 M rows x 164 features (binning + two rounds: 14.9 -> 3.7 ms; one round's
// k_gb_hist 5.2 -> 0.90 ms): the root's histogram (205 us) by its LDS adds and by reading 8 B of bins and,
// per feature group, 16 B of gradient pair a row; the levels below it (150 .. 42 us; 520 us a level on
// average when every node was built from 8-byte gathers) by cache lines and LDS adds.  Building the smaller child alone
// halves the rows and more; the line layout (169 us, once) makes a row cost two lines instead of 21 + 1.
// On 68,182 rows (binning + four rounds: 2.76 -> 1.6 ms) launches and chains of dependent loads bound it:
// three launches a level instead of nine, each level's work list worked out by every workgroup for
// itself.
//
// Split evaluation (k_gb_hist in place: thread = (feature, 8 consecutive bins); k_gb_split: thread = bin):
// an int64 prefix over bins gives GL, HL for every threshold index t; the gain GL^2/(HL+l) + GR^2/(HR+l) -
// G^2/(H+l) is fp64 with contraction off, missing rows tried left, then right (without missing rows both
// are one split); the best is the largest gain, ties to the lowest (feature, t, missing-left first).
// Every decision is therefore bit-identical to a sequential evaluation of the same definitions.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <type_traits>

#include "internal.hpp"

#pragma clang fp contract(off)

namespace harl {
namespace {

constexpr int kThreads = 256;
constexpr int kGroup = 8;           // features per histogram workgroup (one 8-byte load per row)
constexpr int kBins = 256;          // bin 255 holds the missing values
constexpr int kBinStride = 257;     // int64 words per (feature, G|H) histogram row: odd, so that
                                    // the 8 features' rows fall on different LDS banks
constexpr int kSegBytes = 128, kSegGroups = (kSegBytes - 16) / kGroup;
constexpr int kDist = kGroup * kBinStride;  // words from a feature's G row to its H row in LDS
constexpr int kFeatWords = 2 * kBins;  // int64 words of one feature of a stored histogram
constexpr int kMinChunk = 512;       // rows of a histogram chunk, at least
constexpr int kInPlaceRows = 4096;   // sets up to this size: every node one chunk, evaluated in place
constexpr int kManyRows = 1 << 20;   // sets from this size: more chunks, 16 rows per partition thread
// Histogram workgroups of a level below the root, about, at most: three for each that the machine holds,
// which take several chunks in turn and even out chunks of different sizes (trees of thousands of nodes,
// 68,000 rows x 164 features: 1,321 us a round with 768, 1,179 with 1,536, 1,149 with 2,304; 2,058 up to
// 98 for each of the 21 feature groups: 1,131).  A cap per feature group is none for the machine: with 98
// each, 2.1 M rows x 8 features took 917 us and now 732; 5,000 rows x 4,096 features 1,779 and now 1,182.
constexpr int kMaxHistBlocks = 2304;
constexpr int64_t kLineBytes = 96 << 20;  // bin bytes, rows and feature groups from which rows are laid
constexpr int kLineRows = 1 << 19, kLineGroups = 3;  // out in lines (see plan_for)
constexpr int kMaxSegBlocks = 1 << 16;  // k_gb_segments workgroups per segment, at most (rows in turn): a
                                     // thread per 16 bytes of 2^29 rows or more would pass 2^32 threads
constexpr int kQProgs = 32;          // programs per k_gb_row_q workgroup and turn
// Workgroups of programs in k_gb_start and k_gb_row_q, at most (they take more programs in turn): every
// workgroup of the second reads the maxima of all of the first, so without a limit that work grew with
// the square of the programs (16 M programs of one row, 8 features, a round of depth 6: 17.9 ms without the
// limit, 4.4 with it), and beyond 2^29 programs the grid passed 2^32 threads.
constexpr int kMaxProgBlocks = 2048;
constexpr int kBinPasses = 16;       // passes over rows per binning workgroup, at most

struct Params {
    double eta, lambda, gamma, mcw, base;
    int depth;
};

// One split candidate's record; key orders candidates: (feature, t, missing-left first).
struct Best {
    double gain;
    int32_t key, valid;
    int64_t GL, HL, G, H;
};

struct Ws {
    double *gp, *hp, *bmax;      // [P], [P], [2][nblk]
    int32_t *exps;               // [2]
    longlong2 *q;                // [N] gradient and hessian of every row
    int32_t *order, *order2;     // rows grouped by node, this level's and the next one's
    int32_t *start, *cnt, *sf;   // per heap node: first position, rows, split feature (-1: none)
    int32_t *rank;               // per heap node: slot of its kept histogram, or -1
    uint64_t *nlr;               // per heap node: rows moved left | rows moved right << 32
    int32_t *pbase, *nparts;     // level: first partial of a node and their number
    int32_t *list, *lvl;         // level: the nodes k_gb_split evaluates, and their number
    int32_t *alive;              // per level: nodes whose parent was split
    int32_t *zb;                 // [F] the bin of 0.0 per feature
    Best *best;                  // level: [2^d][F]
    int64_t *part, *hist[2];     // [pmax], [slots] by level parity: histograms [F][G|H][kBins]
    uint8_t *seg;                // [segments][N][kSegBytes], large sets
    int pmax, slots;
};

__device__ __forceinline__ int ceil_log2(int64_t n) {
    int c = 0;
    while (((int64_t)1 << c) < n) ++c;
    return c;
}

__device__ __forceinline__ double node_score(double G, double H, double lambda) { return (G * G) / (H + lambda); }

__device__ __forceinline__ int clamp_cuts(const int32_t *n_cuts, int f, int cut_stride) {
    int nc = n_cuts[f];
    nc = nc < 0 ? 0 : nc;
    nc = nc > 254 ? 254 : nc;
    return nc > cut_stride ? cut_stride : nc;
}

// a precedes b: larger gain, then the smaller key
__device__ __forceinline__ bool better(const Best &a, const Best &b) {
    if (!a.valid) return false;
    if (!b.valid) return true;
    if (a.gain > b.gain) return true;
    if (a.gain < b.gain) return false;
    return a.key < b.key;
}

// The candidate split with left sums (gl, hl) of a node with sums (Gi, Hi), if it is admissible and
// gains more than the best so far.
__device__ __forceinline__ void try_split(int64_t gl, int64_t hl, int64_t Gi, int64_t Hi, double parent, int key,
                                          const Params &prm, int eg, int eh, int &bv, double &bg, int &bk, int64_t &bGL,
                                          int64_t &bHL) {
    const double GL = ldexp((double)gl, -eg), HL = ldexp((double)hl, -eh);
    const double GR = ldexp((double)(Gi - gl), -eg), HR = ldexp((double)(Hi - hl), -eh);
    if (!(HL >= prm.mcw) || !(HR >= prm.mcw)) return;
    const double gain = (node_score(GL, HL, prm.lambda) + node_score(GR, HR, prm.lambda)) - parent;
    if (!bv || gain > bg) {
        bv = 1;
        bg = gain;
        bk = key;
        bGL = gl;
        bHL = hl;
    }
}

// The best candidate of each group of W lanes (larger gain, then the smaller key), on all of them.
template <int W>
__device__ __forceinline__ void best_lanes(int &bv, double &bg, int &bk, int64_t &bGL, int64_t &bHL) {
#pragma unroll
    for (int off = W / 2; off > 0; off >>= 1) {
        const double og = __shfl_xor(bg, off, W);
        const int ok = __shfl_xor(bk, off, W), ov = __shfl_xor(bv, off, W);
        const int64_t oGL = __shfl_xor(bGL, off, W), oHL = __shfl_xor(bHL, off, W);
        if (ov && (!bv || og > bg || (og == bg && ok < bk))) {
            bv = ov;
            bg = og;
            bk = ok;
            bGL = oGL;
            bHL = oHL;
        }
    }
}

// ------------------------------------------------------------------------------------------
// binning
// ------------------------------------------------------------------------------------------
// Workgroup = (8-feature group, range of rows).  Per feature a table of 256 buckets of the cut points'
// order-preserving keys is built in LDS first: bucket -> how many cut points lie in lower buckets and
// how many up to it, so a value starts its binary search with the cut points of its own bucket alone.
// A search takes `steps` probes, as many as the fullest bucket of the group needs: 2 or 3 where the cut
// points are spread over the keys, 4 for 152 of them over six decades and one at 0.0 (which stretches the
// window so that a bucket is an octave), 8 at most.  The bucket is any monotone function of the key, the
// same for cut points and values, so the result is the plain count of cut points <= x; -0 counts as +0.
// A thread codes two rows of the group, whose 16 searches overlap; the first rows are loaded while the
// table is built, which 32 lanes per feature do by counting (1 us; a search per bucket took 9).
// 2.1 M rows x 164 features: 760 us with searches over all cut points (8 probes), 402 us now, 4.3 TB/s of
// the features and bins; the probes' LDS reads and the address arithmetic bound it.  16,384 rows x 164
// features: 10.3 us then, 10.7 now.
__device__ __forceinline__ uint32_t bin_key(float v) {
    const uint32_t u = __float_as_uint(v + 0.f);  // -0 + 0 = +0
    return u ^ ((uint32_t)((int32_t)u >> 31) | 0x80000000u);
}

__device__ __forceinline__ uint32_t bin_bucket(float v, uint32_t base, int sh) {
    const uint32_t k = bin_key(v), d = k > base ? k - base : 0u;
    return min(d >> sh, 255u);
}

constexpr int kBinRows = 2;          // rows per thread and pass
constexpr int kCutStride = 264;      // cut points per feature in LDS: NaN past the last one

__global__ __launch_bounds__(kThreads) void k_gb_bin(const float *__restrict__ x, int64_t ldx, int F, int N,
                                                     const float *__restrict__ cuts, int cut_stride,
                                                     const int32_t *__restrict__ n_cuts, uint8_t *__restrict__ bins,
                                                     int64_t ld, int passes) {
    __shared__ float sc[kGroup][kCutStride];
    __shared__ __attribute__((aligned(16))) uint16_t lut[kGroup][256];  // cut points in lower buckets | up to this one << 8
    __shared__ uint32_t cnt[kGroup][64];  // cut points per bucket, a byte each
    __shared__ int snc[kGroup], ssh[kGroup], full;
    __shared__ uint32_t sbase[kGroup];
    const int g = blockIdx.y, t = threadIdx.x;
    const int nf = min(kGroup, F - g * kGroup);
    const float *__restrict__ xg = x + (int64_t)g * kGroup * ldx;
    const int r_first = blockIdx.x * passes * kThreads * kBinRows + t;
    float v[kBinRows][kGroup];
    // the last group of 8 may have fewer features: those past F are neither read nor searched nor stored
    auto fetch = [&](int r0) {  // rows past N are clamped and not stored
#pragma unroll
        for (int j = 0; j < kGroup; ++j)
            if (j < nf)
#pragma unroll
                for (int q = 0; q < kBinRows; ++q) v[q][j] = xg[(int64_t)j * ldx + min(r0 + q * kThreads, N - 1)];
    };
    fetch(r_first);  // in flight while the table is built
    if (t < kGroup) snc[t] = t < nf ? clamp_cuts(n_cuts, g * kGroup + t, cut_stride) : 0;
    if (t == 0) full = 0;
    (&cnt[0][0])[t] = 0;
    (&cnt[0][0])[t + kThreads] = 0;
    __syncthreads();
    for (int e = t; e < kGroup * kCutStride; e += kThreads) {
        const int j = e / kCutStride, i = e % kCutStride;
        sc[j][i] = i < snc[j] ? cuts[(int64_t)(g * kGroup + j) * cut_stride + i] : NAN;
    }
    __syncthreads();
    {  // 32 lanes per feature: its window, its cut points counted per bucket, then their prefix sums
        const int j = t / 32, q = t % 32, nc = snc[j];
        uint32_t base = 0;
        int sh = 0;
        if (nc > 0) {
            const uint32_t k0 = bin_key(sc[j][0]), k1 = bin_key(sc[j][nc - 1]), span = k1 > k0 ? k1 - k0 : 0u;
            sh = max(0, 24 - __builtin_clz(span | 1u));
            sh += (span >> sh) > 253u;
            base = k0 > (1u << sh) ? k0 - (1u << sh) : 0u;  // the first cut point in bucket 1
        }
        for (int i = q; i < nc; i += 32) {
            const uint32_t b = bin_bucket(sc[j][i], base, sh);
            atomicAdd(&cnt[j][b / 4], 1u << (8 * (b % 4)));
        }
        if (q == 0) {
            sbase[j] = base;
            ssh[j] = sh;
        }
        __syncthreads();
        const uint32_t c[2] = {cnt[j][2 * q], cnt[j][2 * q + 1]};
        int n[8], sum = 0, most = 0;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            n[e] = (int)((c[e / 4] >> (8 * (e % 4))) & 255u);
            sum += n[e];
            most = max(most, n[e]);
        }
        int before = sum;
#pragma unroll
        for (int off = 1; off < 32; off <<= 1) {
            const int o = __shfl_up(before, off, 32);
            if (q >= off) before += o;
            most = max(most, __shfl_xor(most, off, 32));
        }
        before -= sum;
        uint32_t e2[4];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const uint32_t w = (uint32_t)before | (uint32_t)(before + n[e]) << 8;
            e2[e / 2] = e % 2 ? e2[e / 2] | w << 16 : w;
            before += n[e];
        }
        *reinterpret_cast<uint4 *>(&lut[j][8 * q]) = make_uint4(e2[0], e2[1], e2[2], e2[3]);
        if (q == 0 && most > 0) atomicMax(&full, most);
    }
    __syncthreads();
    const int steps = 32 - __builtin_clz(full | 1) - (full == 0);  // 2^steps > full
    uint32_t base[kGroup];
    int sh[kGroup];
#pragma unroll
    for (int j = 0; j < kGroup; ++j) {
        base[j] = sbase[j];
        sh[j] = ssh[j];
    }
    auto bin_rows = [&](auto all, int r0) {
        constexpr bool ALL = decltype(all)::value;  // 8 features
        int lo[kBinRows][kGroup], hi[kBinRows][kGroup];
#pragma unroll
        for (int j = 0; j < kGroup; ++j)
            if (ALL || j < nf)
#pragma unroll
                for (int q = 0; q < kBinRows; ++q) {
                    const uint32_t e = lut[j][bin_bucket(v[q][j], base[j], sh[j])];
                    lo[q][j] = (int)(e & 255u);
                    hi[q][j] = (int)(e >> 8);
                }
        for (int s = 0; s < steps; ++s)  // a finished search stays: its next cut point is > v (or the NaN after the last)
#pragma unroll
            for (int j = 0; j < kGroup; ++j)
                if (ALL || j < nf)
#pragma unroll
                    for (int q = 0; q < kBinRows; ++q) {
                        const int mid = (lo[q][j] + hi[q][j]) >> 1;
                        const bool up = sc[j][mid] <= v[q][j];
                        lo[q][j] = up ? mid + 1 : lo[q][j];
                        hi[q][j] = up ? hi[q][j] : mid;
                    }
#pragma unroll
        for (int q = 0; q < kBinRows; ++q) {
            uint32_t w[2] = {0, 0};
#pragma unroll
            for (int j = 0; j < kGroup; ++j)
                if (ALL || j < nf)
                    w[j / 4] |= (v[q][j] != v[q][j] ? 255u : (uint32_t)min(lo[q][j], 254)) << (8 * (j % 4));
            const int r = r0 + q * kThreads;
            if (r < N) *reinterpret_cast<uint2 *>(bins + ((int64_t)g * ld + r) * kGroup) = make_uint2(w[0], w[1]);
        }
    };
    for (int ps = 0; ps < passes; ++ps) {
        const int r0 = r_first + ps * kThreads * kBinRows;
        if (r0 - t >= N) return;
        if (ps > 0) fetch(r0);
        if (nf == kGroup) bin_rows(std::true_type{}, r0);
        else bin_rows(std::false_type{}, r0);
    }
}

// ------------------------------------------------------------------------------------------
// gradients
// ------------------------------------------------------------------------------------------
// Blocks below nblk: per program s_p, g_p, h_p (a thread's programs nblk * kThreads apart) and the block's
// maxima of |g|, |h|.  The others: tree arrays to unreached-node defaults, node state cleared, the features' zero bins.
struct TreeOut {
    int32_t *feature;
    float *threshold;
    int32_t *left, *right;
    uint8_t *default_left;
    float *leaf_value;
};

__global__ __launch_bounds__(kThreads) void k_gb_start(const float *__restrict__ margin,
                                                       const int32_t *__restrict__ prog_ptr, int P,
                                                       const float *__restrict__ label,
                                                       const float *__restrict__ weight, double base, int N, int nblk,
                                                       int n_nodes, int levels, int F,
                                                       const float *__restrict__ cuts, int cut_stride, const int32_t *__restrict__ n_cuts, Ws w,
                                                       TreeOut tr) {
    __shared__ double sg[kThreads], sh[kThreads];
    if ((int)blockIdx.x >= nblk) {
        const int i = ((int)blockIdx.x - nblk) * kThreads + threadIdx.x;
        if (i < n_nodes) {
            tr.feature[i] = -1;
            tr.threshold[i] = 0.f;
            tr.left[i] = 0;
            tr.right[i] = 0;
            tr.default_left[i] = 0;
            tr.leaf_value[i] = 0.f;
            w.sf[i] = -1;
            w.rank[i] = -1;
            w.nlr[i] = 0;
        }
        if (i < levels) w.alive[i] = 0;
        if (i < F) {  // the bin of 0.0: the number of cut points <= 0
            const float *cf = cuts + (int64_t)i * cut_stride;
            int lo = 0, hi = clamp_cuts(n_cuts, i, cut_stride);
            while (lo < hi) {
                const int mid = (lo + hi) >> 1;
                if (cf[mid] <= 0.f) lo = mid + 1;
                else hi = mid;
            }
            w.zb[i] = lo;
        }
        return;
    }
    double ag = 0.0, ah = 0.0;
    for (int64_t p = (int64_t)blockIdx.x * kThreads + threadIdx.x; p < P; p += (int64_t)nblk * kThreads) {
        const int r0 = min(max(prog_ptr[p], 0), N), r1 = min(max(prog_ptr[p + 1], r0), N);
        double s = base;
        int r = r0;
        for (; r + 8 <= r1; r += 8) {  // eight loads in flight, added in row order
            float v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = margin[r + u];
#pragma unroll
            for (int u = 0; u < 8; ++u) s += (double)v[u];
        }
        for (; r < r1; ++r) s += (double)margin[r];
        const double g = (double)weight[p] * (s - (double)label[p]);
        const double h = (double)weight[p];
        w.gp[p] = g;
        w.hp[p] = h;
        if (r1 > r0) {
            ag = fmax(ag, fabs(g));
            ah = fmax(ah, fabs(h));
        }
    }
    sg[threadIdx.x] = ag;
    sh[threadIdx.x] = ah;
    __syncthreads();
    for (int s = kThreads / 2; s > 0; s >>= 1) {
        if (threadIdx.x < s) {
            sg[threadIdx.x] = fmax(sg[threadIdx.x], sg[threadIdx.x + s]);
            sh[threadIdx.x] = fmax(sh[threadIdx.x], sh[threadIdx.x + s]);
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        w.bmax[2 * blockIdx.x] = sg[0];
        w.bmax[2 * blockIdx.x + 1] = sh[0];
    }
}

// The fixed-point exponents (every workgroup from the block maxima; workgroup 0 stores them) and the
// integer pair of every row of the workgroup's 32 programs (several times 32 in turn), row by row so that
// the stores coalesce.
__global__ __launch_bounds__(kThreads) void k_gb_row_q(const int32_t *__restrict__ prog_ptr, int P, int N, int nblk,
                                                       Ws w) {
    __shared__ double sg[kThreads], sh[kThreads];
    __shared__ int64_t qgs[kQProgs], qhs[kQProgs];
    __shared__ int32_t first[kQProgs], last[kQProgs];
    __shared__ int32_t se[2];
    const int t = threadIdx.x;
    double ag = 0.0, ah = 0.0;
    for (int b = t; b < nblk; b += kThreads) {
        ag = fmax(ag, w.bmax[2 * b]);
        ah = fmax(ah, w.bmax[2 * b + 1]);
    }
    sg[t] = ag;
    sh[t] = ah;
    __syncthreads();
    for (int s = kThreads / 2; s > 0; s >>= 1) {
        if (t < s) {
            sg[t] = fmax(sg[t], sg[t + s]);
            sh[t] = fmax(sh[t], sh[t + s]);
        }
        __syncthreads();
    }
    if (t < 2) {
        const double a = t == 0 ? sg[0] : sh[0];
        int e = 0;
        if (a > 0.0) {
            int E;
            frexp(a, &E);
            e = 62 - ceil_log2(N > 0 ? N : 1) - E;
        }
        se[t] = e;
        if (blockIdx.x == 0) w.exps[t] = e;
    }
    __syncthreads();
    for (int64_t p0 = (int64_t)blockIdx.x * kQProgs; p0 < P; p0 += (int64_t)gridDim.x * kQProgs) {
        const int np = (int)min((int64_t)kQProgs, P - p0);
        if (t < np) {
            const int64_t p = p0 + t;
            qgs[t] = (int64_t)rint(ldexp(w.gp[p], se[0]));
            qhs[t] = (int64_t)rint(ldexp(w.hp[p], se[1]));
            const int r0 = min(max(prog_ptr[p], 0), N);  // clamped
            first[t] = r0;
            last[t] = min(max(prog_ptr[p + 1], r0), N);
        }
        __syncthreads();
        for (int r = first[0] + t; r < last[np - 1]; r += kThreads) {
            int lo = 0, hi = np;  // the program whose rows hold r: the number of programs with last <= r
            while (lo < hi) {
                const int mid = (lo + hi) >> 1;
                if (last[mid] <= r) lo = mid + 1;
                else hi = mid;
            }
            lo = min(lo, np - 1);
            w.q[r] = make_longlong2(qgs[lo], qhs[lo]);
        }
        __syncthreads();  // the next turn rewrites the programs in LDS
    }
}

// ------------------------------------------------------------------------------------------
// one depth level
// ------------------------------------------------------------------------------------------
// Node j of level d (heap index k) and how its histogram is made:
//   direct   a node of one chunk whose parent's histogram was not kept: one workgroup per feature
//            group builds it and evaluates it in place
//   parts    built from its rows, one partial histogram per chunk: a node of several chunks, and the
//            smaller child of a node whose own histogram was kept
//   derived  the larger child of such a node: the parent's histogram minus its sibling's, exact in
//            integers, so its rows are not read
// A node's histogram is kept (rank: its slot) when it has more than keep_rows rows and is above the
// last level.  A level's chunks have the rows it builds / plan.chunks, so that few rows still make
// enough workgroups.
struct NodeInfo {
    int alive, s, n, built, from_parent;
    int chunks, parts, listed, kept;
};

__device__ __forceinline__ NodeInfo node_rows(const Ws &w, int d, int j, int N) {
    NodeInfo o{0, 0, 0, 0, 0, 0, 0, 0, 0};
    o.built = 1;
    if (d == 0) {
        o.alive = 1;
        o.n = N;
    } else {
        const int p = ((1 << (d - 1)) - 1) + j / 2;
        const int n = w.cnt[p], nl = (int)(uint32_t)w.nlr[p], s = w.start[p];
        o.from_parent = w.rank[p] >= 0;
        o.alive = w.sf[p] >= 0;
        o.s = (j & 1) ? s + nl : s;
        o.n = (j & 1) ? n - nl : nl;
        if (o.from_parent) o.built = (nl <= n - nl) == !(j & 1);  // the smaller child (the left one of equals)
        if (!o.alive) o = NodeInfo{0, 0, 0, 0, 0, 0, 0, 0, 0};
    }
    return o;
}

__device__ __forceinline__ void node_chunks(NodeInfo &o, int chunk, int keep_rows) {
    if (!o.alive) return;
    o.chunks = o.built ? max(1, (o.n + chunk - 1) / chunk) : 0;
    o.parts = o.built && (o.from_parent || o.chunks > 1) ? o.chunks : 0;
    o.listed = !o.built || o.parts > 0;
    o.kept = o.n > keep_rows;
}

// Histogram words addressed in LDS (32-bit addresses, the G to H distance an instruction offset).
typedef __attribute__((address_space(3))) unsigned long long *lds_words;
__device__ __forceinline__ void lds_add(lds_words p, int64_t v) {
    __hip_atomic_fetch_add(p, (unsigned long long)v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// One row's bins of a feature group.
struct Bytes {
    uint32_t w[2];
    __device__ __forceinline__ void read(const uint8_t *p) {
        const uint2 v = *reinterpret_cast<const uint2 *>(p);
        w[0] = v.x;
        w[1] = v.y;
    }
    // byte (e + k) % 8 becomes byte e
    __device__ __forceinline__ void turn(int k) {
        const uint32_t a = k & 4 ? w[1] : w[0], b = k & 4 ? w[0] : w[1];
        w[0] = __builtin_amdgcn_alignbyte(b, a, k & 3);
        w[1] = __builtin_amdgcn_alignbyte(a, b, k & 3);
    }
};

// Inclusive sums over the workgroup's 64 NW threads of two packed counters.
template <int NW>
__device__ __forceinline__ void scan2(uint64_t &a, uint32_t &b, uint64_t (&wa)[NW], uint32_t (&wb)[NW]) {
    const int lane = threadIdx.x % 64, wv = threadIdx.x / 64;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint64_t ua = __shfl_up(a, o);
        const uint32_t ub = __shfl_up(b, o);
        if (lane >= o) {
            a += ua;
            b += ub;
        }
    }
    if (lane == 63) {
        wa[wv] = a;
        wb[wv] = b;
    }
    __syncthreads();
#pragma unroll
    for (int v = 0; v < NW; ++v)
        if (v < wv) {
            a += wa[v];
            b += wb[v];
        }
}

// Evaluate the splits of a workgroup's features f0 .. of one node from its histogram, G in
// h[feature][kBinStride] and H kDist words further, and cut counts n_cuts, all in LDS; thread =
// (feature j = t / 32, bins 8 (t % 32) ..).  Results in out[j].
__device__ __forceinline__ void evaluate(const int64_t *h, int f0, int F, const int32_t *n_cuts, const Params &prm,
                                         int eg, int eh, Best *out) {
    const int t = threadIdx.x, j = t / 32, q = t % 32, f = f0 + j;
    const int64_t *hg = h + j * kBinStride + 8 * q, *hh = hg + kDist;
    int64_t ig = 0, ih = 0;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        ig += hg[e];
        ih += hh[e];
    }
    int64_t xg = -ig, xh = -ih;  // the sums of the lanes before this one, after the scan
#pragma unroll
    for (int off = 1; off < 32; off <<= 1) {  // inclusive scan over the 32 lanes of this feature
        const int64_t ag = __shfl_up(ig, off, 32), ah = __shfl_up(ih, off, 32);
        if (q >= off) {
            ig += ag;
            ih += ah;
        }
    }
    xg += ig;
    xh += ih;
    const int64_t Gi = __shfl(ig, 31, 32), Hi = __shfl(ih, 31, 32);
    const int64_t Gm = h[j * kBinStride + 255], Hm = h[kDist + j * kBinStride + 255];
    // this lane's best candidate, kept in scalars (a struct copied under a condition spills)
    int bv = 0, bk = 0;
    double bg = 0.0;
    int64_t bGL = 0, bHL = 0;
    if (f < F) {
        const int nc = n_cuts[j];
        const int lo_dir = (Gm | Hm) != 0 ? 0 : 1;  // without missing rows both directions are one split
        const double parent = node_score(ldexp((double)Gi, -eg), ldexp((double)Hi, -eh), prm.lambda);
#pragma unroll 1
        for (int e = 0; e < 8; ++e) {  // the bins read again: their prefix sums in registers cost occupancy
            const int tt = 8 * q + e + 1;
            if (tt > nc) break;
            xg += hg[e];
            xh += hh[e];
            for (int dir = 1; dir >= lo_dir; --dir)
                try_split(xg + (dir ? Gm : 0), xh + (dir ? Hm : 0), Gi, Hi, parent, (f * 256 + tt) * 2 + (1 - dir), prm, eg, eh,
                          bv, bg, bk, bGL, bHL);
        }
    }
    // best over the 32 lanes of the feature: larger gain, then smaller key
    best_lanes<32>(bv, bg, bk, bGL, bHL);
    if (q == 0 && f < F) out[j] = Best{bg, bk, bv, bGL, bHL, Gi, Hi};
}

struct HistArgs {
    const uint8_t *bins;
    int64_t ld;
    int F, n_fg, d, D, N;
    int hx, seg_groups;     // chunks in flight (workgroups per feature group); feature groups per segment
    int chunks, keep_rows;  // chunks a level is cut into; rows above which a histogram is kept
    int cut_stride;
    const int32_t *n_cuts;
    Params prm;
};

// The rows' bins and gradient pairs as one 128-byte line per (segment, row): seg_groups feature groups
// and, in the last 16 bytes, the pair.  A row of a deep node then costs one cache line per segment
// instead of one per feature group and one for the pair.
__global__ __launch_bounds__(kThreads) void k_gb_segments(HistArgs a, Ws w) {
    constexpr int kParts = kSegBytes / 16;  // threads per line, 16 bytes each
    const int part = threadIdx.x % kParts, sgi = blockIdx.y;
    for (int64_t r = ((int64_t)blockIdx.x * kThreads + threadIdx.x) / kParts; r < a.N; r += (int64_t)gridDim.x * (kThreads / kParts)) {
        uint64_t v[2] = {0, 0};
        if (part == kParts - 1) {
            const longlong2 q = w.q[r];
            v[0] = (uint64_t)q.x;
            v[1] = (uint64_t)q.y;
        } else {
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const int k = 2 * part + e, fg = sgi * a.seg_groups + k;
                if (k < a.seg_groups && fg < a.n_fg)
                    v[e] = *reinterpret_cast<const uint64_t *>(a.bins + ((int64_t)fg * a.ld + r) * kGroup);
            }
        }
        *reinterpret_cast<ulonglong2 *>(w.seg + ((int64_t)sgi * a.N + r) * kSegBytes + part * 16) = make_ulonglong2(v[0], v[1]);
    }
}

// Workgroup = (chunk c, feature group fg) of the level's built nodes, several in turn.  Every
// workgroup that can have a chunk works out the level's chunk list from the parents' partition by itself (a scan over at
// most 2^d nodes, cheaper than a launch of its own); workgroup (0, 0) stores it for the kernels that
// follow.
template <bool SEG>
__global__ __launch_bounds__(kThreads, 3) void k_gb_hist(HistArgs a, Ws w) {
    __shared__ int64_t h[2 * kDist];  // 32.1 KB
    __shared__ int64_t tot[2][kThreads / 64];
    __shared__ uint64_t wa[kThreads / 64];
    __shared__ uint32_t wb[kThreads / 64];
    __shared__ int32_t nd[6];  // this unit's node: j, first row, rows, chunk of the node, partial (-1: direct), all chunks
    __shared__ int32_t snc[kGroup], szb[kGroup], sexp[2];
    const int t = threadIdx.x;
    // workgroup -> (first chunk, feature group).  SEG: the feature groups of one segment and chunk, which
    // read the same cache lines, are dealt to one XCD (workgroups go to the 8 XCDs in turn)
    const int n_fg = a.n_fg;
    int fg, bx, nbx;
    if constexpr (SEG) {
        const int i = blockIdx.x / 8, set = i / a.seg_groups * 8 + blockIdx.x % 8;
        const int n_seg = (n_fg + a.seg_groups - 1) / a.seg_groups;
        fg = set % n_seg * a.seg_groups + i % a.seg_groups;
        bx = set / n_seg;
        nbx = a.hx;
        if (fg >= n_fg || bx >= nbx) return;
    } else {
        fg = blockIdx.x % n_fg;
        bx = blockIdx.x / n_fg;
        nbx = a.hx;
    }
    // a level has at most a chunk per node more than the a.chunks its rows are cut into: the others leave
    // before they work out the chunk list
    if (bx >= a.chunks && bx >= a.chunks + w.alive[a.d]) return;
    const int f0 = fg * kGroup;
    const int nf = std::min(kGroup, a.F - f0);
    if (t < kGroup) {
        snc[t] = t < nf ? clamp_cuts(a.n_cuts, f0 + t, a.cut_stride) : 0;
        szb[t] = t < nf ? w.zb[f0 + t] : -1;
        if (t < 2) sexp[t] = w.exps[t];
    }
    const int L = 1 << a.d, base = L - 1;
    const int per = (L + kThreads - 1) / kThreads;  // consecutive nodes per thread
    NodeInfo first{0, 0, 0, 0, 0, 0, 0, 0, 0};  // this thread's first node (its only one up to 256 nodes)
    int64_t rows = 0;  // rows this level builds
    for (int q = 0; q < per; ++q) {
        const int j = t * per + q;
        if (j >= L) break;
        const NodeInfo o = node_rows(w, a.d, j, a.N);
        if (q == 0) first = o;
        rows += o.alive && o.built ? o.n : 0;
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) rows += __shfl_xor(rows, off);
    if (t % 64 == 0) tot[0][t / 64] = rows;
    __syncthreads();
    rows = 0;
#pragma unroll
    for (int v = 0; v < kThreads / 64; ++v) rows += tot[0][v];
    const int chunk = max(kMinChunk, (int)((rows + a.chunks - 1) / a.chunks));
    const int keep_rows = a.d + 1 < a.D ? a.keep_rows : INT32_MAX;
    node_chunks(first, chunk, keep_rows);
    auto node = [&](int q) {
        if (q == 0) return first;
        NodeInfo o = node_rows(w, a.d, t * per + q, a.N);
        node_chunks(o, chunk, keep_rows);
        return o;
    };
    uint64_t mine = 0;   // chunks | parts << 32
    uint32_t mine2 = 0;  // listed nodes | kept nodes << 16
    for (int q = 0; q < per; ++q) {
        if (t * per + q >= L) break;
        const NodeInfo o = node(q);
        mine += (uint64_t)o.chunks | (uint64_t)o.parts << 32;
        mine2 += (uint32_t)o.listed | (uint32_t)o.kept << 16;
    }
    uint64_t incl = mine;
    uint32_t incl2 = mine2;
    scan2(incl, incl2, wa, wb);
    if (t == kThreads - 1) nd[5] = (int)(uint32_t)incl;
    const int c_lo = (int)(uint32_t)(incl - mine), c_hi = (int)(uint32_t)incl;
    if (bx == 0 && fg == 0) {
        int pb = (int)((incl - mine) >> 32), li = (int)((incl2 - mine2) & 0xFFFFu), rk = (int)((incl2 - mine2) >> 16);
        for (int q = 0; q < per; ++q) {
            const int j = t * per + q;
            if (j >= L) break;
            const NodeInfo o = node(q);
            if (!o.alive) continue;
            const int k = base + j;
            w.start[k] = o.s;
            w.cnt[k] = o.n;
            w.pbase[j] = pb;
            w.nparts[j] = o.parts;
            w.rank[k] = o.kept && rk < w.slots ? rk : -1;
            if (o.listed) w.list[li] = j;
            pb += o.parts;
            li += o.listed;
            rk += o.kept;
        }
        if (t == kThreads - 1) w.lvl[0] = (int)(incl2 & 0xFFFFu);
    }
    // the bin of 0.0 (statement features are mostly zeros) is not added row by row: it is the
    // chunk's total minus the other bins, exact in integers.  At add step e lane l adds feature
    // (e + l) % 8, so one instruction spreads its lanes over the 8 features and at most 8 of
    // them can meet on one bin.
    __syncthreads();
    uint32_t zb[kGroup];
    lds_words hb[kGroup];  // the feature's row of h
#pragma unroll
    for (int e = 0; e < kGroup; ++e) {
        const int jj = (e + t) % kGroup;
        zb[e] = szb[jj] < 0 ? 0u : (uint32_t)szb[jj];  // the bytes of features past F are 0: never added
        hb[e] = (lds_words)h + jj * kBinStride;
    }
    const int n_chunks = nd[5];
    for (int c = bx; c < n_chunks; c += nbx) {
        if (c_lo <= c && c < c_hi) {  // the one thread whose nodes hold chunk c
            int c0 = c_lo, pb = (int)((incl - mine) >> 32);
            for (int q = 0; q < per; ++q) {
                const int j = t * per + q;
                if (j >= L) break;
                const NodeInfo o = node(q);
                if (c < c0 + o.chunks) {
                    nd[0] = j;
                    nd[1] = o.s;
                    nd[2] = o.n;
                    nd[3] = c - c0;
                    nd[4] = o.parts ? pb + (c - c0) : -1;
                    break;
                }
                c0 += o.chunks;
                pb += o.parts;
            }
        }
        for (int e = t; e < 2 * kDist; e += kThreads) h[e] = 0;
        __syncthreads();
        const int j = nd[0], s = nd[1], n = nd[2], part = nd[4];
        const int i0 = s + nd[3] * chunk, i1 = std::min(s + n, i0 + chunk);
        int64_t sg = 0, sh = 0;
        // 4 kThreads rows at a time: the loads of the next batch (and the positions of the one after) are
        // in flight while this one is added
        constexpr int U = 4;
        int rn[U];
        Bytes word[U];
        longlong2 q[U];
        auto rows_at = [&](int b0) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int i = b0 + t + kThreads * u;
                rn[u] = i < i1 ? (a.d == 0 ? i : w.order[i]) : -1;
            }
        };
        auto load = [&](Bytes (&wd)[U], longlong2 (&qq)[U]) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int r = rn[u] < 0 ? 0 : rn[u];
                if constexpr (SEG) {
                    const uint8_t *line = w.seg + ((int64_t)(fg / a.seg_groups) * a.N + r) * kSegBytes;
                    wd[u].read(line + fg % a.seg_groups * kGroup);
                    qq[u] = *reinterpret_cast<const longlong2 *>(line + kSegBytes - 16);
                } else {
                    wd[u].read(a.bins + ((int64_t)fg * a.ld + r) * kGroup);
                    qq[u] = w.q[r];
                }
            }
        };
        if (i0 < i1) {  // a node without rows loads nothing: with no rows at all the bins may be null
            rows_at(i0);
            load(word, q);
        }
        for (int b0 = i0; b0 < i1; b0 += (4 * kThreads)) {
            Bytes wc[U];
            longlong2 qc[U];
            bool in[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                wc[u] = word[u];
                qc[u] = q[u];
                in[u] = b0 + t + kThreads * u < i1;
            }
            if (b0 + (4 * kThreads) < i1) {
                rows_at(b0 + (4 * kThreads));
                load(word, q);
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (!in[u]) break;
                sg += qc[u].x;
                sh += qc[u].y;
                // the row's bytes turned so that byte e is feature (e + t) % kGroup's: constant positions
                wc[u].turn(t % kGroup);
#pragma unroll
                for (int e = 0; e < kGroup; ++e) {
                    const uint32_t b = (wc[u].w[e / 4] >> (8 * (e % 4))) & 255u;
                    if (b != zb[e]) {
                        lds_add(hb[e] + b, qc[u].x);
                        lds_add(hb[e] + b + kDist, qc[u].y);
                    }
                }
            }
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            sg += __shfl_xor(sg, off);
            sh += __shfl_xor(sh, off);
        }
        if (t % 64 == 0) {
            tot[0][t / 64] = sg;
            tot[1][t / 64] = sh;
        }
        __syncthreads();
        {  // zero bin = total - the other bins: 16 threads per (G|H, feature) row, 16 bins each
            const int row = t / 16, q = t % 16, gh = row / kGroup, jj = row % kGroup;
            const int b0 = szb[jj];
            int64_t *hr = &h[(gh * kGroup + jj) * kBinStride];
            int64_t rest = 0;
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int b = q + 16 * e;
                rest += b == b0 ? 0 : hr[b];
            }
#pragma unroll
            for (int off = 8; off > 0; off >>= 1) rest += __shfl_xor(rest, off, 16);
            int64_t all = 0;
#pragma unroll
            for (int v = 0; v < kThreads / 64; ++v) all += tot[gh][v];
            __syncthreads();
            if (q == 0 && b0 >= 0) hr[b0] = all - rest;
        }
        __syncthreads();
        if (part < 0) {
            evaluate(h, f0, a.F, snc, a.prm, sexp[0], sexp[1], &w.best[(int64_t)j * a.F + f0]);
        } else if (part < w.pmax) {  // always: fewer than pmax partials exist at any level
            // the partial: bins 0 .. n_cuts and 255 of every feature, [feature][G|H][256]
            int64_t *g = w.part + ((int64_t)part * a.F + f0) * kFeatWords;
#pragma unroll
            for (int jj = 0; jj < kGroup; ++jj)
                if (jj < nf && (t <= snc[jj] || t == 255)) {
                    g[(2 * jj + 0) * kBins + t] = h[jj * kBinStride + t];
                    g[(2 * jj + 1) * kBins + t] = h[kDist + jj * kBinStride + t];
                }
        }
        __syncthreads();  // h and nd are rewritten by the next unit
    }
}

// Histograms and split evaluation of the listed nodes.  Workgroup = (node, feature), several in turn;
// thread (z, t) sums bin t over a quarter z of the node's (or its sibling's) partials.
template <int Z>
__global__ __launch_bounds__(kThreads * Z) void k_gb_split(HistArgs a, Ws w) {
    __shared__ int64_t sz[2][Z][kThreads];
    __shared__ int64_t ws2[2][kThreads / 64];
    __shared__ int64_t miss[2];
    __shared__ Best red[kThreads / 64];
    const int t = threadIdx.x % kThreads, z = threadIdx.x / kThreads, wv = t / 64, lane = t % 64;
    const int L = 1 << a.d, base = L - 1;
    const int units = w.lvl[0] * a.F;
    const int eg = w.exps[0], eh = w.exps[1];
    const int64_t stride = (int64_t)a.F * kFeatWords;
    for (int u = blockIdx.x; u < units; u += gridDim.x) {
        const int j = w.list[u / a.F], f = u % a.F, k = base + j;
        const int nc = clamp_cuts(a.n_cuts, f, a.cut_stride);
        const bool used = t <= nc || t == 255;
        const bool derived = w.nparts[j] == 0;
        const int src = derived ? j ^ 1 : j;
        const int np = w.nparts[src];
        const int64_t *g = w.part + ((int64_t)w.pbase[src] * a.F + f) * kFeatWords + t;
        int64_t G = 0, H = 0;
        if (used) {
            const int q0 = (int)((int64_t)np * z / Z), q1 = (int)((int64_t)np * (z + 1) / Z);
            int q = q0;
            for (; q + 8 <= q1; q += 8) {
                int64_t v[8], x[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    v[e] = g[(q + e) * stride];
                    x[e] = g[(q + e) * stride + kBins];
                }
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    G += v[e];
                    H += x[e];
                }
            }
            for (; q < q1; ++q) {
                G += g[q * stride];
                H += g[q * stride + kBins];
            }
        }
        if constexpr (Z > 1) {
            sz[0][z][t] = G;
            sz[1][z][t] = H;
            __syncthreads();
            if (z == 0) {
#pragma unroll
                for (int v = 1; v < Z; ++v) {
                    G += sz[0][v][t];
                    H += sz[1][v][t];
                }
            }
        }
        int bv = 0, bk = 0;
        double bg = 0.0;
        int64_t bGL = 0, bHL = 0, Gi = 0, Hi = 0;
        if (z == 0) {
            if (derived && used) {
                const int pr = w.rank[(k - 1) / 2];
                const int64_t *ph = w.hist[(a.d + 1) & 1] + ((int64_t)pr * a.F + f) * kFeatWords + t;
                G = ph[0] - G;
                H = ph[kBins] - H;
            }
            const int rk = w.rank[k];
            if (rk >= 0 && used) {
                int64_t *o = w.hist[a.d & 1] + ((int64_t)rk * a.F + f) * kFeatWords + t;
                o[0] = G;
                o[kBins] = H;
            }
            if (t == 255) {
                miss[0] = G;
                miss[1] = H;
            }
        }
        int64_t ig = G, ih = H;  // inclusive sums over the bins
        if (z == 0) {
#pragma unroll
            for (int off = 1; off < 64; off <<= 1) {
                const int64_t ag = __shfl_up(ig, off), ah = __shfl_up(ih, off);
                if (lane >= off) {
                    ig += ag;
                    ih += ah;
                }
            }
            if (lane == 63) {
                ws2[0][wv] = ig;
                ws2[1][wv] = ih;
            }
        }
        __syncthreads();
        if (z == 0) {
#pragma unroll
            for (int v = 0; v < kThreads / 64; ++v) {
                Gi += ws2[0][v];
                Hi += ws2[1][v];
                if (v < wv) {
                    ig += ws2[0][v];
                    ih += ws2[1][v];
                }
            }
            const int tt = t + 1;
            if (tt <= nc) {
                const double parent = node_score(ldexp((double)Gi, -eg), ldexp((double)Hi, -eh), a.prm.lambda);
                const int lo_dir = (miss[0] | miss[1]) != 0 ? 0 : 1;  // without missing rows both directions are one split
                for (int dir = 1; dir >= lo_dir; --dir)
                    try_split(ig + (dir ? miss[0] : 0), ih + (dir ? miss[1] : 0), Gi, Hi, parent, (f * 256 + tt) * 2 + (1 - dir),
                              a.prm, eg, eh, bv, bg, bk, bGL, bHL);
            }
            best_lanes<64>(bv, bg, bk, bGL, bHL);
            if (lane == 0) red[wv] = Best{bg, bk, bv, bGL, bHL, Gi, Hi};
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            int ri = 0;
            for (int v = 1; v < kThreads / 64; ++v)
                if (better(red[v], red[ri])) ri = v;
            w.best[(int64_t)j * a.F + f] = red[ri];
        }
    }
}

__device__ __forceinline__ float leaf_weight(int64_t Gi, int64_t Hi, int eg, int eh, const Params &prm) {
    const double G = ldexp((double)Gi, -eg), H = ldexp((double)Hi, -eh);
    return (float)(-(G / (H + prm.lambda)) * prm.eta);
}

// Decisions and partition of the level's nodes.  Workgroup = chunk of a node's rows (several in
// turn): it takes the node's best split over the features (every chunk for itself; chunk 0 writes the
// tree's arrays), then either adds the leaf's weight to the margins of its rows, which are then
// finished, or moves its rows into the children's ranges: lefts from the front, rights from the back,
// at places taken with one atomic per chunk.  The order of a node's chunks in its children depends
// on scheduling; no result does, since every sum over rows is an integer sum.  The children of the
// last level are leaves: their rows get the margins here and are not moved.
template <int R>
__global__ __launch_bounds__(kThreads) void k_gb_part(HistArgs a, Ws w, const float *__restrict__ cuts, TreeOut tr,
                                                      float *__restrict__ margin) {
    constexpr int pchunk = R * kThreads;
    __shared__ uint64_t wa[kThreads / 64];
    __shared__ uint32_t wb[kThreads / 64];
    __shared__ int32_t nd[5];  // this unit's node: j, first row, rows, chunk of the node; all chunks
    __shared__ Best red[kThreads / 64];
    __shared__ int32_t wl[kThreads / 64], place[2];
    const int t = threadIdx.x, wv = t / 64, lane = t % 64;
    const int L = 1 << a.d, base = L - 1;
    const int per = (L + kThreads - 1) / kThreads;
    auto chunks_of = [&](int j) {
        if (a.d > 0 && w.sf[((1 << (a.d - 1)) - 1) + j / 2] < 0) return 0;
        return max(1, (w.cnt[base + j] + pchunk - 1) / pchunk);
    };
    uint64_t mine = 0, incl;
    uint32_t none = 0;
    for (int q = 0; q < per; ++q)
        if (t * per + q < L) mine += (uint64_t)chunks_of(t * per + q);
    incl = mine;
    scan2(incl, none, wa, wb);
    if (t == kThreads - 1) nd[4] = (int)incl;
    __syncthreads();
    const int n_chunks = nd[4];
    const int eg = w.exps[0], eh = w.exps[1];
    const bool last = a.d + 1 == a.D;
    for (int c = blockIdx.x; c < n_chunks; c += gridDim.x) {
        if ((int)(incl - mine) <= c && c < (int)incl) {
            int c0 = (int)(incl - mine);
            for (int q = 0; q < per; ++q) {
                const int j = t * per + q;
                if (j >= L) break;
                const int n = chunks_of(j);
                if (c < c0 + n) {
                    nd[0] = j;
                    nd[1] = w.start[base + j];
                    nd[2] = w.cnt[base + j];
                    nd[3] = c - c0;
                    break;
                }
                c0 += n;
            }
        }
        __syncthreads();
        const int j = nd[0], s = nd[1], n = nd[2], ci = nd[3], k = base + j;
        const int i0 = s + ci * pchunk, i1 = std::min(s + n, i0 + pchunk);
        int r[R];  // this chunk's rows, read while the decision is taken
#pragma unroll
        for (int u = 0; u < R; ++u) {
            const int i = i0 + u * kThreads + t;
            r[u] = i < i1 ? (a.d == 0 ? i : w.order[i]) : -1;
        }
        // the node's best split: larger gain, then the smaller key
        int bv = 0, bk = 0;
        double bg = 0.0;
        int64_t bGL = 0, bHL = 0;
        const Best *bs = w.best + (int64_t)j * a.F;
        for (int f = t; f < a.F; f += kThreads) {
            const Best o = bs[f];
            if (o.valid && (!bv || o.gain > bg || (o.gain == bg && o.key < bk))) {
                bv = 1;
                bg = o.gain;
                bk = o.key;
                bGL = o.GL;
                bHL = o.HL;
            }
        }
        const int64_t G = bs[0].G, H = bs[0].H;
        best_lanes<64>(bv, bg, bk, bGL, bHL);
        if (lane == 0) red[wv] = Best{bg, bk, bv, bGL, bHL, 0, 0};
        __syncthreads();
        int ri = 0;
#pragma unroll
        for (int v = 1; v < kThreads / 64; ++v)
            if (better(red[v], red[ri])) ri = v;
        const bool split = red[ri].valid && red[ri].gain > a.prm.gamma;
        const int key = red[ri].key, f = key / 512, tt = (key / 2) % 256, dir = 1 - (key & 1);
        if (!split) {
            const float v = leaf_weight(G, H, eg, eh, a.prm);
            if (ci == 0 && t == 0) tr.leaf_value[k] = v;
#pragma unroll
            for (int u = 0; u < R; ++u)
                if (r[u] >= 0) margin[r[u]] = margin[r[u]] + v;
            __syncthreads();
            continue;
        }
        const float vl = last ? leaf_weight(red[ri].GL, red[ri].HL, eg, eh, a.prm) : 0.f;
        const float vr = last ? leaf_weight(G - red[ri].GL, H - red[ri].HL, eg, eh, a.prm) : 0.f;
        if (ci == 0 && t == 0) {
            tr.feature[k] = f;
            tr.threshold[k] = cuts[(int64_t)f * a.cut_stride + tt - 1];
            tr.left[k] = 2 * k + 1;
            tr.right[k] = 2 * k + 2;
            tr.default_left[k] = (uint8_t)dir;
            if (last) {
                tr.leaf_value[2 * k + 1] = vl;
                tr.leaf_value[2 * k + 2] = vr;
            }
            w.sf[k] = f;
            if (!last) atomicAdd(&w.alive[a.d + 1], 2);
        }
        const uint8_t *__restrict__ bf = a.bins + (int64_t)(f / kGroup) * a.ld * kGroup + f % kGroup;
        uint32_t b[R], left = 0;
        int nl = 0, nn = 0;
#pragma unroll
        for (int u = 0; u < R; ++u) b[u] = bf[(int64_t)max(r[u], 0) * kGroup];
#pragma unroll
        for (int u = 0; u < R; ++u) {
            const bool gl = b[u] == 255 ? dir != 0 : (int)b[u] < tt;
            if (r[u] >= 0) {
                ++nn;
                nl += gl;
                left |= (uint32_t)gl << u;
                if (last) margin[r[u]] = margin[r[u]] + (gl ? vl : vr);
            }
        }
        if (!last) {
            // places: this thread's lefts follow those of the threads before it (and its rights likewise)
            int il = nl | nn << 16;
#pragma unroll
            for (int off = 1; off < 64; off <<= 1) {
                const int o = __shfl_up(il, off);
                if (lane >= off) il += o;
            }
            if (lane == 63) wl[wv] = il;
            __syncthreads();
            int all = 0, before = il - (nl | nn << 16);
#pragma unroll
            for (int v = 0; v < kThreads / 64; ++v) {
                if (v < wv) before += wl[v];
                all += wl[v];
            }
            if (t == 0) {
                const int l = all & 0xFFFF, rr = (all >> 16) - l;
                const uint64_t at = atomicAdd(reinterpret_cast<unsigned long long *>(&w.nlr[k]),
                                              (unsigned long long)l | (unsigned long long)rr << 32);
                place[0] = (int)(uint32_t)at;
                place[1] = (int)(at >> 32);
            }
            __syncthreads();
            int pl = s + place[0] + (before & 0xFFFF);
            int pr = s + n - 1 - (place[1] + (before >> 16) - (before & 0xFFFF));
#pragma unroll
            for (int u = 0; u < R; ++u) {
                if (r[u] < 0) continue;
                if (left >> u & 1) w.order2[pl++] = r[u];
                else w.order2[pr--] = r[u];
            }
        }
        __syncthreads();
    }
}

// ------------------------------------------------------------------------------------------
// workspace
// ------------------------------------------------------------------------------------------

// How a level's rows are cut (k_gb_hist): into `chunks` pieces (1: a set small enough that every
// node is evaluated in place), and the rows above which a node's histogram is kept for its children.
struct Plan {
    int chunks, keep_rows, slots, pmax;
    int n_seg, seg_groups;  // segments of the row lines (0: none)
};

// Chunks that a level's rows are cut into, times the feature groups.  Three histogram workgroups fit a CU
// (146 registers a thread): 768 are one full machine, which is also enough for small sets, whose partials
// cost as much as their rows; from kManyRows on the finer cut of 1,024 pays (2.1 M rows x 164 features, a
// round of depth 10: 1,454 us with 768, 1,386 with 1,024).
int hist_blocks(int N) { return N >= kManyRows ? 1024 : 768; }

Plan plan_for(int N, int F) {
    const int n_fg = (F + kGroup - 1) / kGroup;
    Plan p;
    p.chunks = 1;
    if (N > kInPlaceRows) {
        p.chunks = std::max(2, hist_blocks(N) / n_fg);
        p.chunks = std::min(p.chunks, (N + kMinChunk - 1) / kMinChunk);
    }
    // keeping and subtracting a node's histogram moves about as many bytes as building 4,096 rows; at
    // most 192 histograms of a level and 256 MB of them are kept
    const int64_t node = (int64_t)F * kFeatWords * 8;
    const int most = (int)std::max<int64_t>(1, std::min<int64_t>(192, ((int64_t)256 << 20) / node));
    p.keep_rows = p.chunks == 1 ? INT32_MAX : std::max(4096, N / most);
    // kept nodes have more than keep_rows rows.  Partials of a level: nodes of several chunks have
    // fewer than 2 chunks' worth of pieces in all, and the kept nodes' smaller children one each
    p.slots = p.chunks == 1 ? 1 : N / p.keep_rows + 1;
    p.pmax = p.chunks == 1 ? 1 : 2 * p.chunks + p.slots;
    // Lines pay where a node's rows are spread over more memory than the caches hold and where a line has
    // enough in it: bins of a group beyond an XCD's 4 MB L2 (from 2^19 rows), bins in all beyond
    // kLineBytes, and three groups or more (one: 24 of 128 bytes used, and a workspace of 128 bytes a row).
    // One round of depth 10 without and with them, in us: 100 MB of bins as 1 group 2,943 / 3,355, 2:
    // 1,713 / 1,795, 3: 1,350 / 1,288, 8: 923 / 740, 21: 623 / 605; of 437,000 rows x 30 groups 530 / 539;
    // 204,000 x 64 421 / 479; 200 MB as 4 groups 2,349 / 1,917, 21: 1,215 / 945, 409,000 x 64 799 / 817.
    const bool lines = (int64_t)N * n_fg * kGroup >= kLineBytes && N >= kLineRows && n_fg >= kLineGroups;
    p.n_seg = lines ? (n_fg + kSegGroups - 1) / kSegGroups : 0;
    p.seg_groups = lines ? (n_fg + p.n_seg - 1) / p.n_seg : 1;
    return p;
}

// Workgroups for P programs, `per` of them each in a turn.
int prog_blocks(int P, int per) { return (int)std::min<int64_t>(ceil_div(std::max(P, 1), per), kMaxProgBlocks); }

Ws carve(void *base, int F, int N, int P, int depth, size_t *total) {
    const int64_t n_nodes = ((int64_t)1 << (depth + 1)) - 1;
    const int64_t Lmax = (int64_t)1 << (depth - 1);  // widest level that builds histograms
    const int64_t nblk = prog_blocks(P, kThreads);
    char *p = static_cast<char *>(base);
    size_t o = 0;
    auto take = [&](size_t bytes) {
        char *r = p ? p + o : nullptr;
        o += (bytes + 255) / 256 * 256;
        return r;
    };
    Ws w;
    w.gp = reinterpret_cast<double *>(take(sizeof(double) * std::max(P, 1)));
    w.hp = reinterpret_cast<double *>(take(sizeof(double) * std::max(P, 1)));
    w.bmax = reinterpret_cast<double *>(take(sizeof(double) * 2 * nblk));
    w.exps = reinterpret_cast<int32_t *>(take(sizeof(int32_t) * 2));
    w.q = reinterpret_cast<longlong2 *>(take(sizeof(longlong2) * std::max(N, 1)));
    w.order = reinterpret_cast<int32_t *>(take(sizeof(int32_t) * std::max(N, 1)));
    w.order2 = reinterpret_cast<int32_t *>(take(sizeof(int32_t) * std::max(N, 1)));
    w.start = reinterpret_cast<int32_t *>(take(sizeof(int32_t) * n_nodes));
    w.cnt = reinterpret_cast<int32_t *>(take(sizeof(int32_t) * n_nodes));
    w.sf = reinterpret_cast<int32_t *>(take(sizeof(int32_t) * n_nodes));
    w.rank = reinterpret_cast<int32_t *>(take(sizeof(int32_t) * n_nodes));
    w.nlr = reinterpret_cast<uint64_t *>(take(sizeof(uint64_t) * n_nodes));
    w.pbase = reinterpret_cast<int32_t *>(take(sizeof(int32_t) * Lmax));
    w.nparts = reinterpret_cast<int32_t *>(take(sizeof(int32_t) * Lmax));
    w.list = reinterpret_cast<int32_t *>(take(sizeof(int32_t) * Lmax));
    w.lvl = reinterpret_cast<int32_t *>(take(sizeof(int32_t)));
    w.alive = reinterpret_cast<int32_t *>(take(sizeof(int32_t) * (depth + 1)));
    w.zb = reinterpret_cast<int32_t *>(take(sizeof(int32_t) * F));
    w.best = reinterpret_cast<Best *>(take(sizeof(Best) * Lmax * F));
    const Plan plan = plan_for(N, F);
    w.slots = plan.slots;
    w.pmax = plan.pmax;
    const size_t node = sizeof(int64_t) * (size_t)F * kFeatWords;
    w.part = reinterpret_cast<int64_t *>(take(node * (size_t)w.pmax));
    w.hist[0] = reinterpret_cast<int64_t *>(take(node * (size_t)w.slots));
    w.hist[1] = reinterpret_cast<int64_t *>(take(node * (size_t)w.slots));
    w.seg = reinterpret_cast<uint8_t *>(take((size_t)plan.n_seg * N * kSegBytes));
    *total = o;
    return w;
}

}  // namespace

size_t gbdt_ws_bytes(int32_t F, int32_t N, int32_t P, int32_t depth) {
    size_t total = 0;
    carve(nullptr, F, N, P, depth, &total);
    return total;
}

int gbdt_bin_launch(const float *x, int64_t ldx, int32_t F, int32_t N, const float *cuts, int32_t cut_stride,
                    const int32_t *n_cuts, uint8_t *bins, int64_t ld, hipStream_t stream) {
    if (N == 0) return HARL_OK;
    // bytes of features past F in the last group are written as zeros
    // several passes per table on large sets, while keeping about 768 workgroups
    const int64_t n_g = ceil_div(F, kGroup), per = kThreads * kBinRows;
    const int passes = (int)std::max<int64_t>(1, std::min<int64_t>(kBinPasses, ceil_div(N, per) * n_g / 768));
    const dim3 grid((unsigned)ceil_div(N, per * passes), (unsigned)n_g);
    hipLaunchKernelGGL(k_gb_bin, grid, dim3(kThreads), 0, stream, x, ldx, F, N, cuts, cut_stride, n_cuts, bins, ld,
                       passes);
    HARL_HIP_CHECK(hipGetLastError());
    return HARL_OK;
}

int gbdt_round_launch(const harl_gbdt_params *prm_in, const uint8_t *bins, int64_t ld, int32_t F, int32_t N,
                      const float *cuts, int32_t cut_stride, const int32_t *n_cuts, const int32_t *prog_ptr,
                      int32_t P, const float *label, const float *weight, float *margin, int32_t *feature,
                      float *threshold, int32_t *left, int32_t *right, uint8_t *default_left, float *leaf_value,
                      void *ws, hipStream_t stream) {
    Params prm{prm_in->eta, prm_in->reg_lambda, prm_in->gamma, prm_in->min_child_weight, prm_in->base_score,
               prm_in->max_depth};
    const int D = prm.depth;
    const int n_fg = (F + kGroup - 1) / kGroup;
    const int n_nodes = (1 << (D + 1)) - 1;
    size_t total = 0;
    Ws w = carve(ws, F, N, P, D, &total);
    const Plan plan = plan_for(N, F);
    TreeOut tr{feature, threshold, left, right, default_left, leaf_value};
    const int nblk = prog_blocks(P, kThreads);
    hipLaunchKernelGGL(k_gb_start, dim3((unsigned)(nblk + ceil_div(std::max(n_nodes, F), kThreads))), dim3(kThreads), 0,
                       stream, margin, prog_ptr, P, label, weight, prm.base, N, nblk, n_nodes, D + 1, F, cuts, cut_stride, n_cuts,
                       w, tr);
    hipLaunchKernelGGL(k_gb_row_q, dim3((unsigned)prog_blocks(P, kQProgs)), dim3(kThreads), 0, stream, prog_ptr, P, N, nblk, w);
    HARL_HIP_CHECK(hipGetLastError());
    HistArgs ha{bins, ld, F, n_fg, 0, D, N, 1, plan.seg_groups, plan.chunks, plan.keep_rows, cut_stride, n_cuts, prm};
    const int pchunk = N >= kManyRows ? 16 * kThreads : 4 * kThreads;
    for (int d = 0; d < D; ++d) {
        const int64_t L = std::min<int64_t>((int64_t)1 << d, std::max(N, 1));
        ha.d = d;
        const unsigned hx = (unsigned)(d == 0 ? plan.chunks : std::min<int64_t>(2 * plan.chunks + L, ceil_div(kMaxHistBlocks, n_fg)));
        ha.hx = (int)hx;
        if (d > 0 && plan.n_seg > 0) {
            if (d == 1)
                hipLaunchKernelGGL(k_gb_segments,
                                   dim3((unsigned)std::min<int64_t>(ceil_div((int64_t)N * (kSegBytes / 16), kThreads), kMaxSegBlocks),
                                        (unsigned)plan.n_seg),
                                   dim3(kThreads), 0, stream, ha, w);
            hipLaunchKernelGGL(k_gb_hist<true>, dim3((unsigned)(round_up((int64_t)hx * plan.n_seg, 8) * plan.seg_groups)),
                               dim3(kThreads), 0, stream, ha, w);
        } else {
            hipLaunchKernelGGL(k_gb_hist<false>, dim3(hx * (unsigned)n_fg), dim3(kThreads), 0, stream, ha, w);
        }
        HARL_HIP_CHECK(hipGetLastError());  // the kernels below read what this one stores
        if (plan.chunks > 1) {
            if (d == 0)
                hipLaunchKernelGGL(k_gb_split<4>, dim3((unsigned)F), dim3(4 * kThreads), 0, stream, ha, w);
            else
                hipLaunchKernelGGL(k_gb_split<1>, dim3((unsigned)std::min<int64_t>(L * F, 4096)), dim3(kThreads), 0, stream,
                                   ha, w);
        }
        const unsigned px = (unsigned)std::min<int64_t>(ceil_div(std::max(N, 1), pchunk) + L, 2048);
        if (N >= kManyRows)
            hipLaunchKernelGGL(k_gb_part<16>, dim3(px), dim3(kThreads), 0, stream, ha, w, cuts, tr, margin);
        else
            hipLaunchKernelGGL(k_gb_part<4>, dim3(px), dim3(kThreads), 0, stream, ha, w, cuts, tr, margin);
        std::swap(w.order, w.order2);
        HARL_HIP_CHECK(hipGetLastError());
    }
    return HARL_OK;
}

}  // namespace harl
