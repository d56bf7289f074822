// Exact kNN by brute force: the plain definition of the problem the forest approximates
// (Sec. 1: the K points of U nearest to each query), used as the ground truth of the
// accuracy measures of Sec. 5.1 at full data size.
//
// Every (query, point) pair gets its canonical binary64 squared distance D (32 classes of
// fma(delta, delta, s), the same tree as the rest of the library), and each query keeps the
// K points of smallest key (D, index).  Two kernels per chunk of queries:
//   k_exact_dist    D for a chunk of queries against all n points, written to a
//                   [chunk][n] binary64 buffer (a point row is read once per 8 x QL queries:
//                   it stays in registers while the lane group walks the chunk's queries,
//                   which sit in LDS);
//   k_exact_select  one 1024-thread block per query: radix select of the K-th smallest
//                   96-bit key (D bits, index) with 11-bit digits and LDS histograms, stopping
//                   once the key's bucket holds at most 2048 entries; one more pass gathers the
//                   entries below the bucket and the bucket itself; a bitonic sort in LDS
//                   orders the bucket and then the K results.
// Both are HBM / fp64-bound: per pair d binary64 subtractions and fmas; per query a few
// 8-byte reads of its n distances.  Larger problems filter the pairs on the matrix cores first
// (below) and leave only what the filter could not settle to these two.
#include <math.h>

#include <algorithm>
#include <string>

#include "rpf_internal.h"

namespace rpf {
namespace {

constexpr int kQL = 64;          // most queries of a distance block held in LDS (8 per pass)
constexpr int kSelThreads = 1024;
constexpr int kSelBins = 2048;   // 11-bit digits
constexpr int kSelCand = 2048;   // bucket size at which the select gathers and sorts
constexpr uint64_t kInfBits = 0x7ff0000000000000ull;

// The queries of an exhaustive launch: all of [0, nq), or (list) those of a device-side list,
// from its entry `first` on; a launch covers more slots than the list may hold.
struct ExactRows {
    const int32_t *list;
    const uint32_t *count;
    int64_t first;
    __device__ int64_t rows(int64_t nq) const {
        if (!list) return nq;
        const int64_t left = (int64_t)*count - first;
        return left < nq ? (left > 0 ? left : 0) : nq;
    }
    __device__ int64_t query(int64_t slot) const { return list ? list[first + slot] : slot; }
};

// D[r][j] for the queries r < nq of this launch and every point j.  NR > 0: d <= 32 NR,
// d % 4 == 0 and 16-byte rows: each lane holds its NR float4 of the point row in registers.
// NR == 0: any d, the row is re-read (from cache) per group of 8 queries.
template <int NR>
__global__ __launch_bounds__(256) void k_exact_dist(const float *__restrict__ X, int64_t n, int d,
                                                    const float *__restrict__ Q, int64_t nq, ExactRows rows, int ql,
                                                    const int64_t *__restrict__ self, double *__restrict__ D,
                                                    int64_t ldD) {
    extern __shared__ float s_q[];  // [ql][dq], dq = d rounded up to 32, zero-padded; ql % 8 == 0
    const int dq = (d + 31) & ~31;
    const int64_t qb = (int64_t)blockIdx.y * ql;
    nq = rows.rows(nq);
    if (qb >= nq) return;
    const int nql = (int)std::min<int64_t>(ql, nq - qb);
    for (int i = threadIdx.x; i < ql * dq; i += blockDim.x) {
        const int r = i / dq, c = i - r * dq;
        s_q[i] = (r < nql && c < d) ? Q[rows.query(qb + r) * d + c] : 0.f;
    }
    __syncthreads();
    const int g = threadIdx.x & 7;
    const int grp = threadIdx.x >> 3;  // 32 point slots per block
    const int nqg = (nql + 7) >> 3;
    for (int64_t j = (int64_t)blockIdx.x * 32 + grp; j < n; j += (int64_t)gridDim.x * 32) {
        const float *xr = X + j * d;
        float4 row[NR > 0 ? NR : 1];
        if (NR > 0) {
#pragma unroll
            for (int k = 0; k < NR; k++) {
                const int c = 4 * g + 32 * k;
                row[k] = c < d ? *reinterpret_cast<const float4 *>(xr + c) : make_float4(0.f, 0.f, 0.f, 0.f);
            }
        }
        for (int t = 0; t < nqg; t++) {
            double s[8][4];
#pragma unroll
            for (int r = 0; r < 8; r++) s[r][0] = s[r][1] = s[r][2] = s[r][3] = 0.0;
            // one column step: the canonical class of column c is c mod 32, held by lane
            // (c mod 32) / 4 in component c mod 4 -- as in every distance of the library
            auto step = [&](const float4 xv, int c) {
#pragma unroll
                for (int r = 0; r < 8; r++) {
                    const float4 qv = *reinterpret_cast<const float4 *>(&s_q[(t * 8 + r) * dq + c]);
                    const double e0 = (double)qv.x - (double)xv.x, e1 = (double)qv.y - (double)xv.y;
                    const double e2 = (double)qv.z - (double)xv.z, e3 = (double)qv.w - (double)xv.w;
                    s[r][0] = __builtin_fma(e0, e0, s[r][0]);
                    s[r][1] = __builtin_fma(e1, e1, s[r][1]);
                    s[r][2] = __builtin_fma(e2, e2, s[r][2]);
                    s[r][3] = __builtin_fma(e3, e3, s[r][3]);
                }
            };
            if (NR > 0) {
#pragma unroll
                for (int k = 0; k < NR; k++) step(row[k], 4 * g + 32 * k);
            } else {
                for (int c = 4 * g; c < d; c += 32) {
                    // columns past d hold 0 in the query row and are read as 0 here, so they
                    // add fma(0, 0, s) = s (s is never -0: it starts at +0 and adds squares)
                    float4 xv;
                    xv.x = xr[c];
                    xv.y = c + 1 < d ? xr[c + 1] : 0.f;
                    xv.z = c + 2 < d ? xr[c + 2] : 0.f;
                    xv.w = c + 3 < d ? xr[c + 3] : 0.f;
                    step(xv, c);
                }
            }
            double mine = 0.0;
#pragma unroll
            for (int r = 0; r < 8; r++) {
                double v = (s[r][0] + s[r][1]) + (s[r][2] + s[r][3]);
                v = group8_add(v);
                if (r == g) mine = v;
            }
            const int qr = t * 8 + g;  // this lane writes query qr of the block
            if (qr < nql) {
                const int64_t q = qb + qr;
                if (self && self[rows.query(q)] == j) mine = __longlong_as_double((long long)kInfBits);
                D[q * ldD + j] = mine;
            }
        }
    }
}

// 96-bit key of an entry: (bits of D >= 0, point index); order = (D, index) order
__device__ inline unsigned __int128 ekey(uint64_t dbits, uint32_t j) { return ((unsigned __int128)dbits << 32) | j; }

// bitonic sort of s_k[0, m) (m a power of two <= 2 kSelThreads) ascending, by the whole block
__device__ inline void block_bitonic(uint64_t *s_hi, uint32_t *s_lo, int m) {
    for (int size = 2; size <= m; size <<= 1) {
        for (int stride = size >> 1; stride > 0; stride >>= 1) {
            for (int i = threadIdx.x; i < (m >> 1); i += blockDim.x) {
                const int lo = 2 * i - (i & (stride - 1));
                const int hi = lo + stride;
                const bool up = (lo & size) == 0;
                const unsigned __int128 a = ekey(s_hi[lo], s_lo[lo]), b = ekey(s_hi[hi], s_lo[hi]);
                if ((a > b) == up) {
                    const uint64_t th = s_hi[lo];
                    const uint32_t tl = s_lo[lo];
                    s_hi[lo] = s_hi[hi];
                    s_lo[lo] = s_lo[hi];
                    s_hi[hi] = th;
                    s_lo[hi] = tl;
                }
            }
            __syncthreads();
        }
    }
}

__global__ __launch_bounds__(kSelThreads) void k_exact_select(const double *__restrict__ D, int64_t n, int64_t ldD,
                                                             ExactRows rows, int K, int32_t *__restrict__ out_idx,
                                                             float *__restrict__ out_dist) {
    __shared__ uint32_t s_hist[kSelBins];
    __shared__ uint64_t s_ch[kSelCand];  // bucket entries (D bits, index), then the results
    __shared__ uint32_t s_cl[kSelCand];
    __shared__ uint64_t s_rh[256];       // entries below the bucket
    __shared__ uint32_t s_rl[256];
    __shared__ int s_state[4];
    if ((int64_t)blockIdx.x >= rows.rows(gridDim.x)) return;
    const int64_t q = rows.query(blockIdx.x);
    const uint64_t *row = reinterpret_cast<const uint64_t *>(D + blockIdx.x * ldD);
    const int tid = threadIdx.x;
    // the K-th smallest finite key: digits of 11 bits from the top of the 96-bit key (the
    // last digit 8 bits); after each histogram the prefix grows by the digit whose bucket
    // holds the rank
    unsigned __int128 prefix = 0;
    int nbits = 0;
    int need = K;       // entries still to take at or above the prefix
    int below = 0;      // entries known to lie below the prefix (all of them results)
    int bucket = 0;     // entries matching the prefix
    bool all = false;   // fewer finite entries than K: every finite entry is a result
    for (int lev = 0; lev < 9; lev++) {
        const int w = lev < 8 ? 11 : 8;
        const int shift = 96 - nbits - w;
        const unsigned __int128 mask = nbits ? (~(unsigned __int128)0) << (96 - nbits) : 0;
        for (int i = tid; i < kSelBins; i += kSelThreads) s_hist[i] = 0;
        __syncthreads();
        for (int64_t j = tid; j < n; j += kSelThreads) {
            const uint64_t b = row[j];
            if (b >= kInfBits) continue;
            const unsigned __int128 k = ekey(b, (uint32_t)j);
            if ((k & mask) == prefix) atomicAdd(&s_hist[(uint32_t)(k >> shift) & ((1u << w) - 1)], 1u);
        }
        __syncthreads();
        if (tid == 0) {  // the bucket of the rank (2048 bins, one thread: cheap next to the pass)
            uint32_t cum = 0;
            int b = -1;
            for (int i = 0; i < (1 << w); i++) {
                if (cum + s_hist[i] >= (uint32_t)need) {
                    b = i;
                    break;
                }
                cum += s_hist[i];
            }
            s_state[0] = b;
            s_state[1] = (int)cum;
            s_state[2] = b >= 0 ? (int)s_hist[b] : 0;
        }
        __syncthreads();
        const int b = s_state[0];
        if (b < 0) {  // fewer than `need` finite entries match: all of them are results
            all = true;
            break;
        }
        below += s_state[1];
        need -= s_state[1];
        bucket = s_state[2];
        prefix |= (unsigned __int128)b << shift;
        nbits += w;
        __syncthreads();
        if (bucket <= kSelCand) break;
    }
    // gather: entries below the prefix are results; entries matching it are sorted
    if (tid == 0) s_state[0] = s_state[1] = 0;
    __syncthreads();
    const unsigned __int128 mask = nbits ? (~(unsigned __int128)0) << (96 - nbits) : 0;
    for (int64_t j = tid; j < n; j += kSelThreads) {
        const uint64_t b = row[j];
        if (b >= kInfBits) continue;
        const unsigned __int128 k = ekey(b, (uint32_t)j) & mask;
        if (all || k < prefix) {
            const int at = atomicAdd(&s_state[0], 1);
            if (at < 256) {
                s_rh[at] = b;
                s_rl[at] = (uint32_t)j;
            }
        } else if (k == prefix) {
            const int at = atomicAdd(&s_state[1], 1);
            if (at < kSelCand) {
                s_ch[at] = b;
                s_cl[at] = (uint32_t)j;
            }
        }
    }
    __syncthreads();
    const int nr = min(s_state[0], 256), nc = all ? 0 : min(s_state[1], kSelCand);
    int m2 = 1;
    while (m2 < nc) m2 <<= 1;
    for (int i = nc + tid; i < m2; i += kSelThreads) {
        s_ch[i] = ~0ull;
        s_cl[i] = ~0u;
    }
    __syncthreads();
    if (nc > 1) block_bitonic(s_ch, s_cl, m2);
    // results: the nr entries below, then the first `need` of the bucket, sorted together
    const int take = all ? 0 : min(need, nc);
    const int tot = nr + take;
    __syncthreads();
    for (int i = tid; i < take; i += kSelThreads) {  // move the bucket's head behind the below-entries
        s_rh[nr + i] = s_ch[i];
        s_rl[nr + i] = s_cl[i];
    }
    __syncthreads();
    int m3 = 1;
    while (m3 < tot) m3 <<= 1;
    for (int i = tot + tid; i < m3; i += kSelThreads) {
        s_rh[i] = ~0ull;
        s_rl[i] = ~0u;
    }
    __syncthreads();
    if (tot > 1) block_bitonic(s_rh, s_rl, m3);
    for (int i = tid; i < K; i += kSelThreads) {
        if (i < tot) {
            out_idx[q * K + i] = (int32_t)s_rl[i];
            out_dist[q * K + i] = (float)sqrt(__longlong_as_double((long long)s_rh[i]));
        } else {
            out_idx[q * K + i] = -1;
            out_dist[q * K + i] = INFINITY;
        }
    }
    (void)below;
}

// ---------------------------------------------------------------- filtered search
//
// For more than a few queries the binary64 distances of all pairs are not needed: a Gram
// product on the matrix cores brackets every distance, and only the pairs that the bracket
// cannot exclude are measured in binary64.  Per chunk of queries:
//   k_exact_split   rows minus a common centre (any centre is valid: distances do not change),
//                   split into bfloat16 hi + lo and laid out as MFMA fragments, and their norms;
//   k_exact_tile<MODE 0>  upper bounds of the distances to S sampled points (S about K n / 768);
//   k_exact_tau     per query, a threshold at or above the K-th smallest of them: at least K
//                   points lie within it;
//   k_exact_tile<MODE 1>  every point whose lower bound is within the threshold (about 768 a
//                   query on a representative sample) joins the query's list;
//   k_exact_rank    binary64 distance of every listed point, top-K by (D, index).
// A query whose list overflows (many equal or nearly equal distances, or values outside what
// the bracket covers) goes to the exhaustive kernels above, so results are theirs bit for bit.
// Such queries cost the passes before the tiles (k_exact_tau finds most of them), and a wave
// stops listing points of a query once it has seen its list full: 2 000 queries x 500 000 x
// 128 in two clusters far from the centre 21.8 ms (180 when every point was counted by an
// atomic, 23.2 by the exhaustive kernels alone), norms past 1e37 22.1 (325, 23.5), 50 distinct
// rows 32.3 (48.6, 34.4); 64 x 100 000, 10 distinct rows 1.23 (5.6, 1.05).
//
// Bracket: with a' = fl(a - centre), G the computed hi.hi + hi.lo + lo.hi of a'.b' and na, nb
// the squared norms of a', b':  |D - (na + nb - 2G)| <= E (na + nb) + eta.  The split leaves
// out at most 3.1 * 2^-18 |a'||b'| (half of which, twice, meets na + nb >= 2|a'||b'|); the
// accumulation of 3d products errs by at most (3d + 32) 2^-23 |a'||b'|; centring, the norms
// and the tests' own roundings by at most 40 * 2^-24 (na + nb); eta covers underflow.  Norms
// above 1e37 become NaN, which no test excludes.  The accumulation's term allows every one of
// the 3d additions, in any order, an error of one unit in the last place of a partial sum, and
// no partial sum is above |a'||b'| (1 + 2^-6).  The instruction's own rounding is not
// documented; measured against binary64 sums over 512 x 512 pairs of each of ten kinds of rows
// (normal, one sign, exponents over 40 bits, one large value per row or per instruction,
// cancelling pairs, sums of half units) it errs by at most 3.7 units of 2^-23 |a'||b'| at
// d = 16 (80 allowed), 7.7 at 128 (416) and 13.8 at 512 (1 568).
// Bound: MFMA (three bfloat16 products, 6 d flop a pair).  2 000 queries x 500 000 x 128, K 20:
// 1.14 ms a call, 0.75 of it the MODE 1 tiles (1.0 PFLOP/s of bfloat16 products); measuring
// every pair in binary64 took 21.4 ms (0.38 of the binary64 rate and 24 GB of distances).

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int kFiltCap = 4096;     // listed points of a query
constexpr int kFiltQueue = 192;    // pairs a wave holds before it appends them to the lists
constexpr int64_t kFiltBounds = (int64_t)1 << 30;  // bytes of the bounds to the sample
constexpr float kFiltEta = 1e-33f;

// mean of at most 512 rows (every stride-th), 64 columns per block
__global__ __launch_bounds__(1024) void k_exact_centre(const float *__restrict__ X, int64_t n, int d, int64_t stride,
                                                       float *__restrict__ mu) {
    __shared__ float s[16][64];
    const int c = blockIdx.x * 64 + (threadIdx.x & 63), r = threadIdx.x >> 6;
    float v = 0.f;
    const int rows = (int)std::min<int64_t>(512, (n + stride - 1) / stride);
    if (c < d)
        for (int i = r; i < rows; i += 16) v += X[i * stride * d + c] * (1.0f / 512);
    s[r][threadIdx.x & 63] = v;
    __syncthreads();
    if (r) return;
    for (int i = 1; i < 16; i++) v += s[i][threadIdx.x];
    v *= 512.0f / (float)rows;
    if (c < d) mu[c] = v - v == 0.f ? v : 0.f;  // a mean that overflows: no centre
}

// Rows start + stride * i, i < cnt, in tiles of 32: fragment (tile, kstep, part, lane) holds
// columns 16 kstep + 8 (lane / 32) .. + 7 of row 32 tile + lane % 32; part 0 = hi, 1 = lo.
__global__ __launch_bounds__(256) void k_exact_split(const float *__restrict__ X, int64_t n, int d, int64_t stride,
                                                     const float *__restrict__ mu, int KS, __bf16 *__restrict__ F,
                                                     float *__restrict__ nrm) {
    __shared__ double s_n[4][64];
    const int64_t tile = blockIdx.x;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int64_t row = tile * 32 + (lane & 31);
    const bool ok = row * stride < n;
    const float *x = X + (ok ? row * stride : 0) * d;
    double sum = 0.0;
    for (int ks = w; ks < KS; ks += 4) {
        const int c = 16 * ks + 8 * (lane >> 5);
        float v[8];
#pragma unroll
        for (int h = 0; h < 2; h++) {
            const int j = c + 4 * h;
            float4 a = make_float4(0.f, 0.f, 0.f, 0.f), m = a;
            if (ok && j < d) {
                a = load4<false>(x + j, d - j);
                m = load4<false>(mu + j, d - j);
            }
            v[4 * h] = a.x - m.x;
            v[4 * h + 1] = a.y - m.y;
            v[4 * h + 2] = a.z - m.z;
            v[4 * h + 3] = a.w - m.w;
        }
        bf16x8 hi, lo;
#pragma unroll
        for (int e = 0; e < 8; e++) {
            hi[e] = (__bf16)v[e];
            lo[e] = (__bf16)(v[e] - (float)hi[e]);
            sum += (double)v[e] * (double)v[e];
        }
        bf16x8 *f = reinterpret_cast<bf16x8 *>(F) + ((tile * KS + ks) * 2) * 64 + lane;
        f[0] = hi;
        f[64] = lo;
    }
    s_n[w][lane] = sum;
    __syncthreads();
    if (threadIdx.x < 32) {
        double v = 0.0;
        for (int q = 0; q < 4; q++) v += s_n[q][threadIdx.x] + s_n[q][threadIdx.x + 32];
        nrm[tile * 32 + threadIdx.x] = v < 1e37 ? (float)v : __int_as_float(0x7fc00000);
    }
}

// Bounds as the upper halves of their binary32 patterns, lb towards 0 and ub upwards (so the
// pair still brackets the distance); anything that is no number brackets everything.
__device__ inline uint32_t pack_bounds(float lb, float ub) {
    const uint32_t l = lb > 0.f ? __float_as_uint(lb) >> 16 : 0u;
    const uint32_t u = ub < 3e38f ? (__float_as_uint(ub > 0.f ? ub : 0.f) + 0xffffu) >> 16 : 0x7f80u;
    return l | u << 16;
}

// Eight waves; the block's 32 QB queries stay in LDS as fragments, each wave streams point
// tiles of 32 (CH ksteps in flight ahead), so the loop has no barrier.
template <int QB, int CH, int MODE>
__global__ __launch_bounds__(512) void k_exact_tile(const __bf16 *__restrict__ QF, const float *__restrict__ qn,
                                                    int64_t m, const __bf16 *__restrict__ PF,
                                                    const float *__restrict__ pn, int64_t npts, int64_t base, int KS,
                                                    float E, const float *__restrict__ phi, uint32_t *__restrict__ cnt,
                                                    uint2 *__restrict__ cand, float *__restrict__ ub, int64_t ldS) {
    extern __shared__ __align__(16) uint8_t smem[];
    bf16x8 *s_a = reinterpret_cast<bf16x8 *>(smem);                        // [QB][KS][2][64]
    // [8][32 QB], a copy per wave; MODE 1: -inf for a query whose list the wave has seen overflow
    // (and for padding), which no bound passes
    float *s_phis = reinterpret_cast<float *>(s_a + (size_t)QB * KS * 128);
    uint4 *s_queue = reinterpret_cast<uint4 *>(s_phis + 8 * 32 * QB);  // MODE 1: [8][kFiltQueue]
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    float *s_phi = s_phis + w * 32 * QB;
    const int64_t q0 = (int64_t)blockIdx.y * 32 * QB;
    {
        const bf16x8 *src = reinterpret_cast<const bf16x8 *>(QF) + (int64_t)blockIdx.y * QB * KS * 128;
        for (int i = threadIdx.x; i < QB * KS * 128; i += 512) s_a[i] = src[i];
        bool open = MODE == 0;
        for (int i = lane; i < 32 * QB; i += 64) {
            const int64_t q = q0 + i;
            if (MODE == 0) {
                s_phi[i] = (1.0f + E) * qn[q];
            } else {
                const bool take = q < m && cnt[q] <= (uint32_t)kFiltCap;
                s_phi[i] = take ? phi[q] : -INFINITY;
                open |= take;
            }
        }
        if (!__syncthreads_or(open)) return;  // every query of the block is left to the exhaustive kernels
    }
    const int64_t ntile = (npts + 31) / 32, step = (int64_t)gridDim.x * 8;
    const bf16x8 *P = reinterpret_cast<const bf16x8 *>(PF) + lane;
    uint4 *queue = s_queue + w * kFiltQueue;  // (query, point, (1 - E) nb - 2G, nb)
    int nq = 0;
    auto flush = [&]() {
        wave_sync();
        for (int e = lane; e < nq; e += 64) {
            const uint4 it = queue[e];
            if (s_phi[it.x] == -INFINITY) continue;  // (a norm that is no number passes even this)
            const uint32_t at = atomicAdd(&cnt[q0 + it.x], 1u);
            if (at >= (uint32_t)kFiltCap) {
                s_phi[it.x] = -INFINITY;
                continue;
            }
            const float na = qn[q0 + it.x], v = __uint_as_float(it.z), nb = __uint_as_float(it.w);
            const float lb = v + (1.0f - E) * na, ub = lb + 2.0f * E * (na + nb) + 2.0f * kFiltEta + (na + nb) * 1e-6f;
            cand[(q0 + it.x) * kFiltCap + at] = make_uint2(it.y, pack_bounds(lb - (na + nb) * 1e-6f - kFiltEta, ub));
        }
        wave_sync();
        nq = 0;
    };
    int64_t tile = (int64_t)blockIdx.x * 8 + w;
    bf16x8 nx[CH][2];
    if (tile < ntile) {
#pragma unroll
        for (int c = 0; c < CH; c++)
#pragma unroll
            for (int h = 0; h < 2; h++) nx[c][h] = P[(tile * KS + c) * 128 + 64 * h];
    }
    for (; tile < ntile; tile += step) {
        const float nb = pn[tile * 32 + (lane & 31)];
        f32x16 acc[QB];
#pragma unroll
        for (int q = 0; q < QB; q++)
#pragma unroll
            for (int i = 0; i < 16; i++) acc[q][i] = 0.f;
        for (int k0 = 0; k0 < KS; k0 += CH) {
            bf16x8 b[CH][2];
            // the next columns of this tile, or the first ones of the wave's next tile
            int64_t at = (tile * KS + k0 + CH) * 128;
            if (k0 + CH >= KS) at = (tile + step < ntile ? tile + step : tile) * KS * 128;
#pragma unroll
            for (int c = 0; c < CH; c++)
#pragma unroll
                for (int h = 0; h < 2; h++) {
                    b[c][h] = nx[c][h];
                    nx[c][h] = P[at + c * 128 + 64 * h];
                }
#pragma unroll
            for (int c = 0; c < CH; c++) {
                const bf16x8 *a = s_a + (size_t)(k0 + c) * 128 + lane;
#pragma unroll
                for (int q = 0; q < QB; q++) {
                    const bf16x8 hi = a[(size_t)q * KS * 128], lo = a[(size_t)q * KS * 128 + 64];
                    acc[q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(hi, b[c][0], acc[q], 0, 0, 0);
                    acc[q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(hi, b[c][1], acc[q], 0, 0, 0);
                    acc[q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lo, b[c][0], acc[q], 0, 0, 0);
                }
            }
        }
        // lane: point lane % 32; value i: query 8 (i / 4) + 4 (lane / 32) + i % 4 of its 32
        const int64_t col = tile * 32 + (lane & 31);
        const int r0 = 4 * (lane >> 5);
        if (MODE == 0) {
            // (rows up to the block's last are there: the buffer holds whole blocks of queries)
            float *o = ub + (q0 + r0) * ldS + col;
            if (col < npts) {
#pragma unroll
                for (int q = 0; q < QB; q++)
#pragma unroll
                    for (int i = 0; i < 16; i++) {
                        const int r = 32 * q + 8 * (i / 4) + (i & 3);
                        const float v = s_phi[r + r0] + (1.0f + E) * nb - 2.0f * acc[q][i];
                        o[r * ldS] = v > 0.f ? v + kFiltEta : v <= 0.f ? kFiltEta : INFINITY;
                    }
            }
        } else {
            const float lim = (1.0f - E) * nb;
            const bool in = col < npts;
#pragma unroll
            for (int q = 0; q < QB; q++) {
                uint32_t hit = 0;
#pragma unroll
                for (int i = 0; i < 16; i += 4) {
                    const float4 f = *reinterpret_cast<const float4 *>(s_phi + 32 * q + 2 * i + r0);
                    hit |= !(lim - 2.0f * acc[q][i] > f.x) ? 1u << i : 0u;
                    hit |= !(lim - 2.0f * acc[q][i + 1] > f.y) ? 2u << i : 0u;
                    hit |= !(lim - 2.0f * acc[q][i + 2] > f.z) ? 4u << i : 0u;
                    hit |= !(lim - 2.0f * acc[q][i + 3] > f.w) ? 8u << i : 0u;
                }
                if (!in) hit = 0;
                while (true) {  // each turn, every lane with a hit left queues one
                    const uint64_t mask = __ballot(hit != 0);
                    if (!mask) break;
                    if (nq + 64 > kFiltQueue) flush();
                    if (hit) {
                        const int i = __builtin_ctz(hit);
                        hit &= hit - 1;
                        const uint32_t r = (uint32_t)(32 * q + 8 * (i / 4) + r0 + (i & 3));
                        float v = 0.f;
#pragma unroll
                        for (int u = 0; u < 16; u++) v = i == u ? lim - 2.0f * acc[q][u] : v;
                        queue[nq + mask_rank(mask)] = make_uint4(r, (uint32_t)(base + col), __float_as_uint(v),
                                                                 __float_as_uint(nb));
                    }
                    nq += __popcll(mask);
                }
            }
        }
    }
    if (MODE == 1) flush();
}

// phi of a query: its threshold (the upper edge of the 24-bit prefix bucket that holds the
// K-th smallest of its S upper bounds, so at or above it) less its own norm's share.  A query
// of which the sample says that far more points than a list holds would pass (repeated rows,
// clusters far from the centre, norms that are no number) is left to the exhaustive kernels
// here, before the tiles list thousands of its points for nothing: cnt above kFiltCap.
template <int NT>
__global__ __launch_bounds__(NT) void k_exact_tau(const float *__restrict__ ub, int64_t ldS, int64_t S, int K,
                                                   const float *__restrict__ qn, float E,
                                                   const int64_t *__restrict__ self, int64_t n, int64_t stride,
                                                   const float *__restrict__ sn, int probes, int most,
                                                   float *__restrict__ phi, uint32_t *__restrict__ cnt) {
    // 12-bit digits: sixteen bins per octave, so that one query's distances, which share their
    // exponents, do not all meet in one counter
    constexpr int kBins = 4096 / NT;  // bins of a thread
    __shared__ uint32_t s_h[4096];
    __shared__ uint32_t s_w[NT / 64];
    __shared__ uint32_t s_sel[2];
    const uint32_t *row = reinterpret_cast<const uint32_t *>(ub + blockIdx.x * ldS);
    const int tid = threadIdx.x;
    uint32_t prefix = 0, rank = (uint32_t)K - 1;
    // the query's own row, where it is in the sample, bounds nothing
    const int64_t me = self && self[blockIdx.x] >= 0 && self[blockIdx.x] % stride == 0 ? self[blockIdx.x] / stride : -1;
    for (int b = 0; b < 2; b++) {
        for (int i = tid; i < 4096; i += NT) s_h[i] = 0;
        if (tid == 0) s_sel[0] = 4096;
        __syncthreads();
        const int sh = 19 - 12 * b;
#pragma unroll 4
        for (int64_t i = tid; i < S; i += NT) {
            const uint32_t v = row[i];
            if (v < 0x7f800000u && i != me && (b == 0 || v >> 19 == prefix >> 19)) atomicAdd(&s_h[(v >> sh) & 4095u], 1u);
        }
        __syncthreads();
        uint32_t mine = 0;
#pragma unroll
        for (int i = 0; i < kBins; i++) mine += s_h[kBins * tid + i];
        uint32_t excl, total;
        block_excl_scan_w<NT / 64>(mine, s_w, excl, total);
        if (excl <= rank && rank < excl + mine) {
            int i = kBins * tid;
            while (rank >= excl + s_h[i]) excl += s_h[i++];
            s_sel[0] = i;
            s_sel[1] = excl;
        }
        __syncthreads();
        if (s_sel[0] == 4096) {  // fewer than K finite bounds: nothing is excluded
            if (tid == 0) {
                phi[blockIdx.x] = INFINITY;
                cnt[blockIdx.x] = n > kFiltCap ? kFiltCap + 1 : 0;
            }
            return;
        }
        prefix |= s_sel[0] << sh;
        rank -= s_sel[1];
        __syncthreads();
    }
    const float tau = __uint_as_float(prefix | 0x7fu), na = qn[blockIdx.x];
    const float ph = (tau - (1.0f - E) * na) + kFiltEta + (tau + na) * 1e-6f;
    // `probes` of the sampled points, evenly spaced (neighbours in a sorted input fall together), by
    // the tiles' test, (1 - E) nb - 2G from the upper bound
    const float top = ph + (1.0f + E) * na;
    int total = 0;
    for (int e = 0; e < probes; e += 256) {
        uint32_t pass = 0;
        if (tid < 256) {
            const int64_t i = ((e + tid) * S + S / 2) / probes;
            const float u = __uint_as_float(row[i]);
            pass = !(u < 3e38f) || !(u - 2.0f * E * sn[i] > top) ? 1u : 0u;
        }
        total += __syncthreads_count((int)pass);
    }
    if (tid == 0) {
        phi[blockIdx.x] = ph;
        cnt[blockIdx.x] = total > most ? kFiltCap + 1 : 0;
    }
}

// The K nearest of a query's listed points by (D, index): those whose lower bound is within the
// K-th smallest upper bound of the list (a few more than K) are measured in binary64.  Queries
// whose list overflowed go on the exhaustive path's list.
template <bool VEC>
__global__ __launch_bounds__(256) void k_exact_rank(const float *__restrict__ X, int d, const float *__restrict__ Q,
                                                    const int64_t *__restrict__ self, const uint32_t *__restrict__ cnt,
                                                    const uint2 *__restrict__ cand, int K,
                                                    int32_t *__restrict__ out_idx, float *__restrict__ out_dist,
                                                    int32_t q0, int32_t *__restrict__ over,
                                                    uint32_t *__restrict__ n_over) {
    __shared__ uint64_t s_hi[kFiltCap];
    __shared__ uint32_t s_lo[kFiltCap];
    __shared__ uint32_t s_w[8];
    __shared__ uint32_t s_sel[4];
    uint32_t *s_h = reinterpret_cast<uint32_t *>(s_hi);  // 4096 bins, before the distances
    const int64_t q = blockIdx.x;
    const int tid = threadIdx.x, g = tid & 7;
    const uint32_t c = cnt[q];
    if (c > (uint32_t)kFiltCap) {
        if (tid == 0) over[atomicAdd(n_over, 1u)] = q0 + (int32_t)q;
        return;
    }
    const uint2 *list = cand + q * kFiltCap;
    const int64_t me = self ? self[q] : -1;
    // 15 bits of the upper bound: twelve, then three
    uint32_t lim = 0x7f80u, rank = (uint32_t)K - 1;
    for (int i = tid; i < 4096; i += 256) s_h[i] = 0;
    if (tid < 4) s_sel[tid] = 0;
    if (tid == 0) s_sel[0] = ~0u;
    __syncthreads();
    for (uint32_t i = tid; i < c; i += 256)
        if ((int64_t)list[i].x != me) atomicAdd(&s_h[list[i].y >> 19], 1u);
    __syncthreads();
    {
        uint32_t mine = 0;
#pragma unroll
        for (int i = 0; i < 16; i++) mine += s_h[16 * tid + i];
        uint32_t excl, total;
        block_excl_scan256(mine, s_w, excl, total);
        if (excl <= rank && rank < excl + mine) {
            int i = 16 * tid;
            while (rank >= excl + s_h[i]) excl += s_h[i++];
            s_sel[0] = i;
            s_sel[1] = excl;
        }
        __syncthreads();
    }
    const uint32_t bin = s_sel[0];
    if (bin != ~0u) {
        __syncthreads();
        if (tid < 8) s_h[tid] = 0;
        __syncthreads();
        for (uint32_t i = tid; i < c; i += 256)
            if ((int64_t)list[i].x != me && list[i].y >> 19 == bin) atomicAdd(&s_h[(list[i].y >> 16) & 7u], 1u);
        __syncthreads();
        rank -= s_sel[1];
        int i = 0;
        for (; i < 7 && rank >= s_h[i]; i++) rank -= s_h[i];
        lim = bin << 3 | (uint32_t)i;
    }
    __syncthreads();
    for (uint32_t i = tid; i < c; i += 256) {  // (any order: the sort decides)
        const uint2 r = list[i];
        if ((int64_t)r.x != me && (r.y & 0xffffu) <= lim) s_lo[atomicAdd(&s_sel[2], 1u)] = r.x;
    }
    __syncthreads();
    const int nr = (int)s_sel[2];
    int m2 = 1;
    while (m2 < nr) m2 <<= 1;
    const float *qr = Q + q * d;
    for (int i0 = tid >> 3; i0 < nr; i0 += 64) {  // two rows per eight lanes
        const int i1 = i0 + 32 < nr ? i0 + 32 : i0;
        const float *a = X + (int64_t)s_lo[i0] * d, *b = X + (int64_t)s_lo[i1] * d;
        double D[2];
        if (VEC) group8_dist64x2(qr, a, b, d, g, D);
        else {
            D[0] = group8_dist64<false>(qr, a, d, g);
            D[1] = group8_dist64<false>(qr, b, d, g);
        }
        if (g == 0) s_hi[i0] = (uint64_t)__double_as_longlong(D[0]);
        if (g == 1 && i1 != i0) s_hi[i1] = (uint64_t)__double_as_longlong(D[1]);
    }
    for (int i = nr + tid; i < m2; i += 256) {
        s_hi[i] = ~0ull;
        s_lo[i] = ~0u;
    }
    __syncthreads();
    if (m2 > 1) block_bitonic(s_hi, s_lo, m2);
    for (int i = tid; i < K; i += 256) {
        const bool have = i < nr && s_hi[i] < kInfBits;
        out_idx[q * K + i] = have ? (int32_t)s_lo[i] : -1;
        out_dist[q * K + i] = have ? (float)sqrt(__longlong_as_double((long long)s_hi[i])) : INFINITY;
    }
}

// Columns of a row's fragments: a multiple of the ksteps a wave keeps in flight.
int filt_ch(int d) { return d > 96 ? 4 : 2; }
int filt_ks(int d) {
    const int ch = filt_ch(d);
    return ((d + 15) / 16 + ch - 1) / ch * ch;
}

template <int MODE>
void launch_tile(hipStream_t s, int QB, int d, int64_t m, const __bf16 *QF, const float *qn, const __bf16 *PF,
                 const float *pn, int64_t npts, int64_t base, float E, const float *phi, uint32_t *cnt, uint2 *cand,
                 float *ub, int64_t ldS) {
    const int KS = filt_ks(d);
    const unsigned gy = (unsigned)((m + 32 * QB - 1) / (32 * QB));
    // about two blocks per CU in all, in multiples of eight along the points: the query blocks
    // of one range of points then run on one XCD and share its L2
    const int64_t want = std::max<int64_t>(8, 512 / gy / 8 * 8), tiles = (npts + 31) / 32;
    const unsigned gx = (unsigned)std::min<int64_t>(want, (tiles + 7) / 8);
    const size_t lds = (size_t)QB * KS * 2048 + 8 * 128 * QB + (MODE == 1 ? 8 * kFiltQueue * 16 : 0);
    auto go = [&](auto kern) {
        hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        hipLaunchKernelGGL(kern, dim3(gx, gy), dim3(512), lds, s, QF, qn, m, PF, pn, npts, base, KS, E, phi, cnt, cand,
                           ub, ldS);
    };
    const bool c4 = filt_ch(d) == 4;
    if (QB == 4) c4 ? go(k_exact_tile<4, 4, MODE>) : go(k_exact_tile<4, 2, MODE>);
    else if (QB == 2) c4 ? go(k_exact_tile<2, 4, MODE>) : go(k_exact_tile<2, 2, MODE>);
    else c4 ? go(k_exact_tile<1, 4, MODE>) : go(k_exact_tile<1, 2, MODE>);
    launch_check(s, "k_exact_tile");
}

// What the exhaustive kernels take, in us: a fit (within 10% for most, 29% at worst) to 100 calls of
// n 1 000 to 130 000, d 4 to 256 and m 1 to 2 048 that take less than 380.  The filter takes 180 to
// 215 there, so calls below 200 go without it: with it and without,
//   m 512: 2 000 x 16 183, 152    4 000 x 16 185, 166    8 000 x 16 194, 201   4 000 x 64 184, 223
//   m 128: 8 000 x 16 184, 156   16 000 x 16 197, 183   32 000 x 16 201, 232   16 000 x 64 209, 228
//   65 536 points: m 1, d 4 197, 143; d 64 203, 221   m 16, d 4 204, 168; d 64 207, 272
// (One line in n m, as it was, lost up to a third on short rows.)
double exhaustive_us(int64_t n, int64_t m, int d) {
    const double N = (double)n, M = (double)m, d64 = std::min(d, 64), more = d - d64;
    return 96 + 1e-3 * N + 0.067 * M + 1.14e-5 * N * M + 0.34 * d64 + N * (1.16e-5 * d64 + 6.5e-6 * more) +
           2.2e-7 * N * M * d;
}

// The filtered search of all m queries.  False: its workspace could not be had, or a sample that
// its bounds' memory can hold would list too many points (nothing was launched).  over / n_over
// receive the queries left to the exhaustive kernels.
// Workspace: at most 2 GiB of the points' fragments, 1 GiB of bounds to the sample, 0.7 GiB of the
// sample's fragments (a third of the points' at K 256; where the points pass through in slabs, so
// does the sample), 0.5 GiB of lists and a little more.
bool filtered_search(hipStream_t s, const float *X, int64_t n, int d, const float *Q, int64_t m, const int64_t *self,
                     int K, int32_t *out_idx, float *out_dist, int32_t *over, uint32_t *n_over) {
    const int KS = filt_ks(d), dp = 16 * KS;
    // 32 QB queries' fragments in at most 128 KB of LDS
    int QB = dp <= 256 ? 4 : dp <= 512 ? 2 : 1;
    while (QB > 1 && 16 * QB >= m) QB /= 2;
    // the sample: a query lists about K n / S points, with a relative spread of K^-1/2 (for a
    // small K a long tail), so 768 of them, or 256 for K < 8, overflow a list about once in 1e6.
    // The bounds of at least 32 queries have to fit, so 2^23 rows at most; past 2 048 points a
    // list (K n above 2^34) it would overflow too often to be of use.
    const int64_t aim = K < 8 ? 256 : 768, most = kFiltBounds / (4 * 32);
    int64_t S = std::max<int64_t>((K * n + aim - 1) / aim, 16384);
    int64_t stride = std::max<int64_t>(1, (n + S / 8) / std::min(S, n));
    while ((n + stride - 1) / stride > most) stride++;
    S = (n + stride - 1) / stride;
    if (K * n / S > 2048 && S < n) return false;
    const int64_t slab = std::min<int64_t>(n, std::max<int64_t>(32, (((int64_t)2 << 30) / (4 * dp)) & ~(int64_t)31));
    const int64_t rows = std::min<int64_t>(16384, kFiltBounds / (4 * S));
    const int64_t mq = std::min<int64_t>(m, rows >= 128 ? rows & ~(int64_t)127 : rows >= 64 ? 64 : 32);
    while (QB > 1 && 32 * QB > rows) QB /= 2;
    const int64_t qt = (mq + 32 * QB - 1) / (32 * QB) * QB;  // query tiles of 32, whole blocks
    struct { void *p; size_t bytes; } a[10] = {};
    enum { MU, SF, SN, PF, PN, QF, QN, PHI, CNT, CAND };
    void *sbuf = nullptr;
    auto frag = [&](int64_t tiles) { return (size_t)tiles * KS * 2048; };
    a[MU].bytes = 4 * (size_t)(dp + 64);
    a[SF].bytes = slab < n ? 0 : frag((S + 31) / 32);
    a[SN].bytes = 128 * (size_t)((S + 31) / 32);
    a[PF].bytes = frag((slab + 31) / 32);
    a[PN].bytes = 128 * (size_t)((slab + 31) / 32);
    a[QF].bytes = frag(qt);
    a[QN].bytes = 128 * (size_t)qt;
    a[PHI].bytes = 4 * (size_t)mq;
    a[CNT].bytes = 4 * (size_t)mq;
    a[CAND].bytes = 8 * (size_t)mq * kFiltCap;
    bool ok = (sbuf = cache_alloc((size_t)qt * 32 * S * 4, s)) != nullptr;
    for (auto &b : a) ok = ok && (!b.bytes || (b.p = cache_alloc(b.bytes, s)) != nullptr);
    if (ok) {
        const float E = 1.2e-5f + (3.0f * dp + 32) * 1.3e-7f + 3e-6f;
        auto F = [&](int k) { return static_cast<float *>(a[k].p); };
        auto B = [&](int k) { return static_cast<__bf16 *>(a[k].p); };
        uint32_t *cnt = static_cast<uint32_t *>(a[CNT].p);
        uint2 *cand = static_cast<uint2 *>(a[CAND].p);
        auto split = [&](const float *x, int64_t left, int64_t st, int64_t tiles, int f, float *nr) {
            hipLaunchKernelGGL(k_exact_split, dim3((unsigned)tiles), dim3(256), 0, s, x, left, d, st, F(MU), KS, B(f), nr);
            launch_check(s, "k_exact_split");
        };
        ProfScope ps(s, "exact_filter", 4.0 * n * d + 8.0 * m * K, 2.0 * m * n * d);
        hipLaunchKernelGGL(k_exact_centre, dim3((d + 63) / 64), dim3(1024), 0, s, X, n, d, std::max<int64_t>(1, n / 512), F(MU));
        launch_check(s, "k_exact_centre");
        if (slab >= n) {
            split(X, n, stride, (S + 31) / 32, SF, F(SN));
            split(X, n, 1, (n + 31) / 32, PF, F(PN));
        }
        const bool vec = d % 4 == 0 && (uintptr_t)X % 16 == 0 && (uintptr_t)Q % 16 == 0;
        for (int64_t q0 = 0; q0 < m; q0 += mq) {
            const int64_t nq = std::min(mq, m - q0);
            const int64_t *sc = self ? self + q0 : nullptr;
            split(Q + q0 * d, nq, 1, qt, QF, F(QN));
            for (int64_t s0 = 0; s0 < S; s0 += slab) {
                const int64_t ns = std::min(slab, S - s0);
                if (slab < n) split(X + s0 * stride * d, n - s0 * stride, stride, (ns + 31) / 32, PF, F(SN) + s0);
                launch_tile<0>(s, QB, d, nq, B(QF), F(QN), B(slab < n ? PF : SF), F(SN) + s0, ns, 0, E, nullptr, nullptr,
                               nullptr, static_cast<float *>(sbuf) + s0, S);
            }
            // a large sample, of which few queries' bounds are held at once, takes 1024 threads a query
            // (5 000 000 x 128, K 256: 8.5 -> 1.6 ms for 128 queries)
            // a list well above its aim costs more than it saves: above 5/3 of it by three standard
            // deviations of the probes, and twelve of them (of many points a few say little)
            const int probes = nq <= 512 ? 2048 : nq <= 1024 ? 1024 : 256;
            const double per = (double)probes * aim / n;
            const int probe_most = std::max(12, (int)(per * 5 / 3 + 3 * sqrt(per)));
            auto tau = [&](auto kern, int nt) {
                hipLaunchKernelGGL(kern, dim3((unsigned)nq), dim3(nt), 0, s, static_cast<float *>(sbuf), S, S, K, F(QN), E, sc,
                                   n, stride, F(SN), probes, probe_most, F(PHI), cnt);
            };
            if (S >= 65536) tau(k_exact_tau<1024>, 1024);
            else tau(k_exact_tau<256>, 256);
            launch_check(s, "k_exact_tau");
            for (int64_t p0 = 0; p0 < n; p0 += slab) {
                const int64_t np = std::min(slab, n - p0);
                if (slab < n) split(X + p0 * d, np, 1, (np + 31) / 32, PF, F(PN));
                launch_tile<1>(s, QB, d, nq, B(QF), F(QN), B(PF), F(PN), np, p0, E, F(PHI), cnt, cand, nullptr, 0);
            }
            auto rank = [&](auto kern) {
                hipLaunchKernelGGL(kern, dim3((unsigned)nq), dim3(256), 0, s, X, d, Q + q0 * d, sc, cnt, cand, K,
                                   out_idx + q0 * K, out_dist + q0 * K, (int32_t)q0, over, n_over);
            };
            if (vec) rank(k_exact_rank<true>);
            else rank(k_exact_rank<false>);
            launch_check(s, "k_exact_rank");
        }
    }
    if (sbuf) cache_free(sbuf, s);
    for (auto &b : a)
        if (b.p) cache_free(b.p, s);
    return ok;
}

}  // namespace
}  // namespace rpf

using namespace rpf;

extern "C" rpf_status rpf_exact_knn(const float *X, int64_t n, int32_t d, const float *Q, int64_t m,
                                    const int64_t *self, int32_t K, int32_t *out_idx, float *out_dist, void *stream) {
    if (n < 1 || n >= ((int64_t)1 << 31)) return fail(RPF_EINVAL, "rpf_exact_knn: n must be in [1, 2^31)");
    if (d < 1 || d > 2048) return fail(RPF_EINVAL, "rpf_exact_knn: d must be in [1, 2048]");
    if (m < 0) return fail(RPF_EINVAL, "rpf_exact_knn: m must be >= 0");
    if (K < 1 || K > 256) return fail(RPF_EINVAL, "rpf_exact_knn: K must be in [1, 256]");
    if (m == 0) return RPF_OK;
    if (!X || !Q || !out_idx || !out_dist) return fail(RPF_EINVAL, "rpf_exact_knn: NULL pointer");
    hipStream_t s = (hipStream_t)stream;
    {   // finite inputs only (one synchronisation)
        int32_t *flag = static_cast<int32_t *>(cache_alloc(16, s));
        if (!flag) return fail(RPF_ENOMEM, "rpf_exact_knn: allocation");
        fill_u32(flag, 4, 0, s);
        launch_nonfinite(s, X, n * d, flag);
        launch_nonfinite(s, Q, m * d, flag + 1);
        int32_t h[2] = {0, 0};
        hipMemcpyAsync(h, flag, 8, hipMemcpyDeviceToHost, s);
        cache_free(flag, s);
        const rpf_status st = check_hip(hipStreamSynchronize(s), "rpf_exact_knn input check");
        if (st != RPF_OK) return st;
        if (h[0] || h[1]) return fail(RPF_EINVAL, "rpf_exact_knn: X or Q holds NaN or Inf");
    }
    // queries of a distance block (a multiple of 8, LDS within 64 KiB), and per chunk: the
    // distance buffer stays within 4 GiB (at least eight queries)
    const int dq = (d + 31) & ~31;
    const int ql = std::max(8, std::min(kQL, 16384 / dq / 8 * 8));
    const size_t lds = (size_t)ql * dq * 4;
    // rows above 1 024 columns do not fit the filter's LDS
    int32_t *over = nullptr;
    if (m < ((int64_t)1 << 31) && d <= 1024 && (n >= 65536 || (m >= 128 && n * m >= 1000000)) && exhaustive_us(n, m, d) > 200) {
        over = static_cast<int32_t *>(cache_alloc((size_t)(m + 4) * 4, s));
        if (over) {
            fill_u32(reinterpret_cast<uint32_t *>(over), 4, 0, s);
            if (!filtered_search(s, X, n, d, Q, m, self, K, out_idx, out_dist, over + 4, reinterpret_cast<uint32_t *>(over))) {
                cache_free(over, s);
                over = nullptr;
            }
        }
    }
    int64_t chunk = ((int64_t)1 << 29) / n;
    chunk = std::min(m, chunk >= ql ? chunk / ql * ql : std::max<int64_t>(8, chunk & ~(int64_t)7));
    // (after the filter it is usually not read: the answer must not fail for it)
    double *Dbuf = static_cast<double *>(cache_alloc((size_t)chunk * n * 8, s));
    while (!Dbuf && over && chunk > 1) {
        chunk = (chunk + 1) / 2;
        Dbuf = static_cast<double *>(cache_alloc((size_t)chunk * n * 8, s));
    }
    if (!Dbuf) {
        if (over) cache_free(over, s);
        return fail(RPF_ENOMEM, "rpf_exact_knn: distance buffer allocation failed");
    }
    const bool vec = (d % 4) == 0 && ((uintptr_t)X % 16) == 0;
    const int nr = vec && d <= 256 ? (d + 31) / 32 : 0;
    for (int64_t q0 = 0; q0 < m; q0 += chunk) {
        const int64_t nq = std::min(chunk, m - q0);
        const unsigned gy = (unsigned)((nq + ql - 1) / ql);
        const unsigned gx = (unsigned)std::max<int64_t>(1, std::min<int64_t>((n + 31) / 32, std::max<int64_t>(1, (over ? 4096 : 16384) / gy)));
        // after the filter: the queries it left, by the device-side list (usually none)
        const ExactRows rows{over ? over + 4 : nullptr, reinterpret_cast<uint32_t *>(over), q0};
        {
            ProfScope ps(s, "exact_dist", (double)nq * n * 8 + (double)gy * n * d * 4, 2.0 * nq * n * d);
            const float *Qc = over ? Q : Q + q0 * d;
            const int64_t *sc = self && !over ? self + q0 : self;
            switch (nr) {
                case 1: hipLaunchKernelGGL(k_exact_dist<1>, dim3(gx, gy), dim3(256), lds, s, X, n, d, Qc, nq, rows, ql, sc, Dbuf, n); break;
                case 2: hipLaunchKernelGGL(k_exact_dist<2>, dim3(gx, gy), dim3(256), lds, s, X, n, d, Qc, nq, rows, ql, sc, Dbuf, n); break;
                case 3: hipLaunchKernelGGL(k_exact_dist<3>, dim3(gx, gy), dim3(256), lds, s, X, n, d, Qc, nq, rows, ql, sc, Dbuf, n); break;
                case 4: hipLaunchKernelGGL(k_exact_dist<4>, dim3(gx, gy), dim3(256), lds, s, X, n, d, Qc, nq, rows, ql, sc, Dbuf, n); break;
                case 5: hipLaunchKernelGGL(k_exact_dist<5>, dim3(gx, gy), dim3(256), lds, s, X, n, d, Qc, nq, rows, ql, sc, Dbuf, n); break;
                case 6: hipLaunchKernelGGL(k_exact_dist<6>, dim3(gx, gy), dim3(256), lds, s, X, n, d, Qc, nq, rows, ql, sc, Dbuf, n); break;
                case 7: hipLaunchKernelGGL(k_exact_dist<7>, dim3(gx, gy), dim3(256), lds, s, X, n, d, Qc, nq, rows, ql, sc, Dbuf, n); break;
                case 8: hipLaunchKernelGGL(k_exact_dist<8>, dim3(gx, gy), dim3(256), lds, s, X, n, d, Qc, nq, rows, ql, sc, Dbuf, n); break;
                default: hipLaunchKernelGGL(k_exact_dist<0>, dim3(gx, gy), dim3(256), lds, s, X, n, d, Qc, nq, rows, ql, sc, Dbuf, n); break;
            }
            launch_check(s, "k_exact_dist");
        }
        {
            ProfScope ps(s, "exact_select", (double)nq * n * 8 * 3, 0);
            hipLaunchKernelGGL(k_exact_select, dim3((unsigned)nq), dim3(kSelThreads), 0, s, Dbuf, n, n, rows, K,
                               over ? out_idx : out_idx + q0 * K, over ? out_dist : out_dist + q0 * K);
            launch_check(s, "k_exact_select");
        }
    }
    cache_free(Dbuf, s);
    if (over) cache_free(over, s);
    const std::string le = take_launch_error();
    if (!le.empty()) return fail(RPF_EDEVICE, "rpf_exact_knn: " + le);
    return RPF_OK;
}
