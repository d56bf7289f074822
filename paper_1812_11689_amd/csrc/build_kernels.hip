// Tree growth (Alg. 1 with the median split point of Sec. 2, direction choice of Alg. 2),
// level-synchronous over all trees: at level l every internal node of every tree is a
// contiguous segment of that tree's permutation, and one launch processes all of them
// (grid.y = tree).  Per node: project the members onto the node's direction (binary64,
// canonical order), select the member of rank floor(m/2) in (p, index) order, and
// partition stably so that both children stay in ascending original index.
//
// Two paths:
//   - segments of at most kLarge members: one workgroup per (segment, tree) does the whole
//     step in LDS (k_level_small);
//   - larger segments: chunked projection, a median select by one workgroup per segment
//     (the largest segments bracket the median from a sample first), then a stable chunked
//     partition.
#include <type_traits>

#include "rpf_internal.h"

namespace rpf {

// ================================================================ small segments: fused level

template <bool VEC>
__device__ inline void project_segment(const float *__restrict__ X, int d, const float *s_r,
                                       const int32_t *s_perm, int m, double *s_p) {
    const int g = threadIdx.x & 7, pt = threadIdx.x >> 3;
    const int per = blockDim.x >> 3;
    for (int base = 0; base < m; base += per) {
        int i = base + pt;
        int ii = i < m ? i : 0;
        double p = group8_dot64<VEC>(X + (int64_t)s_perm[ii] * d, s_r, d, g);
        if (g == 0 && i < m) s_p[i] = p;
    }
}

// ================================================================ grid rows: projections by digits
//
// Rows of a grid forest are integers k in [0, 255] (x = k / 255), so a projection is nearly
// s / 255 sum k q for a direction rounded to multiples q of s = max|r| / 2^22: three balanced
// base-256 digits of q, one column of v_mfma_i32_16x16x64_i8 each, exact in integers.  The
// node's median is taken from these keys; it is within e of the exact median and every key
// within e of its exact value (e: k_digit_bound), so once the members within 2 e of it hold
// their exact keys, a second selection and the partition give exactly what exact keys give:
// every other member is on its side of the exact median by more than its key's error.
// Binary64 needs a byte extraction, two conversions, a multiplication and three additions per
// coordinate for the three projections of a lead level and was bound by those (10^6 x 784, 48
// trees: 12.4 ms a lead level of multi-block nodes, 3.2 TB/s); the digits take 8.8 ms, bound by
// the gather of the rows (4.6 TB/s, their lines not aligned), and 4.0 ms at the first level,
// where the trees share the rows.  Only rows of 192 to 1024 coordinates: the directions' digits
// of rows below 126 outgrow the LDS held for exact directions, longer rows are not linked.

typedef int digits4 __attribute__((ext_vector_type(4)));
constexpr double kDigitRange = 4194304.0;  // 2^22

struct DigitDir {
    double scale;      // of the integer sums
    long long base;    // 128 sum q: the copy holds k - 128
};

// e per node: (d / 2 s + 2^-23 sum|r|), the rounding of r and that of x to binary32 (2^-24),
// the rest covering the binary64 sums
__global__ __launch_bounds__(256) void k_digit_bound(const float *__restrict__ R, int64_t nodes, int d,
                                                     double *__restrict__ bound) {
    const int lane = threadIdx.x & 63;
    for (int64_t k = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); k < nodes; k += (int64_t)gridDim.x * 4) {
        double mx = 0.0, sum = 0.0;
        for (int j = lane; j < d; j += 64) {
            const double v = fabs((double)R[k * d + j]);
            mx = fmax(mx, v);
            sum += v;
        }
        for (int o = 32; o > 0; o >>= 1) {
            mx = fmax(mx, shfl_xor_d(mx, o));
            sum += shfl_xor_d(sum, o);
        }
        if (lane == 0) bound[k] = 0.501 * d * (mx / kDigitRange) + sum * (1.0 / 8388608.0);
    }
}

// The digits of ND directions as matrix operands, s_b [dq / 64][64 lanes][16 bytes]: lane c +
// 16 g holds coordinates 16 g .. 16 g + 15 of column c; direction k's digit i is column k + 4 i.
template <int NT, int ND>
__device__ inline void digit_stage(const float *const (&dir)[ND], int d, int dq, int8_t *s_b, DigitDir *s_d,
                                   uint32_t *s_max) {
    const int tid = threadIdx.x;
    __syncthreads();
    for (int i = tid; i < dq; i += NT) reinterpret_cast<digits4 *>(s_b)[i] = digits4{0, 0, 0, 0};
    if (tid < ND) {
        s_max[tid] = 0;
        s_d[tid].base = 0;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < ND; k++) {
        float mx = 0.f;
        if (dir[k])
            for (int j = tid; j < d; j += NT) mx = fmaxf(mx, fabsf(dir[k][j]));
        for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o, 64));
        if ((tid & 63) == 0) atomicMax(&s_max[k], __float_as_uint(mx));
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < ND; k++) {
        const double mx = (double)__uint_as_float(s_max[k]);
        const double inv = mx > 0.0 ? kDigitRange / mx : 0.0;
        long long sum = 0;
        if (dir[k])
            for (int j = tid; j < d; j += NT) {
                const int q = (int)rint((double)dir[k][j] * inv);
                const int d0 = (int8_t)q, q1 = (q - d0) >> 8, d1 = (int8_t)q1, d2 = (q1 - d1) >> 8;
                int8_t *at = s_b + ((j >> 6) * 64 + 16 * ((j >> 4) & 3) + k) * 16 + (j & 15);
                at[0] = (int8_t)d0;
                at[4 * 16] = (int8_t)d1;
                at[8 * 16] = (int8_t)d2;
                sum += q;
            }
        for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
        if ((tid & 63) == 0) atomicAdd(reinterpret_cast<unsigned long long *>(&s_d[k].base), (unsigned long long)(128 * sum));
        if (tid == 0) s_d[k].scale = mx / (kDigitRange * 255.0);
    }
    __syncthreads();
}

// out(i, k, p) for each of the m rows id(i) and each direction k < ND, 32 rows per wave
template <int NT, int ND, typename Id, typename Out>
__device__ inline void digit_project(const int8_t *__restrict__ Xq, int dq, const int8_t *s_b, const DigitDir *s_d, int m,
                                     const Id &id, const Out &out) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, col = lane & 15, kg = lane >> 4;
    const int steps = dq >> 6;
    const digits4 *b = reinterpret_cast<const digits4 *>(s_b) + lane;
    for (int base = 32 * w; base < m; base += NT / 2) {
        const int ra = base + col, rb = ra + 16;
        const digits4 *xa = reinterpret_cast<const digits4 *>(Xq + (int64_t)id(ra < m ? ra : 0) * dq + 16 * kg);
        const digits4 *xb = reinterpret_cast<const digits4 *>(Xq + (int64_t)id(rb < m ? rb : 0) * dq + 16 * kg);
        digits4 acc[2] = {digits4{0, 0, 0, 0}, digits4{0, 0, 0, 0}};
        int ks = 0;
        for (; ks + 4 <= steps; ks += 4) {  // eight loads in flight
            digits4 a[4], c[4];
#pragma unroll
            for (int u = 0; u < 4; u++) {
                a[u] = xa[4 * (ks + u)];
                c[u] = xb[4 * (ks + u)];
            }
#pragma unroll
            for (int u = 0; u < 4; u++) {
                const digits4 q = b[64 * (ks + u)];
                acc[0] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[u], q, acc[0], 0, 0, 0);
                acc[1] = __builtin_amdgcn_mfma_i32_16x16x64_i8(c[u], q, acc[1], 0, 0, 0);
            }
        }
        for (; ks < steps; ks++) {
            const digits4 q = b[64 * ks];
            acc[0] = __builtin_amdgcn_mfma_i32_16x16x64_i8(xa[4 * ks], q, acc[0], 0, 0, 0);
            acc[1] = __builtin_amdgcn_mfma_i32_16x16x64_i8(xb[4 * ks], q, acc[1], 0, 0, 0);
        }
        // lane col + 16 kg holds rows 4 kg .. 4 kg + 3 of its column
#pragma unroll
        for (int h = 0; h < 2; h++) {
#pragma unroll
            for (int e = 0; e < 4; e++) {
                const int s1 = __shfl(acc[h][e], lane + 4, 64), s2 = __shfl(acc[h][e], lane + 8, 64);
                const int i = base + 16 * h + 4 * kg + e;
                if (col < ND && i < m) {
                    const long long v = (long long)s2 * 65536 + (long long)s1 * 256 + acc[h][e] + s_d[col].base;
                    out(i, col, (double)v * s_d[col].scale);
                }
            }
        }
    }
}

// Where an eighth of the members and more lie within the bound of their node's median (repeated
// rows, directions over constant columns), the digits decide little, and nearly every member is
// projected a second time.  Each pair of linked levels counts such members, and after a pair with
// that many the next ones project every member exactly from the start.
// 200 000 x 784, 8 trees, half of the rows blank: build 9.2 -> 6.3 ms (5.8 with every level exact;
// the difference is the first pair), directions of which one in twenty is zero 7.7 -> 4.0 (5.6).
__device__ inline bool band_exact(const DigitBand &b) { return b.prev && *b.prev > b.lim; }

// the members of a sample of the level's workgroups (a counter takes some 10 ns an addition)
__device__ inline void band_add(const DigitBand &b, uint32_t members) {
    const uint32_t nb = gridDim.x * gridDim.y, step = (nb >> 10) | 1, id = blockIdx.y * gridDim.x + blockIdx.x;
    if (id % step == 0) atomicAdd(b.cnt, (unsigned long long)members * step);
}

template <bool LEAD>
__global__ __launch_bounds__(256) void k_digit_chunks(const int8_t *__restrict__ Xq, int d, int dq,
                                                      const float *__restrict__ R, int64_t H,
                                                      const SegDesc *__restrict__ segs,
                                                      const ChunkDesc *__restrict__ chunks,
                                                      const int32_t *__restrict__ perm, int64_t n,
                                                      uint64_t *__restrict__ keys, const LookDesc *__restrict__ look,
                                                      double *__restrict__ ahead, int trees_first, DigitBand band) {
    constexpr int ND = LEAD ? 3 : 1;
    extern __shared__ __align__(16) int8_t s_digit[];  // [dq][16]
    __shared__ DigitDir s_d[3];
    __shared__ uint32_t s_max[3];
    const int t = trees_first ? blockIdx.x : blockIdx.y;
    const ChunkDesc c = chunks[trees_first ? blockIdx.y : blockIdx.x];
    const SegDesc sg = segs[c.seg];
    if (band_exact(band)) return;  // k_proj_chunks projects this level
    const float *dir[ND];
    dir[0] = R + ((int64_t)t * H + (sg.heap - 1)) * (int64_t)d;
    if constexpr (LEAD) {
        const LookDesc lk = look[c.seg];
#pragma unroll
        for (int b = 0; b < 2; b++)
            dir[b + 1] = lk.child_heap[b] > 0 ? R + ((int64_t)t * H + (lk.child_heap[b] - 1)) * (int64_t)d : nullptr;
    }
    digit_stage<256, ND>(dir, d, dq, s_digit, s_d, s_max);
    const int64_t at = (int64_t)t * n + c.start;
    const int32_t *pp = perm + at;
    digit_project<256, ND>(Xq, dq, s_digit, s_d, c.len, [&](int i) { return pp[i]; },
                           [&](int i, int k, double p) {
                               if (k == 0) keys[at + i] = key_of(p);
                               else ahead[2 * (at + i) + (k - 1)] = p;
                           });
}

// The exact keys of a chunk's members within 2 e of the first selection's median (where every key is
// exact: none).
template <bool VEC>
__global__ __launch_bounds__(256) void k_digit_refine(const int8_t *__restrict__ Xq, int d, int dq,
                                                      const float *__restrict__ R, int64_t H,
                                                      const SegDesc *__restrict__ segs,
                                                      const ChunkDesc *__restrict__ chunks,
                                                      const int32_t *__restrict__ perm, int64_t n,
                                                      uint64_t *__restrict__ keys, const SelState *__restrict__ state,
                                                      int nseg, const double *__restrict__ bound,
                                                      DigitBand band) {
    extern __shared__ __align__(16) float s_dirf[];  // [d up to a multiple of four]
    __shared__ uint16_t s_list[kChunk];
    __shared__ int s_cnt;
    const int t = blockIdx.y, tid = threadIdx.x;
    const ChunkDesc c = chunks[blockIdx.x];
    const SegDesc sg = segs[c.seg];
    const int64_t node = (int64_t)t * H + (sg.heap - 1), at = (int64_t)t * n + c.start;
    const double mid = val_of(state[(int64_t)t * nseg + c.seg].key), e2 = 2.001 * bound[node];
    if (e2 == 0.0 || band_exact(band)) return;  // (a bound of 0: a direction of zeros)
    if (tid == 0) s_cnt = 0;
    __syncthreads();
    for (int i = tid; i < c.len; i += 256)
        if (fabs(val_of(keys[at + i]) - mid) <= e2) s_list[atomicAdd(&s_cnt, 1)] = (uint16_t)i;
    __syncthreads();
    const int cnt = s_cnt;
    if (cnt == 0) return;
    if (tid == 0 && 8 * cnt > c.len) band_add(band, (uint32_t)cnt);
    for (int j = tid; j < d; j += 256) s_dirf[j] = R[node * d + j];
    __syncthreads();
    const int g = tid & 7;
    for (int k = tid >> 3; k < cnt; k += 32) {
        const int i = s_list[k];
        const double p = group8_dot64_q8<VEC>(Xq + (int64_t)perm[at + i] * dq, s_dirf, d, g);
        if (g == 0) keys[at + i] = key_of(p);
    }
}

// LDS layout: perm[m] int32 | key[m] u64 | dir[d] | hist[256] | misc ; nTry>1 adds p[m], tree[P2]
// Q8: the node projections read rows from the int8 grid copy Xq (stride dq): 1, the same values;
// 2, by digits, the members within 2 `bound` of the median then exactly
// NT: threads of a workgroup (n_try > 1: 256)
template <bool VEC, bool LEAD, int Q8 = 0, int NT = 256>
__global__ __launch_bounds__(NT) void k_level_small(
    const float *__restrict__ X, int d, const float *__restrict__ R, int64_t H, int n_try,
    const SegDesc *__restrict__ segs, const int32_t *__restrict__ perm_in,
    int32_t *__restrict__ perm_out, int64_t n, double *__restrict__ split,
    int32_t *__restrict__ split_idx, int32_t *__restrict__ chosen, int32_t *__restrict__ err,
    const LookDesc *__restrict__ look, double2 *__restrict__ ahead, uint64_t *__restrict__ keys_next,
    const uint64_t *__restrict__ keys_in, const int8_t *__restrict__ Xq, int dq, const double *__restrict__ bound,
    DigitBand band) {
    extern __shared__ __align__(16) uint8_t smem[];
    __shared__ uint32_t s_wide[NT == 256 ? 1 : NT / 64];
    __shared__ DigitDir s_d[3];
    __shared__ uint32_t s_max[3];
    const int t = blockIdx.y;
    const SegDesc sg = segs[blockIdx.x];
    const int m = sg.size;
    const int tid = threadIdx.x;
    const int ds = (d + 3) & ~3;
    int32_t *s_perm = reinterpret_cast<int32_t *>(smem);
    uint64_t *s_key = reinterpret_cast<uint64_t *>(smem + ((4 * m + 15) & ~15));
    // the node's direction (binary32); on a lead level it and its children's, as binary64
    uint8_t *s_dir = smem + ((((4 * m + 15) & ~15) + 8 * m + 15) & ~15);  // 16-byte aligned
    float *s_r = reinterpret_cast<float *>(s_dir);
    double *s_rd = reinterpret_cast<double *>(s_dir);
    uint32_t *s_hist = reinterpret_cast<uint32_t *>(s_rd + 3 * ds);
    uint32_t *s_misc = s_hist + 256;  // 16 words
    uint32_t *s_scan = NT == 256 ? s_misc : s_wide;
    double *s_p = reinterpret_cast<double *>(s_misc + 16);
    int P2 = 1;
    while (P2 < m) P2 <<= 1;
    double *s_tree = s_p + m;

    const int32_t *pin = perm_in + (int64_t)t * n + sg.off;
    for (int i = tid; i < m; i += blockDim.x) s_perm[i] = pin[i];
    const float *Rn = R + ((int64_t)t * H + (sg.heap - 1)) * n_try * (int64_t)d;

    int ch = 0;
    // Alg. 2: keep the try with the largest spread S2 (first wins ties).  Only builds whose memory
    // holds no tries' projections come here; the others score them in k_level_try or over many blocks.
    if (NT == 256 && n_try > 1) {
        double best = 0.0;
        int best_i = -1;
        for (int k = 0; k < n_try; k++) {
            __syncthreads();
            for (int j = tid; j < d; j += blockDim.x) s_r[j] = Rn[(int64_t)k * d + j];
            __syncthreads();
            project_segment<VEC>(X, d, s_r, s_perm, m, s_p);
            __syncthreads();
            for (int i = tid; i < m; i += blockDim.x) s_tree[i] = s_p[i];
            double s1 = block_canon_sum(s_tree, m);
            double mu = s1 / (double)m;
            for (int i = tid; i < m; i += blockDim.x) {
                double dev = s_p[i] - mu;
                s_tree[i] = __dmul_rn(dev, dev);
            }
            double s2 = block_canon_sum(s_tree, m);
            if (s2 > best) { best = s2; best_i = k; }
        }
        ch = best_i < 0 ? 0 : best_i;
    }
    __syncthreads();
    const bool exact = Q8 == 2 && band_exact(band);  // every member projected exactly
    if (Q8 == 2 && LEAD && exact && blockIdx.x == 0 && blockIdx.y == 0 && tid == 0) atomicAdd(band.cnt, band.all);
    if (keys_in) {  // fed level: the keys were made by the partition of the level above
        for (int i = tid; i < m; i += blockDim.x) s_key[i] = keys_in[(int64_t)t * n + sg.off + i];
    } else if (Q8 == 2 && !exact) {
        if constexpr (Q8 == 2) {
            constexpr int ND = LEAD ? 3 : 1;
            const float *dir[ND];
            dir[0] = Rn;
            if constexpr (LEAD) {
                const LookDesc lk = look[blockIdx.x];
#pragma unroll
                for (int b = 0; b < 2; b++)
                    dir[b + 1] = lk.child_heap[b] > 0 ? R + ((int64_t)t * H + (lk.child_heap[b] - 1)) * (int64_t)d : nullptr;
            }
            int8_t *s_b = reinterpret_cast<int8_t *>(s_dir);
            digit_stage<NT, ND>(dir, d, dq, s_b, s_d, s_max);
            double *ah = reinterpret_cast<double *>(ahead + ((int64_t)t * n + sg.off));
            digit_project<NT, ND>(Xq, dq, s_b, s_d, m, [&](int i) { return s_perm[i]; },
                                  [&](int i, int k, double p) {
                                      if (k == 0) s_key[i] = key_of(p);
                                      else ah[2 * i + (k - 1)] = p;
                                  });
        }
    } else if (LEAD) {  // lead level: the children's projections from the same read of X
        const LookDesc lk = look[blockIdx.x];
        for (int j = tid; j < d; j += blockDim.x) {
            s_rd[j] = Rn[j];
#pragma unroll
            for (int b = 0; b < 2; b++)  // a leaf child has no direction: project onto zero
                s_rd[ds * (b + 1) + j] =
                    lk.child_heap[b] > 0 ? R[((int64_t)t * H + (lk.child_heap[b] - 1)) * (int64_t)d + j] : 0.f;
        }
        __syncthreads();
        const int g = tid & 7, pt = tid >> 3;
        for (int base = 0; base < m; base += NT / 4) {
            const int ia = base + pt, ib = ia + NT / 8;
            double p[6];
            if constexpr (Q8 != 0)
                group8_dot64x3r2_q8<VEC>(Xq + (int64_t)s_perm[ia < m ? ia : 0] * dq, Xq + (int64_t)s_perm[ib < m ? ib : 0] * dq,
                                    s_rd, ds, d, g, p);
            else
                group8_dot64x3r2<VEC>(X + (int64_t)s_perm[ia < m ? ia : 0] * d, X + (int64_t)s_perm[ib < m ? ib : 0] * d,
                                      s_rd, ds, d, g, p);
#pragma unroll
            for (int h = 0; h < 2; h++) {
                const int i = h ? ib : ia;
                if (g == 0 && i < m) {
                    s_key[i] = key_of(p[3 * h]);
                    ahead[(int64_t)t * n + sg.off + i] = make_double2(p[3 * h + 1], p[3 * h + 2]);
                }
            }
        }
    } else {
        for (int j = tid; j < d; j += blockDim.x) s_r[j] = Rn[(int64_t)ch * d + j];
        __syncthreads();
        const int g = tid & 7, pt = tid >> 3;
        for (int base = 0; base < m; base += NT / 8) {
            int i = base + pt;
            int ii = i < m ? i : 0;
            double p;
            if constexpr (Q8 != 0) p = group8_dot64_q8<VEC>(Xq + (int64_t)s_perm[ii] * dq, s_r, d, g);
            else p = group8_dot64<VEC>(X + (int64_t)s_perm[ii] * d, s_r, d, g);
            if (g == 0 && i < m) s_key[i] = key_of(p);
        }
    }
    __syncthreads();

    // ---- select rank floor(m/2) in (key, index) order: 8-bit radix passes over the 96-bit key
    uint64_t phi = 0;
    uint32_t plo = 0;
    for (int pass = 0;; pass++) {
        phi = 0;
        plo = 0;
        int nbits = 0;
        uint32_t rank = (uint32_t)(m / 2), cnt = (uint32_t)m;
        while (cnt > 1 && nbits < 96) {
            const int lo_bit = 88 - nbits;
            const unsigned __int128 P = key96(phi, plo);
            if (tid < 256) s_hist[tid] = 0;
            __syncthreads();
            for (int i = tid; i < m; i += blockDim.x) {
                unsigned __int128 K = key96(s_key[i], (uint32_t)s_perm[i]);
                if (nbits == 0 || (K >> (96 - nbits)) == (P >> (96 - nbits)))
                    atomicAdd(&s_hist[(uint32_t)(K >> lo_bit) & 255u], 1u);
            }
            __syncthreads();
            uint32_t v = tid < 256 ? s_hist[tid] : 0u, excl, total;
            block_excl_scan_w<NT / 64>(v, s_scan, excl, total);
            if (excl <= rank && rank < excl + v) {
                s_misc[8] = tid;
                s_misc[9] = excl;
                s_misc[10] = v;
            }
            __syncthreads();
            const uint32_t b = s_misc[8];
            rank -= s_misc[9];
            cnt = s_misc[10];
            unsigned __int128 NP = P | ((unsigned __int128)b << lo_bit);
            phi = (uint64_t)(NP >> 32);
            plo = (uint32_t)NP;
            nbits += 8;
            __syncthreads();
        }
        if (nbits < 96) {  // exactly one key matches the prefix: it is the median
            const unsigned __int128 P = key96(phi, plo);
            for (int i = tid; i < m; i += blockDim.x) {
                unsigned __int128 K = key96(s_key[i], (uint32_t)s_perm[i]);
                if ((K >> (96 - nbits)) == (P >> (96 - nbits))) {
                    s_misc[12] = (uint32_t)s_key[i];
                    s_misc[13] = (uint32_t)(s_key[i] >> 32);
                    s_misc[14] = (uint32_t)s_perm[i];
                }
            }
            __syncthreads();
            phi = ((uint64_t)s_misc[13] << 32) | s_misc[12];
            plo = s_misc[14];
        }
        if (Q8 != 2 || pass || exact) break;
        // exact keys around the digits' median, then the selection over them
        const double mid = val_of(phi), e2 = 2.001 * bound[(int64_t)t * H + (sg.heap - 1)];
        if (e2 == 0.0) break;  // a direction of zeros
        __syncthreads();
        for (int j = tid; j < d; j += NT) s_r[j] = Rn[j];
        if (tid == 0) s_misc[15] = 0;
        __syncthreads();
        const int g = tid & 7;
        for (int i = tid >> 3; i < m; i += NT / 8) {
            if (!(fabs(val_of(s_key[i]) - mid) <= e2)) continue;  // (the same for a row's eight lanes)
            const double p = group8_dot64_q8<VEC>(Xq + (int64_t)s_perm[i] * dq, s_r, d, g);
            if (g == 0) {
                s_key[i] = key_of(p);
                if (atomicAdd(&s_misc[15], 1u) == 0) {
                    s_misc[12] = (uint32_t)s_key[i];
                    s_misc[13] = (uint32_t)(s_key[i] >> 32);
                }
            }
        }
        __syncthreads();
        if (tid == 0 && 8 * (int)s_misc[15] > m) band_add(band, s_misc[15]);
        if (s_misc[15] == 1) {  // alone: the median itself
            phi = ((uint64_t)s_misc[13] << 32) | s_misc[12];
            break;
        }
    }

    // ---- stable partition: left = keys below (c, c_idx), in position (= index) order
    const int half = m / 2;
    int32_t *pout = perm_out + (int64_t)t * n + sg.off;
    uint32_t lefts = 0;
    for (int base = 0; base < m; base += NT) {
        const int i = base + tid;
        const bool valid = i < m;
        const bool left = valid && key_less(s_key[i], (uint32_t)s_perm[i], phi, plo);
        uint32_t excl, total;
        block_excl_scan_w<NT / 64>(left ? 1u : 0u, s_scan, excl, total);
        if (valid) {
            uint32_t lb = lefts + excl;
            int pos = left ? (int)lb : half + (i - (int)lb);
            if (pos >= 0 && pos < m) {  // always true when the select is consistent
                pout[pos] = s_perm[i];
                if (LEAD) {  // the row's key at the next level: its projection onto its child
                    const double2 a = ahead[(int64_t)t * n + sg.off + i];
                    keys_next[(int64_t)t * n + sg.off + pos] = key_of(left ? a.x : a.y);
                }
            }
        }
        lefts += total;
    }
    if (tid == 0) {
        const int64_t hs = (int64_t)t * H + (sg.heap - 1);
        split[hs] = val_of(phi);
        split_idx[hs] = (int32_t)plo;
        if (chosen) chosen[hs] = ch;
        if (lefts != (uint32_t)half) atomicOr(err, 1);
    }
}


// Fed levels of small segments (at most 64 E members, one direction per node): one wave per
// (segment, tree), four segments per workgroup.  The wave holds the keys the lead level's
// partition made and the member ids in registers, E per lane (position i = lane + 64 e),
// selects the member of rank floor(m/2) in (key, index) order with 8-bit
// radix passes over a per-wave LDS histogram, and writes the stable partition: the same
// operations and result as k_level_small on a fed level, without workgroup barriers.
constexpr int kWaveSeg = 1024;  // largest segment of the wave-per-segment fed level

template <int E>
__global__ __launch_bounds__(256) void k_level_fed_wave(const SegDesc *__restrict__ segs, int nseg,
                                                        const int32_t *__restrict__ perm_in,
                                                        int32_t *__restrict__ perm_out, int64_t n, int64_t H,
                                                        double *__restrict__ split, int32_t *__restrict__ split_idx,
                                                        int32_t *__restrict__ chosen, int32_t *__restrict__ err,
                                                        const uint64_t *__restrict__ keys_in) {
    __shared__ uint32_t s_hist[4][256];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int k = blockIdx.x * 4 + w, t = blockIdx.y;
    if (k >= nseg) return;  // a whole wave; nothing below waits on the workgroup
    const SegDesc sg = segs[k];
    const int m = sg.size;
    const int32_t *pin = perm_in + (int64_t)t * n + sg.off;
    const uint64_t *kin = keys_in + (int64_t)t * n + sg.off;
    uint64_t kk[E];
    uint32_t id[E];
#pragma unroll
    for (int e = 0; e < E; e++) {
        const int i = lane + 64 * e;
        kk[e] = i < m ? kin[i] : 0;
        id[e] = i < m ? (uint32_t)pin[i] : 0u;
    }
    uint32_t *h = s_hist[w];
    uint64_t phi = 0;
    uint32_t plo = 0;
    int nbits = 0;
    uint32_t rank = (uint32_t)(m / 2), cnt = (uint32_t)m;
    while (cnt > 1 && nbits < 96) {
        const int lo_bit = 88 - nbits;
        const unsigned __int128 P = key96(phi, plo);
#pragma unroll
        for (int j = 0; j < 4; j++) h[lane + 64 * j] = 0;
        wave_sync();
#pragma unroll
        for (int e = 0; e < E; e++) {
            const int i = lane + 64 * e;
            const unsigned __int128 K = key96(kk[e], id[e]);
            if (i < m && (nbits == 0 || (K >> (96 - nbits)) == (P >> (96 - nbits))))
                atomicAdd(&h[(uint32_t)(K >> lo_bit) & 255u], 1u);
        }
        wave_sync();
        // lane l holds bins 4l .. 4l + 3; an inclusive scan of their sums over the lanes
        uint32_t v[4], sum = 0;
#pragma unroll
        for (int j = 0; j < 4; j++) {
            v[j] = h[4 * lane + j];
            sum += v[j];
        }
        uint32_t incl = sum;
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t y = __shfl_up(incl, o, 64);
            if (lane >= o) incl += y;
        }
        uint32_t run = incl - sum;  // members in the bins below this lane's
        int bsel = -1;
        uint32_t ex = 0, vc = 0;
#pragma unroll
        for (int j = 0; j < 4; j++) {
            if (bsel < 0 && run <= rank && rank < run + v[j]) {
                bsel = 4 * lane + j;
                ex = run;
                vc = v[j];
            }
            run += v[j];
        }
        const uint64_t own = __ballot(bsel >= 0);  // exactly one lane holds the rank
        const int src = own ? __builtin_ctzll(own) : 0;
        const uint32_t b = (uint32_t)__shfl(bsel, src, 64);
        rank -= (uint32_t)__shfl((int)ex, src, 64);
        cnt = (uint32_t)__shfl((int)vc, src, 64);
        const unsigned __int128 NP = P | ((unsigned __int128)b << lo_bit);
        phi = (uint64_t)(NP >> 32);
        plo = (uint32_t)NP;
        nbits += 8;
        wave_sync();  // every read of the histogram is done before the next pass clears it
    }
    if (nbits < 96) {  // exactly one key matches the prefix: it is the median
        const unsigned __int128 P = key96(phi, plo);
        uint64_t mh = 0;
        uint32_t ml = 0;
        bool found = false;
#pragma unroll
        for (int e = 0; e < E; e++) {
            const int i = lane + 64 * e;
            const unsigned __int128 K = key96(kk[e], id[e]);
            if (i < m && (K >> (96 - nbits)) == (P >> (96 - nbits))) {
                mh = kk[e];
                ml = id[e];
                found = true;
            }
        }
        const uint64_t own = __ballot(found);
        const int src = own ? __builtin_ctzll(own) : 0;
        phi = ((uint64_t)(uint32_t)__shfl((int)(uint32_t)(mh >> 32), src, 64) << 32) |
              (uint32_t)__shfl((int)(uint32_t)mh, src, 64);
        plo = (uint32_t)__shfl((int)ml, src, 64);
    }
    // stable partition: left = keys below (c, c_idx), in position (= index) order
    const int half = m / 2;
    int32_t *pout = perm_out + (int64_t)t * n + sg.off;
    uint32_t lefts = 0;
#pragma unroll
    for (int e = 0; e < E; e++) {
        const int i = lane + 64 * e;
        const bool valid = i < m;
        const bool left = valid && key_less(kk[e], id[e], phi, plo);
        const uint64_t mk = __ballot(left);
        if (valid) {
            const int lb = (int)lefts + mask_rank(mk);
            const int pos = left ? lb : half + (i - lb);
            if (pos >= 0 && pos < m) pout[pos] = (int32_t)id[e];
        }
        lefts += (uint32_t)__popcll(mk);
    }
    if (lane == 0) {
        const int64_t hs = (int64_t)t * H + (sg.heap - 1);
        split[hs] = val_of(phi);
        split_idx[hs] = (int32_t)plo;
        if (chosen) chosen[hs] = 0;
        if (lefts != (uint32_t)half) atomicOr(err, 1);
    }
}

// ================================================================ small subtrees: one persistent launch

// One internal node of a subtree, by the whole block (256 threads), nTry = 1: project the
// members s_perm[0 .. m) onto the node's direction r (binary64, canonical order), select the
// member of rank floor(m/2) in (p, index) order, and write the stable partition to s_out.
// The same operations, in the same order, as k_level_small on a one-direction level.
template <bool VEC>
__device__ inline void subtree_node(const float *__restrict__ X, int d, const float *__restrict__ r,
                                    const int32_t *s_perm, int32_t *s_out, int m, uint64_t *s_key, float *s_r,
                                    uint32_t *s_hist, uint32_t *s_misc, double *split_out, int32_t *split_idx_out,
                                    int32_t *chosen_out, int32_t *err) {
    const int tid = threadIdx.x;
    for (int j = tid; j < d; j += blockDim.x) s_r[j] = r[j];
    __syncthreads();
    {
        const int g = tid & 7, pt = tid >> 3;
        for (int base = 0; base < m; base += 32) {
            const int i = base + pt;
            const double p = group8_dot64<VEC>(X + (int64_t)s_perm[i < m ? i : 0] * d, s_r, d, g);
            if (g == 0 && i < m) s_key[i] = key_of(p);
        }
    }
    __syncthreads();
    uint64_t phi = 0;
    uint32_t plo = 0;
    int nbits = 0;
    uint32_t rank = (uint32_t)(m / 2), cnt = (uint32_t)m;
    while (cnt > 1 && nbits < 96) {
        const int lo_bit = 88 - nbits;
        const unsigned __int128 P = key96(phi, plo);
        s_hist[tid] = 0;
        __syncthreads();
        for (int i = tid; i < m; i += blockDim.x) {
            const unsigned __int128 K = key96(s_key[i], (uint32_t)s_perm[i]);
            if (nbits == 0 || (K >> (96 - nbits)) == (P >> (96 - nbits)))
                atomicAdd(&s_hist[(uint32_t)(K >> lo_bit) & 255u], 1u);
        }
        __syncthreads();
        const uint32_t v = s_hist[tid];
        uint32_t excl, total;
        block_excl_scan256(v, s_misc, excl, total);
        if (excl <= rank && rank < excl + v) {
            s_misc[8] = tid;
            s_misc[9] = excl;
            s_misc[10] = v;
        }
        __syncthreads();
        const uint32_t b = s_misc[8];
        rank -= s_misc[9];
        cnt = s_misc[10];
        const unsigned __int128 NP = P | ((unsigned __int128)b << lo_bit);
        phi = (uint64_t)(NP >> 32);
        plo = (uint32_t)NP;
        nbits += 8;
        __syncthreads();
    }
    if (nbits < 96) {  // exactly one key matches the prefix: it is the median
        const unsigned __int128 P = key96(phi, plo);
        for (int i = tid; i < m; i += blockDim.x) {
            const unsigned __int128 K = key96(s_key[i], (uint32_t)s_perm[i]);
            if ((K >> (96 - nbits)) == (P >> (96 - nbits))) {
                s_misc[12] = (uint32_t)s_key[i];
                s_misc[13] = (uint32_t)(s_key[i] >> 32);
                s_misc[14] = (uint32_t)s_perm[i];
            }
        }
        __syncthreads();
        phi = ((uint64_t)s_misc[13] << 32) | s_misc[12];
        plo = s_misc[14];
    }
    const int half = m / 2;
    uint32_t lefts = 0;
    for (int base = 0; base < m; base += 256) {
        const int i = base + tid;
        const bool valid = i < m;
        const bool left = valid && key_less(s_key[i], (uint32_t)s_perm[i], phi, plo);
        uint32_t excl, total;
        block_excl_scan256(left ? 1u : 0u, s_misc, excl, total);
        if (valid) {
            const uint32_t lb = lefts + excl;
            const int pos = left ? (int)lb : half + (i - (int)lb);
            if (pos >= 0 && pos < m) s_out[pos] = s_perm[i];  // always in range when the select is consistent
        }
        lefts += total;
    }
    if (tid == 0) {
        *split_out = val_of(phi);
        *split_idx_out = (int32_t)plo;
        *chosen_out = 0;
        if (lefts != (uint32_t)half) atomicOr(err, 1);
    }
    __syncthreads();
}

// Persistent launch over the small levels: a fixed grid of resident blocks takes items (tree,
// internal node of the first small level) from a device counter until none is left, and
// grows each item's whole subtree inside the block, level by level (a node's children only
// after its partition: the level dependencies stay inside the block).  The item's permutation
// segment stays in LDS (two buffers, one per level parity) and is written once, in leaf order,
// to perm_out.  Every block leaves the loop when the counter passes the item count.
template <bool VEC>
__global__ __launch_bounds__(256) void k_subtree(const float *__restrict__ X, int d, const float *__restrict__ R,
                                                 int64_t H, const SubItem *__restrict__ items, int nitems, int T,
                                                 int n0, const int32_t *__restrict__ perm_in,
                                                 int32_t *__restrict__ perm_out, int64_t n,
                                                 double *__restrict__ split, int32_t *__restrict__ split_idx,
                                                 int32_t *__restrict__ chosen, int32_t *__restrict__ err,
                                                 uint32_t *__restrict__ next, int max_m) {
    extern __shared__ __align__(16) uint8_t smem[];
    const int mp = (max_m + 3) & ~3;
    int32_t *s_pa = reinterpret_cast<int32_t *>(smem);
    int32_t *s_pb = s_pa + mp;
    uint64_t *s_key = reinterpret_cast<uint64_t *>(s_pb + mp);
    float *s_r = reinterpret_cast<float *>(s_key + mp);
    uint32_t *s_hist = reinterpret_cast<uint32_t *>(s_r + ((d + 3) & ~3));
    uint32_t *s_misc = s_hist + 256;  // 16 words; [15] = the block's current item
    const int tid = threadIdx.x;
    const uint32_t total = (uint32_t)nitems * (uint32_t)T;
    while (true) {
        if (tid == 0) s_misc[15] = atomicAdd(next, 1u);
        __syncthreads();
        const uint32_t w = s_misc[15];
        __syncthreads();
        if (w >= total) break;
        const int t = (int)(w / (uint32_t)nitems);
        const SubItem it = items[w % (uint32_t)nitems];
        const int m0 = it.size;
        int32_t *pa = s_pa, *pb = s_pb;
        const int32_t *pin = perm_in + (int64_t)t * n + it.off;
        for (int i = tid; i < m0; i += blockDim.x) pa[i] = pin[i];
        for (int k = 0; k < 31; k++) {  // relative depth k: nodes j = 0 .. 2^k - 1 of the subtree
            for (int i = tid; i < m0; i += blockDim.x) pb[i] = pa[i];  // leaves stay in place
            __syncthreads();
            bool any = false;
            for (int j = 0; j < (1 << k); j++) {
                int lo = 0, sz = m0;
                int64_t hl = it.heap - it.hbase;  // heap id within the data set
                bool present = true;
                for (int b = k - 1; b >= 0; b--) {  // walk down from the item: left = floor(m/2)
                    if (sz <= n0) {
                        present = false;
                        break;
                    }
                    const int left = sz / 2;
                    if ((j >> b) & 1) {
                        lo += left;
                        sz -= left;
                        hl = 2 * hl + 1;
                    } else {
                        sz = left;
                        hl = 2 * hl;
                    }
                }
                if (!present || sz <= n0) continue;
                any = true;
                const int64_t hs = (int64_t)t * H + (it.hbase + hl - 1);
                subtree_node<VEC>(X, d, R + hs * d, pa + lo, pb + lo, sz, s_key, s_r, s_hist, s_misc, split + hs,
                                  split_idx + hs, chosen + hs, err);
            }
            if (!any) break;
            int32_t *tmp = pa;
            pa = pb;
            pb = tmp;
        }
        __syncthreads();
        int32_t *pout = perm_out + (int64_t)t * n + it.off;
        for (int i = tid; i < m0; i += blockDim.x) pout[i] = pa[i];
        __syncthreads();
    }
}

size_t subtree_lds(int max_m, int d) {
    const size_t mp = (size_t)((max_m + 3) & ~3);
    return mp * 4 * 2 + mp * 8 + (size_t)((d + 3) & ~3) * 4 + 4 * (256 + 16);
}

void launch_subtree(hipStream_t s, bool vec, const float *X, int d, const float *R, int64_t H, const SubItem *items,
                    int nitems, int T, int n0, const int32_t *pin, int32_t *pout, int64_t n, double *split,
                    int32_t *split_idx, int32_t *chosen, int32_t *err, uint32_t *next, int max_m, int lds_limit) {
    if (nitems <= 0) return;
    const size_t lds = subtree_lds(max_m, d);
    int dev = 0, cus = 0;
    hipGetDevice(&dev);
    hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    const int per_cu = std::max(1, std::min(8, (int)((size_t)lds_limit / std::max<size_t>(lds, 1))));
    const int64_t total = (int64_t)nitems * T;
    const unsigned blocks = (unsigned)std::max<int64_t>(1, std::min<int64_t>(total, (int64_t)std::max(cus, 1) * per_cu));
    fill_u32(next, 1, 0, s);
    auto go = [&](auto kern) {
        hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        hipLaunchKernelGGL(kern, dim3(blocks), dim3(256), lds, s, X, d, R, H, items, nitems, T, n0, pin, pout, n, split,
                           split_idx, chosen, err, next, max_m);
    };
    if (vec) go(k_subtree<true>);
    else go(k_subtree<false>);
    launch_check(s, "k_subtree");
}

// ================================================================ large segments

// Q8: rows read from the int8 grid copy Xq (stride dq) instead of X; the same values
template <bool VEC, bool LEAD, bool Q8 = false, int NT = 256>
__global__ __launch_bounds__(NT) void k_proj_chunks(
    const float *__restrict__ X, int d, const float *__restrict__ R, int64_t H,
    const SegDesc *__restrict__ segs, const ChunkDesc *__restrict__ chunks,
    const int32_t *__restrict__ perm, int64_t n, uint64_t *__restrict__ keys,
    const LookDesc *__restrict__ look, double2 *__restrict__ ahead, const int8_t *__restrict__ Xq, int dq,
    DigitBand band) {
    if (Q8 && band.prev) {  // a level by digits (k_digit_chunks), but for a band of many members above it
        if (!band_exact(band)) return;
        if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) atomicAdd(band.cnt, band.all);
    }
    // the node's direction (binary32); on a lead level it and its children's, as binary64
    extern __shared__ __align__(16) uint8_t s_dir[];
    float *s_r = reinterpret_cast<float *>(s_dir);
    const int t = blockIdx.y;
    const ChunkDesc c = chunks[blockIdx.x];
    const SegDesc sg = segs[c.seg];
    const int tid = threadIdx.x;
    const float *Rn = R + ((int64_t)t * H + (sg.heap - 1)) * (int64_t)d;
    const int32_t *pp = perm + (int64_t)t * n;
    const int g = tid & 7, pt = tid >> 3;
    if (LEAD && d <= 1024) {  // lead level: the children's projections from the same read of X
        const LookDesc lk = look[c.seg];
        const int ds = (d + 3) & ~3;
        double *s_rd = reinterpret_cast<double *>(s_dir);
        for (int j = tid; j < d; j += NT) {
            s_rd[j] = Rn[j];
#pragma unroll
            for (int b = 0; b < 2; b++)  // a leaf child has no direction: project onto zero
                s_rd[ds * (b + 1) + j] =
                    lk.child_heap[b] > 0 ? R[((int64_t)t * H + (lk.child_heap[b] - 1)) * (int64_t)d + j] : 0.f;
        }
        __syncthreads();
        for (int base = 0; base < c.len; base += NT / 4) {
            const int ia = base + pt, ib = ia + NT / 8;
            const int64_t sa = c.start + (ia < c.len ? ia : 0), sb = c.start + (ib < c.len ? ib : 0);
            double p[6];
            if constexpr (Q8) group8_dot64x3r2_q8<VEC>(Xq + (int64_t)pp[sa] * dq, Xq + (int64_t)pp[sb] * dq, s_rd, ds, d, g, p);
            else group8_dot64x3r2<VEC>(X + (int64_t)pp[sa] * d, X + (int64_t)pp[sb] * d, s_rd, ds, d, g, p);
#pragma unroll
            for (int h = 0; h < 2; h++) {
                const int i = h ? ib : ia;
                const int64_t s = h ? sb : sa;
                if (g == 0 && i < c.len) {
                    keys[(int64_t)t * n + s] = key_of(p[3 * h]);
                    ahead[(int64_t)t * n + s] = make_double2(p[3 * h + 1], p[3 * h + 2]);
                }
            }
        }
    } else if (d <= 1024) {  // longer directions are read from global memory by the scalar loop below
        for (int j = tid; j < d; j += NT) s_r[j] = Rn[j];
        __syncthreads();
        for (int base = 0; base < c.len; base += NT / 8) {
            const int i = base + pt;
            const int64_t s = c.start + (i < c.len ? i : 0);
            double p;
            if constexpr (Q8) p = group8_dot64_q8<VEC>(Xq + (int64_t)pp[s] * dq, s_r, d, g);
            else p = group8_dot64<VEC>(X + (int64_t)pp[s] * d, s_r, d, g);
            if (g == 0 && i < c.len) keys[(int64_t)t * n + s] = key_of(p);
        }
    } else {
        for (int base = 0; base < c.len; base += NT / 8) {
            const int i = base + pt;
            const int64_t s = c.start + (i < c.len ? i : 0);
            double p;
            if constexpr (Q8) p = group8_dot64_q8<false>(Xq + (int64_t)pp[s] * dq, Rn, d, g);
            else p = group8_dot64<false>(X + (int64_t)pp[s] * d, Rn, d, g);
            if (g == 0 && i < c.len) keys[(int64_t)t * n + s] = key_of(p);
        }
    }
}

// ---- median of multi-block segments
//
// One workgroup per (segment, tree) finds the member of rank floor(m/2) in (key, index) order:
// histograms over 2 048 equal parts of the remaining range, each pass narrowing it to the part
// that holds the rank, the members held in registers and the survivors in LDS once 2 048 are left.  (Members
// ascend in index, so equal keys are ordered by position.)  Segments above kSelDirect first
// draw 2 048 evenly spaced keys and bracket the median between the sample's ranks 1 024 +- 120
// (over five standard deviations of a random sample's median); one multi-block pass counts the
// keys below the bracket and at its ends and lists those inside it (about 12%), and the workgroup
// reads only those; a bracket that misses costs it passes over the whole segment.  Bound: one
// read of the keys.  10^6 x 128, 72 trees: 24 launches a level (11-bit digits from the top of
// the key, most of them empty) took 0.54 ms a level, 4.3 ms a step; these take 2.9 ms.  (No
// device-scope fence in the pick: each writes back its XCD's whole L2, and cost 1.2 ms a level.)
constexpr int kSelDirect = 16384;  // members a workgroup keeps in registers, sixteen per thread
constexpr int kSelSample = 2048, kSelMargin = 120;
constexpr int kSelFewer = 65536, kSelSample2 = 512, kSelMargin2 = 60;  // segments below this: a cheaper sample
constexpr int kSelLds = 2048;

// S keys by S / 2 threads
template <int S>
__global__ __launch_bounds__(S / 2) void k_sel_sample(const SegDesc *__restrict__ segs, const uint64_t *__restrict__ keys,
                                                      int64_t n, int direct, SelState *__restrict__ state) {
    constexpr int kMargin = S == kSelSample ? kSelMargin : kSelMargin2;
    __shared__ uint64_t s_k[S];
    const int t = blockIdx.y, tid = threadIdx.x;
    const SegDesc sg = segs[blockIdx.x];
    SelState *st = state + (int64_t)t * gridDim.x + blockIdx.x;
    if (sg.size <= direct) {
        if (tid == 0) st->sampled = 0;
        return;
    }
    const uint64_t *kk = keys + (int64_t)t * n + sg.off;
#pragma unroll
    for (int e = 0; e < 2; e++) {
        const int i = tid + S / 2 * e;
        s_k[i] = kk[((int64_t)i * sg.size + sg.size / 2) / S];
    }
    __syncthreads();
    for (int size = 2; size <= S; size <<= 1)
        for (int stride = size >> 1; stride > 0; stride >>= 1) {
            const int lo = 2 * tid - (tid & (stride - 1)), hi = lo + stride;
            const uint64_t a = s_k[lo], b = s_k[hi];
            if ((a > b) == ((lo & size) == 0)) {
                s_k[lo] = b;
                s_k[hi] = a;
            }
            __syncthreads();
        }
    if (tid == 0) {
        const int a = S / 2 - kMargin, b = S / 2 + kMargin;
        st->lo = s_k[a];
        st->hi = s_k[b];
        // a bracket's key that the sample holds more than once: many members may share it
        st->ties = (s_k[a - 1] == s_k[a] || s_k[a] == s_k[a + 1] ? 1 : 0) |
                   (s_k[b - 1] == s_k[b] || s_k[b] == s_k[b + 1] ? 2 : 0);
        st->cnt = 0;
        st->sampled = 1;
    }
}

// What is kept of a bracketed segment, in its part of the permutation that the partition will
// write (4 m bytes): keys and positions of at most (m - 2) / 3 less the chunks' members inside the
// bracket, and before them, where many members share one of its keys, per chunk the members up to
// the lower key, below the upper key and up to it.
struct SelList {
    uint32_t *upto_lo, *below_hi, *upto_hi;  // [chunks]
    uint64_t *key;
    uint32_t *pos;
    uint32_t cap;
    __device__ SelList(int32_t *perm, int64_t at, int m) {
        const int nch = (m + kChunk - 1) / kChunk;
        upto_lo = reinterpret_cast<uint32_t *>(perm + at);
        below_hi = upto_lo + nch;
        upto_hi = below_hi + nch;
        cap = (uint32_t)(m - 2) / 3 - (uint32_t)nch;
        key = reinterpret_cast<uint64_t *>((reinterpret_cast<uintptr_t>(upto_hi + nch) + 7) & ~(uintptr_t)7);
        pos = reinterpret_cast<uint32_t *>(key + cap);
    }
};

// Members of a chunk below the bracket (lcount) and those inside it, listed.  Where many members
// share a key (repeated rows, few distinct values) the median is most often one of the bracket's
// two keys; members at such a key are counted, not listed.  (Listed, or read by the pick from the
// whole segment where they outgrow the list: 10^6 x 8, 4 trees, two thirds of the rows the same,
// 19.2 ms a build, with the counts 11.6, by 24 launches a level 12.6.)
__global__ __launch_bounds__(256) void k_sel_count(const SegDesc *__restrict__ segs, const ChunkDesc *__restrict__ chunks,
                                                   const uint64_t *__restrict__ keys, int64_t n,
                                                   SelState *__restrict__ state, int nseg, int32_t *__restrict__ list,
                                                   uint32_t *__restrict__ lcount) {
    __shared__ uint32_t s_w[16];
    __shared__ uint32_t s_at;
    const int t = blockIdx.y, tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const ChunkDesc c = chunks[blockIdx.x];
    SelState *st = state + (int64_t)t * nseg + c.seg;
    if (!st->sampled) return;
    const uint64_t lo = st->lo, hi = st->hi;
    const uint64_t *kk = keys + (int64_t)t * n + c.start;
    constexpr int E = kChunk / 256;
    const int ties = st->ties;
    // (keys are integers: a bracket's key that is listed widens the bracket by one)
    const uint64_t lo1 = ties & 1 ? lo : lo - 1, hi1 = ties & 2 ? hi : hi + 1;
    uint32_t below = 0, in = 0, at_hi = 0, at_lo = 0;  // per wave (uniform)
    uint64_t k[E], mine[E];
#pragma unroll
    for (int e = 0; e < E; e++) k[e] = kk[tid + 256 * e < c.len ? tid + 256 * e : 0];
#pragma unroll
    for (int e = 0; e < E; e++) {
        const bool ok = tid + 256 * e < c.len;
        const uint64_t up = __ballot(ok && k[e] <= lo1);
        below += (uint32_t)__popcll(up);
        mine[e] = __ballot(ok && k[e] > lo1 && k[e] < hi1);
        in += (uint32_t)__popcll(mine[e]);
        if (ties) {
            at_lo += (uint32_t)__popcll(up & __ballot(k[e] == lo));
            at_hi += (uint32_t)__popcll(__ballot(ok && k[e] <= hi) & ~up & ~mine[e]);
        }
    }
    if (lane == 0) {
        s_w[w] = in;
        s_w[4 + w] = below - at_lo;
        s_w[8 + w] = at_lo;
        s_w[12 + w] = at_hi;
    }
    __syncthreads();
    const SegDesc sg = segs[c.seg];
    const SelList out(list, (int64_t)t * n + sg.off, sg.size);
    const uint32_t rel = (uint32_t)(c.start - sg.off);
    if (tid == 0) {
        auto sum = [&](int k) { return s_w[k] + s_w[k + 1] + s_w[k + 2] + s_w[k + 3]; };
        const uint32_t tot = sum(0), low = sum(4);
        lcount[(int64_t)t * gridDim.x + blockIdx.x] = low;
        if (ties) {
            const uint32_t upto = low + sum(8), q = rel / kChunk;
            out.upto_lo[q] = upto;
            out.below_hi[q] = upto + tot;
            out.upto_hi[q] = upto + tot + sum(12);
        }
        s_at = tot ? (uint32_t)atomicAdd(&st->cnt, (int)tot) : 0u;
    }
    __syncthreads();
    uint32_t at = s_at;
    for (int q = 0; q < w; q++) at += s_w[q];
#pragma unroll
    for (int e = 0; e < E; e++) {
        const uint32_t slot = at + mask_rank(mine[e]);
        if ((mine[e] >> lane & 1) && slot < out.cap) {  // (a list that overflows is not used)
            out.key[slot] = k[e];
            out.pos[slot] = rel + tid + 256 * e;
        }
        at += (uint32_t)__popcll(mine[e]);
    }
}

__global__ __launch_bounds__(1024) void k_sel_pick(const SegDesc *__restrict__ segs, const uint64_t *__restrict__ keys,
                                                   const int32_t *__restrict__ perm, int64_t n,
                                                   SelState *__restrict__ state, int sampled,
                                                   int32_t *__restrict__ listmem, uint32_t *__restrict__ lcount,
                                                   int nchunk, int64_t H, double *__restrict__ split,
                                                   int32_t *__restrict__ split_idx, int32_t *__restrict__ chosen,
                                                   int32_t *__restrict__ err) {
    constexpr int kBins = 2048, kCnt = 1024;
    __shared__ uint32_t s_h[kBins];
    __shared__ uint64_t s_k[kSelLds];
    __shared__ uint32_t s_p[kSelLds];
    __shared__ uint32_t s_c[kCnt];  // left members per chunk, where the segment has at most kCnt
    __shared__ uint64_t s_fk[64];
    __shared__ uint32_t s_fp[64];
    __shared__ uint64_t s_mm[32];
    __shared__ uint32_t s_w[16];
    __shared__ uint32_t s_sel[4];
    const int t = blockIdx.y, tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const SegDesc sg = segs[blockIdx.x];
    SelState *stp = state + (int64_t)t * gridDim.x + blockIdx.x;
    const uint64_t *kk = keys + (int64_t)t * n + sg.off;
    uint32_t *lc = lcount + (int64_t)t * nchunk + sg.chunk0;
    const int m = sg.size, nch = sg.nchunk;
    uint32_t rank = (uint32_t)(m / 2), N = (uint32_t)m;
    const SelList list(listmem, (int64_t)t * n + sg.off, m);
    uint32_t listN = 0;
    bool listed = false;            // the rank is among the listed members
    const uint32_t *from = nullptr;  // tie: it is among the equal members between these two counts per chunk
    const uint32_t *upto = nullptr;
    const SelState st0 = *stp;
    uint64_t lo = st0.lo, hi = st0.hi;
    const bool counted = sampled && st0.sampled;
    const uint32_t *left0 = lc;     // listed: the chunks' members before the listed ones
    if (counted) {
        uint32_t b1;  // members before the listed ones
        if (st0.ties) {
            uint32_t v[4] = {0, 0, 0, 0};
            for (int q = tid; q < nch; q += 1024) {
                v[0] += lc[q];
                v[1] += list.upto_lo[q];
                v[2] += list.below_hi[q];
                v[3] += list.upto_hi[q];
            }
            if (tid < 4) s_sel[tid] = 0;
            __syncthreads();
#pragma unroll
            for (int k = 0; k < 4; k++) {
                for (int o = 32; o > 0; o >>= 1) v[k] += __shfl_xor(v[k], o, 64);
                if (lane == 0 && v[k]) atomicAdd(&s_sel[k], v[k]);
            }
            __syncthreads();
            const uint32_t b0 = s_sel[0], b2 = s_sel[2], b3 = s_sel[3];
            b1 = s_sel[1];
            __syncthreads();
            left0 = list.upto_lo;
            if (rank >= b0 && rank < b1) {
                from = lc;
                upto = list.upto_lo;
                rank -= b0;
            } else if (rank >= b2 && rank < b3) {
                from = list.below_hi;
                upto = list.upto_hi;
                rank -= b2;
                lo = hi;
            }
        } else {
            uint32_t b = 0;
            for (int q = tid; q < nch; q += 1024) b += lc[q];
            uint32_t excl;
            block_excl_scan_w<16>(b, s_w, excl, b1);
        }
        const uint32_t cnt = (uint32_t)st0.cnt;
        if (!from && rank >= b1 && rank < b1 + cnt && cnt <= list.cap) {
            listed = true;
            N = listN = cnt;
            rank -= b1;
        }
    }
    bool lds = false;  // the survivors are in s_k / s_p
    auto each = [&](auto &&f) {  // f(key, position) of every survivor, perhaps of others
        if (lds) {
            for (uint32_t i = tid; i < N; i += 1024) f(s_k[i], s_p[i]);
            return;
        }
        for (uint32_t i0 = tid; i0 < N; i0 += 8192) {  // eight loads in flight
            uint64_t k[8];
            uint32_t p[8];
#pragma unroll
            for (int u = 0; u < 8; u++) {
                const uint32_t i = i0 + 1024 * u < N ? i0 + 1024 * u : i0;
                p[u] = listed ? list.pos[i] : i;
                k[u] = listed ? list.key[i] : kk[i];
            }
#pragma unroll
            for (int u = 0; u < 8; u++)
                if (i0 + 1024 * u < N) f(k[u], p[u]);
        }
    };
    auto range = [&](auto &&in) {  // lo, hi: the smallest and the largest key that `in` takes
        uint64_t x = ~0ull, y = 0;
        each([&](uint64_t k, uint32_t p) {
            if (!in(k, p)) return;
            x = k < x ? k : x;
            y = k > y ? k : y;
        });
        for (int o = 32; o > 0; o >>= 1) {
            const uint64_t u = __shfl_xor(x, o, 64), v = __shfl_xor(y, o, 64);
            x = u < x ? u : x;
            y = v > y ? v : y;
        }
        if (lane == 0) {
            s_mm[w] = x;
            s_mm[16 + w] = y;
        }
        __syncthreads();
        lo = s_mm[0];
        hi = s_mm[16];
        for (int q = 1; q < 16; q++) {
            lo = s_mm[q] < lo ? s_mm[q] : lo;
            hi = s_mm[16 + q] > hi ? s_mm[16 + q] : hi;
        }
        __syncthreads();
    };
    auto pick_bin = [&]() {  // the part that holds the rank: s_sel = part, members before, members
        const uint32_t h0 = s_h[2 * tid], h1 = s_h[2 * tid + 1];
        uint32_t excl, total;
        block_excl_scan_w<16>(h0 + h1, s_w, excl, total);
        if (rank >= excl && rank < excl + h0 + h1) {
            const bool second = rank >= excl + h0;
            s_sel[0] = 2 * tid + (second ? 1 : 0);
            s_sel[1] = excl + (second ? h0 : 0);
            s_sel[2] = second ? h1 : h0;
        }
        __syncthreads();
    };
    // left members per chunk, for the partition: so far those before the listed ones
    const bool few = nch <= kCnt;
    // the median (key, position): the partition's counts, made a running sum, and the node's split
    auto finish = [&](uint64_t ck, uint32_t cp) {
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        uint32_t run = 0;
        for (int base = 0; base < nch; base += 1024) {
            const int q = base + tid;
            const uint32_t v = q < nch ? (few ? s_c[q] : __hip_atomic_load(&lc[q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) : 0u;
            uint32_t excl, total;
            block_excl_scan_w<16>(v, s_w, excl, total);
            if (q < nch) lc[q] = run + excl;
            run += total;
        }
        if (tid == 0) {
            const int64_t hs = (int64_t)t * H + (sg.heap - 1);
            stp->key = ck;
            stp->idx = perm[(int64_t)t * n + sg.off + cp];
            split[hs] = val_of(ck);
            split_idx[hs] = stp->idx;
            if (chosen) chosen[hs] = 0;  // one direction per node (else Alg. 2's pick stands already)
            if (run != (uint32_t)(m / 2)) atomicOr(err, 16);
        }
    };
    if (from) {  // the median is member `rank` of those equal to lo, in order of position
        uint32_t run = 0;
        for (int base = 0; base < nch; base += 1024) {  // its chunk, and its rank there
            const int q = base + tid;
            const uint32_t v = q < nch ? upto[q] - from[q] : 0u;
            uint32_t excl, total;
            block_excl_scan_w<16>(v, s_w, excl, total);
            if (rank >= run + excl && rank < run + excl + v) {
                s_sel[0] = (uint32_t)q;
                s_sel[1] = rank - run - excl;
            }
            run += total;
        }
        __syncthreads();
        const uint32_t mc = s_sel[0], mr = s_sel[1];
        run = 0;
        for (int i = (int)mc * kChunk + tid, e = 0; e < kChunk; e += 1024, i += 1024) {
            const bool same = i < m && kk[i] == lo;
            uint32_t excl, total;
            block_excl_scan_w<16>(same ? 1u : 0u, s_w, excl, total);
            if (same && run + excl == mr) s_sel[2] = (uint32_t)i;
            run += total;
        }
        for (int q = tid; q < nch; q += 1024) {
            const uint32_t v = q < (int)mc ? upto[q] : from[q] + (q == (int)mc ? mr : 0u);
            if (few) s_c[q] = v;
            else lc[q] = v;
        }
        __syncthreads();
        finish(lo, s_sel[2]);
        return;
    }
    if (few)
        for (int q = tid; q < nch; q += 1024) s_c[q] = listed ? left0[q] : 0u;
    else
        for (int q = tid; q < nch; q += 1024) lc[q] = listed ? left0[q] : 0u;
    __builtin_amdgcn_s_waitcnt(0);  // (the counters in memory: one workgroup's, so no fence is needed)
    __syncthreads();
    auto add = [&](int q, uint32_t v) { atomicAdd(few ? &s_c[q] : &lc[q], v); };
    // The usual case: one histogram over the value range, the members of the rank's part
    // straight to LDS, those of the parts before it counted as left.  Up to sixteen members per
    // thread stay in registers; a longer list (its range is the bracket) is read twice.
    constexpr int E = kSelDirect / 1024;
    const bool reg = N <= (uint32_t)kSelDirect;
    bool fast = reg || listed;
    if (fast) {
        uint64_t rk[E];
        uint32_t bn[E];
        double mn = INFINITY, mx = -INFINITY;
        bool nan = false;
        if (reg) {
#pragma unroll
            for (int e = 0; e < E; e++) {
                if (1024u * e >= N) continue;
                const uint32_t i = tid + 1024u * e < N ? tid + 1024 * e : 0;
                rk[e] = listed ? list.key[i] : kk[i];
            }
#pragma unroll
            for (int e = 0; e < E; e++) {
                if (1024u * e >= N) continue;
                const double v = val_of(rk[e]);
                mn = fmin(mn, v);
                mx = fmax(mx, v);
                nan |= v != v;
            }
            for (int o = 32; o > 0; o >>= 1) {
                mn = fmin(mn, shfl_xor_d(mn, o));
                mx = fmax(mx, shfl_xor_d(mx, o));
            }
            // A plan checks its inputs after the launch, so a key may be a NaN, whose place in the
            // order of the keys its value does not tell: one part for all, and the passes below,
            // which go by the keys.  (By value it counted as left here and as right in the
            // partition, which left a slot of the permutation unwritten.)
            if (__any(nan)) {
                mn = -INFINITY;
                mx = INFINITY;
            }
        } else {
            mn = val_of(lo);
            mx = val_of(hi);
        }
        double *s_v = reinterpret_cast<double *>(s_mm);
        if (lane == 0) {
            s_v[w] = mn;
            s_v[16 + w] = mx;
        }
        for (int i = tid; i < kBins; i += 1024) s_h[i] = 0;
        if (tid == 0) s_sel[3] = 0;
        __syncthreads();
        for (int q = 0; q < 16; q++) {
            mn = fmin(mn, s_v[q]);
            mx = fmax(mx, s_v[16 + q]);
        }
        const double scale = (double)(kBins - 1) / (mx - mn);
        auto bin = [&](uint64_t k) -> uint32_t {
            const double x = (val_of(k) - mn) * scale;  // (no number: a range of one value, or one that overflows)
            return x > 0.0 ? (x < kBins - 1 ? (uint32_t)x : kBins - 1) : 0u;
        };
        if (reg) {
#pragma unroll
            for (int e = 0; e < E; e++) {
                if (1024u * e >= N) continue;
                bn[e] = bin(rk[e]);
                if (tid + 1024u * e < N) atomicAdd(&s_h[bn[e]], 1u);
            }
        } else {
            each([&](uint64_t k, uint32_t) { atomicAdd(&s_h[bin(k)], 1u); });
        }
        __syncthreads();
        pick_bin();
        fast = s_sel[2] <= (uint32_t)kSelLds;
        if (fast) {
            const uint32_t fb = s_sel[0];
            rank -= s_sel[1];
            auto keep = [&](uint64_t k, uint32_t p) {
                const uint32_t at = atomicAdd(&s_sel[3], 1u);
                s_k[at] = k;
                s_p[at] = p;
            };
            if (reg) {
#pragma unroll
                for (int e = 0; e < E; e++) {
                    if (1024u * e >= N) continue;
                    const uint32_t i = tid + 1024 * e;
                    if (i < N && bn[e] == fb) keep(rk[e], listed ? list.pos[i] : i);
                    if (listed) {
                        if (i < N && bn[e] < fb) add((int)(list.pos[i] / kChunk), 1u);
                    } else {  // 1 024 members, of one chunk
                        const uint64_t mask = __ballot(i < N && bn[e] < fb);
                        if (lane == 0 && mask) add(1024 * e / kChunk, (uint32_t)__popcll(mask));
                    }
                }
            } else {
                each([&](uint64_t k, uint32_t p) {
                    const uint32_t b = bin(k);
                    if (b == fb) keep(k, p);
                    else if (b < fb) add((int)(p / kChunk), 1u);
                });
            }
            lds = true;
            N = s_sel[2];
        }
        __syncthreads();
    }
    if (lds ? N > 64 : !listed) range([](uint64_t, uint32_t) { return true; });
    else if (lds) {
        lo = 0;
        hi = ~0ull;
    }
    uint32_t left = N;
    uint64_t plo = 0, phi = (uint64_t)m - 1;  // range of positions (narrowed among equal keys)
    auto inside = [&](uint64_t k, uint32_t p) { return k >= lo && k <= hi && p >= plo && p <= phi; };
    bool by_value = true;
    while (left > 64 && (lo < hi || plo < phi)) {
        // 2 048 parts of the range: of the values (their density is smooth), of the bit patterns
        // where values do not separate the keys, or of the positions of equal keys.  All three
        // are monotone in the order, and the last two always shrink the range.
        const int how = lo == hi ? 2 : by_value ? 0 : 1;
        const double v0 = val_of(lo), scale = (double)(kBins - 1) / (val_of(hi) - v0);
        const uint64_t a = how == 2 ? plo : lo, width = (how == 2 ? phi : hi) - a;
        const int sh = width < kBins ? 0 : 53 - __clzll((long long)width);
        auto bin_of = [&](uint64_t k, uint32_t p) -> uint32_t {
            if (how == 0) {
                const double x = (val_of(k) - v0) * scale;  // (inf or NaN: a range that overflows)
                return x > 0.0 ? (x < kBins - 1 ? (uint32_t)x : kBins - 1) : 0u;
            }
            return (uint32_t)(((how == 2 ? (uint64_t)p : k) - a) >> sh);
        };
        for (int i = tid; i < kBins; i += 1024) s_h[i] = 0;
        __syncthreads();
        each([&](uint64_t k, uint32_t p) {
            if (inside(k, p)) atomicAdd(&s_h[bin_of(k, p)], 1u);
        });
        __syncthreads();
        pick_bin();
        const uint32_t b = s_sel[0], was = left;
        rank -= s_sel[1];
        left = s_sel[2];
        if (how == 0) {
            const uint64_t l0 = lo, h0_ = hi;
            range([&](uint64_t k, uint32_t p) { return k >= l0 && k <= h0_ && bin_of(k, p) == b; });
            by_value = 2 * left < was;
        } else {
            // the part's last key or position, or the range's (past an infinity or a NaN the part's
            // last key could lie beyond 64 bits)
            const uint64_t na = a + ((uint64_t)b << sh), span = ((uint64_t)1 << sh) - 1;
            if (how == 2) {
                phi = phi - na > span ? na + span : phi;
                plo = na;
            } else {
                hi = hi - na > span ? na + span : hi;
                lo = na;
                by_value = true;
            }
            __syncthreads();
        }
        if (!lds && left <= (uint32_t)kSelLds && left > 64) {
            if (tid == 0) s_sel[3] = 0;
            __syncthreads();
            each([&](uint64_t k, uint32_t p) {
                if (inside(k, p)) {
                    const uint32_t at = atomicAdd(&s_sel[3], 1u);
                    s_k[at] = k;
                    s_p[at] = p;
                }
            });
            __syncthreads();
            lds = true;
            N = left;
        }
    }
    if (tid == 0) s_sel[3] = 0;
    __syncthreads();
    each([&](uint64_t k, uint32_t p) {
        if (inside(k, p)) {
            const uint32_t at = atomicAdd(&s_sel[3], 1u);
            s_fk[at & 63] = k;
            s_fp[at & 63] = p;
        }
    });
    __syncthreads();
    const uint32_t fin = s_sel[3];
    if (fin > 64 || rank >= fin) {  // never: the counts above are consistent
        if (tid == 0) atomicOr(err, 2);
        return;
    }
    if (tid < 64 && (uint32_t)tid < fin) {
        uint32_t r = 0;
        for (uint32_t q = 0; q < fin; q++)
            r += s_fk[q] < s_fk[tid] || (s_fk[q] == s_fk[tid] && s_fp[q] < s_fp[tid]) ? 1u : 0u;
        if (r == rank) {
            s_mm[0] = s_fk[tid];
            s_sel[0] = s_fp[tid];
        }
    }
    __syncthreads();
    const uint64_t ck = s_mm[0];
    const uint32_t cp = s_sel[0];
    // the left members not yet counted: those before the median in its part, or all of them
    auto is_left = [&](uint64_t k, uint32_t p) { return k < ck || (k == ck && p < cp); };
    if (fast || listed) {
        lds = fast;
        N = fast ? N : listN;
        each([&](uint64_t k, uint32_t p) {
            if (is_left(k, p)) add((int)(p / kChunk), 1u);
        });
    } else {
        for (int base = 0; base < m; base += 1024) {
            const int i = base + tid;
            const uint64_t mask = __ballot(i < m && is_left(kk[i < m ? i : 0], (uint32_t)i));
            if (lane == 0 && mask) add(base / kChunk, (uint32_t)__popcll(mask));
        }
    }
    finish(ck, cp);
}

template <int NT>
__global__ __launch_bounds__(NT) void k_part_scatter(const SegDesc *__restrict__ segs,
                                                      const ChunkDesc *__restrict__ chunks, int nchunk,
                                                      const uint64_t *__restrict__ keys,
                                                      const int32_t *__restrict__ perm_in,
                                                      int32_t *__restrict__ perm_out, int64_t n,
                                                      const SelState *__restrict__ state, int nseg,
                                                      const uint32_t *__restrict__ lbase,
                                                      const LookDesc *__restrict__ look,
                                                      const double2 *__restrict__ ahead,
                                                      uint64_t *__restrict__ keys_next) {
    __shared__ uint32_t s_w[16];
    const int t = blockIdx.y, tid = threadIdx.x;
    const ChunkDesc c = chunks[blockIdx.x];
    const SegDesc sg = segs[c.seg];
    const SelState st = state[(int64_t)t * nseg + c.seg];
    const int64_t half = sg.size / 2;
    uint32_t lefts = lbase[(int64_t)t * nchunk + blockIdx.x];
    const int64_t rel0 = c.start - sg.off;  // chunk position within the segment
    int32_t *pout = perm_out + (int64_t)t * n + sg.off;
    const bool lead = look != nullptr;
    for (int base = 0; base < c.len; base += NT) {
        const int i = base + tid;
        const bool valid = i < c.len;
        const int64_t s = c.start + (valid ? i : 0);
        const int32_t id = perm_in[(int64_t)t * n + s];
        const bool left = valid && key_less(keys[(int64_t)t * n + s], (uint32_t)id, st.key, (uint32_t)st.idx);
        uint32_t excl, total;
        block_excl_scan_w<NT / 64>(left ? 1u : 0u, s_w, excl, total);
        if (valid) {
            const int64_t lb = (int64_t)lefts + excl;
            const int64_t rel = rel0 + i;
            const int64_t pos = left ? lb : half + (rel - lb);
            if (pos >= 0 && pos < sg.size) {  // always true when the select is consistent
                pout[pos] = id;
                if (lead) {  // the row's key at the next level: its projection onto its child
                    const double2 a = ahead[(int64_t)t * n + s];
                    keys_next[(int64_t)t * n + sg.off + pos] = key_of(left ? a.x : a.y);
                }
            }
        }
        lefts += total;
    }
}

// Lead projections of the first level for every tree from one read of X.  At the roots the
// permutation is the identity in every tree, so the rows of a chunk are the same rows for
// all trees: a block keeps 64 of them in registers (eight lanes per row, two rows per group,
// d <= 128 and d % 4 == 0) and walks the trees, staging each tree's three directions (node
// and children, as binary64) in LDS, double-buffered.  Each projection is computed exactly
// as group8_dot64 computes it.  Writes the keys and the children's projections; the
// first-digit histograms come from a selection pass over the keys.
__global__ __launch_bounds__(256) void k_proj_root(const float *__restrict__ X, int d, const float *__restrict__ R,
                                                   int64_t H, int ntree, const SegDesc *__restrict__ segs,
                                                   const ChunkDesc *__restrict__ chunks,
                                                   const LookDesc *__restrict__ look, int64_t n,
                                                   uint64_t *__restrict__ keys, double2 *__restrict__ ahead) {
    constexpr int NJ = 4;                   // float4 steps per lane: d <= 128
    __shared__ __align__(16) double s_rd[2][3 * 128];
    const ChunkDesc c = chunks[blockIdx.x];
    const int sub0 = 64 * blockIdx.y;
    if (sub0 >= c.len) return;
    const SegDesc sg = segs[c.seg];
    const LookDesc lk = look[c.seg];
    const int tid = threadIdx.x, g = tid & 7, pt = tid >> 3;
    const int ia = sub0 + pt, ib = ia + 32;  // rows within the chunk
    const bool oka = ia < c.len, okb = ib < c.len;
    const float *xa = X + (c.start + (oka ? ia : 0)) * (int64_t)d;
    const float *xb = X + (c.start + (okb ? ib : 0)) * (int64_t)d;
    float4 ra[NJ], rb[NJ];
#pragma unroll
    for (int k = 0; k < NJ; k++) {
        const int j = 4 * g + 32 * k;
        ra[k] = j < d ? *reinterpret_cast<const float4 *>(xa + j) : make_float4(0.f, 0.f, 0.f, 0.f);
        rb[k] = j < d ? *reinterpret_cast<const float4 *>(xb + j) : make_float4(0.f, 0.f, 0.f, 0.f);
    }
    // a tree's three directions (node, left child, right child; zero for a leaf child): thread
    // tid holds elements tid and tid + 256.  The loads for tree t + 2 are issued while tree t
    // is projected, and stored to LDS after it, so their latency is hidden.
    float nv[2];
    auto fetch = [&](int t) {
#pragma unroll
        for (int e = 0; e < 2; e++) {
            const int j = tid + 256 * e, k = j >> 7, jj = j & 127;
            float v = 0.f;
            if (j < 3 * 128 && jj < d) {
                const int heap = k == 0 ? sg.heap : k == 1 ? lk.child_heap[0] : lk.child_heap[1];
                if (heap > 0) v = R[((int64_t)t * H + (heap - 1)) * (int64_t)d + jj];
            }
            nv[e] = v;
        }
    };
    auto put = [&](double *dst) {
#pragma unroll
        for (int e = 0; e < 2; e++)
            if (tid + 256 * e < 3 * 128) dst[tid + 256 * e] = nv[e];
    };
    fetch(0);
    put(s_rd[0]);
    if (ntree > 1) fetch(1);
    for (int t = 0; t < ntree; t++) {
        __syncthreads();  // s_rd[t & 1] is staged; everyone is done with s_rd[(t + 1) & 1]
        const double *r = s_rd[t & 1];
        double s[6][4];
#pragma unroll
        for (int q = 0; q < 6; q++) s[q][0] = s[q][1] = s[q][2] = s[q][3] = 0.0;
#pragma unroll
        for (int k = 0; k < NJ; k++) {
            const int j = 4 * g + 32 * k;
            if (j < d) {
                const double a0 = ra[k].x, a1 = ra[k].y, a2 = ra[k].z, a3 = ra[k].w;
                const double b0 = rb[k].x, b1 = rb[k].y, b2 = rb[k].z, b3 = rb[k].w;
#pragma unroll
                for (int q = 0; q < 3; q++) {
                    const double2 u = *reinterpret_cast<const double2 *>(r + 128 * q + j);
                    const double2 v = *reinterpret_cast<const double2 *>(r + 128 * q + j + 2);
                    s[q][0] = __builtin_fma(a0, u.x, s[q][0]);
                    s[q][1] = __builtin_fma(a1, u.y, s[q][1]);
                    s[q][2] = __builtin_fma(a2, v.x, s[q][2]);
                    s[q][3] = __builtin_fma(a3, v.y, s[q][3]);
                    s[q + 3][0] = __builtin_fma(b0, u.x, s[q + 3][0]);
                    s[q + 3][1] = __builtin_fma(b1, u.y, s[q + 3][1]);
                    s[q + 3][2] = __builtin_fma(b2, v.x, s[q + 3][2]);
                    s[q + 3][3] = __builtin_fma(b3, v.y, s[q + 3][3]);
                }
            }
        }
        double p[6];
#pragma unroll
        for (int q = 0; q < 6; q++) {
            double w = (s[q][0] + s[q][1]) + (s[q][2] + s[q][3]);
            w = group8_add(w);
            p[q] = w + 0.0;
        }
        if (g == 0) {
            const int64_t base = (int64_t)t * n + c.start;
            if (oka) {
                keys[base + ia] = key_of(p[0]);
                ahead[base + ia] = make_double2(p[1], p[2]);
            }
            if (okb) {
                keys[base + ib] = key_of(p[3]);
                ahead[base + ib] = make_double2(p[4], p[5]);
            }
        }
        if (t + 1 < ntree) {  // tree t + 1's directions (loaded during this tree), then t + 2's loads
            put(s_rd[(t + 1) & 1]);
            if (t + 2 < ntree) fetch(t + 2);
        }
    }
}

// ================================================================ several tries per node (Alg. 2)
//
// Every try's projections are made from one read of each row (NT tries at a time), in
// canonical order, and its two canonical sums (of p, then of (p - mean)^2) are pairwise
// trees over the members in position order.  Bound: binary64 arithmetic (d fma per member and
// try); before, each try re-read the rows and each level summed through LDS with a workgroup
// barrier per tree level.
//   - k_level_try: nodes of at most try_cap members, one workgroup per (node, tree): the
//     projections of all tries stay in LDS, one wave sums one try, and the whole step
//     (pick, median, partition) ends in the same workgroup.
//   - larger nodes: k_try_proj / k_try_mean / k_try_dev / k_try_pick / k_try_keys over pieces
//     of 256 members, which are aligned subtrees of the sums; then the level's selection runs
//     from the chosen try's keys as on a fed level.

// directions tr .. tr + cnt - 1 of a node (zero past n_try and past d)
__device__ inline void stage_tries(const float *__restrict__ Rn, int tr, int cnt, int n_try, int d, int ds, float *s_rd) {
    for (int k = 0; k < cnt; k++)
        for (int j = threadIdx.x; j < ds; j += blockDim.x)
            s_rd[k * ds + j] = tr + k < n_try && j < d ? Rn[(int64_t)(tr + k) * d + j] : 0.f;
}

template <bool VEC, int NT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void k_level_try(const float *__restrict__ X, int d, const float *__restrict__ R,
                                                   int64_t H, int n_try, int st, int mp, const SegDesc *__restrict__ segs,
                                                   const int32_t *__restrict__ perm_in, int32_t *__restrict__ perm_out,
                                                   int64_t n, double *__restrict__ split, int32_t *__restrict__ split_idx,
                                                   int32_t *__restrict__ chosen, int32_t *__restrict__ err) {
    extern __shared__ __align__(16) uint8_t smem[];
    const int t = blockIdx.y, tid = threadIdx.x, nthr = blockDim.x;
    const SegDesc sg = segs[blockIdx.x];
    const int m = sg.size, ds = (d + 3) & ~3;
    float *s_rd = reinterpret_cast<float *>(smem);                // [st][ds]
    double *s_p = reinterpret_cast<double *>(s_rd + st * ds);     // [n_try][mp], mp even
    double *s_s2 = s_p + (int64_t)n_try * mp;                     // [n_try]
    int32_t *s_perm = reinterpret_cast<int32_t *>(s_s2 + n_try);  // [mp]
    uint32_t *s_w = reinterpret_cast<uint32_t *>(s_perm + mp);    // [4]
    const int32_t *pin = perm_in + (int64_t)t * n + sg.off;
    for (int i = tid; i < m; i += nthr) s_perm[i] = pin[i];
    const float *Rn = R + ((int64_t)t * H + (sg.heap - 1)) * n_try * (int64_t)d;
    const int g = tid & 7, pt = tid >> 3, per = nthr >> 3;
    for (int t0 = 0; t0 < n_try; t0 += st) {
        __syncthreads();
        stage_tries(Rn, t0, st, n_try, d, ds, s_rd);
        __syncthreads();
        for (int base = 0; base < m; base += 2 * per) {
            const int ia = base + pt, ib = ia + per;
            const float *const x[2] = {X + (int64_t)s_perm[ia < m ? ia : 0] * d, X + (int64_t)s_perm[ib < m ? ib : 0] * d};
            for (int tr = t0; tr < t0 + st && tr < n_try; tr += NT) {  // the rows' later passes hit the caches
                double p[2 * NT];
                group8_dots<VEC, NT, 2>(x, s_rd + (tr - t0) * ds, ds, d, g, p);
#pragma unroll
                for (int k = 0; k < NT; k++)
                    if (g == k && tr + k < n_try) {
                        if (ia < m) s_p[(tr + k) * mp + ia] = p[2 * k];
                        if (ib < m) s_p[(tr + k) * mp + ib] = p[2 * k + 1];
                    }
            }
        }
    }
    __syncthreads();
    // the spread of every try: one wave per try, 256 members of the pairwise tree at a time
    // (at most two such pieces: try_cap <= 512)
    for (int k = tid >> 6; k < n_try; k += nthr >> 6) {
        const double *pk = s_p + k * mp;
        double s1 = wave_canon256([&](int i) { return i < m ? pk[i] : 0.0; });
        if (m > 256) s1 = s1 + wave_canon256([&](int i) { return i + 256 < m ? pk[i + 256] : 0.0; });
        const double mu = s1 / (double)m;
        auto sq = [&](int i) {
            if (i >= m) return 0.0;
            const double dev = pk[i] - mu;
            return __dmul_rn(dev, dev);
        };
        double s2 = wave_canon256(sq);
        if (m > 256) s2 = s2 + wave_canon256([&](int i) { return sq(i + 256); });
        if ((tid & 63) == 0) s_s2[k] = s2;
    }
    __syncthreads();
    int ch = 0;
    double best = 0.0;
    for (int k = 0; k < n_try; k++)  // the largest spread; the first wins ties
        if (s_s2[k] > best) { best = s_s2[k]; ch = k; }
    uint64_t *s_key = reinterpret_cast<uint64_t *>(s_p + ch * mp);
    for (int i = tid; i < mp; i += nthr) s_key[i] = i < m ? key_of(s_p[ch * mp + i]) : ~0ull;
    __syncthreads();
    // rank of every member in (key, position) order: positions ascend with the index, so this
    // is the (p, index) order.  The member of rank floor(m/2) splits the node.
    const int half = m / 2;
    int32_t *pout = perm_out + (int64_t)t * n + sg.off;
    const int64_t hs = (int64_t)t * H + (sg.heap - 1);
    uint32_t lefts = 0;
    for (int base = 0; base < m; base += nthr) {
        const int i = base + tid;
        const bool valid = i < m;
        int rank = m;
        if (valid) {
            const uint64_t u = s_key[i];
            rank = 0;
            for (int q = 0; q < m; q += 2) {
                const ulonglong2 v = *reinterpret_cast<const ulonglong2 *>(s_key + q);
                rank += (v.x < u || (v.x == u && q < i)) ? 1 : 0;
                rank += (v.y < u || (v.y == u && q + 1 < i)) ? 1 : 0;
            }
            if (rank == half) {
                split[hs] = val_of(u);
                split_idx[hs] = s_perm[i];
                chosen[hs] = ch;
            }
        }
        const bool left = valid && rank < half;
        const uint64_t mask = __ballot(left);
        if ((tid & 63) == 0) s_w[tid >> 6] = (uint32_t)__popcll(mask);
        __syncthreads();
        uint32_t lb = lefts + mask_rank(mask);
        for (int w = 0; w < nthr >> 6; w++) {
            if (w < tid >> 6) lb += s_w[w];
            lefts += s_w[w];
        }
        if (valid) {
            const int pos = left ? (int)lb : half + (i - (int)lb);
            if (pos >= 0 && pos < m) pout[pos] = s_perm[i];  // always true when the ranks are consistent
        }
        __syncthreads();
    }
    if (tid == 0 && lefts != (uint32_t)half) atomicOr(err, 1);
}

// Projections of tries tr0 .. tr0 + ntr - 1 over one piece of a node, and the partial of each
// try's sum.
template <bool VEC, int NT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void k_try_proj(const float *__restrict__ X, int d, const float *__restrict__ R,
                                                  int64_t H, int n_try, int st, int tr0, int ntr,
                                                  const SegDesc *__restrict__ segs, const ChunkDesc *__restrict__ subs,
                                                  const int32_t *__restrict__ perm, int64_t n,
                                                  double *__restrict__ praw, double *__restrict__ part) {
    extern __shared__ __align__(16) uint8_t smem[];
    const int ds = (d + 3) & ~3;
    float *s_rd = reinterpret_cast<float *>(smem);             // [st][ds]
    double *s_p = reinterpret_cast<double *>(s_rd + st * ds);  // [st][kTrySub]
    const int t = blockIdx.y, T = gridDim.y, tid = threadIdx.x;
    const ChunkDesc c = subs[blockIdx.x];
    const int32_t *pp = perm + (int64_t)t * n + c.start;
    const float *Rn = R + ((int64_t)t * H + (segs[c.seg].heap - 1)) * n_try * (int64_t)d;
    const int g = tid & 7, pt = tid >> 3;
    for (int t0 = 0; t0 < ntr; t0 += st) {
        __syncthreads();
        stage_tries(Rn, tr0 + t0, st, n_try, d, ds, s_rd);
        __syncthreads();
        for (int base = 0; base < c.len; base += 64) {
            const int ia = base + pt, ib = ia + 32;
            const float *const x[2] = {X + (int64_t)pp[ia < c.len ? ia : 0] * d, X + (int64_t)pp[ib < c.len ? ib : 0] * d};
            for (int tr = 0; tr < st; tr += NT) {  // the rows' later passes hit the caches
                double p[2 * NT];
                group8_dots<VEC, NT, 2>(x, s_rd + tr * ds, ds, d, g, p);
#pragma unroll
                for (int k = 0; k < NT; k++)
                    if (g == k) {
                        s_p[(tr + k) * kTrySub + ia] = ia < c.len ? p[2 * k] : 0.0;
                        s_p[(tr + k) * kTrySub + ib] = ib < c.len ? p[2 * k + 1] : 0.0;
                    }
            }
        }
        __syncthreads();
        for (int k = tid >> 6; k < st && t0 + k < ntr; k += 4) {
            const double *pk = s_p + k * kTrySub;
            const double s1 = wave_canon256([&](int i) { return i < c.len ? pk[i] : 0.0; });
            const int64_t row = (int64_t)(t0 + k) * T + t;
            if ((tid & 63) == 0) part[row * gridDim.x + blockIdx.x] = s1;
            for (int i = tid & 63; i < c.len; i += 64) praw[row * n + c.start + i] = pk[i];
        }
    }
}

// canon_sum of a node's N partials (each an aligned piece of kTrySub members) by one wave; st:
// 32 doubles of LDS of its own.  Pieces of 256 partials combine as a binary counter does.
__device__ inline double wave_canon_list(const double *__restrict__ v, int N, double *st) {
    const int nb = (N + 255) / 256;
    double w = 0.0;
    for (int b = 0; b < nb; b++) {
        w = wave_canon256([&](int i) { return 256 * b + i < N ? v[256 * b + i] : 0.0; });
        int l = 0;
        for (int k = b; k & 1; k >>= 1) w = st[l++] + w;
        st[l] = w;
        wave_sync();
    }
    if (nb & (nb - 1)) {  // the pieces that have no partner meet zeros
        bool have = false;
        for (int l = 0; nb >> l; l++)
            if ((nb >> l) & 1) {
                w = have ? st[l] + w : st[l];
                have = true;
            }
    }
    return w;
}

__global__ __launch_bounds__(256) void k_try_mean(const SegDesc *__restrict__ segs, int nseg, int nsub,
                                                  const double *__restrict__ part, double *__restrict__ mean) {
    __shared__ double s_st[4][32];
    const int k = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (k >= nseg) return;
    const int64_t row = (int64_t)blockIdx.z * gridDim.y + blockIdx.y;  // (try, tree)
    const SegDesc sg = segs[k];
    const double s1 = wave_canon_list(part + row * nsub + sg.sub0, (sg.size + kTrySub - 1) / kTrySub, s_st[threadIdx.x >> 6]);
    if ((threadIdx.x & 63) == 0) mean[row * nseg + k] = s1 / (double)sg.size;
}

__global__ __launch_bounds__(256) void k_try_dev(const ChunkDesc *__restrict__ subs, int ntr,
                                                 const double *__restrict__ praw, int64_t n,
                                                 const double *__restrict__ mean, int nseg,
                                                 double *__restrict__ part) {
    const int t = blockIdx.y, T = gridDim.y;
    const ChunkDesc c = subs[blockIdx.x];
    for (int k = threadIdx.x >> 6; k < ntr; k += 4) {
        const int64_t row = (int64_t)k * T + t;
        const double mu = mean[row * nseg + c.seg];
        const double *pk = praw + row * n + c.start;
        const double s2 = wave_canon256([&](int i) {
            if (i >= c.len) return 0.0;
            const double dev = pk[i] - mu;
            return __dmul_rn(dev, dev);
        });
        if ((threadIdx.x & 63) == 0) part[row * gridDim.x + blockIdx.x] = s2;
    }
}

// The try of largest spread so far (Alg. 2: strictly larger wins), into `chosen`.
__global__ __launch_bounds__(256) void k_try_pick(const SegDesc *__restrict__ segs, int nsub, int tr0, int ntr,
                                                  const double *__restrict__ part, double *__restrict__ best,
                                                  int64_t H, int32_t *__restrict__ chosen) {
    __shared__ double s_st[4][32];
    __shared__ double s_s2[32];  // ntr <= 32
    const int t = blockIdx.y, T = gridDim.y, nseg = gridDim.x, w = threadIdx.x >> 6;
    const SegDesc sg = segs[blockIdx.x];
    for (int k = w; k < ntr; k += 4) {
        const double s2 = wave_canon_list(part + ((int64_t)k * T + t) * nsub + sg.sub0,
                                          (sg.size + kTrySub - 1) / kTrySub, s_st[w]);
        if ((threadIdx.x & 63) == 0) s_s2[k] = s2;
    }
    __syncthreads();
    if (threadIdx.x) return;
    const int64_t hs = (int64_t)t * H + (sg.heap - 1);
    double b = tr0 ? best[(int64_t)t * nseg + blockIdx.x] : 0.0;
    int ch = tr0 ? chosen[hs] : 0;
    for (int k = 0; k < ntr; k++)
        if (s_s2[k] > b) { b = s_s2[k]; ch = tr0 + k; }
    best[(int64_t)t * nseg + blockIdx.x] = b;
    chosen[hs] = ch;
}

// Keys of the chosen try: from the projections when all tries were held at once, else by
// projecting onto the chosen direction again.
template <bool VEC>
__global__ __launch_bounds__(256) void k_try_keys(const float *__restrict__ X, int d, const float *__restrict__ R,
                                                  int64_t H, int n_try, const SegDesc *__restrict__ segs,
                                                  const ChunkDesc *__restrict__ subs, const int32_t *__restrict__ perm,
                                                  int64_t n, const double *__restrict__ praw,
                                                  const int32_t *__restrict__ chosen, uint64_t *__restrict__ keys) {
    extern __shared__ __align__(16) uint8_t smem[];
    const int t = blockIdx.y, tid = threadIdx.x;
    const ChunkDesc c = subs[blockIdx.x];
    const int64_t hs = (int64_t)t * H + (segs[c.seg].heap - 1);
    const int ch = chosen[hs];
    uint64_t *kk = keys + (int64_t)t * n + c.start;
    if (praw) {
        if (tid < c.len) kk[tid] = key_of(praw[((int64_t)ch * gridDim.y + t) * n + c.start + tid]);
        return;
    }
    const int ds = (d + 3) & ~3, g = tid & 7, pt = tid >> 3;
    float *s_rd = reinterpret_cast<float *>(smem);
    stage_tries(R + hs * n_try * (int64_t)d, ch, 1, n_try, d, ds, s_rd);
    __syncthreads();
    const int32_t *pp = perm + (int64_t)t * n + c.start;
    for (int base = 0; base < c.len; base += 64) {
        const int ia = base + pt, ib = ia + 32;
        const float *const x[2] = {X + (int64_t)pp[ia < c.len ? ia : 0] * d, X + (int64_t)pp[ib < c.len ? ib : 0] * d};
        double p[2];
        group8_dots<VEC, 1, 2>(x, s_rd, ds, d, g, p);
        if (g == 0 && ia < c.len) kk[ia] = key_of(p[0]);
        if (g == 0 && ib < c.len) kk[ib] = key_of(p[1]);
    }
}

// Tries projected per read of the rows: at most five (their sums take 80 registers), their
// directions within 40 KB of LDS, evenly spread over the passes.
static int try_width(int n_try, int d) {
    const int ds = (d + 3) & ~3;
    int most = (int)(40 * 1024 / (4 * (size_t)ds));
    most = most > 5 ? 5 : most < 2 ? 2 : most;
    const int passes = (n_try + most - 1) / most;
    const int w = (n_try + passes - 1) / passes;
    return w < 2 ? 2 : w;
}

// Tries whose directions are staged together, a multiple of the width: at most 15, within
// 24 KB (or one width, if that is longer).
static int try_stage(int n_try, int d) {
    const int w = try_width(n_try, d), ds = (d + 3) & ~3, passes = (n_try + w - 1) / w;
    const int per = std::min(24 * 1024 / (4 * ds * w), 15 / w);
    return w * std::max(1, std::min(per, passes));
}

size_t level_try_lds(int max_m, int d, int n_try) {
    const size_t mp = (size_t)((max_m + 1) & ~1), ds = (size_t)((d + 3) & ~3);
    return 4 * try_stage(n_try, d) * ds + 8 * (n_try * mp + n_try) + 4 * (mp + 4);
}

template <typename F>
static void with_tries(bool vec, int w, const F &go) {
    auto nt = [&](auto v) {
        constexpr bool V = decltype(v)::value;
        if (w == 2) go(std::integral_constant<bool, V>{}, std::integral_constant<int, 2>{});
        else if (w == 3) go(std::integral_constant<bool, V>{}, std::integral_constant<int, 3>{});
        else if (w == 4) go(std::integral_constant<bool, V>{}, std::integral_constant<int, 4>{});
        else go(std::integral_constant<bool, V>{}, std::integral_constant<int, 5>{});
    };
    if (vec) nt(std::true_type{});
    else nt(std::false_type{});
}

void launch_level_try(hipStream_t s, bool vec, const float *X, int d, const float *R, int64_t H, int n_try,
                      const SegDesc *segs, int nseg, int max_m, int T, const int32_t *pin, int32_t *pout, int64_t n,
                      double *split, int32_t *split_idx, int32_t *chosen, int32_t *err) {
    const size_t lds = level_try_lds(max_m, d, n_try);
    // a workgroup's rows per step are a quarter of its threads: small nodes take small workgroups
    const int threads = max_m <= 64 ? 64 : max_m <= 128 ? 128 : 256;
    with_tries(vec, try_width(n_try, d), [&](auto v, auto w) {
        auto kern = k_level_try<decltype(v)::value, decltype(w)::value>;
        hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        hipLaunchKernelGGL(kern, dim3(nseg, T), dim3(threads), lds, s, X, d, R, H, n_try, try_stage(n_try, d),
                           (max_m + 1) & ~1, segs, pin, pout, n, split, split_idx, chosen, err);
    });
    launch_check(s, "k_level_try");
}

// Scores the tries of every node of a level over many blocks: `chosen` and the chosen try's
// keys ([T][n], by position).
void launch_level_score(hipStream_t s, bool vec, const float *X, int d, const float *R, int64_t H, int n_try,
                        const SegDesc *segs, int nseg, const ChunkDesc *subs, int nsub, int T, const int32_t *pin,
                        int64_t n, const TryBufs &tb, int32_t *chosen, uint64_t *keys) {
    const dim3 gp(nsub, T);
    const size_t ds = (size_t)((d + 3) & ~3);
    for (int tr0 = 0; tr0 < n_try; tr0 += tb.group) {
        const int ntr = std::min(tb.group, n_try - tr0);
        with_tries(vec, try_width(ntr, d), [&](auto v, auto w) {
            constexpr int NT = decltype(w)::value;
            auto kern = k_try_proj<decltype(v)::value, NT>;
            const int st = try_stage(ntr, d);
            const size_t lds = st * (4 * ds + 8 * kTrySub);
            hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
            hipLaunchKernelGGL(kern, gp, dim3(256), lds, s, X, d, R, H, n_try, st, tr0, ntr, segs, subs, pin, n, tb.praw,
                               tb.part);
        });
        launch_check(s, "k_try_proj");
        hipLaunchKernelGGL(k_try_mean, dim3((nseg + 3) / 4, T, ntr), dim3(256), 0, s, segs, nseg, nsub, tb.part, tb.mean);
        launch_check(s, "k_try_mean");
        hipLaunchKernelGGL(k_try_dev, gp, dim3(256), 0, s, subs, ntr, tb.praw, n, tb.mean, nseg, tb.part);
        launch_check(s, "k_try_dev");
        hipLaunchKernelGGL(k_try_pick, dim3(nseg, T), dim3(256), 0, s, segs, nsub, tr0, ntr, tb.part, tb.best, H, chosen);
        launch_check(s, "k_try_pick");
    }
    const bool held = tb.group >= n_try;
    auto go = [&](auto kern) {
        hipLaunchKernelGGL(kern, gp, dim3(256), held ? 0 : 4 * ds, s, X, d, R, H, n_try, segs, subs, pin, n,
                           held ? tb.praw : nullptr, chosen, keys);
    };
    if (vec) go(k_try_keys<true>);
    else go(k_try_keys<false>);
    launch_check(s, "k_try_keys");
}

__global__ void k_copy_segments(const LeafDesc *__restrict__ segs, int nseg,
                                const int32_t *__restrict__ in, int32_t *__restrict__ out,
                                int64_t n) {
    const int t = blockIdx.y;
    const LeafDesc sg = segs[blockIdx.x];
    for (int i = threadIdx.x; i < sg.size; i += blockDim.x)
        out[(int64_t)t * n + sg.off + i] = in[(int64_t)t * n + sg.off + i];
}

__global__ void k_iota(int32_t *__restrict__ perm, int64_t n) {
    const int t = blockIdx.y;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        perm[(int64_t)t * n + i] = (int32_t)i;
}

// ================================================================ leaves (neighbourhoods)

// leaf_of, leaf centroid mu (binary32 mean of the members), and the leaf-ordered, centred
// copy Xc[t][pos][0..dp) in the tile precision, with |Xc row|^2 (binary32, of the stored
// low-precision values) and |x - mu| (binary32) per position.
template <typename T>
__device__ inline T to_tile(float v);
template <>
__device__ inline float to_tile<float>(float v) { return v; }
template <>
__device__ inline __bf16 to_tile<__bf16>(float v) { return (__bf16)v; }
template <>
__device__ inline _Float16 to_tile<_Float16>(float v) { return (_Float16)v; }

template <typename T>
__global__ __launch_bounds__(256) void k_leaf_finalize(
    const float *__restrict__ X, int d, int dp, const LeafDesc *__restrict__ leaves, int nleaf,
    const int32_t *__restrict__ perm, int64_t n, int32_t *__restrict__ leaf_of,
    float *__restrict__ centroid, T *__restrict__ Xc, float2 *__restrict__ nrm, float range_max, int ids_in_lds) {
    extern __shared__ __align__(16) float s_mu[];  // dp floats, then 4 x dp partial sums, then members
    const int t = blockIdx.y, tid = threadIdx.x;
    const LeafDesc lf = leaves[blockIdx.x];
    const int m = lf.size;
    float *s_part = s_mu + dp;
    const int32_t *pp = perm + (int64_t)t * n + lf.off;
    // member ids: staged in LDS when the launch reserved room for them, else read in place
    int32_t *s_lds_id = reinterpret_cast<int32_t *>(s_part + 4 * dp);
    const int32_t *s_id = ids_in_lds ? s_lds_id : pp;
    for (int i = tid; i < m; i += 256) {
        const int id = pp[i];
        if (ids_in_lds) s_lds_id[i] = id;
        leaf_of[(int64_t)t * n + id] = lf.heap;
    }
    __syncthreads();
    // mean: wave w sums rows w, w+4, ... in order (lane j holds columns j, j+64, ...); four
    // rows are loaded before they are added, then the four partial sums are added in wave
    // order -- a fixed order, so the centroid is reproducible
    const int lane = tid & 63, wv = tid >> 6;
    for (int j0 = 0; j0 < dp; j0 += 64 * 4) {
        float acc[4] = {0.f, 0.f, 0.f, 0.f};
        int i = wv;
        for (; i + 12 < m; i += 16) {
            float v[4][4];
#pragma unroll
            for (int r = 0; r < 4; r++) {
                const float *x = X + (int64_t)s_id[i + 4 * r] * d;
#pragma unroll
                for (int q = 0; q < 4; q++) {
                    const int j = j0 + 64 * q + lane;
                    v[r][q] = j < d ? x[j] : 0.f;
                }
            }
#pragma unroll
            for (int r = 0; r < 4; r++)
#pragma unroll
                for (int q = 0; q < 4; q++) acc[q] += v[r][q];
        }
        for (; i < m; i += 4) {
            const float *x = X + (int64_t)s_id[i] * d;
#pragma unroll
            for (int q = 0; q < 4; q++) {
                const int j = j0 + 64 * q + lane;
                acc[q] += j < d ? x[j] : 0.f;
            }
        }
#pragma unroll
        for (int q = 0; q < 4; q++) {
            const int j = j0 + 64 * q + lane;
            if (j < dp) s_part[wv * dp + j] = acc[q];
        }
    }
    __syncthreads();
    for (int j = tid; j < dp; j += 256) {
        const float sum = ((s_part[j] + s_part[dp + j]) + s_part[2 * dp + j]) + s_part[3 * dp + j];
        const float mu = j < d ? sum / (float)m : 0.f;
        s_mu[j] = mu;
        if (j < d) centroid[((int64_t)t * nleaf + blockIdx.x) * d + j] = mu;
    }
    __syncthreads();
    // centred copy in the tile precision and its norms, two rows per wave at a time
    for (int i0 = wv; i0 < m; i0 += 8) {
        float na[2] = {0.f, 0.f}, ra[2] = {0.f, 0.f};
        bool over[2] = {false, false};
        for (int j0 = 0; j0 < dp; j0 += 64 * 4) {
            float xv[2][4];
#pragma unroll
            for (int r = 0; r < 2; r++) {
                const int i = i0 + 4 * r;
                const float *x = X + (int64_t)s_id[i < m ? i : i0] * d;
#pragma unroll
                for (int q = 0; q < 4; q++) {
                    const int j = j0 + 64 * q + lane;
                    xv[r][q] = j < d ? x[j] : 0.f;
                }
            }
#pragma unroll
            for (int r = 0; r < 2; r++) {
                const int i = i0 + 4 * r;
                if (i >= m) continue;
                T *out = Xc ? Xc + ((int64_t)t * n + lf.off + i) * dp : nullptr;
#pragma unroll
                for (int q = 0; q < 4; q++) {
                    const int j = j0 + 64 * q + lane;
                    if (j >= dp) continue;
                    const float a = j < d ? xv[r][q] - s_mu[j] : 0.f;
                    over[r] |= fabsf(a) > range_max;
                    const T qv = to_tile<T>(a);
                    if (out) out[j] = qv;
                    const float qf = (float)qv;
                    na[r] = __builtin_fmaf(qf, qf, na[r]);
                    ra[r] = __builtin_fmaf(a, a, ra[r]);
                }
            }
        }
#pragma unroll
        for (int r = 0; r < 2; r++) {
            float x = na[r], y = ra[r];
            for (int o = 32; o > 0; o >>= 1) {
                x += __shfl_xor(x, o, 64);
                y += __shfl_xor(y, o, 64);
            }
            const uint64_t ov = __ballot(over[r]);
            const int i = i0 + 4 * r;
            if (lane == 0 && i < m) nrm[(int64_t)t * n + lf.off + i] = make_float2(x, ov ? INFINITY : sqrtf(y));
        }
    }
}

// The leaf-ordered, centred copy alone, for a forest whose leaf pass did not write it: each
// element is x - mu rounded to the tile type (zero past d), from the centroid the leaf pass
// stored, so it holds exactly the values the leaf pass would have written.  One block per
// (leaf, tree); four columns per thread.
template <typename T, bool VEC>
__global__ __launch_bounds__(256) void k_leaf_copy(const float *__restrict__ X, int d, int dp,
                                                   const LeafDesc *__restrict__ leaves, int nleaf,
                                                   const int32_t *__restrict__ perm, int64_t n,
                                                   const float *__restrict__ centroid, T *__restrict__ Xc) {
    const int t = blockIdx.y;
    const LeafDesc lf = leaves[blockIdx.x];
    const float *mu = centroid + ((int64_t)t * nleaf + blockIdx.x) * d;
    const int32_t *pp = perm + (int64_t)t * n + lf.off;
    const int q = dp >> 2;  // four-column groups per row (dp is a multiple of 8)
    for (int v = threadIdx.x; v < lf.size * q; v += 256) {
        const int i = v / q, c = 4 * (v - i * q);
        const float *x = X + (int64_t)pp[i] * d;
        float a[4];
        if (VEC && c < d) {  // d % 4 == 0: the four columns are all below d
            const float4 xv = *reinterpret_cast<const float4 *>(x + c);
            const float4 u = *reinterpret_cast<const float4 *>(mu + c);
            a[0] = xv.x - u.x;
            a[1] = xv.y - u.y;
            a[2] = xv.z - u.z;
            a[3] = xv.w - u.w;
        } else {
#pragma unroll
            for (int e = 0; e < 4; e++) a[e] = c + e < d ? x[c + e] - mu[c + e] : 0.f;
        }
        T qv[4];
#pragma unroll
        for (int e = 0; e < 4; e++) qv[e] = to_tile<T>(a[e]);
        T *out = Xc + ((int64_t)t * n + lf.off + i) * dp + c;
        if constexpr (sizeof(T) == 4) {
            *reinterpret_cast<float4 *>(out) = make_float4(qv[0], qv[1], qv[2], qv[3]);
        } else {
            uint2 w;
            __builtin_memcpy(&w, qv, sizeof(w));
            *reinterpret_cast<uint2 *>(out) = w;
        }
    }
}

// The leaf statistics without the copy, for forests whose all-points search centres the rows
// itself as it stages them (leaves of at most 256 points): leaf_of, the centroid mu (binary32
// mean, a fixed order: each of 32 row groups sums its rows in order, then the groups in
// order) and per position |tile(x - mu)|^2 of the tile-type values and |x - mu| (+inf past
// the tile type's range).  A copy made later from this centroid holds exactly the values
// these norms describe.  One block of 1024 threads per (leaf, tree): 32 lanes per row, four
// columns each per step of 128 columns, and the block's 32 row groups hold all of the leaf's
// rows of a step in registers, so X is read once.
// NT threads hold leaves of up to NT / 4 points (1024 threads for 256-point leaves, 256 for
// leaves of at most 64, where a larger block would leave most of its rows empty).
// Ragged leaves (uniform rule: a few of up to 256 points, most far below 64) run in two launches,
// each for its sizes: 256 threads for leaves of at most 64 points, with the same 32 row groups
// (CL; a thread group of 32 lanes takes CL / RG of them), so the sums do not depend on the
// launch, and 1024 threads for the rest (100 000 x 32, 32 trees, leaves of 21 points on average:
// 1 470 -> 540 us).
template <typename T, bool VEC, int NT, int CL = NT / 32>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(8))) void k_leaf_stats(const float *__restrict__ X, int d, int dp,
                                                     const LeafDesc *__restrict__ leaves, int nleaf,
                                                     const int32_t *__restrict__ perm, int64_t n,
                                                     int32_t *__restrict__ leaf_of, float *__restrict__ centroid,
                                                     float2 *__restrict__ nrm, float range_max, int64_t leaf_stride, int m_lo, int m_hi) {
    constexpr int ML = NT / 4, RG = NT / 32, RK = ML / RG;  // rows, thread groups, rows per thread group
    __shared__ __align__(16) float s_part[CL][128];
    __shared__ __align__(16) float s_mu[128];
    __shared__ int32_t s_id[ML];
    __shared__ float s_na[ML], s_ra[ML];  // the rows' norms, summed over the steps in order
    const int t = blockIdx.y, tid = threadIdx.x, lane = tid & 63;
    const LeafDesc lf = leaves[t * leaf_stride + blockIdx.x];  // (stride 0: one table for all trees)
    const int m = lf.size;
    if (m <= m_lo || m > m_hi) return;  // another launch's leaf, or none: m == 0
    const int32_t *pp = perm + (int64_t)t * n + lf.off;
    for (int i = tid; i < m; i += NT) {
        const int id = pp[i];
        s_id[i] = id;
        leaf_of[(int64_t)t * n + id] = lf.heap;
        s_na[i] = 0.f;
        s_ra[i] = 0.f;
    }
    __syncthreads();
    const int l32 = lane & 31, g = tid >> 5;  // rows g, g + RG, ...
    for (int cb = 0; cb < dp; cb += 128) {
        const int j = cb + 4 * l32;
        float4 x[RK];
#pragma unroll
        for (int k = 0; k < RK; k++) {  // every row of the step in flight at once
            const int r = g + RG * k;
            x[k] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (r < m) {
                const float *xr = X + (int64_t)s_id[r] * d;
                if (VEC) {
                    if (j < d) x[k] = *reinterpret_cast<const float4 *>(xr + j);
                } else {
                    x[k].x = j < d ? xr[j] : 0.f;
                    x[k].y = j + 1 < d ? xr[j + 1] : 0.f;
                    x[k].z = j + 2 < d ? xr[j + 2] : 0.f;
                    x[k].w = j + 3 < d ? xr[j + 3] : 0.f;
                }
            }
        }
#pragma unroll
        for (int c = 0; c < CL / RG; c++) {
            float4 cs = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
            for (int k = c; k < RK; k += CL / RG) {
                if (g + RG * k < m) {
                    cs.x += x[k].x;
                    cs.y += x[k].y;
                    cs.z += x[k].z;
                    cs.w += x[k].w;
                }
            }
            *reinterpret_cast<float4 *>(&s_part[g + RG * c][4 * l32]) = cs;
        }
        __syncthreads();
        if (tid < 128) {
            float v = 0.f;
            for (int q = 0; q < CL; q++) v += s_part[q][tid];
            const int jj = cb + tid;
            const float mu = jj < d ? v / (float)m : 0.f;
            s_mu[tid] = mu;
            if (jj < d) centroid[((int64_t)t * nleaf + blockIdx.x) * d + jj] = mu;
        }
        __syncthreads();
        const float4 u = *reinterpret_cast<const float4 *>(&s_mu[4 * l32]);
#pragma unroll
        for (int k = 0; k < RK; k++) {  // the step's share of each row's norms (past dp: zero)
            const float a[4] = {j < d ? x[k].x - u.x : 0.f, j + 1 < d ? x[k].y - u.y : 0.f,
                                j + 2 < d ? x[k].z - u.z : 0.f, j + 3 < d ? x[k].w - u.w : 0.f};
            float na = 0.f, ra = 0.f;
            bool over = false;
#pragma unroll
            for (int e = 0; e < 4; e++) {
                over |= fabsf(a[e]) > range_max;
                const float qf = (float)to_tile<T>(a[e]);
                na = __builtin_fmaf(qf, qf, na);
                ra = __builtin_fmaf(a[e], a[e], ra);
            }
            for (int o = 1; o < 32; o <<= 1) {
                na += __shfl_xor(na, o, 64);
                ra += __shfl_xor(ra, o, 64);
            }
            const bool ov = ((__ballot(over) >> (lane & 32)) & 0xffffffffull) != 0;
            const int r = g + RG * k;
            if (l32 == 0 && r < m) {
                s_na[r] += na;
                s_ra[r] = ov ? INFINITY : s_ra[r] + ra;
            }
        }
        __syncthreads();  // s_part and s_mu are rewritten by the next step
    }
    for (int r = tid; r < m; r += NT) nrm[(int64_t)t * n + lf.off + r] = make_float2(s_na[r], sqrtf(s_ra[r]));
}

template <typename T>
static void leaf_stats(hipStream_t s, bool vec, const float *X, int d, int dp, const LeafDesc *leaves, int nleaf,
                       int ntree, const int32_t *perm, int64_t n, int32_t *leaf_of, float *centroid, float2 *nrm,
                       float range_max, int max_leaf, int64_t leaf_stride) {
    const dim3 grid(nleaf, ntree);
    auto go = [&](auto kern, int nt, int lo, int hi) {
        hipLaunchKernelGGL(kern, grid, dim3(nt), 0, s, X, d, dp, leaves, nleaf, perm, n, leaf_of, centroid, nrm, range_max,
                           leaf_stride, lo, hi);
    };
    if (max_leaf <= 64) {
        vec ? go(k_leaf_stats<T, true, 256>, 256, 0, 64) : go(k_leaf_stats<T, false, 256>, 256, 0, 64);
    } else {
        const int lo = leaf_stride ? 64 : 0;
        if (lo) vec ? go(k_leaf_stats<T, true, 256, 32>, 256, 0, 64) : go(k_leaf_stats<T, false, 256, 32>, 256, 0, 64);
        vec ? go(k_leaf_stats<T, true, 1024>, 1024, lo, 256) : go(k_leaf_stats<T, false, 1024>, 1024, lo, 256);
    }
    launch_check(s, "k_leaf_stats");
}

// ================================================================ launchers

void launch_leaf_stats(hipStream_t s, int prec, const float *X, int d, int dp, const LeafDesc *leaves, int nleaf,
                       int ntree, const int32_t *perm, int64_t n, int32_t *leaf_of, float *centroid, float2 *nrm,
                       int max_leaf, int64_t leaf_stride) {
    if (nleaf <= 0 || ntree <= 0 || max_leaf > 256) return;  // the caller runs the full leaf pass instead
    const bool vec = (d % 4) == 0;
    if (prec == RPF_DIST_BF16)
        leaf_stats<__bf16>(s, vec, X, d, dp, leaves, nleaf, ntree, perm, n, leaf_of, centroid, nrm, 3.0e38f, max_leaf, leaf_stride);
    else if (prec == RPF_DIST_FP16)
        leaf_stats<_Float16>(s, vec, X, d, dp, leaves, nleaf, ntree, perm, n, leaf_of, centroid, nrm, 60000.f, max_leaf, leaf_stride);
    else
        leaf_stats<float>(s, vec, X, d, dp, leaves, nleaf, ntree, perm, n, leaf_of, centroid, nrm, 3.0e38f, max_leaf, leaf_stride);
}

template <typename T>
static void leaf_copy(hipStream_t s, bool vec, const float *X, int d, int dp, const LeafDesc *leaves, int nleaf,
                      int ntree, const int32_t *perm, int64_t n, const float *centroid, void *Xc) {
    const dim3 grid(nleaf, ntree);
    if (vec)
        hipLaunchKernelGGL((k_leaf_copy<T, true>), grid, dim3(256), 0, s, X, d, dp, leaves, nleaf, perm, n, centroid,
                           (T *)Xc);
    else
        hipLaunchKernelGGL((k_leaf_copy<T, false>), grid, dim3(256), 0, s, X, d, dp, leaves, nleaf, perm, n, centroid,
                           (T *)Xc);
    launch_check(s, "k_leaf_copy");
}

void launch_leaf_copy(hipStream_t s, int prec, const float *X, int d, int dp, const LeafDesc *leaves, int nleaf,
                      int ntree, const int32_t *perm, int64_t n, const float *centroid, void *Xc) {
    if (nleaf <= 0 || ntree <= 0) return;
    const bool vec = (d % 4) == 0;
    if (prec == RPF_DIST_BF16)
        leaf_copy<__bf16>(s, vec, X, d, dp, leaves, nleaf, ntree, perm, n, centroid, Xc);
    else if (prec == RPF_DIST_FP16)
        leaf_copy<_Float16>(s, vec, X, d, dp, leaves, nleaf, ntree, perm, n, centroid, Xc);
    else
        leaf_copy<float>(s, vec, X, d, dp, leaves, nleaf, ntree, perm, n, centroid, Xc);
}

size_t level_small_lds(int max_m, int d, int n_try) {
    size_t lds = ((((4 * (size_t)max_m + 15) & ~(size_t)15) + 8 * (size_t)max_m + 15) & ~(size_t)15) +
                 3 * 8 * (size_t)((d + 3) & ~3) + 4 * (256 + 16);
    lds = (lds + 7) & ~(size_t)7;
    if (n_try > 1) {
        int P2 = 1;
        while (P2 < max_m) P2 <<= 1;
        lds += 8 * (size_t)max_m + 8 * (size_t)P2;
    }
    return lds;
}

void launch_digit_bound(hipStream_t s, const float *R, int64_t nodes, int d, double *bound) {
    const unsigned blocks = (unsigned)((nodes + 3) / 4 < 16384 ? (nodes + 3) / 4 : 16384);
    hipLaunchKernelGGL(k_digit_bound, dim3(blocks), dim3(256), 0, s, R, nodes, d, bound);
    launch_check(s, "k_digit_bound");
}

// A level with at most one workgroup per CU runs 1024 threads in each instead of 256: such a
// level takes the time of one workgroup's walk over its members.  Build at 10 000 x 128, 4 trees:
// 436 -> 349 us; 40 000 x 64, 16 trees: 850 -> 722 (748 with up to 512 workgroups); 200 000 x 128,
// 2 trees: 1 067 -> 760.
static bool few_blocks(int64_t blocks) { return blocks <= 256; }

void launch_level_small(hipStream_t s, bool vec, const float *X, int d, const float *R, int64_t H,
                        int n_try, const SegDesc *segs, int nseg, int max_m, int T,
                        const int32_t *pin, int32_t *pout, int64_t n, double *split,
                        int32_t *split_idx, int32_t *chosen, int32_t *err, const LevelLink &lk) {
    if (!lk.look && lk.keys_in && n_try == 1 && max_m <= kWaveSeg && !lk.bound) {  // fed level of small segments
        auto go = [&](auto kern) {
            hipLaunchKernelGGL(kern, dim3((nseg + 3) / 4, T), dim3(256), 0, s, segs, nseg, pin, pout, n, H, split,
                               split_idx, chosen, err, lk.keys_in);
        };
        if (max_m <= 512) go(k_level_fed_wave<8>);
        else go(k_level_fed_wave<16>);
        launch_check(s, "k_level_fed_wave");
        return;
    }
    const size_t lds = level_small_lds(max_m, d, n_try);
    dim3 grid(nseg, T);
    auto go = [&](auto kern, int nt) {
        hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        hipLaunchKernelGGL(kern, grid, dim3(nt), lds, s, X, d, R, H, n_try, segs, pin, pout, n, split, split_idx,
                           chosen, err, lk.look, lk.ahead, lk.keys_next, lk.keys_in, lk.xq, lk.dq, lk.bound, lk.band);
    };
    const bool q8 = lk.xq && n_try == 1;  // (several tries project through the binary32 rows)
    auto pick = [&](auto w) {
        constexpr int W = decltype(w)::value;
        if (lk.bound) {
            if (lk.look && vec) go(k_level_small<true, true, 2, W>, W);
            else if (lk.look) go(k_level_small<false, true, 2, W>, W);
            else if (vec) go(k_level_small<true, false, 2, W>, W);
            else go(k_level_small<false, false, 2, W>, W);
        } else if (lk.look) {
            if (q8 && vec) go(k_level_small<true, true, 1, W>, W);
            else if (q8) go(k_level_small<false, true, 1, W>, W);
            else if (vec) go(k_level_small<true, true, 0, W>, W);
            else go(k_level_small<false, true, 0, W>, W);
        } else {
            if (q8 && vec) go(k_level_small<true, false, 1, W>, W);
            else if (q8) go(k_level_small<false, false, 1, W>, W);
            else if (vec) go(k_level_small<true, false, 0, W>, W);
            else go(k_level_small<false, false, 0, W>, W);
        }
    };
    if (n_try == 1 && few_blocks((int64_t)nseg * T) && max_m >= 512 && lds <= 128 * 1024)
        pick(std::integral_constant<int, 1024>{});
    else
        pick(std::integral_constant<int, 256>{});
    launch_check(s, "k_level_small");
}

template <bool VEC>
static void proj_chunks(hipStream_t s, dim3 gc, const float *X, int d, const float *R, int64_t H,
                        const SegDesc *segs, const ChunkDesc *chunks, const int32_t *pin, int64_t n,
                        const LargeBufs &b, const LevelLink &lk) {
    const size_t ds = (size_t)((d + 3) & ~3);
    const size_t lds = d > 1024 ? 0 : lk.look ? 3 * ds * sizeof(double) : ds * sizeof(float);
    auto go = [&](auto kern, int nt) {
        hipLaunchKernelGGL(kern, gc, dim3(nt), lds, s, X, d, R, H, segs, chunks, pin, n, b.keys, lk.look, lk.ahead,
                           lk.xq, lk.dq, lk.band);
    };
    const bool q8 = lk.xq != nullptr;
    if (lk.bound) {
        auto digits = [&](auto kern) {
            const int bytes = 16 * lk.dq;
            // the first level: the same rows in every tree, whose workgroups share them in cache
            const bool trees_first = lk.top && gc.x <= 65535;
            hipLaunchKernelGGL(kern, trees_first ? dim3(gc.y, gc.x) : gc, dim3(256), bytes, s, lk.xq, d, lk.dq, R, H,
                               segs, chunks, pin, n, b.keys, lk.look, reinterpret_cast<double *>(lk.ahead),
                               (int)trees_first, lk.band);
        };
        if (lk.look) digits(k_digit_chunks<true>);
        else digits(k_digit_chunks<false>);
        launch_check(s, "k_digit_chunks");
        if (!lk.band.prev) return;
    }
    auto pick = [&](auto w) {
        constexpr int W = decltype(w)::value;
        if (lk.look && q8) go(k_proj_chunks<VEC, true, true, W>, W);
        else if (lk.look) go(k_proj_chunks<VEC, true, false, W>, W);
        else if (q8) go(k_proj_chunks<VEC, false, true, W>, W);
        else go(k_proj_chunks<VEC, false, false, W>, W);
    };
    if (few_blocks((int64_t)gc.x * gc.y)) pick(std::integral_constant<int, 1024>{});
    else pick(std::integral_constant<int, 256>{});
    launch_check(s, "k_proj_chunks");
}

void launch_level_large(hipStream_t s, bool vec, const float *X, int d, const float *R, int64_t H,
                        const SegDesc *segs, int nseg, int max_m, const ChunkDesc *chunks, int nchunk,
                        int T, const int32_t *pin, int32_t *pout, int64_t n, double *split,
                        int32_t *split_idx, int32_t *chosen, int32_t *err, const LargeBufs &b0,
                        double proj_bytes, const LevelLink &lk) {
    dim3 gs(nseg, T), gc(nchunk, T);
    LargeBufs b = b0;
    if (lk.keys_in) b.keys = const_cast<uint64_t *>(lk.keys_in);  // fed level: made by the level above
    if (lk.roots) {  // every tree's root projections from one read of X
        ProfScope ps(s, "proj_roots", proj_bytes, 0);
        hipLaunchKernelGGL(k_proj_root, dim3(nchunk, kChunk / 64), dim3(256), 0, s, X, d, R, H, T, segs, chunks,
                           lk.look, n, b.keys, lk.ahead);
        launch_check(s, "k_proj_root");
    } else if (!lk.keys_in && !lk.keys_ready) {
        ProfScope ps(s, lk.look ? "proj_chunks_x3" : "proj_chunks", proj_bytes, 0);
        if (vec) proj_chunks<true>(s, gc, X, d, R, H, segs, chunks, pin, n, b, lk);
        else proj_chunks<false>(s, gc, X, d, R, H, segs, chunks, pin, n, b, lk);
    }
    auto select = [&]() {
        ProfScope ps(s, "select_passes", 0, 0);
        // with more segments than CUs the pick costs more than the two launches before it save
        // it (72 trees, segments of 7 813: 613 us whole, 320 us bracketed); with few, one launch
        const int direct = (int64_t)nseg * T > 256 ? kChunk : kSelDirect;
        const int sampled = max_m > direct ? 1 : 0;
        if (sampled) {
            if (max_m < kSelFewer)
                hipLaunchKernelGGL(k_sel_sample<kSelSample2>, gs, dim3(kSelSample2 / 2), 0, s, segs, b.keys, n, direct, b.state);
            else
                hipLaunchKernelGGL(k_sel_sample<kSelSample>, gs, dim3(kSelSample / 2), 0, s, segs, b.keys, n, direct, b.state);
            launch_check(s, "k_sel_sample");
            hipLaunchKernelGGL(k_sel_count, gc, dim3(256), 0, s, segs, chunks, b.keys, n, b.state, nseg, pout, b.lcount);
            launch_check(s, "k_sel_count");
        }
        hipLaunchKernelGGL(k_sel_pick, gs, dim3(1024), 0, s, segs, b.keys, pin, n, b.state, sampled, pout, b.lcount,
                           nchunk, H, split, split_idx, chosen, err);
        launch_check(s, "k_sel_pick");
    };
    select();
    if (lk.bound) {  // keys by digits: exact ones around the median, and the median of those
        auto refine = [&](auto kern) {
            hipLaunchKernelGGL(kern, gc, dim3(256), (size_t)((d + 3) & ~3) * 4, s, lk.xq, d, lk.dq, R, H, segs, chunks,
                               pin, n, b.keys, b.state, nseg, lk.bound, lk.band);
        };
        if (vec) refine(k_digit_refine<true>);
        else refine(k_digit_refine<false>);
        launch_check(s, "k_digit_refine");
        select();
    }
    {
        ProfScope ps(s, "partition", 0, 0);
        auto go = [&](auto kern, int nt) {
            hipLaunchKernelGGL(kern, gc, dim3(nt), 0, s, segs, chunks, nchunk, b.keys, pin, pout, n, b.state, nseg,
                               b.lcount, lk.look, lk.ahead, lk.keys_next);
        };
        if (few_blocks((int64_t)nchunk * T)) go(k_part_scatter<1024>, 1024);
        else go(k_part_scatter<256>, 256);
        launch_check(s, "k_part_scatter");
    }
}

void launch_copy_segments(hipStream_t s, const LeafDesc *segs, int nseg, int T, const int32_t *in,
                          int32_t *out, int64_t n) {
    if (nseg == 0) return;
    hipLaunchKernelGGL(k_copy_segments, dim3(nseg, T), dim3(256), 0, s, segs, nseg, in, out, n);
    launch_check(s, "k_copy_segments");
}

void launch_iota(hipStream_t s, int32_t *perm, int64_t n, int T) {
    int blocks = (int)((n + 255) / 256);
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(k_iota, dim3(blocks, T), dim3(256), 0, s, perm, n);
    launch_check(s, "k_iota");
}

// Row stride of a leaf staged in LDS: an odd number of 16-byte chunks, so that the eight rows
// a wave centres at once (one per group of eight lanes) fall in different bank groups.
__host__ __device__ inline int leaf_row_stride(int d) {
    const int s = (d + 3) & ~3;
    return ((s >> 2) & 1) ? s : s + 4;
}

// Mean and centred copy of one leaf whose m rows (stride ds floats) are in LDS, by a block of
// 512 threads: the centroid is a fixed-order sum (R row classes per column, then the classes
// in order), so it is reproducible; then eight lanes per row write the centred row, four
// consecutive columns at a time, and its two norms.
template <typename T>
__device__ __attribute__((always_inline)) inline void leaf_centre_staged(const float *s_rows, float *s_mu, float *s_part, int m, int d, int ds,
                                          int dp, int t, int leaf, int nleaf, const LeafDesc &lf, int64_t n,
                                          float *__restrict__ centroid, T *__restrict__ Xc,
                                          float2 *__restrict__ nrm, float range_max) {
    constexpr int NT = 512, NW = NT / 64;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    if (ds <= NT) {  // R row classes per column: class g sums rows g, g+R, ... (two chains)
        const int R = NT / ds, g = tid / ds, j = tid - g * ds;
        if (g < R) {
            float a0 = 0.f, a1 = 0.f;
            if (j < d) {
                int i = g;
                for (; i + R < m; i += 2 * R) {
                    a0 += s_rows[(size_t)i * ds + j];
                    a1 += s_rows[(size_t)(i + R) * ds + j];
                }
                if (i < m) a0 += s_rows[(size_t)i * ds + j];
            }
            s_part[tid] = a0 + a1;
        }
        __syncthreads();
        if (tid < ds) {
            float sum = 0.f;
            for (int c = 0; c < R; c++) sum += s_part[c * ds + tid];
            const float mu = tid < d ? sum / (float)m : 0.f;
            s_mu[tid] = mu;
            if (tid < d) centroid[((int64_t)t * nleaf + leaf) * d + tid] = mu;
        }
    } else {
        for (int j = tid; j < ds; j += NT) {
            float acc = 0.f;
            if (j < d)
                for (int i = 0; i < m; i++) acc += s_rows[(size_t)i * ds + j];
            const float mu = j < d ? acc / (float)m : 0.f;
            s_mu[j] = mu;
            if (j < d) centroid[((int64_t)t * nleaf + leaf) * d + j] = mu;
        }
    }
    __syncthreads();
    // centred copy and norms: eight lanes per row, each lane four consecutive columns at a
    // time, so a wave has eight rows in flight and reduces each over three shuffle steps
    const int sub = lane & 7, grp = lane >> 3;
    for (int i0 = wv * 8; i0 < m; i0 += NW * 8) {
        const int i = i0 + grp;
        const bool live = i < m;
        const int ir = live ? i : m - 1;
        T *out = Xc ? Xc + ((int64_t)t * n + lf.off + ir) * dp : nullptr;
        float na = 0.f, ra = 0.f;
        bool over = false;
        for (int c = 4 * sub; c < dp; c += 32) {
            float a[4];
            if (c < ds) {
                const float4 x = *reinterpret_cast<const float4 *>(s_rows + (size_t)ir * ds + c);
                const float4 u = *reinterpret_cast<const float4 *>(s_mu + c);
                a[0] = c + 0 < d ? x.x - u.x : 0.f;
                a[1] = c + 1 < d ? x.y - u.y : 0.f;
                a[2] = c + 2 < d ? x.z - u.z : 0.f;
                a[3] = c + 3 < d ? x.w - u.w : 0.f;
            } else {
                a[0] = a[1] = a[2] = a[3] = 0.f;
            }
            T qv[4];
#pragma unroll
            for (int e = 0; e < 4; e++) {
                over |= fabsf(a[e]) > range_max;
                qv[e] = to_tile<T>(a[e]);
                const float qf = (float)qv[e];
                na = __builtin_fmaf(qf, qf, na);
                ra = __builtin_fmaf(a[e], a[e], ra);
            }
            if (live && out) {
                if constexpr (sizeof(T) == 4) {
                    *reinterpret_cast<float4 *>(out + c) = make_float4(qv[0], qv[1], qv[2], qv[3]);
                } else {
                    uint2 w;
                    __builtin_memcpy(&w, qv, sizeof(w));
                    *reinterpret_cast<uint2 *>(out + c) = w;
                }
            }
        }
        for (int o = 4; o > 0; o >>= 1) {
            na += __shfl_xor(na, o, 64);
            ra += __shfl_xor(ra, o, 64);
        }
        const uint64_t ov = (__ballot(over) >> (8 * grp)) & 0xffu;
        if (live && sub == 0) nrm[(int64_t)t * n + lf.off + i] = make_float2(na, ov ? INFINITY : sqrtf(ra));
    }
}

// The same leaf pass with the leaf's rows staged in LDS: X is read once (the two-pass
// kernel reads it once for the mean and again to centre).  One block per (leaf, tree); the
// leaf (up to ~130 KB) is loaded with every load of a thread in flight at once, since one
// block holds the CU's LDS.  The centroid is a fixed-order sum (R row classes per column,
// then the classes in order), so it is reproducible.
template <typename T, bool VEC>
__global__ __launch_bounds__(512) void k_leaf_staged(
    const float *__restrict__ X, int d, int dp, const LeafDesc *__restrict__ leaves, int nleaf,
    const int32_t *__restrict__ perm, int64_t n, int32_t *__restrict__ leaf_of,
    float *__restrict__ centroid, T *__restrict__ Xc, float2 *__restrict__ nrm, float range_max) {
    extern __shared__ __align__(16) float s_rows[];  // m rows of ds floats, centroid (ds), member ids (m)
    __shared__ float s_part[512];
    const int t = blockIdx.y, tid = threadIdx.x;
    constexpr int NT = 512, KV = 16;
    const LeafDesc lf = leaves[blockIdx.x];
    const int m = lf.size;
    const int ds = leaf_row_stride(d);
    float *s_mu = s_rows + (size_t)m * ds;
    int32_t *s_id = reinterpret_cast<int32_t *>(s_mu + ds);
    const int32_t *pp = perm + (int64_t)t * n + lf.off;
    for (int i = tid; i < m; i += NT) {
        const int id = pp[i];
        s_id[i] = id;
        leaf_of[(int64_t)t * n + id] = lf.heap;
    }
    __syncthreads();
    if constexpr (VEC) {  // 16-byte loads, KV of them in flight per thread
        const int q = d >> 2, tot = m * q;
        for (int v0 = 0; v0 < tot; v0 += NT * KV) {
            float4 r[KV];
#pragma unroll
            for (int k = 0; k < KV; k++) {  // past the end: reload the last element, not stored
                const int v = min(v0 + k * NT + tid, tot - 1);
                const int i = v / q, c = v - i * q;
                r[k] = reinterpret_cast<const float4 *>(X + (int64_t)s_id[i] * d)[c];
            }
#pragma unroll
            for (int k = 0; k < KV; k++) {
                const int v = v0 + k * NT + tid;
                const int i = v / q, c = v - i * q;
                if (v < tot) reinterpret_cast<float4 *>(s_rows + (size_t)i * ds)[c] = r[k];
            }
        }
    } else {
        const int tot = m * d;
        for (int v0 = 0; v0 < tot; v0 += NT * KV) {
            float r[KV];
#pragma unroll
            for (int k = 0; k < KV; k++) {
                const int v = min(v0 + k * NT + tid, tot - 1);
                const int i = v / d, j = v - i * d;
                r[k] = X[(int64_t)s_id[i] * d + j];
            }
#pragma unroll
            for (int k = 0; k < KV; k++) {
                const int v = v0 + k * NT + tid;
                const int i = v / d, j = v - i * d;
                if (v < tot) s_rows[(size_t)i * ds + j] = r[k];
            }
        }
    }
    __syncthreads();
    leaf_centre_staged<T>(s_rows, s_mu, s_part, m, d, ds, dp, t, blockIdx.x, nleaf, lf, n, centroid, Xc, nrm,
                          range_max);
}

// The staged leaf pass as a software pipeline: each block (one per CU: a leaf fills its LDS)
// walks the (tree, leaf) items w = blockIdx.x, + gridDim.x, ...; while it centres and writes
// item w from LDS, the rows of the next item are in flight into registers and the member ids
// of the one after are in flight too.  Needs d % 4 == 0, every leaf at most 512 members and
// at most 512 * 16 row quarters.
template <typename T>
__global__ __launch_bounds__(512) void k_leaf_pipe(
    const float *__restrict__ X, int d, int dp, const LeafDesc *__restrict__ leaves, int nleaf, int ntree,
    const int32_t *__restrict__ perm, int64_t n, int32_t *__restrict__ leaf_of,
    float *__restrict__ centroid, T *__restrict__ Xc, float2 *__restrict__ nrm, float range_max, int max_leaf) {
    extern __shared__ __align__(16) float s_rows[];  // max_leaf rows of S floats, centroid (S), ids (max_leaf)
    __shared__ float s_part[512];
    constexpr int NT = 512, KV = 16;
    const int tid = threadIdx.x, q = d >> 2, G = gridDim.x;
    const int items = nleaf * ntree;
    const int S = leaf_row_stride(d);
    float *s_mu = s_rows + (size_t)max_leaf * S;
    int32_t *s_id = reinterpret_cast<int32_t *>(s_mu + S);
    float r0[KV], r1[KV], r2[KV], r3[KV];  // the next item's row quarters (scalars stay in registers)
    // item w -> tree w / nleaf, leaf w % nleaf: neighbouring blocks take neighbouring leaves
    auto id_of = [&](int w) -> int32_t {  // member tid of item w (0 past its end)
        if (w >= items) return 0;
        const int t = w / nleaf;
        const LeafDesc lf = leaves[w - t * nleaf];
        return tid < lf.size ? perm[(int64_t)t * n + lf.off + tid] : 0;
    };
    auto stage_ids = [&](int w, int32_t id) {  // ids of item w into LDS, and its leaf_of entries
        if (w >= items) return;
        const int t = w / nleaf;
        const LeafDesc lf = leaves[w - t * nleaf];
        if (tid < lf.size) {
            s_id[tid] = id;
            leaf_of[(int64_t)t * n + id] = lf.heap;
        }
    };
    // rows of item w into registers (its ids in LDS); past the end of the leaf the last element
    // is loaded again and not stored
#define RPF_ISSUE_ROWS(W)                                                                       \
    {                                                                                           \
        const bool ok_ = (W) < items;  /* past the last item: row 0, never stored */            \
        const int tw_ = ok_ ? (W) / nleaf : 0;                                                  \
        const int tot_ = ok_ ? leaves[(W) - tw_ * nleaf].size * q : 1;                          \
        _Pragma("unroll") for (int k = 0; k < KV; k++) {                                        \
            const int v = min(k * NT + tid, tot_ - 1);                                          \
            const int i = v / q, c = v - i * q;                                                 \
            const int64_t row = ok_ ? s_id[i] : 0;                                              \
            const float4 x_ = reinterpret_cast<const float4 *>(X + row * d)[c];                 \
            r0[k] = x_.x; r1[k] = x_.y; r2[k] = x_.z; r3[k] = x_.w;                             \
        }                                                                                       \
    }
    int w = blockIdx.x;
    stage_ids(w, id_of(w));
    __syncthreads();
    RPF_ISSUE_ROWS(w)
    int32_t idn = id_of(w + G);
    for (; w < items; w += G) {
        const int t = w / nleaf, leaf = w - t * nleaf;
        const LeafDesc lf = leaves[leaf];
        const int m = lf.size, tot = m * q;
        __syncthreads();  // the previous item is done with s_rows and s_id
#pragma unroll
        for (int k = 0; k < KV; k++) {
            const int v = k * NT + tid;
            const int i = v / q, c = v - i * q;
            if (v < tot) reinterpret_cast<float4 *>(s_rows + (size_t)i * S)[c] = make_float4(r0[k], r1[k], r2[k], r3[k]);
        }
        stage_ids(w + G, idn);
        __syncthreads();
        RPF_ISSUE_ROWS(w + G)  // in flight while item w is centred
        idn = id_of(w + 2 * G);
        leaf_centre_staged<T>(s_rows, s_mu, s_part, m, d, S, dp, t, leaf, nleaf, lf, n, centroid, Xc, nrm,
                              range_max);
    }
#undef RPF_ISSUE_ROWS
}

size_t leaf_staged_lds(int d, int max_leaf) {  // dynamic part; 2 KB of static LDS come on top
    return sizeof(float) * (size_t)leaf_row_stride(d) * ((size_t)max_leaf + 1) + sizeof(int32_t) * (size_t)max_leaf;
}

template <typename T>
static void leaf_staged(hipStream_t s, dim3 grid, size_t lds, bool vec, const float *X, int d, int dp,
                        const LeafDesc *leaves, int nleaf, const int32_t *perm, int64_t n, int32_t *leaf_of,
                        float *centroid, void *Xc, float2 *nrm, float range_max) {
    if (vec) {
        hipFuncSetAttribute((const void *)k_leaf_staged<T, true>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        hipLaunchKernelGGL((k_leaf_staged<T, true>), grid, dim3(512), lds, s, X, d, dp, leaves, nleaf, perm, n, leaf_of,
                           centroid, (T *)Xc, nrm, range_max);
    } else {
        hipFuncSetAttribute((const void *)k_leaf_staged<T, false>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        hipLaunchKernelGGL((k_leaf_staged<T, false>), grid, dim3(512), lds, s, X, d, dp, leaves, nleaf, perm, n,
                           leaf_of, centroid, (T *)Xc, nrm, range_max);
    }
    launch_check(s, "k_leaf_staged");
}

template <typename T>
static void leaf_pipe(hipStream_t s, size_t lds, const float *X, int d, int dp, const LeafDesc *leaves, int nleaf,
                      int ntree, const int32_t *perm, int64_t n, int32_t *leaf_of, float *centroid, void *Xc,
                      float2 *nrm, float range_max, int max_leaf) {
    hipFuncSetAttribute((const void *)k_leaf_pipe<T>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    int dev = 0, cus = 0, per = 0;
    hipGetDevice(&dev);
    hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, (const void *)k_leaf_pipe<T>, 512, lds);
    const int64_t items = (int64_t)nleaf * ntree;
    const int grid = (int)std::max<int64_t>(1, std::min<int64_t>(items, (int64_t)std::max(cus, 1) * std::max(per, 1)));
    hipLaunchKernelGGL(k_leaf_pipe<T>, dim3(grid), dim3(512), lds, s, X, d, dp, leaves, nleaf, ntree, perm, n, leaf_of,
                       centroid, (T *)Xc, nrm, range_max, max_leaf);
    launch_check(s, "k_leaf_pipe");
}

template <typename T>
static void leaf_finalize(hipStream_t s, dim3 grid, size_t lds, const float *X, int d, int dp,
                          const LeafDesc *leaves, int nleaf, const int32_t *perm, int64_t n, int32_t *leaf_of,
                          float *centroid, void *Xc, float2 *nrm, float range_max, int ids_in_lds) {
    hipFuncSetAttribute((const void *)k_leaf_finalize<T>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    hipLaunchKernelGGL(k_leaf_finalize<T>, grid, dim3(256), lds, s, X, d, dp, leaves, nleaf, perm, n, leaf_of,
                       centroid, (T *)Xc, nrm, range_max, ids_in_lds);
    launch_check(s, "k_leaf_finalize");
}

size_t leaf_finalize_lds(int dp, int max_leaf, bool ids) {
    return sizeof(float) * 5 * (size_t)dp + (ids ? sizeof(int32_t) * (size_t)max_leaf : 0);
}

void launch_leaf_finalize(hipStream_t s, int prec, const float *X, int d, int dp, const LeafDesc *leaves,
                          int nleaf, int T, const int32_t *perm, int64_t n, int32_t *leaf_of, float *centroid,
                          void *Xc, float2 *nrm, int max_leaf, int lds_limit) {
    dim3 grid(nleaf, T);
    const size_t piped = sizeof(float) * (size_t)leaf_row_stride(d) * ((size_t)max_leaf + 1) +
                         sizeof(int32_t) * (size_t)max_leaf;
    if (d % 4 == 0 && max_leaf <= 512 && max_leaf * (d / 4) <= 512 * 16 && piped + 2048 <= (size_t)lds_limit &&
        (int64_t)nleaf * T < (1ll << 31)) {  // a leaf fits a block's registers and LDS: pipelined
        if (prec == RPF_DIST_BF16)
            leaf_pipe<__bf16>(s, piped, X, d, dp, leaves, nleaf, T, perm, n, leaf_of, centroid, Xc, nrm, 3.0e38f,
                              max_leaf);
        else if (prec == RPF_DIST_FP16)
            leaf_pipe<_Float16>(s, piped, X, d, dp, leaves, nleaf, T, perm, n, leaf_of, centroid, Xc, nrm, 60000.f,
                                max_leaf);
        else
            leaf_pipe<float>(s, piped, X, d, dp, leaves, nleaf, T, perm, n, leaf_of, centroid, Xc, nrm, 3.0e38f,
                             max_leaf);
        return;
    }
    const size_t staged = leaf_staged_lds(d, max_leaf);
    if (staged + 2048 <= (size_t)lds_limit) {  // the leaf's rows fit in LDS: read X once
        const bool vec = (d % 4) == 0;
        if (prec == RPF_DIST_BF16)
            leaf_staged<__bf16>(s, grid, staged, vec, X, d, dp, leaves, nleaf, perm, n, leaf_of, centroid, Xc, nrm, 3.0e38f);
        else if (prec == RPF_DIST_FP16)
            leaf_staged<_Float16>(s, grid, staged, vec, X, d, dp, leaves, nleaf, perm, n, leaf_of, centroid, Xc, nrm,
                                  60000.f);
        else
            leaf_staged<float>(s, grid, staged, vec, X, d, dp, leaves, nleaf, perm, n, leaf_of, centroid, Xc, nrm, 3.0e38f);
        return;
    }
    const int ids = leaf_finalize_lds(dp, max_leaf, true) <= (size_t)lds_limit ? 1 : 0;
    const size_t lds = leaf_finalize_lds(dp, max_leaf, ids != 0);
    if (prec == RPF_DIST_BF16)
        leaf_finalize<__bf16>(s, grid, lds, X, d, dp, leaves, nleaf, perm, n, leaf_of, centroid, Xc, nrm, 3.0e38f, ids);
    else if (prec == RPF_DIST_FP16)
        leaf_finalize<_Float16>(s, grid, lds, X, d, dp, leaves, nleaf, perm, n, leaf_of, centroid, Xc, nrm, 60000.f,
                                ids);
    else
        leaf_finalize<float>(s, grid, lds, X, d, dp, leaves, nleaf, perm, n, leaf_of, centroid, Xc, nrm, 3.0e38f, ids);
}

}  // namespace rpf
