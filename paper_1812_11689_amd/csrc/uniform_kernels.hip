// Tree growth by the uniform split rule that Alg. 1 prints: at a node W the split point c is
// drawn uniformly between a = min and b = max of the members' projections onto the node's
// direction (Alg. 2 picks that direction among nTry random ones), W_L = {p < c} and
// W_R = {p >= c}.  The shape of a tree now depends on the data, so growth is
// level-synchronous over a frontier the host keeps: one level splits every open node of
// every tree in a handful of launches, and the host reads back the left sizes to open the
// next level.
//
// Random numbers.  A node's draws cannot be laid out in advance as the median rule's
// direction array is, so they come from a counter-based generator keyed by (seed, tree, heap
// id of the node): SplitMix64 (Steele, Lea and Flood, "Fast splittable pseudorandom number
// generators", OOPSLA 2014), whose stream with seed s has the outputs
// out(s, i) = mix64(s + (i + 1) GAMMA).  The node's stream has the seed out(out(seed, t), h);
// its draw 0 gives the split fraction u = (draw >> 11) 2^-53 in [0, 1), and coordinate j of
// direction try i is (sum of the 32-bit halves of draws 1 + 6 (i d + j) + q, q < 6) 2^-32 - 6,
// exact in binary64 and rounded once to binary32 (Irwin-Hall: mean 0, variance 1).
// c = RN(a + RN(u RN(b - a))).  A node with an empty child stays whole, as a leaf; nodes at
// depth kUniformDepth are not split (heap ids stay below 2^63).
//
// With one direction per node, nodes of at most kGrowBlock members leave this loop and are grown
// to their leaves on the device (below).  Two paths per level, both writing the node's
// permutation range in place (stable: both
// children keep ascending original index):
//   - nodes of at most kChunk members: one block per node does the whole step in LDS
//     (k_uni_block);
//   - larger nodes: chunks of kChunk positions, aligned at the node's first position, with
//     projections stored in binary64 ([n_try][T n]), the canonical sums of Alg. 2 combined
//     from aligned power-of-two chunk partials (the same balanced tree as one canonical sum),
//     then a stable count / offsets / scatter partition through a scratch permutation.
#include <algorithm>

#include "rpf_internal.h"

namespace rpf {

// ---------------------------------------------------------------- the generator

constexpr uint64_t kSmGamma = 0x9E3779B97F4A7C15ull;

__host__ __device__ inline uint64_t sm64_mix(uint64_t z) {
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

__host__ __device__ inline uint64_t sm64_at(uint64_t seed, uint64_t i) { return sm64_mix(seed + (i + 1) * kSmGamma); }

__host__ __device__ inline uint64_t uni_node_seed(uint64_t seed, int t, int64_t heap) {
    return sm64_at(sm64_at(seed, (uint64_t)t), (uint64_t)heap);
}

__device__ inline double uni_fraction(uint64_t key) { return (double)(sm64_at(key, 0) >> 11) * 0x1p-53; }

__device__ inline float uni_coord(uint64_t key, int tr, int d, int j) {
    const uint64_t base = 1 + 6 * ((uint64_t)tr * (uint64_t)d + (uint64_t)j);
    uint64_t s = 0;
#pragma unroll
    for (int q = 0; q < 6; q++) {
        const uint64_t w = sm64_at(key, base + q);
        s += (w >> 32) + (w & 0xffffffffull);
    }
    // (double)s is exact (s < 12 * 2^32), the scaling and the shift by 6 too
    return (float)__dsub_rn(__dmul_rn((double)s, 0x1p-32), 6.0);
}

__device__ inline double uni_split_point(double a, double b, double u) {
    return __dadd_rn(a, __dmul_rn(u, __dsub_rn(b, a)));
}

// ---------------------------------------------------------------- block helpers

// exclusive scan of one flag per thread over an NT-thread block (NT a multiple of 64);
// s_w needs NT / 64 words
template <int NT>
__device__ inline void block_flag_scan(bool f, uint32_t *s_w, uint32_t &excl, uint32_t &total) {
    const uint64_t b = __ballot(f);
    const uint32_t inw = (uint32_t)mask_rank(b);
    if (NT == 64) {
        excl = inw;
        total = (uint32_t)__popcll(b);
        return;
    }
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) s_w[w] = (uint32_t)__popcll(b);
    __syncthreads();
    uint32_t wb = 0, tot = 0;
#pragma unroll
    for (int k = 0; k < NT / 64; k++) {
        const uint32_t c = s_w[k];
        if (k < w) wb += c;
        tot += c;
    }
    excl = wb + inw;
    total = tot;
    __syncthreads();
}

// min and max over the block (exact in any order); s_r needs 2 NT / 64 doubles
template <int NT>
__device__ inline void block_minmax(double &lo, double &hi, double *s_r) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        lo = fmin(lo, shfl_xor_d(lo, o));
        hi = fmax(hi, shfl_xor_d(hi, o));
    }
    if (NT == 64) return;
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        s_r[w] = lo;
        s_r[NT / 64 + w] = hi;
    }
    __syncthreads();
    lo = s_r[0];
    hi = s_r[NT / 64];
#pragma unroll
    for (int k = 1; k < NT / 64; k++) {
        lo = fmin(lo, s_r[k]);
        hi = fmax(hi, s_r[NT / 64 + k]);
    }
    __syncthreads();
}

template <int NT>
__device__ inline uint32_t block_count(uint32_t v, uint32_t *s_w) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    if (NT == 64) return v;
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) s_w[w] = v;
    __syncthreads();
    uint32_t t = 0;
#pragma unroll
    for (int k = 0; k < NT / 64; k++) t += s_w[k];
    __syncthreads();
    return t;
}

// ---------------------------------------------------------------- nodes of at most kChunk members

size_t uni_block_lds(int max_m, int d, int n_try) {
    int P2 = 2;
    while (P2 < max_m) P2 <<= 1;
    const size_t ds = (size_t)((d + 3) & ~3);
    return (size_t)P2 * 8 * (n_try > 1 ? 3 : 1) + ds * 4 + (size_t)((max_m + 3) & ~3) * 4 + 256;
}

// LDS: p[P2] | (nTry > 1) work[P2], best[P2] | direction[ds] | ids[m] | reductions
template <int NT, bool VEC>
__global__ __launch_bounds__(NT) void k_uni_block(const float *__restrict__ X, int d, int n_try, uint64_t seed,
                                                  const UniSeg *__restrict__ segs, int32_t *__restrict__ perm,
                                                  UniSplit *__restrict__ out) {
    extern __shared__ __align__(16) uint8_t smem[];
    const UniSeg sg = segs[blockIdx.x];
    const int m = sg.size, tid = threadIdx.x;
    int P2 = 2;
    while (P2 < m) P2 <<= 1;
    const int ds = (d + 3) & ~3;
    double *s_p = reinterpret_cast<double *>(smem);
    double *s_work = s_p + P2;
    double *s_best = s_work + P2;
    float *s_dir = reinterpret_cast<float *>(n_try > 1 ? s_best + P2 : s_p + P2);
    int32_t *s_ids = reinterpret_cast<int32_t *>(s_dir + ds);
    double *s_red = reinterpret_cast<double *>(s_ids + ((m + 3) & ~3));
    uint32_t *s_w = reinterpret_cast<uint32_t *>(s_red + 2 * (NT / 64));

    int32_t *pg = perm + sg.pos;
    for (int i = tid; i < m; i += NT) s_ids[i] = pg[i];
    const uint64_t key = uni_node_seed(seed, sg.tree, sg.heap);
    const int g = tid & 7, pt = tid >> 3;
    double best = 0.0;
    int best_i = -1;
    for (int tr = 0; tr < n_try; tr++) {
        __syncthreads();  // the previous try is done with the direction
        for (int j = tid; j < ds; j += NT) s_dir[j] = j < d ? uni_coord(key, tr, d, j) : 0.f;
        __syncthreads();
        for (int base = 0; base < m; base += NT / 4) {  // rows base + pt and base + NT / 8 + pt
            const int ia = base + pt, ib = ia + NT / 8;
            double pa, pb;
            group8_dot64r2<VEC>(X + (int64_t)s_ids[ia < m ? ia : 0] * d, X + (int64_t)s_ids[ib < m ? ib : 0] * d,
                                s_dir, d, g, pa, pb);
            if (g == 0 && ia < m) s_p[ia] = pa;
            if (g == 0 && ib < m) s_p[ib] = pb;
        }
        __syncthreads();
        if (n_try == 1) break;
        // Alg. 2: keep the try with the largest spread S2 (the first wins ties; try 0 when no
        // try has any spread)
        for (int i = tid; i < m; i += NT) s_work[i] = s_p[i];
        const double mu = block_canon_sum(s_work, m) / (double)m;
        for (int i = tid; i < m; i += NT) {
            const double dev = __dsub_rn(s_p[i], mu);
            s_work[i] = __dmul_rn(dev, dev);
        }
        const double s2 = block_canon_sum(s_work, m);
        if (tr == 0 || s2 > best)
            for (int i = tid; i < m; i += NT) s_best[i] = s_p[i];
        if (s2 > best) {
            best = s2;
            best_i = tr;
        }
    }
    __syncthreads();
    const double *P = n_try > 1 ? s_best : s_p;
    double lo = INFINITY, hi = -INFINITY;
    for (int i = tid; i < m; i += NT) {
        lo = fmin(lo, P[i]);
        hi = fmax(hi, P[i]);
    }
    block_minmax<NT>(lo, hi, s_red);
    const double c = uni_split_point(lo, hi, uni_fraction(key));
    uint32_t nl = 0;
    for (int i = tid; i < m; i += NT) nl += P[i] < c ? 1u : 0u;
    nl = block_count<NT>(nl, s_w);
    uint32_t lefts = 0;
    for (int base = 0; base < m; base += NT) {
        const int i = base + tid;
        const bool valid = i < m;
        const bool left = valid && P[i] < c;
        uint32_t excl, total;
        block_flag_scan<NT>(left, s_w, excl, total);
        if (valid) {
            const uint32_t lb = lefts + excl;
            pg[left ? lb : nl + (uint32_t)i - lb] = s_ids[i];
        }
        lefts += total;
    }
    if (tid == 0) out[blockIdx.x] = UniSplit{c, (int32_t)nl, best_i < 0 ? 0 : best_i};
}

// ---------------------------------------------------------------- nodes above kChunk members

// projections of a chunk onto every try (stored), the chunk's min / max per try and, with
// more than one try, its partial canonical sum per try
// (one try and up to 512 chunks, which leave the chip idle: 1024 threads a chunk, 54 -> 24 us a
// level at 100 000 x 32; at 800 chunks 63 -> 78, so no more; several tries sum 4096 squares by
// 256 threads)
template <bool VEC, int NT>
__global__ __launch_bounds__(NT) void k_uni_proj(const float *__restrict__ X, int d, int n_try, uint64_t seed,
                                                  const UniSeg *__restrict__ segs,
                                                  const UniChunk *__restrict__ chunks,
                                                  const int32_t *__restrict__ perm, int64_t TN,
                                                  double *__restrict__ P, double *__restrict__ part,
                                                  double2 *__restrict__ mm) {
    __shared__ __align__(16) float s_dir[4096];
    __shared__ double s_red[2 * (NT / 64)];
    extern __shared__ double s_p[];  // kChunk projections of the chunk, only for several tries
    const UniChunk c = chunks[blockIdx.x];
    const UniSeg sg = segs[c.seg];
    const int tid = threadIdx.x, g = tid & 7, pt = tid >> 3;
    const int ds = (d + 3) & ~3;
    const uint64_t key = uni_node_seed(seed, sg.tree, sg.heap);
    for (int tr = 0; tr < n_try; tr++) {
        __syncthreads();
        for (int j = tid; j < ds; j += NT) s_dir[j] = j < d ? uni_coord(key, tr, d, j) : 0.f;
        __syncthreads();
        double lo = INFINITY, hi = -INFINITY;
        for (int base = 0; base < c.len; base += NT / 4) {
            const int ia = base + pt, ib = ia + NT / 8;
            const int32_t ida = perm[c.pos + (ia < c.len ? ia : 0)];
            const int32_t idb = perm[c.pos + (ib < c.len ? ib : 0)];
            double p2[2];
            group8_dot64r2<VEC>(X + (int64_t)ida * d, X + (int64_t)idb * d, s_dir, d, g, p2[0], p2[1]);
#pragma unroll
            for (int h = 0; h < 2; h++) {
                const int i = h ? ib : ia;
                const double p = p2[h];
                if (g == 0 && i < c.len) {
                    P[(int64_t)tr * TN + c.pos + i] = p;
                    if (n_try > 1) s_p[i] = p;
                    lo = fmin(lo, p);
                    hi = fmax(hi, p);
                }
            }
        }
        block_minmax<NT>(lo, hi, s_red);
        if (tid == 0) mm[(int64_t)blockIdx.x * n_try + tr] = make_double2(lo, hi);
        if (NT == 256 && n_try > 1) {
            const double sum = block_canon_sum(s_p, c.len);  // syncs before reading s_p
            if (tid == 0) part[(int64_t)blockIdx.x * n_try + tr] = sum;
        }
    }
}

// in-place balanced tree over the partials v[0], v[stride], ... of nc chunks: the canonical
// sum of the whole node (a missing right operand is the +0.0 padding)
__device__ inline double chunk_tree(double *v, int nc, int stride) {
    for (int h = 1; h < nc; h <<= 1)
        for (int i = 0; i + h < nc; i += 2 * h) v[(int64_t)i * stride] = v[(int64_t)i * stride] + v[(int64_t)(i + h) * stride];
    return v[0];
}

// per (node, try): the mean of the projections
__global__ void k_uni_mean(const UniSeg *__restrict__ segs, int nseg, int n_try, double *__restrict__ part,
                           double *__restrict__ mu) {
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= (int64_t)nseg * n_try) return;
    const int sgi = (int)(k / n_try), tr = (int)(k % n_try);
    const UniSeg sg = segs[sgi];
    const double s1 = chunk_tree(part + (int64_t)sg.chunk0 * n_try + tr, sg.nchunk, n_try);
    mu[k] = s1 / (double)sg.size;
}

// partial canonical sums of (p - mean)^2 per (chunk, try)
__global__ __launch_bounds__(256) void k_uni_disp(const UniSeg *__restrict__ segs, const UniChunk *__restrict__ chunks,
                                                  int n_try, int64_t TN, const double *__restrict__ P,
                                                  const double *__restrict__ mu, double *__restrict__ part) {
    __shared__ double s_v[kChunk];
    const UniChunk c = chunks[blockIdx.x];
    for (int tr = 0; tr < n_try; tr++) {
        const double m = mu[(int64_t)c.seg * n_try + tr];
        __syncthreads();
        for (int i = threadIdx.x; i < c.len; i += 256) {
            const double dev = __dsub_rn(P[(int64_t)tr * TN + c.pos + i], m);
            s_v[i] = __dmul_rn(dev, dev);
        }
        const double sum = block_canon_sum(s_v, c.len);
        if (threadIdx.x == 0) part[(int64_t)blockIdx.x * n_try + tr] = sum;
    }
}

// per node: the try (Alg. 2), a and b of its projections, and the split point
__global__ void k_uni_decide(const UniSeg *__restrict__ segs, int nseg, int n_try, uint64_t seed,
                             double *__restrict__ part, const double2 *__restrict__ mm, UniSplit *__restrict__ out) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= nseg) return;
    const UniSeg sg = segs[k];
    int ch = 0;
    if (n_try > 1) {
        double best = 0.0;
        int best_i = -1;
        for (int tr = 0; tr < n_try; tr++) {
            const double s2 = chunk_tree(part + (int64_t)sg.chunk0 * n_try + tr, sg.nchunk, n_try);
            if (s2 > best) {
                best = s2;
                best_i = tr;
            }
        }
        ch = best_i < 0 ? 0 : best_i;
    }
    double lo = INFINITY, hi = -INFINITY;
    for (int q = 0; q < sg.nchunk; q++) {
        const double2 v = mm[(int64_t)(sg.chunk0 + q) * n_try + ch];
        lo = fmin(lo, v.x);
        hi = fmax(hi, v.y);
    }
    const uint64_t key = uni_node_seed(seed, sg.tree, sg.heap);
    out[k] = UniSplit{uni_split_point(lo, hi, uni_fraction(key)), 0, ch};
}

__global__ __launch_bounds__(256) void k_uni_count(const UniChunk *__restrict__ chunks, int64_t TN,
                                                   const double *__restrict__ P, const UniSplit *__restrict__ sp,
                                                   uint32_t *__restrict__ lcount) {
    __shared__ uint32_t s_w[4];
    const UniChunk c = chunks[blockIdx.x];
    const UniSplit q = sp[c.seg];
    const double *p = P + (int64_t)q.chosen * TN + c.pos;
    uint32_t v = 0;
    for (int i = threadIdx.x; i < c.len; i += 256) v += p[i] < q.c ? 1u : 0u;
    v = block_count<256>(v, s_w);
    if (threadIdx.x == 0) lcount[blockIdx.x] = v;
}

// per node: left positions before each chunk, and the node's left size
__global__ void k_uni_offsets(const UniSeg *__restrict__ segs, int nseg, const uint32_t *__restrict__ lcount,
                              uint32_t *__restrict__ loff, UniSplit *__restrict__ sp) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= nseg) return;
    const UniSeg sg = segs[k];
    uint32_t run = 0;
    for (int q = 0; q < sg.nchunk; q++) {
        loff[sg.chunk0 + q] = run;
        run += lcount[sg.chunk0 + q];
    }
    sp[k].nl = (int32_t)run;
}

// stable partition of a chunk into the scratch permutation
__global__ __launch_bounds__(256) void k_uni_scatter(const UniSeg *__restrict__ segs,
                                                     const UniChunk *__restrict__ chunks, int64_t TN,
                                                     const double *__restrict__ P, const UniSplit *__restrict__ sp,
                                                     const uint32_t *__restrict__ loff, const int32_t *__restrict__ perm,
                                                     int32_t *__restrict__ tmp) {
    __shared__ uint32_t s_w[4];
    const UniChunk c = chunks[blockIdx.x];
    const UniSeg sg = segs[c.seg];
    const UniSplit q = sp[c.seg];
    const double *p = P + (int64_t)q.chosen * TN + c.pos;
    const int64_t within = c.pos - sg.pos;  // chunk's first position inside the node
    const uint32_t lo0 = loff[blockIdx.x];
    uint32_t lefts = 0;
    for (int base = 0; base < c.len; base += 256) {
        const int i = base + threadIdx.x;
        const bool valid = i < c.len;
        const bool left = valid && p[i] < q.c;
        uint32_t excl, total;
        block_flag_scan<256>(left, s_w, excl, total);
        if (valid) {
            const int64_t lb = (int64_t)lo0 + lefts + excl;  // lefts before this element in the node
            const int64_t dst = left ? lb : (int64_t)q.nl + within + i - lb;
            tmp[sg.pos + dst] = perm[c.pos + i];
        }
        lefts += total;
    }
}

__global__ __launch_bounds__(256) void k_uni_copy(const UniChunk *__restrict__ chunks, const int32_t *__restrict__ tmp,
                                                  int32_t *__restrict__ perm) {
    const UniChunk c = chunks[blockIdx.x];
    for (int i = threadIdx.x; i < c.len; i += 256) perm[c.pos + i] = tmp[c.pos + i];
}

// ---------------------------------------------------------------- whole subtrees on the device
//
// Nodes of at most kGrowBlock members leave the host's level loop: a workgroup grows the node's
// subtree in LDS, depth first, down to nodes of at most kGrowWave members, and one-wave
// workgroups grow those to their leaves, work lists drained through a counter.  One direction
// per node.  Each node is the same step as k_uni_block (projections, extremes, split point,
// stable partition).  Before, every level of every tree cost launches, two copies and a host
// wait (about 60 levels at 100 000 x 32, 32 trees, leaves of at most 64: build 19.5 ms, now
// 6.6, of which 0.86 and 0.87 in the two sizes here and 4.5 in the 25 levels above them).
// Bound: the latency of one node's chain of steps; a uniform split often takes a few members
// off a node, so subtrees are up to 62 levels deep.  kGrowWave of 512 was slower (block size
// 1.36 ms), workgroups of 128 or 256 threads in place of the waves gave nothing.

struct GrowSeg {
    int32_t off, size, depth, small;
    int64_t heap;
};

constexpr int kRecStage = 32;
static_assert(sizeof(UniRec) == 48, "flushed as three int4");

using AliasInt = int32_t __attribute__((may_alias));

size_t uni_grow_lds(int cap, int d) { return (size_t)cap * 12 + (size_t)((d + 3) & ~3) * 4; }

template <int NT, int CAP, bool VEC>
__global__ __launch_bounds__(NT) void k_uni_grow(const float *__restrict__ X, int d, uint64_t seed,
                                                 const UniSeg *__restrict__ items, const uint32_t *__restrict__ count,
                                                 uint32_t most, uint32_t *__restrict__ next, int stop, int n0, int small_max,
                                                 int32_t *__restrict__ perm, UniRec *__restrict__ recs,
                                                 uint32_t *__restrict__ rec_cnt, uint32_t rec_cap,
                                                 int32_t *__restrict__ mark, UniSeg *__restrict__ more,
                                                 uint32_t *__restrict__ more_cnt, uint32_t more_cap) {
    extern __shared__ __align__(16) uint8_t smem[];
    double *s_p = reinterpret_cast<double *>(smem);               // [CAP]
    int32_t *s_id = reinterpret_cast<int32_t *>(s_p + CAP);       // [CAP]
    float *s_dir = reinterpret_cast<float *>(s_id + CAP);         // [d up to a multiple of four]
    __shared__ GrowSeg s_stack[32];  // the larger child waits: at most log2(CAP) + 1 entries
    __shared__ double s_red[2 * (NT / 64)];
    __shared__ uint32_t s_w[NT / 64];
    __shared__ uint32_t s_item, s_base;
    __shared__ __align__(16) UniRec s_rec[kRecStage];
    int nrec = 0;  // records staged: one atomic per kRecStage (one each: 150 000 of them took 1.6 ms)
    const int tid = threadIdx.x, g = tid & 7, pt = tid >> 3;
    const int ds = (d + 3) & ~3;
    const uint32_t nitems = min(*count, most);
    auto flush = [&]() {
        __syncthreads();
        if (tid == 0) s_base = atomicAdd(rec_cnt, (uint32_t)nrec);
        __syncthreads();
        const int4 *from = reinterpret_cast<const int4 *>(s_rec);
        int4 *to = reinterpret_cast<int4 *>(recs);
        for (int i = tid; i < 3 * nrec; i += NT)  // (a record: three times 16 bytes)
            if (s_base + i / 3 < rec_cap) to[3 * (size_t)s_base + i] = from[i];
        __syncthreads();
        nrec = 0;
    };
    for (;;) {  // ends when the list is drained
        __syncthreads();
        if (tid == 0) s_item = atomicAdd(next, 1u);
        __syncthreads();
        if (s_item >= nitems) break;
        const UniSeg sg = items[s_item];
        int32_t *pg = perm + sg.pos;
        for (int i = tid; i < sg.size; i += NT) s_id[i] = pg[i];
        if (tid == 0) s_stack[0] = GrowSeg{0, sg.size, sg.chunk0, sg.nchunk, sg.heap};
        int sp = 1;
        while (sp > 0) {
            __syncthreads();
            const GrowSeg c = s_stack[--sp];
            const uint64_t key = uni_node_seed(seed, sg.tree, c.heap);
            for (int j = tid; j < ds; j += NT) s_dir[j] = j < d ? uni_coord(key, 0, d, j) : 0.f;
            __syncthreads();
            const int m = c.size;
            int32_t *ids = s_id + c.off;
            double *P = s_p + c.off;
            for (int base = 0; base < m; base += NT / 2) {  // four rows per eight lanes in flight
                const float *x[4];
                double pr[4];
#pragma unroll
                for (int k = 0; k < 4; k++) {
                    const int i = base + k * (NT / 8) + pt;
                    x[k] = X + (int64_t)ids[i < m ? i : 0] * d;
                }
                group8_dots<VEC, 1, 4>(x, s_dir, 0, d, g, pr);
                const int i = base + (g & 3) * (NT / 8) + pt;
                if (g < 4 && i < m) P[i] = g == 0 ? pr[0] : g == 1 ? pr[1] : g == 2 ? pr[2] : pr[3];
            }
            __syncthreads();
            double lo = INFINITY, hi = -INFINITY;
            for (int i = tid; i < m; i += NT) {
                lo = fmin(lo, P[i]);
                hi = fmax(hi, P[i]);
            }
            block_minmax<NT>(lo, hi, s_red);
            const double cc = uni_split_point(lo, hi, uni_fraction(key));
            uint32_t nl = 0;
            for (int i = tid; i < m; i += NT) nl += P[i] < cc ? 1u : 0u;
            nl = block_count<NT>(nl, s_w);
            const bool whole = nl == 0 || nl == (uint32_t)m;
            if (!whole) {
                // stable, in place: left members move down among those already read, right
                // members wait where the projections before them stood
                AliasInt *wait = reinterpret_cast<AliasInt *>(P);
                uint32_t lefts = 0;
                for (int base = 0; base < m; base += NT) {
                    const int i = base + tid;
                    const bool valid = i < m, left = valid && P[i] < cc;
                    const int32_t id = valid ? ids[i] : 0;
                    uint32_t excl, total;
                    block_flag_scan<NT>(left, s_w, excl, total);
                    if (valid) {
                        const uint32_t lb = lefts + excl;
                        if (left) ids[lb] = id;
                        else wait[(uint32_t)i - lb] = id;
                    }
                    lefts += total;
                }
                __syncthreads();
                for (int i = tid; i < m - (int)nl; i += NT) ids[nl + i] = wait[i];
            }
            __syncthreads();
            // the children: a leaf and a node for the next list go back to the permutation, a
            // node to split here on the stack, the smaller one on top
            auto settle = [&](int off, int size, int64_t heap, int depth) {
                const int small = c.small < kRecLarge ? c.small : size <= small_max ? depth : kRecLarge;
                const bool leaf = whole || size <= n0 || depth >= kUniformDepth;
                if (!leaf && size > stop) {
                    if (tid == 0) s_stack[sp] = GrowSeg{off, size, depth, small, heap};
                    sp++;
                    return;
                }
                const int32_t *src = s_id + off;
                for (int i = tid; i < size; i += NT) pg[off + i] = src[i];
                if (tid) return;
                if (leaf) {
                    mark[sg.pos + off] = size;
                } else {
                    const uint32_t at = atomicAdd(more_cnt, 1u);
                    if (at < more_cap) more[at] = UniSeg{sg.pos + off, heap, size, sg.tree, depth, small};
                }
            };
            if (whole) {
                settle(c.off, m, c.heap, c.depth);
            } else {
                const int a = (int)nl, b = m - a;
                const bool left_first = a >= b;
                for (int k = 0; k < 2; k++) {
                    const bool left = (k == 0) == left_first;
                    settle(left ? c.off : c.off + a, left ? a : b, 2 * c.heap + (left ? 0 : 1), c.depth + 1);
                }
            }
            if (tid == 0) s_rec[nrec] = UniRec{c.heap, cc, sg.pos + c.off, m, (int32_t)nl, 0, c.depth, sg.tree, c.small};
            if (++nrec == kRecStage) flush();
        }
    }
    flush();
}

// leaves that the host's levels closed
__global__ void k_uni_mark(const UniSeg *__restrict__ leaves, int count, int32_t *__restrict__ mark) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) mark[leaves[i].pos] = leaves[i].size;
}

// The leaf pass's tables are made by several workgroups per tree, each for the leaves that start
// in its range of positions, about 512 in all (build of one tree of 10^7 x 16, leaves of 64: 113 ms
// with one workgroup, 61 with these, 103 level by level from the host).  The jobs of a leaf of many
// tiles are written by its whole workgroup (one leaf of 200 000 copies: 82 ms by one lane, 49, 61).

// per range: leaves, tile jobs with tiles of `TR` rows, members, squared sizes, the largest leaf
__global__ __launch_bounds__(1024) void k_uni_leaf_count(const int32_t *__restrict__ mark, int64_t n, int64_t len, int TR,
                                                         UniTree *__restrict__ out) {
    __shared__ unsigned long long s_v[5];
    const int32_t *mk = mark + blockIdx.y * n;
    if (threadIdx.x < 5) s_v[threadIdx.x] = 0;
    __syncthreads();
    unsigned long long leaves = 0, jobs = 0, pts = 0, sq = 0, most = 0;
    const int64_t end = min(n, (blockIdx.x + 1) * len);
    for (int64_t i = blockIdx.x * len + threadIdx.x; i < end; i += 1024) {
        const unsigned long long v = (unsigned long long)mk[i];
        if (!v) continue;
        const unsigned long long nt = (v + TR - 1) / TR;
        leaves++;
        jobs += nt * nt;
        pts += v;
        sq += v * v;
        most = v > most ? v : most;
    }
    atomicAdd(&s_v[0], leaves);
    atomicAdd(&s_v[1], jobs);
    atomicAdd(&s_v[2], pts);
    atomicAdd(&s_v[3], sq);
    atomicMax(&s_v[4], most);
    __syncthreads();
    if (threadIdx.x == 0)
        out[blockIdx.y * (int64_t)gridDim.x + blockIdx.x] = UniTree{(int64_t)s_v[0], (int64_t)s_v[1], (int64_t)s_v[2], (int64_t)s_v[3], (int64_t)s_v[4]};
}

// the leaf table and the tile jobs, left to right
__global__ __launch_bounds__(1024) void k_uni_leaf_fill(const int32_t *__restrict__ mark, int64_t n, int64_t len, int TR,
                                                        int64_t stride, const UniPart *__restrict__ parts,
                                                        LeafDesc *__restrict__ table, TileJob *__restrict__ jobs,
                                                        int32_t *__restrict__ ident) {
    constexpr uint32_t kMany = 8;  // tiles across a leaf above which the workgroup writes its jobs together
    __shared__ uint32_t s_w[16];
    __shared__ uint32_t s_big[3];
    const int t = blockIdx.y, tid = threadIdx.x;
    const int32_t *mk = mark + t * n;
    LeafDesc *tab = table + t * stride;
    const UniPart pt = parts[t * (int64_t)gridDim.x + blockIdx.x];
    TileJob *out = jobs + pt.job;
    int64_t at = pt.leaf, jat = 0;
    const int64_t end = min(n, (blockIdx.x + 1) * len);
    for (int64_t base = blockIdx.x * len; base < end; base += 1024) {
        const int32_t v = base + tid < end ? mk[base + tid] : 0;
        const uint32_t nt = (uint32_t)((v + TR - 1) / TR);
        uint32_t e1, t1, e2, t2;
        block_excl_scan_w<16>(v ? 1u : 0u, s_w, e1, t1);
        block_excl_scan_w<16>(nt * nt, s_w, e2, t2);
        auto job = [&](int64_t off, int32_t m, int32_t leaf, uint32_t I, uint32_t J) {
            return TileJob{off + (int64_t)I * TR, off + (int64_t)J * TR, min(TR, m - (int)I * TR), min(TR, m - (int)J * TR),
                           t, I == J ? 1 : 0, (int)J * TR, m, leaf, 0};
        };
        if (v) {
            const int64_t off = base + tid;
            const int32_t leaf = (int32_t)(at + e1);
            tab[leaf] = LeafDesc{off, v, leaf};
            if (nt <= kMany) {
                TileJob *q = out + jat + e2;
                for (uint32_t I = 0; I < nt; I++)
                    for (uint32_t J = 0; J < nt; J++) *q++ = job(off, v, leaf, I, J);
            } else {  // (one at most: 1024 positions hold the start of one leaf of so many)
                s_big[0] = (uint32_t)tid;
                s_big[1] = e1;
                s_big[2] = e2;
            }
        }
        if (__syncthreads_or(nt > kMany)) {
            const int64_t off = base + s_big[0];
            const int32_t m = mk[off];
            const uint32_t nb = (uint32_t)((m + TR - 1) / TR);
            TileJob *q = out + jat + s_big[2];
            for (uint64_t k = tid; k < (uint64_t)nb * nb; k += 1024)
                q[k] = job(off, m, (int32_t)(at + s_big[1]), (uint32_t)(k / nb), (uint32_t)(k % nb));
            __syncthreads();
        }
        at += t1;
        jat += t2;
    }
    if (blockIdx.x + 1 == gridDim.x)
        for (int64_t i = at + tid; i < stride; i += 1024) tab[i] = LeafDesc{0, 0, -1};
    if (t == 0)
        for (int64_t i = blockIdx.x * 1024 + tid; i <= stride; i += gridDim.x * 1024) ident[i] = (int32_t)i;
}

// The node records in order: tree, level, small nodes before large ones (by the depth of the
// first small ancestor), left to right.  Two stable passes: by position (ranges of 256 positions
// counted and dealt, ranked inside), then by level and smallness (one workgroup per tree).
__device__ inline int64_t rec_bucket(const UniRec &r, int64_t n, int64_t nb) {
    return r.tree * nb + ((r.pos - r.tree * n) >> 8);
}

__global__ void k_uni_rec_count(const UniRec *__restrict__ recs, uint32_t cnt, int64_t n, int64_t nb,
                                uint32_t *__restrict__ bucket) {
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < cnt; i += gridDim.x * blockDim.x)
        atomicAdd(&bucket[rec_bucket(recs[i], n, nb)], 1u);
}

__global__ void k_uni_rec_deal(const UniRec *__restrict__ recs, uint32_t cnt, int64_t n, int64_t nb,
                               const uint32_t *__restrict__ start, uint32_t *__restrict__ fill,
                               uint32_t *__restrict__ idx) {
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < cnt; i += gridDim.x * blockDim.x) {
        const int64_t b = rec_bucket(recs[i], n, nb);
        idx[start[b] + atomicAdd(&fill[b], 1u)] = i;
    }
}

__global__ void k_uni_rec_rank(const UniRec *__restrict__ recs, uint32_t cnt, int64_t n, int64_t nb,
                               const uint32_t *__restrict__ start, const uint32_t *__restrict__ idx,
                               uint32_t *__restrict__ by_pos, uint32_t *__restrict__ digit) {
    for (uint32_t k = blockIdx.x * blockDim.x + threadIdx.x; k < cnt; k += gridDim.x * blockDim.x) {
        const uint32_t i = idx[k];
        const UniRec r = recs[i];
        const int64_t b = rec_bucket(r, n, nb);
        const uint32_t s0 = start[b], s1 = start[b + 1];
        uint32_t rank = 0;
        for (uint32_t q = s0; q < s1; q++) {
            const UniRec &o = recs[idx[q]];
            rank += (o.pos < r.pos || (o.pos == r.pos && o.depth < r.depth)) ? 1u : 0u;
        }
        by_pos[s0 + rank] = i;
        digit[s0 + rank] = (uint32_t)(r.depth * (kRecLarge + 1) + r.small);
    }
}

constexpr int kRecDigits = 64 * (kRecLarge + 1);

// to[k]: the place of the k-th record by position
__global__ __launch_bounds__(1024) void k_uni_rec_level(const uint32_t *__restrict__ start, int64_t nb,
                                                        const uint32_t *__restrict__ digit, uint32_t *__restrict__ to) {
    __shared__ uint32_t s_at[kRecDigits];
    __shared__ uint32_t s_w[16];
    const int tid = threadIdx.x;
    const uint32_t lo = start[blockIdx.x * nb], hi = start[(blockIdx.x + 1) * nb];
    for (int i = tid; i < kRecDigits; i += 1024) s_at[i] = 0;
    __syncthreads();
    for (uint32_t k = lo + tid; k < hi; k += 1024) atomicAdd(&s_at[digit[k]], 1u);
    __syncthreads();
    uint32_t base = lo;
    for (int i0 = 0; i0 < kRecDigits; i0 += 1024) {
        const int i = i0 + tid;
        uint32_t excl, total;
        block_excl_scan_w<16>(i < kRecDigits ? s_at[i] : 0u, s_w, excl, total);
        if (i < kRecDigits) s_at[i] = base + excl;
        base += total;
    }
    __syncthreads();
    // every wave walks the records in order, 64 at a time, and places those of its levels
    const uint32_t lane = tid & 63, w = tid >> 6;
    uint32_t nextd = lo + lane < hi ? digit[lo + lane] : kRecDigits;
    for (uint32_t k = lo; k < hi; k += 64) {
        const uint32_t d = nextd;
        nextd = k + 64 + lane < hi ? digit[k + 64 + lane] : kRecDigits;
        bool open = d < kRecDigits && ((d / (kRecLarge + 1)) & 15) == w;
        for (uint64_t left = __ballot(open); left; left = __ballot(open)) {
            const uint32_t lead = __builtin_amdgcn_readlane(d, __ffsll((unsigned long long)left) - 1);
            const bool same = open && d == lead;
            const uint64_t b = __ballot(same);
            const uint32_t at = s_at[lead];
            if (same) {
                const uint32_t r = (uint32_t)mask_rank(b);
                to[k + lane] = at + r;
                if (r == 0) s_at[lead] = at + (uint32_t)__popcll(b);
                open = false;
            }
        }
    }
}

__global__ void k_uni_rec_out(const UniRec *__restrict__ recs, uint32_t cnt, const uint32_t *__restrict__ by_pos,
                              const uint32_t *__restrict__ to, rpf_node *__restrict__ out) {
    for (uint32_t k = blockIdx.x * blockDim.x + threadIdx.x; k < cnt; k += gridDim.x * blockDim.x) {
        const UniRec r = recs[by_pos[k]];
        out[to[k]] = rpf_node{r.heap, r.c, r.size, r.left, r.chosen, r.depth};
    }
}

void launch_uni_grow(hipStream_t s, bool wave, const float *X, int d, uint64_t seed, const UniSeg *items,
                     const uint32_t *count, uint32_t *next, int64_t most, int n0, int small_max, int32_t *perm,
                     const UniGrow &u) {
    if (most <= 0) return;
    const bool vec = d % 4 == 0;
    auto go = [&](auto kern, int nt, int cap, int resident) {
        const size_t lds = uni_grow_lds(cap, d);
        hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        hipLaunchKernelGGL(kern, dim3((unsigned)std::min<int64_t>(most, resident)), dim3(nt), lds, s, X, d, seed, items,
                           count, (uint32_t)std::min<int64_t>(most, 0x7fffffff), next, wave ? n0 : kGrowWave, n0,
                           small_max, perm, u.recs, u.rec_cnt, u.rec_cap, u.mark, u.more, u.more_cnt, u.more_cap);
    };
    if (wave)
        vec ? go(k_uni_grow<64, kGrowWave, true>, 64, kGrowWave, 3072)
            : go(k_uni_grow<64, kGrowWave, false>, 64, kGrowWave, 3072);
    else
        vec ? go(k_uni_grow<1024, kGrowBlock, true>, 1024, kGrowBlock, 256)
            : go(k_uni_grow<1024, kGrowBlock, false>, 1024, kGrowBlock, 256);
    launch_check(s, "k_uni_grow");
}

void launch_uni_mark(hipStream_t s, const UniSeg *leaves, int count, int32_t *mark) {
    if (count <= 0) return;
    hipLaunchKernelGGL(k_uni_mark, dim3((count + 255) / 256), dim3(256), 0, s, leaves, count, mark);
    launch_check(s, "k_uni_mark");
}

int uni_leaf_parts(int64_t n, int T) {
    return (int)std::max<int64_t>(1, std::min<int64_t>(512 / T, (n + 4095) / 4096));
}

static int64_t uni_part_len(int64_t n, int parts) { return ((n + parts - 1) / parts + 1023) / 1024 * 1024; }

void launch_uni_leaf_count(hipStream_t s, const int32_t *mark, int64_t n, int T, int parts, int TR, UniTree *out) {
    hipLaunchKernelGGL(k_uni_leaf_count, dim3(parts, T), dim3(1024), 0, s, mark, n, uni_part_len(n, parts), TR, out);
    launch_check(s, "k_uni_leaf_count");
}

void launch_uni_leaf_fill(hipStream_t s, const int32_t *mark, int64_t n, int T, int parts, int TR, int64_t stride,
                          const UniPart *at, LeafDesc *table, TileJob *jobs, int32_t *ident) {
    hipLaunchKernelGGL(k_uni_leaf_fill, dim3(parts, T), dim3(1024), 0, s, mark, n, uni_part_len(n, parts), TR, stride, at,
                       table, jobs, ident);
    launch_check(s, "k_uni_leaf_fill");
}

void launch_uni_rec_count(hipStream_t s, const UniRec *recs, uint32_t cnt, int64_t n, int64_t nb, uint32_t *bucket) {
    if (!cnt) return;
    hipLaunchKernelGGL(k_uni_rec_count, dim3(std::min(cnt / 256 + 1, 2048u)), dim3(256), 0, s, recs, cnt, n, nb, bucket);
    launch_check(s, "k_uni_rec_count");
}

void launch_uni_rec_order(hipStream_t s, const UniRec *recs, uint32_t cnt, int T, int64_t n, int64_t nb,
                          const uint32_t *start, uint32_t *fill, uint32_t *words, uint32_t cap, rpf_node *out) {
    if (!cnt) return;
    uint32_t *idx = words, *by_pos = words + cap, *digit = words + 2 * (size_t)cap;
    const dim3 grid(std::min(cnt / 256 + 1, 4096u)), block(256);
    hipLaunchKernelGGL(k_uni_rec_deal, grid, block, 0, s, recs, cnt, n, nb, start, fill, idx);
    hipLaunchKernelGGL(k_uni_rec_rank, grid, block, 0, s, recs, cnt, n, nb, start, idx, by_pos, digit);
    hipLaunchKernelGGL(k_uni_rec_level, dim3(T), dim3(1024), 0, s, start, nb, digit, idx);
    hipLaunchKernelGGL(k_uni_rec_out, grid, block, 0, s, recs, cnt, by_pos, idx, out);
    launch_check(s, "uniform node records");
}

// ---------------------------------------------------------------- launches of one level

void launch_uni_block(hipStream_t s, const float *X, int d, int n_try, uint64_t seed, const UniSeg *segs, int nseg,
                      int max_m, int32_t *perm, UniSplit *out) {
    if (nseg <= 0) return;
    const size_t lds = uni_block_lds(max_m, d, n_try);
    const bool vec = d % 4 == 0;
    auto go = [&](auto kern, int nt) {
        hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        hipLaunchKernelGGL(kern, dim3((unsigned)nseg), dim3(nt), lds, s, X, d, n_try, seed, segs, perm, out);
    };
    if (max_m <= 128) {  // one wave per node
        if (vec) go(k_uni_block<64, true>, 64);
        else go(k_uni_block<64, false>, 64);
    } else {
        if (vec) go(k_uni_block<256, true>, 256);
        else go(k_uni_block<256, false>, 256);
    }
    launch_check(s, "k_uni_block");
}

void launch_uni_chunked(hipStream_t s, const float *X, int d, int n_try, uint64_t seed, const UniSeg *segs, int nseg,
                        const UniChunk *chunks, int nchunk, int32_t *perm, int64_t TN, const UniBufs &b,
                        UniSplit *out) {
    if (nseg <= 0) return;
    const bool vec = d % 4 == 0;
    auto proj = [&](auto kern, int nt) {
        hipLaunchKernelGGL(kern, dim3(nchunk), dim3(nt), n_try > 1 ? kChunk * sizeof(double) : 0, s, X, d, n_try, seed,
                           segs, chunks, perm, TN, b.P, b.part, b.mm);
    };
    if (n_try > 1 || nchunk > 512) vec ? proj(k_uni_proj<true, 256>, 256) : proj(k_uni_proj<false, 256>, 256);
    else vec ? proj(k_uni_proj<true, 1024>, 1024) : proj(k_uni_proj<false, 1024>, 1024);
    launch_check(s, "k_uni_proj");
    if (n_try > 1) {
        const int64_t items = (int64_t)nseg * n_try;
        hipLaunchKernelGGL(k_uni_mean, dim3((unsigned)((items + 63) / 64)), dim3(64), 0, s, segs, nseg, n_try, b.part,
                           b.mu);
        hipLaunchKernelGGL(k_uni_disp, dim3(nchunk), dim3(256), 0, s, segs, chunks, n_try, TN, b.P, b.mu, b.part);
        launch_check(s, "k_uni_disp");
    }
    hipLaunchKernelGGL(k_uni_decide, dim3((nseg + 63) / 64), dim3(64), 0, s, segs, nseg, n_try, seed, b.part, b.mm,
                       out);
    hipLaunchKernelGGL(k_uni_count, dim3(nchunk), dim3(256), 0, s, chunks, TN, b.P, out, b.lcount);
    hipLaunchKernelGGL(k_uni_offsets, dim3((nseg + 63) / 64), dim3(64), 0, s, segs, nseg, b.lcount, b.loff, out);
    hipLaunchKernelGGL(k_uni_scatter, dim3(nchunk), dim3(256), 0, s, segs, chunks, TN, b.P, out, b.loff, perm, b.tmp);
    hipLaunchKernelGGL(k_uni_copy, dim3(nchunk), dim3(256), 0, s, chunks, b.tmp, perm);
    launch_check(s, "uniform chunked level");
}

}  // namespace rpf
