// Index construction on the GPU (Section 4.1): k-means on a sample of the token
// embeddings, assignment of every token to its nearest centroid, quantile
// bucket cutoffs and weights of the residuals, and packed b-bit residual codes
// grouped by cluster. Every decision is exact, so the result equals the CPU
// definition bit for bit:
//   * assignment: argmax over centroids of the fp64 score S64 (dimension order),
//     lowest id among equal scores (assign.hip);
//   * k-means update: the sum over assigned sample tokens of round(x * 2^30) per
//     dimension (exact int64), normalised in fp64 (dimension-order sum of
//     squares, IEEE sqrt and division) and rounded to fp32; a centroid without
//     tokens keeps its value;
//   * quantiles: the ceil(n p)-th smallest residual component (n components of
//     the first n_quant tokens), cutoffs at p = j / 2^b, weights at
//     p = (j + 1/2) / 2^b;
//   * codes: the number of cutoffs <= the fp32 residual component, packed with
//     the first dimension in the most significant bits; embeddings ordered by
//     cluster, then by input order (a stable sort).
#include <algorithm>
#include <cmath>
#include <string>

#include "engine.h"

namespace warp {

__global__ void k_gather_rows(const float* __restrict__ x, const int64_t* __restrict__ ids, int64_t n,
                              float* __restrict__ out) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n * kDim) return;
    out[i] = x[ids[i / kDim] * kDim + i % kDim];
}

// per centroid: sum of round(x * 2^30) over its assigned sample tokens, and their count
__global__ void k_kmeans_accum(const float* __restrict__ xs, const int32_t* __restrict__ assign, int64_t n,
                               unsigned long long* __restrict__ sums, unsigned long long* __restrict__ counts) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n * kDim) return;
    const int64_t t = i / kDim;
    const int d = (int)(i % kDim);
    const int c = assign[t];
    const long long q = (long long)__builtin_rint((double)xs[i] * 1073741824.0);
    atomicAdd(&sums[(int64_t)c * kDim + d], (unsigned long long)q);  // two's complement sum
    if (d == 0) atomicAdd(&counts[c], 1ull);
}

__global__ void k_kmeans_normalize(const unsigned long long* __restrict__ sums,
                                   const unsigned long long* __restrict__ counts, int32_t n_c,
                                   float* __restrict__ cen) {
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= n_c || counts[c] == 0) return;
    const unsigned long long* s = sums + (int64_t)c * kDim;
    double ss = 0.0;
    for (int d = 0; d < kDim; ++d) {
        const double m = (double)(long long)s[d];
        ss += m * m;
    }
    if (!(ss > 0.0)) return;
    const double norm = __builtin_sqrt(ss);
    for (int d = 0; d < kDim; ++d) cen[(int64_t)c * kDim + d] = (float)((double)(long long)s[d] / norm);
}

// rows of 128 fp32 values scaled to unit norm: (float)(x_d / ||x||), the norm in fp64 (sum
// of squares in dimension order, IEEE sqrt); the rows were checked to be finite and nonzero
__global__ void k_normalize_rows(const float* __restrict__ rows, int32_t n, float* __restrict__ out) {
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= n) return;
    const float* r = rows + (int64_t)c * kDim;
    double ss = 0.0;
    for (int d = 0; d < kDim; ++d) ss += (double)r[d] * (double)r[d];
    const double norm = __builtin_sqrt(ss);
    for (int d = 0; d < kDim; ++d) out[(int64_t)c * kDim + d] = (float)((double)r[d] / norm);
}

// residual components of tokens [0, n): x - C[assign]
__global__ void k_residuals(const float* __restrict__ x, const int32_t* __restrict__ assign, int64_t n,
                            const float* __restrict__ cen, float* __restrict__ out) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n * kDim) return;
    out[i] = x[i] - cen[(int64_t)assign[i / kDim] * kDim + i % kDim];
}

// cutoffs (j = 1 .. 2^b - 1) and weights (j = 0 .. 2^b - 1) from the sorted components
__global__ void k_pick_quantiles(const float* __restrict__ sorted, int64_t n, int32_t nbits,
                                 float* __restrict__ cutoffs, float* __restrict__ weights) {
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    const int nb = 1 << nbits;
    auto at = [&](int64_t num, int shift) {  // the ceil(n * num / 2^shift)-th smallest
        int64_t k = (n * num + ((1ll << shift) - 1)) >> shift;
        k = k < 1 ? 1 : (k > n ? n : k);
        return sorted[k - 1];
    };
    if (j >= 1 && j < nb) cutoffs[j - 1] = at(j, nbits);
    if (j < nb) weights[j] = at(2 * j + 1, nbits + 1);
}

// embeddings in cluster order: codes and document ids at position p of token perm[p]. A thread
// makes four code bytes (32 / NBITS dimensions) from 16-byte loads; the cutoffs stand in LDS.
template <int NBITS>
__global__ __launch_bounds__(256) void k_encode(const float* __restrict__ x, const int32_t* __restrict__ token_docs,
                                                const int32_t* __restrict__ assign, const int64_t* __restrict__ perm,
                                                int64_t n, const float* __restrict__ cen,
                                                const float* __restrict__ cutoffs, uint32_t* __restrict__ codes,
                                                int32_t* __restrict__ doc_ids) {
    constexpr int NB = 1 << NBITS;
    constexpr int WORDS = kDim * NBITS / 32;  // code words per embedding
    constexpr int DIMS = 32 / NBITS;          // dimensions per word
    __shared__ float s_cut[NB];
    if (threadIdx.x < NB - 1) s_cut[threadIdx.x] = cutoffs[threadIdx.x];
    __syncthreads();
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;  // (position, word)
    if (i >= n * WORDS) return;
    const int64_t p = i / WORDS;
    const int word = (int)(i % WORDS);
    const int64_t t = perm[p];
    const int c = assign[t];
    const float4* xr = reinterpret_cast<const float4*>(x + t * kDim + word * DIMS);
    const float4* cr = reinterpret_cast<const float4*>(cen + (int64_t)c * kDim + word * DIMS);
    unsigned v = 0;
#pragma unroll
    for (int k = 0; k < DIMS / 4; ++k) {
        const float4 a = xr[k], b = cr[k];
        const float r[4] = {a.x - b.x, a.y - b.y, a.z - b.z, a.w - b.w};
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int d = 4 * k + u;
            int lo = 0, hi = NB - 1;  // the number of cutoffs <= r (cutoffs ascend)
#pragma unroll
            for (int step = 0; step < NBITS; ++step) {
                const int mid = (lo + hi) >> 1;
                if (s_cut[mid] <= r[u]) lo = mid + 1;
                else hi = mid;
            }
            // the word's bytes in memory order, the first dimension of a byte in its top bits
            const int byte = d * NBITS / 8;
            v |= (unsigned)lo << (8 * byte + 8 - NBITS * (d % (8 / NBITS) + 1));
        }
    }
    if (((uintptr_t)codes & 3) == 0) {  // uniform
        codes[i] = v;
    } else {
        uint8_t* b = reinterpret_cast<uint8_t*>(codes) + 4 * i;
#pragma unroll
        for (int k = 0; k < 4; ++k) b[k] = (uint8_t)(v >> (8 * k));
    }
    if (word == 0) doc_ids[p] = token_docs[t];
}

// Blocks [0, cb): the first starting vector that is not finite or whose squared norm is zero or not
// finite, one thread each: *first becomes the largest ~(2 c + (finite)). Blocks [cb, ...): the first
// sample id outside [0, n_tokens), first[1] the largest ~i.
constexpr int kCheckBlock = 64;
__global__ __launch_bounds__(kCheckBlock) void k_check_build(const float* __restrict__ rows, int32_t n_c, int32_t cb,
                                                             const int64_t* __restrict__ ids, int64_t n, int64_t n_tokens,
                                                             unsigned long long* first) {
    if ((int)blockIdx.x >= cb) {
        const int64_t i = (int64_t)((int)blockIdx.x - cb) * kCheckBlock + threadIdx.x;
        if (i < n && (ids[i] < 0 || ids[i] >= n_tokens)) atomicMax(first + 1, ~(unsigned long long)i);
        return;
    }
    const int c = blockIdx.x * kCheckBlock + threadIdx.x;
    if (c >= n_c) return;
    const float4* r = reinterpret_cast<const float4*>(rows + (int64_t)c * kDim);
    double ss = 0.0;
    bool finite = true;
    for (int d = 0; d < kDim / 4; ++d) {
        const float4 v = r[d];
        finite &= __builtin_isfinite(v.x) && __builtin_isfinite(v.y) && __builtin_isfinite(v.z) && __builtin_isfinite(v.w);
        ss += (double)v.x * v.x;
        ss += (double)v.y * v.y;
        ss += (double)v.z * v.z;
        ss += (double)v.w * v.w;
    }
    if (!finite || !(ss > 0.0) || !__builtin_isfinite(ss)) atomicMax(first, ~(2ull * (unsigned)c + (finite ? 1 : 0)));
}

__global__ void k_count_clusters(const int32_t* __restrict__ assign, int64_t n, unsigned long long* counts) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) atomicAdd(&counts[assign[i]], 1ull);
}

__global__ void k_iota64(int64_t* out, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) out[i] = i;
}

// ---------------------------------------------------------------------------- launchers

static unsigned blocks_for(int64_t n, int per) { return (unsigned)((n + per - 1) / per); }

void launch_gather_rows(const float* x, const int64_t* ids, int64_t n, float* out, hipStream_t s) {
    if (n > 0) hipLaunchKernelGGL(k_gather_rows, dim3(blocks_for(n * kDim, 256)), dim3(256), 0, s, x, ids, n, out);
}

void launch_kmeans_accum(const float* xs, const int32_t* assign, int64_t n, unsigned long long* sums,
                         unsigned long long* counts, hipStream_t s) {
    if (n > 0)
        hipLaunchKernelGGL(k_kmeans_accum, dim3(blocks_for(n * kDim, 256)), dim3(256), 0, s, xs, assign, n, sums,
                           counts);
}

void launch_kmeans_normalize(const unsigned long long* sums, const unsigned long long* counts, int32_t n_c,
                             float* cen, hipStream_t s) {
    hipLaunchKernelGGL(k_kmeans_normalize, dim3(blocks_for(n_c, 64)), dim3(64), 0, s, sums, counts, n_c, cen);
}

void launch_normalize_rows(const float* rows, int32_t n, float* out, hipStream_t s) {
    if (n > 0) hipLaunchKernelGGL(k_normalize_rows, dim3(blocks_for(n, 64)), dim3(64), 0, s, rows, n, out);
}

void launch_residuals(const float* x, const int32_t* assign, int64_t n, const float* cen, float* out,
                      hipStream_t s) {
    if (n > 0) hipLaunchKernelGGL(k_residuals, dim3(blocks_for(n * kDim, 256)), dim3(256), 0, s, x, assign, n, cen, out);
}

void launch_pick_quantiles(const float* sorted, int64_t n, int32_t nbits, float* cutoffs, float* weights,
                           hipStream_t s) {
    hipLaunchKernelGGL(k_pick_quantiles, dim3(1), dim3(256), 0, s, sorted, n, nbits, cutoffs, weights);
}

void launch_encode(int32_t nbits, const float* x, const int32_t* token_docs, const int32_t* assign,
                   const int64_t* perm, int64_t n, const float* cen, const float* cutoffs, uint8_t* codes,
                   int32_t* doc_ids, hipStream_t s) {
    const int64_t work = n * (kDim * nbits / 32);
    if (work <= 0) return;
    uint32_t* words = reinterpret_cast<uint32_t*>(codes);
    const dim3 grid(blocks_for(work, 256)), block(256);
    switch (nbits) {
        case 1: hipLaunchKernelGGL(k_encode<1>, grid, block, 0, s, x, token_docs, assign, perm, n, cen, cutoffs, words, doc_ids); break;
        case 2: hipLaunchKernelGGL(k_encode<2>, grid, block, 0, s, x, token_docs, assign, perm, n, cen, cutoffs, words, doc_ids); break;
        case 4: hipLaunchKernelGGL(k_encode<4>, grid, block, 0, s, x, token_docs, assign, perm, n, cen, cutoffs, words, doc_ids); break;
        default: hipLaunchKernelGGL(k_encode<8>, grid, block, 0, s, x, token_docs, assign, perm, n, cen, cutoffs, words, doc_ids); break;
    }
}

void launch_check_build(const float* rows, int32_t n_c, const int64_t* ids, int64_t n, int64_t n_tokens,
                        unsigned long long* first, hipStream_t s) {
    const unsigned cb = blocks_for(n_c, kCheckBlock);
    hipLaunchKernelGGL(k_check_build, dim3(cb + blocks_for(n, kCheckBlock)), dim3(kCheckBlock), 0, s, rows, n_c, (int32_t)cb,
                       ids, n, n_tokens, first);
}

void launch_count_clusters(const int32_t* assign, int64_t n, unsigned long long* counts, hipStream_t s) {
    if (n > 0) hipLaunchKernelGGL(k_count_clusters, dim3(blocks_for(n, 256)), dim3(256), 0, s, assign, n, counts);
}

void launch_iota64(int64_t* out, int64_t n, hipStream_t s) {
    if (n > 0) hipLaunchKernelGGL(k_iota64, dim3(blocks_for(n, 256)), dim3(256), 0, s, out, n);
}

}  // namespace warp
