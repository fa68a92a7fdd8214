// Nearest centroids for the index construction (Section 4.1): for every token, the centroid of
// the highest fp64 score S64 (dimension order), lowest id among equal scores.
//
// The score matrix is never written. k_assign_gemm multiplies fp16 copies of tokens and
// centroids on the matrix cores (one product, fp32 accumulation): its scores f satisfy
// |f - S64| <= kAssignEps, since each operand is rounded by at most 2^-11 of itself (plus 2^-25
// below the normal range) and sum_d |x_d c_d| <= 1.001 * (1 + 2^-11). Every lane of the product
// sees, per tile of 128 centroids, 16 of one token's scores; it keeps the two tiles of the
// largest maxima of these 16 and the third maximum. k_assign_pick then has, per token, a few
// (tile, lane) blocks of 16 centroids that hold every centroid within 2 kAssignEps of the best
// filter score, hence the fp64 argmax: where a single centroid of theirs lies in the band, by
// its fp16 row again, it is the argmax; else the blocks are scored in fp32 (within 2^-17 of S64),
// and if more than one centroid remains within 2^-15 of the best of these, in fp64. A token with
// a third block in the band (centroids that coincide or nearly so) is scored against every
// centroid again by k_assign_all, sixteen such tokens at a time. So the result is the exact argmax
// for every input.
//
// The product is bound by the matrix cores: a wave computes 64 tokens x 64 centroids with its
// tokens' operands in registers; the centroids stream through two 32 KB LDS tiles that are
// loaded straight from memory (16 bytes per lane, rows swizzled by their number so that the
// operand reads meet no bank twice).
// Measured (1M tokens, 2^14 centroids, with four k-means steps on 125k of them): the whole build
// 96.3 -> 11.0 ms (10.3 ms of kernels; the scratch's allocation and release 0.4 ms, the stream's 0.2 ms);
// the product 5.2 ms (1.19 PFLOP/s), the picks 2.1 + 1.1 + 0.4 ms, against 39 ms for a split-fp16 product
// that wrote fp32 scores and 51 ms to read them. In a process that has freed tens of GB before (large
// indexes), hipMalloc has to reclaim memory: it takes 4 to 12 ms instead of 0.1 and the call 15 to 23 ms.
#include <algorithm>

#include "engine.h"

namespace warp {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half2v __attribute__((ext_vector_type(2)));

constexpr int kAsTile = 128;    // tokens and centroids of a tile
constexpr int kAsStreams = 8;   // lanes that share a token: 4 lane groups x 2 column halves
constexpr int kAsCand = 1024;   // most centroids within 2.5 kFilterEps of the best (else kErrArgOverflow)
// 2 * 2^-11 * 1.0025 for the operands, 128 * 2^-24 for the accumulation, 2^-24 * 12 for values
// below fp16's normal range: 9.9e-4
constexpr float kAssignEps = 1.05e-3f;

struct AsStream {  // what a lane keeps of a token
    float b1, b2, b3;  // the three largest tile maxima
    int32_t t1, t2;    // tiles of the first two
};

// fp16 copies of n rows of 128 values, rows up to n_pad zero; *c0 and *c1 become zero
__global__ __launch_bounds__(256) void k_half_rows(const float* __restrict__ x, int64_t n, int64_t n_pad,
                                                   _Float16* __restrict__ out, int32_t* c0, int32_t* c1) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;  // eight values each
    if (i == 0) *c0 = *c1 = 0;
    if (i >= n_pad * (kDim / 8)) return;
    half8 h = {};
    if (i < n * (kDim / 8)) {
        const float4 u = reinterpret_cast<const float4*>(x)[2 * i], v = reinterpret_cast<const float4*>(x)[2 * i + 1];
        h = (half8){(_Float16)u.x, (_Float16)u.y, (_Float16)u.z, (_Float16)u.w,
                    (_Float16)v.x, (_Float16)v.y, (_Float16)v.z, (_Float16)v.w};
    }
    reinterpret_cast<half8*>(out)[i] = h;
}

// Workgroup (token tile, split): its 128 tokens against the centroid tiles of split blockIdx.y.
__global__ __launch_bounds__(256, 2) void k_assign_gemm(const float* __restrict__ x, int64_t n,
                                                        const _Float16* __restrict__ ch, int32_t n_c,
                                                        AsStream* __restrict__ out) {
    __shared__ __attribute__((aligned(16))) _Float16 s_c[2][kAsTile * kDim];
    const int tid = threadIdx.x;
    const int wave = tid >> 6;
    const int lane = tid & 63;
    const int li = lane & 15;
    const int g = lane >> 4;
    const int wr = (wave >> 1) * 64;  // this wave's tokens within the tile
    const int wc = (wave & 1) * 64;   // and centroids
    const int64_t t_base = (int64_t)blockIdx.x * kAsTile;
    const int tiles = (n_c + kAsTile - 1) / kAsTile;
    const int t0 = (int)((int64_t)tiles * blockIdx.y / gridDim.y), t1 = (int)((int64_t)tiles * (blockIdx.y + 1) / gridDim.y);

    // token operands: block i of 16 tokens, K step s: the lane's 8 values of token 16 i + li
    half8 a[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int64_t t = t_base + wr + 16 * i + li;
        const float4* row = reinterpret_cast<const float4*>(x + (t < n ? t : 0) * kDim);
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const float4 u = row[8 * s + 2 * g], v = row[8 * s + 2 * g + 1];
            a[i][s] = (half8){(_Float16)u.x, (_Float16)u.y, (_Float16)u.z, (_Float16)u.w,
                              (_Float16)v.x, (_Float16)v.y, (_Float16)v.z, (_Float16)v.w};
        }
    }
    // A tile's 128 rows of 16 chunks of 16 bytes, chunk k of row r at position k ^ (r % 16): a wave
    // loads four rows at a time.
    auto load = [&](int t, int b) {
        const char* src = reinterpret_cast<const char*>(ch) + (int64_t)t * kAsTile * kDim * 2;
#pragma unroll
        for (int i = 0; i < kAsTile / 16; ++i) {
            const int r4 = 4 * (wave + 4 * i);  // rows r4 .. r4 + 3
            const int r = r4 + (lane >> 4);
            const char* p = src + r * 256 + ((lane & 15) ^ (r & 15)) * 16;
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)p,
                                             (__attribute__((address_space(3))) void*)&s_c[b][r4 * kDim], 16, 0, 0);
        }
    };
    AsStream best[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) best[i] = {-INFINITY, -INFINITY, -INFINITY, 0, 0};
    if (t0 < t1) load(t0, 0);
    for (int t = t0; t < t1; ++t) {
        const int b = (t - t0) & 1;
        __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): this tile's loads have landed
        __syncthreads();                     // everyone's, and the other buffer is no longer read
        if (t + 1 < t1) load(t + 1, b ^ 1);
        floatx4 acc[4][4];
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) acc[i][j] = (floatx4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            half8 c[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int r = wc + 16 * j + li;
                c[j] = *reinterpret_cast<const half8*>(&s_c[b][r * kDim + ((4 * s + g) ^ (r & 15)) * 8]);
            }
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(c[j], a[i][s], acc[i][j], 0, 0, 0);
        }
        // lane (li, g): centroids 128 t + wc + 16 j + 4 g + r against token wr + 16 i + li
        if ((t + 1) * kAsTile > n_c) {  // uniform: rows past the last centroid do not count
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (t * kAsTile + wc + 16 * j + 4 * g + r >= n_c) {
#pragma unroll
                        for (int i = 0; i < 4; ++i) acc[i][j][r] = -INFINITY;
                    }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float m = acc[i][0][0];
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) m = __builtin_fmaxf(m, acc[i][j][r]);
            AsStream& s = best[i];
            const bool c1 = m > s.b1, c2 = m > s.b2;
            s.b3 = __builtin_fmaxf(s.b3, __builtin_fminf(s.b2, m));
            s.t2 = c1 ? s.t1 : (c2 ? t : s.t2);
            s.b2 = __builtin_amdgcn_fmed3f(s.b1, s.b2, m);
            s.b1 = __builtin_fmaxf(s.b1, m);
            s.t1 = c1 ? t : s.t1;
        }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int64_t t = t_base + wr + 16 * i + li;
        if (t < n) out[(t * gridDim.y + blockIdx.y) * kAsStreams + 4 * (wave & 1) + g] = best[i];
    }
}

// (score desc, id asc)
__device__ __forceinline__ void keep_best(double& best, int& id, double v, int c) {
    if (v > best || (v == best && c < id)) {
        best = v;
        id = c;
    }
}

// A token's streams as a wave reads them (lane q: stream q, at most 64 of them), and the blocks of
// 16 centroids within the band of the best: bit q of m1 (m2): stream q's first (second) tile.
struct AsBlocks {
    AsStream s;
    float thr;
    unsigned long long m1, m2;
    bool over;  // more blocks than were kept, or enough for kAsCand centroids
};
__device__ __forceinline__ AsBlocks as_blocks(const AsStream* streams, int ns, int64_t t, int lane) {
    AsBlocks b;
    b.s = {-INFINITY, -INFINITY, -INFINITY, 0, 0};
    if (lane < ns) b.s = streams[t * ns + lane];
    float mx = b.s.b1;
    for (int off = 32; off > 0; off >>= 1) mx = __builtin_fmaxf(mx, __shfl_xor(mx, off, 64));
    b.thr = mx - 2.1f * kAssignEps;  // (2 eps, and the rounding of either sum)
    b.m1 = __ballot(b.s.b1 >= b.thr);
    b.m2 = __ballot(b.s.b2 >= b.thr);
    b.over = __any(b.s.b3 >= b.thr) || 16 * (__popcll(b.m1) + __popcll(b.m2)) > kAsCand;
    return b;
}
// The blocks in turn: f(centroid of lanes 4 u .. 4 u + 3), u = 4 j + r for centroid 16 j + 4 g + r.
template <typename F>
__device__ __forceinline__ void for_blocks(const AsBlocks& b, int lane, F f) {
    const int u = lane >> 2;
    for (int pass = 0; pass < 2; ++pass)
        for (unsigned long long m = pass ? b.m2 : b.m1; m; m &= m - 1) {  // wave-uniform
            const int q = __builtin_ctzll(m);
            f(__shfl(pass ? b.s.t2 : b.s.t1, q, 64) * kAsTile + ((q & 4) ? 64 : 0) + 16 * (u >> 2) + 4 * (q & 3) + (u & 3));
        }
}

// One wave per token: the blocks' centroids by their fp16 rows again (|f - S64| <= kAssignEps
// whatever the order of the sum), four lanes each. A single one in the band is the argmax; other
// tokens go to `near`, or to `all` where the blocks do not hold the whole band. Bound by the reads
// of the rows (4 KB per token).
__global__ __launch_bounds__(256) void k_assign_pick(const AsStream* __restrict__ streams, int32_t splits, int64_t n,
                                                     const float* __restrict__ x, const _Float16* __restrict__ ch,
                                                     int32_t n_c, int32_t* __restrict__ assign,
                                                     int32_t* __restrict__ near, int32_t* __restrict__ all) {
    const int64_t t = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (t >= n) return;  // wave-uniform
    const int lane = threadIdx.x & 63, part = lane & 3;
    half8 xh[4];
    const float4* xr = reinterpret_cast<const float4*>(x + t * kDim) + 8 * part;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const float4 u = xr[2 * k], v = xr[2 * k + 1];
        xh[k] = (half8){(_Float16)u.x, (_Float16)u.y, (_Float16)u.z, (_Float16)u.w,
                        (_Float16)v.x, (_Float16)v.y, (_Float16)v.z, (_Float16)v.w};
    }
    const AsBlocks b = as_blocks(streams, splits * kAsStreams, t, lane);
    int hits = 0, hit = 0;
    if (!b.over)
        for_blocks(b, lane, [&](int c) {
            const half8* row = reinterpret_cast<const half8*>(ch + (int64_t)c * kDim) + 4 * part;  // (rows past n_c are zero)
            float v = 0.f;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const half8 w = row[k];
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    v = __builtin_amdgcn_fdot2((half2v){w[2 * i], w[2 * i + 1]}, (half2v){xh[k][2 * i], xh[k][2 * i + 1]}, v,
                                               false);
            }
            v += __shfl_xor(v, 1, 64);
            v += __shfl_xor(v, 2, 64);
            const unsigned long long m = __ballot(part == 0 && c < n_c && v >= b.thr);
            hits += __popcll(m);
            if (m) hit = __shfl(c, __builtin_ctzll(m), 64);
        });
    if (lane == 0) {
        if (hits == 1) assign[t] = hit;
        else if (b.over) all[1 + atomicAdd(&all[0], 1)] = (int32_t)t;
        else near[1 + atomicAdd(&near[0], 1)] = (int32_t)t;
    }
}

// The tokens with several centroids in the band (near[0] of them), a wave each: fp32 scores, and
// fp64 ones where several remain.
__global__ __launch_bounds__(256) void k_assign_near(const int32_t* __restrict__ near, const AsStream* __restrict__ streams,
                                                     int32_t splits, const float* __restrict__ x,
                                                     const float* __restrict__ cen, int32_t n_c,
                                                     int32_t* __restrict__ assign) {
    const int lane = threadIdx.x & 63, part = lane & 3;
    const int n = near[0], stride = (int)gridDim.x * 4;
    for (int k0 = (int)blockIdx.x * 4 + (threadIdx.x >> 6); k0 < n; k0 += stride) {  // wave-uniform
        const int64_t t = near[1 + k0];
        const AsBlocks b = as_blocks(streams, splits * kAsStreams, t, lane);
        const float4* xr = reinterpret_cast<const float4*>(x + t * kDim) + 8 * part;
        float4 xv[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) xv[k] = xr[k];
        auto score32 = [&](int c) {
            const float4* row = reinterpret_cast<const float4*>(cen + (int64_t)c * kDim) + 8 * part;
            float v = 0.f;
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const float4 w = row[k];
                v = __builtin_fmaf(w.x, xv[k].x, v);
                v = __builtin_fmaf(w.y, xv[k].y, v);
                v = __builtin_fmaf(w.z, xv[k].z, v);
                v = __builtin_fmaf(w.w, xv[k].w, v);
            }
            v += __shfl_xor(v, 1, 64);
            v += __shfl_xor(v, 2, 64);
            return v;
        };
        float top = -INFINITY;
        for_blocks(b, lane, [&](int c) {
            if (c < n_c) top = __builtin_fmaxf(top, score32(c));  // uniform over the four lanes
        });
        for (int off = 32; off >= 4; off >>= 1) top = __builtin_fmaxf(top, __shfl_xor(top, off, 64));
        const float thr = top - 1.0f / 32768.0f;
        // fp64 in dimension order: the running sum passes through the four lanes of a centroid
        double best = -INFINITY;
        int id = INT32_MAX;
        for_blocks(b, lane, [&](int c) {
            const bool mine = c < n_c && score32(c) >= thr;
            if (!__any(mine)) return;
            const float4* row = reinterpret_cast<const float4*>(cen + (int64_t)(mine ? c : 0) * kDim) + 8 * part;
            double v = 0.0;
#pragma unroll 1
            for (int seg = 0; seg < 4; ++seg) {
                if (part == seg)
                    for (int k = 0; k < 8; ++k) {
                        const float4 w = row[k], y = xr[k];
                        v = __builtin_fma((double)w.x, (double)y.x, v);
                        v = __builtin_fma((double)w.y, (double)y.y, v);
                        v = __builtin_fma((double)w.z, (double)y.z, v);
                        v = __builtin_fma((double)w.w, (double)y.w, v);
                    }
                v = __shfl(v, (lane & ~3) + seg, 64);
            }
            if (mine) keep_best(best, id, v, c);
        });
        for (int off = 32; off > 0; off >>= 1) {
            const double ob = __shfl_xor(best, off, 64);
            const int oi = __shfl_xor(id, off, 64);
            keep_best(best, id, ob, oi);
        }
        if (lane == 0) assign[t] = id;
    }
}

// S64 of two rows of 128 values, in dimension order (each product is exact).
__device__ __forceinline__ double row_dot64(const float* __restrict__ a, const float* __restrict__ b) {
    double v = 0.0;
#pragma unroll 8
    for (int d = 0; d < kDim / 4; ++d) {
        const float4 p = reinterpret_cast<const float4*>(a)[d], q = reinterpret_cast<const float4*>(b)[d];
        v = __builtin_fma((double)p.x, (double)q.x, v);
        v = __builtin_fma((double)p.y, (double)q.y, v);
        v = __builtin_fma((double)p.z, (double)q.z, v);
        v = __builtin_fma((double)p.w, (double)q.w, v);
    }
    return v;
}

constexpr int kAllThreads = 1024;
constexpr int kAllTokens = 16;   // tokens of a workgroup: the columns of one product, and a wave each
constexpr int kAllList = 2048;   // centroids in the band listed per token

// The tokens whose blocks do not hold the whole band (all[0] of them: centroids that coincide or
// nearly so), kAllTokens to a workgroup: its waves stream the centroids' fp16 rows through the matrix
// cores once for all of them and list, per token, the centroids within the band of the best filter
// score (which the streams hold); each wave then scores one token's list in fp64. A token whose list
// overflows is scored against every centroid. Bound by the rows, 4 MB per workgroup at 2^14
// centroids, which 16 tokens share, and by the lists' fp32 rows.
// Whole builds of a million tokens, 2^14 centroids and one k-means step (a workgroup per token that
// reads the fp16 rows twice -> this; a score matrix for all tokens): 64 equal centroids near 1% of the
// tokens 12.7 -> 7.8 ms (76.7), 900 near 5% 49 -> 12.5 ms (79); 900 near each of 300k tokens 257 -> 36 ms
// (41); without equal centroids 7.0 ms (76.5).
__global__ __launch_bounds__(kAllThreads) void k_assign_all(const int32_t* __restrict__ all,
                                                            const AsStream* __restrict__ streams, int32_t splits,
                                                            const float* __restrict__ x,
                                                            const _Float16* __restrict__ ch,
                                                            const float* __restrict__ cen, int32_t n_c,
                                                            int32_t* __restrict__ assign, int32_t* err) {
    constexpr int NW = kAllThreads / 64;
    constexpr int U = 4;  // tiles of 16 centroids in flight per wave
    static_assert(NW == kAllTokens, "a wave per token");
    __shared__ int s_list[kAllTokens][kAllList];
    __shared__ int s_n[kAllTokens];
    __shared__ float s_thr[kAllTokens];
    __shared__ double s_best[NW];
    __shared__ int s_id[NW], s_close;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int li = lane & 15, g = lane >> 4;
    const int n = all[0];
    const int tiles = (n_c + 15) / 16;
    for (int k0 = (int)blockIdx.x * kAllTokens; k0 < n; k0 += (int)gridDim.x * kAllTokens) {  // uniform
        const int m = n - k0 < kAllTokens ? n - k0 : kAllTokens;
        __syncthreads();
        if (wave < m) {
            const AsBlocks b = as_blocks(streams, splits * kAsStreams, all[1 + k0 + wave], lane);
            if (lane == 0) {
                s_thr[wave] = b.thr;
                s_n[wave] = 0;
            }
        }
        __syncthreads();
        // token operands: K step s: the lane's 8 values of token li (columns past the last repeat it)
        half8 a[4];
        const float4* xr = reinterpret_cast<const float4*>(x + (int64_t)all[1 + k0 + (li < m ? li : m - 1)] * kDim);
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const float4 u = xr[8 * s + 2 * g], v = xr[8 * s + 2 * g + 1];
            a[s] = (half8){(_Float16)u.x, (_Float16)u.y, (_Float16)u.z, (_Float16)u.w,
                           (_Float16)v.x, (_Float16)v.y, (_Float16)v.z, (_Float16)v.w};
        }
        const float thr = li < m ? s_thr[li] : INFINITY;
        for (int t0 = wave; t0 < tiles; t0 += U * NW) {  // wave-uniform
            half8 c[U][4];
#pragma unroll
            for (int u = 0; u < U; ++u) {  // (rows past n_c are there, up to a tile of 128)
                const int t = t0 + u * NW < tiles ? t0 + u * NW : t0;
                const half8* row = reinterpret_cast<const half8*>(ch + ((int64_t)t * 16 + li) * kDim);
#pragma unroll
                for (int s = 0; s < 4; ++s) c[u][s] = row[4 * s + g];
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                floatx4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int s = 0; s < 4; ++s) acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(c[u][s], a[s], acc, 0, 0, 0);
                // lane (li, g): centroids 16 t + 4 g + r against token li
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int cc = (t0 + u * NW) * 16 + 4 * g + r;
                    if (acc[r] >= thr && cc < n_c) {
                        const int p = atomicAdd(&s_n[li], 1);
                        if (p < kAllList) s_list[li][p] = cc;
                    }
                }
            }
        }
        __syncthreads();
        if (wave < m && s_n[wave] <= kAllList) {  // wave-uniform: the list in fp64, a lane each
            const int t = __builtin_amdgcn_readfirstlane(all[1 + k0 + wave]);
            const float* xt = x + (int64_t)t * kDim;
            const int nl = s_n[wave];
            double best = -INFINITY;
            int id = INT32_MAX;
            for (int i = lane; i < nl; i += 64) {
                const int c = s_list[wave][i];
                keep_best(best, id, row_dot64(cen + (int64_t)c * kDim, xt), c);
            }
            for (int off = 32; off > 0; off >>= 1) {
                const double ob = __shfl_xor(best, off, 64);
                const int oi = __shfl_xor(id, off, 64);
                keep_best(best, id, ob, oi);
            }
            if (lane == 0) assign[t] = id;
            if (nl > kAsCand) {  // uniform: too many close ones?
                int close = 0;
                for (int i = lane; i < nl; i += 64)
                    close += row_dot64(cen + (int64_t)s_list[wave][i] * kDim, xt) >= best - 2.5 * kFilterEps ? 1 : 0;
                for (int off = 32; off > 0; off >>= 1) close += __shfl_xor(close, off, 64);
                if (lane == 0 && close > kAsCand) atomicOr(err, kErrArgOverflow);
            }
        }
        for (int w = 0; w < m; ++w) {  // every centroid, a thread each
            if (s_n[w] <= kAllList) continue;  // uniform
            const int64_t t = __builtin_amdgcn_readfirstlane(all[1 + k0 + w]);
            const float* xt = x + t * kDim;
            double best = -INFINITY;
            int id = INT32_MAX;
            for (int c = tid; c < n_c; c += kAllThreads) keep_best(best, id, row_dot64(cen + (int64_t)c * kDim, xt), c);
            for (int off = 32; off > 0; off >>= 1) {
                const double ob = __shfl_xor(best, off, 64);
                const int oi = __shfl_xor(id, off, 64);
                keep_best(best, id, ob, oi);
            }
            if (lane == 0) {
                s_best[wave] = best;
                s_id[wave] = id;
            }
            if (tid == 0) s_close = 0;
            __syncthreads();
            for (int v = 0; v < NW; ++v) keep_best(best, id, s_best[v], s_id[v]);
            int close = 0;
            for (int c = tid; c < n_c; c += kAllThreads)
                close += row_dot64(cen + (int64_t)c * kDim, xt) >= best - 2.5 * kFilterEps ? 1 : 0;
            if (close) atomicAdd(&s_close, close);
            __syncthreads();
            if (tid == 0) {
                assign[t] = id;
                if (s_close > kAsCand) atomicOr(err, kErrArgOverflow);
            }
            __syncthreads();
        }
    }
}

// Splits of the centroids per token tile: enough workgroups to fill the GPU several times over,
// and no more (each adds eight streams per token).
static int32_t assign_splits(int64_t n, int32_t n_c) {
    const int64_t row_tiles = (n + kAsTile - 1) / kAsTile, tiles = (n_c + kAsTile - 1) / kAsTile;
    int64_t s = (4096 + row_tiles - 1) / row_tiles;
    if (s > tiles) s = tiles;
    return (int32_t)(s < 1 ? 1 : (s > 8 ? 8 : s));
}

// Tokens assigned at once: 160 bytes of streams each and split, 84 MB for a whole chunk (one split) and at
// most about twice that (two splits, just below it).
static int64_t assign_chunk(int64_t n) { return std::min<int64_t>(n, (int64_t)1 << 19); }

static size_t al256(size_t b) { return (b + 255) & ~(size_t)255; }

size_t assign_scratch_bytes(int64_t n, int32_t n_c) {
    const int64_t chunk = assign_chunk(n);
    size_t streams = 0;
    for (int64_t m : {chunk, n % chunk ? n % chunk : chunk})  // whole chunks and the last
        streams = std::max(streams, (size_t)m * assign_splits(m, n_c) * kAsStreams * sizeof(AsStream));
    const size_t pad = (size_t)(n_c + kAsTile - 1) / kAsTile * kAsTile;
    return al256(pad * kDim * 2) + 2 * al256(((size_t)chunk + 1) * 4) + al256(streams);
}

// out[t] = the nearest centroid of token t; scratch holds assign_scratch_bytes(n, n_c) bytes.
// Small builds are chains of launches: the first chunk's counters are cleared with the centroids' copies, and
// with up to two tiles of centroids k_assign_all is left out (no stream has a third tile, and the at most 16
// streams keep at most 32 blocks, whose 512 centroids fit). With the k-means sums and counts cleared together and
// the inputs checked in fewer launches, 3,000 tokens, 16 centroids and four k-means steps take 70 launches instead
// of 91 and 742 -> 603 us (the score matrix: 63 launches, 624 us).
void launch_assign(const float* x, int64_t n, const float* cen, int32_t n_c, void* scratch, int32_t* out, int32_t* err,
                   hipStream_t s) {
    if (n <= 0) return;
    const int64_t pad = (int64_t)(n_c + kAsTile - 1) / kAsTile * kAsTile, chunk = assign_chunk(n);
    char* p = (char*)scratch;
    _Float16* ch = (_Float16*)p;
    p += al256((size_t)pad * kDim * 2);
    int32_t* near = (int32_t*)p;
    p += al256(((size_t)chunk + 1) * 4);
    int32_t* all = (int32_t*)p;
    p += al256(((size_t)chunk + 1) * 4);
    AsStream* streams = (AsStream*)p;
    hipLaunchKernelGGL(k_half_rows, dim3((unsigned)((pad * (kDim / 8) + 255) / 256)), dim3(256), 0, s, cen, (int64_t)n_c,
                       pad, ch, near, all);
    for (int64_t a = 0; a < n; a += chunk) {
        const int64_t m = std::min(chunk, n - a);
        const int32_t splits = assign_splits(m, n_c);
        if (a > 0) {
            launch_fill_i32(near, 1, 0, s);
            launch_fill_i32(all, 1, 0, s);
        }
        hipLaunchKernelGGL(k_assign_gemm, dim3((unsigned)((m + kAsTile - 1) / kAsTile), (unsigned)splits), dim3(256), 0, s,
                           x + a * kDim, m, ch, n_c, streams);
        hipLaunchKernelGGL(k_assign_pick, dim3((unsigned)((m + 3) / 4)), dim3(256), 0, s, streams, splits, m, x + a * kDim,
                           ch, n_c, out + a, near, all);
        hipLaunchKernelGGL(k_assign_near, dim3(1024), dim3(256), 0, s, near, streams, splits, x + a * kDim, cen, n_c, out + a);
        if (n_c > 2 * kAsTile)
            hipLaunchKernelGGL(k_assign_all, dim3(256), dim3(kAllThreads), 0, s, all, streams, splits, x + a * kDim, ch,
                               cen, n_c, out + a, err);
    }
}

}  // namespace warp
