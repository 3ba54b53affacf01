// Batch norm (training mode, statistics of the worker's own shard) and the
// bias / ReLU backward, all as per-channel column reductions over a row-major
// [M][C] activation matrix followed by an elementwise pass.  HBM-bound.
//
// One launch covers every shard of the pass; statistics and parameter gradients
// are formed per shard (a row block never crosses a shard's end).
//
// Reduction scheme (deterministic, no atomics): the rows are cut into about
// kRedRowBlocks blocks at most; a workgroup of TX x TY lanes owns 32*VEC channels of
// one row block, each lane accumulating one 16-byte channel vector over every
// TY-th row in float32; lanes are combined through LDS; a second tiny kernel
// adds a shard's row blocks in float64.
#include <algorithm>
#include <type_traits>

#include "dev_common.h"
#include "kernels.h"
#include "profiler.h"
#include "tune.h"

namespace edl {

constexpr float kBnEps = 1e-5f;
constexpr float kBnRunningMomentum = 0.1f;

struct RedShape {
    int TX, TY, cvecs, row_blocks, rows_per_block, col_blocks;
    dim3 block;
};

static RedShape red_shape(int64_t M, int C, int VEC) {
    RedShape s;
    s.cvecs = (C + VEC - 1) / VEC;
    int tx = 1;
    while (tx < s.cvecs && tx < 32) tx <<= 1;
    s.TX = tx;
    s.TY = 256 / tx;
    s.col_blocks = (s.cvecs + tx - 1) / tx;
    // aim at ~2048 workgroups, at least TY*4 rows each
    int64_t rb = (2048 + s.col_blocks - 1) / s.col_blocks;
    const int64_t max_rb = (M + (int64_t)s.TY * 4 - 1) / ((int64_t)s.TY * 4);
    if (rb > max_rb) rb = max_rb;
    if (rb > kRedRowBlocks) rb = kRedRowBlocks;
    if (rb < 1) rb = 1;
    s.row_blocks = (int)rb;
    s.rows_per_block = (int)((M + rb - 1) / rb);
    s.block = dim3(s.TX, s.TY);
    return s;
}

size_t norm_sums_floats(int dtype, int64_t M, int C, int p) {
    const int vec = dtype == 1 ? 8 : 4;
    return (size_t)2 * C * (red_shape(M, C, C % vec == 0 ? vec : 1).row_blocks + p);
}

// Loads VEC channels of row r starting at channel c0 (zero beyond C).
template <typename T, int VEC>
__device__ __forceinline__ void load_row(const T* base, int64_t r, int C, int c0, float (&out)[VEC]) {
    if (VEC > 1) {
        const Vec16<T> v = load_vec(base + r * C + c0);
        #pragma unroll
        for (int e = 0; e < VEC; ++e) out[e] = Elem<T>::to_f32(v.e[e]);
    } else {
        out[0] = Elem<T>::to_f32(base[r * C + c0]);
    }
}

// the same through a non-temporal load: for a tensor this pass reads once and nothing reads again soon
typedef unsigned int nt_u32x4 __attribute__((ext_vector_type(4)));
template <typename T, int VEC>
__device__ __forceinline__ void load_row_nt(const T* base, int64_t r, int C, int c0, float (&out)[VEC]) {
    if (VEC > 1) {
        Vec16<T> v;
        const nt_u32x4 q = __builtin_nontemporal_load(reinterpret_cast<const nt_u32x4*>(base + r * C + c0));
        v.u = make_uint4(q.x, q.y, q.z, q.w);
        #pragma unroll
        for (int e = 0; e < VEC; ++e) out[e] = Elem<T>::to_f32(v.e[e]);
    } else {
        out[0] = Elem<T>::to_f32(base[r * C + c0]);
    }
}

template <typename T, int VEC>
__device__ __forceinline__ void store_row(T* base, int64_t r, int C, int c0, const float (&in)[VEC]) {
    if (VEC > 1) {
        Vec16<T> v;
        #pragma unroll
        for (int e = 0; e < VEC; ++e) v.e[e] = Elem<T>::from_f32(in[e]);
        store_vec(base + r * C + c0, v);
    } else {
        base[r * C + c0] = Elem<T>::from_f32(in[0]);
    }
}

// KIND 0: a = x, b = x^2                       (batch-norm statistics)
// KIND 1: a = dy', b = dy' * xhat              (batch-norm backward sums), dy' = dy * (y>0) if relu
// KIND 2: a = dy' (written back in place), b=0 (bias gradient / ReLU mask)
// KIND 3: a = dy', b=0, nothing written back
// LONG: in two levels (see long_blocks)
template <typename T, int VEC, int KIND, bool LONG>
__global__ __launch_bounds__(256) void colreduce_kernel(const T* __restrict__ x, const T* __restrict__ y, T* dy,
                                                        const float* __restrict__ mean_rstd, RowCut cut, int C,
                                                        int relu, float* __restrict__ partial, GradDst dbias) {
    __shared__ float red[2][256 * VEC];
    int r0, r1;
    const int sh = locate_block(cut, blockIdx.y, r0, r1);
    const int tx = threadIdx.x, ty = threadIdx.y, TX = blockDim.x, TY = blockDim.y;
    const int c0 = (blockIdx.x * TX + tx) * VEC;
    const bool active = c0 < C;
    float a[VEC], b[VEC];
    #pragma unroll
    for (int e = 0; e < VEC; ++e) { a[e] = 0.f; b[e] = 0.f; }
    float mu[VEC], rs[VEC];
    if (KIND == 1 && active) {
        const float* const ms = mean_rstd + (int64_t)sh * 2 * C;
        #pragma unroll
        for (int e = 0; e < VEC; ++e) { mu[e] = ms[c0 + e]; rs[e] = ms[C + c0 + e]; }
    }
    if (active) {
        // U rows per trip, every load of a trip issued before the first use: the loads are unconditional
        // (without ReLU y is a valid tensor that is read and ignored), so none of them waits for another.
        auto rows = [&](int64_t r, auto ucount) {
            constexpr int U = decltype(ucount)::value;
            float xv[U][VEC], yv[U][VEC], g[U][VEC];
            #pragma unroll
            for (int u = 0; u < U; ++u) {
                const int64_t rr = r + (int64_t)u * TY;
                if (KIND == 0) {
                    load_row<T, VEC>(x, rr, C, c0, xv[u]);
                } else {
                    load_row<T, VEC>(dy, rr, C, c0, g[u]);
                    load_row<T, VEC>(y, rr, C, c0, yv[u]);
                    if (KIND == 1) load_row<T, VEC>(x, rr, C, c0, xv[u]);
                }
            }
            #pragma unroll
            for (int u = 0; u < U; ++u) {
                if (KIND == 0) {
                    #pragma unroll
                    for (int e = 0; e < VEC; ++e) { a[e] += xv[u][e]; b[e] += xv[u][e] * xv[u][e]; }
                } else {
                    #pragma unroll
                    for (int e = 0; e < VEC; ++e) g[u][e] = (!relu || yv[u][e] > 0.f) ? g[u][e] : 0.f;
                    if (KIND == 1) {
                        #pragma unroll
                        for (int e = 0; e < VEC; ++e) { a[e] += g[u][e]; b[e] += g[u][e] * ((xv[u][e] - mu[e]) * rs[e]); }
                    } else {
                        if (KIND == 2 && relu) store_row<T, VEC>(dy, r + (int64_t)u * TY, C, c0, g[u]);
                        #pragma unroll
                        for (int e = 0; e < VEC; ++e) a[e] += g[u][e];
                    }
                }
            }
        };
        float fa[VEC], fb[VEC];      // LONG: sums of 16 rows are added up here
        #pragma unroll
        for (int e = 0; e < VEC; ++e) { fa[e] = 0.f; fb[e] = 0.f; }
        int64_t r = r0 + ty;
        for (int trip = 1; r + TY < r1; r += 2 * (int64_t)TY, ++trip) {
            rows(r, std::integral_constant<int, 2>());
            if (LONG && (trip & 7) == 0) {
                #pragma unroll
                for (int e = 0; e < VEC; ++e) { fa[e] += a[e]; fb[e] += b[e]; a[e] = 0.f; b[e] = 0.f; }
            }
        }
        if (r < r1) rows(r, std::integral_constant<int, 1>());
        if (LONG)
            #pragma unroll
            for (int e = 0; e < VEC; ++e) { a[e] += fa[e]; b[e] += fb[e]; }
    }
    const int lane = ty * TX + tx;
    #pragma unroll
    for (int e = 0; e < VEC; ++e) { red[0][lane * VEC + e] = a[e]; red[1][lane * VEC + e] = b[e]; }
    __syncthreads();
    if (ty == 0 && active) {
        using Sum = std::conditional_t<LONG, double, float>;
        Sum sa[VEC], sb[VEC];
        #pragma unroll
        for (int e = 0; e < VEC; ++e) { sa[e] = a[e]; sb[e] = b[e]; }
        for (int j = 1; j < TY; ++j) {
            #pragma unroll
            for (int e = 0; e < VEC; ++e) {
                sa[e] += red[0][(j * TX + tx) * VEC + e];
                sb[e] += red[1][(j * TX + tx) * VEC + e];
            }
        }
        #pragma unroll
        for (int e = 0; e < VEC; ++e) { a[e] = (float)sa[e]; b[e] = (float)sb[e]; }
        if (KIND >= 2 && dbias.g != nullptr) {      // a block is a shard: the sums need no finishing kernel
            #pragma unroll
            for (int e = 0; e < VEC; ++e)
                if (c0 + e < C) dbias.g[(int64_t)cut.k[sh] * dbias.stride + c0 + e] = a[e];
            return;
        }
        // partial[sum kind][channel][row block]: a channel's partial sums are contiguous for the finishing kernel
        #pragma unroll
        for (int e = 0; e < VEC; ++e) {
            if (c0 + e < C) {
                partial[(int64_t)(c0 + e) * gridDim.y + blockIdx.y] = a[e];
                partial[(int64_t)(C + c0 + e) * gridDim.y + blockIdx.y] = b[e];
            }
        }
    }
}

// Sums of shard sh's row blocks of one channel by W waves (64 * W lanes): lane L takes blocks L, L + 64*W, ...
// (coalesced) in float64, then a butterfly and, for several waves, LDS.  One wave takes four channels' worth of
// launches off the grid where the blocks are few; the four-wave form is for the first layers of large images, whose
// thousands of blocks would be a long chain of loads for one wave.  Valid in lane 0 of the channel's lanes.
template <int W>
__device__ __forceinline__ void sum_partials(const float* __restrict__ partial, const RowCut& cut, int sh, int C, int c, int sub,
                                             double& s, double& q) {
    s = 0;
    q = 0;
    constexpr int L = 64 * W;
    if (c < C) {
        const int stride = cut.blk0[cut.p], end = cut.blk0[sh + 1];
        const float* ps = partial + (int64_t)c * stride;
        const float* pq = partial + (int64_t)(C + c) * stride;
        // four loads of each kind in flight per lane (the partial sums of a channel are contiguous)
        int j = cut.blk0[sh] + sub;
        for (; j + 3 * L < end; j += 4 * L) {
            const float s0 = ps[j], s1 = ps[j + L], s2 = ps[j + 2 * L], s3 = ps[j + 3 * L];
            const float q0 = pq[j], q1 = pq[j + L], q2 = pq[j + 2 * L], q3 = pq[j + 3 * L];
            s += (double)s0; s += (double)s1; s += (double)s2; s += (double)s3;
            q += (double)q0; q += (double)q1; q += (double)q2; q += (double)q3;
        }
        for (; j < end; j += L) {
            s += (double)ps[j];
            q += (double)pq[j];
        }
    }
    for (int o = 32; o > 0; o >>= 1) {
        s += __shfl_xor(s, o, 64);
        q += __shfl_xor(q, o, 64);
    }
    if (W > 1) {
        __shared__ double part[2][W];
        if ((sub & 63) == 0) { part[0][sub >> 6] = s; part[1][sub >> 6] = q; }
        __syncthreads();
        s = 0;
        q = 0;
        #pragma unroll
        for (int w = 0; w < W; ++w) { s += part[0][w]; q += part[1][w]; }
    }
}

// grid of the finishing kernels: (channels, shards); blockDim = 256 lanes = 4 / W channels
template <int W> __device__ __forceinline__ int fin_channel() { return W > 1 ? blockIdx.x : blockIdx.x * 4 + (threadIdx.x >> 6); }
template <int W> __device__ __forceinline__ int fin_lane() { return W > 1 ? threadIdx.x : (threadIdx.x & 63); }

// mean / rstd from the partial sums; running statistics of the worker whose
// model a joiner would receive (unbiased variance, momentum 0.1): the pass's first shard
template <int W>
__global__ __launch_bounds__(256) void bn_stats_finalize_kernel(const float* __restrict__ partial, RowCut cut,
                                                                int C, float* __restrict__ mean_rstd, float* running) {
    const int c = fin_channel<W>(), sub = fin_lane<W>(), sh = blockIdx.y;
    double s, q;
    sum_partials<W>(partial, cut, sh, C, c, sub, s, q);
    if (c >= C || sub != 0) return;
    const int M = cut.row0[sh + 1] - cut.row0[sh];
    mean_rstd += (int64_t)sh * 2 * C;
    const double mean = s / (double)M;
    double var = q / (double)M - mean * mean;
    if (var < 0) var = 0;
    mean_rstd[c] = (float)mean;
    mean_rstd[C + c] = (float)(1.0 / sqrt(var + (double)kBnEps));
    if (running && sh == 0) {
        const double unbiased = M > 1 ? var * (double)M / (double)(M - 1) : var;
        running[c] = (1.f - kBnRunningMomentum) * running[c] + kBnRunningMomentum * (float)mean;
        running[C + c] = (1.f - kBnRunningMomentum) * running[C + c] + kBnRunningMomentum * (float)unbiased;
    }
}

// dgamma = sum dy'*xhat, dbeta = sum dy'; coef = {dbeta/M, dgamma/M}
template <int W>
__global__ __launch_bounds__(256) void bn_bwd_finalize_kernel(const float* __restrict__ partial, RowCut cut,
                                                              int C, float* __restrict__ dgamma, float* __restrict__ dbeta,
                                                              int64_t grad_stride, float* __restrict__ coef) {
    const int c = fin_channel<W>(), sub = fin_lane<W>(), sh = blockIdx.y;
    double s, q;
    sum_partials<W>(partial, cut, sh, C, c, sub, s, q);
    if (c >= C || sub != 0) return;
    const int M = cut.row0[sh + 1] - cut.row0[sh];
    const int64_t to = (int64_t)cut.k[sh] * grad_stride;
    dbeta[to + c] = (float)s;
    dgamma[to + c] = (float)q;
    coef += (int64_t)sh * 2 * C;
    coef[c] = (float)(s / (double)M);
    coef[C + c] = (float)(q / (double)M);
}

template <int W>
__global__ __launch_bounds__(256) void bias_finalize_kernel(const float* __restrict__ partial, RowCut cut, int C,
                                                            float* __restrict__ dbias, int64_t grad_stride) {
    const int c = fin_channel<W>(), sub = fin_lane<W>(), sh = blockIdx.y;
    double s, q;
    sum_partials<W>(partial, cut, sh, C, c, sub, s, q);
    if (c >= C || sub != 0) return;
    dbias[(int64_t)cut.k[sh] * grad_stride + c] = (float)s;
}

// y = relu(gamma * (x - mean) * rstd + beta + res); grid: (groups of 256 * U vectors of the largest shard, shards)
// No load sits behind a run-time branch, so that all of a lane's loads are in flight together.
// U > 1 (256 a multiple of the vectors per row): a lane's vectors are 256 apart, all of the same channels, whose
// coefficients are read once for all of them - with one vector per lane they are twice the bytes of the data.
template <typename T, int VEC, int U, bool RES, bool NT>
__global__ __launch_bounds__(256) void bn_apply_kernel(const T* __restrict__ x, const T* __restrict__ res,
                                                       T* __restrict__ y, const float* __restrict__ gamma,
                                                       const float* __restrict__ beta, const float* __restrict__ mean_rstd,
                                                       RowCut shards, int C, int cvecs, int relu, unsigned char* __restrict__ sign) {
    const int sh = blockIdx.y, row0 = shards.row0[sh];
    const int64_t total = (int64_t)(shards.row0[sh + 1] - row0) * cvecs;
    const int64_t i0 = (int64_t)blockIdx.x * (256 * U) + threadIdx.x;
    if (i0 >= total) return;
    mean_rstd += (int64_t)sh * 2 * C;
    const int c0 = (int)(i0 % cvecs) * VEC;
    const int64_t base = (int64_t)row0 * cvecs;
    float xv[U][VEC], rv[U][VEC];
    #pragma unroll
    for (int u = 0; u < U; ++u) {
        const int64_t i = base + (i0 + u * 256 < total ? i0 + u * 256 : i0);
        if (NT) load_row_nt<T, VEC>(x, i, VEC, 0, xv[u]); else load_row<T, VEC>(x, i, VEC, 0, xv[u]);
        if (RES) { if (NT) load_row_nt<T, VEC>(res, i, VEC, 0, rv[u]); else load_row<T, VEC>(res, i, VEC, 0, rv[u]); }
    }
    float mu[VEC], sc[VEC], be[VEC];
    #pragma unroll
    for (int e = 0; e < VEC; ++e) { mu[e] = mean_rstd[c0 + e]; sc[e] = gamma[c0 + e] * mean_rstd[C + c0 + e]; be[e] = beta[c0 + e]; }
    #pragma unroll
    for (int u = 0; u < U; ++u) {
        if (i0 + u * 256 >= total) break;
        float out[VEC];
        #pragma unroll
        for (int e = 0; e < VEC; ++e) {
            out[e] = (xv[u][e] - mu[e]) * sc[e] + be[e];
            if (RES) out[e] += rv[u][e];
            if (relu) out[e] = out[e] > 0.f ? out[e] : 0.f;
        }
        store_row<T, VEC>(y, base + i0 + u * 256, VEC, 0, out);
        if (VEC == 8 && sign != nullptr) {
            unsigned bits = 0;      // of the stored values
            #pragma unroll
            for (int e = 0; e < VEC; ++e) bits |= (Elem<T>::to_f32(Elem<T>::from_f32(out[e])) > 0.f ? 1u : 0u) << e;
            sign[base + i0 + u * 256] = (unsigned char)bits;
        }
    }
}

// dx = gamma*rstd*(dy' - coef0 - xhat*coef1) ; dres (+)= dy'; grid as above
// MASK: dy' = dy * (y > 0) is formed here (else dy arrives masked, or there is no ReLU, and y is not read);
// ACC: dres already holds a gradient that dy' is added to.  Compile-time, so that no load sits behind a
// run-time branch and none is issued that is not needed.
template <typename T, int VEC, int U, bool MASK, bool ACC, bool NT>
__global__ __launch_bounds__(256) void bn_bwd_apply_kernel(const T* __restrict__ x, const T* __restrict__ y,
                                                           const T* __restrict__ dy, T* __restrict__ dx, T* dres,
                                                           const float* __restrict__ gamma,
                                                           const float* __restrict__ mean_rstd,
                                                           const float* __restrict__ coef, RowCut shards, int C, int cvecs) {
    const int sh = blockIdx.y, row0 = shards.row0[sh];
    const int64_t total = (int64_t)(shards.row0[sh + 1] - row0) * cvecs;
    const int64_t i0 = (int64_t)blockIdx.x * (256 * U) + threadIdx.x;
    if (i0 >= total) return;
    mean_rstd += (int64_t)sh * 2 * C;
    coef += (int64_t)sh * 2 * C;
    const int c0 = (int)(i0 % cvecs) * VEC;
    const int64_t base = (int64_t)row0 * cvecs;
    float xv[U][VEC], yv[U][VEC], g[U][VEC], old[U][VEC];
    #pragma unroll
    for (int u = 0; u < U; ++u) {
        const int64_t i = base + (i0 + u * 256 < total ? i0 + u * 256 : i0);
        if (NT) load_row_nt<T, VEC>(x, i, VEC, 0, xv[u]); else load_row<T, VEC>(x, i, VEC, 0, xv[u]);
        load_row<T, VEC>(dy, i, VEC, 0, g[u]);
        if (MASK) { if (NT) load_row_nt<T, VEC>(y, i, VEC, 0, yv[u]); else load_row<T, VEC>(y, i, VEC, 0, yv[u]); }
        if (ACC) load_row<T, VEC>(dres, i, VEC, 0, old[u]);
    }
    float mu[VEC], rs[VEC], ga[VEC], k0[VEC], k1[VEC];
    #pragma unroll
    for (int e = 0; e < VEC; ++e) {
        mu[e] = mean_rstd[c0 + e]; rs[e] = mean_rstd[C + c0 + e]; ga[e] = gamma[c0 + e] * rs[e];
        k0[e] = coef[c0 + e]; k1[e] = coef[C + c0 + e];
    }
    #pragma unroll
    for (int u = 0; u < U; ++u) {
        if (i0 + u * 256 >= total) break;
        const int64_t i = base + i0 + u * 256;
        float out[VEC];
        #pragma unroll
        for (int e = 0; e < VEC; ++e) {
            if (MASK) g[u][e] = yv[u][e] > 0.f ? g[u][e] : 0.f;
            const float xh = (xv[u][e] - mu[e]) * rs[e];
            out[e] = ga[e] * (g[u][e] - k0[e] - xh * k1[e]);
        }
        store_row<T, VEC>(dx, i, VEC, 0, out);
        if (dres) {
            if (ACC) {
                #pragma unroll
                for (int e = 0; e < VEC; ++e) g[u][e] += old[u][e];
            }
            store_row<T, VEC>(dres, i, VEC, 0, g[u]);
        }
    }
}

// ---- both finishing steps inside the element-wise pass -------------------------------------------------------------------
// Where a shard's sums are few, every workgroup of the element-wise pass adds up those of the channels that it owns: a launch
// of 4 us between two dependent ones falls away for some hundred loads from the caches, issued behind those of the
// workgroup's own rows.  A workgroup owns a slice of up to 64 channels (all of them in narrow layers) of 256 * U vectors; the
// first of a slice also stores what later passes read.  Latency bounds the pass then: all its loads (rows, sums, scales) are
// issued before the first wait, none behind a branch.
//
// Taken up to 128 blocks of a channel in a shard and 20 MB of sums read by all workgroups together: a workgroup of 98 blocks
// reads 50 KB, and with some 400 to 1,600 workgroups of that it takes as long as the launch that it saves, or longer (us per step
// without / at 20 / 40 / 80 MB: ResNet-50, shard of 32, 4,036 / 3,975 / 3,976 / 3,976; three shards of 161x161 images 4,535 / 4,440 /
// 4,439 / 4,457; ResNet-20, 8 shards of 16, 1,383 / 1,224).

constexpr int kSlice = 64;

// Sums over a shard's row blocks, of SLICE channels from c_lo on: out[kind * SLICE + channel], in float64.  Eight lanes per sum,
// 32 sums at a time, four blocks per load and two loads of each sum in flight.  A load that would end behind the shard
// starts earlier, and what it repeats is not counted (with fewer than four blocks it reads up to three floats behind them,
// which belong to the scratch).
template <int SLICE>
__device__ __forceinline__ void slice_sums(const float* __restrict__ partial, const RowCut& cut, int sh, int C, int c_lo, double* out) {
    const int tid = threadIdx.x, sub = tid & 7, stride = cut.blk0[cut.p], first = cut.blk0[sh], end = cut.blk0[sh + 1];
    constexpr int P = 2 * SLICE / 32;
    struct __attribute__((packed, aligned(4))) Four { float v[4]; };
    const float* p[P];
    double a[P];
    #pragma unroll
    for (int i = 0; i < P; ++i) {
        const int col = i * 32 + (tid >> 3), kind = col / SLICE;
        p[i] = partial + (int64_t)(kind * C + c_lo + col % SLICE) * stride;
        a[i] = 0;
    }
    for (int j0 = first; j0 < end; j0 += 64) {
        Four v[2][P];
        #pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int j = j0 + 32 * h + 4 * sub, at = max(min(j, end - 4), first);
            #pragma unroll
            for (int i = 0; i < P; ++i) v[h][i] = *reinterpret_cast<const Four*>(p[i] + at);
        }
        #pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int j = j0 + 32 * h + 4 * sub, at = max(min(j, end - 4), first);
            #pragma unroll
            for (int i = 0; i < P; ++i)
                #pragma unroll
                for (int k = 0; k < 4; ++k) a[i] += (at + k >= j && at + k < end) ? (double)v[h][i].v[k] : 0.0;
        }
    }
    #pragma unroll
    for (int i = 0; i < P; ++i) {
        #pragma unroll
        for (int o = 4; o > 0; o >>= 1) a[i] += __shfl_xor(a[i], o, 64);
        if (sub == 0) out[i * 32 + (tid >> 3)] = a[i];
    }
}

// 16 bytes that are not converted yet, so that the load stays in flight
__device__ __forceinline__ uint4 raw_vec(const void* base, int64_t i) { return reinterpret_cast<const uint4*>(base)[i]; }
template <typename T> __device__ __forceinline__ void unpack(const uint4& u, float (&out)[Elem<T>::VEC]) {
    Vec16<T> v;
    v.u = u;
    #pragma unroll
    for (int e = 0; e < Elem<T>::VEC; ++e) out[e] = Elem<T>::to_f32(v.e[e]);
}

// The rows and channels of a workgroup: vectors at(u) of the tensor, `inside` the shard or not (then at() is the last row's)
template <int VEC, int SLICE, int U>
struct SliceTile {
    static constexpr int LANES = SLICE / VEC, STEP = 256 / LANES;
    int lane_vec, c_lo, row, rows, cvecs;
    int64_t base;
    __device__ __forceinline__ SliceTile(const RowCut& cut, int sh, int C) {
        cvecs = C / VEC;
        c_lo = blockIdx.y * SLICE;
        lane_vec = (int)threadIdx.x % LANES;
        row = (int)blockIdx.x * (STEP * U) + (int)threadIdx.x / LANES;
        rows = cut.row0[sh + 1] - cut.row0[sh];
        base = (int64_t)cut.row0[sh] * cvecs + blockIdx.y * LANES + lane_vec;
    }
    __device__ __forceinline__ bool empty() const { return (int)blockIdx.x * (STEP * U) >= rows; }
    __device__ __forceinline__ bool inside(int u) const { return row + u * STEP < rows; }
    __device__ __forceinline__ int64_t at(int u) const { return base + (int64_t)(inside(u) ? row + u * STEP : rows - 1) * cvecs; }
};

// bn_stats_finalize_kernel and bn_apply_kernel in one.  grid: (groups of rows of the largest shard, slices, shards)
template <typename T, int SLICE, int U, bool RES>
__global__ __launch_bounds__(256) void bn_finish_apply_kernel(const T* __restrict__ x, const T* __restrict__ res, T* __restrict__ y,
                                                              const float* __restrict__ gamma, const float* __restrict__ beta,
                                                              const float* __restrict__ partial, RowCut cut, int C, int relu,
                                                              float* __restrict__ mean_rstd, float* running, unsigned char* __restrict__ sign) {
    constexpr int VEC = Elem<T>::VEC;
    __shared__ double sums[2 * SLICE];
    __shared__ __attribute__((aligned(16))) float cf[3][SLICE];
    const int sh = blockIdx.z, tid = threadIdx.x;
    const SliceTile<VEC, SLICE, U> t(cut, sh, C);
    if (t.empty()) return;
    uint4 xr[U], rr[U];
    #pragma unroll
    for (int u = 0; u < U; ++u) {
        xr[u] = raw_vec(x, t.at(u));
        if (RES) rr[u] = raw_vec(res, t.at(u));
    }
    // what the sums are finished with is fetched beside them
    const int c = t.c_lo + (tid < SLICE ? tid : 0);
    const bool keeps = blockIdx.x == 0 && running != nullptr && sh == 0;
    const float *const rm = keeps ? running + c : gamma + c, *const rv0 = keeps ? running + C + c : gamma + c;
    const float ga = gamma[c], be0 = beta[c], run_mean = *rm, run_var = *rv0;
    const double M = t.rows, per_row = 1.0 / M;
    slice_sums<SLICE>(partial, cut, sh, C, t.c_lo, sums);
    __syncthreads();
    if (tid < SLICE) {
        const double mean = sums[tid] * per_row;
        double var = sums[SLICE + tid] * per_row - mean * mean;
        if (var < 0) var = 0;
        const float mu = (float)mean, rs = (float)rsqrt(var + (double)kBnEps);
        cf[0][tid] = mu;
        cf[1][tid] = ga * rs;
        cf[2][tid] = be0;
        if (blockIdx.x == 0) {
            mean_rstd[(int64_t)sh * 2 * C + c] = mu;
            mean_rstd[(int64_t)sh * 2 * C + C + c] = rs;
            if (keeps) {
                const double unbiased = t.rows > 1 ? var * M / (M - 1) : var;
                running[c] = (1.f - kBnRunningMomentum) * run_mean + kBnRunningMomentum * mu;
                running[C + c] = (1.f - kBnRunningMomentum) * run_var + kBnRunningMomentum * (float)unbiased;
            }
        }
    }
    __syncthreads();
    float mu[VEC], sc[VEC], be[VEC];
    #pragma unroll
    for (int e = 0; e < VEC; ++e) { mu[e] = cf[0][t.lane_vec * VEC + e]; sc[e] = cf[1][t.lane_vec * VEC + e]; be[e] = cf[2][t.lane_vec * VEC + e]; }
    #pragma unroll
    for (int u = 0; u < U; ++u) {
        if (!t.inside(u)) break;
        float out[VEC], xv[VEC], rv[VEC];
        unpack<T>(xr[u], xv);
        if (RES) unpack<T>(rr[u], rv);
        #pragma unroll
        for (int e = 0; e < VEC; ++e) {
            out[e] = (xv[e] - mu[e]) * sc[e] + be[e];
            if (RES) out[e] += rv[e];
            if (relu) out[e] = out[e] > 0.f ? out[e] : 0.f;
        }
        store_row<T, VEC>(y, t.at(u), VEC, 0, out);
        if (VEC == 8 && sign != nullptr) {
            unsigned bits = 0;      // of the stored values
            #pragma unroll
            for (int e = 0; e < VEC; ++e) bits |= (Elem<T>::to_f32(Elem<T>::from_f32(out[e])) > 0.f ? 1u : 0u) << e;
            sign[t.at(u)] = (unsigned char)bits;
        }
    }
}

// bn_bwd_finalize_kernel and bn_bwd_apply_kernel in one
template <typename T, int SLICE, int U, bool MASK>
__global__ __launch_bounds__(256) void bn_finish_bwd_kernel(const T* __restrict__ x, const T* __restrict__ y, const T* __restrict__ dy,
                                                            T* __restrict__ dx, T* dres, const float* __restrict__ gamma,
                                                            const float* __restrict__ mean_rstd, const float* __restrict__ partial, RowCut cut, int C,
                                                            float* __restrict__ dgamma, float* __restrict__ dbeta, int64_t grad_stride) {
    constexpr int VEC = Elem<T>::VEC;
    __shared__ double sums[2 * SLICE];
    __shared__ __attribute__((aligned(16))) float cf[5][SLICE];
    const int sh = blockIdx.z, tid = threadIdx.x;
    const SliceTile<VEC, SLICE, U> t(cut, sh, C);
    if (t.empty()) return;
    uint4 xr[U], yr[U], gr[U];
    #pragma unroll
    for (int u = 0; u < U; ++u) {
        xr[u] = raw_vec(x, t.at(u));
        gr[u] = raw_vec(dy, t.at(u));
        if (MASK) yr[u] = raw_vec(y, t.at(u));
    }
    const int c = t.c_lo + (tid < SLICE ? tid : 0);
    const float mu0 = mean_rstd[(int64_t)sh * 2 * C + c], rs0 = mean_rstd[(int64_t)sh * 2 * C + C + c], ga0 = gamma[c];
    const double per_row = 1.0 / (double)t.rows;
    slice_sums<SLICE>(partial, cut, sh, C, t.c_lo, sums);
    __syncthreads();
    if (tid < SLICE) {
        const double s = sums[tid], q = sums[SLICE + tid];
        cf[0][tid] = mu0;
        cf[1][tid] = rs0;
        cf[2][tid] = ga0 * rs0;
        cf[3][tid] = (float)(s * per_row);
        cf[4][tid] = (float)(q * per_row);
        if (blockIdx.x == 0) {
            const int64_t to = (int64_t)cut.k[sh] * grad_stride + c;
            dbeta[to] = (float)s;
            dgamma[to] = (float)q;
        }
    }
    __syncthreads();
    float mu[VEC], rs[VEC], ga[VEC], k0[VEC], k1[VEC];
    #pragma unroll
    for (int e = 0; e < VEC; ++e) {
        const int i = t.lane_vec * VEC + e;
        mu[e] = cf[0][i]; rs[e] = cf[1][i]; ga[e] = cf[2][i]; k0[e] = cf[3][i]; k1[e] = cf[4][i];
    }
    #pragma unroll
    for (int u = 0; u < U; ++u) {
        if (!t.inside(u)) break;
        float out[VEC], xv[VEC], yv[VEC], g[VEC];
        unpack<T>(xr[u], xv);
        unpack<T>(gr[u], g);
        if (MASK) unpack<T>(yr[u], yv);
        #pragma unroll
        for (int e = 0; e < VEC; ++e) {
            if (MASK) g[e] = yv[e] > 0.f ? g[e] : 0.f;
            const float xh = (xv[e] - mu[e]) * rs[e];
            out[e] = ga[e] * (g[e] - k0[e] - xh * k1[e]);
        }
        store_row<T, VEC>(dx, t.at(u), VEC, 0, out);
        if (dres) store_row<T, VEC>(dres, t.at(u), VEC, 0, g);
    }
}

// How a pass over S with these sums is cut for the kernels above; slice == 0: it takes two launches
struct SlicePlan { int slice = 0, U = 1; dim3 grid; };
static SlicePlan plan_slices(const ShardSet& S, int hw, int C, int VEC, const RowCut& sums) {
    SlicePlan p;
    if (VEC == 1 || !(C == 16 || C == 32 || C % kSlice == 0) || sums.most > tune().bn_finish_blocks) return p;
    const int slice = std::min(C, kSlice);
    const int64_t groups = (int64_t)S.plan * hw * (C / VEC) / 256;
    p.U = groups >= 4 * 384 ? 4 : groups >= 2 * 384 ? 2 : 1;
    // what the workgroups read of the sums together
    if (groups / p.U * sums.most * slice * 8 > tune().bn_finish_bytes) return p;
    p.slice = slice;
    const int rows = 256 / (slice / VEC) * p.U;
    p.grid = dim3((unsigned)(((int64_t)S.largest() * hw + rows - 1) / rows), C / slice, S.p);
    return p;
}
// LAUNCH(slice, U) for the plan
#define EDL_BN_SLICES(P, LAUNCH)                                                                                      \
    do {                                                                                                              \
        if ((P).slice == 16) { if ((P).U == 4) LAUNCH(16, 4); else if ((P).U == 2) LAUNCH(16, 2); else LAUNCH(16, 1); }  \
        else if ((P).slice == 32) { if ((P).U == 4) LAUNCH(32, 4); else if ((P).U == 2) LAUNCH(32, 2); else LAUNCH(32, 1); } \
        else { if ((P).U == 4) LAUNCH(64, 4); else if ((P).U == 2) LAUNCH(64, 2); else LAUNCH(64, 1); }                  \
    } while (0)

// a finishing kernel over all channels and shards: four waves per channel where a shard has many row blocks
#define EDL_FINALIZE(KERNEL, CUT, CH, ...)                                                                                     \
    do {                                                                                                                       \
        if ((CUT).most > 512) hipLaunchKernelGGL(KERNEL<4>, dim3(CH, (CUT).p), dim3(256), 0, st, partial, CUT, CH, __VA_ARGS__);     \
        else hipLaunchKernelGGL(KERNEL<1>, dim3(((CH) + 3) / 4, (CUT).p), dim3(256), 0, st, partial, CUT, CH, __VA_ARGS__);    \
    } while (0)

static inline dim3 ew_grid(const ShardSet& S, int hw, int cvecs, int u) {
    return dim3((unsigned)(((int64_t)S.largest() * hw * cvecs + 256 * u - 1) / (256 * u)), S.p);
}
// Vectors per lane: as many of 4, 2, 1 as leave three workgroups per CU.  ResNet-50's passes over 256 samples (tensors
// of 25 to 400 MB), us per step at 1 / 2 / 4: forward 2,936 / 2,496 / 2,463, backward 3,740 / 3,052 / 2,850 (4.7 -> 6.2
// TB/s); over 32 samples 548 / 524 / 532 and 600 / 576 / 572.
static int vectors_per_lane(const ShardSet& S, int hw, int cvecs) {
    if (256 % cvecs != 0) return 1;
    const int64_t groups = (int64_t)S.samples() * hw * cvecs / 256;
    return groups >= 4 * 768 ? 4 : groups >= 2 * 768 ? 2 : 1;
}

// Whether the row blocks of a pass are longer than those of its smallest shard alone.  A lane's rows grow with the shards of
// the pass (ResNet-50's stem, 8 shards of 32: 12 -> 98), and with them the rounding error of one float32 chain: those are
// summed in chains of 16 rows, the lanes' sums in float64 (16 layers' scale gradients against float64: alone 9.4e-8, in a
// pass in one chain 1.23e-7, in two levels 8.5e-8; no measurable time).  A shard alone keeps one chain.
static bool long_blocks(const ShardSet& S, int hw, int C, int VEC, const RedShape& pass) {
    return pass.rows_per_block > red_shape((int64_t)S.plan_smallest * hw, C, VEC).rows_per_block;
}
template <typename T, int VEC, int KIND>
static void launch_colreduce(const RedShape& s, bool two_levels, const T* x, const T* y, T* dy, const float* mean_rstd, const RowCut& cut,
                             int C, int relu, float* partial, hipStream_t st, GradDst dbias = GradDst{nullptr, 0}) {
    const dim3 grid(s.col_blocks, cut.blk0[cut.p]);
    if (two_levels) hipLaunchKernelGGL((colreduce_kernel<T, VEC, KIND, true>), grid, s.block, 0, st, x, y, dy, mean_rstd, cut, C, relu, partial, dbias);
    else hipLaunchKernelGGL((colreduce_kernel<T, VEC, KIND, false>), grid, s.block, 0, st, x, y, dy, mean_rstd, cut, C, relu, partial, dbias);
}

template <typename T, int VEC>
static void bn_forward_t(const void* x, const void* res, void* y, const float* gamma, const float* beta,
                         float* save, float* running, const ShardSet& S, int hw, int C, bool relu, unsigned char* sign, float* partial,
                         const RowCut& sums, hipStream_t st) {
    const int64_t M = (int64_t)S.samples() * hw;
    const RedShape s = red_shape((int64_t)S.plan * hw, C, VEC);
    const double tb = (double)sizeof(T) * (double)M * C;   // bytes of one [M][C] tensor
    RowCut cut = sums;
    if (cut.p == 0) {   // else the producer of x left the partial sums
        ProfScope ps(prof_shape_label("bn_stats", M, C), 0.0, tb, st);
        cut = cut_rows(S, hw, s.rows_per_block);
        launch_colreduce<T, VEC, 0>(s, long_blocks(S, hw, C, VEC, s), (const T*)x, (const T*)nullptr, (T*)nullptr, (const float*)nullptr, cut, C, 0, partial, st);
    }
    if constexpr (VEC > 1) {
        const SlicePlan p = plan_slices(S, hw, C, VEC, cut);
        if (p.slice > 0) {
            ProfScope ps(prof_shape_label("bn_finish_apply", M, C), 0.0, tb * ((res ? 3.0 : 2.0) + (sign ? 1.0 / 16 : 0.0)), st);
#define EDL_BN_FINISH(SLICE, U)                                                                                       \
    do {                                                                                                              \
        if (res) hipLaunchKernelGGL((bn_finish_apply_kernel<T, SLICE, U, true>), p.grid, dim3(256), 0, st, (const T*)x, (const T*)res, (T*)y, \
                                    gamma, beta, partial, cut, C, relu ? 1 : 0, save, running, sign);                 \
        else hipLaunchKernelGGL((bn_finish_apply_kernel<T, SLICE, U, false>), p.grid, dim3(256), 0, st, (const T*)x, (const T*)res, (T*)y, \
                                gamma, beta, partial, cut, C, relu ? 1 : 0, save, running, sign);                     \
    } while (0)
            EDL_BN_SLICES(p, EDL_BN_FINISH);
#undef EDL_BN_FINISH
            return;
        }
    }
    {
        ProfScope ps("bn_stats_finalize", 0.0, 8.0 * (double)cut.blk0[cut.p] * C, st);
        EDL_FINALIZE(bn_stats_finalize_kernel, cut, C, save, running);
    }
    ProfScope ps(prof_shape_label("bn_apply", M, C), 0.0, tb * ((res ? 3.0 : 2.0) + (sign ? 1.0 / 16 : 0.0)), st);
    const bool nt = tune().bn_nt != 0 && tb >= (double)tune().bn_nt_bytes;
    const int u = vectors_per_lane(S, hw, s.cvecs);
    const dim3 grid = ew_grid(S, hw, s.cvecs, u);
#define EDL_BN_APPLY(U, RES, NT)                                                                                       \
    hipLaunchKernelGGL((bn_apply_kernel<T, VEC, U, RES, NT>), grid, dim3(256), 0, st, (const T*)x, (const T*)res, (T*)y, gamma, beta, \
                       save, cut, C, s.cvecs, relu ? 1 : 0, sign)
#define EDL_BN_APPLY_U(U)                                                                                              \
    do {                                                                                                               \
        if (res) { if (nt) EDL_BN_APPLY(U, true, true); else EDL_BN_APPLY(U, true, false); }                           \
        else { if (nt) EDL_BN_APPLY(U, false, true); else EDL_BN_APPLY(U, false, false); }                             \
    } while (0)
    if (u == 4) EDL_BN_APPLY_U(4); else if (u == 2) EDL_BN_APPLY_U(2); else EDL_BN_APPLY_U(1);
#undef EDL_BN_APPLY_U
#undef EDL_BN_APPLY
}

void launch_bn_forward(int dtype, const void* x, const void* res, void* y, const float* gamma, const float* beta,
                       float* save, float* running, const ShardSet& S, int hw, int C, bool relu, unsigned char* sign, float* partial,
                       const RowCut& sums, hipStream_t st) {
    if (dtype == 1) {
        if (C % 8 == 0) bn_forward_t<bf16_t, 8>(x, res, y, gamma, beta, save, running, S, hw, C, relu, sign, partial, sums, st);
        else bn_forward_t<bf16_t, 1>(x, res, y, gamma, beta, save, running, S, hw, C, relu, sign, partial, sums, st);
    } else {
        if (C % 4 == 0) bn_forward_t<float, 4>(x, res, y, gamma, beta, save, running, S, hw, C, relu, sign, partial, sums, st);
        else bn_forward_t<float, 1>(x, res, y, gamma, beta, save, running, S, hw, C, relu, sign, partial, sums, st);
    }
}

// what the element-wise pass moves, of tensors of tb bytes
static double bn_backward_bytes(double tb, bool mask, bool dres, bool acc) { return tb * ((mask ? 3.0 : 2.0) + 1.0 + (dres ? (acc ? 2.0 : 1.0) : 0.0)); }

// The element-wise pass, its coefficients given.  mask: dy is yet to be multiplied by y > 0.
template <typename T, int VEC>
static void bn_backward_apply_t(const void* x, const void* y, const void* dy, void* dx, void* dres, bool acc, bool mask, const float* gamma,
                                const float* save, const float* coef, const RowCut& cut, const ShardSet& S, int hw, int C, hipStream_t st) {
    const int64_t M = (int64_t)S.samples() * hw;
    const double tb = (double)sizeof(T) * (double)M * C;
    const int cvecs = (C + VEC - 1) / VEC;
    const bool nt = tune().bn_nt != 0 && tb >= (double)tune().bn_nt_bytes;
    ProfScope ps(prof_shape_label("bn_bwd_apply", M, C), 0.0, bn_backward_bytes(tb, mask, dres != nullptr, acc), st);
    const int u = vectors_per_lane(S, hw, cvecs);
    const dim3 grid = ew_grid(S, hw, cvecs, u);
#define EDL_BN_BWD_APPLY(U, MASK, ACC)                                                                                    \
    do {                                                                                                                  \
        if (nt) hipLaunchKernelGGL((bn_bwd_apply_kernel<T, VEC, U, MASK, ACC, true>), grid, dim3(256), 0, st, (const T*)x, (const T*)y, (const T*)dy, \
                                   (T*)dx, (T*)dres, gamma, save, coef, cut, C, cvecs);                                \
        else hipLaunchKernelGGL((bn_bwd_apply_kernel<T, VEC, U, MASK, ACC, false>), grid, dim3(256), 0, st, (const T*)x, (const T*)y, (const T*)dy, \
                                (T*)dx, (T*)dres, gamma, save, coef, cut, C, cvecs);                                   \
    } while (0)
#define EDL_BN_BWD_APPLY_U(U)                                                                                             \
    do {                                                                                                                  \
        if (mask) { if (acc) EDL_BN_BWD_APPLY(U, true, true); else EDL_BN_BWD_APPLY(U, true, false); }                    \
        else { if (acc) EDL_BN_BWD_APPLY(U, false, true); else EDL_BN_BWD_APPLY(U, false, false); }                       \
    } while (0)
    if (u == 4) EDL_BN_BWD_APPLY_U(4); else if (u == 2) EDL_BN_BWD_APPLY_U(2); else EDL_BN_BWD_APPLY_U(1);
#undef EDL_BN_BWD_APPLY_U
#undef EDL_BN_BWD_APPLY
}

template <typename T, int VEC>
static void bn_backward_t(const void* x, const void* y, const void* dy, void* dx, void* dres, bool dres_acc,
                          const float* gamma, const float* save, GradDst dgamma, GradDst dbeta, const ShardSet& S, int hw, int C,
                          bool relu, float* partial, float* coef, const RowCut& sums, hipStream_t st) {
    const int64_t M = (int64_t)S.samples() * hw;
    const RedShape s = red_shape((int64_t)S.plan * hw, C, VEC);
    const double tb = (double)sizeof(T) * (double)M * C;
    const bool fused = sums.p > 0;
    RowCut cut = sums;
    if (!fused) {   // else the dgrad that produced dy left the sums
        ProfScope ps(prof_shape_label("bn_bwd_reduce", M, C), 0.0, tb * (relu ? 3.0 : 2.0), st);
        cut = cut_rows(S, hw, s.rows_per_block);
        launch_colreduce<T, VEC, 1>(s, long_blocks(S, hw, C, VEC, s), (const T*)x, (const T*)(relu ? y : x), (T*)dy, save, cut, C, relu ? 1 : 0, partial, st);
    }
    // the dgrad that left the sums also left dy masked: the activation is then not read again
    const bool mask = relu && !fused;
    const bool acc = dres && dres_acc;
    if constexpr (VEC > 1) {
        const SlicePlan p = dx == nullptr || acc ? SlicePlan() : plan_slices(S, hw, C, VEC, cut);
        if (p.slice > 0) {
            ProfScope ps(prof_shape_label("bn_finish_bwd", M, C), 0.0, bn_backward_bytes(tb, mask, dres != nullptr, acc), st);
#define EDL_BN_FINISH(SLICE, U)                                                                                       \
    do {                                                                                                              \
        if (mask) hipLaunchKernelGGL((bn_finish_bwd_kernel<T, SLICE, U, true>), p.grid, dim3(256), 0, st, (const T*)x, (const T*)y, (const T*)dy, \
                                     (T*)dx, (T*)dres, gamma, save, partial, cut, C, dgamma.g, dbeta.g, dgamma.stride);  \
        else hipLaunchKernelGGL((bn_finish_bwd_kernel<T, SLICE, U, false>), p.grid, dim3(256), 0, st, (const T*)x, (const T*)y, (const T*)dy, \
                                (T*)dx, (T*)dres, gamma, save, partial, cut, C, dgamma.g, dbeta.g, dgamma.stride);       \
    } while (0)
            EDL_BN_SLICES(p, EDL_BN_FINISH);
#undef EDL_BN_FINISH
            return;
        }
    }
    {
        ProfScope ps("bn_bwd_finalize", 0.0, 8.0 * (double)cut.blk0[cut.p] * C, st);
        EDL_FINALIZE(bn_bwd_finalize_kernel, cut, C, dgamma.g, dbeta.g, dgamma.stride, coef);
    }
    if (dx != nullptr) bn_backward_apply_t<T, VEC>(x, y, dy, dx, dres, acc, mask, gamma, save, coef, cut, S, hw, C, st);
}

void launch_bn_backward(int dtype, const void* x, const void* y, const void* dy, void* dx, void* dres,
                        bool dres_accumulate, const float* gamma, const float* save, GradDst dgamma, GradDst dbeta,
                        const ShardSet& S, int hw, int C, bool relu, float* partial, float* coef, const RowCut& sums,
                        hipStream_t st) {
    if (dtype == 1) {
        if (C % 8 == 0) bn_backward_t<bf16_t, 8>(x, y, dy, dx, dres, dres_accumulate, gamma, save, dgamma, dbeta, S, hw, C, relu, partial, coef, sums, st);
        else bn_backward_t<bf16_t, 1>(x, y, dy, dx, dres, dres_accumulate, gamma, save, dgamma, dbeta, S, hw, C, relu, partial, coef, sums, st);
    } else {
        if (C % 4 == 0) bn_backward_t<float, 4>(x, y, dy, dx, dres, dres_accumulate, gamma, save, dgamma, dbeta, S, hw, C, relu, partial, coef, sums, st);
        else bn_backward_t<float, 1>(x, y, dy, dx, dres, dres_accumulate, gamma, save, dgamma, dbeta, S, hw, C, relu, partial, coef, sums, st);
    }
}

void launch_bn_backward_apply(const void* x, const void* dy, void* dx, const float* gamma, const float* save, const float* coef,
                              const ShardSet& S, int hw, int C, hipStream_t st) {
    // (of the cut only which rows are whose is read)
    bn_backward_apply_t<bf16_t, 8>(x, nullptr, dy, dx, nullptr, false, false, gamma, save, coef, cut_rows(S, hw, hw), S, hw, C, st);
}

// store: the masked gradient is written back (dy <- dy')
template <typename T, int VEC>
static void bias_relu_backward_t(const void* y, void* dy, GradDst dbias, const ShardSet& S, int hw, int C, bool relu, bool store, float* partial,
                                 const RowCut& sums, hipStream_t st) {
    const int64_t M = (int64_t)S.samples() * hw;
    const RedShape s = red_shape((int64_t)S.plan * hw, C, VEC);
    const double tb = (double)sizeof(T) * (double)M * C;
    RowCut cut = sums;
    if (cut.p == 0) {   // else dy is masked already and its column sums are in partial
        ProfScope ps("bias_relu_bwd", 0.0, tb * (relu ? (store ? 3.0 : 2.0) : 1.0), st);
        cut = cut_rows(S, hw, s.rows_per_block);
        // Where a block is a whole shard (few rows: fully connected layers) its sums are the bias gradient: one launch less.
        cut.stored = dbias.g != nullptr && cut.block_per_shard();
        const GradDst direct = cut.stored ? dbias : GradDst{nullptr, 0};
        const bool two = long_blocks(S, hw, C, VEC, s);
        if (store) launch_colreduce<T, VEC, 2>(s, two, (const T*)nullptr, (const T*)(relu ? y : dy), (T*)dy, (const float*)nullptr, cut, C, relu ? 1 : 0, partial, st, direct);
        else launch_colreduce<T, VEC, 3>(s, two, (const T*)nullptr, (const T*)(relu ? y : dy), (T*)dy, (const float*)nullptr, cut, C, relu ? 1 : 0, partial, st, direct);
    }
    if (dbias.g && !cut.stored) {
        ProfScope ps("bias_finalize", 0.0, 4.0 * (double)cut.blk0[cut.p] * C, st);
        EDL_FINALIZE(bias_finalize_kernel, cut, C, dbias.g, dbias.stride);
    }
}

static void bias_relu_backward(int dtype, const void* y, void* dy, GradDst dbias, const ShardSet& S, int hw, int C, bool relu, bool store,
                               float* partial, const RowCut& sums, hipStream_t st) {
    if (dtype == 1) {
        if (C % 8 == 0) bias_relu_backward_t<bf16_t, 8>(y, dy, dbias, S, hw, C, relu, store, partial, sums, st);
        else bias_relu_backward_t<bf16_t, 1>(y, dy, dbias, S, hw, C, relu, store, partial, sums, st);
    } else {
        if (C % 4 == 0) bias_relu_backward_t<float, 4>(y, dy, dbias, S, hw, C, relu, store, partial, sums, st);
        else bias_relu_backward_t<float, 1>(y, dy, dbias, S, hw, C, relu, store, partial, sums, st);
    }
}

int bias_sums_rows(int dtype, const ShardSet& S, int hw, int C, int* side_by_side, bool* in_double) {
    if (C % (dtype == 1 ? 8 : 4) == 0) return 0;
    const RedShape s = red_shape((int64_t)S.plan * hw, C, 1);
    *side_by_side = s.TX;
    *in_double = long_blocks(S, hw, C, 1, s);
    return s.rows_per_block;
}

void launch_bias_relu_backward(int dtype, const void* y, void* dy, GradDst dbias, const ShardSet& S, int hw, int C, bool relu,
                               float* partial, const RowCut& sums, hipStream_t st) {
    if (!relu && !dbias.g) return;
    bias_relu_backward(dtype, y, dy, dbias, S, hw, C, relu, true, partial, sums, st);
}

void launch_pooled_bias_backward(int dtype, const void* pooled, const void* dpooled, GradDst dbias, const ShardSet& S, int hw, int C,
                                 float* partial, hipStream_t st) {
    if (dbias.g) bias_relu_backward(dtype, pooled, const_cast<void*>(dpooled), dbias, S, hw, C, true, false, partial, RowCut(), st);
}

__global__ __launch_bounds__(256) void signs_kernel(const bf16_t* __restrict__ act, unsigned char* __restrict__ sign, int64_t vecs) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= vecs) return;
    const Vec16<bf16_t> v = load_vec(act + i * 8);
    unsigned bits = 0;
    #pragma unroll
    for (int e = 0; e < 8; ++e) bits |= (bf16_to_f32(v.e[e]) > 0.f ? 1u : 0u) << e;
    sign[i] = (unsigned char)bits;
}

void launch_signs(const void* act_bf16, unsigned char* sign, int64_t n, hipStream_t st) {
    hipLaunchKernelGGL(signs_kernel, dim3((unsigned)((n / 8 + 255) / 256)), dim3(256), 0, st, (const bf16_t*)act_bf16, sign, n / 8);
}

}  // namespace edl
