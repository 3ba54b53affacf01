// Small fully connected layers.  First, those with few outputs whose number is no multiple of a vector (a classifier of 10
// classes): the three contractions of such a layer.  Where they are small (thin_fwd_takes and its like say how small) latency bounds them.  The
// tiled kernel took its element-wise path for them (one workgroup of 64x64 outputs, a wait after every load): MLP of 64 samples 12.1 / 10.8 /
// 5.7 us forward / input gradient / weight gradient, here 3.1 / 3.6 / 3.3; a chain of 20 launches of 3 to 8 us each.
//
//   forward           y[m][k]  = sum_c x[m][c] w[k][c] + b[k]       a wave per output, lanes along c
//   input gradient    dx[m][c] = sum_k dy[m][k] w[k][c]             a lane per column c and four rows
//   weight gradient   dw[k][c] = sum_m dy[m][k] x[m][c]             a lane per column c and every 16th row of the shard
//
// All sums in float32, in chains no longer than the tiled kernel's.
//
// Second (small_fc_kernel), forward and input gradient of float32 layers that give the chip less than a workgroup per CU: below.
#include <algorithm>

#include "dev_common.h"
#include "kernels.h"
#include "profiler.h"
#include "thin.h"

namespace edl {

constexpr int kThinOutputs = 128;      // as far as the rules below were measured
constexpr int kThinShard = 1024;       // rows of a shard: a chain of 64 in the weight gradient
constexpr int kThinRows = 16;          // rows of a workgroup of the input gradient

template <typename T, int VEC>
__global__ __launch_bounds__(256) void thin_fwd_kernel(const T* __restrict__ x, const T* __restrict__ w, const float* __restrict__ bias,
                                                       void* __restrict__ y, int M, int K, int C, int relu, int out_fp32) {
    const int lane = threadIdx.x & 63, o = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (o >= M * K) return;
    const int m = o / K, k = o - m * K;
    const T* const xr = x + (size_t)m * C;
    const T* const wr = w + (size_t)k * C;
    float s = 0.f;
    for (int c = lane * VEC; c < C; c += 64 * VEC) {
        if (VEC > 1) {
            const Vec16<T> a = load_vec(xr + c), b = load_vec(wr + c);
            #pragma unroll
            for (int e = 0; e < VEC; ++e) s += Elem<T>::to_f32(a.e[e]) * Elem<T>::to_f32(b.e[e]);
        } else {
            s += Elem<T>::to_f32(xr[c]) * Elem<T>::to_f32(wr[c]);
        }
    }
    for (int d = 32; d > 0; d >>= 1) s += __shfl_xor(s, d, 64);
    if (lane != 0) return;
    if (bias != nullptr) s += bias[k];
    if (relu) s = fmaxf(s, 0.f);
    if (out_fp32) ((float*)y)[o] = s;
    else ((T*)y)[o] = Elem<T>::from_f32(s);
}

// An element through a buffer descriptor: what lies past its end is read as zero.
constexpr unsigned kPastEnd = 0x80000000u;      // (the rules below keep the gradients under that many bytes)
template <typename T> __device__ __forceinline__ float load_or_zero(__amdgpu_buffer_rsrc_t r, unsigned at);
template <> __device__ __forceinline__ float load_or_zero<float>(__amdgpu_buffer_rsrc_t r, unsigned at) {
    return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, at, 0, 0));
}
template <> __device__ __forceinline__ float load_or_zero<bf16_t>(__amdgpu_buffer_rsrc_t r, unsigned at) {
    return bf16_to_f32(__builtin_amdgcn_raw_buffer_load_b16(r, at, 0, 0));
}

// grid: (64 columns, blocks of rows within a shard).  Masked and summed as a bias layer with ReLU wants it (DgradMask with no
// xin); with one block per shard the sums are that layer's bias gradients.
template <typename T>
__global__ __launch_bounds__(256) void thin_dgrad_kernel(const T* __restrict__ dy, const T* __restrict__ w, const T* old, T* dx,
                                                         const T* __restrict__ mask_act, float* __restrict__ sums, GradDst dbias,
                                                         RowCut cut, int K, int C) {
    __shared__ float red[4][64];
    int r0, r1;
    const int shard = locate_block(cut, blockIdx.y, r0, r1);
    const int lane = threadIdx.x & 63, sub = threadIdx.x >> 6;
    const int c = blockIdx.x * 64 + lane;
    const bool active = c < C;
    constexpr int R = kThinRows / 4, KC = 16;
    const __amdgpu_buffer_rsrc_t rdy =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(dy), 0, (unsigned)cut.row0[cut.p] * (unsigned)K * (unsigned)sizeof(T), 0x00020000);
    float acc[R];
    #pragma unroll
    for (int i = 0; i < R; ++i) acc[i] = 0.f;
    for (int k0 = 0; k0 < K; k0 += KC) {
        float wk[KC];
        #pragma unroll
        for (int e = 0; e < KC; ++e) wk[e] = active && k0 + e < K ? Elem<T>::to_f32(w[(size_t)(k0 + e) * C + c]) : 0.f;
        #pragma unroll
        for (int i = 0; i < R; ++i) {
            // (a row past the end is computed and not used)
            const unsigned row = (unsigned)min(r0 + sub + 4 * i, r1 - 1) * (unsigned)K * (unsigned)sizeof(T);
            #pragma unroll
            for (int e = 0; e < KC; ++e) {
                // an output past the last one is read as zero, and not as the last times a zero weight: that may be infinite
                const unsigned col = (unsigned)(k0 + e) * (unsigned)sizeof(T) + (k0 + e < K ? 0u : kPastEnd);
                acc[i] += load_or_zero<T>(rdy, row + col) * wk[e];
            }
        }
    }
    float s = 0.f;
    #pragma unroll
    for (int i = 0; i < R; ++i) {
        const int r = r0 + sub + 4 * i;
        if (r >= r1 || !active) continue;
        const size_t at = (size_t)r * C + c;
        float v = acc[i];
        if (old != nullptr) v += Elem<T>::to_f32(old[at]);
        if (mask_act != nullptr && !(Elem<T>::to_f32(mask_act[at]) > 0.f)) v = 0.f;
        const T o = Elem<T>::from_f32(v);
        dx[at] = o;
        s += Elem<T>::to_f32(o);
    }
    if (sums == nullptr) return;
    red[sub][lane] = s;
    __syncthreads();
    if (sub != 0 || !active) return;
    s = (red[0][lane] + red[1][lane]) + (red[2][lane] + red[3][lane]);
    if (dbias.g != nullptr) dbias.g[(int64_t)cut.k[shard] * dbias.stride + c] = s;
    else {
        sums[(size_t)c * gridDim.y + blockIdx.y] = s;
        sums[(size_t)(C + c) * gridDim.y + blockIdx.y] = 0.f;
    }
}

// grid: (64 columns, outputs / 8, shards); a wave takes every 16th row of the shard (with every fourth, a shard of 512 rows
// was 128 dependent trips, 20 us)
template <typename T>
__global__ __launch_bounds__(1024) void thin_wgrad_kernel(const T* __restrict__ dy, const T* __restrict__ x, GradDst dw, ShardSet S, int K, int C) {
    constexpr int KC = 8, NW = 16;
    __shared__ float red[NW][KC][64];
    const int lane = threadIdx.x & 63, sub = threadIdx.x >> 6;
    const int c = blockIdx.x * 64 + lane, k0 = blockIdx.y * KC, sh = blockIdx.z;
    const int r0 = S.off[sh], r1 = S.off[sh + 1];
    const bool active = c < C;
    float acc[KC];
    #pragma unroll
    for (int e = 0; e < KC; ++e) acc[e] = 0.f;
    #pragma unroll 4
    for (int r = r0 + sub; r < r1; r += NW) {
        const float xv = active ? Elem<T>::to_f32(x[(size_t)r * C + c]) : 0.f;
        #pragma unroll
        for (int e = 0; e < KC; ++e) acc[e] += Elem<T>::to_f32(dy[(size_t)r * K + min(k0 + e, K - 1)]) * xv;
    }
    #pragma unroll
    for (int e = 0; e < KC; ++e) red[sub][e][lane] = acc[e];
    __syncthreads();
    if (sub >= KC || !active || k0 + sub >= K) return;
    float s = 0.f;
    #pragma unroll
    for (int q = 0; q < NW; ++q) s += red[q][sub][lane];
    dw.g[(int64_t)S.k[sh] * dw.stride + (size_t)(k0 + sub) * C + c] = s;
}

static bool thin_shape(int dtype, const ConvGeom& g) {
    return g.H == 1 && g.W == 1 && g.R == 1 && g.S == 1 && g.stride == 1 && g.pad == 0 && g.K % (dtype == 1 ? 8 : 4) != 0 && g.K <= kThinOutputs;
}

// Float32 rows that are no whole vectors: the tiled kernel reads everything element by element then, and takes up to three times as
// long (bf16 as well, but so does the thin one there).
static bool odd_rows(int dtype, const ConvGeom& g) { return dtype != 1 && g.C % 4 != 0; }

// The rules, from launches of 64 to 32,768 rows (M), 63 to 4,096 columns (C) and 10 to 127 outputs (K).  Times are us between events
// around a launch, 5 to 6 of them the events', float32 / bf16 where both are given.
//
// Forward: a wave per output costs 0.14 ns + 0.05 per further 64 vectors of the row, whatever the tiled kernel reuses; that one's time is
// its reduction's, in few workgroups.  Thin against tiled, M x K:
//    65,024 C =   512   15.1 against 15.9 (bf16)                33,280 C = 64      9.7 / 10.1 against 6.5 / 10.9
//   135,168 C =   512   32.4 / 27.6 against 11.6 / 17.7      4,161,536 C = 64      578 / 627 against 16.3 / 15.1
//    65,024 C = 4,096   66.5 / 39.8 against 114 / 114          520,192 C = 4,096   466 / 269 against 116 / 111
//   odd rows: 65,024 C = 511 29.4 / 28.9 against 53.6 / 44.5, 135,168 C = 2,047 180 / 180 against 190 / 141
// and against small_fc_kernel (float32): 5,120 C = 64 6.3 against 6.2, 8,128 C = 512 6.2 against 8.7, 16,896 C = 64 7.8 against 6.2,
// 33,280 C = 512 11.7 against 9.4, 520,192 C = 512 106 against 22.9.
bool thin_fwd_takes(int dtype, const ConvGeom& g, int samples, bool small) {
    const int64_t most = small ? 12288 : 32768 + (odd_rows(dtype, g) ? 110 : 64) * std::min(g.C, 1024);
    return thin_shape(dtype, g) && (int64_t)samples * g.K <= most;
}

// Input gradient: thin against tiled and the launches that come with it (the ReLU's mask and sums, the transposed weights), M x K x C:
//   8.5e6 to 1.7e7   11 to 15 against 34 to 38         1.3e8 to 1.4e8 (K = 65, 127)   29 to 38 against 36 to 49
//   2.7e8 (K = 127)  47 / 57 against 43 to 50          5.5e8 (K = 33)   139 / 181 against 131 / 137    2.1e9 (K = 127)   313 / 425 against 194 / 181
//   odd rows: 2.7e8 (K = 127) 50 against 48 to 53, 2.8e8 (K = 33) 76 against 88 to 90, 1.1e9 167 against 123
// Up to 16 outputs it is one pass over what it reads and writes, at any size: 32,768 x 10 x 512 55 / 66 against 69 / 113.
// (Blocks of 16 rows stay below 65,536.)
bool thin_dgrad_takes(int dtype, const ConvGeom& g) {
    return thin_shape(dtype, g) && (g.K <= 16 ? g.N <= 1000000 : (int64_t)g.N * g.K * g.C <= (odd_rows(dtype, g) ? 400000000 : 200000000));
}

// Weight gradient: thin against tiled and the sum of its pieces, M x K x C:
//   4.2e6 to 1.7e7   13 to 20 against 17 to 25         6.9e7   21 / 23 to 24 against 24 to 25 / 21 to 23
//   1.4e8            30 / 32 against 27 / 22           5.5e8   86 / 97 against 36 / 27
//   odd rows: 1.3e8 24 against 33, 2.8e8 49 against 41
bool thin_wgrad_takes(int dtype, const ConvGeom& g, const ShardSet& S) {
    const int64_t most = odd_rows(dtype, g) ? 200000000 : dtype == 1 ? 70000000 : 100000000;
    return thin_shape(dtype, g) && S.plan_largest <= kThinShard && (int64_t)S.plan * g.K * g.C <= most;
}

template <typename T>
static void fwd(const ConvGeom& g, const void* x, const void* w, const float* bias, bool relu, bool out_fp32, void* y, hipStream_t st) {
    const dim3 grid((g.N * g.K + 3) / 4);
    if (g.C % Elem<T>::VEC == 0 && (((uintptr_t)x | (uintptr_t)w) & 15) == 0)     // (parameters lie at any element)
        hipLaunchKernelGGL((thin_fwd_kernel<T, Elem<T>::VEC>), grid, dim3(256), 0, st, (const T*)x, (const T*)w, bias, y, g.N, g.K, g.C, relu, out_fp32);
    else
        hipLaunchKernelGGL((thin_fwd_kernel<T, 1>), grid, dim3(256), 0, st, (const T*)x, (const T*)w, bias, y, g.N, g.K, g.C, relu, out_fp32);
}

void launch_thin_fwd(int dtype, const ConvGeom& g, const void* x, const void* w, const float* bias, bool relu, bool out_fp32, void* y, hipStream_t st) {
    ProfScope ps(prof_shape_label("thin_fwd", g.N, g.C), 2.0 * g.N * g.K * g.C, (dtype == 1 ? 2.0 : 4.0) * ((double)(g.N + g.K) * g.C + (double)g.N * g.K), st);
    if (dtype == 1) fwd<bf16_t>(g, x, w, bias, relu, out_fp32, y, st);
    else fwd<float>(g, x, w, bias, relu, out_fp32, y, st);
}

RowCut launch_thin_dgrad(int dtype, const ConvGeom& g, const ShardSet& S, const void* dy, const void* w, const void* old, void* dx,
                         const DgradMask* mask, hipStream_t st) {
    RowCut cut = cut_rows(S, 1, kThinRows);
    const int blocks = cut.blk0[cut.p];
    const bool fuse = mask != nullptr && mask->act != nullptr && mask->xin == nullptr && mask->sums.buf != nullptr &&
                      mask->sums.floats >= (size_t)2 * g.C * blocks;
    cut.stored = fuse && mask->dbias.g != nullptr && cut.block_per_shard();
    const void* const act = fuse ? mask->act : nullptr;
    float* const sums = fuse ? mask->sums.buf : nullptr;
    const GradDst dbias = cut.stored ? mask->dbias : GradDst{nullptr, 0};
    ProfScope ps(prof_shape_label("thin_dgrad", g.N, g.C), 2.0 * g.N * g.K * g.C, (dtype == 1 ? 2.0 : 4.0) * ((double)(g.N + g.K) * g.C + (double)g.N * g.K), st);
    const dim3 grid((g.C + 63) / 64, blocks);
    if (dtype == 1)
        hipLaunchKernelGGL(thin_dgrad_kernel<bf16_t>, grid, dim3(256), 0, st, (const bf16_t*)dy, (const bf16_t*)w, (const bf16_t*)old, (bf16_t*)dx,
                           (const bf16_t*)act, sums, dbias, cut, g.K, g.C);
    else
        hipLaunchKernelGGL(thin_dgrad_kernel<float>, grid, dim3(256), 0, st, (const float*)dy, (const float*)w, (const float*)old, (float*)dx,
                           (const float*)act, sums, dbias, cut, g.K, g.C);
    return fuse ? cut : RowCut();
}

void launch_thin_wgrad(int dtype, const ConvGeom& g, const ShardSet& S, const void* x, const void* dy, GradDst dw, hipStream_t st) {
    ProfScope ps(prof_shape_label("thin_wgrad", g.N, g.C), 2.0 * g.N * g.K * g.C, (dtype == 1 ? 2.0 : 4.0) * ((double)g.N * (g.C + g.K)) + 4.0 * S.p * g.K * g.C, st);
    const dim3 grid((g.C + 63) / 64, (g.K + 7) / 8, S.p);
    if (dtype == 1) hipLaunchKernelGGL(thin_wgrad_kernel<bf16_t>, grid, dim3(1024), 0, st, (const bf16_t*)dy, (const bf16_t*)x, dw, S, g.K, g.C);
    else hipLaunchKernelGGL(thin_wgrad_kernel<float>, grid, dim3(1024), 0, st, (const float*)dy, (const float*)x, dw, S, g.K, g.C);
}

// ---------------------------------------------------------------------------------------------------------------------
// Float32 layers of few tiles (an MLP of 64 samples and 256 wide): latency again.  The tiled kernel cut their reduction over
// workgroups to fill some of the chip, with a launch more to add the pieces (784 -> 256: 7.4 + 4.2 us).  Here a workgroup owns
// 32x32 outputs, its sixteen waves a piece of the reduction each (with two sets of sums), which meet in LDS: no pieces
// in memory, no second launch; operands go from global memory into registers, and the input gradient reads the weights as they
// lie, so that these layers need no transposed copy either (3.8 us of the chain).  784 -> 256, 64 rows: 7 us in one launch.
// ---------------------------------------------------------------------------------------------------------------------
typedef float floatx16 __attribute__((ext_vector_type(16)));
constexpr int kSmallTiles = 256, kSmallReduction = 2048, kSmallWaves = 16;     // (chains of 64 products at most)

struct SmallArgs {
    const float *A, *B;          // [M][K]; forward [N][K], input gradient [K][N]
    float* out;                  // [M][N]
    const float *bias, *old, *act;
    float* sums;                 // input gradient, with act: column sums per block (see launch_thin_dgrad)
    GradDst dbias;
    int K, N, relu;
    RowCut cut;
};

template <bool DGRAD>
__global__ __launch_bounds__(64 * kSmallWaves) void small_fc_kernel(SmallArgs a) {
    __shared__ float red[kSmallWaves][32][33];
    int r0, r1;
    const int shard = locate_block(a.cut, blockIdx.y, r0, r1);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, half = lane >> 5;
    const int row = min(r0 + (lane & 31), r1 - 1), col = blockIdx.x * 32 + (lane & 31), colc = min(col, a.N - 1);
    const float* const Ar = a.A + (size_t)row * a.K;
    const float* const Br = DGRAD ? a.B + colc : a.B + (size_t)colc * a.K;
    floatx16 acc[2];
    #pragma unroll
    for (int q = 0; q < 16; ++q) acc[0][q] = acc[1][q] = 0.f;
    const int steps = (a.K + 7) / 8;
    // (reads past the end of the reduction take its last vector and count as zeros; rows and columns past theirs are not stored)
    auto step = [&](int s, floatx16& c) {
        const int k = s * 8 + half * 4, kc = min(k, a.K - 4);
        float4 x = *reinterpret_cast<const float4*>(Ar + kc), w;
        if (DGRAD) w = make_float4(Br[(size_t)kc * a.N], Br[(size_t)(kc + 1) * a.N], Br[(size_t)(kc + 2) * a.N], Br[(size_t)(kc + 3) * a.N]);
        else w = *reinterpret_cast<const float4*>(Br + kc);
        if (k >= a.K) { x = make_float4(0.f, 0.f, 0.f, 0.f); w = x; }
        c = __builtin_amdgcn_mfma_f32_32x32x2f32(x.x, w.x, c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_32x32x2f32(x.y, w.y, c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_32x32x2f32(x.z, w.z, c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_32x32x2f32(x.w, w.w, c, 0, 0, 0);
    };
    // neighbouring steps share their cache lines; with four waves (and 32 KB in flight per workgroup) 784 -> 256 took 14 us
    const int piece = (steps + kSmallWaves - 1) / kSmallWaves, end = min((wave + 1) * piece, steps);
    #pragma unroll 4
    for (int s = wave * piece; s < end; s += 2) {
        step(s, acc[0]);
        step(s + 1 < end ? s + 1 : steps, acc[1]);      // (step `steps` is all zeros)
    }
    #pragma unroll
    for (int q = 0; q < 16; ++q) red[wave][(q >> 2) * 8 + half * 4 + (q & 3)][lane & 31] = acc[0][q] + acc[1][q];
    __syncthreads();
    const int rl = threadIdx.x >> 5, cl = threadIdx.x & 31, r = r0 + rl, c = blockIdx.x * 32 + cl;
    const bool live = r < r1 && c < a.N;
    float v = 0.f;
    #pragma unroll
    for (int w = 0; w < kSmallWaves; w += 4) v += (red[w][rl][cl] + red[w + 1][rl][cl]) + (red[w + 2][rl][cl] + red[w + 3][rl][cl]);
    if (live) {
        const size_t at = (size_t)r * a.N + c;
        if (!DGRAD && a.bias != nullptr) v += a.bias[c];
        if (!DGRAD && a.relu) v = fmaxf(v, 0.f);
        if (DGRAD && a.old != nullptr) v += a.old[at];
        if (DGRAD && a.act != nullptr && !(a.act[at] > 0.f)) v = 0.f;
        a.out[at] = v;
    }
    if (!DGRAD || a.sums == nullptr) return;
    __syncthreads();
    red[0][rl][cl] = live ? v : 0.f;
    __syncthreads();
    if (threadIdx.x >= 32 || blockIdx.x * 32 + (int)threadIdx.x >= a.N) return;
    float p[4] = {0.f, 0.f, 0.f, 0.f};
    #pragma unroll
    for (int i = 0; i < 32; ++i) p[i & 3] += red[0][i][threadIdx.x];
    const float t = (p[0] + p[1]) + (p[2] + p[3]);
    const int cg = blockIdx.x * 32 + threadIdx.x;
    if (a.dbias.g != nullptr) a.dbias.g[(int64_t)a.cut.k[shard] * a.dbias.stride + cg] = t;
    else {
        a.sums[(size_t)cg * gridDim.y + blockIdx.y] = t;
        a.sums[(size_t)(a.N + cg) * gridDim.y + blockIdx.y] = 0.f;
    }
}

// Up to 256 tiles (one per CU) and a reduction of 2,048 (the longest that keeps the chains at 64).  Steps of a job of two such layers of
// equal width, this kernel / tiled, us:
//   width 256, 16 tiles 68 / 90, 256 tiles 105 / 127          1,024, 64 tiles 97 / 106, 256 tiles 120 / 139
//   2,048, 64 tiles 142 / 144, 128 tiles 153 / 153, 256 tiles 173 / 190
// Past the line the short reductions still gain and the long ones lose: 512 tiles 124 / 144, 156 / 171, 239 / 241, and 524 / 487 at 4,096.
bool small_fc_takes(int dtype, const ConvGeom& g, int K, int N, int samples) {
    return dtype != 1 && g.H == 1 && g.W == 1 && g.R == 1 && g.S == 1 && g.stride == 1 && g.pad == 0 && K % 4 == 0 &&
           K <= kSmallReduction && (int64_t)((samples + 31) / 32) * ((N + 31) / 32) <= kSmallTiles;
}

void launch_small_fc_fwd(const ConvGeom& g, const float* x, const float* w, const float* bias, bool relu, float* y, hipStream_t st) {
    ShardSet all = {};
    all.p = 1;
    all.off[1] = g.N;
    all.plan_itself();
    SmallArgs a = {};
    a.A = x; a.B = w; a.out = y; a.bias = bias; a.relu = relu;
    a.K = g.C; a.N = g.K;
    a.cut = cut_rows(all, 1, 32);
    ProfScope ps(prof_shape_label("small_fc_fwd", g.N, g.K), 2.0 * g.N * g.K * g.C, 4.0 * ((double)g.N * (g.C + g.K) + (double)g.K * g.C), st);
    hipLaunchKernelGGL(small_fc_kernel<false>, dim3((a.N + 31) / 32, a.cut.blk0[a.cut.p]), dim3(64 * kSmallWaves), 0, st, a);
}

RowCut launch_small_fc_dgrad(const ConvGeom& g, const ShardSet& S, const float* dy, const float* w, const float* old, float* dx,
                             const DgradMask* mask, hipStream_t st) {
    SmallArgs a = {};
    a.A = dy; a.B = w; a.out = dx; a.old = old;
    a.K = g.K; a.N = g.C;
    a.cut = cut_rows(S, 1, 32);
    const int blocks = a.cut.blk0[a.cut.p];
    const bool fuse = mask != nullptr && mask->act != nullptr && mask->xin == nullptr && mask->sums.buf != nullptr &&
                      mask->sums.floats >= (size_t)2 * g.C * blocks;
    a.cut.stored = fuse && mask->dbias.g != nullptr && a.cut.block_per_shard();
    if (fuse) {
        a.act = (const float*)mask->act;
        a.sums = mask->sums.buf;
        if (a.cut.stored) a.dbias = mask->dbias;
    }
    ProfScope ps(prof_shape_label("small_fc_dgrad", g.N, g.C), 2.0 * g.N * g.K * g.C, 4.0 * ((double)g.N * (g.C + g.K) + (double)g.K * g.C), st);
    hipLaunchKernelGGL(small_fc_kernel<true>, dim3((a.N + 31) / 32, blocks), dim3(64 * kSmallWaves), 0, st, a);
    return fuse ? a.cut : RowCut();
}

}  // namespace edl
