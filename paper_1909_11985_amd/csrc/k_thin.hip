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
#include <type_traits>

#include "dev_common.h"
#include "kernels.h"
#include "profiler.h"
#include "thin.h"
#include "tune.h"

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

// ---------------------------------------------------------------------------------------------------------------------
// A classifier of few ragged outputs with the loss and everything that its backward pass needs, in one launch: what
// thin_fwd_kernel, softmax_ce_small_kernel, thin_dgrad_kernel, thin_wgrad_kernel and the column sums of the logits' gradient leave,
// bit for bit (each sum is formed in the order of those kernels).  Such a chain of five launches is five times the
// latency of one: MLP, four shards of 16, 16.4 us, here 10.4.  A workgroup has 64 columns of one shard and computes the shard's logits for
// itself; the first of a shard stores what belongs to the rows alone.
// ---------------------------------------------------------------------------------------------------------------------
// (fewer than 16: outputs are ragged)
constexpr int kHeadOutputs = 16, kHeadRows = 64, kHeadColumns = 1024;

struct HeadArgs {
    const void *x, *w;               // [M][C], [K][C] in the job's type; x is the output of a ReLU
    const float* bias;
    const int32_t* labels;
    float *logits, *row_loss, *loss;
    void *dlogits, *dx;              // dx: masked by x > 0
    GradDst dw, db, dbias;           // of this layer, and the bias of the layer before
    int K, C, tx, in_double;         // tx: channels side by side in the column sums of dlogits
    ShardSet S;
};

// a step of a butterfly over 2 * HALF sums: a lane keeps the lower or upper half of them
template <int HALF, int D>
__device__ __forceinline__ void give_half(float (&s)[kHeadOutputs], int lane) {
    const bool upper = (lane & D) != 0;
    #pragma unroll
    for (int k = 0; k < HALF; ++k) {
        const float give = upper ? s[k] : s[k + HALF], keep = upper ? s[k + HALF] : s[k];
        s[k] = keep + __shfl_xor(give, D, 64);
    }
}

// Every workgroup runs this code once, and its length is time: instructions that are not there yet come from memory.  Unrolled to 11
// and 18 KB it took 13.5 and 16.2 us, hence the loops that stay loops.
template <typename T>
__global__ __launch_bounds__(1024) void thin_head_kernel(HeadArgs a) {
    constexpr int NW = 16, VEC = Elem<T>::VEC;
    __shared__ __attribute__((aligned(16))) float z[kHeadRows][kHeadOutputs];     // logits, then their gradient (as stored)
    __shared__ float loss[kHeadRows];
    __shared__ float dxs[kHeadRows][64];                                          // the input gradient (as stored)
    __shared__ float red[NW][kHeadOutputs][64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, sh = blockIdx.y;
    const int lo = a.S.off[sh], n = a.S.off[sh + 1] - lo, K = a.K, C = a.C;
    const bool first = blockIdx.x == 0;
    const T* const x = (const T*)a.x + (size_t)lo * C;
    const T* const w = (const T*)a.w;
    const int c = blockIdx.x * 64 + lane, cc = min(c, C - 1);
    // what the later parts read is under way before the logits are there
    int label = a.labels[lo + min(wave, n - 1)];
    T xv = x[(size_t)min(wave, n - 1) * C + cc], wk[kHeadOutputs];
    // logits (thin_fwd_kernel): a wave per row, all its outputs at a time
    #pragma unroll 1
    for (int m = wave; m < n; m += NW) {
        const T* const xr = x + (size_t)m * C;
        float s[kHeadOutputs];
        #pragma unroll
        for (int k = 0; k < kHeadOutputs; ++k) s[k] = 0.f;
        #pragma unroll 1
        for (int i = lane * VEC; i < C; i += 64 * VEC) {
            const T* wr = w + i;
            const Vec16<T> u = load_vec(xr + i);
            Vec16<T> v[kHeadOutputs];
            #pragma unroll
            for (int k = 0; k < kHeadOutputs; ++k) {
                v[k] = load_vec(wr);
                wr += k + 1 < K ? C : 0;
            }
            #pragma unroll
            for (int k = 0; k < kHeadOutputs; ++k)
                #pragma unroll
                for (int e = 0; e < VEC; ++e) s[k] += Elem<T>::to_f32(u.e[e]) * Elem<T>::to_f32(v[k].e[e]);
        }
        // the butterfly over the lanes for all outputs: half of them are given away at each of the first four steps, so that a lane
        // ends with output lane / 4
        give_half<8, 32>(s, lane);
        give_half<4, 16>(s, lane);
        give_half<2, 8>(s, lane);
        give_half<1, 4>(s, lane);
        float mine = s[0];
        mine += __shfl_xor(mine, 2, 64);
        mine += __shfl_xor(mine, 1, 64);
        const int k = lane >> 2;
        if ((lane & 3) == 0 && k < K) {
            if (a.bias != nullptr) mine += a.bias[k];
            z[m][k] = mine;
            if (first) a.logits[(size_t)(lo + m) * K + k] = mine;
        }
    }
    {
        const T* wr = w + cc;
        #pragma unroll
        for (int e = 0; e < kHeadOutputs; ++e) {
            wk[e] = *wr;
            wr += e + 1 < K ? C : 0;
        }
    }
    // loss and the gradient of the logits (softmax_ce_small_kernel); a row's logits are this wave's own, from other lanes
    wave_lds_handover();
    const float invn = 1.f / (float)n;
    #pragma unroll 1
    for (int r = wave; r < n; r += NW) {
        if (r != wave) label = a.labels[lo + r];
        const bool live = lane < K;
        const float v = live ? z[r][lane] : -INFINITY;
        float mx = v;
        #pragma unroll 1
        for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o, 64));
        const float e = live ? expf(v - mx) : 0.f;
        float s = e;
        #pragma unroll 1
        for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
        const float inv = 1.f / s;
        const T d = Elem<T>::from_f32((e * inv - (lane == label ? 1.f : 0.f)) * invn);
        const float zl = __shfl(v, label, 64);
        if (lane < kHeadOutputs) z[r][lane] = live ? Elem<T>::to_f32(d) : 0.f;
        if (first && live) ((T*)a.dlogits)[(size_t)(lo + r) * K + lane] = d;
        if (lane == 0) {
            const float l = logf(s) - (zl - mx);
            loss[r] = l;
            if (first) a.row_loss[lo + r] = l;
        }
    }
    // input gradient (thin_dgrad_kernel) and a wave's part of the weight gradient (thin_wgrad_kernel: every 16th row); all lanes
    // read the row's gradients
    wave_lds_handover();
    float acc[kHeadOutputs];
    #pragma unroll
    for (int e = 0; e < kHeadOutputs; ++e) acc[e] = 0.f;
    #pragma unroll 1
    for (int r = wave; r < kHeadRows; r += NW) {
        float o = 0.f;
        if (r < n) {
            const size_t at = (size_t)r * C + cc;
            if (r != wave) xv = x[at];
            const float xf = Elem<T>::to_f32(xv);
            float v = 0.f;
            #pragma unroll
            for (int e = 0; e < kHeadOutputs; ++e) {
                const float d = z[r][e];
                v += d * (e < K ? Elem<T>::to_f32(wk[e]) : 0.f);
                acc[e] += d * xf;
            }
            if (!(xf > 0.f)) v = 0.f;
            const T t = Elem<T>::from_f32(v);
            if (c < C) ((T*)a.dx)[(size_t)lo * C + at] = t;
            o = Elem<T>::to_f32(t);
        }
        dxs[r][lane] = o;
    }
    #pragma unroll
    for (int e = 0; e < kHeadOutputs; ++e) red[wave][e][lane] = acc[e];
    __syncthreads();
    if (wave < K) {
        float s = 0.f;
        #pragma unroll
        for (int q = 0; q < NW; ++q) s += red[q][wave][lane];
        if (c < C) a.dw.g[(int64_t)a.S.k[sh] * a.dw.stride + (size_t)wave * C + c] = s;
    }
    // the waves that are left: K is less than 16
    if (wave != NW - 1) return;
    // bias gradient of the layer before: sums of 16 rows as thin_dgrad_kernel leaves them; several are added up as bias_finalize_kernel does
    double even = 0, odd = 0;
    float only = 0.f;
    #pragma unroll 1
    for (int b = 0; b < kHeadRows / 16; ++b) {
        float s[4] = {0.f, 0.f, 0.f, 0.f};
        #pragma unroll
        for (int i = 0; i < 16; ++i) s[i & 3] += dxs[b * 16 + i][lane];
        const float t = (s[0] + s[1]) + (s[2] + s[3]);
        if (b == 0) only = t;
        if (b & 1) odd += (double)t;
        else even += (double)t;
    }
    if (c < C) a.dbias.g[(int64_t)a.S.k[sh] * a.dbias.stride + c] = n <= 16 ? only : (float)(even + odd);
    if (!first) return;
    {
        float s = lane < n ? loss[lane] : 0.f;
        #pragma unroll 1
        for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
        if (lane == 0) a.loss[a.S.k[sh]] = s / (float)n;
    }
    // bias gradient (colreduce_kernel: a block per shard, lanes side by side in a.tx channels, 256 / a.tx rows at a time)
    if (lane < K) {
        const int ty = 256 / a.tx;
        double sd = 0;
        float sf = 0.f;
        #pragma unroll 1
        for (int j = 0; j < ty && j < n; ++j) {
            float t = 0.f;
            #pragma unroll 1
            for (int r = j; r < n; r += ty) t += z[r][lane];
            sd += (double)t;
            sf += t;
        }
        a.db.g[(int64_t)a.S.k[sh] * a.db.stride + lane] = a.in_double ? (float)sd : sf;
    }
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
typedef float floatx4 __attribute__((ext_vector_type(4)));
constexpr int kSmallTiles = 256, kSmallReduction = 2048, kSmallWaves = 16;     // (chains of 64 products at most)
// Weight gradient: rows of a shard, 16x16 tiles in all.  us per step with it for shards of up to 64 / 32 / 16 rows: 64 x 256 x 256 50 / 54 / 54,
// 4 x 64 of 512 79 / 83 / 83, 4 x 64 of 256 62 / 68 / 68, 8 x 32 of 256 53 / 53 / 58, 4 x 64 of 1,024 (tiled in any case) 121.
constexpr int kSmallShard = 64, kSmallWgradTiles = 4096;

struct SmallArgs {
    const float *A, *B;          // [M][K]; forward [N][K], input gradient [K][N]
    float* out;                  // [M][N]
    const float *bias, *old, *act;
    float* sums;                 // input gradient, with act: column sums per block (see launch_thin_dgrad)
    GradDst dbias;
    int K, N, relu;
    RowCut cut;
};

// The first layer of a net may take its rows from the data set itself: they are read there, and stored with their labels for the
// backward pass by the workgroups of the first columns.  The samples' numbers travel in the launch's arguments.
struct SmallGather {
    const float* data;
    const int32_t* data_y;
    float* out;
    int32_t* labels;
    int32_t idx[kSmallGather];
};

// One MFMA of TS x TS outputs, TS = 32 or 16: a lane holds row / column lane % TS of the operands, and of the four products of
// four consecutive elements the slice lane / TS; of the outputs column lane % TS and rows out_row(q).
template <int TS> struct Mma;
template <> struct Mma<32> {
    typedef floatx16 acc;
    static __device__ __forceinline__ acc mul(float a, float b, acc c) { return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0); }
    static __device__ __forceinline__ int out_row(int q, int slice) { return (q >> 2) * 8 + slice * 4 + (q & 3); }
};
template <> struct Mma<16> {
    typedef floatx4 acc;
    static __device__ __forceinline__ acc mul(float a, float b, acc c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
    static __device__ __forceinline__ int out_row(int q, int slice) { return slice * 4 + q; }
};

// Tile (bx, by) of TS x TS outputs by the sixteen waves of a workgroup.
template <int TS> using SmallRed = float[kSmallWaves][TS][TS + 1];
template <bool DGRAD, int TS, bool GATHER = false>
__device__ __forceinline__ void small_fc_tile(const SmallArgs& a, int bx, int by, int blocks, SmallRed<TS>& red, const SmallGather* in = nullptr) {
    constexpr int SLICES = 64 / TS, STEP = 4 * SLICES, Q = TS * TS / 64;      // reduction elements per step, outputs per lane
    // Chains of a wave: a 16x16 step has twice the elements of a 32x32 one, so that with two chains, turn and turn about by steps, they
    // were longer (256 elements: one of 16 products where two of 8 were; error against float64 1.04 of the larger tiles').  Four, by
    // the elements of a vector, cost no more.
    constexpr int CHAINS = TS == 16 ? 4 : 2;
    int r0, r1;
    const int shard = locate_block(a.cut, by, r0, r1);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, slice = lane / TS;
    const int row = min(r0 + lane % TS, r1 - 1), col = bx * TS + lane % TS, colc = min(col, a.N - 1);
    const float* const Ar = (GATHER ? in->data + (size_t)in->idx[row] * a.K : a.A + (size_t)row * a.K);
    const float* const Br = DGRAD ? a.B + colc : a.B + (size_t)colc * a.K;
    if (GATHER && bx == 0 && (int)threadIdx.x < r1 - r0) in->labels[r0 + threadIdx.x] = in->data_y[in->idx[r0 + threadIdx.x]];
    typename Mma<TS>::acc acc[CHAINS];
    #pragma unroll
    for (int c = 0; c < CHAINS; ++c)
        #pragma unroll
        for (int q = 0; q < Q; ++q) acc[c][q] = 0.f;
    const int steps = (a.K + STEP - 1) / STEP;
    // neighbouring steps share their cache lines; with four waves (and 32 KB in flight per workgroup) 784 -> 256 took 14 us
    const int piece = (steps + kSmallWaves - 1) / kSmallWaves, begin = wave * piece, end = min(begin + piece, steps);
    // N steps from s on, all their loads before the first product (reads past the end of the piece or of the reduction take the
    // last vector there is and count as zeros; rows and columns past theirs are not stored)
    auto batch = [&](int s, auto count) {
        constexpr int N = decltype(count)::value;
        float4 x[N], w[N];
        #pragma unroll
        for (int i = 0; i < N; ++i) {
            const int kc = min(min(s + i, end - 1) * STEP + slice * 4, a.K - 4);
            x[i] = *reinterpret_cast<const float4*>(Ar + kc);
            if (GATHER && bx == 0 && r0 + lane % TS < r1) *reinterpret_cast<float4*>(in->out + (size_t)row * a.K + kc) = x[i];
            if (DGRAD) w[i] = make_float4(Br[(size_t)kc * a.N], Br[(size_t)(kc + 1) * a.N], Br[(size_t)(kc + 2) * a.N], Br[(size_t)(kc + 3) * a.N]);
            else w[i] = *reinterpret_cast<const float4*>(Br + kc);
        }
        #pragma unroll
        for (int i = 0; i < N; ++i) {
            if (s + i >= end || (s + i) * STEP + slice * 4 >= a.K) { x[i] = make_float4(0.f, 0.f, 0.f, 0.f); w[i] = x[i]; }
            auto chain = [&](int e) -> auto& { return acc[CHAINS == 4 ? e : i & 1]; };
            chain(0) = Mma<TS>::mul(x[i].x, w[i].x, chain(0));
            chain(1) = Mma<TS>::mul(x[i].y, w[i].y, chain(1));
            chain(2) = Mma<TS>::mul(x[i].z, w[i].z, chain(2));
            chain(3) = Mma<TS>::mul(x[i].w, w[i].w, chain(3));
        }
    };
    // (784 -> 256, seven steps a wave: 11 us with a wait every two steps)
    if (piece <= 2) { if (begin < end) batch(begin, std::integral_constant<int, 2>()); }
    else if (piece <= 4) { if (begin < end) batch(begin, std::integral_constant<int, 4>()); }
    else for (int s = begin; s < end; s += 8) batch(s, std::integral_constant<int, 8>());
    #pragma unroll
    for (int q = 0; q < Q; ++q)
        red[wave][Mma<TS>::out_row(q, slice)][lane % TS] = CHAINS == 4 ? (acc[0][q] + acc[1][q]) + (acc[2][q] + acc[CHAINS - 1][q]) : acc[0][q] + acc[1][q];
    __syncthreads();
    const int rl = threadIdx.x / TS, cl = threadIdx.x % TS, r = r0 + rl, c = bx * TS + cl;
    const bool mine = rl < TS, live = mine && r < r1 && c < a.N;
    float v = 0.f;
    if (mine)
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
    if (mine) red[0][rl][cl] = live ? v : 0.f;
    __syncthreads();
    if (threadIdx.x >= TS || bx * TS + (int)threadIdx.x >= a.N) return;
    float p[4] = {0.f, 0.f, 0.f, 0.f};
    #pragma unroll
    for (int i = 0; i < TS; ++i) p[i & 3] += red[0][i][threadIdx.x];
    const float t = (p[0] + p[1]) + (p[2] + p[3]);
    const int cg = bx * TS + threadIdx.x;
    if (a.dbias.g != nullptr) a.dbias.g[(int64_t)a.cut.k[shard] * a.dbias.stride + cg] = t;
    else {
        a.sums[(size_t)cg * blocks + by] = t;
        a.sums[(size_t)(a.N + cg) * blocks + by] = 0.f;
    }
}

// Weight gradient of a layer whose shards have few rows: dw[k][c] = sum_m dy[m][k] x[m][c], a wave per 16x16 of a shard's, its
// rows in one chain, both operands straight from memory (lanes along k and c).
struct SmallWgradArgs {
    const float *dy, *x;         // [M][K], [M][C]
    GradDst dw;
    int K, C, tk, tc, tiles;     // tiles along k and c, in all
    ShardSet S;
};
__device__ __forceinline__ void small_wgrad_tile(const SmallWgradArgs& a, int tile) {
    const int lane = threadIdx.x & 63, slice = lane >> 4;
    const int sh = tile / (a.tk * a.tc), t = tile - sh * (a.tk * a.tc), kt = t / a.tc, ct = t - kt * a.tc;
    const int r0 = a.S.off[sh], r1 = a.S.off[sh + 1], k = kt * 16 + (lane & 15), c = ct * 16 + (lane & 15);
    const float* const yp = a.dy + min(k, a.K - 1);
    const float* const xp = a.x + min(c, a.C - 1);
    floatx4 acc = {0.f, 0.f, 0.f, 0.f};
    for (int r = r0; r < r1; r += 32) {
        float y[8], x[8];
        #pragma unroll
        for (int i = 0; i < 8; ++i) {
            const size_t row = (size_t)min(r + 4 * i + slice, r1 - 1);
            y[i] = yp[row * a.K];
            x[i] = xp[row * a.C];
        }
        #pragma unroll
        for (int i = 0; i < 8; ++i) {
            const bool in = r + 4 * i + slice < r1;
            acc = Mma<16>::mul(in ? y[i] : 0.f, in ? x[i] : 0.f, acc);
        }
    }
    if (c >= a.C) return;
    float* const out = a.dw.g + (int64_t)a.S.k[sh] * a.dw.stride + c;
    #pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int kk = kt * 16 + Mma<16>::out_row(q, slice);
        if (kk < a.K) out[(size_t)kk * a.C] = acc[q];
    }
}

// grid: (tiles of columns, blocks of rows)
template <bool DGRAD, int TS>
__global__ __launch_bounds__(64 * kSmallWaves) void small_fc_kernel(SmallArgs a) {
    __shared__ SmallRed<TS> red;
    small_fc_tile<DGRAD, TS>(a, blockIdx.x, blockIdx.y, gridDim.y, red);
}
template <int TS>
__global__ __launch_bounds__(64 * kSmallWaves) void small_fc_gather_kernel(SmallArgs a, SmallGather in) {
    __shared__ SmallRed<TS> red;
    small_fc_tile<false, TS, true>(a, blockIdx.x, blockIdx.y, gridDim.y, red, &in);
}
// grid: tiles / 16
__global__ __launch_bounds__(64 * kSmallWaves) void small_wgrad_kernel(SmallWgradArgs a) {
    const int tile = blockIdx.x * kSmallWaves + (threadIdx.x >> 6);
    if (tile < a.tiles) small_wgrad_tile(a, tile);
}
// Both gradients of a layer in one launch: grid: tiles of the input gradient (gx columns of them), then of the weights'
template <int TS>
__global__ __launch_bounds__(64 * kSmallWaves) void small_bwd_kernel(SmallArgs a, SmallWgradArgs w, int gx, int gy) {
    __shared__ SmallRed<TS> red;
    const int b = blockIdx.x;
    if (b < gx * gy) {
        small_fc_tile<true, TS>(a, b % gx, b / gx, gy, red);
        return;
    }
    const int tile = (b - gx * gy) * kSmallWaves + (threadIdx.x >> 6);
    if (tile < w.tiles) small_wgrad_tile(w, tile);
}

// Tiles of 16x16 where there are fewer than 64 of 32x32 (a workgroup of those reads twice as much, and what a CU can read is
// what such a launch waits for: 64 rows 784 -> 256, 16 workgroups, 11.2 us, 5.9 with 64), unless the bias gradients of the layer
// before would then be sums of two blocks.
static int small_tile(const ShardSet& S, int N) {
    const int64_t tiles = (int64_t)((S.plan + 31) / 32) * ((N + 31) / 32);
    return tiles < 64 && (S.plan_largest <= 16 || S.plan_largest > 32) ? 16 : 32;
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

void launch_small_fc_fwd(const ConvGeom& g, const ShardSet& S, const float* x, const float* w, const float* bias, bool relu, float* y, const SmallInput* in, hipStream_t st) {
    ShardSet all = {};           // (rows of several shards share a tile)
    all.p = 1;
    all.off[1] = g.N;
    all.plan_itself();
    const int ts = small_tile(S, g.K);
    SmallArgs a = {};
    a.A = x; a.B = w; a.out = y; a.bias = bias; a.relu = relu;
    a.K = g.C; a.N = g.K;
    a.cut = cut_rows(all, 1, ts);
    ProfScope ps(prof_shape_label("small_fc_fwd", g.N, g.K), 2.0 * g.N * g.K * g.C, 4.0 * ((double)g.N * (g.C + g.K) + (double)g.K * g.C), st);
    const dim3 grid((a.N + ts - 1) / ts, a.cut.blk0[a.cut.p]);
    if (in != nullptr) {
        SmallGather gather;
        gather.data = in->data; gather.data_y = in->data_y; gather.out = in->out; gather.labels = in->labels;
        for (int i = 0; i < kSmallGather; ++i) gather.idx[i] = i < g.N ? (int32_t)in->idx[i] : 0;
        if (ts == 16) hipLaunchKernelGGL(small_fc_gather_kernel<16>, grid, dim3(64 * kSmallWaves), 0, st, a, gather);
        else hipLaunchKernelGGL(small_fc_gather_kernel<32>, grid, dim3(64 * kSmallWaves), 0, st, a, gather);
        return;
    }
    if (ts == 16) hipLaunchKernelGGL((small_fc_kernel<false, 16>), grid, dim3(64 * kSmallWaves), 0, st, a);
    else hipLaunchKernelGGL((small_fc_kernel<false, 32>), grid, dim3(64 * kSmallWaves), 0, st, a);
}

static SmallWgradArgs small_wgrad_args(const ConvGeom& g, const ShardSet& S, const float* x, const float* dy, GradDst dw) {
    SmallWgradArgs a = {};
    a.dy = dy; a.x = x; a.dw = dw;
    a.K = g.K; a.C = g.C;
    a.tk = (g.K + 15) / 16; a.tc = (g.C + 15) / 16;
    a.tiles = S.p * a.tk * a.tc;
    a.S = S;
    return a;
}

bool small_wgrad_takes(int dtype, const ConvGeom& g, const ShardSet& S) {
    return dtype != 1 && g.H == 1 && g.W == 1 && g.R == 1 && g.S == 1 && g.stride == 1 && g.pad == 0 && S.plan_largest <= kSmallShard &&
           (int64_t)S.plan_p * ((g.K + 15) / 16) * ((g.C + 15) / 16) <= kSmallWgradTiles;
}

static double small_wgrad_bytes(const ConvGeom& g, const ShardSet& S) { return 4.0 * ((double)g.N * (g.C + g.K) + (double)S.p * g.K * g.C); }

void launch_small_wgrad(const ConvGeom& g, const ShardSet& S, const float* x, const float* dy, GradDst dw, hipStream_t st) {
    const SmallWgradArgs a = small_wgrad_args(g, S, x, dy, dw);
    ProfScope ps(prof_shape_label("small_fc_wgrad", g.N, g.C), 2.0 * g.N * g.K * g.C, small_wgrad_bytes(g, S), st);
    hipLaunchKernelGGL(small_wgrad_kernel, dim3((a.tiles + kSmallWaves - 1) / kSmallWaves), dim3(64 * kSmallWaves), 0, st, a);
}

RowCut launch_small_fc_dgrad(const ConvGeom& g, const ShardSet& S, const float* dy, const float* w, const float* old, float* dx,
                             const DgradMask* mask, const SmallWgrad* wgrad, hipStream_t st) {
    SmallArgs a = {};
    a.A = dy; a.B = w; a.out = dx; a.old = old;
    a.K = g.K; a.N = g.C;
    const int ts = small_tile(S, g.C);
    a.cut = cut_rows(S, 1, ts);
    const int blocks = a.cut.blk0[a.cut.p];
    const bool fuse = mask != nullptr && mask->act != nullptr && mask->xin == nullptr && mask->sums.buf != nullptr &&
                      mask->sums.floats >= (size_t)2 * g.C * blocks;
    a.cut.stored = fuse && mask->dbias.g != nullptr && a.cut.block_per_shard();
    if (fuse) {
        a.act = (const float*)mask->act;
        a.sums = mask->sums.buf;
        if (a.cut.stored) a.dbias = mask->dbias;
    }
    const int gx = (a.N + ts - 1) / ts;
    const double flops = 2.0 * g.N * g.K * g.C, bytes = 4.0 * ((double)g.N * (g.C + g.K) + (double)g.K * g.C);
    ProfScope ps(prof_shape_label("small_fc_dgrad", g.N, g.C), wgrad != nullptr ? 2.0 * flops : flops, wgrad != nullptr ? bytes + small_wgrad_bytes(g, S) : bytes, st);
    if (wgrad != nullptr) {
        const SmallWgradArgs w = small_wgrad_args(g, S, wgrad->x, dy, wgrad->dw);
        const dim3 grid(gx * blocks + (w.tiles + kSmallWaves - 1) / kSmallWaves);
        if (ts == 16) hipLaunchKernelGGL(small_bwd_kernel<16>, grid, dim3(64 * kSmallWaves), 0, st, a, w, gx, blocks);
        else hipLaunchKernelGGL(small_bwd_kernel<32>, grid, dim3(64 * kSmallWaves), 0, st, a, w, gx, blocks);
    } else {
        if (ts == 16) hipLaunchKernelGGL((small_fc_kernel<true, 16>), dim3(gx, blocks), dim3(64 * kSmallWaves), 0, st, a);
        else hipLaunchKernelGGL((small_fc_kernel<true, 32>), dim3(gx, blocks), dim3(64 * kSmallWaves), 0, st, a);
    }
    return fuse ? a.cut : RowCut();
}

// Where each of the launches would be the kernel that this one replaces, for rows of whole vectors, up to 15 outputs, shards of up
// to 64 rows and 64 KB of them (every workgroup reads all of its shard's).  us per step, this launch / the five:
//   float32, shards of 16: C = 256 35 / 46, 1,024 82 / 85     of 32: C = 256 53 / 61, 512 71 / 77, 1,024 85 / 83 and 110 / 111
//   of 64: C = 64 55 / 60, 256 50 / 51, 512 79 / 74, 1,024 99 / 79     odd rows, C = 211, 16 92 / 91, 32 111 / 107, 64 137 / 121
//   bf16, C = 1,024, shards of 16 95 / 109, of 32 106 / 113, of 64 125 / 122
bool thin_head_takes(int dtype, const ConvGeom& g, const ShardSet& S, const void* x, const void* w) {
    bool in_double;
    int tx;
    const bool small = small_fc_takes(dtype, g, g.C, g.K, S.plan);
    ConvGeom all = g;
    all.N = S.plan;
    return tune().thin_head != 0 && g.C % (dtype == 1 ? 8 : 4) == 0 && (((uintptr_t)x | (uintptr_t)w) & 15) == 0 && g.K < kHeadOutputs &&
           g.C <= kHeadColumns && S.plan_largest <= kHeadRows && S.plan_largest * g.C * (dtype == 1 ? 2 : 4) <= 65536 &&
           thin_fwd_takes(dtype, g, S.plan, small) && thin_dgrad_takes(dtype, all) && thin_wgrad_takes(dtype, g, S) && tune().fused_mask != 0 &&
           bias_sums_rows(dtype, S, 1, g.K, &tx, &in_double) >= S.plan_largest;
}

void launch_thin_head(int dtype, const ConvGeom& g, const ShardSet& S, const ThinHead& t, hipStream_t st) {
    HeadArgs a = {};
    a.x = t.x; a.w = t.w; a.bias = t.bias; a.labels = t.labels;
    a.logits = t.logits; a.row_loss = t.row_loss; a.loss = t.loss; a.dlogits = t.dlogits; a.dx = t.dx;
    a.dw = t.dw; a.db = t.db; a.dbias = t.dbias;
    a.K = g.K; a.C = g.C;
    a.S = S;
    bool in_double;
    (void)bias_sums_rows(dtype, S, 1, g.K, &a.tx, &in_double);
    a.in_double = in_double;
    const dim3 grid((g.C + 63) / 64, S.p);
    ProfScope ps("thin_head", 6.0 * g.N * g.K * g.C, (dtype == 1 ? 2.0 : 4.0) * (2.0 * g.N + g.K) * g.C + 4.0 * S.p * g.K * g.C, st);
    if (dtype == 1) hipLaunchKernelGGL(thin_head_kernel<bf16_t>, grid, dim3(1024), 0, st, a);
    else hipLaunchKernelGGL(thin_head_kernel<float>, grid, dim3(1024), 0, st, a);
}

}  // namespace edl
