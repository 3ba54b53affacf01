// Backward pass of a batch norm and of the 1x1 convolution before it that expands K channels into C = 4K (the last
// convolution of a residual block, the projection of the first stage), bf16, over many pixels:
//
//   dx[m][c]   = gamma rstd (dy - k0 - xhat k1)         the batch norm, rounded to bf16 as a stored tensor would be
//   dact[m][k] = sum_c dx[m][c] w[c][k]                  masked by act > 0 and summed for the batch norm before, see DgradMask
//   dw[c][k]   = sum_m dx[m][c] act[m][k]
//
// Memory bounds all three.  As three launches dx, the widest tensor, is written once and read twice; here it is not stored: a
// row is read as dy and x (4C bytes), act and the next batch norm's input (4K), and 2K bytes are written, 1.4 KB instead of
// 3.1 at C = 256.  A workgroup walks a run of rows, 32 at a time:
//   * its lanes form dx of the rows from what they have loaded and leave it in LDS; the next rows are on their way into
//     registers from then on;
//   * each wave contracts 128 channels of c for 32 of the 64 columns k (the weights stay in registers for the whole run), the
//     parts are added in float32 through LDS on the way to the epilogue;
//   * each wave keeps dw of 64 channels of c in registers for the whole run (both operands transposed on the way out of LDS);
//     pieces of runs are added by a second kernel, chains no longer than the smallest shard's own weight gradient would have;
//   * column sums in float64 per lane, one partial sum per run.
// C = 256: four waves, two workgroups per CU; C = 512: eight waves (the same work per wave), two workgroups for the 128
// columns, neighbours on a die that read the same rows.  C = 1,024 would take registers that are not there.
//
// us between events, three launches -> this one and the sum of the pieces, ResNet-50 at 8 shards of 32: M = 802,816, C = 256
// 449 -> 212 + 12 (5.3 TB/s of what has to move), M = 200,704, C = 512 254 -> 160 + 20; a shard of 32: M = 100,352, C = 256
// 61 -> 33 + 10.
#include <algorithm>

#include "bn_pointwise.h"
#include "dev_common.h"
#include "profiler.h"
#include "tune.h"

namespace edl {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef short shortx4 __attribute__((ext_vector_type(4)));

struct BnPointwiseArgs {
    const bf16_t *x, *dy, *act, *wT;
    bf16_t* dact;
    const float *gamma, *save, *coef;          // save, coef: of shard s at 2 * C * s
    const bf16_t* xin;                          // MASKED: the batch norm before
    const float* xin_save;                      // ... of shard s at 2 * K * s
    float* sums;                                // [2][K][runs]
    float* partial;                             // [runs][C][K]
    int K, gx, gy;                              // runs, groups of 64 columns
    RowCut cut;
};

constexpr int kTile = 32, kCols = 64;

// rows of one run: a row past the end reads as zeros and is not written
__device__ __forceinline__ __amdgpu_buffer_rsrc_t run_rsrc(const void* base, size_t first_byte, unsigned bytes) {
    return __builtin_amdgcn_make_buffer_rsrc((char*)const_cast<void*>(base) + first_byte, 0, bytes, 0x00020000);
}
template <bool NT = false>
__device__ __forceinline__ uint4 run_load(__amdgpu_buffer_rsrc_t r, unsigned at) {
    const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(r, at, 0, NT ? 2 : 0);
    return make_uint4(v.x, v.y, v.z, v.w);
}

// 16-byte slot of a row's chunk.  Rows of dx (a multiple of 256 bytes) are read whole, 16 rows at a time, and in 64-byte
// pieces of four consecutive rows (transposed): both spread over all banks.  Rows of act are 128 bytes.
__device__ __forceinline__ int dx_slot(int row, int chunk) { return chunk ^ (((row & 3) << 2) | ((row >> 2) & 3)); }
__device__ __forceinline__ int act_slot(int row, int chunk) { return chunk ^ (((row >> 1) & 1) << 2); }

// MFMA operand of 32 channels from `ch32` on for the rows [r16 + 8 * (lane / 32), + 8): ds_read_tr16_b64 hands a lane one channel
// of four consecutive rows when lane s of 16 reads row s / 4, channels 4 * (s % 4) .. + 3
template <int RB, typename SLOT>
__device__ __forceinline__ bf16x8 transposed(const unsigned char* tile, int ch32, int r16, int lane, SLOT slot) {
    typedef shortx4 __attribute__((address_space(3))) * lds_ptr;
    const int ch = ch32 + ((lane >> 4) & 1) * 16 + 4 * (lane & 3), row = r16 + (lane >> 5) * 8 + ((lane & 15) >> 2);
    const shortx4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(tile + row * RB + slot(row, ch >> 3) * 16 + (ch & 4) * 2));
    const shortx4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(tile + (row + 4) * RB + slot(row + 4, ch >> 3) * 16 + (ch & 4) * 2));
    const uint2 a = __builtin_bit_cast(uint2, lo), b = __builtin_bit_cast(uint2, hi);
    return __builtin_bit_cast(bf16x8, make_uint4(a.x, a.y, b.x, b.y));
}

template <int C, int NW, bool MASKED>
__global__ __launch_bounds__(64 * NW, 2) void bn_pointwise_bwd_kernel(BnPointwiseArgs a) {
    constexpr int NT = 64 * NW, PARTS = NW / 2;
    constexpr int CV = C / 8, RB = C * 2, AB = kCols * 2;              // vectors and bytes of a row of dx, bytes of one of act
    constexpr int ROWS = NT / CV, IT = kTile / ROWS;                    // rows of dx at a time, vectors per lane
    constexpr bool ONCE = C == 256;      // dy and x are read by one workgroup only (non-temporal: 249 -> 212 us; shared, slower)
    static_assert(C / PARTS == 128 && C / NW == 64 && ROWS * IT == kTile && kTile * (kCols / 8) == 256, "work of a wave");
    constexpr int XLD = kCols + 4;                                      // floats per row of the parts of dact
    __shared__ __attribute__((aligned(16))) unsigned char dxs[kTile * RB];
    __shared__ __attribute__((aligned(16))) unsigned char acts[kTile * AB];
    __shared__ __attribute__((aligned(16))) float parts[PARTS * kTile * XLD];
    __shared__ __attribute__((aligned(16))) float cf[4][C];             // mean, rstd k1, k0, gamma rstd

    __shared__ __attribute__((aligned(16))) float xcf[2][kCols];        // MASKED: mean, rstd of the batch norm before

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // a die gets a contiguous run of row blocks (pointwise_kernel)
    int l = blockIdx.x;
    {
        const int total = a.gx * a.gy, q = total >> 3, r = total & 7, die = l & 7, slot = l >> 3;
        l = die * q + (die < r ? die : r) + slot;
    }
    const int bx = l / a.gy, by = l - bx * a.gy;
    int m0, m_end;
    const int shard = locate_block(a.cut, bx, m0, m_end);
    const int rows = m_end - m0, K = a.K;

    const float* const save = a.save + (size_t)shard * 2 * C;
    const float* const coef = a.coef + (size_t)shard * 2 * C;
    for (int c = tid; c < C; c += NT) {
        const float rs = save[C + c];
        cf[0][c] = save[c];
        cf[1][c] = rs * coef[C + c];
        cf[2][c] = coef[c];
        cf[3][c] = a.gamma[c] * rs;
    }

    if (MASKED && tid < 2 * kCols) xcf[tid / kCols][tid % kCols] = a.xin_save[(size_t)shard * 2 * K + (tid / kCols) * K + by * kCols + tid % kCols];

    // the weights of this wave's 32 columns and 128 channels, as MFMA operands
    const int col32 = (wave & 1) * 32, part = wave >> 1;
    bf16x8 wf[8];
    #pragma unroll
    for (int g = 0; g < 8; ++g)
        wf[g] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(a.wT + (size_t)(by * kCols + col32 + (lane & 31)) * C + part * 128 + (2 * g + (lane >> 5)) * 8));

    const __amdgpu_buffer_rsrc_t rDy = run_rsrc(a.dy, (size_t)m0 * RB, (unsigned)rows * RB);
    const __amdgpu_buffer_rsrc_t rX = run_rsrc(a.x, (size_t)m0 * RB, (unsigned)rows * RB);
    const unsigned row_bytes = (unsigned)K * 2u;
    const size_t first = (size_t)m0 * row_bytes;
    const __amdgpu_buffer_rsrc_t rAct = run_rsrc(a.act, first, (unsigned)rows * row_bytes);
    const __amdgpu_buffer_rsrc_t rXin = run_rsrc(MASKED ? a.xin : nullptr, first, MASKED ? (unsigned)rows * row_bytes : 0u);
    const __amdgpu_buffer_rsrc_t rOut = run_rsrc(a.dact, first, (unsigned)rows * row_bytes);

    // this lane's vectors: of dy and x; of act, xin and dact (the first 256 lanes)
    const int chunk = tid % CV, row_c = tid / CV;
    const bool narrow = NT == 256 || wave < 4;
    const int row_k = (tid & 255) >> 3, c8 = (tid & 7) * 8;
    const unsigned at_k = (unsigned)(by * kCols + c8) * 2u;
    uint4 dyv[IT], xv[IT], actv = make_uint4(0, 0, 0, 0), xinv = make_uint4(0, 0, 0, 0);
    auto load = [&](int m) {
        #pragma unroll
        for (int i = 0; i < IT; ++i) {
            const unsigned at = (unsigned)(m + row_c + i * ROWS) * RB + chunk * 16;
            dyv[i] = run_load<ONCE>(rDy, at);
            xv[i] = run_load<ONCE>(rX, at);
        }
        if (narrow) {
            const unsigned at = (unsigned)(m + row_k) * row_bytes + at_k;
            actv = run_load<true>(rAct, at);
            if (MASKED) xinv = run_load(rXin, at);
        }
    };

    double s1[8], s2[8];
    #pragma unroll
    for (int e = 0; e < 8; ++e) s1[e] = s2[e] = 0.0;
    floatx16 dw[2][2];
    #pragma unroll
    for (int i = 0; i < 2; ++i)
        #pragma unroll
        for (int j = 0; j < 2; ++j)
            #pragma unroll
            for (int q = 0; q < 16; ++q) dw[i][j][q] = 0.f;

    load(0);
    __syncthreads();                      // the coefficients are in LDS
    for (int m = 0; m < rows; m += kTile) {
        {
            float4 c4[4][2];
            #pragma unroll
            for (int k = 0; k < 4; ++k)
                #pragma unroll
                for (int h = 0; h < 2; ++h) c4[k][h] = *reinterpret_cast<const float4*>(&cf[k][chunk * 8 + h * 4]);
            const float* const f = reinterpret_cast<const float*>(c4);
            #pragma unroll
            for (int i = 0; i < IT; ++i) {
                const int row = row_c + i * ROWS;
                const uint32_t gw[4] = {dyv[i].x, dyv[i].y, dyv[i].z, dyv[i].w}, xw[4] = {xv[i].x, xv[i].y, xv[i].z, xv[i].w};
                uint32_t out[4];
                #pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float g0 = __uint_as_float(gw[e] << 16), g1 = __uint_as_float(gw[e] & 0xffff0000u);
                    const float x0 = __uint_as_float(xw[e] << 16), x1 = __uint_as_float(xw[e] & 0xffff0000u);
                    const float d0 = f[24 + 2 * e] * (g0 - f[16 + 2 * e] - (x0 - f[2 * e]) * f[8 + 2 * e]);
                    const float d1 = f[25 + 2 * e] * (g1 - f[17 + 2 * e] - (x1 - f[2 * e + 1]) * f[9 + 2 * e]);
                    out[e] = m + row < rows ? pack2_bf16(d0, d1) : 0u;
                }
                *reinterpret_cast<uint4*>(dxs + row * RB + dx_slot(row, chunk) * 16) = make_uint4(out[0], out[1], out[2], out[3]);
            }
        }
        const uint4 act = actv, xin = xinv;
        if (narrow) *reinterpret_cast<uint4*>(acts + row_k * AB + act_slot(row_k, c8 >> 3) * 16) = act;
        load(m + kTile);
        // (the wait is spelled out as in pointwise_kernel: the compiler does not put it before every barrier)
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __syncthreads();
        floatx16 acc;
        #pragma unroll
        for (int q = 0; q < 16; ++q) acc[q] = 0.f;
        #pragma unroll
        for (int g = 0; g < 8; ++g) {
            const int row = lane & 31;
            const uint4 d = *reinterpret_cast<const uint4*>(dxs + row * RB + dx_slot(row, part * 16 + 2 * g + (lane >> 5)) * 16);
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[g], __builtin_bit_cast(bf16x8, d), acc, 0, 0, 0);
        }
        // lane: pixel lane % 32, columns (q / 4) * 8 + (lane / 32) * 4 + q % 4
        #pragma unroll
        for (int q = 0; q < 16; q += 4)
            *reinterpret_cast<float4*>(&parts[(part * kTile + (lane & 31)) * XLD + col32 + (q >> 2) * 8 + (lane >> 5) * 4]) =
                make_float4(acc[q], acc[q + 1], acc[q + 2], acc[q + 3]);
        #pragma unroll
        for (int r16 = 0; r16 < kTile; r16 += 16) {
            bf16x8 fa[2], fb[2];
            #pragma unroll
            for (int i = 0; i < 2; ++i) {
                fa[i] = transposed<RB>(dxs, wave * 64 + i * 32, r16, lane, dx_slot);
                fb[i] = transposed<AB>(acts, i * 32, r16, lane, act_slot);
            }
            #pragma unroll
            for (int i = 0; i < 2; ++i)
                #pragma unroll
                for (int j = 0; j < 2; ++j) dw[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[i], fb[j], dw[i][j], 0, 0, 0);
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __syncthreads();                  // the parts are there, and everyone is done with the tile
        if (narrow) {
            float v[8];
            #pragma unroll
            for (int h = 0; h < 2; ++h) {
                float4 s = *reinterpret_cast<const float4*>(&parts[row_k * XLD + c8 + h * 4]);
                #pragma unroll
                for (int p = 1; p < PARTS; ++p) {
                    const float4 t = *reinterpret_cast<const float4*>(&parts[(p * kTile + row_k) * XLD + c8 + h * 4]);
                    s.x += t.x; s.y += t.y; s.z += t.z; s.w += t.w;
                }
                v[4 * h] = s.x; v[4 * h + 1] = s.y; v[4 * h + 2] = s.z; v[4 * h + 3] = s.w;
            }
            const uint32_t aw[4] = {act.x, act.y, act.z, act.w};
            if (MASKED)
                #pragma unroll
                for (int e = 0; e < 4; ++e) {
                    v[2 * e] = __uint_as_float(aw[e] << 16) > 0.f ? v[2 * e] : 0.f;
                    v[2 * e + 1] = __uint_as_float(aw[e] & 0xffff0000u) > 0.f ? v[2 * e + 1] : 0.f;
                }
            const u32x4 pk = {pack2_bf16(v[0], v[1]), pack2_bf16(v[2], v[3]), pack2_bf16(v[4], v[5]), pack2_bf16(v[6], v[7])};
            __builtin_amdgcn_raw_buffer_store_b128(pk, rOut, (unsigned)(m + row_k) * row_bytes + at_k, 0, 0);
            if (MASKED) {
                // of what a reader of the stored tensor sees (rows past the end are zeros)
                const uint32_t xw[4] = {xin.x, xin.y, xin.z, xin.w};
                const float *const mu = &xcf[0][c8], *const rs = &xcf[1][c8];
                #pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float lo = __uint_as_float(pk[e] << 16), hi = __uint_as_float(pk[e] & 0xffff0000u);
                    s1[2 * e] += (double)lo;
                    s1[2 * e + 1] += (double)hi;
                    s2[2 * e] += (double)(lo * ((__uint_as_float(xw[e] << 16) - mu[2 * e]) * rs[2 * e]));
                    s2[2 * e + 1] += (double)(hi * ((__uint_as_float(xw[e] & 0xffff0000u) - mu[2 * e + 1]) * rs[2 * e + 1]));
                }
            }
        }
    }
    // lane: column lane % 32, channels (q / 4) * 8 + (lane / 32) * 4 + q % 4 of each 32x32 tile
    float* const out = a.partial + ((size_t)bx * C + wave * 64 + (lane >> 5) * 4) * K + by * kCols + (lane & 31);
    #pragma unroll
    for (int i = 0; i < 2; ++i)
        #pragma unroll
        for (int j = 0; j < 2; ++j)
            #pragma unroll
            for (int q = 0; q < 16; ++q) out[(size_t)(i * 32 + (q >> 2) * 8 + (q & 3)) * K + j * 32] = dw[i][j][q];
    if (!MASKED) return;
    // lanes with the same columns differ in lane / 8 and in the wave
    __syncthreads();
    double* const red = reinterpret_cast<double*>(parts);
    static_assert(4 * 2 * kCols * 8 <= sizeof(parts), "column sums fit");
    if (narrow) {
        #pragma unroll
        for (int e = 0; e < 8; ++e) {
            #pragma unroll
            for (int o = 8; o < 64; o <<= 1) {
                s1[e] += __shfl_xor(s1[e], o, 64);
                s2[e] += __shfl_xor(s2[e], o, 64);
            }
            if (lane < 8) {
                red[(wave * 2 + 0) * kCols + c8 + e] = s1[e];
                red[(wave * 2 + 1) * kCols + c8 + e] = s2[e];
            }
        }
    }
    __syncthreads();
    if (tid < 2 * kCols) {
        double s = red[tid];
        #pragma unroll
        for (int w = 1; w < 4; ++w) s += red[w * 2 * kCols + tid];
        const int kind = tid / kCols, c = by * kCols + tid % kCols;
        a.sums[(size_t)(kind * K + c) * a.gx + bx] = (float)s;
    }
}

// dw of a shard = the sum of its runs' pieces: 16 lanes side by side take 16 vectors, 16 groups of them every 16th piece.
// grid: (groups of 16 vectors, shards)
__global__ __launch_bounds__(256) void bn_pointwise_reduce_kernel(const float* __restrict__ part, GradDst dw, RowCut cut, int n, int vec) {
    __shared__ float4 red[16][17];
    const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4, s = blockIdx.y, i = blockIdx.x * 16 + tx;
    const int pieces = cut.blk0[s + 1] - cut.blk0[s], nv = n / 4;
    const float4* const p = reinterpret_cast<const float4*>(part) + (size_t)cut.blk0[s] * nv + i;
    float4 t = make_float4(0.f, 0.f, 0.f, 0.f);
    #pragma unroll 4
    for (int k = ty; k < pieces; k += 16) {
        const float4 v = p[(size_t)k * nv];
        t.x += v.x; t.y += v.y; t.z += v.z; t.w += v.w;
    }
    red[ty][tx] = t;
    __syncthreads();
    if (ty != 0) return;
    #pragma unroll
    for (int k = 1; k < 16; ++k) { t.x += red[k][tx].x; t.y += red[k][tx].y; t.z += red[k][tx].z; t.w += red[k][tx].w; }
    float* const d = dw.g + (int64_t)cut.k[s] * dw.stride + (int64_t)i * 4;
    if (vec) *reinterpret_cast<float4*>(d) = t;
    else { d[0] = t.x; d[1] = t.y; d[2] = t.z; d[3] = t.w; }
}

// Rows of a run: workgroups for two per CU (C = 512: one per CU), chains no longer than the weight gradient of the pass's
// smallest shard alone has, and pieces of at most half the bytes of the batch norm's gradient (they lie in its place: four times
// K rows).
static int rows_per_run(const ConvGeom& g, const ShardSet& S) {
    ConvGeom small = g;
    small.N = S.plan_smallest;
    const int chain = conv_wgrad_chain(1, small) / kTile * kTile;
    const int64_t M = (int64_t)S.plan * g.H * g.W, runs = (g.K == 256 ? 512 : 256) / (g.C / kCols);
    const int64_t rows = ((M + runs - 1) / runs + kTile - 1) / kTile * kTile;
    return (int)std::min<int64_t>(std::max<int64_t>(rows, 4 * g.C), chain);
}

// From 65,536 rows on.  Below, runs of 4K rows leave CUs idle: ResNet-50 at a shard of 32, the layers of 25,088 rows and C = 512
// (98 workgroups) 46 us for 46 in three launches of which one ran beside the chain: the step 4,041 -> 4,058 us.
bool bn_pointwise_takes(int dtype, const ConvGeom& g, const ShardSet& S) {
    if (dtype != 1 || g.R != 1 || g.S != 1 || g.stride != 1 || g.pad != 0 || tune().force_tile >= 0) return false;
    if (g.K != 4 * g.C || (g.C != 64 && g.C != 128)) return false;
    const int64_t hw = (int64_t)g.H * g.W;
    if (S.plan * hw < tune().bn_pointwise_rows || S.plan_smallest * hw < 4 * g.C) return false;
    const int R = rows_per_run(g, S);
    if (R < 4 * g.C) return false;
    // the pieces fit where they go, and the sums where any batch norm's of C channels fit
    const RowCut cut = cut_rows(S, g.H * g.W, R);
    return (int64_t)cut.blk0[cut.p] * g.C * 2 <= S.samples() * hw && (S.plan * hw / R + S.plan_p) * g.C <= (int64_t)kRedRowBlocks * g.K;
}

RowCut launch_bn_pointwise_backward(const ConvGeom& g, const ShardSet& S, const BnPointwiseTask& t, hipStream_t st) {
    BnPointwiseArgs a = {};
    a.x = (const bf16_t*)t.x; a.dy = (const bf16_t*)t.dy; a.act = (const bf16_t*)t.act; a.wT = (const bf16_t*)t.wT;
    a.dact = (bf16_t*)t.dact;
    a.gamma = t.gamma; a.save = t.save; a.coef = t.coef;
    a.partial = t.partial;
    a.K = g.C;
    a.cut = cut_rows(S, g.H * g.W, rows_per_run(g, S));
    a.gx = a.cut.blk0[a.cut.p]; a.gy = g.C / kCols;
    const double M = (double)S.samples() * g.H * g.W;
    ProfScope ps(prof_shape_label("bn_pointwise_bwd", (int64_t)M, g.K), 4.0 * M * g.K * g.C, 2.0 * M * (2.0 * g.K + (t.mask ? 3.0 : 2.0) * g.C), st);
    const dim3 grid(a.gx * a.gy);
    if (t.mask != nullptr) {
        a.xin = (const bf16_t*)t.mask->xin; a.xin_save = t.mask->mean_rstd; a.sums = t.mask->sums.buf;
        if (g.K == 256) hipLaunchKernelGGL((bn_pointwise_bwd_kernel<256, 4, true>), grid, dim3(256), 0, st, a);
        else hipLaunchKernelGGL((bn_pointwise_bwd_kernel<512, 8, true>), grid, dim3(512), 0, st, a);
        return a.cut;
    }
    if (g.K == 256) hipLaunchKernelGGL((bn_pointwise_bwd_kernel<256, 4, false>), grid, dim3(256), 0, st, a);
    else hipLaunchKernelGGL((bn_pointwise_bwd_kernel<512, 8, false>), grid, dim3(512), 0, st, a);
    return RowCut();
}

void launch_bn_pointwise_reduce(const ConvGeom& g, const ShardSet& S, const float* partial, GradDst dw, hipStream_t st) {
    const RowCut cut = cut_rows(S, g.H * g.W, rows_per_run(g, S));
    const int n = g.K * g.C;
    ProfScope ps("wgrad_reduce", 0.0, 4.0 * (double)n * (cut.blk0[cut.p] + S.p), st);
    const int vec = ((uintptr_t)dw.g & 15) == 0 && dw.stride % 4 == 0;
    hipLaunchKernelGGL(bn_pointwise_reduce_kernel, dim3(n / 64, S.p), dim3(256), 0, st, partial, dw, cut, n, vec);
}

}  // namespace edl
