// 1x1 convolutions of stride 1 with a short reduction and a wide output (the expanding layers of a residual block and
// the input gradients that end at its join), bf16, over many pixels:
//
//   out[m][n] = sum_k A[m][k] * B[n][k]      K = 64, 128, 256 or 512;  N a multiple of 256;  M pixels
//
// What bounds them is memory: at K = 64 and N = 256 a row is 128 bytes in and 512 out (a join reads another 1,056), and
// the tiled kernel of k_conv.hip spent its time between a tile's loads and its stores instead (set-up, one or two reduction
// steps, an epilogue, per workgroup of 128x64 outputs: 3.0 TB/s, a join 3.9).  Here a workgroup walks a run of rows:
//   * its waves, four at K = 64 and eight above, own 64 or 32 of 256 columns each; their weights stay in registers for the
//     whole run (32 of them per lane at K = 64 and 128, 64 at 256, 128 at 512), so LDS holds only the rows, read once for
//     256 columns;
//   * the next rows, and what the epilogue of the next 32 reads, are on their way into registers while the present ones are
//     contracted and stored (joins without that: 5 to 15% slower; forward at K = 64 with 32 rows in flight per workgroup
//     instead of 64, both at one workgroup per CU: 148 us for 116; with two it is 102);
//   * the weights are the first operand of the MFMA, so that a lane gets four consecutive channels of one pixel; the wave
//     turns its 32 pixels into rows through LDS of its own, which takes no barrier (one per tile of rows is left);
//   * the column sums a batch norm wants (of the stored values, see ConvArgs::stats and ::msum) are kept in float64 per lane
//     from one tile to the next: one partial sum per channel and run of rows.
// The contraction runs over k in the same order as in the tiled kernel: the outputs are the same bits.
// Measured: 5.0 TB/s at M = 802,816, N = 256, K = 64, a join 5.1 TB/s (pointwise_takes has the times).
// The variants are those without spills.  At K = 512 that takes an instruction more per LDS read: with the read addresses kept
// in registers the join had 23 others in scratch (M = 12,544, N = 2,048: 82 us for 61) and the forward launch fewer loads
// under way (M = 200,704, N = 256: 94 for 77).
#include <algorithm>

#include "dev_common.h"
#include "kernels.h"
#include "pointwise.h"
#include "profiler.h"
#include "tune.h"

namespace edl {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

struct PointwiseArgs {
    const bf16_t* A;                 // [M][K]
    const bf16_t* B;                 // [N][K]
    bf16_t* out;                     // [M][N]
    // JOIN: out = (sum + old) where sign's bit is set, else 0; sums of that and of that times (xin - mean) * rstd
    const bf16_t* old;               // may be out itself: a lane reads what it overwrites
    const unsigned char* sign;
    const bf16_t* xin;
    const float* mean_rstd;          // of shard s at 2 * N * s
    float* sums;                     // [2][N][row blocks], may be null (forward)
    int N, gx, gy;                   // row blocks, column blocks of 256
    RowCut cut;
};

constexpr int kRows = 32, kCols = 256;

// Rows of one run through a buffer descriptor: a row past the end reads as zeros and is not written, so that neither
// needs a branch, and offsets take 32 bits.
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rows_rsrc(const void* base, size_t first_byte, unsigned bytes) {
    return __builtin_amdgcn_make_buffer_rsrc((char*)const_cast<void*>(base) + first_byte, 0, bytes, 0x00020000);
}
__device__ __forceinline__ uint4 rows_load(__amdgpu_buffer_rsrc_t r, unsigned at) {
    const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(r, at, 0, 0);
    return make_uint4(v.x, v.y, v.z, v.w);
}

template <int K, int NW, int SUB, bool JOIN>
__global__ __launch_bounds__(64 * NW, 2) void pointwise_kernel(PointwiseArgs a) {
    constexpr int NT = 64 * NW, TN = 8 / NW;                                  // lanes; MFMA tiles of 32 columns per wave
    constexpr int KV = K / 8, RB = K * 2, RPL = RB >= 256 ? 1 : 256 / RB;     // vectors, bytes per row; rows per 256 bytes
    constexpr int TROWS = kRows * SUB;                                        // rows per barrier
    constexpr int IT = TROWS * KV / NT;                                       // vectors of a tile per lane
    constexpr int G = K / 16;
    constexpr bool AHEAD = JOIN && K <= 256;      // (K = 512: no registers left)
    constexpr int TILE = TROWS * RB;
    // a wave's outputs on their way to rows: float32 where the epilogue adds to them, else bf16; rows of 68 (36) words or 34
    // (18), so that neither the writes of 32 pixels nor the reads of rows meet in a bank
    constexpr int LDS_ROW = JOIN ? (32 * TN + 4) * 4 : (16 * TN + 2) * 4;
    constexpr int STAGE = kRows * LDS_ROW;
    __shared__ __attribute__((aligned(16))) unsigned char smem[2 * TILE + NW * STAGE];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // consecutive workgroups go to the eight dies in turn: a die gets a contiguous run of row blocks, whose column blocks
    // (which read the same rows) are neighbours
    int l = blockIdx.x;
    {
        const int total = a.gx * a.gy, q = total >> 3, r = total & 7, die = l & 7, slot = l >> 3;
        l = die * q + (die < r ? die : r) + slot;
    }
    const int bx = l / a.gy, by = l - bx * a.gy;
    int m0, m_end;
    const int shard = locate_block(a.cut, bx, m0, m_end);
    const int n0 = by * kCols + wave * (32 * TN);
    unsigned char* const stage = smem + 2 * TILE + wave * STAGE;

    // the weights of this wave's columns, as MFMA operands
    uint4 wf[TN][G];
    #pragma unroll
    for (int j = 0; j < TN; ++j)
        #pragma unroll
        for (int g = 0; g < G; ++g)
            wf[j][g] = *reinterpret_cast<const uint4*>(a.B + (size_t)(n0 + j * 32 + (lane & 31)) * K + (2 * g + (lane >> 5)) * 8);

    // the run's rows in the tensors
    const unsigned rows = (unsigned)(m_end - m0), row_bytes = (unsigned)a.N * 2u;
    const __amdgpu_buffer_rsrc_t rA = rows_rsrc(a.A, (size_t)m0 * RB, rows * RB);
    const size_t first = (size_t)m0 * row_bytes;
    const __amdgpu_buffer_rsrc_t rOut = rows_rsrc(a.out, first, rows * row_bytes);
    const __amdgpu_buffer_rsrc_t rOld = rows_rsrc(JOIN ? a.old : nullptr, first, JOIN ? rows * row_bytes : 0);
    const __amdgpu_buffer_rsrc_t rXin = rows_rsrc(JOIN ? a.xin : nullptr, first, JOIN ? rows * row_bytes : 0);
    const __amdgpu_buffer_rsrc_t rSign = rows_rsrc(JOIN ? a.sign : nullptr, first / 16, JOIN ? rows * (row_bytes / 16) : 0);

    // this lane's vectors of the tile at row m of the run
    const int ld_row = tid / KV, ld_chunk = tid % KV;
    auto load_rows = [&](int m, uint4 (&r)[IT]) {
        #pragma unroll
        for (int i = 0; i < IT; ++i) r[i] = rows_load(rA, (unsigned)(m + ld_row + i * (NT / KV)) * RB + ld_chunk * 16);
    };
    auto put_rows = [&](int buf, const uint4 (&r)[IT]) {
        #pragma unroll
        for (int i = 0; i < IT; ++i) {
            const int row = ld_row + i * (NT / KV);
            *reinterpret_cast<uint4*>(smem + buf * TILE + row * RB + ((ld_chunk ^ ((row / RPL) % KV)) * 16)) = r[i];
        }
    };

    // in the output phase a lane holds 8 channels of every ROWS-th row
    constexpr int LANES = 4 * TN, ROWS = 64 / LANES, NK = kRows / ROWS;
    const int cv = lane % LANES, c8 = n0 + cv * 8, r8 = lane / LANES;
    float mu[8], rs[8];
    if (JOIN) {
        const float* const ms = a.mean_rstd + (size_t)shard * 2 * a.N;
        #pragma unroll
        for (int e = 0; e < 8; ++e) { mu[e] = ms[c8 + e]; rs[e] = ms[a.N + c8 + e]; }
    }
    double s1[8], s2[8];
    #pragma unroll
    for (int e = 0; e < 8; ++e) s1[e] = s2[e] = 0.0;

    // what the epilogue of the 32 rows at row m of the run reads
    uint4 oldv[NK], xinv[NK];
    unsigned signv[NK];
    auto load_join = [&](int m) {
        #pragma unroll
        for (int k = 0; k < NK; ++k) {
            const unsigned at = (unsigned)(m + r8 + ROWS * k) * row_bytes + (unsigned)c8 * 2u;
            oldv[k] = rows_load(rOld, at);
            xinv[k] = rows_load(rXin, at);
            signv[k] = __builtin_amdgcn_raw_buffer_load_b8(rSign, at / 16, 0, 0);
        }
    };

    uint4 next[IT];
    load_rows(0, next);
    if (AHEAD) load_join(0);
    put_rows(0, next);
    int buf = 0;
    for (int mt = 0; mt < (int)rows; mt += TROWS, buf ^= 1) {
        // This wave's part of the tile is in LDS ...  (Not redundant: the compiler leaves its own wait out here, where the writes come
        // round the loop, in every one of these kernels; without this line other waves read rows that are not written yet.)
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __syncthreads();      // ... every wave's is, and every wave is done with the tile before
        load_rows(mt + TROWS, next);
        #pragma unroll
        for (int sub = 0; sub < SUB; ++sub) {
            const int m = mt + sub * kRows;
            if (JOIN && !AHEAD) load_join(m);
            floatx16 acc[TN];
            #pragma unroll
            for (int j = 0; j < TN; ++j)
                #pragma unroll
                for (int q = 0; q < 16; ++q) acc[j][q] = 0.f;
            const int row = sub * kRows + (lane & 31);
            int turn = (row / RPL) % KV;
            // (K = 512: the compiler would compute the 32 addresses once, ahead of the loop, into 32 registers that are not there)
            if (K == 512) asm volatile("" : "+v"(turn));
            #pragma unroll
            for (int g = 0; g < G; ++g) {
                const uint4 x = *reinterpret_cast<const uint4*>(smem + buf * TILE + row * RB + (((2 * g + (lane >> 5)) ^ turn) * 16));
                #pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, wf[j][g]), __builtin_bit_cast(bf16x8, x), acc[j], 0, 0, 0);
            }
            // lane: pixel lane % 32, channels j * 32 + (q / 4) * 8 + (lane / 32) * 4 + q % 4
            wave_lds_handover();
            #pragma unroll
            for (int j = 0; j < TN; ++j)
                #pragma unroll
                for (int q = 0; q < 16; q += 4) {
                    const int ch = j * 32 + (q >> 2) * 8 + (lane >> 5) * 4;
                    unsigned char* const p = stage + (lane & 31) * LDS_ROW;
                    if (JOIN) *reinterpret_cast<float4*>(p + ch * 4) = make_float4(acc[j][q], acc[j][q + 1], acc[j][q + 2], acc[j][q + 3]);
                    else *reinterpret_cast<uint2*>(p + ch * 2) = make_uint2(pack2_bf16(acc[j][q], acc[j][q + 1]), pack2_bf16(acc[j][q + 2], acc[j][q + 3]));
                }
            wave_lds_handover();
            float t1[8], t2[8];
            #pragma unroll
            for (int e = 0; e < 8; ++e) t1[e] = t2[e] = 0.f;
            uint4 ov[NK], xv[NK];
            unsigned sv[NK];
            if (JOIN) {
                #pragma unroll
                for (int k = 0; k < NK; ++k) { ov[k] = oldv[k]; xv[k] = xinv[k]; sv[k] = signv[k]; }
                if (AHEAD) load_join(m + kRows);       // of the next 32 rows
            }
            #pragma unroll
            for (int k = 0; k < NK; ++k) {
                const int rl = r8 + ROWS * k;
                const unsigned char* const p = stage + rl * LDS_ROW;
                uint4 pk;
                if (JOIN) {
                    const float4 f0 = *reinterpret_cast<const float4*>(p + cv * 32), f1 = *reinterpret_cast<const float4*>(p + cv * 32 + 16);
                    float v[8] = {f0.x, f0.y, f0.z, f0.w, f1.x, f1.y, f1.z, f1.w};
                    const uint32_t ow[4] = {ov[k].x, ov[k].y, ov[k].z, ov[k].w};
                    #pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        v[2 * e] += __uint_as_float(ow[e] << 16);
                        v[2 * e + 1] += __uint_as_float(ow[e] & 0xffff0000u);
                    }
                    #pragma unroll
                    for (int e = 0; e < 8; ++e) v[e] = (sv[k] >> e) & 1u ? v[e] : 0.f;
                    pk = make_uint4(pack2_bf16(v[0], v[1]), pack2_bf16(v[2], v[3]), pack2_bf16(v[4], v[5]), pack2_bf16(v[6], v[7]));
                } else {
                    const uint2 h0 = *reinterpret_cast<const uint2*>(p + cv * 16), h1 = *reinterpret_cast<const uint2*>(p + cv * 16 + 8);
                    pk = make_uint4(h0.x, h0.y, h1.x, h1.y);
                }
                const u32x4 out = {pk.x, pk.y, pk.z, pk.w};
                __builtin_amdgcn_raw_buffer_store_b128(out, rOut, (unsigned)(m + rl) * row_bytes + (unsigned)c8 * 2u, 0, 0);
                // sums of what a reader of the stored tensor sees (rows past the end are zeros)
                const uint32_t w4[4] = {pk.x, pk.y, pk.z, pk.w};
                const uint32_t xw[4] = {xv[k].x, xv[k].y, xv[k].z, xv[k].w};
                #pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float lo = __uint_as_float(w4[e] << 16), hi = __uint_as_float(w4[e] & 0xffff0000u);
                    t1[2 * e] += lo;
                    t1[2 * e + 1] += hi;
                    if (JOIN) {
                        const float xl = __uint_as_float(xw[e] << 16), xh = __uint_as_float(xw[e] & 0xffff0000u);
                        t2[2 * e] += lo * ((xl - mu[2 * e]) * rs[2 * e]);
                        t2[2 * e + 1] += hi * ((xh - mu[2 * e + 1]) * rs[2 * e + 1]);
                    } else {
                        t2[2 * e] += lo * lo;
                        t2[2 * e + 1] += hi * hi;
                    }
                }
            }
            #pragma unroll
            for (int e = 0; e < 8; ++e) { s1[e] += (double)t1[e]; s2[e] += (double)t2[e]; }
        }
        __builtin_amdgcn_wave_barrier();
        put_rows(buf ^ 1, next);
    }
    if (a.sums == nullptr) return;
    // lanes with the same channels differ in lane / LANES
    #pragma unroll
    for (int e = 0; e < 8; ++e) {
        #pragma unroll
        for (int o = LANES; o < 64; o <<= 1) {
            s1[e] += __shfl_xor(s1[e], o, 64);
            s2[e] += __shfl_xor(s2[e], o, 64);
        }
        if (lane < LANES) {
            a.sums[(size_t)(c8 + e) * a.gx + bx] = (float)s1[e];
            a.sums[(size_t)(a.N + c8 + e) * a.gx + bx] = (float)s2[e];
        }
    }
}

// Rows of a workgroup's run: the chip is filled once, with eight waves per CU (what their registers leave room for; more and
// shorter runs lose: 256 / 512 / 1,024 workgroups for K = 256, M = 50,176, N = 1,024: 90 / 100 / 108 us).
static int rows_per_run(int64_t M, int K, int N) {
    const int64_t target = tune().pointwise_blocks * (K == 64 ? 2 : 1);
    const int64_t runs = std::max<int64_t>(1, target / (N / kCols));
    const int64_t rows = (M + runs - 1) / runs;
    return (int)((rows + kRows - 1) / kRows * kRows);
}

// From 32,768 rows of 256 columns on (four tiles of 32 per workgroup).  Below, a workgroup has too few tiles to pay for the
// weights that it loads.  us between events, tiled / streaming, forward and join (a first block's join and its projection
// have other K than the rest of their stage), of ResNet-50 at 256 samples
//   M = 802,816 N = 256    K =  64 167 / 102 and 344 / 265     K = 128 join 389 / 282
//   M = 200,704 N = 512    K = 128 95 / 68 and 199 / 133       K = 256 join 237 / 151      N = 256 K = 512 forward 104 / 77
//   M = 50,176  N = 1,024  K = 256 59 / 48 and 128 / 79        K = 512 join 164 / 104
//   M = 12,544  N = 2,048  K = 512 48 / 41 and 93 / 61
// at 32 samples
//   M = 100,352 N = 256    K =  64 24.2 / 19.3 and 47.1 / 35.1    K = 128 join 55.0 / 38.5
//   M = 25,088  N = 512    K = 128 19.7 / 17.3 and 30.8 / 24.5    K = 256 join 36.6 / 29.0
// and there below the line
//   M = 6,272   N = 1,024  K = 256 15.8 / 16.6    joins of K = 256 and 512 together 24.3 / 22.6
//   M = 1,568   N = 2,048  K = 512 15.0 / 18.8 and 19.8 / 21.3    M = 25,088 N = 256 K = 512 forward 22.9 / 23.8
bool pointwise_takes(int dtype, const ConvGeom& g, int plan_samples, int K, int N) {
    const int64_t M = (int64_t)plan_samples * g.H * g.W;
    return dtype == 1 && g.R == 1 && g.S == 1 && g.stride == 1 && g.pad == 0 && (K == 64 || K == 128 || K == 256 || K == 512) &&
           N % kCols == 0 && M * (N / kCols) >= tune().pointwise_rows;
}

template <bool JOIN>
static void launch(int K, const PointwiseArgs& a, hipStream_t st) {
    const dim3 grid(a.gx * a.gy);
    if (K == 64) hipLaunchKernelGGL((pointwise_kernel<64, 4, 2, JOIN>), grid, dim3(256), 0, st, a);
    else if (K == 128) hipLaunchKernelGGL((pointwise_kernel<128, 8, 2, JOIN>), grid, dim3(512), 0, st, a);
    else if (K == 256) hipLaunchKernelGGL((pointwise_kernel<256, 8, 1, JOIN>), grid, dim3(512), 0, st, a);
    else hipLaunchKernelGGL((pointwise_kernel<512, 8, 1, JOIN>), grid, dim3(512), 0, st, a);
}

bool launch_pointwise(const ConvGeom& g, const ShardSet& S, const PointwiseTask& t, RowCut* left, hipStream_t st) {
    PointwiseArgs a = {};
    a.A = (const bf16_t*)t.A; a.B = (const bf16_t*)t.B; a.out = (bf16_t*)t.out;
    a.N = t.N;
    a.cut = cut_rows(S, g.H * g.W, rows_per_run((int64_t)S.plan * g.H * g.W, t.K, t.N));
    a.gx = a.cut.blk0[a.cut.p]; a.gy = t.N / kCols;
    const bool sums = t.sums.buf != nullptr && t.sums.floats >= (size_t)2 * t.N * a.gx;
    if (t.join && !sums) return false;
    a.sums = sums ? t.sums.buf : nullptr;
    const double M = (double)S.samples() * g.H * g.W;
    const double bytes = 2.0 * (M * (t.K + t.N) + (double)t.N * t.K) + (t.join ? M * t.N * (2.0 + 2.0 + 1.0 / 8) : 0.0);
    ProfScope ps(prof_shape_label(t.join ? "pointwise_join" : "pointwise_fwd", (int64_t)M, t.N), 2.0 * M * t.N * t.K, bytes, st);
    if (t.join) {
        a.old = (const bf16_t*)t.old; a.sign = t.sign; a.xin = (const bf16_t*)t.xin; a.mean_rstd = t.mean_rstd;
        launch<true>(t.K, a, st);
    } else {
        launch<false>(t.K, a, st);
    }
    *left = sums ? a.cut : RowCut();
    return true;
}

}  // namespace edl
