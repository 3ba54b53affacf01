// 3x3 convolutions of stride 1 with as many channels out as in, 16, 32 or 64, in float32 (the layers of a small residual net),
// forward and input gradient.  Such a launch has 0.6 GFLOP and 4 to 17 MB, 4 us of either, and took 13 to 23: tiles of 32
// columns are half empty at 16 channels, at 64 the reduction was cut over workgroups with a second launch to add the pieces, and
// a chain of reduction steps each waited for its loads.  Here a workgroup has 2,048 / C pixels and all of their outputs:
//   * its pixels' neighbourhood, three runs of pixels (one per kernel row, zeros outside the image), goes into LDS at once, each
//     lane's loads in flight together, the weights beside them into registers for the whole kernel: one wait, one barrier;
//   * a wave owns 16 of the outputs for two tiles of 16 pixels (v_mfma_f32_16x16x4_f32, none of it empty); a lane's 16 bytes
//     from LDS feed four of them;
//   * sums in chains of 32 to 64 products, which a second set adds up (the error against float64 is 0.8 to 0.98 of the tiled
//     kernel's);
//   * the weights are the first operand, so that a lane ends with four channels of a pixel: 16-byte stores, and the epilogue's
//     operands (fetched with the pixels) in the same shape.
// Measured (pixels x channels, forward / input gradient with mask and sums, with the events' 2 us): 131,072 x 16: 20.8 / 24.5 us
// before, 14.8 / 16.2 now; 32,768 x 32: 15.2 / 15.8 and 14.8 / 15.9; 8,192 x 64: 17.7 and 7.7 for the second launch, 17.1 now.
#include "dev_common.h"
#include "magic.h"
#include "narrow.h"
#include "profiler.h"
#include "tune.h"

namespace edl {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

struct NarrowArgs {
    const float *x, *w;
    float* y;
    const float *old, *act, *xin, *mean_rstd;     // act, xin: see DgradMask; mean_rstd of shard s at 2 * C * s
    float* sums;                                  // [2][C][blocks] or null
    int H, W, flip, gx;
    unsigned long long magic_hw, magic_w;         // magic_of
    unsigned bytes;                               // of x
    RowCut cut;
};

constexpr unsigned kOutside = 0x80000000u;        // (x is smaller than 2 GiB)
constexpr int kNarrowTiles = 2;                   // tiles of 16 pixels per wave

// where the 16-byte chunk of a pixel's row lies: 16 neighbouring pixels' same chunk falls into different banks
template <int C> __device__ __forceinline__ int narrow_chunk(int row, int chunk) {
    return chunk ^ (C == 16 ? (row >> 2) & 3 : C == 32 ? (row >> 1) & 7 : row & 15);
}

template <int C>
__global__ __launch_bounds__(256, 2) void narrow_kernel(NarrowArgs a) {
    constexpr int BM = 2048 / C, CH = C / 4, STRIP = BM + 2, ROWS = STRIP + 1;     // pixels, chunks per pixel, pixels of a run (one more: zeros)
    constexpr int VECS = STRIP * CH, IT = (VECS + 255) / 256, CG = C / 16, GROUPS = 4 / CG, RUN = ROWS * C * 4;      // of one run: vectors, per lane, bytes
    struct __attribute__((packed, aligned(4))) Four { float v[4]; };
    __shared__ __attribute__((aligned(256))) unsigned char strip[3 * RUN];
    static_assert(RUN % (C * 4) == 0, "rows of a run lie on multiples of their size");
    static_assert(GROUPS * kNarrowTiles * 16 == BM, "the waves cover the pixels");
    __shared__ float red[4][2][16];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    int bx = blockIdx.x;
    {   // a die gets a contiguous run of blocks
        const int q = a.gx >> 3, r = a.gx & 7, die = bx & 7, slot = bx >> 3;
        bx = die * q + (die < r ? die : r) + slot;
    }
    int m0, m_end;
    const int shard = locate_block(a.cut, bx, m0, m_end);
    const int W = a.W, hw = a.H * W, M = a.cut.row0[a.cut.p];
    const int kt = wave % CG, pg = wave / CG;     // this wave's outputs and group of pixels
    const int slice = lane >> 4, l16 = lane & 15;

    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(a.x), 0, a.bytes, 0x00020000);
    u32x4 in[IT][3];
    int to[IT];
    #pragma unroll
    for (int i = 0; i < IT; ++i) {
        const int v = tid + i * 256, row = v / CH, chunk = v % CH, pix = m0 - 1 + row;
        const int rem = pix - (int)(((unsigned long long)(unsigned)pix * a.magic_hw) >> 40) * hw, h = (int)(((unsigned long long)(unsigned)rem * a.magic_w) >> 40);
        const bool ok = v < VECS && pix >= 0 && pix < M;
        const unsigned off = ((unsigned)pix * C + chunk * 4) * 4u, line = (unsigned)W * C * 4u;
        in[i][0] = __builtin_amdgcn_raw_buffer_load_b128(rx, ok && h > 0 ? off - line : kOutside, 0, 0);
        in[i][1] = __builtin_amdgcn_raw_buffer_load_b128(rx, ok ? off : kOutside, 0, 0);
        in[i][2] = __builtin_amdgcn_raw_buffer_load_b128(rx, ok && h + 1 < a.H ? off + line : kOutside, 0, 0);
        to[i] = v < VECS ? row * (C * 4) + narrow_chunk<C>(row, chunk) * 16 : -1;
    }
    floatx4 wf[9][CG];
    {
        const float* const wp = a.w + (size_t)(kt * 16 + l16) * 9 * C + slice * 4;
        #pragma unroll
        for (int t = 0; t < 9; ++t)
            #pragma unroll
            for (int g = 0; g < CG; ++g) {
                const Four f = *reinterpret_cast<const Four*>(wp + (a.flip ? 8 - t : t) * C + g * 16);
                wf[t][g] = floatx4{f.v[0], f.v[1], f.v[2], f.v[3]};
            }
    }
    // this lane's pixels, and where their neighbours lie in a run (the run of zeros past the image's sides)
    int pix[kNarrowTiles], at[kNarrowTiles][3];
    bool live[kNarrowTiles];
    floatx4 old[kNarrowTiles], act[kNarrowTiles], xin[kNarrowTiles];
    const int k0 = kt * 16 + slice * 4;
    #pragma unroll
    for (int t = 0; t < kNarrowTiles; ++t) {
        const int pl = (pg * kNarrowTiles + t) * 16 + l16;
        const int line = (int)(((unsigned long long)(unsigned)(m0 + pl) * a.magic_w) >> 40), col = m0 + pl - line * W;       // (rows of all images)
        pix[t] = m0 + pl;
        live[t] = pix[t] < m_end;
        #pragma unroll
        for (int s = 0; s < 3; ++s) {
            const int row = col + s - 1 >= 0 && col + s - 1 < W ? pl + s : STRIP;
            at[t][s] = row * (C * 4) + narrow_chunk<C>(row, slice) * 16;       // (the chunk of group g: the same with bits of g flipped)
        }
        const size_t o = live[t] ? (size_t)pix[t] * C + k0 : (size_t)k0;       // (the tensors' start is read and not used)
        if (a.old != nullptr) old[t] = *reinterpret_cast<const floatx4*>(a.old + o);
        if (a.act != nullptr) {
            act[t] = *reinterpret_cast<const floatx4*>(a.act + o);
            xin[t] = *reinterpret_cast<const floatx4*>(a.xin + o);
        }
    }
    #pragma unroll
    for (int i = 0; i < IT; ++i)
        if (to[i] >= 0)
            #pragma unroll
            for (int r = 0; r < 3; ++r) *reinterpret_cast<u32x4*>(strip + r * RUN + to[i]) = in[i][r];
    if (tid < 3 * CH) *reinterpret_cast<u32x4*>(strip + (tid / CH) * RUN + STRIP * (C * 4) + (tid % CH) * 16) = u32x4{0u, 0u, 0u, 0u};
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __syncthreads();

    floatx4 acc[kNarrowTiles], sum[kNarrowTiles];
    #pragma unroll
    for (int t = 0; t < kNarrowTiles; ++t) acc[t] = sum[t] = floatx4{0.f, 0.f, 0.f, 0.f};
    #pragma unroll
    for (int tap = 0; tap < 9; ++tap) {
        const int r = tap / 3, s = tap % 3;
        #pragma unroll
        for (int g = 0; g < CG; ++g)
            #pragma unroll
            for (int t = 0; t < kNarrowTiles; ++t) {
                const floatx4 x = *reinterpret_cast<const floatx4*>(strip + r * RUN + (at[t][s] ^ (g * 64)));
                #pragma unroll
                for (int e = 0; e < 4; ++e) acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(wf[tap][g][e], x[e], acc[t], 0, 0, 0);
            }
        if (C >= 32 || s == 2)
            #pragma unroll
            for (int t = 0; t < kNarrowTiles; ++t) {
                sum[t] += acc[t];
                acc[t] = floatx4{0.f, 0.f, 0.f, 0.f};
            }
    }

    float mu[4], rs[4], s1[4], s2[4];
    #pragma unroll
    for (int e = 0; e < 4; ++e) { mu[e] = rs[e] = s1[e] = s2[e] = 0.f; }
    if (a.act != nullptr) {
        const float* const ms = a.mean_rstd + (size_t)shard * 2 * C + k0;
        #pragma unroll
        for (int e = 0; e < 4; ++e) { mu[e] = ms[e]; rs[e] = ms[C + e]; }
    }
    // lane: pixel l16 of each tile, outputs k0 .. k0 + 3
    #pragma unroll
    for (int t = 0; t < kNarrowTiles; ++t) {
        floatx4 v = sum[t];
        if (!live[t]) continue;
        if (a.old != nullptr) v += old[t];
        if (a.act != nullptr) {
            #pragma unroll
            for (int e = 0; e < 4; ++e) {
                v[e] = act[t][e] > 0.f ? v[e] : 0.f;
                s1[e] += v[e];
                s2[e] += v[e] * ((xin[t][e] - mu[e]) * rs[e]);
            }
        } else {
            #pragma unroll
            for (int e = 0; e < 4; ++e) { s1[e] += v[e]; s2[e] += v[e] * v[e]; }
        }
        *reinterpret_cast<floatx4*>(a.y + (size_t)pix[t] * C + k0) = v;
    }
    if (a.sums == nullptr) return;
    #pragma unroll
    for (int e = 0; e < 4; ++e) {
        #pragma unroll
        for (int d = 1; d < 16; d <<= 1) {
            s1[e] += __shfl_xor(s1[e], d, 64);
            s2[e] += __shfl_xor(s2[e], d, 64);
        }
        if (l16 == 0) { red[wave][0][slice * 4 + e] = s1[e]; red[wave][1][slice * 4 + e] = s2[e]; }
    }
    __syncthreads();
    if (tid >= 2 * C) return;
    const int kind = tid / C, k = tid % C;
    float s = 0.f;
    #pragma unroll
    for (int p = 0; p < GROUPS; ++p) s += red[p * CG + (k >> 4)][kind][k & 15];
    a.sums[(size_t)(kind * C + k) * a.gx + bx] = s;
}

static int narrow_rows(int C) { return 2048 / C; }

// 16 channels always (the step of ResNet-20, 256 to 512 images of 32x32 to 40x40: 2,239 to 4,854 us without, 2,131 to 4,526
// with).  32 and 64 up to 600 workgroups: each loads all the weights (147 KB at 64 channels), which long launches of tiles share
// better (512 images: 2,964 us without, 3,053 and 3,094 with those of 32 and of 64; 8 images: 942 without, 875 and 849 with).
bool narrow_takes(int dtype, const ConvGeom& g, const ShardSet& S) {
    const int C = g.C;
    if (dtype == 1 || g.R != 3 || g.S != 3 || g.stride != 1 || g.pad != 1 || g.K != C || tune().force_tile >= 0 || tune().narrow_blocks == 0) return false;
    if (C != 16 && C != 32 && C != 64) return false;
    const int64_t M = (int64_t)S.plan * g.H * g.W;
    // (the kernel divides the numbers of pixels, the last block's own among them, by H W and by W)
    const double last = (double)M + narrow_rows(C);
    return (C == 16 || M / narrow_rows(C) + S.plan_p <= tune().narrow_blocks) && M * C * 4 < 2147483648ll &&
           magic_fits(last, g.H * g.W) && magic_fits(last, g.W);
}

RowCut launch_narrow(const ConvGeom& g, const ShardSet& S, const NarrowTask& t, hipStream_t st) {
    NarrowArgs a = {};
    a.x = t.x; a.w = t.w; a.y = t.y; a.old = t.old;
    const int C = g.C;
    a.H = g.H; a.W = g.W; a.flip = t.flip;
    a.cut = cut_rows(S, g.H * g.W, narrow_rows(C));
    a.gx = a.cut.blk0[a.cut.p];
    const double M = (double)S.samples() * g.H * g.W;
    a.bytes = (unsigned)(M * C * 4);
    a.magic_hw = magic_of(g.H * g.W);
    a.magic_w = magic_of(g.W);
    const bool sums = t.sums.buf != nullptr && t.sums.floats >= (size_t)2 * C * a.gx && (!t.flip || t.mask != nullptr);
    if (sums) a.sums = t.sums.buf;
    if (sums && t.mask != nullptr) {
        a.act = (const float*)t.mask->act; a.xin = (const float*)t.mask->xin; a.mean_rstd = t.mask->mean_rstd;
    }
    ProfScope ps(prof_shape_label(t.flip ? "narrow_dgrad" : "narrow_fwd", (int64_t)M, C), 18.0 * M * C * C,
                 4.0 * C * (M * (2.0 + (t.old != nullptr) + 2.0 * (a.act != nullptr)) + 9.0 * C), st);
    const dim3 grid(a.gx);
    if (C == 16) hipLaunchKernelGGL(narrow_kernel<16>, grid, dim3(256), 0, st, a);
    else if (C == 32) hipLaunchKernelGGL(narrow_kernel<32>, grid, dim3(256), 0, st, a);
    else hipLaunchKernelGGL(narrow_kernel<64>, grid, dim3(256), 0, st, a);
    return sums ? a.cut : RowCut();
}

}  // namespace edl
