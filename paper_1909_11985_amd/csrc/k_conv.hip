// Implicit-GEMM convolution on the matrix cores: forward, input gradient and
// weight gradient of a channels-last convolution (a fully connected layer is
// the 1x1 case on a 1x1 image).  These are the "computation-intensive
// kernels such as matrix multiplication" of the paper's section 2.1.
//
// All three are Out[M][Nn] = sum_kk A[m][kk] * B[j][kk] with different gathers:
//
//   forward   M = N*Ho*Wo pixels   Nn = K      kk = (r,s,c)   A = x gathered, B = w[K][R][S][C]
//   dgrad     M = N*H*W   pixels   Nn = C      kk = (r,s,k)   A = dy gathered, B = wT[C][R][S][K]
//   wgrad     M = K               Nn = R*S*C   kk = pixel     A = dy^T, B = x^T gathered
//
// A workgroup of 4 waves owns a BM x BN output tile and walks the reduction in
// tiles of BK elements (eight 16-byte vectors per row).  Each wave feeds 32x32
// MFMA tiles from 16-byte fragments: one v_mfma_f32_32x32x16_bf16 per fragment
// pair for bf16, four v_mfma_f32_32x32x2_f32 for float32 (lane L of a fragment
// holds row L%32 and the reduction slice selected by L/32; both operands use
// the same slice order, so any order is a valid contraction).
//
//  * loads: 16-byte buffer loads whose range check returns zeros, so padding
//    taps, ragged edges and the reduction tail need no branch.  The vector
//    kernel (FAST) sends them straight into LDS (buffer_load ... lds: lane L's
//    16 bytes land at M0 + 16*L), PF+1 LDS stages deep, with explicit vmcnt
//    waits and one barrier per tile; it has no element-wise path.  The float32
//    weight gradient, and a second, slow instantiation for operands that are
//    not vector-shaped, keep the register-staged path: their loads land in
//    registers while the previous tile is contracted, then go to the other of
//    two LDS stages.
//  * forward / dgrad tiles: rows of BK elements; on the direct path unpadded,
//    the 16-byte chunks of a row XOR-swizzled by the row index, otherwise padded
//    by one vector (conflict-free fragment reads either way).  Weight-gradient
//    tiles: the reduction index (the pixel) is the slow index in memory; bf16
//    tiles stay [pixel][channel] and are transposed on the way out of LDS
//    (ds_read_tr16_b64), float32 tiles are 32-bit words read one by one.
//  * dgrad of a strided convolution contracts, for each residue class of the
//    input pixel modulo the stride, only the taps that reach the class: one
//    launch for the four classes of stride 2, else one per class.
//  * epilogue: through LDS as float32, out as 16-byte vectors (bf16 packed by
//    the hardware conversion).
//  * long reductions of small problems, and every weight gradient, are cut
//    across workgroups; the float32 partial tiles are summed in split order by
//    a second kernel (no float atomics: results are bit-reproducible).
#include <algorithm>
#include <deque>
#include <string>

#include "dev_common.h"
#include "kernels.h"
#include "magic.h"
#include "narrow.h"
#include "pointwise.h"
#include "profiler.h"
#include "thin.h"
#include "tune.h"

// 1: LDS fragment reads run one fragment group ahead of the MFMAs (tiles of more than one MFMA per group;
// measured -6% on the 128x128 weight gradient, nothing on the others)
#ifndef EDL_FRAG_AHEAD
#define EDL_FRAG_AHEAD 1
#endif

// 1: the vector kernels of forward / dgrad load their tiles from global memory straight into LDS
// (16 bytes per lane, no register staging, PF + 1 LDS stages); 0: through registers, two stages
#ifndef EDL_DIRECT_LDS
#define EDL_DIRECT_LDS 1
#endif
// the same for the bf16 weight gradient
#ifndef EDL_DIRECT_WG
#define EDL_DIRECT_WG 1
#endif

namespace edl {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

struct ConvArgs {
    const void* A;
    const void* B;
    void* out;
    const float* bias;
    int N, H, W, C, K, R, S, stride, pad, Ho, Wo;
    int M, Nn, Kred;
    int relu, out_fp32, accumulate;
    int vecA, vecB;
    int ksplit;  // reduction elements per blockIdx.z
    int fold;    // FOLDED weight gradients and float32: most reduction elements that are summed in one chain
    unsigned bytesA, bytesB;  // extents of the two operands (for the range-checked vector loads)
    // dgrad of a strided convolution, per residue class of the input pixel
    // (h % stride, w % stride) = (ph, pw): only the taps r = r0, r0+stride, ...
    // (nr of them) and s = s0, ... (ns) reach such a pixel, so the reduction runs
    // over nr*ns*K instead of R*S*K.  Hc x Wc pixels per image are in the class.
    // For stride 1 (and the other modes): ph = pw = r0 = s0 = 0, nr = R, ns = S.
    int ph, pw, Hc, Wc, r0, s0, nr, ns;
    int ldb;     // fwd/dgrad: elements between consecutive rows of B
    float* partial;  // fwd/dgrad with a cut reduction: float32 [split][M][Nn] partial sums, else null
    // dgrad with accumulate: the gradient that is added to is read here (same shape and layout as the output;
    // null: from the output buffer itself).  Lets the first reader of a residual join take the shortcut's part
    // from where it already lies instead of from a copy.
    const void* acc_src;
    // fwd, vector path, whole reduction: if not null, the column sums of the stored output and of its
    // squares over this tile's rows go to stats[c * row tiles + row tile] and
    // stats[(Nn + c) * row tiles + row tile] (the layout of the batch-norm reduction's partial sums)
    float* stats;
    // dgrad, vector path, whole reduction, stride 1, not accumulating: the layer that produced this
    // convolution's input ends in a ReLU, and its backward starts with "gradient times (activation > 0)"
    // followed by per-channel sums of that.  With mask_act (the activation, same shape as the output) the
    // gradient is stored already masked, and its column sums over the tile's rows go to msum (the layout of
    // stats above): kind 0 = sum of the masked gradient; kind 1 = sum of masked gradient * (xin - mean) * rstd
    // if xin (the producing batch norm's input) and mean_rstd ([mean[Nn], rstd[Nn]]) are given, else unused.
    // mask_sign (bf16, may be null): the activation's sign, one bit per element, eight channels to a byte, which is
    // then read instead of the activation.
    const void* mask_act;
    const unsigned char* mask_sign;
    const void* xin;
    const float* mean_rstd;     // of shard s at 2 * Nn * s
    float* msum;
    // ceil(2^40 / d) for d = channels per tap and d = taps per kernel row: n / d == (n * magic) >> 40
    // for n * d < 2^40, which keeps the tap bookkeeping of the load loop free of branches
    unsigned long long magic_inner, magic_taps;
    // the same for d = pixels per image and d = pixels per image row of the row index's pixel grid
    // (output pixels in the forward pass, the residue class's input pixels in dgrad), and for the tile grid
    unsigned long long magic_hw, magic_w, magic_gx, magic_gy;
    int stride_shift;                  // dgrad vector path: log2 of the stride (a power of two there)
    // Tile grid (gx row tiles, gy column tiles, gz cuts of the reduction), launched
    // as gx*gy*gz workgroups in one dimension.  The hardware hands consecutive
    // workgroups to the eight dies in turn and each die has its own L2, so with
    // xcd_chunked the kernel gives every die one contiguous run of the tile
    // sequence; n_fastest chooses which operand the neighbours of a run share.
    int gx, gy, gz, xcd_chunked, n_fastest;
    // Several workers' shards in one launch (shards = cut.p > 1).  Forward / dgrad: the row tiles stay within a shard (tile_x
    // runs over the blocks of the cut), so that the epilogue's column sums are those of one shard; without sums the
    // rows are cut without regard to shards (cut.p == 1).  wgrad: the reduction (pixels) is cut per shard, splits
    // pieces each (tile_z = shard * splits + piece); piece z of the sum goes to out + z * zstride floats, or with
    // one piece per shard straight to the shard's gradient (zdirect: out + worker * zstride).
    int shards, splits, zdirect;
    long long zstride;
    int strip;      // forward / dgrad of 3x3, stride 1: the kernel whose steps are a kernel row's three taps (takes_strips)
    int brows;      // dgrad of a fully connected layer: B is the weights as they lie, [K][C] (conv_dgrad_reads_weights)
};

// The tables of a launch over several shards.  One shard takes kernels without them: the table look-ups (and the
// argument loads that they keep from being hoisted) cost 0.3 to 0.9 us per launch, 2% of a ResNet-50 step at a shard
// of 32.
struct ConvArgsShards : ConvArgs { RowCut cut; };
// The residue classes of a stride-2 input gradient in one launch.  Their row tiles take turns (a die gets a contiguous
// run of tiles, and the classes contract one to four taps); what differs between them replaces the fields of ConvArgs of
// the same names.
struct ConvClass {
    int ph, pw, Hc, Wc, r0, s0, nr, ns, M, Kred;
    unsigned long long magic_hw, magic_w, magic_taps;
};
struct ConvArgsClasses : ConvArgs { int classes; ConvClass cls[4]; };
// FOLDED: a weight gradient over shards (or one of them) whose pieces are summed in shorter chains (ConvArgs::fold); a kernel
// of its own because the second set of sums costs the 128x128 tile 64 registers and with them the place of a wave beside it
// (on all weight gradients: VGG-16 1.3%, AlexNet 2.7% slower).
enum LaunchKind { PLAIN, SHARDED, CLASSES, FOLDED };
template <int KIND> struct ArgsOf { typedef ConvArgs type; typedef const ConvArgs& use; };
template <> struct ArgsOf<SHARDED> { typedef ConvArgsShards type; typedef const ConvArgsShards& use; };
template <> struct ArgsOf<FOLDED> { typedef ConvArgsShards type; typedef const ConvArgsShards& use; };
template <> struct ArgsOf<CLASSES> { typedef ConvArgsClasses type; typedef ConvArgs use; };   // a copy, completed by the class


__device__ __forceinline__ int fast_div(int n, unsigned long long magic) {
    return (int)(((unsigned long long)(unsigned)n * magic) >> 40);
}

// (row tile, column tile, reduction cut) of this workgroup
__device__ __forceinline__ void tile_of_block(const ConvArgs& a, int& bx, int& by, int& bz) {
    const int total = a.gx * a.gy * a.gz;
    int l = blockIdx.x;
    if (a.xcd_chunked) {
        const int q = total >> 3, r = total & 7, die = l & 7, slot = l >> 3;
        l = die * q + (die < r ? die : r) + slot;   // die d owns q (+1 for d < r) consecutive tiles
    }
    const bool mg = a.magic_gx != 0;   // 0: the grid is too large for the multiply-shift division
    if (a.n_fastest) {
        const int t = mg ? fast_div(l, a.magic_gy) : l / a.gy;
        by = l - t * a.gy;
        bz = mg ? fast_div(t, a.magic_gx) : t / a.gx;
        bx = t - bz * a.gx;
    } else {
        const int t = mg ? fast_div(l, a.magic_gx) : l / a.gx;
        bx = l - t * a.gx;
        bz = mg ? fast_div(t, a.magic_gy) : t / a.gy;
        by = t - bz * a.gy;
    }
}


// 16-byte load through a buffer descriptor: an offset at or beyond the
// descriptor's extent returns zeros, so padding taps, ragged tile edges and
// the tail of the reduction need no branch and every load of a tile can be in
// flight at once.
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
constexpr unsigned kOutOfRange = 0x80000000u;   // operands are smaller than 2 GiB (checked by the launchers)

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* p, unsigned bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, bytes, 0x00020000);
}
// The same load, landing in LDS instead of registers: lane L's 16 bytes go to LDS byte address
// lds_wave_base + 16*L (lds_wave_base is wave-uniform and travels in M0); a lane whose offset is out of range
// writes zeros.  The instruction is issued from inline assembly, so the compiler does not know of the
// outstanding LDS write: the caller orders it against LDS reads with wait_vmcnt<> and a barrier, and no other
// code of the kernel may use M0.
typedef int i32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ i32x4 make_rsrc_words(const void* p, unsigned bytes) {
    const uint64_t a = (uint64_t)p;
    const i32x4 r = {(int)(uint32_t)a, (int)((uint32_t)(a >> 32) & 0xffffu), (int)bytes, 0x00020000};
    return r;
}
__device__ __forceinline__ void buffer_load16_to_lds(i32x4 rsrc, unsigned lds_wave_base, unsigned byte_offset) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
                 :: "s"(lds_wave_base), "v"(byte_offset), "s"(rsrc) : "memory");
}
// waits until at most N of this wave's vector-memory loads are outstanding (they complete in order)
template <int N> __device__ __forceinline__ void wait_vmcnt() {
    static_assert(N >= 0 && N < 64, "vmcnt is a 6-bit counter");
    asm volatile("s_waitcnt vmcnt(%0)" :: "n"(N) : "memory");
}

__device__ __forceinline__ uint4 buffer_load16(__amdgpu_buffer_rsrc_t r, unsigned byte_offset) {
    const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(r, byte_offset, 0, 0);
    return make_uint4(v.x, v.y, v.z, v.w);
}

template <typename T> struct Frag;
template <> struct Frag<bf16_t> {
    static __device__ __forceinline__ void mma(const uint4& a, const uint4& b, floatx16& c) {
        c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
    }
};
template <> struct Frag<float> {
    static __device__ __forceinline__ void mma(const uint4& a, const uint4& b, floatx16& c) {
        c = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.x), __uint_as_float(b.x), c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.y), __uint_as_float(b.y), c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.z), __uint_as_float(b.z), c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.w), __uint_as_float(b.w), c, 0, 0, 0);
    }
};

// bf16 wgrad tiles in LDS: row = pixel of the reduction step, WIDTH channels per row, no padding; the
// 16-channel (32-byte) chunks of a row are permuted by the row's low bits.  A transposing read (tr_frag) takes,
// per 32 lanes, two neighbouring chunks of four consecutive pixel rows; those eight 32-byte pieces must fall
// into the eight different 32-byte bank groups.  Rows of 256 bytes (WIDTH 128) all start at the same bank, so
// the row moves its chunk pair by two chunks per row (XOR with 2 * (pixel % 4); XOR with pixel % 4, as the
// narrower tiles use, would put the pairs of rows 0/1 and 2/3 on top of each other: measured as 11% of the
// kernel's time in LDS bank conflicts).  Rows of 128 and 64 bytes are already spread by their own offsets.
template <int WIDTH>
__device__ __forceinline__ int wg_swizzle(int pixel) {
    return WIDTH >= 128 ? ((pixel & 3) << 1) : WIDTH >= 64 ? (pixel & 3) : (pixel & (WIDTH / 16 - 1));
}
template <int WIDTH>
__device__ __forceinline__ int wg_lds_index(int pixel, int ch) {
    return pixel * WIDTH + ((((ch >> 4) ^ wg_swizzle<WIDTH>(pixel)) << 4) | (ch & 15));
}

// MFMA operand of a 32-channel tile for reduction pixels [p16 + 8*(lane/32), +8) from such an LDS tile.
// ds_read_tr16_b64 hands lane l of a 16-lane group element (l % 4) of the four 16-bit values read by
// lanes l/4, l/4 + 4, l/4 + 8, l/4 + 12 of the group (lane layout measured on gfx950).  With lane s
// reading pixel s/4, channels 4*(s%4)..+3 of a 16-channel chunk, lane l therefore receives channel l of
// the chunk for four consecutive pixels; two reads give the operand's eight.
typedef short shortx4 __attribute__((ext_vector_type(4)));
template <int WIDTH>
__device__ __forceinline__ uint4 tr_frag(const bf16_t* tile, int ch32, int p16, int lane) {
    const int ch = ch32 + ((lane >> 4) & 1) * 16 + 4 * (lane & 3);
    const int p0 = p16 + (lane >> 5) * 8 + ((lane & 15) >> 2);
    typedef shortx4 __attribute__((address_space(3))) * lds_ptr;
    const shortx4 r0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(tile + wg_lds_index<WIDTH>(p0, ch)));
    const shortx4 r1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(tile + wg_lds_index<WIDTH>(p0 + 4, ch)));
    const uint2 a = __builtin_bit_cast(uint2, r0), b = __builtin_bit_cast(uint2, r1);
    return make_uint4(a.x, a.y, b.x, b.y);
}

// context of one tile row for the pixel-indexed operand of forward / dgrad
struct RowCtx {
    int64_t base;
    int h0, w0;
    bool valid;
};

template <int MODE, bool FAST>
__device__ __forceinline__ RowCtx make_row(const ConvArgs& a, int m, int m_end) {
    RowCtx c;
    c.valid = m < m_end;
    if (MODE == CONV_FWD) {
        const int hw = a.Ho * a.Wo;
        const int n = FAST ? fast_div(m, a.magic_hw) : m / hw, rem = m - n * hw;
        const int ho = FAST ? fast_div(rem, a.magic_w) : rem / a.Wo, wo = rem - ho * a.Wo;
        c.h0 = ho * a.stride - a.pad;
        c.w0 = wo * a.stride - a.pad;
        c.base = (((int64_t)n * a.H + c.h0) * a.W + c.w0) * a.C;
    } else {
        const int hw = a.Hc * a.Wc;
        const int n = FAST ? fast_div(m, a.magic_hw) : m / hw, rem = m - n * hw;
        const int hq = FAST ? fast_div(rem, a.magic_w) : rem / a.Wc, wq = rem - hq * a.Wc;
        c.h0 = a.ph + hq * a.stride + a.pad;
        c.w0 = a.pw + wq * a.stride + a.pad;
        c.base = (int64_t)n * a.Ho * a.Wo * a.K;
    }
    return c;
}

// Element offset of A[m][.] at kernel tap (r,s), channel ch, for forward /
// dgrad; ok = the tap falls inside the image (and, for dgrad, on the stride grid).
template <int MODE>
__device__ __forceinline__ int64_t a_offset_tap(const ConvArgs& a, const RowCtx& c, int r, int s, int ch, bool& ok) {
    if (MODE == CONV_FWD) {
        const int h = c.h0 + r, w = c.w0 + s;
        ok = c.valid && (unsigned)h < (unsigned)a.H && (unsigned)w < (unsigned)a.W;
        return c.base + ((int64_t)r * a.W + s) * a.C + ch;
    } else {
        const int hn = c.h0 - r, wn = c.w0 - s;
        int ho = hn, wo = wn;
        bool on_grid = true;
        if (a.stride == 2) {
            ho = hn >> 1;
            wo = wn >> 1;
            on_grid = ((hn | wn) & 1) == 0;
        } else if (a.stride != 1) {
            ho = hn / a.stride;
            wo = wn / a.stride;
            on_grid = (ho * a.stride == hn) && (wo * a.stride == wn);
        }
        ok = c.valid && hn >= 0 && wn >= 0 && on_grid && ho < a.Ho && wo < a.Wo;
        return c.base + ((int64_t)ho * a.Wo + wo) * a.K + ch;
    }
}

// the same from a flat reduction index (used by the element-wise path only)
template <int MODE>
__device__ __forceinline__ int64_t a_offset(const ConvArgs& a, const RowCtx& c, int kk, bool& ok) {
    const int inner = MODE == CONV_FWD ? a.C : a.K;
    const int tap = kk / inner, ch = kk - tap * inner;
    int r, s;
    if (MODE == CONV_FWD) { r = tap / a.S; s = tap - r * a.S; }
    else { const int ri = tap / a.ns; r = a.r0 + ri * a.stride; s = a.s0 + (tap - ri * a.ns) * a.stride; }
    const int64_t off = a_offset_tap<MODE>(a, c, r, s, ch, ok);
    ok = ok && kk < a.Kred;
    return off;
}

// Vector-path byte offset for forward / dgrad in 32-bit arithmetic (operands
// are below 2 GiB there); tap_off is (r*W + s)*C + ch for the forward pass.
template <int MODE, typename T>
__device__ __forceinline__ unsigned a_voffset(const ConvArgs& a, const RowCtx& c, int r, int s, int ch, int tap_off, bool in_k) {
    if (MODE == CONV_FWD) {
        const int h = c.h0 + r, w = c.w0 + s;
        const bool ok = in_k & c.valid & ((unsigned)h < (unsigned)a.H) & ((unsigned)w < (unsigned)a.W);
        // the offset is formed unconditionally and pushed out of range by its top bit: a select between
        // the two would be compiled into a predicated region, which splits the loop's basic block
        return ((unsigned)((int)c.base + tap_off) * (unsigned)sizeof(T)) | (ok ? 0u : kOutOfRange);
    } else {
        // no branch on the stride (the loop this runs in must stay one basic block): the vector path is taken
        // for strides that are powers of two only.  Negative coordinates are discarded by `ok`.
        const int hn = c.h0 - r, wn = c.w0 - s;
        const int ho = hn >> a.stride_shift, wo = wn >> a.stride_shift;
        const bool on_grid = ((hn | wn) & (a.stride - 1)) == 0;
        const bool ok = in_k & c.valid & ((hn | wn) >= 0) & on_grid & (ho < a.Ho) & (wo < a.Wo);
        return ((unsigned)((int)c.base + (ho * a.Wo + wo) * a.K + ch) * (unsigned)sizeof(T)) | (ok ? 0u : kOutOfRange);
    }
}

// Row of the output matrix a tile row is stored to: the tile row itself, except
// for a residue class of a strided dgrad, whose rows are every stride-th pixel.
template <int MODE, bool FAST = false>
__device__ __forceinline__ int64_t out_row(const ConvArgs& a, int row) {
    if (MODE != CONV_DGRAD || a.stride == 1) return row;
    const int hw = a.Hc * a.Wc;
    const int n = FAST ? fast_div(row, a.magic_hw) : row / hw, rem = row - n * hw;
    const int hq = FAST ? fast_div(rem, a.magic_w) : rem / a.Wc, wq = rem - hq * a.Wc;
    return ((int64_t)n * a.H + a.ph + hq * a.stride) * a.W + a.pw + wq * a.stride;
}

// Tile storage in LDS
//   forward / dgrad: rows of BK reduction elements, padded by one 16-byte vector; a fragment is one
//                    16-byte read (row = lane%32, slice = lane/32).
//   wgrad:           32-bit words [reduction word][row], a word holding the reduction elements 2q, 2q+1
//                    of one row for bf16 (one element for float32); a fragment is four one-word reads,
//                    and the global vectors (channels innermost) go in without any 16-bit scatter.
// FAST: both operands take the 16-byte vector loads and the output width is a
// multiple of a vector, so the kernel has no element-wise paths at all (a
// run-time choice between the two inside the loop would force a wait after
// every load).
// TAPS = 3: 3x3 convolutions of stride 1 (forward and dgrad).  A reduction step is BK channels of the three taps of one
// kernel row: the pixels that the three taps of BM consecutive output pixels read are BM + 2 consecutive pixels, which are
// staged once (a strip) instead of three times, and each tap's fragments are read from the strip one row further on.
// Pixels above and below the image come in as zeros; where a row's neighbour to the left or right is outside the
// image its fragment is read from a row of zeros behind the strip.  What this saves is operand delivery (a 128x64 step
// of 96 elements loads 21 KB instead of 37 KB) and two of three barriers: VGG-16's 64-channel layers at 224x224, shard
// of 32: 278 -> 238 us forward, 362 -> 277 us dgrad (two launches each).
// BROWS: dgrad with B = the weights as they lie ([K][C]: the reduction is the slow index), for fully connected layers.
// B's tile is BK rows of BN channels, loaded and read (transposed on the way out of LDS) like the bf16 weight gradient's;
// the fragments hold the same elements in the same order as those of a transposed copy, so the bits are the same.
template <typename T, int MODE, int WM, int WN, int TM, int TN, int BK, bool FAST, int PF, int KIND, int TAPS = 1, bool BROWS = false>
__global__ __launch_bounds__(256, 2) void conv_igemm_kernel(typename ArgsOf<KIND>::type args) {   // at least two waves per SIMD: 256 registers
    typename ArgsOf<KIND>::use a = args;
    constexpr bool SHARDS = KIND == SHARDED || KIND == FOLDED;
    constexpr bool WG = MODE == CONV_WGRAD;
    constexpr int BM = WM * TM * 32, BN = WN * TN * 32;
    constexpr int VEC = Elem<T>::VEC;
    constexpr int KV = BK / VEC;                    // fwd/dgrad: vectors per tile row
    constexpr int KPD = sizeof(T) == 2 ? 2 : 1;     // wgrad: reduction elements per 32-bit word
    constexpr int KD = BK / KPD;                    // wgrad: words along the reduction
    constexpr int LDPA = BM + 8, LDPB = BN + 8;     // wgrad: words per reduction word-row
    constexpr int RVA = BM / VEC, RVB = BN / VEC;   // wgrad: channel vectors per pixel
    constexpr int TOT_A = WG ? KD * RVA : BM * KV;  // work items per tile (wgrad: KPD vectors each)
    constexpr int TOT_B = WG ? KD * RVB : BN * KV;
    constexpr bool STRIP = TAPS > 1;
    constexpr int STRIP_ROWS = BM + 16;             // BM + TAPS - 1 rounded up to the 16 rows that a wave's load fills
    constexpr int ITER_A = STRIP ? (STRIP_ROWS + 63) / 64 : (TOT_A + 255) / 256;
    constexpr int ITER_B = STRIP ? (TAPS * BN + 63) / 64 : (TOT_B + 255) / 256;
    constexpr int NRA = WG ? ITER_A * KPD : ITER_A, NRB = WG ? ITER_B * KPD : ITER_B;
    // wgrad in bf16 keeps its tiles as they are in memory, [pixel][channel], and transposes on the way out of
    // LDS (ds_read_tr16_b64, see tr_frag); float32 wgrad keeps words [pixel][channel] read one by one
    constexpr bool WGT = WG && sizeof(T) == 2;
    constexpr bool FRAG_AHEAD = EDL_FRAG_AHEAD != 0 && TM * TN > 1;
    // Tiles loaded straight into LDS: rows of BK elements without padding (RB = 64 or 128 bytes); a wave's load
    // instruction fills 64 consecutive 16-byte slots (whole rows), and the slot of chunk c of row r is
    // c ^ ((r / RPL) % KV) with RPL = rows per 256 bytes, which keeps the fragment reads conflict-free.
    constexpr int RB = BK * (int)sizeof(T), RPL = RB > 256 ? 1 : 256 / RB;
    constexpr bool DIRECT = EDL_DIRECT_LDS != 0 && FAST && !WG && (STRIP || (TOT_A % 256 == 0 && TOT_B % 256 == 0)) &&
                            (RB == 64 || RB == 128);
    // The bf16 weight gradient the same way: its tiles are rows of pixels as they are in memory, so a
    // wave's load fills whole pixel rows; item v is the 16-byte slot v % RV of pixel v / RV.
    constexpr bool DIRECT_WG = EDL_DIRECT_LDS != 0 && EDL_DIRECT_WG != 0 && FAST && WGT;
    constexpr int DA = DIRECT_WG ? BK * RVA / 256 : 1, DB = DIRECT_WG ? BK * RVB / 256 : 1;   // loads per tile
    static_assert(!DIRECT_WG || (BK * RVA % 256 == 0 && BK * RVB % 256 == 0), "whole waves of slots");
    constexpr bool DMA = DIRECT || DIRECT_WG;
    constexpr int NST = DMA ? PF + 1 : 2;            // LDS stages
    // Weight gradients with three stages (few workgroups, one per CU) issue a tile's loads between their MFMAs instead of all
    // at once before them: nobody else's MFMAs hide the address arithmetic there (128x128, ResNet-50 at a shard of 32: 27.1
    // -> 24.3 us).  Two stages lose 8 to 13% that way (the loads have one step to land), 128x64 tiles 6%.
    constexpr bool SPREAD = DIRECT_WG && NST >= 3 && TM == TN;
    constexpr int LDK = DIRECT ? BK : BK + VEC;
    static_assert(!STRIP || (DIRECT && RB == 64 && TAPS == 3), "strips are loaded straight into LDS");
    static_assert(!BROWS || (DIRECT && !STRIP && MODE == CONV_DGRAD && sizeof(T) == 2), "rows of weights are loaded straight into LDS");
    constexpr int A_STAGE = STRIP ? STRIP_ROWS * RB : WGT ? BK * BM * 2 : WG ? KD * LDPA * 4 : BM * LDK * (int)sizeof(T);   // bytes per LDS stage
    constexpr int B_STAGE = STRIP ? TAPS * BN * RB : WGT ? BK * BN * 2 : WG ? KD * LDPB * 4 : BN * LDK * (int)sizeof(T);
    // epilogue staging: the rows of one wave row, as float32
    constexpr int STAGE_ROWS = TM * 32, STAGE_LD = BN + 4;
    constexpr int TILE_BYTES = NST * (A_STAGE + B_STAGE);
    constexpr int STAGE_BYTES = STAGE_ROWS * STAGE_LD * 4;
    constexpr int SMEM_BYTES = TILE_BYTES > STAGE_BYTES ? TILE_BYTES : STAGE_BYTES;
    static_assert(WM * WN == 4, "four waves per workgroup");
    static_assert(256 % KV == 0 && 256 % RVA == 0 && 256 % RVB == 0, "per-thread column of the tile must be fixed");
    static_assert(!WG || KD == 32, "wgrad: four fragment groups of eight words");

    __shared__ __attribute__((aligned(16))) unsigned char smem[SMEM_BYTES];
    unsigned char* const As = smem;                  // [NST] stages
    unsigned char* const Bs = smem + NST * A_STAGE;

    const T* __restrict__ Ag = (const T*)a.A;
    const T* __restrict__ Bg = (const T*)a.B;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave / WN, wn = wave % WN;
    int tile_x, tile_y, tile_z;
    tile_of_block(a, tile_x, tile_y, tile_z);
    if constexpr (KIND == CLASSES) {
        const int t = tile_x / args.classes;
        const ConvClass& k = args.cls[tile_x - t * args.classes];
        tile_x = t;
        if (tile_x * BM >= k.M) return;
        a.ph = k.ph; a.pw = k.pw; a.Hc = k.Hc; a.Wc = k.Wc; a.r0 = k.r0; a.s0 = k.s0; a.nr = k.nr; a.ns = k.ns;
        a.M = k.M; a.Kred = k.Kred; a.ksplit = k.Kred;
        a.magic_hw = k.magic_hw; a.magic_w = k.magic_w; a.magic_taps = k.magic_taps;
    }
    const int n0 = tile_y * BN;
    int m0 = tile_x * BM, m_end = a.M;       // rows [m0, m_end) of the output
    int kbeg = tile_z * a.ksplit, kend = kbeg + a.ksplit;
    int shard = 0;
    if (!WG) {
        if constexpr (SHARDS) shard = locate_block(a.cut, tile_x, m0, m_end);
        if (kend > a.Kred) kend = a.Kred;
    } else {
        int last = a.Kred;
        if constexpr (SHARDS) {
            shard = tile_z / a.splits;
            kbeg = a.cut.row0[shard] + (tile_z - shard * a.splits) * a.ksplit;
            kend = kbeg + a.ksplit;
            last = a.cut.row0[shard + 1];
        }
        if (kend > last) kend = last;        // a short shard's last pieces may be empty: they store zeros
    }
    const int nk = (kend - kbeg + TAPS * BK - 1) / (TAPS * BK);

    Vec16<T> ra[PF][NRA], rb[PF][NRB];   // PF register sets: the loads of the next PF tiles are in flight
    const __amdgpu_buffer_rsrc_t rsrcA = make_rsrc(a.A, a.bytesA), rsrcB = make_rsrc(a.B, a.bytesB);
    const i32x4 wordsA = make_rsrc_words(a.A, a.bytesA), wordsB = make_rsrc_words(a.B, a.bytesB);
    // LDS byte address of the 64 slots this wave's first load of a tile fills (DIRECT)
    const unsigned lds_base = (unsigned)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem;
    const unsigned ldsA_wave = __builtin_amdgcn_readfirstlane(lds_base + wave * 1024);
    const unsigned ldsB_wave = ldsA_wave + NST * A_STAGE;

    // ---- per-thread state of the gathers; advanced by BK after every tile ------
    RowCtx rowA[WG ? 1 : ITER_A];
    int64_t offB[WG ? 1 : ITER_B];   // fwd/dgrad: start of the weight row
    bool okB[WG ? 1 : ITER_B];
    int tr = 0, ts = 0, tc = 0, tap_off = 0;   // fwd/dgrad: kernel tap and channel of this thread's vector
    int kcur = 0;                    // reduction index of this thread's vector (fwd/dgrad) or of the tile (wgrad)
    int brow = 0;                    // BROWS: row of the weights of this thread's first vector of B
    constexpr int NOA = DIRECT_WG ? DA : WG ? ITER_A : 1, NPB = DIRECT_WG ? DB : WG ? ITER_B : 1;
    int64_t offA[NOA];               // wgrad: offset of dy[first pixel of the item][first row of the item]
    int pn[NPB], pho[NPB], pwo[NPB]; // wgrad: first pixel of the item
    bool rowA_ok = true;             // wgrad, direct loads: this lane's channels of dy exist
    int wg_r = 0, wg_s = 0, wg_c = 0;  // wgrad: tap and channel of this thread's B rows
    bool wg_j_ok = true;
    int dn = 0, dho = 0, dwo = 0;    // wgrad: BK pixels as (images, rows, columns)
    // strips: byte offsets of this lane's vectors of A and B at kernel row 0, the kernel rows at which the vector of A is
    // inside the image (a bit each), kernel row and channel of the next step
    constexpr int SIA = STRIP ? ITER_A : 1, SIB = STRIP ? ITER_B : 1;
    // (unsigned: in the last image row of a tensor of nearly 2 GiB the offset at row 0 is past it until the row's term, modulo
    // 2^32, brings it back)
    unsigned strip_a[SIA], strip_b[SIB];
    int strip_in[SIA];
    int strip_r = 0, strip_c = 0;
    int strip_frag[STRIP ? TM : 1][TAPS];   // byte offset of this lane's fragment in the strip, by column shift
    if (STRIP) {
        const int inner = MODE == CONV_FWD ? a.C : a.K;
        const int step = kbeg / (TAPS * BK), per_row = inner / BK;
        strip_r = step / per_row;
        strip_c = (step - strip_r * per_row) * BK;
        const int slot = tid % KV;
        const int hw = MODE == CONV_FWD ? a.Ho * a.Wo : a.Hc * a.Wc, wd = a.W;
        #pragma unroll
        for (int it = 0; it < ITER_A; ++it) {
            const int row = (tid + it * 256) / KV, pix = m0 - 1 + row;
            const int chunk = slot ^ ((row / RPL) % KV);
            const int n = fast_div(pix, a.magic_hw), h = fast_div(pix - n * hw, a.magic_w);
            const bool ok = row < BM + TAPS - 1 && pix >= 0 && pix < a.M;     // (m_end is the tile's own end)
            int in = 0;
            #pragma unroll
            for (int r = 0; r < 3; ++r) {
                const int q = MODE == CONV_FWD ? h + r - 1 : h + 1 - r;
                in |= (ok && q >= 0 && q < a.H) ? 1 << r : 0;
            }
            strip_in[it] = in;
            strip_a[it] = ((unsigned)(pix + (MODE == CONV_FWD ? -wd : wd)) * (unsigned)inner + (unsigned)(chunk * VEC)) * (unsigned)sizeof(T);
        }
        #pragma unroll
        for (int it = 0; it < ITER_B; ++it) {
            const int row = (tid + it * 256) / KV, tap = row / BN, j = n0 + row - tap * BN;
            const int chunk = slot ^ ((row / RPL) % KV);
            strip_b[it] = (j < a.Nn && tap < TAPS) ? (unsigned)(j * a.ldb + tap * inner + chunk * VEC) * (unsigned)sizeof(T) : kOutOfRange;
        }
        #pragma unroll
        for (int i = 0; i < TM; ++i) {
            const int row = (wm * TM + i) * 32 + (lane & 31), pix = m0 + row;
            const int n = fast_div(pix, a.magic_hw), rem = pix - n * hw;
            const int w = rem - fast_div(rem, a.magic_w) * wd;
            #pragma unroll
            for (int d = 0; d < TAPS; ++d) {
                const int q = w + d - 1;
                const int sr = (q >= 0 && q < wd) ? row + d : BM + 8;   // a row past the strip is all zeros
                strip_frag[i][d] = sr * RB + (((lane >> 5) ^ ((sr / RPL) % KV)) * 16);
            }
        }
    } else if (!WG) {
        const int inner = MODE == CONV_FWD ? a.C : a.K;
        // DIRECT: the lane fills slot tid % KV of its rows, which holds chunk slot ^ ((row / RPL) % KV); a lane's
        // rows are 256 / KV apart, so this is the same chunk for all of them
        const int chunk = DIRECT ? ((tid % KV) ^ ((tid / KV / RPL) % KV)) : tid % KV;
        kcur = kbeg + chunk * VEC;
        const int tap = FAST ? fast_div(kcur, a.magic_inner) : kcur / inner;
        tc = kcur - tap * inner;
        if (MODE == CONV_FWD) {
            tr = FAST ? fast_div(tap, a.magic_taps) : tap / a.S;
            ts = tap - tr * a.S;
            tap_off = (tr * a.W + ts) * a.C + tc;
        } else {
            const int ri = FAST ? fast_div(tap, a.magic_taps) : (a.ns > 0 ? tap / a.ns : 0);
            tr = a.r0 + ri * a.stride;
            ts = a.s0 + (tap - ri * a.ns) * a.stride;
            tap_off = (tr * a.S + ts) * a.K + tc;      // position inside a row of the transposed weights
        }
        #pragma unroll
        for (int it = 0; it < ITER_A; ++it) rowA[it] = make_row<MODE, FAST>(a, m0 + (tid + it * 256) / KV, m_end);
        if (BROWS) {
            // slots as in the weight gradient below; a lane's rows are 256 / RVB apart, its channels the same in all
            const int pb = tid % RVB;
            const int j = n0 + ((((pb >> 1) ^ wg_swizzle<BN>(tid / RVB)) << 4) | ((pb & 1) << 3));
            brow = kbeg + tid / RVB;
            okB[0] = j < a.Nn;
            offB[0] = j;
        } else {
            #pragma unroll
            for (int it = 0; it < ITER_B; ++it) {
                const int j = n0 + (tid + it * 256) / KV;
                okB[it] = j < a.Nn && (tid + it * 256) < TOT_B;
                offB[it] = !FAST && a.brows ? j : (int64_t)j * a.ldb;
            }
        }
    } else if (DIRECT_WG) {
        // slot p of pixel row x holds the 8 channels starting at (((p >> 1) ^ wg_swizzle(x)) << 4) | ((p & 1) << 3)
        // (wg_lds_index); a lane's pixels are a multiple of 4 apart, so its channels are the same in all of them
        const int pa = tid % RVA, pb = tid % RVB;
        const int chA = ((((pa >> 1) ^ wg_swizzle<BM>(tid / RVA)) << 4) | ((pa & 1) << 3));
        const int chB = ((((pb >> 1) ^ wg_swizzle<BN>(tid / RVB)) << 4) | ((pb & 1) << 3));
        rowA_ok = m0 + chA < a.M;
        const int j0 = n0 + chB;
        const int tap = j0 / a.C;
        wg_c = j0 - tap * a.C;
        wg_r = tap / a.S;
        wg_s = tap - wg_r * a.S;
        const int hw = a.Ho * a.Wo;
        dn = BK / hw;
        dho = (BK - dn * hw) / a.Wo;
        dwo = BK - dn * hw - dho * a.Wo;
        #pragma unroll
        for (int it = 0; it < DA; ++it) offA[it] = (int64_t)(kbeg + (tid + it * 256) / RVA) * a.K + m0 + chA;
        #pragma unroll
        for (int it = 0; it < DB; ++it) {
            const int mm = kbeg + (tid + it * 256) / RVB;
            pn[it] = mm / hw;
            const int rem = mm - pn[it] * hw;
            pho[it] = rem / a.Wo;
            pwo[it] = rem - pho[it] * a.Wo;
        }
        wg_j_ok = j0 < a.Nn;
        kcur = kbeg;
    } else {
        const int j0 = n0 + (tid % RVB) * VEC;
        const int tap = j0 / a.C;
        wg_c = j0 - tap * a.C;
        wg_r = tap / a.S;
        wg_s = tap - wg_r * a.S;
        const int hw = a.Ho * a.Wo;
        dn = BK / hw;
        dho = (BK - dn * hw) / a.Wo;
        dwo = BK - dn * hw - dho * a.Wo;
        #pragma unroll
        for (int it = 0; it < ITER_A; ++it)
            offA[it] = (int64_t)(kbeg + ((tid + it * 256) / RVA) * KPD) * a.K + m0 + (tid % RVA) * VEC;
        #pragma unroll
        for (int it = 0; it < ITER_B; ++it) {
            const int mm = kbeg + ((tid + it * 256) / RVB) * KPD;
            pn[it] = mm / hw;
            const int rem = mm - pn[it] * hw;
            pho[it] = rem / a.Wo;
            pwo[it] = rem - pho[it] * a.Wo;
        }
        kcur = kbeg;
    }

    // Part `part` of `parts` of a tile's loads (the direct kernels); the last one advances to the next tile.
    auto load_part = [&](int set, int part, int parts) {
        constexpr int NA = STRIP || DIRECT ? ITER_A : DA, NB = STRIP || DIRECT ? ITER_B : DB;
        const auto mine = [&](int item) { return item * parts / (NA + NB) == part; };
        const bool last = part == parts - 1;
        if (STRIP) {
            const int inner = MODE == CONV_FWD ? a.C : a.K;
            const unsigned addA = (unsigned)((MODE == CONV_FWD ? strip_r : -strip_r) * a.W * inner + strip_c) * (unsigned)sizeof(T);
            const unsigned addB = (unsigned)(strip_r * TAPS * inner + strip_c) * (unsigned)sizeof(T);
            #pragma unroll
            for (int it = 0; it < ITER_A; ++it) {
                if (!mine(it)) continue;
                const unsigned off = (strip_a[it] + addA) | (((strip_in[it] >> strip_r) & 1) ? 0u : kOutOfRange);
                if ((it + 1) * 64 <= STRIP_ROWS || __builtin_amdgcn_readfirstlane(wave) < (STRIP_ROWS - it * 64) / 16)
                    buffer_load16_to_lds(wordsA, ldsA_wave + set * A_STAGE + it * 4096, off);
            }
            #pragma unroll
            for (int it = 0; it < ITER_B; ++it) {
                if (!mine(NA + it)) continue;
                if ((it + 1) * 64 <= TAPS * BN || __builtin_amdgcn_readfirstlane(wave) < (TAPS * BN - it * 64) / 16)
                    buffer_load16_to_lds(wordsB, ldsB_wave + set * B_STAGE + it * 4096, strip_b[it] + addB);
            }
            if (!last) return;
            strip_c += BK;
            const bool next = strip_c == inner;
            strip_c = next ? 0 : strip_c;
            strip_r += next ? 1 : 0;
        } else if (DIRECT) {
            // `set` is the LDS stage
            const bool in_k = kcur < kend;
            #pragma unroll
            for (int it = 0; it < ITER_A; ++it) {
                if (!mine(it)) continue;
                buffer_load16_to_lds(wordsA, ldsA_wave + set * A_STAGE + it * 4096,
                                     a_voffset<MODE, T>(a, rowA[it], tr, ts, tc, tap_off, in_k));
            }
            #pragma unroll
            for (int it = 0; it < ITER_B; ++it) {
                if (!mine(NA + it)) continue;
                if (BROWS) {
                    const int row = brow + it * (256 / RVB);
                    const unsigned off = ((unsigned)row * (unsigned)a.C + (unsigned)offB[0]) * (unsigned)sizeof(T);
                    buffer_load16_to_lds(wordsB, ldsB_wave + set * B_STAGE + it * 4096, off | ((okB[0] & (row < kend)) ? 0u : kOutOfRange));
                    continue;
                }
                const int boff = MODE == CONV_FWD ? kcur : tap_off;
                buffer_load16_to_lds(wordsB, ldsB_wave + set * B_STAGE + it * 4096,
                                     (okB[it] && in_k) ? (unsigned)((int)offB[it] + boff) * (unsigned)sizeof(T) : kOutOfRange);
            }
            if (!last) return;
            brow += BK;
            const int inner = MODE == CONV_FWD ? a.C : a.K;
            kcur += BK;
            const int tap = fast_div(kcur, a.magic_inner);
            tc = kcur - tap * inner;
            const int ri = fast_div(tap, a.magic_taps);
            if (MODE == CONV_FWD) {
                tr = ri;
                ts = tap - ri * a.S;
                tap_off = (tr * a.W + ts) * a.C + tc;
            } else {
                tr = a.r0 + ri * a.stride;
                ts = a.s0 + (tap - ri * a.ns) * a.stride;
                tap_off = (tr * a.S + ts) * a.K + tc;
            }
        } else if (DIRECT_WG) {
            // `set` is the LDS stage; pixel rows past the end of the reduction come in as zeros
            #pragma unroll
            for (int it = 0; it < DA; ++it) {
                if (!mine(it)) continue;
                const bool ok = rowA_ok & (kcur + (tid + it * 256) / RVA < kend);
                buffer_load16_to_lds(wordsA, ldsA_wave + set * A_STAGE + it * 4096,
                                     ((unsigned)(int)offA[it] * (unsigned)sizeof(T)) | (ok ? 0u : kOutOfRange));
                offA[it] += (int64_t)BK * a.K;
            }
            #pragma unroll
            for (int it = 0; it < DB; ++it) {
                if (!mine(NA + it)) continue;
                const int h = pho[it] * a.stride - a.pad + wg_r, w = pwo[it] * a.stride - a.pad + wg_s;
                const bool ok = wg_j_ok & (kcur + (tid + it * 256) / RVB < kend) & ((unsigned)h < (unsigned)a.H) &
                                ((unsigned)w < (unsigned)a.W);
                const unsigned off = (unsigned)(((pn[it] * a.H + h) * a.W + w) * a.C + wg_c) * (unsigned)sizeof(T);
                buffer_load16_to_lds(wordsB, ldsB_wave + set * B_STAGE + it * 4096, off | (ok ? 0u : kOutOfRange));
                // advance the item's pixel by BK
                int qw = pwo[it] + dwo, qh = pho[it] + dho, qn = pn[it] + dn;
                const bool cw = qw >= a.Wo;
                qw -= cw ? a.Wo : 0;
                qh += cw ? 1 : 0;
                const bool chh = qh >= a.Ho;
                qh -= chh ? a.Ho : 0;
                qn += chh ? 1 : 0;
                pwo[it] = qw; pho[it] = qh; pn[it] = qn;
            }
            if (last) kcur += BK;
        }
    };
    auto load_tiles = [&](int set) {
        if (DMA) {
            load_part(set, 0, 1);
        } else if (!WG) {
            const bool in_k = kcur < kend;
            #pragma unroll
            for (int it = 0; it < ITER_A; ++it) {
                ra[set][it].u = make_uint4(0, 0, 0, 0);
                if (TOT_A % 256 != 0 && tid + it * 256 >= TOT_A) continue;
                if (FAST || a.vecA) {
                    ra[set][it].u = buffer_load16(rsrcA, a_voffset<MODE, T>(a, rowA[it], tr, ts, tc, tap_off, in_k));
                } else {
                    #pragma unroll
                    for (int e = 0; e < VEC; ++e) {
                        bool ok;
                        const int64_t off = a_offset<MODE>(a, rowA[it], kcur + e, ok);
                        if (ok && kcur + e < kend) ra[set][it].e[e] = Ag[off];
                    }
                }
            }
            #pragma unroll
            for (int it = 0; it < ITER_B; ++it) {
                rb[set][it].u = make_uint4(0, 0, 0, 0);
                if (FAST || a.vecB) {
                    const int boff = MODE == CONV_FWD ? kcur : tap_off;
                    rb[set][it].u = buffer_load16(rsrcB, (okB[it] && in_k) ? (unsigned)((int)offB[it] + boff) * (unsigned)sizeof(T) : kOutOfRange);
                } else if (okB[it]) {
                    #pragma unroll
                    for (int e = 0; e < VEC; ++e) {
                        int boff = kcur + e;
                        if (MODE == CONV_DGRAD) {
                            const int tap = (kcur + e) / a.K, ri = a.ns > 0 ? tap / a.ns : 0;
                            boff = ((a.r0 + ri * a.stride) * a.S + a.s0 + (tap - ri * a.ns) * a.stride) * a.K + (kcur + e - tap * a.K);
                        }
                        if (kcur + e < kend) rb[set][it].e[e] = Bg[offB[it] + (a.brows ? (int64_t)boff * a.C : boff)];
                    }
                }
            }
            // advance this thread's vector by BK along (r, s, channel); no branches, so that the
            // loads issued above stay in flight across the following code
            const int inner = MODE == CONV_FWD ? a.C : a.K;
            kcur += BK;
            const int tap = fast_div(kcur, a.magic_inner);
            tc = kcur - tap * inner;
            const int ri = fast_div(tap, a.magic_taps);
            if (MODE == CONV_FWD) {
                tr = ri;
                ts = tap - ri * a.S;
                tap_off = (tr * a.W + ts) * a.C + tc;
            } else {
                tr = a.r0 + ri * a.stride;
                ts = a.s0 + (tap - ri * a.ns) * a.stride;
                tap_off = (tr * a.S + ts) * a.K + tc;
            }
        } else {
            #pragma unroll
            for (int it = 0; it < ITER_A; ++it) {
                const bool live = !(TOT_A % 256 != 0 && tid + it * 256 >= TOT_A);
                const int mm = kcur + ((tid + it * 256) / RVA) * KPD;
                const int row0 = m0 + (tid % RVA) * VEC;
                #pragma unroll
                for (int pp = 0; pp < KPD; ++pp) {
                    Vec16<T>& dst = ra[set][it * KPD + pp];
                    dst.u = make_uint4(0, 0, 0, 0);
                    const bool ok = live && mm + pp < kend;
                    if (FAST || a.vecA) {
                        dst.u = buffer_load16(rsrcA, (ok && row0 < a.M) ? (unsigned)((int)offA[it] + pp * a.K) * (unsigned)sizeof(T) : kOutOfRange);
                    } else if (ok) {
                        #pragma unroll
                        for (int e = 0; e < VEC; ++e)
                            if (row0 + e < a.M) dst.e[e] = Ag[offA[it] + (int64_t)pp * a.K + e];
                    }
                }
                offA[it] += (int64_t)BK * a.K;
            }
            #pragma unroll
            for (int it = 0; it < ITER_B; ++it) {
                const bool live = !(TOT_B % 256 != 0 && tid + it * 256 >= TOT_B);
                const int mm = kcur + ((tid + it * 256) / RVB) * KPD;
                int qn = pn[it], qho = pho[it], qwo = pwo[it];
                #pragma unroll
                for (int pp = 0; pp < KPD; ++pp) {
                    Vec16<T>& dst = rb[set][it * KPD + pp];
                    dst.u = make_uint4(0, 0, 0, 0);
                    const bool okp = live && mm + pp < kend;
                    const int hb = qho * a.stride - a.pad, wb = qwo * a.stride - a.pad;
                    if (FAST || a.vecB) {
                        const int j0 = n0 + (tid % RVB) * VEC;
                        const int h = hb + wg_r, w = wb + wg_s;
                        const bool ok = okp && j0 < a.Nn && (unsigned)h < (unsigned)a.H && (unsigned)w < (unsigned)a.W;
                        const unsigned off = (unsigned)(((qn * a.H + h) * a.W + w) * a.C + wg_c) * (unsigned)sizeof(T);
                        dst.u = buffer_load16(rsrcB, ok ? off : kOutOfRange);
                    } else if (okp) {
                        #pragma unroll
                        for (int e = 0; e < VEC; ++e) {
                            const int j = n0 + (tid % RVB) * VEC + e;
                            const int tap = j / a.C, ch = j - tap * a.C;
                            const int r = tap / a.S, s = tap - r * a.S;
                            const int h = hb + r, w = wb + s;
                            if (j < a.Nn && (unsigned)h < (unsigned)a.H && (unsigned)w < (unsigned)a.W)
                                dst.e[e] = Bg[(((int64_t)qn * a.H + h) * a.W + w) * a.C + ch];
                        }
                    }
                    // the next pixel of the pair
                    if (++qwo == a.Wo) { qwo = 0; if (++qho == a.Ho) { qho = 0; ++qn; } }
                }
                // advance the item's first pixel by BK
                pwo[it] += dwo;
                if (pwo[it] >= a.Wo) { pwo[it] -= a.Wo; ++pho[it]; }
                pho[it] += dho;
                if (pho[it] >= a.Ho) { pho[it] -= a.Ho; ++pn[it]; }
                pn[it] += dn;
            }
            kcur += BK;
        }
    };

    auto store_tiles = [&](int set, int buf) {
        if (!WG) {
            T* const Ad = reinterpret_cast<T*>(As + buf * A_STAGE);
            T* const Bd = reinterpret_cast<T*>(Bs + buf * B_STAGE);
            #pragma unroll
            for (int it = 0; it < ITER_A; ++it) {
                const int v = tid + it * 256;
                if (TOT_A % 256 != 0 && v >= TOT_A) continue;
                store_vec(&Ad[(v / KV) * LDK + (v % KV) * VEC], ra[set][it]);
            }
            #pragma unroll
            for (int it = 0; it < ITER_B; ++it) {
                const int v = tid + it * 256;
                if (TOT_B % 256 != 0 && v >= TOT_B) continue;
                store_vec(&Bd[(v / KV) * LDK + (v % KV) * VEC], rb[set][it]);
            }
        } else if (WGT) {
            bf16_t* const Ad = reinterpret_cast<bf16_t*>(As + buf * A_STAGE);
            bf16_t* const Bd = reinterpret_cast<bf16_t*>(Bs + buf * B_STAGE);
            #pragma unroll
            for (int it = 0; it < ITER_A; ++it) {
                const int v = tid + it * 256;
                if (TOT_A % 256 != 0 && v >= TOT_A) continue;
                #pragma unroll
                for (int pp = 0; pp < KPD; ++pp)
                    *reinterpret_cast<uint4*>(&Ad[wg_lds_index<BM>((v / RVA) * KPD + pp, (v % RVA) * VEC)]) = ra[set][it * KPD + pp].u;
            }
            #pragma unroll
            for (int it = 0; it < ITER_B; ++it) {
                const int v = tid + it * 256;
                if (TOT_B % 256 != 0 && v >= TOT_B) continue;
                #pragma unroll
                for (int pp = 0; pp < KPD; ++pp)
                    *reinterpret_cast<uint4*>(&Bd[wg_lds_index<BN>((v / RVB) * KPD + pp, (v % RVB) * VEC)]) = rb[set][it * KPD + pp].u;
            }
        } else {
            uint32_t* const Ad = reinterpret_cast<uint32_t*>(As + buf * A_STAGE);
            uint32_t* const Bd = reinterpret_cast<uint32_t*>(Bs + buf * B_STAGE);
            #pragma unroll
            for (int it = 0; it < ITER_A; ++it) {
                const int v = tid + it * 256;
                if (TOT_A % 256 != 0 && v >= TOT_A) continue;
                uint32_t* dst = &Ad[(v / RVA) * LDPA + (v % RVA) * VEC];
                if (KPD == 2) {
                    // word e = (pixel 2q, pixel 2q+1) of channel e
                    const uint16_t* p0 = reinterpret_cast<const uint16_t*>(&ra[set][it * KPD]);
                    const uint16_t* p1 = reinterpret_cast<const uint16_t*>(&ra[set][it * KPD + KPD - 1]);
                    uint4 lo, hi;
                    lo.x = p0[0] | ((uint32_t)p1[0] << 16); lo.y = p0[1] | ((uint32_t)p1[1] << 16);
                    lo.z = p0[2] | ((uint32_t)p1[2] << 16); lo.w = p0[3] | ((uint32_t)p1[3] << 16);
                    hi.x = p0[4] | ((uint32_t)p1[4] << 16); hi.y = p0[5] | ((uint32_t)p1[5] << 16);
                    hi.z = p0[6] | ((uint32_t)p1[6] << 16); hi.w = p0[7] | ((uint32_t)p1[7] << 16);
                    *reinterpret_cast<uint4*>(dst) = lo;
                    *reinterpret_cast<uint4*>(dst + 4) = hi;
                } else {
                    *reinterpret_cast<uint4*>(dst) = ra[set][it].u;
                }
            }
            #pragma unroll
            for (int it = 0; it < ITER_B; ++it) {
                const int v = tid + it * 256;
                if (TOT_B % 256 != 0 && v >= TOT_B) continue;
                uint32_t* dst = &Bd[(v / RVB) * LDPB + (v % RVB) * VEC];
                if (KPD == 2) {
                    const uint16_t* p0 = reinterpret_cast<const uint16_t*>(&rb[set][it * KPD]);
                    const uint16_t* p1 = reinterpret_cast<const uint16_t*>(&rb[set][it * KPD + KPD - 1]);
                    uint4 lo, hi;
                    lo.x = p0[0] | ((uint32_t)p1[0] << 16); lo.y = p0[1] | ((uint32_t)p1[1] << 16);
                    lo.z = p0[2] | ((uint32_t)p1[2] << 16); lo.w = p0[3] | ((uint32_t)p1[3] << 16);
                    hi.x = p0[4] | ((uint32_t)p1[4] << 16); hi.y = p0[5] | ((uint32_t)p1[5] << 16);
                    hi.z = p0[6] | ((uint32_t)p1[6] << 16); hi.w = p0[7] | ((uint32_t)p1[7] << 16);
                    *reinterpret_cast<uint4*>(dst) = lo;
                    *reinterpret_cast<uint4*>(dst + 4) = hi;
                } else {
                    *reinterpret_cast<uint4*>(dst) = rb[set][it].u;
                }
            }
        }
    };

    floatx16 acc[TM][TN];
    #pragma unroll
    for (int i = 0; i < TM; ++i)
        #pragma unroll
        for (int j = 0; j < TN; ++j)
            #pragma unroll
            for (int q = 0; q < 16; ++q) acc[i][j][q] = 0.f;
    // Two levels of sums: after at most a.fold elements the accumulators are added to `folded` and start again.  The
    // rounding error of a chain grows with its length, and a pass over several shards cuts each shard's reduction into
    // fewer, longer pieces than the shard alone.  Relative error of a shard's weight gradient against float64, alone / in a
    // pass in one chain / folded: ResNet-50's stem, 8 shards of 32, 4.9e-7 / 1.35e-6 / 4.6e-7; VGG-16's conv2, 4 of 16,
    // 5.3e-7 / 1.17e-6 / 5.1e-7; ResNet-20 in float32, 8 of 64, its 8x8 layers 2.2e-7 / 4.5e-7 / 2.0e-7, their outputs
    // 1.6e-7 / 2.9e-7 / 1.4e-7.  It costs the step of 8 shards of 32 0.2%, AlexNet's of 2 of 64 1.4%.
    constexpr bool FOLDS = KIND == FOLDED || (!WG && sizeof(T) == 4);
    floatx16 folded[FOLDS ? TM : 1][FOLDS ? TN : 1];
    if constexpr (FOLDS)
        #pragma unroll
        for (int i = 0; i < TM; ++i)
            #pragma unroll
            for (int j = 0; j < TN; ++j)
                #pragma unroll
                for (int q = 0; q < 16; ++q) folded[i][j][q] = 0.f;
    auto fold = [&]() {
        if constexpr (FOLDS)
            #pragma unroll
            for (int i = 0; i < TM; ++i)
                #pragma unroll
                for (int j = 0; j < TN; ++j) {
                    folded[i][j] += acc[i][j];
                    #pragma unroll
                    for (int q = 0; q < 16; ++q) acc[i][j][q] = 0.f;
                }
    };
    // tiles between folds: whole rounds of the LDS stages / register sets
    constexpr int ROUND = DMA ? NST : PF;
    const int chain = FOLDS ? (a.fold / (TAPS * BK) > ROUND ? a.fold / (TAPS * BK) / ROUND * ROUND : ROUND) : 0;

    // Software pipeline: two LDS stages and PF register sets.  While tile k is
    // contracted from LDS stage k%2, the global loads of tiles k+1 .. k+PF are in
    // flight; tile k+1 is moved from its registers to the other stage after the
    // MFMAs of tile k.  One barrier per tile.
    static_assert(DMA || PF == 1 || PF % 2 == 0, "the LDS stage of a tile must be known at compile time");
    // Loads past the end of the reduction are issued too: their offsets are out of
    // range, so they touch no memory and return zeros, and the number of loads in
    // flight at every wait is then a compile-time constant.
    // contraction of the tile in LDS stage `buf`
    auto contract = [&](int buf, auto&& between) {
        constexpr int NG = WG ? 4 : TAPS * BK / (2 * VEC);   // fragment groups per tile
        auto read_frags = [&](int g, uint4 (&fa)[TM], uint4 (&fb)[TN]) {
            if (STRIP) {
                constexpr int NT = NG / TAPS;
                static_assert(!STRIP || NT == 2, "two groups per tap");
                const int tap = g / NT, flip = (g - tap * NT) * 32, d = MODE == CONV_FWD ? tap : TAPS - 1 - tap;
                #pragma unroll
                for (int i = 0; i < TM; ++i)
                    fa[i] = *reinterpret_cast<const uint4*>(As + buf * A_STAGE + (strip_frag[STRIP ? i : 0][STRIP ? d : 0] ^ flip));
                const int slot = (lane >> 5) ^ (((lane & 31) / RPL) % KV);
                #pragma unroll
                for (int j = 0; j < TN; ++j)
                    fb[j] = *reinterpret_cast<const uint4*>(Bs + buf * B_STAGE + tap * BN * RB + ((((wn * TN + j) * 32 + (lane & 31)) * RB + slot * 16) ^ flip));
            } else if (!WG) {
                const T* const Ab = reinterpret_cast<const T*>(As + buf * A_STAGE);
                const T* const Bb = reinterpret_cast<const T*>(Bs + buf * B_STAGE);
                // chunk of the row this lane reads, and the slot the tile keeps it in
                const int chunk = 2 * g + (lane >> 5);
                const int slot = DIRECT ? (chunk ^ (((lane & 31) / RPL) % KV)) : chunk;
                #pragma unroll
                for (int i = 0; i < TM; ++i)
                    fa[i] = *reinterpret_cast<const uint4*>(&Ab[((wm * TM + i) * 32 + (lane & 31)) * LDK + slot * VEC]);
                #pragma unroll
                for (int j = 0; j < TN; ++j) {
                    if constexpr (BROWS) fb[j] = tr_frag<BN>(Bb, (wn * TN + j) * 32, g * 16, lane);
                    else fb[j] = *reinterpret_cast<const uint4*>(&Bb[((wn * TN + j) * 32 + (lane & 31)) * LDK + slot * VEC]);
                }
            } else if (WGT) {
                const bf16_t* const Ab = reinterpret_cast<const bf16_t*>(As + buf * A_STAGE);
                const bf16_t* const Bb = reinterpret_cast<const bf16_t*>(Bs + buf * B_STAGE);
                #pragma unroll
                for (int i = 0; i < TM; ++i) fa[i] = tr_frag<BM>(Ab, (wm * TM + i) * 32, g * 16, lane);
                #pragma unroll
                for (int j = 0; j < TN; ++j) fb[j] = tr_frag<BN>(Bb, (wn * TN + j) * 32, g * 16, lane);
            } else {
                const uint32_t* const Ab = reinterpret_cast<const uint32_t*>(As + buf * A_STAGE) + (g * 8 + (lane >> 5) * 4) * LDPA + (lane & 31);
                const uint32_t* const Bb = reinterpret_cast<const uint32_t*>(Bs + buf * B_STAGE) + (g * 8 + (lane >> 5) * 4) * LDPB + (lane & 31);
                #pragma unroll
                for (int i = 0; i < TM; ++i) {
                    const uint32_t* q = Ab + (wm * TM + i) * 32;
                    fa[i] = make_uint4(q[0], q[LDPA], q[2 * LDPA], q[3 * LDPA]);
                }
                #pragma unroll
                for (int j = 0; j < TN; ++j) {
                    const uint32_t* q = Bb + (wn * TN + j) * 32;
                    fb[j] = make_uint4(q[0], q[LDPB], q[2 * LDPB], q[3 * LDPB]);
                }
            }
        };
        // The fragments of group g+1 are read from LDS before the MFMAs of group g are issued
        // (the fences keep the compiler from sinking the reads back to their first use), so the
        // LDS latency of one group hides behind the matrix work of the one before.
        uint4 fa[2][TM], fb[2][TN];
        read_frags(0, fa[0], fb[0]);
        #pragma unroll
        for (int g = 0; g < NG; ++g) {
            if (g + 1 < NG) read_frags(g + 1, fa[(g + 1) & 1], fb[(g + 1) & 1]);
            if (FRAG_AHEAD) __builtin_amdgcn_sched_barrier(0);
            between(g, NG);
            #pragma unroll
            for (int i = 0; i < TM; ++i)
                #pragma unroll
                for (int j = 0; j < TN; ++j) Frag<T>::mma(fa[g & 1][i], fb[g & 1][j], acc[i][j]);
            if (FRAG_AHEAD) __builtin_amdgcn_sched_barrier(0);
        }
    };
    if (DMA) {
        // NST LDS stages filled by direct loads, no registers in between: while tile k is contracted from
        // stage k % NST, the loads of tiles k+1 .. k+NST-1 are in flight.  Per tile: wait until this wave's
        // loads of tile k have landed (loads complete in order, so all but those of the NST-2 younger tiles),
        // barrier (every wave's part of tile k is in LDS and every wave is done reading tile k-1), then
        // refill the stage tile k-1 was in.  Loads past the end of the reduction write zeros into a stage
        // nobody reads; all of them have landed before the epilogue reuses the memory.
        constexpr int PER_TILE = STRIP ? STRIP_ROWS / 64 + TAPS * BN / 64 : DIRECT_WG ? DA + DB : ITER_A + ITER_B;
        #pragma unroll
        for (int u = 0; u < NST - 1; ++u) load_tiles(u);
        for (int kt = 0;;) {
            const int stop = FOLDS && nk - kt > chain ? kt + chain : nk;
            for (; kt < stop; kt += NST) {
                #pragma unroll
                for (int u = 0; u < NST; ++u) {
                    if (kt + u >= nk) break;
                    wait_vmcnt<(NST - 2) * PER_TILE>();
                    __syncthreads();
                    if (!SPREAD) load_tiles((u + NST - 1) % NST);
                    contract(u, [&](int g, int groups) { if (SPREAD) load_part((u + NST - 1) % NST, g, groups); });
                }
            }
            if (!FOLDS || kt >= nk) break;
            fold();
        }
        wait_vmcnt<0>();
        __syncthreads();
    } else {
        #pragma unroll
        for (int u = 0; u < PF; ++u) load_tiles(u);
        store_tiles(0, 0);
        __syncthreads();
        for (int kt = 0;;) {
            const int stop = FOLDS && nk - kt > chain ? kt + chain : nk;
            for (; kt < stop; kt += PF) {
                #pragma unroll
                for (int u = 0; u < PF; ++u) {
                    const int k = kt + u;
                    if (k >= nk) break;
                    const int buf = PF == 1 ? (k & 1) : (u & 1);
                    load_tiles(u);
                    contract(buf, [](int, int) {});
                    store_tiles((u + 1) % PF, buf ^ 1);
                    __syncthreads();
                }
            }
            if (!FOLDS || kt >= nk) break;
            fold();
        }
    }
    if constexpr (FOLDS)
        #pragma unroll
        for (int i = 0; i < TM; ++i)
            #pragma unroll
            for (int j = 0; j < TN; ++j) acc[i][j] += folded[i][j];

    // ---- epilogue: lane holds column lane%32, rows (q/4)*8 + (lane/32)*4 + q%4 of each 32x32 tile ----
    constexpr bool OUT_F32 = WG || sizeof(T) == 4;       // element type of the vector-path output
    constexpr int OSZ = OUT_F32 ? 4 : 2;
    constexpr int OVEC = 16 / OSZ;
    int64_t zoff = 0;   // floats
    if (WG) {
        int z = tile_z;
        if constexpr (SHARDS) z = a.zdirect ? a.cut.k[shard] : tile_z;
        zoff = (int64_t)z * a.zstride;
    }
    if (!FAST) {
        // ragged width (or float32 logits from a bf16 net): element-wise stores
        #pragma unroll
        for (int i = 0; i < TM; ++i) {
            #pragma unroll
            for (int j = 0; j < TN; ++j) {
                const int col = n0 + (wn * TN + j) * 32 + (lane & 31);
                if (col >= a.Nn) continue;
                const float bias = (MODE == CONV_FWD && a.bias) ? a.bias[col] : 0.f;
                #pragma unroll
                for (int q = 0; q < 16; ++q) {
                    const int row = m0 + (wm * TM + i) * 32 + (q >> 2) * 8 + (lane >> 5) * 4 + (q & 3);
                    if (row >= m_end) continue;
                    float v = acc[i][j][q];
                    if (MODE == CONV_FWD) {
                        v += bias;
                        if (a.relu) v = v > 0.f ? v : 0.f;
                        const int64_t o = (int64_t)row * a.Nn + col;
                        if (a.out_fp32) ((float*)a.out)[o] = v;
                        else ((T*)a.out)[o] = Elem<T>::from_f32(v);
                    } else if (MODE == CONV_DGRAD) {
                        const int64_t o = out_row<MODE>(a, row) * a.Nn + col;
                        T* dst = (T*)a.out;
                        if (a.accumulate) v += Elem<T>::to_f32(a.acc_src ? ((const T*)a.acc_src)[o] : dst[o]);
                        dst[o] = Elem<T>::from_f32(v);
                    } else {
                        ((float*)a.out)[zoff + (int64_t)row * a.Nn + col] = v;
                    }
                }
            }
        }
        return;
    }
    // staged: one wave row at a time goes through LDS as float32 (one word per
    // lane and row, conflict-free), then leaves as 16-byte vectors along the output row
    float* const stage = reinterpret_cast<float*>(smem);
    unsigned char* const outp = (unsigned char*)a.out + zoff * 4;
    const unsigned char* const accp = (MODE == CONV_DGRAD && a.acc_src != nullptr) ? (const unsigned char*)a.acc_src : outp;
    const bool to_partial = !WG && a.partial != nullptr;     // cut reduction: raw float32 sums, finished by another kernel
    const bool f32_out = (MODE == CONV_FWD) && a.out_fp32 && !OUT_F32;
    // Every lane stores the same OVEC columns in each of its rows (256 is a multiple of the
    // vectors per row), so column sums of what it stored stay in registers until the end.
    const bool with_stats = MODE == CONV_FWD && a.stats != nullptr;
    float csum[OVEC], csq[OVEC];
    #pragma unroll
    for (int e = 0; e < OVEC; ++e) csum[e] = csq[e] = 0.f;
    constexpr int CV = BN / OVEC;                              // vectors per stored row
    constexpr int NV = (STAGE_ROWS * CV + 255) / 256;          // vectors per lane and pass
    const bool add_old = MODE == CONV_DGRAD && a.accumulate && !to_partial;
    const bool masked = MODE == CONV_DGRAD && a.mask_act != nullptr && !to_partial;
    const bool with_xhat = masked && a.xin != nullptr;
    const bool by_sign = !OUT_F32 && masked && a.mask_sign != nullptr;
    float mu[OVEC], rs[OVEC];      // of this lane's columns
    #pragma unroll
    for (int e = 0; e < OVEC; ++e) { mu[e] = 0.f; rs[e] = 0.f; }
    if (with_xhat) {
        const int c0 = n0 + (tid % CV) * OVEC;
        const float* const ms = a.mean_rstd + (SHARDS ? (int64_t)shard * 2 * a.Nn : 0);
        #pragma unroll
        for (int e = 0; e < OVEC; ++e)
            if (c0 + e < a.Nn) { mu[e] = ms[c0 + e]; rs[e] = ms[a.Nn + c0 + e]; }
    }
    #pragma unroll
    for (int pass = 0; pass < WM; ++pass) {
        // dgrad adding to an existing gradient: its vectors are fetched now, all at once and without a
        // branch (a vector outside the matrix reads the start of the tensor and is ignored), and are
        // there when the staged sums are
        uint4 oldv[NV];
        if (add_old) {
            #pragma unroll
            for (int k = 0; k < NV; ++k) {
                const int v = tid + k * 256, rl = v / CV, cv = v - rl * CV;
                const int row = m0 + pass * STAGE_ROWS + rl, col = n0 + cv * OVEC;
                const bool inside = v < STAGE_ROWS * CV && row < m_end && col < a.Nn;
                const unsigned char* src = inside ? accp + (out_row<MODE, true>(a, row) * a.Nn + col) * OSZ : accp;
                oldv[k] = *reinterpret_cast<const uint4*>(src);
            }
        }
        // the activation or its sign bits (and the batch norm's input) at the positions this lane stores, fetched the
        // same way
        uint4 actv[NV], xinv[NV];
        unsigned signv[NV];
        if (masked) {
            #pragma unroll
            for (int k = 0; k < NV; ++k) {
                const int v = tid + k * 256, rl = v / CV, cv = v - rl * CV;
                const int row = m0 + pass * STAGE_ROWS + rl, col = n0 + cv * OVEC;
                const bool inside = v < STAGE_ROWS * CV && row < m_end && col < a.Nn;
                const int64_t at = inside ? ((int64_t)row * a.Nn + col) * OSZ : 0;
                if (by_sign) signv[k] = a.mask_sign[at / 16];
                else actv[k] = *reinterpret_cast<const uint4*>((const unsigned char*)a.mask_act + at);
                if (with_xhat) xinv[k] = *reinterpret_cast<const uint4*>((const unsigned char*)a.xin + at);
            }
        }
        if (wm == pass) {
            #pragma unroll
            for (int i = 0; i < TM; ++i) {
                #pragma unroll
                for (int j = 0; j < TN; ++j) {
                    const int cl = (wn * TN + j) * 32 + (lane & 31);
                    const int col = n0 + cl;
                    const float bias = (MODE == CONV_FWD && a.bias && col < a.Nn) ? a.bias[col] : 0.f;
                    float* sp = stage + (i * 32 + (lane >> 5) * 4) * STAGE_LD + cl;
                    #pragma unroll
                    for (int q = 0; q < 16; ++q) {
                        float v = acc[i][j][q];
                        if (MODE == CONV_FWD && !to_partial) {
                            v += bias;
                            if (a.relu) v = fmaxf(v, 0.f);
                        }
                        sp[((q >> 2) * 8 + (q & 3)) * STAGE_LD] = v;
                    }
                }
            }
        }
        __syncthreads();
        #pragma unroll
        for (int k = 0; k < NV; ++k) {
            const int v = tid + k * 256;
            if (v >= STAGE_ROWS * CV) break;
            const int rl = v / CV, cv = v - rl * CV;
            const int row = m0 + pass * STAGE_ROWS + rl, col = n0 + cv * OVEC;
            if (row < m_end && col < a.Nn) {
                const float* sp = stage + rl * STAGE_LD + cv * OVEC;
                if (to_partial || f32_out) {
                    float* d = to_partial ? a.partial + ((int64_t)tile_z * a.M + row) * a.Nn + col
                                          : (float*)a.out + (int64_t)row * a.Nn + col;
                    #pragma unroll
                    for (int e = 0; e < OVEC; e += 4) *reinterpret_cast<float4*>(d + e) = *reinterpret_cast<const float4*>(sp + e);
                    continue;
                }
                unsigned char* dst = outp + (out_row<MODE, true>(a, row) * a.Nn + col) * OSZ;
                if (OUT_F32) {
                    float4 o = *reinterpret_cast<const float4*>(sp);
                    if (add_old) {
                        o.x += __uint_as_float(oldv[k].x); o.y += __uint_as_float(oldv[k].y);
                        o.z += __uint_as_float(oldv[k].z); o.w += __uint_as_float(oldv[k].w);
                    }
                    if (masked) {
                        const float am[4] = {__uint_as_float(actv[k].x), __uint_as_float(actv[k].y), __uint_as_float(actv[k].z), __uint_as_float(actv[k].w)};
                        o.x = am[0] > 0.f ? o.x : 0.f; o.y = am[1] > 0.f ? o.y : 0.f;
                        o.z = am[2] > 0.f ? o.z : 0.f; o.w = am[3] > 0.f ? o.w : 0.f;
                        const float gv[4] = {o.x, o.y, o.z, o.w};
                        const float xv[4] = {__uint_as_float(xinv[k].x), __uint_as_float(xinv[k].y), __uint_as_float(xinv[k].z), __uint_as_float(xinv[k].w)};
                        #pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            csum[e % OVEC] += gv[e];
                            if (with_xhat) csq[e % OVEC] += gv[e] * ((xv[e] - mu[e % OVEC]) * rs[e % OVEC]);
                        }
                    }
                    *reinterpret_cast<float4*>(dst) = o;
                    if (with_stats) {
                        csum[0] += o.x; csq[0] += o.x * o.x; csum[1] += o.y; csq[1] += o.y * o.y;
                        csum[2] += o.z; csq[2] += o.z * o.z; csum[3] += o.w; csq[3] += o.w * o.w;
                    }
                } else {
                    float4 o0 = *reinterpret_cast<const float4*>(sp), o1 = *reinterpret_cast<const float4*>(sp + 4);
                    if (add_old) {
                        const uint4 old = oldv[k];
                        o0.x += __uint_as_float(old.x << 16); o0.y += __uint_as_float(old.x & 0xffff0000u);
                        o0.z += __uint_as_float(old.y << 16); o0.w += __uint_as_float(old.y & 0xffff0000u);
                        o1.x += __uint_as_float(old.z << 16); o1.y += __uint_as_float(old.z & 0xffff0000u);
                        o1.z += __uint_as_float(old.w << 16); o1.w += __uint_as_float(old.w & 0xffff0000u);
                    }
                    if (by_sign) {
                        float* const ov[8] = {&o0.x, &o0.y, &o0.z, &o0.w, &o1.x, &o1.y, &o1.z, &o1.w};
                        #pragma unroll
                        for (int e = 0; e < 8; ++e)
                            if (!(signv[k] & (1u << e))) *ov[e] = 0.f;
                    } else if (masked) {   // activation > 0: a positive bf16 (sign clear, not zero)
                        const uint32_t aw[4] = {actv[k].x, actv[k].y, actv[k].z, actv[k].w};
                        float* const ov[8] = {&o0.x, &o0.y, &o0.z, &o0.w, &o1.x, &o1.y, &o1.z, &o1.w};
                        #pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            if (!(__uint_as_float(aw[e] << 16) > 0.f)) *ov[2 * e] = 0.f;
                            if (!(__uint_as_float(aw[e] & 0xffff0000u) > 0.f)) *ov[2 * e + 1] = 0.f;
                        }
                    }
                    uint4 pk;
                    pk.x = pack2_bf16(o0.x, o0.y); pk.y = pack2_bf16(o0.z, o0.w);
                    pk.z = pack2_bf16(o1.x, o1.y); pk.w = pack2_bf16(o1.z, o1.w);
                    *reinterpret_cast<uint4*>(dst) = pk;
                    if (masked) {   // sums of the stored (rounded) gradient
                        const uint32_t w4[4] = {pk.x, pk.y, pk.z, pk.w};
                        const uint32_t xw[4] = {xinv[k].x, xinv[k].y, xinv[k].z, xinv[k].w};
                        #pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const float lo = __uint_as_float(w4[e] << 16), hi = __uint_as_float(w4[e] & 0xffff0000u);
                            csum[(2 * e) % OVEC] += lo;
                            csum[(2 * e + 1) % OVEC] += hi;
                            if (with_xhat) {
                                const float xl = __uint_as_float(xw[e] << 16), xh = __uint_as_float(xw[e] & 0xffff0000u);
                                csq[(2 * e) % OVEC] += lo * ((xl - mu[(2 * e) % OVEC]) * rs[(2 * e) % OVEC]);
                                csq[(2 * e + 1) % OVEC] += hi * ((xh - mu[(2 * e + 1) % OVEC]) * rs[(2 * e + 1) % OVEC]);
                            }
                        }
                    }
                    if (with_stats) {   // of the rounded values, as a reader of the stored tensor would see them
                        const uint32_t w4[4] = {pk.x, pk.y, pk.z, pk.w};
                        #pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const float lo = __uint_as_float(w4[e] << 16), hi = __uint_as_float(w4[e] & 0xffff0000u);
                            csum[(2 * e) % OVEC] += lo; csq[(2 * e) % OVEC] += lo * lo;
                            csum[(2 * e + 1) % OVEC] += hi; csq[(2 * e + 1) % OVEC] += hi * hi;
                        }
                    }
                }
            }
        }
        __syncthreads();
    }
    if (with_stats || masked) {
        float* const sums = with_stats ? a.stats : a.msum;
        // lanes with the same column vector differ in tid / CV: sum over them in a fixed order
        constexpr int GROUPS = 256 / CV;
        static_assert(2 * GROUPS * BN * 4 <= SMEM_BYTES, "column sums fit the tile memory");
        float* const red = stage;
        const int grp = tid / CV, c0 = (tid % CV) * OVEC;
        #pragma unroll
        for (int e = 0; e < OVEC; ++e) {
            red[grp * BN + c0 + e] = csum[e];
            red[(GROUPS + grp) * BN + c0 + e] = csq[e];
        }
        __syncthreads();
        for (int c = tid; c < BN; c += 256) {
            if (n0 + c >= a.Nn) continue;
            float s1 = 0.f, s2 = 0.f;
            #pragma unroll 8
            for (int gq = 0; gq < GROUPS; ++gq) { s1 += red[gq * BN + c]; s2 += red[(GROUPS + gq) * BN + c]; }
            sums[(int64_t)(n0 + c) * a.gx + tile_x] = s1;
            sums[(int64_t)(a.Nn + n0 + c) * a.gx + tile_x] = s2;
        }
    }
}

// dw[i] = sum over a shard's splits, in split order.  One 16-byte vector per lane and
// split (the splits' loads are independent, so they are all in flight together).  grid: (elements, shards)
template <int VECW>
__global__ __launch_bounds__(256) void wgrad_reduce_kernel(const float* __restrict__ part, float* __restrict__ dw, int64_t dw_stride,
                                                           ShardSet S, int64_t n, int splits) {
    part += (int64_t)blockIdx.y * splits * n;
    dw += (int64_t)S.k[blockIdx.y] * dw_stride;
    const int64_t nv = n / VECW;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < nv; i += stride) {
        if (VECW == 4) {
            float4 s = reinterpret_cast<const float4*>(part)[i];
            int k = 1;
            for (; k + 3 < splits; k += 4) {
                const float4 t0 = reinterpret_cast<const float4*>(part + (int64_t)k * n)[i];
                const float4 t1 = reinterpret_cast<const float4*>(part + (int64_t)(k + 1) * n)[i];
                const float4 t2 = reinterpret_cast<const float4*>(part + (int64_t)(k + 2) * n)[i];
                const float4 t3 = reinterpret_cast<const float4*>(part + (int64_t)(k + 3) * n)[i];
                s.x += t0.x; s.y += t0.y; s.z += t0.z; s.w += t0.w;
                s.x += t1.x; s.y += t1.y; s.z += t1.z; s.w += t1.w;
                s.x += t2.x; s.y += t2.y; s.z += t2.z; s.w += t2.w;
                s.x += t3.x; s.y += t3.y; s.z += t3.z; s.w += t3.w;
            }
            for (; k < splits; ++k) {
                const float4 t = reinterpret_cast<const float4*>(part + (int64_t)k * n)[i];
                s.x += t.x; s.y += t.y; s.z += t.z; s.w += t.w;
            }
            reinterpret_cast<float4*>(dw)[i] = s;
        } else {
            float s = part[i];
            for (int k = 1; k < splits; ++k) s += part[(int64_t)k * n + i];
            dw[i] = s;
        }
    }
}

// Finish of a forward / dgrad whose reduction was cut: sum the splits in order,
// add the bias / apply ReLU (forward) or add the existing gradient (dgrad), and
// store in the output type.  Four outputs per lane.
template <typename T, bool MASKED>
__global__ __launch_bounds__(256) void splitk_finish_kernel(const float* __restrict__ part, void* out, const float* __restrict__ bias,
                                                            int64_t M, int Nn, int splits, int relu, int out_fp32, int accumulate,
                                                            RowCut cut, float* __restrict__ stats,
                                                            const T* __restrict__ mask_act, const T* __restrict__ xin,
                                                            const float* __restrict__ mean_rstd, const void* acc_src, GradDst dbias) {
    if (acc_src == nullptr) acc_src = out;      // where the gradient that is added to is read (see ConvArgs)
    // a workgroup owns 64 columns of one block of rows: 16 lanes across (4 columns each), 16 rows at a time
    int r0, r1;
    const int shard = locate_block(cut, blockIdx.y, r0, r1);
    const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
    const int col = (blockIdx.x * 16 + tx) * 4;
    const bool active = col < Nn;
    const int64_t mn = M * Nn;
    float4 bv = make_float4(0.f, 0.f, 0.f, 0.f);
    if (bias && active) bv = *reinterpret_cast<const float4*>(bias + col);
    float cs[4] = {0.f, 0.f, 0.f, 0.f}, cq[4] = {0.f, 0.f, 0.f, 0.f};
    // MASKED (input gradient): the sum is stored where the activation is positive, zero elsewhere, and the
    // column sums are those of the stored gradient and of gradient x normalised input (with xin)
    float mu[4] = {0.f, 0.f, 0.f, 0.f}, rs[4] = {0.f, 0.f, 0.f, 0.f};
    if (MASKED && xin != nullptr && active) {
        #pragma unroll
        for (int e = 0; e < 4; ++e) {
            mu[e] = mean_rstd[(int64_t)shard * 2 * Nn + col + e];
            rs[e] = mean_rstd[(int64_t)shard * 2 * Nn + Nn + col + e];
        }
    }
    if (active) {
        for (int64_t r = r0 + ty; r < r1; r += 16) {
            const int64_t i = r * Nn + col;
            float4 s = *reinterpret_cast<const float4*>(part + i);
            for (int k = 1; k < splits; ++k) {
                const float4 t = *reinterpret_cast<const float4*>(part + (int64_t)k * mn + i);
                s.x += t.x; s.y += t.y; s.z += t.z; s.w += t.w;
            }
            s.x += bv.x; s.y += bv.y; s.z += bv.z; s.w += bv.w;
            if (relu) { s.x = fmaxf(s.x, 0.f); s.y = fmaxf(s.y, 0.f); s.z = fmaxf(s.z, 0.f); s.w = fmaxf(s.w, 0.f); }
            if (out_fp32 || sizeof(T) == 4) {
                float4* d = reinterpret_cast<float4*>((float*)out + i);
                if (accumulate) {
                    const float4 o = *reinterpret_cast<const float4*>((const float*)acc_src + i);
                    s.x += o.x; s.y += o.y; s.z += o.z; s.w += o.w;
                }
                if (MASKED) {
                    const float4 am = *reinterpret_cast<const float4*>((const float*)mask_act + i);
                    s.x = am.x > 0.f ? s.x : 0.f; s.y = am.y > 0.f ? s.y : 0.f;
                    s.z = am.z > 0.f ? s.z : 0.f; s.w = am.w > 0.f ? s.w : 0.f;
                }
                *d = s;
                if (MASKED) {
                    float4 xv = make_float4(0.f, 0.f, 0.f, 0.f);
                    if (xin != nullptr) xv = *reinterpret_cast<const float4*>((const float*)xin + i);
                    cs[0] += s.x; cs[1] += s.y; cs[2] += s.z; cs[3] += s.w;
                    if (xin != nullptr) {
                        cq[0] += s.x * ((xv.x - mu[0]) * rs[0]); cq[1] += s.y * ((xv.y - mu[1]) * rs[1]);
                        cq[2] += s.z * ((xv.z - mu[2]) * rs[2]); cq[3] += s.w * ((xv.w - mu[3]) * rs[3]);
                    }
                    continue;
                }
            } else {
                uint2* d = reinterpret_cast<uint2*>((bf16_t*)out + i);
                if (accumulate) {
                    const uint2 o = *reinterpret_cast<const uint2*>((const bf16_t*)acc_src + i);
                    s.x += __uint_as_float(o.x << 16); s.y += __uint_as_float(o.x & 0xffff0000u);
                    s.z += __uint_as_float(o.y << 16); s.w += __uint_as_float(o.y & 0xffff0000u);
                }
                if (MASKED) {   // activation > 0: a positive bf16
                    const uint2 am = *reinterpret_cast<const uint2*>((const bf16_t*)mask_act + i);
                    if (!(__uint_as_float(am.x << 16) > 0.f)) s.x = 0.f;
                    if (!(__uint_as_float(am.x & 0xffff0000u) > 0.f)) s.y = 0.f;
                    if (!(__uint_as_float(am.y << 16) > 0.f)) s.z = 0.f;
                    if (!(__uint_as_float(am.y & 0xffff0000u) > 0.f)) s.w = 0.f;
                }
                const uint2 pk = make_uint2(pack2_bf16(s.x, s.y), pack2_bf16(s.z, s.w));
                *d = pk;
                // what a reader of the stored tensor sees
                s.x = __uint_as_float(pk.x << 16); s.y = __uint_as_float(pk.x & 0xffff0000u);
                s.z = __uint_as_float(pk.y << 16); s.w = __uint_as_float(pk.y & 0xffff0000u);
                if (MASKED) {
                    uint2 xw = make_uint2(0u, 0u);
                    if (xin != nullptr) xw = *reinterpret_cast<const uint2*>((const bf16_t*)xin + i);
                    const float x0 = __uint_as_float(xw.x << 16), x1 = __uint_as_float(xw.x & 0xffff0000u);
                    const float x2 = __uint_as_float(xw.y << 16), x3 = __uint_as_float(xw.y & 0xffff0000u);
                    cs[0] += s.x; cs[1] += s.y; cs[2] += s.z; cs[3] += s.w;
                    if (xin != nullptr) {
                        cq[0] += s.x * ((x0 - mu[0]) * rs[0]); cq[1] += s.y * ((x1 - mu[1]) * rs[1]);
                        cq[2] += s.z * ((x2 - mu[2]) * rs[2]); cq[3] += s.w * ((x3 - mu[3]) * rs[3]);
                    }
                    continue;
                }
            }
            cs[0] += s.x; cq[0] += s.x * s.x; cs[1] += s.y; cq[1] += s.y * s.y;
            cs[2] += s.z; cq[2] += s.z * s.z; cs[3] += s.w; cq[3] += s.w * s.w;
        }
    }
    if (stats == nullptr) return;
    // column sums of the stored values and of their squares, per row block (the batch-norm reduction's layout)
    __shared__ float red[2][16][64 + 1];
    #pragma unroll
    for (int e = 0; e < 4; ++e) { red[0][ty][tx * 4 + e] = cs[e]; red[1][ty][tx * 4 + e] = cq[e]; }
    __syncthreads();
    if (threadIdx.x < 128) {
        const int kind = threadIdx.x >> 6, c = threadIdx.x & 63, cg = blockIdx.x * 64 + c;
        if (cg < Nn) {
            float t = 0.f;
            #pragma unroll
            for (int j = 0; j < 16; ++j) t += red[kind][j][c];
            if (MASKED && dbias.g != nullptr) {     // a block is a shard: the sums are the producer's bias gradient
                if (kind == 0) dbias.g[(int64_t)cut.k[shard] * dbias.stride + cg] = t;
            } else {
                stats[(int64_t)(kind * Nn + cg) * gridDim.y + blockIdx.y] = t;
            }
        }
    }
}

// ---------------------------------------------------------------------------
// host side: tile selection and launch
// ---------------------------------------------------------------------------
enum TileCfg { T128x128, T128x64, T128x32, T64x64, T32x128 };   // T32x128: float32 weight gradients only

#ifndef EDL_PF_BIG
#define EDL_PF_BIG 1
#endif
#ifndef EDL_PF_SMALL
#define EDL_PF_SMALL 2
#endif
#ifndef EDL_BK_SMALL_MULT
#define EDL_BK_SMALL_MULT 1
#endif
#ifndef EDL_BK_BIG_DIV
#define EDL_BK_BIG_DIV 2
#endif
#ifndef EDL_BK_SMALL_DIV
#define EDL_BK_SMALL_DIV 1
#endif
#ifndef EDL_PF_BIG_HALF
#define EDL_PF_BIG_HALF EDL_PF_BIG
#endif
#ifndef EDL_PF_SMALL_TAIL
#define EDL_PF_SMALL_TAIL 1
#endif
#ifndef EDL_PF_WG_BIG
#define EDL_PF_WG_BIG EDL_PF_BIG
#endif
#ifndef EDL_PF_WG_DEEP
#define EDL_PF_WG_DEEP 2
#endif
#ifndef EDL_PF_WG_SMALL
#define EDL_PF_WG_SMALL 2
#endif

// reduction elements per tile: eight 16-byte vectors per row for either type
template <typename T> constexpr int kConvBK = 8 * Elem<T>::VEC;

// short_fwd: a problem whose epilogue is most of the workgroup's time (a forward pass of one or two
// reduction steps, an input-gradient pass whose epilogue adds, masks and sums); twice as many workgroups of
// half the width measured faster there
static TileCfg pick_tile(int M, int Nn, int Kred, int* bm, int* bn, bool short_fwd = false) {
    // A long reduction takes the 128x128 tile from fewer tiles on (the reduction is cut to fill the chip):
    // VGG-16's 14x14 layers, 196 tiles, measured 64 -> 48 us forward and 71 -> 47 us dgrad.
    const int min128_short = (int)tune().min128, min128_long = (int)tune().min128_long;
    const int min128 = Kred >= 4096 ? std::min(min128_short, min128_long) : min128_short;
    TileCfg t;
    if (Nn <= 32) t = T128x32;
    else if (Nn <= 64) t = (M >= 128) ? T128x64 : T64x64;
    else {
        const int64_t tiles = (int64_t)((M + 127) / 128) * ((Nn + 127) / 128);
        t = (tiles >= min128 && M >= 128) ? (short_fwd ? T128x64 : T128x128) : T64x64;
    }
    // measurement aid: one tile shape for every forward / dgrad problem it fits (0..3 = 128x128, 128x64, 128x32, 64x64)
    const int force = (int)tune().force_tile;
    if (force >= 0 && force <= 3) t = (TileCfg)force;
    switch (t) {
        case T128x128: *bm = 128; *bn = 128; break;
        case T128x64: *bm = 128; *bn = 64; break;
        case T128x32: *bm = 128; *bn = 32; break;
        default: *bm = 64; *bn = 64; break;
    }
    return t;
}

template <typename T, int MODE, int KIND>
static void launch_cfg(TileCfg t, bool fast, dim3 tiles, const typename ArgsOf<KIND>::type& a_in, hipStream_t st) {
    constexpr int BK = kConvBK<T>;
    typename ArgsOf<KIND>::type a = a_in;
    a.gx = (int)tiles.x; a.gy = (int)tiles.y; a.gz = (int)tiles.z;
    const double total = (double)a.gx * a.gy * a.gz;
    const bool mg = magic_fits(total, a.gx) && magic_fits(total, a.gy);
    a.magic_gx = mg ? magic_of(a.gx) : 0; a.magic_gy = mg ? magic_of(a.gy) : 0;
    const dim3 grid(tiles.x * tiles.y * tiles.z);
    // Measured on ResNet-50 at a shard of 32: the 64x64 tile (few registers per set, the least MFMA work per
    // reduction step, often fewer workgroups than the chip has room for) gains a third on long reductions from
    // two register sets of loads in flight; the 128-wide tiles gain nothing from a second set but do from
    // half-length reduction steps (half the LDS per workgroup, so more workgroups per CU).
    constexpr int PF_BIG = EDL_PF_BIG, PF_SMALL = MODE == CONV_WGRAD ? EDL_PF_WG_SMALL : EDL_PF_SMALL;
    constexpr int PF_HALF = MODE == CONV_WGRAD ? EDL_PF_WG_BIG : EDL_PF_BIG_HALF;   // 128-wide tiles on half-length steps
    constexpr int BK_SMALL = MODE == CONV_WGRAD ? BK : EDL_BK_SMALL_MULT * BK / EDL_BK_SMALL_DIV;
    constexpr int BK_BIG = MODE == CONV_WGRAD ? BK : BK / EDL_BK_BIG_DIV;
    // A weight gradient of at most one workgroup per CU has nobody to take turns with: one more tile in flight
    // hides the operand latency its single wave per SIMD leaves exposed (bf16; ResNet-50 at a shard of 32: 128x128 tiles
    // 22.2 -> 20.1 us, 128x64 24.4 -> 18.4 us).  Launches of more workgroups than CUs (VGG-16's long reductions, cut
    // into two workgroups per CU) keep the two-stage form: with a third stage only one workgroup fits a CU's LDS
    // (73.7 -> 113 us).
    constexpr int PF_DEEP = MODE == CONV_WGRAD ? EDL_PF_WG_DEEP : PF_BIG;
    const bool deep = MODE == CONV_WGRAD && total <= (double)tune().wgrad_deep_max;
    if (!fast) {   // element-wise kernel: one tile shape only
        if constexpr (KIND != CLASSES)
            hipLaunchKernelGGL((conv_igemm_kernel<T, MODE, 2, 2, 1, 1, BK, false, 1, KIND>), grid, dim3(256), 0, st, a);
        return;
    }
    if constexpr (MODE != CONV_WGRAD && KIND != CLASSES) {
        if (a.strip) {
            constexpr int BS = 64 / (int)sizeof(T);
            if constexpr (MODE == CONV_DGRAD) {
                // 64x64: a third stage as without strips (53 KB, three workgroups per CU either way)
                if (t == T128x128) hipLaunchKernelGGL((conv_igemm_kernel<T, MODE, 2, 2, 2, 2, BS, true, 1, KIND, 3>), grid, dim3(256), 0, st, a);
                if (t == T64x64) hipLaunchKernelGGL((conv_igemm_kernel<T, MODE, 2, 2, 1, 1, BS, true, 2, KIND, 3>), grid, dim3(256), 0, st, a);
            }
            if (t == T128x64) hipLaunchKernelGGL((conv_igemm_kernel<T, MODE, 2, 2, 2, 1, BS, true, 1, KIND, 3>), grid, dim3(256), 0, st, a);
            if (t == T128x32) hipLaunchKernelGGL((conv_igemm_kernel<T, MODE, 4, 1, 1, 1, BS, true, 1, KIND, 3>), grid, dim3(256), 0, st, a);
            return;
        }
    }
    if constexpr (MODE == CONV_DGRAD && KIND != CLASSES && sizeof(T) == 2 && EDL_DIRECT_LDS != 0) {
        if (a.brows) {      // reduction steps and stages as below (the rows are few: long reductions, full steps for 128x128)
            const bool tail = total > (double)tune().small_tail_from && total <= (double)tune().small_tail_to;
            if (t == T128x128) hipLaunchKernelGGL((conv_igemm_kernel<T, MODE, 2, 2, 2, 2, BK, true, 1, KIND, 1, true>), grid, dim3(256), 0, st, a);
            else if (t == T128x64) hipLaunchKernelGGL((conv_igemm_kernel<T, MODE, 2, 2, 2, 1, BK / 2, true, 1, KIND, 1, true>), grid, dim3(256), 0, st, a);
            else if (t == T128x32) hipLaunchKernelGGL((conv_igemm_kernel<T, MODE, 4, 1, 1, 1, BK, true, 1, KIND, 1, true>), grid, dim3(256), 0, st, a);
            else if (tail) hipLaunchKernelGGL((conv_igemm_kernel<T, MODE, 2, 2, 1, 1, BK, true, 1, KIND, 1, true>), grid, dim3(256), 0, st, a);
            else hipLaunchKernelGGL((conv_igemm_kernel<T, MODE, 2, 2, 1, 1, BK, true, 2, KIND, 1, true>), grid, dim3(256), 0, st, a);
            return;
        }
    }
    switch (t) {
        case T128x128: {
            // Long reductions (VGG-16's 3x3 layers: 1,152 to 4,608 elements) run faster on full-length reduction
            // steps (half the barriers per MFMA: measured 159 -> 135 us forward, 174 -> 154 us dgrad on VGG-16);
            // short ones (ResNet-50's 1x1 layers) want the smaller LDS footprint and more workgroups per CU.
            const int full_steps_from = (int)tune().bk64_kred;
            if constexpr (MODE == CONV_WGRAD && sizeof(T) == 2) {
                if (deep) {
                    hipLaunchKernelGGL((conv_igemm_kernel<T, MODE, 2, 2, 2, 2, BK, true, PF_DEEP, KIND>), grid, dim3(256), 0, st, a);
                    break;
                }
            }
            if (BK_BIG != BK && a.Kred >= full_steps_from)
                hipLaunchKernelGGL((conv_igemm_kernel<T, MODE, 2, 2, 2, 2, BK, true, PF_BIG, KIND>), grid, dim3(256), 0, st, a);
            else
                hipLaunchKernelGGL((conv_igemm_kernel<T, MODE, 2, 2, 2, 2, BK_BIG, true, PF_HALF, KIND>), grid, dim3(256), 0, st, a);
            break;
        }
        case T128x64:
            if constexpr (MODE == CONV_WGRAD && sizeof(T) == 2) {
                if (deep) {
                    hipLaunchKernelGGL((conv_igemm_kernel<T, MODE, 2, 2, 2, 1, BK, true, PF_DEEP, KIND>), grid, dim3(256), 0, st, a);
                    break;
                }
            }
            hipLaunchKernelGGL((conv_igemm_kernel<T, MODE, 2, 2, 2, 1, BK_BIG, true, PF_HALF, KIND>), grid, dim3(256), 0, st, a);
            break;
        case T128x32: hipLaunchKernelGGL((conv_igemm_kernel<T, MODE, 4, 1, 1, 1, BK, true, PF_BIG, KIND>), grid, dim3(256), 0, st, a); break;
        case T32x128:
            if constexpr (MODE == CONV_WGRAD && sizeof(T) == 4)
                hipLaunchKernelGGL((conv_igemm_kernel<T, MODE, 1, 4, 1, 1, BK, true, 1, KIND>), grid, dim3(256), 0, st, a);
            break;
        default:
            if constexpr (MODE != CONV_WGRAD && sizeof(T) == 2) {
                // Three stages of a 64x64 tile are 48 KB of LDS: three workgroups per CU, 768 on the chip.  A launch
                // of a few more (784 and 800 are common: 25,088 pixels x 128 channels, 1,568 x 2,048) ran a second
                // round for its last 16 or 32 workgroups and took almost twice one round.  Such launches run the
                // two-stage form (32 KB, five per CU), so that all of their workgroups are resident at once:
                // 22.1 -> 18.2 us and 25.9 -> 22.2 us for the 3x3 layers at 28x28, 0.490 -> 0.422 ms per ResNet-50
                // step over all launches of that size.
                if (total > (double)tune().small_tail_from && total <= (double)tune().small_tail_to) {
                    hipLaunchKernelGGL((conv_igemm_kernel<T, MODE, 2, 2, 1, 1, BK_SMALL, true, EDL_PF_SMALL_TAIL, KIND>), grid, dim3(256), 0, st, a);
                    break;
                }
            }
            hipLaunchKernelGGL((conv_igemm_kernel<T, MODE, 2, 2, 1, 1, BK_SMALL, true, PF_SMALL, KIND>), grid, dim3(256), 0, st, a);
            break;
    }
}

static const char* conv_label(int dtype, int mode, TileCfg t) {
    if (t == T32x128) return "conv_wgrad_f32_32x128";
    static const char* names[2][3][4] = {
        {{"conv_fwd_f32_128x128", "conv_fwd_f32_128x64", "conv_fwd_f32_128x32", "conv_fwd_f32_64x64"},
         {"conv_dgrad_f32_128x128", "conv_dgrad_f32_128x64", "conv_dgrad_f32_128x32", "conv_dgrad_f32_64x64"},
         {"conv_wgrad_f32_128x128", "conv_wgrad_f32_128x64", "conv_wgrad_f32_128x32", "conv_wgrad_f32_64x64"}},
        {{"conv_fwd_bf16_128x128", "conv_fwd_bf16_128x64", "conv_fwd_bf16_128x32", "conv_fwd_bf16_64x64"},
         {"conv_dgrad_bf16_128x128", "conv_dgrad_bf16_128x64", "conv_dgrad_bf16_128x32", "conv_dgrad_bf16_64x64"},
         {"conv_wgrad_bf16_128x128", "conv_wgrad_bf16_128x64", "conv_wgrad_bf16_128x32", "conv_wgrad_bf16_64x64"}}};
    return names[dtype == 1 ? 1 : 0][mode][(int)t];
}


static bool conv_fast(int dtype, int mode, const ConvArgs& a) {
    const int ovec = (mode == CONV_WGRAD || dtype != 1) ? 4 : 8;
    return a.vecA && a.vecB && a.Nn % ovec == 0;
}

// every multiply-shift division of the vector kernel is exact for this problem
static bool conv_magic_ok(int mode, const ConvArgs& a) {
    if (mode == CONV_WGRAD) return true;
    const int inner = mode == CONV_FWD ? a.C : a.K, taps = mode == CONV_FWD ? a.S : a.ns;
    const int pix = mode == CONV_FWD ? a.Ho * a.Wo : a.Hc * a.Wc, wpix = mode == CONV_FWD ? a.Wo : a.Wc;
    const double kmax = (double)a.Kred + 256.0, mmax = (double)a.M + 256.0;
    return magic_fits(kmax, inner) && magic_fits(kmax / (inner > 0 ? inner : 1) + 1.0, taps) &&
           magic_fits(mmax, pix) && magic_fits((double)pix, wpix);
}

template <int MODE>
static void launch_mode(int dtype, TileCfg t, dim3 grid, const ConvArgsShards& a_in, hipStream_t st, ConvArgsClasses* classes = nullptr) {
    ConvArgsShards a = a_in;
    a.shards = a.cut.p;
    if (MODE == CONV_FWD) { a.magic_inner = magic_of(a.C); a.magic_taps = magic_of(a.S); }
    else if (MODE == CONV_DGRAD) { a.magic_inner = magic_of(a.K); a.magic_taps = magic_of(a.ns); }
    if (MODE == CONV_FWD) { a.magic_hw = magic_of(a.Ho * a.Wo); a.magic_w = magic_of(a.Wo); }
    else if (MODE == CONV_DGRAD) { a.magic_hw = magic_of(a.Hc * a.Wc); a.magic_w = magic_of(a.Wc); }
    a.stride_shift = a.stride >= 4 ? 2 : a.stride >= 2 ? 1 : 0;
    const bool magic_ok = conv_magic_ok(MODE, a);
    const bool fast = conv_fast(dtype, MODE, a) && magic_ok;
    if (!fast) {
        t = T64x64;
        grid.x = (a.M + 63) / 64;
        grid.y = (a.Nn + 63) / 64;
        if (a.brows) a.vecB = 0;      // the element-wise kernel's vectors of B are along the reduction
    }
    // Tile order: the reduction cuts are the slowest index, so a die's run of tiles
    // stays within few cuts; inside a cut the tiles that share the larger operand
    // (activations: the same row tile; weights: the same column tile) are neighbours.
    const int tune_xcd = (int)tune().xcd, tune_order = (int)tune().order;
    a.xcd_chunked = tune_xcd;
    if (tune_order >= 0) a.n_fastest = tune_order;
    else if (MODE == CONV_WGRAD) a.n_fastest = 1;
    else a.n_fastest = (double)a.M * (MODE == CONV_FWD ? a.C : a.K) >= (double)a.Nn * a.Kred;
    // algorithmic work: 2*M*N*K flops; operands and result touched once
    const double esz = dtype == 1 ? 2.0 : 4.0;
    double flops = 2.0 * (double)a.M * a.Nn * a.Kred;
    double bytes;
    if (MODE == CONV_FWD) bytes = esz * ((double)a.N * a.H * a.W * a.C + (double)a.Nn * a.Kred) + (a.out_fp32 ? 4.0 : esz) * (double)a.M * a.Nn;
    else if (MODE == CONV_DGRAD) {
        // dy, weights, dx; plus what a fused epilogue reads at every output position: the gradient already
        // there, the activation that masks it, the batch norm's input for the second sum
        const double extra = (a.accumulate ? 1.0 : 0.0) + (a.mask_act ? (a.mask_sign ? 1.0 / 16 : 1.0) : 0.0) + (a.xin ? 1.0 : 0.0);
        bytes = esz * ((double)a.N * a.Ho * a.Wo * a.K + (double)a.Nn * a.Kred + (1.0 + extra) * (double)a.M * a.Nn);
    } else bytes = esz * ((double)a.Kred * a.K + (double)a.N * a.H * a.W * a.C) + 4.0 * (double)a.M * a.Nn;
    const char* label = conv_label(dtype, MODE, t);
    static const bool by_shape = getenv("EDL_PROFILE_BY_SHAPE") != nullptr;
    if (by_shape && prof_enabled()) {
        // one profile line per distinct problem shape instead of per kernel family
        static std::deque<std::string> names;
        char buf[160];
        snprintf(buf, sizeof(buf), "%s M=%d N=%d K=%d r%d s%d grid=%ux%ux%u", label, a.M, a.Nn, a.Kred, a.R, a.stride, grid.x, grid.y, grid.z);
        const char* found = nullptr;
        for (const std::string& n : names) if (n == buf) { found = n.c_str(); break; }
        if (!found) { names.emplace_back(buf); found = names.back().c_str(); }
        label = found;
    }
    if (MODE == CONV_DGRAD && classes != nullptr) {
        flops = 0;
        bytes = esz * ((double)a.N * a.Ho * a.Wo * a.K + (double)a.Nn * a.ldb + (a.accumulate ? 2.0 : 1.0) * (double)a.N * a.H * a.W * a.Nn);
        for (int c = 0; c < classes->classes; ++c) flops += 2.0 * (double)classes->cls[c].M * a.Nn * classes->cls[c].Kred;
    }
    ProfScope ps(label, flops, bytes, st);
    if (MODE == CONV_DGRAD && classes != nullptr) {
        static_cast<ConvArgs&>(*classes) = a;
        for (int c = 0; c < classes->classes; ++c) {
            ConvClass& k = classes->cls[c];
            k.magic_hw = magic_of(k.Hc * k.Wc);
            k.magic_w = magic_of(k.Wc);
            k.magic_taps = magic_of(k.ns);
        }
        if constexpr (MODE == CONV_DGRAD) {
            if (dtype == 1) launch_cfg<bf16_t, MODE, CLASSES>(t, true, grid, *classes, st);
            else launch_cfg<float, MODE, CLASSES>(t, true, grid, *classes, st);
        }
        return;
    }
    if (MODE == CONV_WGRAD && a.ksplit > a.fold) {
        if constexpr (MODE == CONV_WGRAD) {
            if (dtype == 1) launch_cfg<bf16_t, MODE, FOLDED>(t, fast, grid, a, st);
            else launch_cfg<float, MODE, FOLDED>(t, fast, grid, a, st);
        }
    } else if (a.shards > 1) {
        if (dtype == 1) launch_cfg<bf16_t, MODE, SHARDED>(t, fast, grid, a, st);
        else launch_cfg<float, MODE, SHARDED>(t, fast, grid, a, st);
    } else {
        if (dtype == 1) launch_cfg<bf16_t, MODE, PLAIN>(t, fast, grid, a, st);
        else launch_cfg<float, MODE, PLAIN>(t, fast, grid, a, st);
    }
}

static ConvArgsShards base_args(const ConvGeom& g) {
    ConvArgsShards a = {};
    a.N = g.N; a.H = g.H; a.W = g.W; a.C = g.C; a.K = g.K; a.R = g.R; a.S = g.S;
    a.stride = g.stride; a.pad = g.pad; a.Ho = g.Ho; a.Wo = g.Wo;
    a.ph = a.pw = a.r0 = a.s0 = 0; a.nr = g.R; a.ns = g.S; a.Hc = g.H; a.Wc = g.W;
    a.cut.p = 1;
    a.fold = 128;       // forward and input gradients in float32: about what a cut reduction's shortest pieces are
    return a;
}

int conv_vector_samples(const ConvGeom& g, bool dgrad) {
    constexpr int kMost = 65535;
    const auto ok = [&](int n) {
        ConvArgs f = base_args(g), d = base_args(g);
        // (of a strided input gradient the largest residue class)
        d.Hc = (g.H + g.stride - 1) / g.stride; d.Wc = (g.W + g.stride - 1) / g.stride;
        d.ns = (g.S + g.stride - 1) / g.stride;
        const int64_t fm = (int64_t)n * g.Ho * g.Wo, dm = (int64_t)n * d.Hc * d.Wc;
        if (std::max(fm, dm) >= (1ll << 31)) return false;
        f.M = (int)fm; f.Kred = g.R * g.S * g.C;
        d.M = (int)dm; d.Kred = g.R * g.S * g.K;
        return conv_magic_ok(CONV_FWD, f) && (!dgrad || conv_magic_ok(CONV_DGRAD, d));
    };
    if (!ok(1) || ok(kMost)) return kMost;      // never on the vector path, or always
    int lo = 1, hi = kMost;
    while (hi - lo > 1) (ok((lo + hi) / 2) ? lo : hi) = (lo + hi) / 2;
    return lo;
}

size_t conv_sums_floats(const ConvGeom& g, int p) {
    // the narrowest row tile is 64 rows; the finishing kernel of a cut reduction takes kRedRowBlocks blocks at most
    const auto blocks = [&](int64_t rows) { return std::max<int64_t>(rows / 64, std::min<int64_t>(rows / 16, kRedRowBlocks)) + 1 + p; };
    const size_t fwd = (size_t)(2 * g.K * blocks((int64_t)g.N * g.Ho * g.Wo)), dgrad = (size_t)(2 * g.C * blocks((int64_t)g.N * g.H * g.W));
    return g.stride == 1 ? std::max(fwd, dgrad) : fwd;
}

// How a launch's rows are cut into row tiles of bm: within the shards if it is to leave column sums (and the shards
// are large enough for that not to leave most of a tile idle), else without regard to them.
static RowCut tile_cut(const ShardSet& S, int rows_per_sample, int bm, bool want_sums, bool* per_shard) {
    *per_shard = S.plan_p == 1;
    if (want_sums && S.plan_smallest * rows_per_sample >= bm) *per_shard = true;
    if (*per_shard) return cut_rows(S, rows_per_sample, bm);
    ShardSet all = {};
    all.p = 1;
    all.off[1] = S.samples();
    all.plan_itself();
    return cut_rows(all, rows_per_sample, bm);
}

// Convolutions whose reduction steps are strips: 3x3, stride 1, one pixel of padding, and a number of channels that is a
// multiple of the 64 bytes a strip's rows hold.  Every input-gradient launch of that kind gains (64x64 tiles 2 to 3%,
// 128x128 6%, 128x64 up to 23%), and so do forward launches of narrow outputs (128x64 up to 14%, float32 128x32 8%);
// forward 128x128 tiles lose 2% (full-length steps have fewer barriers than strips there), 64x64 tiles gain nothing.
static bool takes_strips(int dtype, int mode, const ConvGeom& g, TileCfg t) {
    const int inner = mode == CONV_FWD ? g.C : g.K, row = dtype == 1 ? 32 : 16;
    return g.R == 3 && g.S == 3 && g.stride == 1 && g.pad == 1 && g.Ho == g.H && g.Wo == g.W && inner % row == 0 &&
           (mode == CONV_DGRAD || t == T128x64 || t == T128x32);
}

// Cut of the reduction for forward / dgrad problems that give too few tiles to
// fill the chip but have a long reduction (late stages at small batch, fully
// connected layers): returns the number of splits (1 = none).  The target is little more than one
// workgroup per CU: every further cut costs the finishing kernel more partial sums than the fuller chip
// gains (measured on ResNet-50 at a shard of 32: 768 -> 320 workgroups, 4.73 -> 4.69 ms per step;
// VGG-16 5.20 -> 5.14 ms).
static int plan_splitk(int dtype, int M, int Nn, int Kred, int bm, int bn, int* ksplit, bool strip) {
    const int BK = dtype == 1 ? 64 : 32;
    const int unit = strip ? BK / 2 * 3 : BK;      // a cut holds whole steps
    const int64_t tiles = (int64_t)((M + bm - 1) / bm) * ((Nn + bn - 1) / bn);
    const int nk = (Kred + BK - 1) / BK;
    int splits = 1;
    const int max_tiles = (int)tune().splitk_tiles, target = (int)tune().splitk_target;
    if (tiles < max_tiles && nk >= 8) {
        splits = (int)((target + tiles - 1) / tiles);
        if (splits > nk / 4) splits = nk / 4;
        if (splits > 8) splits = 8;
        if (splits < 1) splits = 1;
    }
    const int units = (Kred + unit - 1) / unit, ks = (units + splits - 1) / splits * unit;
    *ksplit = ks;
    return (Kred + ks - 1) / ks;
}

// Returns how the column sums it left in stats are cut (p == 0 if stats.buf is null or too small).
template <typename T>
static RowCut launch_finish(const ConvArgs& a, const ShardSet& S, int rows_per_sample, int splits, SumsBuf stats, hipStream_t st,
                            const DgradMask* mask = nullptr) {
    const int col_blocks = (a.Nn + 63) / 64;
    // about 1024 workgroups, at least 16 rows each
    int64_t rb = (1024 + col_blocks - 1) / col_blocks;
    const int64_t M = (int64_t)S.plan * rows_per_sample;
    const int64_t max_rb = (M + 15) / 16;
    if (rb > max_rb) rb = max_rb;
    if (rb > kRedRowBlocks) rb = kRedRowBlocks;
    if (rb < 1) rb = 1;
    RowCut cut = cut_rows(S, rows_per_sample, (int)((M + rb - 1) / rb));
    const int row_blocks = cut.blk0[cut.p];
    cut.stored = mask != nullptr && mask->xin == nullptr && mask->dbias.g != nullptr && cut.block_per_shard();
    if (stats.buf != nullptr && stats.floats < (size_t)2 * a.Nn * row_blocks) stats.buf = nullptr;   // cannot happen: sized for it
    ProfScope ps("splitk_finish", 0.0, 4.0 * (double)a.M * a.Nn * splits + (a.out_fp32 ? 4.0 : (double)sizeof(T)) * (double)a.M * a.Nn, st);
    if (mask != nullptr && stats.buf != nullptr)
        hipLaunchKernelGGL((splitk_finish_kernel<T, true>), dim3(col_blocks, row_blocks), dim3(256), 0, st, a.partial, a.out, a.bias,
                           (int64_t)a.M, a.Nn, splits, a.relu, a.out_fp32, a.accumulate, cut, stats.buf,
                           (const T*)mask->act, (const T*)mask->xin, mask->mean_rstd, a.acc_src, cut.stored ? mask->dbias : GradDst{nullptr, 0});
    else
        hipLaunchKernelGGL((splitk_finish_kernel<T, false>), dim3(col_blocks, row_blocks), dim3(256), 0, st, a.partial, a.out, a.bias,
                           (int64_t)a.M, a.Nn, splits, a.relu, a.out_fp32, a.accumulate, cut, mask != nullptr ? nullptr : stats.buf,
                           (const T*)nullptr, (const T*)nullptr, (const float*)nullptr, a.acc_src, GradDst{nullptr, 0});
    return stats.buf ? cut : RowCut();
}

size_t conv_splitk_scratch_bytes(int dtype, const ConvGeom& g, int samples) {
    size_t need = 0;
    for (int mode = 0; mode < 2; ++mode) {
        if (mode == 1 && g.stride != 1) continue;
        const int hw = mode == 0 ? g.Ho * g.Wo : g.H * g.W;
        const int Nn = mode == 0 ? g.K : g.C;
        const int Kred = mode == 0 ? g.R * g.S * g.C : g.R * g.S * g.K;
        // the number of cuts does not follow the size of the pass steadily (the tile changes): every size up to those
        // that are not cut on any tile
        for (int n = 1; n <= g.N; ++n) {
            const int M = n * hw;
            if ((int64_t)((M + 127) / 128) * ((Nn + 127) / 128) >= tune().splitk_tiles) break;
            int bm, bn, ks;
            const TileCfg t = pick_tile(M, Nn, Kred, &bm, &bn, mode == 0 && Kred <= 128);
            const int splits = plan_splitk(dtype, M, Nn, Kred, bm, bn, &ks, takes_strips(dtype, mode, g, t));
            if (splits > 1) need = std::max(need, (size_t)splits * std::min(n, samples) * hw * Nn * sizeof(float));
        }
    }
    return need;
}

static bool small_fwd(int dtype, const ConvGeom& g, const ShardSet& S, const void* x, const void* w) {
    return small_fc_takes(dtype, g, g.C, g.K, S.plan) && (((uintptr_t)x | (uintptr_t)w) & 15) == 0 && tune().force_tile < 0;
}

bool conv_fwd_gathers(int dtype, const ConvGeom& g, const ShardSet& S, const void* data, const void* x, const void* w) {
    return g.N <= kSmallGather && ((uintptr_t)data & 15) == 0 && small_fwd(dtype, g, S, x, w) && !thin_fwd_takes(dtype, g, S.plan, true);
}

RowCut launch_conv_fwd(int dtype, const ConvGeom& g, const ShardSet& S, const void* x, const void* w, const float* bias, bool relu,
                       bool out_fp32, void* y, float* scratch, size_t scratch_bytes, SumsBuf stats, hipStream_t st) {
    const bool small = small_fwd(dtype, g, S, x, w);
    if (thin_fwd_takes(dtype, g, S.plan, small)) {
        launch_thin_fwd(dtype, g, x, w, bias, relu, out_fp32, y, st);
        return RowCut();
    }
    if (small) {
        launch_small_fc_fwd(g, S, (const float*)x, (const float*)w, bias, relu, (float*)y, nullptr, st);
        return RowCut();
    }
    if (bias == nullptr && !relu && narrow_takes(dtype, g, S))
        return launch_narrow(g, S, {(const float*)x, (const float*)w, (float*)y, false, nullptr, tune().fused_stats != 0 ? stats : SumsBuf{nullptr, 0}, nullptr}, st);
    const int VEC = dtype == 1 ? 8 : 4;
    ConvArgsShards a = base_args(g);
    a.A = x; a.B = w; a.out = y; a.bias = bias;
    a.M = g.N * g.Ho * g.Wo; a.Nn = g.K; a.Kred = g.R * g.S * g.C;
    a.relu = relu; a.out_fp32 = out_fp32;
    const double esz = dtype == 1 ? 2.0 : 4.0;
    const double bA = esz * (double)g.N * g.H * g.W * g.C, bB = esz * (double)a.Nn * a.Kred;
    a.vecA = (g.C % VEC == 0) && bA < 2147483648.0; a.vecB = (a.Kred % VEC == 0) && bB < 2147483648.0;
    a.bytesA = a.vecA ? (unsigned)bA : 0; a.bytesB = a.vecB ? (unsigned)bB : 0;
    a.ksplit = a.Kred;
    a.ldb = a.Kred;
    int bm, bn;
    const int Mplan = S.plan * g.Ho * g.Wo;
    const TileCfg t = pick_tile(Mplan, a.Nn, a.Kred, &bm, &bn, a.Kred <= 128);
    const bool fast = conv_fast(dtype, CONV_FWD, a);
    if (fast && bias == nullptr && !relu && !out_fp32 && tune().force_tile < 0 && pointwise_takes(dtype, g, S.plan, a.Kred, a.Nn)) {
        PointwiseTask t = {};
        t.K = a.Kred; t.N = a.Nn;
        t.A = x; t.B = w; t.out = y;
        if (tune().fused_stats != 0) t.sums = stats;
        RowCut left;
        if (launch_pointwise(g, S, t, &left, st)) return left;
    }
    int splits = 1, ks = a.Kred;
    a.strip = fast && conv_magic_ok(CONV_FWD, a) && takes_strips(dtype, CONV_FWD, g, t);
    if (fast) {
        splits = plan_splitk(dtype, Mplan, a.Nn, a.Kred, bm, bn, &ks, a.strip);
        if (splits > 1 && (scratch == nullptr || scratch_bytes < (size_t)splits * a.M * a.Nn * sizeof(float))) splits = 1;
    }
    if (splits > 1) { a.ksplit = ks; a.partial = scratch; }
    if (tune().fused_stats == 0 || out_fp32 || !fast || !conv_magic_ok(CONV_FWD, a)) stats.buf = nullptr;
    // whole reduction in one workgroup: the epilogue leaves the sums; cut reduction: the finishing kernel does
    bool per_shard;
    a.cut = tile_cut(S, g.Ho * g.Wo, bm, stats.buf != nullptr && splits == 1, &per_shard);
    const int row_tiles = a.cut.blk0[a.cut.p];
    if (splits == 1 && per_shard && stats.buf != nullptr && stats.floats >= (size_t)2 * a.Nn * row_tiles) a.stats = stats.buf;
    launch_mode<CONV_FWD>(dtype, t, dim3(row_tiles, (a.Nn + bn - 1) / bn, splits), a, st);
    if (splits > 1) {
        const int hw = g.Ho * g.Wo;
        return dtype == 1 ? launch_finish<bf16_t>(a, S, hw, splits, stats, st) : launch_finish<float>(a, S, hw, splits, stats, st);
    }
    return a.stats ? a.cut : RowCut();
}

// Fully connected layers (one pixel, one tap) in bf16: there the transposed copy costs more than the input gradient itself
// (VGG-16, shard of 32: 118 us to copy 124 M weights, 104 us for the three launches that read the copy), which reads every
// weight once, for few rows.  Convolutions read theirs for thousands of rows and keep the copy.  The vectors of B are
// eight channels of one row, so rows are to start on 16 bytes.  Step of VGG-16, shard of 32: 4,946 -> 4,822 us; AlexNet,
// two shards of 64: 1,613 -> 1,578 us.
// Small layers (k_thin.hip) read them so in either type.
bool conv_dgrad_reads_weights(int dtype, const ConvGeom& g, int64_t w_off) {
    if (thin_dgrad_takes(dtype, g) || small_fc_takes(dtype, g, g.K, g.C, g.N)) return true;
    return EDL_DIRECT_LDS != 0 && dtype == 1 && g.R == 1 && g.S == 1 && g.stride == 1 && g.pad == 0 && g.H == 1 && g.W == 1 &&
           g.K % 8 == 0 && g.C % 8 == 0 && w_off % 8 == 0;
}

bool conv_gradients_together(int dtype, const ConvGeom& g, const ShardSet& S, bool w_rows) {
    return w_rows && dtype != 1 && g.K % 4 == 0 && small_wgrad_takes(dtype, g, S);
}

RowCut launch_conv_dgrad(int dtype, const ConvGeom& g, const ShardSet& S, const void* dy, const void* wT, bool accumulate, void* dx,
                         float* scratch, size_t scratch_bytes, const DgradMask* mask, hipStream_t st, const void* acc_src, bool w_rows, const BothGradients* wgrad) {
    RowCut left;
    const bool ragged = g.K % (dtype == 1 ? 8 : 4) != 0;
    if (w_rows && (dtype != 1 || ragged)) {
        const void* const old = accumulate ? (acc_src != nullptr ? acc_src : dx) : nullptr;
        const DgradMask* const m = tune().fused_mask != 0 && (!accumulate || tune().fused_mask_join != 0) ? mask : nullptr;
        if (ragged) return launch_thin_dgrad(dtype, g, S, dy, wT, old, dx, m, st);
        const SmallWgrad both = wgrad != nullptr ? SmallWgrad{(const float*)wgrad->x, wgrad->dw} : SmallWgrad{};
        return launch_small_fc_dgrad(g, S, (const float*)dy, (const float*)wT, (const float*)old, (float*)dx, m, wgrad != nullptr ? &both : nullptr, st);
    }
    const bool mask_here = tune().fused_mask != 0 && mask != nullptr && mask->act != nullptr && (!accumulate || tune().fused_mask_join != 0);
    if (!w_rows && (!mask_here || mask->xin != nullptr) && narrow_takes(dtype, g, S)) {
        const float* const old = accumulate ? (const float*)(acc_src != nullptr ? acc_src : dx) : nullptr;
        return launch_narrow(g, S, {(const float*)dy, (const float*)wT, (float*)dx, true, old, mask_here ? mask->sums : SumsBuf{nullptr, 0},
                                    mask_here ? mask : nullptr}, st);
    }
    const int VEC = dtype == 1 ? 8 : 4;
    ConvArgsShards a = base_args(g);
    a.A = dy; a.B = wT; a.out = dx;
    a.Nn = g.C;
    a.ldb = g.R * g.S * g.K;
    a.accumulate = accumulate;
    a.acc_src = (accumulate && g.stride == 1) ? acc_src : nullptr;
    const double esz = dtype == 1 ? 2.0 : 4.0;
    const double bA = esz * (double)g.N * g.Ho * g.Wo * g.K, bB = esz * (double)a.Nn * a.ldb;
    // the vector gather of dy divides pixel coordinates by the stride with a shift
    const bool stride_pow2 = g.stride == 1 || g.stride == 2 || g.stride == 4;
    a.vecA = (g.K % VEC == 0) && bA < 2147483648.0 && stride_pow2; a.vecB = (a.ldb % VEC == 0) && bB < 2147483648.0;
    a.bytesA = a.vecA ? (unsigned)bA : 0; a.bytesB = a.vecB ? (unsigned)bB : 0;
    a.brows = w_rows;
    const bool want_mask = tune().fused_mask != 0 && mask != nullptr && mask->act != nullptr && g.stride == 1;
    // A residual join: the gradient is added to the shortcut's, masked and summed
    if (want_mask && accumulate && tune().fused_mask_join != 0 && mask->sign != nullptr && mask->xin != nullptr && tune().force_tile < 0 &&
        conv_fast(dtype, CONV_DGRAD, a) && pointwise_takes(dtype, g, S.plan, g.K, g.C)) {
        PointwiseTask t = {};
        t.K = g.K; t.N = g.C;
        t.A = dy; t.B = wT; t.out = dx;
        t.join = true;
        t.old = a.acc_src != nullptr ? a.acc_src : dx;
        t.sign = mask->sign; t.xin = mask->xin; t.mean_rstd = mask->mean_rstd;
        t.sums = mask->sums;
        if (launch_pointwise(g, S, t, &left, st)) return left;
    }
    // Stride 2: the four residue classes of the input pixel modulo the stride in one launch (each alone is a quarter of
    // the pixels, three of a 1x1 convolution's only zeros: 24 launches fewer in ResNet-50's chain)
    if (g.stride == 2 && conv_fast(dtype, CONV_DGRAD, a)) {
        ConvArgsClasses cls = {};
        int64_t work = 0;
        int longest = 0;
        bool ok = true;
        for (int c = 0; c < 4; ++c) {
            const int ph = c >> 1, pw = c & 1;
            if (ph >= g.H || pw >= g.W) continue;
            ConvClass k = {};
            k.ph = ph; k.pw = pw;
            k.Hc = (g.H - ph + 1) / 2; k.Wc = (g.W - pw + 1) / 2;
            k.r0 = (ph + g.pad) % 2; k.s0 = (pw + g.pad) % 2;
            k.nr = k.r0 < g.R ? (g.R - k.r0 + 1) / 2 : 0;
            k.ns = k.s0 < g.S ? (g.S - k.s0 + 1) / 2 : 0;
            k.M = g.N * k.Hc * k.Wc;
            k.Kred = k.nr * k.ns * g.K;
            if (k.Kred == 0 && accumulate) continue;      // nothing reaches these pixels
            ConvArgs probe = a;
            probe.Hc = k.Hc; probe.Wc = k.Wc; probe.ns = k.ns; probe.M = k.M; probe.Kred = k.Kred;
            ok = ok && conv_magic_ok(CONV_DGRAD, probe);
            if (k.Kred > 0) work = std::max(work, (int64_t)S.plan * k.Hc * k.Wc);
            longest = std::max(longest, k.Kred);
            cls.cls[cls.classes++] = k;
        }
        if (ok && cls.classes > 0) {
            int bm, bn, tiles = 0;
            const TileCfg t = pick_tile((int)work, a.Nn, longest, &bm, &bn);
            for (int c = 0; c < cls.classes; ++c) tiles = std::max(tiles, (cls.cls[c].M + bm - 1) / bm);
            tiles *= cls.classes;
            const ConvClass& k = cls.cls[0];
            a.ph = k.ph; a.pw = k.pw; a.Hc = k.Hc; a.Wc = k.Wc; a.r0 = k.r0; a.s0 = k.s0; a.nr = k.nr; a.ns = k.ns; a.M = k.M; a.Kred = k.Kred;
            launch_mode<CONV_DGRAD>(dtype, t, dim3(tiles, (a.Nn + bn - 1) / bn, 1), a, st, &cls);
            return left;
        }
    }
    // one launch per residue class of the input pixel modulo the stride
    for (int ph = 0; ph < g.stride && ph < g.H; ++ph) {
        for (int pw = 0; pw < g.stride && pw < g.W; ++pw) {
            a.ph = ph; a.pw = pw;
            a.Hc = (g.H - ph + g.stride - 1) / g.stride;
            a.Wc = (g.W - pw + g.stride - 1) / g.stride;
            a.r0 = (ph + g.pad) % g.stride;
            a.s0 = (pw + g.pad) % g.stride;
            a.nr = a.r0 < g.R ? (g.R - a.r0 + g.stride - 1) / g.stride : 0;
            a.ns = a.s0 < g.S ? (g.S - a.s0 + g.stride - 1) / g.stride : 0;
            a.M = g.N * a.Hc * a.Wc;
            a.Kred = a.nr * a.ns * g.K;
            a.ksplit = a.Kred > 0 ? a.Kred : 1;
            a.partial = nullptr;
            if (a.Kred == 0 && accumulate) continue;      // nothing reaches these pixels
            int bm, bn;
            // an epilogue that adds to the gradient already there, masks and sums it reads three more tensors
            // than it writes: 128x64 tiles (twice the workgroups, half the vectors in flight per lane; measured
            // -0.4% of the ResNet-50 step, 64x64 tiles +1.5%)
            const bool heavy = tune().join_tile != 0 && mask != nullptr && mask->act != nullptr && accumulate && g.stride == 1;
            const int Mplan = S.plan * a.Hc * a.Wc;
            const TileCfg t = pick_tile(Mplan, a.Nn, a.Kred, &bm, &bn, heavy);
            const bool fast = conv_fast(dtype, CONV_DGRAD, a);
            int splits = 1, ks = a.ksplit;
            a.strip = fast && conv_magic_ok(CONV_DGRAD, a) && takes_strips(dtype, CONV_DGRAD, g, t);
            if (g.stride == 1 && fast) {
                splits = plan_splitk(dtype, Mplan, a.Nn, a.Kred, bm, bn, &ks, a.strip);
                if (splits > 1 && (scratch == nullptr || scratch_bytes < (size_t)splits * a.M * a.Nn * sizeof(float))) splits = 1;
            }
            if (splits > 1) { a.ksplit = ks; a.partial = scratch; }
            // masked store and column sums in the epilogue: one launch that covers every pixel and leaves the
            // final gradient (it may add to what other readers of the tensor have left there)
            const bool want = want_mask && splits == 1 && fast && conv_magic_ok(CONV_DGRAD, a);
            bool per_shard;
            a.cut = tile_cut(S, a.Hc * a.Wc, bm, want, &per_shard);
            const int row_tiles = a.cut.blk0[a.cut.p];
            const bool fuse = want && per_shard && mask->sums.floats >= (size_t)2 * a.Nn * row_tiles;
            a.mask_act = fuse ? mask->act : nullptr;
            a.mask_sign = fuse && dtype == 1 && a.Nn % 8 == 0 ? mask->sign : nullptr;
            a.xin = fuse ? mask->xin : nullptr;
            a.mean_rstd = fuse ? mask->mean_rstd : nullptr;
            a.msum = fuse ? mask->sums.buf : nullptr;
            launch_mode<CONV_DGRAD>(dtype, t, dim3(row_tiles, (a.Nn + bn - 1) / bn, splits), a, st);
            if (fuse) left = a.cut;
            if (splits > 1) {
                // a cut reduction: the finishing kernel masks and sums instead of the epilogue
                const bool cut_mask = tune().fused_mask_cut != 0 && want_mask && mask->sums.buf != nullptr && a.Nn % 4 == 0;
                const DgradMask* fm = cut_mask ? mask : nullptr;
                const SumsBuf fs = cut_mask ? mask->sums : SumsBuf{nullptr, 0};
                const int hw = g.H * g.W;
                left = dtype == 1 ? launch_finish<bf16_t>(a, S, hw, splits, fs, st, fm) : launch_finish<float>(a, S, hw, splits, fs, st, fm);
            }
        }
    }
    return left;
}

struct WgradPlan {
    TileCfg t;
    int bm, bn, splits, ksplit;
    int most;         // splits before the cut's length was rounded: no less for a larger shard
    int64_t tiles;
};

// Tile and split of the weight gradient.  Its output is small and its
// reduction (the pixels) long, so parallelism comes from cutting the reduction;
// every split costs a float32 partial tile that is written and read again, so
// layers whose output already gives enough tiles are split little or not at all.
// g.N: samples of the largest shard.  shards: how many of them the launch covers; they are as good as cuts for filling
// the chip and cost no partial tiles (one cut per shard: straight into the worker's gradient).
static WgradPlan plan_wgrad(int dtype, const ConvGeom& g, int shards) {
    WgradPlan p;
    const int M = g.K, Nn = g.R * g.S * g.C, Kred = g.N * g.Ho * g.Wo;
    const int64_t t128 = (int64_t)((M + 127) / 128) * ((Nn + 127) / 128);
    const int64_t t64 = (int64_t)((M + 63) / 64) * ((Nn + 63) / 64);
    if (Nn <= 32) p.t = T128x32;
    else if (dtype != 1 && M <= 32) p.t = T32x128;      // a 64-row tile would contract rows that are not there
    else if (M <= 64 || Nn <= 64) p.t = (Nn <= 64 && M >= 128) ? T128x64 : T64x64;
    else if (t128 >= 128) p.t = T128x128;
    // Few rows that no cut makes enough workgroups of (fully connected layers): four times as many of a quarter of the size
    // (MLP, four shards of 16, 784 -> 256: 56 workgroups 9.4 us, 208 5.5 us).  Not by the number of shards: a pass in parts
    // would then be cut otherwise than the whole.
    else if (t128 * std::max(1, Kred / 256) < 64) p.t = T64x64;
    else if (t64 >= 256 && Kred < 4096) p.t = T64x64;   // long reductions are cut instead (below)
    else p.t = T128x128;
    switch (p.t) {
        case T128x128: p.bm = 128; p.bn = 128; break;
        case T128x64: p.bm = 128; p.bn = 64; break;
        case T128x32: p.bm = 128; p.bn = 32; break;
        case T32x128: p.bm = 32; p.bn = 128; break;
        default: p.bm = 64; p.bn = 64; break;
    }
    p.tiles = (int64_t)((M + p.bm - 1) / p.bm) * ((Nn + p.bn - 1) / p.bn);
    // The weight gradients run beside the input-gradient chain on a second stream: about one workgroup per
    // two CUs leaves that chain the room it needs (ResNet-50 at a shard of 32: 256 -> 128 workgroups, alone on
    // the chip 3% slower per step, beside the main stream 1.4% faster; ResNet-152 1.8%; below 96 the second
    // stream becomes the longer one).
    const int target = (int)tune().wgrad_blocks;
    const int64_t tiles = p.tiles * shards;
    int64_t splits = (target + tiles - 1) / tiles;
    // A long reduction (VGG-16's layers on large images at a shard of 32) is cut into two workgroups per CU
    // (all that are resident at once), as long as each cut keeps long_ks elements: the partial results are
    // small beside the operands there, and a second workgroup hides the operand latency that one per CU
    // leaves exposed.  Measured on VGG-16: 5.28 -> 5.14 ms per step; three per CU (a second, ragged round
    // of workgroups) is slower again.
    const int long_target = (int)tune().wgrad_long_blocks, long_ks = (int)tune().wgrad_long_ks;
    int64_t more = std::min<int64_t>(long_target / tiles, Kred / (long_ks > 0 ? long_ks : 1));
    // float32: a reduction step is sixteen times the matrix work of a bf16 one (no operand latency to hide behind
    // fewer workgroups), so the chip is filled: three workgroups per CU as long as each keeps 256 elements and the
    // partial results stay small (4 MB).  ResNet-20, 8 shards of 16: 790 -> 480 us of weight gradients per step.
    if (dtype != 1) more = std::max(more, std::min<int64_t>(std::min<int64_t>(768 / tiles, Kred / 256), (1 << 20) / ((int64_t)M * Nn * shards)));
    if (more > splits) splits = more;
    const int64_t max_splits = (Kred + 255) / 256;  // at least 4 reduction steps per split
    if (splits > max_splits) splits = max_splits;
    if (splits < 1) splits = 1;
    p.most = (int)splits;
    int64_t ks = (Kred + splits - 1) / splits;
    ks = (ks + 63) / 64 * 64;
    p.ksplit = (int)ks;
    p.splits = (int)((Kred + ks - 1) / ks);
    return p;
}

static size_t wgrad_partial_bytes(const ConvGeom& g, int shards, int splits) {
    return splits <= 1 ? 0 : (size_t)shards * splits * g.K * g.R * g.S * g.C * sizeof(float);
}

size_t conv_wgrad_scratch_bytes(int dtype, const ConvGeom& g, int shards) {
    return wgrad_partial_bytes(g, shards, plan_wgrad(dtype, g, shards).most);
}

size_t conv_wgrad_needs(int dtype, const ConvGeom& g, const ShardSet& S) {
    ConvGeom one = g;
    one.N = S.plan_largest;
    return wgrad_partial_bytes(g, S.p, plan_wgrad(dtype, one, S.plan_p).splits);
}

int conv_wgrad_chain(int dtype, const ConvGeom& g) { return plan_wgrad(dtype, g, 1).ksplit; }

void launch_conv_wgrad(int dtype, const ConvGeom& g, const ShardSet& S, const void* x, const void* dy, GradDst dw, float* scratch,
                       size_t scratch_bytes, hipStream_t st) {
    if (thin_wgrad_takes(dtype, g, S)) {
        launch_thin_wgrad(dtype, g, S, x, dy, dw, st);
        return;
    }
    if (small_wgrad_takes(dtype, g, S)) {
        launch_small_wgrad(g, S, (const float*)x, (const float*)dy, dw, st);
        return;
    }
    const int VEC = dtype == 1 ? 8 : 4;
    ConvGeom one = g;
    one.N = S.plan_largest;
    WgradPlan p = plan_wgrad(dtype, one, S.plan_p);
    ConvArgsShards a = base_args(g);
    a.A = dy; a.B = x;
    a.M = g.K; a.Nn = g.R * g.S * g.C; a.Kred = g.N * g.Ho * g.Wo;
    const double esz = dtype == 1 ? 2.0 : 4.0;
    const double bA = esz * (double)a.Kred * g.K, bB = esz * (double)g.N * g.H * g.W * g.C;
    a.vecA = (g.K % VEC == 0) && bA < 2147483648.0; a.vecB = (g.C % VEC == 0) && bB < 2147483648.0;
    a.bytesA = a.vecA ? (unsigned)bA : 0; a.bytesB = a.vecB ? (unsigned)bB : 0;
    const int64_t n = (int64_t)a.M * a.Nn;
    const bool direct = p.splits <= 1 || scratch == nullptr || scratch_bytes < wgrad_partial_bytes(g, S.p, p.splits);
    if (direct) {
        p.splits = 1;
        p.ksplit = one.N * g.Ho * g.Wo;
    }
    a.ksplit = p.ksplit;
    a.splits = p.splits;
    ConvGeom small = g;
    small.N = S.plan_smallest;
    a.fold = conv_wgrad_chain(dtype, small);     // no longer chains than those of the smallest shard alone
    a.cut = cut_rows(S, g.Ho * g.Wo, p.ksplit);
    a.zdirect = direct;
    // (a kernel with the table of shards finds the worker's gradient itself)
    a.out = direct ? (S.p == 1 && a.ksplit <= a.fold ? dw.g + S.k[0] * dw.stride : dw.g) : scratch;
    a.zstride = direct ? dw.stride : n;
    const dim3 grid((a.M + p.bm - 1) / p.bm, (a.Nn + p.bn - 1) / p.bn, S.p * p.splits);
    launch_mode<CONV_WGRAD>(dtype, p.t, grid, a, st);
    if (!direct) {
        ProfScope ps("wgrad_reduce", 0.0, 4.0 * (double)n * (p.splits + 1) * S.p, st);
        // dw may sit at any float offset of the flat gradient vector: vectors only if it is 16-byte aligned
        const int vec = (n % 4 == 0 && ((uintptr_t)dw.g & 15) == 0 && dw.stride % 4 == 0) ? 4 : 1;
        int64_t blocks = (n / vec + 255) / 256;
        if (blocks > 8192) blocks = 8192;
        const dim3 rgrid((unsigned)blocks, S.p);
        if (vec == 4) hipLaunchKernelGGL(wgrad_reduce_kernel<4>, rgrid, dim3(256), 0, st, scratch, dw.g, dw.stride, S, n, p.splits);
        else hipLaunchKernelGGL(wgrad_reduce_kernel<1>, rgrid, dim3(256), 0, st, scratch, dw.g, dw.stride, S, n, p.splits);
    }
}

}  // namespace edl
