// Pooling and the softmax cross-entropy loss.  All HBM- or latency-bound.
#include "dev_common.h"
#include "kernels.h"
#include "profiler.h"

namespace edl {

static inline int ew_grid(int64_t total) {
    int64_t b = (total + 255) / 256;
    if (b > (1 << 30)) b = 1 << 30;
    if (b < 1) b = 1;
    return (int)b;
}

// ---------------------------------------------------------------------------
// max pool: one lane per output element (channel innermost, so neighbouring
// lanes read neighbouring channels).  arg = r*k + s of the first maximum in
// row-major window order (255 = no tap in range, which cannot happen for the
// geometries used).
// ---------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(256) void maxpool_fwd_kernel(const T* __restrict__ x, T* __restrict__ y,
                                                          uint8_t* __restrict__ arg, int N, int H, int W, int C, int k,
                                                          int stride, int pad, int Ho, int Wo) {
    const int64_t total = (int64_t)N * Ho * Wo * C;
    const int64_t step = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += step) {
        const int c = (int)(i % C);
        int64_t t = i / C;
        const int wo = (int)(t % Wo); t /= Wo;
        const int ho = (int)(t % Ho);
        const int n = (int)(t / Ho);
        float best = 0.f;
        int where = 255;
        for (int r = 0; r < k; ++r) {
            const int h = ho * stride - pad + r;
            if (h < 0 || h >= H) continue;
            for (int s = 0; s < k; ++s) {
                const int w = wo * stride - pad + s;
                if (w < 0 || w >= W) continue;
                const float v = Elem<T>::to_f32(x[(((int64_t)n * H + h) * W + w) * C + c]);
                if (where == 255 || v > best) { best = v; where = r * k + s; }
            }
        }
        y[i] = Elem<T>::from_f32(best);
        arg[i] = (uint8_t)where;
    }
}

// gather form of the backward: an input element collects dy from every window
// that recorded it as its arg-max (no atomics, deterministic)
template <typename T>
__global__ __launch_bounds__(256) void maxpool_bwd_kernel(const T* __restrict__ dy, const uint8_t* __restrict__ arg,
                                                          T* dx, int accumulate, int N, int H, int W, int C, int k,
                                                          int stride, int pad, int Ho, int Wo) {
    const int64_t total = (int64_t)N * H * W * C;
    const int64_t step = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += step) {
        const int c = (int)(i % C);
        int64_t t = i / C;
        const int w = (int)(t % W); t /= W;
        const int h = (int)(t % H);
        const int n = (int)(t / H);
        float g = 0.f;
        for (int r = 0; r < k; ++r) {
            const int hn = h + pad - r;
            if (hn < 0 || hn % stride) continue;
            const int ho = hn / stride;
            if (ho >= Ho) continue;
            for (int s = 0; s < k; ++s) {
                const int wn = w + pad - s;
                if (wn < 0 || wn % stride) continue;
                const int wo = wn / stride;
                if (wo >= Wo) continue;
                const int64_t o = (((int64_t)n * Ho + ho) * Wo + wo) * C + c;
                if (arg[o] == r * k + s) g += Elem<T>::to_f32(dy[o]);
            }
        }
        if (accumulate) g += Elem<T>::to_f32(dx[i]);
        dx[i] = Elem<T>::from_f32(g);
    }
}

// Work items of the vector kernels below: blocks of 256 channel vectors of one image row, so that only the vector's
// place within the row is divided per lane (by a shift for the usual channel counts), in 32 bits; the row and image are
// uniform.  With one flat 64-bit index the divisions took longer than the memory (VGG-16's pools at a shard of 32: 182
// us backward and 110 us forward per step).
struct RowItems { int per_row, vecs, cv, cv_shift; };     // blocks per row, vectors per row, vectors per pixel, log2 or -1
static RowItems row_items(int W, int C, int vec) {
    RowItems r;
    r.cv = C / vec;
    r.vecs = W * r.cv;
    r.per_row = (r.vecs + 255) / 256;
    r.cv_shift = -1;
    for (int k = 0; k < 16; ++k)
        if (r.cv == 1 << k) r.cv_shift = k;
    return r;
}
// A die gets a contiguous run of blocks: rows that several windows read stay in its L2 (forward, 256 images of 112x112x64 in windows of
// 3x3: 153 us with neighbours on different dies, 136 so).
__device__ __forceinline__ int block_of_die() {
    const int q = gridDim.x >> 3, r = gridDim.x & 7, die = blockIdx.x & 7;
    return die * q + min(die, r) + (blockIdx.x >> 3);
}
// row of the image stack, pixel and first vector of this lane; false for the lanes past the row's end
__device__ __forceinline__ bool locate_vector(const RowItems& r, int& row, int& pixel, int& cvec) {
    const int block = block_of_die();
    row = block / r.per_row;
    const int v = (block - row * r.per_row) * 256 + threadIdx.x;
    pixel = r.cv_shift >= 0 ? v >> r.cv_shift : v / r.cv;
    cvec = v - pixel * r.cv;
    return v < r.vecs;
}

// 16-byte channel vectors per lane (C a multiple of the vector width); window size and stride known at compile time
// (KK = 0: not), so that all of a window's loads are in flight together
template <typename T, int KK>
__global__ __launch_bounds__(256) void maxpool_fwd_vec_kernel(const T* __restrict__ x, T* __restrict__ y,
                                                              uint8_t* __restrict__ arg, RowItems items, int H, int W, int C, int kk,
                                                              int stride, int pad, int Ho, int Wo) {
    constexpr int VEC = Elem<T>::VEC;
    const int k = KK > 0 ? KK : kk;
    int row, wo, cvec;
    if (!locate_vector(items, row, wo, cvec)) return;
    const int n = row / Ho, ho = row - n * Ho, c0 = cvec * VEC;
    float best[VEC];
    int where[VEC];
    #pragma unroll
    for (int e = 0; e < VEC; ++e) { best[e] = 0.f; where[e] = 255; }
    const int h0 = ho * stride - pad, w0 = wo * stride - pad;
    auto tap = [&](const Vec16<T>& v, int t) {
        #pragma unroll
        for (int e = 0; e < VEC; ++e) {
            const float f = Elem<T>::to_f32(v.e[e]);
            if (where[e] == 255 || f > best[e]) { best[e] = f; where[e] = t; }
        }
    };
    if (KK > 0) {
        Vec16<T> v[KK > 0 ? KK * KK : 1];
        #pragma unroll
        for (int r = 0; r < KK; ++r)
            #pragma unroll
            for (int s = 0; s < KK; ++s) {      // a tap outside the image reads the nearest pixel and is ignored
                const int h = min(max(h0 + r, 0), H - 1), w = min(max(w0 + s, 0), W - 1);
                v[r * KK + s] = load_vec(x + ((int64_t)(n * H + h) * W + w) * C + c0);
            }
        #pragma unroll
        for (int r = 0; r < KK; ++r)
            #pragma unroll
            for (int s = 0; s < KK; ++s)
                if ((unsigned)(h0 + r) < (unsigned)H && (unsigned)(w0 + s) < (unsigned)W) tap(v[r * KK + s], r * KK + s);
    } else {
        for (int r = 0; r < k; ++r)
            for (int s = 0; s < k; ++s)
                if ((unsigned)(h0 + r) < (unsigned)H && (unsigned)(w0 + s) < (unsigned)W)
                    tap(load_vec(x + ((int64_t)(n * H + h0 + r) * W + w0 + s) * C + c0), r * k + s);
    }
    const int64_t o = ((int64_t)row * Wo + wo) * C + c0;
    Vec16<T> out;
    uint8_t am[VEC];
    #pragma unroll
    for (int e = 0; e < VEC; ++e) { out.e[e] = Elem<T>::from_f32(best[e]); am[e] = (uint8_t)where[e]; }
    if (VEC == 8) *reinterpret_cast<uint2*>(arg + o) = *reinterpret_cast<const uint2*>(am);
    else *reinterpret_cast<uint32_t*>(arg + o) = *reinterpret_cast<const uint32_t*>(am);
    store_vec(y + o, out);
}

template <typename T>
__global__ __launch_bounds__(256) void maxpool_bwd_vec_kernel(const T* __restrict__ dy, const uint8_t* __restrict__ arg,
                                                              T* dx, int accumulate, int N, int H, int W, int C, int k,
                                                              int stride, int pad, int Ho, int Wo) {
    constexpr int VEC = Elem<T>::VEC;
    const int cv = C / VEC;
    const int64_t total = (int64_t)N * H * W * cv;
    const int64_t step = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += step) {
        const int c0 = (int)(i % cv) * VEC;
        int64_t t = i / cv;
        const int w = (int)(t % W); t /= W;
        const int h = (int)(t % H);
        const int n = (int)(t / H);
        float g[VEC];
        #pragma unroll
        for (int e = 0; e < VEC; ++e) g[e] = 0.f;
        for (int r = 0; r < k; ++r) {
            const int hn = h + pad - r;
            if (hn < 0 || hn % stride) continue;
            const int ho = hn / stride;
            if (ho >= Ho) continue;
            for (int s = 0; s < k; ++s) {
                const int wn = w + pad - s;
                if (wn < 0 || wn % stride) continue;
                const int wo = wn / stride;
                if (wo >= Wo) continue;
                const int64_t o = (((int64_t)n * Ho + ho) * Wo + wo) * C + c0;
                const Vec16<T> v = load_vec(dy + o);
                uint8_t am[VEC];
                if (VEC == 8) *reinterpret_cast<uint2*>(am) = *reinterpret_cast<const uint2*>(arg + o);
                else *reinterpret_cast<uint32_t*>(am) = *reinterpret_cast<const uint32_t*>(arg + o);
                #pragma unroll
                for (int e = 0; e < VEC; ++e)
                    if (am[e] == r * k + s) g[e] += Elem<T>::to_f32(v.e[e]);
            }
        }
        const int64_t xo = (((int64_t)n * H + h) * W + w) * C + c0;
        if (accumulate) {
            const Vec16<T> old = load_vec(dx + xo);
            #pragma unroll
            for (int e = 0; e < VEC; ++e) g[e] += Elem<T>::to_f32(old.e[e]);
        }
        Vec16<T> out;
        #pragma unroll
        for (int e = 0; e < VEC; ++e) out.e[e] = Elem<T>::from_f32(g[e]);
        store_vec(dx + xo, out);
    }
}

// The backward of a pool of 3x3 windows with stride 2: a lane has the square of (up to) four pixels that the same four windows reach
// - rows h + pad = 2 i - 1 and 2 i, from windows i - 1 and i, and so with the columns - so that four loads of each of the pooled tensors
// serve four pixels; pixel by pixel they were read sixteen times.  MASK: as below, and since a window's gradient goes to the pixel
// whose value the pool's output is, the ReLU's sign is read from that output, a quarter of the activation's bytes.
// SUMS: the producer is a batch norm, whose own gradients are sums over what is stored here and its input: they are left as
// column sums (DgradMask's), and its pass over both falls away.
// Measured (256 images of 112x112x64 in bf16, with the mask): 233 us, and 179 for the sums, before; 225 for all of it now (1.08 GB at
// 4.8 TB/s; held to 128 registers instead of 153 it spills and takes 583).  Without sums, AlexNet's three at 128 images: 73 us before, 54 now.
struct PoolQuads {
    int H, W, Ho, Wo, pad, cv, C;
    int i0, j0, cols, quads;      // first row and column of squares, squares per row and per image
    int groups, per_group;        // blocks per image, squares of each
};
template <typename T, bool MASK, bool SUMS>
__global__ __launch_bounds__(256) void maxpool_bwd_quad_kernel(const T* __restrict__ dy, const uint8_t* __restrict__ arg, T* __restrict__ dx,
                                                               const T* __restrict__ pooled, const T* __restrict__ xin,
                                                               const float* __restrict__ mean_rstd, float* __restrict__ sums, RowCut cut, PoolQuads a) {
    constexpr int VEC = Elem<T>::VEC;
    __shared__ float red[SUMS ? 2 * VEC : 1][SUMS ? 256 : 1];
    const int block = block_of_die();
    const int tid = threadIdx.x, n = block / a.groups, group = block - n * a.groups;
    const int side = 256 / a.cv, mine = tid / a.cv, c0 = (tid - mine * a.cv) * VEC;       // squares at a time, this lane's among them
    const int first = group * a.per_group, end = min(first + a.per_group, a.quads);
    float mu[VEC], rs[VEC], s1[VEC], s2[VEC];
    #pragma unroll
    for (int e = 0; e < VEC; ++e) { mu[e] = rs[e] = s1[e] = s2[e] = 0.f; }
    if (SUMS) {
        const float* const ms = mean_rstd + (size_t)shard_of_block(cut, block) * 2 * a.C + c0;
        #pragma unroll
        for (int e = 0; e < VEC; ++e) { mu[e] = ms[e]; rs[e] = ms[a.C + e]; }
    }
    for (int q = first + mine; q < end && mine < side; q += side) {
        const int iq = q / a.cols, i = a.i0 + iq, j = a.j0 + q - iq * a.cols;
        Vec16<T> v[2][2], sign[2][2], x[2][2];
        uint8_t am[2][2][VEC];
        int64_t to[2][2];
        bool in[2][2], ok[2][2];
        #pragma unroll
        for (int r = 0; r < 2; ++r)
            #pragma unroll
            for (int s = 0; s < 2; ++s) {
                const int ho = i - 1 + r, wo = j - 1 + s;       // window, and the square's pixel
                ok[r][s] = ho >= 0 && wo >= 0 && ho < a.Ho && wo < a.Wo;
                const int64_t o = ok[r][s] ? (((int64_t)n * a.Ho + ho) * a.Wo + wo) * a.C + c0 : c0;
                v[r][s] = load_vec(dy + o);
                if (VEC == 8) *reinterpret_cast<uint2*>(am[r][s]) = *reinterpret_cast<const uint2*>(arg + o);
                else *reinterpret_cast<uint32_t*>(am[r][s]) = *reinterpret_cast<const uint32_t*>(arg + o);
                if (MASK) sign[r][s] = load_vec(pooled + o);
                const int h = 2 * i - 1 + r - a.pad, w = 2 * j - 1 + s - a.pad;
                in[r][s] = h >= 0 && w >= 0 && h < a.H && w < a.W;
                to[r][s] = in[r][s] ? (((int64_t)n * a.H + h) * a.W + w) * a.C + c0 : c0;
                if (SUMS) x[r][s] = load_vec(xin + to[r][s]);
            }
        Vec16<T> out[2][2];
        #pragma unroll
        for (int e = 0; e < VEC; ++e) {
            float g[2][2];
            int t[2][2];
            #pragma unroll
            for (int r = 0; r < 2; ++r)
                #pragma unroll
                for (int s = 0; s < 2; ++s) {
                    g[r][s] = Elem<T>::to_f32(v[r][s].e[e]) + 0.f;       // (-0 goes as 0)
                    t[r][s] = ok[r][s] && (!MASK || Elem<T>::to_f32(sign[r][s].e[e]) > 0.f) ? am[r][s][e] : 255;
                }
            // a pixel's windows in the order of the kernel below: the later row first, in it the later column
            float d[2][2];
            d[0][0] = t[0][0] == 4 ? g[0][0] : 0.f;
            d[0][1] = (t[0][1] == 3 ? g[0][1] : 0.f) + (t[0][0] == 5 ? g[0][0] : 0.f);
            d[1][0] = (t[1][0] == 1 ? g[1][0] : 0.f) + (t[0][0] == 7 ? g[0][0] : 0.f);
            d[1][1] = (((t[1][1] == 0 ? g[1][1] : 0.f) + (t[1][0] == 2 ? g[1][0] : 0.f)) + (t[0][1] == 6 ? g[0][1] : 0.f)) + (t[0][0] == 8 ? g[0][0] : 0.f);
            #pragma unroll
            for (int r = 0; r < 2; ++r)
                #pragma unroll
                for (int s = 0; s < 2; ++s) {
                    out[r][s].e[e] = Elem<T>::from_f32(d[r][s]);
                    if (SUMS) {
                        const float stored = in[r][s] ? Elem<T>::to_f32(out[r][s].e[e]) : 0.f;
                        s1[e] += stored;
                        s2[e] += in[r][s] ? stored * ((Elem<T>::to_f32(x[r][s].e[e]) - mu[e]) * rs[e]) : 0.f;
                    }
                }
        }
        #pragma unroll
        for (int r = 0; r < 2; ++r)
            #pragma unroll
            for (int s = 0; s < 2; ++s)
                if (in[r][s]) store_vec(dx + to[r][s], out[r][s]);
    }
    if (!SUMS) return;
    #pragma unroll
    for (int e = 0; e < VEC; ++e) { red[e][tid] = s1[e]; red[VEC + e][tid] = s2[e]; }
    __syncthreads();
    for (int o = tid; o < 2 * a.C; o += 256) {
        const int kind = o / a.C, c = o - kind * a.C;
        double s = 0.0;      // (as the pass of sums: float32 chains of 16 terms, float64 across lanes)
        for (int l = 0; l < side; ++l) s += (double)red[kind * VEC + c % VEC][l * a.cv + c / VEC];
        sums[(size_t)o * gridDim.x + block] = (float)s;
    }
}

// The same with the window positions that can reach an input pixel enumerated without branches: at most
// NC = ceil(k / stride) per dimension.  All NC*NC loads are issued before the first use (a position outside
// the output reads a clamped one and is ignored), instead of one load and one wait per tap.
// MASK: the pooled tensor is the output of a ReLU; the gradient is stored already multiplied by (act > 0),
// so that the producer's backward need not read its activation again.  The pixel a window picked holds the window's
// maximum: where a pixel has one window (NC = 1) the sign comes from the pooled value, a quarter of the bytes of the
// activation; with several it is one load of the activation.
template <typename T, int NC, bool MASK>
__global__ __launch_bounds__(256) void maxpool_bwd_win_kernel(const T* __restrict__ dy, const uint8_t* __restrict__ arg,
                                                              T* dx, const T* __restrict__ act, const T* __restrict__ pooled, int accumulate,
                                                              RowItems items, int H, int W, int C, int k, int stride, int pad, int Ho, int Wo) {
    constexpr int VEC = Elem<T>::VEC;
    int row, w, cvec;
    if (!locate_vector(items, row, w, cvec)) return;
    const int n = row / H, h = row - n * H, c0 = cvec * VEC;
    // output rows ho with ho*stride - pad <= h < ho*stride - pad + k: ho in [ho_hi - NC + 1, ho_hi]
    const int ho_hi = (h + pad) / stride, wo_hi = (w + pad) / stride;
    Vec16<T> v[NC][NC];
    uint8_t am[NC][NC][VEC];
    bool ok[NC][NC];
    int tap[NC][NC];
    Vec16<T> old, sign;
    #pragma unroll
    for (int a = 0; a < NC; ++a) {
        #pragma unroll
        for (int b = 0; b < NC; ++b) {
            const int ho = ho_hi - a, wo = wo_hi - b;
            const int r = h + pad - ho * stride, s2 = w + pad - wo * stride;      // tap of this pixel in that window
            ok[a][b] = ho >= 0 && wo >= 0 && ho < Ho && wo < Wo && r < k && s2 < k;
            tap[a][b] = r * k + s2;
            const int hc = ho < 0 ? 0 : (ho >= Ho ? Ho - 1 : ho), wc = wo < 0 ? 0 : (wo >= Wo ? Wo - 1 : wo);
            const int64_t o = ((int64_t)(n * Ho + hc) * Wo + wc) * C + c0;
            v[a][b] = load_vec(dy + o);
            if (VEC == 8) *reinterpret_cast<uint2*>(am[a][b]) = *reinterpret_cast<const uint2*>(arg + o);
            else *reinterpret_cast<uint32_t*>(am[a][b]) = *reinterpret_cast<const uint32_t*>(arg + o);
            if (MASK && NC == 1) sign = load_vec(pooled + o);
        }
    }
    const int64_t xo = ((int64_t)row * W + w) * C + c0;
    old.u = make_uint4(0, 0, 0, 0);
    if (accumulate) old = load_vec(dx + xo);
    if (MASK && NC > 1) sign = load_vec(act + xo);
    float g[VEC];
    #pragma unroll
    for (int e = 0; e < VEC; ++e) g[e] = 0.f;
    // taps in the order of the kernel above (r ascending, then s): the tap grows with a and b
    #pragma unroll
    for (int a = 0; a < NC; ++a) {
        #pragma unroll
        for (int b = 0; b < NC; ++b) {
            #pragma unroll
            for (int e = 0; e < VEC; ++e)
                if (ok[a][b] && am[a][b][e] == tap[a][b]) g[e] += Elem<T>::to_f32(v[a][b].e[e]);
        }
    }
    if (accumulate) {
        #pragma unroll
        for (int e = 0; e < VEC; ++e) g[e] += Elem<T>::to_f32(old.e[e]);
    }
    Vec16<T> out;
    #pragma unroll
    for (int e = 0; e < VEC; ++e) out.e[e] = Elem<T>::from_f32((!MASK || Elem<T>::to_f32(sign.e[e]) > 0.f) ? g[e] : 0.f);
    store_vec(dx + xo, out);
}

void launch_maxpool_forward(int dtype, const void* x, void* y, uint8_t* arg, int N, int H, int W, int C, int k,
                            int stride, int pad, int Ho, int Wo, hipStream_t st) {
    const int grid = ew_grid((int64_t)N * Ho * Wo * C);
    const double esz = dtype == 1 ? 2.0 : 4.0;
    ProfScope ps("maxpool_fwd", 0.0, esz * (double)N * H * W * C + (esz + 1.0) * (double)N * Ho * Wo * C, st);
    const int vec = dtype == 1 ? 8 : 4;
    const RowItems items = row_items(Wo, C, vec);
    if (C % vec == 0 && (double)N * Ho * items.per_row < 2147483648.0) {
        const dim3 vgrid((unsigned)(N * Ho * items.per_row));
#define EDL_POOL_FWD(TT, KK)                                                                                             \
    hipLaunchKernelGGL((maxpool_fwd_vec_kernel<TT, KK>), vgrid, dim3(256), 0, st, (const TT*)x, (TT*)y, arg, items, H, W, C, k, \
                       stride, pad, Ho, Wo)
        if (dtype == 1) { if (k == 2) EDL_POOL_FWD(bf16_t, 2); else if (k == 3) EDL_POOL_FWD(bf16_t, 3); else EDL_POOL_FWD(bf16_t, 0); }
        else { if (k == 2) EDL_POOL_FWD(float, 2); else if (k == 3) EDL_POOL_FWD(float, 3); else EDL_POOL_FWD(float, 0); }
#undef EDL_POOL_FWD
        return;
    }
    if (dtype == 1)
        hipLaunchKernelGGL(maxpool_fwd_kernel<bf16_t>, dim3(grid), dim3(256), 0, st, (const bf16_t*)x, (bf16_t*)y, arg, N,
                           H, W, C, k, stride, pad, Ho, Wo);
    else
        hipLaunchKernelGGL(maxpool_fwd_kernel<float>, dim3(grid), dim3(256), 0, st, (const float*)x, (float*)y, arg, N, H,
                           W, C, k, stride, pad, Ho, Wo);
}

// The squares' kernel, for a pool that it takes (launch_maxpool_backward).  A block has four rounds of squares, fewer where that
// leaves less than eight blocks per CU.
static RowCut launch_maxpool_quads(int dtype, const void* dy, const uint8_t* arg, void* dx, const ShardSet& S, int H, int W, int C, int pad,
                                   int Ho, int Wo, const DgradMask* mask, const void* relu_pooled, hipStream_t st) {
    const int vec = dtype == 1 ? 8 : 4;
    PoolQuads a = {H, W, Ho, Wo, pad, C / vec, C, pad, pad, (W + pad) / 2 - pad + 1, 0, 0, 0};
    a.quads = ((H + pad) / 2 - pad + 1) * a.cols;
    const int side = 256 / a.cv, rounds = (a.quads + side - 1) / side;
    const int64_t all = (int64_t)S.plan * rounds;
    a.per_group = side * (int)std::max<int64_t>(1, std::min<int64_t>(4, all / 2048));
    a.groups = (a.quads + a.per_group - 1) / a.per_group;
    RowCut cut;
    const int blocks = S.samples() * a.groups;
    const bool masked = mask != nullptr, sums = masked && mask->xin != nullptr && mask->sums.buf != nullptr && mask->sums.floats >= (size_t)2 * C * blocks;
    if (sums) {      // (blocks of squares, not of rows; who reads the sums goes by the blocks of each shard)
        cut = cut_rows(S, H * W, H * W);
        for (int s = 0; s <= S.p; ++s) cut.blk0[s] = S.off[s] * a.groups;
        cut.most = S.plan_largest * a.groups;
    }
    const double esz = dtype == 1 ? 2.0 : 4.0, N = S.samples();
    ProfScope ps(sums ? "maxpool_bwd_sums" : "maxpool_bwd", 0.0, esz * N * H * W * C * (sums ? 2.0 : 1.0) + (esz * (masked ? 2.0 : 1.0) + 1.0) * N * Ho * Wo * C, st);
#define EDL_POOL_QUADS(TT, MM, SS)                                                                                                  \
    hipLaunchKernelGGL((maxpool_bwd_quad_kernel<TT, MM, SS>), dim3(blocks), dim3(256), 0, st, (const TT*)dy, arg, (TT*)dx, (const TT*)relu_pooled, \
                       (const TT*)(sums ? mask->xin : nullptr), sums ? mask->mean_rstd : nullptr, sums ? mask->sums.buf : nullptr, cut, a)
    if (dtype == 1) { if (sums) EDL_POOL_QUADS(bf16_t, true, true); else if (masked) EDL_POOL_QUADS(bf16_t, true, false); else EDL_POOL_QUADS(bf16_t, false, false); }
    else { if (sums) EDL_POOL_QUADS(float, true, true); else if (masked) EDL_POOL_QUADS(float, true, false); else EDL_POOL_QUADS(float, false, false); }
#undef EDL_POOL_QUADS
    return cut;
}

bool launch_maxpool_backward(int dtype, const void* dy, const uint8_t* arg, void* dx, bool accumulate, const ShardSet& S, int H,
                             int W, int C, int k, int stride, int pad, int Ho, int Wo, const DgradMask* mask, const void* relu_pooled, RowCut* sums,
                             hipStream_t st) {
    const int N = S.samples();
    const int grid = ew_grid((int64_t)N * H * W * C);
    const double esz = dtype == 1 ? 2.0 : 4.0;
    const int vec = dtype == 1 ? 8 : 4;
    const void* const relu_act = mask != nullptr ? mask->act : nullptr;
    // (pad 0 or 1: every window starts inside the image or one before it; up to 256 vectors per pixel; blocks counted in 31 bits)
    if (k == 3 && stride == 2 && pad <= 1 && !accumulate && C % vec == 0 && C / vec <= 256 && (double)N * H * W < 2147483648.0) {
        *sums = launch_maxpool_quads(dtype, dy, arg, dx, S, H, W, C, pad, Ho, Wo, relu_act != nullptr ? mask : nullptr, relu_pooled, st);
        return relu_act != nullptr;
    }
    const int nc = (k + stride - 1) / stride;
    const RowItems items = row_items(W, C, vec);
    const bool win = C % vec == 0 && nc <= 2 && (double)N * H * items.per_row < 2147483648.0;
    const bool masked = win && relu_act != nullptr && !accumulate;
    ProfScope ps("maxpool_bwd", 0.0, esz * (double)N * H * W * C * ((accumulate ? 2.0 : 1.0) + (masked && nc > 1 ? 1.0 : 0.0)) +
                                       (esz * (masked && nc == 1 ? 2.0 : 1.0) + 1.0) * (double)N * Ho * Wo * C, st);
    if (C % vec == 0) {
        const int vgrid = ew_grid((int64_t)N * H * W * (C / vec));
        if (win) {
            const dim3 g1((unsigned)(N * H * items.per_row));
#define EDL_POOL_BWD(TT, NCC, MM)                                                                                               \
    hipLaunchKernelGGL((maxpool_bwd_win_kernel<TT, NCC, MM>), g1, dim3(256), 0, st, (const TT*)dy, arg, (TT*)dx, (const TT*)relu_act, \
                       (const TT*)relu_pooled, accumulate ? 1 : 0, items, H, W, C, k, stride, pad, Ho, Wo)
            if (dtype == 1) {
                if (nc == 1) { if (masked) EDL_POOL_BWD(bf16_t, 1, true); else EDL_POOL_BWD(bf16_t, 1, false); }
                else { if (masked) EDL_POOL_BWD(bf16_t, 2, true); else EDL_POOL_BWD(bf16_t, 2, false); }
            } else {
                if (nc == 1) { if (masked) EDL_POOL_BWD(float, 1, true); else EDL_POOL_BWD(float, 1, false); }
                else { if (masked) EDL_POOL_BWD(float, 2, true); else EDL_POOL_BWD(float, 2, false); }
            }
#undef EDL_POOL_BWD
            return masked;
        }
        if (dtype == 1)
            hipLaunchKernelGGL(maxpool_bwd_vec_kernel<bf16_t>, dim3(vgrid), dim3(256), 0, st, (const bf16_t*)dy, arg,
                               (bf16_t*)dx, accumulate ? 1 : 0, N, H, W, C, k, stride, pad, Ho, Wo);
        else
            hipLaunchKernelGGL(maxpool_bwd_vec_kernel<float>, dim3(vgrid), dim3(256), 0, st, (const float*)dy, arg, (float*)dx,
                               accumulate ? 1 : 0, N, H, W, C, k, stride, pad, Ho, Wo);
        return false;
    }
    if (dtype == 1)
        hipLaunchKernelGGL(maxpool_bwd_kernel<bf16_t>, dim3(grid), dim3(256), 0, st, (const bf16_t*)dy, arg, (bf16_t*)dx,
                           accumulate ? 1 : 0, N, H, W, C, k, stride, pad, Ho, Wo);
    else
        hipLaunchKernelGGL(maxpool_bwd_kernel<float>, dim3(grid), dim3(256), 0, st, (const float*)dy, arg, (float*)dx,
                           accumulate ? 1 : 0, N, H, W, C, k, stride, pad, Ho, Wo);
    return false;
}

// ---------------------------------------------------------------------------
// global average pool: y[n][c] = mean over the HW pixels
// ---------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(256) void gavgpool_fwd_kernel(const T* __restrict__ x, T* __restrict__ y, int N, int HW, int C) {
    const int64_t total = (int64_t)N * C;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (int64_t)gridDim.x * blockDim.x) {
        const int c = (int)(i % C);
        const int64_t n = i / C;
        float s = 0.f;
        for (int q = 0; q < HW; ++q) s += Elem<T>::to_f32(x[(n * HW + q) * C + c]);
        y[i] = Elem<T>::from_f32(s / (float)HW);
    }
}

// The same on 16-byte vectors of channels: a block takes 64 channel vectors of one sample, its four
// quarter-blocks every fourth pixel each, and the four partial sums meet in LDS (a fixed order).
template <typename T>
__global__ __launch_bounds__(256) void gavgpool_fwd_vec_kernel(const T* __restrict__ x, T* __restrict__ y, int HW, int C) {
    constexpr int VEC = Elem<T>::VEC;
    __shared__ float part[3][64][VEC + 1];
    const int lane = threadIdx.x >> 6;
    const int cv = blockIdx.x * 64 + (threadIdx.x & 63);
    const int64_t n = blockIdx.y;
    const bool live = cv * VEC < C;
    float s[VEC];
#pragma unroll
    for (int j = 0; j < VEC; ++j) s[j] = 0.f;
    if (live) {
        const T* base = x + n * HW * C + (int64_t)cv * VEC;
#pragma unroll 4
        for (int q = lane; q < HW; q += 4) {
            const Vec16<T> v = load_vec(base + (int64_t)q * C);
#pragma unroll
            for (int j = 0; j < VEC; ++j) s[j] += Elem<T>::to_f32(v.e[j]);
        }
    }
    if (lane > 0) {
#pragma unroll
        for (int j = 0; j < VEC; ++j) part[lane - 1][threadIdx.x & 63][j] = s[j];
    }
    __syncthreads();
    if (lane == 0 && live) {
        Vec16<T> o;
#pragma unroll
        for (int j = 0; j < VEC; ++j) {
            const float t = ((s[j] + part[0][threadIdx.x][j]) + part[1][threadIdx.x][j]) + part[2][threadIdx.x][j];
            o.e[j] = Elem<T>::from_f32(t / (float)HW);
        }
        store_vec(y + n * C + (int64_t)cv * VEC, o);
    }
}

template <typename T>
__global__ __launch_bounds__(256) void gavgpool_bwd_kernel(const T* __restrict__ dy, T* dx, int accumulate, int N, int HW,
                                                           int C) {
    const int64_t total = (int64_t)N * HW * C;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (int64_t)gridDim.x * blockDim.x) {
        const int c = (int)(i % C);
        const int64_t n = i / ((int64_t)HW * C);
        float g = Elem<T>::to_f32(dy[n * C + c]) / (float)HW;
        if (accumulate) g += Elem<T>::to_f32(dx[i]);
        dx[i] = Elem<T>::from_f32(g);
    }
}

void launch_gavgpool_forward(int dtype, const void* x, void* y, int N, int HW, int C, hipStream_t st) {
    const int grid = ew_grid((int64_t)N * C);
    ProfScope ps("gavgpool_fwd", 0.0, (dtype == 1 ? 2.0 : 4.0) * (double)N * (HW + 1) * C, st);
    const int vec = dtype == 1 ? 8 : 4;
    const bool aligned = ((uintptr_t)x | (uintptr_t)y) % 16 == 0;
    if (C % vec == 0 && aligned && N >= 1 && N <= 65535) {
        const dim3 vgrid((unsigned)((C / vec + 63) / 64), (unsigned)N);
        if (dtype == 1)
            hipLaunchKernelGGL(gavgpool_fwd_vec_kernel<bf16_t>, vgrid, dim3(256), 0, st, (const bf16_t*)x, (bf16_t*)y, HW, C);
        else
            hipLaunchKernelGGL(gavgpool_fwd_vec_kernel<float>, vgrid, dim3(256), 0, st, (const float*)x, (float*)y, HW, C);
    } else if (dtype == 1)
        hipLaunchKernelGGL(gavgpool_fwd_kernel<bf16_t>, dim3(grid), dim3(256), 0, st, (const bf16_t*)x, (bf16_t*)y, N, HW, C);
    else
        hipLaunchKernelGGL(gavgpool_fwd_kernel<float>, dim3(grid), dim3(256), 0, st, (const float*)x, (float*)y, N, HW, C);
}

void launch_gavgpool_backward(int dtype, const void* dy, void* dx, bool accumulate, int N, int HW, int C,
                              hipStream_t st) {
    const int grid = ew_grid((int64_t)N * HW * C);
    ProfScope ps("gavgpool_bwd", 0.0, (dtype == 1 ? 2.0 : 4.0) * (double)N * (HW + 1) * C, st);
    if (dtype == 1)
        hipLaunchKernelGGL(gavgpool_bwd_kernel<bf16_t>, dim3(grid), dim3(256), 0, st, (const bf16_t*)dy, (bf16_t*)dx,
                           accumulate ? 1 : 0, N, HW, C);
    else
        hipLaunchKernelGGL(gavgpool_bwd_kernel<float>, dim3(grid), dim3(256), 0, st, (const float*)dy, (float*)dx,
                           accumulate ? 1 : 0, N, HW, C);
}

// ---------------------------------------------------------------------------
// softmax cross-entropy: one workgroup per sample.  loss_i = log(sum exp(z -
// max)) - (z_label - max); dz = (softmax - onehot) / n.
// ---------------------------------------------------------------------------
__device__ __forceinline__ float block_reduce(float v, float* sm, bool is_max) {
    for (int o = 32; o > 0; o >>= 1) {
        const float other = __shfl_xor(v, o, 64);
        v = is_max ? fmaxf(v, other) : v + other;
    }
    const int wave = threadIdx.x >> 6;
    __syncthreads();
    if ((threadIdx.x & 63) == 0) sm[wave] = v;
    __syncthreads();
    float r = sm[0];
    for (int i = 1; i < (int)(blockDim.x >> 6); ++i) r = is_max ? fmaxf(r, sm[i]) : r + sm[i];
    return r;
}

template <typename T>
__global__ __launch_bounds__(256) void softmax_ce_kernel(const float* __restrict__ logits, const int32_t* __restrict__ labels,
                                                         T* __restrict__ dlogits, float* __restrict__ row_loss, RowCut shards, int C) {
    __shared__ float sm[4];
    const int i = blockIdx.x;
    const int sh = shard_of_block(shards, i);        // one block per sample
    const int n = shards.row0[sh + 1] - shards.row0[sh];
    const float* z = logits + (int64_t)i * C;
    float mx = -INFINITY;
    for (int c = threadIdx.x; c < C; c += blockDim.x) mx = fmaxf(mx, z[c]);
    mx = block_reduce(mx, sm, true);
    float s = 0.f;
    for (int c = threadIdx.x; c < C; c += blockDim.x) s += expf(z[c] - mx);
    s = block_reduce(s, sm, false);
    const int label = labels[i];
    const float inv = 1.f / s, invn = 1.f / (float)n;
    for (int c = threadIdx.x; c < C; c += blockDim.x) {
        const float pr = expf(z[c] - mx) * inv;
        dlogits[(int64_t)i * C + c] = Elem<T>::from_f32((pr - (c == label ? 1.f : 0.f)) * invn);
    }
    if (threadIdx.x == 0) row_loss[i] = logf(s) - (z[label] - mx);
}

// mean of the per-sample losses of each shard, summed in sample order by one wave; grid: shards
__global__ void loss_mean_kernel(const float* __restrict__ row_loss, ShardSet S, float* __restrict__ out) {
    const int lo = S.off[blockIdx.x], hi = S.off[blockIdx.x + 1];
    float s = 0.f;
    for (int i = lo + threadIdx.x; i < hi; i += 64) s += row_loss[i];
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
    if (threadIdx.x == 0) out[S.k[blockIdx.x]] = s / (float)(hi - lo);
}

// The same for small shards and few classes, the means included: a workgroup per shard, a wave per row, a lane per class.  As two
// launches (a block per row, then the means) it took 8 us of an MLP's 64 us chain, so 4.
constexpr int kSmallClasses = 64, kSmallLossRows = 64;
template <typename T>
__global__ __launch_bounds__(1024) void softmax_ce_small_kernel(const float* __restrict__ logits, const int32_t* __restrict__ labels,
                                                                T* __restrict__ dlogits, float* __restrict__ row_loss, ShardSet S, int C,
                                                                float* __restrict__ out) {
    __shared__ float loss[kSmallLossRows];
    const int lo = S.off[blockIdx.x], n = S.off[blockIdx.x + 1] - lo;
    const int lane = threadIdx.x & 63;
    const bool live = lane < C;
    const float invn = 1.f / (float)n;
    for (int r = threadIdx.x >> 6; r < n; r += 16) {
        const int i = lo + r;
        const float z = live ? logits[(int64_t)i * C + lane] : -INFINITY;
        const int label = labels[i];
        float mx = z;
        for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o, 64));
        const float e = live ? expf(z - mx) : 0.f;
        float s = e;
        for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
        const float inv = 1.f / s;
        if (live) dlogits[(int64_t)i * C + lane] = Elem<T>::from_f32((e * inv - (lane == label ? 1.f : 0.f)) * invn);
        const float zl = __shfl(z, label, 64);
        if (lane == 0) {
            const float l = logf(s) - (zl - mx);
            row_loss[i] = l;
            loss[r] = l;
        }
    }
    __syncthreads();
    if (threadIdx.x >= 64) return;
    float s = lane < n ? loss[lane] : 0.f;      // as in loss_mean_kernel
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
    if (lane == 0) out[S.k[blockIdx.x]] = s / (float)n;
}

void launch_softmax_ce(int dtype, const float* logits, const int32_t* labels, void* dlogits, float* row_loss,
                       float* loss_out, const ShardSet& S, int C, hipStream_t st) {
    const int n = S.samples();
    ProfScope ps("softmax_ce", 0.0, (4.0 + (dtype == 1 ? 2.0 : 4.0)) * (double)n * C, st);
    if (C <= kSmallClasses && S.largest() <= kSmallLossRows) {
        if (dtype == 1) hipLaunchKernelGGL(softmax_ce_small_kernel<bf16_t>, dim3(S.p), dim3(1024), 0, st, logits, labels, (bf16_t*)dlogits, row_loss, S, C, loss_out);
        else hipLaunchKernelGGL(softmax_ce_small_kernel<float>, dim3(S.p), dim3(1024), 0, st, logits, labels, (float*)dlogits, row_loss, S, C, loss_out);
        return;
    }
    const RowCut shards = cut_rows(S, 1, 1);
    if (dtype == 1)
        hipLaunchKernelGGL(softmax_ce_kernel<bf16_t>, dim3(n), dim3(256), 0, st, logits, labels, (bf16_t*)dlogits, row_loss, shards, C);
    else
        hipLaunchKernelGGL(softmax_ce_kernel<float>, dim3(n), dim3(256), 0, st, logits, labels, (float*)dlogits, row_loss, shards, C);
    hipLaunchKernelGGL(loss_mean_kernel, dim3(S.p), dim3(64), 0, st, row_loss, S, loss_out);
}

// ---------------------------------------------------------------------------
// Attainable matrix rate: every wave keeps four independent 32x32 accumulators
// and issues MFMAs on register operands only (no memory in the loop).  What the
// convolutions' MFMA fractions can be held against besides the data sheet.
// ---------------------------------------------------------------------------
typedef float mfma_acc_t __attribute__((ext_vector_type(16)));
typedef __bf16 mfma_bf16x8_t __attribute__((ext_vector_type(8)));

template <bool BF16>
__global__ __launch_bounds__(256) void mfma_rate_kernel(int iters, float* __restrict__ sink) {
    mfma_acc_t acc[4];
    #pragma unroll
    for (int q = 0; q < 4; ++q)
        #pragma unroll
        for (int e = 0; e < 16; ++e) acc[q][e] = 0.f;
    const float seed = 1.0f + (float)(threadIdx.x & 7) * 0.125f;
    mfma_bf16x8_t a, b;
    #pragma unroll
    for (int e = 0; e < 8; ++e) { a[e] = (__bf16)seed; b[e] = (__bf16)(1.0f / seed); }
    for (int i = 0; i < iters; ++i) {
        #pragma unroll
        for (int q = 0; q < 4; ++q) {
            if (BF16) acc[q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc[q], 0, 0, 0);
            else acc[q] = __builtin_amdgcn_mfma_f32_32x32x2f32(seed, 1.0f / seed, acc[q], 0, 0, 0);
        }
    }
    float t = 0.f;
    #pragma unroll
    for (int q = 0; q < 4; ++q)
        #pragma unroll
        for (int e = 0; e < 16; ++e) t += acc[q][e];
    if (t == 12345.678f) sink[0] = t;   // never true; keeps the accumulators alive
}

// flops issued: blocks * 4 waves * iters * 4 MFMAs * 2*32*32*k
double launch_mfma_rate(int dtype, int blocks, int iters, float* sink, hipStream_t st) {
    const double per_mfma = dtype == 1 ? 2.0 * 32 * 32 * 16 : 2.0 * 32 * 32 * 2;
    const double flops = (double)blocks * 4.0 * (double)iters * 4.0 * per_mfma;
    ProfScope ps(dtype == 1 ? "mfma_rate_bf16" : "mfma_rate_f32", flops, 0.0, st);
    if (dtype == 1) hipLaunchKernelGGL(mfma_rate_kernel<true>, dim3(blocks), dim3(256), 0, st, iters, sink);
    else hipLaunchKernelGGL(mfma_rate_kernel<false>, dim3(blocks), dim3(256), 0, st, iters, sink);
    return flops;
}

}  // namespace edl
