// The module's convolutions for every shape without a fused kernel: any C, H, W, fp32 or bf16 storage, as implicit GEMMs on
// the matrix cores.  Shared by the forward executor and the backward pass (whose data gradients are convolutions too).
//
// One launch runs one convolution for all items of a launch group.  A workgroup of four waves owns one item's MT x 16
// pixels times NT x 16 output channels:
//     D[16 channels][16 pixels] += W[16 channels][k] * X[k][16 pixels],  k = taps x input channels
// The input pixels it needs, halo included, are staged once into LDS (zeros outside the map and behind the last channel) and
// serve all taps; weights go from the caller's layout straight into registers, a ring of RD steps ahead (a step is one
// tap and 16 (fp32) or 32 (bf16) input channels: one 16-byte piece per lane and channel tile).  The four waves split the
// steps, not the tile: every weight is then read by one wave of the workgroup, and a tile small enough to give
// every CU work in a narrow launch group still keeps four SIMDs busy.  Their partial sums meet in LDS, in wave order.
//
// fp32 operands use v_mfma_f32_16x16x4 (fp32 products and sums: 157 TFLOP/s on the chip, the vector unit without packed
// instructions half of that), bf16 operands v_mfma_f32_16x16x32_bf16.  The kernel before this one gave every output element
// to a thread that read its 9 C products' operands from the caches: 21 training programs in fp32 at C = 128, 14 x 14
// went from 179 to 3.2 ms, 64 programs in bf16 at 7 x 7 from 45 to 0.61 ms.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>

#include "device_utils.h"
#include "plan_internal.h"

namespace {

// forward: join (1x1 over two arguments), first and second 3x3; backward: data gradients of the second and the first 3x3
// and of the join
enum ConvMode { CV_JOIN, CV_FIRST, CV_SECOND, CV_DSECOND, CV_DFIRST, CV_DJOIN };

struct ConvArgs {
    const dynb_item* items;
    const uint8_t* arity;         // device [n_types]
    int32_t first_item;           // index of items[0] among the items that gy, dm and du hold a map for
    int32_t first_kept;           // index of items[0] among the maps of u and mid
    const void* feats;
    void* out;
    void* slots;
    void* u;                      // results of joins, one map per item
    void* mid;                    // results of first convolutions, one map per item
    const void* w;                // the weights of this mode's convolution, in the caller's layout
    const float* bias;
    // backward
    const int32_t* gdst0;         // where the gradient of an argument goes
    const int32_t* gdst1;
    float* gy;                    // gradient with respect to every item's result
    float* gleaf;                 // ... arriving at every SCENE leaf
    float* dm;                    // gradient with respect to mid, masked by its ReLU
    float* du;                    // two-argument functions: gradient with respect to u, masked by its ReLU
    int32_t C, H, W;
    // tiling (conv_tiling)
    int32_t sw;                   // columns of a segment: wide maps are cut into segments of equal width
    int32_t tiles_per_seg;        // workgroup tiles of a segment's H x sw pixels
    int32_t n_ctile;              // channel tiles
    int32_t ck;                   // input channels staged at a time
};

typedef u32x4 u32x4_any __attribute__((aligned(2)));      // 16 and 8 bytes at any element's address
typedef u32x2 u32x2_any __attribute__((aligned(2)));
typedef f32x4 f32x4_any __attribute__((aligned(4)));

template <typename T> __device__ __forceinline__ const T* conv_src(const ConvArgs& a, int32_t s, size_t chw)
{
    return s >= 0 ? (const T*)a.slots + size_t(s) * chw : (const T*)a.feats + size_t(-1 - s) * chw;
}
template <typename T> __device__ __forceinline__ T* conv_dst(const ConvArgs& a, int32_t d, size_t chw)
{
    return d >= 0 ? (T*)a.slots + size_t(d) * chw : (T*)a.out + size_t(-1 - d) * chw;
}
__device__ __forceinline__ float* conv_route(const ConvArgs& a, int32_t r, size_t chw)
{
    return r >= 0 ? a.gy + size_t(r) * chw : a.gleaf + size_t(-1 - r) * chw;
}

// elements p[0 .. 3] as floats, zeros from n on (n may be negative); reads nothing behind p[n - 1]
template <typename T> __device__ __forceinline__ f32x4 load4(const T* p, int n)
{
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
    if (n >= 4) {
        if constexpr (sizeof(T) == 4) v = *reinterpret_cast<const f32x4_any*>(p);
        else {
            const u32x2 q = *reinterpret_cast<const u32x2_any*>(p);
            v = f32x4{__uint_as_float(q.x << 16), __uint_as_float(q.x & 0xffff0000u), __uint_as_float(q.y << 16), __uint_as_float(q.y & 0xffff0000u)};
        }
    } else
        for (int i = 0; i < 4; ++i)
            if (i < n) v[i] = load_f32(p + i);
    return v;
}
template <typename T> __device__ __forceinline__ void store4(T* p, int n, const f32x4& v)
{
    if (n >= 4) {
        if constexpr (sizeof(T) == 4) *reinterpret_cast<f32x4_any*>(p) = v;
        else *reinterpret_cast<u32x2_any*>(p) = u32x2{pack_bf16x2(v.x, v.y), pack_bf16x2(v.z, v.w)};
    } else
        for (int i = 0; i < 4; ++i)
            if (i < n) store_f32(p + i, v[i]);
}
// one 16-byte piece of a row in its own type: 4 floats or 8 bfloat16, zeros from n on
template <typename T> __device__ __forceinline__ u32x4 load_piece(const T* p, int n)
{
    constexpr int N = 16 / int(sizeof(T));
    if (n >= N) return *reinterpret_cast<const u32x4_any*>(p);
    u32x4 v = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int i = 0; i < N; ++i)
        if (i < n) {
            if constexpr (sizeof(T) == 4) v[i] = __float_as_uint(p[i]);
            else v[i / 2] |= uint32_t(p[i]) << (16 * (i & 1));
        }
    return v;
}

// The gradient that enters an item's second convolution, g = gy [y > 0], four channels of it
template <typename T> __device__ __forceinline__ f32x4 masked_gy(const float* gy, const T* y, int n)
{
    f32x4 g = load4(gy, n);
    const f32x4 v = load4(y, n);
#pragma unroll
    for (int i = 0; i < 4; ++i) g[i] = v[i] > 0.f ? g[i] : 0.f;
    return g;
}

// v / d for v * d < 2^32, d > 1, with m = recip_of(d)
__device__ __forceinline__ uint32_t recip_of(uint32_t d) { return 0xffffffffu / d + 1u; }
__device__ __forceinline__ uint32_t div_by(uint32_t v, uint32_t m) { return __umulhi(v, m); }

template <ConvMode MODE> struct ConvTraits {
    static constexpr bool JOINS = MODE == CV_JOIN || MODE == CV_DJOIN;
    static constexpr int TAPS = JOINS ? 1 : 9, HALO = JOINS ? 0 : 1;
    static constexpr bool BWD = MODE == CV_DSECOND || MODE == CV_DFIRST || MODE == CV_DJOIN;
};

// LDS of a workgroup: rows x columns of staged pixels, `ck` channels each.  A pixel takes an odd number of 16-byte granules,
// so that the 16 consecutive pixels that a quarter of a fragment read touches lie on different banks.
__host__ __device__ inline int conv_pixel_bytes(int ck, int elt) { return ck * elt + 16; }
__host__ __device__ inline int conv_rows(int first, int n_pix, int sw, int halo) { return (first + n_pix - 1) / sw - first / sw + 1 + 2 * halo; }

template <typename T, ConvMode MODE, int MT, int NT>
__global__ __launch_bounds__(256, 2) void k_conv(ConvArgs a)
{
    using Tr = ConvTraits<MODE>;
    using E = std::conditional_t<Tr::BWD, float, T>;      // element type of the staged input: gradients are fp32
    constexpr bool F32 = sizeof(E) == 4;
    constexpr int TAPS = Tr::TAPS, HALO = Tr::HALO, ES = int(sizeof(E)), KS = F32 ? 16 : 32, PE = 16 / ES, RD = 4;
    constexpr int BM = MT * 16;
    extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];

    const int i = blockIdx.y;
    const dynb_item it = a.items[i];
    const bool binary = a.arity[it.type] == 2;            // uniform over the workgroup
    if (Tr::JOINS && !binary) return;
    const int C = a.C, H = a.H, W = a.W, sw = a.sw;
    const size_t chw = size_t(H) * W * C;
    const int ctile = blockIdx.x % a.n_ctile, ptile = blockIdx.x / a.n_ctile;      // channel tiles of the same pixels are neighbours
    const int seg = ptile / a.tiles_per_seg, q0 = (ptile % a.tiles_per_seg) * BM, n_q = H * sw;
    const int x0 = seg * sw, y0 = q0 / sw;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, r = lane & 15, g = lane >> 4;
    const int NO = MODE == CV_DJOIN ? 2 * C : C;          // output channels
    const int n0 = ctile * NT * 16;

    const int pix_bytes = conv_pixel_bytes(a.ck, ES), cols = sw + 2 * HALO, row_bytes = cols * pix_bytes;
    const int n_q_here = min(BM, n_q - q0);
    const int rows = conv_rows(q0, n_q_here, sw, HALO);

    // this lane's weights: output channel n0 + 16 nt + r (the last one again behind the end, whose results are dropped)
    int n_of[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) n_of[nt] = min(n0 + nt * 16 + r, NO - 1);
    const T* w_type = (const T*)a.w + size_t(it.type) * C * (Tr::JOINS ? 2 * C : 9 * C);

    // this lane's pixels: LDS address of the top left tap, first channel of its piece
    uint32_t x_at[MT];
#pragma unroll
    for (int t = 0; t < MT; ++t) {
        const int q = min(q0 + t * 16 + r, n_q - 1), y = q / sw, x = q - y * sw;
        x_at[t] = uint32_t((y - y0) * row_bytes + x * pix_bytes + g * 16);
    }
    f32x4 acc[MT][NT];
#pragma unroll
    for (int t = 0; t < MT; ++t)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) acc[t][nt] = f32x4{0.f, 0.f, 0.f, 0.f};

    // the map whose convolution this is (in the join: argument `arg`)
    auto input_map = [&](int arg) -> const E* {
        if constexpr (MODE == CV_JOIN) return conv_src<E>(a, arg ? it.src1 : it.src0, chw);
        else if constexpr (MODE == CV_FIRST) return binary ? (const E*)a.u + size_t(a.first_kept + i) * chw : conv_src<E>(a, it.src0, chw);
        else if constexpr (MODE == CV_SECOND) return (const E*)a.mid + size_t(a.first_kept + i) * chw;
        else if constexpr (MODE == CV_DSECOND) return a.gy + size_t(a.first_item + i) * chw;
        else if constexpr (MODE == CV_DFIRST) return a.dm + size_t(a.first_item + i) * chw;
        else return a.du + size_t(a.first_item + i) * chw;
    };
    const T* y_map = MODE == CV_DSECOND || MODE == CV_DFIRST ? conv_dst<T>(a, it.dst, chw) : nullptr;   // the item's result

    const int panels = (C + a.ck - 1) / a.ck;
#pragma unroll 1
    for (int panel = 0; panel < panels * (MODE == CV_JOIN ? 2 : 1); ++panel) {
        const int arg = MODE == CV_JOIN && panel >= panels ? 1 : 0;
        const int c0 = (panel - arg * panels) * a.ck;
        const int nj = min(a.ck / KS, (C - c0 + KS - 1) / KS);
        const int S = nj * TAPS, s0 = S * wave / 4, s1 = S * (wave + 1) / 4;
        const uint32_t m_nj = recip_of(nj);
        auto tap_of = [&](int s) -> int { return TAPS == 1 ? 0 : nj == 1 ? s : int(div_by(s, m_nj)); };
        // weights of step s = tap * nj + j
        auto load_w = [&](int s, u32x4 (&w)[NT]) {
            const int tap = tap_of(s), j = s - tap * nj;
            const int c = c0 + j * KS + g * PE;           // first of this lane's PE input channels
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                if constexpr (!Tr::BWD) {
                    const T* p = w_type + (Tr::JOINS ? size_t(n_of[nt]) * 2 * C + arg * C : (size_t(n_of[nt]) * 9 + tap) * C) + c;
                    w[nt] = load_piece(p, c0 + (j + 1) * KS <= C ? PE : C - c);
                } else {
                    // W[k][o]: the channels that are summed are the weights' output channels (rows)
                    const size_t pitch = Tr::JOINS ? size_t(2) * C : size_t(9) * C;
                    const T* p = w_type + size_t(c) * pitch + (Tr::JOINS ? 0 : (8 - tap) * C) + n_of[nt];
                    const int n = c0 + (j + 1) * KS <= C ? 4 : C - c;
#pragma unroll
                    for (int e = 0; e < 4; ++e) w[nt][e] = __float_as_uint(e < n ? load_f32(p + size_t(e) * pitch) : 0.f);
                }
            }
        };
        u32x4 ring[RD][NT];
#pragma unroll
        for (int u = 0; u < RD; ++u)
            if (s0 + u < s1) load_w(s0 + u, ring[u]);

        // ---- stage rows x cols pixels x nj * KS channels
        if (panel > 0) __syncthreads();
        {
            const E* src = input_map(arg);
            const int np = nj * (KS / PE), n_pieces = rows * cols * np;
            const uint32_t m_np = recip_of(np), m_cols = recip_of(cols);
            constexpr int UN = 8;
            for (int base = tid; base < n_pieces; base += 256 * UN) {
                u32x4 v[UN];
                uint32_t at[UN];
#pragma unroll
                for (int k = 0; k < UN; ++k) {
                    const int c = base + k * 256;
                    v[k] = u32x4{0u, 0u, 0u, 0u};
                    const uint32_t pix = div_by(c, m_np), part = c - pix * np, row = cols == 1 ? pix : div_by(pix, m_cols), col = pix - row * cols;
                    at[k] = row * row_bytes + col * pix_bytes + part * 16;
                    const int y = y0 - HALO + int(row), x = x0 - HALO + int(col), ch = c0 + int(part) * PE;
                    if (c < n_pieces && unsigned(y) < unsigned(H) && unsigned(x) < unsigned(W)) {
                        const size_t e = (size_t(y) * W + x) * C + ch;
                        if constexpr (MODE == CV_DSECOND) v[k] = __builtin_bit_cast(u32x4, masked_gy(src + e, y_map + e, C - ch));
                        else v[k] = load_piece(src + e, C - ch);
                    }
                }
#pragma unroll
                for (int k = 0; k < UN; ++k)
                    if (base + k * 256 < n_pieces) *reinterpret_cast<u32x4*>(lds_raw + at[k]) = v[k];
            }
        }
        __syncthreads();

        // ---- this wave's steps
#pragma unroll 1
        for (int s = s0; s < s1; s += RD) {
#pragma unroll
            for (int u = 0; u < RD; ++u) {
                if (s + u >= s1) break;
                const int tap = tap_of(s + u), j = s + u - tap * nj, kh = tap * 11 >> 5, kw = tap - 3 * kh;
                const uint32_t off = uint32_t(kh * row_bytes + kw * pix_bytes + j * KS * ES);
                u32x4 x[MT];
#pragma unroll
                for (int t = 0; t < MT; ++t) x[t] = *reinterpret_cast<const u32x4*>(lds_raw + x_at[t] + off);
                if constexpr (F32) {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
#pragma unroll
                        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                            for (int t = 0; t < MT; ++t)
                                acc[t][nt] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(ring[u][nt][e]), __uint_as_float(x[t][e]), acc[t][nt], 0, 0, 0);
                } else {
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                        for (int t = 0; t < MT; ++t)
                            acc[t][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, ring[u][nt]), __builtin_bit_cast(bf16x8, x[t]), acc[t][nt], 0, 0, 0);
                }
                if (s + u + RD < s1) load_w(s + u + RD, ring[u]);
            }
        }
    }

    // ---- partial sums through LDS; wave w finishes tiles w, w + 4, ...
    __syncthreads();
    f32x4* red = reinterpret_cast<f32x4*>(lds_raw);
#pragma unroll
    for (int t = 0; t < MT; ++t)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) red[(wave * MT * NT + t * NT + nt) * 64 + lane] = acc[t][nt];
    __syncthreads();
    for (int tt = wave; tt < MT * NT; tt += 4) {
        const int t = tt / NT, nt = tt % NT;
        const int q = q0 + t * 16 + r, y = q / sw, x = x0 + q - y * sw;
        const int o = n0 + nt * 16 + g * 4, n = min(4, NO - o);          // lane: pixel r, output channels o .. o + 3
        if (q >= n_q || x >= W || n <= 0) continue;
        f32x4 v = red[tt * 64 + lane];
#pragma unroll
        for (int w = 1; w < 4; ++w) {
            const f32x4 p = red[(w * MT * NT + tt) * 64 + lane];
            v.x += p.x; v.y += p.y; v.z += p.z; v.w += p.w;
        }
        const size_t e = (size_t(y) * W + x) * C + o;
        if constexpr (!Tr::BWD) {
            if (a.bias) {
                const f32x4 b = load4(a.bias + size_t(it.type) * C + o, n);
                v.x += b.x; v.y += b.y; v.z += b.z; v.w += b.w;
            }
            T* dst;
            if constexpr (MODE == CV_JOIN) dst = (T*)a.u + size_t(a.first_kept + i) * chw;
            else if constexpr (MODE == CV_FIRST) dst = (T*)a.mid + size_t(a.first_kept + i) * chw;
            else {
                const T* u = binary ? (const T*)a.u + size_t(a.first_kept + i) * chw : conv_src<T>(a, it.src0, chw);
                const f32x4 b = load4(u + e, n);
                v.x += b.x; v.y += b.y; v.z += b.z; v.w += b.w;
                dst = conv_dst<T>(a, it.dst, chw);
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) v[k] = fmaxf(v[k], 0.f);
            store4(dst + e, n, v);
        } else if constexpr (MODE == CV_DSECOND) {                       // dmid = result [mid > 0]
            const f32x4 m = load4((const T*)a.mid + size_t(a.first_kept + i) * chw + e, n);
#pragma unroll
            for (int k = 0; k < 4; ++k) v[k] = m[k] > 0.f ? v[k] : 0.f;
            store4(a.dm + size_t(a.first_item + i) * chw + e, n, v);
        } else if constexpr (MODE == CV_DFIRST) {                        // du = result + g
            const f32x4 b = masked_gy(a.gy + size_t(a.first_item + i) * chw + e, y_map + e, n);
            v.x += b.x; v.y += b.y; v.z += b.z; v.w += b.w;
            if (binary) {                                                // dc = du [u > 0]
                const f32x4 u = load4((const T*)a.u + size_t(a.first_kept + i) * chw + e, n);
#pragma unroll
                for (int k = 0; k < 4; ++k) v[k] = u[k] > 0.f ? v[k] : 0.f;
                store4(a.du + size_t(a.first_item + i) * chw + e, n, v);
            } else store4(conv_route(a, a.gdst0[i], chw) + e, n, v);
        } else {                                                         // channels 0 .. C - 1: first argument, C .. 2 C - 1: second
            float* d0 = conv_route(a, a.gdst0[i], chw) + e;
            float* d1 = conv_route(a, a.gdst1[i], chw) + e - C;
            if (o + n <= C) store4(d0, n, v);
            else if (o >= C) store4(d1, n, v);
            else
                for (int k = 0; k < 4; ++k)
                    if (k < n) (o + k < C ? d0 : d1)[k] = v[k];
        }
    }
}

template <typename T, ConvMode MODE, int MT, int NT>
int launch_conv_tile(ConvArgs a, int count, hipStream_t st)
{
    using Tr = ConvTraits<MODE>;
    constexpr int ES = Tr::BWD ? 4 : int(sizeof(T)), KS = ES == 4 ? 16 : 32;
    constexpr int LDS_MAX = 80 * 1024;                                   // two workgroups per CU
    static std::atomic<uint64_t> attr_set{0};                            // one bit per device
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return DYNB_E_HIP;
    if (!(attr_set.load() >> (dev & 63) & 1)) {
        if (hipFuncSetAttribute(reinterpret_cast<const void*>(k_conv<T, MODE, MT, NT>), hipFuncAttributeMaxDynamicSharedMemorySize, LDS_MAX) != hipSuccess)
            return DYNB_E_HIP;
        attr_set.fetch_or(uint64_t(1) << (dev & 63));
    }
    const int n_q = a.H * a.sw, n_seg = (a.W + a.sw - 1) / a.sw;
    a.tiles_per_seg = (n_q + MT * 16 - 1) / (MT * 16);
    a.n_ctile = ((MODE == CV_DJOIN ? 2 * a.C : a.C) + NT * 16 - 1) / (NT * 16);
    // a tile's pixels start anywhere in a row
    const int n_pix = std::min(MT * 16, n_q);
    const int pixels = std::min(conv_rows(a.sw - 1, n_pix, a.sw, Tr::HALO), a.H + 2 * Tr::HALO) * (a.sw + 2 * Tr::HALO);
    // as many channels at a time as fit, in panels of nearly equal size
    const int steps = (a.C + KS - 1) / KS;
    const int fit = std::max(1, (LDS_MAX / pixels - 16) / (KS * ES));
    const int panels = (steps + fit - 1) / fit;
    a.ck = (steps + panels - 1) / panels * KS;
    const size_t lds = std::max<size_t>(size_t(pixels) * conv_pixel_bytes(a.ck, ES), size_t(4) * MT * NT * 1024);
    if (lds > LDS_MAX) return DYNB_E_UNSUPPORTED;                        // cannot happen: sw <= 32
    hipLaunchKernelGGL((k_conv<T, MODE, MT, NT>), dim3(unsigned(n_seg * a.tiles_per_seg * a.n_ctile), unsigned(count)), dim3(256), lds, st, a);
    return DYNB_OK;
}

// One convolution for `count` (<= 65535) items.  The tile is the largest that still makes two workgroups per CU (256 CUs): small
// tiles read the weights and stage the halo more often per output, but a launch that leaves CUs idle takes as long
// as its one workgroup does.
template <typename T, ConvMode MODE>
int launch_conv(ConvArgs a, int count, hipStream_t st)
{
    const int n_seg = (a.W + 31) / 32;
    a.sw = (a.W + n_seg - 1) / n_seg;
    const long long ptiles = (long long)n_seg * ((a.H * a.sw + 15) / 16), ctiles = ((MODE == CV_DJOIN ? 2 * a.C : a.C) + 15) / 16;
    auto groups = [&](int mt, int nt) { return (long long)count * ((ptiles + mt - 1) / mt) * ((ctiles + nt - 1) / nt); };
    if (groups(4, 2) >= 512) return launch_conv_tile<T, MODE, 4, 2>(a, count, st);
    if (groups(4, 1) >= 512) return launch_conv_tile<T, MODE, 4, 1>(a, count, st);
    if (groups(2, 1) >= 512) return launch_conv_tile<T, MODE, 2, 1>(a, count, st);
    return launch_conv_tile<T, MODE, 1, 1>(a, count, st);
}

}  // namespace
