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
// went from 179 to 2.5 ms, 64 programs in bf16 at 7 x 7 from 45 to 0.6 ms (0.46 with what stands at ConvSteps, k_conv and launch_conv).
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <climits>
#include <type_traits>

#include "device_utils.h"
#include "plan_internal.h"

namespace {

// forward: join (1x1 over two arguments), first and second 3x3; backward: data gradients of the second and the first 3x3
// and of the join
// (CV_JOIN_BOTH: a join with both arguments in LDS, one behind the other)
enum ConvMode { CV_JOIN, CV_FIRST, CV_SECOND, CV_DSECOND, CV_DFIRST, CV_DJOIN, CV_JOIN_BOTH };

struct ConvArgs {
    int32_t first_item;           // index of items[0] among the items that gy, dm and du hold a map for
    int32_t first_kept;           // index of items[0] among the maps of u and mid
    // (u and du of kept plans hold maps for two-argument functions only, and the pointers are such that the same indices find them)
    const void* feats;
    void* out;
    void* slots;
    void* u;                      // results of joins
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
    uint32_t m_sw;                // recip20_of(sw)
    // runs of items for the dies: recip_of(workgroups of an item) or 0 (they stay in their order); workgroups of an item; an eighth of all
    // workgroups, and how many are left over.  (Last: what a workgroup waits for first brings these arguments' line with it.)
    uint32_t runs, n_groups, run_q, run_r;
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

// elements p[0 .. 3] as floats, zeros from n on (n may be negative); reads nothing behind p[n - 1].  FULL: n >= 4 is known
template <bool FULL, typename T> __device__ __forceinline__ f32x4 load4(const T* p, int n)
{
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
    if (FULL || n >= 4) {
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
template <bool FULL, typename T> __device__ __forceinline__ void store4(T* p, int n, const f32x4& v)
{
    if (FULL || n >= 4) {
        if constexpr (sizeof(T) == 4) *reinterpret_cast<f32x4_any*>(p) = v;
        else *reinterpret_cast<u32x2_any*>(p) = u32x2{pack_bf16x2(v.x, v.y), pack_bf16x2(v.z, v.w)};
    } else
        for (int i = 0; i < 4; ++i)
            if (i < n) store_f32(p + i, v[i]);
}
// one 16-byte piece of a row in its own type: 4 floats or 8 bfloat16, zeros from n on
template <bool FULL, typename T> __device__ __forceinline__ u32x4 load_piece(const T* p, int n)
{
    constexpr int N = 16 / int(sizeof(T));
    if (FULL || n >= N) return *reinterpret_cast<const u32x4_any*>(p);
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
template <bool FULL, typename T> __device__ __forceinline__ f32x4 masked_gy(const float* gy, const T* y, int n)
{
    f32x4 g = load4<FULL>(gy, n);
    const f32x4 v = load4<FULL>(y, n);
#pragma unroll
    for (int i = 0; i < 4; ++i) g[i] = v[i] > 0.f ? g[i] : 0.f;
    return g;
}

// Divisions (some thirty instructions) by a few values that a workgroup divides by again and again:
// v / d for d > 1, v * d < 2^32, with m = recip_of(d)
__host__ __device__ constexpr uint32_t recip_of(uint32_t d) { return 0xffffffffu / d + 1u; }
__device__ __forceinline__ uint32_t div_by(uint32_t v, uint32_t m) { return __umulhi(v, m); }
// v / d for v < 4096, v * d < 2^20, with m = recip20_of(d); here v are the steps of a 3x3's panel (at most 9 x 142: it stages
// at least 9 pixels), pixels of a tile (1300) and columns of a segment (32)
__host__ __device__ constexpr uint32_t recip20_of(uint32_t d) { return ((1u << 20) + d - 1) / d; }
__host__ __device__ constexpr uint32_t div20_by(uint32_t v, uint32_t m) { return v * m >> 20; }
// The tap of a panel's step s: nj steps a tap, m_nj = recip20_of(nj).  (Two taps, a join's arguments, are told apart without a division: on maps of a
// pixel or two nj goes as far as LDS does, and from 756 on s * nj beyond what div20_by is exact for.)
template <int TAPS> __host__ __device__ constexpr int tap_of(int s, int nj, uint32_t m_nj)
{
    return TAPS == 1 ? 0 : TAPS == 2 ? int(s >= nj) : int(div20_by(uint32_t(s), m_nj));
}

template <ConvMode MODE> struct ConvTraits {
    static constexpr bool JOINS = MODE == CV_JOIN || MODE == CV_DJOIN || MODE == CV_JOIN_BOTH;
    static constexpr int TAPS = MODE == CV_JOIN_BOTH ? 2 : JOINS ? 1 : 9, HALO = JOINS ? 0 : 1;
    static constexpr bool BWD = MODE == CV_DSECOND || MODE == CV_DFIRST || MODE == CV_DJOIN;
};

// LDS of a workgroup: rows x columns of staged pixels, `ck` channels each.  A pixel takes an odd number of 16-byte granules,
// so that the 16 consecutive pixels that a quarter of a fragment read touches lie on different banks.
__host__ __device__ inline int conv_pixel_bytes(int ck, int elt) { return ck * elt + 16; }
__host__ __device__ inline int conv_rows(int first, int n_pix, int sw, int halo) { return (first + n_pix - 1) / sw - first / sw + 1 + 2 * halo; }

// The steps of a sum: step s is a tap and KS input channels, channels first.  A wave takes steps s0 .. s0 + n_steps of NT
// channel tiles and MT pixel tiles.  Weights and pixels of a step lie at uniform offsets from the lane's own places.
// (The data gradient of a 3x3 takes the weights' taps backwards and sums over their rows.)
// request() asks for the first RD steps' weights, run() multiplies.  There is no branch around a request: the counter that
// a wave waits on counts requests, and behind a branch the compiler can only wait for all of them.  Past the end the
// last step is requested again.  The pixels of the next step are read under the MFMAs of this one.
// FULL: C is a multiple of KS, so that no piece is ever cut short.  (What handles the others doubles the code, and a launch of
// a few microseconds feels every line of it that the instruction cache has to fetch.)
// G = 2 (FULL, panels of an even number of steps, forward): weights are requested for two steps together.  A fragment wants the pieces of 16
// rows in neighbouring lanes; asked for like that, four lanes' 64 bytes come from four lines, and a CU is answered at 15.6 bytes a clock
// however many waves ask (590 KB, all CUs or a quarter of them).  Here two neighbouring lanes ask for consecutive pieces of one row (four,
// in groups of four steps, were no faster: 23 to 38 bytes a clock, but such groups divide badly among the waves and the exchange doubles),
// and the two fragments are put together by an exchange between these lanes:
__device__ __forceinline__ void exchange(u32x4& a, u32x4& b)           // a's odd lanes against b's even ones
{
    const bool odd = (threadIdx.x & 1) != 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int pa = __builtin_amdgcn_mov_dpp(int(a[e]), 0xB1, 0xF, 0xF, true), pb = __builtin_amdgcn_mov_dpp(int(b[e]), 0xB1, 0xF, 0xF, true);   // quad_perm [1,0,3,2]
        const uint32_t na = odd ? uint32_t(pb) : a[e], nb = odd ? b[e] : uint32_t(pa);
        a[e] = na;
        b[e] = nb;
    }
}

template <typename T, ConvMode MODE, int MT, int NT, bool FULL, int G = 1>
struct ConvSteps {
    using Tr = ConvTraits<MODE>;
    using E = std::conditional_t<Tr::BWD, float, T>;      // element type of the staged input: gradients are fp32
    static constexpr bool F32 = sizeof(E) == 4;
    static constexpr int TAPS = Tr::TAPS, ES = int(sizeof(E)), KS = F32 ? 16 : 32, PE = 16 / ES;
    static constexpr int X_LANE = G * 16;                 // bytes between the pixel data of the lane groups g
    static_assert(G == 1 || (G == 2 && FULL && !Tr::BWD), "weights in groups of steps");
    // Steps that the weights are requested ahead: a step is 128 (fp32) or 16 (bf16) clocks of MFMAs per 16 x 16 tile, an
    // answer takes 500 to 2000.  Even; at C = 128 a wave of k_conv has 18 or up to 10 steps.
    static constexpr int RD = F32 ? 6 : G == 2 ? 12 : 10, NG = RD / G;
    static_assert(RD % G == 0 && RD % 2 == 0, "ring");

    uint32_t w_at[G == 2 ? 1 : NT], x_at[MT];             // this lane's weights (bytes from w_panel) and pixels (LDS address of the top left tap)
    uint32_t w_tile[G == 2 ? NT : 1];                     // G = 2: bytes from w_panel to the channel tiles, uniform
    const char* w_panel;
    int C, c0, nj, s0, n_steps, w_pitch, w_chan, w_tap, g, row_bytes, pix_bytes;
    uint32_t m_nj;
    u32x4 ring[NG][NT][G];

    // weights of `type` for output channels n0 .. of NO (the last one again behind the end, whose results are dropped)
    __device__ __forceinline__ const char* weights(const void* w, int type, int C_, int n0, int NO, int lane)
    {
        C = C_;
        g = lane >> 4;
        w_pitch = (Tr::JOINS ? 2 : 9) * C;                // elements between two rows of weights
        w_chan = KS * (Tr::BWD ? w_pitch : 1);
        w_tap = Tr::BWD ? -C : C;
        if constexpr (G == 2) {                           // request i of a group: row (lane % 16 / G) G + i, piece lane % G of the lane group's G
            w_at[0] = (uint32_t(lane & 15 & ~(G - 1)) * uint32_t(w_pitch) + uint32_t((g * G + (lane & (G - 1))) * PE)) * uint32_t(sizeof(T));
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) w_tile[nt] = uint32_t(min(n0 + nt * 16, NO - 16) - n0) * uint32_t(w_pitch) * uint32_t(sizeof(T));
        } else {
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                const uint32_t n = uint32_t(min(n0 + nt * 16 + (lane & 15), NO - 1) - n0);
                w_at[nt] = Tr::BWD ? (uint32_t(g * PE) * uint32_t(w_pitch) + n) * uint32_t(sizeof(T)) : (n * uint32_t(w_pitch) + uint32_t(g * PE)) * uint32_t(sizeof(T));
            }
        }
        return reinterpret_cast<const char*>((const T*)w + size_t(type) * C * w_pitch + (Tr::BWD ? size_t(n0) : size_t(n0) * w_pitch));
    }
    // summed channels first .. of `pieces` KS channels; of the join: of argument `arg`
    __device__ __forceinline__ void panel(const char* w_tile, int first, int pieces, int arg)
    {
        c0 = first;
        nj = pieces;
        m_nj = recip20_of(nj);
        w_panel = w_tile + (Tr::BWD ? ptrdiff_t(c0) * w_pitch + (Tr::JOINS ? 0 : 8 * C) : ptrdiff_t(arg * C) + c0) * ptrdiff_t(sizeof(T));
    }
    // wave w of 4: its share of the panel's steps, whole groups
    __device__ __forceinline__ void share(int w)
    {
        const int groups = nj * TAPS / G;
        s0 = groups * w / 4 * G;
        n_steps = groups * (w + 1) / 4 * G - s0;
    }
    // steps step .. step + G - 1 (one group)
    __device__ __forceinline__ void load_w(int step, u32x4 (&w)[NT][G]) const
    {
        const int s = s0 + step, tap = tap_of<TAPS>(s, nj, m_nj), j = s - tap * nj;
        const char* p = w_panel + (ptrdiff_t(tap) * w_tap + ptrdiff_t(j) * w_chan) * ptrdiff_t(sizeof(T));
        if constexpr (G == 2) {
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                for (int i = 0; i < G; ++i)
                    w[nt][i] = *reinterpret_cast<const u32x4_any*>(p + w_tile[nt] + uint32_t(i * w_pitch) * uint32_t(sizeof(T)) + w_at[0]);
        } else {
            const bool inside = FULL || c0 + (j + 1) * KS <= C;          // uniform
            const int c = c0 + j * KS + g * PE;           // first of this lane's PE summed channels
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                if constexpr (!Tr::BWD) w[nt][0] = load_piece<FULL>(reinterpret_cast<const T*>(p + w_at[nt]), inside ? PE : C - c);
                else {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        w[nt][0][e] = inside || c + e < C ? __float_as_uint(load_f32(reinterpret_cast<const T*>(p + (w_at[nt] + uint32_t(e * w_pitch) * uint32_t(sizeof(T)))))) : 0u;
                }
            }
        }
    }
    // a group as it was requested -> its steps' fragments: lane: row lane % 16, step i: piece g G + i of the group
    static __device__ __forceinline__ void sort(u32x4 (&w)[NT][G])
    {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            if constexpr (G == 2) exchange(w[nt][0], w[nt][1]);
        }
    }
    // LDS offset of a group's pixels: of its first step; step i lies i pieces further
    __device__ __forceinline__ uint32_t x_group(int step) const
    {
        const int s = s0 + step, tap = tap_of<TAPS>(s, nj, m_nj), j = s - tap * nj, kh = tap * 11 >> 5, kw = tap - 3 * kh;
        return uint32_t(kh * row_bytes + kw * pix_bytes + j * (KS * ES));
    }
    __device__ __forceinline__ void read_x(uint32_t off, int i, u32x4 (&v)[MT]) const
    {
        extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
#pragma unroll
        for (int t = 0; t < MT; ++t) v[t] = *reinterpret_cast<const u32x4*>(lds_raw + (x_at[t] + off) + i * 16);
    }
    template <typename W> static __device__ __forceinline__ void multiply(f32x4 (&acc)[MT][NT], const W& w, int i, const u32x4 (&v)[MT])
    {
        if constexpr (F32) {
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                    for (int t = 0; t < MT; ++t)
                        acc[t][nt] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(w[nt][i][e]), __uint_as_float(v[t][e]), acc[t][nt], 0, 0, 0);
        } else {
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                for (int t = 0; t < MT; ++t)
                    acc[t][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w[nt][i]), __builtin_bit_cast(bf16x8, v[t]), acc[t][nt], 0, 0, 0);
        }
    }
    __device__ __forceinline__ void request()
    {
#pragma unroll
        for (int u = 0; u < NG; ++u) load_w(max(0, min(u * G, n_steps - G)), ring[u]);
    }
    // (Two loops, for steps in groups and for single ones: one loop for both, which carries a group's place in LDS to the next, has ten instructions
    // fewer of 5935 and took k_node, fp32, C = 20, 7 x 7 2.5 % longer, C = 16, 8 x 8 1 %.  Behind the last request single steps go without fences: with
    // them k_node, fp32, C = 16, 14 x 14 takes 14.56 us instead of 14.41.)
    __device__ __forceinline__ void run(f32x4 (&acc)[MT][NT])
    {
        if (n_steps <= 0) return;
        u32x4 x[2][MT];
        const int last = n_steps - G;                     // the last group
        uint32_t off = x_group(0);
        read_x(off, 0, x[0]);
        int s = 0;
        if constexpr (G == 1) {
#pragma unroll 1
            for (; s + RD < n_steps; s += RD) {
#pragma unroll
                for (int u = 0; u < RD; ++u) {
                    read_x(x_group(min(s + u + 1, last)), 0, x[(u + 1) & 1]);
                    __builtin_amdgcn_sched_barrier(0);
                    multiply(acc, ring[u], 0, x[u & 1]);
                    __builtin_amdgcn_sched_barrier(0);
                    load_w(min(s + u + RD, last), ring[u]);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
#pragma unroll
            for (int u = 0; u < RD; ++u) {
                if (s + u >= n_steps) break;
                read_x(x_group(min(s + u + 1, last)), 0, x[(u + 1) & 1]);
                multiply(acc, ring[u], 0, x[u & 1]);
            }
        } else {
            // one group, its weights in w; what comes after it is read under its MFMAs
            auto group = [&](u32x4 (&w)[NT][G], int u, int next) {
                sort(w);
                const uint32_t then = x_group(min(next, last));
#pragma unroll
                for (int i = 0; i < G; ++i) {
                    const int k = u * G + i;
                    if (i + 1 < G) read_x(off, i + 1, x[(k + 1) & 1]);
                    else read_x(then, 0, x[(k + 1) & 1]);
                    __builtin_amdgcn_sched_barrier(0);
                    multiply(acc, w, i, x[k & 1]);
                    __builtin_amdgcn_sched_barrier(0);
                }
                off = then;
            };
#pragma unroll 1
            for (; s + RD < n_steps; s += RD) {
#pragma unroll
                for (int u = 0; u < NG; ++u) {
                    group(ring[u], u, s + (u + 1) * G);
                    load_w(min(s + u * G + RD, last), ring[u]);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
#pragma unroll
            for (int u = 0; u < NG; ++u) {
                if (s + u * G >= n_steps) break;
                group(ring[u], u, s + (u + 1) * G);
            }
        }
    }
};

// A tap outside the map contributes nothing, whatever its weight; the matrix instructions multiply a zero with it, which is NaN for
// a weight that is not finite.  Nothing else brings a NaN in from outside, so a sum at the map's border that came out NaN is taken
// again, tap by tap: rare, and out of the way of the others.
__device__ __forceinline__ bool any_nan(const f32x4& v)                 // (one too many is no harm: a direct sum is always right)
{
    return __builtin_expect(__builtin_isunordered(v.x, v.y) | __builtin_isunordered(v.z, v.w), 0);
}
__device__ __forceinline__ bool at_border(int y, int x, int H, int W) { return y == 0 || x == 0 || y == H - 1 || x == W - 1; }
// Ends the wave unless one of its lanes says otherwise.  (The compiler's branch to the end over what follows waits for instructions
// that nobody has fetched, 1.5 % of a pass at 7 x 7, where launches are short.)
__device__ __forceinline__ void end_unless(bool lane)
{
    asm volatile("s_cmp_lg_u64 %0, 0\n\ts_cbranch_scc1 1f\n\ts_endpgm\n1:" ::"s"(__ballot(lane)) : "scc", "memory");
}
// w: the function's weights.  pixel(kh, kw, c): channel c of the pixel under tap (kh, kw), as a float.  BWD: the data gradient (taps
// backwards, sums over the weights' rows)
template <bool BWD, typename T, typename Pixel>
__device__ __forceinline__ f32x4 direct_sum(const T* w, int C, int H, int W, int y, int x, int o, int n, Pixel&& pixel)
{
    f32x4 sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
    for (int tap = 0; tap < 9; ++tap) {
        const int kh = tap / 3, kw = tap - 3 * kh;
        if (unsigned(y + kh - 1) >= unsigned(H) || unsigned(x + kw - 1) >= unsigned(W)) continue;
#pragma unroll 1
        for (int c = 0; c < C; ++c) {
            const float v = pixel(kh, kw, c);
            const T* p = BWD ? w + (size_t(c) * 9 + 8 - tap) * C + o : w + (size_t(o) * 9 + tap) * C + c;
            for (int e = 0; e < n; ++e) sum[e] += v * load_f32(p + size_t(e) * (BWD ? 1 : 9 * size_t(C)));
        }
    }
    return sum;
}

// Waves per SIMD, which are workgroups per CU: three where the sums are in fp32 and 168 registers hold the tile.  (The staging of pixels ahead of the
// weights took ten more and left two: kernel time of a pass over 64 balanced trees, fp32, the joins in 4 x 2 tiles, C = 256, 14 x 14 1233 us,
// with three 1141; a training step's, C = 128, 14 x 14, the first convolution's data gradients in 2 x 2 790 / 725, the joins' 366 / 310.)
template <typename T, ConvMode MODE, int MT, int NT, bool FULL>
constexpr int conv_waves()
{
    constexpr int tiles = MODE == CV_DSECOND ? 2 : MODE == CV_DFIRST || MODE == CV_SECOND ? 4 : 8;
    return FULL && (ConvTraits<MODE>::BWD || sizeof(T) == 4) && MT * NT <= tiles ? 3 : 2;
}

template <typename T, ConvMode MODE, int MT, int NT, bool FULL, int G>
__global__ __launch_bounds__(256, (conv_waves<T, MODE, MT, NT, FULL>())) void k_conv(const dynb_item* items, ConvArgs a)
{
    using Tr = ConvTraits<MODE>;
    using Steps = ConvSteps<T, MODE, MT, NT, FULL, G>;
    using E = typename Steps::E;
    constexpr int HALO = Tr::HALO, ES = Steps::ES, KS = Steps::KS, PE = Steps::PE;
    constexpr int BM = MT * 16;
    extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];

    // Consecutive workgroups go to the chip's 8 dies in turn: every die gets one run of the items' tiles, so that an item's map and its function's
    // weights (items are sorted by function) are fetched behind one L2 and not behind all (21 training programs, fp32, C = 128, 14 x 14: 2496 ->
    // 2374 us; 64 programs, bf16, 7 x 7: 492 -> 470).
    // (Without a branch, and nothing of it from the grid's size: behind a branch the pointer to the items and the grid's size were waits of their own
    // ahead of the item, 0.2 us a launch: training step of 3 programs, fp32, C = 16, 14 x 14 703 -> 697 us; of 9 programs, bf16, C = 64, 9 x 9 811 -> 798.)
    uint32_t i = blockIdx.y, tile = blockIdx.x;
    {
        const uint32_t b = i * a.n_groups + tile, die = b & 7, l = die * a.run_q + min(die, a.run_r) + (b >> 3), run_i = div_by(l, a.runs);
        tile = a.runs ? l - run_i * a.n_groups : tile;
        i = a.runs ? run_i : i;
    }
    const dynb_item it = items[i];
    const bool binary = it.src1 != DYNB_NO_ARG;           // uniform over the workgroup
    if (Tr::JOINS && !binary) return;
    const int C = a.C, H = a.H, W = a.W, sw = a.sw;
    const size_t chw = size_t(H) * W * C;
    const int ptile = int(tile) / a.n_ctile, ctile = int(tile) - ptile * a.n_ctile;   // channel tiles of the same pixels are neighbours
    const int seg = sw == W ? 0 : ptile / a.tiles_per_seg, q0 = (ptile - seg * a.tiles_per_seg) * BM, n_q = H * sw;
    const int x0 = seg * sw, y0 = q0 / sw, r0 = q0 - y0 * sw;     // the tile's first pixel: row y0, column x0 + r0
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, r = lane & 15, g = lane >> 4;
    const int NO = MODE == CV_DJOIN ? 2 * C : C;          // output channels
    const int n0 = ctile * NT * 16;

    const int pix_bytes = conv_pixel_bytes(a.ck, ES), cols = sw + 2 * HALO, row_bytes = cols * pix_bytes;
    const int rows = int(div20_by(r0 + min(BM, n_q - q0) - 1, a.m_sw)) + 1 + 2 * HALO;

    Steps steps;
    const char* const w_tile = steps.weights(a.w, it.type, C, n0, NO, lane);
    steps.row_bytes = row_bytes;
    steps.pix_bytes = pix_bytes;
#pragma unroll
    for (int t = 0; t < MT; ++t) {
        const int q = r0 + min(t * 16 + r, n_q - 1 - q0), y = int(div20_by(q, a.m_sw)), x = q - y * sw;
        steps.x_at[t] = uint32_t(y * row_bytes + x * pix_bytes + g * Steps::X_LANE);
    }
    f32x4 acc[MT][NT];
#pragma unroll
    for (int t = 0; t < MT; ++t)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) acc[t][nt] = f32x4{0.f, 0.f, 0.f, 0.f};

    // the map whose convolution this is (in the join: argument `arg`)
    auto input_map = [&](int arg) -> const E* {
        if constexpr (MODE == CV_JOIN || MODE == CV_JOIN_BOTH) return conv_src<E>(a, arg ? it.src1 : it.src0, chw);
        else if constexpr (MODE == CV_FIRST) return binary ? (const E*)a.u + size_t(a.first_kept + i) * chw : conv_src<E>(a, it.src0, chw);
        else if constexpr (MODE == CV_SECOND) return (const E*)a.mid + size_t(a.first_kept + i) * chw;
        else if constexpr (MODE == CV_DSECOND) return a.gy + size_t(a.first_item + i) * chw;
        else if constexpr (MODE == CV_DFIRST) return a.dm + size_t(a.first_item + i) * chw;
        else return a.du + size_t(a.first_item + i) * chw;
    };
    const T* y_map = MODE == CV_DSECOND || MODE == CV_DFIRST ? conv_dst<T>(a, it.dst, chw) : nullptr;   // the item's result
    const T* u_map = binary ? (const T*)a.u + size_t(a.first_kept + i) * chw : conv_src<T>(a, it.src0, chw);

    // ---- what the results of this wave (tiles wave, wave + 4, ...) are combined with
    constexpr int NF = (MT * NT + 3) / 4;
    struct Out { f32x4 p, q; size_t e; int o, n; };       // n: channels of this lane's pixel that exist (0: no such pixel)
    Out fin[NF];
    auto request_operands = [&]() {
#pragma unroll
        for (int k = 0; k < NF; ++k) {
            const int tt = wave + 4 * k, t = tt / NT, nt = tt % NT;
            const int q = r0 + t * 16 + r, y = int(div20_by(q, a.m_sw)), x = x0 + q - y * sw;
            Out& f = fin[k];
            f.o = n0 + nt * 16 + g * 4;                   // lane: pixel r, output channels o .. o + 3
            f.n = tt < MT * NT && q0 - r0 + q < n_q && x < W ? max(0, min(4, NO - f.o)) : 0;
            f.e = (size_t(y0 + y) * W + x) * C + f.o;
            f.p = f.q = f32x4{0.f, 0.f, 0.f, 0.f};
            if (f.n <= 0) continue;
            if (!Tr::BWD && a.bias) f.p = load4<FULL>(a.bias + size_t(it.type) * C + f.o, f.n);
            if constexpr (MODE == CV_SECOND) f.q = load4<FULL>(u_map + f.e, f.n);
            if constexpr (MODE == CV_DSECOND) f.p = load4<FULL>((const T*)a.mid + size_t(a.first_kept + i) * chw + f.e, f.n);
            if constexpr (MODE == CV_DFIRST) {
                f.p = masked_gy<FULL>(a.gy + size_t(a.first_item + i) * chw + f.e, y_map + f.e, f.n);
                if (binary) f.q = load4<FULL>(u_map + f.e, f.n);
            }
        }
    };

    const int panels = (C + a.ck - 1) / a.ck;
#pragma unroll 1
    for (int panel = 0; panel < panels * (MODE == CV_JOIN ? 2 : 1); ++panel) {
        const int arg = MODE == CV_JOIN && panel >= panels ? 1 : 0;
        const int c0 = (panel - arg * panels) * a.ck;
        const int nj = min(a.ck / KS, (C - c0 + KS - 1) / KS);
        steps.panel(w_tile, c0, nj, arg);
        steps.share(wave);
        if constexpr (MODE == CV_JOIN_BOTH) {
            steps.row_bytes = 0;
            steps.pix_bytes = rows * row_bytes;           // from one argument to the other
        }

        // ---- stage rows x cols pixels x nj * KS channels
        if (panel > 0) __syncthreads();
        const int np = nj * (KS / PE), n_map = rows * cols * np, n_pieces = MODE == CV_JOIN_BOTH ? 2 * n_map : n_map;
        const uint32_t m_np = recip_of(np), m_cols = recip20_of(cols);
        const E* const src = input_map(arg);
        const E* const src1 = MODE == CV_JOIN_BOTH ? input_map(1) : nullptr;
        constexpr int UN = 6;
        u32x4 v[UN];
        uint32_t at[UN], keep[UN];
        auto load = [&](int base) {
#pragma unroll
            for (int k = 0; k < UN; ++k) {
                const int c = base + k * 256;
                const bool second = MODE == CV_JOIN_BOTH && c >= n_map;
                const uint32_t cc = second ? c - n_map : c;
                const uint32_t pix = div_by(cc, m_np), part = cc - pix * np, row = div20_by(pix, m_cols), col = pix - row * cols;
                at[k] = row * row_bytes + col * pix_bytes + part * 16 + (second ? uint32_t(rows * row_bytes) : 0u);
                const int y = y0 - HALO + int(row), x = x0 - HALO + int(col), ch = c0 + int(part) * PE;
                const bool inside = c < n_pieces && unsigned(y) < unsigned(H) && unsigned(x) < unsigned(W);
                keep[k] = inside ? ~0u : 0u;
                const size_t e = inside ? (size_t(y) * W + x) * C + ch : 0;      // outside: any piece, replaced by zeros below
                if constexpr (MODE == CV_DSECOND) v[k] = __builtin_bit_cast(u32x4, masked_gy<FULL>(src + e, y_map + e, inside ? C - ch : 0));
                else v[k] = load_piece<FULL>((second ? src1 : src) + e, inside ? C - ch : 0);
            }
        };
        auto store = [&](int base) {
#pragma unroll
            for (int k = 0; k < UN; ++k)
                if (base + k * 256 < n_pieces) *reinterpret_cast<u32x4*>(__builtin_assume_aligned(lds_raw + at[k], 16)) = v[k] & keep[k];
        };
        if constexpr (Steps::F32) {
            steps.request();
            for (int base = tid; base < n_pieces; base += 256 * UN) {
                load(base);
                store(base);
                // Everything has arrived.  Said aloud, because pieces that were requested and not stored would otherwise count
                // as outstanding, and every wait from here on would be for more than it needs.
                __builtin_amdgcn_s_waitcnt(0x0f70);       // vmcnt(0)
            }
        } else {
            // in bf16 the first pieces go ahead of the weights, which arrive while the pixels are written (fp32 has no registers for it, conv_waves)
            load(tid);
            __builtin_amdgcn_sched_barrier(0);
            steps.request();
            __builtin_amdgcn_sched_barrier(0);
            store(tid);
            for (int base = tid + 256 * UN; base < n_pieces; base += 256 * UN) {
                load(base);
                store(base);
                __builtin_amdgcn_s_waitcnt(0x0f70);
            }
        }
        if (panel == 0) request_operands();
        __syncthreads();

        steps.run(acc);
    }

    // ---- partial sums through LDS; wave w finishes tiles w, w + 4, ...
    __syncthreads();
    f32x4* red = reinterpret_cast<f32x4*>(lds_raw);
#pragma unroll
    for (int t = 0; t < MT; ++t)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) red[(wave * MT * NT + t * NT + nt) * 64 + lane] = acc[t][nt];
    __syncthreads();
    auto finish = [&](const Out& f, f32x4 v) {
        const int o = f.o, n = f.n;
        if constexpr (!Tr::BWD) {
            v.x += f.p.x; v.y += f.p.y; v.z += f.p.z; v.w += f.p.w;
            if constexpr (MODE == CV_SECOND) { v.x += f.q.x; v.y += f.q.y; v.z += f.q.z; v.w += f.q.w; }
#pragma unroll
            for (int c = 0; c < 4; ++c) v[c] = fmaxf(v[c], 0.f);
            T* dst = MODE == CV_SECOND ? conv_dst<T>(a, it.dst, chw) : (T*)(Tr::JOINS ? a.u : a.mid) + size_t(a.first_kept + i) * chw;
            store4<FULL>(dst + f.e, n, v);
        } else if constexpr (MODE == CV_DSECOND) {                       // dmid = result [mid > 0]
#pragma unroll
            for (int c = 0; c < 4; ++c) v[c] = f.p[c] > 0.f ? v[c] : 0.f;
            store4<FULL>(a.dm + size_t(a.first_item + i) * chw + f.e, n, v);
        } else if constexpr (MODE == CV_DFIRST) {                        // du = result + g
            v.x += f.p.x; v.y += f.p.y; v.z += f.p.z; v.w += f.p.w;
            if (binary) {                                                // dc = du [u > 0]
#pragma unroll
                for (int c = 0; c < 4; ++c) v[c] = f.q[c] > 0.f ? v[c] : 0.f;
                store4<FULL>(a.du + size_t(a.first_item + i) * chw + f.e, n, v);
            } else store4<FULL>(conv_route(a, a.gdst0[i], chw) + f.e, n, v);
        } else {                                                         // channels 0 .. C - 1: first argument, C .. 2 C - 1: second
            float* d0 = conv_route(a, a.gdst0[i], chw) + f.e;
            float* d1 = conv_route(a, a.gdst1[i], chw) + f.e - C;
            if (FULL || o + n <= C || o >= C) store4<FULL>(o >= C ? d1 : d0, n, v);
            else
                for (int c = 0; c < 4; ++c)
                    if (c < n) (o + c < C ? d0 : d1)[c] = v[c];
        }
    };
    bool again[NF];
#pragma unroll
    for (int k = 0; k < NF; ++k) {
        const Out& f = fin[k];
        again[k] = false;
        if (f.n <= 0) continue;
        const int tt = wave + 4 * k;
        f32x4 v = red[tt * 64 + lane];
#pragma unroll
        for (int w = 1; w < 4; ++w) {
            const f32x4 p = red[(w * MT * NT + tt) * 64 + lane];
            v.x += p.x; v.y += p.y; v.z += p.z; v.w += p.w;
        }
        if (!Tr::JOINS) again[k] = any_nan(v);
        finish(f, v);
    }
    if constexpr (!Tr::JOINS) {
        bool any = again[0];
#pragma unroll
        for (int k = 1; k < NF; ++k) any |= again[k];
        end_unless(any);
#pragma unroll
        for (int k = 0; k < NF; ++k) {
            const Out& f = fin[k];
            const int p = int((f.e - f.o) / C), y = p / W, x = p - y * W;
            if (!again[k] || !at_border(y, x, H, W)) continue;
            const E* in = input_map(0);
            finish(f, direct_sum<Tr::BWD>((const T*)a.w + size_t(it.type) * C * 9 * C, C, H, W, y, x, f.o, f.n, [&](int kh, int kw, int c) {
                const size_t e = (size_t(y + kh - 1) * W + (x + kw - 1)) * C + c;
                if constexpr (MODE == CV_DSECOND) return load_f32(y_map + e) > 0.f ? in[e] : 0.f;
                else return load_f32(in + e);
            }));
        }
    }
}

// ---- one thread per output element ----------------------------------------------------------------------------------
// Few channels, or maps of a few pixels: a 16 x 16 tile of the matrix instructions is then mostly padding, and taps that lie
// outside the map (8 of 9 on a 1 x 1 map) are multiplied all the same.  1000 modules, us, this kernel / k_conv / k_node:
// fp32 C = 3, 14 x 14: 33 / 89 / 55; bf16 C = 4, 28 x 28: 140 / 701 / 318; 20000 modules, fp32 C = 24, 1 x 1: 53 / 387 / 475.
template <typename T, ConvMode MODE>
__global__ __launch_bounds__(256) void k_conv_plain(const dynb_item* items, ConvArgs a)
{
    using Tr = ConvTraits<MODE>;
    static_assert(!Tr::BWD, "forward convolutions");
    const int i = blockIdx.y;
    const dynb_item it = items[i];
    const bool binary = it.src1 != DYNB_NO_ARG;           // uniform over the workgroup
    if (Tr::JOINS && !binary) return;
    const int C = a.C, H = a.H, W = a.W;
    const size_t chw = size_t(H) * W * C;
    const int e = int(blockIdx.x * 256u + threadIdx.x);
    if (unsigned(e) >= chw) return;
    const int p = e / C, co = e - p * C;
    float acc = a.bias ? a.bias[size_t(it.type) * C + co] : 0.f;
    if constexpr (Tr::JOINS) {
        const T* w = (const T*)a.w + (size_t(it.type) * C + co) * 2 * C;
        const T* x0 = conv_src<T>(a, it.src0, chw) + size_t(p) * C;
        const T* x1 = conv_src<T>(a, it.src1, chw) + size_t(p) * C;
        for (int ci = 0; ci < C; ++ci) acc += load_f32(x0 + ci) * load_f32(w + ci);
        for (int ci = 0; ci < C; ++ci) acc += load_f32(x1 + ci) * load_f32(w + C + ci);
        store_f32((T*)a.u + size_t(a.first_kept + i) * chw + e, fmaxf(acc, 0.f));
    } else {
        T* const mid = (T*)a.mid + size_t(a.first_kept + i) * chw;
        const T* const u = binary ? (const T*)a.u + size_t(a.first_kept + i) * chw : conv_src<T>(a, it.src0, chw);
        const T* const in = MODE == CV_SECOND ? mid : u;
        const T* const w = (const T*)a.w + (size_t(it.type) * C + co) * 9 * C;
        const int y = p / W, x = p - y * W;
        for (int kh = 0; kh < 3; ++kh) {
            if (unsigned(y + kh - 1) >= unsigned(H)) continue;
            for (int kw = 0; kw < 3; ++kw) {
                if (unsigned(x + kw - 1) >= unsigned(W)) continue;
                const T* px = in + (size_t(y + kh - 1) * W + (x + kw - 1)) * C;
                const T* wk = w + (kh * 3 + kw) * C;
                for (int ci = 0; ci < C; ++ci) acc += load_f32(px + ci) * load_f32(wk + ci);
            }
        }
        if constexpr (MODE == CV_SECOND) store_f32(conv_dst<T>(a, it.dst, chw) + e, fmaxf(acc + load_f32(u + e), 0.f));
        else store_f32(mid + e, fmaxf(acc, 0.f));
    }
}

// ---- a whole module per workgroup -----------------------------------------------------------------------------------
// Small maps and few channels: a module is then a few microseconds of one CU, no more than a launch takes to get going (the
// kernel's arguments, the item, its map: three memory latencies, one after the other), and three launches for it would be
// spent on that (8 programs, fp32, C = 16, 8 x 8, whole pass: 53 -> 34 us).  A workgroup of 8 waves owns an item; the input map and mid live in two LDS tiles with zero borders, a unit of
// work is MT x 16 pixels x 16 output channels, a wave takes every eighth.  Joins read their arguments' fragments straight
// from global memory (every element is used once per channel tile) and leave u in the first tile.
struct NodeArgs {
    const void* w1; const float* b1;
    const void* w3a; const float* b3a;
    const void* w3b; const float* b3b;
    int32_t count;
    int32_t keep;                 // u and mid are also written to the maps of the backward pass
};

struct NodeKernelArgs { const dynb_item* items; NodeArgs nw; ConvArgs a; };             // k_node's parameters

// The rare end of k_node: sums that any_nan speaks of.  mid_nan (all waves): mid's border and every result are taken again, else this
// lane's results at the border.  Everything is read anew, so that the kernel need not hold registers for it (it had to move
// scalar registers into vector lanes: 2 % of a pass, fp32, C = 32, 8 x 8).
template <typename T, int MT>
__device__ __forceinline__ void node_again(bool mid_nan, bool nan)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
    const void* args = (const void*)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(args));
    const NodeKernelArgs k = *static_cast<const NodeKernelArgs*>(args);
    const ConvArgs& a = k.a;
    const int i = int(blockIdx.x & 7) * int(gridDim.x >> 3) + int(blockIdx.x >> 3);
    const dynb_item it = k.items[i];
    const int C = a.C, H = a.H, W = a.W, P = H * W, pix_bytes = conv_pixel_bytes(a.ck, int(sizeof(T))), row_bytes = (W + 2) * pix_bytes;
    const uint32_t second = uint32_t((H + 2) * row_bytes);                              // the second tile
    const size_t chw = size_t(P) * C;
    const int lane = threadIdx.x & 63, n_ct = (C + 15) / 16, n_units = n_ct * ((P + MT * 16 - 1) / (MT * 16));
    T* const dst = conv_dst<T>(a, it.dst, chw);
    // this wave's results of a convolution: fn(pixel, y, x, channels o .. o + n - 1, sum, bias, address of the pixel's top left tap)
    auto each = [&](const void* w, const float* bias, uint32_t tile, bool inner, auto&& fn) {
#pragma unroll 1
        for (int u = threadIdx.x >> 6; u < n_units; u += 8)
#pragma unroll 1
            for (int t = 0; t < MT; ++t) {
                const int pt = u / n_ct, p = (pt * MT + t) * 16 + (lane & 15), y = p / W, x = p - y * W;
                const int o = (u - pt * n_ct) * 16 + (lane >> 4) * 4, n = min(4, C - o);
                if (p >= P || n <= 0 || !(inner || at_border(y, x, H, W))) continue;
                const uint32_t at = uint32_t(y * row_bytes + x * pix_bytes);
                const f32x4 b = bias ? load4<false>(bias + size_t(it.type) * C + o, n) : f32x4{0.f, 0.f, 0.f, 0.f};
                fn(p, o, n, at + uint32_t(row_bytes + pix_bytes), b,
                   direct_sum<false>((const T*)w + size_t(it.type) * C * 9 * C, C, H, W, y, x, o, n, [&](int kh, int kw, int c) {
                       return load_f32(reinterpret_cast<const T*>(lds_raw + tile + at + uint32_t(kh * row_bytes + kw * pix_bytes)) + c);
                   }));
            }
    };
    if (mid_nan) {
        __syncthreads();
        each(k.nw.w3a, k.nw.b3a, 0, false, [&](int p, int o, int n, uint32_t centre, const f32x4& b, f32x4 v) {
            for (int c = 0; c < 4; ++c) v[c] = fmaxf(v[c] + b[c], 0.f);
            store4<false>(reinterpret_cast<T*>(lds_raw + second + centre) + o, n, v);
            if (k.nw.keep) store4<false>((T*)a.mid + size_t(a.first_kept + i) * chw + size_t(p) * C + o, n, v);
        });
        __syncthreads();
    }
    if (mid_nan || nan)
        each(k.nw.w3b, k.nw.b3b, second, mid_nan, [&](int p, int o, int n, uint32_t centre, const f32x4& b, f32x4 v) {
            const f32x4 res = load4<false>(reinterpret_cast<const T*>(lds_raw + centre) + o, n);
            for (int c = 0; c < 4; ++c) v[c] = fmaxf(v[c] + b[c] + res[c], 0.f);
            store4<false>(dst + size_t(p) * C + o, n, v);
        });
}

template <typename T, int MT, bool FULL, int G>
__global__ __launch_bounds__(512, MT == 1 ? 4 : 2) void k_node(const dynb_item* items, NodeArgs nw, ConvArgs a)
{
    using First = ConvSteps<T, CV_FIRST, MT, 1, FULL, G>;
    using Second = ConvSteps<T, CV_SECOND, MT, 1, FULL, G>;
    using Join = ConvSteps<T, CV_JOIN, MT, 1, FULL>;
    constexpr int ES = int(sizeof(T)), KS = First::KS, PE = First::PE, NTHR = 512, NWAVE = 8;
    extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
    // consecutive workgroups go to the chip's 8 dies in turn: every die gets one run of items (they are sorted by function)
    const int i = int(blockIdx.x & 7) * int(gridDim.x >> 3) + int(blockIdx.x >> 3);
    if (i >= nw.count) return;
    const dynb_item it = items[i];
    const bool binary = it.src1 != DYNB_NO_ARG;           // uniform over the workgroup
    const int C = a.C, H = a.H, W = a.W, P = H * W, cols = W + 2;
    const size_t chw = size_t(P) * C;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, r = lane & 15, g = lane >> 4;
    const int nj = a.ck / KS, pix_bytes = conv_pixel_bytes(a.ck, ES), row_bytes = cols * pix_bytes, tile_bytes = (H + 2) * row_bytes;
    const int n_ct = (C + 15) / 16, n_units = n_ct * ((P + MT * 16 - 1) / (MT * 16));

    // unit u: channel tile u % n_ct of pixel tiles u / n_ct * MT ..
    int n0 = 0, p0 = 0;
    uint32_t at[MT];                                      // tile offset of this lane's pixel (top left tap), without channels
    auto unit = [&](int u) {
        const int pt = u / n_ct;
        n0 = (u - pt * n_ct) * 16;
        p0 = pt * MT * 16;
#pragma unroll
        for (int t = 0; t < MT; ++t) {
            const int p = min(p0 + t * 16 + r, P - 1), y = int(div20_by(p, a.m_sw));
            at[t] = uint32_t(y * row_bytes + (p - y * W) * pix_bytes);
        }
    };
    const uint32_t centre = uint32_t(row_bytes + pix_bytes);
    f32x4 acc[MT][1];
    auto clear = [&]() {
#pragma unroll
        for (int t = 0; t < MT; ++t) acc[t][0] = f32x4{0.f, 0.f, 0.f, 0.f};
    };
    auto prepare = [&](auto& steps, const void* w, uint32_t tile) {
        steps.panel(steps.weights(w, it.type, C, n0, C, lane), 0, nj, 0);
        steps.row_bytes = row_bytes;
        steps.pix_bytes = pix_bytes;
        steps.s0 = 0;
        steps.n_steps = nj * 9;
#pragma unroll
        for (int t = 0; t < MT; ++t) steps.x_at[t] = tile + at[t] + uint32_t(g * First::X_LANE);
        steps.request();
    };
    auto bias_of = [&](const float* b) -> f32x4 {
        return b ? load4<FULL>(b + size_t(it.type) * C + n0 + g * 4, C - n0 - g * 4) : f32x4{0.f, 0.f, 0.f, 0.f};
    };
    // fn(pixel index, its tile offset, channels o .. o + n - 1 of it): this lane's results of pixel tile t
    auto results = [&](auto&& fn) {
        const int o = n0 + g * 4, n = min(4, C - o);
#pragma unroll
        for (int t = 0; t < MT; ++t) {
            const int p = p0 + t * 16 + r;
            if (p < P && n > 0) fn(t, p, o, n);
        }
    };

    if (wave < n_units) unit(wave);
    First first;
    if (!binary && wave < n_units) prepare(first, nw.w3a, 0);

    // ---- both tiles: zeros, and the argument's map in the middle of the first
    {
        const T* src = conv_src<T>(a, it.src0, chw);
        const int np = a.ck * ES / 16, n_map = binary ? 0 : (H + 2) * cols * np;       // 16-byte pieces
        const uint32_t m_np = recip_of(np), m_cols = recip20_of(cols);
        constexpr int UN = 4;
        for (int base = tid; base < n_map; base += NTHR * UN) {
            u32x4 v[UN];
            uint32_t to[UN], mask[UN];
#pragma unroll
            for (int k = 0; k < UN; ++k) {
                const int c = base + k * NTHR;
                const uint32_t pix = div_by(c, m_np), part = c - pix * np, row = div20_by(pix, m_cols), col = pix - row * cols;
                to[k] = row * row_bytes + col * pix_bytes + part * 16;
                const int y = int(row) - 1, x = int(col) - 1, ch = int(part) * PE;
                const bool inside = c < n_map && unsigned(y) < unsigned(H) && unsigned(x) < unsigned(W);
                mask[k] = inside ? ~0u : 0u;
                v[k] = load_piece<FULL>(src + (inside ? (size_t(y) * W + x) * C + ch : 0), inside ? C - ch : 0);
            }
#pragma unroll
            for (int k = 0; k < UN; ++k)
                if (base + k * NTHR < n_map) *reinterpret_cast<u32x4*>(__builtin_assume_aligned(lds_raw + to[k], 16)) = v[k] & mask[k];
            __builtin_amdgcn_s_waitcnt(0x0f70);           // vmcnt(0), see k_conv
        }
        for (int c = tid + (binary ? 0 : tile_bytes / 16); c < 2 * tile_bytes / 16; c += NTHR)
            *reinterpret_cast<u32x4*>(lds_raw + size_t(c) * 16) = u32x4{0u, 0u, 0u, 0u};
    }
    __syncthreads();

    if (binary) {
        // ---- u = ReLU(conv1x1(concat(arguments)) + b1) into the first tile
        for (int u = wave; u < n_units; u += NWAVE) {
            unit(u);
            const f32x4 b = bias_of(nw.b1);
            Join join;
            const char* w_tile = join.weights(nw.w1, it.type, C, n0, C, lane);
            join.s0 = 0;
            join.n_steps = nj;
            clear();
#pragma unroll 1
            for (int arg = 0; arg < 2; ++arg) {
                const T* src = conv_src<T>(a, arg ? it.src1 : it.src0, chw);
                join.panel(w_tile, 0, nj, arg);
                constexpr int UN = 4;
#pragma unroll 1
                for (int j0 = 0; j0 < nj; j0 += UN) {
                    u32x4 w[UN][1][1], x[UN][MT];
#pragma unroll
                    for (int k = 0; k < UN; ++k) {
                        const int j = min(j0 + k, nj - 1), c = j * KS + g * PE;
                        join.load_w(j, w[k]);
#pragma unroll
                        for (int t = 0; t < MT; ++t) x[k][t] = load_piece<FULL>(src + size_t(min(p0 + t * 16 + r, P - 1)) * C + c, C - c);
                    }
#pragma unroll
                    for (int k = 0; k < UN; ++k)
                        if (j0 + k < nj) Join::multiply(acc, w[k], 0, x[k]);
                }
            }
            results([&](int t, int p, int o, int n) {
                f32x4 v = acc[t][0];
#pragma unroll
                for (int c = 0; c < 4; ++c) v[c] = fmaxf(v[c] + b[c], 0.f);
                store4<FULL>(reinterpret_cast<T*>(lds_raw + at[t] + centre) + o, n, v);
                if (nw.keep) store4<FULL>((T*)a.u + size_t(a.first_kept + i) * chw + size_t(p) * C + o, n, v);
            });
        }
        if (wave < n_units) { unit(wave); prepare(first, nw.w3a, 0); }
        __syncthreads();
    }

    auto put_mid = [&](int t, int p, int o, int n, f32x4 v, const f32x4& b) {
#pragma unroll
        for (int c = 0; c < 4; ++c) v[c] = fmaxf(v[c] + b[c], 0.f);
        store4<FULL>(reinterpret_cast<T*>(lds_raw + tile_bytes + at[t] + centre) + o, n, v);
        if (nw.keep) store4<FULL>((T*)a.mid + size_t(a.first_kept + i) * chw + size_t(p) * C + o, n, v);
    };
    T* const dst = conv_dst<T>(a, it.dst, chw);
    auto put_result = [&](int t, int p, int o, int n, f32x4 v, const f32x4& b) {
        const f32x4 res = load4<FULL>(reinterpret_cast<const T*>(lds_raw + at[t] + centre) + o, n);
#pragma unroll
        for (int c = 0; c < 4; ++c) v[c] = fmaxf(v[c] + b[c] + res[c], 0.f);
        store4<FULL>(dst + size_t(p) * C + o, n, v);
    };
    // (any_nan: a NaN in mid concerns all waves and is noted in the padding of the second tile's first pixel, which is zero)
    uint32_t* const flag = reinterpret_cast<uint32_t*>(lds_raw + tile_bytes + a.ck * ES);
    bool nan = false;

    // ---- mid = ReLU(conv3x3(first tile) + b3a) into the second tile
    for (int u = wave; u < n_units; u += NWAVE) {
        if (u != wave) { unit(u); prepare(first, nw.w3a, 0); }
        const f32x4 b = bias_of(nw.b3a);
        clear();
        first.run(acc);
        results([&](int t, int p, int o, int n) {
            nan |= any_nan(acc[t][0]);
            put_mid(t, p, o, n, acc[t][0], b);
        });
    }
    if (nan) *flag = 1;
    Second second;
    if (wave < n_units) { unit(wave); prepare(second, nw.w3b, uint32_t(tile_bytes)); }
    __syncthreads();

    // ---- result = ReLU(conv3x3(second tile) + b3b + first tile)
    nan = false;
    for (int u = wave; u < n_units; u += NWAVE) {
        if (u != wave) { unit(u); prepare(second, nw.w3b, uint32_t(tile_bytes)); }
        const f32x4 b = bias_of(nw.b3b);
        clear();
        second.run(acc);
        results([&](int t, int p, int o, int n) {
            nan |= any_nan(acc[t][0]);
            put_result(t, p, o, n, acc[t][0], b);
        });
    }
    // (Read before these sums, the flag would wait for their weights: the compiler gives it a register that they return behind.)
    const uint32_t mid_nan = __builtin_amdgcn_readfirstlane(*flag);
    end_unless(nan || mid_nan != 0);
    node_again<T, MT>(mid_nan != 0, nan);
}

// ---- launching
constexpr int CONV_LDS_MAX = 80 * 1024;                                  // two workgroups per CU

// staged pixels of a tile of mt x 16 pixels, which start anywhere in a row
inline int conv_tile_pixels(const ConvArgs& a, int mt, int halo)
{
    const int n_pix = std::min(mt * 16, a.H * a.sw);
    return std::min(conv_rows(a.sw - 1, n_pix, a.sw, halo), a.H + 2 * halo) * (a.sw + 2 * halo);
}

// Channels staged at a time: as many as fit beside the pixels of the largest tile, whatever this tile has, in panels of nearly equal
// size: a panel is what the waves split, so the panels are part of the order of summation, and a launch group's width (which
// picks the tile) must not change a result's bits.
template <int HALO, int ES>
int conv_panel(const ConvArgs& a)
{
    constexpr int KS = ES == 4 ? 16 : 32;
    const int steps = (a.C + KS - 1) / KS;
    const int fit = std::max(1, (CONV_LDS_MAX / conv_tile_pixels(a, 4, HALO) - 16) / (KS * ES));
    const int panels = (steps + fit - 1) / fit;
    return (steps + panels - 1) / panels * KS;
}

// both arguments of a join, all channels, of a tile of mt x 16 pixels
template <int ES>
size_t conv_both_bytes(const ConvArgs& a, int mt)
{
    constexpr int KS = ES == 4 ? 16 : 32;
    return size_t(2) * conv_tile_pixels(a, mt, 0) * conv_pixel_bytes((a.C + KS - 1) / KS * KS, ES);
}

template <typename T, ConvMode MODE, int MT, int NT, bool FULL, int G>
int launch_conv_tile(const dynb_item* items, ConvArgs a, int count, hipStream_t st)
{
    using Tr = ConvTraits<MODE>;
    constexpr int ES = Tr::BWD ? 4 : int(sizeof(T)), KS = ES == 4 ? 16 : 32;
    static std::atomic<uint64_t> attr_set{0};                            // one bit per device
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return DYNB_E_HIP;
    if (!(attr_set.load() >> (dev & 63) & 1)) {
        if (hipFuncSetAttribute(reinterpret_cast<const void*>(k_conv<T, MODE, MT, NT, FULL, G>), hipFuncAttributeMaxDynamicSharedMemorySize, CONV_LDS_MAX) != hipSuccess)
            return DYNB_E_HIP;
        attr_set.fetch_or(uint64_t(1) << (dev & 63));
    }
    const int n_q = a.H * a.sw, n_seg = (a.W + a.sw - 1) / a.sw;
    a.tiles_per_seg = (n_q + MT * 16 - 1) / (MT * 16);
    a.n_ctile = ((MODE == CV_DJOIN ? 2 * a.C : a.C) + NT * 16 - 1) / (NT * 16);
    const int pixels = conv_tile_pixels(a, MT, Tr::HALO);
    a.ck = MODE == CV_JOIN_BOTH ? (a.C + KS - 1) / KS * KS : conv_panel<Tr::HALO, ES>(a);
    a.m_sw = recip20_of(a.sw);
    const size_t lds = std::max<size_t>(MODE == CV_JOIN_BOTH ? conv_both_bytes<ES>(a, MT) : size_t(pixels) * conv_pixel_bytes(a.ck, ES), size_t(4) * MT * NT * 1024);
    if (lds > CONV_LDS_MAX) return DYNB_E_UNSUPPORTED;                   // cannot happen: sw <= 32
    // A row of a grid holds less than 2^32 threads (and nobody says so: the launch just does less).  Only the gradients of maps of
    // half a billion pixels with fewer than 4 channels would need more, which a parameter gradient's workgroup walks for many seconds.
    const long long groups = (long long)n_seg * a.tiles_per_seg * a.n_ctile;
    if (groups >= 1 << 24) return DYNB_E_UNSUPPORTED;
    // Runs of items for the dies as long as a function's weights stay in a die's L2 of 4 MB.  Larger ones every die would read for itself, for its
    // items alone; in the plain order the items of a function run at the same time and a die reads its channel tiles' share for all of them.  Kernel
    // time of the 3x3s of 64 balanced trees, runs / plain order: C = 1024 fp32, 4 x 4 10070 / 7740 us, bf16, 5 x 5 4800 / 2630; C = 512, 5 x 5,
    // fp32 2730 / 2700; C = 256, 7 x 7, fp32 (2.4 MB) 1360 / 1390.
    const long long weights = (long long)Tr::TAPS * a.C * (MODE == CV_DJOIN ? 2 * a.C : a.C) * int(sizeof(T));
    a.runs = groups > 1 && count >= 16 && weights <= 4 << 20 && groups * groups * count < 1ll << 32 ? recip_of(uint32_t(groups)) : 0;
    a.n_groups = uint32_t(groups);
    a.run_q = uint32_t(groups * count >> 3);
    a.run_r = uint32_t(groups * count & 7);
    hipLaunchKernelGGL((k_conv<T, MODE, MT, NT, FULL, G>), dim3(unsigned(groups), unsigned(count)), dim3(256), lds, st, items, a);
    return DYNB_OK;
}

// One convolution for `count` (<= 65535) items.  The tile is the one that finishes first in a simple account of a CU's time:
// it runs ceil(workgroups / 256) workgroups, each with its MFMAs (a quarter of the steps per SIMD), the staging of its
// pixels at about 24 bytes per clock, and about 1200 clocks of its own.  Large tiles read weights and halos less
// often per output; small ones split the launch into CU-sized shares more finely.  Measured for fp32, C = 128, 14 x 14, us:
//     items      1     2     4     6     9     12    15    18    21    25
//     4 x 2    15.2  15.0  15.1  15.4  15.8  16.3  16.6  27.1  27.1  27.2
//     2 x 2    10.4  10.5  10.6  10.8  10.9  17.4  17.7  18.1  23.6  23.2
//     2 x 1     7.6   7.6   7.9  11.5  11.6  15.4  19.7  21.7  23.3  26.3
//     1 x 1     6.5   6.7   9.0  11.2  15.1  17.6  23.1  25.6  28.0  32.6
template <typename T, ConvMode MODE, bool FULL, int G>
int launch_conv_full(const dynb_item* items, ConvArgs a, int count, hipStream_t st)
{
    using Tr = ConvTraits<MODE>;
    constexpr int ES = Tr::BWD ? 4 : int(sizeof(T)), KS = ES == 4 ? 16 : 32, STEP_CLOCKS = ES == 4 ? 128 : 16;
    const long long ptiles = (long long)((a.W + a.sw - 1) / a.sw) * ((a.H * a.sw + 15) / 16), ctiles = ((MODE == CV_DJOIN ? 2 * a.C : a.C) + 15) / 16;
    const long long steps = (long long)((a.C + KS - 1) / KS) * Tr::TAPS * (MODE == CV_JOIN ? 2 : 1);
    auto clocks = [&](int mt, int nt) {
        if (MODE == CV_JOIN_BOTH && conv_both_bytes<ES>(a, mt) > CONV_LDS_MAX) return LLONG_MAX;
        const long long groups = (long long)count * ((ptiles + mt - 1) / mt) * ((ctiles + nt - 1) / nt);
        const long long staged = (long long)conv_tile_pixels(a, mt, Tr::HALO) * a.C * ES * (MODE == CV_JOIN || MODE == CV_JOIN_BOTH || MODE == CV_DSECOND ? 2 : 1);
        return (groups + 255) / 256 * (mt * nt * ((steps + 3) / 4) * STEP_CLOCKS + staged / 24 + 1200);
    };
    const long long c42 = clocks(4, 2), c22 = clocks(2, 2), c21 = clocks(2, 1), c11 = clocks(1, 1);
    const long long best = std::min(std::min(c42, c22), std::min(c21, c11));
    if (best == c42) return launch_conv_tile<T, MODE, 4, 2, FULL, G>(items, a, count, st);
    if (best == c22) return launch_conv_tile<T, MODE, 2, 2, FULL, G>(items, a, count, st);
    if (best == c21) return launch_conv_tile<T, MODE, 2, 1, FULL, G>(items, a, count, st);
    return launch_conv_tile<T, MODE, 1, 1, FULL, G>(items, a, count, st);
}

template <typename T, ConvMode MODE>
int launch_conv(const dynb_item* items, const ConvArgs& args, int count, hipStream_t st)
{
    ConvArgs a = args;
    using Tr = ConvTraits<MODE>;
    constexpr int ES = Tr::BWD ? 4 : int(sizeof(T)), KS = ES == 4 ? 16 : 32;
    const int n_seg = (a.W + 31) / 32;
    a.sw = (a.W + n_seg - 1) / n_seg;
    // A join takes both arguments at once where a 2 x 2 tile's fit beside another workgroup's (a rule by the shape: it is part of the order of
    // summation), and a 4 x 2 tile if its own do.  One after the other they were two waits for memory: 8.0 us a lone workgroup of bf16, C = 128, 7 x 7; at
    // once 5 for the whole launch.  With one workgroup a CU, or in 1 x 1 tiles, both at once take longer: kernel time of the joins of 64
    // balanced trees, fp32, one after the other / at once: C = 128, 14 x 14 354 / 430 us in 4 x 2 tiles, 349 in 2 x 2; C = 256, 7 x 7 263 / 337 in
    // 4 x 2, 570 in 1 x 1; C = 512, 5 x 5 470 / 655 in 2 x 2; C = 1024, 4 x 4 1580 / 2640 in 1 x 1.
    if constexpr (MODE == CV_JOIN) {
        if (conv_both_bytes<ES>(a, 2) <= CONV_LDS_MAX) {
            if (a.C % KS != 0) return launch_conv_full<T, CV_JOIN_BOTH, false, 1>(items, a, count, st);
            if (a.C % (2 * KS) == 0) return launch_conv_full<T, CV_JOIN_BOTH, true, 2>(items, a, count, st);
            return launch_conv_full<T, CV_JOIN_BOTH, true, 1>(items, a, count, st);
        }
    }
    if (a.C % KS != 0) return launch_conv_full<T, MODE, false, 1>(items, a, count, st);
    if constexpr (!Tr::JOINS && !Tr::BWD) {
        if (a.C % (KS * 2) == 0 && conv_panel<Tr::HALO, ES>(a) % (KS * 2) == 0) return launch_conv_full<T, MODE, true, 2>(items, a, count, st);
    }
    return launch_conv_full<T, MODE, true, 1>(items, a, count, st);
}

// The three ways to run a module's convolutions are chosen by the shape alone, never by how many modules there are: each adds up in
// an order of its own, and another schedule must not change a result's bits.

// k_conv_plain, where its products cost less than the tiles' padding: a product inside the map takes it some 3 ps (all CUs
// busy), a 16 x 16 tile takes k_conv 9 ns (fp32), 14 to 22 ns (bf16, fewer than 16 channels: 32 are summed at a time) or 10 ns (bf16).
// 20000 modules, us, plain / tiles, on the two sides of the line: fp32 4 x 4, C = 5: 166 / 196, C = 6: 213 / 198; 14 x 14, C = 4:
// 885 / 906, C = 5: 2210 / 1571; 1 x 1, C = 100: 825 / 2636; bf16 10 x 10, C = 6: 1353 / 2560, C = 8: 1800 / 1382; 3 x 3, C = 12:
// 356 / 404, C = 16: 988 / 292.
template <typename T>
bool plain_shape(const ConvArgs& a)
{
    const double taps = (3.0 * a.H - 2) * (3.0 * a.W - 2);               // inside the map, over all pixels
    const double tiles = double((size_t(a.H) * a.W + 15) / 16) * ((a.C + 15) / 16);
    return double(a.C) * a.C * taps <= tiles * (sizeof(T) == 4 ? 3000 : a.C < 16 ? 7100 : 3500);
}

template <typename T, ConvMode MODE>
int launch_conv_plain(const dynb_item* items, const ConvArgs& a, int count, hipStream_t st)
{
    const size_t chw = size_t(a.H) * a.W * a.C;
    hipLaunchKernelGGL((k_conv_plain<T, MODE>), dim3(unsigned((chw + 255) / 256), unsigned(count)), dim3(256), 0, st, items, a);
    return DYNB_OK;
}

// k_node: pixel tiles per unit: 4 read the weights a quarter as often, 1 gives all waves work where there are few tiles.  us for one
// module, 1 / 4 tiles: fp32 C = 16, 8 x 8 6.1 / 9.5, 14 x 14 12.3 / 10.1; C = 32, 7 x 7 12.0 / 14.5; bf16 C = 16, 14 x 14 21.6 / 14.4, 20 x 20 33.8 /
// 16.1; C = 24, 14 x 14 34.8 / 16.1; C = 32, 14 x 14 14.7 / 9.8.
inline bool node_wide(int pt, int ct) { return ((pt + 3) / 4 * ct + 7) / 8 * 4 <= (pt * ct + 7) / 8; }

// Whole modules by k_node, where that takes one CU no longer than two or three launches of k_conv take to get going (5 us
// each) and two tiles fit LDS.  A CU's time: its MFMAs, or its weights, of which one CU was seen to take in some 12 bytes a clock
// (fp32, C = 16, 8 x 8: 8 us an item against 3 x 5; bf16, C = 128, 7 x 7, 590 KB of weights: 16 to 22 us, in pairs of steps, against 2 x 5 to 5 + 2 x 9,
// which costs a pass over 1, 8 and 64 programs with their narrow labels 328, 520 and 658 us against 180, 293 and 484, and saves one over 256, and
// over 256 balanced trees, 692 against 764 and 365 against 552: the rule goes by the shape alone and decides for the narrow ones),
// and with every round of units a wait for weights: one lone module, bf16 C = 48, 14 x 14, 5 rounds: 58 us against 15 by k_conv;
// C = 20, 20 x 20, 7 rounds: 79 / 20 (and 35 by k_conv_plain); C = 24, 14 x 14, 1 round of wide units: 16 / 15.  Below 16 channels the
// tiles are cut short and k_conv wins from two rounds on (bf16 C = 8, 14 x 14: 21 / 14) or with many modules (fp32 C = 6, 4 x 4,
// 20000: 335 / 198); so it does on maps of a few pixels with cut steps (2 x 2, 20000: fp32 C = 20 474 / 386, bf16 C = 16 420 / 282).
template <typename T>
bool node_shape(const ConvArgs& a)
{
    constexpr int ES = int(sizeof(T)), KS = ES == 4 ? 16 : 32, STEP_CLOCKS = ES == 4 ? 128 : 16;
    const long long steps = (a.C + KS - 1) / KS, P = (long long)a.H * a.W;
    const long long lds = 2ll * (a.H + 2) * (a.W + 2) * conv_pixel_bytes(int(steps * KS), ES);
    if (a.C < 16 || a.W > 64 || P > 2048 || lds > 160 * 1024 || (P < 9 && a.C < 24 && a.C % KS != 0)) return false;
    const int pt = int(P + 15) / 16, ct = (a.C + 15) / 16;
    const int rounds = ((node_wide(pt, ct) ? (pt + 3) / 4 : pt) * ct + 7) / 8;
    const long long mfma = (long long)pt * ct * steps * 9 * 2 * STEP_CLOCKS / 4, weights = 2ll * 9 * a.C * a.C * ES / 12;
    return rounds <= 2 && std::max(mfma, weights) <= 10000;
}

template <typename T, int MT, bool FULL, int G>
int launch_node_tile(const dynb_item* items, const NodeArgs& nw, const ConvArgs& a, hipStream_t st)
{
    static std::atomic<uint64_t> attr_set{0};                            // one bit per device
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return DYNB_E_HIP;
    if (!(attr_set.load() >> (dev & 63) & 1)) {
        if (hipFuncSetAttribute(reinterpret_cast<const void*>(k_node<T, MT, FULL, G>), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024) != hipSuccess)
            return DYNB_E_HIP;
        attr_set.fetch_or(uint64_t(1) << (dev & 63));
    }
    const size_t lds = size_t(2) * (a.H + 2) * (a.W + 2) * conv_pixel_bytes(a.ck, int(sizeof(T)));
    hipLaunchKernelGGL((k_node<T, MT, FULL, G>), dim3(unsigned((nw.count + 7) / 8 * 8)), dim3(512), lds, st, items, nw, a);
    return DYNB_OK;
}

template <typename T>
int launch_node(const dynb_item* items, const NodeArgs& nw, ConvArgs a, hipStream_t st)
{
    constexpr int KS = sizeof(T) == 4 ? 16 : 32;
    a.ck = (a.C + KS - 1) / KS * KS;
    a.m_sw = recip20_of(a.W);
    const int pt = (a.H * a.W + 15) / 16, ct = (a.C + 15) / 16;
    const bool wide = node_wide(pt, ct);
    if (a.C % KS != 0) return wide ? launch_node_tile<T, 4, false, 1>(items, nw, a, st) : launch_node_tile<T, 1, false, 1>(items, nw, a, st);
    auto with = [&](auto group) {
        constexpr int G = decltype(group)::value;
        return wide ? launch_node_tile<T, 4, true, G>(items, nw, a, st) : launch_node_tile<T, 1, true, G>(items, nw, a, st);
    };
    return a.C % (2 * KS) == 0 ? with(std::integral_constant<int, 2>{}) : with(std::integral_constant<int, 1>{});
}

}  // namespace
