// Backward pass of an executed plan (paper: Results / IEP times the backward pass next to inference and
// expects the same gains from batching, since the pools are the same).  The launch groups are walked in
// reverse; inside a group every node is independent.  The gradients of the parameters are summed function by function
// afterwards, over all its nodes in item order, so the result does not depend on scheduling.
//
// For a node with residual block input u, mid = ReLU(conv_a(u) + b_a), y = ReLU(u + conv_b(mid) + b_b) and
// incoming gradient gy:
//     g    = gy * [y > 0]                      db_b += sum_p g      dW_b += g (x) mid
//     dmid = conv_b^T(g) * [mid > 0]           db_a += sum_p dmid   dW_a += dmid (x) u
//     du   = g + conv_a^T(dmid)
// and for a two-argument function, u = ReLU(conv1x1(concat(a0, a1)) + b1):
//     dc   = du * [u > 0]                      db_1 += sum_p dc     dW_1 += dc (x) concat
//     da0  = W1[:, :C]^T dc,  da1 = W1[:, C:]^T dc
// The node results y, u of two-argument functions and mid come from the forward pass (a plan made with DYNB_PLAN_KEEP
// leaves every one of them in the workspace).
// Two kernel families with the same semantics, like the forward pass: fused kernels for bf16, C = 128, 14 x 14 (further
// down), and for any other shape, fp32 or bf16 values and weights, one launch per transposed convolution of a launch
// group (k_conv, iep_conv.h) and one for the parameter gradients of the whole plan (k_wgrad); fp32 gradients throughout.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <string>
#include <type_traits>
#include <vector>

#include "device_utils.h"
#include "iep_conv.h"
#include "iep_mfma.h"
#include "plan_internal.h"

using dynb::fail;

#define HIP_TRY(expr, what)                                                                   \
    do {                                                                                      \
        hipError_t e_ = (expr);                                                               \
        if (e_ != hipSuccess)                                                                 \
            return fail(DYNB_E_HIP, std::string(what) + ": " + hipGetErrorString(e_));        \
    } while (0)

namespace {

// Parameter gradients of every function, any shape: a workgroup owns a 32 x 32 block (output x input channels) of one
// function's weight gradient, all taps of it, and sums it over the function's items and their pixels,
//     D[32 co][32 ci] += G[32 co][2 pixels] * IN[2 pixels][32 ci]     (v_mfma_f32_32x32x2: fp32 products and sums)
// Second 3x3: G = g, IN = mid; first 3x3: G = dmid, IN = u; JOIN: the 1x1 (G = dc, IN = the arguments).  The functions with the most items come
// first, of both 3x3s: a workgroup takes some 14 us an item beside another on its CU, and the last
// ones should be short (fp32, C = 128, 14 x 14: a training step of 21 programs 2685 us with the functions in order, 2633 so; of 8 programs 1435 / 1387).
// An item's 32 + 32 channels are staged into LDS as fp32, pixel-major without padding (a fragment, two pixels x 32
// channels, is then 64 consecutive words), the input with its halo; a step of two pixels reads 1 + TAPS fragments
// for TAPS MFMAs of 64 clocks.  The waves split an item's pixels and meet in LDS at the end, in wave order.  Maps that do
// not fit are taken in bands of rows and segments of columns; of maps of a few pixels several items are staged at a time.
// (Per launch group, one thread per gradient element, the sums took most of a training step's 179 ms at 21 programs,
// C = 128, 14 x 14.)
struct WgradArgs {
    const dynb_item* items;       // all items of the plan
    const uint8_t* arity;
    const int32_t* fn_first;      // the items of function t: fn_items[fn_first[t] .. fn_first[t + 1])
    const int32_t* fn_items;
    const int32_t* fn_order;      // functions, those with the most items first
    const int32_t* u_at;          // where an item's u and du lie among the kept ones
    const void* feats;
    const void* out;
    const void* slots;
    const void* u;
    const void* mid;
    const float* gy;
    const float* dm;
    const float* du;
    float* dw[2];                 // of the second and the first 3x3 (JOIN: the first only)
    float* db[2];
    int32_t first_type;           // place in fn_order of blockIdx.y = 0
    int32_t C, H, W;
    int32_t sw, band;             // columns of a segment, rows of a band
    int32_t many;                 // MANY: items staged at a time (sw = W, band = H)
};

template <typename T, bool JOIN, bool MANY>
__global__ __launch_bounds__(256, 2) void k_wgrad(WgradArgs a)
{
    constexpr int TAPS = JOIN ? 1 : 9, HALO = JOIN ? 0 : 1, PIX = 32 * 4;       // bytes of a staged pixel
    extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
    const int C = a.C, H = a.H, W = a.W, sw = a.sw;
    const int cb = (C + 31) / 32, n_in = JOIN ? 2 * cb : cb;                     // input blocks; of the join: per argument
    const int which = JOIN ? 0 : int(blockIdx.x) / (cb * cb), block = int(blockIdx.x) - which * (cb * cb);
    const int co0 = block / n_in * 32, arg = JOIN && block % n_in >= cb ? 1 : 0;
    const int ci0 = (block % n_in - arg * cb) * 32;
    const int type = a.fn_order[a.first_type + blockIdx.y];
    const int ar = a.arity[type];
    const size_t chw = size_t(H) * W * C;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, r = lane & 31, hk = lane >> 5;

    // staged pixels of G: band rows x wp columns (even: a step never crosses a row), of the input: with halo
    const int wp = (sw + 1) & ~1, half = wp / 2, icols = wp + 2 * HALO;
    const int NI = MANY ? a.many : 1;
    const uint32_t in_off = uint32_t(NI * a.band * wp * PIX);
    const uint32_t m_wp = recip_of(wp), m_icols = recip_of(icols);

    f32x16 acc[TAPS];
#pragma unroll
    for (int k = 0; k < TAPS; ++k)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[k][i] = 0.f;
    float bias = 0.f;                                                            // sum of this lane's G values

    const int lo = JOIN && ar != 2 ? 0 : a.fn_first[type], hi = JOIN && ar != 2 ? 0 : a.fn_first[type + 1];
    struct Maps { const float* G; const T* Y; const T* IN; };                    // Y: the item's result, whose ReLU masks G (which 0)
    auto maps = [&](int idx) -> Maps {
        const int32_t item = a.fn_items[idx];
        const dynb_item it = a.items[item];
        const size_t off = size_t(item) * chw, u_off = ar == 2 ? size_t(a.u_at[item]) * chw : 0;
        const int32_t s = arg ? it.src1 : it.src0;
        const T* A = s >= 0 ? (const T*)a.slots + size_t(s) * chw : (const T*)a.feats + size_t(-1 - s) * chw;
        return {JOIN ? a.du + u_off : which == 0 ? a.gy + off : a.dm + off,
                it.dst >= 0 ? (const T*)a.slots + size_t(it.dst) * chw : (const T*)a.out + size_t(-1 - it.dst) * chw,
                JOIN ? A : which == 0 ? (const T*)a.mid + off : ar == 2 ? (const T*)a.u + u_off : A};
    };
#pragma unroll 1
    for (int idx = lo; idx < hi; idx += NI) {
        const int n = MANY ? min(NI, hi - idx) : 1;
        const Maps one = maps(idx);
#pragma unroll 1
        for (int x0 = 0; x0 < W; x0 += sw)
#pragma unroll 1
            for (int y0 = 0; y0 < H; y0 += a.band) {
                const int rows = min(a.band, H - y0), cols = min(sw, W - x0), irows = rows + 2 * HALO;
                __syncthreads();                                                 // the last band's fragments have been read
                constexpr int UN = 4;
                const int ng = n * rows * wp * 8, ni = n * irows * icols * 8;            // 16-byte pieces
                for (int base = tid; base < ng; base += 256 * UN) {
                    f32x4 v[UN];
#pragma unroll
                    for (int k = 0; k < UN; ++k) {
                        const int c = base + k * 256;
                        const uint32_t pix = uint32_t(c) >> 3, line = div_by(pix, m_wp), col = pix - line * wp;
                        const int it = MANY ? int(line) / rows : 0, row = int(line) - it * rows;
                        const int ch = co0 + (c & 7) * 4;
                        v[k] = f32x4{0.f, 0.f, 0.f, 0.f};
                        if (c < ng && int(col) < cols) {
                            const Maps m = MANY ? maps(idx + it) : one;
                            const size_t e = (size_t(y0 + row) * W + x0 + col) * C + ch;
                            v[k] = !JOIN && which == 0 ? masked_gy<false>(m.G + e, m.Y + e, C - ch) : load4<false>(m.G + e, C - ch);
                        }
                    }
#pragma unroll
                    for (int k = 0; k < UN; ++k)
                        if (base + k * 256 < ng) *reinterpret_cast<f32x4*>(lds_raw + size_t(base + k * 256) * 16) = v[k];
                }
                for (int base = tid; base < ni; base += 256 * UN) {
                    f32x4 v[UN];
#pragma unroll
                    for (int k = 0; k < UN; ++k) {
                        const int c = base + k * 256;
                        const uint32_t pix = uint32_t(c) >> 3, line = div_by(pix, m_icols), col = pix - line * icols;
                        const int it = MANY ? int(line) / irows : 0, row = int(line) - it * irows;
                        const int ch = ci0 + (c & 7) * 4, y = y0 + row - HALO, x = x0 + int(col) - HALO;
                        v[k] = f32x4{0.f, 0.f, 0.f, 0.f};
                        if (c < ni && unsigned(y) < unsigned(H) && unsigned(x) < unsigned(W)) {
                            const Maps m = MANY ? maps(idx + it) : one;
                            v[k] = load4<false>(m.IN + (size_t(y) * W + x) * C + ch, C - ch);
                        }
                    }
#pragma unroll
                    for (int k = 0; k < UN; ++k)
                        if (base + k * 256 < ni) *reinterpret_cast<f32x4*>(lds_raw + in_off + size_t(base + k * 256) * 16) = v[k];
                }
                __syncthreads();
                // this wave's steps: (row y, pixels 2 x and 2 x + 1), read one step ahead; the rows of the staged items follow each
                // other, iy is the row of the input that goes with y
                const int S = n * rows * half, s0 = S * wave / 4, s1 = S * (wave + 1) / 4;
                struct Step { float g, in[TAPS]; };
                auto read = [&](int y, int iy, int x, Step& v) {
                    const uint32_t ga = uint32_t(((y * half + x) * 2 + hk) * PIX + r * 4);
                    const uint32_t ia = in_off + uint32_t((iy * icols + x * 2 + hk) * PIX + r * 4);
                    v.g = *reinterpret_cast<const float*>(lds_raw + ga);
#pragma unroll
                    for (int k = 0; k < TAPS; ++k)
                        v.in[k] = *reinterpret_cast<const float*>(lds_raw + ia + uint32_t(((k / 3) * icols + k % 3) * PIX));
                };
                auto multiply = [&](const Step& v) {
                    bias += v.g;
#pragma unroll
                    for (int k = 0; k < TAPS; ++k) acc[k] = __builtin_amdgcn_mfma_f32_32x32x2f32(v.g, v.in[k], acc[k], 0, 0, 0);
                };
                if (s0 < s1) {
                    int y = s0 / half, x = s0 - y * half, left = 0, iy = y;
                    if constexpr (MANY) { const int it = y / rows; left = (it + 1) * rows - y; iy += it * 2 * HALO; }     // rows left of this item
                    auto advance = [&]() {
                        if (++x < half) return;
                        x = 0; ++y; ++iy;
                        if (MANY && --left == 0) { left = rows; iy += 2 * HALO; }
                    };
                    Step p, q;
                    read(y, iy, x, p);
#pragma unroll 1
                    for (int st = s0; st < s1; st += 2) {
                        advance();
                        if (st + 1 < s1) read(y, iy, x, q);
                        multiply(p);
                        if (st + 1 >= s1) break;
                        advance();
                        if (st + 2 < s1) read(y, iy, x, p);
                        multiply(q);
                    }
                }
            }
    }
    // The staged zeros (outside the map, in the padding column of an odd width) are factors here, and a zero times an infinity is
    // NaN: a sum that came out NaN is taken again without them (again: bit 4 tap + e for the thread's four rows).
    uint64_t again = 0;
    auto direct = [&](int tap, int co, int ci) -> float {
        float sum = 0.f;
#pragma unroll 1
        for (int idx = lo; idx < hi; ++idx) {
            const Maps m = maps(idx);
#pragma unroll 1
            for (int p = 0; p < H * W; ++p) {
                const int y = p / W + (JOIN ? 0 : tap / 3 - 1), x = p % W + (JOIN ? 0 : tap % 3 - 1);
                if (unsigned(y) >= unsigned(H) || unsigned(x) >= unsigned(W)) continue;
                const size_t e = size_t(p) * C + co;
                const float g = !JOIN && which == 0 && !(load_f32(m.Y + e) > 0.f) ? 0.f : m.G[e];
                sum += g * load_f32(m.IN + (size_t(y) * W + x) * C + ci);
            }
        }
        return sum;
    };
    // partial sums of the waves through LDS, three taps at a time: [wave][tap][b][lane] of four rows each
    f32x4* red = reinterpret_cast<f32x4*>(lds_raw);
    constexpr int R = JOIN ? 1 : 3;
#pragma unroll
    for (int k0 = 0; k0 < TAPS; k0 += R) {
        __syncthreads();
#pragma unroll
        for (int k = 0; k < R; ++k)
#pragma unroll
            for (int b = 0; b < 4; ++b)
                red[((wave * R + k) * 4 + b) * 64 + lane] = f32x4{acc[k0 + k][4 * b], acc[k0 + k][4 * b + 1], acc[k0 + k][4 * b + 2], acc[k0 + k][4 * b + 3]};
        __syncthreads();
#pragma unroll
        for (int k = 0; k < R; ++k) {                                            // this thread: rows 8 wave + 4 hk .. + 3, column r
            f32x4 v = red[(k * 4 + wave) * 64 + lane];
#pragma unroll
            for (int w = 1; w < 4; ++w) {
                const f32x4 q = red[((w * R + k) * 4 + wave) * 64 + lane];
                v.x += q.x; v.y += q.y; v.z += q.z; v.w += q.w;
            }
            const int co = co0 + 8 * wave + 4 * hk, ci = ci0 + r;
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (co + e < C && ci < C) {
                    if (v[e] != v[e]) again |= uint64_t(1) << ((k0 + k) * 4 + e);
                    const size_t row = size_t(type) * C + co + e;
                    a.dw[which][JOIN ? row * 2 * C + arg * C + ci : (row * 9 + k0 + k) * C + ci] = v[e];
                }
        }
    }
    if (ci0 == 0 && arg == 0) {                                                  // bias: the lane halves and the waves in order
        __syncthreads();
        float* sum = reinterpret_cast<float*>(lds_raw);
        sum[tid] = bias;
        __syncthreads();
        if (tid < 32 && co0 + tid < C) {
            float v = 0.f;
            for (int w = 0; w < 8; ++w) v += sum[w * 32 + tid];
            a.db[which][size_t(type) * C + co0 + tid] = v;
        }
    }
    end_unless(again != 0);
#pragma unroll 1
    for (; again; again &= again - 1) {
        const int b = __builtin_ctzll(again), co = co0 + 8 * wave + 4 * hk + (b & 3), ci = ci0 + r;
        const size_t row = size_t(type) * C + co;
        a.dw[which][JOIN ? row * 2 * C + arg * C + ci : (row * 9 + (b >> 2)) * C + ci] = direct(b >> 2, co, ci);
    }
}

__global__ void k_bwd_fill(float* p, size_t n, float v)
{
    for (size_t i = size_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n; i += size_t(gridDim.x) * blockDim.x) p[i] = v;
}

// V: floats per access, 4 where every map starts 16-byte aligned (chw a multiple of 4, dout and dfeats aligned).  Both kernels only
// move memory: 256 examples of 14 x 14 x 128 took 20 and 40 us with single floats.
template <int V> using floats = float __attribute__((ext_vector_type(V)));

// gy[root item of example e] = dout[e]
template <int V>
__global__ void k_bwd_seed(const float* __restrict__ dout, const int32_t* __restrict__ root_item, float* __restrict__ gy, size_t chw)
{
    const int e = blockIdx.y;
    const int32_t r = root_item[e];
    if (r < 0) return;
    for (size_t i = (size_t(blockIdx.x) * blockDim.x + threadIdx.x) * V; i < chw; i += size_t(gridDim.x) * blockDim.x * V)
        *reinterpret_cast<floats<V>*>(gy + size_t(r) * chw + i) = *reinterpret_cast<const floats<V>*>(dout + size_t(e) * chw + i);
}

// dfeats[e] = sum of the gradients of e's SCENE leaves in leaf order; a program that is one SCENE token passes dout through
template <int V>
__global__ void k_bwd_leaves(const float* __restrict__ gleaf, const int32_t* __restrict__ leaf_first,
                             const int32_t* __restrict__ root_item, const float* __restrict__ dout, float* __restrict__ dfeats, size_t chw)
{
    const int e = blockIdx.y;
    const int32_t lo = leaf_first[e], hi = root_item[e] < 0 ? lo : leaf_first[e + 1];
    for (size_t i = (size_t(blockIdx.x) * blockDim.x + threadIdx.x) * V; i < chw; i += size_t(gridDim.x) * blockDim.x * V) {
        floats<V> acc = 0.f;
        if (root_item[e] < 0) acc = *reinterpret_cast<const floats<V>*>(dout + size_t(e) * chw + i);
#pragma unroll 4
        for (int32_t l = lo; l < hi; ++l) {
            const floats<V> v = *reinterpret_cast<const floats<V>*>(gleaf + size_t(l) * chw + i);
#pragma unroll
            for (int c = 0; c < V; ++c) acc[c] += v[c];
        }
        *reinterpret_cast<floats<V>*>(dfeats + size_t(e) * chw + i) = acc;
    }
}

// (gy and gleaf lie in the workspace, 256-byte aligned)
bool wide_maps(size_t chw, const void* p) { return chw % 4 == 0 && (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

void launch_seed(const dynb_plan* p, const float* dout, const int32_t* root_item, float* gy, size_t chw, hipStream_t st)
{
    const bool wide = wide_maps(chw, dout);
    const unsigned bx = unsigned(std::min<size_t>((chw / (wide ? 4 : 1) + 255) / 256, 64));
    for (int e0 = 0; e0 < p->B; e0 += 32768)
        hipLaunchKernelGGL(wide ? k_bwd_seed<4> : k_bwd_seed<1>, dim3(bx, unsigned(std::min(32768, p->B - e0))), dim3(256), 0, st,
                           dout + size_t(e0) * chw, root_item + e0, gy, chw);
}

void launch_leaves(const dynb_plan* p, const float* gleaf, const int32_t* leaf_first, const int32_t* root_item, const float* dout,
                   float* dfeats, size_t chw, hipStream_t st)
{
    const bool wide = wide_maps(chw, dout) && wide_maps(chw, dfeats);
    const unsigned bx = unsigned(std::min<size_t>((chw / (wide ? 4 : 1) + 255) / 256, 64));
    for (int e0 = 0; e0 < p->B; e0 += 32768)
        hipLaunchKernelGGL(wide ? k_bwd_leaves<4> : k_bwd_leaves<1>, dim3(bx, unsigned(std::min(32768, p->B - e0))), dim3(256), 0, st, gleaf,
                           leaf_first + e0, root_item + e0, dout + size_t(e0) * chw, dfeats + size_t(e0) * chw, chw);
}

// ------------------------------------------------------------------------------------------
// MFMA path: bf16, C = 128, 14 x 14 (the shape of the fused forward kernel)
// ------------------------------------------------------------------------------------------
// The transposed convolutions are convolutions with the taps flipped and the channel roles exchanged, so a node's
// backward step has the shape of its forward step and runs on the same building blocks (LDS halo tile, packed
// weight fragments, software-pipelined K loop), a node or a part of one per workgroup, wave w owning channel tile w.  The forward
// pass of a DYNB_PLAN_KEEP plan has left u (two-argument functions) and mid of every item in its workspace.
//   tile <- g = gy * [y > 0]   (bf16)
//   conv(g; W_b flipped^T)     -> dmid = result * [mid > 0], written into the tile in place of g
//   conv(dmid; W_a flipped^T)  -> du = that + g (the residual path, in fp32 from the gradient map), written as fp32
//                                 to the argument's gradient map; two-argument functions: dc = du * [u > 0] into the
//                                 tile, then two 1x1 convolutions with the halves of W_1^T
// Everything that enters or leaves in the accumulator layout (masks, the residual term, results) goes through LDS so
// that all global accesses are coalesced 16-byte pieces.
// Gradients travel between nodes as fp32 maps and enter the MFMAs as bf16 (like every other operand of this
// path).  g, dmid and dc are saved as bf16 maps per item for the parameter gradients, which one kernel sums
// function by function afterwards.
struct BmArgs {
    const dynb_item* items;       // the launch group's items
    const int32_t* gdst0;         // routes of the group's items
    const int32_t* gdst1;
    int32_t first_item;
    int32_t count;
    const bf16_t* pk3bT;          // packed fragments: conv_b, taps flipped, channels exchanged
    const bf16_t* pk3aT;          //                   conv_a, taps flipped, channels exchanged
    const bf16_t* pk1T;           //                   conv1x1 halves, channels exchanged
    float* gy;                    // [n_items][P*C]
    const float* dout;            // the gradient of a root's result, read where it is (null: it has been copied to gy)
    float* gleaf;                 // [n_leaves][P*C]
    const bf16_t* sv_u;           // [n_items][P*C] each; u: in the forward pass's workspace
    const unsigned char* mask_y;  // [n_items][P*C/8], of the results and of mid: from the forward pass
    const unsigned char* mask_m;
    bf16_t* sv_g;
    bf16_t* sv_dm;
    bf16_t* sv_dc;
    int32_t per_xcd;              // workgroups of a die's run
};

__device__ __forceinline__ float* route_mf(const BmArgs& a, int32_t r)
{
    return r >= 0 ? a.gy + size_t(r) * (mf::P * mf::C) : a.gleaf + size_t(-1 - r) * (mf::P * mf::C);
}

// dst[function][tile][fragment][lane][i] = W(o, tap, k) with o = tile*32 + rho(lane % 32) (the row permutation of the
// forward pass's packed weights), k = (lane/32)*64 + j*8 + i, (tap, j) of the fragment as in iep_mfma.h, where
//   ntap 9: W = src[function][k][8 - tap][o]             conv3x3 transposed, taps flipped
//   ntap 2: W = src[function][k][tap*128 + o]            conv1x1 transposed, half `tap`
// blockIdx.y: w3a, w3b, w1
__global__ void k_bwd_pack(PackArgs a)
{
    const bf16_t* __restrict__ const src = a.src[blockIdx.y];
    u32x4* __restrict__ const dst = a.dst[blockIdx.y];
    const int ntap = blockIdx.y == 2 ? 2 : 9;
    const size_t total = size_t(a.n_types) * 4 * ntap * 8 * 64;
    for (size_t q = size_t(blockIdx.x) * blockDim.x + threadIdx.x; q < total; q += size_t(gridDim.x) * blockDim.x) {
        // a workgroup's four waves take the four channel tiles of a fragment: together they read whole rows
        const int lane = int(q & 63), tile = int(q >> 6) & 3, f = int((q >> 8) % (size_t(ntap) * 8));
        const size_t type = (q >> 8) / (size_t(ntap) * 8);
        const int tap = ntap == 9 ? mf::frag_kh(f) * 3 + mf::frag_kw(f) : f >> 3, j = ntap == 9 ? mf::frag_step(f) : f & 7;
        const int m = lane & 31;
        const int o = tile * 32 + ((m >> 2) & 1) * 16 + (m >> 3) * 4 + (m & 3), k0 = (lane >> 5) * 64 + j * 8;
        uint32_t v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int k = k0 + i;
            v[i] = src[ntap == 9 ? ((type * 128 + k) * 9 + (8 - tap)) * 128 + o : (type * 128 + k) * 256 + tap * 128 + o];
        }
        dst[((type * 4 + tile) * (size_t(ntap) * 8) + f) * 64 + lane] = u32x4{v[0] | (v[1] << 16), v[2] | (v[3] << 16), v[4] | (v[5] << 16), v[6] | (v[7] << 16)};
    }
}

// LDS of the backward node kernel: the halo tile, parts: the mask bytes of their rows of y, and an
// fp32 staging area through which accumulators (lane = pixel) leave as coalesced 16-byte pieces.  A global access in
// which every lane touches a line of its own costs about 125 clocks to issue, so nothing but the mask of mid (two bytes a lane, eight lanes a line) is
// loaded or stored in the accumulator layout: the residual term and the result go through the staging area.
namespace bn {
constexpr int MASK_OFF = (mf::TILE_BYTES + 255) / 256 * 256; // y mask bytes [P][16]
constexpr int MASK_BYTES = mf::P * 16 + 192;             // (+ padding to a multiple of 256)
constexpr int STAGE_OFF = MASK_OFF + MASK_BYTES;
constexpr int STAGE_PITCH = mf::C * 4 + 16;              // bytes per pixel: 128 floats + a bank-shifting pad
constexpr int STAGE_PIX = 112;                           // pixels per round: four pixel tiles (8 image rows)
constexpr int LDS_BYTES = STAGE_OFF + STAGE_PIX * STAGE_PITCH;
static_assert(MASK_BYTES % 256 == 0 && LDS_BYTES <= 160 * 1024, "LDS budget of one CU");
}  // namespace bn

// PARTS workgroups share a node (PartShape): narrow launch groups took 37 us with one.
// SPLIT: workgroups that share a part of a one-argument function's node, each with 4 / SPLIT channel tiles of du (parts_for); a two-argument one's
// join needs all channels of dc, and the first of them does it alone.
template <int PARTS, int SPLIT = 1>
__global__ __launch_bounds__(256, 1) void k_bwd_node_mfma(BmArgs a)
{
    using namespace mf;
    using Shape = PartShape<PARTS>;
    constexpr int MTA = Shape::MTA, MTB = Shape::MTB, UROWS = Shape::UROWS, RW = Shape::RW, NTHR = 256;
    constexpr int XA = PARTS == 1 ? 6 : Shape::XA, XB = PARTS == 1 ? 6 : Shape::XB;
    extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
    const int logical = (blockIdx.x & 7) * a.per_xcd + (blockIdx.x >> 3);
    const int node = logical / (PARTS * SPLIT), part = logical / SPLIT % PARTS, share = logical % SPLIT;
    if (node >= a.count) return;
    // image rows: results [orow0, orow1), windows of the two convs from row_a and row_b, g from urow0
    const int orow0 = part * Shape::ROWS, orow1 = min(orow0 + Shape::ROWS, S);
    const int row_a = min(max(orow0 - 1, 0), S - 2 * MTA), row_b = min(orow0, S - 2 * MTB), urow0 = min(max(row_a - 1, 0), S - UROWS);
    const int own_lo = orow0 * S * 16, own_hi = orow1 * S * 16;       // 16-byte pieces of this workgroup's rows of a map
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int r = lane & 31, h = lane >> 5, n0 = wave * 32;
#ifdef DYNB_NODE_CLOCKS
    long long tck[10], tck0 = clock64();
#define NCLK(i) tck[i] = clock64() - tck0
#else
#define NCLK(i) do {} while (0)
#endif
    const dynb_item it = a.items[node];
    const bool binary = it.src1 != DYNB_NO_ARG;                        // uniform over the workgroup
    if (SPLIT > 1 && binary && share > 0) return;
    const bool shared = SPLIT > 1 && !binary;
    const int tile_b = shared ? share * (4 / SPLIT) + wave % (4 / SPLIT) : wave;      // channel tile of the second conv
    const bool second = !shared || wave < 4 / SPLIT;                   // this wave has one
    auto mine = [&](int c) { return !shared || (c & 15) / (16 / SPLIT) == share; };   // piece c of a map: this workgroup's channels
    const size_t item_off = size_t(a.first_item + node) * (P * C);

    const size_t frag3 = (size_t(it.type) * 4 + wave) * 72, frag1 = (size_t(it.type) * 4 + wave) * 16;
    const bf16_t* wrow_bT = a.pk3bT + frag3 * FRAG + lane * 8;
    const bf16_t* wrow_aT = a.pk3aT + (size_t(it.type) * 4 + tile_b) * 72 * FRAG + lane * 8;
    bf16x8 ring[RW];

    auto centre_addr = [&](int c) -> uint32_t {                       // 16-byte piece c of a map -> its place in the halo tile
        const int p = c >> 4, part = c & 15;
        return uint32_t((p / S + 1) * ROW_BYTES + (p % S + 1) * PIX_BYTES + part * 16);
    };
    const float* gyp = a.dout && it.dst < 0 ? a.dout + size_t(-1 - it.dst) * (P * C) : a.gy + item_off;
    const unsigned char* const y_mask = a.mask_y + size_t(a.first_item + node) * (P * C / 8);
    const unsigned char* const m_mask = a.mask_m + size_t(a.first_item + node) * (P * C / 8);

    // ---- g = gy * [y > 0] as bf16 into the tile, saved for dW_b and db_b; all loads are issued before the first use.
    // A whole node's g stays in registers (half of them are free) until it is added to du: reading gy again was 100 of the 500 KB that a node
    // moved, in a phase that waits for them.
    constexpr int NIT = (UROWS * S * 16 + NTHR - 1) / NTHR;
    struct Grad { f32x4 g0, g1; };
    Grad whole[PARTS == 1 ? NIT : 1];
    {
        const int c_lo = urow0 * S * 16 + tid, c_hi = (urow0 + UROWS) * S * 16;
        const f32x4* gy4 = reinterpret_cast<const f32x4*>(gyp);
        u32x4* sg4 = reinterpret_cast<u32x4*>(a.sv_g + item_off);
        Grad in[NIT];
        uint32_t yb[NIT];
#pragma unroll
        for (int i = 0; i < NIT; ++i) {
            const int c = c_lo + i * NTHR;
            if (c < c_hi) { in[i].g0 = gy4[2 * c]; in[i].g1 = gy4[2 * c + 1]; yb[i] = y_mask[c]; }
        }
        __builtin_amdgcn_sched_barrier(0);
        ring_fill<RW>(ring, wrow_bT);                             // arrives while the tile is written
        zero_border<NTHR>(tid, row_a, row_a + 2 * MTA + 1);
#pragma unroll
        for (int i = 0; i < NIT; ++i) {
            const int c = c_lo + i * NTHR;
            if (c < c_hi) {
                Grad g;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    g.g0[e] = masked_by(yb[i], mask_bit(e), in[i].g0[e]);
                    g.g1[e] = masked_by(yb[i], mask_bit(e + 4), in[i].g1[e]);
                }
                const u32x4 pk = {pack_bf16x2(g.g0.x, g.g0.y), pack_bf16x2(g.g0.z, g.g0.w), pack_bf16x2(g.g1.x, g.g1.y), pack_bf16x2(g.g1.z, g.g1.w)};
                *reinterpret_cast<u32x4*>(lds_raw + centre_addr(c)) = pk;
                if (PARTS == 1 || (c >= own_lo && c < own_hi && mine(c))) sg4[c] = pk;
                if constexpr (PARTS == 1) whole[i] = g;
                else lds_raw[bn::MASK_OFF + c] = static_cast<unsigned char>(yb[i]);
            }
        }
    }

    // this lane's LDS address for the first row pair of the windows; in tile t it holds the pixel in column px of window row
    // 2 t + py
    const uint32_t x_a = pair_lane_addr(lane) + uint32_t(row_a * ROW_BYTES), x_b = pair_lane_addr(lane) + uint32_t(row_b * ROW_BYTES);
    const int px = r & 15, py = r >> 4;
    const bool real = px < S;                                         // columns 14, 15 are padding
    auto pixel = [&](int row, int t) { return (row + 2 * t + py) * S + px; };
    const int chan = n0 + 16 * h, chan_b = tile_b * 32 + 16 * h;      // this lane's 16 accumulator elements: channels chan .. chan+15; of the second conv
    f32x16 acc_a[MTA];
    constexpr bool SAME = MTA == MTB;                                 // one window: the second conv takes the first's registers
    f32x16 acc_own[SAME ? 1 : MTB];
    auto& acc = [&]() -> auto& { if constexpr (SAME) return acc_a; else return acc_own; }();
    auto zero = [](auto& accs) {
#pragma unroll
        for (auto& v : accs)
#pragma unroll
            for (int i = 0; i < 16; ++i) v[i] = 0.f;
    };
    auto centre = [&](uint32_t x, int t) -> uint32_t { return x - uint32_t(h * 128) + uint32_t(CENTER + 2 * t * ROW_BYTES); };
    // acc[8q .. 8q+7] where the mask bit is set, as 8 packed bf16
    auto packed_masked = [&](const f32x16& acc, int q, uint32_t bits) -> u32x4 {
        float v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = masked_by(bits, 8 * q + mask_bit(i), acc[8 * q + i]);
        return u32x4{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]), pack_bf16x2(v[4], v[5]), pack_bf16x2(v[6], v[7])};
    };
    // Accumulators of the second window -> the fp32 staging area, four pixel tiles per round; then every thread takes 16-byte pieces
    // (8 channels of a pixel) out of it: fn(c, lo, hi, pre(c), i) with c the piece's index in the whole map and i its number among the thread's
    // (of whole nodes the thread's i-th as it staged them).  pre(c) is evaluated for all of a thread's pieces before the round's barriers, so what it
    // loads is there afterwards.
    constexpr int NI = ((MTB < 4 ? MTB : 4) * 28 * 16 + NTHR - 1) / NTHR;     // pieces per thread of the larger round
    auto through_lds = [&](auto&& pre, auto&& fn) {
#pragma unroll
        for (int round = 0; round < (MTB + 3) / 4; ++round) {
            const int t0 = round * 4, t1 = min(t0 + 4, MTB), p0 = row_b * S + t0 * 28;
            const int lo = PARTS == 1 ? p0 * 16 : own_lo, hi = PARTS == 1 ? p0 * 16 + (t1 - t0) * 28 * 16 : own_hi;   // (parts: one round)
            decltype(pre(0)) ahead[NI];
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                const int c = lo + tid + i * NTHR;
                if (c < hi && mine(c)) ahead[i] = pre(c);
            }
            __syncthreads();                                          // the area (and, the first time, the tile) is free
#pragma unroll
            for (int t = 0; t < MTB; ++t)
                if (t >= t0 && t < t1 && real && second) {
#pragma unroll
                    for (int b = 0; b < 4; ++b)
                        *reinterpret_cast<f32x4*>(lds_raw + bn::STAGE_OFF + uint32_t((pixel(row_b, t) - p0) * bn::STAGE_PITCH + (chan_b + 4 * b) * 4)) =
                            f32x4{acc[t][4 * b], acc[t][4 * b + 1], acc[t][4 * b + 2], acc[t][4 * b + 3]};
                }
            __syncthreads();
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                const int c = lo + tid + i * NTHR;
                if (c < hi && mine(c)) {
                    const uint32_t at = bn::STAGE_OFF + uint32_t(((c >> 4) - p0) * bn::STAGE_PITCH + (c & 15) * 32);
                    fn(c, *reinterpret_cast<const f32x4*>(lds_raw + at), *reinterpret_cast<const f32x4*>(lds_raw + at + 16), ahead[i], round * NI + i);
                }
            }
        }
    };
    static_assert(PARTS > 1 || 4 * 28 * 16 % NTHR == 0, "a whole node's rounds begin where a thread's pieces do");
    struct Nothing {};
    auto store_piece = [](float* dst, int c, const f32x4& lo, const f32x4& hi) {
        *reinterpret_cast<f32x4*>(dst + size_t(c) * 8) = lo;
        *reinterpret_cast<f32x4*>(dst + size_t(c) * 8 + 4) = hi;
    };
    NCLK(0);
    __syncthreads();

    // ---- dmid = conv(g; W_b flipped, transposed) * [mid > 0], written into the tile in place of g
    // (this lane's 16 bits of mid's mask, the bytes of the two pieces that hold its channels, are requested now)
    uint32_t mm[MTA];
#pragma unroll
    for (int t = 0; t < MTA; ++t) mm[t] = real ? *reinterpret_cast<const uint16_t*>(m_mask + pixel(row_a, t) * 16 + (chan >> 3)) : 0u;
    zero(acc_a);
    NCLK(1);
    kloop3<MTA, RW, XA>(acc_a, x_a, ring, wrow_bT, wrow_aT);
    NCLK(2);
    __syncthreads();
#pragma unroll
    for (int t = 0; t < MTA; ++t)
        if (real) {
#pragma unroll
            for (int q = 0; q < 2; ++q)
                *reinterpret_cast<u32x4*>(lds_raw + centre(x_a, t) + uint32_t((chan + q * 8) * 2)) = packed_masked(acc_a[t], q, mm[t]);
        }
    __syncthreads();
    {                                                                 // dmid saved for dW_a and db_a, out of the tile
        u32x4* sdm4 = reinterpret_cast<u32x4*>(a.sv_dm + item_off);
#pragma unroll
        for (int i = 0; i < (Shape::ROWS * S * 16 + NTHR - 1) / NTHR; ++i) {
            const int c = own_lo + tid + i * NTHR;
            if (c < own_hi && mine(c)) sdm4[c] = *reinterpret_cast<const u32x4*>(lds_raw + centre_addr(c));
        }
    }

    // ---- du = g + conv(dmid; W_a flipped, transposed).  The residual term g is added in fp32, from the gradient map
    // itself, not from its bf16 copy in the tile: down a chain of modules the convolution's share is small against
    // the residual's and would vanish below the bfloat16 quantum of the latter at every level.
    // (a part's pieces of it are requested here: behind the loop they were a trip to memory that nothing hid)
    Grad residue[PARTS > 1 ? NI : 1];
    if constexpr (PARTS > 1) {
        const f32x4* gy4 = reinterpret_cast<const f32x4*>(gyp);
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int c = own_lo + tid + i * NTHR;
            if (c < own_hi && mine(c)) residue[i] = Grad{gy4[2 * c], gy4[2 * c + 1]};
        }
    }
    auto grad = [&](int i) -> const Grad& { if constexpr (PARTS > 1) return residue[i]; else return whole[i]; };
    zero(acc);
    NCLK(3);
    if (second) kloop3<MTB, RW, XB, false>(acc, x_b, ring, wrow_aT, wrow_aT);
    NCLK(4);
    auto residual = [&](int c, f32x4& lo, f32x4& hi, const Grad& g) {
        const uint32_t yb = PARTS > 1 ? lds_raw[bn::MASK_OFF + c] : 0u;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            lo[e] += PARTS > 1 ? masked_by(yb, mask_bit(e), g.g0[e]) : g.g0[e];
            hi[e] += PARTS > 1 ? masked_by(yb, mask_bit(e + 4), g.g1[e]) : g.g1[e];
        }
    };
    if (!binary) {
        float* dst = route_mf(a, a.gdst0[node]);
        through_lds([](int) { return Nothing{}; },
                    [&](int c, f32x4 lo, f32x4 hi, const Nothing&, int i) {
                        residual(c, lo, hi, grad(i));
                        store_piece(dst, c, lo, hi);
                    });
        NCLK(5);
#ifdef DYNB_NODE_CLOCKS
        if (logical == 0 && (threadIdx.x & 63) == 0)
            printf("node count %d wave %d: staged %lld | conv1 %lld..%lld | conv2 %lld..%lld | stored %lld\n", a.count, int(threadIdx.x >> 6), tck[0],
                   tck[1], tck[2], tck[3], tck[4], tck[5]);
#endif
        return;
    }
    // ---- two-argument functions: dc = du * [u > 0] into the tile, then da0 = dc W_1[:, :C], da1 = dc W_1[:, C:]
    {
        const u32x4* u4 = reinterpret_cast<const u32x4*>(a.sv_u + item_off);
        u32x4* sdc4 = reinterpret_cast<u32x4*>(a.sv_dc + item_off);
        through_lds([&](int c) { return u4[c]; },
                    [&](int c, f32x4 lo, f32x4 hi, const u32x4& u, int i) {
                        residual(c, lo, hi, grad(i));
                        const uint32_t ub = positive_mask(u);
#pragma unroll
                        for (int e = 0; e < 4; ++e) { lo[e] = masked_by(ub, mask_bit(e), lo[e]); hi[e] = masked_by(ub, mask_bit(e + 4), hi[e]); }
                        const u32x4 pk = {pack_bf16x2(lo.x, lo.y), pack_bf16x2(lo.z, lo.w), pack_bf16x2(hi.x, hi.y), pack_bf16x2(hi.z, hi.w)};
                        *reinterpret_cast<u32x4*>(lds_raw + centre_addr(c)) = pk;
                        sdc4[c] = pk;
                    });
    }
    __syncthreads();
    {
        const bf16_t* t1row = a.pk1T + frag1 * FRAG + lane * 8;
        bf16x8 w1f[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) w1f[j] = *reinterpret_cast<const bf16x8*>(t1row + j * FRAG);
        auto caddr = [&](int t) { return centre(x_b, t) + uint32_t(h * 128); };
        zero(acc);
        kloop1<MTB, true>(acc, caddr, w1f, t1row + 8 * FRAG);
        float* d0 = route_mf(a, a.gdst0[node]);
        through_lds([](int) { return Nothing{}; }, [&](int c, f32x4 lo, f32x4 hi, const Nothing&, int) { store_piece(d0, c, lo, hi); });
        zero(acc);
        kloop1<MTB, false>(acc, caddr, w1f, nullptr);
        float* d1 = route_mf(a, a.gdst1[node]);
        through_lds([](int) { return Nothing{}; }, [&](int c, f32x4 lo, f32x4 hi, const Nothing&, int) { store_piece(d1, c, lo, hi); });
    }
}

// Parameter gradients.  A unit is the partial sum over one chunk of a function's items for one (mode, part):
//   mode 0: conv_b, part = kernel row kh:  dW_b[co][kh][kw][ci] = sum_items sum_p g[p][co]    mid[p + (kh-1, kw-1)][ci]
//   mode 1: conv_a, part = kernel row kh:  dW_a[co][kh][kw][ci] = sum_items sum_p dmid[p][co] u[p + (kh-1, kw-1)][ci]
//   mode 2: conv1x1, part = argument:      dW_1[co][part*C + ci] = sum_items sum_p dc[p][co]  arg_part[p][ci]
// and with part 0 the bias gradient, the sum of g / dmid / dc over items and pixels.  k_bwd_wgrad_sum adds the units of a (function,
// part) in chunk order.  Nothing is atomic.
//
// A workgroup sums one chunk for a quadrant of the channels, 64 output x 64 input ones, and all nine taps (of the 1x1: one argument); a
// wave 32 x 32 of them:  D[co][ci] += G[co][16 pixels] IN[16 pixels][ci]  (v_mfma_f32_32x32x16_bf16), a K step being an image row
// (14 pixels and 2 zeros).  The contraction runs over pixels, the dimension in which neither map is contiguous: both
// half maps of an item are copied into LDS as they are, pixel by pixel, and read with the transposing LDS load, whose lanes get four
// pixels of one channel each.  An input row is read for the three tap columns and multiplied with the three gradient rows that its
// tap rows want, so a step of 9 MFMAs (288 clocks) reads 8 KB, where one kernel row at a time for all 128 x 128 channels reads 18 KB four
// bytes a lane and packs the operands with 72 permutes for 12.  57 KB of LDS and 256 registers: two workgroups share a CU, and one's
// copying runs under the other's MFMAs.  256 programs (4276 modules): 747 -> 397 us, MFMA
// busy 0.38 -> 0.66 of the time, no bank conflicts; the rest is the end of the last round of workgroups and waits for maps.
// A staged pixel is 128 bytes without padding; its halves (32 channels, what a wave reads) are exchanged in every other pair
// of pixels, so that the four pixels x 64 bytes that 32 lanes read lie on all 64 banks.
struct WgArgs {
    const dynb_item* items;       // all items of the plan
    const dynb_wg_unit* units;
    const int32_t* order;         // the units, longest chunks first (planner.cpp)
    const int32_t* fn_first;
    const int32_t* fn_items;
    int32_t n_chunks;             // chunks of the 3x3s: three units each
    int32_t n_joins;              // units of the 1x1, behind the others in the order
    const bf16_t* feats;
    const bf16_t* slots;
    const bf16_t* sv_u;
    const bf16_t* sv_m;
    const bf16_t* sv_g;
    const bf16_t* sv_dm;
    const bf16_t* sv_dc;
    float* partial;               // [unit][3][C][C] weight gradient ([tap][co][ci]; conv1x1: tap 0 only), then [C] bias gradient
    float* dw3a; float* db3a; float* dw3b; float* db3b; float* dw1; float* db1;
};
constexpr size_t WG_PARTIAL = size_t(3) * 128 * 128 + 128;           // floats per unit
constexpr int WG_ROW = 16 * 128, WG_MAP = mf::S * WG_ROW;            // LDS: bytes of an image row (columns 14, 15 are zeros), of a half map

// four pixels (at this lane's pixel address and its three neighbours') of one channel per lane
__device__ __forceinline__ i16x4 lds_read_pixels(uint32_t addr)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
    using lds_i16x4 = __attribute__((address_space(3))) i16x4;
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16(reinterpret_cast<lds_i16x4*>((__attribute__((address_space(3))) unsigned char*)lds_raw + addr));
}

// chunks: the function's; a single one is the whole sum and goes where the gradients go.  CONV: un is the first of the chunk's three units (kernel
// row 0), the others follow `chunks` units apart
template <bool CONV>
__device__ __forceinline__ void wgrad_chunk(const WgArgs& a, const dynb_wg_unit un, const int32_t unit, const int32_t chunks, const int quad)
{
    using namespace mf;
    constexpr int K = CONV ? 3 : 1, NTHR = 256;
    extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int wi = wave & 1, wj = wave >> 1, ci_half = quad & 1, co_half = quad >> 1;

    // the chunk's items, one per lane (at most 16): where the input map and the gradient map start, this quadrant's halves of them
    uint64_t in_at, g_at;
    {
        const int32_t item = a.fn_items[min(un.begin + (lane & (DYNB_WG_CHUNK - 1)), un.end - 1)];
        const dynb_item it = a.items[item];
        const size_t off = size_t(item) * (P * C);
        const int32_t s = !CONV && un.part == 1 ? it.src1 : it.src0;
        const bf16_t* IN = un.mode == 0                              ? a.sv_m + off
                           : un.mode == 1 && it.src1 != DYNB_NO_ARG ? a.sv_u + off
                           : s >= 0                                  ? a.slots + size_t(s) * (P * C)
                                                                     : a.feats + size_t(-1 - s) * (P * C);
        const bf16_t* G = (un.mode == 0 ? a.sv_g : un.mode == 1 ? a.sv_dm : a.sv_dc) + off;
        in_at = reinterpret_cast<uint64_t>(IN + ci_half * 64);
        g_at = reinterpret_cast<uint64_t>(G + co_half * 64);
    }
    // (said to be global: a flat load would count among the LDS accesses, and every wait for a fragment would be for the maps too)
    using global_bytes = const __attribute__((address_space(1))) unsigned char*;
    using global_piece = const __attribute__((address_space(1))) u32x4*;
    auto of_lane = [](uint64_t v, int l) -> global_bytes {
        const uint32_t lo = uint32_t(__builtin_amdgcn_readlane(int(uint32_t(v)), l)), hi = uint32_t(__builtin_amdgcn_readlane(int(uint32_t(v >> 32)), l));
        return reinterpret_cast<global_bytes>(uint64_t(hi) << 32 | lo);
    };
    // zeros in columns 14 and 15 of both maps' rows
    for (int c = tid; c < 2 * S * 16; c += NTHR) *reinterpret_cast<u32x4*>(lds_raw + uint32_t((c >> 4) * WG_ROW + S * 128 + (c & 15) * 16)) = u32x4{0u, 0u, 0u, 0u};

    // copying: 16-byte pieces, eight per pixel.  Their addresses are made anew for every item (here(), whose value the compiler cannot carry
    // through the loop): kept, they would take the registers that the next item's maps wait in.
    constexpr int NP = (P * 8 + NTHR - 1) / NTHR;
    u32x4 tin[NP], tg[NP];
    auto here = [&]() -> uint32_t {
        uint32_t t = uint32_t(tid);
        asm volatile("" : "+v"(t));
        return t;
    };
    auto load = [&](int n) {
        const global_bytes in = of_lane(in_at, n), g = of_lane(g_at, n);
        const uint32_t t = here();
#pragma unroll
        for (int i = 0; i < NP; ++i) {                                // (the last pixel again where there are no more)
            const uint32_t p = (t >> 3) + uint32_t(i * (NTHR / 8)), at = (i + 1 < NP ? p : min(p, uint32_t(P - 1))) * (C * 2) + (t & 7) * 16;
            tin[i] = *reinterpret_cast<global_piece>(in + at);
            tg[i] = *reinterpret_cast<global_piece>(g + at);
        }
    };
    auto store = [&]() {
        const uint32_t t = here();
#pragma unroll
        for (int i = 0; i < NP; ++i)
            if (i + 1 < NP || t + uint32_t(i * NTHR) < uint32_t(P * 8)) {
                const uint32_t p = (t >> 3) + uint32_t(i * (NTHR / 8)), y = p / S, x = p - y * S;
                const uint32_t at = y * WG_ROW + x * 128 + (((t >> 2) ^ (x >> 1)) & 1u) * 64 + (t & 3) * 16;
                *reinterpret_cast<u32x4*>(lds_raw + at) = tin[i];
                *reinterpret_cast<u32x4*>(lds_raw + WG_MAP + at) = tg[i];
            }
    };
    // This lane's address for pixels x .. x + 3 (x = its K half's first pixel, plus 4 for the second four, plus the tap column's -1, 0, 1):
    // the group of 16 lanes reads 16 channels, four lanes a pixel.  Columns beyond the row are zeros: column 15.
    auto lane_at = [&](int half, int shift) -> uint32_t {
        int x = (lane >> 5) * 8 + ((lane >> 2) & 3) + shift;
        if (x < 0 || x > 15) x = 15;
        return uint32_t(x * 128 + ((half ^ (x >> 1)) & 1) * 64 + ((lane >> 4) & 1) * 32 + (lane & 3) * 8);
    };
    uint32_t in_lane[K][2];
#pragma unroll
    for (int kw = 0; kw < K; ++kw)
#pragma unroll
        for (int q = 0; q < 2; ++q) in_lane[kw][q] = lane_at(wi, 4 * q + kw - K / 2);
    const uint32_t g_lane = lane_at(wj, 0) + uint32_t(WG_MAP);
    auto frag = [](i16x4 lo, i16x4 hi) -> bf16x8 { return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7)); };
    auto read_in = [&](int y, int kw) { return frag(lds_read_pixels(in_lane[kw][0] + uint32_t(y * WG_ROW)), lds_read_pixels(in_lane[kw][1] + uint32_t(y * WG_ROW))); };
    auto read_g = [&](int y) { return frag(lds_read_pixels(g_lane + uint32_t(y * WG_ROW)), lds_read_pixels(g_lane + uint32_t(y * WG_ROW + 4 * 128))); };

    f32x16 acc[K][K];
    float bias = 0.f;                                                 // sum of this lane's channel of G
#pragma unroll
    for (int kh = 0; kh < K; ++kh)
#pragma unroll
        for (int kw = 0; kw < K; ++kw)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[kh][kw][i] = 0.f;
    const bool with_bias = (!CONV && un.part == 1) ? false : wi == 0 && ci_half == 0;      // uniform over the wave
    // (every wave sums G: the fifteen additions of a row cost nothing beside its MFMAs, a second copy of the loop costs registers)
    auto add_bias = [&](const bf16x8& v) {
        const u32x4 w = __builtin_bit_cast(u32x4, v);
        float s[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) s[i] = __uint_as_float(w[i] << 16) + __uint_as_float(w[i] & 0xffff0000u);
        bias += (s[0] + s[1]) + (s[2] + s[3]);
    };
    // steps (input row y, tap column kw): the fragments of step s + 2 and of gradient row y + 2 are requested ahead of its MFMAs
    constexpr int STEPS = S * K, AHEAD = 2;
    auto multiply = [&]() {
        bf16x8 in[AHEAD + 1], g[4];
        g[0] = read_g(0);
#pragma unroll
        for (int s = 0; s < AHEAD; ++s) in[s] = read_in(s / K, s % K);
        g[1] = read_g(1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int s = 0; s < STEPS; ++s) {
            const int y = s / K, kw = s % K;
            if (s + AHEAD < STEPS) in[(s + AHEAD) % (AHEAD + 1)] = read_in((s + AHEAD) / K, (s + AHEAD) % K);
            if (kw == 0 && y + 2 < S) g[(y + 2) & 3] = read_g(y + 2);
            if (kw == 0) add_bias(g[y & 3]);
            auto mul = [&](int kh, int row) {
                acc[kh][kw] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(g[row & 3], in[s % (AHEAD + 1)], acc[kh][kw], 0, 0, 0);
            };
            if constexpr (K == 1) mul(0, y);
            else {
                mul(1, y);
                if (y > 0) mul(2, y - 1);                             // tap row kh of output row y + 1 - kh
                if (y + 1 < S) mul(0, y + 1);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    const int n_items = un.end - un.begin;
    load(0);
#pragma unroll 1
    for (int n = 0; n < n_items; ++n) {
        __syncthreads();                                              // the previous item's fragments have been read
        store();
        __syncthreads();
        load(min(n + 1, n_items - 1));                                // arrives under this item's MFMAs
        multiply();
    }
    // D[co][ci]: lane ci = lane % 32, element i: co = 8 (i / 4) + 4 (lane / 32) + i % 4; a store writes two rows of 128 bytes
    const int m = lane & 31, hk = lane >> 5, co = co_half * 64 + wj * 32 + 4 * hk, ci = ci_half * 64 + wi * 32 + m;
    const bool whole = chunks == 1;
    float* const out = a.partial + size_t(unit) * WG_PARTIAL;
    // elements between kernel rows, taps of a row, output channels
    const size_t to_row = CONV ? (whole ? size_t(3 * C) : size_t(chunks) * WG_PARTIAL) : 0;
    const uint32_t to_tap = whole ? C : C * C, to_co = !whole ? C : CONV ? 9 * C : 2 * C;
    float* const dw = !whole ? out : !CONV ? a.dw1 + (size_t(un.type) * C * 2 + un.part) * C : (un.mode == 0 ? a.dw3b : a.dw3a) + size_t(un.type) * C * 9 * C;
    float* const to = dw + size_t(co) * to_co + ci;
#pragma unroll
    for (int kh = 0; kh < K; ++kh)
#pragma unroll
        for (int kw = 0; kw < K; ++kw)
#pragma unroll
            for (int i = 0; i < 16; ++i) (to + kh * to_row)[kw * to_tap + uint32_t(8 * (i / 4) + i % 4) * to_co] = acc[kh][kw][i];
    if (with_bias) {
        bias += __shfl_xor(bias, 32);
        float* const db = !whole ? out + size_t(3) * C * C : (!CONV ? a.db1 : un.mode == 0 ? a.db3b : a.db3a) + size_t(un.type) * C;
        if (hk == 0) db[co_half * 64 + wj * 32 + m] = bias;
    }
}

// Workgroups come in sets of 32: eight chunks, whose four quadrants are taken by workgroups 8 apart, which run on one die and share the
// maps in its L2.
__global__ __launch_bounds__(256, 2) void k_bwd_wgrad_mfma(WgArgs a)
{
    const int set = int(blockIdx.x >> 5), x = blockIdx.x & 7, quad = (blockIdx.x >> 3) & 3, conv_sets = (a.n_chunks + 7) / 8;
    auto chunks_of = [&](int type) { return (a.fn_first[type + 1] - a.fn_first[type] + DYNB_WG_CHUNK - 1) / DYNB_WG_CHUNK; };
    if (set < conv_sets) {
        if (set * 8 + x >= a.n_chunks) return;
        const int32_t u = a.order[set * 24 + x];                      // (the parts of eight chunks follow each other in the order)
        const dynb_wg_unit un = a.units[u];
        wgrad_chunk<true>(a, un, u, chunks_of(un.type), quad);
    } else {
        const int j = (set - conv_sets) * 8 + x;
        if (j >= a.n_joins) return;
        const int32_t u = a.order[3 * a.n_chunks + j];
        const dynb_wg_unit un = a.units[u];
        wgrad_chunk<false>(a, un, u, chunks_of(un.type), quad);
    }
}

// dW / db of one (mode, function, part) = its units' partial results added in chunk order.  Bound by memory: 340 MB at 256 programs.  They are read once, past the
// caches (78 us with ordinary loads, 61 so; eight of them ahead 62, ordinary ones ahead 76; partial results written past the caches as well 68)
struct WsArgs {
    const dynb_wg_group* groups;
    const float* partial;
    float* dw3a; float* db3a; float* dw3b; float* db3b; float* dw1; float* db1;
};

__global__ void k_bwd_wgrad_sum(WsArgs a)
{
    constexpr int C = 128;
    const dynb_wg_group g = a.groups[blockIdx.y];
    if (g.n_units == 1) return;                                       // written by k_bwd_wgrad_mfma
    const int ntap = g.mode == 2 ? 1 : 3;
    const int e = blockIdx.x * blockDim.x + threadIdx.x;              // float4 index inside [tap][co][ci]
    if (e < ntap * C * C / 4) {
        f32x4 s = {0.f, 0.f, 0.f, 0.f};
        for (int c = 0; c < g.n_units; ++c) {
            const f32x4 v = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(a.partial + size_t(g.first_unit + c) * WG_PARTIAL) + e);
            s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
        }
        const int ci = (e * 4) % C, co = (e * 4 / C) % C, k = e * 4 / (C * C);
        float* dst = g.mode == 2 ? a.dw1 + (size_t(g.type) * C + co) * (2 * C) + g.part * C + ci
                                 : (g.mode == 0 ? a.dw3b : a.dw3a) + ((size_t(g.type) * C + co) * 9 + g.part * 3 + k) * C + ci;
        *reinterpret_cast<f32x4*>(dst) = s;
    }
    if (g.part == 0 && blockIdx.x == 0 && threadIdx.x < C) {
        float s = 0.f;
        for (int c = 0; c < g.n_units; ++c) s += a.partial[size_t(g.first_unit + c) * WG_PARTIAL + size_t(3) * C * C + threadIdx.x];
        (g.mode == 2 ? a.db1 : g.mode == 0 ? a.db3b : a.db3a)[size_t(g.type) * C + threadIdx.x] = s;
    }
}

size_t align256(size_t v) { return (v + 255) & ~size_t(255); }

// workspace away from the fused kernels' shape: fp32 maps, gy and dm of every item, du of two-argument functions
struct BwdLayout {
    size_t gy, gleaf, dm, du, total;
};

BwdLayout bwd_layout(const dynb_plan* p, const dynb_shape* s)
{
    BwdLayout L;
    const size_t chw = size_t(s->C) * s->H * s->W, n_items = p->items.size();
    const size_t n_leaf = p->leaf_first.empty() ? 0 : size_t(p->leaf_first.back());
    size_t o = 0;
    auto take = [&](size_t bytes) { size_t at = o; o += align256(std::max<size_t>(bytes, 4)); return at; };
    L.gy = take(n_items * chw * 4);
    L.gleaf = take(n_leaf * chw * 4);
    L.dm = take(n_items * chw * 4);
    L.du = take(p->n_u * chw * 4);
    L.total = o;
    return L;
}

constexpr int WGRAD_LDS_MAX = 80 * 1024;                                  // two workgroups per CU
template <typename T, bool JOIN, bool MANY>
int launch_wgrad_items(WgradArgs a, int n_types, size_t lds, hipStream_t st)
{
    static std::atomic<uint64_t> attr_set{0};                             // one bit per device
    int dev = 0;
    HIP_TRY(hipGetDevice(&dev), "hipGetDevice");
    if (!(attr_set.load() >> (dev & 63) & 1)) {
        HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(k_wgrad<T, JOIN, MANY>), hipFuncAttributeMaxDynamicSharedMemorySize, WGRAD_LDS_MAX),
                "hipFuncSetAttribute(k_wgrad)");
        attr_set.fetch_or(uint64_t(1) << (dev & 63));
    }
    const int cb = (a.C + 31) / 32;
    for (int t0 = 0; t0 < n_types; t0 += 32768) {
        a.first_type = t0;
        hipLaunchKernelGGL((k_wgrad<T, JOIN, MANY>), dim3(unsigned(cb * cb * 2), unsigned(std::min(32768, n_types - t0))),
                           dim3(256), lds, st, a);
    }
    return DYNB_OK;
}

// parameter gradients of all functions, zeros for functions without items
template <typename T, bool JOIN>
int launch_wgrad(WgradArgs a, int n_types, hipStream_t st)
{
    constexpr int HALO = JOIN ? 0 : 1;
    const int n_seg = (a.W + 31) / 32;
    a.sw = (a.W + n_seg - 1) / n_seg;
    const int wp = (a.sw + 1) & ~1, icols = wp + 2 * HALO;
    a.band = std::min(a.H, (WGRAD_LDS_MAX / 128 - 2 * HALO * icols) / (wp + icols));      // >= 8: sw <= 32
    // Maps of up to 16 pixels: several items at a time, some 64 pixels, where one item would be a trip to memory (3 us) for a few
    // MFMAs.  10000 programs of 2 modules, fp32, 1 x 1, a training step: C = 1 31 -> 4.0 ms, C = 16 30 -> 4.2.
    const long long pixels = (long long)a.H * wp;
    a.many = pixels <= 16 ? int(64 / pixels) : 1;
    const size_t lds = std::max<size_t>(size_t(a.many) * (a.band * wp + (a.band + 2 * HALO) * icols) * 128, size_t(JOIN ? 1 : 3) * 16 * 1024);
    return a.many > 1 ? launch_wgrad_items<T, JOIN, true>(a, n_types, lds, st) : launch_wgrad_items<T, JOIN, false>(a, n_types, lds, st);
}

template <typename T>
int run_backward(const dynb_plan* p, const dynb_shape* s, const dynb_module_weights* w, const void* feats, const void* out,
                 const void* fwd_ws, const float* dout, const dynb_module_grads* g, char* ws, hipStream_t st)
{
    const BwdLayout L = bwd_layout(p, s);
    const size_t chw = size_t(s->C) * s->H * s->W;
    // the routing tables were uploaded with the plan
    const dynb_keep_tables KT = dynb_plan_keep_tables(p);
    const char* pd = static_cast<const char*>(p->dev_buf);
    const int32_t* d_leaf_first = reinterpret_cast<const int32_t*>(pd + KT.leaf_first);
    const int32_t* d_root_item = reinterpret_cast<const int32_t*>(pd + KT.root_item);

    float* gy = reinterpret_cast<float*>(ws + L.gy);
    launch_seed(p, dout, d_root_item, gy, chw, st);

    const dynb_item* d_items = reinterpret_cast<const dynb_item*>(pd);
    ConvArgs a = {};
    a.feats = feats; a.out = const_cast<void*>(out); a.slots = const_cast<void*>(fwd_ws);
    const size_t map = chw * sizeof(T);
    a.mid = static_cast<char*>(const_cast<void*>(fwd_ws)) + dynb_generic_mid_offset(p, map);
    T* const u = reinterpret_cast<T*>(static_cast<char*>(a.mid) + dynb_generic_mids(p) * map);
    a.gy = gy; a.gleaf = reinterpret_cast<float*>(ws + L.gleaf);
    a.dm = reinterpret_cast<float*>(ws + L.dm);
    float* const du = reinterpret_cast<float*>(ws + L.du);
    a.C = s->C; a.H = s->H; a.W = s->W;
    for (size_t li = p->launches.size(); li-- > 0;) {
        const dynb_launch& l = p->launches[li];
        a.u = dynb_u_of_group(u, l, chw);
        a.du = dynb_u_of_group(du, l, chw);
        // a launch group wider than one grid (65535 rows) is walked in slices; its nodes are independent
        for (int off = 0; off < l.count; off += 32768) {
            const int cnt = std::min(32768, l.count - off);
            a.first_item = a.first_kept = l.start + off;
            const dynb_item* items = d_items + a.first_item;
            a.gdst0 = reinterpret_cast<const int32_t*>(pd + KT.gdst0) + a.first_item;
            a.gdst1 = reinterpret_cast<const int32_t*>(pd + KT.gdst1) + a.first_item;
            a.w = w->w3b;
            int rc = launch_conv<T, CV_DSECOND>(items, a, cnt, st);
            a.w = w->w3a;
            if (rc == DYNB_OK) rc = launch_conv<T, CV_DFIRST>(items, a, cnt, st);
            const int lo = std::max(l.bin_lo, l.start + off), hi = std::min(l.bin_hi, l.start + off + cnt);
            if (rc == DYNB_OK && lo < hi) {
                ConvArgs j = a;
                const int skip = lo - (l.start + off);
                j.w = w->w1;
                j.first_item += skip; j.first_kept += skip;
                j.gdst0 += skip; j.gdst1 += skip;
                rc = launch_conv<T, CV_DJOIN>(items + skip, j, hi - lo, st);
            }
            if (rc != DYNB_OK) return fail(rc, "dynbatch_backward: a convolution could not be launched");
        }
    }
    WgradArgs q = {};
    q.items = d_items; q.arity = reinterpret_cast<const uint8_t*>(pd + dynb_plan_arity_offset(p));
    q.fn_first = reinterpret_cast<const int32_t*>(pd + KT.fn_first);
    q.fn_items = reinterpret_cast<const int32_t*>(pd + KT.fn_items);
    q.fn_order = reinterpret_cast<const int32_t*>(pd + KT.fn_order);
    q.u_at = reinterpret_cast<const int32_t*>(pd + KT.u_at);
    q.feats = feats; q.out = out; q.slots = fwd_ws; q.u = u; q.mid = a.mid;
    q.gy = gy; q.dm = a.dm; q.du = du;
    q.C = s->C; q.H = s->H; q.W = s->W;
    q.dw[0] = g->dw3b; q.db[0] = g->db3b; q.dw[1] = g->dw3a; q.db[1] = g->db3a;
    int rc = launch_wgrad<T, false>(q, p->n_types, st);
    if (rc != DYNB_OK) return rc;
    if (p->has_binary) {
        q.dw[0] = g->dw1; q.db[0] = g->db1;
        rc = launch_wgrad<T, true>(q, p->n_types, st);
        if (rc != DYNB_OK) return rc;
    } else {
        auto fill = [&](float* ptr, size_t n) {
            if (ptr && n) hipLaunchKernelGGL(k_bwd_fill, dim3(unsigned(std::min<size_t>((n + 255) / 256, 4096))), dim3(256), 0, st, ptr, n, 0.f);
        };
        fill(g->dw1, size_t(p->n_types) * s->C * 2 * s->C);
        fill(g->db1, size_t(p->n_types) * s->C);
    }
    launch_leaves(p, a.gleaf, d_leaf_first, d_root_item, dout, g->dfeats, chw, st);
    HIP_TRY(hipGetLastError(), "dynbatch_backward");
    return DYNB_OK;
}

bool fast_shape(const dynb_shape* s) { return s->dtype == DYNB_BF16 && s->C == 128 && s->H == 14 && s->W == 14; }

// workspace of the MFMA path
struct BmLayout {
    size_t gy, gleaf, sv_g, sv_dm, sv_dc, pk3bT, pk3aT, pk1T;
    size_t partial, total;
};

BmLayout bm_layout(const dynb_plan* p)
{
    BmLayout L;
    const size_t chw = size_t(mf::P) * mf::C, n_items = p->items.size(), nt = size_t(p->n_types);
    const size_t n_leaf = p->leaf_first.empty() ? 0 : size_t(p->leaf_first.back());
    size_t o = 0;
    auto take = [&](size_t bytes) { size_t at = o; o += align256(std::max<size_t>(bytes, 4)); return at; };
    L.gy = take(n_items * chw * 4);
    L.gleaf = take(n_leaf * chw * 4);
    L.sv_g = take(n_items * chw * 2);
    L.sv_dm = take(n_items * chw * 2);
    L.sv_dc = take(p->has_binary ? n_items * chw * 2 : 0);
    L.pk3bT = take(nt * 9 * 128 * 128 * 2);
    L.pk3aT = take(nt * 9 * 128 * 128 * 2);
    L.pk1T = take(nt * 2 * 128 * 128 * 2);
    L.partial = take(p->wg_units.size() * WG_PARTIAL * 4);
    L.total = o;
    return L;
}

int run_backward_mfma(const dynb_plan* p, const dynb_module_weights* w, const void* feats, const void* fwd_ws, const float* dout,
                      const dynb_module_grads* g, char* ws, hipStream_t st)
{
    static std::atomic<uint64_t> attr_set{0};                 // one bit per device
    int dev = 0;
    HIP_TRY(hipGetDevice(&dev), "hipGetDevice");
    if (!(attr_set.load() >> (dev & 63) & 1)) {
        for (const void* f : {reinterpret_cast<const void*>(k_bwd_node_mfma<1>), reinterpret_cast<const void*>(k_bwd_node_mfma<2>),
                              reinterpret_cast<const void*>(k_bwd_node_mfma<4>), reinterpret_cast<const void*>(k_bwd_node_mfma<7>),
                              reinterpret_cast<const void*>(k_bwd_node_mfma<7, 2>), reinterpret_cast<const void*>(k_bwd_node_mfma<7, 4>)})
            HIP_TRY(hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, bn::LDS_BYTES), "hipFuncSetAttribute(k_bwd_node_mfma)");
        attr_set.fetch_or(uint64_t(1) << (dev & 63));
    }
    const BmLayout L = bm_layout(p);
    const size_t chw = size_t(mf::P) * mf::C, n_items_all = p->items.size();
    const int C = mf::C, nt = p->n_types;
    // the routing tables, item lists and work units were uploaded with the plan
    const dynb_keep_tables KT = dynb_plan_keep_tables(p);
    const char* pd = static_cast<const char*>(p->dev_buf);
    const int32_t* d_leaf_first = reinterpret_cast<const int32_t*>(pd + KT.leaf_first);
    const int32_t* d_root_item = reinterpret_cast<const int32_t*>(pd + KT.root_item);

    // (every function's parameter gradients are written below, by k_bwd_wgrad_mfma where they are one chunk's sum, else, and zeros
    // too, by k_bwd_wgrad_sum; without a two-argument function in the batch there is no conv1x1 gradient to sum)
    if (!p->has_binary) {
        auto fill = [&](float* ptr, size_t n) {
            if (ptr && n) hipLaunchKernelGGL(k_bwd_fill, dim3(unsigned(std::min<size_t>((n + 255) / 256, 4096))), dim3(256), 0, st, ptr, n, 0.f);
        };
        fill(g->dw1, size_t(nt) * C * 2 * C);
        fill(g->db1, size_t(nt) * C);
    }

    // transposed weights in fragment order
    PackArgs pa = {};
    const void* const src[3] = {w->w3a, w->w3b, w->w1};
    const size_t at[3] = {L.pk3aT, L.pk3bT, L.pk1T};
    for (int i = 0; i < 3; ++i) {
        pa.src[i] = static_cast<const bf16_t*>(src[i]);
        pa.dst[i] = reinterpret_cast<u32x4*>(ws + at[i]);
    }
    pa.n_types = nt;
    hipLaunchKernelGGL(k_bwd_pack, dim3(unsigned(std::min<size_t>((size_t(nt) * 4 * 9 * 512 + 255) / 256, 4096)), p->has_binary ? 3 : 2), dim3(256), 0, st, pa);

    // 16-byte aligned: roots read dout itself (the copy took 12 us for 256 examples; a training step 2507 -> 2491, of 16 examples 738 -> 730)
    float* gy = reinterpret_cast<float*>(ws + L.gy);
    const bool in_place = wide_maps(chw, dout);
    if (!in_place) launch_seed(p, dout, d_root_item, gy, chw, st);

    const char* d = static_cast<const char*>(p->dev_buf);
    const dynb_item* d_items = reinterpret_cast<const dynb_item*>(d);
    BmArgs a;
    a.pk3bT = reinterpret_cast<const bf16_t*>(ws + L.pk3bT); a.pk3aT = reinterpret_cast<const bf16_t*>(ws + L.pk3aT);
    a.pk1T = reinterpret_cast<const bf16_t*>(ws + L.pk1T);
    a.gy = gy; a.dout = in_place ? dout : nullptr; a.gleaf = reinterpret_cast<float*>(ws + L.gleaf);
    // u and mid of every item: where the forward pass of a DYNB_PLAN_KEEP plan put them
    const bf16_t* const sv_m = reinterpret_cast<const bf16_t*>(static_cast<const char*>(fwd_ws) + dynb_fast_maps_offset(p));
    a.sv_u = sv_m + n_items_all * chw;
    a.mask_y = static_cast<const unsigned char*>(fwd_ws) + dynb_fast_keep_offset(p);
    a.mask_m = a.mask_y + n_items_all * dynb_fast_mask_bytes();
    a.sv_g = reinterpret_cast<bf16_t*>(ws + L.sv_g); a.sv_dm = reinterpret_cast<bf16_t*>(ws + L.sv_dm);
    a.sv_dc = reinterpret_cast<bf16_t*>(ws + L.sv_dc);
    for (size_t li = p->launches.size(); li-- > 0;) {
        const dynb_launch& l = p->launches[li];
        a.items = d_items + l.start; a.first_item = l.start; a.count = l.count;
        a.gdst0 = reinterpret_cast<const int32_t*>(pd + KT.gdst0) + l.start;
        a.gdst1 = reinterpret_cast<const int32_t*>(pd + KT.gdst1) + l.start;
        const int parts = p->throughput ? 1 : parts_for(l.count);
        const unsigned grid = unsigned((parts * l.count + 7) / 8 * 8);
        a.per_xcd = int32_t(grid / 8);
        auto* kernel = parts == 28 ? k_bwd_node_mfma<7, 4> : parts == 14 ? k_bwd_node_mfma<7, 2> : parts == 7 ? k_bwd_node_mfma<7> : parts == 4 ? k_bwd_node_mfma<4> : parts == 2 ? k_bwd_node_mfma<2> : k_bwd_node_mfma<1>;
        hipLaunchKernelGGL(kernel, dim3(grid), dim3(256), bn::LDS_BYTES, st, a);
    }
    {
        WgArgs q;
        q.items = d_items;
        q.units = reinterpret_cast<const dynb_wg_unit*>(pd + KT.units);
        q.order = reinterpret_cast<const int32_t*>(pd + KT.order);
        q.fn_first = reinterpret_cast<const int32_t*>(pd + KT.fn_first);
        q.fn_items = reinterpret_cast<const int32_t*>(pd + KT.fn_items);
        q.n_chunks = 0; q.n_joins = 0;
        for (const dynb_wg_group& wg : p->wg_groups) (wg.mode == 2 ? q.n_joins : q.n_chunks) += wg.n_units;
        q.n_chunks /= 3;                                      // (a unit for each kernel row)
        q.feats = static_cast<const bf16_t*>(feats); q.slots = static_cast<const bf16_t*>(fwd_ws);
        q.sv_u = a.sv_u; q.sv_m = sv_m; q.sv_g = a.sv_g; q.sv_dm = a.sv_dm; q.sv_dc = a.sv_dc;
        q.partial = reinterpret_cast<float*>(ws + L.partial);
        q.dw3a = g->dw3a; q.db3a = g->db3a; q.dw3b = g->dw3b; q.db3b = g->db3b; q.dw1 = g->dw1; q.db1 = g->db1;
        const unsigned sets = unsigned((q.n_chunks + 7) / 8 + (q.n_joins + 7) / 8);
        if (sets > 0) hipLaunchKernelGGL(k_bwd_wgrad_mfma, dim3(sets * 32), dim3(256), 2 * WG_MAP, st, q);
        WsArgs r;
        r.groups = reinterpret_cast<const dynb_wg_group*>(pd + KT.groups);
        r.partial = q.partial;
        r.dw3a = g->dw3a; r.db3a = g->db3a; r.dw3b = g->dw3b; r.db3b = g->db3b; r.dw1 = g->dw1; r.db1 = g->db1;
        // groups without units: the sum writes their zeros
        hipLaunchKernelGGL(k_bwd_wgrad_sum, dim3(3 * 128 * 128 / 4 / 256, unsigned(p->wg_groups.size())), dim3(256), 0, st, r);
    }
    launch_leaves(p, a.gleaf, d_leaf_first, d_root_item, dout, g->dfeats, chw, st);
    HIP_TRY(hipGetLastError(), "dynbatch_backward(mfma kernels)");
    return DYNB_OK;
}

int check_backward(const dynb_plan* p, const dynb_shape* s, const char* who)
{
    if (!p || !s) return fail(DYNB_E_INVAL, std::string(who) + ": NULL argument");
    if (s->C <= 0 || s->H <= 0 || s->W <= 0) return fail(DYNB_E_INVAL, std::string(who) + ": C, H, W must be positive");
    if (s->dtype != DYNB_F32 && s->dtype != DYNB_BF16) return fail(DYNB_E_UNSUPPORTED, std::string(who) + ": unknown dtype");
    if (!p->keep) return fail(DYNB_E_UNSUPPORTED, std::string(who) + ": the plan was not made with DYNB_PLAN_KEEP");
    if (p->shared_nodes) return fail(DYNB_E_UNSUPPORTED, std::string(who) + ": dependency graphs with shared nodes have no backward pass yet");
    if (size_t(s->C) * s->H * s->W >= (size_t(1) << 31) || size_t(s->C) * 9 * s->C >= (size_t(1) << 31))
        return fail(DYNB_E_UNSUPPORTED, std::string(who) + ": map too large");
    return DYNB_OK;
}

}  // namespace

extern "C" size_t dynbatch_backward_workspace_bytes(const dynb_plan* p, const dynb_shape* s)
{
    if (check_backward(p, s, "dynbatch_backward_workspace_bytes") != DYNB_OK) return 0;
    if (fast_shape(s)) return std::max<size_t>(bm_layout(p).total, 256);
    return std::max<size_t>(bwd_layout(p, s).total, 256);
}

extern "C" int dynbatch_backward(const dynb_plan* p, const dynb_shape* s, const dynb_module_weights* w, const void* feats,
                                 const void* out, const void* forward_workspace, const float* dout,
                                 const dynb_module_grads* grads, void* workspace, size_t workspace_bytes, void* stream)
{
    int rc = check_backward(p, s, "dynbatch_backward");
    if (rc != DYNB_OK) return rc;
    if (!w || !feats || !out || !forward_workspace || !dout || !grads || !workspace)
        return fail(DYNB_E_INVAL, "dynbatch_backward: NULL argument");
    if (!w->w3a || !w->w3b) return fail(DYNB_E_INVAL, "dynbatch_backward: conv3x3 weights missing");
    if (!grads->dfeats || !grads->dw3a || !grads->db3a || !grads->dw3b || !grads->db3b)
        return fail(DYNB_E_INVAL, "dynbatch_backward: a gradient tensor is missing");
    if (p->has_binary && (!w->w1 || !grads->dw1 || !grads->db1))
        return fail(DYNB_E_INVAL, "dynbatch_backward: two-argument functions need w1, dw1 and db1");
    if (!p->dev_buf) return fail(DYNB_E_WORKSPACE, "dynbatch_backward: plan not uploaded");
    if (workspace_bytes < (fast_shape(s) ? bm_layout(p).total : bwd_layout(p, s).total))
        return fail(DYNB_E_WORKSPACE, "dynbatch_backward: workspace too small");
    if (reinterpret_cast<uintptr_t>(workspace) & 255) return fail(DYNB_E_INVAL, "dynbatch_backward: workspace not 256-byte aligned");
    hipStream_t st = static_cast<hipStream_t>(stream);
    char* ws = static_cast<char*>(workspace);
    if (fast_shape(s)) return run_backward_mfma(p, w, feats, forward_workspace, dout, grads, ws, st);
    if (s->dtype == DYNB_BF16) return run_backward<bf16_t>(p, s, w, feats, out, forward_workspace, dout, grads, ws, st);
    return run_backward<float>(p, s, w, feats, out, forward_workspace, dout, grads, ws, st);
}
