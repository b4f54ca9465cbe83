// GPU executor of a plan: gather -> batched residual conv module -> scatter, one launch group
// per label (paper: Methods / Improved topological sort, a pool is executed as one batch; Results / IEP, data stacking).
//
// Two kernel families with the same semantics:
//   * k_module_mfma  — bf16, C = 128, 14 x 14: one fused kernel per launch group.  A workgroup
//                      owns a node or a part of one; the node's input map is gathered straight into an
//                      LDS halo tile, conv1x1 (binary functions), conv3x3, ReLU, conv3x3, residual
//                      add and ReLU all run from that tile on MFMA, and the result is scattered to
//                      the node's slot (or to the output tensor for a root).
//   * k_conv         — any C/H/W, fp32 or bf16 storage, fp32 accumulate (iep_conv.h): one launch per convolution of a
//                      launch group, tiles small enough to spread narrow groups over the chip; for small maps k_node, a
//                      whole module per workgroup, for a few channels or pixels k_conv_plain.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cstdlib>
#include <cstring>
#include <string>

#include "device_utils.h"
#include "iep_conv.h"
#include "iep_mfma.h"
#include "plan_internal.h"
#include "timing.h"

using dynb::fail;

#define HIP_TRY(expr, what)                                                                   \
    do {                                                                                      \
        hipError_t e_ = (expr);                                                               \
        if (e_ != hipSuccess)                                                                 \
            return fail(DYNB_E_HIP, std::string(what) + ": " + hipGetErrorString(e_));        \
    } while (0)

namespace {

// out[example] = feats[example] for programs that are a single SCENE token
__global__ void k_copy_leaf_roots(const int32_t* examples, int n, const uint32_t* feats, uint32_t* out,
                                  size_t words_per_map)
{
    if (int(blockIdx.y) >= n) return;
    const int ex = examples[blockIdx.y];
    for (size_t w = size_t(blockIdx.x) * blockDim.x + threadIdx.x; w < words_per_map;
         w += size_t(gridDim.x) * blockDim.x)
        out[size_t(ex) * words_per_map + w] = feats[size_t(ex) * words_per_map + w];
}

// ------------------------------------------------------------------------------------------
// Fused MFMA module kernel: bf16, C = 128, 14 x 14
// ------------------------------------------------------------------------------------------
// Development aid, compiled in only with -DDYNB_PHASE_CLOCKS: lane 0 of every wave stores the
// shader clock at the phase boundaries of k_module_mfma into a caller-provided device buffer.
#ifdef DYNB_PHASE_CLOCKS
__device__ long long* g_phase_clk = nullptr;      // [workgroup][wave][16]
#define PHASE(i)                                                                             \
    do {                                                                                     \
        if ((threadIdx.x & 63) == 0 && g_phase_clk)                                          \
            g_phase_clk[(size_t(blockIdx.x) * 4 + (threadIdx.x >> 6)) * 16 + (i)] = clock64(); \
        if ((threadIdx.x & 63) == 0 && g_phase_clk && ((i) == 0 || (i) == 9))                 \
            g_phase_clk[(size_t(blockIdx.x) * 4 + (threadIdx.x >> 6)) * 16 + 10 + ((i) != 0)] = wall_clock64(); \
    } while (0)
#else
#define PHASE(i) do {} while (0)
#endif

struct MfArgs {
    const dynb_item* items;
    int32_t count;
    int32_t first_item;       // index of items[0] in the plan
    const bf16_t* feats;
    bf16_t* out;
    bf16_t* slots;
    const bf16_t* w1;
    const float* b1;
    const bf16_t* w3a;
    const float* b3a;
    const bf16_t* w3b;
    const float* b3b;
    // Workgroups of a die's run.  (Here and not next to count: the arguments lie in host memory, a cache line of 64 bytes at a time, and what a workgroup wants
    // first should bring both lines with it.  With the grid's size for it and two fields more, which put that into a third line, a launch took
    // 0.15 us longer, and so it did with this field in the first: one program 162.6 / 166 us.)
    int32_t per_xcd;
    // plans that keep what the backward pass needs (dynb_fast_keep_offset, plan_internal.h): masks of the results and of mid, mid, and u of two-argument
    // functions, one of each per item
    int32_t n_items;
    char* keep;
};


// dst[function][tile][fragment][lane][i] = src[function][co = tile*32 + rho(lane%32)][tap][ci = (lane/32)*64 + j*8 + i] with
// (tap, j) of the fragment as in iep_mfma.h; a thread takes a row's half for one tap, the 128 bytes of all eight j; ntap = 9 for a conv3x3, 2 for the two
// halves of the conv1x1 over 2C inputs.
// rho permutes the channels inside a tile: MFMA output row m = 8b + 4h + c (accumulator element 4b + c
// of lane half h) is given channel 16h + 4b + c, so that the 16 accumulator elements of a lane are 16
// consecutive channels and leave the kernel as two 16-byte stores.
// blockIdx.y: w3a, w3b, w1.  (In a launch each, a thread per 16-byte piece, so that up to eight XCDs fetched every line, they took 18, 11 and 4 us for 41
// functions; in one launch 28; with whole lines 13.4.)
__global__ void k_pack_weights(PackArgs a)
{
    const u32x4* __restrict__ const src = reinterpret_cast<const u32x4*>(a.src[blockIdx.y]);
    u32x4* __restrict__ const dst = a.dst[blockIdx.y];
    const int ntap = blockIdx.y == 2 ? 2 : 9;
    const size_t total = size_t(a.n_types) * ntap * 4 * 64;
    for (size_t q = size_t(blockIdx.x) * blockDim.x + threadIdx.x; q < total; q += size_t(gridDim.x) * blockDim.x) {
        const int lane = int(q & 63), tile = int(q >> 6) & 3, tap = int((q >> 8) % ntap), m = lane & 31;
        const size_t type = (q >> 8) / ntap;
        const int co = tile * 32 + ((m >> 2) & 1) * 16 + (m >> 3) * 4 + (m & 3), kh = tap / 3;
        const u32x4* const from = src + ((((type * 128 + co) * ntap + tap) * 128 + (lane >> 5) * 64) >> 3);
        // fragments of this tap: one per step
        const int f0 = ntap == 9 ? tap % 3 * 24 + (kh == 0 ? 0 : 3 - kh) : tap * 8, step = ntap == 9 ? 3 : 1;
        u32x4* const to = dst + ((type * 4 + tile) * (size_t(ntap) * 8) + f0) * 64 + lane;
        u32x4 v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = from[j];
#pragma unroll
        for (int j = 0; j < 8; ++j) to[j * step * 64] = v[j];
    }
}

// (How a node is spread over workgroups: PartShape, iep_mfma.h.)
// All fit 256 registers and half of a CU's LDS, so that two workgroups share a CU where a launch group is wide enough,
// and one's staging, swap and epilogue run under the other's MFMAs.  (A whole-node layout of its own for groups of
// up to one node per CU, with twice the weight ring in 346 registers, was 3 % slower: the accumulators then live in
// the upper half of the register file, and every other use of them is a copy.)
// One workgroup's share of a launch group: position `logical` (a node, or a part of one) of the items a.items[0 .. a.count).
// KEEP: u (two-argument functions) and mid are also written behind a.keep, and the masks of mid and the result.  SPLIT: workgroups that share a part, each with
// 4 / SPLIT channel tiles of the second conv (parts_for).
template <int PARTS, bool KEEP = false, int SPLIT = 1>
__device__ __forceinline__ void module_body(const MfArgs& a, const int logical)
{
    using namespace mf;
    using Shape = PartShape<PARTS>;
    constexpr bool WHOLE = PARTS == 1;
    constexpr int MTA = Shape::MTA, MTB = Shape::MTB, UROWS = Shape::UROWS;
    constexpr int MTU = WHOLE ? MT7 : (UROWS * S + 31) / 32;     // tiles of the join: row pairs, or 32 consecutive pixels
    constexpr int NTHR = 256;
    constexpr int RW = Shape::RW;
    extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];

    const int node = logical / (PARTS * SPLIT), part = logical / SPLIT % PARTS, share = logical % SPLIT;
    if (node >= a.count) return;
    // image rows: output [orow0, orow1), windows of the convs [row_a, row_a + 2 MTA) and [row_b, row_b + 2 MTB), u
    // [urow0, urow0 + UROWS), every one of them moved inside the map
    const int orow0 = part * Shape::ROWS, orow1 = min(orow0 + Shape::ROWS, S);
    const int row_a = min(max(orow0 - 1, 0), S - 2 * MTA), row_b = min(orow0, S - 2 * MTB);
    const int urow0 = min(max(row_a - 1, 0), S - UROWS);

    PHASE(0);
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const dynb_item it = a.items[node];
    const bool binary = it.src1 != DYNB_NO_ARG;                        // uniform over the workgroup
    const int r = lane & 31, h = lane >> 5;
    const int n0 = wave * 32;                 // first output channel of this wave
    const size_t keep_at = size_t(a.first_item + node) * P;           // first pixel of this item's kept maps

    // packed weights of this wave's channel tile
    const bf16_t* wrow_a = a.w3a + (size_t(it.type) * 4 + wave) * 72 * FRAG + lane * 8;
    const int tile_b = SPLIT == 1 ? wave : share * (4 / SPLIT) + wave % (4 / SPLIT);  // the second conv's; waves beyond 4 / SPLIT have none
    const bf16_t* wrow_b = a.w3b + (size_t(it.type) * 4 + tile_b) * 72 * FRAG + lane * 8;
    bf16x8 ring[RW];

    // ---- gather: zero border once, then the argument map into the centre of the halo tile;
    // all global loads of the map are issued before the first LDS write, so one memory latency is paid
    // (the rows of u are those that the first conv's taps can touch)
    constexpr int NIT = (UROWS * S * 16 + NTHR - 1) / NTHR;
    const int c_lo = urow0 * S * 16, c_hi = c_lo + UROWS * S * 16;
    u32x4 tmp[NIT];
    auto stage_load = [&](const bf16_t* src) {
        const u32x4* s4 = reinterpret_cast<const u32x4*>(src);
#pragma unroll
        for (int i = 0; i < NIT; ++i) {
            const int c = c_lo + tid + i * NTHR;
            if (c < c_hi) tmp[i] = s4[c];
        }
    };
    auto stage_store = [&]() {
#pragma unroll
        for (int i = 0; i < NIT; ++i) {
            const int c = c_lo + tid + i * NTHR;
            if (c < c_hi) {
                const int p = c >> 4, part = c & 15;
                const uint32_t addr = uint32_t((p / S + 1) * ROW_BYTES + (p % S + 1) * PIX_BYTES + part * 16);
                *reinterpret_cast<u32x4*>(lds_raw + addr) = tmp[i];
            }
        }
    };
    // the centre of the halo tile -> a map, this workgroup's output rows (and share of the channels), in coalesced 16-byte pieces, and the map's mask
    // (a launch of whole nodes 31.9 -> 34.9 us, of halves 21.4 -> 22.4, of quarters 15.7 -> 16.2; the backward pass gains 8.1, 2.3 and 1.4.  Four lanes'
    // bytes put together, for a quarter of the stores: the registers do not suffice, 41 us.)
    auto copy_out = [&](bf16_t* dst, auto&& mask) {
        constexpr int OUTPIECES = Shape::ROWS * S * 16;
        int t = tid;
        if constexpr (KEEP) asm volatile("" : "+v"(t));          // (the pieces' addresses made anew, not kept beside the sums from one map to the next)
#pragma unroll
        for (int i = 0; i < (OUTPIECES + NTHR - 1) / NTHR; ++i) {
            const int c = orow0 * S * 16 + t + i * NTHR;
            if (c < orow1 * S * 16 && (SPLIT == 1 || (c & 15) / (16 / SPLIT) == share)) {
                const int p = c >> 4, part = c & 15;
                const u32x4 v = *reinterpret_cast<const u32x4*>(lds_raw + uint32_t((p / S + 1) * ROW_BYTES + (p % S + 1) * PIX_BYTES + part * 16));
                reinterpret_cast<u32x4*>(dst)[c] = v;
                mask(c, v);
            }
        }
    };
    auto no_mask = [](int, const u32x4&) {};
    // kept: masks of the results | of mid | (256-byte aligned) mid | u
    unsigned char* const mask_y = KEEP ? reinterpret_cast<unsigned char*>(a.keep) : nullptr;
    unsigned char* const mask_m = KEEP ? mask_y + size_t(a.n_items) * (P * C / 8) : nullptr;
    bf16_t* const keep_m = KEEP ? reinterpret_cast<bf16_t*>(a.keep + dynb_align256(2 * size_t(a.n_items) * (P * C / 8))) : nullptr;
    bf16_t* const keep_u = KEEP ? keep_m + size_t(a.n_items) * (P * C) : nullptr;
    auto mask_to = [&](unsigned char* masks) {
        unsigned char* const m = masks + keep_at * (C / 8);
        return [m](int c, const u32x4& v) { m[uint32_t(c)] = static_cast<unsigned char>(positive_mask(v)); };
    };
    auto arg_map = [&](int32_t s) { return s >= 0 ? a.slots + size_t(s) * (P * C) : a.feats + size_t(-1 - s) * (P * C); };
    // Loads return in the order they were issued: the argument map (needed first) goes ahead of the weight ring,
    // whose fragments then arrive while the map is written to the tile.
    stage_load(arg_map(it.src0));
    __builtin_amdgcn_sched_barrier(0);
    // biases through LDS: b3a, b3b, b1 (requested here, not where a wave would wait for them)
    float bias_reg[2] = {0.f, 0.f};
    {
        const float* const b0 = tid < C ? a.b3a : a.b3b;
        if (b0) bias_reg[0] = b0[size_t(it.type) * C + (tid & (C - 1))];
        if (binary && a.b1 && tid < C) bias_reg[1] = a.b1[size_t(it.type) * C + tid];
    }
    __builtin_amdgcn_sched_barrier(0);
    if (!binary) ring_fill<RW>(ring, wrow_a);
    zero_border<NTHR>(tid, row_a, row_a + 2 * MTA + 1);
    *reinterpret_cast<float*>(lds_raw + BIAS_OFF + tid * 4) = bias_reg[0];
    if (tid < C) *reinterpret_cast<float*>(lds_raw + BIAS_OFF + (2 * C + tid) * 4) = bias_reg[1];
    stage_store();

    // this lane's LDS address for the first row pair of the convs' windows; the pixel it ends up with in tile t is column
    // r & 15 of window row 2 t + r / 16 (columns 14 and 15 are padding)
    const uint32_t x_a = pair_lane_addr(lane) + uint32_t(row_a * ROW_BYTES), x_b = pair_lane_addr(lane) + uint32_t(row_b * ROW_BYTES);
    const bool real = (r & 15) < S;
    // its 16 accumulator elements are channels chan .. chan + 15 (the packed weights carry the matching row permutation)
    const int chan = n0 + 16 * h, chan_b = tile_b * 32 + 16 * h;             // (of the first and of the second conv)

    auto bias4 = [&](int which, int b) {      // channels chan + 4 b .. + 3 of b3a (0), b3b (1), b1 (2)
        return *reinterpret_cast<const f32x4*>(lds_raw + BIAS_OFF + uint32_t((which * C + (which == 1 ? chan_b : chan) + b * 4) * 4));
    };
    auto init_bias = [&](auto& acc, int which) {
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const f32x4 v = bias4(which, b);
#pragma unroll
            for (auto& t : acc) {
                t[4 * b + 0] = v.x; t[4 * b + 1] = v.y;
                t[4 * b + 2] = v.z; t[4 * b + 3] = v.w;
            }
        }
    };
    // byte address of this lane's centre pixel of tile t of a window, its first channel
    auto centre = [&](uint32_t x, int t) -> uint32_t { return x - uint32_t(h * 128) + uint32_t(CENTER + chan * 2 + 2 * t * ROW_BYTES); };
    auto centre_b = [&](int t) -> uint32_t { return x_b - uint32_t(h * 128) + uint32_t(CENTER + chan_b * 2 + 2 * t * ROW_BYTES); };
    // ReLU(acc[8q .. 8q+7]) as 8 packed bf16 (q = 0, 1)
    auto packed = [&](const f32x16& acc, int q) -> u32x4 {
        u32x4 pk;
        pk.x = relu_bf16x2(pack_bf16x2(acc[8 * q + 0], acc[8 * q + 1]));
        pk.y = relu_bf16x2(pack_bf16x2(acc[8 * q + 2], acc[8 * q + 3]));
        pk.z = relu_bf16x2(pack_bf16x2(acc[8 * q + 4], acc[8 * q + 5]));
        pk.w = relu_bf16x2(pack_bf16x2(acc[8 * q + 6], acc[8 * q + 7]));
        return pk;
    };

    PHASE(1);
    __syncthreads();
    PHASE(2);

    // ---- binary functions: u = ReLU(conv1x1(concat(arg0, arg1)) + b1), built in the same tile.
    // The first conv3x3 reads u one row beyond its window, so in parts of a node the 1x1 runs on its own window of
    // UROWS rows, in tiles of 32 consecutive pixels.
    f32x16 acc_a[MTA];
    if (binary) {
        constexpr int UPIX = UROWS * S;
        f32x16 acc_u[WHOLE ? 1 : MTU];                   // (whole nodes: the registers of acc_a)
        auto& acc = [&]() -> auto& { if constexpr (WHOLE) return acc_a; else return acc_u; }();
        uint32_t ua[WHOLE ? 1 : MTU];
        if constexpr (!WHOLE) {
#pragma unroll
            for (int t = 0; t < MTU; ++t) {
                const int p = urow0 * S + min(t * 32 + r, UPIX - 1);
                ua[t] = uint32_t(CENTER + (p / S) * ROW_BYTES + (p % S) * PIX_BYTES + h * 128);
            }
        } else ua[0] = x_a + uint32_t(CENTER);
        auto uaddr = [&](int t) { return WHOLE ? ua[0] + uint32_t(2 * t * ROW_BYTES) : ua[WHOLE ? 0 : t]; };
        // the first half of the 1x1 weights (argument 0), then the second: its fragments are fetched under the first
        // half's loop and wait while the second argument is staged
        const bf16_t* w1row = a.w1 + (size_t(it.type) * 4 + wave) * 16 * FRAG + lane * 8;
        bf16x8 w1f[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) w1f[j] = *reinterpret_cast<const bf16x8*>(w1row + j * FRAG);
        stage_load(arg_map(it.src1));                     // arrives under the first half's loop
        __builtin_amdgcn_sched_barrier(0);
        init_bias(acc, 2);
        kloop1<MTU, true>(acc, uaddr, w1f, w1row + 8 * FRAG);
        __syncthreads();
        stage_store();
        __syncthreads();
        kloop1<MTU, false>(acc, uaddr, w1f, nullptr);
        ring_fill<RW>(ring, wrow_a);                      // (only now: the loops above need the registers)
        __syncthreads();
#pragma unroll
        for (int t = 0; t < MTU; ++t)                     // ReLU(acc) -> bf16 -> centre of the halo tile (in place)
            if (WHOLE ? real : t * 32 + r < UPIX) {
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    const u32x4 pk = packed(acc[t], q);
                    *reinterpret_cast<u32x4*>(lds_raw + uaddr(t) - uint32_t(h * 128) + uint32_t((chan + q * 8) * 2)) = pk;
                }
            }
        __syncthreads();
        if constexpr (KEEP) copy_out(keep_u + keep_at * C, no_mask);
    }

    // ---- first conv3x3 + ReLU, result replaces the tile; the old centre values become the residual
    PHASE(3);
    init_bias(acc_a, 0);
    kloop3<MTA, RW, Shape::XA>(acc_a, x_a, ring, wrow_a, wrow_b);       // leaves the ring filled for the second conv
    PHASE(4);
    // (one window for both convs: the second accumulates in the registers of the first)
    constexpr bool SAME = MTA == MTB;
    static_assert(!SAME || SPLIT == 1, "a part that is shared has its own window for the second conv");
    f32x16 acc_own[SAME ? 1 : MTB];
    auto& acc_b = [&]() -> auto& { if constexpr (SAME) return acc_a; else return acc_own; }();
    const bool second = SPLIT == 1 || wave < 4 / SPLIT;                // uniform over the wave
    auto old = [&](int t, int q) { return *reinterpret_cast<const u32x4*>(lds_raw + centre_b(t) + uint32_t(q * 16)); };
    auto residual = [&](int t, int q, const u32x4& res) {
        const f32x4 blo = bias4(1, 2 * q), bhi = bias4(1, 2 * q + 1);
        f32x16& acc = acc_b[t];
        acc[8 * q + 0] = __uint_as_float(res.x << 16) + blo.x;
        acc[8 * q + 1] = __uint_as_float(res.x & 0xffff0000u) + blo.y;
        acc[8 * q + 2] = __uint_as_float(res.y << 16) + blo.z;
        acc[8 * q + 3] = __uint_as_float(res.y & 0xffff0000u) + blo.w;
        acc[8 * q + 4] = __uint_as_float(res.z << 16) + bhi.x;
        acc[8 * q + 5] = __uint_as_float(res.z & 0xffff0000u) + bhi.y;
        acc[8 * q + 6] = __uint_as_float(res.w << 16) + bhi.z;
        acc[8 * q + 7] = __uint_as_float(res.w & 0xffff0000u) + bhi.w;
    };
    auto residuals = [&]() {
#pragma unroll
        for (int t = 0; t < MTB; ++t) { residual(t, 0, old(t, 0)); residual(t, 1, old(t, 1)); }
    };
    // (of a shared part, a wave's channels of the second conv are another wave's of the first: read before anyone replaces them)
    if (SPLIT > 1 && second && real) residuals();
    __syncthreads();
    PHASE(5);
    if (real) {
        // ReLU(acc_a) into the tile, old centre values + bias into acc_b.  A wave reads and writes its own channels only, and
        // its reads come first: where the windows are the same, piece by piece, else all of them
        auto replace = [&](int t, int q) { *reinterpret_cast<u32x4*>(lds_raw + centre(x_a, t) + uint32_t(q * 16)) = packed(acc_a[t], q); };
        if constexpr (SAME) {
#pragma unroll
            for (int q = 0; q < 2; ++q)
#pragma unroll
                for (int t = 0; t < MTA; ++t) {
                    const u32x4 res = old(t, q);
                    replace(t, q);
                    residual(t, q, res);
                }
        } else {
            if constexpr (SPLIT == 1) residuals();
#pragma unroll
            for (int t = 0; t < MTA; ++t) { replace(t, 0); replace(t, 1); }
        }
    }
    PHASE(6);
    __syncthreads();
    PHASE(7);

    if constexpr (KEEP) copy_out(keep_m + keep_at * C, mask_to(mask_m));

    // ---- second conv3x3 on top of (residual + bias), ReLU, scatter.  The result leaves through the tile: in the
    // accumulators a lane holds 32 bytes of a pixel, and stores in which every lane touches a line of its own take 4.4k
    // clocks of a whole-node workgroup's 53k, the way through LDS with coalesced stores 3.6k.
    if (second) kloop3<MTB, RW, Shape::XB, false>(acc_b, x_b, ring, wrow_b, wrow_b);
    PHASE(8);
    __syncthreads();
    if (second && real) {
#pragma unroll
        for (int t = 0; t < MTB; ++t)
#pragma unroll
            for (int q = 0; q < 2; ++q) *reinterpret_cast<u32x4*>(lds_raw + centre_b(t) + uint32_t(q * 16)) = packed(acc_b[t], q);
    }
    __syncthreads();
    bf16_t* const dst = it.dst >= 0 ? a.slots + size_t(it.dst) * (P * C) : a.out + size_t(-1 - it.dst) * (P * C);
    if constexpr (KEEP) copy_out(dst, mask_to(mask_y));
    else copy_out(dst, no_mask);
    PHASE(9);
}

template <int PARTS, bool KEEP = false, int SPLIT = 1>
__global__ __launch_bounds__(256, 2) void k_module_mfma(MfArgs a)
{
    // Workgroup -> position in the launch group.  Consecutive workgroup ids land on different
    // XCDs; give every XCD one contiguous run of items (items are sorted by function id) so that
    // a function's weights stay in as few L2s as possible.
    module_body<PARTS, KEEP, SPLIT>(a, (blockIdx.x & 7) * a.per_xcd + (blockIdx.x >> 3));
}

// ---- one dependency-driven launch per batch ---------------------------------------------------------
// Resident workgroups claim units of work (tickets) in the plan's execution order from one device
// counter.  A unit's arguments are results of units with smaller tickets; those were claimed by
// workgroups that are already running and that in turn only wait for still smaller tickets, so the unit
// with the smallest unfinished ticket never waits and every wait ends.  The waits are bounded all the
// same: a workgroup that gives up raises the status word, and from then on every workgroup only drains
// the counter.  ready[slot] counts published halves of a result (a whole node adds 2).
struct PersistArgs {
    const int32_t* tickets;   // device [n_tickets]: 4 * item + part
    int32_t n_tickets;
    int32_t spin_limit;
    int32_t* ready;           // device [n_slots], zero before the launch
    int32_t* counter;         // device, zero before the launch
    int32_t* status;          // device, zero before the launch; 1 = a wait expired
};

__device__ __forceinline__ int32_t load_relaxed(const int32_t* p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__global__ __launch_bounds__(256, 1) void k_module_persist(MfArgs a, PersistArgs q)
{
    __shared__ int32_t s_ticket, s_go;
    const dynb_item* items = a.items;
    for (;;) {
        if (threadIdx.x == 0) {
            const int32_t tk = __hip_atomic_fetch_add(q.counter, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            int32_t go = 0;                                   // 0: stop, 1: compute, 2: skip (draining after an error)
            if (tk < q.n_tickets) {
                go = 1;
                const dynb_item it = items[q.tickets[tk] >> 2];
                for (int s = 0; s < 2 && go == 1; ++s) {
                    const int32_t src = s == 0 ? it.src0 : it.src1;
                    if (src < 0) continue;                    // an example's feature map (always there) or no argument
                    int32_t polls = 0;
                    while (load_relaxed(q.ready + src) < 2) {
                        if (polls >= q.spin_limit || load_relaxed(q.status) != 0) {
                            __hip_atomic_store(q.status, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                            go = 2;
                            break;
                        }
                        ++polls;
                        __builtin_amdgcn_s_sleep(8);
                    }
                }
                if (go == 1 && load_relaxed(q.status) != 0) go = 2;
                // The arguments' maps were written by other CUs, possibly behind another L2: drop what this CU's
                // vector cache and this L2 may still hold of those addresses.  One wave does it for the
                // workgroup (its waves share both caches); the others load only after the barrier below.
                if (go == 1) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
            }
            s_ticket = tk;
            s_go = go;
        }
        __syncthreads();
        const int32_t tk = s_ticket, go = s_go;
        __syncthreads();                                      // both are read before thread 0 writes them again
        if (go == 0) return;
        if (go == 2) continue;
        const int32_t t = q.tickets[tk];
        MfArgs b = a;
        b.items = items + (t >> 2);
        b.count = 1;
        const int part = t & 3;
        if (part == 0) module_body<1>(b, 0);
        else module_body<2>(b, part - 1);
        // Publish: every wave waits until its stores of the result have reached the L2 (all waves of a
        // workgroup sit behind the same one), then one thread writes that L2's dirty lines back to memory,
        // where every CU can see them, and raises the flag (the agent-scope release does both).
        wait_for_stores();
        __syncthreads();                                      // also frees the LDS tile for the next unit
        const int32_t dst = b.items[0].dst;
        if (threadIdx.x == 0 && dst >= 0)
            __hip_atomic_fetch_add(q.ready + dst, part == 0 ? 2 : 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
    }
}

__global__ void k_fill_i32(int32_t* p, size_t n, int32_t v)
{
    for (size_t i = size_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n; i += size_t(gridDim.x) * blockDim.x) p[i] = v;
}

size_t elt_bytes(int dtype) { return dtype == DYNB_BF16 ? 2 : 4; }

bool fast_shape(const dynb_shape* s) { return s->dtype == DYNB_BF16 && s->C == 128 && s->H == 14 && s->W == 14; }

size_t align256(size_t v) { return (v + 255) & ~size_t(255); }

size_t packed_weight_bytes(int n_types) { return dynb_fast_packed_weight_bytes(n_types); }

}  // namespace

#ifdef DYNB_PHASE_CLOCKS
extern "C" int dynb_debug_phase_clocks(void* device_buf)
{
    long long* p = static_cast<long long*>(device_buf);
    return hipMemcpyToSymbol(HIP_SYMBOL(g_phase_clk), &p, sizeof(p)) == hipSuccess ? DYNB_OK : DYNB_E_HIP;
}
#endif

// Device buffer layout of an uploaded plan: items | leaf-root example ids | arity table | tickets
static size_t plan_items_bytes(const dynb_plan* p) { return dynb_plan_items_bytes(p); }
static size_t plan_leaf_bytes(const dynb_plan* p) { return dynb_plan_leaf_bytes(p); }
static size_t plan_arity_bytes(const dynb_plan* p) { return dynb_plan_arity_bytes(p); }
static size_t plan_ticket_bytes(const dynb_plan* p) { return dynb_plan_ticket_bytes(p); }

extern "C" size_t dynbatch_plan_device_bytes(const dynb_plan* p)
{
    if (!p) return 0;
    return dynb_plan_keep_tables(p).end + 256;
}

// Workspace tail of the dependency-driven launch: ready[n_slots] | counter | status (after the slots and,
// without prepared weights, the packed weights)
static size_t persist_sync_bytes(const dynb_plan* p) { return dynb_fast_sync_bytes(p); }

// offset of that tail: behind the slots and the room for packed weights
static size_t persist_sync_offset(const dynb_plan* p)
{
    return dynb_fast_sync_offset(p);
}

static std::atomic<int32_t> g_spin_limit{1 << 22};

extern "C" int32_t dynb_set_spin_limit(int32_t polls) { return g_spin_limit.exchange(polls < 0 ? 0 : polls); }

extern "C" int dynbatch_plan_upload(dynb_plan* p, void* dev_buf, size_t bytes, void* stream)
{
    if (!p || !dev_buf) return fail(DYNB_E_INVAL, "dynbatch_plan_upload: NULL argument");
    if (bytes < dynbatch_plan_device_bytes(p)) return fail(DYNB_E_WORKSPACE, "dynbatch_plan_upload: buffer too small");
    if (reinterpret_cast<uintptr_t>(dev_buf) & 15) return fail(DYNB_E_INVAL, "dynbatch_plan_upload: buffer not 16-byte aligned");
    hipStream_t st = static_cast<hipStream_t>(stream);
    // One copy: the parts are laid out in a host image of the device buffer (a separate copy per part costs a few
    // microseconds of stream time each, which shows in a step of less than a millisecond).  The image belongs to the
    // plan, so it lives as long as the copy may need it.
    const dynb_keep_tables t = dynb_plan_keep_tables(p);
    p->image.assign(t.end, 0);
    char* h = p->image.data();
    auto put = [&](size_t at, const void* src, size_t n) { if (n) memcpy(h + at, src, n); };
    put(0, p->items.data(), p->items.size() * sizeof(dynb_item));
    put(plan_items_bytes(p), p->leaf_roots.data(), p->leaf_roots.size() * sizeof(int32_t));
    put(plan_items_bytes(p) + plan_leaf_bytes(p), p->arity.data(), p->arity.size());
    put(plan_items_bytes(p) + plan_leaf_bytes(p) + plan_arity_bytes(p), p->tickets.data(), p->tickets.size() * sizeof(int32_t));
    if (p->keep) {                                            // what the backward pass works from
        put(t.gdst0, p->grad_dst0.data(), p->grad_dst0.size() * 4);
        put(t.gdst1, p->grad_dst1.data(), p->grad_dst1.size() * 4);
        put(t.leaf_first, p->leaf_first.data(), p->leaf_first.size() * 4);
        put(t.root_item, p->root_item.data(), p->root_item.size() * 4);
        put(t.fn_first, p->fn_first.data(), p->fn_first.size() * 4);
        put(t.fn_items, p->fn_items.data(), p->fn_items.size() * 4);
        put(t.fn_order, p->fn_order.data(), p->fn_order.size() * 4);
        put(t.units, p->wg_units.data(), p->wg_units.size() * sizeof(dynb_wg_unit));
        put(t.groups, p->wg_groups.data(), p->wg_groups.size() * sizeof(dynb_wg_group));
        put(t.order, p->wg_order.data(), p->wg_order.size() * 4);
        put(t.u_at, p->u_at.data(), p->u_at.size() * 4);
    }
    if (t.end) HIP_TRY(hipMemcpyAsync(dev_buf, h, t.end, hipMemcpyHostToDevice, st), "dynbatch_plan_upload");
    p->dev_buf = dev_buf;
    p->dev_bytes = bytes;
    return DYNB_OK;
}

extern "C" size_t dynbatch_workspace_bytes(const dynb_plan* p, const dynb_shape* s)
{
    if (!p || !s || s->C <= 0 || s->H <= 0 || s->W <= 0) return 0;
    if (s->dtype != DYNB_F32 && s->dtype != DYNB_BF16) return 0;
    const size_t map = size_t(s->C) * s->H * s->W * elt_bytes(s->dtype);    // slots are packed
    size_t n = size_t(p->n_slots);
    if (!fast_shape(s)) n += dynb_generic_mids(p) + dynb_generic_us(p);
    size_t bytes = align256(n * map);
    if (fast_shape(s)) bytes += align256(packed_weight_bytes(p->n_types));    // weights in MFMA fragment order
    if (fast_shape(s)) bytes += persist_sync_bytes(p);                        // ready flags, ticket counter, status
    if (fast_shape(s)) bytes += dynb_fast_keep_bytes(p);                      // u and mid of every item for the backward pass
    return std::max<size_t>(bytes, 256);
}

// Shapes without a fused kernel.  mid and u live behind the slots: one map each per item of the widest group, or, for the backward
// pass of a DYNB_PLAN_KEEP plan, mid of every item of the plan and u of its two-argument functions.
template <typename T>
static int run_generic(const dynb_plan* p, const dynb_shape* s, const dynb_module_weights* w, const void* feats,
                       void* out, char* ws, hipStream_t st)
{
    const size_t map = size_t(s->C) * s->H * s->W * sizeof(T);
    const char* d = static_cast<const char*>(p->dev_buf);
    ConvArgs a = {};
    a.feats = feats; a.out = out; a.slots = ws;
    a.mid = ws + dynb_generic_mid_offset(p, map);
    T* const u = reinterpret_cast<T*>(static_cast<char*>(a.mid) + dynb_generic_mids(p) * map);
    a.u = u;
    a.C = s->C; a.H = s->H; a.W = s->W;
    const bool timed = dynb::timing_on(), coarse = dynb::timing_coarse();
    if (timed) dynb::timing_mark(st, dynb::ST_SETUP, 0);
    int32_t evals = 0;
    const bool plain = plain_shape<T>(a), whole = !plain && node_shape<T>(a);
    for (const dynb_launch& l : p->launches) {
        evals += l.count;
        if (p->keep) a.u = dynb_u_of_group(u, l, map / sizeof(T));
        // a grid has at most 65535 rows and 2^32 threads a row: very wide launch groups are split
        const int slice = whole ? 1 << 22 : 32768;
        for (int off = 0; off < l.count; off += slice) {
            const int count = std::min(slice, l.count - off);
            const dynb_item* items = reinterpret_cast<const dynb_item*>(d) + l.start + off;
            a.first_kept = p->keep ? l.start + off : off;
            if (whole) {
                const NodeArgs nw = {w->w1, w->b1, w->w3a, w->b3a, w->w3b, w->b3b, count, p->keep ? 1 : 0};
                const int rc = launch_node<T>(items, nw, a, st);
                if (rc != DYNB_OK) return fail(rc, "dynbatch_execute: a launch group could not be launched");
                continue;
            }
            int rc = DYNB_OK;
            // (only the items that may be joins: a launch group's others would each start workgroups that find nothing to do)
            const int lo = std::max(l.bin_lo, l.start + off), hi = std::min(l.bin_hi, l.start + off + count);
            if (lo < hi) {
                ConvArgs j = a;
                j.w = w->w1; j.bias = w->b1;
                j.first_kept += lo - (l.start + off);
                rc = (plain ? launch_conv_plain<T, CV_JOIN> : launch_conv<T, CV_JOIN>)(items + (lo - (l.start + off)), j, hi - lo, st);
            }
            a.w = w->w3a; a.bias = w->b3a;
            if (rc == DYNB_OK) rc = (plain ? launch_conv_plain<T, CV_FIRST> : launch_conv<T, CV_FIRST>)(items, a, count, st);
            a.w = w->w3b; a.bias = w->b3b;
            if (rc == DYNB_OK) rc = (plain ? launch_conv_plain<T, CV_SECOND> : launch_conv<T, CV_SECOND>)(items, a, count, st);
            if (rc != DYNB_OK) return fail(rc, "dynbatch_execute: a convolution could not be launched");
        }
        if (timed && !coarse) dynb::timing_mark(st, int32_t(&l - p->launches.data()), l.count);
    }
    if (coarse) dynb::timing_mark(st, 0, evals);
    HIP_TRY(hipGetLastError(), "dynbatch_execute(convolution kernels)");
    return DYNB_OK;
}

// w1 (2 halves), w3a, w3b (9 taps each) -> fragment order at pk: [w3a | w3b | w1]
static void launch_pack(const dynb_module_weights* w, int n_types, char* pk, hipStream_t st)
{
    const size_t tap_bytes = size_t(n_types) * 128 * 128 * 2;
    PackArgs a = {};
    const void* const src[3] = {w->w3a, w->w3b, w->w1};
    for (int i = 0; i < 3; ++i) {
        a.src[i] = static_cast<const bf16_t*>(src[i]);
        a.dst[i] = reinterpret_cast<u32x4*>(pk + size_t(i) * 9 * tap_bytes);
    }
    a.n_types = n_types;
    const unsigned grid = unsigned(std::min<size_t>(size_t(n_types) * 9, 4096));
    hipLaunchKernelGGL(k_pack_weights, dim3(grid, w->w1 ? 3 : 2), dim3(256), 0, st, a);
}

static int run_mfma(const dynb_plan* p, const dynb_module_weights* w, const void* feats, void* out, char* ws,
                    hipStream_t st)
{
    static std::atomic<uint64_t> attr_set{0};                 // one bit per device
    static int cu_count[64] = {};
    int dev = 0;
    HIP_TRY(hipGetDevice(&dev), "hipGetDevice");
    if (!(attr_set.load() >> (dev & 63) & 1)) {
        int cus = 0;
        HIP_TRY(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev), "hipDeviceGetAttribute");
        cu_count[dev & 63] = cus > 0 ? cus : 256;
        for (const void* f : {reinterpret_cast<const void*>(k_module_persist),
                              reinterpret_cast<const void*>(k_module_mfma<1, false>), reinterpret_cast<const void*>(k_module_mfma<1, true>),
                              reinterpret_cast<const void*>(k_module_mfma<2, false>), reinterpret_cast<const void*>(k_module_mfma<2, true>),
                              reinterpret_cast<const void*>(k_module_mfma<4, false>), reinterpret_cast<const void*>(k_module_mfma<4, true>),
                              reinterpret_cast<const void*>(k_module_mfma<7, false>), reinterpret_cast<const void*>(k_module_mfma<7, true>),
                              reinterpret_cast<const void*>(k_module_mfma<7, false, 2>), reinterpret_cast<const void*>(k_module_mfma<7, true, 2>),
                              reinterpret_cast<const void*>(k_module_mfma<7, false, 4>), reinterpret_cast<const void*>(k_module_mfma<7, true, 4>)})
            HIP_TRY(hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, mf::LDS_BYTES), "hipFuncSetAttribute(module kernels)");
        attr_set.fetch_or(uint64_t(1) << (dev & 63));
    }
    const char* d = static_cast<const char*>(p->dev_buf);
    MfArgs a = {};
    a.feats = static_cast<const bf16_t*>(feats);
    a.out = static_cast<bf16_t*>(out);
    a.slots = reinterpret_cast<bf16_t*>(ws);
    // weights in fragment order: the caller's prepared copy, or a fresh one behind the slots
    // (about 0.6 MB per function)
    const size_t tap_bytes = size_t(p->n_types) * 128 * 128 * 2;
    char* pk = w->packed ? static_cast<char*>(const_cast<void*>(w->packed))
                         : ws + align256(size_t(p->n_slots) * mf::P * mf::C * 2);
    bf16_t* pk3a = reinterpret_cast<bf16_t*>(pk);
    bf16_t* pk3b = reinterpret_cast<bf16_t*>(pk + 9 * tap_bytes);
    bf16_t* pk1 = reinterpret_cast<bf16_t*>(pk + 18 * tap_bytes);
    if (!w->packed) launch_pack(w, p->n_types, pk, st);
    a.w1 = pk1; a.b1 = w->b1;
    a.w3a = pk3a; a.b3a = w->b3a;
    a.w3b = pk3b; a.b3b = w->b3b;
    a.first_item = 0;
    a.n_items = int32_t(p->items.size());
    a.keep = p->keep ? ws + dynb_fast_keep_offset(p) : nullptr;
    const bool timed = dynb::timing_on(), coarse = dynb::timing_coarse();
    if (p->persistent) {
        // one launch for the whole batch: clear the ready flags, the ticket counter and the status word with a
        // fill kernel (no memset node: the call may be captured into a graph), then the resident workgroups
        PersistArgs q;
        q.tickets = reinterpret_cast<const int32_t*>(d + plan_items_bytes(p) + plan_leaf_bytes(p) + plan_arity_bytes(p));
        q.n_tickets = int32_t(p->tickets.size());
        q.spin_limit = g_spin_limit.load();
        q.ready = reinterpret_cast<int32_t*>(ws + persist_sync_offset(p));
        q.counter = q.ready + p->n_slots;
        q.status = q.counter + 1;
        const size_t nsync = size_t(p->n_slots) + 2;
        hipLaunchKernelGGL(k_fill_i32, dim3(unsigned(std::min<size_t>((nsync + 255) / 256, 256))), dim3(256), 0, st, q.ready, nsync, 0);
        if (timed) dynb::timing_mark(st, dynb::ST_SETUP, 0);
        // a plan that also keeps u and mid for the backward pass runs one launch per label (below); its status
        // word stays clear
        if (!p->keep) {
            a.items = reinterpret_cast<const dynb_item*>(d);
            a.count = int32_t(p->items.size());
            const int resident = cu_count[dev & 63];          // one workgroup per CU (78 KB of LDS, all registers)
            const unsigned grid = unsigned(std::min<int>(q.n_tickets, resident));
            hipLaunchKernelGGL(k_module_persist, dim3(grid), dim3(256), mf::LDS_BYTES, st, a, q);
            if (timed) dynb::timing_mark(st, 0, a.count);
            HIP_TRY(hipGetLastError(), "dynbatch_execute(dependency-driven kernel)");
            return DYNB_OK;
        }
    }
    if (timed && !p->persistent) dynb::timing_mark(st, dynb::ST_SETUP, 0);
    int32_t evals = 0;
    for (const dynb_launch& l : p->launches) {
        evals += l.count;
        a.items = reinterpret_cast<const dynb_item*>(d) + l.start;
        a.first_item = l.start;
        a.count = l.count;
        // as many workgroups per node as still fit the chip's 256 CUs in one round; beyond that, and whenever several batches are in
        // flight (their narrow groups share the chip), one node per workgroup
        const int parts = p->throughput ? 1 : parts_for(l.count);
        const unsigned grid = unsigned((parts * l.count + 7) / 8 * 8);
        a.per_xcd = int32_t(grid / 8);
        auto* kernel = parts == 28  ? (p->keep ? k_module_mfma<7, true, 4> : k_module_mfma<7, false, 4>)
                       : parts == 14 ? (p->keep ? k_module_mfma<7, true, 2> : k_module_mfma<7, false, 2>)
                       : parts == 7 ? (p->keep ? k_module_mfma<7, true> : k_module_mfma<7>)
                       : parts == 4 ? (p->keep ? k_module_mfma<4, true> : k_module_mfma<4>)
                       : parts == 2 ? (p->keep ? k_module_mfma<2, true> : k_module_mfma<2>)
                                    : (p->keep ? k_module_mfma<1, true> : k_module_mfma<1>);
        hipLaunchKernelGGL(kernel, dim3(grid), dim3(256), mf::LDS_BYTES, st, a);
        if (timed && !coarse) dynb::timing_mark(st, int32_t(&l - p->launches.data()), l.count);
    }
    if (coarse) dynb::timing_mark(st, 0, evals);
    HIP_TRY(hipGetLastError(), "dynbatch_execute(mfma kernels)");
    return DYNB_OK;
}

extern "C" size_t dynbatch_packed_weights_bytes(const dynb_shape* s, int32_t n_types)
{
    if (!s || n_types <= 0 || !fast_shape(s)) return 0;
    return align256(packed_weight_bytes(n_types));
}

extern "C" int dynbatch_pack_weights(const dynb_shape* s, int32_t n_types, const dynb_module_weights* w, void* packed,
                                     size_t packed_bytes, void* stream)
{
    if (!s || !w || !packed || n_types <= 0) return fail(DYNB_E_INVAL, "dynbatch_pack_weights: NULL argument or n_types <= 0");
    if (!fast_shape(s)) return fail(DYNB_E_UNSUPPORTED, "dynbatch_pack_weights: this shape has no packed layout");
    if (!w->w3a || !w->w3b) return fail(DYNB_E_INVAL, "dynbatch_pack_weights: conv3x3 weights missing");
    if (reinterpret_cast<uintptr_t>(packed) & 255) return fail(DYNB_E_INVAL, "dynbatch_pack_weights: buffer not 256-byte aligned");
    if (packed_bytes < dynbatch_packed_weights_bytes(s, n_types))
        return fail(DYNB_E_WORKSPACE, "dynbatch_pack_weights: buffer too small");
    launch_pack(w, n_types, static_cast<char*>(packed), static_cast<hipStream_t>(stream));
    HIP_TRY(hipGetLastError(), "dynbatch_pack_weights");
    return DYNB_OK;
}

extern "C" int dynbatch_execute(const dynb_plan* p, const dynb_shape* s, const dynb_module_weights* w,
                                const void* feats, void* out, void* workspace, size_t workspace_bytes,
                                void* stream)
{
    if (!p || !s || !w || !feats || !out || !workspace) return fail(DYNB_E_INVAL, "dynbatch_execute: NULL argument");
    if (s->C <= 0 || s->H <= 0 || s->W <= 0) return fail(DYNB_E_INVAL, "dynbatch_execute: C, H, W must be positive");
    if (s->dtype != DYNB_F32 && s->dtype != DYNB_BF16) return fail(DYNB_E_UNSUPPORTED, "dynbatch_execute: unknown dtype");
    if (!w->w3a || !w->w3b) return fail(DYNB_E_INVAL, "dynbatch_execute: conv3x3 weights missing");
    if (p->has_binary && !w->w1) return fail(DYNB_E_UNSUPPORTED, "dynbatch_execute: binary functions need w1");
    if (!p->dev_buf) return fail(DYNB_E_WORKSPACE, "dynbatch_execute: plan not uploaded");
    if (workspace_bytes < dynbatch_workspace_bytes(p, s)) return fail(DYNB_E_WORKSPACE, "dynbatch_execute: workspace too small");
    if (reinterpret_cast<uintptr_t>(workspace) & 255) return fail(DYNB_E_INVAL, "dynbatch_execute: workspace not 256-byte aligned");
    if (size_t(s->C) * s->H * s->W >= (size_t(1) << 31)) return fail(DYNB_E_UNSUPPORTED, "dynbatch_execute: map too large");
    hipStream_t st = static_cast<hipStream_t>(stream);
    char* ws = static_cast<char*>(workspace);

    if (dynb::timing_on()) dynb::timing_begin(st);
    if (!p->leaf_roots.empty()) {
        const size_t words = size_t(s->C) * s->H * s->W * elt_bytes(s->dtype) / 4;
        if ((size_t(s->C) * s->H * s->W * elt_bytes(s->dtype)) % 4) return fail(DYNB_E_UNSUPPORTED, "dynbatch_execute: odd-sized bf16 map");
        const int32_t* ex = reinterpret_cast<const int32_t*>(static_cast<const char*>(p->dev_buf) + plan_items_bytes(p));
        for (size_t off = 0; off < p->leaf_roots.size(); off += 32768) {
            const unsigned n = unsigned(std::min<size_t>(32768, p->leaf_roots.size() - off));
            dim3 grid(unsigned(std::min<size_t>((words + 255) / 256, 64)), n);
            hipLaunchKernelGGL(k_copy_leaf_roots, grid, dim3(256), 0, st, ex + off, int(n),
                               static_cast<const uint32_t*>(feats), static_cast<uint32_t*>(out), words);
        }
    }
    if (p->items.empty()) {
        HIP_TRY(hipGetLastError(), "dynbatch_execute(copy)");
        return DYNB_OK;
    }
    if (fast_shape(s)) return run_mfma(p, w, feats, out, ws, st);
    if (s->dtype == DYNB_BF16) return run_generic<bf16_t>(p, s, w, feats, out, ws, st);
    return run_generic<float>(p, s, w, feats, out, ws, st);
}

extern "C" int dynbatch_execute_check(const dynb_plan* p, const dynb_shape* s, const void* workspace, void* stream)
{
    if (!p || !s || !workspace) return fail(DYNB_E_INVAL, "dynbatch_execute_check: NULL argument");
    if (!p->persistent) return fail(DYNB_E_INVAL, "dynbatch_execute_check: the plan was not made with DYNB_PLAN_PERSISTENT");
    hipStream_t st = static_cast<hipStream_t>(stream);
    HIP_TRY(hipStreamSynchronize(st), "dynbatch_execute_check(synchronize)");
    if (!fast_shape(s) || p->items.empty()) return DYNB_OK;   // those run one launch per label: nothing waits
    int32_t status = 0;
    const char* w = static_cast<const char*>(workspace) + persist_sync_offset(p) + (size_t(p->n_slots) + 1) * sizeof(int32_t);
    HIP_TRY(hipMemcpy(&status, w, sizeof(status), hipMemcpyDeviceToHost), "dynbatch_execute_check(read status)");
    if (status != 0)
        return fail(DYNB_E_HIP, "dynbatch_execute: a workgroup gave up waiting for an argument of its node; the results are invalid");
    return DYNB_OK;
}
