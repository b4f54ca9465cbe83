// MFMA building blocks of the fused module kernels (bf16, C = 128, 14 x 14), shared by the forward executor and the
// backward pass: the LDS halo tile's geometry, the packed weight fragment order and the software-pipelined K loop.
#pragma once

#include <hip/hip_runtime.h>

#include "device_utils.h"

namespace {

namespace mf {
constexpr int C = 128;
constexpr int S = 14;                    // spatial size
constexpr int P = S * S;                 // 196 pixels
constexpr int HALO = 16;                 // tile side with zero border
constexpr int PIX_BYTES = 272;           // 128 channels bf16 + 16 bytes pad: 17 granules of 16 bytes
// A row is 304 granules of 16 bytes apart from the next, a multiple of the banks: pixel (y, x) sits at granule x (mod 16), and the lanes
// that an LDS pass takes from the two image rows of a fragment (four consecutive ones of either, shifted against each other) meet
// distinct banks.  (17 pixels, 289 granules, put the second row one granule further: a conflict in every pass, 0.45 of the LDS
// cycles.  With 304 the counters say 0.014.  The MFMAs above them hide most of it: with zero_border below, which came with it, 1000 programs
// 2127 -> 2110 us, 256 programs 721 -> 716, 23 programs 285 -> 277.)
// Of a row 14 pixels are the map's; the pixel before and all behind are zeros, which is what the two padding columns
// of a pixel tile (below) read, whatever the tap.  (Zeros and not the last pixel again: the chip is at its power limit in
// these kernels, and the matrix pipes take less of it for zeros: builds that run the K loop alone, on all CUs, reach 1.62 instead
// of 1.52 PFLOP/s.)
constexpr int ROW_BYTES = 304 * 16;
static_assert(ROW_BYTES >= (HALO + 1) * PIX_BYTES, "room for the zeros on the right");
constexpr int TILE_BYTES = HALO * ROW_BYTES + PIX_BYTES;   // (the last row's neighbours are zeros of their own)
constexpr int RIM = (S + 1) * PIX_BYTES;                // first byte of a row behind its last pixel
constexpr int TOP_PIECES = (ROW_BYTES + PIX_BYTES) / 16, RIM_PIECES = (ROW_BYTES - RIM + PIX_BYTES) / 16;
constexpr int BIAS_OFF = TILE_BYTES;                    // behind the tile: three vectors of C biases
constexpr int LDS_BYTES = TILE_BYTES + 3 * C * 4;       // 79632: two workgroups per CU
constexpr int CENTER = ROW_BYTES + PIX_BYTES;           // (+1,+1) from the top-left tap
}  // namespace mf

__device__ __forceinline__ bf16x8 lds_read_frag(uint32_t addr)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
    return *reinterpret_cast<const bf16x8*>(lds_raw + addr);
}

// ---- MFMA tiling ------------------------------------------------------------------------------
// v_mfma_f32_32x32x16_bf16 is the efficient bf16 instruction of gfx950 (measured: ~2.1 PFLOP/s chip
// wide, against ~1.5 for the 16x16x32 form), so a convolution is tiled as
//     D[32 channels][32 pixels] += W[32 channels][16 k] * X[16 k][32 pixels]
// with the weights as the A operand and the activations as the B operand: a lane then ends up with
// 16 channels of one pixel (consecutive ones, thanks to the row permutation of the packed weights),
// which it can store as 16-byte pieces.  A pixel tile is two image rows of 14 pixels, each padded to 16 columns (the
// padding columns read zeros and are dropped): 14 rows make 7 tiles, 224 columns for 196 pixels, the same
// as tiles of 32 consecutive pixels would need, but a fragment then depends on its first image row alone: the
// fragment that the upper tap row reads for one tile is the one that the lower tap row reads for the tile above.
// A wave owns one channel tile and all pixel tiles of its node.
//
// K order.  dx (tap column) outermost, then the 128 input channels in 8 steps of 16, then the tap rows in the order 0, 2,
// 1; lane half h = lane/32 supplies channels h*64 + j*8 .. +7 in step j (any pairing works as long as both
// operands agree).  All layouts and both passes keep this order, so results do not depend on the layout.
// Weight fragments.  In the caller's [Cout][kh][kw][Cin] layout one fragment load would touch 64
// different cache lines (32 rows x 2 halves), which makes the vector L1 the bottleneck.  The
// weights are therefore repacked (k_pack_weights) into fragment order, in the order of their use,
//     conv3x3 [function][channel tile 4][dx 3][step 8][tap row 0, 2, 1][lane 64][8 bf16]
//     conv1x1 [function][channel tile 4][argument 2][step 8][lane 64][8 bf16]
// so that the 64 lanes of a fragment load read one contiguous kilobyte.
constexpr int MT7 = 7;

namespace mf {
constexpr int FRAG = 512;   // elements of one packed weight fragment: 64 lanes x 8 bf16 = 1 KB

// tap (kh, kw) and step of fragment f (0 .. 71) of a packed conv3x3
__host__ __device__ constexpr int frag_kw(int f) { return f / 24; }
__host__ __device__ constexpr int frag_step(int f) { return f / 3 % 8; }
__host__ __device__ constexpr int frag_kh(int f) { return f % 3 == 0 ? 0 : f % 3 == 1 ? 2 : 1; }
}

// The three weight tensors that are brought into fragment order, by blockIdx.y: one launch.
struct PackArgs { const bf16_t* src[3]; u32x4* dst[3]; int n_types; };

// LDS byte offset, from the tile's first byte, of what lane `lane` reads for the tile row pair that starts at tile row 0,
// tap column 0: image row lane%32/16, column lane%16 (for columns 14, 15 the zeros from column 15 on), its half of the channels
__device__ __forceinline__ uint32_t pair_lane_addr(int lane)
{
    const int r = lane & 31;
    return uint32_t((r >> 4) * mf::ROW_BYTES + ((r & 15) < mf::S ? r & 15 : mf::S + 1) * mf::PIX_BYTES + (lane >> 5) * 128);
}

// Zeros around the map in tile rows lo .. hi (what a workgroup's first conv reads; all sixteen of them took a part of a node 0.2 us more, 2 to 4 % of
// a narrow level), by threads tid, tid + NTHR, ...: between the last pixel of a row and the first of the next
// (rim r: behind row r), the whole top row and bottom row where they are among them.
template <int NTHR>
__device__ __forceinline__ void zero_border(int tid, int lo, int hi)
{
    using namespace mf;
    extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
    const int top = lo == 0 ? TOP_PIECES : 0, rim0 = lo == 0 ? 1 : lo - 1, rims = ((hi == HALO - 1 ? HALO - 2 : hi) - rim0 + 1) * RIM_PIECES;
    const int all = top + rims + (hi == HALO - 1 ? ROW_BYTES / 16 : 0);
    for (int c = tid; c < all; c += NTHR) {
        const int q = c - top, row = q / RIM_PIECES;
        const int at = q < 0 ? c * 16 : q < rims ? (rim0 + row) * ROW_BYTES + RIM + (q - row * RIM_PIECES) * 16
                                                 : (HALO - 1) * ROW_BYTES + PIX_BYTES + (q - rims) * 16;
        *reinterpret_cast<u32x4*>(lds_raw + uint32_t(at)) = u32x4{0u, 0u, 0u, 0u};
    }
}

// ---- K loop of a conv3x3 ----------------------------------------------------------------------------
// acc[t] += W * X over 9 taps x 8 steps of 16 input channels.  x0: this lane's address for the first row pair of the
// window (pair_lane_addr of the window's first tile row).  Per (dx, step) the wave reads the 2 MTW + 1 fragments whose
// row pairs start at tile rows 0 .. 2 MTW and multiplies each with every tap row that needs it: even ones with tap row 0
// (tile s/2) and tap row 2 (tile s/2 - 1), odd ones with tap row 1.  MTW = 7: 15 LDS reads for 21 MFMAs.
// The loop itself is bound by the matrix pipes: 17.4k clocks per conv3x3 of a lone workgroup with everything hot in L2
// (504 MFMAs per wave are 16.1k; the LDS reads add 0.1k, the weight loads 0.6k), 18.3k in the kernel.  On the whole chip it
// is bound by power, not by any pipe (the clock falls to 1.7-1.9 GHz of 2.4): in such builds register-only MFMAs on random data reach
// 1.70 PFLOP/s, the LDS reads cost 7 % of that and the weight loads 11 %, which is why every fragment is read once per
// use of its rows and once per workgroup.
// Software pipelined by hand:
//   * activation fragments live in XW register sets and are requested XW - 1 fragments ahead, one request before the
//     MFMAs of each fragment;
//   * weight fragments live in a ring of RW register sets (RW/3 steps); the previous step's are refilled from global
//     memory behind the first MFMAs of the current step, RW/3 - 1 steps ahead of their use (issuing the load directly
//     behind the MFMAs that still read the slot would stall the wave);
//   * scheduler fences keep that order (the compiler would otherwise sink every load to its use).
// The ring is filled by ring_fill, a call of its own so that the caller can issue it long before the loop; the
// last chunk refills the ring with the first fragments of the NEXT loop (wnext), which then starts full (NEXT = false: there
// is none, and the requests, which cannot be left out without losing count of the others, are for one fragment).
// Consecutive MFMAs never use the same accumulator (but for MTW = 1, which has one).
template <int RW>
__device__ __forceinline__ void ring_fill(bf16x8 (&wf)[RW], const bf16_t* wrow)
{
#pragma unroll
    for (int j = 0; j < RW - 3; ++j) {
        wf[j] = *reinterpret_cast<const bf16x8*>(wrow + j * mf::FRAG);
        __builtin_amdgcn_sched_barrier(0);
    }
}

template <int MTW, int RW, int XW, bool NEXT = true>
__device__ __forceinline__ void kloop3(f32x16 (&acc)[MTW], const uint32_t x0, bf16x8 (&wf)[RW], const bf16_t* wrow, const bf16_t* wnext)
{
    constexpr int NF = 2 * MTW + 1, STEPS = RW / 3, NCHUNK = 24 / STEPS, G = STEPS * NF;
    static_assert(RW % 3 == 0 && (STEPS == 8 || STEPS == 4) && G % XW == 0, "ring shapes");
    // the row pairs are taken in the order 0, 2, 1, 4, 3, 6, 5, ...: one and two MFMAs per fragment in turn
    auto row_of = [](int k) -> int { return k == 0 ? 0 : (k & 1) ? k + 1 : k - 1; };
    // fragment g of a chunk: byte offset from the chunk's first tap and channel step
    auto at = [&](int g) -> uint32_t {
        return uint32_t(row_of(g % NF) * mf::ROW_BYTES + (g / NF) * 16);
    };
    auto chunk_base = [](int c) -> uint32_t {
        return STEPS == 8 ? uint32_t(c) * mf::PIX_BYTES : uint32_t(c >> 1) * mf::PIX_BYTES + uint32_t(c & 1) * 64;
    };
    bf16x8 x[XW];
#pragma unroll
    for (int g = 0; g < XW - 1; ++g) {
        x[g] = lds_read_frag(x0 + at(g));
        __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll 1
    for (int c = 0; c < NCHUNK; ++c) {
        const bool last = c + 1 >= NCHUNK;
        const uint32_t xa = x0 + chunk_base(c), xn = x0 + chunk_base(last ? c : c + 1);   // after the last chunk: re-read valid data
        const bf16_t* cur = wrow + (c * RW + RW - 3) * mf::FRAG;        // the last step of this chunk
        const bf16_t* nxt = last ? wnext : wrow + (c + 1) * RW * mf::FRAG;   // the next chunk / the next loop
        const int nfrag = !NEXT && last ? 0 : mf::FRAG;                      // (no next loop: one fragment again and again)
#pragma unroll
        for (int st = 0; st < STEPS; ++st) {
#pragma unroll
            for (int k = 0; k < NF; ++k) {
                const int g = st * NF + k, ga = g + XW - 1;
                x[ga % XW] = lds_read_frag(ga >= G ? xn + at(ga - G) : xa + at(ga));
                const int s = row_of(k), t = s / 2;
                auto mul = [&](int tile, int w) { acc[tile] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[st * 3 + w], x[g % XW], acc[tile], 0, 0, 0); };
                if (s & 1) mul(t, 2);                  // tap row 1
                else {
                    if (t > 0) mul(t - 1, 1);          // tap row 2 of the tile above
                    if (t < MTW) mul(t, 0);            // tap row 0
                }
                __builtin_amdgcn_sched_barrier(0);
                constexpr int K0 = NF > 3 ? 1 : 0;
                if (k >= K0 && k < K0 + 3) {           // refill the slots of the previous step
                    wf[(st * 3 + k - K0 + RW - 3) % RW] = *reinterpret_cast<const bf16x8*>(st == 0 ? cur + (k - K0) * mf::FRAG : nxt + ((st - 1) * 3 + k - K0) * nfrag);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        }
    }
}

// ---- conv1x1 over one argument ----------------------------------------------------------------------
// acc[t] += W * X over 8 steps of 16 input channels; xaddr(t): this lane's pixel of tile t (centre of the halo tile, its
// half of the channels).  The 8 weight fragments are the caller's registers; WNEXT: they are replaced by those of the
// next call as they are used.
template <int MTW, bool WNEXT, typename Addr>
__device__ __forceinline__ void kloop1(f32x16 (&acc)[MTW], const Addr& xaddr, bf16x8 (&wf)[8], const bf16_t* wnext)
{
    constexpr int XW = 6, G = 8 * MTW;          // activation fragments: register sets, fragments in all
    bf16x8 x[XW];
    auto at = [&](int g) { return xaddr(g % MTW) + uint32_t(g / MTW * 16); };
#pragma unroll
    for (int g = 0; g < XW - 1; ++g) {
        x[g] = lds_read_frag(at(g));
        __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) {
#pragma unroll
        for (int t = 0; t < MTW; ++t) {
            const int g = j * MTW + t, ga = g + XW - 1;
            if (ga < G) x[ga % XW] = lds_read_frag(at(ga));
            acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[j], x[g % XW], acc[t], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            if (WNEXT && t == 0 && j > 0) wf[j - 1] = *reinterpret_cast<const bf16x8*>(wnext + (j - 1) * mf::FRAG);
        }
    }
    if (WNEXT) wf[7] = *reinterpret_cast<const bf16x8*>(wnext + 7 * mf::FRAG);
}

// ---- ReLU masks ---------------------------------------------------------------------------------------
// What the backward pass wants to know of a result or of mid is which elements are positive.  The forward pass of a DYNB_PLAN_KEEP plan notes it
// in one byte per 16-byte piece (8 channels of a pixel): 6 KB a node that the backward pass reads instead of 100 KB of maps.
constexpr int mask_bit(int e) { return (e >> 1) + 4 * (e & 1); }       // element e's bit
// of a piece behind a ReLU (no half is negative: positive is not zero), in the low eight bits
__device__ __forceinline__ uint32_t positive_mask(const u32x4& v)
{
    typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
    uint32_t r = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) r |= __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_bit_cast(u16x2, uint32_t(v[i])), u16x2{1, 1})) << i;
    return r | r >> 12;
}
// v where bit `bit` of m is set, else 0
__device__ __forceinline__ float masked_by(uint32_t m, int bit, float v)
{
    return __uint_as_float(__float_as_uint(v) & uint32_t(__builtin_amdgcn_sbfe(int(m), bit, 1)));
}

// ---- parts of a node --------------------------------------------------------------------------------
// A node is spread over PARTS workgroups, each with a share of the output rows:
//   PARTS      output rows      rows of the first conv's window (pixel tiles)    of the second's
//     1            14                      14 (7)                                    14 (7)
//     2             7                       8 (4)                                     8 (4)
//     4             4                       6 (3)                                     4 (2)
//     7             2                       4 (2)                                     2 (1)
// (the second conv needs one row of the first conv's output beyond its own rows on either side).  Wave w owns channel
// tile w of all of them.  More parts shorten narrow launch groups at the price of MFMA work (14, 16, 20, 21 tiles a
// node) and of reading the weights once per part: one node takes 14.7 us in 2 parts, of which 7.7 are MFMAs.
// The backward pass has the same geometry: du is the result, dmid what lies between the convs, g (rows of u) what goes in.
template <int PARTS> struct PartShape;        // output rows, pixel tiles of the two convs, rows of u, fragments in the weight ring, activation register sets
template <> struct PartShape<1> { static constexpr int ROWS = 14, MTA = 7, MTB = 7, UROWS = 14, RW = 12, XA = 10, XB = 10; };
template <> struct PartShape<2> { static constexpr int ROWS = 7, MTA = 4, MTB = 4, UROWS = 9, RW = 12, XA = 12, XB = 12; };
template <> struct PartShape<4> { static constexpr int ROWS = 4, MTA = 3, MTB = 2, UROWS = 8, RW = 24, XA = 8, XB = 8; };
template <> struct PartShape<7> { static constexpr int ROWS = 2, MTA = 2, MTB = 1, UROWS = 6, RW = 24, XA = 8, XB = 8; };

// Workgroups per node of a launch group of `count` nodes: as many as still fit the chip's 256 CUs in one round.  14 and 28: 7 parts whose
// second conv is shared by 2 or 4 workgroups, 64 or 32 output channels each (SPLIT): what a part waits for are weights, 295 KB a conv at some
// 30 bytes a clock, and of the second conv each then reads a half or a quarter.  (The first conv's channels are all needed by every
// one.)  us a pass, 7 parts / shared: one program 193 / 170, three 230 / 205; 5 training programs 660 / 631.  (Requesting the first conv's weights
// into the die's L2 while the argument is on its way, a share per workgroup: 3-5 % slower.)
inline int parts_for(int count) { return count > 128 ? 1 : count > 64 ? 2 : count > 36 ? 4 : count > 18 ? 7 : count > 9 ? 14 : 28; }

}  // namespace
