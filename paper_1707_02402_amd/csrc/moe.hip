// Sparsely gated mixture-of-experts layer with the paper's degenerate one-level batching
// (Results / Sparsely Gated Mixture of Experts): the k*b expert uses known after gating are
// grouped by expert so that each of the n experts is called once on its stacked rows.
//
// Stages (all on the caller's stream, no host synchronisation):
//   gate      logits = x Wg^T + noise * softplus(x Wn^T)                 MFMA, fp32 accumulate
//   top-k     k largest per token (ties -> lower expert), softmax        one wave per token
//   group     stable counting sort of the T*k uses by expert             rank-by-prefix-sum, no
//                                                                        order-dependent atomics
//   permute   xs[inv[t*k+j]] = x[t]  (= xs[pos] = x[perm[pos] / k])       HBM-bound scatter
//   experts   hid = ReLU(xs W1_e^T), y = hid W2_e^T per group             grouped MFMA GEMM, ragged
//                                                                        and empty groups allowed
//   combine   out[t] = sum_j w[t][j] * y[inv[t*k+j]]                      HBM-bound, fixed order
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <initializer_list>
#include <type_traits>
#include <mutex>
#include <string>
#include <vector>

#include "device_utils.h"
#include "moe_deal.h"
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

constexpr int SORT_BLOCK = 256;   // uses ranked together by one workgroup
constexpr int TM = 64;            // rows of one grouped-GEMM tile
constexpr int XR = 256, XF = 256; // rows and features of a whole tile of k_grouped_stream
constexpr int XM = 128;           // most rows of its other kind
constexpr int TN = 256;           // output features of one grouped-GEMM tile
constexpr int NTW = TN / 64;      // 16-feature sub-tiles per wave (4 waves split the features)
constexpr int MAX_K = 8;          // uses of a token whose places are kept in registers (more are looked up)
constexpr int MG = 8;             // row tiles of one expert that walk the feature tiles together
constexpr int XCD_CHUNK = 128;    // most consecutive grouped-GEMM tiles dealt to one XCD
constexpr uint32_t XCD_CUS = 32;
struct alignas(16) RowTile { int32_t expert, row0, rows, alone; };   // alone: k_grouped_stream's, no other tile has this expert

__device__ __forceinline__ bf16x8 ldg_frag(const bf16_t* p) { return *reinterpret_cast<const bf16x8*>(p); }

// ------------------------------------------------------------------------------------------ rows on their way into LDS
// A unit: 64 rows x 64 channels of a matrix, copied without registers on the way.  Eight neighbouring lanes copy 128 bytes of a row, in their order (in any other a
// request is answered lane by lane, 13.5 bytes a clock instead of 64); a unit is eight blocks of 8 rows.  What an LDS pass of a fragment's read takes
// together, 16 of its 32 rows (lanes 0-3, 12-15, 20-23, 24-27 or the others), are two rows of every block, an even and an odd one, and the blocks are 16 bytes
// further apart than their size: all banks.
constexpr int XBLOCK = 1040, XUNIT = 8 * XBLOCK;
// the row of its fragment (lane / 32) that lane `lane` copies into block `block`
__device__ __forceinline__ int copied_row(int block, int lane)
{
    const int odd = lane >> 3 & 1, g = lane >> 4 & 1;
    return (block >> 1) * 8 + (g ^ (block >> 1 & 1) ^ (block >> 2 & 1)) * 4 + (block & 1) * 2 + odd;
}
// where in a unit lane q + 32 hk reads row q of the first fragment (the second lies 512 bytes further), its half of K-step 0 (each next one 32 bytes further)
__device__ __forceinline__ uint32_t fragment_at(int q, int hk)
{
    return uint32_t(((q >> 3) * 2 + (q >> 1 & 1)) * XBLOCK + (((q >> 2 ^ q >> 3 ^ q >> 4) & 1) * 2 + (q & 1)) * 128 + hk * 16);
}
template <bool ONCE = false>                                   // ONCE: nobody else wants these bytes, they need not stay in any cache
__device__ __forceinline__ void lds_copy16(const char* base, uint32_t off, uint32_t lds_at)   // 64 lanes x 16 bytes -> LDS at lds_at, lane after lane
{
    extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
    asm volatile("" : "+s"(base), "+v"(off));                                      // (a scalar base and a lane's offset, and no address of 64 bits per lane kept for every request)
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) uint32_t*)(base + off),
                                     (__attribute__((address_space(3))) uint32_t*)(lds_raw + lds_at), 16, 0, ONCE ? 2 : 0);
}
// *p by the scalar unit: the address is the same for the whole wave, and nobody writes there during the kernel
__device__ __forceinline__ int32_t uniform_load(const int32_t* p)
{
    return __builtin_amdgcn_readfirstlane(*(const __attribute__((address_space(4))) int32_t*)(p));
}
// All but this wave's newest N requests and stores have been answered
template <int N> __device__ __forceinline__ void answered_but() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }
// (Not __syncthreads, which waits for all requests into LDS)
__device__ __forceinline__ void meet() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// ------------------------------------------------------------------------------------------ gate
// Workgroup tile: 64 tokens x 64 experts, both gate matrices at once.  Operands are staged through
// LDS in K-chunks of 64 with coalesced 128-byte row reads (see the grouped GEMM below for why), the
// next chunk is prefetched into registers.  A wave owns a 32-token x 32-expert quarter of the tile
// for both matrices (clean and noise accumulators), multiplied with 32x32x16 MFMAs.
constexpr int GKC = 64;                // K-chunk
constexpr int GLDP = GKC + 8;          // LDS row pitch in elements (144 bytes, conflict free)

// softplus(z) = max(z, 0) + log(1 + u), u = exp(-|z|) in (0, 1], from the hardware's exp2 and log2 (good to about
// 1e-7).  w = 1 + u is rounded; c = u - (w - 1) is exactly what the rounding dropped (w - 1 and the difference are
// exact for w in [1, 2]), and log(1 + u) = log(w) + c / w, where leaving out the division costs less than 2^-25: small
// u keep their relative accuracy without a second code path (u < 2^-24 gives w = 1, log(w) = 0, c = u).
__device__ __forceinline__ float softplus_f(float z)
{
    const float u = __builtin_amdgcn_exp2f(-1.4426950408889634f * fabsf(z));
    const float w = 1.f + u;
    const float c = u - (w - 1.f);
    return fmaxf(z, 0.f) + fmaf(0.6931471805599453f, __builtin_amdgcn_logf(w), c);
}

// clear (if not null): a counter that the next launch wants at zero
__global__ __launch_bounds__(256) void k_gate(const bf16_t* __restrict__ x, const bf16_t* __restrict__ Wg,
                                              const bf16_t* __restrict__ Wn, const float* __restrict__ noise,
                                              float* __restrict__ logits, int T, int d, int E, int32_t* __restrict__ clear)
{
    if (clear && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) *clear = 0;
    __shared__ __attribute__((aligned(16))) bf16_t Ws[128 * GLDP];   // rows 0..63 Wg, 64..127 Wn
    __shared__ __attribute__((aligned(16))) bf16_t Xs[64 * GLDP];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int t0 = blockIdx.y * 64, e0 = blockIdx.x * 64;
    const int part = tid & 7, srow = tid >> 3;          // staging: 32 rows x 8 pieces of 16 bytes per pass
    const bf16_t* wsrc[4];
    const bf16_t* xsrc[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const size_t row = size_t(min(e0 + srow + i * 32, E - 1)) * d + part * 8;
        wsrc[i] = Wg + row;
        wsrc[2 + i] = (noise ? Wn : Wg) + row;
        xsrc[i] = x + size_t(min(t0 + srow + i * 32, T - 1)) * d + part * 8;
    }
    u32x4 wreg[4], xreg[2];
    auto fetch = [&](int kc) {
        const bool inside = kc * GKC + part * 8 < d;
#pragma unroll
        for (int i = 0; i < 4; ++i)
            wreg[i] = inside ? *reinterpret_cast<const u32x4*>(wsrc[i] + kc * GKC) : u32x4{0u, 0u, 0u, 0u};
#pragma unroll
        for (int i = 0; i < 2; ++i)
            xreg[i] = inside ? *reinterpret_cast<const u32x4*>(xsrc[i] + kc * GKC) : u32x4{0u, 0u, 0u, 0u};
    };
    // 4 waves = 2 token halves x 2 expert halves; each wave one 32 x 32 tile per gate matrix (32x32x16 MFMAs)
    const int q = lane & 31, hk = lane >> 5, th = wave & 1, eh = wave >> 1;
    f32x16 ag, an;
#pragma unroll
    for (int i = 0; i < 16; ++i) { ag[i] = 0.f; an[i] = 0.f; }
    const int nchunk = (d + GKC - 1) / GKC;
    fetch(0);
    // lane holds expert e0 + eh*32 + q, tokens t0 + th*32 + 8*(i/4) + 4*hk + i%4 in element i.  Its noise values are requested here: behind the
    // sums, each between the branches around its store, they were sixteen trips to memory in a row (15943 tokens, 359 experts: 21.4 -> 17.9 us).
    const int e = e0 + eh * 32 + q;
    auto token = [&](int i) { return t0 + th * 32 + 8 * (i / 4) + 4 * hk + (i % 4); };
    float nz[16];
    if (noise) {
#pragma unroll
        for (int i = 0; i < 16; ++i) nz[i] = noise[size_t(min(token(i), T - 1)) * E + min(e, E - 1)];
    }
    for (int kc = 0; kc < nchunk; ++kc) {
#pragma unroll
        for (int i = 0; i < 4; ++i) *reinterpret_cast<u32x4*>(Ws + (srow + i * 32) * GLDP + part * 8) = wreg[i];
#pragma unroll
        for (int i = 0; i < 2; ++i) *reinterpret_cast<u32x4*>(Xs + (srow + i * 32) * GLDP + part * 8) = xreg[i];
        __syncthreads();
        if (kc + 1 < nchunk) fetch(kc + 1);
#pragma unroll
        for (int ks = 0; ks < GKC / 16; ++ks) {
            const bf16x8 xf = *reinterpret_cast<const bf16x8*>(Xs + (th * 32 + q) * GLDP + ks * 16 + hk * 8);
            const bf16x8 gf = *reinterpret_cast<const bf16x8*>(Ws + (eh * 32 + q) * GLDP + ks * 16 + hk * 8);
            ag = __builtin_amdgcn_mfma_f32_32x32x16_bf16(xf, gf, ag, 0, 0, 0);
            if (noise) {
                const bf16x8 nf = *reinterpret_cast<const bf16x8*>(Ws + (64 + eh * 32 + q) * GLDP + ks * 16 + hk * 8);
                an = __builtin_amdgcn_mfma_f32_32x32x16_bf16(xf, nf, an, 0, 0, 0);
            }
        }
        __syncthreads();
    }
    if (e >= E) return;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        float v = ag[i];
        if (noise) v += nz[i] * softplus_f(an[i]);
        if (token(i) < T) logits[size_t(token(i)) * E + e] = v;
    }
}

// The same tiles where d is a multiple of 64: the K-chunks go straight into LDS, two ahead, with one barrier each, instead of one ahead by way of registers
// with two.  (What k_gate waits for are d / 64 trips to memory, one after the other.)  The sums are k_gate's bit for bit.
constexpr int GS_BUFS = 3, GS_LDS = GS_BUFS * 3 * XUNIT;     // x rows, Wg rows, Wn rows of three chunks: two workgroups a CU

template <bool NOISY>
__global__ __launch_bounds__(256, 2) void k_gate_stream(const bf16_t* __restrict__ x, const bf16_t* __restrict__ Wg, const bf16_t* __restrict__ Wn,
                                                        const float* __restrict__ noise, float* __restrict__ logits, int T, int d, int E, int32_t* __restrict__ clear)
{
    if (clear && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) *clear = 0;
    extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
    constexpr int UNITS = NOISY ? 3 : 2, PIECES = 2 * UNITS;
    constexpr uint32_t BUF = uint32_t(UNITS * XUNIT);
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, q = lane & 31, hk = lane >> 5;
    const int t0 = blockIdx.y * 64, e0 = blockIdx.x * 64, th = wave & 1, eh = wave >> 1;
    // wave w copies blocks 2 w and 2 w + 1 of every unit
    uint32_t x_off[2], w_off[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int row = (lane >> 5) * 32 + copied_row(2 * wave + i, lane);
        x_off[i] = (uint32_t(min(t0 + row, T - 1) - t0) * uint32_t(d) + uint32_t(lane & 7) * 8u) * 2u;
        w_off[i] = (uint32_t(min(e0 + row, E - 1) - e0) * uint32_t(d) + uint32_t(lane & 7) * 8u) * 2u;
    }
    const char* x_next = reinterpret_cast<const char*>(x + size_t(t0) * d);
    const char* g_next = reinterpret_cast<const char*>(Wg + size_t(e0) * d);
    const char* n_next = reinterpret_cast<const char*>((NOISY ? Wn : Wg) + size_t(e0) * d);
    uint32_t fill = 0, take = 0;
    auto request = [&]() {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const uint32_t at = fill + uint32_t((2 * wave + i) * XBLOCK);
            lds_copy16(x_next, x_off[i], at);
            lds_copy16(g_next, w_off[i], at + XUNIT);
            if (NOISY) lds_copy16(n_next, w_off[i], at + 2 * XUNIT);
        }
        x_next += 128;
        g_next += 128;
        n_next += 128;
        fill = fill == (GS_BUFS - 1) * BUF ? 0 : fill + BUF;
    };
    const int nchunk = d / 64;
    // the noise values first (k_gate): they are there when the first chunk is
    const int e = e0 + eh * 32 + q;
    auto token = [&](int i) { return t0 + th * 32 + 8 * (i / 4) + 4 * hk + (i % 4); };
    float nz[16];
    if (NOISY) {
#pragma unroll
        for (int i = 0; i < 16; ++i) nz[i] = noise[size_t(min(token(i), T - 1)) * E + min(e, E - 1)];
        __builtin_amdgcn_sched_barrier(0);
    }
    request();
    if (nchunk > 1) request();
    f32x16 ag, an;
#pragma unroll
    for (int i = 0; i < 16; ++i) { ag[i] = 0.f; an[i] = 0.f; }
    const uint32_t slot = fragment_at(q, hk);
#pragma unroll 1
    for (int c = 0; c < nchunk; ++c) {
        if (c + 1 < nchunk) answered_but<PIECES>();
        else answered_but<0>();
        meet();
        if (c + 2 < nchunk) request();                         // (into the place of chunk c - 1, which all waves are done with)
        const uint32_t xf = take + uint32_t(th * 512) + slot, wf = take + XUNIT + uint32_t(eh * 512) + slot;
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            const bf16x8 fx = *reinterpret_cast<const bf16x8*>(lds_raw + xf + ks * 32);
            ag = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fx, *reinterpret_cast<const bf16x8*>(lds_raw + wf + ks * 32), ag, 0, 0, 0);
            if (NOISY) an = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fx, *reinterpret_cast<const bf16x8*>(lds_raw + wf + XUNIT + ks * 32), an, 0, 0, 0);
        }
        take = take == (GS_BUFS - 1) * BUF ? 0 : take + BUF;
    }
    if (e >= E) return;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        float v = ag[i];
        if (NOISY) v += nz[i] * softplus_f(an[i]);
        if (token(i) < T) logits[size_t(token(i)) * E + e] = v;
    }
}

// The same product for a few tokens: a workgroup owns 16 tokens x 16 experts, both matrices, and its four waves split the
// sum, so that a handful of tokens still gives a workgroup to many CUs and every wave has all it needs in flight at once
// (37 tokens, d = 512, 256 experts: 4 workgroups of k_gate and 8 K-chunks one after the other, 7.4 us, against 48
// workgroups that wait for memory once).  Fragments come straight from global memory.
constexpr int GS_UN = 4;               // K-steps of 32 requested together

__global__ __launch_bounds__(256) void k_gate_small(const bf16_t* __restrict__ x, const bf16_t* __restrict__ Wg,
                                                    const bf16_t* __restrict__ Wn, const float* __restrict__ noise,
                                                    float* __restrict__ logits, int T, int d, int E, int32_t* __restrict__ clear)
{
    if (clear && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) *clear = 0;
    __shared__ f32x4 part[4][2][64];
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, r = lane & 15, g = lane >> 4;
    const int t0 = blockIdx.y * 16, e0 = blockIdx.x * 16;
    const bf16_t* const px = x + size_t(min(t0 + r, T - 1)) * d;
    const bf16_t* const pg = Wg + size_t(min(e0 + r, E - 1)) * d;
    const bf16_t* const pn = (noise ? Wn : Wg) + size_t(min(e0 + r, E - 1)) * d;
    const int S = (d + 31) / 32, s1 = S * (wave + 1) / 4;
    f32x4 ag = {0.f, 0.f, 0.f, 0.f}, an = {0.f, 0.f, 0.f, 0.f};
    for (int s = S * wave / 4; s < s1; s += GS_UN) {
        u32x4 vx[GS_UN], vg[GS_UN], vn[GS_UN];
#pragma unroll
        for (int u = 0; u < GS_UN; ++u) {
            const int k = (s + u) * 32 + g * 8;
            const bool in = s + u < s1 && k < d;              // d is a multiple of 8; outside: anything, replaced by zeros
            const int at = in ? k : 0;
            const uint32_t m = in ? ~0u : 0u;
            vx[u] = *reinterpret_cast<const u32x4*>(px + at) & m;
            vg[u] = *reinterpret_cast<const u32x4*>(pg + at) & m;
            if (noise) vn[u] = *reinterpret_cast<const u32x4*>(pn + at) & m;
        }
#pragma unroll
        for (int u = 0; u < GS_UN; ++u) {
            const bf16x8 fx = __builtin_bit_cast(bf16x8, vx[u]);
            ag = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fx, __builtin_bit_cast(bf16x8, vg[u]), ag, 0, 0, 0);
            if (noise) an = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fx, __builtin_bit_cast(bf16x8, vn[u]), an, 0, 0, 0);
        }
    }
    part[wave][0][lane] = ag;
    part[wave][1][lane] = an;
    __syncthreads();
    // thread: expert e0 + r, token t0 + 4 g + wave (element `wave` of the lane's accumulators)
    const int e = e0 + r, t = t0 + 4 * g + wave;
    if (e >= E || t >= T) return;
    float v = 0.f, z = 0.f;
#pragma unroll
    for (int w = 0; w < 4; ++w) { v += part[w][0][lane][wave]; z += part[w][1][lane][wave]; }
    if (noise) v += noise[size_t(t) * E + e] * softplus_f(z);
    logits[size_t(t) * E + e] = v;
}

// The same product for wide gates: a workgroup owns a CU and a tile of 256 tokens x 128 experts, both gate matrices
// at once.  A 64 x 64 tile takes in 24 KB per K-chunk for 8 MFMAs per wave (96 B per MFMA clock), three times what
// a CU receives from L2; this tile takes in 64 KB for 64 MFMAs per wave (32 B per MFMA clock).  Operands go through LDS in K-chunks of 64, double buffered, one barrier per chunk.  A wave owns 128
// tokens x 64 experts of both matrices: 16 accumulator tiles.  It is alone on its SIMD, so nothing but its own
// instruction order hides latency: every request is issued between two MFMA groups - an LDS fragment of the next
// K-step; a 16-byte piece of chunk c+1 going from its register to the other LDS buffer, and the piece of chunk c+2
// that takes its place; during the last four chunks half of the epilogue's noise values.  Tiles that share token
// rows are given to one die: its L2 keeps the rows, and the gate matrices too.  Whole tiles only: E a multiple of
// 128, d of 64 and at least 256; the tokens behind the last whole tile of 256, and every other shape, go to k_gate.
constexpr int GB_TOK = 256, GB_EXP = 128;
constexpr int GB_BUF = (GB_TOK + 2 * GB_EXP) * GLDP;       // elements of one LDS buffer: x rows, Wg rows, Wn rows
constexpr int GB_LDS_BYTES = 2 * GB_BUF * 2;

template <bool NOISY>
__global__ __launch_bounds__(256, 1) void k_gate_big(const bf16_t* __restrict__ x, const bf16_t* __restrict__ Wg,
                                                     const bf16_t* __restrict__ Wn, const float* __restrict__ noise,
                                                     float* __restrict__ logits, int T, int d, int E, int n_tok_tiles, int n_exp_tiles,
                                                     int tok_tiles_per_die)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char gb_lds[];
    const int die = blockIdx.x & 7, j = blockIdx.x >> 3;
    const int tok_tile = die * tok_tiles_per_die + j / n_exp_tiles, exp_tile = j % n_exp_tiles;
    if (j / n_exp_tiles >= tok_tiles_per_die || tok_tile >= n_tok_tiles) return;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int t0 = tok_tile * GB_TOK, e0 = exp_tile * GB_EXP;
    const int part = tid & 7, srow = tid >> 3;          // staging: 32 rows x 8 pieces of 16 bytes per pass
    constexpr int NP = NOISY ? 16 : 12;                 // pieces of a chunk per thread: 8 of x, 4 of Wg, 4 of Wn
    constexpr int NF = NOISY ? 8 : 6;                   // fragments of a K-step: 4 token tiles, 2 (+2) expert tiles
    const int q = lane & 31, hk = lane >> 5, th = wave & 1, eh = wave >> 1;   // 2 token halves x 2 expert halves
    bf16_t* const lds = reinterpret_cast<bf16_t*>(gb_lds);

    // piece i of a chunk: 16 bytes of row srow + 32 i of the x tile (i < 8), of the Wg tile (i < 12), of the Wn tile;
    // 32-bit offsets from the tiles' corners, one register for all of them (a tile spans 256 d < 2^31 elements)
    const bf16_t* const x_tile = x + size_t(t0) * d;
    const bf16_t* const wg_tile = Wg + size_t(e0) * d;
    const bf16_t* const wn_tile = NOISY ? Wn + size_t(e0) * d : nullptr;
    // (byte offsets: a uniform base plus a 32-bit lane offset is an addressing mode of the loads and stores)
    const unsigned row_bytes = unsigned(d) * 2u, lane_off = unsigned(srow) * row_bytes + unsigned(part * 16);
    u32x4 stage[NP];                                    // a chunk on its way to LDS
    auto fetch_piece = [&](int i, int kc) {
        const char* src = reinterpret_cast<const char*>(i < 8 ? x_tile : i < 12 ? wg_tile : wn_tile);
        const unsigned row32 = unsigned(i < 8 ? i : (i - 8) & 3) * 32u;
        stage[i] = *reinterpret_cast<const u32x4*>(src + (lane_off + row32 * row_bytes + unsigned(kc * GKC * 2)));
    };
    auto store_piece = [&](int i, bf16_t* buf) {        // piece i covers rows srow + 32 i of the buffer's 512
        *reinterpret_cast<u32x4*>(buf + (srow + i * 32) * GLDP + part * 8) = stage[i];
    };
    // element i of accumulator tile n = 4 b + a (expert column b, token tile a) belongs to expert e0 + eh*64 + b*32
    // + q and token t0 + th*128 + a*32 + 4*hk + 8*(i/4) + i%4; its place in the tile of logits (and of noise values)
    // is a 32-bit byte offset from the tile's corner
    const unsigned uE = unsigned(E) * 4u;                 // bytes of a row of logits
    const unsigned lane_at = unsigned(th * 128 + 4 * hk) * uE + unsigned(eh * 64 + q) * 4u;
    auto at = [&](int n, int i) { return lane_at + unsigned((n & 3) * 32 + 8 * (i / 4) + (i % 4)) * uE + unsigned((n >> 2) * 128); };
    const char* const noise_tile = NOISY ? reinterpret_cast<const char*>(noise + size_t(t0) * E + e0) : nullptr;
    float nz[NOISY ? 8 : 1][16];                          // noise values, 16 per accumulator tile

    f32x16 ag[4][2], an[NOISY ? 4 : 1][2];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int i = 0; i < 16; ++i) { ag[a][b][i] = 0.f; if (NOISY) an[NOISY ? a : 0][b][i] = 0.f; }

    // one chunk: 4 K-steps of 8 MFMA groups (a token tile x an expert tile, both matrices); `side(g)` issues what
    // else has to be requested before group g, g = 0..31
    auto chunk = [&](const bf16_t* buf, auto&& side) {
        const bf16_t* Xs = buf;
        const bf16_t* Ws = buf + GB_TOK * GLDP;          // rows 0..127 Wg, 128..255 Wn
        auto read_frag = [&](int r, int ks) -> bf16x8 {
            const bf16_t* row = r < 4   ? Xs + (th * 128 + r * 32 + q) * GLDP
                                : r < 6 ? Ws + (eh * 64 + (r - 4) * 32 + q) * GLDP
                                        : Ws + (GB_EXP + eh * 64 + (r - 6) * 32 + q) * GLDP;
            return *reinterpret_cast<const bf16x8*>(row + ks * 16 + hk * 8);
        };
        bf16x8 fr[2][NF];
#pragma unroll
        for (int r = 0; r < NF; ++r) fr[0][r] = read_frag(r, 0);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int ks = 0; ks < GKC / 16; ++ks) {
#pragma unroll
            for (int g = 0; g < 8; ++g) {
                const int a = g >> 1, b = g & 1;
                if (ks + 1 < GKC / 16 && g < NF) fr[(ks + 1) & 1][g] = read_frag(g, ks + 1);
                side(ks * 8 + g);
                __builtin_amdgcn_sched_barrier(0);
                ag[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[ks & 1][a], fr[ks & 1][4 + b], ag[a][b], 0, 0, 0);
                if (NOISY)
                    an[NOISY ? a : 0][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[ks & 1][a], fr[ks & 1][NOISY ? 6 + b : 0],
                                                                                  an[NOISY ? a : 0][b], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };

    const int nchunk = d / GKC;
#pragma unroll
    for (int i = 0; i < NP; ++i) fetch_piece(i, 0);
#pragma unroll
    for (int i = 0; i < NP; ++i) {
        store_piece(i, lds);
        fetch_piece(i, min(1, nchunk - 1));
    }
    __syncthreads();
    // chunk kc multiplies out of buffer kc & 1 while chunk kc+1 moves from the registers to the other buffer (all
    // waves left that buffer before the last barrier) and chunk kc+2 is requested into the registers; past the end
    // the requests repeat the last chunk, which nobody reads.  The last four chunks also request the noise values
    // of accumulator tiles 0..3, one tile each: every workgroup of the launch reaches its epilogue at about the
    // same time, and what they all ask of HBM then is what bounds the epilogue.
    auto steady = [&](int kc, auto&& also) {
        bf16_t* other = lds + ((kc + 1) & 1) * GB_BUF;
        const int k2 = min(kc + 2, nchunk - 1);
        chunk(lds + (kc & 1) * GB_BUF, [&](int g) {
            if ((g >> 1) < NP) {
                if ((g & 1) == 0) store_piece(g >> 1, other);
                else fetch_piece(g >> 1, k2);
            }
            also(g);
        });
        __syncthreads();
    };
    auto noise_of = [&](auto n) {                     // tile n's 16 values, in the even groups
        return [&, n](int g) {
            if (NOISY && (g & 1) == 0) nz[NOISY ? decltype(n)::value : 0][g >> 1] = *reinterpret_cast<const float*>(noise_tile + at(decltype(n)::value, g >> 1));
        };
    };
    for (int kc = 0; kc + 4 < nchunk; ++kc) steady(kc, [](int) {});
    steady(nchunk - 4, noise_of(std::integral_constant<int, 0>{}));
    steady(nchunk - 3, noise_of(std::integral_constant<int, 1>{}));
    steady(nchunk - 2, noise_of(std::integral_constant<int, 2>{}));
    chunk(lds + ((nchunk - 1) & 1) * GB_BUF, noise_of(std::integral_constant<int, 3>{}));

    // the noise values of tile n+4 are requested before tile n is worked on
    char* const tile = reinterpret_cast<char*>(logits + size_t(t0) * E + e0);
#pragma unroll
    for (int n = 0; n < 8; ++n) {
        const int a = n & 3, b = n >> 2;
        if (NOISY && n + 4 < 8) {
#pragma unroll
            for (int i = 0; i < 16; ++i) nz[NOISY ? n + 4 : 0][i] = *reinterpret_cast<const float*>(noise_tile + at(n + 4, i));
            __builtin_amdgcn_sched_barrier(0);
        }
        // a wave alone on its SIMD waits out every dependent instruction, so the softplus of 8 elements advances
        // stage by stage
#pragma unroll
        for (int i0 = 0; i0 < 16; i0 += 8) {
            float v[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] = ag[a][b][i0 + i];
            if (NOISY) {
                float z[8], u[8], w[8], c[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) z[i] = an[NOISY ? a : 0][b][i0 + i];
#pragma unroll
                for (int i = 0; i < 8; ++i) u[i] = __builtin_amdgcn_exp2f(-1.4426950408889634f * fabsf(z[i]));
#pragma unroll
                for (int i = 0; i < 8; ++i) w[i] = 1.f + u[i];
#pragma unroll
                for (int i = 0; i < 8; ++i) c[i] = u[i] - (w[i] - 1.f);
#pragma unroll
                for (int i = 0; i < 8; ++i) w[i] = __builtin_amdgcn_logf(w[i]);
#pragma unroll
                for (int i = 0; i < 8; ++i) c[i] = __builtin_amdgcn_fmed3f(z[i], 0.f, INFINITY) + fmaf(0.6931471805599453f, w[i], c[i]);
#pragma unroll
                for (int i = 0; i < 8; ++i) v[i] = fmaf(nz[NOISY ? n : 0][i0 + i], c[i], v[i]);
            }
#pragma unroll
            for (int i = 0; i < 8; ++i) *reinterpret_cast<float*>(tile + at(n, i0 + i)) = v[i];
        }
        __builtin_amdgcn_sched_barrier(0);
    }
}

// ------------------------------------------------------------------------------------------ top-k
// One wave per token. Selection compares fp32 logits exactly: larger first, equal -> lower id.
// The row is read once into registers (lane l holds experts l, l+64, ...; up to NV*64 experts) and the
// k selection rounds run on registers with a wave-wide argmax; NV = 0 re-reads the row every round
// (any E).  Selections come out in strictly descending (value, then ascending id) order, so "already
// taken" is simply "not below the previous selection": no list of chosen ids is kept and k may be
// anything up to E.  A NaN logit counts as -inf.
template <int NV>
__global__ __launch_bounds__(256) void k_topk(const float* __restrict__ logits, int32_t* __restrict__ topk_idx,
                                              float* __restrict__ topk_w, int T, int E, int k)
{
    const int lane = threadIdx.x & 63;
    const int t = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (t >= T) return;
    const float* row = logits + size_t(t) * E;
    auto clean = [](float v) -> float { return v != v ? -INFINITY : v; };
    float reg[NV > 0 ? NV : 1];
    if (NV > 0) {
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int e = lane + 64 * i;
            reg[i] = e < E ? clean(row[e]) : 0.f;
        }
    }
    constexpr int NONE = 0x7fffffff;
    float last_v = INFINITY, v0 = 0.f, den = 0.f;
    int last_e = -1;
    int32_t* idx_t = topk_idx + size_t(t) * k;
    float* w_t = topk_w + size_t(t) * k;
    for (int j = 0; j < k; ++j) {
        float bv = -INFINITY;
        int bi = NONE;
        auto offer = [&](float v, int e) {
            const bool open = v < last_v || (v == last_v && e > last_e);       // below the previous selection
            if (open && (v > bv || bi == NONE)) { bv = v; bi = e; }
        };
        if (NV > 0) {
#pragma unroll
            for (int i = 0; i < NV; ++i)
                if (lane + 64 * i < E) offer(reg[i], lane + 64 * i);
        } else {
            for (int e = lane; e < E; e += 64) offer(clean(row[e]), e);
        }
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) {
            const float ov = __shfl_xor(bv, off);
            const int oi = __shfl_xor(bi, off);
            if (oi != NONE && (bi == NONE || ov > bv || (ov == bv && oi < bi))) { bv = ov; bi = oi; }
        }
        // k <= E: a candidate always exists.  The selection is uniform over the wave.
        last_v = bv;
        last_e = bi;
        if (j == 0) v0 = bv;
        den += expf(bv - v0);
        if ((j & 63) == lane) { idx_t[j] = bi; w_t[j] = bv; }                  // raw logit until den is complete
    }
    for (int j = lane; j < k; j += 64) w_t[j] = expf(w_t[j] - v0) / den;       // each lane revisits its own stores
}

// The same selection for k <= MAX_K with the row in registers, as integer keys whose order is the logits' order
// (-0 is read as +0, NaN as -infinity, like above).  A round finds the largest key of the wave (per lane, then
// across lanes with data-parallel-primitive moves: inside rows of 16, then two row broadcasts to lane 63), and then
// its owner: the registers are asked in turn which lanes hold that key; the registers go up through the expert ids
// in groups of 256, so the first group with an answer holds the lowest expert id, the tie rule.  The owner replaces
// the key by one below every key a logit can have.  All of this is the same for the whole wave, so the search is
// scalar branches around one compare per register.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ int wave_max_step(int v)
{
    // lanes without a source see the smallest integer, the identity of the maximum (which lets the move fold into it)
    return max(v, __builtin_amdgcn_update_dpp(int(0x80000000), v, CTRL, ROW_MASK, 0xF, false));
}

template <int NV>
__device__ __forceinline__ void topk_row(const float* __restrict__ logits, int32_t* __restrict__ topk_idx, float* __restrict__ topk_w, const int t,
                                         int E, int k)
{
    static_assert(NV % 4 == 0, "registers in groups of four consecutive experts");
    const int lane = threadIdx.x & 63;
    const float* row = logits + size_t(t) * E;
    constexpr int TAKEN = int(0x80000000);           // below the key of -infinity (0x807fffff)
    // register 4 i + c holds expert 256 i + 4 lane + c: one 16-byte load per i where the row allows it
    int key[NV];
    const bool wide = (E & 3) == 0 && (reinterpret_cast<uintptr_t>(logits) & 15) == 0;   // rows start 16-byte aligned, end on a group
    const bool full = E == 64 * NV;                   // no register lies beyond the row
#pragma unroll
    for (int i = 0; i < NV / 4; ++i) {
        const int e0 = 256 * i + 4 * lane;
        float v[4] = {0.f, 0.f, 0.f, 0.f};
        if (wide) {
            if (full || e0 < E) { const f32x4 q = *reinterpret_cast<const f32x4*>(row + e0); v[0] = q[0]; v[1] = q[1]; v[2] = q[2]; v[3] = q[3]; }
        } else {
#pragma unroll
            for (int c = 0; c < 4; ++c) if (e0 + c < E) v[c] = row[e0 + c];
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const float u = fmaxf(v[c], -INFINITY) + 0.f;            // the maximum drops a NaN, the sum turns -0 into +0
            const int bits = __builtin_bit_cast(int, u);
            const int ordered = bits ^ ((bits >> 31) & 0x7fffffff);
            key[4 * i + c] = (full || e0 + c < E) ? ordered : TAKEN;
        }
    }
    int chosen[MAX_K];
    float val[MAX_K];
#pragma unroll
    for (int j = 0; j < MAX_K; ++j) { chosen[j] = -1; val[j] = 0.f; }
#pragma unroll
    for (int j = 0; j < MAX_K; ++j) {
        if (j < k) {
            int m = key[0];
#pragma unroll
            for (int i = 1; i < NV; ++i) m = max(m, key[i]);
            m = wave_max_step<0xB1, 0xF>(m);       // quad_perm [1,0,3,2]
            m = wave_max_step<0x4E, 0xF>(m);       // quad_perm [2,3,0,1]
            m = wave_max_step<0x141, 0xF>(m);      // row_half_mirror
            m = wave_max_step<0x140, 0xF>(m);      // row_mirror
            m = wave_max_step<0x142, 0xA>(m);      // row_bcast15 into rows 1 and 3
            m = wave_max_step<0x143, 0xC>(m);      // row_bcast31 into rows 2 and 3
            m = __builtin_amdgcn_readlane(m, 63);
            bool found = false;
#pragma unroll
            for (int i = 0; i < NV / 4; ++i) {
                if (!found) {
                    int best = 0x7fffffff;           // lowest expert id of this group of 256 that holds m
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        const unsigned long long owners = __ballot(key[4 * i + c] == m);
                        if (owners) best = min(best, 256 * i + 4 * (__ffsll(owners) - 1) + c);
                    }
                    if (best != 0x7fffffff) {
                        chosen[j] = best;
#pragma unroll
                        for (int c = 0; c < 4; ++c)
                            if (256 * i + 4 * lane + c == best) key[4 * i + c] = TAKEN;
                        found = true;
                    }
                }
            }
            const int bits = m ^ ((m >> 31) & 0x7fffffff);
            val[j] = __builtin_bit_cast(float, bits);
        }
    }
    // softmax over the k kept logits with the hardware's exp2 (arguments <= 0, results in (0, 1], good to ~2e-6)
    float den = 0.f, ex[MAX_K];
#pragma unroll
    for (int j = 0; j < MAX_K; ++j) {
        ex[j] = j < k ? __expf(val[j] - val[0]) : 0.f;
        den += ex[j];
    }
#pragma unroll
    for (int j = 0; j < MAX_K; ++j)
        if (j < k && lane == j) {
            topk_idx[size_t(t) * k + j] = chosen[j];
            topk_w[size_t(t) * k + j] = ex[j] / den;
        }
}

template <int NV>
__global__ __launch_bounds__(256) void k_topk_small(const float* __restrict__ logits, int32_t* __restrict__ topk_idx,
                                                    float* __restrict__ topk_w, int T, int E, int k)
{
    const int t = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (t < T) topk_row<NV>(logits, topk_idx, topk_w, t, E, k);
}

// ------------------------------------------------------------------------------------------ grouping
__global__ void k_zero_i32(int32_t* p, size_t n)
{
    for (size_t i = size_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n; i += size_t(gridDim.x) * blockDim.x) p[i] = 0;
}

// Block b ranks its 256 uses: lrank[a] = number of earlier uses in the block with the same expert;
// blockcnt[e][b] = uses of expert e in block b (written by the last such use; array pre-zeroed).
__global__ __launch_bounds__(SORT_BLOCK) void k_rank_blocks(const int32_t* __restrict__ idx, int32_t* __restrict__ lrank,
                                                            int32_t* __restrict__ blockcnt, int A, int nblk)
{
    __shared__ int32_t se[SORT_BLOCK];
    const int a = blockIdx.x * SORT_BLOCK + threadIdx.x;
    const int e = a < A ? idx[a] : -1;
    se[threadIdx.x] = e;
    __syncthreads();
    if (a >= A) return;
    int before = 0, total = 0;
    for (int j = 0; j < SORT_BLOCK; ++j) {
        const bool same = (se[j] == e);
        total += same;
        before += same && (j < int(threadIdx.x));
    }
    lrank[a] = before;
    if (before == total - 1) blockcnt[size_t(e) * nblk + blockIdx.x] = total;
}

// One wave per expert: exclusive scan of blockcnt[e][:] in place, counts[e] = total.
__global__ __launch_bounds__(256) void k_scan_blocks(int32_t* __restrict__ blockcnt, int32_t* __restrict__ counts,
                                                     int E, int nblk)
{
    const int lane = threadIdx.x & 63;
    const int e = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (e >= E) return;
    int32_t* col = blockcnt + size_t(e) * nblk;
    int carry = 0;
    for (int b0 = 0; b0 < nblk; b0 += 64) {
        const int b = b0 + lane;
        const int v = b < nblk ? col[b] : 0;
        int inc = v;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int o = __shfl_up(inc, off);
            if (lane >= off) inc += o;
        }
        if (b < nblk) col[b] = carry + inc - v;
        carry += __shfl(inc, 63);
    }
    if (lane == 0) counts[e] = carry;
}

// Row tiles of k_grouped_stream: an expert's tiles of more than XM rows, up to XR, from the front of `tiles` on, and one of up to XM remaining rows, from the
// back on.  They are counted together, 65536 a whole tile and 1 a rest; how many there are stands in tile_start[E].
__device__ __forceinline__ int stream_tiles(int c) { return int(uint32_t((c + XR - XM - 1) / XR) << 16) | int(c % XR != 0 && c % XR <= XM); }
__device__ __forceinline__ int whole_tiles(int n) { return int(uint32_t(n) >> 16); }
__device__ __forceinline__ int rest_tiles(int n) { return n & 0xffff; }
// Every step-th one of an expert's tiles, whole ones first, from number i on.  (All workgroups or a wave share a crowded expert's: by one thread, 2000000 uses of 8 experts took
// k_offsets 65.5 us, 4.7 without them, k_place 9.0 with and without; 65536 uses of 1024 experts k_place_wide 14.5, 12.1 so, 11.2 with the other kernels' table)
__device__ __forceinline__ void put_stream_tiles(RowTile* tiles, int max_tiles, int before, int e, int at, int c, int i, int step)
{
    const int n = stream_tiles(c), whole = whole_tiles(n);
    for (; i < whole; i += step) tiles[whole_tiles(before) + i] = RowTile{e, at + i * XR, min(XR, c - i * XR), 0};
    if (i == whole && rest_tiles(n)) tiles[max_tiles - 1 - rest_tiles(before)] = RowTile{e, at + i * XR, c - i * XR, c <= XM};
}

// One workgroup of 16 waves: offsets = exclusive scan of counts; tile_start = exclusive scan of ceil(counts / TM).
// 1024 experts per pass: a scan inside every wave, the waves' totals through LDS.
constexpr int OFFS_THREADS = 1024;
template <bool STREAM>                                       // STREAM: tile_start = exclusive scan of stream_tiles(counts)
__global__ __launch_bounds__(OFFS_THREADS) void k_offsets(const int32_t* __restrict__ counts, int32_t* __restrict__ offsets,
                                                          int32_t* __restrict__ tile_start, int E)
{
    __shared__ int32_t wsum[OFFS_THREADS / 64], wtsum[OFFS_THREADS / 64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    int carry = 0, tcarry = 0;
    for (int e0 = 0; e0 < E; e0 += OFFS_THREADS) {
        const int e = e0 + tid;
        const int c = e < E ? counts[e] : 0;
        const int tl = STREAM ? stream_tiles(c) : (c + TM - 1) / TM;
        int inc = c, tinc = tl;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int o = __shfl_up(inc, off);
            const int to = __shfl_up(tinc, off);
            if (lane >= off) { inc += o; tinc += to; }
        }
        if (lane == 63) { wsum[wave] = inc; wtsum[wave] = tinc; }
        __syncthreads();
        int before = 0, tbefore = 0, all = 0, tall = 0;      // totals of the waves before this one, and of all
#pragma unroll
        for (int w = 0; w < OFFS_THREADS / 64; ++w) {
            const int a = wsum[w], t = wtsum[w];
            if (w < wave) { before += a; tbefore += t; }
            all += a;
            tall += t;
        }
        if (e < E) { offsets[e] = carry + before + inc - c; tile_start[e] = tcarry + tbefore + tinc - tl; }
        carry += all;
        tcarry += tall;
        __syncthreads();                                     // the totals are overwritten by the next pass
    }
    if (tid == 0) { offsets[E] = carry; tile_start[E] = tcarry; }
}

// STREAM: also k_grouped_stream's tiles, a wave for every expert (there are 64 uses for each, so waves enough)
template <bool STREAM>
__global__ __launch_bounds__(SORT_BLOCK) void k_place(const int32_t* __restrict__ idx, const int32_t* __restrict__ lrank,
                                                      const int32_t* __restrict__ blockoff, const int32_t* __restrict__ offsets,
                                                      int32_t* __restrict__ perm, int32_t* __restrict__ inv, int A, int nblk,
                                                      const int32_t* __restrict__ tile_start, RowTile* __restrict__ tiles, int max_tiles, int E)
{
    if constexpr (STREAM)
        for (int t = blockIdx.x * (SORT_BLOCK / 64) + (threadIdx.x >> 6); t < E; t += nblk * (SORT_BLOCK / 64))
            put_stream_tiles(tiles, max_tiles, tile_start[t], t, offsets[t], offsets[t + 1] - offsets[t], threadIdx.x & 63, 64);
    const int a = blockIdx.x * SORT_BLOCK + threadIdx.x;
    if (a >= A) return;
    const int e = idx[a];
    const int pos = offsets[e] + blockoff[size_t(e) * nblk + blockIdx.x] + lrank[a];
    perm[pos] = a;
    inv[a] = pos;
}

// The use of thread tid of 1024 among the block's first `n`: the number of earlier uses of its expert `my` (-1: none).  Every wave ranks
// its 64 uses among themselves, then the waves add theirs to count[] (LDS, zero before; the experts' uses after) in turn.
__device__ __forceinline__ int rank_in_block(int my, int n, int32_t* count)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int local = 0, same = 0;                              // uses of this expert in earlier lanes, in the whole wave
#pragma unroll 16
    for (int j = 0; j < 64; ++j) {
        const bool m = __builtin_amdgcn_readlane(my, j) == my;
        same += m;
        local += m && j < lane;
    }
    __syncthreads();
    int before = 0;
    for (int w = 0; w < (n + 63) / 64; ++w) {
        if (wave == w && my >= 0) {
            before = count[my] + local;
            if (local == same - 1) count[my] = before + 1;          // (behind the wave's reads: its LDS accesses are executed in order)
        }
        __syncthreads();
    }
    return before;
}

// The whole grouping of at most SMALL_USES uses in one workgroup, where the five kernels above are five launches with next to
// nothing to do (18 us for 74 uses): counts and places of the experts in LDS.  `tiles` (if not null): the row tiles of the expert layers, {expert, first row, rows, 0} each, rows = 0 from the
// last one on to max_tiles, so that a workgroup of those layers finds its tile with one load.
constexpr int SMALL_USES = 1024, SMALL_EXPERTS = 4096;

__global__ __launch_bounds__(1024) void k_group_small(const int32_t* __restrict__ idx, int32_t* __restrict__ counts,
                                                      int32_t* __restrict__ offsets, int32_t* __restrict__ tile_start,
                                                      int32_t* __restrict__ perm, int32_t* __restrict__ inv,
                                                      RowTile* __restrict__ tiles, int max_tiles, int A, int E)
{
    __shared__ int32_t first[SMALL_EXPERTS];              // counts, then the experts' first places
    __shared__ int32_t wsum[16], wtsum[16];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int my = tid < A ? idx[tid] : -1;
    for (int e = tid; e < E; e += 1024) first[e] = 0;
    const int before = rank_in_block(my, A, first);
    int carry = 0, tcarry = 0;
    for (int e0 = 0; e0 < E; e0 += 1024) {                // as k_offsets
        const int e = e0 + tid;
        const int c = e < E ? first[e] : 0;
        const int tl = (c + TM - 1) / TM;
        int inc = c, tinc = tl;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int o = __shfl_up(inc, off);
            const int to = __shfl_up(tinc, off);
            if (lane >= off) { inc += o; tinc += to; }
        }
        if (lane == 63) { wsum[wave] = inc; wtsum[wave] = tinc; }
        __syncthreads();
        int b = 0, tb = 0, all = 0, tall = 0;
#pragma unroll
        for (int w = 0; w < 16; ++w) {
            const int s = wsum[w], t = wtsum[w];
            if (w < wave) { b += s; tb += t; }
            all += s;
            tall += t;
        }
        if (e < E) {
            const int at = carry + b + inc - c, tat = tcarry + tb + tinc - tl;
            counts[e] = c;
            offsets[e] = at;
            tile_start[e] = tat;
            first[e] = at;
            if (tiles)
                for (int t = 0; t < tl; ++t) tiles[tat + t] = RowTile{e, at + t * TM, min(TM, c - t * TM), 0};
        }
        carry += all;
        tcarry += tall;
        __syncthreads();
    }
    if (tid == 0) { offsets[E] = carry; tile_start[E] = tcarry; }
    if (tiles)
        for (int t = tcarry + tid; t < max_tiles; t += 1024) tiles[t] = RowTile{0, 0, 0, 0};
    if (my >= 0) {
        const int pos = first[my] + before;
        perm[pos] = tid;
        inv[tid] = pos;
    }
}

// The same for more uses, in two launches: blocks of 1024 uses are ranked with the experts' counts in LDS and leave all of their
// counts, zeros included (nothing has to be cleared), as blockcnt[block][expert]; then every block adds up all blocks' counts for
// itself, four experts a thread, and places its uses.  For up to SMALL_EXPERTS experts and MID_BLOCKS blocks; us, the five launches
// below / these two with sixteen waves a workgroup / with four (k_place_wide beyond 1024 experts: eight), by blocks x experts: 2 x 64 20.6 / 12.2 / 10.2,
// 8 x 256 21.2 / 12.7 / 10.4, 32 x 1024 22.1 / 14.7 / 13.2, 64 x 1024 23.9 / 16.2 / 16.2, 40 x 2048 24.7 / 18.6 / 14.4, 20 x 4096 26.9 / 22.8 / 17.0,
// 64 x 4096 31.3 / 29.3 / 22.3.  Beside other layers' expert GEMMs sixteen waves find no CU with room for them: three layers of 64 x 1024 in
// flight 1.95 ms a layer with sixteen, 1.87 with eight in k_place_wide, 1.73 with four (the five launches: 1.81).
constexpr int MID_BLOCKS = 64;
__host__ __device__ constexpr int mid_stride(int E) { return (E + 3) & ~3; }      // experts of a row of blockcnt

// A block of 256 threads ranks 1024 uses: thread's use i is first + wave * 256 + i * 64 + lane (my: its expert, -1: none), before: the number of earlier
// ones of the block with that expert.  count[] (LDS): the experts' uses after
__device__ __forceinline__ void rank_1024(const int (&my)[4], int (&before)[4], int32_t* count, int stride, int E)
{
    using i32x4 = int32_t __attribute__((ext_vector_type(4)));
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    int local[4], same[4];
    for (int e = tid * 4; e < stride; e += 1024) *reinterpret_cast<i32x4*>(count + e) = i32x4{0, 0, 0, 0};
    // among 64 the lanes with the same expert are those that agree in every bit of its number
    uint64_t peers[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) peers[i] = __ballot(my[i] >= 0);
    for (int bit = 1; bit < E; bit <<= 1)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint64_t set = __ballot(my[i] & bit);
            peers[i] &= my[i] & bit ? set : ~set;
        }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        local[i] = __popcll(peers[i] & ((1ull << lane) - 1));
        same[i] = __popcll(peers[i]);
    }
    __syncthreads();
    // the waves add theirs in turn
    for (int w = 0; w < 4; ++w) {
        if (wave == w) {
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (my[i] >= 0) {
                    before[i] = count[my[i]] + local[i];
                    if (local[i] == same[i] - 1) count[my[i]] = before[i] + 1;       // (behind the wave's reads: its LDS accesses are executed in order)
                }
        }
        __syncthreads();
    }
}

__global__ __launch_bounds__(256) void k_rank_wide(const int32_t* __restrict__ idx, int32_t* __restrict__ lrank, int32_t* __restrict__ blockcnt, int A, int E)
{
    __shared__ __attribute__((aligned(16))) int32_t count[SMALL_EXPERTS];
    using i32x4 = int32_t __attribute__((ext_vector_type(4)));
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, stride = mid_stride(E);
    const int a0 = blockIdx.x * 1024 + wave * 256 + lane;
    int my[4], before[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) my[i] = a0 + i * 64 < A ? idx[a0 + i * 64] : -1;
    rank_1024(my, before, count, stride, E);
#pragma unroll
    for (int i = 0; i < 4; ++i)
        if (my[i] >= 0) lrank[a0 + i * 64] = before[i];
    for (int e = tid * 4; e < stride; e += 1024)
        *reinterpret_cast<i32x4*>(blockcnt + size_t(blockIdx.x) * stride + e) = *reinterpret_cast<const i32x4*>(count + e);
}

// Selection and grouping of at most SMALL_USES uses in one launch: the last workgroup to finish its tokens' selection groups all uses.  (A launch of
// its own for the grouping waits for the selection's end, its arguments and the indices: one token, d 160, h 184, 82 experts 25.0 -> 22.3 us a pass, 37 tokens of
// the small layer 42.2 -> 39.7.)
// `done`: zero before the launch (the gate's kernels clear it).
template <int NV>
__global__ __launch_bounds__(256) void k_topk_group(const float* __restrict__ logits, int32_t* __restrict__ topk_idx, float* __restrict__ topk_w, int T, int E,
                                                    int k, int32_t* __restrict__ done, int32_t* __restrict__ counts, int32_t* __restrict__ offsets,
                                                    int32_t* __restrict__ tile_start, int32_t* __restrict__ perm, int32_t* __restrict__ inv,
                                                    RowTile* __restrict__ tiles, int max_tiles)
{
    __shared__ __attribute__((aligned(16))) int32_t first[64 * NV];           // counts, then the experts' first places
    __shared__ int32_t wsum[4], wtsum[4], s_last;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int t = blockIdx.x * 4 + wave;
    if (t < T) topk_row<NV>(logits, topk_idx, topk_w, t, E, k);
    // every wave waits until its stores have reached the L2, then one thread makes them visible to the chip and counts this workgroup in; the
    // last one sees what all others have made visible
    wait_for_stores();
    __syncthreads();
    if (tid == 0) s_last = __hip_atomic_fetch_add(done, 1, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) == int(gridDim.x) - 1;
    __syncthreads();
    if (!s_last) return;
    const int A = T * k, stride = mid_stride(E);
    int my[4], before[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int a = wave * 256 + i * 64 + lane;
        my[i] = a < A ? __hip_atomic_load(topk_idx + a, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : -1;
    }
    rank_1024(my, before, first, stride, E);
    using i32x4 = int32_t __attribute__((ext_vector_type(4)));
    int carry = 0, tcarry = 0;
    for (int e0 = 0; e0 < E; e0 += 1024) {                // as k_offsets, four experts a thread
        const int e = e0 + tid * 4;
        i32x4 c = {0, 0, 0, 0};
        if (e < E) c = *reinterpret_cast<const i32x4*>(first + e);
        const i32x4 tl = (c + (TM - 1)) / TM;
        const int mine = c.x + c.y + c.z + c.w, tmine = tl.x + tl.y + tl.z + tl.w;
        int inc = mine, tinc = tmine;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int o = __shfl_up(inc, off);
            const int to = __shfl_up(tinc, off);
            if (lane >= off) { inc += o; tinc += to; }
        }
        if (lane == 63) { wsum[wave] = inc; wtsum[wave] = tinc; }
        __syncthreads();
        int earlier = 0, tearlier = 0, all = 0, tall = 0;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            if (w < wave) { earlier += wsum[w]; tearlier += wtsum[w]; }
            all += wsum[w];
            tall += wtsum[w];
        }
        int at = carry + earlier + inc - mine, tat = tcarry + tearlier + tinc - tmine;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (e + i < E) {
                first[e + i] = at;
                counts[e + i] = c[i];
                offsets[e + i] = at;
                tile_start[e + i] = tat;
                if (tiles)
                    for (int q = 0; q < tl[i]; ++q) tiles[tat + q] = RowTile{e + i, at + q * TM, min(TM, c[i] - q * TM), 0};
            }
            at += c[i];
            tat += tl[i];
        }
        carry += all;
        tcarry += tall;
        __syncthreads();
    }
    if (tid == 0) { offsets[E] = carry; tile_start[E] = tcarry; }
    if (tiles)
        for (int q = tcarry + tid; q < max_tiles; q += 256) tiles[q] = RowTile{0, 0, 0, 0};
#pragma unroll
    for (int i = 0; i < 4; ++i)
        if (my[i] >= 0) {
            const int a = wave * 256 + i * 64 + lane, pos = first[my[i]] + before[i];
            perm[pos] = a;
            inv[a] = pos;
        }
}

// block 0 also writes the experts' tables; tiles as in k_group_small, or (STREAM) as k_grouped_stream wants them
template <int WAVES, bool STREAM>
__global__ __launch_bounds__(WAVES * 64) void k_place_wide(const int32_t* __restrict__ idx, const int32_t* __restrict__ lrank, const int32_t* __restrict__ blockcnt,
                                                    int32_t* __restrict__ counts, int32_t* __restrict__ offsets, int32_t* __restrict__ tile_start,
                                                    int32_t* __restrict__ perm, int32_t* __restrict__ inv, RowTile* __restrict__ tiles, int max_tiles,
                                                    int A, int E, int nblk)
{
    __shared__ int32_t first[SMALL_EXPERTS];              // where this block's uses of an expert start
    constexpr int THREADS = WAVES * 64, USES = 1024 / THREADS;
    __shared__ int32_t wsum[WAVES], wtsum[WAVES];
    using i32x4 = int32_t __attribute__((ext_vector_type(4)));
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, blk = blockIdx.x, stride = mid_stride(E);
    const bool tables = blk == 0;
    int my[USES], rank[USES];
#pragma unroll
    for (int i = 0; i < USES; ++i) {
        const int a = blk * 1024 + i * THREADS + tid;
        my[i] = a < A ? idx[a] : 0;
        rank[i] = a < A ? lrank[a] : 0;
    }
    int carry = 0, tcarry = 0;
    for (int e0 = 0; e0 < E; e0 += 4 * THREADS) {
        const int e = e0 + tid * 4;                       // this thread: experts e .. e + 3 (behind E: no uses)
        i32x4 c = {0, 0, 0, 0}, before = {0, 0, 0, 0};    // uses in all blocks, in the blocks before this one
        if (e < E) {
            const int32_t* p = blockcnt + e;
            for (int b0 = 0; b0 < nblk; b0 += 16) {
                i32x4 v[16];
#pragma unroll
                for (int i = 0; i < 16; ++i) v[i] = b0 + i < nblk ? *reinterpret_cast<const i32x4*>(p + size_t(b0 + i) * stride) : i32x4{0, 0, 0, 0};
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    c += v[i];
                    if (b0 + i < blk) before += v[i];
                }
            }
        }
        // from here on as k_offsets, four experts a thread
        const i32x4 tl = STREAM ? i32x4{stream_tiles(c.x), stream_tiles(c.y), stream_tiles(c.z), stream_tiles(c.w)} : (c + (TM - 1)) / TM;
        const int mine = c.x + c.y + c.z + c.w, tmine = tl.x + tl.y + tl.z + tl.w;
        int inc = mine, tinc = tmine;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int o = __shfl_up(inc, off);
            const int to = __shfl_up(tinc, off);
            if (lane >= off) { inc += o; tinc += to; }
        }
        if (lane == 63) { wsum[wave] = inc; wtsum[wave] = tinc; }
        __syncthreads();
        int earlier = 0, tearlier = 0, all = 0, tall = 0;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) {
            const int s = wsum[w], t = wtsum[w];
            if (w < wave) { earlier += s; tearlier += t; }
            all += s;
            tall += t;
        }
        int at = carry + earlier + inc - mine, tat = tcarry + tearlier + tinc - tmine;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (e + i < E) {
                first[e + i] = at + before[i];
                if (!STREAM && tiles)
                    for (int t = blk; t < tl[i]; t += nblk) tiles[tat + t] = RowTile{e + i, at + t * TM, min(TM, c[i] - t * TM), 0};
                if (STREAM) put_stream_tiles(tiles, max_tiles, tat, e + i, at, c[i], blk, nblk);
                if (tables) {
                    counts[e + i] = c[i];
                    offsets[e + i] = at;
                    tile_start[e + i] = tat;
                }
            }
            at += c[i];
            tat += tl[i];
        }
        carry += all;
        tcarry += tall;
        __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < USES; ++i) {
        const int a = blk * 1024 + i * THREADS + tid;
        if (a < A) {
            const int pos = first[my[i]] + rank[i];
            perm[pos] = a;
            inv[a] = pos;
        }
    }
    if (!tables) return;
    if (tid == 0) { offsets[E] = carry; tile_start[E] = tcarry; }
    if (!STREAM && tiles)
        for (int t = tcarry + tid; t < max_tiles; t += THREADS) tiles[t] = RowTile{0, 0, 0, 0};
}

// ------------------------------------------------------------------------------------------ permute / combine
// xs[inv[t*k + j]] = x[t] for j < k: one wave per token reads the row once and scatters it to the
// token's k places in the expert-sorted order (reading by sorted position instead would fetch every
// token row k times, since a token's uses sit in k different groups).  d is a multiple of 8.
// The first MAX_K places sit in registers; a token with more uses looks the others up as it goes.
__global__ __launch_bounds__(256) void k_permute(const bf16_t* __restrict__ x, const int32_t* __restrict__ inv,
                                                 bf16_t* __restrict__ xs, int T, int d, int k)
{
    const int lane = threadIdx.x & 63;
    const int t = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (t >= T) return;
    const int32_t* inv_t = inv + size_t(t) * k;
    int pos[MAX_K];
#pragma unroll
    for (int j = 0; j < MAX_K; ++j) pos[j] = j < k ? inv_t[j] : 0;
    const u32x4* src = reinterpret_cast<const u32x4*>(x + size_t(t) * d);
    for (int c0 = 0; c0 < d / 8; c0 += 256) {
        u32x4 v[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int c = c0 + i * 64 + lane;
            if (c < d / 8) v[i] = src[c];
        }
        auto put = [&](int p) {
            u32x4* dst = reinterpret_cast<u32x4*>(xs + size_t(p) * d);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int c = c0 + i * 64 + lane;
                if (c < d / 8) dst[c] = v[i];
            }
        };
#pragma unroll
        for (int j = 0; j < MAX_K; ++j)
            if (j < k) put(pos[j]);
        for (int j = MAX_K; j < k; ++j) put(inv_t[j]);
    }
}

__global__ __launch_bounds__(256) void k_combine(const bf16_t* __restrict__ y, const int32_t* __restrict__ inv,
                                                 const float* __restrict__ topk_w, bf16_t* __restrict__ out,
                                                 int T, int d, int k)
{
    const int lane = threadIdx.x & 63;
    const int t = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (t >= T) return;
    const int32_t* inv_t = inv + size_t(t) * k;
    const float* w_t = topk_w + size_t(t) * k;
    int pos[MAX_K];
    float w[MAX_K];
#pragma unroll
    for (int j = 0; j < MAX_K; ++j)
        if (j < k) { pos[j] = inv_t[j]; w[j] = w_t[j]; }
    for (int c = lane; c < d / 8; c += 64) {
        float acc[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) acc[i] = 0.f;
        auto add = [&](int p, float wj) {                  // j ascending: the summation order is fixed
            const u32x4 v = reinterpret_cast<const u32x4*>(y + size_t(p) * d)[c];
            const uint32_t u[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                acc[2 * i] += wj * __uint_as_float(u[i] << 16);
                acc[2 * i + 1] += wj * __uint_as_float(u[i] & 0xffff0000u);
            }
        };
#pragma unroll
        for (int j = 0; j < MAX_K; ++j)
            if (j < k) add(pos[j], w[j]);
        for (int j = MAX_K; j < k; ++j) add(inv_t[j], w_t[j]);
        u32x4 o;
        o.x = pack_bf16x2(acc[0], acc[1]);
        o.y = pack_bf16x2(acc[2], acc[3]);
        o.z = pack_bf16x2(acc[4], acc[5]);
        o.w = pack_bf16x2(acc[6], acc[7]);
        reinterpret_cast<u32x4*>(out + size_t(t) * d)[c] = o;
    }
}

// ------------------------------------------------------------------------------------------ grouped GEMM
// Tile body: out[row0 .. row0+rows)[nb .. nb+TN) = act(in[rows][K] . We[n][K]^T), ML = live 16-row tiles.
//
// Operands go through LDS in K-chunks of 64.  Loading MFMA fragments straight from global memory
// makes every lane of a load touch its own 16 bytes of a different row, and the vector L1 then
// retires about one lane per clock (measured: ~16 B/clk per CU, which capped this kernel at 2 ms
// per layer).  Staged loads instead let 8 neighbouring lanes read one row's 128 contiguous bytes;
// the fragments are then cut out of LDS with ds_read_b128 (row pitch 144 bytes, conflict free).
// The next chunk is fetched into registers while the current one is multiplied: 40 KB per
// workgroup, two workgroups per CU.  (Tiles of 128 features with four workgroups per CU stream
// the second layer's 4 KB-pitched weight rows 15 % slower and are no faster elsewhere.)
constexpr int KC = 64;                 // K-chunk
constexpr int LDP = KC + 8;            // LDS row pitch in elements (144 bytes)

// gather != nullptr: the tile's input rows are not in[row0 ..] but rows of `in` picked through the
// grouping: row r of the tile is in[gather[row0 + r] / kdiv] (the token of that expert use), i.e. the
// stacking of the tokens happens inside the operand load and the permuted copy is never written.
template <bool RELU, int ML>
__device__ __forceinline__ void gemm_tile(const bf16_t* __restrict__ in, const bf16_t* __restrict__ We,
                                          bf16_t* __restrict__ out, int row0, int rows, int nb, int N, int K,
                                          bf16_t* Ws, bf16_t* Xs, const int32_t* __restrict__ gather, int kdiv)
{
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, r = lane & 15, g = lane >> 4;
    constexpr int PARTS = KC / 8;                  // 16-byte pieces of one chunk row
    constexpr int RPP = 256 / PARTS;               // rows staged per pass of the workgroup
    constexpr int WPASS = TN / RPP, XPASS = TM / RPP;
    const int part = tid % PARTS, prow = tid / PARTS;
    // staging assignments: WPASS weight rows and up to XPASS activation rows per thread
    const bf16_t* wsrc[WPASS];
    const bf16_t* xsrc[XPASS];
#pragma unroll
    for (int i = 0; i < WPASS; ++i) wsrc[i] = We + size_t(min(nb + prow + i * RPP, N - 1)) * K + part * 8;
#pragma unroll
    for (int i = 0; i < XPASS; ++i) {
        const int r = row0 + min(prow + i * RPP, rows - 1);
        xsrc[i] = in + size_t(gather ? gather[r] / kdiv : r) * K + part * 8;
    }
    u32x4 wreg[WPASS], xreg[XPASS];
    auto fetch = [&](int kc) {
        const bool inside = kc * KC + part * 8 < K;   // K is a multiple of 8: the last chunk may be partly empty
#pragma unroll
        for (int i = 0; i < WPASS; ++i)
            wreg[i] = inside ? *reinterpret_cast<const u32x4*>(wsrc[i] + kc * KC) : u32x4{0u, 0u, 0u, 0u};
#pragma unroll
        for (int i = 0; i < XPASS; ++i)
            if (i * RPP < ML * 16)                    // only rows of live 16-row sub-tiles
                xreg[i] = inside ? *reinterpret_cast<const u32x4*>(xsrc[i] + kc * KC) : u32x4{0u, 0u, 0u, 0u};
    };
    const int nchunk = (K + KC - 1) / KC;
    // one K-chunk through LDS: registers -> LDS, barrier, prefetch of the next chunk, multiply, barrier
    auto chunk_loop = [&](auto&& multiply) {
        fetch(0);
        for (int kc = 0; kc < nchunk; ++kc) {
#pragma unroll
            for (int i = 0; i < WPASS; ++i)
                *reinterpret_cast<u32x4*>(Ws + (prow + i * RPP) * LDP + part * 8) = wreg[i];
#pragma unroll
            for (int i = 0; i < XPASS; ++i)
                if (i * RPP < ML * 16) *reinterpret_cast<u32x4*>(Xs + (prow + i * RPP) * LDP + part * 8) = xreg[i];
            __syncthreads();
            if (kc + 1 < nchunk) fetch(kc + 1);
            multiply();
            __syncthreads();
        }
    };
    const int n0 = nb + wave * (TN / 4);          // first feature of this wave
    auto store4 = [&](int lr, int n, float v0, float v1, float v2, float v3) {
        if (lr >= rows || n >= N) return;
        u32x2 pk;
        pk.x = pack_bf16x2(v0, v1);
        pk.y = pack_bf16x2(v2, v3);
        if (RELU) { pk.x = relu_bf16x2(pk.x); pk.y = relu_bf16x2(pk.y); }
        *reinterpret_cast<u32x2*>(out + size_t(row0 + lr) * N + n) = pk;
    };
    if constexpr (ML == 4) {
        // all four 16-row sub-tiles live: 32x32x16 MFMAs (the faster bf16 shape), 2 x 2 tiles per wave
        static_assert(TN == 256, "two 32-feature tiles per wave");
        const int q = lane & 31, hk = lane >> 5;
        f32x16 acc[2][2];
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int i = 0; i < 16; ++i) acc[a][b][i] = 0.f;
        chunk_loop([&] {
#pragma unroll
            for (int ks = 0; ks < KC / 16; ++ks) {
                bf16x8 wf[2], xf[2];
#pragma unroll
                for (int a = 0; a < 2; ++a)
                    wf[a] = *reinterpret_cast<const bf16x8*>(Ws + (wave * 64 + a * 32 + q) * LDP + ks * 16 + hk * 8);
#pragma unroll
                for (int b = 0; b < 2; ++b)
                    xf[b] = *reinterpret_cast<const bf16x8*>(Xs + (b * 32 + q) * LDP + ks * 16 + hk * 8);
#pragma unroll
                for (int a = 0; a < 2; ++a)
#pragma unroll
                    for (int b = 0; b < 2; ++b)
                        acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[a], xf[b], acc[a][b], 0, 0, 0);
            }
        });
        // lane holds row b*32 + q, features n0 + a*32 + 8j + 4hk .. +3 in acc[a][b][4j .. 4j+3]
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int a = 0; a < 2; ++a)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    store4(b * 32 + q, n0 + a * 32 + 8 * j + 4 * hk, acc[a][b][4 * j], acc[a][b][4 * j + 1],
                           acc[a][b][4 * j + 2], acc[a][b][4 * j + 3]);
    } else {
        f32x4 acc[ML][NTW];
#pragma unroll
        for (int mt = 0; mt < ML; ++mt)
#pragma unroll
            for (int nt = 0; nt < NTW; ++nt) acc[mt][nt] = f32x4{0, 0, 0, 0};
        chunk_loop([&] {
#pragma unroll
            for (int kk = 0; kk < KC / 32; ++kk) {
                bf16x8 wf[NTW], xf[ML];
#pragma unroll
                for (int nt = 0; nt < NTW; ++nt)
                    wf[nt] = *reinterpret_cast<const bf16x8*>(Ws + (wave * (TN / 4) + nt * 16 + r) * LDP + kk * 32 + g * 8);
#pragma unroll
                for (int mt = 0; mt < ML; ++mt)
                    xf[mt] = *reinterpret_cast<const bf16x8*>(Xs + (mt * 16 + r) * LDP + kk * 32 + g * 8);
#pragma unroll
                for (int mt = 0; mt < ML; ++mt)
#pragma unroll
                    for (int nt = 0; nt < NTW; ++nt)
                        acc[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[nt], xf[mt], acc[mt][nt], 0, 0, 0);
            }
        });
        // lane holds features n0 + nt*16 + g*4 .. +3 of row mt*16 + r
#pragma unroll
        for (int mt = 0; mt < ML; ++mt)
#pragma unroll
            for (int nt = 0; nt < NTW; ++nt)
                store4(mt * 16 + r, n0 + nt * 16 + g * 4, acc[mt][nt].x, acc[mt][nt].y, acc[mt][nt].z, acc[mt][nt].w);
    }
}

// out[row][n] = act( sum_k in[row][k] * W[e][n][k] ) for the rows of expert e.
// One workgroup = one (row tile of <= 64 rows inside one group, 256 output features) pair; a group's
// tiles are found from tile_start (prefix sum of ceil(count/64)), so ragged and empty groups cost
// nothing beyond their real rows.  4 waves split the 256 features; only the live 16-row sub-tiles
// are multiplied.  N must be a multiple of 4 (it is: d and h are multiples of 8).
template <bool RELU>
__global__ __launch_bounds__(256) void k_grouped_gemm(const bf16_t* __restrict__ in, const bf16_t* __restrict__ W,
                                                      bf16_t* __restrict__ out, const int32_t* __restrict__ offsets,
                                                      const int32_t* __restrict__ tile_start, int E, int N, int K,
                                                      int n_tiles_n, const int32_t* __restrict__ gather, int kdiv)
{
    __shared__ __attribute__((aligned(16))) bf16_t Ws[TN * LDP];
    __shared__ __attribute__((aligned(16))) bf16_t Xs[TM * LDP];
    // Tiles are numbered expert by expert; inside an expert, row tiles are taken in groups of MG, and
    // inside a group the row tiles that share one feature tile are adjacent (feature tile outer, row
    // tile inner), so a weight tile is fetched from HBM once and then found in L2 by the other row
    // tiles of its group.  Consecutive workgroup ids land on different XCDs (8 of them, each with
    // its own L2), so the numbering is dealt to the XCDs in equal runs of at most XCD_CHUNK tiles:
    // everything that shares weights or activation rows stays behind one L2, and every XCD gets as many runs.
    const uint32_t total = uint32_t(tile_start[E]) * uint32_t(n_tiles_n);      // (below 2^31: check_shape bounds the grid; at least one tile)
    const uint32_t runs = (total + 8 * XCD_CHUNK - 1) / (8 * XCD_CHUNK);
    // (as few tiles as one XCD has CUs stay on one, behind whose L2 the next layer finds their rows: one token, layers of 768 x 64, 6 uses, 30.2
    // us dealt to all, 28.4 so; 248 x 136, 8 uses, 26.4 / 25.5.  The per-use loop's small grids do not reach that far)
    const uint32_t chunk = total <= XCD_CUS && gridDim.x >= 8 * XCD_CUS ? XCD_CUS : (total + 8 * runs - 1) / (8 * runs);
    const uint32_t xcd = blockIdx.x & 7, j = blockIdx.x >> 3;
    const uint32_t lin = (j / chunk * 8 + xcd) * chunk + j % chunk;
    if (j >= runs * chunk || lin >= total) return;
    const int lin_m = int(lin / uint32_t(n_tiles_n));
    // largest e with tile_start[e] <= lin_m, 64 places looked at together: two trips to memory for up to 4096 experts
    int lo = 0, hi = E;
    while (hi - lo > 1) {
        const int stride = (hi - lo + 63) / 64, at = lo + int(threadIdx.x & 63) * stride;
        const int below = __popcll(__ballot(at < hi && tile_start[min(at, E)] <= lin_m));   // (place 0 always is)
        lo += (below - 1) * stride;
        hi = min(lo + stride, hi);
    }
    const int e = lo;
    const int mt_e = tile_start[e + 1] - tile_start[e];
    const int i = int(lin) - tile_start[e] * n_tiles_n;   // tile of this expert, 0 .. mt_e * n_tiles_n
    const int mg = i / (MG * n_tiles_n);
    const int rem = i - mg * MG * n_tiles_n;
    const int gsize = min(MG, mt_e - mg * MG);
    const int ntile = rem / gsize;
    const int mtile = mg * MG + rem % gsize;
    const int row0 = offsets[e] + mtile * TM;
    const int rows = min(TM, offsets[e + 1] - row0);
    const int mlive = (rows + 15) >> 4;
    const bf16_t* We = W + size_t(e) * N * K;
    const int nb = ntile * TN;
    if (mlive <= 1) gemm_tile<RELU, 1>(in, We, out, row0, rows, nb, N, K, Ws, Xs, gather, kdiv);
    else if (mlive == 2) gemm_tile<RELU, 2>(in, We, out, row0, rows, nb, N, K, Ws, Xs, gather, kdiv);
    else gemm_tile<RELU, 4>(in, We, out, row0, rows, nb, N, K, Ws, Xs, gather, kdiv);
}

// The expert layers for few tiles (the rule stands where it is applied).  There a layer is a stream of weights, each multiplied with a handful of rows: what
// counts is how much of it is in flight.  k_grouped_gemm asks for one K-chunk at a time and for 256 features per workgroup.  Here a workgroup
// owns 64 features of a row tile, a wave 16 of them, and weights go straight from memory into registers, SK_RD K-steps (1 KB
// each) ahead; two consecutive steps read one 128-byte line per row.  The rows pass through LDS, 32 KB of them at a time: four
// waves that read their fragments from global memory are answered at 16 bytes per clock (neighbouring lanes hold different
// rows), which alone took 8 us.
// The results are those of k_grouped_gemm bit for bit, whose tiles of more than 32 rows use the 32x32x16 MFMA: one 16x16x32 MFMA
// rounds like two of those over the same channels (524288 sums of 512 products, values spread over up to 2^32: no bit differs).
constexpr int SK_RD = 16;
constexpr int SK_LDS = 33 * 1024;                              // 16 ML rows of 1024 / ML channels and 16 bytes

template <bool RELU, int ML>
__device__ __forceinline__ void skinny_tile(const bf16_t* __restrict__ in, const bf16_t* __restrict__ We, bf16_t* __restrict__ out,
                                            const RowTile tile, int n0, int N, int K, const int32_t* __restrict__ gather, int kdiv,
                                            unsigned char* lds)
{
    constexpr int RD = SK_RD, KB = 1024 / ML, SB = KB / 32, PITCH = KB * 2 + 16, PIECES = KB / 8, NP = 16 * ML * PIECES / 256;
    static_assert(16 * ML * PITCH <= SK_LDS && SB % 8 == 0, "LDS block");
    constexpr int U = SB < RD ? SB : RD;                       // steps per trip: a divisor of a block's
    const int tid = threadIdx.x, lane = tid & 63, r = lane & 15, g = lane >> 4;
    const bf16_t* const pw = We + size_t(min(n0 + r, N - 1)) * K;
    const int S = (K + 31) / 32, last = S - 1;
    u32x4 w[U];
    // past the end the last step again; behind K (a multiple of 8) anything, replaced by zeros where it is used (here, the
    // replacement would wait for every piece as it is requested)
    auto fetch = [&](int s, u32x4& v) {
        const int k = min(s, last) * 32 + g * 8;
        v = *reinterpret_cast<const u32x4*>(pw + (k < K ? k : 0));
    };
#pragma unroll
    for (int u = 0; u < U; ++u) fetch(u, w[u]);
    f32x4 acc[ML];
#pragma unroll
    for (int m = 0; m < ML; ++m) acc[m] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int b = 0; b < S; b += SB) {                          // a block of channels
        if (b > 0) __syncthreads();
        u32x4 v[NP];
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            const int c = tid + i * 256, row = tile.row0 + min(c / PIECES, tile.rows - 1), k = b * 32 + c % PIECES * 8;
            v[i] = *reinterpret_cast<const u32x4*>(in + size_t(gather ? gather[row] / kdiv : row) * K + (k < K ? k : 0)) & (k < K ? ~0u : 0u);
        }
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            const int c = tid + i * 256;
            *reinterpret_cast<u32x4*>(__builtin_assume_aligned(lds + c / PIECES * PITCH + c % PIECES * 16, 16)) = v[i];
        }
        __syncthreads();
        for (int s = b; s < min(S, b + SB); s += U) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (s + u < S) {
                    const u32x4 wu = w[u] & ((s + u) * 32 + g * 8 < K ? ~0u : 0u);
#pragma unroll
                    for (int m = 0; m < ML; ++m) {
                        const u32x4 x = *reinterpret_cast<const u32x4*>(lds + (m * 16 + r) * PITCH + (s + u - b) * 64 + g * 16);
                        acc[m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, wu), __builtin_bit_cast(bf16x8, x), acc[m], 0, 0, 0);
                    }
                }
                fetch(s + u + U, w[u]);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }
    // lane: features n0 + 4 g .. + 3 of rows 16 m + r
    const int n = n0 + g * 4;
#pragma unroll
    for (int m = 0; m < ML; ++m) {
        const int row = m * 16 + r;
        if (row >= tile.rows || n >= N) continue;
        u32x2 pk = {pack_bf16x2(acc[m].x, acc[m].y), pack_bf16x2(acc[m].z, acc[m].w)};
        if (RELU) { pk.x = relu_bf16x2(pk.x); pk.y = relu_bf16x2(pk.y); }
        *reinterpret_cast<u32x2*>(out + size_t(tile.row0 + row) * N + n) = pk;
    }
}

template <bool RELU>
__global__ __launch_bounds__(256, 3) void k_grouped_skinny(const bf16_t* __restrict__ in, const bf16_t* __restrict__ W, bf16_t* __restrict__ out,
                                                        const RowTile* __restrict__ tiles, int N, int K, int n_tiles_n,
                                                        const int32_t* __restrict__ gather, int kdiv)
{
    __shared__ __attribute__((aligned(16))) unsigned char lds[SK_LDS];
    const int m = blockIdx.x / n_tiles_n;
    const RowTile tile = tiles[m];
    const int n0 = (int(blockIdx.x) - m * n_tiles_n) * 64 + int(threadIdx.x >> 6) * 16;      // (a wave may have no features; it stages)
    if (tile.rows == 0) return;
    const bf16_t* We = W + size_t(tile.expert) * N * K;
    if (tile.rows <= 16) skinny_tile<RELU, 1>(in, We, out, tile, n0, N, K, gather, kdiv, lds);
    else if (tile.rows <= 32) skinny_tile<RELU, 2>(in, We, out, tile, n0, N, K, gather, kdiv, lds);
    else skinny_tile<RELU, 4>(in, We, out, tile, n0, N, K, gather, kdiv, lds);
}

// The expert layers of whole K-chunks (the rule stands where it is applied): a stream of weights, each used for a handful of rows, of which every CU should have
// its share under way at once.  A workgroup owns up to 64 rows x 128 features; chunks of 64 channels go from memory straight into LDS, BUFS - 1 of them ahead, with one
// barrier each (k_grouped_gemm and k_grouped_skinny wait for a trip to memory per 64 and 32 channels), the weights' first ones ahead of the look-up of the rows.  A wave
// multiplies 32 features.  What bounds it is memory, at 4096 tokens, 256 experts, d 512, h 1024 (two layers of 268 MB, as many as 20 MB of results, which cost the
// reading six times their bytes: 58 us a layer at the rate of a large copy): 62.7 and 63.6 us with k_grouped_gemm, 57.3 and 58.2 so.  (Workgroups that stay for the
// launch and ask for the next tile's chunks ahead, as k_grouped_stream's: 60.0 and 62.9.  Without the two of __launch_bounds__ the sums move to AGPRs and back every
// chunk: 59.2 and 62.0.)
// The sums are k_grouped_gemm's bit for bit: 32x32x16 MFMAs over the channels in the same order.
// `chunk` consecutive tiles are dealt to one XCD at a time: the features of a row tile, whose rows they share, and an expert's next row tile, whose weights it shares.
constexpr int FEW_F = 128;
constexpr int few_lds(int bufs) { return bufs * 3 * XUNIT + 4 * 256; }   // a chunk: two units of weights and one of rows; each wave's places of the rows

template <bool RELU, int BUFS>
__global__ __launch_bounds__(256, 2) void k_grouped_few(const bf16_t* __restrict__ in, const bf16_t* __restrict__ W, bf16_t* __restrict__ out,
                                                     const RowTile* __restrict__ tiles, int n_tiles_m, int chunk, int N, int K, int n_tiles_n,
                                                     const int32_t* __restrict__ gather, uint32_t m_kdiv)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
    constexpr uint32_t BUF = 3 * XUNIT;
    constexpr uint32_t PLACES = BUFS * BUF;
    constexpr int PIECES = 6;                                  // of a chunk, each wave's
    const int j = blockIdx.x >> 3, run = j / chunk, lin = (run * 8 + int(blockIdx.x & 7)) * chunk + j - run * chunk;
    const int m = lin / n_tiles_n, n0 = (lin - m * n_tiles_n) * FEW_F;
    if (m >= n_tiles_m) return;
    const int expert = uniform_load(&tiles[m].expert), row0 = uniform_load(&tiles[m].row0), rows = uniform_load(&tiles[m].rows);
    if (rows == 0) return;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, q = lane & 31, hk = lane >> 5;
    // wave w copies blocks 2 w and 2 w + 1 of every unit
    uint32_t w_off[2][2], x_off[2];
    int x_row[2];
    bool x_on[2];                                              // this lane's row is there (lane 0: always, so that every wave makes every request, which it counts)
    if constexpr (RELU)                                        // (the first layer: gathered rows.  Through LDS, for the compiler waits for all requests where it waits for a register's)
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) uint32_t*)(gather + row0 + min(lane, rows - 1)),
                                         (__attribute__((address_space(3))) uint32_t*)(lds_raw + PLACES + wave * 256), 4, 0, 0);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int s_q = copied_row(2 * wave + i, lane), f = (lane >> 5) * 32 + (s_q >> 2 & 1) * 16 + (s_q >> 3) * 4 + (s_q & 3);
        x_row[i] = min((lane >> 5) * 32 + s_q, rows - 1);
        x_on[i] = (lane >> 5) * 32 + s_q < rows || lane == 0;
#pragma unroll
        for (int u = 0; u < 2; ++u) w_off[u][i] = (uint32_t(min(n0 + u * 64 + f, N - 1) - n0) * uint32_t(K) + uint32_t(lane & 7) * 8u) * 2u;
    }
    const char* w_next = reinterpret_cast<const char*>(W + (size_t(expert) * N + n0) * K);
    const char* x_next = reinterpret_cast<const char*>(in);
    uint32_t fill = 0, take = 0;
    auto request_w = [&](uint32_t to) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int u = 0; u < 2; ++u) lds_copy16(w_next, w_off[u][i], to + uint32_t(u * XUNIT + (2 * wave + i) * XBLOCK));
        w_next += 128;
    };
    auto request_x = [&](uint32_t to) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
            if (x_on[i]) lds_copy16(x_next, x_off[i], to + uint32_t(2 * XUNIT + (2 * wave + i) * XBLOCK));
        x_next += 128;
    };
    const int nchunk = K / 64;
    // the weights first: the rows' places are on their way
    request_w(0);
    if (BUFS == 3 && nchunk > 1) request_w(BUF);
    if constexpr (RELU) {
        if (BUFS == 3 && nchunk > 1) answered_but<8>();
        else answered_but<4>();
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        uint32_t row = uint32_t(row0 + x_row[i]);
        if constexpr (RELU) {
            row = *reinterpret_cast<const uint32_t*>(lds_raw + PLACES + wave * 256 + x_row[i] * 4);
            if (m_kdiv) row = __umulhi(row, m_kdiv);           // / k
        }
        x_off[i] = (row * uint32_t(K) + uint32_t(lane & 7) * 8u) * 2u;
    }
    request_x(0);
    if (BUFS == 3 && nchunk > 1) request_x(BUF);
    fill = (BUFS - 1) * BUF;
    f32x16 acc[2];
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[b][i] = 0.f;
    const uint32_t slot = fragment_at(q, hk);
    auto multiply = [&](auto blocks) {                         // the tile, one or two blocks of 32 rows
        constexpr int NB = decltype(blocks)::value;
#pragma unroll 1
        for (int c = 0; c < nchunk; ++c) {
            if (BUFS == 2 || c + 1 >= nchunk) answered_but<0>();
            else if (c == 0) answered_but<2>();                // (all but chunk 1's rows)
            else answered_but<PIECES>();
            meet();
            if (c + BUFS - 1 < nchunk) {                       // (into the place of chunk c - 1, which all waves are done with)
                request_w(fill);
                request_x(fill);
                fill = fill == (BUFS - 1) * BUF ? 0 : fill + BUF;
            }
            const uint32_t wu = take + uint32_t((wave >> 1) * XUNIT + (wave & 1) * 512) + slot, xu = take + 2 * XUNIT + slot;
            bf16x8 wf[4], xf[NB][4];
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                wf[ks] = *reinterpret_cast<const bf16x8*>(lds_raw + wu + ks * 32);
#pragma unroll
                for (int b = 0; b < NB; ++b) xf[b][ks] = *reinterpret_cast<const bf16x8*>(lds_raw + xu + b * 512 + ks * 32);
            }
#pragma unroll
            for (int ks = 0; ks < 4; ++ks)
#pragma unroll
                for (int b = 0; b < NB; ++b) acc[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[ks], xf[b][ks], acc[b], 0, 0, 0);
            take = take == (BUFS - 1) * BUF ? 0 : take + BUF;
        }
    };
    if (rows > 32) multiply(std::integral_constant<int, 2>{});
    else multiply(std::integral_constant<int, 1>{});
    // lane: features n .. + 15 of row 32 b + q
    const int n = n0 + wave * 32 + 16 * hk;
    if (n >= N) return;
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        if (32 * b + q >= rows) continue;
        bf16_t* const to = out + size_t(row0 + 32 * b + q) * N + n;
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            const f32x16& v = acc[b];
            u32x4 o = {pack_bf16x2(v[8 * p + 0], v[8 * p + 1]), pack_bf16x2(v[8 * p + 2], v[8 * p + 3]), pack_bf16x2(v[8 * p + 4], v[8 * p + 5]), pack_bf16x2(v[8 * p + 6], v[8 * p + 7])};
            if (RELU) { o.x = relu_bf16x2(o.x); o.y = relu_bf16x2(o.y); o.z = relu_bf16x2(o.z); o.w = relu_bf16x2(o.w); }
            *reinterpret_cast<u32x4*>(to + p * 8) = o;
        }
    }
}

// The expert layers for crowded experts (the rule stands where it is applied): one workgroup per CU that stays for the launch and sees its tiles as one stream
// of K-chunks (but for the last four of a die, where they leave ahead of the others).  Chunks of 64 channels go from memory straight into LDS, one or two of them ahead, across the border of one tile to the next: the pipeline does
// not run dry for a tile's first chunk or while its results leave, and a chunk costs one barrier.  A whole tile has 256 rows and 256 features, so that an
// expert's weights and rows enter a CU at 31 bytes for every clock of its matrix instructions (k_grouped_gemm's tiles of 64 rows: 78; the L2 gives a CU
// 64 a clock, 135 GB/s, to copies of 128 bytes of a row at a time, and memory all of them 6.3 TB/s, one alone 58 GB/s, with two chunks in flight or
// four); an expert's remaining rows, up to 128, are another kind, a stream of weights with two chunks ahead.  18 workgroups of a die begin with the
// whole tiles, 14 with the rests: products beside the stream (one kind after the other on all CUs: 950 us a layer of 16384 tokens, 1024 experts, instead of 900).
// What bounds it: whole tiles, the matrix instructions at the clock the card grants (16384 tokens, d 1024, h 2048, 16 experts, 4 uses: 0.92 PFLOP/s the
// pass, k_grouped_gemm 0.68); the others, memory, where results that are written cost the reading six times their bytes (4 GiB of weights alone in 675
// us, with 64 MB of results 737).
// The sums are k_grouped_gemm's bit for bit: 32x32x16 MFMAs over the channels in the same order.
constexpr int XIDX = 18 * XUNIT;                               // behind the chunks (2 of 8 units, 3 of 6): the rows' places in `gather`, two tiles'
constexpr int XLIST = XIDX + 2 * XR * 4, XLIST_LEN = 512;      // ... and the workgroup's next tiles
constexpr int X_LDS = XLIST + XLIST_LEN * 16;
constexpr int X_GRID = StreamDeal::WORKGROUPS;

template <bool RELU>
__global__ __launch_bounds__(512, 1) void k_grouped_stream(const bf16_t* __restrict__ in, const bf16_t* __restrict__ W, bf16_t* __restrict__ out,
                                                           const RowTile* __restrict__ tiles, const int32_t* __restrict__ n_tiles, int max_tiles,
                                                           int N, int K, int nt, const int32_t* __restrict__ gather, uint32_t m_kdiv, int once)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, q = lane & 31, hk = lane >> 5;
    const int fg = wave & 3, rg = wave >> 2;                   // this wave: features 64 fg .. of a tile, the first or second half of its rows
    const int nchunk = K / 64;
    const int die = blockIdx.x & 7, slot = blockIdx.x >> 3;

    // ---- where things lie in LDS: wave w copies block w of every unit
    const int s_q = copied_row(wave, lane);
    const uint32_t x_slot = fragment_at(q, hk);
    // accumulator row 8 b + 4 h + c of lane half h is given feature 16 h + 4 b + c: a lane ends up with 16 consecutive features of a row
    const int x_row = (lane >> 5) * 32 + s_q, w_row = (lane >> 5) * 32 + (s_q >> 2 & 1) * 16 + (s_q >> 3) * 4 + (s_q & 3);
    const size_t w_unit = size_t(K) * 128;                     // bytes from one unit of features to the next
    const uint32_t piece = uint32_t(lane & 7) * 16u, w_off = uint32_t(w_row) * uint32_t(K) * 2u + piece;

    struct Tile { int expert, row0, rows, nb; bool once; };
    // this workgroup's tiles of one kind, of up to ROWS rows, BUFS chunks in LDS; find(s): the tile's place in `tiles` and its feature tile
    auto run = [&](auto rows_const, auto bufs_const, const int count, auto&& find) {
        constexpr int ROWS = decltype(rows_const)::value, BUFS = decltype(bufs_const)::value, AHEAD = BUFS - 1;
        constexpr int RU = ROWS / 64, PIECES = 4 + RU;         // units of rows; of a chunk
        constexpr uint32_t BUF = uint32_t(PIECES * XUNIT);
        static_assert(BUFS * BUF <= uint32_t(XIDX) && ROWS <= XR && ROWS % 64 == 0, "room");
        if (count == 0) return;
        // where the tiles are is looked up for 512 of them at once (one at a time, it would be a trip to memory for each)
        auto list_tiles = [&](int s0) {
            if (s0 + tid < count) {
                const int2 at = find(s0 + tid);
                const RowTile t = tiles[at.x];
                *reinterpret_cast<u32x4*>(lds_raw + XLIST + tid * 16) = u32x4{uint32_t(t.expert), uint32_t(t.row0), uint32_t(t.rows), uint32_t(at.y * XF + (once & t.alone))};
            }
            answered_but<0>();
            meet();
        };
        auto tile_at = [&](int s) {
            const u32x4 v = *reinterpret_cast<const u32x4*>(lds_raw + XLIST + s % XLIST_LEN * 16);
            const int nb = int(__builtin_amdgcn_readfirstlane(v.w));
            return Tile{int(__builtin_amdgcn_readfirstlane(v.x)), int(__builtin_amdgcn_readfirstlane(v.y)), int(__builtin_amdgcn_readfirstlane(v.z)), nb & ~1,
                        (nb & 1) != 0};
        };
        uint32_t x_off[RU];
        bool x_on[RU];                                         // this lane's row is there (lane 0: always, so that every wave makes every request, which it counts)
        const char* w_next = nullptr;                          // weights of the chunk that is requested next
        const char* x_next = nullptr;
        int w_units = 0;                                       // ... that exist (the last one is copied again)
        bool w_once = false;
        uint32_t fill = 0, take = 0;                           // the chunk's place that is filled next, and the one that is read
        auto request_rows = [&](const Tile& t, int buf) {      // the places of a tile's rows
            if (gather && wave * 64 < t.rows)
                __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) uint32_t*)(gather + t.row0 + min(wave * 64 + lane, t.rows - 1)),
                                                 (__attribute__((address_space(3))) uint32_t*)(lds_raw + XIDX + buf * (XR * 4) + wave * 256), 4, 0, 0);
        };
        auto open = [&](const Tile& t, int buf) {
            w_next = reinterpret_cast<const char*>(W + (size_t(t.expert) * N + t.nb) * K);
            x_next = reinterpret_cast<const char*>(in);
            w_units = (N - t.nb) / 64;
            w_once = t.once;
#pragma unroll
            for (int i = 0; i < RU; ++i) {
                const int r = min(i * 64 + x_row, t.rows - 1);
                x_on[i] = i * 64 + x_row < t.rows || lane == 0;
                uint32_t row = uint32_t(t.row0 + r);
                if (gather) {
                    row = *reinterpret_cast<const uint32_t*>(lds_raw + XIDX + buf * (XR * 4) + r * 4);
                    if (m_kdiv) row = __umulhi(row, m_kdiv);   // / k
                }
                x_off[i] = row * uint32_t(K) * 2u + piece;
            }
        };
        auto request_piece = [&](int i) {
            const uint32_t at = fill + uint32_t(i * XUNIT + wave * XBLOCK);
            if (i < 4 && ROWS == XM && w_once) lds_copy16<true>(w_next + (i < w_units ? i : 0) * w_unit, w_off, at);
            else if (i < 4) lds_copy16(w_next + (i < w_units ? i : 0) * w_unit, w_off, at);
            else if (x_on[(i - 4) % RU]) lds_copy16(x_next, x_off[(i - 4) % RU], at);
        };
        auto requested = [&]() {
            w_next += 128;
            x_next += 128;
            fill = fill == AHEAD * BUF ? 0 : fill + BUF;
        };

        list_tiles(0);
        Tile now = tile_at(0);
        request_rows(now, 0);
        answered_but<0>();
        meet();
        open(now, 0);
        for (int c = 0; c < AHEAD; ++c) {
#pragma unroll
            for (int i = 0; i < PIECES; ++i) request_piece(i);
            requested();
        }
        int stores = 0;                                        // of this wave, behind the last tile's last request
#pragma unroll 1
        for (int s = 0; s < count; ++s) {
            if ((s + 1) % XLIST_LEN == 0 && s + 1 < count) list_tiles(s + 1);   // (all waves have met since they read the list's last)
            const Tile then = tile_at(min(s + 1, count - 1));
            const int rows = now.rows;
            const bool few = RU < 4 && rows <= 64, more = s + 1 < count;      // few: one block of 32 rows a wave
            const int first = few ? rg : rg * RU;              // this wave's first block
            const int mine = now.nb + fg * 64 < N ? max(0, min(few ? 1 : RU, (rows + 31) / 32 - first)) : 0;
            auto arrive = [&](int c) {                         // chunk c of this tile is there, and all waves are done with the one before
                if (c < AHEAD && stores > 0) {
                    constexpr int A = (AHEAD - 1) * PIECES;
                    if (stores >= 16) answered_but<A + 16>();
                    else if (stores >= 12) answered_but<A + 12>();
                    else if (stores >= 8) answered_but<A + 8>();
                    else answered_but<A + 4>();
                } else answered_but<(AHEAD - 1) * PIECES>();
                meet();
            };
            // the tile, with NB blocks for this wave
            auto work = [&](auto nb_const) {
                constexpr int NB = decltype(nb_const)::value;
                f32x16 acc[2][NB > 0 ? NB : 1];
#pragma unroll
                for (int a = 0; a < 2; ++a)
#pragma unroll
                    for (int b = 0; b < NB; ++b)
#pragma unroll
                        for (int i = 0; i < 16; ++i) acc[a][b][i] = 0.f;
                // products of the chunk at `take`, and the requests for another one under them
                auto chunk = [&](bool ask) {
                    const uint32_t wu = take + uint32_t(fg * XUNIT) + x_slot;
                    const uint32_t xu = take + uint32_t((4 + first / 2) * XUNIT + first % 2 * 512) + x_slot;
                    bf16x8 wf[2][2], xf[2][NB > 0 ? NB : 1];
                    auto read = [&](int ks) {
#pragma unroll
                        for (int a = 0; a < 2; ++a) wf[ks & 1][a] = *reinterpret_cast<const bf16x8*>(lds_raw + wu + (a * 512 + ks * 32));
#pragma unroll
                        for (int b = 0; b < NB; ++b) xf[ks & 1][b] = *reinterpret_cast<const bf16x8*>(lds_raw + xu + (b / 2 * XUNIT + b % 2 * 512 + ks * 32));
                    };
                    auto request = [&](int ks) {
                        if (ask && ks < 2) {
#pragma unroll
                            for (int i = ks * PIECES / 2; i < (ks + 1) * PIECES / 2; ++i) request_piece(i);
                        }
                        __builtin_amdgcn_sched_barrier(0);
                    };
                    if constexpr (NB == 0) { request(0); request(1); }
                    else {
                        if (RU < 4) { request(0); request(1); }           // (a stream of weights: first of all)
                        read(0);
                        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                        for (int ks = 0; ks < 4; ++ks)
#pragma unroll
                            for (int b = 0; b < NB; ++b) {
#pragma unroll
                                for (int a = 0; a < 2; ++a) acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[ks & 1][a], xf[ks & 1][b], acc[a][b], 0, 0, 0);
                                __builtin_amdgcn_sched_barrier(0);
                                if (b == 0 && ks < 3) {
                                    read(ks + 1);
                                    __builtin_amdgcn_sched_barrier(0);
                                }
                                if (RU == 4 && b == NB / 2) request(ks);
                            }
                    }
                    if (ask) requested();
                    take = take == AHEAD * BUF ? 0 : take + BUF;
                };
#pragma unroll 1
                for (int c = 0; c < nchunk - AHEAD; ++c) {
                    arrive(c);
                    if (c == 0 && more) request_rows(then, (s + 1) & 1);
                    chunk(true);
                }
                // (the places of its rows: asked for ahead of chunk 0's requests, and there when all have met for chunk AHEAD)
                if (nchunk < 2 * AHEAD + 1) { answered_but<0>(); meet(); }
                if (more) open(then, (s + 1) & 1);
#pragma unroll 1
                for (int c = nchunk - AHEAD; c < nchunk; ++c) {
                    if (more) arrive(c);
                    else { answered_but<0>(); meet(); }
                    chunk(more);
                }
#pragma unroll
                for (int b = 0; b < NB; ++b) {
                    const int r = (first + b) * 32 + q;
                    if (b < mine && r < rows) {
                        bf16_t* const to = out + size_t(now.row0 + r) * N + now.nb + fg * 64 + 16 * hk;
#pragma unroll
                        for (int a = 0; a < 2; ++a)
#pragma unroll
                            for (int p = 0; p < 2; ++p) {
                                const f32x16& v = acc[a][b];
                                u32x4 o = {pack_bf16x2(v[8 * p + 0], v[8 * p + 1]), pack_bf16x2(v[8 * p + 2], v[8 * p + 3]),
                                           pack_bf16x2(v[8 * p + 4], v[8 * p + 5]), pack_bf16x2(v[8 * p + 6], v[8 * p + 7])};
                                if (RELU) { o.x = relu_bf16x2(o.x); o.y = relu_bf16x2(o.y); o.z = relu_bf16x2(o.z); o.w = relu_bf16x2(o.w); }
                                *reinterpret_cast<u32x4*>(to + a * 32 + p * 8) = o;
                            }
                    }
                }
                // (an end of its own for every size: ends that the compiler has merged are reached from stores that only some lanes make, and what it
                // then takes for different from lane to lane is all of the state above)
                asm volatile("; %0" ::"n"(NB));
            };
            if constexpr (RU > 2) work(std::integral_constant<int, RU>{});
            else if (mine == 0) work(std::integral_constant<int, 0>{});
            else if (few) work(std::integral_constant<int, 1>{});
            else work(std::integral_constant<int, RU>{});
            stores = 4 * mine;
            now = then;
        }
        meet();                                                // (the other kind's chunks lie in the same place)
    };

    const int n_all = uniform_load(n_tiles);
    const StreamDeal deal(blockIdx.x, whole_tiles(n_all), rest_tiles(n_all), nt, K);
#pragma unroll 1
    for (int phase = 0; phase < 2; ++phase) {
        if (phase == deal.half) {
            run(std::integral_constant<int, XR>{}, std::integral_constant<int, 2>{}, deal.whole_count(), [&](int s) {
                const StreamDeal::Place at = deal.whole(s);
                return int2{at.row, at.column};
            });
        } else {
            run(std::integral_constant<int, XM>{}, std::integral_constant<int, 3>{}, deal.rest_count(), [&](int s) {
                const StreamDeal::Place at = deal.rest(s);
                return int2{max_tiles - 1 - at.row, at.column};
            });
        }
    }
}

size_t align256(size_t v) { return (v + 255) & ~size_t(255); }

struct Layout {
    size_t logits, topk_idx, topk_w, counts, offsets, tile_start, perm, inv, lrank, blockcnt, xs, hid, y, total;
    int nblk;
};

Layout layout(const moe_shape* s)
{
    Layout L;
    const size_t T = size_t(s->T), E = size_t(s->E), A = T * size_t(s->k);
    L.nblk = int((A + SORT_BLOCK - 1) / SORT_BLOCK);
    size_t o = 0;
    auto take = [&](size_t bytes) { size_t at = o; o += align256(std::max<size_t>(bytes, 4)); return at; };
    L.logits = take(T * E * 4);
    L.topk_idx = take(A * 4);
    L.topk_w = take(A * 4);
    L.counts = take(E * 4);
    L.offsets = take((E + 1) * 4);
    L.tile_start = take((E + 1) * 4);
    L.perm = take(A * 4);
    L.inv = take(A * 4);
    L.lrank = take(A * 4);
    L.blockcnt = take(E * size_t(std::max(L.nblk, 1)) * 4);
    L.xs = take(A * size_t(s->d) * 2);
    L.hid = take(A * size_t(s->h) * 2);
    L.y = take(A * size_t(s->d) * 2);
    L.total = o;
    return L;
}

// Which kernels a pass runs on: by its sizes, by its tensors' addresses (the kernels that copy straight into LDS ask for pieces of 16 bytes; registers are loaded from any
// address, by the others), and nothing else.
struct Choice {
    int T_big;                    // tokens of k_gate_big; the others' logits:
    bool gate_small, gate_stream; // k_gate_small, k_gate_stream or k_gate
    bool small, joined, mid;      // the grouping in one workgroup, in the selection's launch, in two launches, or (none) in five
    bool fused_permute;
    int skinny_tiles, stream_most;  // most row tiles
    bool streamed, few1, few2, skinny1, skinny2;  // k_grouped_stream, or k_grouped_few, k_grouped_skinny, k_grouped_gemm for the first and the second expert layer
    long long few_tiles(int N) const { return (long long)skinny_tiles * ((N + FEW_F - 1) / FEW_F); }
    bool tables() const { return streamed || few1 || few2 || skinny1 || skinny2; }   // of the row tiles, in the stacked tokens' room
};

Choice choose(const moe_shape* s, bool noisy, bool gate_on16, bool layers_on16, int naive_stride)
{
    const int T = s->T, d = s->d, h = s->h, E = s->E, k = s->k, A = T * k;
    Choice c = {};
    // whole tiles of 256 tokens go to k_gate_big where the expert and model widths allow it and there are enough tiles (a workgroup of
    // it has a CU for itself, and takes as long however few there are), the tokens behind the last whole tile (and every other shape)
    // to k_gate.  us, k_gate_big / k_gate by tiles and d:
    //   noisy: 32 x 512 22 / 13, 64 x 1024 31 / 22, 128 x 256 18.8 / 16.3, 128 x 512 23 / 22, 128 x 1024 32.5 / 33.7, 256 x 1024 43 / 62
    //   without noise: 32 x 512 12.4 / 11.3, 64 x 512 13.2 / 12.8, 64 x 1024 18.4 / 18.5, 96 x 512 14.0 / 15.4, 128 x 256 12.1 / 13.3, 128 x 1024
    //   20 / 27; 500 tokens, d 1024, 256 experts (2 tiles and a rest; k_gate_small): 45 / 11
    // The whole pass, noisy: 96 x 2048 143 / 140, 128 x 2048 142 / 150, 96 x 4096 249 / 249, 256 x 256 74 / 76; without noise: 16 x 4096 117 / 116,
    // 32 x 2048 77 / 77, 32 x 4096 134 / 139, 64 x 2048 102 / 105.  (Of 120 shapes of 8 to 512 tiles, d 256 to 4096, three go to the slower one by more
    // than 3 % of the pass, all without noise and by 2.8 us at most: 128 x 256 twice and 64 x 1024 in 4 x 16 tiles.)
    const size_t big_tiles = size_t(T / GB_TOK) * size_t(E / GB_EXP);
    const bool many_tiles = noisy ? big_tiles * (size_t(d) + 5120) >= 128 * 6144 : big_tiles * (size_t(d) + 1280) >= 64 * 2304;
    c.T_big = (many_tiles && E % GB_EXP == 0 && d % GKC == 0 && d >= 4 * GKC && size_t(GB_TOK) * size_t(std::max(E, d)) < (size_t(1) << 30))
                          ? T / GB_TOK * GB_TOK : 0;
    const int T_big = c.T_big;
    // up to some five 16 x 16 tiles per CU: the kernel with the small tiles.  us, k_gate / k_gate_small by the number of small tiles: d =
    // 1024, noisy: 500 21 / 11, 1008 20 / 18, 1764 21 / 25, 2000 21 / 31; without noise: 1000 15.5 / 12.8, 2000 16.4 / 20; d = 64: 1764
    // 8.8 / 10.2; d = 512, few tokens: 48 12 / 6.5
    c.gate_small = T_big == 0 && size_t((E + 15) / 16) * size_t((T + 15) / 16) <= 1200;
    // Of k_gate's tiles, those of whole K-chunks go to k_gate_stream: all of them without noise, and with noise as many as two workgroups a CU hold at once;
    // beyond that the five of k_gate hide more.  The whole pass in us, k_gate / k_gate_stream, by tiles and d: noisy 256 x 512 153.6 / 150.5, 306 x 576 300.0 / 298.2,
    // 222 x 768 101.1 / 97.6, 80 x 320 54.1 / 52.1, 376 x 192 47.5 / 47.6, and on the other side 518 x 192 79.2 / 80.5, 845 x 256 81.1 / 82.6, 2370 x 768 312 / 321; without
    // noise 90 x 384 62.1 / 59.0, 240 x 832 91.1 / 85.1, 430 x 128 38.2 / 36.8, 2057 x 448 191.3 / 186.2
    const long long tiles = (long long)((E + 63) / 64) * ((T - T_big + 63) / 64);
    c.gate_stream = !c.gate_small && T > T_big && d % 64 == 0 && d <= 1 << 20 && (!noisy || tiles <= 512) && gate_on16;
    // few uses, up to eight per token: the selection's last workgroup groups them (its counter lies where the ranks of many uses do), as long as the
    // selection has no more than 128 workgroups to count.  us a pass replayed from a graph, d = h = 64, a launch more / so, by tokens x experts, uses of a
    // token: 16 x 64, 2 20.0 / 17.7; 64 x 1024, 4 25.6 / 22.7; 128 x 256, 8 26.8 / 23.7; 256 x 64, 2 22.1 / 19.7; 512 x 256, 2 23.9 / 22.9; 512 x 2048,
    // 2 34.9 / 32.7; 1024 x 64, 1 24.2 / 25.4; 1024 x 1024, 1 28.8 / 29.6
    const bool small = c.small = A <= SMALL_USES && E <= SMALL_EXPERTS;
    c.joined = small && k <= MAX_K && E <= 32 * 64 && T > T_big && T <= 512;
    // the tokens are stacked inside the first expert layer's operand load (token perm[pos] / k for sorted position pos), or
    // by a kernel of its own (MOE_SEPARATE_PERMUTE, and for the per-use loop)
    const bool fused_permute = c.fused_permute = !(s->flags & MOE_SEPARATE_PERMUTE) && naive_stride <= 0;
    // m3 stable counting sort: few uses in one workgroup, more in two launches, beyond that in five.
    // An expert layer of few tiles and long sums that k_grouped_few (below) does not take runs on k_grouped_skinny, each layer for itself.  k_grouped_gemm pays 1.2 to 1.5 us for
    // every 64 summed channels however few tiles there are.  k_grouped_skinny reads an expert's weights once per row tile, and where a tile
    // has many rows, every wave multiplies up to four fragments of them with each of the weights.  us, k_grouped_gemm / k_grouped_skinny, by
    // features x summed channels and rounds of 768 workgroups (three a CU):
    //   a layer of few rows a tile: 256 x 2048 0.1: 30 / 15;  768 x 2048 0.9: 47 / 29;  256 x 1024 0.1: 18 / 11, 0.6: 20 / 14;
    //     512 x 1024 0.25: 21 / 12;  256 x 512 0.7: 13.4 / 9.3;  240 x 432 0.2: 12 / 8.6;  128 x 216 0.6: 10.4 / 8.8;  512 x 512 1.4: 16 / 24;
    //     2048 x 512 2.0: 18 / 31;  1024 x 256 1.4: 10 / 20;  192 x 320 1.2: 15 / 23;  128 x 192 0.6: 10.3 / 14;  128 x 128 0.5: 7.5 / 10
    //   a layer of few uses, 20 to 45 rows a tile: 1728 x 128 0.2: 6.4 / 4.8;  256 x 200 0.15: 7.8 / 5.2;  528 x 200 0.15: 8.0 / 4.2
    //   the whole pass, 43 to 64 rows a tile: 512 x 2048 0.4: 69 / 62, 2.75: 160 / 200;  1024 x 4096 0.5: 133 / 103, 0.75: 122 / 124, 1.5: 171 / 197;
    //     512 x 1024 0.75: 55 / 58;  1024 x 2048 1.5: 103 / 116, 2.8: 154 / 187;  1024 x 8192 21: 3076 / 4253
    //   one token, 160 x 184: 21.5 / 24.3 the pass (a few workgroups of short sums pay for their start)
    // (4646 passes of 64 to 2048 x 64 to 4096 channels and up to 65536 uses take 1.3 % longer than with the better kernel for each layer, in the
    // mean, and 26 % at worst; with the first limit alone, whatever the rows, 1.8 and 90 %.)
    // The tiles' table takes the room of the stacked tokens, which no kernel writes then (at most one tile per use, 16 bytes
    // each like the smallest token).
    const bool mid = c.mid = !small && E <= SMALL_EXPERTS && A <= MID_BLOCKS * 1024;
    const int skinny_tiles = c.skinny_tiles = std::min(A, std::min(A, E) + A / TM);     // at least as many row tiles as there are
    auto skinny_layer = [&](int N, int K) {
        const long long groups = (long long)skinny_tiles * ((N + 63) / 64), rows16 = A / (16ll * skinny_tiles);
        if (!(small || mid) || !fused_permute) return false;
        // few uses, 16 rows a tile and more: 0.1 to 0.25 rounds also of short sums
        if (small && rows16 >= 1 && K >= 96 && groups * 10 >= 768 && groups * 4 <= 768) return true;
        // rounds <= (K - 128) / 600 and 3; from 32 rows a tile 0.3 (few uses: 0.4), with long sums (K - 128) / 2560, at most 0.8
        const long long most = rows16 < 2 ? 3 * 768 : std::max(small ? 307ll : 230ll, std::min(614ll, (K - 128) * 3ll / 10));
        return groups * 600 <= 768ll * (K - 128) && groups <= most && (K >= 224 || A >= 128 || groups * 5 >= 768);
    };
    c.stream_most = std::min(A, E + A / XR);           // at least as many tiles of k_grouped_stream as there are
    // Crowded experts, 64 uses each and more in the mean, and products for a tile of 256 x 256 on every CU and more (2^24 = 256 of them, both layers
    // together): k_grouped_stream.  Its tiles are few and large: where k_grouped_few can take the layers (up to 65536 uses), from 384 features on, which fill 256 + 128, and from
    // 2^33 products a layer.  The whole pass, others / so in us: k_grouped_gemm, by mean uses of an expert and tiles: 2250, 692: 204 / 157;
    // 3870, 1180: 288 / 217; 541, 1087: 343 / 271; 788, 863: 192 / 139; 553, 422: 103 / 92; 508, 283: 78 / 67; 370, 2430: 660 / 553; 116, 291: 154 / 136; 99, 525: 171 /
    // 164; 64, 3072 (Zipf 1.2): 2010 / 1930; 152, 372: 91 / 94; and on the other side of the line 1190, 167: 51 / 55; 187, 135: 48 / 55; 399, 38: 40 / 49; 48, 561: 313 /
    // 312; 63, 1127: 444 / 450; 37, 395: 301 / 303; 32, 192: 153 / 159.  k_grouped_few, by uses, experts, d x h: 20216, 54, 1536 x 384: 126 / 122; 15200, 7, 1600 x 768:
    // 96 / 91; 10902, 54, 448 x 1280: 117 / 106; 17964, 22, 1792 x 1536 400 / 266; and on the other side 6435, 2, 512 x 3072 82 / 120; 7906, 16, 384 x 1792 66 / 81; 17965, 4, 448 x
    // 896 80 / 91; 13256, 119, 320 x 2112 97 / 109; 28110, 3, 256 x 1920 121 / 129 (of 70 shapes within the old line 19 were faster with k_grouped_few, all others 2 to 50 % slower)
    const bool streamed = c.streamed = fused_permute && layers_on16 && naive_stride <= 0 && !small && d % 64 == 0 && h % 64 == 0 && d >= 256 && h >= 256 && E <= SMALL_EXPERTS && A < 1 << 22 && k <= 1024 &&
                        size_t(A) * size_t(std::max(d, h)) < size_t(1) << 31 && A >= 64 * E && size_t(A) * size_t(d + h) >= size_t(1) << 24 &&
                        (!mid || (std::min(d, h) >= 384 && double(A) * d * h >= double(1ll << 33)));
    // All other layers of whole K-chunks whose row tiles have a table (up to 65536 uses and 4096 experts): k_grouped_few, but for single chunks of few rows a tile
    // (where it saves no trip to memory), and long sums in a fraction of a tile for every fourth CU (a CU alone gets 58 GB/s: k_grouped_skinny has half the features).  Three chunks
    // in LDS, two workgroups a CU, where that holds all of them and for long sums, else two chunks and three workgroups.  112 passes over 4 to 32768 tokens, 2 to 2048
    // experts, 64 to 4096 channels, uniform and skewed, take 0.82 of the time in the geometric mean, 0.59 to 1.00 (always two chunks: 1.02 times as long as so, up to 1.23; always three 1.02, up to 1.13).  us a
    // pass, before / so, by tokens x experts, uses, d x h: 37 x 256, 2, 512 x 1024 31.0 / 25.4; 4096 x 256, 2, 512 x 1024 86 / 80; 86 x 72, 1, 1856 x 1344 73 / 43;
    // 542 x 51, 4, 896 x 256 54 / 36; 13879 x 184, 4, 64 x 640 98 / 72; 22 x 38, 4, 64 x 192 21.7 / 19.5; 15959 x 1631, 4, 448 x 512 469 / 446; what is left out: one chunk of few
    // rows, 4811 x 1394, 1, 64 x 3904 279 / 286; few tiles of long sums, 55 x 57, 2, 128 x 3776 42.0 / 43.9
    auto few_layer = [&](int N, int K) {
        return (small || mid) && fused_permute && naive_stride <= 0 && !streamed && layers_on16 && N % 64 == 0 && K % 64 == 0 && size_t(A) * size_t(std::max(N, K)) < size_t(1) << 31 && K <= 1 << 20 &&
               (K >= 128 || A >= 16ll * skinny_tiles) && (c.few_tiles(N) >= 64 || K < 2560);
    };
    c.few1 = few_layer(h, d);
    c.few2 = few_layer(d, h);
    c.skinny1 = !streamed && !c.few1 && skinny_layer(h, d);
    c.skinny2 = !streamed && !c.few2 && skinny_layer(d, h);
    return c;
}

bool on16(std::initializer_list<const void*> pointers)
{
    for (const void* at : pointers)
        if (reinterpret_cast<uintptr_t>(at) & 15) return false;
    return true;
}

int check_shape(const moe_shape* s, const char* who)
{
    if (!s) return fail(DYNB_E_INVAL, std::string(who) + ": NULL shape");
    if (size_t(s->T) > size_t(65535) * 64) return fail(DYNB_E_UNSUPPORTED, std::string(who) + ": more than 4194240 tokens");
    if (s->T < 0 || s->d <= 0 || s->h <= 0 || s->E <= 0 || s->k <= 0)
        return fail(DYNB_E_INVAL, std::string(who) + ": sizes must be positive");
    if (s->k > s->E) return fail(DYNB_E_INVAL, std::string(who) + ": k > E");
    if (s->d % 8 || s->h % 8)
        return fail(DYNB_E_UNSUPPORTED, std::string(who) + ": d and h must be multiples of 8 (rows are moved in 16-byte pieces)");
    if (s->dtype != DYNB_BF16) return fail(DYNB_E_UNSUPPORTED, std::string(who) + ": only bf16");
    if (s->flags & ~uint32_t(MOE_SEPARATE_PERMUTE)) return fail(DYNB_E_UNSUPPORTED, std::string(who) + ": unknown flag bits");
    if (size_t(s->T) * size_t(s->k) >= (size_t(1) << 30) || size_t(s->T) * size_t(s->E) >= (size_t(1) << 40))
        return fail(DYNB_E_UNSUPPORTED, std::string(who) + ": too many expert uses");
    // the grouped expert layers launch one workgroup per (row tile, feature tile): at most ceil(A/TM) + E row tiles
    const long long max_mtiles = ((long long)s->T * s->k + TM - 1) / TM + s->E;
    const long long nt = (std::max(s->h, s->d) + TN - 1) / TN;
    if (max_mtiles * nt + 8ll * XCD_CHUNK >= (1ll << 31)) return fail(DYNB_E_UNSUPPORTED, std::string(who) + ": grid too large");
    return DYNB_OK;
}

}  // namespace

extern "C" size_t moe_workspace_bytes(const moe_shape* s)
{
    if (check_shape(s, "moe_workspace_bytes") != DYNB_OK) return 0;
    return std::max<size_t>(layout(s).total, 256);
}

__global__ void k_unit_group(int32_t* p)      // offsets {0,1} and tile table {0,1} of a one-row group
{
    if (threadIdx.x < 4) p[threadIdx.x] = threadIdx.x & 1;
}

// naive_stride = 0: batched layer.  naive_stride >= 1: the expert stage is run one use at a time
// (every naive_stride-th use), which needs the group sizes on the host.
static int moe_run(const moe_shape* s, const void* x, const void* Wg, const void* Wn, const float* noise,
                   const void* W1, const void* W2, void* out, const moe_aux* aux, void* workspace,
                   size_t workspace_bytes, void* stream, int naive_stride)
{
    int rc = check_shape(s, "moe_forward");
    if (rc != DYNB_OK) return rc;
    if (s->T == 0) return DYNB_OK;
    if (!x || !Wg || !W1 || !W2 || !out || !workspace) return fail(DYNB_E_INVAL, "moe_forward: NULL argument");
    if (noise && !Wn) return fail(DYNB_E_INVAL, "moe_forward: noise given without Wn");
    const Layout L = layout(s);
    if (workspace_bytes < L.total) return fail(DYNB_E_WORKSPACE, "moe_forward: workspace too small");
    if (reinterpret_cast<uintptr_t>(workspace) & 255) return fail(DYNB_E_INVAL, "moe_forward: workspace not 256-byte aligned");
    hipStream_t st = static_cast<hipStream_t>(stream);
    char* ws = static_cast<char*>(workspace);
    const int T = s->T, d = s->d, h = s->h, E = s->E, k = s->k, A = T * k;

    float* logits = (aux && aux->logits) ? aux->logits : reinterpret_cast<float*>(ws + L.logits);
    int32_t* topk_idx = (aux && aux->topk_idx) ? aux->topk_idx : reinterpret_cast<int32_t*>(ws + L.topk_idx);
    float* topk_w = (aux && aux->topk_w) ? aux->topk_w : reinterpret_cast<float*>(ws + L.topk_w);
    int32_t* counts = (aux && aux->counts) ? aux->counts : reinterpret_cast<int32_t*>(ws + L.counts);
    int32_t* offsets = (aux && aux->offsets) ? aux->offsets : reinterpret_cast<int32_t*>(ws + L.offsets);
    int32_t* perm = (aux && aux->perm) ? aux->perm : reinterpret_cast<int32_t*>(ws + L.perm);
    int32_t* inv = (aux && aux->inv) ? aux->inv : reinterpret_cast<int32_t*>(ws + L.inv);
    int32_t* tile_start = reinterpret_cast<int32_t*>(ws + L.tile_start);
    int32_t* lrank = reinterpret_cast<int32_t*>(ws + L.lrank);
    int32_t* blockcnt = reinterpret_cast<int32_t*>(ws + L.blockcnt);
    bf16_t* xs = reinterpret_cast<bf16_t*>(ws + L.xs);
    bf16_t* hid = reinterpret_cast<bf16_t*>(ws + L.hid);
    bf16_t* y = reinterpret_cast<bf16_t*>(ws + L.y);
    const bf16_t* xb = static_cast<const bf16_t*>(x);

    const Choice c = choose(s, noise != nullptr, on16({x, Wg, noise ? Wn : nullptr}), on16({x, W1, W2}), naive_stride);
    const bool joined = c.joined, small = c.small, mid = c.mid, fused_permute = c.fused_permute, streamed = c.streamed;
    const int T_big = c.T_big, skinny_tiles = c.skinny_tiles, stream_most = c.stream_most;

    const bool timed = dynb::timing_on();
    if (timed) dynb::timing_begin(st);
    // m1 gate
    if (T_big > 0) {
        static std::atomic<uint64_t> attr_set{0};             // one bit per device: LDS beyond 64 KB
        int dev = 0;
        HIP_TRY(hipGetDevice(&dev), "hipGetDevice");
        if (!(attr_set.load() >> (dev & 63) & 1)) {
            HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(k_gate_big<true>), hipFuncAttributeMaxDynamicSharedMemorySize, GB_LDS_BYTES),
                    "hipFuncSetAttribute(k_gate_big)");
            HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(k_gate_big<false>), hipFuncAttributeMaxDynamicSharedMemorySize, GB_LDS_BYTES),
                    "hipFuncSetAttribute(k_gate_big)");
            attr_set.fetch_or(uint64_t(1) << (dev & 63));
        }
        const int ntt = T_big / GB_TOK, net = E / GB_EXP, per_die = (ntt + 7) / 8;
        const dim3 grid(unsigned(8 * per_die * net));
        if (noise)
            hipLaunchKernelGGL((k_gate_big<true>), grid, dim3(256), GB_LDS_BYTES, st, xb, static_cast<const bf16_t*>(Wg),
                               static_cast<const bf16_t*>(Wn), noise, logits, T_big, d, E, ntt, net, per_die);
        else
            hipLaunchKernelGGL((k_gate_big<false>), grid, dim3(256), GB_LDS_BYTES, st, xb, static_cast<const bf16_t*>(Wg),
                               static_cast<const bf16_t*>(Wn), noise, logits, T_big, d, E, ntt, net, per_die);
    }
    int32_t* const done = joined ? lrank : nullptr;
    if (c.gate_small)
        hipLaunchKernelGGL(k_gate_small, dim3((E + 15) / 16, (T + 15) / 16), dim3(256), 0, st, xb, static_cast<const bf16_t*>(Wg),
                           static_cast<const bf16_t*>(Wn), noise, logits, T, d, E, done);
    else if (c.gate_stream) {
        static std::atomic<uint64_t> attr_set{0};             // one bit per device: LDS beyond 64 KB
        int dev = 0;
        HIP_TRY(hipGetDevice(&dev), "hipGetDevice");
        if (!(attr_set.load() >> (dev & 63) & 1)) {
            for (const void* f : {reinterpret_cast<const void*>(k_gate_stream<true>), reinterpret_cast<const void*>(k_gate_stream<false>)})
                HIP_TRY(hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, GS_LDS), "hipFuncSetAttribute(k_gate_stream)");
            attr_set.fetch_or(uint64_t(1) << (dev & 63));
        }
        hipLaunchKernelGGL(noise ? k_gate_stream<true> : k_gate_stream<false>, dim3((E + 63) / 64, (T - T_big + 63) / 64), dim3(256),
                           noise ? GS_LDS : GS_LDS / 3 * 2, st, xb + size_t(T_big) * d,
                           static_cast<const bf16_t*>(Wg), static_cast<const bf16_t*>(Wn), noise ? noise + size_t(T_big) * E : nullptr,
                           logits + size_t(T_big) * E, T - T_big, d, E, done);
    } else if (T > T_big)
        hipLaunchKernelGGL(k_gate, dim3((E + 63) / 64, (T - T_big + 63) / 64), dim3(256), 0, st, xb + size_t(T_big) * d,
                           static_cast<const bf16_t*>(Wg), static_cast<const bf16_t*>(Wn), noise ? noise + size_t(T_big) * E : nullptr,
                           logits + size_t(T_big) * E, T - T_big, d, E, done);
    if (timed) dynb::timing_mark(st, dynb::ST_GATE, 0);
    RowTile* const tiles = c.tables() ? reinterpret_cast<RowTile*>(xs) : nullptr;
    // m2 top-k + softmax
    const dim3 tk_grid((T + 3) / 4), tk_block(256);
    if (joined) {
        auto* const kernel = E <= 4 * 64 ? k_topk_group<4> : E <= 16 * 64 ? k_topk_group<16> : k_topk_group<32>;
        hipLaunchKernelGGL(kernel, tk_grid, tk_block, 0, st, logits, topk_idx, topk_w, T, E, k, done, counts, offsets, tile_start, perm, inv, tiles, skinny_tiles);
    } else if (k <= MAX_K && E <= 4 * 64)
        hipLaunchKernelGGL((k_topk_small<4>), tk_grid, tk_block, 0, st, logits, topk_idx, topk_w, T, E, k);
    else if (k <= MAX_K && E <= 16 * 64)
        hipLaunchKernelGGL((k_topk_small<16>), tk_grid, tk_block, 0, st, logits, topk_idx, topk_w, T, E, k);
    else if (k <= MAX_K && E <= 32 * 64)
        hipLaunchKernelGGL((k_topk_small<32>), tk_grid, tk_block, 0, st, logits, topk_idx, topk_w, T, E, k);
    else if (E <= 4 * 64)
        hipLaunchKernelGGL((k_topk<4>), tk_grid, tk_block, 0, st, logits, topk_idx, topk_w, T, E, k);
    else if (E <= 16 * 64)
        hipLaunchKernelGGL((k_topk<16>), tk_grid, tk_block, 0, st, logits, topk_idx, topk_w, T, E, k);
    else if (E <= 32 * 64)
        hipLaunchKernelGGL((k_topk<32>), tk_grid, tk_block, 0, st, logits, topk_idx, topk_w, T, E, k);
    else
        hipLaunchKernelGGL((k_topk<0>), tk_grid, tk_block, 0, st, logits, topk_idx, topk_w, T, E, k);
    if (timed) dynb::timing_mark(st, dynb::ST_TOPK, 0);
    if (joined) {
    } else if (small) {
        hipLaunchKernelGGL(k_group_small, dim3(1), dim3(1024), 0, st, topk_idx, counts, offsets, tile_start, perm, inv, tiles,
                           skinny_tiles, A, E);
    } else if (mid) {
        const int nblk = (A + 1023) / 1024;                    // (a quarter of the blocks that blockcnt has room for; a single expert's rows of four counts fill that)
        hipLaunchKernelGGL(k_rank_wide, dim3(nblk), dim3(256), 0, st, topk_idx, lrank, blockcnt, A, E);
        auto* const place = E <= 1024 ? (streamed ? k_place_wide<4, true> : k_place_wide<4, false>) : streamed ? k_place_wide<8, true> : k_place_wide<8, false>;
        hipLaunchKernelGGL(place, dim3(nblk), dim3(E <= 1024 ? 256 : 512), 0, st, topk_idx, lrank, blockcnt,
                           counts, offsets, tile_start, perm, inv, tiles, streamed ? stream_most : skinny_tiles, A, E, nblk);
    } else {
        const size_t nbc = size_t(E) * L.nblk;
        hipLaunchKernelGGL(k_zero_i32, dim3(unsigned(std::min<size_t>((nbc + 255) / 256, 2048))), dim3(256), 0, st, blockcnt, nbc);
        hipLaunchKernelGGL(k_rank_blocks, dim3(L.nblk), dim3(SORT_BLOCK), 0, st, topk_idx, lrank, blockcnt, A, L.nblk);
        hipLaunchKernelGGL(k_scan_blocks, dim3((E + 3) / 4), dim3(256), 0, st, blockcnt, counts, E, L.nblk);
        hipLaunchKernelGGL(streamed ? k_offsets<true> : k_offsets<false>, dim3(1), dim3(OFFS_THREADS), 0, st, counts, offsets, tile_start, E);
        hipLaunchKernelGGL(streamed ? k_place<true> : k_place<false>, dim3(L.nblk), dim3(SORT_BLOCK), 0, st, topk_idx, lrank, blockcnt, offsets, perm, inv, A,
                           L.nblk, tile_start, tiles, stream_most, E);
    }
    if (timed) dynb::timing_mark(st, dynb::ST_SORT, 0);
    // m4 permute
    if (!fused_permute) hipLaunchKernelGGL(k_permute, dim3((T + 3) / 4), dim3(256), 0, st, xb, inv, xs, T, d, k);
    if (timed) dynb::timing_mark(st, dynb::ST_PERMUTE, 0);
    // m5 grouped expert FFN: at most ceil(A/TM) + E row tiles exist
    const long long max_mtiles = (long long)(A + TM - 1) / TM + E;
    const int nt1 = (h + TN - 1) / TN, nt2 = (d + TN - 1) / TN;
    const long long span = 8ll * XCD_CHUNK;                   // every XCD's longest run
    if (streamed) {
        static std::atomic<uint64_t> attr_set{0};             // one bit per device
        int dev = 0;
        HIP_TRY(hipGetDevice(&dev), "hipGetDevice");
        if (!(attr_set.load() >> (dev & 63) & 1)) {
            for (const void* f : {reinterpret_cast<const void*>(k_grouped_stream<true>), reinterpret_cast<const void*>(k_grouped_stream<false>)})
                HIP_TRY(hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, X_LDS), "hipFuncSetAttribute(k_grouped_stream)");
            attr_set.fetch_or(uint64_t(1) << (dev & 63));
        }
        // Where a layer's weights are more than the memory side's cache holds (256 MB), those of an expert with a single tile pass by the caches.  The whole pass, without / so, by
        // weights of a layer: 245 MiB 309 / 309 us (less than the cache, and all experts' rests so: 53 MB 134 / 157, 76 MB 102 / 122); 304 241 / 214; 504 252 / 227; 569 188 / 180; 894 650 / 651;
        // 4096 1877 / 1849 (with all rests so, those of experts with whole tiles too: 569 188 / 200, 322 217 / 227 instead of 204)
        const int once = size_t(E) * d * h >= size_t(1) << 27;
        hipLaunchKernelGGL((k_grouped_stream<true>), dim3(X_GRID), dim3(512), X_LDS, st, xb, static_cast<const bf16_t*>(W1), hid, tiles, tile_start + E,
                           stream_most, h, d, (h + XF - 1) / XF, perm, k > 1 ? 0xffffffffu / uint32_t(k) + 1u : 0u, once);
        if (timed) dynb::timing_mark(st, dynb::ST_FFN1, 0);
        hipLaunchKernelGGL((k_grouped_stream<false>), dim3(X_GRID), dim3(512), X_LDS, st, hid, static_cast<const bf16_t*>(W2), y, tiles, tile_start + E,
                           stream_most, d, h, (d + XF - 1) / XF, nullptr, 0u, once);
        if (timed) dynb::timing_mark(st, dynb::ST_FFN2, 0);
    } else if (naive_stride <= 0) {
        if (c.few1 || c.few2) {
            static std::atomic<uint64_t> attr_set{0};         // one bit per device
            int dev = 0;
            HIP_TRY(hipGetDevice(&dev), "hipGetDevice");
            if (!(attr_set.load() >> (dev & 63) & 1)) {
                for (const void* f : {reinterpret_cast<const void*>(k_grouped_few<true, 3>), reinterpret_cast<const void*>(k_grouped_few<false, 3>)})
                    HIP_TRY(hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, few_lds(3)), "hipFuncSetAttribute(k_grouped_few)");
                attr_set.fetch_or(uint64_t(1) << (dev & 63));
            }
        }
        auto few = [&](auto relu, const bf16_t* from, const void* W, bf16_t* to, int N, int K, const int32_t* rows_at) {
            const long long all = c.few_tiles(N);
            const bool three = all <= 512 || K >= 1024;
            // (tiles dealt to an XCD at once: sixteen, or as many as leave all eight eight turns)
            const int chunk = int(std::min(16ll, std::max(1ll, all / 64))), nt = (N + FEW_F - 1) / FEW_F;
            hipLaunchKernelGGL((three ? k_grouped_few<decltype(relu)::value, 3> : k_grouped_few<decltype(relu)::value, 2>),
                               dim3(unsigned((all + 8 * chunk - 1) / (8 * chunk) * (8 * chunk))), dim3(256), few_lds(three ? 3 : 2), st, from,
                               static_cast<const bf16_t*>(W), to, tiles, skinny_tiles, chunk, N, K, nt, rows_at,
                               k > 1 ? 0xffffffffu / uint32_t(k) + 1u : 0u);   // (exact: places below 65536, and k no more)
        };
        if (c.few1) few(std::true_type{}, xb, W1, hid, h, d, perm);
        else if (c.skinny1)
            hipLaunchKernelGGL((k_grouped_skinny<true>), dim3(unsigned(skinny_tiles * ((h + 63) / 64))), dim3(256), 0, st, xb,
                               static_cast<const bf16_t*>(W1), hid, tiles, h, d, (h + 63) / 64, perm, k);
        else
            hipLaunchKernelGGL((k_grouped_gemm<true>), dim3(unsigned((max_mtiles * nt1 + span - 1) / span * span)), dim3(256), 0, st,
                               fused_permute ? xb : xs, static_cast<const bf16_t*>(W1), hid, offsets, tile_start, E, h, d, nt1,
                               fused_permute ? perm : nullptr, k);
        if (timed) dynb::timing_mark(st, dynb::ST_FFN1, 0);
        if (c.few2) few(std::false_type{}, hid, W2, y, d, h, nullptr);
        else if (c.skinny2)
            hipLaunchKernelGGL((k_grouped_skinny<false>), dim3(unsigned(skinny_tiles * ((d + 63) / 64))), dim3(256), 0, st, hid,
                               static_cast<const bf16_t*>(W2), y, tiles, d, h, (d + 63) / 64, nullptr, 1);
        else
            hipLaunchKernelGGL((k_grouped_gemm<false>), dim3(unsigned((max_mtiles * nt2 + span - 1) / span * span)), dim3(256), 0, st,
                               hid, static_cast<const bf16_t*>(W2), y, offsets, tile_start, E, d, h, nt2, nullptr, 1);
        if (timed) dynb::timing_mark(st, dynb::ST_FFN2, 0);
    } else {
        // the paper's naive version: loop over the k*b expert uses, one expert call (two layers) per use; where the tiles are more than
        // a run for every XCD, the runs are rounded up one by one, and the grid has to be whole runs
        auto unit_grid = [&](int nt) { return dim3(unsigned(nt <= span ? (nt + 7) / 8 * 8 : (nt + span - 1) / span * span)); };
        std::vector<int32_t> off(size_t(E) + 1);
        int32_t* unit = lrank;                                // free again after k_place
        hipLaunchKernelGGL(k_unit_group, dim3(1), dim3(64), 0, st, unit);
        HIP_TRY(hipMemcpyAsync(off.data(), offsets, off.size() * sizeof(int32_t), hipMemcpyDeviceToHost, st), "moe_forward_naive");
        HIP_TRY(hipStreamSynchronize(st), "moe_forward_naive");
        const bf16_t* w1 = static_cast<const bf16_t*>(W1);
        const bf16_t* w2 = static_cast<const bf16_t*>(W2);
        for (int e = 0; e < E; ++e)
            for (int pos = off[e]; pos < off[e + 1]; ++pos) {
                if (pos % naive_stride) continue;
                hipLaunchKernelGGL((k_grouped_gemm<true>), unit_grid(nt1), dim3(256), 0, st, xs + size_t(pos) * d,
                                   w1 + size_t(e) * h * d, hid + size_t(pos) * h, unit, unit + 2, 1, h, d, nt1, nullptr, 1);
                hipLaunchKernelGGL((k_grouped_gemm<false>), unit_grid(nt2), dim3(256), 0, st, hid + size_t(pos) * h,
                                   w2 + size_t(e) * d * h, y + size_t(pos) * d, unit, unit + 2, 1, d, h, nt2, nullptr, 1);
            }
        if (timed) { dynb::timing_mark(st, dynb::ST_FFN1, 0); dynb::timing_mark(st, dynb::ST_FFN2, 0); }
    }
    // m6 combine
    hipLaunchKernelGGL(k_combine, dim3((T + 3) / 4), dim3(256), 0, st, y, inv, topk_w, static_cast<bf16_t*>(out), T, d, k);
    if (timed) dynb::timing_mark(st, dynb::ST_COMBINE, 0);
    HIP_TRY(hipGetLastError(), "moe_forward");
    return DYNB_OK;
}

// The kernels of moe_forward for tensors on 16-byte borders, for the tests: bit 0 k_gate_stream, 1 k_gate_small, 2 k_gate_big, 3 k_grouped_stream, 4 and 5
// k_grouped_few, 6 and 7 k_grouped_skinny (first and second layer); a negative code where the shape is refused
extern "C" int dynb_moe_kernels(const moe_shape* s, int noisy)
{
    const int rc = check_shape(s, "dynb_moe_kernels");
    if (rc != DYNB_OK) return rc;
    const Choice c = choose(s, noisy != 0, true, true, 0);
    return c.gate_stream | c.gate_small << 1 | (c.T_big > 0) << 2 | c.streamed << 3 | c.few1 << 4 | c.few2 << 5 | c.skinny1 << 6 | c.skinny2 << 7;
}

extern "C" int moe_forward(const moe_shape* s, const void* x, const void* Wg, const void* Wn, const float* noise,
                           const void* W1, const void* W2, void* out, const moe_aux* aux, void* workspace,
                           size_t workspace_bytes, void* stream)
{
    return moe_run(s, x, Wg, Wn, noise, W1, W2, out, aux, workspace, workspace_bytes, stream, 0);
}

// ------------------------------------------------------------------------------------------
// Entry point for callers that cannot allocate device memory.  The routing tables and the
// xs / hid / y buffers that moe_forward keeps in its caller-provided workspace live in a device
// array that is part of the library's code object; every GPU holds its own copy at its own address.
static __device__ __align__(256) unsigned char scratch[MOE_STATIC_SCRATCH_BYTES];

// Device address of `scratch` on the current GPU.  In host code the array's name is only a
// stand-in for the symbol, so the address is asked for once per device and kept.
static int static_scratch_ptr(void** out)
{
    constexpr int MAX_DEVICES = 64;
    static std::mutex mu;
    static void* ptr_of[MAX_DEVICES] = {};
    int dev = 0;
    HIP_TRY(hipGetDevice(&dev), "moe_forward_static(hipGetDevice)");
    if (dev < 0 || dev >= MAX_DEVICES) return fail(DYNB_E_UNSUPPORTED, "moe_forward_static: device ordinal beyond 63");
    std::lock_guard<std::mutex> lock(mu);
    if (!ptr_of[dev]) {
        void* p = nullptr;
        HIP_TRY(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)), "moe_forward_static(hipGetSymbolAddress)");
        if (!p) return fail(DYNB_E_HIP, "moe_forward_static: no device address for the scratch array");
        ptr_of[dev] = p;
    }
    *out = ptr_of[dev];
    return DYNB_OK;
}

extern "C" int moe_forward_static(const moe_shape* s, const void* x, const void* Wg, const void* Wn, const float* noise,
                                  const void* W1, const void* W2, void* out, const moe_aux* aux, void* stream)
{
    int rc = check_shape(s, "moe_forward_static");
    if (rc != DYNB_OK) return rc;
    const size_t need = layout(s).total;
    if (need > size_t(MOE_STATIC_SCRATCH_BYTES))
        return fail(DYNB_E_WORKSPACE, "moe_forward_static: this shape needs " + std::to_string(need) +
                                          " bytes of scratch memory, the built-in array holds " +
                                          std::to_string(size_t(MOE_STATIC_SCRATCH_BYTES)) + "; use moe_forward");
    void* ws = nullptr;
    rc = static_scratch_ptr(&ws);
    if (rc != DYNB_OK) return rc;
    // every buffer of the layout is written before it is read (blockcnt, where it has to start at zero, by a fill kernel
    // inside the layer): the previous call's contents do not matter
    return moe_run(s, x, Wg, Wn, noise, W1, W2, out, aux, ws, size_t(MOE_STATIC_SCRATCH_BYTES), stream, 0);
}

extern "C" int moe_forward_naive(const moe_shape* s, const void* x, const void* Wg, const void* Wn, const float* noise,
                                 const void* W1, const void* W2, void* out, const moe_aux* aux, void* workspace,
                                 size_t workspace_bytes, void* stream, int32_t use_stride)
{
    if (use_stride < 1) return fail(DYNB_E_INVAL, "moe_forward_naive: use_stride must be >= 1");
    return moe_run(s, x, Wg, Wn, noise, W1, W2, out, aux, workspace, workspace_bytes, stream, use_stride);
}
