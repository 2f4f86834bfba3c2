// Convolution over the fragment batch as an MFMA implicit GEMM (gfx950).
//
// Every fragment is an independent signal (Definition "fragmentwise
// evaluation", Sect. 4.2), so all fragments of a layer form one batch of
// ordinary valid convolutions (Sect. 3.3 and its 2-D form in Sect. 6.1):
//   out[f][y][x][o] = act( bias[o] + sum_{t_h,t_w,i} W[o][i][t_h][t_w] * in[f][y+t_h][x+t_w][i] )
// As a GEMM: M = output samples (a TH x TW spatial tile of one fragment per
// workgroup), N = output channels, K = fh * fw * Cin.
//
// Workgroup = 4 wavefronts of 64 lanes; each wave owns (16 MT) samples x (16 NT)
// channels of the output tile (128 x 64 for the wide layers: the wider the wave
// tile, the fewer operand bytes per flop) in 16 x 16 MFMA tiles.  The weights are
// the MFMAs' first operand, so a lane ends with one sample and four consecutive
// channels of every tile, which the epilogues store without a transposition.
// K loop: input channels in chunks of 32 x filter taps; a step is one (chunk,
// tap) pair.  For each chunk the input halo tile (TH + fh - 1) x (TW + fw - 1) is
// staged in LDS once and read by all fh * fw taps.  The weights of a step go from
// global memory (L2-resident: every workgroup of an N block reads the same
// slices) straight into each lane's registers ahead of their use.
//
//  bfloat16: one v_mfma_f32_16x16x32_bf16 per tile and step, accumulating over
//   the whole K loop; the halo is copied by LDS-DMA, double-buffered where two
//   workgroups still fit a CU.
//
//  binary32: every operand is split into two binary16 numbers, x S = hi + lo with
//   hi = fl16(x S), lo = fl16(x S - hi) and S a power of two, and a product is
//   hi hi + hi lo + lo hi: three v_mfma_f32_16x16x32_f16 per tile and step in 48
//   cycles, against 256 cycles for the same 32 channels on the binary32 matrix
//   instruction.  Both parts together hold 22 to 23 bits, and the dropped lo lo is
//   below 2^-22 of the product.  The sums keep more than that loses: a step's
//   32-channel sum starts from zero and is added to the accumulator by a binary32
//   fma (which also takes S out again), one rounding to nearest per step where the
//   binary32 instruction rounds once per product.  Relative error (2-norm) of a
//   sum of K products relu(N(0,1)) x N(0,1) against 64 bits, binary32 instruction
//   -> this: K = 64 1.03e-7 -> 0.92e-7, 288 2.15e-7 -> 1.04e-7, 1152 4.3e-7 ->
//   1.5e-7, 9216 1.22e-6 -> 3.4e-7.  (Three bfloat16 parts and six products need
//   no scale and reach 3.3e-7 at K = 9216, at twice the matrix cycles.)
//   S is chosen per staged sample and 32-channel chunk, the power of two that
//   takes the sample's largest magnitude into [2^14, 2^15) (for the weights one per
//   output channel, which the epilogue takes out again): it depends on nothing but
//   the sample itself, so every fashion, tile shape and batch gives the same bits.
//   A value keeps all its bits down to 2^-17 of its sample's (filter's) largest and
//   an absolute 2^-40 of that below.  That is lost only where the large values meet
//   small or no weights, so every output is certified: the sum of what its samples'
//   parts left out (kept beside the sample in LDS) and of what its filter's did,
//   each times the largest value it can have met, must stay below sqrt(K) 2^-24 of
//   the output's own magnitude, what the K additions themselves lose in binary32.  Outputs that fail, and those that are not finite (an
//   infinity leaves no finite parts), are summed again with the binary32 matrix
//   instruction from the inputs and weights as they are.  The certificate is a
//   property of the output's window alone too.  On N(0,1) data a few outputs
//   of a layer fail, if any (the certificate costs 0.1 to 4 % of a call, most on layers
//   of few taps: HD frame 42.1 -> 42.6 ms, twelve layers of 128 maps 0.862 -> 0.895);
//   on channels that differ by 2^20 and more against their weights all do.
//
// Spatial tiles may read a virtual zero border of pad_h x pad_w samples around
// every fragment (the input gradient of the backward pass); small fragments can
// instead be read as one flat sequence, and the dilated fashion tiles one signal
// by phase (see the kernel's parameters).
//
// K-index assignment inside one MFMA issue: lane group g (lanes 16g..16g+15)
// holds channels 8g .. 8g+7 of the chunk; both operands use the same assignment.
//
// Epilogue: + bias, activation, masked 16-byte stores (edge tiles, padded
// channels) in the channels-last output layout.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "dev_common.h"
#include "dss_internal.h"

namespace dss {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));   // one 16-byte unit

constexpr int kCC = 32;             // channels per chunk
constexpr int kThreads = 256;
constexpr int kBM = 256;            // output samples per workgroup
// LDS bytes per staged sample.  bfloat16: the chunk's 64 bytes, its four 16-byte
// units rotated by two where bit 2 of the halo column is set.  binary32: 64 bytes
// of hi parts, 64 of lo parts, the sample's scale, padding.  An operand read
// (ds_read_b128) is served in four passes of 16 lanes; lane l shares its pass
// with the lanes whose bits 2, 3 and 4 have the same parity as its own, i.e. a
// pass reads unit u of samples {0-3, 12-15} (or {4-11}) of the 16 and unit u + 1
// of the others.  With a pitch of 16-byte units = 2 (mod 4) (160 bytes) those 16
// units fall in 16 different bank groups, with 64 bytes the rotation does it.
constexpr int kPitchBf16 = 64, kPitchF32 = 160;
constexpr int kScaleAt = 128;       // binary32: byte offset of 2^-14 / S of a sample's chunk
constexpr int kLossAt = 136;        // ... and of what its parts left out (times that, summed over the chunks
                                    // so far) and of the largest 2^-14 / S of the chunks
constexpr int kBadAt = 144;         // ... and the outputs of this sample that failed their certificate
constexpr int kLdsHead = 128;       // bytes before the halo (binary32: both of the above over the workgroup)
constexpr int kMaxLds = 78 * 1024;  // two workgroups per CU (160 KB of LDS)
constexpr int kMaxLds1 = 156 * 1024;  // one workgroup per CU (filters too wide for two)
constexpr int kXcds = 8;            // accelerator complex dies of an MI355X
constexpr int kGroup = 16;          // neighbouring tiles scheduled together

// WGM x WGN waves of (16 MT samples) x (16 NT channels)
template <int WGM, int WGN, int MT, int NT>
struct MfmaCfg {
    static constexpr int BN = 16 * NT * WGN;            // output channels per workgroup
    static_assert(16 * MT * WGM == kBM && 64 * WGM * WGN == kThreads, "256 samples, four waves");
    static_assert(NT % 2 == 0, "bfloat16 tiles pair up into runs of 8 channels");
};

// Bytes of one 16-row weight tile of a step: 64 lanes x 16 bytes, binary32 hi and lo parts.
constexpr int tile_bytes(bool bf16) { return bf16 ? 1024 : 2048; }
// Channel of row r (0..15) of tile nt (even/odd pairs) within a group of tiles.
// binary32: consecutive.  bfloat16: a lane's rows 4g..4g+3 of tiles 2k and 2k + 1 are
// channels 32k + 8g .. + 7, one 16-byte store.
__host__ __device__ constexpr int tile_channel(bool bf16, int nt, int r) {
    return bf16 ? (nt >> 1) * 32 + (r >> 2) * 8 + (nt & 1) * 4 + (r & 3) : nt * 16 + r;
}

// 16 zero bytes: the source of every staged unit that lies outside the fragment
// or in the zero-padded channels of the last chunk.
__device__ __attribute__((aligned(16))) const unsigned int g_zero16[4] = {0u, 0u, 0u, 0u};

typedef __attribute__((address_space(3))) void lds_void;

// Direct global -> LDS copy of one 16-byte unit per active lane: the unit lands in
// LDS at wave_dst + 16 * lane (gfx950 global_load_lds_dwordx4).
__device__ __forceinline__ void dma16(const void* src, char* wave_dst) {
    __builtin_amdgcn_global_load_lds(src, (lds_void*)wave_dst, 16, 0, 0);
}

__device__ __forceinline__ floatx4 mfma_bf16(u32x4 w, u32x4 x, floatx4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w), __builtin_bit_cast(bf16x8, x), c, 0,
                                                   0, 0);
}
__device__ __forceinline__ floatx4 mfma_f16(u32x4 w, u32x4 x, floatx4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, w), __builtin_bit_cast(f16x8, x), c, 0, 0,
                                                  0);
}

// The two binary16 parts of v[i] * scale (scale a power of two).
__device__ __forceinline__ void split_f16(const float (&v)[8], float scale, u32x4& hi, u32x4& lo) {
    f16x8 h, l;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const float y = v[i] * scale;
        h[i] = (_Float16)y;
        l[i] = (_Float16)(y - (float)h[i]);
    }
    hi = __builtin_bit_cast(u32x4, h);
    lo = __builtin_bit_cast(u32x4, l);
}

// What the parts leave out of the values that may lose bits, in the same unit (a bound
// for the smallest, whose product with the scale may underflow): 0 or 2^-83 and more.
__device__ __forceinline__ float split_loss(const float (&v)[8], float scale) {
    float sum = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const float y = v[i] * scale, r = y - (float)(_Float16)y;
        sum += fabsf(y) >= 0.25f || v[i] == 0.f ? 0.f : fabsf(y) < 0x1p-60f ? 0x1p-60f : fabsf(r - (float)(_Float16)r);
    }
    return sum;
}

// Power of two S that takes a largest magnitude with these bits into [2^14, 2^15):
// 2^110 for magnitudes below 2^-96 (zero among them).  The bits of 2^-14 / S are
// kUnscale minus S's.
constexpr uint32_t kUnscale = 240u << 23;
__device__ __forceinline__ uint32_t scale_bits(uint32_t max_bits) {
    return min((268u << 23) - (max_bits & 0x7f800000u), 237u << 23);
}

// Epilogue variants: kEpiStore writes the activations, kEpiProj the partial
// projections of a folded 1x1 convolution, kEpiPool the sliding-window maxima of
// a 1-D pool written straight to their fragments.
constexpr int kEpiStore = 0, kEpiProj = 1, kEpiPool = 2;

template <bool BF16, typename Tout, int WGM, int WGN, int MT, int NT, int EPI = kEpiStore>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2))) void conv_mfma_kernel(
    const char* __restrict__ in,       // [F][Hin][Win][Cin] of BF16 ? bfloat16 : binary32
    int Hin, int Win, int Cin,
    const char* __restrict__ wp,       // packed weights: slices [N block of pack_rows][chunk][th][tw] of 16-row tiles
    int pack_rows,
    const float* __restrict__ bias,    // [Cout_pad]
    int fh, int fw, int Cout, int act, int nchunks,
    Tout* __restrict__ out,            // [F][Hout][Wout][Cout]; kEpiPool: the fragments [k F][1][pool_U][Cout]
                                       // (unused with kEpiProj)
    int Hout, int Wout, int TH, int TW, int tilesY, int tilesX, int nbs, int dbl_halo,
    int flat_h, int flat_w,             // flat mode: input fragments of flat_h x flat_w (0: spatial tiles)
    int dil_h, int dil_w,               // dilated mode (> 1): taps dil apart on one signal, tiled by phase
    int pad_h, int pad_w,               // spatial tiles: a zero border of pad samples around every fragment
    const float* __restrict__ w2,       // kEpiProj: 1x1 projection weights [Cout_pad][4] (binary32, zero padded)
    float* __restrict__ part,           // kEpiProj: partial projections [nbs * WGN][F * Hout * Wout][4]
    int64_t part_stride,                // kEpiProj: floats per channel group of part
    int tile_step_w,                    // columns between neighbouring tiles (TW, or TW - k + 1 with kEpiPool)
    int pool_k, int pool_U,             // kEpiPool: pool size along the row, pooled samples per fragment
    const float* __restrict__ w32,      // binary32: the weights as they are, in the packed tiles' order
    float cert,                         // binary32: how often an output must exceed what its sum may have lost
    const float* __restrict__ w_scale) {   // binary32: [Cout_pad][2], e_n and what the parts of the weights leave out
    using Cfg = MfmaCfg<WGM, WGN, MT, NT>;
    constexpr int THREADS = kThreads;
    constexpr int PITCH = BF16 ? kPitchBf16 : kPitchF32;
    constexpr int PLANES = BF16 ? 1 : 2;
    constexpr int ES = BF16 ? 2 : 4;
    extern __shared__ __attribute__((aligned(16))) char lds[];
    // The bfloat16 kernel with 128x64 wave tiles keeps its accumulators in the
    // accumulation registers (AGPRs): an AGPR use the compiler cannot rule out
    // (this empty clobber) makes it pick that form of the MFMA instructions.
    if constexpr (BF16 && MT == 8 && NT == 4) asm volatile("" ::: "a0");

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // uniform: a scalar register
    const int wm = wave % WGM;           // wave position along M
    const int wn = wave / WGM;           // wave position along N
    const int grp = lane >> 4;           // lane group: K slot of the MFMA operands, channel run of the results
    const int l16 = lane & 15;           // sample of a tile (operands and results), weight row (operands)

    // workgroup -> (fragment, tile row, tile column, N block).  Workgroups are
    // handed to the 8 XCDs round-robin by id; the remap gives every XCD one
    // contiguous range of work items.  Items are ordered in groups of kGroup
    // neighbouring tiles (which share halo samples); inside a group the N block
    // is the outer index, so the workgroups that run together on an XCD read the
    // same weight slices and the same input tiles from its L2.
    const int total = gridDim.x;
    const int xcd = blockIdx.x % kXcds, slot = blockIdx.x / kXcds;
    const int q8 = total / kXcds, r8 = total % kXcds;
    const int item = xcd < r8 ? xcd * (q8 + 1) + slot : r8 * (q8 + 1) + (xcd - r8) * q8 + slot;
    const int ntiles = total / nbs;
    const int gi = item / (kGroup * nbs);
    const int gsize = min(kGroup, ntiles - gi * kGroup);
    const int grem = item - gi * kGroup * nbs;
    const int nb = grem / gsize;
    const int tile = gi * kGroup + grem % gsize;
    const int tiles = tilesY * tilesX;
    const int f = tile / tiles;
    const int trem = tile % tiles;
    const int ty0 = (trem / tilesX) * TH;
    const int tx0 = (trem % tilesX) * tile_step_w;

    // Spatial tiles: a TH x TW block of one fragment, halo (TH + fh - 1) x (TW + fw - 1).
    // Flat mode (small fragments): the fragment batch is read as one sequence of
    // samples, a tile is TW consecutive positions of it (TH = 1), tap (th, tw)
    // sits th * flat_w + tw samples further on, and only positions that are valid
    // outputs of their own fragment are stored.
    const int HW = flat_w ? TW + (fh - 1) * flat_w + fw - 1 : TW + fw - 1;   // halo row width
    const int tap_row = flat_w ? flat_w : HW;
    const int halo_px = (flat_w ? TH : TH + fh - 1) * HW;
    const int halo_bytes = ((halo_px * PITCH + 127) / 128) * 128;
    char* const halo0 = lds + kLdsHead;
    char* const halo1 = BF16 && dbl_halo ? halo0 + halo_bytes : halo0;

    // Tile sample m -> tile row.  Tiles 16 or more samples wide are row-major: the
    // 16 samples of an MFMA tile lie side by side.  An 8-wide tile puts them on two
    // rows, whose operand reads are free of bank conflicts when the rows are
    // d apart with HW * d = 0 (mod 8); d = 8 >> (trailing zero bits of HW).
    const int tw_log2 = __builtin_ctz(TW);   // spatial and dilated tiles are 2^k samples wide
    const int row_lg = TW == 8 ? 3 - min(3, __builtin_ctz(HW)) : 0;
    auto tile_dy = [&](int m) -> int {
        if (TW != 8) return m >> tw_log2;
        const int b = m >> 4;
        return ((b >> row_lg) << (row_lg + 1)) + (b & ((1 << row_lg) - 1)) + (((m >> 3) & 1) << row_lg);
    };
    // byte offset of a lane's sample of MFMA tile mt inside the halo: a scalar per
    // tile plus one vector value (summed ahead per tile for bfloat16, whose
    // accumulators leave the vector registers for it)
    const int lane_off = ((TW == 8 ? ((l16 >> 3) << row_lg) * HW + (l16 & 7) : l16) * PITCH) + (BF16 ? 0 : grp * 16);
    auto tile_off = [&](int mt) -> int {
        const int m = (wm * MT + mt) * 16;
        return (tile_dy(m) * HW + (m & (TW - 1))) * PITCH;
    };
    int a_off[BF16 ? MT : 1];
    if constexpr (BF16) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            const int m = (wm * MT + mt) * 16 + l16;
            a_off[mt] = (tile_dy(m) * HW + (m & (TW - 1))) * PITCH;
        }
    }

    floatx4 acc[MT][NT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = floatx4{0.f, 0.f, 0.f, 0.f};

    const size_t row_bytes = (size_t)Cin * ES;
    // Where the tile's halo lives.  Spatial tiles: fragment f, rows and columns
    // adjacent.  Dilated mode: the "fragments" are the dil_h x dil_w phases of one
    // signal; phase (py, px) holds samples (py + dil_h a, px + dil_w b), so a tap
    // step is dil samples and every tile reads and writes one phase only.
    const bool dilated = dil_h * dil_w > 1;
    const int py = dilated ? f / dil_w : 0, px = dilated ? f - py * dil_w : 0;
    const size_t row_step = (size_t)(dilated ? dil_h : 1) * Win * row_bytes;
    const size_t col_step = (size_t)(dilated ? dil_w : 1) * row_bytes;
    const size_t f_base = dilated ? ((size_t)py * Win + px) * row_bytes : (size_t)f * Hin * Win * row_bytes;
    const int lim_h = dilated ? (Hin - py + dil_h - 1) / dil_h : Hin;   // samples of this phase / fragment
    const int lim_w = dilated ? (Win - px + dil_w - 1) / dil_w : Win;
    // top-left input sample of the tile's halo (negative inside the zero border)
    const int hy0 = ty0 - pad_h, hx0 = tx0 - pad_w;
    const char* in_f = in + f_base;
    const int taps = fh * fw;
    const int steps = nchunks * taps;
    const char* zero = reinterpret_cast<const char*>(g_zero16);

    // Staging: thread t takes 16-byte LDS unit (bfloat16) or 8-channel unit
    // (binary32) t & 3 of halo samples t / 4, t / 4 + 64, ...; a round moves on
    // by 64 samples, so the sample's halo row and column are divided out once and
    // then advanced by additions.
    const int dy_step = 64 / HW, dx_step = 64 - dy_step * HW;
    auto advance = [&](int& dy, int& dx) {
        dy += dy_step;
        dx += dx_step;
        if (dx >= HW) {
            dx -= HW;
            ++dy;
        }
    };
    auto wait_staged = [] {
        __builtin_amdgcn_s_waitcnt(0);   // this wave's copies have landed in LDS
        __syncthreads();                 // ... and every other wave's
    };

    // Weights: a wave's NT tiles of a slice are consecutive; lane (row l16, group
    // grp) holds 16 bytes, channels 8 grp .. 8 grp + 7 of its row, per part, and
    // one load instruction reads a contiguous kilobyte.  Slices are packed for
    // pack_rows rows, of which a narrower launch takes a part.
    const int n_base = nb * Cfg::BN + wn * 16 * NT;      // first channel of the wave
    const size_t slice_bytes = (size_t)(pack_rows >> 4) * tile_bytes(BF16);
    const char* w_lane = wp + (size_t)(n_base / pack_rows) * steps * slice_bytes +
                         (size_t)((n_base % pack_rows) >> 4) * tile_bytes(BF16) + lane * 16;
    auto load_b = [&](int st, u32x4 (&bb)[NT][PLANES]) {
        const char* src = w_lane + (size_t)st * slice_bytes;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int p = 0; p < PLANES; ++p)
                bb[nt][p] = *reinterpret_cast<const u32x4*>(src + nt * tile_bytes(BF16) + p * 1024);
    };

    int step = 0, cc = 0, th = 0, tw = 0;   // step, chunk and tap of the next step
    if constexpr (BF16) {
        auto stage_halo = [&](int cn, char* dst) {
            const char* src_c = in_f + (size_t)cn * (kCC * ES);
            const int c_base = cn * kCC;
            const int st_q = tid & 3;
            int dy = (tid >> 2) / HW, dx = (tid >> 2) - dy * HW;
            for (int r0 = 0; r0 < halo_px * 4; r0 += THREADS) {
                const int yy = hy0 + dy, xx = hx0 + dx, q = st_q ^ (((dx >> 2) & 1) << 1);
                const bool ok = (unsigned)yy < (unsigned)lim_h && (unsigned)xx < (unsigned)lim_w && c_base + q * 8 < Cin;
                if (r0 + tid < halo_px * 4)
                    dma16(ok ? src_c + (size_t)yy * row_step + (size_t)xx * col_step + q * 16 : zero,
                          dst + (r0 + wave * 64) * 16);
                advance(dy, dx);
            }
        };
        // The next chunk's halo is staged by the same copies as stage_halo, but
        // issued as inline assembly.  To the compiler, LDS-DMA completes out of
        // order with ordinary loads, so with one in flight that it knows of,
        // every wait for a B operand would become a wait for all loads; unseen,
        // they leave those waits partial.  The hardware counts them in issue order
        // with the B loads (a partial wait that the compiler computes without
        // them still covers its own loads), and the full wait before the chunk's
        // closing barrier drains them.  M0 (the LDS destination) is saved and
        // restored around each copy.
        const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)lds;
        auto stage_halo_unseen = [&](int cn, char* dst) {
            const char* src_c = in_f + (size_t)cn * (kCC * ES);
            const int c_base = cn * kCC;
            const uint32_t dst_lds = lds_base + (uint32_t)(dst - lds);
            const int st_q = tid & 3;
            int dy = (tid >> 2) / HW, dx = (tid >> 2) - dy * HW;
            for (int r0 = 0; r0 < halo_px * 4; r0 += THREADS) {
                const int yy = hy0 + dy, xx = hx0 + dx, q = st_q ^ (((dx >> 2) & 1) << 1);
                const bool ok = (unsigned)yy < (unsigned)lim_h && (unsigned)xx < (unsigned)lim_w && c_base + q * 8 < Cin;
                const char* src = ok ? src_c + (size_t)yy * row_step + (size_t)xx * col_step + q * 16 : zero;
                const uint32_t m0v = __builtin_amdgcn_readfirstlane(dst_lds + (uint32_t)(r0 + wave * 64) * 16);
                if (r0 + tid < halo_px * 4) {
                    uint32_t saved;
                    asm volatile(
                        "s_mov_b32 %0, m0\n\t"
                        "s_mov_b32 m0, %2\n\t"
                        "s_nop 0\n\t"
                        "global_load_lds_dwordx4 %1, off\n\t"
                        "s_mov_b32 m0, %0"
                        : "=&s"(saved)
                        : "v"(src), "s"(m0v)
                        : "memory");
                }
                advance(dy, dx);
            }
        };
        // One step: this tap's samples from the halo, then the step's MFMAs with
        // the weights bb.
        auto mma_step = [&](const char* halo, const u32x4 (&bb)[NT][1]) {
            const int shift = flat_w ? th * flat_w + tw : tw;
            const int off = (th * tap_row + tw) * PITCH + ((grp ^ ((((l16 + shift) >> 2) & 1) << 1)) << 4);
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                const u32x4 a = *reinterpret_cast<const u32x4*>(halo + (a_off[mt] + off));
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = mfma_bf16(bb[nt][0], a, acc[mt][nt]);
            }
        };
        // B operands two steps ahead in three register sets whose roles rotate
        // with the step, over all steps of all chunks in threes, so no register
        // copy waits for a load (the loads past the last step repeat the last
        // slice).  A chunk ends inside the rotation: its closing drain and barrier
        // leave the next chunk's halo in place, and the copies of the one after
        // it go out.
        u32x4 bA[NT][1], bB[NT][1], bC[NT][1];
        load_b(0, bA);
        load_b(min(1, steps - 1), bB);
        stage_halo(0, halo0);
        wait_staged();
        if (dbl_halo && nchunks > 1) stage_halo_unseen(1, halo1);
        const char* halo = halo0;
        auto next_chunk = [&]() {
            if (++cc >= nchunks) return;
            if (!dbl_halo) {
                __syncthreads();               // every wave is done with the previous chunk's halo
                stage_halo(cc, halo0);
            }
            wait_staged();                     // chunk cc's halo has landed, for every wave
            halo = (cc & 1) ? halo1 : halo0;
            // chunk cc + 1 goes to the buffer of chunk cc - 1, which every wave is done with
            if (dbl_halo && cc + 1 < nchunks) stage_halo_unseen(cc + 1, (cc & 1) ? halo0 : halo1);
        };
        auto sub_step = [&](const u32x4 (&bb)[NT][1], u32x4 (&bl)[NT][1]) {
            load_b(min(step + 2, steps - 1), bl);
            mma_step(halo, bb);
            ++step;
            if (++tw == fw) {
                tw = 0;
                if (++th == fh) {
                    th = 0;
                    next_chunk();
                }
            }
        };
        while (step + 2 < steps) {
            sub_step(bA, bC);
            sub_step(bB, bA);
            sub_step(bC, bB);
        }
        if (step < steps) sub_step(bA, bC);
        if (step < steps) sub_step(bB, bA);
    } else {
        // Stages chunk cn: rounds of 64 samples, kRounds rounds' loads in flight
        // together.  The four threads of a sample find its largest magnitude, hence
        // its scale, by two exchanges within their quad.
        constexpr int kRounds = MT * NT == 32 ? 4 : MT * NT == 16 && EPI != kEpiPool ? 3 : 2;   // (registers)
        float* const head = reinterpret_cast<float*>(lds);
        auto stage_split = [&](int cn) __attribute__((always_inline)) {
            // computed here each time: held through the K loop, these would take
            // registers from the accumulators
            int tid_s = tid;
            asm volatile("" : "+v"(tid_s));
            const int st_q = tid_s & 3;
            const char* src_c = in_f + (size_t)cn * (kCC * ES) + st_q * 32;
            const int c0 = cn * kCC + st_q * 8;
            int dy = (tid_s >> 2) / HW, dx = (tid_s >> 2) - dy * HW;
            // channels c0 .. c0 + 7 of halo sample p
            auto load = [&](int p, int sy, int sx, float (&q)[8]) {
                const int yy = hy0 + sy, xx = hx0 + sx;
                const bool ok = p < halo_px && (unsigned)yy < (unsigned)lim_h && (unsigned)xx < (unsigned)lim_w &&
                                c0 < Cin;
                const char* src = src_c + (size_t)yy * row_step + (size_t)xx * col_step;
                const floatx4 a = *reinterpret_cast<const floatx4*>(ok ? src : zero);
                const floatx4 b = *reinterpret_cast<const floatx4*>(ok && c0 + 4 < Cin ? src + 16 : zero);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    q[e] = a[e];
                    q[4 + e] = b[e];
                }
            };
            auto top_bits = [](const float (&q)[8]) {
                // (v_max3_f32 takes magnitudes for nothing and passes NaN by)
                float top = 0.f;
#pragma unroll
                for (int e = 0; e < 8; e += 2)
                    asm("v_max3_f32 %0, |%1|, |%2|, %0" : "+v"(top) : "v"(q[e]), "v"(q[e + 1]));
                uint32_t mb = __float_as_uint(top);
                mb = max(mb, (uint32_t)__builtin_amdgcn_mov_dpp((int)mb, 0xB1, 0xf, 0xf, true));   // lane ^ 1
                return max(mb, (uint32_t)__builtin_amdgcn_mov_dpp((int)mb, 0x4E, 0xf, 0xf, true));  // lane ^ 2
            };
            uint32_t un_max = 0;
            for (int p0 = tid_s >> 2; p0 < halo_px; p0 += 64 * kRounds) {
                float v[kRounds][8];
                uint32_t lossy = 0;
#pragma unroll
                for (int r = 0; r < kRounds; ++r) {
                    load(p0 + 64 * r, dy, dx, v[r]);
                    advance(dy, dx);
                }
#pragma unroll
                for (int r = 0; r < kRounds; ++r) {
                    if (p0 + 64 * r >= halo_px) break;
                    const uint32_t mb = top_bits(v[r]), sb = scale_bits(mb);
                    const uint32_t un = kUnscale - sb;
                    u32x4 hi, lo;
                    split_f16(v[r], __uint_as_float(sb), hi, lo);
                    char* dst = halo0 + (p0 + 64 * r) * PITCH + st_q * 16;
                    *reinterpret_cast<u32x4*>(dst) = hi;
                    *reinterpret_cast<u32x4*>(dst + 64) = lo;
                    const uint32_t x = mb ? un : 0u;          // (a sample of zeros loses nothing)
                    if (st_q == 0) {
                        *reinterpret_cast<uint32_t*>(dst + kScaleAt) = un;
                        uint32_t* const rec = reinterpret_cast<uint32_t*>(dst + kLossAt);
                        if (cn == 0) *reinterpret_cast<uint2*>(rec) = make_uint2(0u, x);
                        else atomicMax(rec + 1, x);
                    }
                    un_max = max(un_max, x);
                    // a value other than 0 below 2^-2 / S may lose bits (twice its magnitude less 1: 0 comes last)
                    uint32_t mn = ~0u;
#pragma unroll
                    for (int e = 0; e < 8; ++e) mn = min(mn, (__float_as_uint(v[r][e]) << 1) - 1u);
                    lossy |= (uint32_t)(mn < (((252u << 23) - sb) << 1) - 1u);
                }
                if (__any(lossy != 0)) {
#pragma unroll
                    for (int r = 0; r < kRounds; ++r) {
                        if (p0 + 64 * r >= halo_px) break;
                        const uint32_t mb = top_bits(v[r]), sb = scale_bits(mb);
                        float lost = split_loss(v[r], __uint_as_float(sb));
                        if (lost > 0.f) lost = fmaxf(lost * __uint_as_float(kUnscale - sb), 0x1p-149f);
                        if (mb < (31u << 23) && mb != 0) lost = __builtin_inff();   // S could not follow
                        lost += __uint_as_float(__builtin_amdgcn_mov_dpp(__float_as_uint(lost), 0xB1, 0xf, 0xf, true));
                        lost += __uint_as_float(__builtin_amdgcn_mov_dpp(__float_as_uint(lost), 0x4E, 0xf, 0xf, true));
                        if (st_q == 0 && lost > 0.f) {
                            *reinterpret_cast<float*>(halo0 + (p0 + 64 * r) * PITCH + kLossAt) += lost;
                            atomicAdd(&head[0], lost);
                        }
                    }
                }
            }
            // over the wave: within rows of 16 lanes, then row by row into lane 63
            un_max = max(un_max, (uint32_t)__builtin_amdgcn_mov_dpp((int)un_max, 0x124, 0xf, 0xf, true));   // rotated by 4
            un_max = max(un_max, (uint32_t)__builtin_amdgcn_mov_dpp((int)un_max, 0x128, 0xf, 0xf, true));   // ... by 8
            un_max = max(un_max, (uint32_t)__builtin_amdgcn_mov_dpp((int)un_max, 0x142, 0xf, 0xf, true));   // row before
            un_max = max(un_max, (uint32_t)__builtin_amdgcn_mov_dpp((int)un_max, 0x143, 0xf, 0xf, true));   // two rows
            if ((tid_s & 63) == 63) atomicMax(reinterpret_cast<uint32_t*>(head) + 1, un_max);
        };
        // One step.  A tile's sum over the step's 32 channels starts from zero, the
        // smallest products first, and is added unscaled to its accumulator.  Two
        // tiles at a time: while their six MFMAs run, the previous two tiles' sums are
        // added, and a sample tile's operands are read one tile ahead (512 x 512 6x6
        // layer 1.26 -> 1.20 ms, 22-GFLOP 3x3 layers of 128 maps 0.104 -> 0.093 ms
        // against one sample tile after the other).  The 1-D pool's 64x64 wave tile
        // takes one sample tile after the other: its 9 steps gain more from three
        // waves per SIMD, which the 168 registers of that form allow (0.170 against
        // 0.194 ms on the conv9 32->64 layer).
        constexpr bool AHEAD = !(EPI == kEpiPool && MT * NT == 16);
        auto mma_step = [&](const u32x4 (&bb)[NT][2]) {
            const int off = lane_off + (th * tap_row + tw) * PITCH;
            const int s_delta = kScaleAt - grp * 16;
            u32x4 hi, lo;
            float un;
            auto read_tile = [&](int mt, u32x4& h, u32x4& l, float& u) {
                const char* p = halo0 + (tile_off(mt) + off);
                h = *reinterpret_cast<const u32x4*>(p);
                l = *reinterpret_cast<const u32x4*>(p + 64);
                u = *reinterpret_cast<const float*>(p + s_delta);
            };
            if constexpr (!AHEAD) {
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) {
                    read_tile(mt, hi, lo, un);
                    floatx4 t[NT];
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt) t[nt] = mfma_f16(bb[nt][1], hi, floatx4{0.f, 0.f, 0.f, 0.f});
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt) t[nt] = mfma_f16(bb[nt][0], lo, t[nt]);
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt) t[nt] = mfma_f16(bb[nt][0], hi, t[nt]);
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt) {
#pragma unroll
                        for (int v = 0; v < 4; ++v) acc[mt][nt][v] = fmaf(t[nt][v], un, acc[mt][nt][v]);
                        asm volatile("" : "+v"(acc[mt][nt]));   // see add() below
                    }
                }
                return;
            }
            read_tile(0, hi, lo, un);
            u32x4 nhi = hi, nlo = lo;
            float nun = un;
            floatx4 tp[2];        // the previous pair's sums, and their factor
            float un_p = 0.f;
            auto add = [&](int pair, int k) {      // tile k of pair (mt NT / 2 + nt / 2)
                const int mt = pair / (NT / 2), nt = pair % (NT / 2) * 2 + k;
#pragma unroll
                for (int v = 0; v < 4; ++v) acc[mt][nt][v] = fmaf(tp[k][v], un_p, acc[mt][nt][v]);
                // here, not after the step, where all tiles' sums would be alive at once
                asm volatile("" : "+v"(acc[mt][nt]));
            };
#pragma unroll
            for (int pair = 0; pair < MT * NT / 2; ++pair) {
                const int mt = pair / (NT / 2), nt = pair % (NT / 2) * 2;
                if (nt == 0 && mt + 1 < MT) read_tile(mt + 1, nhi, nlo, nun);
                floatx4 t[2];
#pragma unroll
                for (int k = 0; k < 2; ++k) t[k] = mfma_f16(bb[nt + k][1], hi, floatx4{0.f, 0.f, 0.f, 0.f});
                if (pair > 0) add(pair - 1, 0);
#pragma unroll
                for (int k = 0; k < 2; ++k) t[k] = mfma_f16(bb[nt + k][0], lo, t[k]);
                if (pair > 0) add(pair - 1, 1);
#pragma unroll
                for (int k = 0; k < 2; ++k) t[k] = mfma_f16(bb[nt + k][0], hi, t[k]);
                tp[0] = t[0];
                tp[1] = t[1];
                un_p = un;
                if (nt + 2 == NT) {
                    hi = nhi;
                    lo = nlo;
                    un = nun;
                }
            }
            add(MT * NT / 2 - 1, 0);
            add(MT * NT / 2 - 1, 1);
        };
        u32x4 bA[NT][2], bB[NT][2];
        if (tid < 2) head[tid] = 0.f;
        __syncthreads();
        load_b(0, bA);
        stage_split(0);
        __syncthreads();
        auto sub_step = [&](const u32x4 (&bb)[NT][2], u32x4 (&bl)[NT][2]) {
            load_b(min(step + 1, steps - 1), bl);
            mma_step(bb);
            ++step;
            if (++tw == fw) {
                tw = 0;
                if (++th == fh) {
                    th = 0;
                    if (++cc < nchunks) {
                        __syncthreads();               // every wave is done with the previous chunk's halo
                        stage_split(cc);
                        __syncthreads();
                    }
                }
            }
        };
        while (step + 1 < steps) {
            sub_step(bA, bB);
            sub_step(bB, bA);
        }
        if (step < steps) sub_step(bA, bB);
    }

    // -- epilogue: lane (le_grp, le_16) holds sample le_16 and rows 4 le_grp + v of every
    // tile.  The lane's position again, from the lane-id instructions: the values
    // computed at entry feed the K loop, and sharing them would keep them (and
    // what is derived from them here) live through it.
    int lane_e = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
    asm volatile("" : "+v"(lane_e));
    const int le_16 = lane_e & 15, le_grp = lane_e >> 4;
    const size_t f_off = (size_t)f * Hout * Wout;
    const int frag_px = flat_h * flat_w;
    // output sample of tile position m: whether it exists, and its index
    auto out_pos = [&](int m, size_t& o) -> bool {
        if (flat_w) {
            const int p = tx0 + m;                 // TH = 1: position in the flat sequence (Win long)
            const int fr = p / frag_px, r = p - fr * frag_px;
            const int y = r / flat_w, x = r - y * flat_w;
            o = ((size_t)fr * Hout + y) * Wout + x;
            return p < Win && y < Hout && x < Wout;
        }
        if (dilated) {
            const int y = py + dil_h * (ty0 + tile_dy(m)), x = px + dil_w * (tx0 + (m & (TW - 1)));
            o = (size_t)y * Wout + x;
            return y < Hout && x < Wout;
        }
        const int y = ty0 + tile_dy(m), x = tx0 + (m & (TW - 1));
        o = f_off + (size_t)y * Wout + x;
        return y < Hout && x < Wout;
    };
    // byte offset of the lane's sample of MFMA tile mt inside the halo, as tile_off() and lane_off
    auto sample_off = [&](int mt, int ln) {
        return tile_off(mt) + (TW == 8 ? (((ln & 15) >> 3) << row_lg) * HW + (ln & 7) : ln & 15) * PITCH;
    };
    // where the lane keeps which of its outputs of tile row mt have failed: beside its own sample, 16 bits a lane
    auto bad_mask = [&](int mt, int ln) {
        return reinterpret_cast<uint16_t*>(halo0 + sample_off(mt, ln) + kBadAt + (wn * 4 + (ln >> 4)) * 2);
    };
    // The sums of tiles (mt, nt) .. (mt, nt + N - 1) from the inputs and weights as they are, in
    // global memory, U steps' operands loaded together: K slot g of matrix instruction j holds
    // channel 8 g + j of the chunk.
    auto exact_sums = [&](int mt, int nt, int ln, auto& sum, auto u_c) __attribute__((always_inline)) {
        constexpr int N = sizeof(sum) / sizeof(floatx4), U = decltype(u_c)::value;
        const int m = (wm * MT + mt) * 16 + (ln & 15);
        const int y0 = flat_w ? 0 : hy0 + tile_dy(m), x0 = flat_w ? tx0 + m : hx0 + (m & (TW - 1));
        const float* ws = w32 + ln * 8 +
                          ((size_t)(n_base / pack_rows) * steps * (pack_rows >> 4) + ((n_base % pack_rows) >> 4) + nt) * 512;
#pragma unroll
        for (int n = 0; n < N; ++n) sum[n] = floatx4{0.f, 0.f, 0.f, 0.f};
        int a = 0, b = 0, c0 = (ln >> 4) * 8;
#pragma nounroll
        for (int st = 0; st < steps; st += U) {
            floatx4 x[U][2], w[U][N][2];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int yy = flat_w ? 0 : y0 + a, xx = flat_w ? x0 + a * flat_w + b : x0 + b;
                const bool on = st + u < steps;              // past the last step: zeros
                const bool in_range = on && (unsigned)yy < (unsigned)lim_h && (unsigned)xx < (unsigned)lim_w && c0 < Cin;
                const char* src = in_f + (size_t)yy * row_step + (size_t)xx * col_step + (size_t)c0 * ES;
                x[u][0] = *reinterpret_cast<const floatx4*>(in_range ? src : zero);
                x[u][1] = *reinterpret_cast<const floatx4*>(in_range && c0 + 4 < Cin ? src + 16 : zero);
#pragma unroll
                for (int n = 0; n < N; ++n)
#pragma unroll
                    for (int k = 0; k < 2; ++k)
                        w[u][n][k] = *reinterpret_cast<const floatx4*>(on ? (const char*)(ws + n * 512 + k * 4) : zero);
                ws += (size_t)(pack_rows >> 4) * 512;
                if (++b == fw) {
                    b = 0;
                    if (++a == fh) {
                        a = 0;
                        c0 += kCC;
                    }
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int j = 0; j < 8; ++j)
#pragma unroll
                    for (int n = 0; n < N; ++n)
                        sum[n] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[u][n][j >> 2][j & 3], x[u][j >> 2][j & 3], sum[n], 0, 0,
                                                                      0);
        }
    };
    // the lane number again: a value of its own, so that nothing derived from it is shared with other places and
    // kept in registers between them
    auto lane_again = [] {
        int ln = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
        asm volatile("" : "+v"(ln));
        return ln;
    };
    // e_n and the loss of the weights of the lane's channels of tile nt
    auto load_scale = [&](const float* sc, int nt, int ln, floatx4& e, floatx4& wl) {
        const size_t c = n_base + tile_channel(false, nt, (ln >> 4) * 4);
        const floatx4 s0 = *reinterpret_cast<const floatx4*>(sc + 2 * c), s1 = *reinterpret_cast<const floatx4*>(sc + 2 * c + 4);
        e = floatx4{s0[0], s0[2], s1[0], s1[2]};
        wl = floatx4{s0[1], s0[3], s1[1], s1[3]};
    };
    bool redo = false;                  // binary32, wave-uniform: some output has failed
    // binary32: the powers of two of the channels' weights, and the certificate.  In
    // units of e_n an output's sums are off by at most 2^15 (L + X w_n): L the loss of the
    // window's samples (times 2^-14 / S; weights are below 2 e_n), X the largest
    // 2^-14 / S among them (a sample is below 2^15 / S, its parts' loss in units of
    // 1 / S) and w_n the loss of the channel's weights (in units of 2^-14 e_n).  First
    // with the workgroup's L and X for all outputs, then, hardly ever, with the
    // window's own.
    if constexpr (!BF16) {
        // 2^15 times the certificate's factor, of which 2^28 go to L and X ahead of their products.
        // (X at least 2^-94: then its product with a filter's loss does not underflow.  Signals
        // below 2^-65 are summed again somewhat more often for it.)
        const float kCert = cert * 0x1p-13f;
        auto largest = [](float x) { return x > 0.f ? fmaxf(x * 0x1p28f, 0x1p-66f) : 0.f; };
        const float* const head = reinterpret_cast<const float*>(lds);
        const float l_all = 0x1p29f * head[0], x_all = 2.f * largest(head[1]);
        uint32_t worst = 0;                              // of |sum| - threshold: negative, infinite and NaN come last
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            floatx4 e, wl, thr;
            load_scale(w_scale, nt, lane_e, e, wl);
#pragma unroll
            for (int v = 0; v < 4; ++v) thr[v] = kCert * (l_all + x_all * wl[v]) * e[v];
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                acc[mt][nt] *= e;
#pragma unroll
                for (int v = 0; v < 4; ++v) worst = max(worst, __float_as_uint(fabsf(acc[mt][nt][v]) - thr[v]));
            }
        }
        if (__any(worst >= 0x7f800000u)) {
            const int ln = lane_again();
            // the same without the tile's positions that are no outputs, some of them sums of nothing
            worst = 0;
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                size_t o;
                if (!out_pos((wm * MT + mt) * 16 + (ln & 15), o)) continue;
                int here = 0;                 // keeps the loads below in their place
                asm volatile("" : "+s"(here));
                const float* const sc = w_scale + here;
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) {
                    floatx4 e, wl;
                    load_scale(sc, nt, ln, e, wl);
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        worst = max(worst, __float_as_uint(fabsf(acc[mt][nt][v]) - kCert * (l_all + x_all * wl[v]) * e[v]));
                }
            }
        }
        if (__any(worst >= 0x7f800000u)) {
            const int ln = lane_again();
            float l[MT], x[MT];
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) l[mt] = x[mt] = 0.f;
            const char* rec = halo0 + (TW == 8 ? (((ln & 15) >> 3) << row_lg) * HW + (ln & 7) : ln & 15) * PITCH + kLossAt;
#pragma nounroll
            for (int a = 0; a < fh; ++a)
#pragma nounroll
                for (int b = 0; b < fw; ++b)
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt) {
                        const float2 q = *reinterpret_cast<const float2*>(rec + (tile_off(mt) + (a * tap_row + b) * PITCH));
                        l[mt] += q.x;
                        x[mt] = fmaxf(x[mt], q.y);
                    }
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                size_t o;
                const bool ok = out_pos((wm * MT + mt) * 16 + (ln & 15), o);
                int here = 0;
                asm volatile("" : "+s"(here));
                const float* const sc = w_scale + here;
                const float xs = largest(x[mt]);
                // bit nt 4 + v: output v of tile (mt, nt).  (Padded channels have zero weights and no
                // threshold; an infinity makes them NaN, which a projection would add.)
                uint32_t bad = 0;
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) {
                    floatx4 e, wl;
                    load_scale(sc, nt, ln, e, wl);
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        // (explicit fmas: the same decision in every instantiation)
                        const float d = fmaf(-kCert * fmaf(xs, wl[v], 0x1p28f * l[mt]), e[v], fabsf(acc[mt][nt][v]));
                        bad |= (uint32_t)(__float_as_uint(d) >= 0x7f800000u) << (nt * 4 + v);
                    }
                }
                if (!ok) bad = 0;
                if constexpr (EPI == kEpiPool) {
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt) {
                        if (!__any(bad >> (nt * 4) & 15)) continue;
                        floatx4 sum[1];
                        exact_sums(mt, nt, ln, sum, std::integral_constant<int, 2>{});
#pragma unroll
                        for (int v = 0; v < 4; ++v) acc[mt][nt][v] = bad >> (nt * 4 + v) & 1 ? sum[0][v] : acc[mt][nt][v];
                    }
                } else {
                    redo |= __any(bad != 0);
                    *bad_mask(mt, ln) = (uint16_t)bad;
                }
            }
        }
    }
    // first channel of the lane's run of four in tile nt
    auto chan = [&](int nt) { return n_base + tile_channel(BF16, nt, le_grp * 4); };
    // The stores of one activation (a compile-time constant, so the per-value
    // code has no branch on it).
    auto store_tile = [&](auto act_c) {
        constexpr int ACT = decltype(act_c)::value;
        constexpr int RUN = sizeof(Tout) == 2 ? 8 : 4;      // channels of a 16-byte store
        const bool vec = Cout % RUN == 0 && ((uintptr_t)out & 15) == 0;
        floatx4 bv[NT];
        if constexpr (BF16) {
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) bv[nt] = *reinterpret_cast<const floatx4*>(bias + chan(nt));
        }
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            size_t o;
            if (!out_pos(wm * 16 * MT + mt * 16 + le_16, o)) continue;
            Tout* dst = out + o * Cout;
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    float a = activate(ACT, BF16 ? acc[mt][nt][v] + bv[nt][v] : acc[mt][nt][v]);
                    if constexpr (ACT == 2) asm volatile("" : "+v"(a));   // one long tanh at a time
                    acc[mt][nt][v] = a;
                }
            if (vec) {
                if constexpr (sizeof(Tout) == 2) {
#pragma unroll
                    for (int nt = 0; nt < NT; nt += 2) {
                        const int c = chan(nt);
                        bf16x8 h;
#pragma unroll
                        for (int v = 0; v < 4; ++v) {
                            h[v] = (__bf16)acc[mt][nt][v];
                            h[4 + v] = (__bf16)acc[mt][nt + 1][v];
                        }
                        if (c < Cout) *reinterpret_cast<u32x4*>(dst + c) = __builtin_bit_cast(u32x4, h);
                    }
                } else {
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt)
                        if (chan(nt) < Cout) *reinterpret_cast<floatx4*>(dst + chan(nt)) = acc[mt][nt];
                }
            } else {
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        if (chan(nt) + v < Cout) store_elem(dst + chan(nt) + v, acc[mt][nt][v]);
            }
        }
    };
    // The following 1x1 convolution folded into this epilogue (kEpiProj): per output
    // sample and projection channel o (four, zero padded), the partial dot
    // product over each wave's group of 16 NT channels (64 with the 64- and
    // 128-channel N tiles, 32 with the 32-channel one),
    //   part[group][sample][o] = sum_{n in group} w2[n][o] * act(acc[sample][n] + bias[n]),
    // summed over the groups in order, with the projection's bias and activation,
    // by the step that reads it.  The groups do not depend on the N tile of the
    // launch, so every evaluation fashion sums in the same order: a lane adds the
    // products of its 4 NT channels of its sample, tile by tile, and two exchanges
    // across the four lane groups add the others', after which lane group g holds
    // output g of the sample.
    auto store_proj = [&](auto act_c) {
        constexpr int ACT = decltype(act_c)::value;
        // Loads from the read-only kernel arguments are invariant to the
        // compiler, which may move them anywhere, up to before the K loop, where
        // their registers would stay live through it: an opaque zero added to
        // the pointer per use keeps each load in its place.
        auto pinned = [](const float* q) {
            int zero_off = 0;
            asm volatile("" : "+s"(zero_off));
            return q + zero_off;
        };
        float ps[MT][4];
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int o = 0; o < 4; ++o) ps[mt][o] = 0.f;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            // One tile column at a time: its weights, then its values.
            const int c = chan(nt);
            const floatx4 b = *reinterpret_cast<const floatx4*>(pinned(bias) + c);
            const float* w2g = pinned(w2);
            floatx4 wq[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) wq[u] = *reinterpret_cast<const floatx4*>(w2g + 4 * (size_t)(c + u));
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    // Each value passes through an (empty) ordered asm statement, so
                    // the activations cannot all be computed up front, where their
                    // results would not fit beside the accumulators.
                    float x = acc[mt][nt][u];
                    asm volatile("" : "+v"(x));
                    const float a = activate(ACT, x + b[u]);
#pragma unroll
                    for (int o = 0; o < 4; ++o) ps[mt][o] += a * wq[u][o];
                }
            // ... and the column's sums are complete before the next one's values
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int o = 0; o < 4; ++o) asm volatile("" : "+v"(ps[mt][o]));
        }
        float* part_g = part + (size_t)(nb * WGN + wn) * part_stride;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            size_t o;
            const bool ok = out_pos(wm * 16 * MT + mt * 16 + le_16, o);
            // groups 0 + 2 and 1 + 3: the lower groups keep outputs 0 and 1, the upper 2 and 3
            const auto r0 = __builtin_amdgcn_permlane32_swap(__float_as_uint(ps[mt][0]), __float_as_uint(ps[mt][2]),
                                                             false, false);
            const auto r1 = __builtin_amdgcn_permlane32_swap(__float_as_uint(ps[mt][1]), __float_as_uint(ps[mt][3]),
                                                             false, false);
            const float s0 = __uint_as_float(r0[0]) + __uint_as_float(r0[1]);
            const float s1 = __uint_as_float(r1[0]) + __uint_as_float(r1[1]);
            // even and odd groups: the even ones keep the first of their two outputs
            const auto r2 = __builtin_amdgcn_permlane16_swap(__float_as_uint(s0), __float_as_uint(s1), false, false);
            const float sum = __uint_as_float(r2[0]) + __uint_as_float(r2[1]);
            if (ok) part_g[o * 4 + le_grp] = sum;
        }
    };
    // kEpiPool (fragments of one row, binary32, one wave column): per group of
    // 32 channels (two tile columns of every wave) the tile's activations
    // go to LDS as [256][32 + 4] floats (37 KB: within the halo's 42 KB, so three
    // workgroups still fit a CU); each thread then forms the maxima of k
    // consecutive samples for the tile's first TW - k + 1 positions
    // (neighbouring tiles overlap by k - 1 samples, so every window lies inside
    // one tile) and writes each maximum straight to its fragment: sample x of
    // input fragment f goes to sample x div k of fragment (x mod k) F + f, F the
    // launch's fragment count (Lemma "frag-ops" along the row).
    auto store_pool = [&](auto act_c) {
        constexpr int ACT = decltype(act_c)::value;
        constexpr int POOL_PITCH = 32 + 4;
        constexpr int CQ = 32 / 4;
        float* tl = reinterpret_cast<float*>(lds);
        const int nfrag = ntiles / tilesX;                       // fragments of the launch (tilesY = 1)
        const int npos = TW - pool_k + 1;
#pragma unroll
        for (int n2 = 0; n2 < NT; n2 += 2) {
            __syncthreads();                                     // the halo / the previous group is done with
#pragma unroll
            for (int nt = n2; nt < n2 + 2; ++nt) {
                const floatx4 b = *reinterpret_cast<const floatx4*>(bias + chan(nt));
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) {
                    const int m = wm * 16 * MT + mt * 16 + le_16;
                    floatx4 a;
#pragma unroll
                    for (int v = 0; v < 4; ++v) a[v] = activate(ACT, acc[mt][nt][v] + b[v]);
                    *reinterpret_cast<floatx4*>(tl + m * POOL_PITCH + (nt - n2) * 16 + le_grp * 4) = a;
                }
            }
            __syncthreads();
            // a thread takes channels 4 cq .. of every 32nd window; (xq, xr) = window x div and mod k
            const int cq = tid % CQ, c0 = n_base + n2 * 16 + cq * 4;
            int xq = (tx0 + tid / CQ) / pool_k, xr = tx0 + tid / CQ - xq * pool_k;
            for (int pp = tid / CQ; pp < npos; pp += THREADS / CQ) {
                if (tx0 + pp >= pool_k * pool_U || c0 >= Cout) break;
                floatx4 mx = *reinterpret_cast<const floatx4*>(tl + pp * POOL_PITCH + cq * 4);
                for (int t = 1; t < pool_k; ++t) {
                    const floatx4 q = *reinterpret_cast<const floatx4*>(tl + (pp + t) * POOL_PITCH + cq * 4);
#pragma unroll
                    for (int e = 0; e < 4; ++e) mx[e] = fmaxf(mx[e], q[e]);
                }
                *reinterpret_cast<floatx4*>(reinterpret_cast<float*>(out) + (size_t)(xr * nfrag + f) * pool_U * Cout +
                                            (size_t)xq * Cout + c0) = mx;
                xq += (THREADS / CQ) / pool_k;
                xr += (THREADS / CQ) % pool_k;
                if (xr >= pool_k) {
                    xr -= pool_k;
                    ++xq;
                }
            }
        }
    };
    if constexpr (EPI == kEpiStore && !BF16) {
        // the bias once, ahead of the activations' code, in place
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            int here = 0;                     // keeps the load in its place
            asm volatile("" : "+s"(here));
            const floatx4 b = *reinterpret_cast<const floatx4*>(bias + here + chan(nt));
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) acc[mt][nt] += b;
        }
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) asm volatile("" : "+v"(acc[mt][nt]));
    }
    auto epilogue = [&](auto act_c) {
        if constexpr (EPI == kEpiPool) store_pool(act_c);
        else if constexpr (EPI == kEpiProj) store_proj(act_c);
        else store_tile(act_c);
    };
    if (act == 1)
        epilogue(std::integral_constant<int, 1>{});
    else if (act == 2)
        epilogue(std::integral_constant<int, 2>{});
    else
        epilogue(std::integral_constant<int, 0>{});
    if constexpr (!BF16 && EPI != kEpiPool) {
        if (!redo) return;
        // what has failed, over what the epilogue stored: single outputs, or (kEpiProj) the
        // group's projections of a sample with a failed channel, from all its exact sums
#pragma nounroll
        for (int mt = 0; mt < MT; ++mt) {
            const int ln = lane_again();
            const uint32_t bad = *bad_mask(mt, ln);
            const uint64_t any = __ballot(bad != 0);
            if (any == 0) continue;
            size_t o;
            const bool ok = out_pos((wm * MT + mt) * 16 + (ln & 15), o);
            int here = 0;                     // keeps the loads below in their place
            asm volatile("" : "+s"(here));
            const float* const bias_p = bias + here;
            if constexpr (EPI == kEpiStore) {
                auto store_failed = [&](int nt, const floatx4& sum) {
                    const int c = n_base + tile_channel(false, nt, (ln >> 4) * 4);
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        if (c + v < Cout && (bad >> (nt * 4 + v) & 1))
                            store_elem(out + o * Cout + c + v, activate(act, sum[v] + bias_p[c + v]));
                };
                uint32_t tiles = 0;
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) tiles |= (uint32_t)(__any(bad >> (nt * 4) & 15) != 0) << nt;
                if (tiles == (1u << NT) - 1) {               // channels that differ: all tiles side by side
                    floatx4 sum[NT];
                    exact_sums(mt, 0, ln, sum, std::integral_constant<int, 2>{});
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt) store_failed(nt, sum[nt]);
                    continue;
                }
#pragma nounroll
                for (int nt = 0; nt < NT; ++nt) {            // a single output as a rule
                    if (!(tiles >> nt & 1)) continue;
                    floatx4 sum[1];
                    exact_sums(mt, nt, ln, sum, std::integral_constant<int, 4>{});
                    store_failed(nt, sum[0]);
                }
            } else {
                const float* const w2_p = w2 + here;
                floatx4 sum[NT];
                exact_sums(mt, 0, ln, sum, std::integral_constant<int, 2>{});
                float ps[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const int c = n_base + tile_channel(false, nt, (ln >> 4) * 4 + v);
                        const float a = c < Cout ? activate(act, sum[nt][v] + bias_p[c]) : 0.f;
#pragma unroll
                        for (int q = 0; q < 4; ++q) ps[q] += a * w2_p[4 * (size_t)c + q];
                    }
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    ps[q] += __shfl_xor(ps[q], 16);
                    ps[q] += __shfl_xor(ps[q], 32);
                }
                const float p = ln < 16 ? ps[0] : ln < 32 ? ps[1] : ln < 48 ? ps[2] : ps[3];
                if (ok && ((any | any >> 16 | any >> 32 | any >> 48) >> (ln & 15) & 1))
                    part[(size_t)(nb * WGN + wn) * part_stride + o * 4 + (ln >> 4)] = p;
            }
        }
    }
}

// e_n, the power of two at or below the largest finite magnitude of channel n's
// weights (at least 2^-112, so that the weights' scale 2^14 / e_n is finite; 0 for
// a channel without any), and what the weights' parts leave out.  One workgroup per
// channel.
__global__ __launch_bounds__(256) void weight_scale_kernel(WeightView wv, int cout, int cin, int taps,
                                                          float* __restrict__ w_scale) {
    __shared__ uint32_t top;
    __shared__ float loss[256];
    const int n = blockIdx.x;
    if (threadIdx.x == 0) top = 0u;
    __syncthreads();
    uint32_t m = 0;
    const int64_t count = n < cout ? (int64_t)cin * taps : 0;
    for (int64_t i = threadIdx.x; i < count; i += 256) {
        const int64_t c = i / taps;
        const uint32_t b = __float_as_uint(wv.w[(int64_t)n * wv.sn + c * wv.sc + (i - c * taps)]) & 0x7fffffffu;
        m = max(m, b < 0x7f800000u ? b : 0u);
    }
    atomicMax(&top, m);
    __syncthreads();
    const float e = top == 0u ? 0.f : __uint_as_float(max(top & 0x7f800000u, 15u << 23));
    float sum = 0.f;
    for (int64_t i = threadIdx.x; e > 0.f && i < count; i += 256) {
        const int64_t c = i / taps;
        const float w[8] = {wv.w[(int64_t)n * wv.sn + c * wv.sc + (i - c * taps)], 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        sum += split_loss(w, 16384.f / e);
    }
    loss[threadIdx.x] = sum;
    for (int d = 128; d >= 1; d >>= 1) {
        __syncthreads();
        if ((int)threadIdx.x < d) loss[threadIdx.x] += loss[threadIdx.x + d];
    }
    if (threadIdx.x == 0) {
        w_scale[2 * n] = e;
        w_scale[2 * n + 1] = loss[0];
    }
}

// Packs a convolution's weights into the order the kernel's lanes load: slices
// [N block of rows][chunk][th][tw] of rows / 16 tiles, each 64 lanes x 16 bytes per
// part (lane 16 g + r: channels 8 g .. 8 g + 7 of row r); w32: the values themselves,
// 32 bytes a lane.  One thread per lane of a tile; rows and channels past the layer's
// are zero.
template <bool BF16>
__global__ __launch_bounds__(256) void pack_weights_kernel(WeightView wv, int cout, int cin, int taps, int rows,
                                                          int nchunks, const float* __restrict__ w_scale,
                                                          u32x4* __restrict__ dst, floatx4* __restrict__ w32,
                                                          int64_t nthreads) {
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= nthreads) return;
    const int lane = (int)(idx & 63), tiles = rows >> 4;
    int64_t t = idx >> 6;
    const int64_t tile_index = t;
    const int nt = (int)(t % tiles);
    t /= tiles;
    const int tap = (int)(t % taps);
    t /= taps;
    const int ch = (int)(t % nchunks);
    const int n = (int)(t / nchunks) * rows + tile_channel(BF16, nt, lane & 15);
    float v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const int c = ch * kCC + (lane >> 4) * 8 + e;
        v[e] = n < cout && c < cin
                   ? wv.w[(int64_t)n * wv.sn + (int64_t)c * wv.sc + (wv.flip ? taps - 1 - tap : tap)]
                   : 0.f;
    }
    if constexpr (BF16) {
        bf16x8 h;
#pragma unroll
        for (int e = 0; e < 8; ++e) h[e] = (__bf16)v[e];
        dst[tile_index * 64 + lane] = __builtin_bit_cast(u32x4, h);
    } else {
        u32x4 hi, lo;
        split_f16(v, n < cout && w_scale[2 * n] > 0.f ? 16384.f / w_scale[2 * n] : 0.f, hi, lo);
        dst[tile_index * 128 + lane] = hi;
        dst[tile_index * 128 + 64 + lane] = lo;
        w32[(tile_index * 64 + lane) * 2] = floatx4{v[0], v[1], v[2], v[3]};
        w32[(tile_index * 64 + lane) * 2 + 1] = floatx4{v[4], v[5], v[6], v[7]};
    }
}

// ------------------------------------------------------------------ host side

int mfma_pick_bn(int cout) { return cout >= 128 ? 128 : cout >= 64 ? 64 : 32; }

size_t mfma_packed_bytes(const PlanConv& pc) {
    return (size_t)(pc.cout_pad / 16) * (pc.cin_pad / kCC) * pc.fh * pc.fw * tile_bytes(pc.impl == CONV_MFMA_BF16);
}

hipError_t launch_pack_mfma(const PlanConv& pc, hipStream_t s) {
    const bool bf16 = pc.impl == CONV_MFMA_BF16;
    const int64_t n = (int64_t)(mfma_packed_bytes(pc) / tile_bytes(bf16)) * 64;
    const dim3 grid((unsigned)ceil_div64(n, 256));
    if (!bf16)
        weight_scale_kernel<<<dim3((unsigned)pc.cout_pad), 256, 0, s>>>(pc.wv, pc.cout, pc.cin, pc.fh * pc.fw, pc.w_scale);
    if (bf16)
        pack_weights_kernel<true><<<grid, 256, 0, s>>>(pc.wv, pc.cout, pc.cin, pc.fh * pc.fw, pc.pack_rows,
                                                       pc.cin_pad / kCC, pc.w_scale, (u32x4*)pc.w, nullptr, n);
    else
        pack_weights_kernel<false><<<grid, 256, 0, s>>>(pc.wv, pc.cout, pc.cin, pc.fh * pc.fw, pc.pack_rows,
                                                        pc.cin_pad / kCC, pc.w_scale, (u32x4*)pc.w,
                                                        (floatx4*)pc.w32, n);
    return hipGetLastError();
}

struct Tile {
    int TH, TW;
    size_t lds;
    int dbl;    // halo double-buffered
};

static size_t halo_lds(int64_t halo_px, bool bf16) {
    return (size_t)((halo_px * (bf16 ? kPitchBf16 : kPitchF32) + 127) / 128) * 128;
}

// LDS of a workgroup with one (or, bfloat16, preferably two) halo buffers of
// halo_px samples within `cap` bytes; false if not even one fits.
static bool fit_halo(int64_t halo_px, bool bf16, size_t cap, Tile* t) {
    const size_t h = halo_lds(halo_px, bf16);
    if (kLdsHead + h > cap) return false;
    t->dbl = bf16 && kLdsHead + 2 * h <= cap;
    t->lds = kLdsHead + (t->dbl ? 2 : 1) * h;
    return true;
}

// Spatial tile TH x TW = 256 output samples: the shape that wastes the fewest
// masked samples on this layer's fragment extent; among those, one whose halo can
// be double-buffered within the LDS budget of two workgroups per CU, then the
// smallest halo.  Filters whose halo fits no such budget get the LDS of a whole
// CU.  (8-wide tiles cost no more per sample than wider ones: neither read pattern
// has bank conflicts.)
static Tile pick_tile(int Hout, int Wout, int fh, int fw, size_t lds_max, bool bf16) {
    Tile best{0, 0, 0, 0};
    for (const size_t cap : {std::min(lds_max, (size_t)kMaxLds), std::min(lds_max, (size_t)kMaxLds1)}) {
        int64_t best_work = -1, best_halo = -1;
        for (int TW = 8; TW <= kBM; TW *= 2) {
            const int TH = kBM / TW;
            const int64_t halo_px = (int64_t)(TH + fh - 1) * (TW + fw - 1);
            Tile t{TH, TW, 0, 0};
            if (!fit_halo(halo_px, bf16, cap, &t)) continue;
            const int64_t work = ceil_div64(Hout, TH) * TH * ceil_div64(Wout, TW) * TW;
            const bool better = best_work < 0 || work < best_work ||
                                (work == best_work && (t.dbl > best.dbl || (t.dbl == best.dbl && halo_px < best_halo)));
            if (better) {
                best = t;
                best_work = work;
                best_halo = halo_px;
            }
        }
        if (best.TH > 0) break;
    }
    return best;
}

// Whether an fh x fw filter runs on the MFMA kernel: some spatial tile's halo has
// at most 819 samples (which fit the LDS in either type).
bool mfma_supports(int fh, int fw) {
    for (int TW = 8; TW <= kBM; TW *= 2)
        if ((int64_t)(kBM / TW + fh - 1) * (TW + fw - 1) <= 819) return true;
    return false;
}

// Flat-mode tile (TH = 1, TW = 256 consecutive positions of the flattened
// fragment batch) for fragments of Hin x Win input samples, or TH = 0 if its
// single-row halo does not fit.
static Tile flat_tile(int Win, int fh, int fw, size_t lds_max, bool bf16) {
    Tile t{1, kBM, 0, 0};
    const int64_t halo_px = kBM + (int64_t)(fh - 1) * Win + fw - 1;
    return fit_halo(halo_px, bf16, std::min(lds_max, (size_t)kMaxLds), &t) ? t : Tile{0, 0, 0, 0};
}

// The grid of one launch: a spatial tile per fragment (per phase when dilated),
// or the flat reading of the whole fragment batch when that computes at least
// 10 % fewer positions (small fragments waste most of a spatial tile; the flat
// sequence computes Hin*Win positions per fragment, of which only the last
// fh-1 rows and fw-1 columns are discarded).
struct LaunchShape {
    Tile t;
    int flat;
    int tilesY, tilesX;
    int64_t nblocks;    // 0 if no tile fits
};

// Hin x Win: the fragment extent including any zero border (which rules out the
// flat reading, allow_flat = false).
static LaunchShape launch_shape(bool bf16, int F, int Hin, int Win, int dil_h, int dil_w, int fh, int fw,
                                int nbs, bool allow_flat = true) {
    LaunchShape L{Tile{0, 0, 0, 0}, 0, 0, 0, 0};
    const size_t lds = device_lds_limit();
    if (dil_h * dil_w > 1) {
        const int Hout = Hin - dil_h * (fh - 1), Wout = Win - dil_w * (fw - 1);
        const int Hp = (int)ceil_div64(Hout, dil_h), Wp = (int)ceil_div64(Wout, dil_w);
        L.t = pick_tile(Hp, Wp, fh, fw, lds, bf16);
        if (L.t.TH == 0) return L;
        L.tilesY = (int)ceil_div64(Hp, L.t.TH);
        L.tilesX = (int)ceil_div64(Wp, L.t.TW);
        L.nblocks = (int64_t)dil_h * dil_w * L.tilesY * L.tilesX * nbs;
        return L;
    }
    const int Hout = Hin - fh + 1, Wout = Win - fw + 1;
    L.t = pick_tile(Hout, Wout, fh, fw, lds, bf16);
    const int64_t flat_len = (int64_t)F * Hin * Win;
    if (allow_flat && flat_len < (1ll << 30)) {
        const Tile ft = flat_tile(Win, fh, fw, lds, bf16);
        const int64_t work_tiles =
            L.t.TH ? (int64_t)F * ceil_div64(Hout, L.t.TH) * L.t.TH * ceil_div64(Wout, L.t.TW) * L.t.TW : -1;
        const int64_t work_flat = ceil_div64(flat_len, kBM) * kBM;
        if (ft.TH && (work_tiles < 0 || 10 * work_flat < 9 * work_tiles)) {
            L.t = ft;
            L.flat = 1;
            L.tilesY = 1;
            L.tilesX = (int)ceil_div64(flat_len, ft.TW);
            L.nblocks = (int64_t)L.tilesX * nbs;
            return L;
        }
    }
    if (L.t.TH == 0) return L;
    L.tilesY = (int)ceil_div64(Hout, L.t.TH);
    L.tilesX = (int)ceil_div64(Wout, L.t.TW);
    L.nblocks = (int64_t)F * L.tilesY * L.tilesX * nbs;
    return L;
}

// The 128-channel N tile or the 64-channel one for a launch.  A launch of fewer
// workgroups than the 512 that the GPU holds at once (two per CU) leaves CUs
// idle or half-loaded; the 64-channel tile doubles the workgroup count at 5 to 12 %
// more time per MFMA where both fill the GPU (900 to 1,300 workgroups of the 3x3
// 128 -> 128, 5x5 64 -> 256 and 6x6 256 -> 512 layers, both types).  With every
// workgroup resident, the busiest CU sets the time: ceil(blocks / 256) workgroups
// of the 128-channel tile against ceil(blocks64 / 256) of half the work each.  A lone
// workgroup per CU (one wave per SIMD) hides no MFMA latency, so up to 256
// workgroups the 64-channel tile is taken (binary32 6x6 layer, 100 workgroups: 225
// against 373 us; 3x3, 256: 65.8 against 70.0).  Over 50 to 512 workgroups of those
// layers the rule takes the faster tile or one within 5 %; from 513 to about 640,
// where the second round of the 128-channel tile is nearly empty, the 64-channel
// one would be 4 to 9 % faster, from 650 on the 128-channel one is.
PlanConv mfma_launch_variant(const PlanConv& pc, int F, int Hin, int Win, int dil_h, int dil_w, int pad_h,
                             int pad_w) {
    if (pc.impl == CONV_DIRECT || pc.bn != 128) return pc;
    const bool bf16 = pc.impl == CONV_MFMA_BF16;
    const bool flat = pad_h == 0 && pad_w == 0;
    Hin += 2 * pad_h;
    Win += 2 * pad_w;
    const LaunchShape a = launch_shape(bf16, F, Hin, Win, dil_h, dil_w, pc.fh, pc.fw,
                                       pc.cout_pad / pc.bn, flat);
    if (a.nblocks == 0 || a.nblocks >= 512) return pc;
    const LaunchShape b =
        launch_shape(bf16, F, Hin, Win, dil_h, dil_w, pc.fh, pc.fw,
                     (pc.cout + 63) / 64, flat);
    if (b.nblocks == 0) return pc;
    if (a.nblocks > 256 && 11 * ceil_div64(b.nblocks, 256) >= 20 * ceil_div64(a.nblocks, 256)) return pc;
    PlanConv alt = pc;
    alt.bn = 64;             // half of a slice of the 128-row packing
    alt.cout_pad = (pc.cout + 63) / 64 * 64;
    return alt;
}

int mfma_tile_mode(const PlanConv& pc, int F, int Hin, int Win, int dil_h, int dil_w, int pad_h, int pad_w) {
    if (pc.impl == CONV_DIRECT) return -1;
    if (dil_h * dil_w > 1) return 2;
    const bool padded = pad_h > 0 || pad_w > 0;
    const LaunchShape L = launch_shape(pc.impl == CONV_MFMA_BF16, F, Hin + 2 * pad_h, Win + 2 * pad_w, dil_h,
                                       dil_w, pc.fh, pc.fw, pc.cout_pad / pc.bn, !padded);
    return L.flat ? 1 : 0;
}

// The halo of a one-row pooled tile (kEpiPool) in the LDS of two workgroups per CU,
// or false: a filter of more than 244 columns, or of two rows and more, is wider than
// that and takes the tile that suits it, with the pool in a launch of its own.
static bool pool_halo(const PlanConv& pc, Tile* t) {
    *t = Tile{1, kBM, 0, 0};
    return fit_halo((int64_t)pc.fh * (kBM + pc.fw - 1), pc.impl == CONV_MFMA_BF16,
                    std::min(device_lds_limit(), (size_t)kMaxLds), t);
}

bool mfma_pool_fits(const PlanConv& pc) {
    Tile t;
    return pool_halo(pc, &t);
}

template <bool BF16, typename Tout, int WGM, int WGN, int MT, int NT, int EPI>
static hipError_t run_mfma(const void* in, int F, int Hin, int Win, int dil_h, int dil_w, int pad_h, int pad_w,
                           const PlanConv& pc, void* out, float* part, int pool_k, hipStream_t s) {
    using Cfg = MfmaCfg<WGM, WGN, MT, NT>;
    const bool dilated = dil_h * dil_w > 1;
    const bool padded = pad_h > 0 || pad_w > 0;
    if (dilated && F != 1) return hipErrorInvalidValue;   // dilated: one signal, tiled per phase
    if (padded && (dilated || pad_h < 0 || pad_w < 0)) return hipErrorInvalidValue;
    const int nbs = pc.cout_pad / Cfg::BN;
    LaunchShape L = launch_shape(BF16, F, Hin + 2 * pad_h, Win + 2 * pad_w, dil_h, dil_w, pc.fh, pc.fw, nbs,
                                 !padded);
    if (L.nblocks == 0) return hipErrorInvalidConfiguration;
    // A single channel chunk reads one halo: the second buffer would only halve
    // the workgroups that fit a CU.
    if (pc.cin_pad == kCC && L.t.dbl) {
        L.t.dbl = 0;
        L.t.lds = kLdsHead + (L.t.lds - kLdsHead) / 2;
    }
    // kEpiPool: spatial tiles of one row of BM samples, stepped by BM - k + 1
    // columns, and LDS for the tile's activations
    int tile_step_w = L.t.TW, pool_U = 0;
    if constexpr (EPI == kEpiPool) {
        const int Wout = Win - pc.fw + 1;
        if (BF16 || WGN != 1 || dil_h * dil_w > 1 || pad_h || pad_w || Hin != pc.fh || pool_k < 2 ||
            pool_k >= kBM || (Wout - pool_k + 1) % pool_k != 0 || pc.cout % 4 != 0)
            return hipErrorInvalidValue;
        pool_U = (Wout - pool_k + 1) / pool_k;
        tile_step_w = kBM - pool_k + 1;
        if (!pool_halo(pc, &L.t)) return hipErrorInvalidValue;
        L.t.lds = std::max(L.t.lds, (size_t)kBM * (32 + 4) * sizeof(float));
        L.flat = 0;
        L.tilesY = 1;
        L.tilesX = (int)ceil_div64((int64_t)pool_k * pool_U, tile_step_w);
        L.nblocks = (int64_t)F * L.tilesX * nbs;
    }
    if (L.nblocks >= (1ll << 31)) return hipErrorInvalidConfiguration;
    auto kern = conv_mfma_kernel<BF16, Tout, WGM, WGN, MT, NT, EPI>;
    hipError_t e = allow_dynamic_lds((const void*)kern, L.t.lds);
    if (e != hipSuccess) return e;
    const int nchunks = pc.cin_pad / kCC;
    const int Hout = Hin + 2 * pad_h - dil_h * (pc.fh - 1), Wout = Win + 2 * pad_w - dil_w * (pc.fw - 1);
    if (EPI == kEpiProj && (padded || !pc.w2)) return hipErrorInvalidValue;
    const int64_t part_stride = EPI == kEpiProj ? (int64_t)F * Hout * Wout * 4 : 0;
    // what K binary32 additions lose as a random walk: sqrt(K) 2^-24 of the sum
    const float cert = 16777216.f / std::sqrt((float)pc.fh * (float)pc.fw * (float)pc.cin);
    if (L.flat) {
        // one "fragment" of 1 x (F * Hin * Win) samples for the staging and the tile grid
        const int flat_len = (int)((int64_t)F * Hin * Win);   // below 2^30 in flat mode
        kern<<<dim3((unsigned)L.nblocks), kThreads, L.t.lds, s>>>(
            (const char*)in, 1, flat_len, pc.cin, (const char*)pc.w, pc.pack_rows, pc.b, pc.fh, pc.fw, pc.cout, pc.act, nchunks,
            (Tout*)out, Hout, Wout, 1, L.t.TW, 1, L.tilesX, nbs, L.t.dbl, Hin, Win, 1, 1, 0, 0, pc.w2, part,
            part_stride, L.t.TW, 0, 0, pc.w32, cert, pc.w_scale);
        return hipGetLastError();
    }
    kern<<<dim3((unsigned)L.nblocks), kThreads, L.t.lds, s>>>(
        (const char*)in, Hin, Win, pc.cin, (const char*)pc.w, pc.pack_rows, pc.b, pc.fh, pc.fw, pc.cout, pc.act, nchunks,
        (Tout*)out, Hout, Wout, L.t.TH, L.t.TW, L.tilesY, L.tilesX, nbs, L.t.dbl, 0, 0, dil_h, dil_w, pad_h, pad_w,
        pc.w2, part, part_stride, tile_step_w, pool_k, pool_U, pc.w32, cert, pc.w_scale);
    return hipGetLastError();
}

template <bool BF16, typename Tout, int EPI = kEpiStore>
static hipError_t dispatch_bn(const void* in, int F, int Hin, int Win, int dh, int dw, int ph, int pw,
                              const PlanConv& pc, void* out, hipStream_t s, float* part = nullptr, int pool_k = 0) {
    switch (pc.bn) {
        case 128:
            if constexpr (EPI == kEpiPool) return hipErrorInvalidValue;   // one wave column only
            else return run_mfma<BF16, Tout, 2, 2, 8, 4, EPI>(in, F, Hin, Win, dh, dw, ph, pw, pc, out, part, 0, s);
        case 64: return run_mfma<BF16, Tout, 4, 1, 4, 4, EPI>(in, F, Hin, Win, dh, dw, ph, pw, pc, out, part, pool_k, s);
        case 32: return run_mfma<BF16, Tout, 4, 1, 4, 2, EPI>(in, F, Hin, Win, dh, dw, ph, pw, pc, out, part, pool_k, s);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_conv_mfma_f32(const float* in, int F, int Hin, int Win, int dil_h, int dil_w, const PlanConv& pc,
                                float* out, hipStream_t s) {
    return dispatch_bn<false, float>(in, F, Hin, Win, dil_h, dil_w, 0, 0, pc, out, s);
}

hipError_t launch_conv_mfma_f32_padded(const float* in, int F, int Hin, int Win, int pad_h, int pad_w,
                                       const PlanConv& pc, float* out, hipStream_t s) {
    return dispatch_bn<false, float>(in, F, Hin, Win, 1, 1, pad_h, pad_w, pc, out, s);
}

hipError_t launch_conv_mfma_bf16(dss_dtype tout, const uint16_t* in, int F, int Hin, int Win, int dil_h, int dil_w,
                                 const PlanConv& pc, void* out, hipStream_t s) {
    if (tout == DSS_F32) return dispatch_bn<true, float>(in, F, Hin, Win, dil_h, dil_w, 0, 0, pc, out, s);
    return dispatch_bn<true, uint16_t>(in, F, Hin, Win, dil_h, dil_w, 0, 0, pc, out, s);
}

hipError_t launch_conv_mfma_proj(const void* in, int F, int Hin, int Win, int dil_h, int dil_w, const PlanConv& pc,
                                 float* part, hipStream_t s) {
    if (pc.impl == CONV_MFMA_BF16)
        return dispatch_bn<true, float, kEpiProj>(in, F, Hin, Win, dil_h, dil_w, 0, 0, pc, nullptr, s, part);
    if (pc.impl == CONV_MFMA_F32)
        return dispatch_bn<false, float, kEpiProj>(in, F, Hin, Win, dil_h, dil_w, 0, 0, pc, nullptr, s, part);
    return hipErrorInvalidValue;
}

hipError_t launch_conv_mfma_pool(const float* in, int F, int Hin, int Win, const PlanConv& pc, int pool_k, float* out,
                                 hipStream_t s) {
    if (pc.impl != CONV_MFMA_F32) return hipErrorInvalidValue;
    return dispatch_bn<false, float, kEpiPool>(in, F, Hin, Win, 1, 1, 0, 0, pc, out, s, nullptr, pool_k);
}

}  // namespace dss
