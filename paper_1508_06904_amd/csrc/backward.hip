// Kernels of the backward pass through the dense evaluation (binary32).
//
// The transformed network computes the same function as the strided network on
// every window (Theorem "processing chain", Sect. 4.3), so its gradients for a
// whole image are obtained by backpropagating through its own steps in reverse;
// the paper notes (Sect. 6.2, fine-tuning on entire images) that the gradients
// of Stuff and Trim are trivial, that Frag and Defrag are inverse permutations
// of each other, and that the sliding max-pool needs only elementary calculus.
//
//  frag_scatter_grad   transpose of Defrag_{k*_L} + Trim: the upstream gradient
//                      of the dense output [C][O_h][O_w] written into the final
//                      fragment layout [F][U_h][U_w][C] (zero for the trimmed
//                      positions).
//  pool_frag_backward  transpose of Frag_k after the sliding max-pool, fused with
//                      the activation's derivative: every pool input sample
//                      gathers the gradients of the (at most k_h k_w) sliding
//                      windows whose maximum it is.  The maximum of a window is
//                      its first maximal sample in row-major order, the rule the
//                      strided network's max-pool gradient uses too.
//  act_backward        dy = g * act'(a) for a convolution without a pool.
//  pad_grad            zero border of fh-1 x fw-1 around every fragment: the input
//                      gradient is a valid convolution of the bordered gradient
//                      with the transposed, flipped filters.  The MFMA convolution
//                      reads the border virtually; this copy feeds the direct
//                      kernel (input gradients into few channels).
//  wgrad_mfma          dW[o][i][t] = sum_p dy[p][o] x[p + t][i]: per tap a GEMM
//                      over all output positions p of all fragments (MFMA
//                      32x32x2 binary32); a workgroup takes the taps of one
//                      filter row, which share their operand rows shifted by
//                      the tap; split over p, partial sums reduced in a fixed
//                      order by wgrad_reduce.  The same launch sums dy over p for
//                      the bias gradient db[o].
//  narrow_backward     the whole backward step of a final 1x1 layer to few outputs
//                      in one pass over its input.
//  crop_to_planar      transpose of Stuff: the stuffed input's gradient cropped
//                      to the signal and written planar.
#include <algorithm>
#include <type_traits>

#include "dev_common.h"
#include "dss_internal.h"

namespace dss {

constexpr int kBT = 256;

// ------------------------------------------------------------------ frag_scatter_grad
__global__ __launch_bounds__(kBT) void frag_scatter_grad_kernel(const float* __restrict__ g, int C, int O_h, int O_w,
                                                               int K_h, int K_w, int U_h, int U_w,
                                                               float* __restrict__ out) {
    const int64_t p = (int64_t)blockIdx.x * kBT + threadIdx.x;
    const int64_t per = (int64_t)U_h * U_w;
    if (p >= (int64_t)K_h * K_w * per) return;
    const int f = (int)(p / per);
    const int q = (int)(p % per);
    const int y = q / U_w, x = q % U_w;
    const int i = y * K_h + f / K_w, j = x * K_w + f % K_w;    // dense position of this fragment sample
    const bool in = i < O_h && j < O_w;
    float* o = out + p * C;
    for (int c = 0; c < C; ++c) o[c] = in ? g[((int64_t)c * O_h + i) * O_w + j] : 0.f;
}

hipError_t launch_frag_scatter_grad(const float* g, int C, int O_h, int O_w, int K_h, int K_w, int U_h, int U_w,
                                    float* out, hipStream_t s) {
    const int64_t n = (int64_t)K_h * K_w * U_h * U_w;
    frag_scatter_grad_kernel<<<dim3((unsigned)ceil_div64(n, kBT)), kBT, 0, s>>>(g, C, O_h, O_w, K_h, K_w, U_h, U_w, out);
    return hipGetLastError();
}

// ------------------------------------------------------------------ activation derivative
__device__ __forceinline__ float act_grad(int act, float a) {
    if (act == DSS_ACT_RELU) return a > 0.f ? 1.f : 0.f;
    if (act == DSS_ACT_TANH) return 1.f - a * a;
    return 1.f;
}

// ------------------------------------------------------------------ pool_frag_backward
// One thread per (input fragment, pool-input sample, group of V channels).
template <int V>
__global__ __launch_bounds__(kBT) void pool_frag_backward_kernel(const float* __restrict__ g,
                                                                const float* __restrict__ a, int S_h, int S_w,
                                                                int E_h, int E_w, int C, int k_h, int k_w, int act,
                                                                float* __restrict__ out) {
    const int CV = C / V;
    const int P_h = E_h - k_h + 1, P_w = E_w - k_w + 1;      // sliding-pool extents
    const int U_h = P_h / k_h, U_w = P_w / k_w;
    const int64_t total = (int64_t)S_h * S_w * E_h * E_w * CV;
    const int64_t idx = (int64_t)blockIdx.x * kBT + threadIdx.x;
    if (idx >= total) return;
    const int cv = (int)(idx % CV);
    int64_t t = idx / CV;
    const int x = (int)(t % E_w);
    t /= E_w;
    const int y = (int)(t % E_h);
    const int s = (int)(t / E_h);
    const int b_h = s / S_w, b_w = s % S_w;
    const float* frag = a + (int64_t)s * E_h * E_w * C + cv * V;

    float acc[V];
#pragma unroll
    for (int e = 0; e < V; ++e) acc[e] = 0.f;
    for (int dy = 0; dy < k_h; ++dy) {
        const int py = y - dy;
        if (py < 0 || py >= P_h) continue;
        for (int dx = 0; dx < k_w; ++dx) {
            const int px = x - dx;
            if (px < 0 || px >= P_w) continue;
            // first maximum of window (py, px), per channel
            float best[V];
            int arg[V];
            VecIO<float, V>::load(frag + ((int64_t)py * E_w + px) * C, best);
#pragma unroll
            for (int e = 0; e < V; ++e) arg[e] = 0;
            for (int a2 = 0; a2 < k_h; ++a2)
                for (int b2 = 0; b2 < k_w; ++b2) {
                    if ((a2 | b2) == 0) continue;
                    float v[V];
                    VecIO<float, V>::load(frag + ((int64_t)(py + a2) * E_w + px + b2) * C, v);
#pragma unroll
                    for (int e = 0; e < V; ++e)
                        if (v[e] > best[e]) {
                            best[e] = v[e];
                            arg[e] = a2 * k_w + b2;
                        }
                }
            const int f_new = ((py % k_h) * S_h + b_h) * (k_w * S_w) + (px % k_w) * S_w + b_w;
            float gv[V];
            VecIO<float, V>::load(g + (((int64_t)f_new * U_h + py / k_h) * U_w + px / k_w) * C + cv * V, gv);
            const int me = dy * k_w + dx;
#pragma unroll
            for (int e = 0; e < V; ++e)
                if (arg[e] == me) acc[e] += gv[e];
        }
    }
    if (act != DSS_ACT_NONE) {
        float av[V];
        VecIO<float, V>::load(frag + ((int64_t)y * E_w + x) * C, av);
#pragma unroll
        for (int e = 0; e < V; ++e) acc[e] *= act_grad(act, av[e]);
    }
    VecIO<float, V>::store(out + (((int64_t)s * E_h + y) * E_w + x) * C + cv * V, acc);
}

// The same for 2 x 2 windows: a thread walks NY rows of one column (four channels),
// so a sample is loaded three times (its own column and both neighbours') instead of
// 17 times, a window is compared twice instead of four times, and the index divisions are
// made once per strip.  A window row gives its two gradients to the sample row it
// starts in at once and keeps those of the next one; every sample adds its windows'
// gradients in the general kernel's order, so the bits are the same.
// Bound by HBM: a and g read once, out written once.  256 channels of 1,877,089 positions
// 2.97 -> 1.26 ms (4.6 TB/s), of 200,704 0.176 -> 0.096 ms.  Strips of 16 rows read a
// sixteenth more than their rows; without them each row would be read twice.
template <int NY>
__global__ __launch_bounds__(kBT) void pool_frag_backward_2x2_kernel(const float* __restrict__ g,
                                                                    const float* __restrict__ a, int S_h, int S_w,
                                                                    int E_h, int E_w, int C, int act,
                                                                    float* __restrict__ out) {
    const int CV = C / 4;
    const int P_h = E_h - 1, P_w = E_w - 1;      // sliding-pool extents
    const int U_h = P_h / 2, U_w = P_w / 2;
    const int strips = (E_h + NY - 1) / NY;
    const int64_t total = (int64_t)S_h * S_w * strips * E_w * CV;
    const int64_t idx = (int64_t)blockIdx.x * kBT + threadIdx.x;
    if (idx >= total) return;
    const int cv = (int)(idx % CV);
    int64_t t = idx / CV;
    const int x = (int)(t % E_w);
    t /= E_w;
    const int y0 = (int)(t % strips) * NY, y1 = min(y0 + NY, E_h);
    const int s = (int)(t / strips);
    const int b_h = s / S_w, b_w = s - b_h * S_w;
    const int64_t row = (int64_t)E_w * C;
    const float* frag = a + (int64_t)s * E_h * row + cv * 4;
    const int64_t col[3] = {(int64_t)max(x - 1, 0) * C, (int64_t)x * C, (int64_t)min(x + 1, E_w - 1) * C};
    // windows starting in column x (d = 0) and x - 1 (d = 1): whether there are any, and their place in g
    const bool has[2] = {x < P_w, x > 0};
    const int64_t per = (int64_t)U_h * U_w * C;
    int64_t g_col[2];
#pragma unroll
    for (int d = 0; d < 2; ++d) {
        const int px = max(x - d, 0);
        g_col[d] = ((px & 1) * S_w + b_w) * per + (int64_t)(px >> 1) * C + cv * 4;
    }
    float4 up[3], lo[3];                         // a at rows py and py + 1, columns x - 1 .. x + 1
    float4 carry[2];
    auto load_row = [&](int y, float4(&r)[3]) {
        const float* q = frag + y * row;
#pragma unroll
        for (int k = 0; k < 3; ++k) r[k] = *reinterpret_cast<const float4*>(q + col[k]);
    };
    auto at = [](const float4& v, int e) { return e == 0 ? v.x : e == 1 ? v.y : e == 2 ? v.z : v.w; };
    auto put = [](float4& v, int e, float f) { (e == 0 ? v.x : e == 1 ? v.y : e == 2 ? v.z : v.w) = f; };
    carry[0] = carry[1] = make_float4(0.f, 0.f, 0.f, 0.f);
    load_row(max(y0 - 1, 0), up);
    for (int py = y0 - 1; py < y1; ++py) {
        load_row(min(py + 1, E_h - 1), lo);
        float4 now[2], next[2];
#pragma unroll
        for (int d = 0; d < 2; ++d) {
            now[d] = next[d] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (py < 0 || py >= P_h || !has[d]) continue;
            const float4 gv = *reinterpret_cast<const float4*>(
                g + ((int64_t)((py & 1) * S_h + b_h) * (2 * S_w)) * per + (int64_t)(py >> 1) * U_w * C + g_col[d]);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                // first maximum of the window, row-major
                float best = at(up[1 - d], e);
                int arg = 0;
                const float v1 = at(up[2 - d], e), v2 = at(lo[1 - d], e), v3 = at(lo[2 - d], e);
                if (v1 > best) { best = v1; arg = 1; }
                if (v2 > best) { best = v2; arg = 2; }
                if (v3 > best) { best = v3; arg = 3; }
                put(now[d], e, arg == d ? at(gv, e) : 0.f);
                put(next[d], e, arg == 2 + d ? at(gv, e) : 0.f);
            }
        }
        if (py >= y0) {
            float4 r;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                float v = 0.f;
                v += at(now[0], e);
                v += at(now[1], e);
                v += at(carry[0], e);
                v += at(carry[1], e);
                if (act != DSS_ACT_NONE) v *= act_grad(act, at(up[1], e));
                put(r, e, v);
            }
            *reinterpret_cast<float4*>(out + ((int64_t)s * E_h + py) * row + (int64_t)x * C + cv * 4) = r;
        }
#pragma unroll
        for (int k = 0; k < 3; ++k) up[k] = lo[k];
        carry[0] = next[0];
        carry[1] = next[1];
    }
}

hipError_t launch_pool_frag_backward(const float* g, const float* a, int S_h, int S_w, int E_h, int E_w, int C,
                                     int k_h, int k_w, int act, float* out, hipStream_t s) {
    const int64_t n = (int64_t)S_h * S_w * E_h * E_w;
    if (C % 4 == 0 && k_h == 2 && k_w == 2) {
        constexpr int NY = 16;
        const int64_t m = (int64_t)S_h * S_w * ((E_h + NY - 1) / NY) * E_w * (C / 4);
        pool_frag_backward_2x2_kernel<NY><<<dim3((unsigned)ceil_div64(m, kBT)), kBT, 0, s>>>(g, a, S_h, S_w, E_h, E_w, C,
                                                                                            act, out);
        return hipGetLastError();
    }
    if (C % 4 == 0) {
        pool_frag_backward_kernel<4><<<dim3((unsigned)ceil_div64(n * (C / 4), kBT)), kBT, 0, s>>>(
            g, a, S_h, S_w, E_h, E_w, C, k_h, k_w, act, out);
    } else {
        pool_frag_backward_kernel<1><<<dim3((unsigned)ceil_div64(n * C, kBT)), kBT, 0, s>>>(
            g, a, S_h, S_w, E_h, E_w, C, k_h, k_w, act, out);
    }
    return hipGetLastError();
}

// ------------------------------------------------------------------ act_backward
__global__ __launch_bounds__(kBT) void act_backward_kernel(const float* __restrict__ g, const float* __restrict__ a,
                                                          int64_t n, int act, float* __restrict__ out) {
    const int64_t p = (int64_t)blockIdx.x * kBT + threadIdx.x;
    if (p < n) out[p] = g[p] * act_grad(act, a[p]);
}

hipError_t launch_act_backward(const float* g, const float* a, int64_t n, int act, float* out, hipStream_t s) {
    act_backward_kernel<<<dim3((unsigned)ceil_div64(n, kBT)), kBT, 0, s>>>(g, a, n, act, out);
    return hipGetLastError();
}

// ------------------------------------------------------------------ pad_grad
__global__ __launch_bounds__(kBT) void pad_grad_kernel(const float* __restrict__ in, int F, int E_h, int E_w, int C,
                                                      int p_h, int p_w, float* __restrict__ out) {
    const int Wp = E_w + 2 * p_w, Hp = E_h + 2 * p_h;
    const int64_t total = (int64_t)F * Hp * Wp * C;
    const int64_t idx = (int64_t)blockIdx.x * kBT + threadIdx.x;
    if (idx >= total) return;
    const int c = (int)(idx % C);
    int64_t t = idx / C;
    const int x = (int)(t % Wp) - p_w;
    t /= Wp;
    const int y = (int)(t % Hp) - p_h;
    const int64_t f = t / Hp;
    const bool in_range = y >= 0 && y < E_h && x >= 0 && x < E_w;
    out[idx] = in_range ? in[((f * E_h + y) * E_w + x) * C + c] : 0.f;
}

hipError_t launch_pad_grad(const float* in, int F, int E_h, int E_w, int C, int p_h, int p_w, float* out,
                           hipStream_t s) {
    const int64_t n = (int64_t)F * (E_h + 2 * p_h) * (E_w + 2 * p_w) * C;
    pad_grad_kernel<<<dim3((unsigned)ceil_div64(n, kBT)), kBT, 0, s>>>(in, F, E_h, E_w, C, p_h, p_w, out);
    return hipGetLastError();
}

// ------------------------------------------------------------------ wgrad (MFMA)
typedef float floatx16 __attribute__((ext_vector_type(16)));

constexpr int kWT = 64;               // workgroup tile: 64 output x 64 input channels
constexpr int kKC = 32;               // positions per chunk
constexpr int kWP = kWT + 32;         // LDS row pitch in floats: the two half-waves of a read
                                      // (rows p and p + 1) hit disjoint banks
constexpr int kMaxTT = 8;             // taps of one filter row per workgroup
constexpr int kMaxSplitTT = 7;        // the same for the bfloat16-part kernel (accumulators and shifted operands)
constexpr int kMaxPackedTT = 4;       // MFMA tiles per wave in the packed (narrow-layer) mode

static size_t wgrad_lds_bytes(int tt) { return 2 * (size_t)(kKC + kKC + tt - 1) * kWP * sizeof(float); }

// Workgroup (o tile, i tile, tap row t_h, tap group, split) computes
//   dW[o][i][t_h][t_w] = sum_p dy[p][o] x[f][y + t_h][x + t_w][i]
// for 64 output channels, 64 input channels and the taps t_w of one group of up
// to TT consecutive taps of filter row t_h.  4 waves in a 2 x 2 grid, each a
// 32 x 32 MFMA tile per tap.
//
// Positions are numbered over the input width: q = (f E_h + y) U_w + x for
// x < U_w, of which x < E_w are output positions (dy row (f E_h + y) E_w + x)
// and the rest carry a zero gradient.  Then the input sample of tap (t_h, t_w)
// at q is the tap (t_h, 0) sample at q + t_w: within a row x + t_w < U_w for
// every output position.  A chunk of 32 positions therefore stages the dy rows
// of its 32 positions and the x rows of 32 + TT - 1 positions once, and every tap
// of the group reads its operand rows t_w further on in LDS -- TT times fewer
// global reads than one workgroup per tap.
//
// PACKED (narrow layers, at most 32 input channels): the 64 columns of an MFMA
// tile hold g = 64 / cpt taps of cpt channels each (cpt: Cin rounded up to a
// power of two, at least 4), column j being tap j / cpt and channel j % cpt, so
// a narrow layer does not spend 64-column tiles on a few channels.  Tile t of a
// workgroup covers taps t g .. t g + g - 1 of its group; the staged x rows are
// cpt floats apart and column j of tap row q reads row q + j / cpt.
template <bool VEC, int TT, bool PACKED>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void wgrad_mfma_kernel(
    const float* __restrict__ dy, const float* __restrict__ x, int E_h, int E_w, int U_h, int U_w, int Cout, int Cin,
    int fh, int fw, int Q, int nchunks, int chunk_mul, int otiles, int itiles, int ntg, int splits, int cpt,
    const uint32_t* __restrict__ flags, float* __restrict__ partial, float* __restrict__ bias_partial) {
    constexpr int RB = kKC + TT - 1;              // staged x rows per chunk (unpacked; bounds the buffer)
    extern __shared__ __attribute__((aligned(16))) float wl[];
    auto lds_a = [&](int buf) { return wl + buf * (kKC * kWP); };                  // dy rows
    auto lds_b = [&](int buf) { return wl + 2 * kKC * kWP + buf * (RB * kWP); };   // x rows
    // Workgroups are handed to the 8 XCDs round-robin by id; remap so that every
    // XCD runs one contiguous range of the logical order (o tile, i tile, tap
    // group, tap row fastest, split slowest): the workgroups on an XCD then read
    // the same chunks of dy and x from its L2.
    const int total = gridDim.x;
    const int xcd = blockIdx.x % 8, slot = blockIdx.x / 8;
    const int q8 = total / 8, r8 = total % 8;
    int bid = xcd < r8 ? xcd * (q8 + 1) + slot : r8 * (q8 + 1) + (xcd - r8) * q8 + slot;
    if (flags && !flags[bid]) return;             // after wgrad_split_kernel: only the workgroups it marked
    const int ot = bid % otiles;
    bid /= otiles;
    const int it = bid % itiles;
    bid /= itiles;
    const int tg = bid % ntg;
    bid /= ntg;
    const int th = bid % fh;
    const int split = bid / fh;
    const int g = PACKED ? kWT / cpt : 1;         // taps per MFMA tile
    const int span = TT * g;                      // taps per group
    const int tw0 = tg * span;
    const int ntt = min(span, fw - tw0);          // taps of this group
    const int rows_b = kKC + span - 1;            // staged x rows per chunk
    const int c0 = (int)((int64_t)nchunks * split / splits) * chunk_mul;
    const int c1 = (int)((int64_t)nchunks * (split + 1) / splits) * chunk_mul;
    const int o0 = ot * kWT, i0 = it * kWT;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave & 1, wn = wave >> 1, half = lane >> 5, l32 = lane & 31;
    const int s_col = (tid & 15) * 4, s_row = tid >> 4;          // staging: 16 float4 per row, 16 rows per pass
    const int rowlen = E_h * U_w;                                // positions per fragment

    floatx16 acc[TT];
#pragma unroll
    for (int t = 0; t < TT; ++t)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[t][v] = 0.f;

    float bsum = 0.f;   // sum of this lane's dy column over its positions (bias gradient)
    float4 ra[2], rb[3];
    auto load4 = [&](const float* base, int c_lo, int C, bool ok) -> float4 {
        if (!ok) return make_float4(0.f, 0.f, 0.f, 0.f);
        if (VEC) return c_lo + 3 < C ? *reinterpret_cast<const float4*>(base + c_lo) : make_float4(0.f, 0.f, 0.f, 0.f);
        float v[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = c_lo + e < C ? base[c_lo + e] : 0.f;
        return make_float4(v[0], v[1], v[2], v[3]);
    };
    auto load_chunk = [&](int c) {
        const int qc = c * kKC;
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int q = qc + s_row + 16 * k;
            const int r = q / U_w, xx = q - r * U_w;              // r = f E_h + y
            ra[k] = load4(dy + ((int64_t)r * E_w + xx) * Cout, o0 + s_col, Cout, q < Q && xx < E_w);
        }
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            int row, col;
            if constexpr (PACKED) {                 // rows of cpt floats, cpt / 4 units each
                const int u = tid + 256 * k;
                row = u / (cpt / 4);
                col = (u - row * (cpt / 4)) * 4;
            } else {
                row = s_row + 16 * k;
                col = i0 + s_col;
            }
            const int q = qc + tw0 + row;
            const int f = q / rowlen;
            const int64_t src = (int64_t)q + (int64_t)f * (fh - 1) * U_w + (int64_t)th * U_w;
            rb[k] = row < rows_b ? load4(x + src * Cin, col, Cin, q < Q) : make_float4(0.f, 0.f, 0.f, 0.f);
        }
    };
    auto store_chunk = [&](int buf) {
#pragma unroll
        for (int k = 0; k < 2; ++k)
            *reinterpret_cast<float4*>(lds_a(buf) + (s_row + 16 * k) * kWP + s_col) = ra[k];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            if constexpr (PACKED) {
                const int u = tid + 256 * k;
                if (u < rows_b * (cpt / 4)) *reinterpret_cast<float4*>(lds_b(buf) + u * 4) = rb[k];
            } else {
                if (s_row + 16 * k < RB) *reinterpret_cast<float4*>(lds_b(buf) + (s_row + 16 * k) * kWP + s_col) = rb[k];
            }
        }
    };

    if (c0 < c1) {
        load_chunk(c0);
        store_chunk(0);
    }
    __syncthreads();
    for (int c = c0; c < c1; ++c) {
        const int buf = (c - c0) & 1;
        const bool more = c + 1 < c1;
        if (more) load_chunk(c + 1);
        const float* A = lds_a(buf) + wm * 32 + l32;
        const float* Bm = lds_b(buf) + wn * 32 + l32;   // packed: column j = wn 32 + l32 of row 0
        const int bstep = PACKED ? cpt : kWP;           // floats between staged rows
        // all TT taps even in a ragged last group (the extra ones are not stored):
        // a tap-dependent branch here would keep a second copy of the accumulators
#pragma unroll 4
        for (int ks = 0; ks < kKC / 2; ++ks) {
            const int p = 2 * ks + half;
            const float av = A[p * kWP];
            bsum += av;
            float bv[TT];
#pragma unroll
            for (int t = 0; t < TT; ++t) bv[t] = PACKED ? Bm[(p + t * g) * bstep] : Bm[(p + t) * kWP];
#pragma unroll
            for (int t = 0; t < TT; ++t) acc[t] = __builtin_amdgcn_mfma_f32_32x32x2f32(av, bv[t], acc[t], 0, 0, 0);
        }
        if (more) store_chunk(buf ^ 1);
        __syncthreads();
    }

    // db[o] = sum_p dy[p][o]: one wave per output-channel half of the workgroups
    // of the first input tile, tap row and tap group adds its two half-wave sums
    bsum += __shfl_xor(bsum, 32);
    if (it == 0 && tg == 0 && th == 0 && wn == 0 && half == 0 && o0 + wm * 32 + l32 < Cout)
        bias_partial[(size_t)split * Cout + o0 + wm * 32 + l32] = bsum;

    // D[i][j] of a 32x32 tile sits in lane j + 32*((i/4)%2), register (i/8)*4 + i%4
    const int taps = fh * fw;
    const int jj = wn * 32 + l32;
    const int ii = PACKED ? jj % cpt : i0 + jj;     // input channel of this lane's column
    const int tl = PACKED ? jj / cpt : 0;           // tap of this lane's column within a tile
#pragma unroll
    for (int t = 0; t < TT; ++t) {
        const int k = t * g + tl;                   // tap within the group
        if (k >= ntt) continue;
        float* dst = partial + ((size_t)split * taps + th * fw + tw0 + k) * Cout * Cin;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int o = o0 + wm * 32 + (v >> 2) * 8 + half * 4 + (v & 3);
            if (o < Cout && ii < Cin) dst[(size_t)o * Cin + ii] = acc[t][v];
        }
    }
}

// ------------------------------------------------------------------ wgrad on bfloat16 parts
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

constexpr int kSC = 64;                    // positions per chunk
constexpr int kSParts = 3;
constexpr int kSRow = 2 * kWT + 16;        // LDS bytes per staged position and part (the 16 bytes put the four
                                           // rows of a transposing read on different banks)
constexpr int kSRowsX = kSC + 8;           // staged x positions (taps read up to 7 further on)
constexpr int kSPlaneA = kSC * kSRow, kSPlaneB = kSRowsX * kSRow;
constexpr int kSLds = kSParts * (kSPlaneA + kSPlaneB) + 64;   // the parts of dy and x, and the flags

// n / d for 0 <= n < 2^31 and a divisor of at least 2 (multiplication by its rounded-up reciprocal)
struct FastDiv {
    uint32_t mul, shift;
};
static FastDiv fast_div(uint32_t d) {
    uint32_t l = 1;
    while ((1ull << l) < d) ++l;
    return {(uint32_t)(((1ull << (31 + l)) + d - 1) / d), l - 1};
}
__device__ __forceinline__ uint32_t div_by(uint32_t n, FastDiv f) { return __umulhi(n, f.mul) >> f.shift; }

// The same weight gradient (unpacked layers, channels in fours) with every operand
// split into three bfloat16 numbers, v = b0 + b1 + b2 with b0 = bf16(v), b1 =
// bf16(v - b0), b2 = bf16(v - b0 - b1): together they hold all 24 bits, and a product
// is b0 b0 + b0 b1 + b1 b0 + b1 b1 + b0 b2 + b2 b0 (what is left out is below 2^-24 of
// it), six v_mfma_f32_16x16x32_bf16.  bfloat16 has binary32's exponents, so channels
// and positions of any magnitude stand side by side without a scale.  (Two binary16
// parts and three products under one scale per operand take half the matrix cycles,
// but lose what is 2^-15 and less of the scale's largest value, and real gradients have
// channels that are hardly ever active beside busy ones.)
//
// The contraction runs over the positions, 32 per issue.  The matrix instruction wants
// eight consecutive positions of one channel per lane; the chunk is staged as it lies
// in memory, positions of 64 channels, and read by the transposing LDS loads
// (ds_read_b64_tr_b16: four positions of a lane's channel).  A lane reads 16 positions
// of x once and shifts them in registers for every tap.  The next chunk's loads are in
// flight while a chunk is computed; its parts go to the same LDS buffer, so that two
// workgroups fit a CU, one computing while the other converts.
//
// Infinities have no finite parts, magnitudes below 2^-117 parts below bfloat16's
// subnormal numbers (which the instruction takes), and products near binary32's
// largest parts that may overflow both ways: workgroups that met such values set their
// flag, and the binary32 kernel computes their sums again.
template <int TT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void wgrad_split_kernel(
    const float* __restrict__ dy, const float* __restrict__ x, int E_h, int E_w, int U_w, int Cout, int Cin, int fh,
    int fw, int Q, int nchunks, int otiles, int itiles, int ntg, int splits, FastDiv by_row, FastDiv by_frag,
    uint32_t* __restrict__ flags, float* __restrict__ partial, float* __restrict__ bias_partial) {
    extern __shared__ __attribute__((aligned(16))) float wl[];
    char* const lds = reinterpret_cast<char*>(wl);
    uint32_t* const flag = reinterpret_cast<uint32_t*>(lds + kSLds - 64);
    const int total = gridDim.x;
    const int xcd = blockIdx.x % 8, slot = blockIdx.x / 8;
    const int q8 = total / 8, r8 = total % 8;
    const int id = xcd < r8 ? xcd * (q8 + 1) + slot : r8 * (q8 + 1) + (xcd - r8) * q8 + slot;
    int bid = id;
    const int ot = bid % otiles;
    bid /= otiles;
    const int it = bid % itiles;
    bid /= itiles;
    const int tg = bid % ntg;
    bid /= ntg;
    const int th = bid % fh;
    const int split = bid / fh;
    const int tw0 = tg * TT;
    const int ntt = min(TT, fw - tw0);
    const int c0 = (int)((int64_t)nchunks * split / splits), c1 = (int)((int64_t)nchunks * (split + 1) / splits);
    const int o0 = ot * kWT, i0 = it * kWT;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave & 1, wn = wave >> 1, grp = lane >> 4, l16 = lane & 15;
    const int s_col = (tid & 15) * 4, s_row = tid >> 4;          // staging: 16 float4 per row, 16 rows per pass

    floatx4 acc[TT][2][2];
#pragma unroll
    for (int t = 0; t < TT; ++t)
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int b = 0; b < 2; ++b) acc[t][a][b] = floatx4{0.f, 0.f, 0.f, 0.f};

    constexpr int NA = kSC / 16, NB = (kSC + TT - 1 + 15) / 16;
    floatx4 ra[NA], rb[NB];
    const bool col_a = o0 + s_col < Cout, col_b = i0 + s_col < Cin;
    auto load_chunk = [&](int c) {
        const int qc = c * kSC + s_row;
#pragma unroll
        for (int k = 0; k < NA; ++k) {
            const int q = qc + 16 * k;
            const int r = (int)div_by((uint32_t)q, by_row), xx = q - r * U_w;   // r = f E_h + y
            const float* src = dy + ((int64_t)r * E_w + xx) * Cout + o0 + s_col;
            ra[k] = q < Q && xx < E_w && col_a ? *reinterpret_cast<const floatx4*>(src) : floatx4{0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll
        for (int k = 0; k < NB; ++k) {
            const int q = qc + 16 * k + tw0;
            const int f = (int)div_by((uint32_t)q, by_frag);
            const float* src = x + ((int64_t)q + (int64_t)(f * (fh - 1) + th) * U_w) * Cin + i0 + s_col;
            rb[k] = q < Q && col_b && (16 * k + 15 < kSC + TT - 1 || s_row + 16 * k < kSC + TT - 1)
                        ? *reinterpret_cast<const floatx4*>(src)
                        : floatx4{0.f, 0.f, 0.f, 0.f};
        }
    };
    // The matrix instruction rounds its sums down a little (the mean error of a sum
    // is negative, whatever its sign), which over the positions of all splits would
    // add up.  Every other split therefore sums -dy x, and its sums are negated back.
    const uint32_t sign = split & 1 ? 0x80000000u : 0u;
    uint32_t low = ~0u;                    // twice the smallest magnitude but 0, less 1
    float high_a = 0.f, high_b = 0.f;      // the largest magnitudes (NaN, which stays NaN in every part, passes by)
    auto store_parts = [&](char* plane, int plane_bytes, int row, floatx4 r) {
        char* dst = plane + row * kSRow + s_col * 2;
#pragma unroll
        for (int p = 0; p < kSParts; ++p) {
            bf16x4 b;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                b[e] = (__bf16)r[e];
                r[e] -= (float)b[e];
            }
            *reinterpret_cast<u32x2*>(dst + p * plane_bytes) = __builtin_bit_cast(u32x2, b);
        }
    };
    auto note = [&](floatx4 r, float& high) {
#pragma unroll
        for (int e = 0; e < 4; ++e) low = min(low, (__float_as_uint(r[e]) << 1) - 1u);
        asm("v_max3_f32 %0, |%1|, |%2|, %0" : "+v"(high) : "v"(r[0]), "v"(r[1]));
        asm("v_max3_f32 %0, |%1|, |%2|, %0" : "+v"(high) : "v"(r[2]), "v"(r[3]));
    };
    auto store_chunk = [&] {
        char* const A = lds;
        char* const B = lds + kSParts * kSPlaneA;
#pragma unroll
        for (int k = 0; k < NA; ++k) {
            note(ra[k], high_a);
            floatx4 r;
#pragma unroll
            for (int e = 0; e < 4; ++e) r[e] = __uint_as_float(__float_as_uint(ra[k][e]) ^ sign);
            store_parts(A, kSPlaneA, s_row + 16 * k, r);
        }
#pragma unroll
        for (int k = 0; k < NB; ++k) {
            note(rb[k], high_b);
            if (s_row + 16 * k < kSRowsX) store_parts(B, kSPlaneB, s_row + 16 * k, rb[k]);
        }
    };

    // db[o] = sum_p dy[p][o]: the workgroups of the first input tile, tap row and tap group add their dy rows
    const bool do_bias = it == 0 && tg == 0 && th == 0;
    floatx4 bsum = {0.f, 0.f, 0.f, 0.f};
    if (tid < 3) flag[tid] = 0u;
    if (c0 < c1) load_chunk(c0);
    // transposing reads: lane j of group g reads positions 8 g + j / 4, channels 4 (j % 4) .. + 3
    // of a 16-channel tile, and receives four positions of channel j
    const int tr_off = (8 * grp + (l16 >> 2)) * kSRow + (l16 & 3) * 8;
    auto tr_read = [&](const char* p) {
        return __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)p));
    };
    const char* const A = lds + tr_off + wm * 64;
    const char* const B = lds + kSParts * kSPlaneA + tr_off + wn * 64;
    for (int c = c0; c < c1; ++c) {
        __syncthreads();                       // every wave is done with the chunk before
        store_chunk();
        if (do_bias) {
#pragma unroll
            for (int k = 0; k < NA; ++k) bsum += ra[k];
        }
        __syncthreads();
        if (c + 1 < c1) load_chunk(c + 1);
#pragma unroll
        for (int ks = 0; ks < kSC / 32; ++ks) {
            bf16x8 a[2][kSParts];
#pragma unroll
            for (int oi = 0; oi < 2; ++oi)
#pragma unroll
                for (int p = 0; p < kSParts; ++p) {
                    const char* src = A + p * kSPlaneA + ks * 32 * kSRow + oi * 32;
                    const u32x2 lo = tr_read(src), hi = tr_read(src + 4 * kSRow);
                    a[oi][p] = __builtin_bit_cast(bf16x8, u32x4{lo[0], lo[1], hi[0], hi[1]});
                }
#pragma unroll
            for (int ii = 0; ii < 2; ++ii) {
                __builtin_amdgcn_sched_barrier(0);
                // the smallest parts of x first; with part pb, dy's parts 2 - pb .. 0
#pragma unroll
                for (int pb = kSParts - 1; pb >= 0; --pb) {
                    // 16 positions of the lane's channel, and the same one position on
                    uint32_t even[8], odd[8];
                    const char* src = B + pb * kSPlaneB + ks * 32 * kSRow + ii * 32;
#pragma unroll
                    for (int k = 0; k < (TT > 1 ? 4 : 2); ++k) {
                        const u32x2 v = tr_read(src + 4 * k * kSRow);
                        even[2 * k] = v[0];
                        even[2 * k + 1] = v[1];
                    }
                    if constexpr (TT > 1) {
#pragma unroll
                        for (int k = 0; k < 7; ++k) odd[k] = __builtin_amdgcn_alignbit(even[k + 1], even[k], 16);
                    }
                    auto tap = [&](int t) {
                        const uint32_t* q = t & 1 ? odd : even;
                        const int k = t >> 1;
                        return __builtin_bit_cast(bf16x8, u32x4{q[k], q[k + 1], q[k + 2], q[k + 3]});
                    };
                    // b2's product goes to the sums; b1's two and b0's three are added up from zero first, so that
                    // 32 positions round a sum three times instead of six (relative error of N(0,1) gradients
                    // over 93,000 positions 7.0e-7 -> 3.7e-7, on the binary32 instruction 8.2e-7; 5 % of a
                    // gradient step's time)
#pragma unroll
                    for (int t0 = 0; t0 < TT; t0 += 2) {
                        floatx4 sum[2][2];
#pragma unroll
                        for (int pa = kSParts - 1 - pb; pa >= 0; --pa)
#pragma unroll
                            for (int t = t0; t < (t0 + 2 < TT ? t0 + 2 : TT); ++t)
#pragma unroll
                                for (int oi = 0; oi < 2; ++oi) {
                                    const floatx4 from = pb == kSParts - 1         ? acc[t][oi][ii]
                                                         : pa == kSParts - 1 - pb ? floatx4{0.f, 0.f, 0.f, 0.f}
                                                                                  : sum[t - t0][oi];
                                    sum[t - t0][oi] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[oi][pa], tap(t), from, 0, 0, 0);
                                }
#pragma unroll
                        for (int t = t0; t < (t0 + 2 < TT ? t0 + 2 : TT); ++t)
#pragma unroll
                            for (int oi = 0; oi < 2; ++oi) {
                                if (pb == kSParts - 1) acc[t][oi][ii] = sum[t - t0][oi];
                                else acc[t][oi][ii] += sum[t - t0][oi];
                            }
                    }
                }
            }
        }
    }

    if (low < ((10u << 23) << 1) - 1u) *flag = 1u;       // 2^-117
    atomicMax(flag + 1, __float_as_uint(high_a));
    atomicMax(flag + 2, __float_as_uint(high_b));
    __syncthreads();
    if (tid == 0) {
        // (what bfloat16 rounds to infinity, or products of parts that may be infinities of both signs)
        const float a = __uint_as_float(flag[1]), b = __uint_as_float(flag[2]);
        flags[id] = *flag != 0u || !(fmaxf(a, b) < __uint_as_float(0x7f7f8000u)) || a * b >= 0x1p120f ? 1u : 0u;
    }
    if (do_bias) {
        // rows s_row of the 16 column quads, added in order
        *reinterpret_cast<floatx4*>(lds + tid * 16) = bsum;
        __syncthreads();
        if (tid < kWT && o0 + tid < Cout) {
            const float* v = wl + (tid >> 2) * 4 + (tid & 3);
            float s = 0.f;
            for (int k = 0; k < 16; ++k) s += v[k * 64];
            bias_partial[(size_t)split * Cout + o0 + tid] = s;
        }
    }
    const int taps = fh * fw;
#pragma unroll
    for (int t = 0; t < TT; ++t) {
        if (t >= ntt) continue;
        float* dst = partial + ((size_t)split * taps + th * fw + tw0 + t) * Cout * Cin;
#pragma unroll
        for (int oi = 0; oi < 2; ++oi)
#pragma unroll
            for (int ii = 0; ii < 2; ++ii) {
                const int i = i0 + wn * 32 + ii * 16 + l16;
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int o = o0 + wm * 32 + oi * 16 + grp * 4 + v;
                    if (o < Cout && i < Cin)
                        dst[(size_t)o * Cin + i] = __uint_as_float(__float_as_uint(acc[t][oi][ii][v]) ^ sign);
                }
            }
    }
}

// dW[o][i][th][tw] = sum over splits (in order) of partial[s][tap][o][i], and
// db[o] = sum over splits (in order) of bias_partial[s][o].
__global__ __launch_bounds__(kBT) void wgrad_reduce_kernel(const float* __restrict__ partial,
                                                          const float* __restrict__ bias_partial, int splits,
                                                          int taps, int Cout, int Cin, float* __restrict__ dw,
                                                          float* __restrict__ db) {
    const int64_t n = (int64_t)Cout * Cin * taps;
    const int64_t p = (int64_t)blockIdx.x * kBT + threadIdx.x;
    if (p >= n) {
        const int64_t o = p - n;
        if (o >= Cout) return;
        float s = 0.f;
        for (int k = 0; k < splits; ++k) s += bias_partial[(int64_t)k * Cout + o];
        db[o] = s;
        return;
    }
    const int tap = (int)(p % taps);
    const int64_t oi = p / taps;                 // o * Cin + i
    const int64_t stride = (int64_t)taps * Cout * Cin;
    const float* src = partial + (int64_t)tap * Cout * Cin + oi;
    float s = 0.f;
    for (int k = 0; k < splits; ++k) s += src[k * stride];
    dw[p] = s;                                   // [o][i][th][tw] with tap = th * fw + tw
}

WgradPlan wgrad_plan(int F, int E_h, int E_w, int Cout, int Cin, int fh, int fw) {
    WgradPlan w;
    // the bfloat16-part kernel: whole float4 channel groups, and rows that its division takes
    // (more than 16 input channels: at 32 its tile is half padding and still faster than two taps side by
    // side on the binary32 instruction, 0.167 against 0.238 ms for a 5x5 32 -> 64 layer of 255 x 255 samples,
    // 0.087 against 0.111 for a 1x1 one; at 16 four taps fill that one's tile and the two are 5 % apart)
    const bool vec = Cout % 4 == 0 && Cin % 4 == 0;
    w.positions = (int64_t)F * E_h * (E_w + fw - 1);
    w.split = Cin > kWT / 4 && vec && E_w + fw - 1 >= 2 && w.positions + kMaxSplitTT + kSC < (1ll << 31);
    if (Cin <= kWT / 2 && !w.split) {
        // packed: cpt columns per tap, g taps per tile; at most kMaxPackedTT tiles,
        // the fewest MFMA tiles per row (ntg * tt), then the most taps per group
        w.packed = true;
        w.cpt = 4;
        while (w.cpt < Cin) w.cpt *= 2;
        const int g = kWT / w.cpt;
        int best_work = -1;
        for (int tt = kMaxPackedTT; tt >= 1; --tt) {
            const int ntg = (fw + tt * g - 1) / (tt * g);
            if (best_work < 0 || ntg * tt < best_work) {
                best_work = ntg * tt;
                w.tt = tt;
                w.ntg = ntg;
            }
        }
    } else {
        // the largest group of taps (at most kMaxTT) whose ragged last group wastes
        // at most a tenth of the row's MFMA work
        for (int tt = std::min(fw, vec ? kMaxSplitTT : kMaxTT); tt >= 1; --tt) {
            const int ntg = (fw + tt - 1) / tt;
            if (10 * (ntg * tt - fw) <= fw) {
                w.tt = tt;
                w.ntg = ntg;
                break;
            }
        }
    }
    const int64_t chunk = w.split ? kSC : kKC;
    w.nchunks = (w.positions + chunk - 1) / chunk;
    w.otiles = (Cout + kWT - 1) / kWT;
    w.itiles = w.packed ? 1 : (Cin + kWT - 1) / kWT;
    const int64_t base = (int64_t)w.otiles * w.itiles * fh * w.ntg;
    // About 512 workgroups run at once (two or three per CU, 53-55 KB of LDS
    // each).  Take at least eight rounds of 512 and, among the split counts up
    // to twice that, the one whose last round is fullest; every split keeps at
    // least 64 chunks, so that a workgroup's prologue and partial-sum stores stay
    // small against its loop (measured on the 512 x 512 frame: 8 -> 64 chunks
    // makes its weight gradients 6.6 -> 5.5 ms).
    const int64_t max_splits = std::max<int64_t>(1, std::min<int64_t>(4096, w.nchunks * chunk / (64 * kKC)));
    const int64_t lo = std::min(max_splits, std::max<int64_t>(1, (512 * 8 + base - 1) / base));
    const int64_t hi = std::min(max_splits, 2 * lo);
    int64_t best = lo;
    double best_fill = -1.0;
    for (int64_t sp = lo; sp <= hi; ++sp) {
        const int64_t total = base * sp;
        const double fill = (double)total / (double)(((total + 511) / 512) * 512);
        if (fill > best_fill + 1e-9) {
            best_fill = fill;
            best = sp;
        }
    }
    w.splits = (int)best;
    w.partial_floats = (int64_t)w.splits * fh * fw * Cout * Cin;
    w.bias_partial_floats = (int64_t)w.splits * Cout + (w.split ? base * w.splits : 0);   // and a flag per workgroup
    return w;
}

template <bool VEC, int TT, bool PACKED>
static hipError_t run_wgrad(const float* dy, const float* x, int E_h, int E_w, int U_h, int U_w, int Cout, int Cin,
                            int fh, int fw, const WgradPlan& w, float* partial, float* bpart, hipStream_t s) {
    const int64_t nblocks = (int64_t)w.otiles * w.itiles * fh * w.ntg * w.splits;
    if (nblocks >= (1ll << 31)) return hipErrorInvalidConfiguration;
    uint32_t* flags = nullptr;
    if constexpr (VEC && !PACKED && TT <= kMaxSplitTT) {
        if (w.split) {
            auto kern = wgrad_split_kernel<TT>;
            hipError_t e = allow_dynamic_lds((const void*)kern, kSLds);
            if (e != hipSuccess) return e;
            flags = reinterpret_cast<uint32_t*>(bpart + (int64_t)w.splits * Cout);
            kern<<<dim3((unsigned)nblocks), 256, kSLds, s>>>(
                dy, x, E_h, E_w, U_w, Cout, Cin, fh, fw, (int)w.positions, (int)w.nchunks, w.otiles, w.itiles, w.ntg,
                w.splits, fast_div((uint32_t)U_w), fast_div((uint32_t)(E_h * U_w)), flags, partial, bpart);
            e = hipGetLastError();
            if (e != hipSuccess) return e;
        }
    }
    auto kern = wgrad_mfma_kernel<VEC, TT, PACKED>;
    const size_t lds = wgrad_lds_bytes(TT);
    hipError_t e = allow_dynamic_lds((const void*)kern, lds);
    if (e != hipSuccess) return e;
    kern<<<dim3((unsigned)nblocks), 256, lds, s>>>(dy, x, E_h, E_w, U_h, U_w, Cout, Cin, fh, fw, (int)w.positions,
                                                   (int)w.nchunks, w.split ? kSC / kKC : 1, w.otiles, w.itiles, w.ntg,
                                                   w.splits, w.cpt, flags, partial, bpart);
    return hipGetLastError();
}

template <bool VEC>
static hipError_t dispatch_wgrad(const float* dy, const float* x, int E_h, int E_w, int U_h, int U_w, int Cout,
                                 int Cin, int fh, int fw, const WgradPlan& w, float* partial, float* bpart,
                                 hipStream_t s) {
    if (w.packed) {
        switch (w.tt) {
            case 1: return run_wgrad<VEC, 1, true>(dy, x, E_h, E_w, U_h, U_w, Cout, Cin, fh, fw, w, partial, bpart, s);
            case 2: return run_wgrad<VEC, 2, true>(dy, x, E_h, E_w, U_h, U_w, Cout, Cin, fh, fw, w, partial, bpart, s);
            case 3: return run_wgrad<VEC, 3, true>(dy, x, E_h, E_w, U_h, U_w, Cout, Cin, fh, fw, w, partial, bpart, s);
            case 4: return run_wgrad<VEC, 4, true>(dy, x, E_h, E_w, U_h, U_w, Cout, Cin, fh, fw, w, partial, bpart, s);
        }
        return hipErrorInvalidValue;
    }
    switch (w.tt) {
        case 1: return run_wgrad<VEC, 1, false>(dy, x, E_h, E_w, U_h, U_w, Cout, Cin, fh, fw, w, partial, bpart, s);
        case 2: return run_wgrad<VEC, 2, false>(dy, x, E_h, E_w, U_h, U_w, Cout, Cin, fh, fw, w, partial, bpart, s);
        case 3: return run_wgrad<VEC, 3, false>(dy, x, E_h, E_w, U_h, U_w, Cout, Cin, fh, fw, w, partial, bpart, s);
        case 4: return run_wgrad<VEC, 4, false>(dy, x, E_h, E_w, U_h, U_w, Cout, Cin, fh, fw, w, partial, bpart, s);
        case 5: return run_wgrad<VEC, 5, false>(dy, x, E_h, E_w, U_h, U_w, Cout, Cin, fh, fw, w, partial, bpart, s);
        case 6: return run_wgrad<VEC, 6, false>(dy, x, E_h, E_w, U_h, U_w, Cout, Cin, fh, fw, w, partial, bpart, s);
        case 7: return run_wgrad<VEC, 7, false>(dy, x, E_h, E_w, U_h, U_w, Cout, Cin, fh, fw, w, partial, bpart, s);
        case 8:
            if constexpr (!VEC)
                return run_wgrad<VEC, 8, false>(dy, x, E_h, E_w, U_h, U_w, Cout, Cin, fh, fw, w, partial, bpart, s);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_wgrad(const float* dy, const float* x, int F, int E_h, int E_w, int U_h, int U_w, int Cout, int Cin,
                        int fh, int fw, const WgradPlan& w, float* partial, float* dw, float* db, hipStream_t s) {
    (void)F;
    // positions and chunks are 32-bit in the kernel
    const int span = w.packed ? w.tt * (kWT / w.cpt) : w.tt;   // taps per group
    if (w.positions + span + (w.split ? kSC : kKC) >= (1ll << 31) || U_w != E_w + fw - 1 || U_h != E_h + fh - 1)
        return hipErrorInvalidConfiguration;
    float* bpart = partial + w.partial_floats;
    const bool vec = Cout % 4 == 0 && Cin % 4 == 0;
    hipError_t e = vec ? dispatch_wgrad<true>(dy, x, E_h, E_w, U_h, U_w, Cout, Cin, fh, fw, w, partial, bpart, s)
                       : dispatch_wgrad<false>(dy, x, E_h, E_w, U_h, U_w, Cout, Cin, fh, fw, w, partial, bpart, s);
    if (e != hipSuccess) return e;
    const int64_t n = (int64_t)Cout * Cin * fh * fw + Cout;
    wgrad_reduce_kernel<<<dim3((unsigned)ceil_div64(n, kBT)), kBT, 0, s>>>(partial, bpart, w.splits, fh * fw, Cout,
                                                                           Cin, dw, db);
    return hipGetLastError();
}

// ------------------------------------------------------------------ 1x1 layer to few outputs
// A 1x1 convolution to CO <= 4 channels after a convolution without a pool, backward
// in one pass over its input a: the weight and bias gradients, and the gradient of
// the previous convolution before its activation (what dgrad and act_backward give,
// in their order, so the same bits).  Separately these steps read a twice and
// write and read the CO -> C gradient in between: 0.37 ms on 200,704 positions of
// 256 channels, 5.83 ms on 1,877,089 of 512.  A lane owns four channels, 1 << lg_lanes lanes
// a position (at most 32: then short signals still make a block per CU); the weight
// gradient stays in registers over the block's positions.
// Bound by HBM: a read once, dx written once, now 0.093 and 1.55 ms (5.0 TB/s).
constexpr int kHT = 1024, kHLanes = 32, kHBlocks = 1024;

template <int CO>
__global__ __launch_bounds__(kHT) void narrow_backward_kernel(const float* __restrict__ g, const float* __restrict__ a,
                                                             const float* __restrict__ w, int w_pitch, int64_t npos,
                                                             int C, int lg_lanes, int act, float* __restrict__ dx,
                                                             float* __restrict__ partial, float* __restrict__ bpart) {
    __shared__ float4 red[kHT];
    const int tid = threadIdx.x, lanes = 1 << lg_lanes, subs = kHT >> lg_lanes;
    const int quad = (tid & (lanes - 1)) + blockIdx.y * kHLanes;
    const bool on = quad < C / 4;
    const int64_t p0 = npos * blockIdx.x / gridDim.x, p1 = npos * (blockIdx.x + 1) / gridDim.x;
    float wq[CO][4], acc[CO][4], bs[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int o = 0; o < CO; ++o)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            wq[o][e] = on ? w[(int64_t)(4 * quad + e) * w_pitch + o] : 0.f;
            acc[o][e] = 0.f;
        }
    constexpr int U = 4;                         // positions in flight
    for (int64_t p = p0 + (tid >> lg_lanes); p < p1; p += (int64_t)U * subs) {
        float av[U][4], gv[U][CO];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t q = p + (int64_t)u * subs;
            const bool in = q < p1;
#pragma unroll
            for (int e = 0; e < 4; ++e) av[u][e] = 0.f;
            if (in && on) VecIO<float, 4>::load(a + q * C + 4 * quad, av[u]);
#pragma unroll
            for (int o = 0; o < CO; ++o) gv[u][o] = in ? g[q * CO + o] : 0.f;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t q = p + (int64_t)u * subs;
            float r[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int o = 0; o < CO; ++o) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    r[e] = fmaf(gv[u][o], wq[o][e], r[e]);
                    acc[o][e] = fmaf(gv[u][o], av[u][e], acc[o][e]);
                }
                bs[o] += gv[u][o];
            }
            if (act != DSS_ACT_NONE) {
#pragma unroll
                for (int e = 0; e < 4; ++e) r[e] *= act_grad(act, av[u][e]);
            }
            if (q < p1 && on) VecIO<float, 4>::store(dx + q * C + 4 * quad, r);
        }
    }
    // over the threads of the same channels: a tree in LDS
    auto sum = [&](const float (&v)[4]) {
        __syncthreads();
        red[tid] = make_float4(v[0], v[1], v[2], v[3]);
        for (int d = kHT / 2; d >= lanes; d >>= 1) {
            __syncthreads();
            if (tid < d) {
                const float4 x = red[tid], y = red[tid + d];
                red[tid] = make_float4(x.x + y.x, x.y + y.y, x.z + y.z, x.w + y.w);
            }
        }
        return red[tid];                         // complete in threads 0 .. lanes - 1, by themselves
    };
#pragma unroll
    for (int o = 0; o < CO; ++o) {
        const float4 v = sum(acc[o]);
        if (tid < lanes && on)
            *reinterpret_cast<float4*>(partial + ((int64_t)blockIdx.x * CO + o) * C + 4 * quad) = v;
    }
    const float4 v = sum(bs);
    if (tid == 0 && blockIdx.y == 0) {
        const float b[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int o = 0; o < CO; ++o) bpart[(int64_t)blockIdx.x * CO + o] = b[o];
    }
}

// dw[i] = sum over blocks of partial[block][i], n values a block, then db likewise
// from bpart: 16 values a workgroup, 16 threads a value.
__global__ __launch_bounds__(256) void narrow_reduce_kernel(const float* __restrict__ partial,
                                                           const float* __restrict__ bpart, int nb, int n, int nbias,
                                                           float* __restrict__ dw, float* __restrict__ db) {
    __shared__ float red[16][17];
    const int i = blockIdx.x * 16 + (threadIdx.x & 15), slice = threadIdx.x >> 4;
    const bool bias = i >= n;
    float s = 0.f;
    if (i < n + nbias)
        for (int b = slice; b < nb; b += 16)
            s += bias ? bpart[(int64_t)b * nbias + i - n] : partial[(int64_t)b * n + i];
    red[threadIdx.x & 15][slice] = s;
    __syncthreads();
    if (slice != 0 || i >= n + nbias) return;
    s = 0.f;
    for (int k = 0; k < 16; ++k) s += red[threadIdx.x][k];
    (bias ? db[i - n] : dw[i]) = s;
}

hipError_t launch_narrow_backward(const float* g, const float* a, const PlanConv& pc, int64_t npos, int act,
                                  const WgradPlan& wp, float* partial, float* dx, float* dw, float* db,
                                  hipStream_t s) {
    const int C = pc.cin, CO = pc.cout;
    if (C % 4 != 0 || CO < 1 || CO > 4) return hipErrorInvalidValue;
    int lg = 0;
    while ((1 << lg) < kHLanes && (1 << lg) < C / 4) ++lg;
    const int groups = (C / 4 + kHLanes - 1) / kHLanes;
    // at least 4 positions a thread, kHBlocks blocks in all, and no more partial sums
    // than the layer's weight-gradient plan has room for (one per split)
    const int64_t by_size = ceil_div64(npos, 4 * (kHT >> lg));
    const int nb = (int)std::max<int64_t>(
        1, std::min({by_size, (int64_t)wp.splits, (int64_t)std::max(1, kHBlocks / groups)}));
    float* bpart = partial + (int64_t)nb * CO * C;
    const dim3 grid((unsigned)nb, (unsigned)groups);
    auto run = [&](auto co) {
        narrow_backward_kernel<decltype(co)::value><<<grid, kHT, 0, s>>>(g, a, (const float*)pc.w, pc.cout_pad, npos, C,
                                                                        lg, act, dx, partial, bpart);
    };
    if (CO == 1) run(std::integral_constant<int, 1>{});
    else if (CO == 2) run(std::integral_constant<int, 2>{});
    else if (CO == 3) run(std::integral_constant<int, 3>{});
    else run(std::integral_constant<int, 4>{});
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    narrow_reduce_kernel<<<dim3((unsigned)((C * CO + CO + 15) / 16)), 256, 0, s>>>(partial, bpart, nb, C * CO, CO, dw,
                                                                                  db);
    return hipGetLastError();
}

// ------------------------------------------------------------------ crop_to_planar
__global__ __launch_bounds__(kBT) void crop_to_planar_kernel(const float* __restrict__ in, int D_w, int C, int H, int W,
                                                            float* __restrict__ out) {
    const int64_t p = (int64_t)blockIdx.x * kBT + threadIdx.x;
    if (p >= (int64_t)H * W) return;
    const int y = (int)(p / W), x = (int)(p % W);
    const float* src = in + ((int64_t)y * D_w + x) * C;
    for (int c = 0; c < C; ++c) out[(int64_t)c * H * W + p] = src[c];
}

hipError_t launch_crop_to_planar(const float* in, int D_w, int C, int H, int W, float* out, hipStream_t s) {
    crop_to_planar_kernel<<<dim3((unsigned)ceil_div64((int64_t)H * W, kBT)), kBT, 0, s>>>(in, D_w, C, H, W, out);
    return hipGetLastError();
}

}  // namespace dss
