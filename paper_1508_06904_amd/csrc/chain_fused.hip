// The dense evaluation of a small network in one launch (binary32).
//
// A network whose layers have at most 16 channels (every convolution on the
// direct kernel) does so little per window that the separate launches of Stuff,
// each convolution, each pool + Frag and Defrag are bound by their latencies: 7
// launches of 6 to 14 us for 5 MFLOP on the 64 x 64 image.  Here a workgroup takes
// a tile of the dense output and carries it through the whole network in LDS, in
// the dilated fashion (appendix, Definition "evaldilate": layer j's convolution and
// maximum take taps k*_{j-1} apart, and layer L is the dense output): the signal
// region of a TH x TW tile is (TH + B_h - 1) x (TW + B_w - 1) samples, and each step
// shrinks it.  Neighbouring tiles compute their common border again, which the
// tile size is chosen against (fused_plan).
//
// Every output is summed in the direct convolution kernel's order (the bias, then
// filter rows, columns and input channels, one fma each), so its bits are those of
// the separate launches.
//
// Bound by LDS latency and the vector ALU of the busiest CU: several positions of a
// thread share each weight read, and the filter loop keeps several reads in
// flight.  64 x 64 image 50.8 -> 19.6 us an evaluation (fused_plan has other sizes
// and networks).
#include <algorithm>
#include <type_traits>

#include "dev_common.h"
#include "dss_internal.h"

namespace dss {

constexpr int kFT = 512;

// Positions x channels a thread accumulates at once: COB channels of PP positions
// 512 apart, from `in` (region in_w wide, cin channels a sample) to `out`.  VEC:
// input channels in fours.
template <int COB, int PP, bool VEC>
__device__ __forceinline__ void fused_conv_form(const FusedLayer& L, const float* __restrict__ wl,
                                                const float* __restrict__ in, float* __restrict__ out) {
    const int npos = L.e_h * L.e_w, e_w = L.e_w, in_w = L.in_w, cin = L.cin, cout_pad = L.cout_pad, cout = L.cout;
    const int fw = L.fw, act = L.act;
    const int row_step = L.dil_h * in_w * cin, col_step = L.dil_w * cin;
    constexpr int CI = VEC ? 4 : 1;
    constexpr int UNROLL = VEC && COB >= 8 ? (PP * COB >= 32 ? 1 : 2) : 4;   // within 128 registers: two workgroups per CU
    const int nsteps = L.fh * fw * cin / CI;
    for (int base = threadIdx.x; base < npos; base += kFT * PP) {
        const float* src[PP];
#pragma unroll
        for (int k = 0; k < PP; ++k) {
            const int p = min(base + kFT * k, npos - 1), y = p / e_w;
            src[k] = in + (y * in_w + p - y * e_w) * cin;
        }
        for (int og = 0; og < cout_pad; og += COB) {
            float acc[PP][COB];
#pragma unroll
            for (int o = 0; o < COB; ++o) {
                const float bo = L.b[og + o];
#pragma unroll
                for (int k = 0; k < PP; ++k) acc[k][o] = bo;
            }
            // filter rows, columns and input channels as one loop, so that several
            // of its LDS reads are in flight
            const float* wr = wl + og;
            int off = 0, i = 0, tw = 0, row = 0;
#pragma unroll UNROLL
            for (int t = 0; t < nsteps; ++t, wr += CI * cout_pad) {
                float v[PP][CI];
#pragma unroll
                for (int k = 0; k < PP; ++k) {
                    if constexpr (VEC) {
                        const float4 q = *reinterpret_cast<const float4*>(src[k] + off + i);
                        v[k][0] = q.x;
                        v[k][1] = q.y;
                        v[k][2] = q.z;
                        v[k][3] = q.w;
                    } else {
                        v[k][0] = src[k][off + i];
                    }
                }
                i += CI;
                if (i == cin) {
                    i = 0;
                    off += col_step;
                    if (++tw == fw) {
                        tw = 0;
                        off = row += row_step;
                    }
                }
#pragma unroll
                for (int e = 0; e < CI; ++e) {
                    float wv[COB];
                    if constexpr (COB >= 4) {
#pragma unroll
                        for (int o = 0; o < COB; o += 4) {
                            const float4 q = *reinterpret_cast<const float4*>(wr + e * cout_pad + o);
                            wv[o] = q.x;
                            wv[o + 1] = q.y;
                            wv[o + 2] = q.z;
                            wv[o + 3] = q.w;
                        }
                    } else {
#pragma unroll
                        for (int o = 0; o < COB; ++o) wv[o] = wr[e * cout_pad + o];
                    }
#pragma unroll
                    for (int k = 0; k < PP; ++k)
#pragma unroll
                        for (int o = 0; o < COB; ++o) acc[k][o] = fmaf(v[k][e], wv[o], acc[k][o]);
                }
            }
#pragma unroll
            for (int k = 0; k < PP; ++k)
                if (base + kFT * k < npos)
#pragma unroll
                    for (int o = 0; o < COB; ++o)
                        if (og + o < cout) out[(base + kFT * k) * cout + og + o] = activate(act, acc[k][o]);
        }
    }
}

template <int COB>
__device__ __forceinline__ void fused_conv(const FusedLayer& L, const float* __restrict__ wl,
                                           const float* __restrict__ in, float* __restrict__ out) {
    const int npos = L.e_h * L.e_w;
    if (L.cin % 4 == 0) {
        if (npos <= kFT) fused_conv_form<COB, 1, true>(L, wl, in, out);
        else fused_conv_form<COB, 2, true>(L, wl, in, out);
    } else {
        if (npos <= kFT) fused_conv_form<COB, 1, false>(L, wl, in, out);
        else if (npos <= 2 * kFT || COB >= 16) fused_conv_form<COB, 2, false>(L, wl, in, out);
        else fused_conv_form<COB, 4, false>(L, wl, in, out);
    }
}

__global__ __launch_bounds__(kFT, 4) void fused_chain_kernel(const float* __restrict__ signal, int H, int W, FusedChain fc,
                                                         float* __restrict__ outp, int out_h, int out_w) {
    extern __shared__ __attribute__((aligned(16))) float fl[];
    float* cur = fl;
    float* nxt = fl + fc.buf_floats[0];
    float* const wl = fl + fc.buf_floats[0] + fc.buf_floats[1];
    const int ty = blockIdx.x / fc.tiles_x, tx = blockIdx.x - ty * fc.tiles_x;
    const int y0 = ty * fc.TH, x0 = tx * fc.TW;
    const int tid = threadIdx.x;
    // n floats from global memory to LDS, four loads of a thread in flight at once
    auto stage = [&](int n, auto&& load, auto&& store) {
        for (int i = tid; i < n; i += 4 * kFT) {
            float v[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) v[k] = i + k * kFT < n ? load(i + k * kFT) : 0.f;
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (i + k * kFT < n) store(i + k * kFT, v[k]);
        }
    };
    // the tile's signal region, channels last; past the signal: 0 (it feeds no kept output)
    const int rh = fc.L[0].in_h, rw = fc.L[0].in_w;
    for (int c = 0; c < fc.in_c; ++c)
        stage(
            rh * rw,
            [&](int p) {
                const int y = y0 + p / rw, x = x0 + p % rw;
                return y < H && x < W ? signal[((int64_t)c * H + y) * W + x] : 0.f;
            },
            [&](int p, float v) { cur[p * fc.in_c + c] = v; });
    for (int j = 0; j < fc.n; ++j) {     // every layer's weights
        const FusedLayer& L = fc.L[j];
        if (L.has_conv)
            stage(
                L.fh * L.fw * L.cin * L.cout_pad, [&](int i) { return L.w[i]; },
                [&](int i, float v) { wl[L.w_at + i] = v; });
    }
    __syncthreads();
    for (int j = 0; j < fc.n; ++j) {
        const FusedLayer& L = fc.L[j];
        if (L.has_conv) {
            const float* wj = wl + L.w_at;
            switch (L.cob) {
                case 16: fused_conv<16>(L, wj, cur, nxt); break;
                case 8: fused_conv<8>(L, wj, cur, nxt); break;
                case 4: fused_conv<4>(L, wj, cur, nxt); break;
                case 2: fused_conv<2>(L, wj, cur, nxt); break;
                default: fused_conv<1>(L, wj, cur, nxt); break;
            }
            float* t = cur;
            cur = nxt;
            nxt = t;
            __syncthreads();
        }
        if (L.k_h * L.k_w > 1) {
            // channels in fours where they are
            auto pool = [&](auto vec_c) {
                constexpr int V = decltype(vec_c)::value;
                const int C = L.cout, CV = C / V, row = L.u_w * CV, n = L.u_h * row;
#pragma unroll 2
                for (int i = tid; i < n; i += kFT) {
                    const int y = i / row, xc = i - y * row;
                    const float* src = cur + y * L.e_w * C + xc * V;
                    float m[V];
                    VecIO<float, V>::load(src, m);
#pragma unroll 2
                    for (int a = 0; a < L.k_h; ++a)
#pragma unroll 2
                        for (int b = 0; b < L.k_w; ++b) {
                            float v[V];
                            VecIO<float, V>::load(src + (a * L.dil_h * L.e_w + b * L.dil_w) * C, v);
#pragma unroll
                            for (int e = 0; e < V; ++e) m[e] = fmaxf(m[e], v[e]);
                        }
                    VecIO<float, V>::store(nxt + i * V, m);
                }
            };
            if (L.cout % 4 == 0) pool(std::integral_constant<int, 4>{});
            else pool(std::integral_constant<int, 1>{});
            float* t = cur;
            cur = nxt;
            nxt = t;
            __syncthreads();
        }
    }
    const int C = fc.L[fc.n - 1].cout, n = fc.TH * fc.TW;
    for (int c = 0; c < C; ++c)
        for (int p = tid; p < n; p += kFT) {
            const int y = p / fc.TW, x = p - y * fc.TW;
            if (y0 + y < out_h && x0 + x < out_w)
                outp[((int64_t)c * out_h + y0 + y) * out_w + x0 + x] = cur[p * C + c];
        }
}

// Regions of a TH x TW output tile, back to front.  Returns the tile's multiply-adds
// (0 if it does not fit).
static int64_t fused_regions(const Chain& ch, int TH, int TW, FusedChain* fc) {
    const int L = ch.L();
    int h = TH, w = TW;
    int64_t macs = 0, wtotal = 0;
    for (int j = L; j >= 1; --j) {
        const ChainLayer& c = ch.layers[j - 1];
        FusedLayer& f = fc->L[j - 1];
        f.dil_h = ch.kstar_h[j - 1];
        f.dil_w = ch.kstar_w[j - 1];
        f.k_h = c.k_h;
        f.k_w = c.k_w;
        f.u_h = h;
        f.u_w = w;
        f.e_h = h + f.dil_h * (c.k_h - 1);
        f.e_w = w + f.dil_w * (c.k_w - 1);
        f.in_h = h = f.e_h + f.dil_h * (c.c_h - 1);
        f.in_w = w = f.e_w + f.dil_w * (c.c_w - 1);
        f.cin = c.has_conv ? c.cin : c.cout;
        f.cout = c.cout;
        f.fh = c.c_h;
        f.fw = c.c_w;
        f.act = c.act;
        f.has_conv = c.has_conv;
        if ((int64_t)h * w > (1 << 16)) return 0;
        if (c.has_conv) {
            macs += (int64_t)f.e_h * f.e_w * c.cout * c.cin * c.c_h * c.c_w;
            f.w_at = (int)wtotal;
            wtotal += ((int64_t)c.c_h * c.c_w * c.cin * f.cout_pad + 3) / 4 * 4;
        }
    }
    // the steps alternate between two LDS buffers, the signal in the first
    int64_t need[2] = {(int64_t)fc->L[0].in_h * fc->L[0].in_w * fc->in_c, 0};
    int which = 0;
    auto step = [&](int64_t floats) {
        which ^= 1;
        need[which] = std::max(need[which], floats);
    };
    for (int j = 0; j < L; ++j) {
        const FusedLayer& f = fc->L[j];
        if (f.has_conv) step((int64_t)f.e_h * f.e_w * f.cout);
        if (f.k_h * f.k_w > 1) step((int64_t)f.u_h * f.u_w * f.cout);
    }
    for (int i = 0; i < 2; ++i) fc->buf_floats[i] = (int)((need[i] + 3) / 4 * 4);
    const int64_t lds = (need[0] + need[1] + 8 + wtotal) * 4;
    if (lds > 64 * 1024) return 0;
    fc->TH = TH;
    fc->TW = TW;
    fc->lds_bytes = (size_t)lds;
    return std::max<int64_t>(macs, 1);
}

// One workgroup's tile: its threads' chains of LDS reads and multiply-adds, layer by layer.
static double thread_cost(const FusedChain& fc) {
    double cost = 0.0;
    for (int j = 0; j < fc.n; ++j) {
        const FusedLayer& f = fc.L[j];
        if (!f.has_conv) continue;
        const bool vec = f.cin % 4 == 0;
        const int npos = f.e_h * f.e_w, ci = vec ? 4 : 1;
        const int pp = npos <= kFT ? 1 : vec || npos <= 2 * kFT || f.cob >= 16 ? 2 : 4;      // as in fused_conv
        const double iters = (double)((npos + kFT * pp - 1) / (kFT * pp)) * (f.cout_pad / f.cob);
        cost += 2.2 + iters * (0.085 + (double)(f.fh * f.fw * f.cin / ci) * (0.04 + 0.0078 * ci * pp * f.cob));
    }
    return cost;
}

// The separate launches: their number, the longest chain of each convolution's threads,
// and its operations and input reads.
static double separate_cost(const Chain& ch, const std::vector<PlanConv>& convs, int out_h, int out_w, double conv_flops,
                            int launches) {
    double cost = 5.8 * launches + 3e-8 * conv_flops;
    int64_t h = out_h, w = out_w;
    for (int j = ch.L(); j >= 1; --j) {
        const ChainLayer& c = ch.layers[j - 1];
        h += (int64_t)ch.kstar_h[j - 1] * (c.k_h - 1);
        w += (int64_t)ch.kstar_w[j - 1] * (c.k_w - 1);
        if (c.has_conv) {
            const double K = (double)c.cin * c.c_h * c.c_w;
            cost += 0.13 * K + 3.2e-7 * h * w * K * (convs[j - 1].cout_pad / convs[j - 1].cob);
        }
        h += (int64_t)ch.kstar_h[j - 1] * (c.c_h - 1);
        w += (int64_t)ch.kstar_w[j - 1] * (c.c_w - 1);
    }
    return cost;
}

bool fused_plan(const Chain& ch, const std::vector<PlanConv>& convs, int out_h, int out_w, double conv_flops,
                FusedChain* fc) {
    const int L = ch.L();
    // one-dimensional networks have their pools in their convolutions' launches already
    if (L < 1 || L > kMaxFused || ch.ndim == 1) return false;
    fc->n = L;
    fc->in_c = ch.in_c;
    int launches = 2;            // Stuff and Defrag
    for (int j = 0; j < L; ++j) {
        const ChainLayer& c = ch.layers[j];
        FusedLayer& f = fc->L[j];
        f = FusedLayer{};
        if (c.cout > 16) return false;
        launches += (c.has_conv ? 1 : 0) + (c.has_pool ? 1 : 0);
        if (!c.has_conv) continue;
        const PlanConv& pc = convs[j];
        if (pc.impl != CONV_DIRECT || c.cin >= 16) return false;   // the plain direct kernel's summation order
        f.w = (const float*)pc.w;
        f.b = pc.b;
        f.cob = pc.cob;
        f.cout_pad = pc.cout_pad;
    }
    // The tile that finishes first, and whether the separate launches finish before it.
    // Both sides' costs are fitted together to the choices that eleven networks (1 to 4
    // layers, filters of 2x2 to 11x11, 1 to 16 channels, pools of 2 to 4) on 48 x 48 to
    // 600 x 800 samples call for, every tile side and the separate launches measured: they
    // are in one unit, not in microseconds.  Up to 512 tiles run at once, two a CU, and
    // further ones in whole rounds.  Of those 77 calls 73 take the fastest way or one within
    // 10 %; the others lose 7 to 17 % to another tile side, none more than 5 % to the separate
    // launches.  For instance, separate / tiles of 4 / 8 / 16 in us:
    //   conv5x5 1-4, pool, conv5x5 4-8, pool, conv4x4 8-1   48 x 48    50.5 / 20.5 / 21.1 / 25.9
    //                                                       400 x 400  68.9 / 329 / 101 / 52.0
    //                                                       600 x 800  94.7 / 1013 / 295 / 105
    //   conv3x3 1-12, 12-12, 12-12, pool, conv3x3 12-2      150 x 150  47.7 / 93.4 / 34.9
    //                                                       200 x 320  58.2 / 242 / 68.2
    //   conv11x11 3-14, conv5x5 14-1                        200 x 320  91.9 / 496 / 138 / 70.0
    double best = 0.0;
    FusedChain pick = *fc;
    for (int side = 4; side <= 64; side *= 2) {
        const int TH = side, TW = side;
        FusedChain t = *fc;
        const int64_t macs = fused_regions(ch, TH, TW, &t);
        if (macs == 0) break;
        const int64_t tiles = ceil_div64(out_h, TH) * ceil_div64(out_w, TW);
        const double cost = (double)ceil_div64(tiles, 512) *
                            (8.0 + std::max(thread_cost(t), (tiles > 256 ? 2.0 : 1.0) * macs / 48000.0));
        if (tiles < (1ll << 31) && (best == 0.0 || cost < best)) {
            best = cost;
            pick = t;
        }
    }
    if (best == 0.0) return false;
    *fc = pick;
    fc->tiles_x = (int)ceil_div64(out_w, fc->TW);
    return best < separate_cost(ch, convs, out_h, out_w, conv_flops, launches);
}

hipError_t launch_fused_chain(const FusedChain& fc, const float* signal, int H, int W, float* out, int out_h, int out_w,
                              hipStream_t s) {
    const int64_t tiles = ceil_div64(out_h, fc.TH) * fc.tiles_x;
    fused_chain_kernel<<<dim3((unsigned)tiles), kFT, fc.lds_bytes, s>>>(signal, H, W, fc, out, out_h, out_w);
    return hipGetLastError();
}

}  // namespace dss
