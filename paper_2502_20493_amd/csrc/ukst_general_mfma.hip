// Stride-s transpose convolution and dilation-d convolution of wide layers on the bf16 matrix pipe
// (ukst_parts.h: fp32 operands as three exact parts, bf16 operands as one).
//
// Both are, per parity class, a plain stride-1 correlation (ukst_general.hip):
//     y[b][co][oy0 + os*i][ox0 + os*j] = sum_ci sum_{u<Tr, v<Tc} x[b][ci][i + rb + u*xs][j + cb + v*xs]
//                                                                * w[co][ci][r + u*ws][c + v*ws]
// with os = ws = s, xs = 1 and s*s classes (r, c) for the transpose convolution, os = ws = 1, xs = d and one
// class for the dilated one: an implicit GEMM with M = output channels, N = the class's pixels flattened
// over (image, row, column), K = input channels, 16 per MFMA, one pair of fragments per tap.
//
// A block is 4 waves on 32*MT channels x 256 pixels of one class (a wave: MT x 2 accumulator tiles), small
// enough in registers and usually in LDS (two taps of weights in two buffers, the pixel rows of 16 channels)
// that two blocks share a compute unit and one's staging runs beside the other's MFMAs.  A wave reads
// (MT + 2) fragments per part and tap for 2*MT products of parts: 12 KiB per 24 MFMAs at MT = 2, three
// parts, well inside the LDS rate.  The weights of the group of two taps after next are on their way while
// a group is multiplied, the next group's are split and written between its two taps.  Blocks of the s*s
// classes of one pixel tile are neighbours: they read the same rows and complete each other's lines of y.
// Measured, vector-ALU kernel of ukst_general.hip -> this one: stride 3, 16 x 128 -> 64 channels, 32 x 32, n = 5: fp32
// 547 -> 81 us (79 TFLOP/s), bf16 528 -> 59; dilation 2, 16 x 64 -> 64, 64 x 64, n = 3: 236 -> 44 (105), 200 -> 26.
#include "ukst_parts.h"

namespace ukst {
namespace {

constexpr int KC = 16, TN = 256, T = 256;
constexpr int LDS_LIMIT = 160 * 1024 - 256;  // (256 bytes belong to __syncthreads_or)

struct ConvArgs {
    int B, Cin, Cout, H, W, n, P, k, OH, OW;
    int dilated;
    int classes;  // k*k or 1
    int group;    // pixel tiles whose blocks lie together, the classes of most taps first
    unsigned long long order;  // the classes by taps, four bits each
    int nco, nqt; // channel blocks, pixel tiles of the largest class
    int XPL;      // bytes of one part's activation stage
};

// the class geometry, from the class number (uniform over a block)
struct Class {
    int r, c, Tr, Tc;     // first tap, taps per axis
    int xs, ws, os;       // steps: input rows per tap, taps, output rows per lattice row
    int oy0, ox0, NI, NJ; // lattice of output pixels
    int rb, cb;           // input row / column of lattice row / column 0 at tap 0
    int EH, LW;           // staged rows per image, columns
    int col0, cols;       // staged columns that hold input columns: col0 .. col0 + cols - 1
};
__host__ __device__ inline Class class_of(const ConvArgs& a, int cls)
{
    Class q;
    if (a.dilated) {
        q.r = q.c = 0;
        q.Tr = q.Tc = a.n;
        q.xs = a.k;
        q.ws = q.os = 1;
        q.oy0 = q.ox0 = 0;
        q.rb = q.cb = -a.P;
    } else {
        const int k = a.k;
        q.oy0 = cls / k;
        q.ox0 = cls % k;
        q.r = ((a.P - q.oy0) % k + k) % k;
        q.c = ((a.P - q.ox0) % k + k) % k;
        q.Tr = q.r < a.n ? (a.n - q.r + k - 1) / k : 0;
        q.Tc = q.c < a.n ? (a.n - q.c + k - 1) / k : 0;
        if (q.Tr == 0 || q.Tc == 0) q.Tr = q.Tc = 0;
        q.xs = 1;
        q.ws = q.os = k;
        q.rb = (q.oy0 + q.r - a.P) / k;  // exact
        q.cb = (q.ox0 + q.c - a.P) / k;
    }
    q.NI = a.OH > q.oy0 ? (a.OH - q.oy0 + q.os - 1) / q.os : 0;
    q.NJ = a.OW > q.ox0 ? (a.OW - q.ox0 + q.os - 1) / q.os : 0;
    const int sr = q.Tr ? (q.Tr - 1) * q.xs : 0, sc = q.Tc ? (q.Tc - 1) * q.xs : 0;
    q.EH = q.NI + sr;
    q.LW = q.NJ + sc;
    q.col0 = q.cb < 0 ? -q.cb : 0;
    const int end = q.LW < a.W - q.cb ? q.LW : a.W - q.cb;
    q.cols = end > q.col0 ? end - q.col0 : 0;
    return q;
}

// n / d for 0 <= n < 2^24, d >= 1
__device__ __forceinline__ int small_div(int n, int d, float rcp)
{
    int q = (int)((float)n * rcp);
    const int rem = n - q * d;
    q += rem >= d ? 1 : 0;
    q -= rem < 0 ? 1 : 0;
    return q;
}

// MT: groups of 32 output channels; XU: activation units per thread
template <int MT, int XU, typename TIn>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2)))
void ukst_general_mfma_kernel(const TIn* __restrict__ x, const TIn* __restrict__ w, float* __restrict__ y, ConvArgs a)
{
    constexpr int PARTS = sizeof(TIn) == 4 ? 3 : 1;
    constexpr int ES = (int)sizeof(TIn);
    constexpr int TM = 32 * MT;
    constexpr int WTS = (TM + 4) * 16;            // a tap's 16-byte slots [channel]; two taps, then the other
    constexpr int WHS = 2 * WTS;                  // channel half: the staging lanes (tap, half, 4 channels) of a
    constexpr int WPL = 2 * WHS;                  // 16-lane pass hit 16 different slots modulo 16
    constexpr int WBUF = PARTS * WPL;
    constexpr int XS_OFF = 2 * WBUF;
    constexpr int PX = PARTS == 3 ? 1 : 4;        // pixels of an activation unit
    typedef PartProducts<PARTS> PP;
    extern __shared__ __align__(16) unsigned char lds[];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, gk = lane >> 5;
    int bid = xcd_contiguous(blockIdx.x, gridDim.x);
    const int gs = a.group * a.classes * a.nco, grp = bid / gs;
    bid -= grp * gs;
    const int gt = a.nqt - grp * a.group < a.group ? a.nqt - grp * a.group : a.group;  // tiles of this group
    const int cb = bid / (gt * a.classes);
    bid -= cb * gt * a.classes;
    const int rank = bid / gt, qt = grp * a.group + bid - rank * gt;
    const int cls = a.group > 1 ? (int)(a.order >> (4 * rank)) & 15 : rank;
    const Class g = class_of(a, cls);
    const int IJ = g.NI * g.NJ, Q = a.B * IJ;
    const int co0 = cb * TM, q0 = qt * TN;
    if (q0 >= Q) return;  // (classes differ by a lattice row or column)
    const int q_last = q0 + TN - 1 < Q ? q0 + TN - 1 : Q - 1;
    const float rIJ = 1.f / (float)IJ, rNJ = 1.f / (float)g.NJ, rEH = 1.f / (float)g.EH;
    const int taps = g.Tr * g.Tc, NN = a.n * a.n;

    // lattice row rho = b*NI + i reads staged rows e = b*EH + i + u*xs, less the tile's first
    const int bf0 = small_div(q0, IJ, rIJ), if0 = small_div(q0 - bf0 * IJ, g.NJ, rNJ);
    const int e_first = bf0 * g.EH + if0;
    const int bl = small_div(q_last, IJ, rIJ), il = small_div(q_last - bl * IJ, g.NJ, rNJ);
    const int rows = bl * g.EH + il + g.EH - g.NI - e_first + 1;
    const int XPL = a.XPL, XH = rows * g.LW * 16;  // (the other channel half follows the first)

    if (taps) {
        for (int i = tid; i < PARTS * XPL / 16; i += T)
            *reinterpret_cast<u4v_t*>(lds + XS_OFF + i * 16) = u4v_t{0u, 0u, 0u, 0u};
    }

    const __amdgpu_buffer_rsrc_t rs_x = __builtin_amdgcn_make_buffer_rsrc(
        (void*)x, 0, (int)((size_t)a.B * a.Cin * a.H * a.W * ES), kRawBuffer);
    const __amdgpu_buffer_rsrc_t rs_w =
        __builtin_amdgcn_make_buffer_rsrc((void*)w, 0, (int)((size_t)a.Cout * a.Cin * NN * ES), kRawBuffer);
    const unsigned x_cstride = (unsigned)(a.H * a.W * ES);

    // activation units: (channel half, row, PX columns), columns fastest
    unsigned x_goff[XU];
    int x_loff[XU], x_ci[XU];
    {
        const int cpr = (g.cols + PX - 1) / PX, per_half = rows * cpr;
        const float rC = 1.f / (float)(cpr > 0 ? cpr : 1), rR = 1.f / (float)(per_half > 0 ? per_half : 1);
#pragma unroll
        for (int j = 0; j < XU; ++j) {
            const int e = tid + T * j;
            x_goff[j] = kNoByte;
            x_loff[j] = -1;
            x_ci[j] = 0;
            if (e < 2 * per_half) {
                const int h = small_div(e, per_half, rR), rem = e - h * per_half;
                const int row = small_div(rem, cpr, rC), pc = rem - row * cpr;
                const int col = g.col0 + (PX * pc + PX <= g.cols ? PX * pc : g.cols - PX);
                const int er = e_first + row, b = small_div(er, g.EH, rEH), i = er - b * g.EH + g.rb;
                if (i >= 0 && i < a.H)
                    x_goff[j] = (unsigned)((((b * a.Cin + 8 * h) * a.H + i) * a.W + col + g.cb) * ES);
                x_loff[j] = XS_OFF + h * XH + (row * g.LW + col) * 16;
                x_ci[j] = 8 * h;
            }
        }
    }
    // weight unit of the thread: (output channel, channel half, tap of the group)
    const int w_t = tid & 1, w_h = (tid >> 1) & 1, w_co = tid >> 2;
    const bool w_on = w_co < TM;  // uniform per wave
    const unsigned w_goff = w_on && co0 + w_co < a.Cout ? (unsigned)(((co0 + w_co) * a.Cin + 8 * w_h) * NN * ES) : kNoByte;
    const int w_loff = w_h * WHS + w_t * WTS + w_co * 16;

    unsigned xr[XU][8][PARTS == 3 ? 1 : 2], wr[8];
    auto load_x = [&](int s) {
#pragma unroll
        for (int j = 0; j < XU; ++j)
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const unsigned soff = (unsigned)(s * KC + k) * x_cstride;
                if constexpr (PARTS == 3) {
                    xr[j][k][0] = __builtin_amdgcn_raw_buffer_load_b32(rs_x, x_goff[j], soff, 0);
                } else {
                    const u2v_t v = __builtin_amdgcn_raw_buffer_load_b64(rs_x, x_goff[j], soff, 0);
                    xr[j][k][0] = v.x;
                    xr[j][k][1] = v.y;
                }
            }
    };
    auto store_x = [&](int s) {
#pragma unroll
        for (int j = 0; j < XU; ++j) {
            if (s * KC + KC > a.Cin) {  // channels past the last one: zeros
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    const bool in = s * KC + x_ci[j] + k < a.Cin;
                    xr[j][k][0] = in ? xr[j][k][0] : 0u;
                    if constexpr (PARTS == 1) xr[j][k][1] = in ? xr[j][k][1] : 0u;
                }
            }
            if (x_loff[j] < 0) continue;
            if constexpr (PARTS == 3) {
                unsigned v[8];
#pragma unroll
                for (int k = 0; k < 8; ++k) v[k] = xr[j][k][0];
                u4v_t p[3];
                to_parts<3>(v, p);
#pragma unroll
                for (int i = 0; i < 3; ++i) *reinterpret_cast<u4v_t*>(lds + i * XPL + x_loff[j]) = p[i];
            } else {
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    u4v_t v;
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        v[i] = __builtin_amdgcn_perm(xr[j][2 * i + 1][t >> 1], xr[j][2 * i][t >> 1],
                                                     (t & 1) ? 0x07060302u : 0x05040100u);
                    *reinterpret_cast<u4v_t*>(lds + x_loff[j] + t * 16) = v;
                }
            }
        }
    };
    const float rTc = 1.f / (float)(g.Tc > 0 ? g.Tc : 1);
    const int groups = (taps + 1) / 2, stages = (a.Cin + KC - 1) / KC;
    // taps 2*grp and 2*grp + 1 of stage s (a group past the last: the next stage's; past the last stage: anything)
    auto load_w = [&](int s, int grp) {
        while (grp >= groups) { grp -= groups; ++s; }  // (a class of one or two taps: two stages on)
        if (s >= stages) s = stages - 1;
        const int t = 2 * grp + w_t;
        const int u = small_div(t, g.Tc, rTc), v = t - u * g.Tc;
        const unsigned voff = w_on && t < taps ? w_goff + (unsigned)(((g.r + u * g.ws) * a.n + g.c + v * g.ws) * ES) : kNoByte;
#pragma unroll
        for (int k = 0; k < 8; ++k) wr[k] = load_element<TIn>(rs_w, voff, (unsigned)((s * KC + k) * NN * ES));
    };
    auto store_w = [&](int s, int grp, int buf) {
        if (!w_on) return;
        if (grp >= groups) { grp -= groups; ++s; }
        if (s * KC + KC > a.Cin) {
#pragma unroll
            for (int k = 0; k < 8; ++k) wr[k] = s * KC + 8 * w_h + k < a.Cin ? wr[k] : 0u;
        }
        u4v_t p[PARTS];
        to_parts<PARTS>(wr, p);
#pragma unroll
        for (int i = 0; i < PARTS; ++i) *reinterpret_cast<u4v_t*>(lds + buf * WBUF + i * WPL + w_loff) = p[i];
    };

    const int a_lds = gk * WHS + l32 * 16;
    int b_lds[2];
#pragma unroll
    for (int nt = 0; nt < 2; ++nt) {
        int q = q0 + (wave * 2 + nt) * 32 + l32;
        if (q > q_last) q = q_last;
        const int b = small_div(q, IJ, rIJ), rem = q - b * IJ;
        const int i = small_div(rem, g.NJ, rNJ), j = rem - i * g.NJ;
        b_lds[nt] = XS_OFF + gk * XH + ((b * g.EH + i - e_first) * g.LW + j) * 16;
    }
    f32x16_t acc[MT][2];
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int nt = 0; nt < 2; ++nt)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[m][nt][i] = 0.f;

    auto tap = [&](int buf, int t, int xoff) {  // t: 0 or 1; xoff: bytes of the tap's window position
        bf16x8_t af[MT][PARTS], bf[2][PARTS];
#pragma unroll
        for (int i = PARTS - 1; i >= 0; --i) {
#pragma unroll
            for (int m = 0; m < MT; ++m)
                af[m][i] = *reinterpret_cast<const bf16x8_t*>(lds + buf * WBUF + a_lds + i * WPL + t * WTS + m * 512);
#pragma unroll
            for (int nt = 0; nt < 2; ++nt)
                bf[nt][i] = *reinterpret_cast<const bf16x8_t*>(lds + b_lds[nt] + i * XPL + xoff);
        }
#pragma unroll
        for (int p = 0; p < PP::count; ++p)
#pragma unroll
            for (int m = 0; m < MT; ++m)
#pragma unroll
                for (int nt = 0; nt < 2; ++nt)
                    acc[m][nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[m][PP::a[p]], bf[nt][PP::b[p]], acc[m][nt],
                                                                         0, 0, 0);
    };

    if (taps) {
        load_w(0, 0);
        load_x(0);
        __syncthreads();  // zero fill done before the first activation writes
        store_w(0, 0, 0);
        store_x(0);
        load_w(0, 1);
        __syncthreads();
        int buf = 0;
        for (int s = 0; s < stages; ++s) {
            const int s_next = s + 1 < stages ? s + 1 : s;
            int u = 0, v = 0;
            for (int grp = 0; grp < groups; ++grp) {
                const bool last = grp + 1 == groups;
                if (last) load_x(s_next);
                __builtin_amdgcn_sched_barrier(0);
                tap(buf, 0, (u * g.LW + v) * g.xs * 16);
                if (++v == g.Tc) { v = 0; ++u; }
                __builtin_amdgcn_sched_barrier(0);
                store_w(s, grp + 1, buf ^ 1);
                load_w(s, grp + 2);
                __builtin_amdgcn_sched_barrier(0);
                if (2 * grp + 1 < taps) {
                    tap(buf, 1, (u * g.LW + v) * g.xs * 16);
                    if (++v == g.Tc) { v = 0; ++u; }
                }
                __syncthreads();
                if (last) {
                    store_x(s_next);
                    __syncthreads();
                }
                buf ^= 1;
            }
        }
    }

    // accumulator register i of a tile holds channel 8*(i/4) + 4*gk + (i%4), for the lane's pixel
    const __amdgpu_buffer_rsrc_t rs_y = __builtin_amdgcn_make_buffer_rsrc(
        (void*)y, 0, (int)((size_t)a.B * a.Cout * a.OH * a.OW * 4), kRawBuffer);
    const unsigned plane = (unsigned)(a.OH * a.OW * 4);
#pragma unroll
    for (int nt = 0; nt < 2; ++nt) {
        const int q = q0 + (wave * 2 + nt) * 32 + l32;
        const int qq = q <= q_last ? q : q_last;
        const int b = small_div(qq, IJ, rIJ), rem = qq - b * IJ;
        const int i = small_div(rem, g.NJ, rNJ), j = rem - i * g.NJ;
        const unsigned off =
            (unsigned)(((b * a.Cout + co0 + 4 * gk) * a.OH + g.oy0 + i * g.os) * a.OW + g.ox0 + j * g.os) * 4u;
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int ch = 32 * m + 8 * (e / 4) + (e % 4);
                const float val = PARTS == 3 ? acc[m][nt][e] * kPartsDown : acc[m][nt][e];
                const bool on = q <= q_last && co0 + 4 * gk + ch < a.Cout;
                __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(val), rs_y, on ? off : kNoByte, (unsigned)ch * plane, 0);
            }
    }

    float most = 0.f;
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int nt = 0; nt < 2; ++nt) most = peak(acc[m][nt], most);
    if (!__syncthreads_or(most < __builtin_inff() ? 0 : 1)) return;
    // tiles that hold a sum that is not finite (ukst_parts.h)
    unsigned tiles = 0u;
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int nt = 0; nt < 2; ++nt)
            if (!wave_finite(acc[m][nt])) tiles |= 1u << (2 * m + nt);
    if (tid == 0) *reinterpret_cast<unsigned*>(lds) = 0u;
    __syncthreads();
    const unsigned w_cstride = (unsigned)(NN * ES);
    const size_t pixels = (size_t)a.OH * a.OW;
    // group: (four channels, pixel) of the block's outputs
#pragma unroll 1
    for (int m = 0; m < MT; ++m) {
        if ((tiles >> (2 * m) & 3) == 0u) continue;
        const int ch = co0 + 32 * m + l32 < a.Cout ? co0 + 32 * m + l32 : a.Cout - 1;
        bool on[2], halo[2];
        int b[2], i0[2], j0[2];
        f32x16_t sum[2];
#pragma unroll
        for (int nt = 0; nt < 2; ++nt) {
            const int ql = q0 + (wave * 2 + nt) * 32 + l32;
            on[nt] = ql <= q_last;
            halo[nt] = false;
            const int q = on[nt] ? ql : q_last;
            b[nt] = small_div(q, IJ, rIJ);
            const int rem = q - b[nt] * IJ;
            i0[nt] = small_div(rem, g.NJ, rNJ);
            j0[nt] = rem - i0[nt] * g.NJ;
#pragma unroll
            for (int i = 0; i < 16; ++i) sum[nt][i] = 0.f;
        }
        for (int u = 0; u < g.Tr; ++u)
            for (int v = 0; v < g.Tc; ++v) {
                unsigned xo[2];
#pragma unroll
                for (int nt = 0; nt < 2; ++nt) {
                    const int i = i0[nt] + g.rb + u * g.xs, j = j0[nt] + g.cb + v * g.xs;
                    const bool in = on[nt] && i >= 0 && i < a.H && j >= 0 && j < a.W;
                    halo[nt] = halo[nt] || !in;
                    xo[nt] = in ? (unsigned)(((b[nt] * a.Cin * a.H + i) * a.W + j) * ES) : kNoByte;
                }
                sum_tiles<TIn>(sum, rs_w, (unsigned)((ch * a.Cin * NN + (g.r + u * g.ws) * a.n + g.c + v * g.ws) * ES),
                               w_cstride, rs_x, xo, x_cstride, 0, a.Cin);
            }
#pragma unroll
        for (int nt = 0; nt < 2; ++nt) {
            if (!(tiles >> (2 * m + nt) & 1) || !on[nt]) continue;
            float* const out =
                y + ((size_t)b[nt] * a.Cout * a.OH + g.oy0 + i0[nt] * g.os) * a.OW + g.ox0 + j0[nt] * g.os;
            put_tile(
                lds, sum[nt], halo[nt],
                [&](int i, float v) {
                    const int c = co0 + 32 * m + 8 * (i / 4) + 4 * gk + i % 4;
                    if (c < a.Cout) out[c * pixels] = v;
                },
                [&](int i) { return (8 * m + 2 * i + gk) * TN + (wave * 2 + nt) * 32 + l32; });
        }
    }
    __threadfence();  // what was stored lies in memory before it is stored again
    __syncthreads();
    const int listed = *reinterpret_cast<const int*>(lds);
    for (int e = tid; e < listed; e += T) {
        const int group = reinterpret_cast<const unsigned short*>(lds + 16)[e];
        const int q = q0 + group % TN, cbase = co0 + group / TN * 4;
        if (cbase >= a.Cout) continue;
        const int b = small_div(q, IJ, rIJ), rem = q - b * IJ;
        const int i0 = small_div(rem, g.NJ, rNJ), j0 = rem - i0 * g.NJ;
        float sum[4] = {0.f, 0.f, 0.f, 0.f};
        for (int u = 0; u < g.Tr; ++u) {
            const int i = i0 + g.rb + u * g.xs;
            if (i < 0 || i >= a.H) continue;
            for (int v = 0; v < g.Tc; ++v) {
                const int j = j0 + g.cb + v * g.xs;
                if (j < 0 || j >= a.W) continue;
                unsigned wo[4];
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    wo[k] = (unsigned)(((cbase + k < a.Cout ? cbase + k : a.Cout - 1) * a.Cin * NN +
                                        (g.r + u * g.ws) * a.n + g.c + v * g.ws) * ES);
                sum_products<TIn>(sum, rs_x, (unsigned)(((b * a.Cin * a.H + i) * a.W + j) * ES), x_cstride, rs_w, wo,
                                  w_cstride, 0, a.Cin);
            }
        }
        float* const out = y + ((size_t)b * a.Cout * a.OH + g.oy0 + i0 * g.os) * a.OW + g.ox0 + j0 * g.os;
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (cbase + k < a.Cout) out[(cbase + k) * pixels] = sum[k];
    }
}

// LDS bytes, XU and grid of a layer on blocks of 32 * mt channels; false if the kernel cannot run it
struct ConvPlan { ConvArgs a; int mt, xu; size_t lds; unsigned blocks; };

bool make_plan(ConvArgs a, int es, int mt, ConvPlan& p)
{
    const size_t lim = 0x7FFFFFF0u;  // single buffer descriptors, 32-bit byte offsets
    const int NN = a.n * a.n, parts = es == 4 ? 3 : 1;
    if ((size_t)a.B * a.Cin * a.H * a.W * es > lim || (size_t)a.Cout * a.Cin * NN * es > lim ||
        (size_t)a.B * a.Cout * a.OH * a.OW * 4 > lim)
        return false;
    a.classes = a.dilated ? 1 : a.k * a.k;
    p.mt = mt;
    a.nco = (a.Cout + 32 * p.mt - 1) / (32 * p.mt);
    long long slots = 0, units = 0, qmax = 0;
    for (int c = 0; c < a.classes; ++c) {
        const Class g = class_of(a, c);
        const long long ij = (long long)g.NI * g.NJ, q = a.B * ij;
        if (q == 0) continue;
        if (q >= (1 << 24) || (long long)a.B * g.EH >= (1 << 24)) return false;  // small_div
        if (g.Tr && parts == 1 && g.cols > 0 && g.cols < 4) return false;        // pieces of four columns
        // TN consecutive pixels touch at most this many lattice rows / images
        const long long nrho = TN % g.NJ == 0 ? TN / g.NJ : (TN - 2) / g.NJ + 2;
        const long long nimg = ij % TN == 0 ? 1 : TN % ij == 0 ? TN / ij : (TN - 2) / ij + 2;
        const long long rows = nrho + (g.EH - g.NI) * nimg;
        if (rows * g.LW > slots) slots = rows * g.LW;
        const long long un = 2 * rows * ((g.cols + (parts == 3 ? 0 : 3)) / (parts == 3 ? 1 : 4));
        if (un > units) units = un;
        if (q > qmax) qmax = q;
    }
    if (qmax == 0 || slots > 8192) return false;
    a.XPL = (int)(2 * slots * 16);
    const int per = (int)((units + T - 1) / T);
    if (parts == 3) p.xu = per <= 3 ? 3 : per <= 5 ? 5 : 8;
    else p.xu = per <= 1 ? 1 : per <= 2 ? 2 : 4;
    if (per > p.xu) return false;
    p.lds = 2 * (size_t)parts * 4 * (32 * p.mt + 4) * 16 + (size_t)parts * a.XPL;
    if (p.lds < redo_bytes(TN * 8 * p.mt)) p.lds = redo_bytes(TN * 8 * p.mt);
    if (p.lds > LDS_LIMIT) return false;
    a.nqt = (int)((qmax + TN - 1) / TN);
    const long long nb = (long long)a.nqt * a.nco * a.classes;
    if (nb > 0x3FFFFFFF) return false;
    // Classes of unequal taps, an incomplete second round of blocks and a sum of some length (fp32): within four pixel tiles
    // the classes of most taps start first, so that the blocks that start last are the short ones.  Neighbouring classes
    // write y later than one another, which few channels do not repay.  Time class by class over time by taps, geometric means
    // of 18000 layers, from 64 channels on (48 to 63: stride 3 1.07 at 513 to 576 blocks, 1.00 beyond): stride 2 1.21 to 1.25 at 513 to
    // 576 blocks, 1.09 to 1.18 up to 1024; stride 3, two blocks to a compute unit 1.07 to 1.12 and 1.01 to 1.02, but where LDS
    // holds one, whose rounds are of 256, 0.98 to 1.04 and 0.99; stride 4, n = 5, 6 1.03 to 1.12 from 577 blocks on, below (a second
    // round of a few blocks, most of them of one tap) 0.95 to 1.00, n = 7, one class in four short, 0.93 to 1.00.
    // 128 -> 64 channels, 16 of 32 x 32, n = 5, stride 3, 576 blocks 80.2 / 70.5 us; beyond 1024 blocks 336 -> 72, 13 of 34 x 34,
    // n = 5, 1116 blocks 233 / 243, below 513 49.5 / 52.4, equal taps, 168 -> 152, n = 4, stride 4 231 / 244.
    const bool unequal = !a.dilated && a.classes <= 16 && a.n > a.k && a.n % a.k != 0;
    const bool second_round = nb > (a.k == 4 ? 576 : 512) && nb <= 1024;
    a.group = unequal && second_round && es == 4 && a.Cin >= 64 && (a.k != 3 || 2 * p.lds <= LDS_LIMIT) &&
              (a.k != 4 || a.n < 7) ? 4 : 1;
    a.order = 0;
    for (int c = 0; a.group > 1 && c < a.classes; ++c) {
        const Class g = class_of(a, c);
        int rank = 0;
        for (int d = 0; d < a.classes; ++d) {
            const Class h = class_of(a, d);
            rank += h.Tr * h.Tc > g.Tr * g.Tc || (h.Tr * h.Tc == g.Tr * g.Tc && d < c) ? 1 : 0;
        }
        a.order |= (unsigned long long)c << (4 * rank);
    }
    p.blocks = (unsigned)nb;
    p.a = a;
    return true;
}

// Blocks of 64 channels read less per product; of 32 where those do not fit LDS (14 images, 184 -> 152 channels, 45 x 10, n = 5,
// dilation 4: 1122 us on the vector ALUs, 176 so), where there are no more than 32, and where even twice the blocks leave
// every one a compute unit of its own (us, 64 / 32: 72 -> 128, 10 of 38 x 38, n = 5, dilation 2, 228 blocks of 32 120 / 87; 216 -> 144
// bf16, 250 blocks 70 / 55; but 40 -> 184, 294 blocks 51 / 71, strided layers of 800 to 12000 blocks 0.7 to 1.2 times as fast).
// fp32: also where all of them are resident at once, two to a compute unit, and cover each other's waits (dilation 2, 64 -> 64 at
// 64 x 64, n = 3: 11 images, 352 blocks 46.3 / 41.3, 16 images, 512 blocks 44.0 / 40.4; 20, 640 blocks 61 / 65; n = 5, where LDS
// holds one, 100 / 131; bf16, whose loop waits less, 27.0 / 27.2).  Classes of one tap have little to
// share (stride 3, 64 -> 64, n = 3, one of 64 x 64 17.8 / 18.5, two of 40 x 40 17.5 / 16.5; n = 4 27.1 / 25.1, 26.8 / 22.5)
bool pick_plan(const ConvArgs& a, int es, ConvPlan& p)
{
    if (a.Cout <= 32) return make_plan(a, es, 1, p);
    if (!make_plan(a, es, 2, p)) return make_plan(a, es, 1, p);
    ConvPlan q;
    if (p.blocks <= 256 && (a.dilated || a.n > a.k) && make_plan(a, es, 1, q) &&
        (q.blocks <= 256 || (es == 4 && q.blocks <= 512 && 2 * q.lds <= LDS_LIMIT)))
        p = q;
    return true;
}

template <int MT, int XU, typename TIn>
hipError_t launch_v(const ConvPlan& p, const void* x, const void* w, float* y, hipStream_t stream)
{
    const hipError_t e = hipFuncSetAttribute((const void*)ukst_general_mfma_kernel<MT, XU, TIn>,
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)p.lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((ukst_general_mfma_kernel<MT, XU, TIn>), dim3(p.blocks), dim3(T), p.lds, stream, (const TIn*)x,
                       (const TIn*)w, y, p.a);
    return hipGetLastError();
}

}  // namespace

bool general_mfma_fits(int dilated, int B, int Cin, int Cout, int H, int W, int n, int P, int k, int OH, int OW, int dtype)
{
    ConvArgs a;
    a.B = B; a.Cin = Cin; a.Cout = Cout; a.H = H; a.W = W; a.n = n; a.P = P; a.k = k; a.OH = OH; a.OW = OW;
    a.dilated = dilated;
    ConvPlan p;
    return pick_plan(a, dtype == 0 ? 4 : 2, p);
}

bool launch_general_mfma(int dilated, int B, int Cin, int Cout, int H, int W, int n, int P, int k, int OH, int OW,
                         const void* x, const void* w, float* y, int dtype, hipStream_t stream, hipError_t* err)
{
    // from 16 channels on the smallest layers gain too (16 -> 16 channels, 8 x 8 maps, stride 3: 9.3 -> 7.2 us;
    // 16 x 16 maps, dilation 2: 30 -> 11.5); what does not fit LDS (long rows under a wide dilation) is for the small tiles
    if (Cin < 16 || Cout < 8) return false;
    // one stage of channels and many lattice pixels: writing y with a stride is all there is (16 -> 16 channels,
    // 8 x 48 x 48, stride 3, fp32: 17.2 against 17.7 us)
    if (!dilated && dtype == 0 && Cin * Cout < 512 && (long long)B * H * W > 4096) return false;
    // one or two stages of channels and no class with more than one tap: little to multiply, and the vector ALUs neither
    // pad the channels nor write y a class at a time.  fp32, 24 x 25 maps, 4 images, vector ALUs against this kernel, us:
    // 17 -> 64 channels, n = 1, stride 1 9.2 / 11.2, n = 2, stride 2 10.2 / 12.4, 17 -> 8, n = 1, stride 5 9.0 / 10.6 (16
    // images of 40 x 41, 17 -> 64, n = 1, stride 1 14.7 / 12.5; 17 -> 200, n = 1, stride 5 39 / 33); stride 8 16 -> 32,
    // n = 1 19.1 / 22.1, 16 -> 200, n = 2 71 / 86, 17 -> 8, n = 3 12.2 / 15.9 (17 -> 32, n = 3 25.8 / 24.8); bf16
    // 16 -> 64, n = 2, stride 8 28.0 / 32.2, and 16 images of 40 x 41, 17 -> 8, n = 4, stride 4 23.1 / 27.4, 16 -> 8, n = 5,
    // stride 8 62.6 / 71.2 (stride 5 29.7 / 27.6)
    if (!dilated && Cin < 20 && n <= k) {
        const bool few = (long long)B * H * W < 4096;
        if (dtype != 0 && !few && Cout <= 8 && k % 4 == 0) return false;
        if (dtype == 0 && few && n <= 3 && Cin > 16 && Cout <= 64 && k < 8) return false;
        if (k >= 8 && n <= 3 && ((n == 2 && few) || (dtype == 0 && (n == 1 || Cout <= 8)))) return false;
    }
    ConvArgs a;
    a.B = B; a.Cin = Cin; a.Cout = Cout; a.H = H; a.W = W; a.n = n; a.P = P; a.k = k; a.OH = OH; a.OW = OW;
    a.dilated = dilated;
    ConvPlan p;
    if (!pick_plan(a, dtype == 0 ? 4 : 2, p)) return false;
    if (dtype == 0) {
        if (p.mt == 2)
            *err = p.xu == 3 ? launch_v<2, 3, float>(p, x, w, y, stream)
                 : p.xu == 5 ? launch_v<2, 5, float>(p, x, w, y, stream) : launch_v<2, 8, float>(p, x, w, y, stream);
        else
            *err = p.xu == 3 ? launch_v<1, 3, float>(p, x, w, y, stream)
                 : p.xu == 5 ? launch_v<1, 5, float>(p, x, w, y, stream) : launch_v<1, 8, float>(p, x, w, y, stream);
    } else {
        if (p.mt == 2)
            *err = p.xu == 1 ? launch_v<2, 1, uint16_t>(p, x, w, y, stream)
                 : p.xu == 2 ? launch_v<2, 2, uint16_t>(p, x, w, y, stream) : launch_v<2, 4, uint16_t>(p, x, w, y, stream);
        else
            *err = p.xu == 1 ? launch_v<1, 1, uint16_t>(p, x, w, y, stream)
                 : p.xu == 2 ? launch_v<1, 2, uint16_t>(p, x, w, y, stream) : launch_v<1, 4, uint16_t>(p, x, w, y, stream);
    }
    return true;
}

}  // namespace ukst
