// Gradient with respect to the input of wide fp32 layers on the bf16 matrix pipe, operands as three exact bf16 parts
// (ukst_parts.h); n = 2..7, any sizes.
//
// dx[b][ci][i][j] = sum_co sum_{a,c} dy[b][co][2i+P-a][2j+P-c] * w[co][ci][a][c].  Tap rows of one parity meet the dy
// rows of one parity (Sec. 3.1 read backwards), so the sum falls into four stride-1 correlations, one per parity class
// of dy, each with its ceil or floor(n/2) squared taps:
//     dx[i][j] += sum_co sum_{u<Tr, v<Tc} D[co][i + rb + u][j + cb + v] * w[co][ci][a0 + 2(Tr-1-u)][c0 + 2(Tc-1-v)],
//     D[co][r][s] = dy[co][2r + pr][2s + pc].
// An implicit GEMM with M = input channels, N = pixels flattened over (image, row, column), K = output channels, 16
// per MFMA; a stage is 16 output channels of one class, staged as a dense sub-image (columns two apart in memory, the
// other column parity's stage next, while the lines are near).
//
// A sub-image serves a quarter of the taps only (2.25 of them at n = 3), so staging is what could bound it: with more
// than 64 input channels eight waves share one (128 channels x 256 pixels, two waves per SIMD), else four waves take 64
// channels and two blocks share a compute unit.  A wave owns 64 channels x 64 pixels and reads 12 KiB of fragments per
// tap for 24 MFMAs.  Weights go through LDS two taps at a time, the group after next on its way in registers.
// fp32 pipe -> this kernel, 32 x 128 -> 128 channels: 63 x 63, n = 3 444 -> 259 us; 64 x 64, n = 4 671 -> 388, n = 5 953 -> 610.
#include "ukst_parts.h"

namespace ukst {
namespace {

constexpr int KC = 16, TN = 256;
constexpr int LDS_LIMIT = 160 * 1024 - 256;  // (256 bytes belong to __syncthreads_or)

struct GiPartsArgs {
    int B, Cin, Cout, H, W, n, P, OH, OW;
    int nci, nqt;  // channel blocks, pixel tiles
    int EH, LW;    // staged rows per image, staged columns (of the largest class)
    int XPL;       // bytes of one part's sub-image stage
    FastDiv dHW, dW, dEH, dLW;
};

// a parity class of dy (uniform over a block): first tap, taps per axis, row and column parity, sub-image origin
struct Class { int a0, c0, Tr, Tc, pr, pc, rb, cb; };
__device__ __forceinline__ Class class_of(const GiPartsArgs& a, int cls)
{
    Class q;
    q.a0 = cls >> 1;
    q.c0 = cls & 1;
    q.Tr = (a.n - q.a0 + 1) >> 1;
    q.Tc = (a.n - q.c0 + 1) >> 1;
    q.pr = (a.P - q.a0) & 1;
    q.pc = (a.P - q.c0) & 1;
    q.rb = ((a.P - q.a0 - q.pr) >> 1) - (q.Tr - 1);
    q.cb = ((a.P - q.c0 - q.pc) >> 1) - (q.Tc - 1);
    return q;
}

// CW: 64-channel groups per block (4 waves each); XU: sub-image units per thread
template <int CW, int XU>
__global__ __launch_bounds__(256 * CW) __attribute__((amdgpu_waves_per_eu(2, 2)))
void ukst_grad_input_mfma_kernel_parts(const float* __restrict__ dy, const float* __restrict__ w,
                                       float* __restrict__ dx, GiPartsArgs a)
{
    constexpr int T = 256 * CW, TM = 64 * CW;
    constexpr int WTS = (TM + 4) * 16;  // a tap's 16-byte slots [channel]; the staging lanes (tap, half, 4 channels) of a
    constexpr int WHS = 2 * WTS;        // 16-lane pass hit 16 different slots modulo 16
    constexpr int WPL = 2 * WHS, WBUF = 3 * WPL, XS_OFF = 2 * WBUF;
    typedef PartProducts<3> PP;
    extern __shared__ __align__(16) unsigned char lds[];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int cw = wave % CW, qw = wave / CW;
    const int l32 = lane & 31, gk = lane >> 5;
    const int bid = xcd_contiguous(blockIdx.x, gridDim.x);
    const int ci0 = bid % a.nci * TM, q0 = bid / a.nci * TN;
    const int HW = a.H * a.W, Q = a.B * HW, NN = a.n * a.n;
    const int q_last = q0 + TN - 1 < Q ? q0 + TN - 1 : Q - 1;
    // pixel row rho = b*H + i reads staged rows e = b*EH + i + u, less the tile's first
    const int bf0 = fdiv(q0, a.dHW), if0 = fdiv(q0 - bf0 * HW, a.dW);
    const int e_first = bf0 * a.EH + if0;
    const int bl = fdiv(q_last, a.dHW), il = fdiv(q_last - bl * HW, a.dW);
    const int rows = bl * a.EH + il + a.EH - a.H - e_first + 1;
    const int XPL = a.XPL, XH = rows * a.LW * 16;  // (the other channel half follows the first)

    const __amdgpu_buffer_rsrc_t rs_dy = __builtin_amdgcn_make_buffer_rsrc(
        (void*)dy, 0, (int)((size_t)a.B * a.Cout * a.OH * a.OW * 4), kRawBuffer);
    const __amdgpu_buffer_rsrc_t rs_w =
        __builtin_amdgcn_make_buffer_rsrc((void*)w, 0, (int)((size_t)a.Cout * a.Cin * NN * 4), kRawBuffer);
    const unsigned y_cstride = (unsigned)(a.OH * a.OW * 4);

    // sub-image units: (channel half, row, column), column fastest; every unit is written in every stage
    int x_base[XU], x_loff[XU], x_ij[XU];
#pragma unroll
    for (int j = 0; j < XU; ++j) {
        const int e = tid + T * j, per_half = rows * a.LW;
        const int h = e >= per_half ? 1 : 0, rem = e - h * per_half;
        const int row = fdiv(rem, a.dLW), col = rem - row * a.LW;
        const int er = e_first + row, b = fdiv(er, a.dEH), i = er - b * a.EH;
        x_loff[j] = e < 2 * per_half ? XS_OFF + h * XH + rem * 16 : -1;
        x_base[j] = ((b * a.Cout + 8 * h) * a.OH + 2 * i) * a.OW + 2 * col;
        x_ij[j] = (h << 31) | (i << 15) | col;  // (b < B: the tile's rows end with its last image)
    }
    // weight unit of the thread: (input channel, channel half, tap of the group)
    const int w_t = tid & 1, w_h = (tid >> 1) & 1, w_ci = tid >> 2;
    const int w_base = (8 * w_h * a.Cin + ci0 + w_ci) * NN;
    const bool w_on = ci0 + w_ci < a.Cin;
    const int w_loff = w_h * WHS + w_t * WTS + w_ci * 16;

    const int stages = (a.Cout + KC - 1) / KC;
    unsigned xr[XU][8], wr[8];
    // a group of two taps: stage of 16 channels, class, group of the class
    struct At { int s, cls, grp; };
    auto next = [&](At t) {
        const Class q = class_of(a, t.cls);
        if (2 * ++t.grp >= q.Tr * q.Tc) {
            t.grp = 0;
            if (++t.cls == 4) { t.cls = 0; ++t.s; }
        }
        return t;
    };
    auto load_x = [&](const At& t) {
        const Class q = class_of(a, t.cls);
        const int shift = (2 * q.rb + q.pr) * a.OW + 2 * q.cb + q.pc;
#pragma unroll
        for (int j = 0; j < XU; ++j) {
            const int oy = 2 * (((x_ij[j] >> 15) & 0xFFFF) + q.rb) + q.pr, ox = 2 * ((x_ij[j] & 0x7FFF) + q.cb) + q.pc;
            const bool in = x_loff[j] >= 0 && oy >= 0 && oy < a.OH && ox >= 0 && ox < a.OW;
            const unsigned voff = in ? (unsigned)(x_base[j] + shift) * 4u : kNoByte;
#pragma unroll
            for (int k = 0; k < 8; ++k)
                xr[j][k] = __builtin_amdgcn_raw_buffer_load_b32(rs_dy, voff, (unsigned)(t.s * KC + k) * y_cstride, 0);
        }
    };
    auto store_x = [&](const At& t) {
#pragma unroll
        for (int j = 0; j < XU; ++j) {
            if (t.s * KC + KC > a.Cout) {  // channels past the last one: zeros
#pragma unroll
                for (int k = 0; k < 8; ++k)
                    xr[j][k] = t.s * KC + (x_ij[j] < 0 ? 8 : 0) + k < a.Cout ? xr[j][k] : 0u;
            }
            u4v_t p[3];
            to_parts<3>(xr[j], p);
            if (x_loff[j] < 0) continue;
#pragma unroll
            for (int i = 0; i < 3; ++i) *reinterpret_cast<u4v_t*>(lds + i * XPL + x_loff[j]) = p[i];
        }
    };
    auto load_w = [&](const At& t) {  // (past the last stage: nothing)
        const Class q = class_of(a, t.cls);
        const int tap = 2 * t.grp + w_t;
        const int u = (tap >= q.Tc ? 1 : 0) + (tap >= 2 * q.Tc ? 1 : 0) + (tap >= 3 * q.Tc ? 1 : 0), v = tap - u * q.Tc;
        const int off = (q.a0 + 2 * (q.Tr - 1 - u)) * a.n + q.c0 + 2 * (q.Tc - 1 - v);
        const bool in = w_on && t.s < stages && tap < q.Tr * q.Tc;
        const unsigned voff = in ? (unsigned)(w_base + off) * 4u : kNoByte;
#pragma unroll
        for (int k = 0; k < 8; ++k)
            wr[k] = __builtin_amdgcn_raw_buffer_load_b32(
                rs_w, voff, in ? (unsigned)((t.s * KC + k) * a.Cin * NN) * 4u : 0u, 0);
    };
    auto store_w = [&](const At& t, int buf) {
        if (t.s * KC + KC > a.Cout) {
#pragma unroll
            for (int k = 0; k < 8; ++k) wr[k] = t.s * KC + 8 * w_h + k < a.Cout ? wr[k] : 0u;
        }
        u4v_t p[3];
        to_parts<3>(wr, p);
#pragma unroll
        for (int i = 0; i < 3; ++i) *reinterpret_cast<u4v_t*>(lds + buf * WBUF + i * WPL + w_loff) = p[i];
    };

    const int a_lds = gk * WHS + (cw * 64 + l32) * 16;
    int b_lds[2];
#pragma unroll
    for (int nt = 0; nt < 2; ++nt) {
        int q = q0 + (qw * 2 + nt) * 32 + l32;
        if (q > q_last) q = q_last;
        const int b = fdiv(q, a.dHW), rem = q - b * HW;
        const int i = fdiv(rem, a.dW), j = rem - i * a.W;
        b_lds[nt] = XS_OFF + gk * XH + ((b * a.EH + i - e_first) * a.LW + j) * 16;
    }
    f32x16_t acc[2][2];
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int nt = 0; nt < 2; ++nt)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[m][nt][i] = 0.f;

    auto tap = [&](int buf, int t, int xoff) {  // t: 0 or 1; xoff: bytes of the tap's place in the sub-image
        bf16x8_t af[2][3], bf[2][3];
#pragma unroll
        for (int i = 2; i >= 0; --i) {
#pragma unroll
            for (int m = 0; m < 2; ++m)
                af[m][i] = *reinterpret_cast<const bf16x8_t*>(lds + buf * WBUF + a_lds + i * WPL + t * WTS + m * 512);
#pragma unroll
            for (int nt = 0; nt < 2; ++nt)
                bf[nt][i] = *reinterpret_cast<const bf16x8_t*>(lds + b_lds[nt] + i * XPL + xoff);
        }
#pragma unroll
        for (int p = 0; p < PP::count; ++p)
#pragma unroll
            for (int m = 0; m < 2; ++m)
#pragma unroll
                for (int nt = 0; nt < 2; ++nt)
                    acc[m][nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[m][PP::a[p]], bf[nt][PP::b[p]], acc[m][nt],
                                                                         0, 0, 0);
    };

    At at = {0, 0, 0};
    load_w(at);
    load_x(at);
    store_w(at, 0);
    store_x(at);
    At n1 = next(at);
    load_w(n1);
    __syncthreads();
    int buf = 0, u = 0, v = 0;
    while (at.s < stages) {
        const Class q = class_of(a, at.cls);
        const At n2 = next(n1);
        const bool last = n1.grp == 0;  // last group of its stage
        if (last && n1.s < stages) load_x(n1);
        __builtin_amdgcn_sched_barrier(0);
        tap(buf, 0, (u * a.LW + v) * 16);
        if (++v == q.Tc) { v = 0; ++u; }
        __builtin_amdgcn_sched_barrier(0);
        store_w(n1, buf ^ 1);
        load_w(n2);
        __builtin_amdgcn_sched_barrier(0);
        if (2 * at.grp + 1 < q.Tr * q.Tc) {
            tap(buf, 1, (u * a.LW + v) * 16);
            if (++v == q.Tc) { v = 0; ++u; }
        }
        __syncthreads();
        if (last) {
            if (n1.s < stages) store_x(n1);
            u = v = 0;
            __syncthreads();
        }
        buf ^= 1;
        at = n1;
        n1 = n2;
    }

    // accumulator register e of a tile holds channel 8*(e/4) + 4*gk + (e%4), for the lane's pixel
#pragma unroll
    for (int nt = 0; nt < 2; ++nt) {
        const int q = q0 + (qw * 2 + nt) * 32 + l32;
        if (q > q_last) continue;
        const int b = fdiv(q, a.dHW), rem = q - b * HW;
        float* const out = dx + (size_t)b * a.Cin * HW + rem;
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int ci = ci0 + cw * 64 + 32 * m + 8 * (e / 4) + 4 * gk + (e % 4);
                const float val = acc[m][nt][e] * kPartsDown;
                if (ci < a.Cin) out[(size_t)ci * HW] = val;
            }
    }

    float most = 0.f;
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int nt = 0; nt < 2; ++nt) most = peak(acc[m][nt], most);
    if (!__syncthreads_or(most < __builtin_inff() ? 0 : 1)) return;
    // tiles that hold a sum that is not finite (ukst_parts.h)
    unsigned tiles = 0u;
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int nt = 0; nt < 2; ++nt)
            if (!wave_finite(acc[m][nt])) tiles |= 1u << (2 * m + nt);
    if (tid == 0) *reinterpret_cast<unsigned*>(lds) = 0u;
    __syncthreads();
    const unsigned w_cstride = (unsigned)(a.Cin * NN) * 4u;
    // group: (four channels, pixel) of the block's outputs
    for (; tiles != 0u; tiles &= tiles - 1) {
        const int t = __builtin_ctz(tiles), m = t >> 1, ql = (qw * 2 + (t & 1)) * 32 + l32;
        const bool on = q0 + ql <= q_last;
        const int q = on ? q0 + ql : q_last;
        const int b = fdiv(q, a.dHW), rem = q - b * HW;
        const int i = fdiv(rem, a.dW), j = rem - i * a.W;
        const int cl = 64 * cw + 32 * m, ch = ci0 + cl + l32 < a.Cin ? ci0 + cl + l32 : a.Cin - 1;
        bool halo = false;
        f32x16_t sum[1];
#pragma unroll
        for (int k = 0; k < 16; ++k) sum[0][k] = 0.f;
        for (int ta = 0; ta < a.n; ++ta)
            for (int tc = 0; tc < a.n; ++tc) {
                const int oy = 2 * i + a.P - ta, ox = 2 * j + a.P - tc;
                const bool in = on && oy >= 0 && oy < a.OH && ox >= 0 && ox < a.OW;
                halo = halo || !in;
                const unsigned dyo[1] = {in ? (unsigned)((b * a.Cout * a.OH + oy) * a.OW + ox) * 4u : kNoByte};
                sum_tiles<float>(sum, rs_w, (unsigned)(ch * NN + ta * a.n + tc) * 4u, w_cstride, rs_dy, dyo, y_cstride, 0,
                                 a.Cout);
            }
        float* const out = dx + (size_t)b * a.Cin * HW + rem;
        if (on)
            put_tile(
                lds, sum[0], halo,
                [&](int k, float v) {
                    const int c = ci0 + cl + 8 * (k / 4) + 4 * gk + k % 4;
                    if (c < a.Cin) out[(size_t)c * HW] = v;
                },
                [&](int k) { return (cl / 4 + 2 * k + gk) * TN + ql; });
    }
    __threadfence();  // what was stored lies in memory before it is stored again
    __syncthreads();
    const int listed = *reinterpret_cast<const int*>(lds);
    for (int e = tid; e < listed; e += T) {
        const int group = reinterpret_cast<const unsigned short*>(lds + 16)[e];
        const int q = q0 + group % TN, cbase = ci0 + group / TN * 4;
        if (cbase >= a.Cin) continue;
        const int b = fdiv(q, a.dHW), rem = q - b * HW;
        const int i = fdiv(rem, a.dW), j = rem - i * a.W;
        float sum[4] = {0.f, 0.f, 0.f, 0.f};
        for (int ta = 0; ta < a.n; ++ta) {
            const int oy = 2 * i + a.P - ta;
            if (oy < 0 || oy >= a.OH) continue;
            for (int tc = 0; tc < a.n; ++tc) {
                const int ox = 2 * j + a.P - tc;
                if (ox < 0 || ox >= a.OW) continue;
                unsigned wo[4];
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    wo[k] = (unsigned)((cbase + k < a.Cin ? cbase + k : a.Cin - 1) * NN + ta * a.n + tc) * 4u;
                sum_products<float>(sum, rs_dy, (unsigned)((b * a.Cout * a.OH + oy) * a.OW + ox) * 4u, y_cstride, rs_w,
                                    wo, w_cstride, 0, a.Cout);
            }
        }
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (cbase + k < a.Cin) dx[((size_t)b * a.Cin + cbase + k) * HW + rem] = sum[k];
    }
}

struct GiPlan { GiPartsArgs a; int cw, xu; size_t lds; unsigned blocks; };

bool make_plan(const GeomBase& g, GiPlan& p)
{
    if (g.Cin < 32 || g.Cout < 16 || g.n < 2 || g.n > 7) return false;
    const size_t lim = 0x7FFFFFF0u;  // single buffer descriptors, 32-bit byte offsets
    if ((size_t)g.B * g.Cout * g.OH * g.OW * 4 > lim || (size_t)g.Cout * g.Cin * g.n * g.n * 4 > lim) return false;
    if (g.H >= (1 << 15) - 8 || g.W >= (1 << 15) - 8) return false;  // packed row and column of a unit
    GiPartsArgs a;
    a.B = g.B; a.Cin = g.Cin; a.Cout = g.Cout; a.H = g.H; a.W = g.W; a.n = g.n; a.P = g.P; a.OH = g.OH; a.OW = g.OW;
    const long long hw = (long long)g.H * g.W, Q = g.B * hw;
    if (Q > 0x3FFFFFFFLL) return false;
    const int span = (g.n + 1) / 2 - 1;
    a.EH = g.H + span;
    a.LW = g.W + span;
    p.cw = g.Cin > 64 ? 2 : 1;
    const int T = 256 * p.cw;
    // TN consecutive pixels touch at most this many rows / images
    const long long nrho = TN % g.W == 0 ? TN / g.W : (TN - 2) / g.W + 2;
    const long long nimg = hw % TN == 0 ? 1 : TN % hw == 0 ? TN / hw : (TN - 2) / hw + 2;
    const long long slots = (nrho + span * nimg) * a.LW;
    if (slots > 8192) return false;
    a.XPL = (int)(2 * slots * 16);
    const int per = (int)((2 * slots + T - 1) / T);
    p.xu = p.cw == 2 ? (per <= 2 ? 2 : per <= 3 ? 3 : 4) : (per <= 4 ? 4 : 6);
    if (per > p.xu) return false;
    p.lds = 2 * (size_t)3 * 4 * (64 * p.cw + 4) * 16 + (size_t)3 * a.XPL;
    if (p.lds < redo_bytes(TN * 16 * p.cw)) p.lds = redo_bytes(TN * 16 * p.cw);
    if (p.lds > LDS_LIMIT) return false;
    a.nci = (g.Cin + 64 * p.cw - 1) / (64 * p.cw);
    a.nqt = (int)((Q + TN - 1) / TN);
    const long long nb = (long long)a.nci * a.nqt;
    // a tile is one block's serial work: few of them lose to the fp32 pipe, which splits the sum over channels (64
    // tiles, 64 images of 128 -> 64 channels, 16 x 16, n = 4: 68 against 84 us; 102 tiles of 128 -> 128, 51 x 51, n = 2 /
    // 3 / 4 / 5 / 7: 131 / 193 / 276 / 383 / 667 against 90 / 118 / 168 / 257 / 478).  Blocks of four waves, up to 64
    // input channels, take as long for half the channels, and that pipe splits further with many output channels: from
    // there on they gain at n = 3 and 4 only (33 -> 160 channels, n = 4, 102 tiles: 202 against 197).  n = 5 and 7, 33 ->
    // 160: 102 tiles 263 / 441 against 297 / 502, 122 tiles 265 / 445 against 298 / 502, 133 tiles 330 / 559 against
    // 297 / 504; n = 6 355 against 399 at 102, 428 against 400 at 122; 33 -> 256, n = 5, 122 tiles 484 against 472; n = 2 only
    // 33 -> 96, 59 against 70 (-> 64 and -> 128 gain); with few output channels all of them, 64 -> 64 as 64 -> 16 (n = 5,
    // 102 tiles: 129 against 118, 56 against 34; 33 -> 64, n = 7: 191 against 204); 64 -> 160, n = 7, 122 tiles 525 against 480
    int line = 100;
    if (p.cw == 1 && g.n >= 5 && (g.Cout > 64 || (g.Cout > 32 && g.Cin < 40)))
        line = (g.n == 7 && g.Cin < 56) || (g.n == 5 && g.Cout <= 160) ? 130 : 115;
    if (p.cw == 1 && g.n == 2 && g.Cout > 64 && g.Cout <= 96) line = 115;
    if (nb < line || nb > 0x3FFFFFFF) return false;
    p.blocks = (unsigned)nb;
    a.dHW = make_fastdiv((unsigned)hw);
    a.dW = make_fastdiv((unsigned)g.W);
    a.dEH = make_fastdiv((unsigned)a.EH);
    a.dLW = make_fastdiv((unsigned)a.LW);
    p.a = a;
    return true;
}

template <int CW, int XU>
hipError_t launch(const GiPlan& p, const float* dy, const float* w, float* dx, hipStream_t stream)
{
    const hipError_t e = hipFuncSetAttribute((const void*)ukst_grad_input_mfma_kernel_parts<CW, XU>,
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)p.lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((ukst_grad_input_mfma_kernel_parts<CW, XU>), dim3(p.blocks), dim3(256 * CW), p.lds, stream, dy, w,
                       dx, p.a);
    return hipGetLastError();
}

}  // namespace

bool grad_input_parts_supported(const GeomBase& g)
{
    GiPlan p;
    return make_plan(g, p);
}

hipError_t launch_grad_input_parts(const GeomBase& g, const float* dy, const float* w, float* dx, hipStream_t stream)
{
    GiPlan p;
    if (!make_plan(g, p)) return hipErrorInvalidValue;
    if (p.cw == 2)
        return p.xu == 2 ? launch<2, 2>(p, dy, w, dx, stream) : p.xu == 3 ? launch<2, 3>(p, dy, w, dx, stream)
                                                              : launch<2, 4>(p, dy, w, dx, stream);
    return p.xu == 4 ? launch<1, 4>(p, dy, w, dx, stream) : launch<1, 6>(p, dy, w, dx, stream);
}

}  // namespace ukst
