// Stride-2 forward layers on the bf16 matrix pipe from bf16 parts: fp32 operands as three exact parts
// (ukst_parts.h), bf16 operands as one.  Any row length, any channel counts, n = 2..5.
//
// The product is the one of ukst_mfma_f32.hip: per quad the four parity classes of Algorithm 2 share a
// window of the input (quads aligned to the output for even n and P, shifted quads otherwise); class
// (r, s) multiplies window position p by its tap w[r+2u][s+2v] (Eqs. 1-4).  M = output channels, N =
// quads flattened over (image, quad row, quad column), K = input channels, 16 per MFMA.
//
// What bounds it and why it is laid out like this.  With three parts a pair of fragment triples feeds
// six MFMAs, so the LDS reads of a tap (3 KiB of weights, 6 KiB of activations that two taps share) come
// with 12 MFMAs = 384 clocks and the matrix pipe is the bound; what has to be kept off its back is
// staging.  Splitting costs about 7 vector instructions per element, hence a wide tile (64 channels x
// 256 quads x 4 classes on 8 waves, two per SIMD, so that one wave's splitting runs beside the other's
// MFMAs); a load costs the address unit about 16 clocks whatever its width, hence weights in pieces of
// four taps x 2 (or 8) input channels, transposed in registers.  Weights are staged a run of 4 or 5
// taps at a time into the other of two buffers while the current one is multiplied, activations of 16
// channels once per n*n taps.  Only element alignment is needed anywhere.
#pragma once
#include "ukst_parts.h"

namespace ukst {
namespace parts {

constexpr int KC = 16;  // input channels per stage (one MFMA K step)
constexpr int LDS_LIMIT = 160 * 1024 - 256;  // (256 bytes belong to __syncthreads_or)

struct PartsArgs {
    GeomBase g;
    int KHq, KWq;  // quad rows / columns
    int cb_major;  // tile order: 1 = consecutive blocks share the channel block (big weights)
    int Q;         // total quads
    int EH;        // input rows one image's quad rows touch
    int ROWS;      // input rows an activation stage holds
    int LWX;       // 16-byte slots per staged row
    int XPL;       // bytes of one part's activation stage (both channel halves)
    int SH;        // slot of input column 0 = floor(P/2)
    int CPR;       // activation units per row
    int nco, nqt;
    int ksplit, kstages;
    size_t copy_bytes;  // distance of the slices' copies of y
    FastDiv dKHW, dKW, dEH, dRW, dW;
};

typedef unsigned u3v_t __attribute__((ext_vector_type(3)));

// tap of class c = 2r + s at window position (pa, pb) lies at tap row a = r + 2u, pa = u (+ r if aligned)
template <bool AL>
constexpr int pos_of(int a) { return AL ? (a >> 1) + (a & 1) : a >> 1; }

// Weights are staged in pieces of four consecutive taps (one 16- or 8-byte load per channel); a weight
// stage is a run of taps, its pieces start where piece_at says (the last piece of a run that is no
// multiple of four taps repeats some of its neighbour's).  Three parts: runs of 4 (or 5) taps, so that
// two weight stages fit LDS beside the activations; one part: all taps at once.
constexpr int sub_count(int n, int parts) { return parts == 1 ? 1 : n * n / 4; }
constexpr int sub_first(int n, int parts, int sub)  // first tap of a stage; sub == sub_count: n*n
{
    return sub == 0 ? 0 : sub == sub_count(n, parts) ? n * n : 4 * sub;
}
constexpr int sub_taps(int n, int parts, int sub) { return sub_first(n, parts, sub + 1) - sub_first(n, parts, sub); }
constexpr int sub_pieces(int n, int parts, int sub) { return (sub_taps(n, parts, sub) + 3) / 4; }
constexpr int piece_at(int taps, int piece) { return 4 * piece + 4 <= taps ? 4 * piece : taps - 4; }  // within the stage
// One part, odd n: a channel's taps start in the middle of a dword half the time, and such loads keep the address unit
// busy for a multiple of the time that whole dwords take (it was busy 73% of the kernel's time, the matrix pipe 31%).
// Whole dwords are read and shifted, and a load is 16 bytes long so that there are half as many of them.  Pieces are of
// seven taps, the least that such a load holds.  (even n: taps start at whole dwords; pieces of 8 at n = 4 measured slower,
// 58 -> 65 us on [26,388->72,21x54].)
constexpr int long_piece(int n) { return n % 2 ? 7 : 4; }
constexpr int long_pieces(int n) { return (n * n + long_piece(n) - 1) / long_piece(n); }
constexpr int long_piece_at(int n, int piece)
{
    return long_piece(n) * (piece + 1) <= n * n ? long_piece(n) * piece : n * n - long_piece(n);
}
constexpr int max_taps(int n, int parts) { return parts == 1 ? n * n : 4 + n * n % 4; }
constexpr int max_pieces(int n, int parts) { return (max_taps(n, parts) + 3) / 4; }
// LDS image of one part of a weight stage: 16-byte slots [channel half][tap][output channel], with strides
// that spread the staging lanes over the banks: three parts, a wave writes 8 channels x 8 dwords of one
// tap (halves 8 slots apart modulo 16); one part, 16-byte slots of pieces, halves and output channels
// (pieces 4, halves 2 apart modulo 16).  The slots between the halves take what has no place.
constexpr int w_tap_slots(int parts, int tm) { return parts == 3 ? tm : tm + 1; }
constexpr int w_half_slots(int n, int parts, int tm)
{
    const int used = max_taps(n, parts) * w_tap_slots(parts, tm), want = parts == 3 ? 8 : 2;
    return used + 1 + (want + 31 - used % 16) % 16;
}

// One part: the taps in the order of their window positions, so that the activations of a position are read once
// (n = 5: 43 fragments of 50 MFMAs instead of 55); the i-th tap of that order, and the number of taps before position (pa, pb)
template <int N, bool AL>
constexpr int tap_in_order(int i)
{
    for (int p = 0; p < 64; ++p)
        for (int tap = 0; tap < N * N; ++tap)
            if (pos_of<AL>(tap / N) * 8 + pos_of<AL>(tap % N) == p && i-- == 0) return tap;
    return 0;
}

template <int N, bool AL>
constexpr int pos_in_order(int i) { return pos_of<AL>(tap_in_order<N, AL>(i) / N) * 8 + pos_of<AL>(tap_in_order<N, AL>(i) % N); }
template <int N, bool AL>
constexpr int positions_until(int i)  // changes of position up to the i-th tap
{
    int k = 0;
    for (int j = 1; j <= i; ++j) k += pos_in_order<N, AL>(j) != pos_in_order<N, AL>(j - 1);
    return k;
}
// f(integral_constant<int, 0>) .. f(integral_constant<int, N - 1>): constants before the loops are unrolled
template <int N, class F>
__device__ __forceinline__ void in_turn(F&& f)
{
    if constexpr (N > 0) {
        in_turn<N - 1>(f);
        f(std::integral_constant<int, N - 1>{});
    }
}

// CW x QW waves: block tile = 32*CW channels x 32*NT*QW quads; a wave owns 32 channels x 32*NT quads x 4 classes.
// XU: staging units of activations per thread.  EPI / OUT16 as in the other kernels.
template <int N, int CW, int QW, int NT, int XU, bool AL, bool EPI, typename TIn, bool OUT16>
__global__ __launch_bounds__(64 * CW * QW) __attribute__((amdgpu_waves_per_eu(2, 2)))
void ukst_mfma_f32_kernel_parts(const TIn* __restrict__ x, const TIn* __restrict__ w, void* __restrict__ y,
                                PartsArgs a, Epilogue ep)
{
    constexpr int PARTS = sizeof(TIn) == 4 ? 3 : 1;
    constexpr int ES = (int)sizeof(TIn);
    constexpr int T = 64 * CW * QW;      // threads
    constexpr int TM = 32 * CW, TN = 32 * NT * QW;
    constexpr int NN = N * N;
    constexpr int NSUB = sub_count(N, PARTS);   // weight stages per 16 channels
    constexpr int WTS = w_tap_slots(PARTS, TM) * 16, WHS = w_half_slots(N, PARTS, TM) * 16;
    constexpr int WPL = 2 * WHS;                // bytes of one part's weight stage
    constexpr int WBUF = PARTS * WPL;
    constexpr int UK = PARTS == 3 ? 2 : 8;      // input channels of a weight unit
    constexpr int UPC = KC / UK;                // weight units per (output channel, piece)
    constexpr int WCG = PARTS == 3 ? (TM * UPC + T - 1) / T : 1;  // (groups of output channels per thread)
    constexpr int WU = PARTS == 3 ? WCG * max_pieces(N, PARTS) : (TM * UPC * long_pieces(N) + T - 1) / T;
    // (WU: weight units per thread)
    constexpr int PX = PARTS == 3 ? 1 : 4;      // pixels of an activation unit
    constexpr int XS_OFF = 2 * WBUF;
    typedef PartProducts<PARTS> PP;
    extern __shared__ __align__(16) unsigned char lds[];

    const GeomBase& g = a.g;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int cw = wave % CW, qw = wave / CW;
    const int l32 = lane & 31, gk = lane >> 5;
    const int KHW = a.KHq * a.KWq;

    const int bid_all = xcd_contiguous(blockIdx.x, gridDim.x);
    const int ks = bid_all % a.ksplit, bid = bid_all / a.ksplit;
    const int cb = a.cb_major ? bid / a.nqt : bid % a.nco;
    const int qt = a.cb_major ? bid % a.nqt : bid / a.nco;
    const int co0 = cb * TM, q0 = qt * TN;
    const int q_last = (q0 + TN - 1 < a.Q ? q0 + TN - 1 : a.Q - 1);
    // quad row rho = b*KHq + kk uses input rows e = b*EH + kk + pa
    const int bf0 = fdiv(q0, a.dKHW), kf0 = fdiv(q0 - bf0 * KHW, a.dKW);
    const int e_first = bf0 * a.EH + kf0;

    // ---- zero the activation stage once: halo columns are never written again
    for (int i = tid; i < PARTS * a.XPL / 16; i += T)
        *reinterpret_cast<u4v_t*>(lds + XS_OFF + i * 16) = u4v_t{0u, 0u, 0u, 0u};

    // (FUNNEL_X: activations of odd images are read in whole dwords too, and shifted.  Not where a thread has two units:
    // there are no registers for it (weights fetched eight taps later to make room: 119 -> 132 us on [16,200->72,93x61]); nor
    // at n = 2, whose few MFMAs per unit wait for memory: 62 us without, 64 with it
    // on [1,649->208,34x34].  Neither shifted, weights only, both, at n = 5: [16,200->72,93x61]
    // 143, 123, 119 us; [12,256->56,80x80] 106, 94, 89; [32,256->128,128x128] 1180, 1077, 1030)
    constexpr bool FUNNEL_X = PARTS == 1 && XU == 1 && N > 2;
    const int x_low = FUNNEL_X ? (int)((uintptr_t)x & 2) : 0;
    const size_t x_bytes = (size_t)g.B * g.Cin * g.H * g.W * ES;
    const __amdgpu_buffer_rsrc_t rs_x = __builtin_amdgcn_make_buffer_rsrc(
        (void*)((const char*)x - x_low), 0, (int)(FUNNEL_X ? (x_low + x_bytes + 3) & ~(size_t)3 : x_bytes), kRawBuffer);
    const int x_odd = FUNNEL_X && g.H * g.W % 2 ? 2 : 0;  // bytes by which an odd channel starts past a dword
    // (FUNNEL: w is read in whole dwords; the first and the last of them may hold two bytes of something else)
    constexpr bool FUNNEL = PARTS == 1 && N % 2;
    constexpr int PT = PARTS == 3 ? 4 : long_piece(N);  // taps of a weight unit
    const int w_low = FUNNEL ? (int)((uintptr_t)w & 2) : 0;
    const size_t w_bytes = (size_t)g.Cout * g.Cin * NN * ES;
    const __amdgpu_buffer_rsrc_t rs_w = __builtin_amdgcn_make_buffer_rsrc(
        (void*)((const char*)w - w_low), 0, (int)(FUNNEL ? (w_low + w_bytes + 3) & ~(size_t)3 : w_bytes), kRawBuffer);
    const unsigned x_cstride = (unsigned)(g.H * g.W * ES);

    // ---- staging units.  Activations: (channel half, row, PX columns), columns fastest; the last unit of a
    // row whose length is no multiple of PX starts inside its neighbour
    unsigned x_goff[XU];
    int x_loff[XU];
#pragma unroll
    for (int j = 0; j < XU; ++j) {
        const int e = tid + T * j;
        const int h = fdiv(e, a.dRW);
        const int rem = e - h * (a.ROWS * a.CPR);
        const int row = fdiv(rem, a.dW), c = rem - row * a.CPR;
        const int col = PX * c + PX <= g.W ? PX * c : g.W - PX;
        x_goff[j] = kNoByte;
        x_loff[j] = -1;
        if (h < 2) {
            const int er = e_first + row;
            const int b = fdiv(er, a.dEH), i = er - b * a.EH - (g.P >> 1);
            if (b < g.B && i >= 0 && i < g.H)
                x_goff[j] = (unsigned)((((b * g.Cin + 8 * h) * g.H + i) * g.W + col) * ES) + x_low;
            x_loff[j] = XS_OFF + ((h * a.ROWS + row) * a.LWX + a.SH + col) * 16;
        }
    }
    // weights.  Three parts: the thread's unit j is (output channel tid/8 + (j % WCG)*T/8, two input channels,
    // piece j / WCG), every unit exists; channels past the last output channel lie past the end of w and
    // arrive as zeros.  One part: unit tid + T*j = (output channel, eight input channels, piece), piece
    // fastest; units that do not exist read nothing and write to a pad slot.
    int w_goff[PARTS == 3 ? 1 : WU], w_loff[PARTS == 3 ? 1 : WU];
    if constexpr (PARTS == 3) {
        const int cg = tid % UPC, co = tid / UPC;
        w_goff[0] = (((co0 + co) * g.Cin + UK * cg) * NN) * ES;
        w_loff[0] = (UK * cg >> 3) * WHS + co * 16 + (UK * cg & 7) * 2;
        if (TM * UPC < T && co >= TM) w_goff[0] = (int)kNoByte;  // (TM = 32 on 8 waves)
    } else {
#pragma unroll
        for (int j = 0; j < WU; ++j) {
            constexpr int pieces = long_pieces(N);
            const int e = tid + T * j;
            const int t = e / pieces, tap = long_piece_at(N, e - t * pieces);
            const int cg = t % UPC, co = t / UPC;
            w_goff[j] = co < TM && co0 + co < g.Cout ? (((co0 + co) * g.Cin + UK * cg) * NN + tap) * ES + w_low : (int)kNoByte;
            w_loff[j] = co < TM ? cg * WHS + tap * WTS + co * 16 : -1;
        }
    }
    const int w_gstep = T / UPC * g.Cin * NN * ES;
    // raw registers of the stage being fetched: UK (8) values of PT taps (PX pixels) per unit
    constexpr int WD = PARTS == 1 && N % 2 == 0 ? 2 : 4, XD = PARTS == 3 ? 1 : FUNNEL_X ? 3 : 2;  // dwords per load
    unsigned xr[XU][8][XD], wr[WU][UK][WD];
    auto load_x = [&](int s) {
#pragma unroll
        for (int j = 0; j < XU; ++j)
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const unsigned soff = (unsigned)(s * KC + k) * x_cstride;
                if constexpr (FUNNEL_X) {
                    const int odd = k & 1 ? x_odd : 0;
                    const u3v_t v = __builtin_amdgcn_raw_buffer_load_b96(rs_x, (x_goff[j] + odd) & ~3u, soff - odd, 0);
#pragma unroll
                    for (int i = 0; i < 3; ++i) xr[j][k][i] = v[i];
                } else if constexpr (XD == 1) {
                    xr[j][k][0] = __builtin_amdgcn_raw_buffer_load_b32(rs_x, x_goff[j], soff, 0);
                } else {
                    const u2v_t v = __builtin_amdgcn_raw_buffer_load_b64(rs_x, x_goff[j], soff, 0);
                    xr[j][k][0] = v.x;
                    xr[j][k][1] = v.y;
                }
            }
    };
    auto w_units = [&](int sub) { return PARTS == 3 ? WCG * sub_pieces(N, PARTS, sub) : WU; };
    auto load_w = [&](int s, int sub) {
#pragma unroll
        for (int j = 0; j < w_units(sub); ++j) {
            const int tap0 = PARTS == 3 ? sub_first(N, PARTS, sub) + piece_at(sub_taps(N, PARTS, sub), j / WCG) : 0;
#pragma unroll
            for (int k = 0; k < UK; ++k) {
                unsigned voff = (unsigned)(PARTS == 3 ? w_goff[0] + (j % WCG) * w_gstep : w_goff[j]);
                unsigned soff = (unsigned)(((s * KC + k) * NN + tap0) * ES);
                if constexpr (FUNNEL) {
                    // an odd channel starts two bytes past a dword of its own where an even one does not, and the
                    // other way round: the dwords that hold the taps are read, and align_w shifts them
                    voff = (voff + 2 * (k & 1)) & ~3u;
                    soff -= 2 * (k & 1);
                }
                if constexpr (WD == 4) {
                    const u4v_t v = __builtin_amdgcn_raw_buffer_load_b128(rs_w, voff, soff, 0);
#pragma unroll
                    for (int i = 0; i < 4; ++i) wr[j][k][i] = v[i];
                } else {
                    const u2v_t v = __builtin_amdgcn_raw_buffer_load_b64(rs_w, voff, soff, 0);
                    wr[j][k][0] = v.x;
                    wr[j][k][1] = v.y;
                }
            }
        }
    };
    // registers -> LDS.  A stage that reaches past the last input channel holds zeros there (what was
    // loaded for them belongs to another image or output channel)
    auto trim_w = [&](int s, int sub) {
        if (s * KC + KC <= g.Cin) return;
#pragma unroll
        for (int j = 0; j < w_units(sub); ++j)
#pragma unroll
            for (int k = 0; k < UK; ++k) {
                int e = tid + (PARTS == 3 ? 0 : T * j);
                asm("" : "+v"(e));
                const int cg = PARTS == 3 ? e % UPC : e / long_pieces(N) % UPC;
                const bool in = s * KC + UK * cg + k < g.Cin;
#pragma unroll
                for (int i = 0; i < WD; ++i) wr[j][k][i] = in ? wr[j][k][i] : 0u;
            }
    };
    auto align_w = [&]() {  // odd n: the taps of a unit from the start of its registers on
        if constexpr (FUNNEL) {
#pragma unroll
            for (int j = 0; j < WU; ++j)
#pragma unroll
                for (int k = 0; k < UK; ++k) {
                    const unsigned sh = (unsigned)((w_goff[j] + 2 * (k & 1)) & 2) * 8;
#pragma unroll
                    for (int i = 0; i < 3; ++i) wr[j][k][i] = __builtin_amdgcn_alignbit(wr[j][k][i + 1], wr[j][k][i], sh);
                    wr[j][k][3] >>= sh;
                }
        }
    };
    auto store_w_tap = [&](int sub, int buf, int t) {  // tap t of every unit's piece
#pragma unroll
        for (int j = 0; j < w_units(sub); ++j) {
            if constexpr (PARTS == 3) {
                unsigned char* const dst = lds + buf * WBUF + w_loff[0] + (j % WCG) * (T / UPC * 16) +
                                           (piece_at(sub_taps(N, PARTS, sub), j / WCG) + t) * WTS;
                if (TM * UPC < T && wave >= TM * UPC / 64) continue;  // uniform
                unsigned p[3];
                split_pair(__uint_as_float(wr[j][0][t]), __uint_as_float(wr[j][1][t]), p[0], p[1], p[2]);
#pragma unroll
                for (int i = 0; i < 3; ++i) *reinterpret_cast<unsigned*>(dst + i * WPL) = p[i];
            } else {
                u4v_t v;
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    v[i] = __builtin_amdgcn_perm(wr[j][2 * i + 1][t >> 1], wr[j][2 * i][t >> 1],
                                                 (t & 1) ? 0x07060302u : 0x05040100u);
                *reinterpret_cast<u4v_t*>(lds + buf * WBUF + (w_loff[j] < 0 ? WHS - 16 : w_loff[j] + t * WTS)) = v;
            }
        }
    };
    u4v_t xp[XU][PARTS * PX];
    auto trim_x = [&](int s) {
        if (s * KC + KC <= g.Cin) return;
#pragma unroll
        for (int j = 0; j < XU; ++j) {
            int e = tid + T * j;
            asm("" : "+v"(e));  // (worked out here, once per call, and not kept across the loop: registers are short)
            const int h = fdiv(e, a.dRW);
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const bool in = s * KC + 8 * h + k < g.Cin;
#pragma unroll
                for (int i = 0; i < XD; ++i) xr[j][k][i] = in ? xr[j][k][i] : 0u;
            }
        }
    };
    auto align_x = [&]() {
        if constexpr (FUNNEL_X) {
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const unsigned sh = ((x_goff[0] + (k & 1 ? x_odd : 0)) & 2) * 8;
#pragma unroll
                for (int i = 0; i < 2; ++i) xr[0][k][i] = __builtin_amdgcn_alignbit(xr[0][k][i + 1], xr[0][k][i], sh);
            }
        }
    };
    auto pack_x = [&](int i) {  // items 0 .. 4*XU - 1
        const int j = i >> 2, q = i & 3;
        if constexpr (PARTS == 3) {
            unsigned p0, p1, p2;
            split_pair(__uint_as_float(xr[j][2 * q][0]), __uint_as_float(xr[j][2 * q + 1][0]), p0, p1, p2);
            xp[j][0][q] = p0;
            xp[j][1][q] = p1;
            xp[j][2][q] = p2;
        } else {
#pragma unroll
            for (int k = 0; k < 4; ++k)
                xp[j][q][k] = __builtin_amdgcn_perm(xr[j][2 * k + 1][q >> 1], xr[j][2 * k][q >> 1],
                                                    (q & 1) ? 0x07060302u : 0x05040100u);
        }
    };
    auto store_x = [&]() {
#pragma unroll
        for (int j = 0; j < XU; ++j)
            if (x_loff[j] >= 0) {
#pragma unroll
                for (int i = 0; i < PARTS * PX; ++i)
                    *reinterpret_cast<u4v_t*>(lds + (PARTS == 3 ? i * a.XPL : i * 16) + x_loff[j]) = xp[j][i];
            }
    };

    // ---- operand positions of this lane
    const int a_lds = gk * WHS + (cw * 32 + l32) * 16;
    int b_lds[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        int q = q0 + (qw * NT + nt) * 32 + l32;
        if (q > q_last) q = q_last;
        const int b = fdiv(q, a.dKHW);
        const int rem = q - b * KHW;
        const int kk = fdiv(rem, a.dKW), mm = rem - kk * a.KWq;
        b_lds[nt] = XS_OFF + ((gk * a.ROWS + b * a.EH + kk - e_first) * a.LWX + mm) * 16;
    }

    f32x16_t acc[NT][2][2];  // [quad group][row class][column class]
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[nt][c >> 1][c & 1][i] = 0.f;

    // One weight stage (sub is a constant once unrolled), with the staging of the next ones dealt out
    // between its MFMAs: two waves that share a SIMD get through their MFMAs side by side, so whatever is
    // left for the end is left for both and finds the matrix pipe idle.
    //   weights: the next stage's registers go to the other buffer under taps 1 and 2 and are refilled at once for
    //     the stage after it (one part: fetched before the first tap, written under the second half of them)
    //   activations of the next 16 channels: fetched before, split under the last tap of their last stage
    const int s0 = ks * a.kstages;
    const int nstages = (g.Cin + KC - 1) / KC;
    const int s1 = s0 + a.kstages < nstages ? s0 + a.kstages : nstages;
    auto stage_after = [&](int s, int sub, int d) {  // (the last stages fetch the last one again: unused)
        const int r = s + (sub + d) / NSUB;
        return r < s1 ? r : s1 - 1;
    };
    auto compute = [&](int buf, int s, int sub) {
        const unsigned char* const wb = lds + buf * WBUF + a_lds;
        const int taps = sub_taps(N, PARTS, sub);
        const int s_w = stage_after(s, sub, 1), sub_w = (sub + 1) % NSUB;
        bf16x8_t bf[NT][PARTS];
        int have = -1;
        if (sub + 1 == NSUB) load_x(stage_after(s, sub, 1));
#pragma unroll
        for (int t = 0; t < taps; ++t) {
            const int tap = sub_first(N, PARTS, sub) + t, tr = tap / N, tc = tap % N;
            const int pa = pos_of<AL>(tr), pb = pos_of<AL>(tc);
            __builtin_amdgcn_sched_barrier(0);
            bf16x8_t af[PARTS];
#pragma unroll
            for (int i = 0; i < PARTS; ++i) af[i] = *reinterpret_cast<const bf16x8_t*>(wb + i * WPL + t * WTS);
            if (pa * 8 + pb != have) {
                have = pa * 8 + pb;
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                    for (int i = 0; i < PARTS; ++i)
                        bf[nt][i] = *reinterpret_cast<const bf16x8_t*>(lds + b_lds[nt] + i * a.XPL + pa * a.LWX * 16 +
                                                                       pb * 16);
            }
            if (t == 1) trim_w(s_w, sub_w);
            if (t + 1 == taps && sub + 1 == NSUB) trim_x(stage_after(s, sub, 1));
#pragma unroll
            for (int m = 0; m < PP::count; ++m) {
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
                    acc[nt][tr & 1][tc & 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                        af[PP::a[m]], bf[nt][PP::b[m]], acc[nt][tr & 1][tc & 1], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
                if ((t == 1 || t == 2) && (m == 1 || m == 3)) store_w_tap(sub_w, buf ^ 1, 2 * (t - 1) + m / 2);
                if (t == 2 && m == 4) load_w(stage_after(s, sub, 2), (sub + 2) % NSUB);
                if (t + 1 == taps && sub + 1 == NSUB) {
#pragma unroll
                    for (int i = m * 4 * XU / 6; i < (m + 1) * 4 * XU / 6; ++i) pack_x(i);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    };

    // One part: a tap is only NT MFMAs, and a wave issues in order, so reading a tap's fragments right before them
    // left the matrix pipe waiting for LDS at every tap.  Here a tap's fragments are read while the tap before it is
    // multiplied, and the taps go by window position, so that the activations are read once per position.
    // [16,200->72,93x61] n=5 ragged bf16 152 -> 143 us; [26,388->72,21x54] n=4 68 -> 58; [64,128->64,33x33] n=4
    // 50 -> 45; [32,256->128,128x128] n=5 1287 -> 1180.
    auto compute1 = [&](int buf, int s) {
        const unsigned char* const wb = lds + buf * WBUF + a_lds;
        const int s_w = stage_after(s, 0, 1);
        bf16x8_t af[2], bf[2][NT];
        auto fetch = [&](auto ic) {
            constexpr int i = decltype(ic)::value, tap = tap_in_order<N, AL>(i), pos = pos_in_order<N, AL>(i);
            constexpr int p = positions_until<N, AL>(i) & 1, before = pos_in_order<N, AL>(i > 0 ? i - 1 : 0);
            af[i & 1] = *reinterpret_cast<const bf16x8_t*>(wb + tap * WTS);
            if constexpr (i == 0 || pos != before) {
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
                    bf[p][nt] =
                        *reinterpret_cast<const bf16x8_t*>(lds + b_lds[nt] + (pos >> 3) * a.LWX * 16 + (pos & 7) * 16);
            }
        };
        fetch(std::integral_constant<int, 0>{});
        load_x(s_w);
        load_w(s_w, 0);
        in_turn<NN>([&](auto ic) {
            constexpr int i = decltype(ic)::value, tap = tap_in_order<N, AL>(i), tr = tap / N, tc = tap % N;
            constexpr int p = positions_until<N, AL>(i) & 1;
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (i + 1 < NN) fetch(std::integral_constant<int, i + 1>{});
            if (i == NN / 2) {
                trim_w(s_w, 0);
                align_w();
            }
            if (i + 1 == NN) {
                trim_x(s_w);
                align_x();
            }
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
                acc[nt][tr & 1][tc & 1] =
                    __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[i & 1], bf[p][nt], acc[nt][tr & 1][tc & 1], 0, 0, 0);
            // weights: tap k of the pieces under tap NN/2 + k*(NN - NN/2)/PT; activations under the last one
#pragma unroll
            for (int k = 0; k < PT; ++k)
                if (i == NN / 2 + k * (NN - NN / 2) / PT) store_w_tap(0, buf ^ 1, k);
            if (i + 1 == NN) {
#pragma unroll
                for (int k = 0; k < 4 * XU; ++k) pack_x(k);
            }
        });
        __builtin_amdgcn_sched_barrier(0);
    };
    load_w(s0, 0);
    load_x(s0);
    __syncthreads();  // zero fill done before the first activation writes
    trim_w(s0, 0);
    align_w();
#pragma unroll
    for (int t = 0; t < PT; ++t) store_w_tap(0, 0, t);
    trim_x(s0);
    align_x();
#pragma unroll
    for (int i = 0; i < 4 * XU; ++i) pack_x(i);
    store_x();
    if constexpr (PARTS == 3) load_w(stage_after(s0, 0, 1), 1 % NSUB);
    __syncthreads();
    int buf = 0;
    for (int s = s0; s < s1; ++s) {
#pragma unroll
        for (int sub = 0; sub < NSUB; ++sub) {
            // addresses are worked out again in every weight stage: hoisted out of the loop, one per (part,
            // window row, tap run), they would push the accumulators out of the register file
            #pragma unroll
            for (int nt = 0; nt < NT; ++nt) asm("" : "+v"(b_lds[nt]));
            if constexpr (PARTS == 3) compute(buf, s, sub);
            else compute1(buf, s);
            __syncthreads();
            buf ^= 1;
        }
        store_x();
        __syncthreads();
    }

    // ---- results
    constexpr int OS = OUT16 ? 2 : 4;
    const size_t ybytes = (size_t)g.B * g.Cout * g.OH * g.OW * OS;
    unsigned char* const yb = (unsigned char*)y + (size_t)ks * a.copy_bytes;

    // accumulator register i of a tile holds channel 8*(i/4) + 4*gk + (i%4) of the wave's 32, for the
    // lane's quad; the two column classes of a quad are neighbours in memory
    const __amdgpu_buffer_rsrc_t rs_y = __builtin_amdgcn_make_buffer_rsrc((void*)yb, 0, (int)ybytes, kRawBuffer);
    const unsigned plane = (unsigned)(g.OH * g.OW * OS);
    const int co_w = co0 + cw * 32 + 4 * gk;  // channel of register 0
    auto drain = [&](auto act_tag) {
        constexpr int ACT = decltype(act_tag)::value;  // -1: no epilogue at all
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            const int q = q0 + (qw * NT + nt) * 32 + l32;
            const bool qv = q <= q_last;
            const int qq = qv ? q : q_last;
            const int b = fdiv(qq, a.dKHW);
            const int rem = qq - b * KHW;
            const int kk = fdiv(rem, a.dKW), mm = rem - kk * a.KWq;
            // first row / column of the quad in the output (-1 where only the second one exists)
            const int oy = AL ? 2 * kk : 2 * (g.k_min + kk) - 1 - g.P;
            const int ox = AL ? 2 * mm : 2 * (g.m_min + mm) - 1 - g.P;
            const bool c0v = ox >= 0, c1v = ox + 1 < g.OW;
            const unsigned y_off = (unsigned)(((b * g.Cout + co_w) * g.OH + oy) * g.OW + ox) * (unsigned)OS;
#pragma unroll
            for (int rr = 0; rr < 2; ++rr) {
                const bool vrow = qv && oy + rr >= 0 && oy + rr < g.OH;
                const unsigned base = y_off + (unsigned)(rr * g.OW * OS);
                const unsigned off_pair = vrow && c0v && c1v ? base : kNoByte;
                const bool only0 = vrow && c0v && !c1v, only1 = vrow && !c0v && c1v;
                const unsigned off_edge = only0 ? base : only1 ? base + (unsigned)OS : kNoByte;
                const bool any_edge = !AL && __builtin_amdgcn_ballot_w64(only0 || only1) != 0;
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const int ch = 8 * (i / 4) + (i % 4);
                    if (co0 + cw * 32 + ch >= g.Cout) continue;  // uniform
                    const bool chv = co_w + ch < g.Cout;         // (the upper four of a partial group of 8)
                    const unsigned soff = (unsigned)ch * plane;
                    // shifted quads hold class 1 in their first row / column
                    float v0 = AL ? acc[nt][rr][0][i] : acc[nt][1 - rr][1][i];
                    float v1 = AL ? acc[nt][rr][1][i] : acc[nt][1 - rr][0][i];
                    if constexpr (PARTS == 3) {
                        v0 *= kPartsDown;
                        v1 *= kPartsDown;
                    }
                    if constexpr (ACT >= 0) {
                        const float bv = ep.bias ? ep.bias[chv ? co_w + ch : 0] : 0.f;
                        v0 = epilogue_t<ACT>(v0, bv);
                        v1 = epilogue_t<ACT>(v1, bv);
                    }
                    const unsigned op = chv ? off_pair : kNoByte, oe = chv ? off_edge : kNoByte;
                    if constexpr (OUT16) {
                        const unsigned bits = pack_bf16(v0, v1);
                        __builtin_amdgcn_raw_buffer_store_b32(bits, rs_y, op, soff, 0);
                        if (any_edge)
                            __builtin_amdgcn_raw_buffer_store_b16((short)(only0 ? bits & 0xFFFFu : bits >> 16), rs_y, oe,
                                                                  soff, 0);
                    } else {
                        u2v_t d;
                        d.x = __float_as_uint(v0);
                        d.y = __float_as_uint(v1);
                        __builtin_amdgcn_raw_buffer_store_b64(d, rs_y, op, soff, 0);
                        if (any_edge)
                            __builtin_amdgcn_raw_buffer_store_b32(only0 ? d.x : d.y, rs_y, oe, soff, 0);
                    }
                }
            }
        }
    };
    if constexpr (EPI) with_activation(ep.act, drain);
    else drain(std::integral_constant<int, -1>{});

    float most = 0.f;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int c = 0; c < 4; ++c) most = peak(acc[nt][c >> 1][c & 1], most);
    if (!__syncthreads_or(most < __builtin_inff() ? 0 : 1)) return;
    // tiles that hold a sum that is not finite (ukst_parts.h)
    unsigned tiles[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        tiles[nt] = 0u;
#pragma unroll
        for (int c = 0; c < 4; ++c)
            if (!wave_finite(acc[nt][c >> 1][c & 1])) tiles[nt] |= 1u << c;
    }
    if (tid == 0) *reinterpret_cast<unsigned*>(lds) = 0u;
    __syncthreads();
    const int ci0 = s0 * KC, ci1 = s1 * KC < g.Cin ? s1 * KC : g.Cin;
    const unsigned w_cstride = NN * ES;
    const size_t planes = (size_t)g.OH * g.OW;
    // the class's place of quad q in channel 0 of y (and image, row, column of the quad); false if there is none
    auto place = [&](int q, int cls, size_t& o, int& b, int& kk, int& mm) {
        b = fdiv(q, a.dKHW);
        const int rem = q - b * KHW;
        kk = fdiv(rem, a.dKW);
        mm = rem - kk * a.KWq;
        const int oy = AL ? 2 * kk + (cls >> 1) : 2 * (g.k_min + kk) - (cls >> 1) - g.P;
        const int ox = AL ? 2 * mm + (cls & 1) : 2 * (g.m_min + mm) - (cls & 1) - g.P;
        o = ((size_t)b * g.Cout * g.OH + oy) * g.OW + ox;
        return oy >= 0 && oy < g.OH && ox >= 0 && ox < g.OW;
    };
    auto put = [&](size_t o, int ch, float v) {
        if (ch >= g.Cout) return;
        if constexpr (EPI) v = epilogue(v, ep.bias ? ep.bias[ch] : 0.f, ep.act);
        if constexpr (OUT16) ((uint16_t*)yb)[o + ch * planes] = __builtin_bit_cast(uint16_t, (__bf16)v);
        else ((float*)yb)[o + ch * planes] = v;
    };
    // Group: (class, four channels, quad) of the block's outputs.  The four classes of 32 quads together: a lane's
    // weights, which lie in as many cache lines as there are lanes, come four taps to a load
#pragma unroll 1
    for (int nt = 0; nt < NT; ++nt) {
        const unsigned todo = NT > 1 && nt == 1 ? tiles[NT - 1] : tiles[0];
        if (todo == 0u) continue;
        const int ql = (qw * NT + nt) * 32 + l32;
        const bool on = q0 + ql <= q_last;
        size_t o;
        int b, kk, mm;
        place(on ? q0 + ql : q_last, 0, o, b, kk, mm);
        const int ch = co0 + cw * 32 + l32 < g.Cout ? co0 + cw * 32 + l32 : g.Cout - 1;
        const unsigned wo = (unsigned)((ch * g.Cin + gk) * NN * ES);
        constexpr int W = pos_of<AL>(N - 1) + 1;  // window side
        unsigned xo[W][W];
        bool halo = false;
#pragma unroll
        for (int pa = 0; pa < W; ++pa)
#pragma unroll
            for (int pb = 0; pb < W; ++pb) {
                const int i = kk + pa - (g.P >> 1), j = mm + pb - (g.P >> 1);
                const bool in = on && i >= 0 && i < g.H && j >= 0 && j < g.W;
                halo = halo || !in;
                xo[pa][pb] = in ? (unsigned)((((b * g.Cin + gk) * g.H + i) * g.W + j) * ES) : kNoByte;
            }
        f32x16_t sum[4];
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int i = 0; i < 16; ++i) sum[c][i] = 0.f;
#pragma unroll 1
        for (int ci = ci0; ci < ci1; ci += 2) {
            if (wave_nan(sum[0]) && wave_nan(sum[1]) && wave_nan(sum[2]) && wave_nan(sum[3])) break;
            const bool in = ci + gk < ci1;
            float wv[NN], xv[W][W];
#pragma unroll
            for (int p = 0; p < (NN + 3) / 4; ++p) {
                const unsigned soff = (unsigned)((ci * NN + piece_at(NN, p)) * ES);
                if constexpr (ES == 4) {
                    const u4v_t v = __builtin_amdgcn_raw_buffer_load_b128(rs_w, in ? wo : kNoByte, soff, 0);
#pragma unroll
                    for (int t = 0; t < 4; ++t) wv[piece_at(NN, p) + t] = __uint_as_float(v[t]);
                } else {
                    const u2v_t v = __builtin_amdgcn_raw_buffer_load_b64(rs_w, in ? wo : kNoByte, soff, 0);
#pragma unroll
                    for (int t = 0; t < 4; ++t)
                        wv[piece_at(NN, p) + t] = __uint_as_float(t & 1 ? v[t >> 1] & 0xFFFF0000u : v[t >> 1] << 16);
                }
            }
#pragma unroll
            for (int pa = 0; pa < W; ++pa)
#pragma unroll
                for (int pb = 0; pb < W; ++pb) xv[pa][pb] = load_f32<TIn>(rs_x, in ? xo[pa][pb] : kNoByte, ci * x_cstride);
#pragma unroll
            for (int tap = 0; tap < NN; ++tap) {
                const int ta = tap / N, tc = tap % N, c = 2 * (ta & 1) + (tc & 1);
                sum[c] = __builtin_amdgcn_mfma_f32_32x32x2f32(wv[tap], xv[pos_of<AL>(ta)][pos_of<AL>(tc)], sum[c], 0, 0, 0);
            }
        }
#pragma unroll
        for (int c = 0; c < 4; ++c)
            if ((todo >> c & 1) && place(on ? q0 + ql : q_last, c, o, b, kk, mm) && on)
                put_tile(lds, sum[c], halo, [&](int i, float v) { put(o, co0 + cw * 32 + 8 * (i / 4) + 4 * gk + i % 4, v); },
                         [&](int i) { return (c * (TM / 4) + cw * 8 + 2 * i + gk) * TN + ql; });
    }
    __threadfence();  // what was stored lies in memory before it is stored again
    __syncthreads();
    const int listed = *reinterpret_cast<const int*>(lds);
    for (int e = tid; e < listed; e += T) {
        const int group = reinterpret_cast<const unsigned short*>(lds + 16)[e];
        const int cbase = co0 + group / TN % (TM / 4) * 4, cls = group / (TN * (TM / 4));
        if (cbase >= g.Cout) continue;
        size_t o;
        int b, kk, mm;
        place(q0 + group % TN, cls, o, b, kk, mm);
        float sum[4] = {0.f, 0.f, 0.f, 0.f};
        for (int ta = cls >> 1; ta < N; ta += 2) {
            const int i = kk + pos_of<AL>(ta) - (g.P >> 1);
            if (i < 0 || i >= g.H) continue;
            for (int tc = cls & 1; tc < N; tc += 2) {
                const int j = mm + pos_of<AL>(tc) - (g.P >> 1);
                if (j < 0 || j >= g.W) continue;
                unsigned wo[4];
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    wo[k] = (unsigned)(((cbase + k < g.Cout ? cbase + k : g.Cout - 1) * g.Cin * NN + ta * N + tc) * ES);
                sum_products<TIn>(sum, rs_x, (unsigned)(((b * g.Cin * g.H + i) * g.W + j) * ES), x_cstride, rs_w, wo,
                                  w_cstride, ci0, ci1);
            }
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) put(o, cbase + k, sum[k]);
    }
}

// tile configuration: cw x qw waves of 32 channels x 32*nt quads, xu activation units per thread
struct Config { int cw, qw, nt, xu; };

inline int weight_stage_bytes(int n, int parts, int cw) { return parts * 2 * w_half_slots(n, parts, 32 * cw) * 16; }

template <int N, int CW, int QW, int NT, int XU, bool AL, typename TIn, bool OUT16>
hipError_t launch_c(const PartsArgs& a, const Epilogue& ep, const void* x, const void* w, void* y, hipStream_t stream)
{
    constexpr size_t list = redo_bytes(32 * CW * 32 * NT * QW);
    size_t lds = 2 * (size_t)weight_stage_bytes(N, sizeof(TIn) == 4 ? 3 : 1, CW) +
                 (size_t)(sizeof(TIn) == 4 ? 3 : 1) * a.XPL;
    if (lds < list) lds = list;
    typedef void (*kernel_t)(const TIn*, const TIn*, void*, PartsArgs, Epilogue);
    const kernel_t kfn = has_epilogue(ep) ? ukst_mfma_f32_kernel_parts<N, CW, QW, NT, XU, AL, true, TIn, OUT16>
                                          : ukst_mfma_f32_kernel_parts<N, CW, QW, NT, XU, AL, false, TIn, OUT16>;
    const hipError_t e = hipFuncSetAttribute((const void*)kfn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kfn, dim3((unsigned)(a.nco * a.nqt * a.ksplit)), dim3(64 * CW * QW), lds, stream,
                       (const TIn*)x, (const TIn*)w, y, a, ep);
    return hipGetLastError();
}

template <int N, bool AL, typename TIn, bool OUT16>
hipError_t launch_n(const PartsArgs& a, const Config& c, const Epilogue& ep, const void* x, const void* w, void* y,
                    hipStream_t st)
{
#define UKST_PARTS_CASE(CW, QW, NT, XU)                          \
    if (c.cw == CW && c.qw == QW && c.nt == NT && c.xu == XU)    \
        return launch_c<N, CW, QW, NT, XU, AL, TIn, OUT16>(a, ep, x, w, y, st);
    if constexpr (sizeof(TIn) == 4) {
        UKST_PARTS_CASE(2, 4, 2, 2) UKST_PARTS_CASE(2, 4, 2, 3) UKST_PARTS_CASE(2, 4, 2, 4)
        UKST_PARTS_CASE(2, 4, 1, 2) UKST_PARTS_CASE(2, 4, 1, 4)
        UKST_PARTS_CASE(1, 4, 2, 2) UKST_PARTS_CASE(1, 4, 2, 4) UKST_PARTS_CASE(1, 8, 2, 2) UKST_PARTS_CASE(1, 8, 2, 4)
    } else {
        UKST_PARTS_CASE(2, 4, 2, 1) UKST_PARTS_CASE(2, 4, 2, 2)
        UKST_PARTS_CASE(2, 4, 1, 1) UKST_PARTS_CASE(2, 4, 1, 2)
        UKST_PARTS_CASE(1, 4, 2, 1) UKST_PARTS_CASE(1, 4, 2, 2)
    }
#undef UKST_PARTS_CASE
    return hipErrorInvalidValue;
}

// every instance of one kernel side and operand type (one translation unit each: ukst_mfma_parts_*.hip)
template <int N, typename TIn>
hipError_t launch_side(const PartsArgs& a, const Config& c, const Epilogue& ep, const void* x, const void* w, void* y,
                       bool out16, hipStream_t st);

template <>
hipError_t launch_side<2, float>(const PartsArgs&, const Config&, const Epilogue&, const void*, const void*, void*,
                           bool, hipStream_t);
template <>
hipError_t launch_side<2, uint16_t>(const PartsArgs&, const Config&, const Epilogue&, const void*, const void*, void*,
                           bool, hipStream_t);
template <>
hipError_t launch_side<3, float>(const PartsArgs&, const Config&, const Epilogue&, const void*, const void*, void*,
                           bool, hipStream_t);
template <>
hipError_t launch_side<3, uint16_t>(const PartsArgs&, const Config&, const Epilogue&, const void*, const void*, void*,
                           bool, hipStream_t);
template <>
hipError_t launch_side<4, float>(const PartsArgs&, const Config&, const Epilogue&, const void*, const void*, void*,
                           bool, hipStream_t);
template <>
hipError_t launch_side<4, uint16_t>(const PartsArgs&, const Config&, const Epilogue&, const void*, const void*, void*,
                           bool, hipStream_t);
template <>
hipError_t launch_side<5, float>(const PartsArgs&, const Config&, const Epilogue&, const void*, const void*, void*,
                           bool, hipStream_t);
template <>
hipError_t launch_side<5, uint16_t>(const PartsArgs&, const Config&, const Epilogue&, const void*, const void*, void*,
                           bool, hipStream_t);

template <int N, typename TIn>
hipError_t launch_side_impl(const PartsArgs& a, const Config& c, const Epilogue& ep, const void* x, const void* w,
                            void* y, bool out16, hipStream_t st)
{
    if constexpr (sizeof(TIn) == 2) {
        if (out16) {
            if constexpr (N % 2 == 0) {
                if (a.g.P % 2 == 0) return launch_n<N, true, TIn, true>(a, c, ep, x, w, y, st);
            }
            return launch_n<N, false, TIn, true>(a, c, ep, x, w, y, st);
        }
    }
    if constexpr (N % 2 == 0) {
        if (a.g.P % 2 == 0) return launch_n<N, true, TIn, false>(a, c, ep, x, w, y, st);
    }
    return launch_n<N, false, TIn, false>(a, c, ep, x, w, y, st);
}

}  // namespace parts
}  // namespace ukst
