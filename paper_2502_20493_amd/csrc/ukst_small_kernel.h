// Layers of few tiles on the fp32 matrix pipe: one small tile per block, the sum over the input channels dealt to
// the block's waves.  Stride-2 forward layers, input gradients, stride-S and dilated layers; fp32 operands, or bf16
// operands widened (exactly) on their way into LDS; n = 2..5, any other size, element alignment only.
//
// All of them are the same product: output channel (row) m, lattice position p = (image, u, v), summed index k,
//     Y_c[m][p] = sum_k sum_{taps t of class c} A[m][k][t] * X[k][PS*(u, v) + window place of t]
//   shifted quads / stride S (KIND 0)  S*S classes, tap (a, b) belongs to class (a % S, b % S), window place (a / S, b / S)
//   output-aligned quads (KIND 1)      even n and P, stride 2: window place (a / 2 + a % 2, ...) as in ukst_mfma_f32.hip
//   input gradient (KIND 2)            one class, X = dy, positions two dy rows / columns apart (PS = 2)
//   dilation d (KIND 3)                one class; the d*d residues of the output coordinates are lattices of their own,
//                                      each a dense correlation on a sub-sampled map (Sec. 5's segregated input)
//
// What bounds it and why it looks like this.  Such layers are a long sum (hundreds of channels) over few outputs:
// a tile that fills a compute unit with 64 x 256 outputs leaves most of the chip idle and is one serial chain.  So the
// tile is the smallest that the matrix instructions take, 32 x 32 (or 16 x 16) outputs of every class, and the WV waves
// of a block split k: a wave owns every WV-th stage of KC channels, stages them in LDS of its own and multiplies them
// without a block barrier anywhere in the loop; two waves per SIMD cover each other's waits.  At the end the waves add
// their accumulators through LDS in wave order (bit-reproducible).  One launch, no workspace; given one, a forward layer
// of a few blocks and many stages is cut into slices of the stages over blocks, whose sums a second kernel adds in order.
// A wave fetches a stage's weights as they lie in memory, consecutive lanes 16 bytes each (the operand order would
// touch a cache line per lane: the address unit bounded that, 46.9 us for 64 images of 512 -> 256 channels, 4 x 4, n = 4,
// where this kernel takes 37 and its MFMAs alone 27),
// and the matrix operands are then single dwords from LDS, one or two per instruction of 64 (32) clocks.
// The halo needs no special case: a staged cell outside the map is a load that is out of range, which returns zero.
// Sums that are not finite and whose window reaches outside the map are taken again without the outside cells,
// whose zeros would make NaN of an infinite weight (likewise where a last stage repeats channels against zeros).
#pragma once
#include "ukst_internal.h"
#include <utility>

namespace ukst {
namespace small {

typedef float f4v_t __attribute__((ext_vector_type(4)));
typedef float f16v_t __attribute__((ext_vector_type(16)));
typedef unsigned u4v_t __attribute__((ext_vector_type(4)));
typedef unsigned u2v_t __attribute__((ext_vector_type(2)));

constexpr int kRaw = 0x00020000;           // raw 32-bit buffer, gfx9 family
constexpr unsigned kNone = 0xFFFFFF00u;    // byte offset that is out of range for any buffer

enum { kShifted = 0, kAligned = 1, kInputGrad = 2, kDilated = 3 };

struct SmallArgs {
    int B, K, M;              // images, summed channels, output channels
    int XH, XW, OH, OW;       // maps of X and Y
    int LH, LW;               // lattice positions per image (of one residue)
    int TCW, nct;             // columns of a column tile, column tiles
    int Q;                    // positions of a column tile = B * LH * TCW
    int EH;                   // staged rows of one image = PS * (LH - 1) + window rows
    int COLS;                 // staged columns
    int g0, xs;               // row (column) of X of staged row (column) r: g0 + xs * r (+ the residue)
    int o0, os;               // row (column) of Y of lattice row u, class r: o0 + os * u -+ r (+ the residue)
    int res;                  // residues per axis
    int nmt, npt;             // tiles of output channels; of the positions of a column tile
    int m_major;              // consecutive blocks share the tile of output channels
    int out16;
    int ksplit, kslice;       // slices of the stages over blocks, stages per slice
    size_t copy_bytes;        // distance of the slices' copies of y
    FastDiv dT, dH, dE, dC;   // by TCW, LH, EH, COLS
    FastDiv dMajor, dP, dN, dR, dK;  // by the tiles of the faster axis, npt, nct, res, ksplit
};

// channels per stage: stages of about a thousand clocks and more of multiplication
constexpr int kc_of(int kind, int n, int mt)
{
    return mt == 16 ? (n == 2 ? 16 : 8) : n == 2 || (n == 3 && kind != kInputGrad) ? 8 : 4;
}
constexpr int window_of(int kind, int n, int s) { return kind == kShifted ? (n + s - 1) / s : kind == kAligned ? n / 2 + 1 : n; }
constexpr int place_of(int kind, int n, int s, int a)
{
    return kind == kShifted ? a / s : kind == kAligned ? a / 2 + a % 2 : kind == kInputGrad ? n - 1 - a : a;
}
// passes of 64 lanes over the staged cells of a channel: what tiles of 4 x 8 (2 x 8) positions and of ragged small maps take
constexpr int jr_of(int kind, int n, int mt)
{
    return mt == 32 ? (kind == kInputGrad ? n + 1 : kind == kDilated && n > 3 ? n - 1 : 2)
                    : (kind == kInputGrad ? (n > 3 ? 3 : 2) : kind == kDilated && n > 3 ? n - 2 : 1);
}
constexpr int classes_of(int kind, int s) { return kind <= kAligned ? s * s : 1; }

// f(0), ..., f(COUNT - 1), the arguments constants (the main loop's bodies are too large for the compiler's own unrolling)
template <int FIRST, class F, int... I>
__device__ __forceinline__ void unrolled_from(F&& f, std::integer_sequence<int, I...>)
{
    (f(std::integral_constant<int, FIRST + I>{}), ...);
}
template <int FIRST, int END, class F>
__device__ __forceinline__ void unrolled(F&& f)
{
    if constexpr (FIRST < END) unrolled_from<FIRST>(f, std::make_integer_sequence<int, END - FIRST>{});
}

template <int KIND, int N, int S, int MT>
struct Layout {
    static constexpr bool TW = KIND == kInputGrad;  // weights [k][m][tap] instead of [m][k][tap]
    static constexpr int NN = N * N, KC = kc_of(KIND, N, MT), NC = classes_of(KIND, S);
    static constexpr int PS = KIND == kInputGrad ? 2 : 1, WIN = window_of(KIND, N, S);
    static constexpr int KI = MT == 32 ? 2 : 4;      // channels per matrix instruction
    static constexpr int R = MT == 32 ? 16 : 4;      // accumulator registers of a class
    // weights in LDS, floats: rows of m (k with TW) a multiple of 16 bytes long, so that pieces of four are whole, and
    // an odd number of such pieces apart, so that the lanes of an operand read spread over the banks
    static constexpr int PPR = (TW ? MT : KC) * NN / 4;                    // pieces of a row
    static constexpr int MS = TW ? (NN == 16 ? 20 : NN) : 4 * (PPR | 1);   // from one m to the next
    static constexpr int KS = TW ? MT * MS : NN;                           // from one k to the next
    static constexpr int AFL = TW ? KC * KS : MT * MS;
    static constexpr int RPI = TW ? 1 : (PPR >= 64 ? 1 : 64 / PPR);        // rows per load instruction
    static constexpr int IPR = (PPR + 63) / 64;                            // load instructions per row
    static constexpr int NROWS = TW ? KC : MT;
    static constexpr int NI = (NROWS + RPI - 1) / RPI * IPR;
    static constexpr int JR = jr_of(KIND, N, MT);
    static constexpr int XPL = JR * 64 + (MT == 32 ? 32 : 16);             // floats of a channel's cells
    static constexpr int STAGE = AFL + KC * XPL;                           // floats per wave
};

// WV waves per block
template <int KIND, int N, int S, int MT, int WV, typename TIn>
__device__ __forceinline__ void small_tile(const TIn* __restrict__ x, const TIn* __restrict__ w, void* __restrict__ y,
                                           const SmallArgs& a, const Epilogue& ep)
{
    typedef Layout<KIND, N, S, MT> L;
    constexpr int ES = (int)sizeof(TIn), NN = L::NN, KC = L::KC, NC = L::NC, WIN = L::WIN, R = L::R, KI = L::KI;
    constexpr bool TW = L::TW, B16 = ES == 2;
    constexpr int PD = B16 ? 2 : 4;  // dwords of a piece
    typedef typename std::conditional<MT == 32, f16v_t, f4v_t>::type acc_t;
    extern __shared__ __align__(16) float lds[];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l = lane % MT, gk = lane / MT;

    const int tk = xcd_contiguous(blockIdx.x, gridDim.x);
    const int t = fdiv(tk, a.dK), ks = tk - t * a.ksplit;
    const int slow = fdiv(t, a.dMajor), fast = t - slow * (int)a.dMajor.d;
    const int mt = a.m_major ? slow : fast, tile = a.m_major ? fast : slow;  // tile: (residue, column tile, its positions)
    const int pc = fdiv(tile, a.dP), p0 = (tile - pc * a.npt) * MT;
    const int pr = fdiv(pc, a.dN), v0 = (pc - pr * a.nct) * a.TCW;
    const int rr = fdiv(pr, a.dR), rc = pr - rr * a.res;
    const int m0 = mt * MT;

    // ---- the lane's position and the block's staged cells
    const int p_first_row = fdiv(p0, a.dT);
    const int b_first = fdiv(p_first_row, a.dH);
    const int e_first = b_first * a.EH + L::PS * (p_first_row - b_first * a.LH);
    const int p = p0 + l < a.Q ? p0 + l : a.Q - 1;
    const int prow = fdiv(p, a.dT), pv = p - prow * a.TCW;
    const int pb = fdiv(prow, a.dH), pu = prow - pb * a.LH;
    const int pos = (pb * a.EH + L::PS * pu - e_first) * a.COLS + L::PS * pv;

    const __amdgpu_buffer_rsrc_t rs_x = __builtin_amdgcn_make_buffer_rsrc(
        (void*)x, 0, (int)((size_t)a.B * a.K * a.XH * a.XW * ES), kRaw);
    const __amdgpu_buffer_rsrc_t rs_w = __builtin_amdgcn_make_buffer_rsrc(
        (void*)w, 0, (int)((size_t)a.M * a.K * NN * ES), kRaw);
    const unsigned xcs = (unsigned)(a.XH * a.XW * ES);
    unsigned xg[L::JR];
#pragma unroll
    for (int j = 0; j < L::JR; ++j) {
        const int e = lane + 64 * j;
        const int row = fdiv(e, a.dC), col = e - row * a.COLS;
        const int er = e_first + row;
        const int b = fdiv(er, a.dE);
        const int i = a.g0 + rr + a.xs * (er - b * a.EH), c = a.g0 + rc + a.xs * (L::PS * v0 + col);
        xg[j] = b < a.B && i >= 0 && i < a.XH && c >= 0 && c < a.XW
                    ? (unsigned)(((b * a.K * a.XH + i) * a.XW + c) * ES) : kNone;
    }
    // weights: the lane's piece of load instruction i is row i / IPR * RPI + lane / PPR, piece lane % PPR + i % IPR * 64
    const int wrow = L::RPI > 1 ? lane / L::PPR : 0;
    const int wq = L::RPI > 1 ? lane - wrow * L::PPR : lane;
    const unsigned wv = TW ? (unsigned)((m0 * NN + 4 * wq) * ES) : (unsigned)(((m0 + wrow) * a.K * NN + 4 * wq) * ES);
    // (a row of m is pieces in a row; with TW and 16 taps, four pieces of an m and a gap)
    const int wl = TW && NN == 16 ? wq / 4 * L::MS + wq % 4 * 4 : wrow * L::MS + 4 * wq;
    auto piece_on = [&](int i) __attribute__((always_inline)) {  // (i: a constant once unrolled)
        const int q = i % L::IPR * 64;
        return (L::RPI == 1 ? wq + q < L::PPR : lane < L::RPI * L::PPR) && i / L::IPR * L::RPI + wrow < L::NROWS;
    };
    auto row_step = [&](int i) __attribute__((always_inline)) { return i / L::IPR * L::RPI; };
    // rows past the last output channel are fetched from its row (they reach no output): the scalar offset stays inside w
    const int m_last = a.M - 1 - m0;
    auto row_in = [&](int i) __attribute__((always_inline)) {
        const int r = row_step(i);
        return TW || r < m_last ? r : m_last;
    };

    unsigned xr[KC][L::JR], wr[L::NI][PD];
    // A last stage that reaches past channel K - 1 is moved down to end there; the channels it shares with the stage
    // before are zeros of X
    auto first_of = [&](int s) { return s * KC + KC <= a.K ? s * KC : a.K - KC; };
    // (stages that do not exist are out of range)
    auto load_x = [&](int s, bool on, int k, int j) __attribute__((always_inline)) {
        const int k_new = s * KC, k0 = first_of(s);
        const unsigned voff = on && k0 + k >= k_new ? xg[j] : kNone;
        if constexpr (B16)
            xr[k][j] = (unsigned)(unsigned short)__builtin_amdgcn_raw_buffer_load_b16(rs_x, voff, (unsigned)(k0 + k) * xcs, 0);
        else
            xr[k][j] = __builtin_amdgcn_raw_buffer_load_b32(rs_x, voff, (unsigned)(k0 + k) * xcs, 0);
    };
    auto load_w = [&](int s, bool on, int i) __attribute__((always_inline)) {
        const int k0 = first_of(s);
        const unsigned voff = on && piece_on(i) ? wv + (unsigned)(i % L::IPR * 256 * ES) : kNone;
        const unsigned soff = (unsigned)((TW ? (k0 + row_in(i)) * a.M * NN : (row_in(i) * a.K + k0) * NN) * ES);
        if constexpr (B16) {
            const u2v_t v = __builtin_amdgcn_raw_buffer_load_b64(rs_w, voff, soff, 0);
            wr[i][0] = v.x;
            wr[i][1] = v.y;
        } else {
            const u4v_t v = __builtin_amdgcn_raw_buffer_load_b128(rs_w, voff, soff, 0);
#pragma unroll
            for (int e = 0; e < 4; ++e) wr[i][e] = v[e];
        }
    };
    float* const As = lds + wave * L::STAGE;
    float* const Xs = As + L::AFL;
    auto store_w = [&](int i) __attribute__((always_inline)) {
        u4v_t v;
        if constexpr (B16) v = u4v_t{wr[i][0] << 16, wr[i][0] & 0xFFFF0000u, wr[i][1] << 16, wr[i][1] & 0xFFFF0000u};
        else v = u4v_t{wr[i][0], wr[i][1], wr[i][2], wr[i][3]};
        const int step = TW ? row_step(i) * L::KS + (NN == 16 ? i % L::IPR * 16 * L::MS : i % L::IPR * 256)
                            : row_step(i) * L::MS + i % L::IPR * 256;
        if (piece_on(i)) *reinterpret_cast<u4v_t*>(As + wl + step) = v;
    };
    auto store_x = [&](int k, int j) __attribute__((always_inline)) { Xs[k * L::XPL + 64 * j + lane] = __uint_as_float(B16 ? xr[k][j] << 16 : xr[k][j]); };

    // (one class: its taps in turn on four accumulators, a quarter of the roundings in a chain)
    constexpr int NA = NC == 1 ? 4 : NC;
    acc_t acc[NA];
#pragma unroll
    for (int c = 0; c < NA; ++c)
#pragma unroll
        for (int i = 0; i < R; ++i) acc[c][i] = 0.f;

    const float* const ap = As + l * L::MS + gk * L::KS;
    const float* const bp = Xs + gk * L::XPL + pos;
    // operands of KI channels: every tap's weight, every window place
    float av[2][NN], bv[2][WIN * WIN];
    constexpr int FA = (NN + 3) / 4, FETCHES = FA + WIN;  // groups of reads: four taps' weights, a row of window places
    auto fetch = [&](int kk, int g) __attribute__((always_inline)) {  // (constants once unrolled)
        if (g < FA) {
#pragma unroll
            for (int i = 4 * g; i < (4 * g + 4 < NN ? 4 * g + 4 : NN); ++i) av[kk & 1][i] = ap[kk * KI * L::KS + i];
        } else {
            const float* const brow = bp + kk * KI * L::XPL + (g - FA) * a.COLS;
#pragma unroll
            for (int wb = 0; wb < WIN; ++wb) bv[kk & 1][(g - FA) * WIN + wb] = brow[wb];
        }
    };
    auto multiply = [&](int kk, int t) __attribute__((always_inline)) {
        const int ta = t / N, tb = t % N, c = NC == 1 ? t % 4 : ta % S * S + tb % S;
        const float af = av[kk & 1][t], bf = bv[kk & 1][place_of(KIND, N, S, ta) * WIN + place_of(KIND, N, S, tb)];
        if constexpr (MT == 32) acc[c] = __builtin_amdgcn_mfma_f32_32x32x2f32(af, bf, acc[c], 0, 0, 0);
        else acc[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(af, bf, acc[c], 0, 0, 0);
    };
    auto own_wave_in_order = [&]() {  // (LDS serves a wave in order; the compiler has to be told)
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    };

    const int stages = (a.K + KC - 1) / KC, s_first = ks * a.kslice;
    const int s_end = s_first + a.kslice < stages ? s_first + a.kslice : stages;
    // The operands of the next KI channels are read while those of the last are multiplied.  Once the last operands of a
    // stage have been read, the next stage goes from its registers to LDS, the registers are refilled and its first operands
    // read, one or two instructions after each MFMA of the last KI channels: a wave that issues more than an MFMA's time of
    // anything else leaves the matrix pipe to the other wave of its SIMD, which does the same at the same time (all of it
    // between two groups of MFMAs: a stage of n = 4 took two waves 5150 clocks for 4096 of MFMAs; in five lots 4970).
    // No branches: the compiler would wait for loads just issued where it waits for the last stage's.
    constexpr int KK = KC / KI, XL = KC * L::JR;
    static_assert(KK % 2 == 0, "operand registers by parity");
    int s = s_first + wave;
    auto op_last = [&](int q, int s_load) __attribute__((always_inline)) {  // 2 * NI + XL + FETCHES of them
        if (q < 2 * L::NI) {
            if (q % 2 == 0) store_w(q / 2);
            else load_w(s_load, s_load < s_end, q / 2);
        } else if (q < 2 * L::NI + XL) {
            store_x((q - 2 * L::NI) % KC, (q - 2 * L::NI) / KC);
        } else {
            if (q == 2 * L::NI + XL) own_wave_in_order();
            fetch(0, q - 2 * L::NI - XL);
        }
    };
    auto op_more = [&](int kk, int q, int s_load) __attribute__((always_inline)) {  // XL of them for kk = 0, then FETCHES
        if (kk == 0 && q < XL) load_x(s_load, s_load < s_end, q % KC, q / KC);
        else fetch(kk + 1, q - (kk == 0 ? XL : 0));
    };
    constexpr int LAST = 2 * L::NI + XL + FETCHES;
    if (s < s_end) {
#pragma unroll
        for (int i = 0; i < L::NI; ++i) load_w(s, true, i);
#pragma unroll
        for (int i = 0; i < XL; ++i) load_x(s, true, i % KC, i / KC);
        unrolled<0, LAST>([&](auto q) __attribute__((always_inline)) { op_last(q, s + WV); });
    }
    for (; s < s_end; s += WV) {
        unrolled<0, KK>([&](auto kk) __attribute__((always_inline)) {
            constexpr bool last = kk + 1 == KK;
            constexpr int ops = last ? LAST : FETCHES + (kk == 0 ? XL : 0);
            if constexpr (last) own_wave_in_order();
            unrolled<0, NN>([&](auto t) __attribute__((always_inline)) {
                multiply(kk, t);
                __builtin_amdgcn_sched_barrier(0);
                unrolled<ops * t / NN, ops * (t + 1) / NN>([&](auto q) __attribute__((always_inline)) {
                    if constexpr (last) op_last(q, s + 2 * WV);
                    else op_more(kk, q, s + WV);
                });
                __builtin_amdgcn_sched_barrier(0);
            });
        });
    }

    if constexpr (NC == 1) acc[0] = (acc[0] + acc[1]) + (acc[2] + acc[3]);
    // ---- the waves' sums meet in LDS, four rows (output channels) at a time: [wave][class][row group][lane]
    __syncthreads();
    constexpr int RG = R / 4;
    f4v_t* const meet = reinterpret_cast<f4v_t*>(lds);
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int g = 0; g < RG; ++g)
            meet[((wave * NC + c) * RG + g) * 64 + lane] =
                f4v_t{acc[c][4 * g], acc[c][4 * g + 1], acc[c][4 * g + 2], acc[c][4 * g + 3]};
    __syncthreads();
    const size_t ybytes = (size_t)a.B * a.M * a.OH * a.OW * (a.out16 ? 2 : 4);
    const __amdgpu_buffer_rsrc_t rs_y = __builtin_amdgcn_make_buffer_rsrc(
        (void*)((unsigned char*)y + (size_t)ks * a.copy_bytes), 0, (int)ybytes, kRaw);
    const bool pv_on = p0 + l < a.Q && v0 + pv < a.LW;
    // the sum of one output without the cells outside the map, if its window reaches any (or repeats channels)
    auto inside_only = [&](float v, int c, int m) {
        const int k_lo = s_first * KC, k_hi = s_end * KC < a.K ? s_end * KC : a.K;
        const int ra = NC == 1 ? 0 : c / S, ca = NC == 1 ? 0 : c % S, st = NC == 1 ? 1 : S;
        const int i0 = a.g0 + rr + a.xs * L::PS * pu, j0 = a.g0 + rc + a.xs * L::PS * (v0 + pv);
        auto place = [&](int ta) { return KIND == kShifted ? ta / S : KIND == kAligned ? ta / 2 + ta % 2 :
                                          KIND == kInputGrad ? N - 1 - ta : ta; };
        bool outside = a.K % KC != 0;
        for (int ta = ra; ta < N; ta += st) {
            const int r = i0 + a.xs * place(ta);
            outside = outside || r < 0 || r >= a.XH;
        }
        for (int tb = ca; tb < N; tb += st) {
            const int q = j0 + a.xs * place(tb);
            outside = outside || q < 0 || q >= a.XW;
        }
        if (!outside) return v;
        v = 0.f;
        for (int ta = ra; ta < N; ta += st)
            for (int tb = ca; tb < N && v == v; tb += st) {
                const int r = i0 + a.xs * place(ta), q = j0 + a.xs * place(tb);
                if (r < 0 || r >= a.XH || q < 0 || q >= a.XW) continue;
                const TIn* xp = x + ((size_t)(pb * a.K + k_lo) * a.XH + r) * a.XW + q;
                const TIn* wp = w + (TW ? (size_t)k_lo * a.M + m : (size_t)m * a.K + k_lo) * NN + ta * N + tb;
                const size_t xstep = (size_t)a.XH * a.XW, wstep = TW ? (size_t)a.M * NN : NN;
                for (int k = k_lo; k < k_hi; ++k, xp += xstep, wp += wstep) {
                    if constexpr (B16) v = fmaf(__uint_as_float((unsigned)*xp << 16), __uint_as_float((unsigned)*wp << 16), v);
                    else v = fmaf(*xp, *wp, v);
                }
            }
        return v;
    };
    auto sums_of = [&](int c, int g) {  // (uniform)
        f4v_t v = meet[(c * RG + g) * 64 + lane];
#pragma unroll
        for (int q = 1; q < WV; ++q) v += meet[((q * NC + c) * RG + g) * 64 + lane];
        return v;
    };
    // rows m_of(g) .. + 3
    auto m_of = [&](int g) { return m0 + (MT == 32 ? 8 * g + 4 * gk : 4 * gk); };
    const int oyb = a.o0 + rr + a.os * pu, oxb = a.o0 + rc + a.os * (v0 + pv);
    const unsigned OSZ = a.out16 ? 2u : 4u, plane = (unsigned)(a.OH * a.OW) * OSZ;
    if constexpr (NC == 4) {
        // both column classes of a row class: neighbours in memory
#pragma unroll 1
        for (int it = wave; it < 2 * RG; it += WV) {
            const int r = it / RG, g = it % RG, m = m_of(g);
            const int oy = KIND == kAligned ? oyb + r : oyb - r;
            // first column of the pair: class 0 (aligned) or class 1 (shifted)
            const int ox = KIND == kAligned ? oxb : oxb - 1, c0 = 2 * r + (KIND == kAligned ? 0 : 1), c1 = c0 ^ 1;
            const f4v_t s0 = sums_of(c0, g), s1 = sums_of(c1, g);
            const bool on = pv_on && oy >= 0 && oy < a.OH;
            const bool on0 = on && ox >= 0 && ox < a.OW, on1 = on && ox + 1 >= 0 && ox + 1 < a.OW;
            const unsigned off = (unsigned)(((pb * a.M + m) * a.OH + oy) * a.OW + ox) * OSZ;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                float v0f = s0[e], v1f = s1[e];
                if (m + e >= a.M) break;
                if (__builtin_expect(!(fabsf(v0f) + fabsf(v1f) < __builtin_inff()), 0)) {
                    if (on0 && !(fabsf(v0f) < __builtin_inff())) v0f = inside_only(v0f, c0, m + e);
                    if (on1 && !(fabsf(v1f) < __builtin_inff())) v1f = inside_only(v1f, c1, m + e);
                }
                if (has_epilogue(ep)) {
                    const float bv = ep.bias ? ep.bias[m + e] : 0.f;
                    v0f = epilogue(v0f, bv, ep.act);
                    v1f = epilogue(v1f, bv, ep.act);
                }
                const unsigned o = off + e * plane;
                if (a.out16) {
                    typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
                    const bf16x2_t b2 = {(__bf16)v0f, (__bf16)v1f};
                    const unsigned bits = __builtin_bit_cast(unsigned, b2);
                    __builtin_amdgcn_raw_buffer_store_b32(bits, rs_y, on0 && on1 ? o : kNone, 0, 0);
                    if (on0 != on1)
                        __builtin_amdgcn_raw_buffer_store_b16((short)(on0 ? bits & 0xFFFFu : bits >> 16), rs_y, on0 ? o : o + 2u, 0, 0);
                } else {
                    __builtin_amdgcn_raw_buffer_store_b64(u2v_t{__float_as_uint(v0f), __float_as_uint(v1f)}, rs_y,
                                                          on0 && on1 ? o : kNone, 0, 0);
                    if (on0 != on1)
                        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(on0 ? v0f : v1f), rs_y, on0 ? o : o + 4u, 0, 0);
                }
            }
        }
    } else {  // (gradients, strided and dilated layers: fp32 results, no epilogue)
#pragma unroll 1
        for (int it = wave; it < NC * RG; it += WV) {
            const int c = it / RG, g = it % RG, m = m_of(g);
            const int oy = NC == 1 ? oyb : oyb - c / S, ox = NC == 1 ? oxb : oxb - c % S;
            const f4v_t sum = sums_of(c, g);
            const bool on = pv_on && oy >= 0 && oy < a.OH && ox >= 0 && ox < a.OW;
            const unsigned off = (unsigned)(((pb * a.M + m) * a.OH + oy) * a.OW + ox) * 4u;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                float v = sum[e];
                if (__builtin_expect(!(fabsf(v) < __builtin_inff()), 0))
                    if (on && m + e < a.M) v = inside_only(v, c, m + e);
                __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), rs_y, on && m + e < a.M ? off + e * plane : kNone, 0, 0);
            }
        }
    }
}

template <int KIND, int N, int S, int MT, int WV, typename TIn>
__global__ __launch_bounds__(64 * WV) __attribute__((amdgpu_waves_per_eu(2, 2)))
void ukst_mfma_f32_kernel_small(const TIn* __restrict__ x, const TIn* __restrict__ w, void* __restrict__ y, SmallArgs a,
                                Epilogue ep)
{
    small_tile<KIND, N, S, MT, WV, TIn>(x, w, y, a, ep);
}
// (under the name of the kernels it belongs to)
template <int N, int MT, int WV, typename TIn>
__global__ __launch_bounds__(64 * WV) __attribute__((amdgpu_waves_per_eu(2, 2)))
void ukst_grad_input_mfma_kernel_small(const TIn* __restrict__ x, const TIn* __restrict__ w, void* __restrict__ y,
                                       SmallArgs a, Epilogue ep)
{
    small_tile<kInputGrad, N, 1, MT, WV, TIn>(x, w, y, a, ep);
}

template <int KIND, int N, int S, int MT, int WV, typename TIn>
hipError_t launch_one(const SmallArgs& a, const Epilogue& ep, const void* x, const void* w, void* y, hipStream_t stream)
{
    typedef Layout<KIND, N, S, MT> L;
    constexpr size_t stage = (size_t)WV * L::STAGE * 4, sums = (size_t)WV * L::NC * L::R * 256;
    constexpr size_t bytes = stage > sums ? stage : sums;
    static_assert(bytes <= 160 * 1024, "LDS");
    typedef void (*kernel_t)(const TIn*, const TIn*, void*, SmallArgs, Epilogue);
    kernel_t kfn;
    if constexpr (KIND == kInputGrad) kfn = ukst_grad_input_mfma_kernel_small<N, MT, WV, TIn>;
    else kfn = ukst_mfma_f32_kernel_small<KIND, N, S, MT, WV, TIn>;
    const hipError_t e = hipFuncSetAttribute((const void*)kfn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
    if (e != hipSuccess) return e;
    const unsigned blocks = (unsigned)(a.nmt * a.npt * a.nct * a.res * a.res * a.ksplit);
    hipLaunchKernelGGL(kfn, dim3(blocks), dim3(64 * WV), bytes, stream, (const TIn*)x, (const TIn*)w, y, a, ep);
    return hipGetLastError();
}

// every instance of one kind and operand type (one translation unit each: ukst_small_*.hip); mt 32 or 16, wv 4 or 8
template <int KIND, typename TIn>
hipError_t launch_kind(const SmallArgs& a, int n, int s, int mt, int wv, const Epilogue& ep, const void* x, const void* w,
                       void* y, hipStream_t stream);

#define UKST_SMALL_DECLARE(KIND, T)                                                                                 \
    template <> hipError_t launch_kind<KIND, T>(const SmallArgs&, int, int, int, int, const Epilogue&, const void*, \
                                                const void*, void*, hipStream_t);
UKST_SMALL_DECLARE(kShifted, float) UKST_SMALL_DECLARE(kShifted, uint16_t)
UKST_SMALL_DECLARE(kAligned, float) UKST_SMALL_DECLARE(kAligned, uint16_t)
UKST_SMALL_DECLARE(kInputGrad, float) UKST_SMALL_DECLARE(kInputGrad, uint16_t)
UKST_SMALL_DECLARE(kDilated, float) UKST_SMALL_DECLARE(kDilated, uint16_t)
#undef UKST_SMALL_DECLARE

template <int KIND, int N, int S, typename TIn>
hipError_t launch_sizes(const SmallArgs& a, int mt, int wv, const Epilogue& ep, const void* x, const void* w, void* y,
                        hipStream_t st)
{
    if constexpr (classes_of(KIND, S) <= 4) {
        if (mt == 32 && wv == 8) return launch_one<KIND, N, S, 32, 8, TIn>(a, ep, x, w, y, st);
        if (mt == 32 && wv == 4) return launch_one<KIND, N, S, 32, 4, TIn>(a, ep, x, w, y, st);
    }
    if (mt == 16) return launch_one<KIND, N, S, 16, 8, TIn>(a, ep, x, w, y, st);
    return hipErrorInvalidValue;
}

template <int KIND, typename TIn>
hipError_t launch_kind_impl(const SmallArgs& a, int n, int s, int mt, int wv, const Epilogue& ep, const void* x,
                            const void* w, void* y, hipStream_t st)
{
#define UKST_SMALL_CASE(N, S) \
    if (n == N && s == S) return launch_sizes<KIND, N, S, TIn>(a, mt, wv, ep, x, w, y, st);
    if constexpr (KIND == kShifted) {
        UKST_SMALL_CASE(2, 2) UKST_SMALL_CASE(3, 2) UKST_SMALL_CASE(4, 2) UKST_SMALL_CASE(5, 2)
        UKST_SMALL_CASE(2, 3) UKST_SMALL_CASE(3, 3) UKST_SMALL_CASE(4, 3) UKST_SMALL_CASE(5, 3)
        UKST_SMALL_CASE(2, 4) UKST_SMALL_CASE(3, 4) UKST_SMALL_CASE(4, 4) UKST_SMALL_CASE(5, 4)
    } else if constexpr (KIND == kAligned) {
        UKST_SMALL_CASE(2, 2) UKST_SMALL_CASE(4, 2)
    } else {
        UKST_SMALL_CASE(2, 1) UKST_SMALL_CASE(3, 1) UKST_SMALL_CASE(4, 1) UKST_SMALL_CASE(5, 1)
    }
#undef UKST_SMALL_CASE
    return hipErrorInvalidValue;
}

}  // namespace small
}  // namespace ukst
