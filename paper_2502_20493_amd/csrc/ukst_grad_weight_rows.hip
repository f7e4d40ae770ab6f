// Gradient with respect to the kernel of wide layers on the bf16 matrix pipe: fp32 operands as three exact bf16 parts
// (ukst_parts.h), bf16 operands as one; n = 2..5, rows of any length.
//
// The product is that of the other kernel gradients, DW_tap[co][ci] += sum_pixel DY_tap[co][pixel] * X[ci][pixel],
// with the pixel axis as the K axis of v_mfma_f32_32x32x16_bf16: a lane's operand is 8 consecutive pixels of one
// channel, x as it lies in memory, dy rows split by column parity on their way into LDS.
//
// What bounds kernels of this kind is filling LDS, so the fill is laid out to run beside the multiplication:
//  * A block (8 waves, two per SIMD, one block per compute unit) takes 32 output channels x 128 input channels (n = 5: 64)
//    and walks down a strip of the images, 8*GPR columns wide, TI rows at a time.  x rows are double buffered; dy rows live in a
//    ring, and of the 2*TI + n - 2 rows that TI rows of x meet, only the 2*TI new ones are staged.  Images follow each
//    other without a break: an image has HS = H + ceil((n-2)/2) rows in this walk, the first ones without pixels, in which
//    the ring fills with its first dy rows.  Row `r` of the walk meets dy rows 2*r + 1 - a (a: tap row) of the walk of dy.
//  * What a stage needs is loaded a whole stage earlier, into registers, and written to LDS while the stage before it is
//    multiplied.  bf16: slot by slot between the units of a step, whose operands are read one unit ahead; a wave that did
//    its staging in one go took as long for it as for its MFMAs.  fp32, six MFMAs for one: by the second wave of a SIMD
//    before its MFMAs, by the first one after them.  One barrier a stage.
//  * K steps are 2 groups of 8 pixels, one per half of the wave, each in a row of its own if need be: narrow maps fill
//    the steps as well as wide ones.
//  * Taps are dealt to the waves in units of one (tap row, column parity): the taps of a unit are one element apart
//    and share an LDS read, the shift is made in registers.  n = 4: a row of taps per wave; n = 5: units of 3 and 2
//    taps, 6, 6, 7 and 6 a wave; n = 3: 5 and 4; n = 2: 2.
// Measured with the sum of the copies, us, the kernels before it / this one: bf16, 64 x 1024 -> 512 channels, 16 x 16, n = 4 459 / 277
// (matrix pipes busy 0.29 / 0.55), 32 x 256 -> 128, 128 x 128, n = 4 895 / 541, 21 x 128 -> 147, 44 x 58, n = 5 664 / 113; fp32, 32 x 128 -> 128,
// 63 x 63, n = 3 344 / 234, 64 x 64, n = 5 1178 / 540.  On the way (the first): addresses and row ends worked out per piece 600; once per
// lane, branches in the staging 328; staging between the units 307; dy rows one element before whole 16 bytes 280.
// Rows past their end: x is masked to zeros, so the pixels there take no part in a sum; a dy operand that is not finite makes a
// NaN of them, and tiles with a sum that is not finite are taken again from memory (ukst_parts.h).  Loads of bf16 rows are whole
// 16 bytes of memory: no byte outside the 16-byte lines that hold the tensor is touched.
#include <math.h>

#include "ukst_parts.h"

namespace ukst {
namespace {

struct GwRowsArgs {
    GeomBase g;
    int GPR, TI;                // groups of 8 pixels of a row, rows of a stage
    int HS, V;                  // rows of an image in the walk, those of them without pixels
    int HC, R, DP, XP;          // half row, ring rows, channel strides of dy and x (elements)
    int flushRows;              // rows after which the sums are added to the copy of dw (fp32)
    int ragged;                 // rows of x are no multiple of 8: 1
    int rowsPerSlice, slicesPerTile, tilesX, nSlices, coTiles, ciTiles;
    int c8, dl, xl;             // 8-column pieces of a row of dy; lanes that load a row of dy, of x
    int dRowsPerWave, dWaves, xRowsPerWave, xWaves;  // rows a wave loads at once, and how often a stage's row asks for that
    FastDiv dHS, dGPR, dDL, dXL, dDWaves, dXWaves;
};

constexpr int T_ROWS = 512;  // threads
// pieces a thread stages of x and dy, at most (four or eight registers each)
constexpr int x_slots(int es, int ci_t, bool ragged) { return es == 4 ? 1 : (ci_t == 64 ? 1 : 2) + (ragged ? 1 : 0); }
constexpr int dy_slots(int es) { return es == 4 ? 2 : 4; }

// the taps' deal: groups of waves, and a wave's units (a row of taps, first tap column 0 or 1, taps 2 columns apart)
constexpr int tap_groups(int n) { return n <= 3 ? 2 : 4; }
constexpr int wave_taps(int n) { return n == 2 ? 2 : n == 3 ? 5 : n == 4 ? 4 : 7; }  // (accumulators, at most)
// unit u of group grp: row * 2 + first column; the number of its taps; -1: none
constexpr int unit_of(int n, int grp, int u)
{
    if (n == 2) return u < 2 ? grp * 2 + u : -1;
    if (n == 3) {
        const int t[2][3] = {{0, 2, 1}, {4, 3, 5}};  // {row 0 even, row 1 even, row 0 odd}, {row 2 even, row 1 odd, row 2 odd}
        return t[grp][u];
    }
    if (n == 4) return u < 2 ? grp * 2 + u : -1;
    const int t[4][3] = {{0, 2, -1}, {4, 6, -1}, {8, 1, 3}, {5, 7, 9}};
    return t[grp][u];
}
constexpr int unit_taps(int n, int unit) { return unit < 0 ? 0 : (n - (unit & 1) + 1) / 2; }
constexpr int max_units(int n) { return n == 3 || n == 5 ? 3 : 2; }
// accumulator of tap k of unit u
constexpr int acc_of(int n, int u, int k) { return n == 3 ? (u == 0 ? k : u == 1 ? 2 + k : 4) : n == 5 ? (u == 2 ? 5 : 3 * u) + k : (n / 2) * u + k; }
constexpr int most_taps(int n, int u)
{
    int m = 0;
    for (int grp = 0; grp < tap_groups(n); ++grp) {
        const int t = unit_taps(n, unit_of(n, grp, u));
        m = t > m ? t : m;
    }
    return m;
}
constexpr int least_taps(int n, int u)
{
    int m = 99;
    for (int grp = 0; grp < tap_groups(n); ++grp) {
        const int t = unit_taps(n, unit_of(n, grp, u));
        m = t < m ? t : m;
    }
    return m;
}

// eight elements of a row as loaded: fp32 values, or packed bf16
template <typename TIn>
struct Eight { u4v_t h[sizeof(TIn) / 2]; };

template <typename TIn>
__device__ __forceinline__ Eight<TIn> load_eight(const __amdgpu_buffer_rsrc_t& rs, unsigned off)
{
    Eight<TIn> q;
#pragma unroll
    for (int h = 0; h < (int)sizeof(TIn) / 2; ++h) {
        unsigned at = off + 16 * h;
        if (h) asm("" : "+v"(at));  // (added here, modulo 2^32: the first half of a piece may lie before the tensor)
        q.h[h] = __builtin_amdgcn_raw_buffer_load_b128(rs, at, 0, 0);
    }
    return q;
}
// eight bf16 from element sh/2 of the lane's eight on, the lane above holding the eight behind them
__device__ __forceinline__ unsigned of_lane_above(unsigned v)
{
    return (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x130, 0xF, 0xF, true);  // wave_shl:1
}
__device__ __forceinline__ void funnel(u4v_t& q, int sh)
{
    const unsigned bits = (unsigned)(sh & 2) << 3;
    unsigned w[8];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        w[i] = q[i];
        w[i + 4] = of_lane_above(q[i]);
    }
    const unsigned by2 = (unsigned)-(sh >> 3 & 1), by1 = (unsigned)-(sh >> 2 & 1);  // (bit selects: of conditions the compiler makes
#pragma unroll                                                                       // an index into memory)
    for (int i = 0; i < 6; ++i) w[i] = (w[i] & ~by2) | (w[i + 2] & by2);
#pragma unroll
    for (int i = 0; i < 5; ++i) w[i] = (w[i] & ~by1) | (w[i + 1] & by1);
#pragma unroll
    for (int i = 0; i < 4; ++i) q[i] = __builtin_amdgcn_alignbit(w[i + 1], w[i], bits);
}
// element k becomes element k + s, 0 < s < 8 (only where a row begins before the tensor)
__device__ __forceinline__ void move_up(Eight<float>& q, int s)
{
#pragma unroll
    for (int k = 7; k >= 0; --k) {
        unsigned r = 0u;
#pragma unroll
        for (int j = 0; j < k; ++j) r = k - s == j ? q.h[j >> 2][j & 3] : r;
        q.h[k >> 2][k & 3] = s > 0 ? r : q.h[k >> 2][k & 3];
    }
}

// N kernel side; NC groups of 32 input channels per wave; STEPS K steps of a stage; RAGGED: rows of
// x are no multiple of 8; ONE: every piece of dy begins one element before whole 16 bytes (bf16, n = 4, P = 2, aligned rows)
template <int N, int NC, int STEPS, bool RAGGED, bool ONE, typename TIn>
__device__ __forceinline__ void grad_weight_rows(const TIn* __restrict__ x, const TIn* __restrict__ dy,
                                                 float* __restrict__ part, const GwRowsArgs& a)
{
    constexpr int PARTS = sizeof(TIn) == 4 ? 3 : 1;
    constexpr int ES = (int)sizeof(TIn);
    constexpr int NN = N * N;
    constexpr int GROUPS = tap_groups(N), CIW = 8 / GROUPS;
    constexpr int CO_T = 32, CI_T = 32 * NC * CIW;
    constexpr int MX = x_slots(ES, CI_T, RAGGED), MD = dy_slots(ES);
    typedef PartProducts<PARTS> PP;
    extern __shared__ __align__(16) unsigned char lds[];
    const GeomBase& g = a.g;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, kk = lane >> 5;
    // wave w and w + 4 share a SIMD: of n = 5 no two groups of seven and six taps meet there more than once, n = 3 five and four
    const int grp = GROUPS == 2 ? wave >> 2 : N == 5 && wave >= 4 ? (wave + 1) & 3 : wave & 3;
    const int ciw = GROUPS == 2 ? wave & 3 : wave >> 2;

    // bytes of one part: an x buffer, the ring; 256 behind them take what lanes without a piece write (a branch around the
    // write would keep it from the MFMAs it is written under)
    const int XPB = CI_T * a.XP * 2 + 256, DPB = CO_T * a.DP * 2 + 256;
    unsigned char* const xs = lds;                           // [buffer][part][ci][row of the stage][column]
    unsigned char* const dys = lds + 2 * PARTS * XPB;        // [part][co][ring row][column parity][column / 2]
    // bf16 (rows of x: if they are no multiple of 8): loads are whole 16 bytes of memory, at addresses of 16 bytes; what they
    // hold of other rows, or of the 16 bytes in which the tensor begins or ends, is masked
    const unsigned x_align = ES == 2 && RAGGED ? 15u : 0u, dy_align = ES == 2 ? 15u : 0u;
    const unsigned x_in = (unsigned)(uintptr_t)x & x_align, dy_in = (unsigned)(uintptr_t)dy & dy_align;
    const __amdgpu_buffer_rsrc_t rs_x = __builtin_amdgcn_make_buffer_rsrc(
        (void*)((uintptr_t)x - x_in), 0,
        (int)(((size_t)g.B * g.Cin * g.H * g.W * ES + x_in + x_align) & ~(size_t)x_align), kRawBuffer);
    const __amdgpu_buffer_rsrc_t rs_dy = __builtin_amdgcn_make_buffer_rsrc(
        (void*)((uintptr_t)dy - dy_in), 0,
        (int)(((size_t)g.B * g.Cout * g.OH * g.OW * ES + dy_in + dy_align) & ~(size_t)dy_align), kRawBuffer);

    int bid = xcd_contiguous(blockIdx.x, gridDim.x);  // neighbours in this numbering share an L2
    const int cit = bid % a.ciTiles; bid /= a.ciTiles;
    const int cot = bid % a.coTiles;
    const int slice = bid / a.coTiles;
    const int co0 = cot * CO_T, ci0 = cit * CI_T;
    const int tile = slice / a.slicesPerTile;
    const int j0 = tile * 8 * a.GPR;
    const int row0 = (slice - tile * a.slicesPerTile) * a.rowsPerSlice;
    const int rows = g.B * a.HS;
    const int row_end = row0 + a.rowsPerSlice < rows ? row0 + a.rowsPerSlice : rows;
    int first = row0, row1 = first + a.flushRows < row_end ? first + a.flushRows : row_end;  // the run of rows at hand

    {
        const int total = 2 * PARTS * XPB + PARTS * DPB;
        for (int i = tid * 16; i < total; i += T_ROWS * 16) *reinterpret_cast<u4v_t*>(lds + i) = u4v_t{0u, 0u, 0u, 0u};
    }

    // ---- staging.  A piece is eight columns of a row.  (No load under a condition: those are waited for where the paths
    // meet.)  bf16 pieces are fetched as they lie in memory, from the last whole 16 bytes at or before their first column
    // on, by one lane more than the row has pieces, and shifted into place with the help of the lane above; fetched at
    // their own addresses they cost the address unit a cycle or two per lane, which bounded the kernel, and LDS takes far
    // longer for writes at odd addresses.  fp32 pieces are fetched from their own addresses
    const int hw = g.H * g.W, ohw = g.OH * g.OW;
    const int ox0 = 2 * j0 + g.P - (N - 1);
    // the lane's piece is the same one of every row: what is past the ends of a row (read from LDS for every piece, the masks
    // were waited for behind the writes of the piece before and cost a third of the time)
    Eight<TIn> x_in_row, d_in_row;
    auto in_row = [&](int col, int end, Eight<TIn>& m) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            auto is = [&](int c) { return c >= 0 && c < end ? ~0u : 0u; };
            if constexpr (ES == 4) {
                m.h[0][k] = is(col + k);
                m.h[1][k] = is(col + 4 + k);
            } else {
                m.h[0][k] = (is(col + 2 * k) & 0xFFFFu) | (is(col + 2 * k + 1) & 0xFFFF0000u);
            }
        }
    };
    auto image_of = [&](int row) { return (int)(__umulhi((unsigned)row, a.dHS.M) >> a.dHS.sh); };  // (HS > 1)
    const int x_image = g.Cin * hw * ES, x_line = g.W * ES, dy_image = g.Cout * ohw * ES, dy_line = g.OW * ES;
    Eight<TIn> xq[MX], dq[MD];
    unsigned x_off[MX];  // (no such piece: past the end, whatever is added)
    int x_dst[MX], d_off[MD], d_dst[MD], d_bit[MD];
    int x_sh[MX], d_sh[MD];  // by how much the piece in flight has to be shifted
    int x_tr[MX], d_tr[MD];  // (uniform) row of the stage
    constexpr int kNever = 0x40000000;
    {
        const int li = fdiv(lane, a.dXL), m = lane - li * a.xl;
        in_row(j0 + 8 * m, g.W, x_in_row);
#pragma unroll
        for (int k = 0; k < MX; ++k) {
            const int turn = wave + 8 * k;
            x_tr[k] = fdiv(turn, a.dXWaves);
            const int ch = (turn - x_tr[k] * a.xWaves) * a.xRowsPerWave + li;
            const bool on = li < a.xRowsPerWave && ch < CI_T && x_tr[k] < a.TI;
            const bool in = on && ci0 + ch < g.Cin && j0 + 8 * m - (ES == 2 && RAGGED ? 7 : 0) < g.W;
            x_off[k] = in ? (unsigned)(((ci0 + ch) * hw + j0 + 8 * m) * ES) + x_in : 0x80000000u;
            x_dst[k] = on && m < a.GPR ? (ch * a.XP + (x_tr[k] * a.GPR + m) * 8) * 2 : CI_T * a.XP * 2 + lane % 16 * 16;
        }
    }
    const int d_li = fdiv(lane, a.dDL), d_m = lane - d_li * a.dl - (ONE ? 1 : 0);
    in_row(ox0 + 8 * d_m, g.OW, d_in_row);
    // the lane's piece of the pair of rows in the wave's turn `turn` at it
    auto dy_lane = [&](int turn, bool last, int& off, int& dst, int& bit) {
        const int row = turn * a.dRowsPerWave + d_li, ch = row < CO_T ? row : row - CO_T, ox = ox0 + 8 * d_m + (ONE ? 1 : 0);  // (ONE: the lane's own 16 bytes, the last element of the lane below before them)
        const bool on = d_li < a.dRowsPerWave && row < 2 * CO_T && last;
        bit = row < CO_T ? 0 : 1;
        off = ((co0 + ch) * ohw + bit * g.OW + ox) * ES + (int)dy_in;
        dst = on && d_m >= 0 && d_m < a.c8 ? (ch * a.DP + bit * 2 * a.HC + 4 * d_m) * 2 : -1 - lane % 8 * 8;
        if (!on || co0 + ch >= g.Cout || ox + 7 < 0 || ox - (ES == 2 && !ONE ? 7 : 0) >= g.OW) bit = kNever;
    };
#pragma unroll
    for (int k = 0; k < MD; ++k) {
        const int turn = wave + 8 * k;
        d_tr[k] = fdiv(turn, a.dDWaves);
        dy_lane(turn - d_tr[k] * a.dWaves, d_tr[k] < a.TI, d_off[k], d_dst[k], d_bit[k]);
    }
    auto masked = [&](Eight<TIn>& q, const Eight<TIn>& m) {
#pragma unroll
        for (int h = 0; h < ES / 2; ++h) q.h[h] &= m.h[h];
    };
    auto load_x = [&](int k, int row_s) {  // slot k of the stage that begins with row row_s of the walk
        const int row = row_s + x_tr[k], b = image_of(row), i = row - b * a.HS - a.V;  // (uniform)
        const unsigned at = x_off[k] + (unsigned)(b * x_image + i * x_line);
        x_sh[k] = (int)(at & x_align);
        xq[k] = load_eight<TIn>(rs_x, row < row1 && i >= 0 ? at & ~x_align : kNoByte);
    };
    auto write_x = [&](int k, int buf) {
        Eight<TIn> q8 = xq[k];
        if constexpr (RAGGED) {
            if constexpr (ES == 2) funnel(q8.h[0], x_sh[k]);
            masked(q8, x_in_row);
        }
        unsigned char* const dst = xs + buf * PARTS * XPB + x_dst[k];
        if constexpr (PARTS == 3) {
            u4v_t p[3];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                unsigned q[3];
                split_pair(__uint_as_float(q8.h[i >> 1][2 * i & 3]), __uint_as_float(q8.h[i >> 1][(2 * i & 3) + 1]), q[0], q[1], q[2]);
#pragma unroll
                for (int m = 0; m < 3; ++m) p[m][i] = q[m];
            }
#pragma unroll
            for (int m = 0; m < 3; ++m) *reinterpret_cast<u4v_t*>(dst + m * XPB) = p[m];
        } else {
            *reinterpret_cast<u4v_t*>(dst) = q8.h[0];
        }
    };
    // the two dy rows of row `row` of the walk.  (Rows past the last image, as rows before the first one, do not exist or
    // belong to no pixels)
    auto dy_load = [&](int row, int off, int bit, int& sh) {
        const int b = row < 0 ? 0 : image_of(row), oy = 2 * (row - b * a.HS - a.V) - 1 + g.P;  // (uniform)
        const int at = off + b * dy_image + oy * dy_line;
        const bool on = b < g.B && (unsigned)(oy + bit) < (unsigned)g.OH;
        if constexpr (ES == 2) {
            sh = at & 15;  // (ONE: 0)
            return load_eight<TIn>(rs_dy, on ? (unsigned)at & (ONE ? ~0u : ~15u) : kNoByte);
        } else {
            const int from = at < 0 ? 0 : at;  // (the tensor's first row)
            sh = on ? from - at : 0;
            return load_eight<TIn>(rs_dy, on ? (unsigned)from : kNoByte);
        }
    };
    auto dy_write = [&](int slot, int dst_off, int sh, Eight<TIn> q) {
        if constexpr (ONE) {
            const unsigned below = (unsigned)__builtin_amdgcn_update_dpp(0, (int)q.h[0].w, 0x138, 0xF, 0xF, true);  // wave_shr:1
            q.h[0] = u4v_t{__builtin_amdgcn_alignbit(q.h[0].x, below, 16), __builtin_amdgcn_alignbit(q.h[0].y, q.h[0].x, 16),
                           __builtin_amdgcn_alignbit(q.h[0].z, q.h[0].y, 16), __builtin_amdgcn_alignbit(q.h[0].w, q.h[0].z, 16)};
        } else if constexpr (ES == 2) {
            funnel(q.h[0], sh);
        } else {
            if (__builtin_amdgcn_ballot_w64(sh != 0)) move_up(q, sh / ES);  // (hardly ever)
        }
        masked(q, d_in_row);
        unsigned char* const dst = dys + (dst_off < 0 ? CO_T * a.DP * 2 - 1 - dst_off : slot * 4 * a.HC + dst_off);
        if constexpr (PARTS == 3) {
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                unsigned u[2][3];
#pragma unroll
                for (int h = 0; h < 2; ++h)
                    split_pair(__uint_as_float(q.h[h][p]), __uint_as_float(q.h[h][2 + p]), u[h][0], u[h][1], u[h][2]);
#pragma unroll
                for (int i = 0; i < 3; ++i) *reinterpret_cast<u2v_t*>(dst + i * DPB + p * a.HC * 2) = u2v_t{u[0][i], u[1][i]};
            }
        } else {
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                const unsigned sel = p ? 0x07060302u : 0x05040100u;
                *reinterpret_cast<u2v_t*>(dst + p * a.HC * 2) =
                    u2v_t{__builtin_amdgcn_perm(q.h[0].y, q.h[0].x, sel), __builtin_amdgcn_perm(q.h[0].w, q.h[0].z, sel)};
            }
        }
    };
    auto load_dy = [&](int k, int row_s) { dq[k] = dy_load(row_s + d_tr[k], d_off[k], d_bit[k], d_sh[k]); };
    auto write_dy = [&](int k, int slot_s) {  // slot_s: ring row of the stage's first dy row (even, as is the ring)
        const int slot = slot_s + 2 * d_tr[k];
        dy_write(slot < a.R ? slot : slot - a.R, d_dst[k], d_sh[k], dq[k]);
    };
    constexpr int ITEMS = MX + MD;  // slots of a stage: of x, then of dy
    auto load_item = [&](int k, int row_s) {
        if (k < MX) load_x(k, row_s);
        else load_dy(k - MX, row_s);
    };
    auto write_item = [&](int k, int buf, int slot_s) {
        if (k < MX) write_x(k, buf);
        else write_dy(k - MX, slot_s);
    };

    // n = 2: every other step on accumulators of its own, half the roundings in a chain
    constexpr int SETS = N == 2 ? 2 : 1;
    f32x16_t acc[SETS * wave_taps(N)][NC];
    auto clear = [&]() {
#pragma unroll
        for (int t = 0; t < SETS * wave_taps(N); ++t)
#pragma unroll
            for (int c = 0; c < NC; ++c)
#pragma unroll
                for (int i = 0; i < 16; ++i) acc[t][c][i] = 0.f;
    };

    // ---- the wave's units
    constexpr int U = max_units(N);
    int u_row[U], u_par[U], u_taps[U], u_col[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        int un = -1, nt = 0;
#pragma unroll
        for (int q = 0; q < GROUPS; ++q)
            if (grp == q) {
                un = unit_of(N, q, u);
                nt = unit_taps(N, unit_of(N, q, u));
            }
        u_taps[u] = nt;
        u_row[u] = un >> 1;
        u_col[u] = un & 1;
        u_par[u] = (N - 1 - u_col[u]) & 1;
    }
    const int b_lane = (ciw * 32 * NC + l32) * a.XP * 2;
    int a_lane[U];
#pragma unroll
    for (int u = 0; u < U; ++u) a_lane[u] = l32 * a.DP * 2 + u_par[u] * a.HC * 2;
    // the lane's group of K step sp, 2*sp + kk: bytes from the ring row of the stage's first row on
    const int line = 4 * a.HC, ring = a.R * line;
    int rel[STEPS], xrel[STEPS];
#pragma unroll
    for (int sp = 0; sp < STEPS; ++sp) {
        const int q = 2 * sp + kk, t = fdiv(q, a.dGPR), c = q - t * a.GPR;
        rel[sp] = (t < a.TI ? 2 * t : 0) * line + 16 * c;
        xrel[sp] = (t < a.TI ? t * a.GPR + c : a.TI * a.GPR) * 16;  // (groups past the stage: zeros)
    }

    // the K steps of a stage whose first dy row is in ring row slot_s, stage(k), k = 0 .. ITEMS - 1, dealt out between them
    constexpr bool DEAL = PARTS == 1;  // the staging dealt out between the products, or before them or after them
    auto multiply = [&](int slot_s, int buf, auto&& stage) {
        int first[U];  // (uniform) where the unit's tap row of the stage's first row is, not yet taken modulo the ring
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int r = slot_s + 1 - u_row[u];
            first[u] = u > 0 && N % 2 == 0 ? first[0] : (r < 0 ? r + a.R : r) * line;  // (n = 2, 4: units of one row)
        }
        const unsigned char* const bp = xs + buf * PARTS * XPB + b_lane;
        constexpr int AHEAD = DEAL ? 1 : 0;  // units whose operands are read ahead
        bf16x8_t bv[1 + AHEAD][NC][PARTS];
        u4v_t h[1 + AHEAD][PARTS];
        unsigned next[1 + AHEAD][PARTS];
        auto fetch = [&](int r) {  // operands of unit r % U of step r / U
            const int sp = r / U, u = r % U;
            if (u == 0) {
#pragma unroll
                for (int c = 0; c < NC; ++c)
#pragma unroll
                    for (int i = 0; i < PARTS; ++i)
                        bv[sp & AHEAD][c][i] = *reinterpret_cast<const bf16x8_t*>(bp + i * XPB + c * 64 * a.XP + xrel[sp]);
            }
            const unsigned pos = (unsigned)(first[u] + rel[sp]), back = pos - (unsigned)ring;
            const unsigned char* const ap = dys + a_lane[u] + (pos < back ? pos : back);
#pragma unroll
            for (int i = 0; i < PARTS; ++i) {
                h[r & AHEAD][i] = *reinterpret_cast<const u4v_t*>(ap + i * DPB);
                if (most_taps(N, u) > 1) next[r & AHEAD][i] = *reinterpret_cast<const unsigned*>(ap + i * DPB + 16);
            }
        };
        if (AHEAD) fetch(0);
#pragma unroll
        for (int r = 0; r < STEPS * U; ++r) {
            const int sp = r / U, u = r % U;
            // the next unit's operands, a share of the staging, the products: one wave issues in order, so the compiler is asked
            // for a few vector instructions behind every MFMA
            if (DEAL) __builtin_amdgcn_sched_barrier(0);
            if (!AHEAD) fetch(r);
            else if (r + 1 < STEPS * U) fetch(r + 1);
            int items = 0;
            if (DEAL && u < 2) {
#pragma unroll
                for (int k = 0; k < ITEMS; ++k)
                    if (k * 2 * STEPS / ITEMS == 2 * sp + u) {
                        stage(k);
                        ++items;
                    }
            }
            bf16x8_t av[3][PARTS];
#pragma unroll
            for (int i = 0; i < PARTS; ++i) {
                const u4v_t v = h[r & AHEAD][i];
                const unsigned n = next[r & AHEAD][i];
                av[0][i] = __builtin_bit_cast(bf16x8_t, v);
                if (most_taps(N, u) > 1)
                    av[1][i] = __builtin_bit_cast(
                        bf16x8_t, u4v_t{__builtin_amdgcn_alignbit(v.y, v.x, 16), __builtin_amdgcn_alignbit(v.z, v.y, 16),
                                        __builtin_amdgcn_alignbit(v.w, v.z, 16), __builtin_amdgcn_alignbit(n, v.w, 16)});
                if (most_taps(N, u) > 2) av[2][i] = __builtin_bit_cast(bf16x8_t, u4v_t{v.y, v.z, v.w, n});
            }
            // (a unit's last tap column is the one that is not shifted: k here counts from it)
            const int at = sp % SETS * wave_taps(N);
            auto products = [&](int k0, int k1) {
#pragma unroll
                for (int m = 0; m < PP::count; ++m)
#pragma unroll
                    for (int k = k0; k < k1; ++k)
#pragma unroll
                        for (int c = 0; c < NC; ++c)
                            acc[at + acc_of(N, u, k)][c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                                av[k][PP::a[m]], bv[sp & AHEAD][c][PP::b[m]], acc[at + acc_of(N, u, k)][c], 0, 0, 0);
            };
            // the taps every group has in this unit, then the one that only some have (uniform)
            const int some = least_taps(N, u) == 0 ? most_taps(N, u) : least_taps(N, u);
            if (least_taps(N, u) > 0 || u_taps[u] > 0) products(0, some);
            if (items > 0) {
                const int mfmas = some * NC, per = ((ONE ? 24 : 40) * items + mfmas - 1) / mfmas;
#pragma unroll
                for (int i = 0; i < mfmas; ++i) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                    if (per <= 4) __builtin_amdgcn_sched_group_barrier(0x002, 4, 0);
                    else if (per <= 6) __builtin_amdgcn_sched_group_barrier(0x002, 6, 0);
                    else if (per <= 10) __builtin_amdgcn_sched_group_barrier(0x002, 10, 0);
                    else __builtin_amdgcn_sched_group_barrier(0x002, 20, 0);
                }
            }
            if (some < most_taps(N, u) && u_taps[u] > some) products(some, most_taps(N, u));
        }
        __builtin_amdgcn_sched_barrier(0);
    };

    // ---- the walk, in runs where chains are long (fp32): a run's sums are added to the block's copy of dw, which the first one
    // writes.  Registers hold the stage after the one that is multiplied
    const __amdgpu_buffer_rsrc_t rs_out = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(part + (size_t)slice * g.Cout * g.Cin * NN), 0, (int)((size_t)g.Cout * g.Cin * NN * 4), kRawBuffer);
    unsigned again = 0u;  // tiles that hold a sum that is not finite
#pragma unroll 1
    for (;;) {
        clear();
        __syncthreads();
        int slot = 2 * first % a.R;  // ring row of dy row 2*first (even)
        // the dy rows before it, in pairs, and the first stage
        for (int p = -((N - 1) / 2); p < 0; ++p)
            for (int turn = wave; turn < a.dWaves; turn += 8) {
                int off, dst, bit, sh;
                dy_lane(turn, true, off, dst, bit);
                Eight<TIn> q = dy_load(first + p, off, bit, sh);
                dy_write(slot + 2 * p < 0 ? slot + 2 * p + a.R : slot + 2 * p, dst, sh, q);
            }
#pragma unroll
        for (int k = 0; k < ITEMS; ++k) load_item(k, first);
#pragma unroll
        for (int k = 0; k < ITEMS; ++k) {
            write_item(k, 0, slot);
            load_item(k, first + a.TI);
        }
        __syncthreads();
        int buf = 0;
        for (int row = first; row < row1; row += a.TI) {
            int nslot = slot + 2 * a.TI;
            nslot = nslot >= a.R ? nslot - a.R : nslot;
            auto stage = [&](int k) {  // (past the last stage: zeros and rows that no product meets)
                write_item(k, buf ^ 1, nslot);
                load_item(k, row + 2 * a.TI);
            };
            auto all = [&]() {
#pragma unroll
                for (int k = 0; k < ITEMS; ++k) stage(k);
            };
            if (!DEAL && wave >= 4) all();
            multiply(slot, buf, stage);
            if (!DEAL && wave < 4) all();
            __syncthreads();
            slot = nslot;
            buf ^= 1;
        }
        // accumulator register i: output channel 8*(i/4) + 4*kk + (i%4) of the 32, input channel l32
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int k = 0; k < most_taps(N, u); ++k) {
                if (k >= u_taps[u]) continue;  // uniform
                const int tap = u_row[u] * N + u_col[u] + 2 * (u_taps[u] - 1 - k);
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                    f32x16_t v = acc[acc_of(N, u, k)][c];
                    if constexpr (SETS == 2) v += acc[wave_taps(N) + acc_of(N, u, k)][c];
                    if (!wave_finite(v)) again |= 1u << ((u * 3 + k) * NC + c);
                    const int ci = ci0 + (ciw * NC + c) * 32 + l32;
                    const unsigned at = ci < g.Cin ? (unsigned)((((co0 + 4 * kk) * NN + tap) * g.Cin + ci) * 4) : kNoByte;
#pragma unroll
                    for (int q = 0; q < 16; q += 8) {
                        float r[8], before[8];
                        if (first != row0) {  // uniform
#pragma unroll
                            for (int i = 0; i < 8; ++i)
                                before[i] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(
                                    rs_out, at, (unsigned)((8 * ((q + i) / 4) + i % 4) * NN * g.Cin * 4), 0));
                        } else {
#pragma unroll
                            for (int i = 0; i < 8; ++i) before[i] = 0.f;
                        }
#pragma unroll
                        for (int i = 0; i < 8; ++i) {
                            const float w = v[q + i];
                            r[i] = (PARTS == 3 ? w * kPartsDown : w) + before[i];
                        }
#pragma unroll
                        for (int i = 0; i < 8; ++i)
                            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(r[i]), rs_out, at,
                                                                  (unsigned)((8 * ((q + i) / 4) + i % 4) * NN * g.Cin * 4), 0);
                    }
                }
            }
        if (row1 >= row_end) break;
        first = row1;
        row1 = first + a.flushRows < row_end ? first + a.flushRows : row_end;
    }
    float* const out = part + (size_t)slice * g.Cout * g.Cin * NN;
    for (; again != 0u; again &= again - 1) {
        const int t = __builtin_ctz(again), c = t % NC, uk = t / NC, u = uk / 3, k = uk % 3;
        int row_t = 0, col_t = 0;
#pragma unroll
        for (int q = 0; q < U; ++q)
            if (q == u) {
                row_t = u_row[q];
                col_t = u_col[q] + 2 * (u_taps[q] - 1 - k);
            }
        const int com = co0 + l32, cor = com < g.Cout ? com : g.Cout - 1;
        const int cil = ci0 + (ciw * NC + c) * 32 + l32, cir = cil < g.Cin ? cil : g.Cin - 1;
        int ja = (col_t - g.P + 1) >> 1, jb = ((g.OW - 1 - g.P + col_t) >> 1) + 1;  // 0 <= 2j + P - col_t < OW
        if (ja < j0) ja = j0;
        if (jb > g.W) jb = g.W;
        if (jb > j0 + 8 * a.GPR) jb = j0 + 8 * a.GPR;
        f32x16_t sum[1];
#pragma unroll
        for (int i = 0; i < 16; ++i) sum[0][i] = 0.f;
        for (int row = row0; row < row_end && ja < jb; ++row) {
            const int b = image_of(row), i = row - b * a.HS - a.V, oy = 2 * i + g.P - row_t;
            if (i < 0 || oy < 0 || oy >= g.OH) continue;
            const unsigned xo[1] = {(unsigned)(((b * g.Cin + cir) * hw + i * g.W + ja) * ES)};
            sum_tiles<TIn>(sum, rs_dy, (unsigned)(((b * g.Cout + cor) * ohw + oy * g.OW + 2 * ja + g.P - col_t) * ES),
                           2 * ES, rs_x, xo, ES, 0, jb - ja);
        }
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int co = co0 + 8 * (i / 4) + 4 * kk + i % 4;
            if (co < g.Cout && cil < g.Cin) out[((size_t)co * NN + row_t * N + col_t) * g.Cin + cil] = sum[0][i];
        }
    }
}

template <int N, int NC, int STEPS, bool RAGGED, typename TIn>
__global__ __launch_bounds__(T_ROWS) __attribute__((amdgpu_waves_per_eu(2, 2)))
void ukst_grad_weight_mfma_kernel_parts_rows(const TIn* __restrict__ x, const TIn* __restrict__ dy,
                                             float* __restrict__ part, GwRowsArgs a)
{
    grad_weight_rows<N, NC, STEPS, RAGGED, false, TIn>(x, dy, part, a);
}

constexpr int rows_nc(int n) { return n == 4 ? 2 : 1; }
constexpr int rows_ci(int n) { return 32 * rows_nc(n) * (8 / tap_groups(n)); }  // input channels of a block (32 output channels)

// (bf16 operands in rows of whole 16 bytes: the name of the kernel that took them alone)
template <int N, int NC, int STEPS, bool ONE>
__global__ __launch_bounds__(T_ROWS) __attribute__((amdgpu_waves_per_eu(2, 2)))
void ukst_grad_weight_mfma_bf16_kernel_rows(const uint16_t* __restrict__ x, const uint16_t* __restrict__ dy,
                                            float* __restrict__ part, GwRowsArgs a)
{
    grad_weight_rows<N, NC, STEPS, false, ONE, uint16_t>(x, dy, part, a);
}

size_t rows_lds(const GwRowsArgs& a, int es)
{
    return (size_t)(es == 4 ? 3 : 1) * (2 * (2 * (size_t)rows_ci(a.g.n) * a.XP + (size_t)32 * a.DP) + 3 * 256);
}

bool rows_args(const GeomBase& g, int es, int max_slices, int chain, bool bf16_pipe, GwRowsArgs& a, int& steps)
{
    const int N = g.n;
    if (N < 2 || N > 5 || g.Cin < 32 || g.Cout < 32) return false;
    // single buffer descriptors, 32-bit offsets of elements and bytes; pieces of eight elements
    const size_t xe = (size_t)g.B * g.Cin * g.H * g.W, de = (size_t)g.B * g.Cout * g.OH * g.OW;
    if (xe * es > 0x7FFFFFE0u || de * es > 0x7FFFFFE0u || (size_t)g.Cout * g.Cin * N * N * 4 > 0x7FFFFFF0u) return false;
    const int CO_T = 32, CI_T = rows_ci(N);
    a.g = g;
    a.V = N > 2 ? (N - 1) / 2 : g.H > 1 ? 0 : 1;
    a.HS = g.H + a.V;
    const int most = es == 4 ? 4 : 8;
    const int groups = (g.W + 7) / 8;
    a.tilesX = (groups + most - 1) / most;
    a.GPR = (groups + a.tilesX - 1) / a.tilesX;
    a.HC = 8 * a.GPR + 8;
    a.c8 = (16 * a.GPR + N - 2 + 7) / 8;
    a.ragged = g.W % 8 != 0 ? 1 : 0;
    a.dl = a.c8 + (es == 2 ? 1 : 0);
    a.xl = a.GPR + (es == 2 ? a.ragged : 0);
    a.dRowsPerWave = 64 / a.dl;
    a.xRowsPerWave = 64 / a.xl;
    a.dWaves = (2 * CO_T + a.dRowsPerWave - 1) / a.dRowsPerWave;
    a.xWaves = (CI_T + a.xRowsPerWave - 1) / a.xRowsPerWave;
    if ((long long)g.B * a.HS > 0x3FFFFFFF) return false;
    // rows of a stage: up to 4 (fp32) or 8 groups, fewer if LDS asks for it
    int TI = most / a.GPR;
    for (;; --TI) {
        if (TI < 1) return false;
        a.TI = TI;
        steps = (TI * a.GPR + 1) / 2;
        const int least = es == 4 ? 2 : 3;
        steps = steps < least ? least : steps;
        a.R = 4 * TI + (N - 1) / 2 * 2;  // (even: the two dy rows of a row stay together)
        a.DP = a.R * 2 * a.HC;
        if ((a.DP / 8) % 2 == 0) a.DP += 8;
        a.XP = 8 * TI * a.GPR + (TI * a.GPR < 2 * steps ? 8 : 0);  // (with a group of zeros where one is read)
        if ((a.XP / 8) % 2 == 0) a.XP += 8;
        if (TI * a.xWaves <= x_slots(es, CI_T, a.ragged != 0) * 8 && TI * a.dWaves <= dy_slots(es) * 8 && rows_lds(a, es) <= 160 * 1024)
            break;
    }
    a.coTiles = (g.Cout + CO_T - 1) / CO_T;
    a.ciTiles = (g.Cin + CI_T - 1) / CI_T;
    const long long rows = (long long)g.B * a.HS, stages = (rows + a.TI - 1) / a.TI;
    long long want = 256 / ((long long)a.coTiles * a.ciTiles * a.tilesX);
    if (want < 1) want = 1;
    if (want > stages) want = stages;
    if (want * a.tilesX > max_slices) want = max_slices / a.tilesX;
    if (want < 1) return false;
    const long long per = (stages + want - 1) / want;
    a.rowsPerSlice = (int)(per * a.TI);
    a.slicesPerTile = (int)((stages + per - 1) / per);
    a.nSlices = a.slicesPerTile * a.tilesX;
    // chains of at most `chain` pixels (or a little more: one more chain costs as much as it begins with), of equal length;
    // of three parts the pixels that fill up a group count too, six roundings a step
    const double px = (double)a.rowsPerSlice * g.H / a.HS * (es == 2 && g.W < 8 * a.GPR ? g.W : 8 * a.GPR);
    long long runs = (long long)ceil(px / (N == 2 ? 2 : 1) / chain - (es == 4 ? 0.1 : 0.03));
    if (runs < 1) runs = 1;
    if (runs > per) runs = per;
    const long long perRun = (per + runs - 1) / runs;
    a.flushRows = (int)(perRun * TI);
    // Against the kernels before it (ratio of the times, 110 drawn layers each): fp32 from four stages a chain on 1.1 to 2.1, with
    // fewer 0.5 to 1.1 (a chain begins with an empty ring); tiles of input channels less than 0.6 full 0.86 to 1.04.  bf16 layers
    // that ran on the bf16 pipe 1.2 to 2.0 with most of the multiplications at work, 0.77 to 1.08 with less than 0.6 of them;
    // layers that ran on the fp32 pipe 1.1 to 5.2, whatever their size
    const double filled = (double)g.Cin / ((double)a.ciTiles * CI_T);
    const double busy = filled * g.W / (8. * a.GPR * a.tilesX) * (TI * a.GPR) / (2. * steps);
    if (es == 4 ? perRun < 4 || filled < 0.6 || busy < 0.5
                : (perRun < 4 && (runs > 1 || bf16_pipe)) || (busy < 0.6 && bf16_pipe))
        return false;
    a.dHS = make_fastdiv((unsigned)a.HS);
    a.dGPR = make_fastdiv((unsigned)a.GPR);
    a.dDL = make_fastdiv((unsigned)a.dl);
    a.dXL = make_fastdiv((unsigned)a.xl);
    a.dDWaves = make_fastdiv((unsigned)a.dWaves);
    a.dXWaves = make_fastdiv((unsigned)a.xWaves);
    return true;
}

template <int N, int STEPS, bool RAGGED, bool ONE, typename TIn>
hipError_t launch_rows_t(const GwRowsArgs& a, const void* x, const void* dy, float* part, hipStream_t stream)
{
    const size_t lds = rows_lds(a, (int)sizeof(TIn));
    void (*kernel)(const TIn*, const TIn*, float*, GwRowsArgs);
    if constexpr (sizeof(TIn) == 2 && N <= 4 && !RAGGED) kernel = ukst_grad_weight_mfma_bf16_kernel_rows<N, rows_nc(N), STEPS, ONE>;
    else kernel = ukst_grad_weight_mfma_kernel_parts_rows<N, rows_nc(N), STEPS, RAGGED, TIn>;
    const hipError_t e = hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kernel, dim3((unsigned)((long long)a.nSlices * a.coTiles * a.ciTiles)), dim3(T_ROWS), lds, stream,
                       (const TIn*)x, (const TIn*)dy, part, a);
    return hipGetLastError();
}

template <int N, typename TIn>
hipError_t launch_rows(const GwRowsArgs& a, int steps, const void* x, const void* dy, float* part, hipStream_t stream)
{
    if constexpr (sizeof(TIn) == 4) {
        return a.ragged ? launch_rows_t<N, 2, true, false, TIn>(a, x, dy, part, stream)
                        : launch_rows_t<N, 2, false, false, TIn>(a, x, dy, part, stream);
    } else {
        if (a.ragged)
            return steps == 3 ? launch_rows_t<N, 3, true, false, TIn>(a, x, dy, part, stream)
                              : launch_rows_t<N, 4, true, false, TIn>(a, x, dy, part, stream);
        if constexpr (N == 4) {
            // dy rows of whole 16 bytes, the first column of a tile one element before them
            if (a.g.OW % 8 == 0 && ((uintptr_t)dy & 15) == 0 && ((a.g.P - (N - 1)) & 7) == 7)
                return steps == 3 ? launch_rows_t<N, 3, false, true, TIn>(a, x, dy, part, stream)
                                  : launch_rows_t<N, 4, false, true, TIn>(a, x, dy, part, stream);
        }
        return steps == 3 ? launch_rows_t<N, 3, false, false, TIn>(a, x, dy, part, stream)
                          : launch_rows_t<N, 4, false, false, TIn>(a, x, dy, part, stream);
    }
}

}  // namespace

int grad_weight_rows_slices(const GeomBase& g, int es, int max_slices, int chain, bool bf16_pipe, int* runs)
{
    GwRowsArgs a;
    int steps;
    if (!rows_args(g, es, max_slices, chain, bf16_pipe, a, steps)) return 0;
    if (runs) *runs = (a.rowsPerSlice + a.flushRows - 1) / a.flushRows;
    return a.nSlices;
}

hipError_t launch_grad_weight_rows(const GeomBase& g, const void* x, const void* dy, float* part, int es, int max_slices,
                                   int chain, bool bf16_pipe, hipStream_t stream)
{
    GwRowsArgs a;
    int steps;
    if (!rows_args(g, es, max_slices, chain, bf16_pipe, a, steps)) return hipErrorInvalidValue;
    switch (g.n * 8 + es) {
        case 20: return launch_rows<2, float>(a, steps, x, dy, part, stream);
        case 18: return launch_rows<2, uint16_t>(a, steps, x, dy, part, stream);
        case 28: return launch_rows<3, float>(a, steps, x, dy, part, stream);
        case 26: return launch_rows<3, uint16_t>(a, steps, x, dy, part, stream);
        case 36: return launch_rows<4, float>(a, steps, x, dy, part, stream);
        case 34: return launch_rows<4, uint16_t>(a, steps, x, dy, part, stream);
        case 44: return launch_rows<5, float>(a, steps, x, dy, part, stream);
        case 42: return launch_rows<5, uint16_t>(a, steps, x, dy, part, stream);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace ukst
