// Gradient with respect to the kernel of wide layers on the bf16 matrix pipe from bf16 parts (ukst_parts.h):
// fp32 operands as three exact parts, bf16 operands as one; n = 3, 4, rows of at least 16 pixels, any length.
//
// The product is that of the other kernel gradients, DW_tap[co][ci] += sum_pixel DY_tap[co][pixel] * X[ci][pixel],
// with the pixel axis as the K axis of v_mfma_f32_32x32x16_bf16: a lane's operand is 8 consecutive pixels of one
// channel, x as it lies in memory, dy rows split by column parity on their way into LDS, the one-element shift
// between the taps of a column parity made in registers.
//
// Block = 4 waves on 32 output x 64 input channels, two blocks per compute unit (LDS and registers), so that one's
// staging and splitting run beside the other's MFMAs.  Wave w owns input channels 32*(w & 1) .. +31; the other bit
// halves the work: n = 4 two tap rows each (8 accumulator tiles), n = 3 all nine taps and every other K step, the
// two halves added through LDS at the end.  (Nine taps dealt to four waves leave a quarter of the
// matrix pipes idle.)  Of a 16-pixel step at n = 3 a wave reads 23 KiB of fragments for 54 MFMAs of three parts,
// about 0.4 of the LDS rate; staging a piece of four elements costs about 30 vector instructions and is what keeps
// the pipes from more.  No more copies of dw than the fp32-pipe kernel writes, in the same layout.  fp32 pipe -> this
// kernel, with the sum of the copies: fp32 32 x 128 -> 128 channels, 63 x 63, n = 3 509 -> 343 us, 64 x 64, n = 4 724 -> 544;
// bf16 16 x 64 -> 64, 61 x 61, n = 3 / 4 96 -> 59 / 122 -> 55.
#include "ukst_parts.h"

namespace ukst {
namespace {

struct GwPartsArgs {
    GeomBase g;
    int TJ, logTJ, TI, logTI, TB, TR, logPix;  // stage: TR (image, pixel row) pairs x TJ columns
    int LR, HC, cols, DP, XP;                  // dy rows per image, half row, row, channel strides (elements)
    int tilesX, tilesY, nStages, stagesPerSlice, nSlices, coTiles, ciTiles;
    int c4, npass;                             // four-column pieces per dy row, passes of 64 lanes per channel
    FastDiv dC4, dLR;
};

constexpr int CI_T = 64;

// four raw elements: fp32 values or bf16 bit patterns, one per dword
struct Piece { unsigned v[4]; };
// moved sh places up (sh > 0) or down, zeros moving in; 0 < |sh| < 4
__device__ __forceinline__ Piece shifted(const Piece& q, int sh)
{
    Piece r;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        unsigned v = 0u;
#pragma unroll
        for (int e = 0; e < 4; ++e) v = k - sh == e ? q.v[e] : v;
        r.v[k] = v;
    }
    return r;
}
template <typename TIn>
__device__ __forceinline__ Piece load_piece(const __amdgpu_buffer_rsrc_t& rs, unsigned voff, unsigned soff)
{
    if constexpr (sizeof(TIn) == 4) {
        const u4v_t t = __builtin_amdgcn_raw_buffer_load_b128(rs, voff, soff, 0);
        return Piece{{t.x, t.y, t.z, t.w}};
    } else {
        const u2v_t t = __builtin_amdgcn_raw_buffer_load_b64(rs, voff, soff, 0);
        return Piece{{t.x & 0xFFFFu, t.x >> 16, t.y & 0xFFFFu, t.y >> 16}};
    }
}
// two elements -> PARTS packed dwords
template <int PARTS>
__device__ __forceinline__ void pair_parts(unsigned a, unsigned b, unsigned (&p)[PARTS])
{
    if constexpr (PARTS == 3) split_pair(__uint_as_float(a), __uint_as_float(b), p[0], p[1], p[2]);
    else p[0] = a | (b << 16);
}

template <int N, typename TIn>
__global__ __launch_bounds__(256, 2) void ukst_grad_weight_mfma_kernel_parts(const TIn* __restrict__ x,
                                                                            const TIn* __restrict__ dy,
                                                                            float* __restrict__ part, GwPartsArgs a)
{
    constexpr int PARTS = sizeof(TIn) == 4 ? 3 : 1;
    constexpr int ES = (int)sizeof(TIn);
    constexpr int NN = N * N;
    constexpr bool KHALF = N == 3;               // the waves' second bit: K steps, or tap rows
    constexpr int RW = KHALF ? N : N / 2;        // tap rows per wave
    typedef PartProducts<PARTS> PP;
    extern __shared__ __align__(16) unsigned char lds[];
    const GeomBase& g = a.g;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, kk = lane >> 5, wc = wave & 1, wh = wave >> 1;
    const int XPB = CI_T * a.XP * 2, DPB = 32 * a.DP * 2;  // bytes of one part's tiles
    unsigned char* const xs = lds;                         // [part][ci][pixel]
    unsigned char* const dys = lds + PARTS * XPB;          // [part][co][row][column parity][column / 2]
    const __amdgpu_buffer_rsrc_t rs_x = __builtin_amdgcn_make_buffer_rsrc(
        (void*)x, 0, (int)((size_t)g.B * g.Cin * g.H * g.W * ES), kRawBuffer);
    const __amdgpu_buffer_rsrc_t rs_dy = __builtin_amdgcn_make_buffer_rsrc(
        (void*)dy, 0, (int)((size_t)g.B * g.Cout * g.OH * g.OW * ES), kRawBuffer);

    int bid = xcd_contiguous(blockIdx.x, gridDim.x);  // neighbours in this numbering share an L2
    const int cit = bid % a.ciTiles; bid /= a.ciTiles;
    const int cot = bid % a.coTiles;
    const int slice = bid / a.coTiles;
    const int co0 = cot * 32, ci0 = cit * CI_T;

    f32x16_t acc[RW][N];
#pragma unroll
    for (int r = 0; r < RW; ++r)
#pragma unroll
        for (int c = 0; c < N; ++c)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[r][c][i] = 0.f;

    const int a_lane = (l32 * a.DP + 8 * kk) * 2, b_lane = ((wc * 32 + l32) * a.XP + 8 * kk) * 2;
    const int st0 = slice * a.stagesPerSlice;
    const int st_end = st0 + a.stagesPerSlice < a.nStages ? st0 + a.stagesPerSlice : a.nStages;
    const int per_co = a.TB * a.LR * a.c4;
    const unsigned co_bytes = (unsigned)(g.OH * g.OW * ES);
    int turn = 0;  // K steps so far, of all rows (KHALF)
    for (int st = st0; st < st_end; ++st) {
        int t = st;
        const int tx = t % a.tilesX; t /= a.tilesX;
        const int ty = t % a.tilesY;
        const int b0 = t / a.tilesY * a.TB, i0 = ty * a.TI, j0 = tx * a.TJ;
        const int oy_base = 2 * i0 + g.P - (N - 1), ox_base = 2 * j0 + g.P - (N - 1);
        __syncthreads();
        // every wave stages a quarter of the channels: what depends on the lane (row, piece, validity) is worked
        // out once per pass, the channel enters through the scalar offset.  Rows, images and channels that do not
        // exist arrive as zeros (out-of-range offset); a piece that hangs over an end of its row is fetched from
        // inside the row and shifted into place.
        constexpr int GRP = 4;
        unsigned dvoff;
        int dsh, ddst;
        auto lane_pass = [&](int pp) {
            const int idx = lane + 64 * pp;
            const int rem = fdiv(idx, a.dC4), m = idx - rem * a.c4;
            const int bl = fdiv(rem, a.dLR), rr = rem - bl * a.LR;
            const int b = b0 + bl, oy = oy_base + rr, ox = ox_base + 4 * m;
            const bool ok = idx < per_co && b < g.B && oy >= 0 && oy < g.OH && ox + 3 >= 0 && ox < g.OW;
            const int oxl = ox < 0 ? 0 : (ox > g.OW - 4 ? g.OW - 4 : ox);
            dsh = oxl - ox;
            dvoff = ok ? (unsigned)((((b * g.Cout) * g.OH + oy) * g.OW + oxl) * ES) : kNoByte;
            ddst = idx < per_co ? (rem * a.cols + 2 * m) * 2 : -1;
        };
        auto load_group = [&](int h, Piece (&q)[GRP]) {
#pragma unroll
            for (int c = 0; c < GRP; ++c) {
                const int co = co0 + wave * 8 + h * GRP + c;  // uniform
                const bool on = co < g.Cout;
                q[c] = load_piece<TIn>(rs_dy, on ? dvoff : kNoByte, on ? (unsigned)co * co_bytes : 0u);
            }
        };
        auto write_group = [&](int h, int sh, int dst, const Piece (&q)[GRP]) {
            if (dst < 0) return;
#pragma unroll
            for (int c = 0; c < GRP; ++c) {
                unsigned char* const base = dys + (wave * 8 + h * GRP + c) * a.DP * 2 + dst;
                const Piece v = sh != 0 ? shifted(q[c], sh) : q[c];
                unsigned ev[PARTS], od[PARTS];
                pair_parts<PARTS>(v.v[0], v.v[2], ev);
                pair_parts<PARTS>(v.v[1], v.v[3], od);
#pragma unroll
                for (int i = 0; i < PARTS; ++i) {
                    *reinterpret_cast<unsigned*>(base + i * DPB) = ev[i];
                    *reinterpret_cast<unsigned*>(base + i * DPB + a.HC * 2) = od[i];
                }
            }
        };
        Piece qa[GRP], qb[GRP];
        lane_pass(0);
        load_group(0, qa);
        {
            const int logCPC = a.logPix - 2, CPC = 1 << logCPC;  // pieces per channel
            const int xpasses = (16 << logCPC) >> 6;             // >= 1: a stage holds at least 16 pixels
            for (int p0 = 0; p0 < xpasses; p0 += 4) {
                Piece q[4];
                int dst[4], sh[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    dst[u] = -1;
                    sh[u] = 0;
                    if (p0 + u < xpasses) {
                        const int flat = lane + 64 * (p0 + u);
                        const int cl = wave * 16 + (flat >> logCPC), pix = (flat & (CPC - 1)) << 2;
                        const int tr = pix >> a.logTJ, lj = pix & (a.TJ - 1);
                        const int b = b0 + (tr >> a.logTI), i = i0 + (tr & (a.TI - 1)), j = j0 + lj, ci = ci0 + cl;
                        const bool ok = ci < g.Cin && b < g.B && i < g.H && j < g.W;
                        const int jl = j > g.W - 4 ? g.W - 4 : j;
                        sh[u] = jl - j;
                        q[u] = load_piece<TIn>(
                            rs_x, ok ? (unsigned)((((b * g.Cin + ci) * g.H + i) * g.W + jl) * ES) : kNoByte, 0u);
                        dst[u] = (cl * a.XP + pix) * 2;
                    }
                }
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    if (dst[u] >= 0) {
                        const Piece v = sh[u] <= -4 ? Piece{{0u, 0u, 0u, 0u}} : sh[u] != 0 ? shifted(q[u], sh[u]) : q[u];
                        unsigned lo[PARTS], hi[PARTS];
                        pair_parts<PARTS>(v.v[0], v.v[1], lo);
                        pair_parts<PARTS>(v.v[2], v.v[3], hi);
#pragma unroll
                        for (int i = 0; i < PARTS; ++i)
                            *reinterpret_cast<u2v_t*>(xs + i * XPB + dst[u]) = u2v_t{lo[i], hi[i]};
                    }
            }
        }
#pragma unroll 1
        for (int pp = 0; pp < a.npass; ++pp) {
            const int sh_c = dsh, dst_c = ddst;
            load_group(1, qb);
            write_group(0, sh_c, dst_c, qa);
            if (pp + 1 < a.npass) {
                lane_pass(pp + 1);
                load_group(0, qa);
            }
            write_group(1, sh_c, dst_c, qb);
        }
        __syncthreads();
        // K steps of 16 pixels along a row; pixels past the end of the row are zeros in x
        const int wj = g.W - j0 < a.TJ ? g.W - j0 : a.TJ;
        const int steps = (wj + 15) >> 4;
        for (int tr = 0; tr < a.TR; ++tr) {
            const int bl = tr >> a.logTI, li = tr & (a.TI - 1);
            if (b0 + bl >= g.B || i0 + li >= g.H) continue;  // uniform
            const unsigned char* ap = dys + a_lane + (bl * a.LR + 2 * li) * a.cols * 2;
            const unsigned char* bp = xs + b_lane + tr * a.TJ * 2;
            for (int sp = 0; sp < steps; ++sp) {
                if (KHALF && (turn++ & 1) != wh) continue;  // uniform
                bf16x8_t bv[PARTS];
#pragma unroll
                for (int i = 0; i < PARTS; ++i) bv[i] = *reinterpret_cast<const bf16x8_t*>(bp + i * XPB + 32 * sp);
#pragma unroll
                for (int r = 0; r < RW; ++r) {
                    const int ta = KHALF ? r : wh * RW + r;  // tap row
                    const unsigned char* const rp = ap + (N - 1 - ta) * a.cols * 2 + 32 * sp;
                    bf16x8_t av[N][PARTS];
#pragma unroll
                    for (int i = 0; i < PARTS; ++i) {
                        u4v_t h[2];
                        unsigned next[2];
#pragma unroll
                        for (int p = 0; p < 2; ++p) {
                            h[p] = *reinterpret_cast<const u4v_t*>(rp + i * DPB + p * a.HC * 2);
                            if (p < N - 2) next[p] = *reinterpret_cast<const unsigned*>(rp + i * DPB + p * a.HC * 2 + 16);
                        }
#pragma unroll
                        for (int c = 0; c < N; ++c) {  // tap column
                            const int p = (N - 1 - c) & 1;
                            u4v_t v = h[p];
                            if ((N - 1 - c) >> 1)
                                v = u4v_t{__builtin_amdgcn_alignbit(h[p].y, h[p].x, 16),
                                          __builtin_amdgcn_alignbit(h[p].z, h[p].y, 16),
                                          __builtin_amdgcn_alignbit(h[p].w, h[p].z, 16),
                                          __builtin_amdgcn_alignbit(next[p], h[p].w, 16)};
                            av[c][i] = __builtin_bit_cast(bf16x8_t, v);
                        }
                    }
#pragma unroll
                    for (int m = 0; m < PP::count; ++m)
#pragma unroll
                        for (int c = 0; c < N; ++c)
                            acc[r][c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av[c][PP::a[m]], bv[PP::b[m]], acc[r][c],
                                                                               0, 0, 0);
                }
            }
        }
    }

    float* out = part + (size_t)slice * g.Cout * g.Cin * NN;
    if constexpr (KHALF) {
        __syncthreads();  // every wave is done with the tiles
        float* const lf = reinterpret_cast<float*>(lds);  // [wc][tap][register][lane]
        if (wh == 1) {
#pragma unroll
            for (int r = 0; r < RW; ++r)
#pragma unroll
                for (int c = 0; c < N; ++c)
#pragma unroll
                    for (int i = 0; i < 16; ++i) lf[((wc * NN + r * N + c) * 16 + i) * 64 + lane] = acc[r][c][i];
        }
        __syncthreads();
        if (wh == 0) {
#pragma unroll
            for (int r = 0; r < RW; ++r)
#pragma unroll
                for (int c = 0; c < N; ++c)
#pragma unroll
                    for (int i = 0; i < 16; ++i) acc[r][c][i] += lf[((wc * NN + r * N + c) * 16 + i) * 64 + lane];
        }
    }
    const bool owner = !KHALF || wh == 0;  // uniform
    // tiles that hold a sum that is not finite (ukst_parts.h)
    unsigned tiles = 0u;
    if (owner) {
#pragma unroll
        for (int r = 0; r < RW; ++r)
#pragma unroll
            for (int c = 0; c < N; ++c)
                if (!wave_finite(acc[r][c])) tiles |= 1u << (r * N + c);
    }
    // accumulator register i: output channel 8*(i/4) + 4*kk + (i%4) of the 32, input channel l32
    if (owner) {
        const int ci = ci0 + wc * 32 + l32;
#pragma unroll
        for (int r = 0; r < RW; ++r)
#pragma unroll
            for (int c = 0; c < N; ++c) {
                const int tap = (KHALF ? r : wh * RW + r) * N + c;
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const int co = co0 + 8 * (i / 4) + 4 * kk + (i % 4);
                    const float v = PARTS == 3 ? acc[r][c][i] * kPartsDown : acc[r][c][i];
                    if (co < g.Cout && ci < g.Cin) out[((size_t)co * NN + tap) * g.Cin + ci] = v;
                }
            }
    }

    for (; tiles != 0u; tiles &= tiles - 1) {
        const int t = __builtin_ctz(tiles), tap = (KHALF ? 0 : wh * RW * N) + t, ta = tap / N, tc = tap % N;
        const int co = co0 + l32 < g.Cout ? co0 + l32 : g.Cout - 1, cil = ci0 + wc * 32 + l32;
        const int j_lo = (tc - g.P + 1) >> 1, j_hi = ((g.OW - 1 - g.P + tc) >> 1) + 1;  // 0 <= 2j + P - tc < OW
        f32x16_t sum[1];
#pragma unroll
        for (int i = 0; i < 16; ++i) sum[0][i] = 0.f;
        for (int st = st0; st < st_end; ++st) {
            int t = st;
            const int tx = t % a.tilesX; t /= a.tilesX;
            const int ty = t % a.tilesY, b0 = t / a.tilesY * a.TB;
            int j0 = tx * a.TJ, j1 = j0 + a.TJ < g.W ? j0 + a.TJ : g.W;
            if (j0 < j_lo) j0 = j_lo;
            if (j1 > j_hi) j1 = j_hi;
            if (j0 >= j1) continue;
            for (int tr = 0; tr < a.TR; ++tr) {
                const int b = b0 + (tr >> a.logTI), i = ty * a.TI + (tr & (a.TI - 1));
                const int oy = 2 * i + g.P - ta, ci = cil < g.Cin ? cil : g.Cin - 1;
                if (b >= g.B || i >= g.H || oy < 0 || oy >= g.OH) continue;
                const unsigned xo[1] = {(unsigned)((((b * g.Cin + ci) * g.H + i) * g.W + j0) * ES)};
                sum_tiles<TIn>(sum, rs_dy, (unsigned)((((b * g.Cout + co) * g.OH + oy) * g.OW + 2 * j0 + g.P - tc) * ES),
                               2 * ES, rs_x, xo, ES, 0, j1 - j0);
            }
        }
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int c = co0 + 8 * (i / 4) + 4 * kk + i % 4;
            if (c < g.Cout && cil < g.Cin) out[((size_t)c * NN + tap) * g.Cin + cil] = sum[0][i];
        }
    }
}

int log2_of(int v) { int l = 0; while ((1 << l) < v) ++l; return l; }

size_t lds_bytes(const GwPartsArgs& a, int es)
{
    const size_t tiles = (size_t)(es == 4 ? 3 : 1) * 2 * (CI_T * a.XP + 32 * a.DP);
    const size_t halves = a.g.n == 3 ? (size_t)2 * a.g.n * a.g.n * 4096 : 0;  // where the K halves meet
    return tiles > halves ? tiles : halves;
}

bool make_args(const GeomBase& g, int es, int max_slices, GwPartsArgs& a)
{
    const int least = es == 2 ? 16 : 32;  // (fp32: see gw_mfma_args)
    if (g.Cin < least || g.Cout < least || g.n < 3 || g.n > 4 || g.W < 16 || g.OW < 4) return false;
    // (n = 2, 64 x 64 maps: 290 against 289 us, four taps do not pay for their staging)  Few pixels leave the
    // slices a stage or two and gain nothing: 64 -> 64 channels, 2 images of 16 x 16, n = 3 18.8 against 19.2 us, 4 of
    // 20 x 33 28.2 against 28.0, 64 of 16 x 16 with n = 4 58 against 46
    if ((long long)g.B * g.H * g.W < 8192) return false;
    // fp32: rows that fill less than 5/8 of their column tiles multiply too many zeros for n = 4 (64 images of 17 x 17,
    // 128 -> 128 channels, n = 3 / 4: 111 / 157 us on the fp32 pipe against 101 / 156; 64 of 18 x 18 115 / 162 against
    // 107 / 163; 32 of 33 x 33, 64 -> 64, n = 3 83 against 75; 64 of 20 x 20, 128 -> 128, 129 / 186 against 115 / 178; 40
    // of 31 x 31, n = 3 167 against 118)
    const int tiled_cols = g.W > 16 ? (g.W + 31) / 32 * 32 : 16;
    if (es == 4 && g.W * 8 < tiled_cols * 5) return false;
    // single buffer descriptors, 32-bit byte offsets
    if ((size_t)g.B * g.Cin * g.H * g.W * es > 0x7FFFFFF0u || (size_t)g.B * g.Cout * g.OH * g.OW * es > 0x7FFFFFF0u)
        return false;
    const int N = g.n;
    a.g = g;
    a.TJ = g.W > 16 ? 32 : 16;
    a.logTJ = log2_of(a.TJ);
    a.HC = a.TJ + 8;  // half rows: TJ + 1 columns are read, at most TJ + 4 written, whole 16-byte slots
    a.cols = 2 * a.HC;
    a.c4 = (2 * a.TJ + N - 2 + 3) / 4;
    const bool few = few_channels(g);
    for (int TR = (few ? kFewStage : 512) / a.TJ;; TR >>= 1) {
        if (TR < 1) return false;
        a.TR = TR;
        a.TI = 1 << log2_of(g.H < TR ? g.H : TR);
        a.TB = TR / a.TI;
        a.LR = 2 * a.TI + N - 2;
        // channel strides: an odd number of 16-byte slots, so that the 16 lanes of a read pass fall into
        // different bank groups
        a.DP = a.TB * a.LR * a.cols;
        if ((a.DP / 8) % 2 == 0) a.DP += 8;
        a.XP = TR * a.TJ + 8;
        if (lds_bytes(a, es) <= 78 * 1024) break;
    }
    a.logTI = log2_of(a.TI);
    a.logPix = log2_of(a.TR * a.TJ);
    a.tilesX = (g.W + a.TJ - 1) / a.TJ;
    a.tilesY = (g.H + a.TI - 1) / a.TI;
    const long long stages = (long long)a.tilesX * a.tilesY * ((g.B + a.TB - 1) / a.TB);
    if (stages > 0x7fffffffLL) return false;
    a.nStages = (int)stages;
    a.coTiles = (g.Cout + 31) / 32;
    a.ciTiles = (g.Cin + CI_T - 1) / CI_T;
    long long want = 512 / ((long long)a.coTiles * a.ciTiles);
    if (few) want = few_slices(g, stages * a.TR * a.TJ, want);
    if (want < 1) want = 1;
    if (want > stages) want = stages;
    if (!few && want > max_slices) want = max_slices;
    a.stagesPerSlice = (int)((stages + want - 1) / want);
    a.nSlices = (int)((stages + a.stagesPerSlice - 1) / a.stagesPerSlice);
    if (few && (long long)a.stagesPerSlice * a.TR * a.TJ > kFewChainMax) return false;
    a.npass = (a.TB * a.LR * a.c4 + 63) / 64;
    a.dC4 = make_fastdiv((unsigned)a.c4);
    a.dLR = make_fastdiv((unsigned)a.LR);
    return true;
}

template <int N, typename TIn>
hipError_t launch(const GwPartsArgs& a, const void* x, const void* dy, float* part, hipStream_t stream)
{
    const size_t lds = lds_bytes(a, (int)sizeof(TIn));
    const hipError_t e = hipFuncSetAttribute((const void*)ukst_grad_weight_mfma_kernel_parts<N, TIn>,
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((ukst_grad_weight_mfma_kernel_parts<N, TIn>),
                       dim3((unsigned)((long long)a.nSlices * a.coTiles * a.ciTiles)), dim3(256), lds, stream,
                       (const TIn*)x, (const TIn*)dy, part, a);
    return hipGetLastError();
}

}  // namespace

int grad_weight_parts_slices(const GeomBase& g, int es, int max_slices)
{
    GwPartsArgs a;
    return make_args(g, es, max_slices, a) ? a.nSlices : 0;
}

hipError_t launch_grad_weight_parts(const GeomBase& g, const void* x, const void* dy, float* part, int es,
                                    int max_slices, hipStream_t stream)
{
    GwPartsArgs a;
    if (!make_args(g, es, max_slices, a)) return hipErrorInvalidValue;
    if (es == 4)
        return g.n == 3 ? launch<3, float>(a, x, dy, part, stream) : launch<4, float>(a, x, dy, part, stream);
    return g.n == 3 ? launch<3, uint16_t>(a, x, dy, part, stream) : launch<4, uint16_t>(a, x, dy, part, stream);
}

}  // namespace ukst
