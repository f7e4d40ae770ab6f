// The two generalisations Sec. 5 of the paper points to, on the vector ALUs, one kernel for both (layers of at
// least 16 input and 8 output channels run on the matrix cores where they fit: ukst_general_mfma.hip):
//
//  * transpose convolution with a general stride s: s-1 zeros are inserted between neighbouring
//    pixels (Algorithm 1 with s in place of 2), so tap a of output row oy meets a pixel only where
//    oy + a - P is a multiple of s.  Algorithm 2 carries over with s*s classes instead of four:
//    row class r = (P - oy) mod s, taps r, r+s, r+2s, ... (the sub-kernel k_rc[u][v] =
//    K[r+s*u][c+s*v]), tap r+s*u reads input row (oy + r - P)/s + u.  Each thread selects the
//    class of its output pixel at run time and never touches an inserted zero.
//  * dilated convolution with dilation d: here the KERNEL is the bed of nails (d-1 zeros between
//    neighbouring taps), and the computation pattern is applied to the segregated INPUT: output
//    pixel (oy, ox) only meets input pixels congruent to (oy - P, ox - P) modulo d, i.e. one of the
//    d*d sub-sampled input maps, with the unmodified n x n kernel.  A thread reads its sub-map in
//    place (input row oy - P + d*a for tap a); the sub-maps are never built.
//
// Both are the gather  y[oy][ox] = sum_ci sum_{u<Tr} sum_{v<Tc} x[i0 + u*xs][j0 + v*xs] *
// w[r + u*ws][c + v*ws]  with (xs, ws) = (1, s) or (d, 1).  Block = 32 x 8 output pixels x 8
// output channels; the weights of 8 input channels at a time sit in LDS as [ci][tap][co] and are
// read as two 16-byte broadcasts per input value; out-of-range window pixels (the padding) are
// skipped by a bounds predicate.
#include "ukst_internal.h"

namespace ukst {
namespace {

constexpr int CO_BLK = 8;   // output channels per thread
constexpr int CI_CH = 8;    // input channels per weight stage
constexpr int MAX_NN = 49;  // n <= 7

struct GenArgs {
    int B, Cin, Cout, H, W, n, P, k, OH, OW;
    int dilated;  // 0: stride-k transpose convolution, 1: dilation-k convolution
    int tilesX, tilesY, coBlocks;
};

__device__ __forceinline__ float to_f32(float v) { return v; }
__device__ __forceinline__ float to_f32(uint16_t v) { return __uint_as_float((unsigned)v << 16); }

template <typename TIn>
__global__ __launch_bounds__(256) void ukst_general_kernel(const TIn* __restrict__ x,
                                                          const TIn* __restrict__ w,
                                                          float* __restrict__ y, GenArgs a)
{
    __shared__ __align__(16) float wl[CI_CH * MAX_NN * CO_BLK];
    const int tid = threadIdx.x;
    int bid = blockIdx.x;
    const int tile = bid % (a.tilesX * a.tilesY); bid /= a.tilesX * a.tilesY;
    const int cob = bid % a.coBlocks;
    const int b = bid / a.coBlocks;
    const int ox = (tile % a.tilesX) * 32 + (tid & 31);
    const int oy = (tile / a.tilesX) * 8 + (tid >> 5);
    const bool valid = ox < a.OW && oy < a.OH;
    const int co0 = cob * CO_BLK;
    const int n = a.n, NN = n * n, k = a.k;

    // run-time class selection: first tap (r, c), tap stride, window start, input stride, taps
    int r = 0, c = 0, i0, j0, Tr, Tc, xstep, wstep;
    if (a.dilated) {
        i0 = oy - a.P; j0 = ox - a.P; Tr = Tc = n; xstep = k; wstep = 1;
    } else {
        r = ((a.P - oy) % k + k) % k;
        c = ((a.P - ox) % k + k) % k;
        i0 = (oy + r - a.P) / k;  // exact: the numerator is a multiple of k (also when negative)
        j0 = (ox + c - a.P) / k;
        Tr = r < n ? (n - r + k - 1) / k : 0;
        Tc = c < n ? (n - c + k - 1) / k : 0;
        xstep = 1; wstep = k;
    }

    float acc[CO_BLK];
#pragma unroll
    for (int co = 0; co < CO_BLK; ++co) acc[co] = 0.f;

    for (int ci0 = 0; ci0 < a.Cin; ci0 += CI_CH) {
        __syncthreads();
        for (int e = tid; e < CI_CH * NN * CO_BLK; e += 256) {
            const int co = e % CO_BLK, t = (e / CO_BLK) % NN, ci = e / (CO_BLK * NN);
            float v = 0.f;
            if (co0 + co < a.Cout && ci0 + ci < a.Cin)
                v = to_f32(w[((size_t)(co0 + co) * a.Cin + ci0 + ci) * NN + t]);
            wl[e] = v;
        }
        __syncthreads();
        if (!valid) continue;
        const int nci = a.Cin - ci0 < CI_CH ? a.Cin - ci0 : CI_CH;
        for (int ci = 0; ci < nci; ++ci) {
            const TIn* xp = x + ((size_t)b * a.Cin + ci0 + ci) * a.H * a.W;
            for (int u = 0; u < Tr; ++u) {
                const int i = i0 + u * xstep;
                if (i < 0 || i >= a.H) continue;
                for (int v = 0; v < Tc; ++v) {
                    const int j = j0 + v * xstep;
                    if (j < 0 || j >= a.W) continue;
                    const float xv = to_f32(xp[(size_t)i * a.W + j]);
                    const int tap = (r + u * wstep) * n + (c + v * wstep);
                    const float4* wp = reinterpret_cast<const float4*>(&wl[(ci * NN + tap) * CO_BLK]);
                    const float4 w0 = wp[0], w1 = wp[1];
                    acc[0] = fmaf(xv, w0.x, acc[0]); acc[1] = fmaf(xv, w0.y, acc[1]);
                    acc[2] = fmaf(xv, w0.z, acc[2]); acc[3] = fmaf(xv, w0.w, acc[3]);
                    acc[4] = fmaf(xv, w1.x, acc[4]); acc[5] = fmaf(xv, w1.y, acc[5]);
                    acc[6] = fmaf(xv, w1.z, acc[6]); acc[7] = fmaf(xv, w1.w, acc[7]);
                }
            }
        }
    }
    if (!valid) return;
#pragma unroll
    for (int co = 0; co < CO_BLK; ++co)
        if (co0 + co < a.Cout)
            y[(((size_t)b * a.Cout + co0 + co) * a.OH + oy) * a.OW + ox] = acc[co];
}

}  // namespace

// Layers of few tiles (ukst_small_kernel.h), in 32 x 32 tiles of a dilated layer, 16 x 16 tiles of every class of a strided
// one.  Up to these the kernel on parts, whose blocks take 64 channels x 256 lattice pixels of one class, is a serial chain
// on a part of the chip (us, its time against the small tiles': dilation 2, 192 -> 120 channels, 18 of 9 x 9, n = 5 251 / 28;
// dilation 3, 72 -> 39, 2 of 16 x 85, n = 3 128 / 10; stride 4, 136 -> 96, 2 of 14 x 14, n = 3 29.3 / 9.5), beyond them it
// catches up (fp32 dilation 2, 328 -> 23, n = 3, 2940 tiles 178 / 198; bf16 40 -> 136, n = 3, 912 tiles 41 / 38, 24 -> 272, n = 4, 1440
// tiles 23.1 / 25.5; stride 3, 16 -> 40, n = 5, 756 tiles 13.1 / 17.9, bf16 96 -> 214, 1638 tiles 24.5 / 49)
static bool prefer_small(const SmallProblem& q)
{
    if (q.K < 16 || q.M < 8 || q.n < 2 || q.n > 5) return false;
    if (q.op == SmallOp::strided && q.step != 3 && q.step != 4) return false;
    const long long tiles = small_blocks(q, q.op == SmallOp::strided ? 16 : 32);
    if (tiles > 0 && tiles <= (q.op == SmallOp::strided ? (q.dtype == 0 ? 512 : 256) : q.dtype == 0 ? 1200 : 512)) return true;
    // dilated layers that do not fit that kernel's LDS (long rows under a wide dilation) have only the vector ALUs besides (us,
    // dilation 4, n = 5: 64 -> 64 channels, 4 of 100 x 100 452 / 125; 160 -> 200, 8 of 96 x 96 4178 / 1267; 17 -> 40, 13 of 56 x 56
    // 96 / 58; bf16, 16 -> 16, 6 of 128 x 128, dilation 8 82 / 57)
    return q.op == SmallOp::dilated && tiles > 0 &&
           !general_mfma_fits(1, q.B, q.K, q.M, q.XH, q.XW, q.n, q.P, q.step, q.OH, q.OW, q.dtype);
}

int general_plan(int dilated, int B, int Cin, int Cout, int H, int W, int n, int P, int k, int OH, int OW, int dtype)
{
    const SmallProblem q{dilated ? SmallOp::dilated : SmallOp::strided, B, Cin, Cout, H, W, OH, OW, n, P, k, dtype};
    return prefer_small(q) ? small_plan(q, 0) : 0;
}

// k = stride (dilated == 0) or dilation (dilated == 1); shapes validated by the caller
hipError_t launch_general(int dilated, int B, int Cin, int Cout, int H, int W, int n, int P, int k,
                          int OH, int OW, const void* x, const void* w, float* y, int dtype,
                          hipStream_t stream)
{
    const SmallProblem q{dilated ? SmallOp::dilated : SmallOp::strided, B, Cin, Cout, H, W, OH, OW, n, P, k, dtype};
    if (prefer_small(q)) {
        Workspace none;
        return launch_small(q, Epilogue{nullptr, 0}, x, w, y, none, stream);
    }
    hipError_t err = hipSuccess;
    if (launch_general_mfma(dilated, B, Cin, Cout, H, W, n, P, k, OH, OW, x, w, y, dtype, stream, &err)) return err;
    GenArgs a;
    a.B = B; a.Cin = Cin; a.Cout = Cout; a.H = H; a.W = W; a.n = n; a.P = P; a.k = k;
    a.OH = OH; a.OW = OW; a.dilated = dilated;
    a.tilesX = (OW + 31) / 32;
    a.tilesY = (OH + 7) / 8;
    a.coBlocks = (Cout + CO_BLK - 1) / CO_BLK;
    const long long nb = (long long)a.tilesX * a.tilesY * a.coBlocks * B;
    if (nb > 0x7fffffffLL) return hipErrorInvalidConfiguration;
    if (dtype == 0)
        hipLaunchKernelGGL(ukst_general_kernel<float>, dim3((unsigned)nb), dim3(256), 0, stream,
                           (const float*)x, (const float*)w, y, a);
    else
        hipLaunchKernelGGL(ukst_general_kernel<uint16_t>, dim3((unsigned)nb), dim3(256), 0, stream,
                           (const uint16_t*)x, (const uint16_t*)w, y, a);
    return hipGetLastError();
}

}  // namespace ukst
