// Geometry and launch of the small-tile kernels (ukst_small_kernel.h).
#include "ukst_small_kernel.h"

namespace ukst {
using namespace small;
namespace {

int floor_div(int a, int b) { return a >= 0 ? a / b : -((-a + b - 1) / b); }

bool make_args(const SmallProblem& q, int mt, SmallArgs& a)
{
    const bool forward = q.op == SmallOp::forward, dx = q.op == SmallOp::grad_input;
    const bool strided = q.op == SmallOp::strided, dilated = q.op == SmallOp::dilated;
    if (q.n < 2 || q.n > 5) return false;
    const int s = strided ? q.step : 2;
    if (strided && (s < 2 || s > 4)) return false;
    const int kind = dx ? kInputGrad : dilated ? kDilated : forward && q.n % 2 == 0 && q.P % 2 == 0 ? kAligned : kShifted;
    const int cs = kind <= kAligned ? s : 1;  // classes per axis
    if (mt == 32 && cs > 2) return false;
    const int es = q.dtype == 0 ? 4 : 2, ps = dx ? 2 : 1, win = window_of(kind, q.n, s);
    a.B = q.B;
    a.K = q.K;
    a.M = q.M;
    a.XH = q.XH;
    a.XW = q.XW;
    a.OH = q.OH;
    a.OW = q.OW;
    a.out16 = q.dtype == 2 ? 1 : 0;
    const size_t lim = 0x7FFFFFF0u;  // single buffer descriptors, 32-bit byte offsets
    if ((size_t)q.B * q.K * q.XH * q.XW * es > lim || (size_t)q.M * q.K * q.n * q.n * es > lim ||
        (size_t)q.B * q.M * q.OH * q.OW * 4 > lim)
        return false;
    if (q.K < kc_of(kind, q.n, mt)) return false;
    // bf16 weights of an input gradient whose last piece hangs over the end of w in the middle of a dword
    if (dx && q.dtype != 0 && q.M % mt != 0 && q.M * q.n % 2 != 0) return false;
    a.res = 1;
    a.xs = 1;
    if (kind == kShifted) {
        const int k_min = -(q.P / s);
        a.LH = floor_div(q.OH - 1 - q.P + s - 1, s) - k_min + 1;
        a.LW = floor_div(q.OW - 1 - q.P + s - 1, s) - k_min + 1;
        a.g0 = k_min;
        a.o0 = q.P % s;
        a.os = s;
    } else if (kind == kAligned) {
        a.LH = q.OH / 2;
        a.LW = q.OW / 2;
        a.g0 = -(q.P / 2);
        a.o0 = 0;
        a.os = 2;
    } else if (kind == kInputGrad) {
        a.LH = q.OH;
        a.LW = q.OW;
        a.g0 = q.P - (q.n - 1);
        a.o0 = 0;
        a.os = 1;
    } else {
        a.LH = (q.OH + q.step - 1) / q.step;
        a.LW = (q.OW + q.step - 1) / q.step;
        a.g0 = -q.P;
        a.xs = a.os = a.res = q.step;
        a.o0 = 0;
    }
    if (a.LH < 1 || a.LW < 1) return false;
    // Column tiles of about eight columns keep the halo small; the widest whose staged cells fit
    bool fits = false;
    for (int nct = (a.LW + 7) / 8, tries = 0; !fits && tries < 4 && nct <= a.LW; ++nct, ++tries) {
        a.nct = nct;
        a.TCW = (a.LW + nct - 1) / nct;
        const long long Q = (long long)q.B * a.LH * a.TCW;
        if (Q > 0x3FFFFFFF) return false;
        a.Q = (int)Q;
        // rows and images that a tile's positions touch at most
        const long long per = (long long)a.LH * a.TCW;
        long long rows = mt % a.TCW == 0 ? mt / a.TCW : (mt - 2) / a.TCW + 2;
        long long images = per % mt == 0 ? 1 : mt % per == 0 ? mt / per : (mt - 2) / per + 2;
        if (rows > (long long)q.B * a.LH) rows = (long long)q.B * a.LH;
        if (images > q.B) images = q.B;
        a.COLS = ps * (a.TCW - 1) + win;
        fits = (ps * (rows - 1) + (images - 1) * (win - ps) + win) * a.COLS <= 64 * jr_of(kind, q.n, mt);
    }
    if (!fits) return false;
    a.EH = ps * (a.LH - 1) + win;
    a.nmt = (q.M + mt - 1) / mt;
    a.npt = (a.Q + mt - 1) / mt;
    const long long blocks = (long long)a.nmt * a.npt * a.nct * a.res * a.res;
    if (blocks > 0xFFFFFF) return false;
    a.m_major = (size_t)q.M * q.K * q.n * q.n > (size_t)q.B * q.K * q.XH * q.XW ? 1 : 0;
    a.ksplit = 1;
    a.kslice = (q.K + kc_of(kind, q.n, mt) - 1) / kc_of(kind, q.n, mt);
    a.copy_bytes = 0;
    return true;
}

void add_divisors(SmallArgs& a)
{
    a.dMajor = make_fastdiv((unsigned)(a.m_major ? a.npt * a.nct * a.res * a.res : a.nmt));
    a.dP = make_fastdiv((unsigned)a.npt);
    a.dN = make_fastdiv((unsigned)a.nct);
    a.dR = make_fastdiv((unsigned)a.res);
    a.dT = make_fastdiv((unsigned)a.TCW);
    a.dH = make_fastdiv((unsigned)a.LH);
    a.dE = make_fastdiv((unsigned)a.EH);
    a.dC = make_fastdiv((unsigned)a.COLS);
    a.dK = make_fastdiv((unsigned)a.ksplit);
}

// Time of a plan in us, fitted to 900 layers of every operation (17 % off on average; the choice it makes costs 1 % against the
// best plan of each): rounds of blocks, each with a fixed part and its waves' MFMAs, two waves per SIMD.  Input gradients
// of small kernels stage more than they multiply (four cells of dy and n * n weights for n * n products): with their MFMAs alone the
// 16 x 16 tiles looked three times as fast as they are for n = 2, and were taken where the 32 x 32 ones are up to 1.7 times as fast
// (398 <- 344 channels, 16 x 16 24.1 / 15.0 us; 1 % of 1700 layers by more than 1.5 for n = 2, 1.2 for n = 3; now 1.07 and 1.08)
double estimate(const SmallProblem& q, const SmallArgs& a, int mt, int wv)
{
    const int kind = q.op == SmallOp::grad_input ? kInputGrad : q.op == SmallOp::dilated ? kDilated : kShifted;
    const int kc = kc_of(kind, q.n, mt), per_wave = ((q.K + kc - 1) / kc + wv - 1) / wv;
    const double staging = kind != kInputGrad || q.n > 3 ? 1. : q.n == 2 ? (mt == 32 ? 1.9 : 3.4) : (mt == 32 ? 1.35 : 1.75);
    const double mfma = staging * (mt == 32 ? 64. * kc / 2 : 32. * kc / 4) * q.n * q.n / 2400. * per_wave;
    const long long blocks = (long long)a.nmt * a.npt * a.nct * a.res * a.res;
    const double rounds = (double)((blocks + 255) / 256);
    if (mt == 16) return rounds * (2.6 + 1.95 * 2. * mfma);
    if (wv == 8) return rounds * (3.5 + 1.36 * 2. * mfma);
    const long long rest = blocks % 512;  // blocks of four waves: two to a compute unit
    const double twos = (double)(blocks / 512 + (rest > 256 ? 1 : 0)), one = rest > 0 && rest <= 256 ? 1. : 0.;
    return 4. * (twos + one) + 1.33 * (2. * twos + 1.2 * one) * mfma;
}

// the quickest plan; false if none fits
bool pick(const SmallProblem& q, SmallArgs& a, int& mt, int& wv)
{
    const int order[3][2] = {{32, 8}, {32, 4}, {16, 8}};
    double best = 0.;
    for (const auto& o : order) {
        SmallArgs t;
        if (!make_args(q, o[0], t)) continue;
        const double e = estimate(q, t, o[0], o[1]);
        if (best != 0. && e >= best) continue;
        best = e;
        a = t;
        mt = o[0];
        wv = o[1];
    }
    return best != 0.;
}

// cuts the stages of a plan into slices over blocks; false if that is no use (see small_workspace())
bool slice(const SmallProblem& q, SmallArgs& a, int mt, int wv)
{
    const long long blocks = (long long)a.nmt * a.npt * a.nct;
    const int per_wave = (a.kslice + wv - 1) / wv;
    const int least = q.n == 3 || (q.n == 2 && mt == 32) ? 5 : 4;
    if (q.op != SmallOp::forward || q.dtype != 0 || blocks > 128 || per_wave < least) return false;
    a.copy_bytes = ws_align((size_t)q.B * q.M * q.OH * q.OW * 4);
    int ks = (int)(256 / blocks);
    if (ks > per_wave) ks = per_wave;
    while (ks > 1 && ks * a.copy_bytes > ((size_t)1 << 26)) --ks;
    if (ks < 2) return false;
    const int stages = a.kslice;
    a.kslice = (stages + ks - 1) / ks;
    a.ksplit = (stages + a.kslice - 1) / a.kslice;
    return a.ksplit > 1;
}

template <typename TIn>
hipError_t launch_t(const SmallProblem& q, const SmallArgs& a, int mt, int wv, const Epilogue& ep, const void* x,
                    const void* w, void* y, hipStream_t st)
{
    switch (q.op) {
        case SmallOp::forward:
            if (q.n % 2 == 0 && q.P % 2 == 0) return launch_kind<kAligned, TIn>(a, q.n, 2, mt, wv, ep, x, w, y, st);
            return launch_kind<kShifted, TIn>(a, q.n, 2, mt, wv, ep, x, w, y, st);
        case SmallOp::strided: return launch_kind<kShifted, TIn>(a, q.n, q.step, mt, wv, ep, x, w, y, st);
        case SmallOp::grad_input: return launch_kind<kInputGrad, TIn>(a, q.n, 1, mt, wv, ep, x, w, y, st);
        case SmallOp::dilated: return launch_kind<kDilated, TIn>(a, q.n, 1, mt, wv, ep, x, w, y, st);
    }
    return hipErrorInvalidValue;
}

}  // namespace

double small_estimate(const SmallProblem& q)
{
    SmallArgs a;
    int mt = 0, wv = 0;
    return pick(q, a, mt, wv) ? estimate(q, a, mt, wv) : 0.;
}

long long small_blocks(const SmallProblem& q, int edge)
{
    SmallArgs a;
    if (!make_args(q, 16, a) && !make_args(q, 32, a)) return 0;
    const long long m = (q.M + edge - 1) / edge, p = (a.Q + edge - 1) / edge;
    return m * p * a.nct * a.res * a.res;
}

// Slices of the stages, given a workspace: fp32 layers that leave half of the compute units idle and have at least four stages
// for every wave, five of the shorter ones of n = 3 and of n = 2 in 32 x 32 tiles (us, unsliced -> sliced with the sum: one image,
// 512 -> 256 channels, 4 x 4, n = 4 13.3 -> 8.6, 500 -> 256 13.4 -> 8.6, n = 5, P = 1 23.7 -> 10.8, n = 3 11.0 -> 7.9; two, 1024 -> 64,
// 8 x 8 22.4 -> 10.6; eight, 512 -> 256, 4 x 4 14.3 -> 12.2; 60, 512 -> 24, 4 x 4 14.4 -> 12.2; at the line, n = 2, 449 -> 16, 6 of 7 x 6
// 9.0 -> 7.9, n = 4, 256 -> 128, 8 x 8 8.6 -> 7.9, but n = 3, 256 -> 128, 2 of 8 x 8 7.9 -> 8.0, 210 -> 313, 6 x 8 7.3 -> 8.4, n = 2, 211 -> 482,
// 2 of 7 x 15 10.3 -> 11.6; 128 layers 1.49 times as fast on average)
size_t small_workspace(const SmallProblem& q)
{
    SmallArgs a;
    int mt, wv;
    return pick(q, a, mt, wv) && slice(q, a, mt, wv) ? a.ksplit * a.copy_bytes : 0;
}

int small_plan(const SmallProblem& q, size_t workspace_bytes)
{
    SmallArgs a;
    int mt, wv;
    if (!pick(q, a, mt, wv)) return 0;
    const bool sliced = slice(q, a, mt, wv) && workspace_bytes >= a.ksplit * a.copy_bytes;
    return mt | wv << 8 | (sliced ? a.ksplit : 1) << 16;
}

hipError_t launch_small(const SmallProblem& q, const Epilogue& ep, const void* x, const void* w, void* y, Workspace& ws,
                        hipStream_t stream)
{
    SmallArgs a;
    int mt, wv;
    if (!pick(q, a, mt, wv)) return hipErrorInvalidValue;
    const bool sliced = ws.ptr != nullptr && slice(q, a, mt, wv) && ws.bytes >= a.ksplit * a.copy_bytes;
    if (!sliced) {
        a.ksplit = 1;
        a.kslice = q.K;  // (at least the stages)
    }
    add_divisors(a);
    const Epilogue none = {nullptr, 0};
    const Epilogue& first = sliced ? none : ep;
    void* const out = sliced ? ws.ptr : y;
    const hipError_t e = q.dtype == 0 ? launch_t<float>(q, a, mt, wv, first, x, w, out, stream)
                                      : launch_t<uint16_t>(q, a, mt, wv, first, x, w, out, stream);
    if (e != hipSuccess || !sliced) return e;
    return launch_sum_slices(ws.ptr, a.copy_bytes, (float*)y, (size_t)q.B * q.M * q.OH * q.OW, a.ksplit, ep,
                             (unsigned)(q.OH * q.OW), (unsigned)q.M, stream);
}

}  // namespace ukst
