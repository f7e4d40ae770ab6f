// Tile selection and launch of the matrix-core kernels on bf16 parts (ukst_mfma_parts_kernel.h).
#include "ukst_mfma_parts_kernel.h"

namespace ukst {
using namespace parts;
namespace {

// y[i] = part[0][i] + part[1][i] + ... in this order, four elements per thread, then the epilogue
__global__ __launch_bounds__(256) void ukst_sum_part_slices_kernel(const float4* __restrict__ part, size_t copy4,
                                                                   float* __restrict__ y, int total, int ksplit,
                                                                   const float* __restrict__ bias, int act,
                                                                   unsigned plane, unsigned cout)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (4 * i >= total) return;
    float4 s = part[i];
#pragma unroll 4
    for (int k = 1; k < ksplit; ++k) {
        const float4 p = part[(size_t)k * copy4 + i];
        s.x += p.x; s.y += p.y; s.z += p.z; s.w += p.w;
    }
    float v[4] = {s.x, s.y, s.z, s.w};
    if (bias != nullptr || act != 0) {  // uniform
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const unsigned idx = 4u * (unsigned)i + e;  // element of y[B][Cout][plane]
            v[e] = epilogue(v[e], bias ? bias[(idx / plane) % cout] : 0.f, act);
        }
    }
    if (4 * i + 4 <= total && ((uintptr_t)y & 15) == 0) {
        reinterpret_cast<float4*>(y)[i] = make_float4(v[0], v[1], v[2], v[3]);
        return;
    }
#pragma unroll
    for (int e = 0; e < 4; ++e)
        if (4 * i + e < total) y[4 * i + e] = v[e];
}

// geometry of a tile configuration; false if it does not fit
bool make_args(const Geom& g, int dtype, int cw, int qw, int nt, PartsArgs& a, Config& c)
{
    const int parts = dtype == 0 ? 3 : 1, es = dtype == 0 ? 4 : 2, os = dtype == 2 ? 2 : 4;
    const int TM = 32 * cw, TN = 32 * nt * qw, T = 64 * cw * qw;
    if (g.n < 2 || g.n > 5) return false;
    const size_t lim = 0x7FFFFFF0u;  // single buffer descriptors, 32-bit byte offsets
    if ((size_t)g.B * g.Cin * g.H * g.W * es > lim || (size_t)g.Cout * g.Cin * g.n * g.n * es > lim ||
        (size_t)g.B * g.Cout * g.OH * g.OW * 4 > lim)
        return false;
    const int HI = (g.n + 1) / 2;
    const bool al = g.n % 2 == 0 && g.P % 2 == 0;
    a.g = g;
    a.KHq = al ? g.OH / 2 : g.KH;
    a.KWq = al ? g.OW / 2 : g.KW;
    const int wrows = al ? HI + 1 : HI;
    const long long khw = (long long)a.KHq * a.KWq, Q = (long long)g.B * khw;
    if (Q > 0x3FFFFFFFLL) return false;
    a.Q = (int)Q;
    a.EH = a.KHq + wrows - 1;
    // TN consecutive quads touch at most this many quad rows / images
    const long long nrho = TN % a.KWq == 0 ? TN / a.KWq : (TN - 2) / a.KWq + 2;
    const long long nimg = khw % TN == 0 ? 1 : TN % khw == 0 ? TN / khw : (TN - 2) / khw + 2;
    a.ROWS = (int)(nrho + (wrows - 1) * nimg);
    a.SH = g.P >> 1;
    a.LWX = a.SH + g.W;  // the staged columns, or the last column a quad reads if that is further right
    if (a.LWX < a.KWq + wrows - 1) a.LWX = a.KWq + wrows - 1;
    if ((long long)a.LWX * a.ROWS > 16384) return false;
    a.XPL = 2 * a.ROWS * a.LWX * 16;
    if (dtype != 0 && g.W < 4) return false;  // bf16 rows are staged four columns at a time
    a.CPR = dtype == 0 ? g.W : (g.W + 3) / 4;
    const int units = 2 * a.ROWS * a.CPR;
    c.cw = cw;
    c.qw = qw;
    c.nt = nt;
    c.xu = dtype == 0 ? (units <= 2 * T ? 2 : units <= 3 * T && cw == 2 && nt == 2 ? 3 : 4) : units <= T ? 1 : 2;
    if (units > c.xu * T) return false;
    if (2 * weight_stage_bytes(g.n, parts, cw) + parts * a.XPL > LDS_LIMIT) return false;
    a.nco = (g.Cout + TM - 1) / TM;
    a.nqt = (int)((Q + TN - 1) / TN);
    if ((long long)a.nco * a.nqt * 32 > 0x3FFFFFFFLL) return false;
    a.cb_major = (size_t)g.Cout * g.Cin * g.n * g.n > (size_t)g.B * g.Cin * g.H * g.W ? 1 : 0;
    a.ksplit = 1;
    a.kstages = (g.Cin + KC - 1) / KC;
    a.copy_bytes = ws_align((size_t)g.B * g.Cout * g.OH * g.OW * os);
    a.dKHW = make_fastdiv((unsigned)khw);
    a.dKW = make_fastdiv((unsigned)a.KWq);
    a.dEH = make_fastdiv((unsigned)a.EH);
    a.dRW = make_fastdiv((unsigned)(a.ROWS * a.CPR));
    a.dW = make_fastdiv((unsigned)a.CPR);
    return true;
}

// The tile with the shortest estimated run: blocks a compute unit gets times the MFMAs of a wave times the
// waves per SIMD of a block.  Four waves alone on a compute unit (one per SIMD) have nothing beside their
// staging and take about 1.3 times as long per MFMA as eight; a wave with one group of quads reads more
// fragments per MFMA and its block stages as many weights for half the quads (1.2).
bool pick(const Geom& g, int dtype, PartsArgs& a, Config& c)
{
    const int parts = dtype == 0 ? 3 : 1;
    const Config order[] = {{2, 4, 2, 0}, {2, 4, 1, 0}, {1, 8, 2, 0}, {1, 4, 2, 0}};
    double best = 0.;
    for (const Config& o : order) {
        if (g.Cout <= 32 && o.cw == 2) continue;
        if (dtype != 0 && o.qw == 8) continue;
        PartsArgs t;
        Config tc;
        if (!make_args(g, dtype, o.cw, o.qw, o.nt, t, tc)) continue;
        const double per_cu = (double)(((long long)t.nco * t.nqt + 255) / 256);
        const bool alone = o.cw * o.qw == 4 &&
                           (per_cu == 1. || 2 * (2 * weight_stage_bytes(g.n, parts, o.cw) + parts * t.XPL) > LDS_LIMIT);
        const double est = per_cu * (o.cw * o.qw / 4) * o.nt * (alone ? 1.3 : o.nt == 1 ? 1.2 : 1.);
        if (best != 0. && est >= best) continue;
        best = est;
        a = t;
        c = tc;
    }
    return best != 0.;
}

}  // namespace

double mfma_parts_tiles(const Geom& g, int dtype)
{
    PartsArgs a;
    Config c;
    return pick(g, dtype, a, c) ? (double)a.nco * a.nqt * (c.cw * c.qw * c.nt) / 16. : 0.;
}

// Layers of few tiles: 64 channels x 128 quads and slices of the input channels, about one block per compute
// unit, each slice at least three stages; 0 if that is no use
static int pick_split(const Geom& g, int dtype, PartsArgs& a, Config& c)
{
    if (!make_args(g, dtype, 2, 4, 1, a, c)) return 0;
    const long long tiles = (long long)a.nco * a.nqt;
    const int stages = a.kstages;
    int ks = (int)(256 / tiles);
    if (ks > stages / 3) ks = stages / 3;
    while (ks > 1 && (size_t)ks * a.copy_bytes > ((size_t)1 << 26)) --ks;
    if (ks < 2) return 0;
    a.kstages = (stages + ks - 1) / ks;
    a.ksplit = (stages + a.kstages - 1) / a.kstages;
    // fewer blocks than that lose to the small tiles of the fp32 pipe (16 images of 128 -> 64 channels, 16 x 16,
    // n = 4: 64 blocks, 30 against 17.5 us; 64 images, 256 blocks: 42 against 49)
    if (tiles * a.ksplit < 192) return 0;
    return a.ksplit;
}

int mfma_parts_split_slices(const Geom& g, int dtype)
{
    PartsArgs a;
    Config c;
    return dtype == 0 ? pick_split(g, dtype, a, c) : 0;
}

static hipError_t launch_sides(const PartsArgs& a, const Config& c, const Epilogue& ep, const void* x, const void* w,
                               void* y, int dtype, hipStream_t stream)
{
    switch (a.g.n * 2 + (dtype == 0 ? 0 : 1)) {
        case 4: return launch_side<2, float>(a, c, ep, x, w, y, false, stream);
        case 5: return launch_side<2, uint16_t>(a, c, ep, x, w, y, dtype == 2, stream);
        case 6: return launch_side<3, float>(a, c, ep, x, w, y, false, stream);
        case 7: return launch_side<3, uint16_t>(a, c, ep, x, w, y, dtype == 2, stream);
        case 8: return launch_side<4, float>(a, c, ep, x, w, y, false, stream);
        case 9: return launch_side<4, uint16_t>(a, c, ep, x, w, y, dtype == 2, stream);
        case 10: return launch_side<5, float>(a, c, ep, x, w, y, false, stream);
        case 11: return launch_side<5, uint16_t>(a, c, ep, x, w, y, dtype == 2, stream);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_sum_slices(const void* part, size_t copy_bytes, float* y, size_t total, int ks, const Epilogue& ep,
                             unsigned plane, unsigned cout, hipStream_t stream)
{
    hipLaunchKernelGGL(ukst_sum_part_slices_kernel, dim3((unsigned)((total + 1023) / 1024)), dim3(256), 0, stream,
                       (const float4*)part, copy_bytes / 16, y, (int)total, ks, ep.bias, ep.act, plane, cout);
    return hipGetLastError();
}

// fp32 layers with a workspace: partial sums of the slices, added in slice order
hipError_t launch_mfma_parts_split(const Geom& g, const void* x, const void* w, float* y, Workspace& ws, hipStream_t stream)
{
    PartsArgs a;
    Config c;
    if (pick_split(g, 0, a, c) < 2) return hipErrorInvalidValue;
    ws.need = (size_t)a.ksplit * a.copy_bytes;
    if (ws.query) return hipSuccess;
    if (ws.ptr == nullptr || ws.bytes < ws.need) return kWorkspaceTooSmall;
    const Epilogue none = {nullptr, 0};
    const hipError_t e = launch_sides(a, c, none, x, w, ws.ptr, 0, stream);
    if (e != hipSuccess) return e;
    return launch_sum_slices(ws.ptr, a.copy_bytes, y, (size_t)g.B * g.Cout * g.OH * g.OW, a.ksplit, g.ep,
                             (unsigned)(g.OH * g.OW), (unsigned)g.Cout, stream);
}

hipError_t launch_mfma_parts(const Geom& g, const void* x, const void* w, void* y, int dtype, Workspace& ws,
                             hipStream_t stream)
{
    PartsArgs a;
    Config c;
    if (!pick(g, dtype, a, c)) return hipErrorInvalidValue;
    ws.need = 0;
    if (ws.query) return hipSuccess;
    return launch_sides(a, c, g.ep, x, w, y, dtype, stream);
}

}  // namespace ukst
