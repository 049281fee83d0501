// Convolution on the float32 matrix instruction, any kernel up to 7^3, any
// stride and padding: the float32 workloads.
//
// v_mfma_f32_16x16x4_f32 does 2048 flops in 32 cycles, a sixteenth of the
// bf16 rate, so one 4-byte LDS read per operand lane feeds it with room to
// spare and the operands need no special order: an input box is staged as it
// lies in memory ([channel][depth][row][column], zeros outside the volume)
// and a lane finds its operand at (offset of its voxel) + (offset of its
// channel and tap).  So a tile may be any box of voxels -- chosen per shape
// so that few of its lanes fall outside the map -- and a stride only changes
// the voxels' offsets.
//
// Forward (conv_box_fwd): rows M = output channels (A = weights), columns =
// voxels of the box (B = the staged input), K = (input channel, tap).
// Input gradient (conv_box_dgrad): the same with K = (output channel, tap);
// the target voxels of stride s fall into s^3 residue classes, and the voxels
// i = r + s m of a class see the taps t0 + s j only: a stride-1 convolution of
// dy with those taps in reverse.
// Weight gradient (conv_box_wgrad): M = output channels (A = dy), columns =
// (tap, input channel), K = the voxels of a range of boxes; partial sums of
// the ranges are added in order afterwards.
//
// Bound: MFMA issue (153 TFLOP/s for a large float32 matrix product).  Measured
// against the gather kernel, 3^3, 64 -> 64 channels, us: 2 x 24x28x24 forward
// 232 -> 78 (92 TFLOP/s), input gradient 310 -> 83, weight gradient 168 -> 109;
// 8 x 46x55x46 3576 -> 1858 (111 TFLOP/s), 5248 -> 1933, 5009 -> 2620; 2 x
// 6x7x6, 256 channels 770 -> 105, 1017 -> 75, 68 -> 48.
#include <cmath>

#include "common.hpp"
#include "kernels.hpp"
#include "prof.hpp"

namespace rat3d {

namespace {

constexpr int kBoxMaxK = 7;
constexpr size_t kBoxLds = 64 * 1024;
constexpr int64_t kLim = (int64_t)1 << 31;  // 32-bit element offsets
// Launch limits: work-items of the first dimension in 32 bits, workgroups of
// the others in 16
constexpr int64_t kGridX = (((int64_t)1 << 32) - 1) / 256, kGridYZ = 65535;

__device__ __forceinline__ f32x4 mfma4(float a, float b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

constexpr uint32_t kNoOff = 0x80000000u;  // a buffer offset past any end: reads zero
constexpr int kBoxXr = 12, kBoxWr = 28;   // dgrad: words a thread stages per chunk, source and weights
constexpr int kFwdXr = 12, kFwdWr = 6;    // forward: source words, 16-byte weight units (of 64 rows)
// LDS floats per staged K entry: an odd multiple of 16, so that the four K
// entries of an operand read lie in different quarters of the banks; each K
// step of four entries is shifted by one more float, so that a store of 16
// consecutive K entries by 4 channels hits 64 different banks as well
__host__ __device__ constexpr int box_ws(int ct) { return ct == 4 ? 80 : ct == 2 ? 48 : 16; }
__host__ __device__ constexpr int box_ws4(int ct) { return 4 * box_ws(ct) + 1; }

__device__ __forceinline__ float buf_ldf(__amdgpu_buffer_rsrc_t r, uint32_t off) {
    return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0));
}

struct FdBox {
    const float* src;   // [N][Cs][Sd][Sh][Sw]
    const float* w;     // [Co][Ci][k^3]
    const float* bias;  // forward: [Ct] or null
    float* dst;         // [N][Ct][Dd][Dh][Dw]
    int N, Cs, Ct, Sd, Sh, Sw, Dd, Dh, Dw;
    int k, s, p, accumulate;
    int wM, wC;              // dgrad: weight strides of a target and of a source channel
    int TN, TD, TH, TW;      // box
    int tn, td, th, tw;      // boxes per axis (of the largest class)
    int CK;                  // source channels per chunk
    int KC;                  // forward: K entries per chunk, a multiple of 16
    int w16;                 // forward: weight rows are 16-byte aligned
    int chs;                 // LDS floats per staged channel
    int kmax;                // entries of the tap tables
    int wrows;               // staged weight rows
    int xtot;                // LDS floats of the staged channels
    int zero;                // LDS floats of the channel of zeros behind them (0: none)
};

// One axis of a residue class: target position of index m is s m + r, its
// source positions are m + off + j, j < n, and tap j of the sweep is weight
// tap ta - s j.
struct Axis {
    int M, n, off, ta;
};
__host__ __device__ __forceinline__ Axis box_axis(int D, int k, int s, int p, int r) {
    Axis a;
    const int t0 = (r + p) % s;
    a.M = r < D ? (D - r + s - 1) / s : 0;
    a.n = t0 < k ? (k - t0 + s - 1) / s : 0;
    a.off = (r + p - t0) / s - (a.n - 1);
    a.ta = t0 + s * (a.n - 1);
    return a;
}

}  // namespace

// A workgroup of four waves: each VT * 16 voxels of the box by the same CT *
// 16 output channels.  K runs in the order (channel, tap), 16 entries at a
// time: lane group kg holds entries 4 kg + j of the 16, and MFMA j multiplies
// those -- the order of the gather kernel, whose sums these are bit for bit.
// So a weight row is staged as it lies in memory and one 16-byte LDS read
// gives a lane its four A operands; the four LDS offsets of its B operands are
// another.  A chunk of KC entries spans CK channels (the first and last
// perhaps in part); the next chunk's operands are loaded into registers while
// the current one multiplies.  Every load is a buffer load whose out-of-range
// offset reads zero: a conditional load would be waited for on the spot.
template <int CT, int VT>
__global__ __launch_bounds__(256, 2) void conv_box_fwd(FdBox a) {
    constexpr int XR = kFwdXr, WR = (kFwdWr * CT + 3) / 4;  // staged words, 16-byte weight units
    extern __shared__ __align__(16) float lds[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int li = lane & 15, kg = lane >> 4;
    const int S = a.s;
    int b = blockIdx.x;
    const int w0 = (b % a.tw) * a.TW;
    b /= a.tw;
    const int h0 = (b % a.th) * a.TH;
    b /= a.th;
    const int d0 = (b % a.td) * a.TD;
    const int n0 = b / a.td * a.TN;
    const int c0t = blockIdx.y * CT * 16;
    const int NT = a.k * a.k * a.k, K = a.Cs * NT, KC = a.KC;
    const int PH = (a.TH - 1) * S + a.k, PW = (a.TW - 1) * S + a.k;
    const int P1 = ((a.TD - 1) * S + a.k) * PH * PW, P = a.TN * P1;
    const int64_t Vs = (int64_t)a.Sd * a.Sh * a.Sw, Vd = (int64_t)a.Dd * a.Dh * a.Dw;

    // LDS: staged channels (one more, all zero, for K entries past the end),
    // weights [channel][KC + 8] (16 rows at a stride of 32 or 96 bytes mod 128
    // take one pass), LDS byte offsets of the chunk's entries and of the taps,
    // source offsets of the staged positions
    float* xs = lds;
    float* wsm = xs + a.xtot + a.zero;
    const int ws_row = KC + 8;
    int* koff = (int*)(wsm + CT * 16 * ws_row);
    int* toff = koff + KC;
    uint32_t* poff = (uint32_t*)(toff + ((NT + 3) & ~3));
    const Div byNT(NT), byKK(a.k * a.k), byK(a.k), byP1(P1), byPHW(PH * PW), byPW(PW);
    const Div byChs(a.chs), byBox(a.TD * a.TH * a.TW), byTHW(a.TH * a.TW), byTW(a.TW);
    const Div byKQ(KC >> 2);
    for (int t = tid; t < NT; t += 256) {
        const int jd = byKK(t), r = t - jd * a.k * a.k, jh = byK(r);
        toff[t] = 4 * ((jd * PH + jh) * PW + r - jh * a.k);
    }
    for (int i = tid; i < P; i += 256) {
        const int n = byP1(i);
        int r = i - n * P1;
        const int dd = byPHW(r);
        r -= dd * PH * PW;
        const int hh = byPW(r), ww = r - hh * PW;
        const int d = d0 * S - a.p + dd, h = h0 * S - a.p + hh, w = w0 * S - a.p + ww;
        const bool ok = n0 + n < a.N && (unsigned)d < (unsigned)a.Sd &&
                        (unsigned)h < (unsigned)a.Sh && (unsigned)w < (unsigned)a.Sw;
        poff[i] = ok ? 4u * (uint32_t)((int)(n * a.Cs * Vs) + (d * a.Sh + h) * a.Sw + w) : kNoOff;
    }
    for (int i = tid; i < a.zero; i += 256) xs[a.xtot + i] = 0.f;

    // this lane's voxels: LDS address, and target offset (-1: not a voxel)
    const char* vb[VT];
    int64_t vd[VT];
#pragma unroll
    for (int v = 0; v < VT; ++v) {
        const int i = (wave * VT + v) * 16 + li;
        const int n = byBox(i);
        int r = i - n * a.TD * a.TH * a.TW;
        const int d = byTHW(r);
        r -= d * a.TH * a.TW;
        const int h = byTW(r), w = r - h * a.TW;
        const bool in = n < a.TN;
        vb[v] = (const char*)(xs + (in ? n * P1 + (d * S * PH + h * S) * PW + w * S : 0));
        const bool ok = in && n0 + n < a.N && d0 + d < a.Dd && h0 + h < a.Dh && w0 + w < a.Dw;
        vd[v] = ok ? (int64_t)(n0 + n) * a.Ct * Vd + ((int64_t)(d0 + d) * a.Dh + h0 + h) * a.Dw +
                         w0 + w
                   : -1;
    }
    f32x4 acc[CT][VT];
#pragma unroll
    for (int c = 0; c < CT; ++c)
#pragma unroll
        for (int v = 0; v < VT; ++v) acc[c][v] = f32x4{0.f, 0.f, 0.f, 0.f};
    __syncthreads();

    // staged word e of a chunk: position e % chs of channel e / chs (LDS offset e)
    uint32_t gx[XR], gw[WR];
    const int nx = (a.CK * a.chs + 255) >> 8, nq = CT * 16 * (KC >> 2);
#pragma unroll
    for (int r = 0; r < XR; ++r) {
        const int e = tid + 256 * r, c = byChs(e), i = e - c * a.chs;
        const uint32_t o = poff[i < P ? i : 0];
        gx[r] = c < a.CK && i < P && o != kNoOff ? o + 4u * (uint32_t)(c * Vs) : kNoOff;
    }
    // weight unit e: entries 4 q .. 4 q + 3 of row e / (KC / 4)
#pragma unroll
    for (int r = 0; r < WR; ++r) {
        const int e = tid + 256 * r, row = byKQ(e), q = e - row * (KC >> 2);
        const bool ok = e < nq && c0t + row < a.Ct;
        gw[r] = ok ? 4u * ((uint32_t)(c0t + row) * (uint32_t)K + 4u * q) : kNoOff;
    }
    const float* sbase = a.src + (int64_t)n0 * a.Cs * Vs;
    const int ns = a.N - n0 < a.TN ? a.N - n0 : a.TN;
    float vx[XR];
    uint4 vw[WR];
    // (channels past the last are past the buffer's end, or another sample's
    // where a box holds several: no K entry refers to them)
    auto load = [&](int k0, bool x) {
        if (x) {
            const int cf = byNT(k0);
            const int64_t left = ((int64_t)ns * a.Cs - cf) * Vs * 4;
            const __amdgpu_buffer_rsrc_t r =
                buf_rsrc_u(sbase + (int64_t)cf * Vs, (uint32_t)(left < kNoOff ? left : kNoOff));
#pragma unroll
            for (int i = 0; i < XR; ++i)
                if (i < nx) vx[i] = buf_ldf(r, gx[i]);
        }
        const __amdgpu_buffer_rsrc_t r =
            buf_rsrc_u(a.w + k0, (uint32_t)(((int64_t)a.Ct * K - k0) * 4));
        if (a.w16) {
#pragma unroll
            for (int i = 0; i < WR; ++i) vw[i] = buf_ld16(r, gw[i], 0);
        } else {
#pragma unroll
            for (int i = 0; i < WR; ++i)
                vw[i] = make_uint4(__float_as_uint(buf_ldf(r, gw[i])),
                                   __float_as_uint(buf_ldf(r, gw[i] + 4)),
                                   __float_as_uint(buf_ldf(r, gw[i] + 8)),
                                   __float_as_uint(buf_ldf(r, gw[i] + 12)));
        }
    };
    auto store = [&](int k0, bool x) {
        const int cf = byNT(k0);
        if (tid < KC) {
            const int k = k0 + tid, c = byNT(k);
            koff[tid] = k < K ? 4 * (c - cf) * a.chs + toff[k - c * NT] : 4 * a.xtot;
        }
        if (x) {
#pragma unroll
            for (int i = 0; i < XR; ++i)
                if (i < nx) xs[tid + 256 * i] = vx[i];
        }
        // entries past the end are zeros, not the next row's weights
        const int left = K - k0;
#pragma unroll
        for (int i = 0; i < WR; ++i) {
            const int e = tid + 256 * i, row = byKQ(e), k = 4 * (e - row * (KC >> 2));
            if (e >= nq) break;
            uint4 v = vw[i];
            if (left < KC) {
                v.x = k < left ? v.x : 0u;
                v.y = k + 1 < left ? v.y : 0u;
                v.z = k + 2 < left ? v.z : 0u;
                v.w = k + 3 < left ? v.w : 0u;
            }
            *reinterpret_cast<uint4*>(wsm + row * ws_row + k) = v;
        }
    };
    // 16 K entries per step.  A step's operands are read while the one before
    // multiplies, its B offsets one step earlier still; the scheduling groups
    // spread the reads over the MFMAs (left alone, the compiler sinks them to
    // their use and every step waits out the LDS latency).
    auto compute = [&](int groups) {
        const float* wl = wsm + li * ws_row + 4 * kg;
        const int* kt = koff + 4 * kg;
        float4 A[2][CT];
        float B[2][4][VT];
        auto read = [&](float4 (&x)[CT], float (&y)[4][VT], int g, const int4& ko) {
#pragma unroll
            for (int v = 0; v < VT; ++v) {
                y[0][v] = *(const float*)(vb[v] + ko.x);
                y[1][v] = *(const float*)(vb[v] + ko.y);
                y[2][v] = *(const float*)(vb[v] + ko.z);
                y[3][v] = *(const float*)(vb[v] + ko.w);
            }
#pragma unroll
            for (int c = 0; c < CT; ++c)
                x[c] = *reinterpret_cast<const float4*>(wl + c * 16 * ws_row + 16 * g);
        };
        auto mul = [&](const float4 (&x)[CT], const float (&y)[4][VT]) {
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int c = 0; c < CT; ++c)
#pragma unroll
                    for (int v = 0; v < VT; ++v)
                        acc[c][v] = mfma4(j == 0 ? x[c].x : j == 1 ? x[c].y : j == 2 ? x[c].z : x[c].w,
                                          y[j][v], acc[c][v]);
        };
        auto spread = [&] {
#pragma unroll
            for (int i = 0; i < 4 * CT * VT; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // MFMA
                __builtin_amdgcn_sched_group_barrier(0x002, 2, 0);  // VALU
                __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);  // LDS read
            }
            __builtin_amdgcn_sched_barrier(0);
        };
        auto ko_at = [&](int g) {  // (past the last step: the last again)
            return *reinterpret_cast<const int4*>(kt + 16 * (g < groups ? g : groups - 1));
        };
        auto clip = [&](int g) { return g < groups ? g : groups - 1; };
        read(A[0], B[0], 0, ko_at(0));
        int4 ko = ko_at(1);
        for (int g = 1; g < groups; g += 2) {
            read(A[1], B[1], g, ko);
            ko = ko_at(g + 1);
            mul(A[0], B[0]);
            spread();
            read(A[0], B[0], clip(g + 1), ko);
            ko = ko_at(g + 2);
            mul(A[1], B[1]);
            spread();
        }
        if (groups & 1) mul(A[0], B[0]);
    };

    load(0, true);
    store(0, true);
    __syncthreads();
    for (int k0 = 0; k0 < K; k0 += KC) {
        const bool more = k0 + KC < K;
        // (the same first channel: the same staged channels)
        const bool x = more && byNT(k0 + KC) != byNT(k0);
        if (more) load(k0 + KC, x);
        compute(((K - k0 < KC ? K - k0 : KC) + 15) >> 4);
        __syncthreads();
        if (more) {
            store(k0 + KC, x);
            __syncthreads();
        }
    }

    const int room = a.Ct - c0t - 4 * kg;  // rows of this lane's that exist
#pragma unroll
    for (int v = 0; v < VT; ++v) {
        if (vd[v] < 0) continue;
        float* q = a.dst + vd[v] + (int64_t)(c0t + 4 * kg) * Vd;
        if (a.bias) {
#pragma unroll
            for (int c = 0; c < CT; ++c)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    acc[c][v][e] += a.bias[c * 16 + e < room ? c0t + 4 * kg + c * 16 + e : 0];
        }
#pragma unroll
        for (int c = 0; c < CT; ++c)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (c * 16 + e < room) q[(int64_t)(c * 16 + e) * Vd] = acc[c][v][e];
    }
}

// Input gradient.  A workgroup of four waves: WV = 4 / WK groups of VT * 16
// voxels by CT * 16 target channels, the K steps of each group dealt to WK
// waves (summed through LDS at the end) where a map has too few voxels to
// fill the chip.  Staged and pipelined like the forward; weights go to LDS as
// [K entry][target channel].  Sums are kept in two levels (a chunk's, then
// the total): the rounding error of K = 1728 products falls by about 3
// against one running sum.
template <int CT, int VT, int WK>
__global__ __launch_bounds__(256, 2) void conv_box_dgrad(FdBox a) {
    constexpr int WV = 4 / WK;
    constexpr int WS = box_ws(CT), WS4 = box_ws4(CT);
    constexpr int XR = kBoxXr, WR = kBoxWr, WK16 = WR / CT;  // staged words per thread
    extern __shared__ __align__(16) float lds[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int li = lane & 15, kg = lane >> 4;

    const int s = a.s, cls = blockIdx.z;
    const int rd = cls / (s * s), rh = (cls / s) % s, rw = cls % s;
    const Axis ad = box_axis(a.Dd, a.k, s, a.p, rd);
    const Axis ah = box_axis(a.Dh, a.k, s, a.p, rh);
    const Axis aw = box_axis(a.Dw, a.k, s, a.p, rw);
    int b = blockIdx.x;
    const int w0 = (b % a.tw) * a.TW;
    b /= a.tw;
    const int h0 = (b % a.th) * a.TH;
    b /= a.th;
    const int d0 = (b % a.td) * a.TD;
    const int n0 = b / a.td * a.TN;
    if (d0 >= ad.M || h0 >= ah.M || w0 >= aw.M) return;  // past this class's voxels
    const int c0t = blockIdx.y * CT * 16;

    const int NT = ad.n * ah.n * aw.n;
    const int PD = a.TD - 1 + ad.n, PH = a.TH - 1 + ah.n, PW = a.TW - 1 + aw.n;
    const int P1 = PD * PH * PW, P = a.TN * P1;
    const int64_t Vs = (int64_t)a.Sd * a.Sh * a.Sw, Vd = (int64_t)a.Dd * a.Dh * a.Dw;

    // LDS: staged channels (one more, all zero, for K entries past the end),
    // weights [k][WS], then the tables
    float* xs = lds;
    float* wsm = xs + a.xtot + a.zero;
    int* koff = (int*)(wsm + (a.wrows >> 2) * WS4);    // LDS byte offset of (channel, tap)
    uint32_t* wtap = (uint32_t*)(koff + a.kmax);      // weight byte offset of (channel, tap)
    uint32_t* poff = wtap + a.kmax;                   // source byte offset of a staged position
    const int K1 = a.CK * NT, K4 = (K1 + 3) & ~3;
    const Div byNT(NT), byHW(ah.n * aw.n), byW(aw.n), byP1(P1), byPHW(PH * PW), byPW(PW);
    const Div byChs(a.chs), byBox(a.TD * a.TH * a.TW), byTHW(a.TH * a.TW), byTW(a.TW);
    for (int i = tid; i < a.kmax; i += 256) {
        int ko = i < K4 ? 4 * a.xtot : 0;  // (read ahead past the last step: not used)
        uint32_t wo = kNoOff;
        if (i < K1) {
            const int c = byNT(i), t = i - c * NT;
            const int jd = byHW(t), r = t - jd * ah.n * aw.n, jh = byW(r);
            const int jw = r - jh * aw.n;
            ko = 4 * (c * a.chs + (jd * PH + jh) * PW + jw);
            wo = 4u * (uint32_t)(c * a.wC + ((ad.ta - s * jd) * a.k + ah.ta - s * jh) * a.k +
                                 aw.ta - s * jw);
        }
        koff[i] = ko;
        wtap[i] = wo;
    }
    for (int i = tid; i < P; i += 256) {
        const int n = byP1(i);
        int r = i - n * P1;
        const int dd = byPHW(r);
        r -= dd * PH * PW;
        const int hh = byPW(r), ww = r - hh * PW;
        const int d = d0 + ad.off + dd, h = h0 + ah.off + hh, w = w0 + aw.off + ww;
        const bool ok = n0 + n < a.N && (unsigned)d < (unsigned)a.Sd &&
                        (unsigned)h < (unsigned)a.Sh && (unsigned)w < (unsigned)a.Sw;
        poff[i] = ok ? 4u * (uint32_t)((int)(n * a.Cs * Vs) + (d * a.Sh + h) * a.Sw + w) : kNoOff;
    }
    for (int i = tid; i < a.zero; i += 256) xs[a.xtot + i] = 0.f;

    // this lane's voxels: LDS offset, and target offset (-1: not a voxel)
    const int wv = wave % WV, wk = wave / WV;
    const char* vb[VT];
    int64_t vd[VT];
#pragma unroll
    for (int v = 0; v < VT; ++v) {
        const int i = (wv * VT + v) * 16 + li;
        const int n = byBox(i);
        int r = i - n * a.TD * a.TH * a.TW;
        const int d = byTHW(r);
        r -= d * a.TH * a.TW;
        const int h = byTW(r), w = r - h * a.TW;
        const bool in = n < a.TN;
        vb[v] = (const char*)(xs + (in ? n * P1 + (d * PH + h) * PW + w : 0));
        const bool ok = in && n0 + n < a.N && d0 + d < ad.M && h0 + h < ah.M && w0 + w < aw.M;
        const int td = s * (d0 + d) + rd, th = s * (h0 + h) + rh, tw = s * (w0 + w) + rw;
        vd[v] = ok ? (int64_t)(n0 + n) * a.Ct * Vd + ((int64_t)td * a.Dh + th) * a.Dw + tw : -1;
    }

    f32x4 acc[CT][VT];
#pragma unroll
    for (int c = 0; c < CT; ++c)
#pragma unroll
        for (int v = 0; v < VT; ++v) acc[c][v] = f32x4{0.f, 0.f, 0.f, 0.f};
    __syncthreads();

    // resources starting at source channel c0: what lies past the last
    // channel is past the end and reads zero (a box of several samples only
    // has whole chunks)
    const float* sbase = a.src + (int64_t)n0 * a.Cs * Vs;
    const int ns = a.N - n0 < a.TN ? a.N - n0 : a.TN;
    auto src_rsrc = [&](int c0) {
        const int64_t left = ((int64_t)ns * a.Cs - c0) * Vs * 4;
        return buf_rsrc_u(sbase + (int64_t)c0 * Vs, (uint32_t)(left < kNoOff ? left : kNoOff));
    };
    auto w_rsrc = [&](int c0) {
        const int64_t KT = a.k * a.k * a.k;
        const int64_t left = ((int64_t)a.Cs * a.Ct * KT - (int64_t)c0 * a.wC) * 4;
        return buf_rsrc_u(a.w + (int64_t)c0 * a.wC, (uint32_t)left);
    };
    // weights: word (kb, c) of a thread is K entry 16 kb + lane % 16 of target
    // channel 16 c + 4 (lane / 16) + wave: a load reads 64 contiguous bytes of
    // four rows
    const int kl = lane & 15, wcl = 4 * (lane >> 4) + wave;
    uint32_t wrow[CT];
#pragma unroll
    for (int c = 0; c < CT; ++c)
        wrow[c] = c0t + c * 16 + wcl < a.Ct ? 4u * (uint32_t)(c0t + c * 16 + wcl) * (uint32_t)a.wM
                                            : kNoOff;
    // byte offset of K entry 16 kb + kl (rows past the chunk read zero)
    auto w_tap = [&](int rows, int kb) {
        const int kk = 16 * kb + kl;
        const uint32_t t = wtap[kk < rows ? kk : 0];
        return kk < rows ? t : kNoOff;
    };
    // kv: K entries of the chunk that exist (those of channels past the last
    // would be other channels' weights)
    float* wst = wsm + (kl >> 2) * WS4 + (kl & 3) * WS + wcl;
    auto w_store = [&](int nkb, int kv, const float (&v)[WR]) {
        const bool whole = kv >= 16 * nkb;
#pragma unroll
        for (int kb = 0; kb < WK16; ++kb)
            if (kb < nkb) {
#pragma unroll
                for (int c = 0; c < CT; ++c)
                    wst[4 * kb * WS4 + c * 16] =
                        whole || 16 * kb + kl < kv ? v[kb * CT + c] : 0.f;
            }
    };
    // K steps of four entries.  A step's operands are read while the one
    // before multiplies, its (channel, tap) offset one step earlier still; the
    // scheduling groups spread the reads over the MFMAs (left alone, the
    // compiler sinks them to their use and every step waits out the LDS
    // latency; all in front of the MFMAs, their issue is not hidden).
    auto compute = [&](int rows) {
        const int steps = rows >> 2;
        if (wk >= steps) return;
        const int n = (steps - wk + WK - 1) / WK;  // this wave's steps
        const int* kt = koff + kg + wk * 4;
        const float* wl = wsm + wk * WS4 + kg * WS + li;
        float A[2][CT], B[2][VT];
        f32x4 part[CT][VT];
#pragma unroll
        for (int c = 0; c < CT; ++c)
#pragma unroll
            for (int v = 0; v < VT; ++v) part[c][v] = f32x4{0.f, 0.f, 0.f, 0.f};
        auto read = [&](float (&x)[CT], float (&y)[VT], const float* w, int ko) {
#pragma unroll
            for (int v = 0; v < VT; ++v) y[v] = *(const float*)(vb[v] + ko);
#pragma unroll
            for (int c = 0; c < CT; ++c) x[c] = w[c * 16];
        };
        auto mul = [&](const float (&x)[CT], const float (&y)[VT]) {
#pragma unroll
            for (int c = 0; c < CT; ++c)
#pragma unroll
                for (int v = 0; v < VT; ++v) part[c][v] = mfma4(x[c], y[v], part[c][v]);
        };
        auto spread = [&] {
#pragma unroll
            for (int i = 0; i < CT * VT; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // MFMA
                __builtin_amdgcn_sched_group_barrier(0x002, 2, 0);  // VALU
                __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);  // LDS read
            }
            __builtin_amdgcn_sched_barrier(0);
        };
        constexpr int WP = WK * WS4, KP = 4 * WK;
        read(A[0], B[0], wl, kt[0]);
        int ko = kt[KP];
        for (int i = 1; i < n; i += 2) {
            read(A[1], B[1], wl + WP, ko);
            ko = kt[2 * KP];
            mul(A[0], B[0]);
            spread();
            read(A[0], B[0], wl + 2 * WP, ko);
            ko = kt[3 * KP];
            mul(A[1], B[1]);
            spread();
            wl += 2 * WP;
            kt += 2 * KP;
        }
        if (n & 1) mul(A[0], B[0]);
#pragma unroll
        for (int c = 0; c < CT; ++c)
#pragma unroll
            for (int v = 0; v < VT; ++v) acc[c][v] += part[c][v];
    };
    const int rows1 = K4;
    // words per thread (whole workgroup rows: the LDS regions are padded to them)
    const int nx = (a.CK * a.chs + 255) >> 8;
    // word e of the chunk is position e % chs of channel e / chs, at LDS offset e
    uint32_t gx[XR], gw[WK16];
    const int nkb = (rows1 + 15) >> 4;
#pragma unroll
    for (int r = 0; r < XR; ++r) {
        const int e = tid + 256 * r, c = byChs(e), i = e - c * a.chs;
        const uint32_t o = poff[i < P ? i : 0];
        gx[r] = c < a.CK && i < P && o != kNoOff ? o + 4u * (uint32_t)(c * Vs) : kNoOff;
    }
#pragma unroll
    for (int kb = 0; kb < WK16; ++kb) gw[kb] = kb < nkb ? w_tap(rows1, kb) : kNoOff;
    float vx[XR], vw[WR];
    auto load = [&](int c0) {
        const __amdgpu_buffer_rsrc_t xr = src_rsrc(c0), wr = w_rsrc(c0);
#pragma unroll
        for (int r = 0; r < XR; ++r)
            if (r < nx) vx[r] = buf_ldf(xr, gx[r]);
#pragma unroll
        for (int kb = 0; kb < WK16; ++kb)
            if (kb < nkb) {
#pragma unroll
                for (int c = 0; c < CT; ++c) vw[kb * CT + c] = buf_ldf(wr, wrow[c] + gw[kb]);
            }
    };
    auto store = [&](int c0) {
#pragma unroll
        for (int r = 0; r < XR; ++r)
            if (r < nx) xs[tid + 256 * r] = vx[r];
        w_store(nkb, (a.Cs - c0 < a.CK ? a.Cs - c0 : a.CK) * NT, vw);
    };
    if (NT > 0) {
        load(0);
        store(0);
        __syncthreads();
        for (int c0 = 0; c0 < a.Cs; c0 += a.CK) {
            const bool more = c0 + a.CK < a.Cs;
            if (more) load(c0 + a.CK);
            compute(rows1);
            __syncthreads();
            if (more) {
                store(c0 + a.CK);
                __syncthreads();
            }
        }
    }

    if constexpr (WK > 1) {
        // the other waves' sums, added in wave order
        float* red = lds;
        constexpr int R = CT * VT * 4;
        if (wk > 0) {
#pragma unroll
            for (int c = 0; c < CT; ++c)
#pragma unroll
                for (int v = 0; v < VT; ++v)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        red[(((wk - 1) * WV + wv) * R + (c * VT + v) * 4 + e) * 64 + lane] =
                            acc[c][v][e];
        }
        __syncthreads();
        if (wk > 0) return;
#pragma unroll
        for (int k = 1; k < WK; ++k)
#pragma unroll
            for (int c = 0; c < CT; ++c)
#pragma unroll
                for (int v = 0; v < VT; ++v)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        acc[c][v][e] +=
                            red[(((k - 1) * WV + wv) * R + (c * VT + v) * 4 + e) * 64 + lane];
    }
    // rows c * 16 + 4 kg + e of the tile; old values (accumulate) are all
    // loaded before the first is used (rows past the last channel load the
    // last channel's: room may be zero or negative for a lane)
    const int room = a.Ct - c0t - 4 * kg;
#pragma unroll
    for (int v = 0; v < VT; ++v) {
        if (vd[v] < 0) continue;
        float* q = a.dst + vd[v] + (int64_t)(c0t + 4 * kg) * Vd;
        if (a.accumulate) {
            f32x4 old[CT];
#pragma unroll
            for (int c = 0; c < CT; ++c)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    old[c][e] = q[(int64_t)(c * 16 + e < room ? c * 16 + e : room - 1) * Vd];
#pragma unroll
            for (int c = 0; c < CT; ++c) acc[c][v] += old[c];
        }
#pragma unroll
        for (int c = 0; c < CT; ++c)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (c * 16 + e < room) q[(int64_t)(c * 16 + e) * Vd] = acc[c][v][e];
    }
}

// ---------------------------------------------------------------- wgrad
namespace {
struct WgBox {
    const float* x;   // [N][Ci][D][H][W]
    const float* dy;  // [N][Co][Do][Ho][Wo]
    float* part;      // [splits][Co][Ci * k^3]
    ConvGeom g;
    int TN, TD, TH, TW, tn, td, th, tw;
    int CI;           // input channels per workgroup
    int chs;          // LDS floats per staged channel
    int boxes, per;   // boxes in all, boxes per split
};
__device__ __forceinline__ float buf_ldf_s(__amdgpu_buffer_rsrc_t r, uint32_t off, uint32_t soff) {
    return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, off, soff, 0));
}
// input channels a thread stages: 32 words in all (64 where few columns
// leave the registers free)
__host__ __device__ constexpr int box_cs(int jt, int pr) { return (jt == 1 ? 64 : 32) / pr; }
constexpr int kWgVox = 128;          // voxels per box
// Whether a box's sum is formed apart and added to the range's: the error is then
// that of sums of 128 products and of some boxes, not of one running sum over all
// voxels of the range (against float64, with one running sum, apart, and with the
// general kernel: 4 x 128 -> 32 at 38x52x40, stride 2, 1.2e-6, 2.3e-7 and 5.7e-7;
// 2 x 64 -> 64 at 31x26x32 7.1e-7, 2.2e-7 and 4.7e-7).  The largest shapes have no
// registers for it: their ranges are no longer than the general kernel's.  It costs
// 0.6% of the time on average over 578 random layers, up to 26% (5 x 96 -> 48, 5^3,
// stride 2, at 25x23x19: 179 and 225 us, the general kernel 261); one sum over
// several boxes costs as much.
__host__ __device__ constexpr bool box_two(int ct, int jt, int pr) {
    return ct * jt <= (pr == 16 ? 8 : 16);
}
constexpr int kDyRow = kWgVox + 4;   // LDS floats per staged dy row: 16 rows x 4 voxels hit 64 banks
}  // namespace

// dw of CT * 16 output channels by up to 4 * JT * 16 columns (tap, channel),
// wave w owning column tiles w, w + 4, ...; K = the voxels of a split's boxes.
// The next box's operands are loaded into registers while the current box
// multiplies: a thread stages PR positions of the input region for CI <= CS
// channels, and one voxel of dy for half of the output channels.
template <int CT, int JT, int PR>
__global__ __launch_bounds__(256, 2) void conv_box_wgrad(WgBox a) {
    constexpr int CS = box_cs(JT, PR), YR = CT * 16 * kWgVox / 256;
    extern __shared__ __align__(16) float lds[];
    const ConvGeom& g = a.g;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int li = lane & 15, kg = lane >> 4;
    const int KT = g.k * g.k * g.k;
    const int co0 = blockIdx.x * CT * 16, ci0 = blockIdx.y * a.CI;
    const int nci = g.Ci - ci0 < a.CI ? g.Ci - ci0 : a.CI;
    const int nco = g.Co - co0 < CT * 16 ? g.Co - co0 : CT * 16;
    const int PH = (a.TH - 1) * g.s + g.k, PW = (a.TW - 1) * g.s + g.k;
    const int P1 = ((a.TD - 1) * g.s + g.k) * PH * PW, P = a.TN * P1;
    const int Vi = g.D * g.H * g.W, Vo = g.Do * g.Ho * g.Wo;

    float* dys = lds;
    float* xs = dys + CT * 16 * kDyRow;
    int* voff = (int*)(xs + a.CI * a.chs);  // staged byte offset of a voxel, -1 where there is none
    if (tid < 8) voff[kWgVox + tid] = -1;

    // this lane's columns: c = tap * CI + channel
    const char* col[JT];
#pragma unroll
    for (int j = 0; j < JT; ++j) {
        const int c = (wave + 4 * j) * 16 + li;
        const int t = c / a.CI, ci = c - t * a.CI;
        const int kd = t / (g.k * g.k), r = t - kd * g.k * g.k, kh = r / g.k;
        col[j] = (const char*)(xs + (t < KT ? ci * a.chs + (kd * PH + kh) * PW + (r - kh * g.k) : 0));
    }
    // this thread's staged positions (packed: sample, depth, row, column) and
    // its dy voxel
    uint32_t pos[PR];
#pragma unroll
    for (int q = 0; q < PR; ++q) {
        const int i = tid + 256 * q, n = i / P1;
        int r = i - n * P1;
        const int dd = r / (PH * PW);
        r -= dd * PH * PW;
        const int hh = r / PW, ww = r - hh * PW;
        pos[q] = i < P ? (uint32_t)n << 24 | (uint32_t)dd << 16 | (uint32_t)hh << 8 | (uint32_t)ww
                       : 0xffffffffu;
    }
    const int v = tid & (kWgVox - 1);
    int vn, vdd, vh, vw, vbase;
    {
        const int box = a.TD * a.TH * a.TW;
        vn = v / box;
        int r = v - vn * box;
        vdd = r / (a.TH * a.TW);
        r -= vdd * a.TH * a.TW;
        vh = r / a.TW;
        vw = r - vh * a.TW;
        vbase = 4 * (vn * P1 + (vdd * g.s * PH + vh * g.s) * PW + vw * g.s);
    }
    constexpr bool TWO = box_two(CT, JT, PR);
    f32x4 acc[CT][JT], box[TWO ? CT : 1][TWO ? JT : 1];
#pragma unroll
    for (int c = 0; c < CT; ++c)
#pragma unroll
        for (int j = 0; j < JT; ++j) acc[c][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    float vx[PR][CS], vy[YR];
    int vo_next = -1;
    auto load = [&](int bi) {
        int b = bi;
        const int w0 = (b % a.tw) * a.TW;
        b /= a.tw;
        const int h0 = (b % a.th) * a.TH;
        b /= a.th;
        const int d0 = (b % a.td) * a.TD;
        const int n0 = b / a.td * a.TN;
        const int ns = g.N - n0 < a.TN ? g.N - n0 : a.TN;
        // dy: rows past the last output channel repeat it (their sums are not stored)
        {
            const bool ok = vn < ns && d0 + vdd < g.Do && h0 + vh < g.Ho && w0 + vw < g.Wo;
            vo_next = ok ? vbase : -1;
            const uint32_t o = ok ? 4u * (uint32_t)(vn * g.Co * Vo +
                                                    ((d0 + vdd) * g.Ho + h0 + vh) * g.Wo + w0 + vw)
                                  : kNoOff;
            const __amdgpu_buffer_rsrc_t r =
                buf_rsrc_u(a.dy + ((int64_t)n0 * g.Co + co0) * Vo, kNoOff);
#pragma unroll
            for (int q = 0; q < YR; ++q) {
                int c = 2 * q + (wave >> 1);
                c = c < nco ? c : nco - 1;
                vy[q] = buf_ldf_s(r, o, 4u * (uint32_t)c * (uint32_t)Vo);
            }
        }
        // x: channels past the last are not staged here (their columns are not stored)
        const __amdgpu_buffer_rsrc_t r = buf_rsrc_u(a.x + ((int64_t)n0 * g.Ci + ci0) * Vi, kNoOff);
#pragma unroll
        for (int q = 0; q < PR; ++q) {
            const int n = pos[q] >> 24, d = d0 * g.s - g.p + (int)((pos[q] >> 16) & 255u);
            const int h = h0 * g.s - g.p + (int)((pos[q] >> 8) & 255u);
            const int w = w0 * g.s - g.p + (int)(pos[q] & 255u);
            const bool ok = pos[q] != 0xffffffffu && n < ns && (unsigned)d < (unsigned)g.D &&
                            (unsigned)h < (unsigned)g.H && (unsigned)w < (unsigned)g.W;
            const uint32_t o = ok ? 4u * (uint32_t)(n * g.Ci * Vi + (d * g.H + h) * g.W + w) : kNoOff;
#pragma unroll
            for (int c = 0; c < CS; ++c)
                if (c < nci) vx[q][c] = buf_ldf_s(r, o, 4u * (uint32_t)c * (uint32_t)Vi);
        }
    };

    const int b0 = blockIdx.z * a.per;
    const int b1 = b0 + a.per < a.boxes ? b0 + a.per : a.boxes;
    load(b0);
    for (int bi = b0; bi < b1; ++bi) {
#pragma unroll
        for (int q = 0; q < YR; ++q) dys[(2 * q + (wave >> 1)) * kDyRow + v] = vy[q];
        if (tid < kWgVox) voff[tid] = vo_next;
#pragma unroll
        for (int q = 0; q < PR; ++q)
#pragma unroll
            for (int c = 0; c < CS; ++c)
                if (c < nci && tid + 256 * q < P) xs[c * a.chs + tid + 256 * q] = vx[q][c];
        __syncthreads();
        if (bi + 1 < b1) load(bi + 1);
        // a step: four voxels.  Operands are read one step ahead, the voxels'
        // offsets two, spread over the MFMAs (as in the forward)
        const float* al = dys + li * kDyRow + kg;
        const int* vt = voff + kg;
        float A[2][CT], B[2][JT];
        auto read = [&](int st, int vo, float (&x)[CT], float (&y)[JT]) {
            const int va = vo >= 0 ? vo : 0;
#pragma unroll
            for (int j = 0; j < JT; ++j) y[j] = *(const float*)(col[j] + va);
#pragma unroll
            for (int c = 0; c < CT; ++c) x[c] = al[c * 16 * kDyRow + st * 4];
        };
        if constexpr (TWO) {
#pragma unroll
            for (int c = 0; c < CT; ++c)
#pragma unroll
                for (int j = 0; j < JT; ++j) box[c][j] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
        // a lane without a voxel takes part with zero (never 0 * x)
        auto mul = [&](int vo, const float (&x)[CT], const float (&y)[JT]) {
#pragma unroll
            for (int j = 0; j < JT; ++j) {
                const float yj = vo >= 0 ? y[j] : 0.f;
#pragma unroll
                for (int c = 0; c < CT; ++c) {
                    f32x4& s = TWO ? box[TWO ? c : 0][TWO ? j : 0] : acc[c][j];
                    s = mfma4(x[c], yj, s);
                }
            }
        };
        auto spread = [&] {
#pragma unroll
            for (int i = 0; i < CT * JT; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // MFMA
                __builtin_amdgcn_sched_group_barrier(0x002, 2, 0);  // VALU
                __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);  // LDS read
            }
            __builtin_amdgcn_sched_barrier(0);
        };
        int vo0 = vt[0], vo1 = vt[4];
        read(0, vo0, A[0], B[0]);
        for (int st = 0; st < kWgVox / 4; st += 2) {
            // (voff has two entries' steps past the end; what they read is not used)
            read(st + 1, vo1, A[1], B[1]);
            const int vo2 = vt[(st + 2) * 4];
            mul(vo0, A[0], B[0]);
            spread();
            read(st + 2, vo2, A[0], B[0]);
            const int vo3 = vt[(st + 3) * 4];
            mul(vo1, A[1], B[1]);
            spread();
            vo0 = vo2;
            vo1 = vo3;
        }
        if constexpr (TWO) {
#pragma unroll
            for (int c = 0; c < CT; ++c)
#pragma unroll
                for (int j = 0; j < JT; ++j) acc[c][j] += box[c][j];
        }
        __syncthreads();
    }

    float* out = a.part + (int64_t)blockIdx.z * g.Co * g.Ci * KT;
#pragma unroll
    for (int j = 0; j < JT; ++j) {
        const int c = (wave + 4 * j) * 16 + li;
        const int t = c / a.CI, ci = c - t * a.CI;
        if (t >= KT || ci >= nci) continue;
#pragma unroll
        for (int k = 0; k < CT; ++k)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int co = co0 + k * 16 + 4 * kg + e;
                if (co < g.Co) out[((int64_t)co * g.Ci + ci0 + ci) * KT + t] = acc[k][j][e];
            }
    }
}

// ---------------------------------------------------------------- plans
namespace {

struct Box {
    int TN, TD, TH, TW, tn, td, th, tw;
    int64_t count() const { return (int64_t)tn * td * th * tw; }
};

// The box of at most `vox` voxels that covers an N x D x H x W map with the
// least work: the MFMAs of `vox` voxels (whether or not they exist) and, at a
// quarter of the weight, the staged positions (stride S, n taps per axis), at
// most `maxp` of them.  Several samples share a
// box only where it holds the whole map.
bool pick_box(int N, int D, int H, int W, int vox, int S, int n, int maxp, Box* out) {
    int64_t best = -1;
    auto next = [](int L, int parts) { return (int)(((unsigned)L + parts - 1) / (unsigned)parts); };
    // lengths of the balanced cuts of an axis, from the longest that fits down
    // (no more steps than the box has voxels, however long the axis is)
    for (int tw = W < vox ? W : vox; tw >= 1; --tw) {
        const int TW = next(W, next(W, tw));
        if (TW != tw) continue;
        for (int th = H < vox / TW ? H : vox / TW; th >= 1; --th) {
            const int TH = next(H, next(H, th));
            if (TH != th) continue;
            const int room = vox / (TW * TH);
            const int TD = next(D, next(D, room));
            const int PW = (TW - 1) * S + n, PH = (TH - 1) * S + n, PD = (TD - 1) * S + n;
            int TN = 1;
            if (TD == D && TH == H && TW == W) {
                TN = vox / (D * H * W);
                if (TN > N) TN = N;
                TN = next(N, next(N, TN));
                while (TN > 1 && (int64_t)TN * PD * PH * PW > maxp) --TN;
            }
            const int64_t P = (int64_t)TN * PD * PH * PW;
            if (P > maxp) continue;
            const Box b{TN, TD, TH, TW, next(N, TN), next(D, TD), next(H, TH), next(W, TW)};
            const int64_t cost = b.count() * (4 * vox + P);
            if (best < 0 || cost < best) {
                best = cost;
                *out = b;
            }
        }
    }
    return best > 0;
}

struct FdPlan {
    bool ok;
    int ct, vt, wk;
    Box box;
    int CK, KC, chs, kmax, wrows, xtot, zero;
    size_t lds;
    int blocks_x, blocks_y, classes;
};

// Cycles of the busiest CU.  A lone wave per SIMD issues a float32 MFMA every
// 40 to 43 cycles, not 32, and an LDS round trip takes about 130; each staged
// word or unit of a thread costs about 75 in a chunk, and the tables, first
// loads and stores of a workgroup 15000 to 18000 (measured with cycle
// counters).  Either the CU's MFMAs and staging add up, or the chain of
// workgroups that run one after another (`side` of them side by side) is longer.
double box_cycles(double wgs, double side, double mfma, double chain, double chunks, double words,
                  double around) {
    const double one = chain + chunks * (500 + 75 * words) + around;
    const double mul = wgs * (mfma * 1.05 + chunks * (250 + 40 * words) + around / 2);
    return mul > ceil(wgs / side) * one ? mul : ceil(wgs / side) * one;
}

// Microseconds of a pass on the gather kernels (conv_gather.hip), fitted to
// their times of 10320 random layers (k 1, 2, 3, 5, 7, strides 1 to 3, 1 to 256
// channels, 1 to 125 voxels per axis; 7 to 19 % off at one standard deviation).
double gather_us(const ConvGeom& g, int pass) {
    const int cus = device_cus();
    const double NT = g.k * g.k * g.k, Vo = (double)g.N * g.Do * g.Ho * g.Wo;
    auto up = [](double a, double b) { return ceil(a / b); };
    if (pass == 0) {
        const double steps = up(g.Ci * NT, 16), w = up(up(Vo, 64) * up(g.Co, 64), cus);
        return 3.9 + 1.0 * steps + w * (0.33 + 0.418 * steps) + 0.45 * 4e-6 * g.Co * Vo;
    }
    if (pass == 1 && g.s == 1) {
        const double steps = up(g.Co * NT, 16);
        const double w = up(up((double)g.N * g.D * g.H * g.W, 64) * up(g.Ci, 64), cus);
        const double mb = 4e-6 * g.N * g.Ci * (double)g.D * g.H * g.W;
        return 4.3 + 1.45 * steps + w * (0.35 + 0.741 * steps) + 0.33 * mb;
    }
    if (pass == 1) {  // residue classes, of n taps per axis or one fewer, and strided stores
        const double n = up(g.k, g.s), classes = (double)g.s * g.s * g.s;
        const double rows = (double)g.N * up(g.D, g.s) * up(g.H, g.s) * up(g.W, g.s);
        const double tiles = up(rows, 64) * up(g.Ci, 64) * classes;
        const double mb = 4e-6 * g.N * g.Ci * (double)g.D * g.H * g.W;
        return 5.4 + 1.51 * up(g.Co * n * n * n, 16) +
               tiles / cus * (0.84 + 0.45 * g.Co * NT / 16 / classes) + 0.34 * g.s * mb;
    }
    const double one = (double)g.Co * g.Ci * NT, tiles = up(g.Co, 64) * up(g.Ci * NT, 64);
    const double want = (double)(wgrad_gather_ws(g) / sizeof(float)) / one;
    const double steps = up(up(Vo, want), 16), splits = up(Vo, 16 * steps);
    return 3.8 + 1.34 * steps + up(tiles * splits, cus) * 0.415 * steps + 3.5e-6 * one * (splits + 1);
}
// The same of a pass planned here: `fixed`, a lone workgroup's tables, first
// loads and stores; then the planned cycles (us, at 2.4 GHz) beyond it, of
// which `share` remains (residue classes have fewer taps than the largest), or
// the megabytes of the 64-byte lines that the staged and the stored (weight
// gradient: dy) rows touch: a box of short rows costs the MFMAs nothing and
// moves up to sixteen times its voxels.  A plan is taken where it is expected to
// be faster, by the margin of the pass.  Of those layers a plan taken whenever
// there was one was more than 5 % slower than the gather kernel for 4 % of the
// forward, 5 % of the input and 26 % of the weight gradients (8 x 32 -> 32, 1^3,
// 60x50x77 forward 271 and 1100 us; 4 x 96 -> 128, 7^3 stride 3, 27x21x35
// weight gradient 623 and 1069).  With this rule, 16, 39 and 20 of 3464 further
// layers (1.46, 1.57 and 1.44 times at most), and the time of all of them is
// within 0.2 % of what the faster kernel of each would take.
constexpr double kTake[3] = {1.0, 0.95, 0.9};
double box_us(double fixed, double cycles_us, double share, double staged_mb, double stored_mb) {
    const double a = cycles_us > fixed ? share * (cycles_us - fixed) : 0;
    const double b = 0.14 * staged_mb + 0.15 * stored_mb;
    return fixed + sqrt(a * a + b * b);
}

// Shapes of workgroup that conv_box_fwd is built for: (CT, VT).
constexpr int kFwdShapes[][2] = {{4, 2}, {2, 2}, {2, 1}, {1, 4}, {1, 1}};

FdPlan make_fwd_plan(const ConvGeom& g) {
    FdPlan best{};
    double best_cost = 0;
    const int NT = g.k * g.k * g.k, K = g.Ci * NT;
    const int64_t Vs = (int64_t)g.D * g.H * g.W;
    const int cus = device_cus();
    for (const auto& sh : kFwdShapes) {
        FdPlan f{};
        f.ct = sh[0];
        f.vt = sh[1];
        f.wk = 1;
        if (f.ct > 1 && (f.ct / 2) * 16 >= g.Co) continue;  // half the rows would hold C_out
        if (f.ct == 1 && f.vt == 4 && g.Co > 16) continue;
        if (!pick_box(g.N, g.Do, g.Ho, g.Wo, f.vt * 64, g.s, g.k, kFwdXr * 256, &f.box)) continue;
        if (f.box.TN * Vs * g.Ci * 4 >= kLim) {  // 32-bit byte offsets within a box
            f.box.TN = 1;
            f.box.tn = g.N;
        }
        f.chs = f.box.TN * ((f.box.TD - 1) * g.s + g.k) * ((f.box.TH - 1) * g.s + g.k) *
                ((f.box.TW - 1) * g.s + g.k);
        // (whole 16-byte units: the weights and offsets behind it are read in those)
        f.zero = K % 16 ? (f.chs + 3) & ~3 : 0;
        f.blocks_x = (int)f.box.count();
        f.blocks_y = (int)ceil_div(g.Co, f.ct * 16);
        f.classes = 1;
        if (f.box.count() > kGridX || f.blocks_y > kGridYZ) continue;
        // K entries per chunk: what the staging registers and 52 KB of LDS
        // hold, by the same measure
        const int k16 = (K + 15) & ~15;
        for (int kc = 16; kc <= 16 * kFwdWr && kc <= k16; kc += 16) {
            const int span = (NT - 1 + kc - 1) / NT + 1, ck = span < g.Ci ? span : g.Ci;
            const size_t xtot = ((size_t)ck * f.chs + 255) & ~(size_t)255;
            const size_t lds =
                sizeof(float) * (xtot + f.chs + f.zero + (size_t)f.ct * 16 * (kc + 8) + kc +
                                 ((NT + 3) & ~3));
            if (xtot > kFwdXr * 256 || lds > 52 * 1024 || ck * Vs * 4 >= kLim) continue;
            const double groups = (K + 15) / 16, chunks = (double)ceil_div(K, kc);
            const double mf = 4 * 32.0 * f.ct * f.vt;
            const double lone = 1.25 * mf > 190 ? 1.25 * mf : 190;
            const double words = xtot / 256.0 * (ck == 1 && g.Ci == 1 ? 0 : 1) +
                                 f.ct * 16.0 * kc / 4 / 256 + 2;
            const double wgs = (double)ceil_div((int64_t)f.blocks_x * f.blocks_y, cus);
            const double side = f.ct * f.vt >= 8 || lds > 40 * 1024 ? 3 : 4;
            const double cost =
                box_cycles(wgs, side, groups * mf, groups * lone, chunks, words, 15000);
            if (!best.ok || cost < best_cost) {
                best = f;
                best.KC = kc;
                best.CK = ck;
                best.xtot = (int)xtot;
                best.lds = lds;
                best.ok = true;
                best_cost = cost;
            }
        }
    }
    if (best.ok) {
        const Box& b = best.box;
        const double rows = (double)b.count() * b.TN * ((b.TD - 1) * g.s + g.k) *
                            ((b.TH - 1) * g.s + g.k) * best.blocks_y * g.Ci;
        const double staged = 4e-6 * rows * ((b.TW - 1) * g.s + g.k + 15);
        const double stored = 4e-6 * g.N * g.Co * (double)g.Do * g.Ho * g.Wo * (b.TW + 15) / b.TW;
        // (1^3: tables of one tap and boxes without halo: half of the cycles planned)
        best.ok = box_us(5.5, best_cost / 2400, g.k == 1 ? 0.5 : 1.0, staged, stored) <
                  kTake[0] * gather_us(g, 0);
    }
    return best;
}

// Shapes of workgroup that conv_box_dgrad is built for: (CT, VT, WK).
constexpr int kFdShapes[][3] = {{4, 4, 1}, {4, 2, 1}, {2, 4, 1}, {2, 2, 1}, {1, 4, 1},
                                {2, 2, 4}, {1, 2, 4}, {1, 1, 4}};

FdPlan make_dgrad_plan(const ConvGeom& g) {
    FdPlan best{};
    double best_cost = 0;
    // voxels of the largest residue class, and the most taps of one
    const int Md = (int)ceil_div(g.D, g.s), Mh = (int)ceil_div(g.H, g.s);
    const int Mw = (int)ceil_div(g.W, g.s), n = (int)ceil_div(g.k, g.s);
    const int NT = n * n * n, cus = device_cus();
    const int64_t Vs = (int64_t)g.Do * g.Ho * g.Wo;
    for (const auto& sh : kFdShapes) {
        FdPlan f{};
        f.ct = sh[0];
        f.vt = sh[1];
        f.wk = sh[2];
        f.classes = g.s * g.s * g.s;
        if (f.ct > 1 && (f.ct / 2) * 16 >= g.Ci) continue;  // half the rows would hold C_in
        if (f.ct == 1 && f.vt == 4 && g.Ci > 16) continue;  // (2, 2) reads less: 82 vs 97 us
        const int WS4 = box_ws4(f.ct);
        if (!pick_box(g.N, Md, Mh, Mw, 4 / f.wk * f.vt * 16, 1, n, kBoxXr * 256, &f.box)) continue;
        if (f.box.TN * Vs * g.Co * 4 >= kLim) {  // 32-bit byte offsets within a box
            f.box.TN = 1;
            f.box.tn = g.N;
        }
        f.chs = f.box.TN * (f.box.TD - 1 + n) * (f.box.TH - 1 + n) * (f.box.TW - 1 + n);
        auto bytes = [&](int ck) {
            f.xtot = (ck * f.chs + 255) & ~255;
            f.zero = f.classes > 1 || ck * NT % 4 ? f.chs : 0;  // (a class may have fewer taps)
            f.wrows = (ck * NT + 15) & ~15;
            f.kmax = ((ck * NT + 3) & ~3) + 12 * f.wk;      // two steps are read ahead
            // (the weights' read-ahead runs over the tables behind them)
            const size_t tables = 2 * (size_t)f.kmax + f.chs, ahead = 2 * (size_t)f.wk * WS4;
            return sizeof(float) * ((size_t)f.xtot + f.zero + (size_t)(f.wrows / 4) * WS4 +
                                    (tables > ahead ? tables : ahead));
        };
        // source channels per chunk: what the staging registers and 52 KB of
        // LDS (three workgroups per CU) hold, in chunks of equal size
        const int maxrows = kBoxWr * 16 / f.ct;
        int ck = 0;
        for (int c = 1; c <= g.Co && c <= 64; ++c) {
            if (f.box.TN > 1 && g.Co % c) continue;
            if (((c * NT + 3) & ~3) <= maxrows && c * f.chs <= kBoxXr * 256 &&
                bytes(c) <= 52 * 1024 && c * Vs * 4 < kLim)
                ck = c;
        }
        if (!ck) continue;
        if (f.box.TN == 1) {
            ck = (int)ceil_div(g.Co, ceil_div(g.Co, ck));
            if (ck * NT % 4 && ck > 4 && ck * NT > 16) ck &= ~3;  // whole K steps
        }
        f.CK = ck;
        f.lds = bytes(ck);
        const size_t red = f.wk > 1 ? (size_t)(f.wk - 1) * (4 / f.wk) * f.ct * f.vt * 4 * 64 * 4 : 0;
        if (f.lds < red) f.lds = red;
        f.blocks_x = (int)f.box.count();
        f.blocks_y = (int)ceil_div(g.Ci, f.ct * 16);
        if (f.box.count() > kGridX || f.blocks_y > kGridYZ || f.classes > kGridYZ) continue;
        const double wgs = (double)ceil_div((int64_t)f.blocks_x * f.blocks_y * f.classes, cus);
        const double mf = 32.0 * f.ct * f.vt, lone = 1.33 * mf > 130 ? 1.33 * mf : 130;
        const double chunks = (double)ceil_div(g.Co, f.CK), ksteps = (double)g.Co * NT / 4 / f.wk;
        const double side = f.ct * f.vt >= 8 || f.lds > 53 * 1024 ? 2 : 3;
        const double cost = box_cycles(wgs, side, ksteps * mf, ksteps * lone, chunks,
                                       (f.xtot + 16.0 * f.ct * f.wrows) / 256, 18000);
        if (!best.ok || cost < best_cost) {
            best = f;
            best.ok = true;
            best_cost = cost;
        }
    }
    if (best.ok) {
        const Box& b = best.box;
        const double rows = (double)b.count() * b.TN * (b.TD - 1 + n) * (b.TH - 1 + n) *
                            best.blocks_y * best.classes * g.Co;
        // products of an average class against the largest
        const double f = (double)g.k * g.k * g.k / ((double)best.classes * NT);
        const double staged = 4e-6 * rows * f * (b.TW - 1 + n + 15);
        // (a class stores every s-th word of a row)
        const double stored = 4e-6 * g.N * g.Ci * (double)g.D * g.H * g.W * (b.TW * g.s + 15) / b.TW;
        best.ok = box_us(7.0, best_cost / 2400, 1.1 * (0.4 + 0.6 * f), staged, stored) <
                  kTake[1] * gather_us(g, 1);
    }
    return best;
}

struct WgPlan {
    bool ok;
    int ct, jt, pr;
    Box box;
    int CI, chs, splits, per;
    size_t lds;
};

// Splits whose partial sums the general path's workspace would hold, or 24 MiB
// of it where that is more, or what the bias gradient's sums leave of the
// bytes of the weight gradient without a workspace, which so refuses no more
// than with the general kernel; and no more than one launch takes.
int64_t wg_splits_max(const ConvGeom& g) {
    const int64_t one = (int64_t)g.Co * g.Ci * g.k * g.k * g.k * sizeof(float);
    const int64_t left = (int64_t)kNoallocBytes - 256 - (int64_t)bias_grad_ws(g);
    const int64_t cap = (int64_t)24 << 20;
    const int64_t a = (int64_t)wgrad_gather_ws(g) / one, b = (left < cap ? left : cap) / one;
    const int64_t m = a > b ? a : b;
    return m < kGridYZ ? m : kGridYZ;
}

WgPlan make_wg_plan(const ConvGeom& g) {
    WgPlan f{};
    const int KT = g.k * g.k * g.k;
    f.ct = g.Co > 32 ? 4 : g.Co > 16 ? 2 : 1;
    const size_t dyb = (size_t)f.ct * 16 * kDyRow * sizeof(float);
    const int maxp = (int)((kBoxLds - dyb - (kWgVox + 8) * 4) / 4) - 64;
    if (!pick_box(g.N, g.Do, g.Ho, g.Wo, kWgVox, g.s, g.k, maxp < 4096 ? maxp : 4096, &f.box))
        return f;
    const int64_t Vi = (int64_t)g.D * g.H * g.W, Vo = (int64_t)g.Do * g.Ho * g.Wo;
    if (f.box.TN * Vi * g.Ci * 4 >= kLim || f.box.TN * Vo * g.Co * 4 >= kLim) {
        f.box.TN = 1;
        f.box.tn = g.N;
    }
    const int PD = (f.box.TD - 1) * g.s + g.k, PH = (f.box.TH - 1) * g.s + g.k;
    const int PW = (f.box.TW - 1) * g.s + g.k, P = f.box.TN * PD * PH * PW;
    if (PD > 255 || PH > 255 || PW > 255 || f.box.TN > 254) return f;  // packed positions
    f.chs = ((P + 59) & ~63) + 4;  // 4 (mod 64): 16 channels x 4 voxels hit 64 banks
    f.pr = P <= 256 ? 1 : P <= 512 ? 2 : P <= 1024 ? 4 : 16;
    auto lds = [&](int ci) { return dyb + sizeof(float) * ((size_t)ci * f.chs + kWgVox + 8); };
    auto tiles4 = [&](int ci) { return (int)ceil_div(ceil_div(ci * KT, 16), 4); };
    // 32-bit byte offsets: channels of a box through the scalar offset
    if ((int64_t)f.ct * 16 * Vo * 4 >= kLim) return f;
    const int64_t boxes = f.box.count(), most = wg_splits_max(g);
    if (boxes >= kLim / 2) return f;  // (box indices are ints)
    double best = 0;
    for (int jt : {1, 2, 4, 7}) {
        // the most input channels jt column tiles per wave hold
        int ci = 0;
        for (int c = 1; c <= g.Ci && c <= 64; ++c)
            if (tiles4(c) <= jt && c <= box_cs(jt, f.pr) && lds(c) <= kBoxLds &&
                (int64_t)c * Vi * 4 < kLim)
                ci = c;
        if (!ci) continue;
        if (ci > 16) ci &= ~15;
        ci = (int)ceil_div(g.Ci, ceil_div(g.Ci, ci));
        // boxes per split: the time of the busiest CU's boxes (its MFMAs, or the
        // chain of one workgroup's boxes, two workgroups side by side) plus
        // writing and adding the partial sums at about 4.5 TB/s
        const int64_t groups = ceil_div(g.Co, f.ct * 16) * ceil_div(g.Ci, ci);
        if (ceil_div(g.Co, f.ct * 16) > kGridX || ceil_div(g.Ci, ci) > kGridYZ) continue;
        // voxels of a range of the general kernel
        const int64_t gather = ceil_div(g.N * Vo, (int64_t)(wgrad_gather_ws(g) / sizeof(float)) /
                                                  ((int64_t)g.Co * g.Ci * KT));
        const int64_t longest =
            box_two(f.ct, jt, f.pr) ? boxes : gather / kWgVox > 1 ? gather / kWgVox : 1;
        const double mf = f.ct * jt * 32.0 * (kWgVox / 4);
        const double lone = 1.3 * mf > 160 * kWgVox / 4 ? 1.3 * mf : 160 * kWgVox / 4;
        const double words = f.ct * 16 * kWgVox / 256.0 + f.pr * ci;
        const double one = lone + 500 + 140 * words;  // cycles of a lone workgroup's box
        for (int64_t per = ceil_div(boxes, most), tried = 0;
             per <= boxes && per <= longest && tried < 64; ++per, ++tried) {
            const int64_t splits = ceil_div(boxes, per);
            const double cu = (double)ceil_div(groups * splits, device_cus());
            const double a = cu * per * (mf * 1.1 + 70 * words);
            const double b = ceil(cu / 2) * (per * one + 15000);
            const double us = (a > b ? a : b) / 2400 + 8.0 * splits * g.Co * g.Ci * KT / 4.5e6;
            if (!f.ok || us < best) {
                best = us;
                f.per = (int)per;
                f.splits = (int)splits;
                f.CI = ci;
                f.jt = jt;
                f.lds = lds(ci);
                f.ok = true;
            }
        }
    }
    if (f.ok) {
        const Box& b = f.box;
        const double rows = (double)boxes * b.TN * PD * PH * ceil_div(g.Co, f.ct * 16) * g.Ci;
        const double dyrows =
            (double)boxes * b.TN * b.TD * b.TH * ceil_div(g.Ci, f.CI) * g.Co;
        const double us =
            box_us(7.0, best, 1.0, 4e-6 * rows * (PW + 15), 4e-6 * dyrows * (b.TW + 15)) +
            3.6e-6 * f.splits * g.Co * g.Ci * KT;
        f.ok = us < kTake[2] * gather_us(g, 2);
    }
    return f;
}

// A plan depends on the sizes alone; each thread keeps the last ones it made
// (a search takes some microseconds, and every call asks two or three times).
template <typename Plan> struct PlanMemo {
    struct Entry {
        ConvGeom g;
        int pass, cus;
        bool set;
        Plan plan;
    } e[64] = {};
    template <typename F> const Plan& get(const ConvGeom& g, int pass, F make) {
        uint32_t h = (uint32_t)pass;
        for (int v : {g.N, g.Ci, g.Co, g.D, g.H, g.W, g.k, g.s, g.p}) h = h * 31u + (uint32_t)v;
        Entry& x = e[(h ^ (h >> 8)) & 63];
        const int cus = device_cus();
        if (!(x.set && x.pass == pass && x.cus == cus && x.g.N == g.N && x.g.Ci == g.Ci &&
              x.g.Co == g.Co && x.g.D == g.D && x.g.H == g.H && x.g.W == g.W && x.g.k == g.k &&
              x.g.s == g.s && x.g.p == g.p))
            x = Entry{g, pass, cus, true, make()};
        return x.plan;
    }
};

const FdPlan& fd_plan(const ConvGeom& g, bool dgrad) {
    thread_local PlanMemo<FdPlan> memo;
    return memo.get(g, dgrad ? 1 : 0, [&] { return dgrad ? make_dgrad_plan(g) : make_fwd_plan(g); });
}

const WgPlan& wg_plan(const ConvGeom& g) {
    thread_local PlanMemo<WgPlan> memo;
    return memo.get(g, 2, [&] { return make_wg_plan(g); });
}

}  // namespace

bool box_fd_ok(const ConvGeom& g, rat3d_dtype dt, bool dgrad) {
    if (dt != RAT3D_F32 || g.k > kBoxMaxK) return false;
    // 1^3: a workgroup's tables and staging outweigh its few K steps on small
    // maps, where the gather kernel's short blocks are faster (us, gather vs
    // this; 64 -> 64 at 2 x 24x28x24 15.5 vs 16.7, 128 -> 128 at 2 x 21x23x22
    // 30 vs 40; 64 -> 64 at 2 x 48x56x48 69 vs 46; strided input gradient, 64 ->
    // 128 at 2 x 24x28x24, 26 vs 18)
    if (g.k == 1 && !(dgrad && g.s > 1) && (int64_t)g.N * g.Do * g.Ho * g.Wo < 131072) return false;
    // one input channel, large kernel: the region a box stages outweighs its 343
    // products per voxel (1 -> 32, 7^3 stride 2, 2 x 96x112x95: gather 184 us, this 194)
    if (!dgrad && g.Ci == 1 && g.k > 3) return false;
    const int64_t Vs = dgrad ? (int64_t)g.Do * g.Ho * g.Wo : (int64_t)g.D * g.H * g.W;
    const int64_t Vd = dgrad ? (int64_t)g.D * g.H * g.W : (int64_t)g.Do * g.Ho * g.Wo;
    const int64_t NT = (int64_t)g.k * g.k * g.k;
    if (Vs >= kLim || Vd >= kLim || (int64_t)g.Co * g.Ci * NT * 4 >= kLim) return false;
    // (a K entry's channel: Div's range, with a chunk's entries past the end)
    if (!dgrad && (g.Ci * NT + 16 * kFwdWr) * NT >= (int64_t)1 << 32) return false;
    return fd_plan(g, dgrad).ok;
}

rat3d_status conv_fd_box(const ConvGeom& g, bool dgrad, const void* src, const void* w,
                         const float* bias, void* dst, int accumulate, hipStream_t st) {
    const FdPlan& f = fd_plan(g, dgrad);
    const int KT = g.k * g.k * g.k;
    FdBox a;
    a.src = (const float*)src;
    a.w = (const float*)w;
    a.bias = bias;
    a.dst = (float*)dst;
    a.N = g.N;
    a.Cs = dgrad ? g.Co : g.Ci;
    a.Ct = dgrad ? g.Ci : g.Co;
    a.Sd = dgrad ? g.Do : g.D;
    a.Sh = dgrad ? g.Ho : g.H;
    a.Sw = dgrad ? g.Wo : g.W;
    a.Dd = dgrad ? g.D : g.Do;
    a.Dh = dgrad ? g.H : g.Ho;
    a.Dw = dgrad ? g.W : g.Wo;
    a.k = g.k;
    a.s = g.s;
    a.p = g.p;
    a.accumulate = accumulate;
    a.wM = KT;
    a.wC = g.Ci * KT;
    a.TN = f.box.TN;
    a.TD = f.box.TD;
    a.TH = f.box.TH;
    a.TW = f.box.TW;
    a.tn = f.box.tn;
    a.td = f.box.td;
    a.th = f.box.th;
    a.tw = f.box.tw;
    a.CK = f.CK;
    a.KC = f.KC;
    a.w16 = ((uintptr_t)w & 15u) == 0 && g.Ci * KT % 4 == 0 ? 1 : 0;
    a.chs = f.chs;
    a.kmax = f.kmax;
    a.wrows = f.wrows;
    a.xtot = f.xtot;
    a.zero = f.zero;
    ProfScope ps(dgrad ? "conv_box_dgrad" : "conv_box_fwd", st, conv_flops(g), conv_bytes(g, 4));
    const dim3 grid((unsigned)f.blocks_x, (unsigned)f.blocks_y, (unsigned)f.classes);
#define RAT3D_FF(C, V)                                                \
    if (!dgrad && f.ct == C && f.vt == V) {                           \
        conv_box_fwd<C, V><<<grid, 256, f.lds, st>>>(a);              \
        RAT3D_LAUNCH_CHECK();                                         \
        return RAT3D_OK;                                              \
    }
#define RAT3D_FB(C, V, K)                                             \
    if (dgrad && f.ct == C && f.vt == V && f.wk == K) {               \
        conv_box_dgrad<C, V, K><<<grid, 256, f.lds, st>>>(a);         \
        RAT3D_LAUNCH_CHECK();                                         \
        return RAT3D_OK;                                              \
    }
    RAT3D_FF(4, 2)
    RAT3D_FF(2, 2)
    RAT3D_FF(2, 1)
    RAT3D_FF(1, 4)
    RAT3D_FF(1, 1)
    RAT3D_FB(4, 4, 1)
    RAT3D_FB(4, 2, 1)
    RAT3D_FB(2, 4, 1)
    RAT3D_FB(2, 2, 1)
    RAT3D_FB(1, 4, 1)
    RAT3D_FB(2, 2, 4)
    RAT3D_FB(1, 2, 4)
    RAT3D_FB(1, 1, 4)
#undef RAT3D_FB
#undef RAT3D_FF
    set_error("conv_fd_box: no kernel for the plan");
    return RAT3D_EUNSUPPORTED;
}

bool box_wgrad_ok(const ConvGeom& g, rat3d_dtype dt) {
    if (dt != RAT3D_F32 || g.k > kBoxMaxK) return false;
    // 1^3: few products per staged word; the gather kernel is faster on large
    // maps and many channels (us, gather vs this; 64 x 64 at 2 x 24x28x24 39 vs
    // 25, 64 x 128 at 9 x 12x13x11 35 vs 33, 128 x 128 at 2 x 21x23x22 48 vs 77,
    // 64 x 64 at 2 x 48x56x48 81 vs 89)
    if (g.k == 1 && ((int64_t)g.N * g.Do * g.Ho * g.Wo > 65536 || g.Ci > 64 || g.Co > 128))
        return false;
    const int64_t Vi = (int64_t)g.D * g.H * g.W, Vo = (int64_t)g.Do * g.Ho * g.Wo;
    if (Vi >= kLim || Vo >= kLim) return false;
    return wg_plan(g).ok;
}

size_t box_wgrad_ws(const ConvGeom& g) {
    return (size_t)wg_plan(g).splits * g.Co * g.Ci * g.k * g.k * g.k * sizeof(float);
}

rat3d_status conv_wgrad_box(const ConvGeom& g, const void* x, const void* dy, float* dw,
                            int accumulate, void* ws, hipStream_t st) {
    const WgPlan& f = wg_plan(g);
    const int KT = g.k * g.k * g.k;
    WgBox a{(const float*)x, (const float*)dy, (float*)ws, g,
            f.box.TN, f.box.TD, f.box.TH, f.box.TW, f.box.tn, f.box.td, f.box.th, f.box.tw,
            f.CI, f.chs, (int)f.box.count(), f.per};
    const dim3 grid((unsigned)ceil_div(g.Co, f.ct * 16), (unsigned)ceil_div(g.Ci, f.CI),
                    (unsigned)f.splits);
    {
        ProfScope ps("conv_box_wgrad", st, conv_flops(g), conv_bytes(g, 4));
#define RAT3D_WB(C, J, R) \
    if (f.ct == C && f.jt == J && f.pr == R) conv_box_wgrad<C, J, R><<<grid, 256, f.lds, st>>>(a);
#define RAT3D_WBR(C, J) RAT3D_WB(C, J, 1) RAT3D_WB(C, J, 2) RAT3D_WB(C, J, 4) RAT3D_WB(C, J, 16)
#define RAT3D_WBJ(C) RAT3D_WBR(C, 1) RAT3D_WBR(C, 2) RAT3D_WBR(C, 4) RAT3D_WBR(C, 7)
        RAT3D_WBJ(1)
        RAT3D_WBJ(2)
        RAT3D_WBJ(4)
#undef RAT3D_WBJ
#undef RAT3D_WBR
#undef RAT3D_WB
        RAT3D_LAUNCH_CHECK();
    }
    const int64_t count = (int64_t)g.Co * g.Ci * KT;
    ProfScope ps("wgrad_reduce", st, 0.0, 4.0 * count * (f.splits + 1 + accumulate));
    return wgrad_reduce_launch((const float*)ws, f.splits, count, dw, accumulate, st);
}

}  // namespace rat3d

// What a float32 convolution pass is planned as, for the tests that keep every
// built shape of workgroup covered and the launches within their limits.
// Returns 0 where the pass does not take these kernels, else 1 and out = {CT,
// VT, WK or (weight gradient) CT, JT, PR; grid x, y, z; LDS bytes; LDS offset of
// the operand rows that are read 16 bytes at a time (forward), else 0}.
extern "C" int rat3d_box_plan(const rat3d_conv3d_desc* desc, int pass, int64_t out[8]) {
    using namespace rat3d;
    ConvGeom g;
    if (!desc || !out || check_conv_desc(desc, &g) != RAT3D_OK) return 0;
    if (pass == 2) {
        if (!box_wgrad_ok(g, desc->dtype)) return 0;
        const WgPlan& f = wg_plan(g);
        const int64_t o[8] = {f.ct, f.jt, f.pr, ceil_div(g.Co, f.ct * 16), ceil_div(g.Ci, f.CI),
                              f.splits, (int64_t)f.lds, 0};
        for (int i = 0; i < 8; ++i) out[i] = o[i];
        return 1;
    }
    if (!box_fd_ok(g, desc->dtype, pass == 1)) return 0;
    const FdPlan& f = fd_plan(g, pass == 1);
    const int64_t o[8] = {f.ct, f.vt, f.wk, f.blocks_x, f.blocks_y, f.classes, (int64_t)f.lds,
                          pass == 0 ? 4 * ((int64_t)f.xtot + f.zero) : 0};
    for (int i = 0; i < 8; ++i) out[i] = o[i];
    return 1;
}
