// Generic 3D convolution as an implicit GEMM on MFMA, any kernel size,
// stride and padding, float32 or bfloat16 storage.
//
// forward:  rows = output voxels (n, o), cols = C_out, K = C_in * k^3
//           A[m][(ci,t)] = x[n, ci, o*s - p + t]   (gathered, zero outside)
//           B[(ci,t)][co] = w[co, ci, t]           (contiguous in K)
// dgrad:    rows = input voxels (n, i), cols = C_in, K = C_out * k^3
//           A[m][(co,t)] = dy[n, co, (i + p - t)/s] when divisible and in range
//           B[(co,t)][ci] = w[co, ci, t]
// wgrad:    rows = C_out, cols = C_in * k^3, K = output voxels (split over
//           workgroups; partial tiles reduced in a fixed order afterwards)
//           A[co][(n,o)] = dy[n, co, o],  B[(n,o)][(ci,t)] = x[n, ci, o*s - p + t]
//
// Workgroup tile 64 x 64, four waves of 32 x 32 (2 x 2 MFMA 16x16 tiles).
// Each K step stages a 64 x BK slab of A and of B in LDS with the K index
// innermost, so that every lane fetches its MFMA operand with one 16-byte
// LDS read: bf16 uses v_mfma_f32_16x16x32_bf16 (8 K values per lane),
// float32 uses four v_mfma_f32_16x16x4_f32 (4 K values per lane).
#include <type_traits>

#include "common.hpp"
#include "kernels.hpp"
#include "vec.hpp"
#include "prof.hpp"

namespace rat3d {

template <typename T> struct MfmaCfg;
template <> struct MfmaCfg<bf16> { static constexpr int KV = 8, BK = 32; };
template <> struct MfmaCfg<float> { static constexpr int KV = 4, BK = 16; };

union Frag16 {
    uint4 u;
    bf16x8 b;
    float f[4];
    bf16 h[8];
};

template <typename T> __device__ __forceinline__ void mma16(f32x4& acc, const Frag16& a,
                                                            const Frag16& b);
template <> __device__ __forceinline__ void mma16<bf16>(f32x4& acc, const Frag16& a,
                                                        const Frag16& b) {
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.b, b.b, acc, 0, 0, 0);
}
template <> __device__ __forceinline__ void mma16<float>(f32x4& acc, const Frag16& a,
                                                         const Frag16& b) {
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a.f[0], b.f[0], acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a.f[1], b.f[1], acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a.f[2], b.f[2], acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a.f[3], b.f[3], acc, 0, 0, 0);
}

constexpr int kRow = 80;  // LDS bytes per staged row: 64 bytes of K values + 16 pad

template <typename T>
__device__ __forceinline__ void store_frag(unsigned char* lds, const T (&v)[16 / sizeof(T)]) {
    Frag16 f;
#pragma unroll
    for (int j = 0; j < (int)(16 / sizeof(T)); ++j) {
        if constexpr (sizeof(T) == 2) f.h[j] = (bf16)v[j];
        else f.f[j] = (float)v[j];
    }
    *reinterpret_cast<uint4*>(lds) = f.u;
}

// One K step of the 64x64 tile: each wave multiplies its 32x32 quarter.
template <typename T>
__device__ __forceinline__ void tile_mma(const unsigned char* As, const unsigned char* Bs,
                                         f32x4 (&acc)[2][2], int lane, int wm, int wn) {
    Frag16 a[2], b[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        a[i].u = *reinterpret_cast<const uint4*>(As + (wm * 32 + i * 16 + (lane & 15)) * kRow +
                                                 (lane >> 4) * 16);
        b[i].u = *reinterpret_cast<const uint4*>(Bs + (wn * 32 + i * 16 + (lane & 15)) * kRow +
                                                 (lane >> 4) * 16);
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) mma16<T>(acc[i][j], a[i], b[j]);
}

// ---------------------------------------------------------------- fwd / dgrad
template <typename T, bool DGRAD>
__global__ __launch_bounds__(256) void conv_gather_fd(ConvGeom g, const T* __restrict__ src,
                                                      const T* __restrict__ wt,
                                                      const float* __restrict__ bias,
                                                      T* __restrict__ dst, int accumulate) {
    constexpr int KV = MfmaCfg<T>::KV, BK = MfmaCfg<T>::BK;
    __shared__ __align__(16) unsigned char As[64 * kRow];
    __shared__ __align__(16) unsigned char Bs[64 * kRow];
    __shared__ int4 ktab[BK];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave & 1, wn = wave >> 1;
    // GEMM rows are voxels of the destination tensor.
    const int RD = DGRAD ? g.D : g.Do, RH = DGRAD ? g.H : g.Ho, RW = DGRAD ? g.W : g.Wo;
    const int64_t Vrow = (int64_t)RD * RH * RW;
    const int64_t M = (int64_t)g.N * Vrow;
    const int Ncol = DGRAD ? g.Ci : g.Co;
    const int Csrc = DGRAD ? g.Co : g.Ci;
    const int SD = DGRAD ? g.Do : g.D, SH = DGRAD ? g.Ho : g.H, SW = DGRAD ? g.Wo : g.W;
    const int64_t Vsrc = (int64_t)SD * SH * SW;
    const int KT = g.k * g.k * g.k;
    const int K = Csrc * KT;
    const int64_t m0 = (int64_t)blockIdx.x * 64;
    const int c0 = blockIdx.y * 64;

    const int ar = tid >> 2, aq = tid & 3;
    const int64_t am = m0 + ar;
    const bool arow_ok = am < M;
    int a_d = 0, a_h = 0, a_w = 0;
    int64_t a_base = 0;
    if (arow_ok) {
        const int64_t n = am / Vrow;
        int64_t sp = am - n * Vrow;
        a_d = (int)(sp / ((int64_t)RH * RW));
        sp -= (int64_t)a_d * RH * RW;
        a_h = (int)(sp / RW);
        a_w = (int)(sp - (int64_t)a_h * RW);
        a_base = n * Csrc * Vsrc;
    }
    const int bcol = c0 + (tid >> 2), bq = tid & 3;

    f32x4 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    for (int k0 = 0; k0 < K; k0 += BK) {
        if (tid < BK) {
            const int k = k0 + tid;
            int4 e = make_int4(-1, 0, 0, 0);
            if (k < K) {
                const int c = k / KT;
                const int t = k - c * KT;
                const int kd = t / (g.k * g.k);
                const int r = t - kd * g.k * g.k;
                const int kh = r / g.k;
                e = make_int4(c, kd, kh, r - kh * g.k);
            }
            ktab[tid] = e;
        }
        __syncthreads();
        {
            T v[KV];
#pragma unroll
            for (int j = 0; j < KV; ++j) {
                const int4 e = ktab[aq * KV + j];
                T val = Elt<T>::to_bits(0.f);
                if (arow_ok && e.x >= 0) {
                    if constexpr (!DGRAD) {
                        const int id = a_d * g.s - g.p + e.y, ih = a_h * g.s - g.p + e.z,
                                  iw = a_w * g.s - g.p + e.w;
                        if ((unsigned)id < (unsigned)g.D && (unsigned)ih < (unsigned)g.H &&
                            (unsigned)iw < (unsigned)g.W)
                            val = src[a_base + e.x * Vsrc + ((int64_t)id * g.H + ih) * g.W + iw];
                    } else {
                        const int nd = a_d + g.p - e.y, nh = a_h + g.p - e.z,
                                  nw = a_w + g.p - e.w;
                        if (nd >= 0 && nh >= 0 && nw >= 0 && nd % g.s == 0 && nh % g.s == 0 &&
                            nw % g.s == 0) {
                            const int od = nd / g.s, oh = nh / g.s, ow = nw / g.s;
                            if (od < g.Do && oh < g.Ho && ow < g.Wo)
                                val = src[a_base + e.x * Vsrc + ((int64_t)od * g.Ho + oh) * g.Wo +
                                          ow];
                        }
                    }
                }
                v[j] = val;
            }
            store_frag<T>(As + ar * kRow + aq * 16, v);
        }
        {
            T v[KV];
#pragma unroll
            for (int j = 0; j < KV; ++j) {
                const int k = k0 + bq * KV + j;
                T val = Elt<T>::to_bits(0.f);
                if (bcol < Ncol && k < K) {
                    if constexpr (!DGRAD) {
                        val = wt[(int64_t)bcol * K + k];
                    } else {
                        const int co = ktab[bq * KV + j].x;
                        val = wt[((int64_t)co * g.Ci + bcol) * KT + (k - co * KT)];
                    }
                }
                v[j] = val;
            }
            store_frag<T>(Bs + (tid >> 2) * kRow + bq * 16, v);
        }
        __syncthreads();
        tile_mma<T>(As, Bs, acc, lane, wm, wn);
    }

#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int row = wm * 32 + i * 16 + 4 * (lane >> 4) + e;
                const int col = wn * 32 + j * 16 + (lane & 15);
                const int64_t m = m0 + row;
                const int c = c0 + col;
                if (m < M && c < Ncol) {
                    const int64_t n = m / Vrow, sp = m - n * Vrow;
                    const int64_t off = (n * Ncol + c) * Vrow + sp;
                    float v = acc[i][j][e];
                    if (bias) v += bias[c];
                    if (accumulate) v += Elt<T>::ld(dst + off);
                    Elt<T>::st(dst + off, v);
                }
            }
}

// A thread's operands of one K step as they were loaded: eight 2-byte values
// each (or, forward weights, four words in b).  They are packed when they are
// written to LDS; packing at the load would wait for it there.
struct PipeOps {
    uint32_t a[8], b[8];
};
__device__ __forceinline__ uint4 pack8(const uint32_t (&v)[8]) {
    return make_uint4(v[0] | v[1] << 16, v[2] | v[3] << 16, v[4] | v[5] << 16, v[6] | v[7] << 16);
}
// S K steps, the loads two steps ahead of their multiplication (the grids of
// strided maps leave a CU two workgroups or so: too few waves to hide a load
// behind one step).  load(st, R) issues step st's loads, stage(st, R) writes
// them to LDS buffer st & 1, mul(st) multiplies from it.  No load sits behind a
// branch inside the loop, where it would be waited for at the branch's end.
// Every thread passes the same barriers.
template <class L, class G, class M>
__device__ __forceinline__ void pipe_steps(int S, L&& load, G&& stage, M&& mul) {
    __syncthreads();  // tables the loads read
    if (S <= 0) return;
    PipeOps R0, R1;
    load(0, R0);
    if (S > 1) load(1, R1);
    stage(0, R0);
    __syncthreads();
    int st = 0;
    for (; st + 3 < S; st += 2) {
        load(st + 2, R0);
        mul(st);
        stage(st + 1, R1);
        __syncthreads();
        load(st + 3, R1);
        mul(st + 1);
        stage(st + 2, R0);
        __syncthreads();
    }
    const int left = S - st;  // 1, 2 or 3
    if (left == 3) load(st + 2, R0);
    mul(st);
    if (left >= 2) {
        stage(st + 1, R1);
        __syncthreads();
        mul(st + 1);
    }
    if (left == 3) {
        stage(st + 2, R0);
        __syncthreads();
        mul(st + 2);
    }
}

// Forward, bfloat16, source channels a multiple of 32 (every K step of 32
// is whole): the same 64 x 64 tiles and the same order of sums, pipelined by
// pipe_steps through two LDS buffers.  A thread's 8 K values are consecutive
// taps of one or two channels: the channel and tap of the first come from one
// division, the rest by stepping the tap with a wrap.  A tap's offset and its
// coordinates as bits come from a table in LDS; a row knows which coordinates
// are outside the volume for it, so a tap costs one test, one addition and a
// buffer load that reads zero when it is outside (WIDE, for tensors of 2 GiB
// and more: 64-bit addresses).  Bound by the latency of those 2-byte loads.
// With the offset in 64-bit arithmetic per element and the loads one step
// ahead, packed at once: 8 x 64 -> 128 at 24x28x24, stride 2, 96.7 us, now
// 65.4; 8 x 128 -> 256 at 12x14x12 159.6 -> 109.4; 4 x 64 -> 128 at 46x55x46
// 238.7 -> 154.0.
constexpr int kGatherMaxTaps = 343;
template <bool WIDE>
__global__ __launch_bounds__(256) void conv_gather_fwd_pipe(ConvGeom g, const bf16* __restrict__ src,
                                                            const bf16* __restrict__ wt,
                                                            const float* __restrict__ bias,
                                                            bf16* __restrict__ dst) {
    constexpr int KV = 8, BK = 32;
    __shared__ __align__(16) unsigned char As[2][64 * kRow];
    __shared__ __align__(16) unsigned char Bs[2][64 * kRow];
    // a tap's element offset, and its bits kd | 8 + kh | 16 + kw
    __shared__ int2 taps[kGatherMaxTaps];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave & 1, wn = wave >> 1;
    const int KT = g.k * g.k * g.k, K = g.Ci * KT;
    const int64_t Vrow = (int64_t)g.Do * g.Ho * g.Wo, M = (int64_t)g.N * Vrow;
    const int64_t Vsrc = (int64_t)g.D * g.H * g.W;
    const int64_t m0 = (int64_t)blockIdx.x * 64;
    const int c0 = blockIdx.y * 64;
    for (int t = tid; t < KT; t += 256) {
        const int kd = t / (g.k * g.k), r = t - kd * g.k * g.k, kh = r / g.k;
        const int kw = r - kh * g.k;
        taps[t] = make_int2((int)(((int64_t)kd * g.H + kh) * g.W + kw),
                            1 << kd | 256 << kh | 65536 << kw);
    }

    // this thread's A row (an output voxel) and B row (an output channel)
    const int ar = tid >> 2, aq = tid & 3;
    const int64_t am = m0 + ar;
    const bool arow_ok = am < M;
    int64_t a_base = 0;  // element of tap 0 of channel 0 (may lie before the row)
    uint32_t a_out = ~0u;  // bit set: that tap coordinate is outside the volume
    if (arow_ok) {
        const int64_t n = am / Vrow;
        int64_t sp = am - n * Vrow;
        const int od = (int)(sp / ((int64_t)g.Ho * g.Wo));
        sp -= (int64_t)od * g.Ho * g.Wo;
        const int oh = (int)(sp / g.Wo), ow = (int)(sp - (int64_t)oh * g.Wo);
        const int id0 = od * g.s - g.p, ih0 = oh * g.s - g.p, iw0 = ow * g.s - g.p;
        a_base = n * g.Ci * Vsrc + ((int64_t)id0 * g.H + ih0) * g.W + iw0;
        for (int q = 0; q < g.k; ++q) {
            if ((unsigned)(id0 + q) < (unsigned)g.D) a_out &= ~(1u << q);
            if ((unsigned)(ih0 + q) < (unsigned)g.H) a_out &= ~(256u << q);
            if ((unsigned)(iw0 + q) < (unsigned)g.W) a_out &= ~(65536u << q);
        }
    }
    const __amdgpu_buffer_rsrc_t src_r =
        buf_rsrc(src, WIDE ? 0u : (uint32_t)(2 * g.N * g.Ci * (int)Vsrc));
    const int bcol = c0 + (tid >> 2);
    const bool bcol_ok = bcol < g.Co;
    const bf16* wrow = wt + (int64_t)(bcol_ok ? bcol : 0) * K;

    auto load = [&](int st, PipeOps& R) {
        const int k0 = st * BK, kf = k0 + aq * KV;
        const int c = kf / KT;
        int t = kf - c * KT;
        int64_t base = a_base + c * Vsrc;
        uint32_t base32 = (uint32_t)base * 2u;
#pragma unroll
        for (int j = 0; j < KV; ++j) {
            const int2 e = taps[t];
            const bool ok = (a_out & (uint32_t)e.y) == 0;
            if constexpr (WIDE) {
                const bf16 x = src[ok ? base + e.x : 0];
                R.a[j] = ok ? x : (bf16)0;
            } else {
                R.a[j] = buf_ld2(src_r, ok ? base32 + 2u * (uint32_t)e.x : 0x80000000u, 0u);
            }
            if (++t == KT) {
                t = 0;
                base += Vsrc;
                base32 += 2u * (uint32_t)Vsrc;
            }
        }
        const uint4 u = *reinterpret_cast<const uint4*>(wrow + k0 + aq * KV);
        R.b[0] = u.x; R.b[1] = u.y; R.b[2] = u.z; R.b[3] = u.w;
    };
    auto stage = [&](int st, const PipeOps& R) {
        const int buf = st & 1;
        *reinterpret_cast<uint4*>(As[buf] + ar * kRow + aq * 16) = pack8(R.a);
        *reinterpret_cast<uint4*>(Bs[buf] + (tid >> 2) * kRow + aq * 16) =
            bcol_ok ? make_uint4(R.b[0], R.b[1], R.b[2], R.b[3]) : make_uint4(0u, 0u, 0u, 0u);
    };

    f32x4 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    const int S = K / BK;
    pipe_steps(S, load, stage, [&](int st) {
        tile_mma<bf16>(As[st & 1], Bs[st & 1], acc, lane, wm, wn);
    });

#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int row = wm * 32 + i * 16 + 4 * (lane >> 4) + e;
                const int col = wn * 32 + j * 16 + (lane & 15);
                const int64_t m = m0 + row;
                const int c = c0 + col;
                if (m < M && c < g.Co) {
                    const int64_t n = m / Vrow, sp = m - n * Vrow;
                    float v = acc[i][j][e];
                    if (bias) v += bias[c];
                    dst[(n * g.Co + c) * Vrow + sp] = f2bf(v);
                }
            }
}

// ---------------------------------------------------------------- strided dgrad
// Input gradient of a strided convolution, decomposed by phase: input voxel
// i (per axis) receives from tap t only when s divides i + p - t, i.e. when
// t = (i + p) mod s (mod s).  The voxels of one residue class r = i mod s per
// axis therefore share one tap set (t0 + s j < k, t0 = (r + p) mod s), and
// for such a voxel i = r + s m the source position is od = m + (r + p - t)/s.
// blockIdx.z picks the class (rd, rh, rw); its rows are the class's voxels
// (n, md, mh, mw) and its K the Co x (its taps) products, so no product is a
// structural zero (the k^3 taps are split over the s^3 classes).  A class
// without taps (k < s) stores zeros (or leaves an accumulated dx unchanged).
template <typename T>
__global__ __launch_bounds__(256) void conv_gather_dgrad_phase(ConvGeom g,
                                                               const T* __restrict__ dy,
                                                               const T* __restrict__ wt,
                                                               T* __restrict__ dx,
                                                               int accumulate) {
    constexpr int KV = MfmaCfg<T>::KV, BK = MfmaCfg<T>::BK;
    __shared__ __align__(16) unsigned char As[64 * kRow];
    __shared__ __align__(16) unsigned char Bs[64 * kRow];
    __shared__ int4 ktab[BK];  // (co or -1, od offset, oh offset, ow offset)
    __shared__ int ttab[BK];   // flattened tap kd * k^2 + kh * k + kw

    const int s = g.s;
    const int cls = blockIdx.z;
    const int rd = cls / (s * s), rh = (cls / s) % s, rw = cls % s;
    // rows: the class's voxels; taps per axis
    const int Md = rd < g.D ? (g.D - rd + s - 1) / s : 0;
    const int Mh = rh < g.H ? (g.H - rh + s - 1) / s : 0;
    const int Mw = rw < g.W ? (g.W - rw + s - 1) / s : 0;
    const int t0d = (rd + g.p) % s, t0h = (rh + g.p) % s, t0w = (rw + g.p) % s;
    const int nd = t0d < g.k ? (g.k - t0d + s - 1) / s : 0;
    const int nh = t0h < g.k ? (g.k - t0h + s - 1) / s : 0;
    const int nw = t0w < g.k ? (g.k - t0w + s - 1) / s : 0;
    const int KTc = nd * nh * nw;
    const int Kc = g.Co * KTc;
    const int64_t Vc = (int64_t)Md * Mh * Mw;
    const int64_t M = (int64_t)g.N * Vc;
    const int64_t m0 = (int64_t)blockIdx.x * 64;
    if (m0 >= M) return;  // this class has fewer rows than the grid covers
    const int c0 = blockIdx.y * 64;
    const int KT = g.k * g.k * g.k;
    const int64_t Vsrc = (int64_t)g.Do * g.Ho * g.Wo;
    const int64_t Vdst = (int64_t)g.D * g.H * g.W;

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave & 1, wn = wave >> 1;
    const int ar = tid >> 2, aq = tid & 3;
    const int64_t am = m0 + ar;
    const bool arow_ok = am < M;
    int a_d = 0, a_h = 0, a_w = 0;
    int64_t a_base = 0;
    if (arow_ok) {
        const int64_t n = am / Vc;
        int64_t sp = am - n * Vc;
        a_d = (int)(sp / ((int64_t)Mh * Mw));
        sp -= (int64_t)a_d * Mh * Mw;
        a_h = (int)(sp / Mw);
        a_w = (int)(sp - (int64_t)a_h * Mw);
        a_base = n * g.Co * Vsrc;
    }
    const int bcol = c0 + (tid >> 2), bq = tid & 3;

    f32x4 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    for (int k0 = 0; k0 < Kc; k0 += BK) {
        if (tid < BK) {
            const int k = k0 + tid;
            int4 e = make_int4(-1, 0, 0, 0);
            int t = 0;
            if (k < Kc) {
                const int co = k / KTc;
                int r = k - co * KTc;
                const int jd = r / (nh * nw);
                r -= jd * nh * nw;
                const int jh = r / nw, jw = r - (r / nw) * nw;
                const int td = t0d + s * jd, th = t0h + s * jh, tw = t0w + s * jw;
                e = make_int4(co, (rd + g.p - td) / s, (rh + g.p - th) / s, (rw + g.p - tw) / s);
                t = (td * g.k + th) * g.k + tw;
            }
            ktab[tid] = e;
            ttab[tid] = t;
        }
        __syncthreads();
        {
            T v[KV];
#pragma unroll
            for (int j = 0; j < KV; ++j) {
                const int4 e = ktab[aq * KV + j];
                T val = Elt<T>::to_bits(0.f);
                if (arow_ok && e.x >= 0) {
                    const int od = a_d + e.y, oh = a_h + e.z, ow = a_w + e.w;
                    if ((unsigned)od < (unsigned)g.Do && (unsigned)oh < (unsigned)g.Ho &&
                        (unsigned)ow < (unsigned)g.Wo)
                        val = dy[a_base + e.x * Vsrc + ((int64_t)od * g.Ho + oh) * g.Wo + ow];
                }
                v[j] = val;
            }
            store_frag<T>(As + ar * kRow + aq * 16, v);
        }
        {
            T v[KV];
#pragma unroll
            for (int j = 0; j < KV; ++j) {
                const int kk = bq * KV + j;
                T val = Elt<T>::to_bits(0.f);
                const int co = ktab[kk].x;
                if (bcol < g.Ci && co >= 0)
                    val = wt[((int64_t)co * g.Ci + bcol) * KT + ttab[kk]];
                v[j] = val;
            }
            store_frag<T>(Bs + (tid >> 2) * kRow + bq * 16, v);
        }
        __syncthreads();
        tile_mma<T>(As, Bs, acc, lane, wm, wn);
    }

#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int row = wm * 32 + i * 16 + 4 * (lane >> 4) + e;
                const int col = wn * 32 + j * 16 + (lane & 15);
                const int64_t m = m0 + row;
                const int c = c0 + col;
                if (m < M && c < g.Ci) {
                    const int64_t n = m / Vc;
                    int64_t sp = m - n * Vc;
                    const int md = (int)(sp / ((int64_t)Mh * Mw));
                    sp -= (int64_t)md * Mh * Mw;
                    const int mh = (int)(sp / Mw), mw = (int)(sp - (sp / Mw) * Mw);
                    const int64_t off = (n * g.Ci + c) * Vdst +
                                        ((int64_t)(rd + s * md) * g.H + rh + s * mh) * g.W + rw +
                                        s * mw;
                    float v = acc[i][j][e];
                    if (accumulate) v += Elt<T>::ld(dx + off);
                    Elt<T>::st(dx + off, v);
                }
            }
}

// The strided input gradient in bf16 with C_out (the channels its K runs
// over) a multiple of 32, pipelined like conv_gather_fwd_pipe: the class's
// taps (at most (k / s + 1)^3) in an LDS table built once, each thread's 8
// consecutive K values (co, tap) stepped through it.  Weights are 2-byte loads
// too (a class's taps are not adjacent).  Before -> after, shapes as there:
// 144.5 -> 130.8 us, 119.8 -> 86.9, 442.5 -> 426.5.
constexpr int kPhaseMaxTaps = 64;
template <bool WIDE>
__global__ __launch_bounds__(256) void conv_gather_dgrad_phase_pipe(ConvGeom g,
                                                                    const bf16* __restrict__ dy,
                                                                    const bf16* __restrict__ wt,
                                                                    bf16* __restrict__ dx,
                                                                    int accumulate) {
    constexpr int KV = 8, BK = 32;
    __shared__ __align__(16) unsigned char As[2][64 * kRow];
    __shared__ __align__(16) unsigned char Bs[2][64 * kRow];
    // a tap's dy element offset, bits jd | 8 + jh | 16 + jw, flattened weight
    // tap kd * k^2 + kh * k + kw
    __shared__ int4 taps[kPhaseMaxTaps];

    const int s = g.s;
    const int cls = blockIdx.z;
    const int rd = cls / (s * s), rh = (cls / s) % s, rw = cls % s;
    const int Md = rd < g.D ? (g.D - rd + s - 1) / s : 0;
    const int Mh = rh < g.H ? (g.H - rh + s - 1) / s : 0;
    const int Mw = rw < g.W ? (g.W - rw + s - 1) / s : 0;
    const int t0d = (rd + g.p) % s, t0h = (rh + g.p) % s, t0w = (rw + g.p) % s;
    const int nd = t0d < g.k ? (g.k - t0d + s - 1) / s : 0;
    const int nh = t0h < g.k ? (g.k - t0h + s - 1) / s : 0;
    const int nw = t0w < g.k ? (g.k - t0w + s - 1) / s : 0;
    const int KTc = nd * nh * nw;
    const int Kc = g.Co * KTc;
    const int64_t Vc = (int64_t)Md * Mh * Mw;
    const int64_t M = (int64_t)g.N * Vc;
    const int64_t m0 = (int64_t)blockIdx.x * 64;
    if (m0 >= M) return;  // this class has fewer rows than the grid covers
    const int c0 = blockIdx.y * 64;
    const int KT = g.k * g.k * g.k;
    const int64_t Vsrc = (int64_t)g.Do * g.Ho * g.Wo;
    const int64_t Vdst = (int64_t)g.D * g.H * g.W;

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave & 1, wn = wave >> 1;
    for (int j = tid; j < KTc; j += 256) {
        const int jd = j / (nh * nw), r = j - jd * nh * nw, jh = r / nw, jw = r - jh * nw;
        const int td = t0d + s * jd, th = t0h + s * jh, tw = t0w + s * jw;
        const int64_t off = ((int64_t)((rd + g.p - td) / s) * g.Ho + (rh + g.p - th) / s) * g.Wo +
                            (rw + g.p - tw) / s;
        taps[j] = make_int4((int)off, 1 << jd | 256 << jh | 65536 << jw,
                            (td * g.k + th) * g.k + tw, 0);
    }
    const int ar = tid >> 2, aq = tid & 3;
    const int64_t am = m0 + ar;
    const bool arow_ok = am < M;
    int64_t a_base = 0;    // dy element of channel 0 at the row's own index
    uint32_t a_out = ~0u;  // bit set: that tap of the class is outside dy
    if (arow_ok) {
        const int64_t n = am / Vc;
        int64_t sp = am - n * Vc;
        const int a_d = (int)(sp / ((int64_t)Mh * Mw));
        sp -= (int64_t)a_d * Mh * Mw;
        const int a_h = (int)(sp / Mw), a_w = (int)(sp - (int64_t)a_h * Mw);
        a_base = n * g.Co * Vsrc + ((int64_t)a_d * g.Ho + a_h) * g.Wo + a_w;
        for (int q = 0; q < nd; ++q)
            if ((unsigned)(a_d + (rd + g.p - t0d - s * q) / s) < (unsigned)g.Do) a_out &= ~(1u << q);
        for (int q = 0; q < nh; ++q)
            if ((unsigned)(a_h + (rh + g.p - t0h - s * q) / s) < (unsigned)g.Ho) a_out &= ~(256u << q);
        for (int q = 0; q < nw; ++q)
            if ((unsigned)(a_w + (rw + g.p - t0w - s * q) / s) < (unsigned)g.Wo)
                a_out &= ~(65536u << q);
    }
    const __amdgpu_buffer_rsrc_t dy_r =
        buf_rsrc(dy, WIDE ? 0u : (uint32_t)(2 * g.N * g.Co * (int)Vsrc));
    const __amdgpu_buffer_rsrc_t wt_r = buf_rsrc(wt, WIDE ? 0u : (uint32_t)(2 * g.Co * g.Ci * KT));
    const int bcol = c0 + (tid >> 2);
    const bool bcol_ok = bcol < g.Ci;
    const int bc = bcol_ok ? bcol : 0;

    auto load = [&](int st, PipeOps& R) {
        const int kf = st * BK + aq * KV;
        const int co = kf / KTc;
        int j = kf - co * KTc;
        int64_t ab = a_base + co * Vsrc, bb = ((int64_t)co * g.Ci + bc) * KT;
        uint32_t ab32 = (uint32_t)ab * 2u, bb32 = (uint32_t)bb * 2u;
#pragma unroll
        for (int q = 0; q < KV; ++q) {
            const int4 e = taps[j];
            const bool ok = (a_out & (uint32_t)e.y) == 0;
            if constexpr (WIDE) {
                const bf16 xa = dy[ok ? ab + e.x : 0];
                R.a[q] = ok ? xa : (bf16)0;
                const bf16 xb = wt[bb + e.z];
                R.b[q] = bcol_ok ? xb : (bf16)0;
            } else {
                R.a[q] = buf_ld2(dy_r, ok ? ab32 + 2u * (uint32_t)e.x : 0x80000000u, 0u);
                R.b[q] = buf_ld2(wt_r, bcol_ok ? bb32 + 2u * (uint32_t)e.z : 0x80000000u, 0u);
            }
            if (++j == KTc) {
                j = 0;
                ab += Vsrc;
                ab32 += 2u * (uint32_t)Vsrc;
                bb += (int64_t)g.Ci * KT;
                bb32 += 2u * (uint32_t)(g.Ci * KT);
            }
        }
    };
    auto stage = [&](int st, const PipeOps& R) {
        const int buf = st & 1;
        *reinterpret_cast<uint4*>(As[buf] + ar * kRow + aq * 16) = pack8(R.a);
        *reinterpret_cast<uint4*>(Bs[buf] + (tid >> 2) * kRow + aq * 16) = pack8(R.b);
    };

    f32x4 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    const int S = Kc / BK;  // 0: no tap reaches this class
    pipe_steps(S, load, stage, [&](int st) {
        tile_mma<bf16>(As[st & 1], Bs[st & 1], acc, lane, wm, wn);
    });

#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int row = wm * 32 + i * 16 + 4 * (lane >> 4) + e;
                const int col = wn * 32 + j * 16 + (lane & 15);
                const int64_t m = m0 + row;
                const int c = c0 + col;
                if (m < M && c < g.Ci) {
                    const int64_t n = m / Vc;
                    int64_t sp = m - n * Vc;
                    const int md = (int)(sp / ((int64_t)Mh * Mw));
                    sp -= (int64_t)md * Mh * Mw;
                    const int mh = (int)(sp / Mw), mw = (int)(sp - (sp / Mw) * Mw);
                    const int64_t off = (n * g.Ci + c) * Vdst +
                                        ((int64_t)(rd + s * md) * g.H + rh + s * mh) * g.W + rw +
                                        s * mw;
                    float v = acc[i][j][e];
                    if (accumulate) v += bf2f(dx[off]);
                    dx[off] = f2bf(v);
                }
            }
}

// ---------------------------------------------------------------- wgrad
template <typename T>
__global__ __launch_bounds__(256) void conv_gather_wgrad(ConvGeom g, const T* __restrict__ x,
                                                         const T* __restrict__ dy,
                                                         float* __restrict__ part,
                                                         int64_t kchunk) {
    constexpr int KV = MfmaCfg<T>::KV, BK = MfmaCfg<T>::BK;
    __shared__ __align__(16) unsigned char As[64 * kRow];
    __shared__ __align__(16) unsigned char Bs[64 * kRow];
    __shared__ int4 vtab[BK];    // (n or -1, od*s-p, oh*s-p, ow*s-p)
    __shared__ int64_t vdy[BK];  // n*Co*Vo + o

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave & 1, wn = wave >> 1;
    const int KT = g.k * g.k * g.k;
    const int Ncols = g.Ci * KT;
    const int64_t Vo = (int64_t)g.Do * g.Ho * g.Wo, Vi = (int64_t)g.D * g.H * g.W;
    const int64_t Ktot = (int64_t)g.N * Vo;
    const int64_t kbeg = (int64_t)blockIdx.z * kchunk;
    const int64_t kend = kbeg + kchunk < Ktot ? kbeg + kchunk : Ktot;
    const int co0 = blockIdx.x * 64, col0 = blockIdx.y * 64;

    const int aco = co0 + (tid >> 2), aq = tid & 3;
    const int bcol = col0 + (tid >> 2), bq = tid & 3;
    int b_ci = 0, b_kd = 0, b_kh = 0, b_kw = 0;
    const bool bcol_ok = bcol < Ncols;
    if (bcol_ok) {
        b_ci = bcol / KT;
        const int t = bcol - b_ci * KT;
        b_kd = t / (g.k * g.k);
        const int r = t - b_kd * g.k * g.k;
        b_kh = r / g.k;
        b_kw = r - b_kh * g.k;
    }

    f32x4 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    for (int64_t v0 = kbeg; v0 < kend; v0 += BK) {
        if (tid < BK) {
            const int64_t v = v0 + tid;
            int4 e = make_int4(-1, 0, 0, 0);
            int64_t off = 0;
            if (v < kend) {
                const int64_t n = v / Vo;
                int64_t o = v - n * Vo;
                const int od = (int)(o / ((int64_t)g.Ho * g.Wo));
                const int64_t r = o - (int64_t)od * g.Ho * g.Wo;
                const int oh = (int)(r / g.Wo), ow = (int)(r - (int64_t)oh * g.Wo);
                e = make_int4((int)n, od * g.s - g.p, oh * g.s - g.p, ow * g.s - g.p);
                off = n * g.Co * Vo + o;
            }
            vtab[tid] = e;
            vdy[tid] = off;
        }
        __syncthreads();
        {
            T v[KV];
#pragma unroll
            for (int j = 0; j < KV; ++j) {
                T val = Elt<T>::to_bits(0.f);
                if (aco < g.Co && vtab[aq * KV + j].x >= 0)
                    val = dy[vdy[aq * KV + j] + (int64_t)aco * Vo];
                v[j] = val;
            }
            store_frag<T>(As + (tid >> 2) * kRow + aq * 16, v);
        }
        {
            T v[KV];
#pragma unroll
            for (int j = 0; j < KV; ++j) {
                T val = Elt<T>::to_bits(0.f);
                const int4 e = vtab[bq * KV + j];
                if (bcol_ok && e.x >= 0) {
                    const int id = e.y + b_kd, ih = e.z + b_kh, iw = e.w + b_kw;
                    if ((unsigned)id < (unsigned)g.D && (unsigned)ih < (unsigned)g.H &&
                        (unsigned)iw < (unsigned)g.W)
                        val = x[((int64_t)e.x * g.Ci + b_ci) * Vi + ((int64_t)id * g.H + ih) * g.W +
                                iw];
                }
                v[j] = val;
            }
            store_frag<T>(Bs + (tid >> 2) * kRow + bq * 16, v);
        }
        __syncthreads();
        tile_mma<T>(As, Bs, acc, lane, wm, wn);
    }

    float* out = part + (int64_t)blockIdx.z * g.Co * Ncols;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int co = co0 + wm * 32 + i * 16 + 4 * (lane >> 4) + e;
                const int col = col0 + wn * 32 + j * 16 + (lane & 15);
                if (co < g.Co && col < Ncols) out[(int64_t)co * Ncols + col] = acc[i][j][e];
            }
}

// The same weight gradient in bf16, k <= 7, tensors below 2 GiB (but for a few
// rows over many voxels, see the launcher), pipelined: a
// K step's 32 voxels are table entries in LDS (a ring of four, filled two steps
// ahead), {x element of tap 0, bits of the tap coordinates outside the volume,
// dy element, 0}, and an operand is a buffer load at entry + column offset.
// Tiles, K ranges and the order of the sums are those of conv_gather_wgrad,
// which waits for each step's loads before it multiplies.  It against this,
// shapes as for conv_gather_fwd_pipe: 121.9 and 113.9 us, 61.8 and 55.2, 433.4
// and 384.8; stride 1, 8 x 256 -> 256 at 3x4x3 37.1 and 33.4.
__global__ __launch_bounds__(256) void conv_gather_wgrad_pipe(ConvGeom g, const bf16* __restrict__ x,
                                                              const bf16* __restrict__ dy,
                                                              float* __restrict__ part,
                                                              int kchunk) {
    constexpr int KV = 8, BK = 32;
    __shared__ __align__(16) unsigned char As[2][64 * kRow];
    __shared__ __align__(16) unsigned char Bs[2][64 * kRow];
    __shared__ int4 vtab[4][BK];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave & 1, wn = wave >> 1;
    const int KT = g.k * g.k * g.k;
    const int Ncols = g.Ci * KT;
    const int HWo = g.Ho * g.Wo, Vo = g.Do * HWo, Vi = g.D * g.H * g.W;
    const int Ktot = g.N * Vo;
    const int kbeg = (int)blockIdx.z * kchunk;
    const int kend = Ktot - kbeg < kchunk ? Ktot : kbeg + kchunk;
    const int co0 = blockIdx.x * 64, col0 = blockIdx.y * 64;

    const int row = tid >> 2, aq = tid & 3;
    const bool a_ok = co0 + row < g.Co, b_ok = col0 + row < Ncols;
    const uint32_t a_off = (uint32_t)(co0 + row) * (uint32_t)Vo * 2u;
    uint32_t b_off = 0, b_bits = 0;
    if (b_ok) {
        const int ci = (col0 + row) / KT, t = col0 + row - ci * KT;
        const int kd = t / (g.k * g.k), r = t - kd * g.k * g.k, kh = r / g.k, kw = r - kh * g.k;
        b_off = 2u * ((uint32_t)ci * (uint32_t)Vi + (uint32_t)((kd * g.H + kh) * g.W + kw));
        b_bits = 1u << kd | 256u << kh | 65536u << kw;
    }
    const __amdgpu_buffer_rsrc_t x_r = buf_rsrc(x, (uint32_t)(2 * g.N * g.Ci * Vi));
    const __amdgpu_buffer_rsrc_t dy_r = buf_rsrc(dy, (uint32_t)(2 * g.N * g.Co * Vo));

    auto fill = [&](int st) {
        if (tid >= BK) return;
        const int v = kbeg + st * BK + tid;
        int4 e = make_int4(0, -1, -1, 0);
        if (v < kend) {
            const int n = v / Vo, o = v - n * Vo, od = o / HWo, r = o - od * HWo;
            const int oh = r / g.Wo, ow = r - oh * g.Wo;
            const int id = od * g.s - g.p, ih = oh * g.s - g.p, iw = ow * g.s - g.p;
            uint32_t out = ~0u;
            for (int q = 0; q < g.k; ++q) {
                if ((unsigned)(id + q) < (unsigned)g.D) out &= ~(1u << q);
                if ((unsigned)(ih + q) < (unsigned)g.H) out &= ~(256u << q);
                if ((unsigned)(iw + q) < (unsigned)g.W) out &= ~(65536u << q);
            }
            e = make_int4((int)(2u * ((uint32_t)(n * g.Ci) * (uint32_t)Vi +
                                      (uint32_t)((id * g.H + ih) * g.W + iw))),
                          (int)out, (int)(2u * ((uint32_t)(n * g.Co) * (uint32_t)Vo + (uint32_t)o)),
                          0);
        }
        vtab[st & 3][tid] = e;
    };
    auto load = [&](int st, PipeOps& R) {
#pragma unroll
        for (int j = 0; j < KV; ++j) {
            const int4 e = vtab[st & 3][aq * KV + j];
            R.a[j] = buf_ld2(dy_r, a_ok && e.z != -1 ? (uint32_t)e.z + a_off : 0x80000000u, 0u);
            R.b[j] = buf_ld2(x_r, b_ok && ((uint32_t)e.y & b_bits) == 0 ? (uint32_t)e.x + b_off
                                                                      : 0x80000000u, 0u);
        }
        fill(st + 2);
    };
    auto stage = [&](int st, const PipeOps& R) {
        *reinterpret_cast<uint4*>(As[st & 1] + row * kRow + aq * 16) = pack8(R.a);
        *reinterpret_cast<uint4*>(Bs[st & 1] + row * kRow + aq * 16) = pack8(R.b);
    };

    f32x4 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    fill(0);
    fill(1);
    pipe_steps((kend - kbeg + BK - 1) / BK, load, stage, [&](int st) {
        tile_mma<bf16>(As[st & 1], Bs[st & 1], acc, lane, wm, wn);
    });

    float* out = part + (int64_t)blockIdx.z * g.Co * Ncols;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int co = co0 + wm * 32 + i * 16 + 4 * (lane >> 4) + e;
                const int col = col0 + wn * 32 + j * 16 + (lane & 15);
                if (co < g.Co && col < Ncols) out[(int64_t)co * Ncols + col] = acc[i][j][e];
            }
}

// Sums `splits` partial weight-gradient slabs in split order into dw; four
// consecutive elements per thread (count is a multiple of 4 on that path).
// dw (+)= sum of the split partials, float4 lanes.  A block owns 16
// consecutive float4 outputs; its 256 threads cut the splits into 16
// contiguous chunks (thread t: output t % 16, chunk t / 16), sum them in
// split order, and the chunk sums are combined in chunk order through LDS:
// a fixed summation order with every split read by a different thread.
__global__ __launch_bounds__(256) void wgrad_reduce4(const float4* __restrict__ part, int splits,
                                                     int64_t count4, float4* __restrict__ dw,
                                                     int accumulate) {
    __shared__ float4 red[16][16];
    const int j = threadIdx.x & 15, c = threadIdx.x >> 4;
    const int64_t i = (int64_t)blockIdx.x * 16 + j;
    const int per = (splits + 15) / 16;
    const int z0 = c * per, z1 = z0 + per < splits ? z0 + per : splits;
    float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
    if (i < count4) {
#pragma unroll 4
        for (int z = z0; z < z1; ++z) {
            const float4 v = part[(int64_t)z * count4 + i];
            s.x += v.x;
            s.y += v.y;
            s.z += v.z;
            s.w += v.w;
        }
    }
    red[c][j] = s;
    __syncthreads();
    if (c == 0 && i < count4) {
        float4 t = accumulate ? dw[i] : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            t.x += red[k][j].x;
            t.y += red[k][j].y;
            t.z += red[k][j].z;
            t.w += red[k][j].w;
        }
        dw[i] = t;
    }
}

__global__ void wgrad_reduce(const float* __restrict__ part, int splits, int64_t count,
                             float* __restrict__ dw, int accumulate) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= count) return;
    float s = accumulate ? dw[i] : 0.f;
#pragma unroll 8
    for (int z = 0; z < splits; ++z) s += part[(int64_t)z * count + i];
    dw[i] = s;
}

// dbias: stage 1 sums one segment of one (n, c) plane per block (each plane
// split into SP segments), stage 2 adds each channel's N*SP segment sums in
// order.
static int bias_segments(const ConvGeom& g) {
    const int sp = (int)ceil_div(64, g.N);
    return sp < 1 ? 1 : sp;
}

// Block (c, n * SP + segment): the sum of one segment of plane (n, c).
// Segments are multiples of 8 elements; with V % 8 == 0 every thread reads
// 8 elements per 16-byte load, four loads in flight (clamped in-segment
// addresses, out-of-segment lanes masked), else one element per load.
template <typename T>
__global__ __launch_bounds__(256) void bias_grad_part(const T* __restrict__ dy, int C, int64_t V,
                                                      int SP, float* __restrict__ part) {
    __shared__ float red[256];
    const int c = blockIdx.x, sl = blockIdx.y;  // sl = n * SP + segment
    const int n = sl / SP, seg = sl - n * SP;
    const int64_t len = ((V + SP - 1) / SP + 7) & ~(int64_t)7;
    const int64_t beg = seg * len, end = beg + len < V ? beg + len : V;
    const T* p = dy + ((int64_t)n * C + c) * V;
    float s = 0.f;
    constexpr int VEC = 16 / (int)sizeof(T);
    if (V % VEC == 0 && end > beg) {
        constexpr int64_t STEP = 256 * VEC;
        for (int64_t e0 = beg + threadIdx.x * VEC; e0 < end; e0 += 4 * STEP) {
            float v[4][VEC];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int64_t e = e0 + u * STEP;
                vload<T, VEC>(p + (e < end ? e : end - VEC), v[u]);
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const bool ok = e0 + u * STEP < end;
#pragma unroll
                for (int j = 0; j < VEC; ++j) s += ok ? v[u][j] : 0.f;
            }
        }
    } else {
        for (int64_t e = beg + threadIdx.x; e < end; e += 256) s += Elt<T>::ld(p + e);
    }
    red[threadIdx.x] = s;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[(int64_t)c * gridDim.y + sl] = red[0];
}

__global__ void bias_grad_final(const float* __restrict__ part, int C, int S,
                                float* __restrict__ db, int accumulate) {
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= C) return;
    float s = accumulate ? db[c] : 0.f;
    for (int i = 0; i < S; ++i) s += part[(int64_t)c * S + i];
    db[c] = s;
}

size_t bias_grad_ws(const ConvGeom& g) {
    return (size_t)g.Co * g.N * bias_segments(g) * sizeof(float);
}

// ---------------------------------------------------------------- launchers
int wgrad_gather_splits(const ConvGeom& g) {
    const int64_t Ktot = (int64_t)g.N * g.Do * g.Ho * g.Wo;
    const int64_t tiles = ceil_div(g.Co, 64) * ceil_div((int64_t)g.Ci * g.k * g.k * g.k, 64);
    int64_t splits = ceil_div(2048, tiles);
    const int64_t max_splits = ceil_div(Ktot, 256);  // at least 256 voxels per split
    if (splits > max_splits) splits = max_splits;
    if (splits < 1) splits = 1;
    if (splits > 4096) splits = 4096;
    return (int)splits;
}

size_t wgrad_gather_ws(const ConvGeom& g) {
    return (size_t)wgrad_gather_splits(g) * g.Co * g.Ci * g.k * g.k * g.k * sizeof(float);
}

double conv_flops(const ConvGeom& g) {
    return 2.0 * g.N * g.Co * g.Ci * (double)(g.k * g.k * g.k) * g.Do * g.Ho * g.Wo;
}

double conv_bytes(const ConvGeom& g, size_t esz) {
    return (double)esz * ((double)g.N * g.Ci * g.D * g.H * g.W +
                          (double)g.Co * g.Ci * g.k * g.k * g.k +
                          (double)g.N * g.Co * g.Do * g.Ho * g.Wo);
}

// The pipelined kernels address whole tensors with 32-bit byte offsets into a
// buffer whose out-of-range reads are zero; tensors of 2 GiB and more take
// 64-bit addresses (WIDE).
static bool pipe_narrow(const ConvGeom& g) {
    const int64_t lim = (int64_t)1 << 30;  // 2-byte elements
    return (int64_t)g.N * g.Ci * g.D * g.H * g.W < lim &&
           (int64_t)g.N * g.Co * g.Do * g.Ho * g.Wo < lim &&
           (int64_t)g.Co * g.Ci * g.k * g.k * g.k < lim;
}

template <typename T>
static rat3d_status gather_fd(const ConvGeom& g, bool dgrad, const void* src, const void* w,
                              const float* bias, void* dst, int accumulate, hipStream_t st) {
    ProfScope ps(dgrad ? "conv_gather_dgrad" : "conv_gather_fwd", st, conv_flops(g),
                 conv_bytes(g, sizeof(T)));
    const int64_t rows = (int64_t)g.N * (dgrad ? (int64_t)g.D * g.H * g.W
                                               : (int64_t)g.Do * g.Ho * g.Wo);
    const int cols = dgrad ? g.Ci : g.Co;
    dim3 grid((unsigned)ceil_div(rows, 64), (unsigned)ceil_div(cols, 64));
    if constexpr (std::is_same<T, bf16>::value) {
        // (16-byte weight loads: K = Ci k^3 is a multiple of 8, the base must be aligned;
        // a tap's offset in 32 bits)
        if (!dgrad && !accumulate && g.Ci % 32 == 0 && g.k * g.k * g.k <= kGatherMaxTaps &&
            ((uintptr_t)w & 15u) == 0 && (int64_t)g.k * g.H * g.W < ((int64_t)1 << 31)) {
            if (pipe_narrow(g))
                conv_gather_fwd_pipe<false><<<grid, 256, 0, st>>>(g, (const bf16*)src,
                                                                  (const bf16*)w, bias, (bf16*)dst);
            else
                conv_gather_fwd_pipe<true><<<grid, 256, 0, st>>>(g, (const bf16*)src,
                                                                 (const bf16*)w, bias, (bf16*)dst);
            RAT3D_LAUNCH_CHECK();
            return RAT3D_OK;
        }
    }
    if (dgrad)
        conv_gather_fd<T, true><<<grid, 256, 0, st>>>(g, (const T*)src, (const T*)w, nullptr,
                                                      (T*)dst, accumulate);
    else
        conv_gather_fd<T, false><<<grid, 256, 0, st>>>(g, (const T*)src, (const T*)w, bias,
                                                       (T*)dst, accumulate);
    RAT3D_LAUNCH_CHECK();
    return RAT3D_OK;
}

rat3d_status conv_fwd_gather(const ConvGeom& g, rat3d_dtype dt, const void* x, const void* w,
                             const float* bias, void* y, hipStream_t st) {
    return dt == RAT3D_BF16 ? gather_fd<bf16>(g, false, x, w, bias, y, 0, st)
                            : gather_fd<float>(g, false, x, w, bias, y, 0, st);
}

template <typename T>
static rat3d_status gather_dgrad_phase(const ConvGeom& g, const void* dy, const void* w, void* dx,
                                       int accumulate, hipStream_t st) {
    ProfScope ps("conv_gather_dgrad_s2", st, conv_flops(g), conv_bytes(g, sizeof(T)));
    // the largest class (residue 0 on every axis) sets the row grid
    const int64_t rows = (int64_t)g.N * ceil_div(g.D, g.s) * ceil_div(g.H, g.s) *
                         ceil_div(g.W, g.s);
    dim3 grid((unsigned)ceil_div(rows, 64), (unsigned)ceil_div(g.Ci, 64),
              (unsigned)(g.s * g.s * g.s));
    if constexpr (std::is_same<T, bf16>::value) {
        // class tap sets of at most (k / s + 1)^3 taps, a tap's offset in 32 bits
        const int tps = g.k / g.s + 1;
        if (g.Co % 32 == 0 && tps * tps * tps <= kPhaseMaxTaps &&
            (int64_t)g.k * g.Ho * g.Wo < ((int64_t)1 << 31)) {
            if (pipe_narrow(g))
                conv_gather_dgrad_phase_pipe<false><<<grid, 256, 0, st>>>(
                    g, (const bf16*)dy, (const bf16*)w, (bf16*)dx, accumulate);
            else
                conv_gather_dgrad_phase_pipe<true><<<grid, 256, 0, st>>>(
                    g, (const bf16*)dy, (const bf16*)w, (bf16*)dx, accumulate);
            RAT3D_LAUNCH_CHECK();
            return RAT3D_OK;
        }
    }
    conv_gather_dgrad_phase<T><<<grid, 256, 0, st>>>(g, (const T*)dy, (const T*)w, (T*)dx,
                                                     accumulate);
    RAT3D_LAUNCH_CHECK();
    return RAT3D_OK;
}

rat3d_status conv_dgrad_gather(const ConvGeom& g, rat3d_dtype dt, const void* dy, const void* w,
                               void* dx, int accumulate, hipStream_t st) {
    if (g.s > 1)  // phase-decomposed: no structurally zero products
        return dt == RAT3D_BF16 ? gather_dgrad_phase<bf16>(g, dy, w, dx, accumulate, st)
                                : gather_dgrad_phase<float>(g, dy, w, dx, accumulate, st);
    return dt == RAT3D_BF16 ? gather_fd<bf16>(g, true, dy, w, nullptr, dx, accumulate, st)
                            : gather_fd<float>(g, true, dy, w, nullptr, dx, accumulate, st);
}

rat3d_status conv_wgrad_gather(const ConvGeom& g, rat3d_dtype dt, const void* x, const void* dy,
                               float* dw, int accumulate, void* ws, hipStream_t st) {
    const int splits = wgrad_gather_splits(g);
    const int64_t Ktot = (int64_t)g.N * g.Do * g.Ho * g.Wo;
    const int BK = dt == RAT3D_BF16 ? 32 : 16;
    const int64_t kchunk = ceil_div(ceil_div(Ktot, splits), BK) * BK;
    const int real_splits = (int)ceil_div(Ktot, kchunk);
    const int Ncols = g.Ci * g.k * g.k * g.k;
    dim3 grid((unsigned)ceil_div(g.Co, 64), (unsigned)ceil_div(Ncols, 64), (unsigned)real_splits);
    float* part = (float*)ws;
    {
    ProfScope ps("conv_gather_wgrad", st, conv_flops(g),
                 conv_bytes(g, dt == RAT3D_BF16 ? 2 : 4));
    // Few live rows of a tile's 64 + 64 over many voxels: the plain kernel loads
    // nothing for the others, the pipelined one issues every load (us, plain and
    // pipelined: 1^3, 5 x 8 -> 8 at 83x82x111 218 and 279, 8 x 12 -> 12 at 87x76x76
    // 242 and 302, 5 x 20 -> 20 at 66x59x62 98 and 109; 3^3, 16 x 1 -> 1 at 88x88x104
    // 859 and 967; 4 x 4 -> 8 at 42x40x49 37 and 40; with more rows or fewer voxels the
    // pipelined one is as fast or faster: 3^3, 16 x 2 -> 2 at 70x105x102 947 and 852)
    const bool sparse = g.Co + Ncols <= 48 && Ktot >= 320000;
    if (dt == RAT3D_BF16 && g.k <= 7 && pipe_narrow(g) && !sparse)
        conv_gather_wgrad_pipe<<<grid, 256, 0, st>>>(g, (const bf16*)x, (const bf16*)dy, part,
                                                     (int)kchunk);
    else if (dt == RAT3D_BF16)
        conv_gather_wgrad<bf16><<<grid, 256, 0, st>>>(g, (const bf16*)x, (const bf16*)dy, part,
                                                      kchunk);
    else
        conv_gather_wgrad<float><<<grid, 256, 0, st>>>(g, (const float*)x, (const float*)dy,
                                                       part, kchunk);
    RAT3D_LAUNCH_CHECK();
    }
    const int64_t count = (int64_t)g.Co * Ncols;
    ProfScope ps("wgrad_reduce", st, 0.0, 4.0 * count * (real_splits + 1 + accumulate));
    return wgrad_reduce_launch(part, real_splits, count, dw, accumulate, st);
}

rat3d_status wgrad_reduce_launch(const float* part, int splits, int64_t count, float* dw,
                                 int accumulate, hipStream_t st) {
    if (count % 4 == 0 && ((uintptr_t)dw & 15u) == 0 && ((uintptr_t)part & 15u) == 0)
        wgrad_reduce4<<<(unsigned)ceil_div(count / 4, 16), 256, 0, st>>>(
            (const float4*)part, splits, count / 4, (float4*)dw, accumulate);
    else
        wgrad_reduce<<<(unsigned)ceil_div(count, 256), 256, 0, st>>>(part, splits, count, dw,
                                                                     accumulate);
    RAT3D_LAUNCH_CHECK();
    return RAT3D_OK;
}

rat3d_status conv_bias_grad(const ConvGeom& g, rat3d_dtype dt, const void* dy, float* db,
                            int accumulate, void* ws, hipStream_t st) {
    const int64_t Vo = (int64_t)g.Do * g.Ho * g.Wo;
    float* part = (float*)ws;
    ProfScope ps("bias_grad", st, 0.0, (dt == RAT3D_BF16 ? 2.0 : 4.0) * g.N * g.Co * Vo);
    const int SP = bias_segments(g);
    const dim3 grid(g.Co, g.N * SP);
    if (dt == RAT3D_BF16)
        bias_grad_part<bf16><<<grid, 256, 0, st>>>((const bf16*)dy, g.Co, Vo, SP, part);
    else
        bias_grad_part<float><<<grid, 256, 0, st>>>((const float*)dy, g.Co, Vo, SP, part);
    RAT3D_LAUNCH_CHECK();
    bias_grad_final<<<(unsigned)ceil_div(g.Co, 64), 64, 0, st>>>(part, g.Co, g.N * SP, db,
                                                                 accumulate);
    RAT3D_LAUNCH_CHECK();
    return RAT3D_OK;
}

// One wave per channel: lane l adds partials l, l + 64, ... in turn, then an
// xor butterfly (a fixed order for a given S).
__global__ __launch_bounds__(64) void bias_sum_wave(const float* __restrict__ part, int S,
                                                    float* __restrict__ db, int accumulate) {
    const int c = blockIdx.x, lane = threadIdx.x;
    const float* p = part + (int64_t)c * S;
    float s = 0.f;
    for (int i = lane; i < S; i += 64) s += p[i];
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) s += __shfl_xor(s, m, 64);
    if (lane == 0) db[c] = accumulate ? db[c] + s : s;
}

rat3d_status bias_grad_from_partials(const float* part, int C, int S, float* db, int accumulate,
                                     hipStream_t st) {
    bias_sum_wave<<<(unsigned)C, 64, 0, st>>>(part, S, db, accumulate);
    RAT3D_LAUNCH_CHECK();
    return RAT3D_OK;
}

}  // namespace rat3d
