// Per-degree channel contraction (Eqs. struct-H, struct-phi), fp32, in whole rows:
//   Y[b*y_sb + o*y_so + k*y_sk] (+)= sum_i W[l(k)*w_sl + i*w_si + o*w_so] * X[b*x_sb + i*K + k].
//
// k_contract_mfma works degree by degree, so that a row of Y leaves in runs of 2l+1 floats, a
// degree at a time, and the L2's write requests (16 to 21 bytes each) bound it. Here a workgroup
// owns 16 consecutive k, of whatever degrees, of 16 nodes and 64 outputs: for each k it forms the
// [16 outputs x inputs] x [inputs x 16 nodes] product with that degree's weights, and every
// output row leaves as one run of 16 floats (through LDS); the input rows load the same way.
//
// A k needs operands of its own, which the fp32 matrix instructions pay for (every layout of
// this kind measured slower on them). The products therefore run on 16x16x32 bf16 instructions,
// 16 times faster, over three-part operands x = h + m + l (24 bits of significand): hh, hm, mh, mm,
// hl, lh, accumulated in fp32; what is left out is below 2^-24 of the term. The parts are exact
// where the third is no smaller than bf16's smallest step, 2^-133, so from 2^-109 on, and up to
// bf16's largest value; an infinite operand has none. A workgroup that meets a node's row or a
// group of weights outside that range (parts_lose) forms its sums in plain fp32 instead, so that
// tiny, huge and infinite operands give what k_contract_mfma gives, whichever of the two a size
// selects (the check costs 1 to 3% of a call). X is split once per workgroup into LDS, in the order
// the lanes read it; a wave splits the weights of its own 16 outputs in registers, once per degree
// and slice, loaded a degree ahead.
//
// Measured, k_contract_mfma and this kernel: on-site calls of 4,096 nodes, lmax 12, 128 channels
// and ranks 2.96 -> 2.48 ms; 2,048 nodes, lmax 4, 64/64 85 -> 75 us; 1,237 nodes, lmax 17, 72/56
// 1.02 -> 0.92 ms; edge fields, 1,000 atoms, lmax 6, 64/64 10.8 -> 10.1 ms; 10^4 atoms, lmax 6,
// 128/128 9.79 -> 9.54 ms. Errors of the whole calls against 64 bits fall (lmax 12 3.9e-7 -> 3.1e-7:
// a slice of 32 inputs is one instruction's sum). Bound by latency at three waves per SIMD, which
// registers (155) and LDS (49 KB a workgroup) set.
#include "internal.h"

namespace cgtp {

namespace {

typedef float float4_t __attribute__((ext_vector_type(4)));
typedef float float2_t __attribute__((ext_vector_type(2)));
typedef unsigned uint4_t __attribute__((ext_vector_type(4)));
typedef __bf16 bf2_t __attribute__((ext_vector_type(2)));
typedef __bf16 bf8_t __attribute__((ext_vector_type(8)));

constexpr int kThreadsR = 256;  // 4 waves of 16 outputs
constexpr int kNodes = 16;      // nodes per workgroup: the products' columns
constexpr int kRows = 64;       // outputs per workgroup
constexpr int kNk = 16;         // consecutive k per workgroup
constexpr int kSl = 32;         // inputs per slice: one matrix instruction's reduction
// A staged slice: per k the vectors [part][lane group][node] of 8 inputs, and one vector of
// padding, so that the staging lanes, consecutive in k, write to different banks.
constexpr int kStride = 3 * 4 * kNodes + 1;
constexpr int kYs = kNk + 4;    // row stride of the output transpose, clear of bank conflicts
static_assert(4 * 8 * kNodes * kYs * 4 <= kNk * kStride * 16, "the transpose reuses the slice");

// A byte offset past every resource here: loads return 0.
constexpr unsigned kOut = 0x80000000u;

__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(const void *base, unsigned bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), (short)0, (int)bytes,
                                             0x00020000);
}

__device__ __forceinline__ float bload(__amdgpu_buffer_rsrc_t rs, unsigned voff, unsigned soff)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, voff, soff, 0));
}

// The three bf16 parts of 8 values.
__device__ __forceinline__ void split8(const float *x, uint4_t (&part)[3])
{
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        float2_t r = {x[2 * k], x[2 * k + 1]};
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const unsigned bits = __builtin_bit_cast(unsigned, __builtin_convertvector(r, bf2_t));
            part[c][k] = bits;
            r[0] -= __builtin_bit_cast(float, bits << 16);
            r[1] -= __builtin_bit_cast(float, bits & 0xffff0000u);
        }
    }
}

// Whether parts lose bits of operands whose largest magnitude is m (a maximum that skips NaN, which
// parts propagate): all of them below the range (one inside dwarfs what the others lose, 2^-134
// each), or one above it.
__device__ __forceinline__ bool parts_lose(float m)
{
    return (m < 0x1p-104f && m != 0.f) || m > 0x1.fep127f;
}

// The largest of m, |a| and |b| (fmaxf would first quieten each operand, an instruction of its own).
__device__ __forceinline__ void max_abs(float &m, float a, float b)
{
    asm("v_max3_f32 %0, %0, |%1|, |%2|" : "+v"(m) : "v"(a), "v"(b));
}

// Orders a wave's LDS writes before its other lanes' reads (a wave's LDS operations complete in
// order).
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// WT: the weights are contiguous along the input (w_si == 1) and Cin is a multiple of 4. GATHER: input rows [c rows,
// (c + 1) rows) come from xg.base[c]; rows is a multiple of the slice.
template <bool WT, bool GATHER>
__global__ __launch_bounds__(kThreadsR, 3) void k_contract_rows(
    int64_t B, int Cin, int Cout, int K, int otiles, int ktiles, const float *__restrict__ W,
    unsigned w_bytes, int w_sl, int w_si, int w_so, const float *__restrict__ X, int x_sb,
    float *__restrict__ Y, int64_t y_sb, int64_t y_so, int64_t y_sk, bool accumulate, XGather xg,
    Pair2 second)
{
    __shared__ uint4_t sh[kNk * kStride];
    __shared__ int plain;  // some operand is outside the range of parts
    // Block b runs on XCD b % 8: the blocks of a node group, which share lines of X and Y, get
    // consecutive ids on one XCD.
    const int64_t nblk = gridDim.x, per = nblk / 8, rem = nblk % 8;
    const int64_t xcd = blockIdx.x % 8, slot = blockIdx.x / 8;
    int64_t bid = (xcd < rem) ? xcd * (per + 1) + slot : rem * (per + 1) + (xcd - rem) * per + slot;
    if (second.nper > 0 && bid >= second.nper) {
        bid -= second.nper;
        W = second.W;
        X = second.X;
        Y = second.Y;
    }
    const int o0 = (int)(bid % otiles) * kRows;
    const int64_t rest = bid / otiles;
    const int k0 = (int)(rest % ktiles) * kNk;
    const int64_t b0 = rest / ktiles * kNodes;
    const int nk = K - k0 < kNk ? K - k0 : kNk;
    const int nb = B - b0 < kNodes ? (int)(B - b0) : kNodes;
    int l0 = (int)sqrtf((float)k0);
    while (l0 * l0 > k0) --l0;
    while ((l0 + 1) * (l0 + 1) <= k0) ++l0;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 4, n = lane & 15;

    // staging: this thread's k and node, all inputs of the slice
    const int tk = tid & 15, tb = tid >> 4;
    const unsigned xvo = (tk < nk && tb < nb) ? (unsigned)(tb * x_sb + k0 + tk) * 4u : kOut;
    const int rows_in = GATHER ? xg.rows : Cin;
    const unsigned x_bytes = (unsigned)((nb - 1) * x_sb + rows_in * K) * 4u;
    float xr[kSl];
    auto fetch = [&](int i0) {
        const int src = GATHER ? i0 / xg.rows : 0;
        const __amdgpu_buffer_rsrc_t xs =
            rsrc((GATHER ? xg.base[src] : X) + b0 * (int64_t)x_sb, x_bytes);
        const int ib = GATHER ? i0 - src * xg.rows : i0;
#pragma unroll
        for (int i = 0; i < kSl; ++i)
            xr[i] = i0 + i < Cin ? bload(xs, xvo, (unsigned)((ib + i) * K) * 4u) : bload(xs, kOut, 0);
    };
    // weights: output o0 + 16 wave + n, inputs 8 g .. 8 g + 7 of the slice
    const __amdgpu_buffer_rsrc_t ws = rsrc(W, w_bytes);
    const int ow = o0 + 16 * wave + n;
    const unsigned wvo = ow < Cout ? (unsigned)(ow * w_so + 8 * g * w_si) * 4u : kOut;
    // scalar offsets stay within the resource (one past its end has no lane that reads)
    auto wclamp = [&](unsigned so) { return so < w_bytes ? so : 0u; };
    float wr[8];
    auto wfetch = [&](int i0, int l) {
        const unsigned so = (unsigned)(l * w_sl + i0 * w_si) * 4u;
        const int left = Cin - i0 - 8 * g;  // inputs from this lane's first one on
        if (WT) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const float4_t v = __builtin_bit_cast(
                    float4_t, __builtin_amdgcn_raw_buffer_load_b128(ws, left > 4 * h ? wvo : kOut,
                                                                    wclamp(so + 16u * h), 0));
#pragma unroll
                for (int e = 0; e < 4; ++e) wr[4 * h + e] = v[e];
            }
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e)
                wr[e] = bload(ws, left > e ? wvo : kOut, wclamp(so + (unsigned)(e * w_si) * 4u));
        }
    };

    float4_t acc[kNk];
#pragma unroll
    for (int k = 0; k < kNk; ++k) acc[k] = float4_t{0.f, 0.f, 0.f, 0.f};
    float xmax = 0.f;   // of this thread's node and k, all inputs
    bool lose = false;  // its weights, group by group

    if (tid == 0) plain = 0;
    fetch(0);
    wfetch(0, l0);
    for (int i0 = 0; i0 < Cin; i0 += kSl) {
        __syncthreads();  // the previous slice is consumed
#pragma unroll
        for (int i = 0; i < kSl; i += 2) max_abs(xmax, xr[i], xr[i + 1]);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            uint4_t part[3];
            split8(xr + 8 * q, part);
#pragma unroll
            for (int c = 0; c < 3; ++c) sh[tk * kStride + (c * 4 + q) * kNodes + tb] = part[c];
        }
        __syncthreads();
        if (i0 + kSl < Cin) fetch(i0 + kSl);
        uint4_t wp[3];
        int l = l0 - 1, kb = 0;  // the degree in wp and the k at which it ends
        uint4_t xn[3];  // the next k's vectors, read while this one's are multiplied
#pragma unroll
        for (int c = 0; c < 3; ++c) xn[c] = sh[c * 4 * kNodes + lane];
#pragma unroll
        for (int k = 0; k < kNk; ++k) {
            if (k == kb) {
                split8(wr, wp);
                float wmax = 0.f;
#pragma unroll
                for (int e = 0; e < 8; e += 2) max_abs(wmax, wr[e], wr[e + 1]);
                lose |= parts_lose(wmax);
                ++l;
                kb = (l + 1) * (l + 1) - k0;
                const bool more = kb < nk;  // else the next slice's first degree (zeros past Cin)
                wfetch(more ? i0 : i0 + kSl, more ? l + 1 : l0);
            }
            bf8_t w[3], x[3];
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                w[c] = __builtin_bit_cast(bf8_t, wp[c]);
                x[c] = __builtin_bit_cast(bf8_t, xn[c]);
                if (k + 1 < kNk) xn[c] = sh[(k + 1) * kStride + c * 4 * kNodes + lane];
            }
            if (k < nk) {
                float4_t a = acc[k];
                a = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[0], x[2], a, 0, 0, 0);
                a = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[2], x[0], a, 0, 0, 0);
                a = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[1], x[1], a, 0, 0, 0);
                a = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[0], x[1], a, 0, 0, 0);
                a = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[1], x[0], a, 0, 0, 0);
                acc[k] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[0], x[0], a, 0, 0, 0);
            }
        }
    }

    if (lose || parts_lose(xmax)) plain = 1;
    __syncthreads();  // (also: the last slice is consumed)
    if (plain) {
        const int ob = o0 + 16 * wave + 4 * g;
#pragma unroll
        for (int k = 0; k < kNk; ++k) {
            acc[k] = float4_t{0.f, 0.f, 0.f, 0.f};
            if (k >= nk || n >= nb) continue;
            int lk = l0;
            while ((lk + 1) * (lk + 1) <= k0 + k) ++lk;
            for (int i = 0; i < Cin; ++i) {
                const int src = GATHER ? i / xg.rows : 0, ii = GATHER ? i - src * xg.rows : i;
                const float x = (GATHER ? xg.base[src] : X)[(b0 + n) * x_sb + (int64_t)ii * K + k0 + k];
                const float *w = W + (int64_t)lk * w_sl + (int64_t)i * w_si;
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (ob + j < Cout) acc[k][j] += w[(int64_t)(ob + j) * w_so] * x;
            }
        }
    }
    // D[o = 4 g + j][b = n] of each k: rows (b, o) of 16 k leave through LDS, two j at a time
    float *ys = reinterpret_cast<float *>(sh) + wave * (8 * kNodes * kYs);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
        for (int jj = 0; jj < 2; ++jj)
#pragma unroll
            for (int q = 0; q < kNk / 4; ++q) {
                const int j = 2 * h + jj;
                *reinterpret_cast<float4_t *>(ys + (8 * n + 2 * g + jj) * kYs + 4 * q) =
                    float4_t{acc[4 * q][j], acc[4 * q + 1][j], acc[4 * q + 2][j], acc[4 * q + 3][j]};
            }
        wave_sync();
        // lane (g, n) stores k = n of row 4 t + g: node t / 2, output slot 4 (t % 2) + g
#pragma unroll
        for (int odd = 0; odd < 2; ++odd) {
            const int q = 4 * odd + g;
            const int o = o0 + 16 * wave + 4 * (q >> 1) + 2 * h + (q & 1);
            if (o < Cout && n < nk) {
                float *y = Y + b0 * y_sb + (int64_t)o * y_so + (int64_t)(k0 + n) * y_sk;
#pragma unroll
                for (int b = 0; b < kNodes; ++b)
                    if (b < nb) {
                        float v = ys[(8 * b + q) * kYs + n];
                        if (accumulate) v += y[b * y_sb];
                        y[b * y_sb] = v;
                    }
            }
        }
        wave_sync();
    }
}

template <bool GATHER>
hipError_t launch(int64_t blocks, int64_t B, int Cin, int Cout, int K, const float *W, int64_t w_sl,
                  int64_t w_si, int64_t w_so, const float *X, int64_t x_sb, float *Y, int64_t y_sb,
                  int64_t y_so, int64_t y_sk, bool accumulate, const XGather &xg,
                  const Pair2 &second, hipStream_t s)
{
    const int otiles = (Cout + kRows - 1) / kRows, ktiles = (K + kNk - 1) / kNk;
    const unsigned w_bytes = (unsigned)contract_rows_w_bytes(Cin, Cout, K, w_sl, w_si, w_so);
    auto *kernel = w_si == 1 && Cin % 4 == 0 ? k_contract_rows<true, GATHER> : k_contract_rows<false, GATHER>;
    hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(kThreadsR), 0, s, B, Cin, Cout, K, otiles,
                       ktiles, W, w_bytes, (int)w_sl, (int)w_si, (int)w_so, X, (int)x_sb, Y, y_sb,
                       y_so, y_sk, accumulate, xg, second);
    return hipGetLastError();
}

int64_t block_count(int64_t B, int Cout, int K)
{
    return (B + kNodes - 1) / kNodes * ((K + kNk - 1) / kNk) * ((Cout + kRows - 1) / kRows);
}

}  // namespace

bool contract_rows_takes(int64_t B, int Cin, int Cout, int K, int64_t w_sl, int64_t w_si,
                         int64_t w_so, int64_t x_sb, bool accumulate, int problems)
{
    const int64_t blocks = block_count(B, Cout, K);
    const bool large = (int64_t)Cin * Cout >= kRowsWork, wide = Cout >= kRowsWide;
    if (K < kNk || blocks < kRowsMinBlocks) return false;
    if (problems * blocks < 2 * kRowsMinBlocks && !large && !wide) return false;
    if (accumulate && !wide && (Cout <= kRows || blocks < 2 * kRowsMinBlocks)) return false;
    return 2 * blocks <= 0x7fffffffLL && w_sl >= 0 && w_si >= 0 && w_so >= 0 &&
           contract_rows_w_bytes(Cin, Cout, K, w_sl, w_si, w_so) < (int64_t)kOut &&
           4 * (kNodes * x_sb + (int64_t)(Cin + kSl) * K) < (int64_t)kOut;
}

hipError_t launch_contract_rows(int64_t B, int Cin, int Cout, int K, const float *W, int64_t w_sl,
                                int64_t w_si, int64_t w_so, const float *X, int64_t x_sb, float *Y,
                                int64_t y_sb, int64_t y_so, int64_t y_sk, bool accumulate,
                                const XGather *xg, Pair2 second, hipStream_t s)
{
    const int64_t one = block_count(B, Cout, K);
    second.nper = second.W ? one : 0;
    const int64_t blocks = second.W ? 2 * one : one;
    return xg ? launch<true>(blocks, B, Cin, Cout, K, W, w_sl, w_si, w_so, nullptr, x_sb, Y, y_sb,
                             y_so, y_sk, accumulate, *xg, second, s)
              : launch<false>(blocks, B, Cin, Cout, K, W, w_sl, w_si, w_so, X, x_sb, Y, y_sb, y_so,
                              y_sk, accumulate, XGather{}, second, s);
}

}  // namespace cgtp
