// On-site grid stage, fp32, lmax <= kOnsiteFoldedMaxL: one workgroup per
// (node, block of rb ranks), one thread per (rank, Gauss-Legendre node u).
//
// A thread keeps the Legendre coefficients F[m] and dF/dx[m] of both operands in
// registers (Eq. struct-F and its x-derivative pass), then sweeps the azimuth four points at a
// time. The integrand needs V >= 3 lmax + 1 equispaced azimuths wherever they start, so the
// sweep takes V4 = 4 Q of them at half steps, phi_v = 2 pi (v + 1/2) / V4: phi, -phi, pi - phi
// and pi + phi then are four different points whose cos(m phi) and sin(m phi) differ in sign
// only, by the parity of m (at low degrees whole steps, fold_whole, which are more accurate
// there: a step more, whose ends count half). Four partial sums per field (cosine and sine, even and odd m)
// give its values (Eq. struct-tildeA) at all four, where the product (Eq. struct-S) and the
// surface curl (Eq. poisson-S2-x) are formed, and four signed sums of those go back into the
// Fourier analysis (Eq. struct-Tmu): a quarter of the products of a plain sweep, half of those
// of one folded once (v, V - v), for 3% more points at most above lmax 10. The Gauss-Legendre
// analysis across u (Eq. struct-Tlm) goes through LDS, one output field at a time, in the space
// the coefficient rows held (they are dead once the Legendre pass is in registers); a thread
// keeps one (l, m) and its weight row in registers over the ranks it serves. The curl is swept
// first and the product after it, when the derivative coefficients are dead.
//
// Bound by vector instructions (VALU issue 0.85 to 1.0). Measured, before (azimuths folded once,
// one sweep for both products, weights read per rank) and now: 4,096 nodes, 128 ranks, lmax 12
// 1.94 -> 1.35 ms; 2,048 nodes, 64 ranks: lmax 4 46 -> 36 us, lmax 6 100 -> 76 us, lmax 10
// 390 -> 164 us, lmax 14 1204 -> 681 us. With one sweep's registers gone it also beats
// k_onsite_mfma up to lmax 20 (same sizes: lmax 15 1.54 -> 0.72 ms, 17 2.80 -> 1.12, 20 4.58 ->
// 2.81); beyond, four coefficient rows and a Fourier row pass 256 registers.
//
// With per-block factors (general parameterization) the Gaunt product takes the values of the
// Gaunt factors' contractions HA, HB and the surface curl the derivative fields of the curl
// factors' contractions HAc, HBc; that kernel sweeps the two one after the other, with both
// output rows in registers and the same LDS reuse.
#include "internal.h"

namespace cgtp {

namespace {

typedef float float4_t __attribute__((ext_vector_type(4)));

// Partial sums of a field at one azimuth phi of the first quadrant: cosine sums over even and
// odd m, sine sums over even and odd m.
struct Quad {
    float ce, co, se, so;
};

// Adds order k's cosine coefficient fc (factor c) and sine coefficient fs (factor s).
__device__ __forceinline__ void quad_add(Quad &a, int k, float c, float fc, float s, float fs)
{
    if (k & 1) {
        a.co += c * fc;
        a.so += s * fs;
    } else {
        a.ce += c * fc;
        a.se += s * fs;
    }
}

// The field at phi, -phi, pi - phi, pi + phi: cos(k (pi - phi)) = (-1)^k cos(k phi),
// sin(k (pi - phi)) = -(-1)^k sin(k phi).
__device__ __forceinline__ void quad_values(const Quad &a, float (&v)[4])
{
    const float p = a.ce + a.co, m = a.ce - a.co, q = a.se + a.so, r = a.so - a.se;
    v[0] = p + q;
    v[1] = p - q;
    v[2] = m + r;
    v[3] = m - r;
}

// Adds the Fourier analysis of a field's four values: T[m] += sum_v q_vm S_v.
template <int LM>
__device__ __forceinline__ void quad_analyse(const float (&v)[4], const float *qr, float *T)
{
    const float p = v[0] + v[1], q = v[2] + v[3], m = v[0] - v[1], n = v[2] - v[3];
    const float ce = p + q, co = p - q, se = m - n, so = m + n;
    T[LM] += ce;
#pragma unroll
    for (int k = 1; k <= LM; ++k) {
        T[LM + k] += qr[LM + k] * (k & 1 ? co : ce);
        T[LM - k] += qr[LM - k] * (k & 1 ? so : se);
    }
}

// Row strides in LDS: the Legendre tables' rows (an odd length, so that the lanes' rows u start
// on different banks) and the Fourier rows [m][ts] (16-byte words; an odd number of them per row
// keeps the reads of consecutive m off each other's banks).
__host__ __device__ constexpr int table_stride(int P) { return P | 1; }
__host__ __device__ constexpr int tm_stride(int ut) { return ut + (ut % 8 == 0 ? 4 : 0); }

// Writes one thread's Fourier row (rank q, node u) of a field into Tm [rank][m][ts], with zeros
// in the padding of the last node.
template <int LM>
__device__ __forceinline__ void store_fourier(float *Tm, int ts, int q, int u, int U,
                                              const float *T)
{
    constexpr int M = 2 * LM + 1;
    float *tm = Tm + q * M * ts + u;
#pragma unroll
    for (int mi = 0; mi < M; ++mi) tm[mi * ts] = T[mi];
    if (u == U - 1)
        for (int mi = 0; mi < M; ++mi)
            for (int p = 1; (u + p) % 4 != 0; ++p) tm[mi * ts + p] = 0.f;
}

// Gauss-Legendre analysis of one field's Fourier rows of nr ranks (Eq. struct-Tlm): dst[q][k] =
// sum_u wpf[(l, |m|)][u] Tm[q][m][u]. A thread keeps one k = (l, m), its weight row in registers
// (UT nodes, the default grid of the call; other grids read it per rank), over every gq-th rank.
template <int LM, int UT>
__device__ __forceinline__ void gl_analyse(const Tabs<float> &tb, const float *Tm, int nr,
                                           float *__restrict__ dst)
{
    constexpr int M = 2 * LM + 1, K = (LM + 1) * (LM + 1);
    const int nt = blockDim.x, ut = (tb.d.U + 3) / 4 * 4, ts = tm_stride(ut);
    const int gq = K < nt ? nt / K : 1;
    for (int kq = threadIdx.x; kq < K * gq; kq += nt) {
        const int q0 = kq / K, k = kq - q0 * K;
        // sqrt(k + 1/2) lies at least 1/(4 (l + 1)) from an integer, far more than the hardware
        // square root's error at these k
        const int l = (int)__builtin_amdgcn_sqrtf((float)k + 0.5f);
        const int m = k - l * l - l, am = m < 0 ? -m : m;
        const float4_t *w4 =
            reinterpret_cast<const float4_t *>(tb.wpf + (l * (l + 1) / 2 + am) * ut);
        if (ut == UT) {
            constexpr int NC = UT / 4;
            float4_t w[NC];
#pragma unroll
            for (int c = 0; c < NC; ++c) w[c] = w4[c];
            for (int q = q0; q < nr; q += gq) {
                const float4_t *t4 =
                    reinterpret_cast<const float4_t *>(Tm + (q * M + m + LM) * tm_stride(UT));
                float s = 0.f;
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                    const float4_t t = t4[c];
                    s += w[c][0] * t[0] + w[c][1] * t[1] + w[c][2] * t[2] + w[c][3] * t[3];
                }
                dst[q * K + k] = s;
            }
        } else {
            for (int q = q0; q < nr; q += gq) {
                const float4_t *t4 =
                    reinterpret_cast<const float4_t *>(Tm + (q * M + m + LM) * ts);
                float s = 0.f;
                for (int c = 0; c < ut / 4; ++c) {
                    const float4_t w = w4[c], t = t4[c];
                    s += w[0] * t[0] + w[1] * t[1] + w[2] * t[2] + w[3] * t[3];
                }
                dst[q * K + k] = s;
            }
        }
    }
}

// GL nodes, rounded up to 4, of the default grid of a product of nu fields (Ut of the plan).
constexpr int default_ut(int lm, int nu)
{
    const int u = nu == 2 ? (3 * lm + 3) / 2 : ((nu + 1) * lm + 2) / 2;
    return ((u < 1 ? 1 : u) + 3) / 4 * 4;
}

// Whole steps (fold_whole): the first and last step's four points are two, each counted twice, so
// one factor of the product counts half there (its partial sums, exactly: the products and their
// sums keep their rounding).
template <int LM>
__device__ __forceinline__ void halve_ends(Quad &a, int step, int steps, bool whole)
{
    if (LM < 1 || LM > kFoldWholeMaxL) return;  // always half steps
    const float w = whole && (step == 0 || step == steps - 1) ? 0.5f : 1.f;
    a.ce *= w;
    a.co *= w;
    a.se *= w;
    a.so *= w;
}

// Azimuth sweep of one row at latitude u for the Gaunt product (Eq. struct-S): synthesise
// A from FA and B from FB at the four points of each quadrant step and add the Fourier analysis
// (Eq. struct-Tmu) of A B into T. qs: the plan's qf, passed down from a read-only kernel argument
// so that each row is read with scalar loads.
template <int LM>
__device__ __forceinline__ void sweep_product(const float *FA, const float *FB, const float *qs,
                                              int steps, bool whole, float *T)
{
    constexpr int M = 2 * LM + 1;
    for (int v = 0; v < steps; ++v) {
        const float *qr = qs + v * M;
        Quad a{FA[LM], 0.f, 0.f, 0.f}, c{FB[LM], 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 1; k <= LM; ++k) {
            quad_add(a, k, qr[LM + k], FA[LM + k], qr[LM - k], FA[LM - k]);
            quad_add(c, k, qr[LM + k], FB[LM + k], qr[LM - k], FB[LM - k]);
        }
        halve_ends<LM>(a, v, steps, whole);
        float va[4], vc[4];
        quad_values(a, va);
        quad_values(c, vc);
#pragma unroll
        for (int p = 0; p < 4; ++p) va[p] *= vc[p];
        quad_analyse<LM>(va, qr, T);
    }
}

// The same sweep for the surface curl (Eq. poisson-S2-x): dA/dphi dB/dx - dA/dx dB/dphi,
// with the phi-derivatives taken from FA, FB by swapping the cosine and sine halves.
template <int LM>
__device__ __forceinline__ void sweep_curl(const float *FA, const float *FxA, const float *FB,
                                           const float *FxB, const float *qs, const float *qds,
                                           int steps, bool whole, float *T)
{
    constexpr int M = 2 * LM + 1;
    for (int v = 0; v < steps; ++v) {
        const float *qr = qs + v * M, *qdr = qds + v * M;
        Quad ax{FxA[LM], 0.f, 0.f, 0.f}, ap{0.f, 0.f, 0.f, 0.f};
        Quad cx{FxB[LM], 0.f, 0.f, 0.f}, cp{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 1; k <= LM; ++k) {
            const float cs = qr[LM + k], sn = qr[LM - k];
            const float kc = qdr[LM + k], mks = qdr[LM - k];  // k cos, -k sin
            quad_add(ax, k, cs, FxA[LM + k], sn, FxA[LM - k]);
            quad_add(ap, k, kc, FA[LM - k], mks, FA[LM + k]);
            quad_add(cx, k, cs, FxB[LM + k], sn, FxB[LM - k]);
            quad_add(cp, k, kc, FB[LM - k], mks, FB[LM + k]);
        }
        halve_ends<LM>(ap, v, steps, whole);
        halve_ends<LM>(ax, v, steps, whole);
        float vx[4], vp[4], sb[4];
        quad_values(ap, vp);
        quad_values(cx, vx);
#pragma unroll
        for (int p = 0; p < 4; ++p) sb[p] = vp[p] * vx[p];
        quad_values(ax, vx);
        quad_values(cp, vp);
#pragma unroll
        for (int p = 0; p < 4; ++p) sb[p] -= vx[p] * vp[p];
        quad_analyse<LM>(sb, qr, T);
    }
}

// Degree 0 on one node and one quadruple of azimuths: a field is its one value there, so a thread
// takes a rank from coefficient to coefficient, with the sweeps' arithmetic and without their LDS
// passes (20,000 nodes, 16 ranks, whole call 28 -> 25 us; on the former kernels 25).
__device__ __forceinline__ float analyse_constant(const Tabs<float> &tb, float v)
{
    return tb.wpf[0] * (4.f * v);
}

// Waves per SIMD of k_onsite_folded: what the registers of four coefficient rows and one Fourier
// row leave room for (unforced, the scheduler takes a wave's registers more at lmax 8 and 9 and
// the grid stage 176 instead of 149 us, 2,048 nodes, 64 ranks).
constexpr int folded_waves(int lm) { return lm >= 15 ? 2 : lm >= 11 ? 3 : lm >= 7 ? 4 : 1; }

// qg, qdg: the plan's qf and qdf as read-only arguments: the azimuth sweep reads one row of each
// per step, the same for every thread, as scalar loads (operands from scalar registers, no LDS
// traffic in the sweep).
template <int LM>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(folded_waves(LM))))
void k_onsite_folded(Tabs<float> tb, int R, int rb, int steps, bool whole,
                     const float *__restrict__ qg, const float *__restrict__ qdg,
                     const float *__restrict__ HA, const float *__restrict__ HB,
                     float *__restrict__ Ta, float *__restrict__ Tb)
{
    constexpr int M = 2 * LM + 1, L = LM + 1, K = L * L, P = L * (L + 1) / 2;
    constexpr int PS = table_stride(P);
    extern __shared__ __attribute__((aligned(16))) float smem[];
    const int U = tb.d.U, ts = tm_stride((U + 3) / 4 * 4);
    float *Tm = smem;  // [rb][M][ts]: one field's Fourier rows, in the space of
    float *Hs = smem;  // [2][rb][K]: the coefficient rows
    const int shared = 2 * rb * K > rb * M * ts ? 2 * rb * K : rb * M * ts;
    float *ps = smem + (shared + 3) / 4 * 4;  // [U][PS]
    float *dps = ps + U * PS;                 // [U][PS]

    const int nrb = (R + rb - 1) / rb;
    const int64_t b = blockIdx.x / nrb;
    const int r0 = (int)(blockIdx.x - b * nrb) * rb;
    const int nr = (R - r0 < rb) ? (R - r0) : rb;
    const int64_t row0 = (b * R + r0) * (int64_t)K;
    if (LM == 0 && U == 1 && steps == 1) {
        if ((int)threadIdx.x < nr) {
            const float h1 = HA[row0 + threadIdx.x], h2 = HB[row0 + threadIdx.x];
            const float p = tb.p[0], dp = tb.dp[0];
            Ta[row0 + threadIdx.x] = analyse_constant(tb, (p * h1) * (p * h2));
            Tb[row0 + threadIdx.x] = analyse_constant(tb, 0.f * (dp * h2) - (dp * h1) * 0.f);
        }
        return;
    }
    for (int k = threadIdx.x; k < U * P; k += blockDim.x) {
        const int uu = k / P, o = uu * PS + k - uu * P;
        ps[o] = tb.p[k];
        dps[o] = tb.dp[k];
    }
    for (int k = threadIdx.x; k < nr * K; k += blockDim.x) {
        Hs[k] = HA[row0 + k];
        Hs[rb * K + k] = HB[row0 + k];
    }
    __syncthreads();

    const int q = threadIdx.x / U, u = threadIdx.x - q * U;
    const bool active = q < nr;
    float FA[M], FxA[M], FB[M], FxB[M], T[M];
    if (active) {
        const float *h1 = Hs + q * K, *h2 = Hs + (rb + q) * K;
        const float *pu = ps + u * PS, *dpu = dps + u * PS;
#pragma unroll
        for (int mi = 0; mi < M; ++mi) {
            const int m = mi - LM, am = m < 0 ? -m : m;
            float f1 = 0.f, g1 = 0.f, f2 = 0.f, g2 = 0.f;
#pragma unroll
            for (int l = am; l <= LM; ++l) {
                const float p = pu[l * (l + 1) / 2 + am], dp = dpu[l * (l + 1) / 2 + am];
                const float c1 = h1[l * l + l + m], c2 = h2[l * l + l + m];
                f1 += p * c1;
                g1 += dp * c1;
                f2 += p * c2;
                g2 += dp * c2;
            }
            FA[mi] = f1;
            FxA[mi] = g1;
            FB[mi] = f2;
            FxB[mi] = g2;
        }
    }
    __syncthreads();  // every thread has its coefficients: Hs is free for Tm
    // The curl's sweep and analysis, then the product's: the derivative coefficients are dead
    // once the curl is done, so the registers hold four coefficient rows and one Fourier row at
    // most
#pragma unroll
    for (int mi = 0; mi < M; ++mi) T[mi] = 0.f;
    if (active) {
        sweep_curl<LM>(FA, FxA, FB, FxB, qg, qdg, steps, whole, T);
        store_fourier<LM>(Tm, ts, q, u, U, T);
    }
    __syncthreads();
    gl_analyse<LM, default_ut(LM, 2)>(tb, Tm, nr, Tb + row0);
#pragma unroll
    for (int mi = 0; mi < M; ++mi) T[mi] = 0.f;
    if (active) sweep_product<LM>(FA, FB, qg, steps, whole, T);
    __syncthreads();  // the curl's Fourier rows are read
    if (active) store_fourier<LM>(Tm, ts, q, u, U, T);
    __syncthreads();
    gl_analyse<LM, default_ut(LM, 2)>(tb, Tm, nr, Ta + row0);
}

// LDS bytes of a folded kernel: `rows` staged coefficient rows per rank (whose space then holds
// one field's Fourier rows) and `tables` Legendre tables.
size_t folded_lds(const Dims &d, int rb, int rows, int tables)
{
    const size_t M = d.M, K = d.K, ts = tm_stride((d.U + 3) / 4 * 4);
    const size_t shared = rows * K > M * ts ? rows * K : M * ts;
    return sizeof(float) * ((rb * shared + 3) / 4 * 4 + (size_t)tables * d.U * table_stride(d.P));
}

template <int LM>
hipError_t launch_folded(const Tabs<float> &tb, int64_t B, int R, const float *HA,
                         const float *HB, float *Ta, float *Tb, hipStream_t s)
{
    const int U = tb.d.U;
    int rb = 256 / U;
    if (rb > R) rb = R;
    if (rb < 1) return hipErrorInvalidValue;
    while (rb > 1 && folded_lds(tb.d, rb, 2, 2) > (size_t)tb.d.lds_max) --rb;
    const size_t lds = folded_lds(tb.d, rb, 2, 2);
    if (lds > (size_t)tb.d.lds_max) return hipErrorInvalidValue;
    const int threads = (rb * U + 63) / 64 * 64;
    const int64_t blocks = B * ((R + rb - 1) / rb);
    hipLaunchKernelGGL((k_onsite_folded<LM>), dim3((unsigned)blocks), dim3(threads), lds, s, tb, R,
                       rb, fold_rows(tb.d), fold_whole(tb.d), tb.qf, tb.qdf, HA, HB, Ta, Tb);
    return hipGetLastError();
}

// Per-block factors: the workgroup stages the Gaunt rows HA, HB and the curl rows HAc, HBc
// once; each (rank, u) thread sweeps the surface curl from the second pair (values and
// x-derivatives), then the Gaunt product from the first (values only: the smaller register set
// while the curl's Fourier row is held), keeping both Fourier rows in registers. Once every thread has its coefficients the staged rows are dead and their LDS
// holds one output field's Fourier rows at a time for the Gauss-Legendre analysis, as in
// k_onsite_folded.
template <int LM>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(LM == 11 || LM == 12 ? 3 : 1)))
void k_onsite_split(Tabs<float> tb, int R, int rb, int steps, bool whole, const float *__restrict__ qg,
                    const float *__restrict__ qdg, const float *__restrict__ HA,
                    const float *__restrict__ HB, const float *__restrict__ HAc,
                    const float *__restrict__ HBc, float *__restrict__ Ta,
                    float *__restrict__ Tb)
{
    constexpr int M = 2 * LM + 1, L = LM + 1, K = L * L, P = L * (L + 1) / 2;
    constexpr int PS = table_stride(P);
    extern __shared__ __attribute__((aligned(16))) float smem[];
    const int U = tb.d.U, ts = tm_stride((U + 3) / 4 * 4);
    float *Tm = smem;  // [rb][M][ts]: one field's Fourier rows, in the space of
    float *Hs = smem;  // [4][rb][K]: HA, HB, HAc, HBc rows
    const int shared = 4 * rb * K > rb * M * ts ? 4 * rb * K : rb * M * ts;
    float *ps = smem + (shared + 3) / 4 * 4;  // [U][PS]
    float *dps = ps + U * PS;                 // [U][PS]

    const int nrb = (R + rb - 1) / rb;
    const int64_t b = blockIdx.x / nrb;
    const int r0 = (int)(blockIdx.x - b * nrb) * rb;
    const int nr = (R - r0 < rb) ? (R - r0) : rb;
    for (int k = threadIdx.x; k < U * P; k += blockDim.x) {
        const int uu = k / P, o = uu * PS + k - uu * P;
        ps[o] = tb.p[k];
        dps[o] = tb.dp[k];
    }
    const int64_t row0 = (b * R + r0) * (int64_t)K;
    if (LM == 0 && U == 1 && steps == 1) {
        if ((int)threadIdx.x < nr) {
            const float h1 = HA[row0 + threadIdx.x], h2 = HB[row0 + threadIdx.x];
            const float c1 = HAc[row0 + threadIdx.x], c2 = HBc[row0 + threadIdx.x];
            const float p = tb.p[0], dp = tb.dp[0];
            Ta[row0 + threadIdx.x] = analyse_constant(tb, (p * h1) * (p * h2));
            Tb[row0 + threadIdx.x] = analyse_constant(tb, 0.f * (dp * c2) - (dp * c1) * 0.f);
        }
        return;
    }
    for (int k = threadIdx.x; k < nr * K; k += blockDim.x) {
        Hs[k] = HA[row0 + k];
        Hs[rb * K + k] = HB[row0 + k];
        Hs[2 * rb * K + k] = HAc[row0 + k];
        Hs[3 * rb * K + k] = HBc[row0 + k];
    }
    __syncthreads();

    const int q = threadIdx.x / U, u = threadIdx.x - q * U;
    const bool active = q < nr;
    float TA[M], TB[M];
#pragma unroll
    for (int mi = 0; mi < M; ++mi) TA[mi] = TB[mi] = 0.f;
    if (active) {
        const float *pu = ps + u * PS, *dpu = dps + u * PS;
        {
            const float *h1 = Hs + (2 * rb + q) * K, *h2 = Hs + (3 * rb + q) * K;
            float FA[M], FxA[M], FB[M], FxB[M];
#pragma unroll
            for (int mi = 0; mi < M; ++mi) {
                const int m = mi - LM, am = m < 0 ? -m : m;
                float f1 = 0.f, g1 = 0.f, f2 = 0.f, g2 = 0.f;
#pragma unroll
                for (int l = am; l <= LM; ++l) {
                    const float p = pu[l * (l + 1) / 2 + am], dp = dpu[l * (l + 1) / 2 + am];
                    const float c1 = h1[l * l + l + m], c2 = h2[l * l + l + m];
                    f1 += p * c1;
                    g1 += dp * c1;
                    f2 += p * c2;
                    g2 += dp * c2;
                }
                FA[mi] = f1;
                FxA[mi] = g1;
                FB[mi] = f2;
                FxB[mi] = g2;
            }
            sweep_curl<LM>(FA, FxA, FB, FxB, qg, qdg, steps, whole, TB);
        }
        {
            const float *h1 = Hs + q * K, *h2 = Hs + (rb + q) * K;
            float FA[M], FB[M];
#pragma unroll
            for (int mi = 0; mi < M; ++mi) {
                const int m = mi - LM, am = m < 0 ? -m : m;
                float f1 = 0.f, f2 = 0.f;
#pragma unroll
                for (int l = am; l <= LM; ++l) {
                    const float p = pu[l * (l + 1) / 2 + am];
                    f1 += p * h1[l * l + l + m];
                    f2 += p * h2[l * l + l + m];
                }
                FA[mi] = f1;
                FB[mi] = f2;
            }
            sweep_product<LM>(FA, FB, qg, steps, whole, TA);
        }
    }
    __syncthreads();  // every thread has its Fourier rows: Hs is free for Tm
    // Gauss-Legendre analysis, one field at a time
#pragma unroll
    for (int which = 0; which < 2; ++which) {
        if (active) store_fourier<LM>(Tm, ts, q, u, U, which ? TB : TA);
        __syncthreads();
        gl_analyse<LM, default_ut(LM, 2)>(tb, Tm, nr, (which ? Tb : Ta) + row0);
        __syncthreads();  // Tm is read before the next field overwrites it
    }
}

template <int LM>
hipError_t launch_split(const Tabs<float> &tb, int64_t B, int R, const float *HA,
                        const float *HB, const float *HAc, const float *HBc, float *Ta,
                        float *Tb, hipStream_t s)
{
    const int U = tb.d.U;
    int rb = 256 / U;
    if (rb > R) rb = R;
    if (rb < 1) return hipErrorInvalidValue;
    auto lds = [&](int r) { return folded_lds(tb.d, r, 4, 2); };
    while (rb > 1 && lds(rb) > (size_t)tb.d.lds_max) --rb;
    if (lds(rb) > (size_t)tb.d.lds_max) return hipErrorInvalidValue;
    const int threads = (rb * U + 63) / 64 * 64;
    const int64_t blocks = B * ((R + rb - 1) / rb);
    hipLaunchKernelGGL((k_onsite_split<LM>), dim3((unsigned)blocks), dim3(threads), lds(rb), s,
                       tb, R, rb, fold_rows(tb.d), fold_whole(tb.d), tb.qf, tb.qdf, HA, HB, HAc,
                       HBc, Ta, Tb);
    return hipGetLastError();
}

// nu-body product in the folded form (fp32, lmax <= kNbodyFoldedMaxL, NU operands): one
// thread per (rank, Gauss-Legendre node u) keeps the Legendre coefficients F_t[m] of every
// operand in registers (Eq. struct-F), sweeps the azimuth four points at a time as the on-site kernel,
// multiplies the NU values at each point and accumulates the Fourier analysis (Eq. struct-Tmu) of
// the product in registers. The Gauss-Legendre analysis across u (Eq. struct-Tlm)
// goes through LDS. The grid (U, V) is the plan's, exact for the (NU + 1) lmax integrand.
template <int LM, int NU>
__global__ __launch_bounds__(256) void k_nbody_folded(Tabs<float> tb, int R, int rb, int steps,
                                                      bool whole,
                                                      const float *__restrict__ qg,
                                                      NbodyOperands<float> H,
                                                      float *__restrict__ Tout)
{
    constexpr int M = 2 * LM + 1, L = LM + 1, K = L * L, P = L * (L + 1) / 2;
    constexpr int PS = table_stride(P);
    extern __shared__ __attribute__((aligned(16))) float smem[];
    const int U = tb.d.U, ts = tm_stride((U + 3) / 4 * 4);
    float *Tm = smem;  // [rb][M][ts]: the Fourier rows, in the space of
    float *Hs = smem;  // [NU][rb][K]: the coefficient rows
    const int shared = NU * rb * K > rb * M * ts ? NU * rb * K : rb * M * ts;
    float *ps = smem + (shared + 3) / 4 * 4;  // [U][PS]

    const int nrb = (R + rb - 1) / rb;
    const int64_t b = blockIdx.x / nrb;
    const int r0 = (int)(blockIdx.x - b * nrb) * rb;
    const int nr = (R - r0 < rb) ? (R - r0) : rb;
    for (int k = threadIdx.x; k < U * P; k += blockDim.x) {
        const int uu = k / P;
        ps[uu * PS + k - uu * P] = tb.p[k];
    }
    const int64_t row0 = (b * R + r0) * (int64_t)K;
    if (LM == 0 && U == 1 && steps == 1) {
        if ((int)threadIdx.x < nr) {
            float v = 1.f;
#pragma unroll
            for (int t = 0; t < NU; ++t) v *= tb.p[0] * H.h[t][row0 + threadIdx.x];
            Tout[row0 + threadIdx.x] = analyse_constant(tb, v);
        }
        return;
    }
#pragma unroll
    for (int t = 0; t < NU; ++t) {
        const float *h = H.h[t] + row0;
        for (int k = threadIdx.x; k < nr * K; k += blockDim.x) Hs[t * rb * K + k] = h[k];
    }
    __syncthreads();

    const int q = threadIdx.x / U, u = threadIdx.x - q * U;
    const bool active = q < nr;
    float F[NU][M], T[M];
#pragma unroll
    for (int mi = 0; mi < M; ++mi) T[mi] = 0.f;
    if (active) {
        const float *pu = ps + u * PS;
#pragma unroll
        for (int t = 0; t < NU; ++t) {
            const float *h = Hs + (t * rb + q) * K;
#pragma unroll
            for (int mi = 0; mi < M; ++mi) {
                const int m = mi - LM, am = m < 0 ? -m : m;
                float f = 0.f;
#pragma unroll
                for (int l = am; l <= LM; ++l) f += pu[l * (l + 1) / 2 + am] * h[l * l + l + m];
                F[t][mi] = f;
            }
        }
    }
    __syncthreads();  // every thread has its coefficients: Hs is free for Tm
    if (active) {
        for (int v = 0; v < steps; ++v) {
            const float *qr = qg + v * M;
            float s[4];
#pragma unroll
            for (int t = 0; t < NU; ++t) {
                Quad a{F[t][LM], 0.f, 0.f, 0.f};
#pragma unroll
                for (int k = 1; k <= LM; ++k)
                    quad_add(a, k, qr[LM + k], F[t][LM + k], qr[LM - k], F[t][LM - k]);
                if (t == 0) halve_ends<LM>(a, v, steps, whole);
                float x[4];
                quad_values(a, x);
#pragma unroll
                for (int p = 0; p < 4; ++p) s[p] = t ? s[p] * x[p] : x[p];
            }
            quad_analyse<LM>(s, qr, T);
        }
        store_fourier<LM>(Tm, ts, q, u, U, T);
    }
    __syncthreads();
    gl_analyse<LM, default_ut(LM, NU)>(tb, Tm, nr, Tout + row0);
}

template <int LM, int NU>
hipError_t launch_nbody_folded_lm(const Tabs<float> &tb, int64_t B, int R,
                                  const NbodyOperands<float> &H, float *Tout, hipStream_t s)
{
    const int U = tb.d.U;
    int rb = 256 / U;
    if (rb > R) rb = R;
    if (rb < 1) return hipErrorNotSupported;
    while (rb > 1 && folded_lds(tb.d, rb, NU, 1) > (size_t)tb.d.lds_max) --rb;
    const size_t lds = folded_lds(tb.d, rb, NU, 1);
    if (lds > (size_t)tb.d.lds_max) return hipErrorNotSupported;
    const int threads = (rb * U + 63) / 64 * 64;
    const int64_t blocks = B * ((R + rb - 1) / rb);
    if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    hipLaunchKernelGGL((k_nbody_folded<LM, NU>), dim3((unsigned)blocks), dim3(threads), lds, s, tb,
                       R, rb, fold_rows(tb.d), fold_whole(tb.d), tb.qf, H, Tout);
    return hipGetLastError();
}

template <int LM>
hipError_t launch_nbody_folded_nu(const Tabs<float> &tb, int64_t B, int R, int nu,
                                  const NbodyOperands<float> &H, float *Tout, hipStream_t s)
{
    switch (nu) {
    case 2: return launch_nbody_folded_lm<LM, 2>(tb, B, R, H, Tout, s);
    case 3: return launch_nbody_folded_lm<LM, 3>(tb, B, R, H, Tout, s);
    case 4: return launch_nbody_folded_lm<LM, 4>(tb, B, R, H, Tout, s);
    default: return hipErrorNotSupported;
    }
}

}  // namespace

bool onsite_split_supported(const Dims &d)
{
    return d.lmax <= kOnsiteSplitMaxL && d.U <= 256 && folded_lds(d, 1, 4, 2) <= (size_t)d.lds_max;
}

hipError_t launch_onsite_folded(const Tabs<float> &tb, int64_t B, int R, const float *HA,
                                const float *HB, float *Ta, float *Tb, hipStream_t s,
                                const float *HAc, const float *HBc)
{
    if (B == 0) return hipSuccess;
    if ((HAc == nullptr) != (HBc == nullptr)) return hipErrorInvalidValue;
    if (HAc) {
        switch (tb.d.lmax) {
#define CGTP_CASE(LMV) \
    case LMV: return launch_split<LMV>(tb, B, R, HA, HB, HAc, HBc, Ta, Tb, s);
            CGTP_CASE(0) CGTP_CASE(1) CGTP_CASE(2) CGTP_CASE(3) CGTP_CASE(4) CGTP_CASE(5)
            CGTP_CASE(6) CGTP_CASE(7) CGTP_CASE(8) CGTP_CASE(9) CGTP_CASE(10) CGTP_CASE(11)
            CGTP_CASE(12) CGTP_CASE(13) CGTP_CASE(14)
#undef CGTP_CASE
        default: return hipErrorNotSupported;
        }
    }
    switch (tb.d.lmax) {
#define CGTP_CASE(LMV) \
    case LMV: return launch_folded<LMV>(tb, B, R, HA, HB, Ta, Tb, s);
        CGTP_CASE(0) CGTP_CASE(1) CGTP_CASE(2) CGTP_CASE(3) CGTP_CASE(4) CGTP_CASE(5)
        CGTP_CASE(6) CGTP_CASE(7) CGTP_CASE(8) CGTP_CASE(9) CGTP_CASE(10) CGTP_CASE(11)
        CGTP_CASE(12) CGTP_CASE(13) CGTP_CASE(14) CGTP_CASE(15) CGTP_CASE(16) CGTP_CASE(17)
        CGTP_CASE(18) CGTP_CASE(19) CGTP_CASE(20)
#undef CGTP_CASE
    default: return hipErrorNotSupported;
    }
}

hipError_t launch_nbody_folded(const Tabs<float> &tb, int64_t B, int R, int nu,
                               const NbodyOperands<float> &H, float *Tout, hipStream_t s)
{
    if (B == 0) return hipSuccess;
    switch (tb.d.lmax) {
#define CGTP_CASE(LMV) \
    case LMV: return launch_nbody_folded_nu<LMV>(tb, B, R, nu, H, Tout, s);
        CGTP_CASE(0) CGTP_CASE(1) CGTP_CASE(2) CGTP_CASE(3) CGTP_CASE(4) CGTP_CASE(5)
        CGTP_CASE(6) CGTP_CASE(7) CGTP_CASE(8) CGTP_CASE(9) CGTP_CASE(10)
#undef CGTP_CASE
    default: return hipErrorNotSupported;
    }
}

}  // namespace cgtp
