// Message-passing receiver pass reading sender values only (fp32, default grid, rank padded to
// a multiple of 16), the edge-field synthesis on MFMA.
//
// For an edge e the zonal edge field and its t-derivative at grid point p are
//   a[r][p] = sum_l Rt[e][l][r] P_l(t_p),   g[r][p] = sum_l Rt[e][l][r] P_l'(t_p),
// t_p = rhat_e . Omega_p (addition theorem; the (2l+1)/(4 pi) weights are folded into Rt): two
// [16 ranks x L] x [L x 16 points] products per tile. The surface curl takes the
// moved-derivative form (integration by parts on the sphere): its coefficient is the analysis
// of S1 = sum_j B_j dA_j/dx against dY/dphi minus that of S2 = sum_j B_j dA_j/dphi against
// dY/dx, with dA/dx = g dt/dx and dA/dphi = g dt/dphi of the edge field. So a receiver reads the
// value plane B_j of its senders alone and sums the Gaunt product a B and the pair (S1, S2);
// S [N][R][3][UVs] (six planes with two node slots) goes to the MFMA analysis in its moved modes.
//
// Products on bf16 triples. The fp32 matrix instructions run on the vector ALU's data path:
// on this chip they do not overlap vector instructions of other waves (16x16x4 fp32 products
// and FMAs that take 229 and 296 us apart take 510 us together), so a receiver on them paid the
// sum of its matrix and vector time. The 16x16x32 bf16 instruction is 16 times faster and does
// overlap (128 and 144 us apart, 192 together). Both operands are therefore held as sums of three
// bf16 parts, x = h + m + l (24 bits of significand, round to nearest each time; exact from 2^-109
// on, within 2^-134 below: a coefficient down there keeps fewer bits than fp32 held, and an
// infinite one becomes NaN), and a
// product is formed from the parts' products hh, hm, mh, mm, hl, lh (up to lmax 7, where there is
// room, also ml and lm), accumulated in fp32: what is left out is below 2^-24 of the term.
//
// Operand layout (lane = 16 g + n, 8 consecutive reduction slots per lane): a slot vector is 8
// degrees of one part. With one degree group (lmax <= 7) the four lane groups take four part
// pairs of it, two instructions; with two groups (lmax <= 15) two part pairs of both, three
// instructions; above, one part pair of up to four groups, six instructions.
//
// fp32 form (F32). The split costs vector instructions per degree and point, paid once per wave,
// and a slot vector costs 48 bytes per rank however few of its degrees exist. Where a wave has one
// rank tile to share the split, or the degrees fill the slots badly, the products run on the fp32
// instructions (16x16x4, four degrees a step) from P rows and coefficients held as floats; the
// tiles, waves and sums are the same. receiver_values_f32 (internal.h) has the rule and both sides.
//
// Sender values come in tiles of 16 ranks x 16 points, 1 KB each in the order a wave reads
// them: SF [N][R/16][UVs/16][64 lanes][4], lane 16 g + n holding ranks 4 g .. 4 g + 3 of point
// n (with per-block factors a second such plane follows). One 16-byte load per lane then
// fetches whole lines; the same bytes as rows [R][UVs], 16 segments of 64 bytes per load, ran
// at two thirds of the rate (the loads alone, 10^4 nodes, lmax 6, R = 128, 525,308 edges, Hilbert
// order: 5.4 to 5.6 ms in rows, 3.5 to 3.7 ms in tiles).
//
// A wave owns RT rank tiles x PT point tiles of one receiver and works alone. P_l and P_l' of an
// edge do not depend on the rank: a lane runs the recurrence at one point for one of 4 / PT
// edges, splits the values into parts once for all ranks and leaves them in wave-private LDS
// (no barrier). Sharing them between the waves of a workgroup instead halves that work but left
// the waves waiting for each other (6.5 ms at 10^4 nodes, lmax 6, R = 128, 525,308 edges).
// The waves of a workgroup take neighbouring points, so that the edge coefficients they all
// read meet in L1.
//
// Measured (receiver alone, before: fp32 products, values in rows, one wave per 16 ranks and 64
// points): 10^4 nodes, lmax 6, R = 128, 525,308 edges 6.98 -> 5.58 ms; 5,000 nodes, lmax 20,
// R = 64, 35.0 -> 27.9 ms; two slots, 5,000 nodes, lmax 6, R = 128, 6.81 -> 4.56 ms; per-block
// factors, 3,000 nodes, lmax 6, 128 stacked ranks, 3.78 -> 3.06 ms. What bounds it now is the
// power limit: it needs a third fewer cycles than the fp32 form, but with matrix cores (32% busy),
// vector ALU (50%) and gather all running the clock falls to 1.76 to 1.87 GHz (2.2 in the
// contractions, 2.4 in the gather alone). The per-block factors are on the fp32 form by now.
#include <type_traits>

#include "internal.h"
#include "receiver_tiles.h"

namespace cgtp {

namespace {

typedef float float4_t __attribute__((ext_vector_type(4)));
typedef float float2_t __attribute__((ext_vector_type(2)));
typedef unsigned uint2_t __attribute__((ext_vector_type(2)));
typedef unsigned uint4_t __attribute__((ext_vector_type(4)));
typedef __bf16 bf2_t __attribute__((ext_vector_type(2)));
typedef __bf16 bf8_t __attribute__((ext_vector_type(8)));

__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(const void *base, unsigned bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), (short)0, (int)bytes,
                                             0x00020000);
}

template <typename V>
__device__ __forceinline__ V bload16(__amdgpu_buffer_rsrc_t rs, unsigned voff, unsigned soff)
{
    return __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b128(rs, voff, soff, 0));
}

// A byte offset past every resource here: loads return 0.
constexpr unsigned kOut = 0x80000000u;
// Waves per workgroup (neighbouring points): two, so that few of them lie past the grid; four
// with two coefficient sets, which share twice the coefficients through L1 (3.05 against 3.14 ms,
// 3,000 nodes, lmax 6, 128 stacked ranks; at lmax 24 four would take 100 KB of LDS, one workgroup
// per compute unit), one with a single rank tile, whose 64 points are a larger share of the grid.
constexpr int waves_for(bool split, int rt, int ndg)
{
    return split && ndg < 4 ? 4 : rt == 1 && !split ? 1 : 2;
}
// Waves per SIMD that the registers are to leave room for: two; with a single rank tile, whose
// waves have the least to hide their latency behind, as many as its sums allow.
constexpr int simd_waves(int lm, int rt, bool half)
{
    return rt > 1 || half || lm >= 24 ? 2 : lm <= 11 ? 4 : 3;
}
constexpr int kSplitWaves = 4;  // waves per workgroup that share one wave's edges (ES)

// Wave-private LDS in bytes: 64 (edge, point) pairs, each with the slot vectors of P_l, then of
// P_l' (8 bf16 each; with one degree group a zero vector after each), and dt/dx and dt/dphi.
// Layout [edge][P, P'][part][degree group][points][8 bf16], then [edge][2][points].
constexpr int plane_vecs(int ndg) { return 3 * ndg + (ndg == 1 ? 1 : 0); }
constexpr int wave_bytes(int ndg) { return 64 * (2 * plane_vecs(ndg) * 16 + 2 * 4); }

// fp32 form: reduction steps of 4 degrees of the value sum and of the derivative sum. P_0' = 0:
// where lmax is a multiple of 4 the derivative sum starts at degree f32_first = 1 and takes a
// step fewer. Wave-private LDS: rows of P_l, then of P_l', of the 64 (edge, point) pairs, and
// dt/dx and dt/dphi: [edge][row][points], then [edge][2][points].
constexpr int f32_first(int lm) { return lm > 0 && lm % 4 == 0 ? 1 : 0; }
constexpr int f32_steps(int lm) { return lm / 4 + 1; }
constexpr int f32_dsteps(int lm) { return (lm - f32_first(lm)) / 4 + 1; }
constexpr int f32_wave_bytes(int lm) { return 64 * 4 * (4 * (f32_steps(lm) + f32_dsteps(lm)) + 2); }

// Operand vectors by degree groups. Lane group g of instruction i multiplies a part (0 h, 1 m,
// 2 l, 3 zero) of A vector av(i) with one of B vector bv(i), of the degree group group(g):
//   NDG 1: A h m l h with B h h h m, then B l m m 0: hh mh lh hm, hl mm lm
//   NDG 2: A h h m m with B h h h h, then B m m m m; A h h l l with B l l h h: hh mh, hm mm, hl lh
//   above: one part pair per instruction: hh hm mh mm hl lh
template <int NDG>
struct Slots {
    static constexpr int NI = NDG == 1 ? 2 : NDG == 2 ? 3 : 6;
    static constexpr int NA = NDG <= 2 ? NDG : 3, NB = NDG == 1 ? 2 : 3;
    static constexpr int av(int i) { return NDG == 1 ? 0 : NDG == 2 ? i / 2 : (const int[6]){0, 0, 1, 1, 0, 2}[i]; }
    static constexpr int bv(int i) { return NDG <= 2 ? i : (const int[6]){0, 1, 0, 1, 2, 0}[i]; }
    static __device__ int apart(int k, int g)
    {
        if (NDG == 1) return g == 3 ? 0 : g;
        if (NDG == 2) return k == 0 ? g >> 1 : (g >> 1) * 2;
        return k;
    }
    static __device__ int bpart(int k, int g)
    {
        if (NDG == 1) return k == 0 ? (g == 3 ? 1 : 0) : (g == 0 ? 2 : g == 3 ? 3 : 1);
        if (NDG == 2) return k < 2 ? k : 2 - (g >> 1) * 2;
        return k;
    }
    // degree group of lane group g (>= NDG: none)
    static __device__ int group(int g) { return NDG == 1 ? 0 : NDG == 2 ? g & 1 : g; }
};

// The three bf16 parts of 8 values (degrees past the last are zero), as slot vectors. The
// residual x - part is one dot product instruction (exact: the parts cancel leading bits).
__device__ __forceinline__ void split8(const float (&x)[8], uint4_t (&part)[3])
{
    // (-1, 0) and (0, -1), kept from the compiler: as an inline constant the first would be read
    // as the second. So would a part known at compile time (P_0 = 1).
    unsigned lob = 0x0000bf80u, hib = 0xbf800000u;
    asm("" : "+s"(lob), "+s"(hib));
    const bf2_t lo = __builtin_bit_cast(bf2_t, lob), hi = __builtin_bit_cast(bf2_t, hib);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        float2_t r = {x[2 * k], x[2 * k + 1]};
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            unsigned bits = __builtin_bit_cast(unsigned, __builtin_convertvector(r, bf2_t));
            asm("" : "+v"(bits));
            const bf2_t w = __builtin_bit_cast(bf2_t, bits);
            part[c][k] = bits;
            if (c < 2) {
                r[0] = __builtin_amdgcn_fdot2_f32_bf16(w, lo, r[0], false);
                r[1] = __builtin_amdgcn_fdot2_f32_bf16(w, hi, r[1], false);
            }
        }
    }
}

// Block order of the receiver: rank group by rank group; inside, each XCD takes a contiguous
// span of the receiver sequence (as recv_block) and the point chunks of one receiver run back to
// back, so that the edge coefficients they share stay in its L2.
__device__ __forceinline__ bool recv_chunk_block(int64_t N, const int32_t *order, int nchunks,
                                                 int &rg, int64_t &i, int &chunk)
{
    const int64_t m = recv_span(N), k = blockIdx.x / kXcds, per = m * nchunks;
    rg = (int)(k / per);
    const int64_t rem = k - rg * per, q = rem / nchunks;
    chunk = (int)(rem - q * nchunks);
    const int64_t pos = (blockIdx.x % kXcds) * m + q;
    if (pos >= N) return false;
    i = order ? (int64_t)order[pos] : pos;
    return true;
}

// Wave-scope ordering of LDS accesses (LDS operations of a wave complete in order; the fences
// keep the compiler from moving accesses across).
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// TWO: the senders carry a second, parity-flipped node slot SFf (same layout as SF); by
// Table 1 its curl then feeds S_alpha's slot (natural parity) and its Gaunt product S_beta's.
// SPLIT: per-block factors. The derivative sum g multiplies P' with the curl factors' edge
// coefficients Rtg and its products take the curl factors' values, plane 1 of SF.
// Rt, Rtg: edge coefficients in parts, [E][R/16][3 parts][NDG][16 ranks][8 degrees] bf16.
// ES: the workgroup's waves (kSplitWaves) take one wave's tiles together, a share of the edges
// each, and add up their sums in wave order.
// rt_first: the first rank tile of the launch. PART: the last wave may have fewer than RT rank
// tiles and skips the others; without it every wave has RT.
// F32: products on the fp32 matrix instructions; Rt, Rtg are [E][LM + 1][R] floats.
template <int LM, int RT, int PT, bool TWO, bool SPLIT, bool ES, bool PART, bool F32>
__global__ __launch_bounds__(64 * (ES ? kSplitWaves : waves_for(SPLIT, RT, rt_groups(LM))))
__attribute__((amdgpu_waves_per_eu(simd_waves(LM, RT, TWO || SPLIT)))) void k_receiver_values(Tabs<float> tb, int R, int rt_first, int nchunks, int64_t N,
                       const int32_t *__restrict__ row_ptr, const int32_t *__restrict__ col,
                       const int32_t *__restrict__ order, const float *__restrict__ unit,
                       const void *__restrict__ Rt, const void *__restrict__ Rtg,
                       const float *__restrict__ SF, const float *__restrict__ SFf,
                       float *__restrict__ S)
{
    constexpr int NDG = rt_groups(LM);
    constexpr int TB = 3 * NDG * 16 * 16;  // bytes of a rank tile's slot vectors
    using SL = Slots<NDG>;
    constexpr int KS = f32_steps(LM), KSG = f32_dsteps(LM), DO = f32_first(LM);
    constexpr bool AG = SPLIT || (F32 && DO);  // the derivative sum has operands of its own
    constexpr int NA = F32 ? KS : SL::NA, NB = F32 ? KS : SL::NB;
    using vec_t = typename std::conditional<F32, float, bf8_t>::type;  // one lane's operand
    constexpr int PW = 16 * PT, EG = 64 / PW;  // points of a wave, edges per recurrence pass
    // bytes of one edge's P vectors (rows) and of both, and where dt/dx and dt/dphi start
    constexpr int PLANE = F32 ? 4 * KS * PW * 4 : plane_vecs(NDG) * PW * 16;
    constexpr int PLANES = F32 ? PLANE + 4 * KSG * PW * 4 : 2 * PLANE, DXS = EG * PLANES;
    const Dims &d = tb.d;
    const int UV = d.UV, UVs = d.UVs, NT = UVs / 16, RTL = R / 16;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int g = lane >> 4, n = lane & 15;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    char *lds = smem + wave * (F32 ? f32_wave_bytes(LM) : wave_bytes(NDG));
    // fp32 rows: column of point p in row j. The two rows that half a wave reads at once lie on
    // different halves of the banks, and a row's writes stay a permutation of them.
    auto fslot = [](int j, int p) { return j * PW + (p ^ ((j & (PT - 1)) << 4)); };

    int64_t i;
    int rg, ch;
    if (!recv_chunk_block(N, order, nchunks, rg, i, ch)) return;  // the whole workgroup
    const int p0 = (ES ? ch : ch * waves_for(SPLIT, RT, NDG) + wave) * PW;  // first point of the wave
    const int rt0 = rt_first + rg * RT;                                 // its first rank tile
    if (p0 >= UV) return;  // waves never wait for each other (ES: the whole workgroup)
    // its rank tiles: wave-uniform, so a tile it does not have costs a scalar branch
    const int na = wave_rank_tiles(RT, PART, RTL, rt0);

    // This lane's recurrence point (points past the grid compute on point 0, never stored).
    const int hl = lane & (PW - 1), he = lane / PW;
    const int prc = p0 + hl < UV ? p0 + hl : 0;
    const int ur = prc / d.V, vr = prc - ur * d.V;
    const float rx = tb.x[ur], rsx = tb.sx[ur], rxsx = tb.xsx[ur], rcp = tb.cphi[vr],
                rsp = tb.sphi[vr];
    // the wave's edges: the receiver's, or (ES) a quarter of them
    int e0 = row_ptr[i], e1 = row_ptr[i + 1];
    if (ES) {
        const int len = e1 - e0, first = e0;
        e0 = first + (int)((int64_t)len * wave / kSplitWaves);
        e1 = first + (int)((int64_t)len * (wave + 1) / kSplitWaves);
    }
    // the direction of this lane's edge of a pass, loaded a pass ahead
    float nux = 0.f, nuy = 0.f, nuz = 1.f;
    auto load_unit = [&](int b) {
        const float *v = unit + 3 * (int64_t)(b + he < e1 ? b + he : e0);
        nux = v[0];
        nuy = v[1];
        nuz = v[2];
    };
    // P_l, P_l' of edges b .. b + EG - 1 at the wave's points, in parts, into LDS
    auto legendre = [&]() {
        // renormalised by the hardware reciprocal square root (within 1 ulp)
        const float inv = __builtin_amdgcn_rsqf(nux * nux + nuy * nuy + nuz * nuz);
        const float ux = nux * inv, uy = nuy * inv, uz = nuz * inv;
        // t = rhat . Omega at this lane's point; P_l(t) and P_l'(t) by the Legendre and
        // derivative recurrences
        const float h = ux * rcp + uy * rsp;
        const float t = uz * rx + rsx * h;
        float *dxs = reinterpret_cast<float *>(lds + DXS) + he * 2 * PW + hl;
        dxs[0] = uz - rxsx * h;
        dxs[PW] = rsx * (uy * rcp - ux * rsp);
        uint4_t *o = reinterpret_cast<uint4_t *>(lds + he * PLANES) + hl;
        float *of = reinterpret_cast<float *>(lds + he * PLANES);
        // P_l = ((2l-1) t P_{l-1} - (l-1) P_{l-2}) / l,  P_l' = l P_{l-1} + t P_{l-1}' (the form
        // P_{l-2}' + (2l-1) P_{l-1} is one operation shorter and measured less accurate)
        float p0v = 0.f, p1v = 0.f, d1 = 0.f;  // P_{l-2}, P_{l-1}, P_{l-1}'
#pragma unroll
        for (int dg = 0; dg < NDG; ++dg) {
            float v[8], w[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const int l = 8 * dg + k;
                v[k] = w[k] = 0.f;
                if (l > LM) continue;
                float p2 = l == 0 ? 1.f : t;
                float d2 = l == 0 ? 0.f : 1.f;
                if (l >= 2) {
                    const float c1 = (float)(2 * l - 1) / (float)l, c2 = (float)(l - 1) / (float)l;
                    p2 = c1 * t * p1v - c2 * p0v;
                    d2 = (float)l * p1v + t * d1;
                }
                v[k] = p2;
                w[k] = d2;
                if (F32) {
                    of[fslot(l, hl)] = p2;
                    if (l >= DO) of[4 * KS * PW + fslot(l - DO, hl)] = d2;
                }
                p0v = p1v;
                p1v = p2;
                d1 = d2;
            }
            if (F32) continue;
            uint4_t part[3];
            split8(v, part);
#pragma unroll
            for (int c = 0; c < 3; ++c) o[(c * NDG + dg) * PW] = part[c];
            split8(w, part);
#pragma unroll
            for (int c = 0; c < 3; ++c) o[(plane_vecs(NDG) + c * NDG + dg) * PW] = part[c];
        }
    };

    // D[row = rank 4 g + j][col = point n]: a lane holds four ranks of one point. sa, sb: the
    // Gaunt sums into S_alpha, S_beta; (ca1, ca2) the moved curl pair into S_alpha (the flipped
    // slot's, TWO), (cb1, cb2) into S_beta (the natural slot's).
    float4_t sa[RT][PT], sb[RT][PT], ca1[RT][PT], ca2[RT][PT], cb1[RT][PT], cb2[RT][PT];
#pragma unroll
    for (int a = 0; a < RT; ++a)
#pragma unroll
        for (int t = 0; t < PT; ++t)
            sa[a][t] = sb[a][t] = ca1[a][t] = ca2[a][t] = cb1[a][t] = cb2[a][t] =
                float4_t{0.f, 0.f, 0.f, 0.f};

    const int64_t jstride = (int64_t)R * UVs;  // sender stride of a value plane
    const int64_t sfo = ((int64_t)rt0 * NT + p0 / 16) * 256;
    const float *sfb = SF + sfo;
    const float *sfx = (TWO ? SFf : SF + N * jstride) + sfo;  // flipped slot, or plane 1
    const unsigned sfbytes = value_bytes(na, NT, p0 / 16);
    int pt[PT];
#pragma unroll
    for (int t = 0; t < PT; ++t) pt[t] = value_point_tile(PT, t, NT, p0 / 16);
    // A operands: slot vectors of the edge's rank tiles; B operands: slot
    // vectors of P, P' at the wave's points. Lane groups without a degree group take zeros for A
    // and any (finite) vector for B.
    // F32: A degree 4 k + g (zero past lmax) of rank n, B the same row at point n.
    unsigned ao[NA], ago[NA], bo[NB];
    const int dgl = SL::group(g);
#pragma unroll
    for (int k = 0; k < NA; ++k) {
        if constexpr (F32) {
            ao[k] = 4 * k + g <= LM ? (unsigned)((4 * k + g) * R + n) * 4u : kOut;
            ago[k] = 4 * k + g + DO <= LM ? (unsigned)((4 * k + g + DO) * R + n) * 4u : kOut;
        } else {
            ao[k] = ago[k] = dgl < NDG ? (unsigned)((SL::apart(k, g) * NDG + dgl) * 16 + n) * 16u : kOut;
        }
    }
#pragma unroll
    for (int k = 0; k < NB; ++k)
        bo[k] = F32 ? 0u : (unsigned)((SL::bpart(k, g) * NDG + (dgl < NDG ? dgl : 0)) * (PW * 16) + n * 16);
    // an edge's coefficients from the wave's first rank tile on, a rank tile's bytes, an edge's
    // and those up to the wave's last rank tile
    constexpr unsigned TA = F32 ? 16 * 4 : TB;
    const char *rtb = static_cast<const char *>(Rt) + rt0 * TA;
    const char *rtgb = static_cast<const char *>(Rtg) + (SPLIT ? rt0 * TA : 0);
    const int64_t estride = F32 ? (int64_t)(LM + 1) * R * 4 : (int64_t)RTL * TB;
    const unsigned abytes = F32 ? (unsigned)(LM * R) * 4u + na * TA : na * TA;

    // sender indices in batches of 64 edges: lane k holds that of edge k of the batch, read out
    // with readlane, so no load of an index sits on an edge's critical path (coln: the next 64)
    int colv = 0, coln = 0;
    auto load_col = [&](int e) { return e + lane < e1 ? col[e + lane] : 0; };
    // An edge's values and coefficients are requested one edge ahead, tile by tile, each right
    // after its registers' last use (past the last edge the last is requested again).
    float4_t f[RT][PT], x[RT][PT];
    vec_t A[RT][NA], Ag[AG ? RT : 1][NA];
    auto load_a = [&](__amdgpu_buffer_rsrc_t rs, int a, const unsigned (&off)[NA], int steps,
                      vec_t (&v)[NA]) {
#pragma unroll
        for (int k = 0; k < NA; ++k) {
            if (k >= steps) continue;
            if constexpr (F32)
                v[k] = __builtin_bit_cast(
                    float, __builtin_amdgcn_raw_buffer_load_b32(rs, off[k], (unsigned)a * TA, 0));
            else
                v[k] = bload16<bf8_t>(rs, off[k], (unsigned)a * TA);
        }
    };
    auto load_f = [&](__amdgpu_buffer_rsrc_t rs, int a, int t) {
        return bload16<float4_t>(rs, lane * 16u, value_offset(a, pt[t], NT));
    };
    struct Next {
        __amdgpu_buffer_rsrc_t f, x, a, ag;
    };
    auto next_edge = [&](int e) {
        const int ec = e < e1 ? e : e1 - 1;
        const int k = (ec - e0) & 63;
        if (k == 0 && e > e0 && e < e1) {
            colv = coln;
            coln = load_col(e + 64);
        }
        const int64_t j = __builtin_amdgcn_readlane(colv, k);
        Next r;
        r.f = rsrc(sfb + j * jstride, sfbytes);
        r.x = rsrc(sfx + j * jstride, sfbytes);
        r.a = rsrc(rtb + ec * estride, abytes);
        r.ag = SPLIT ? rsrc(rtgb + ec * estride, abytes) : r.a;
        return r;
    };
    auto edge = [&](int e, int q) {
        const Next nx = next_edge(e + 1);
        const char *u = lds + q * PLANES;
        const float *dxs = reinterpret_cast<const float *>(lds + DXS) + q * 2 * PW + n;
#pragma unroll
        for (int t = 0; t < PT; ++t) {
            vec_t pv[NB], dv[NB];
#pragma unroll
            for (int k = 0; k < NB; ++k) {
                if constexpr (F32) {
                    const int at = fslot(4 * k + g, 16 * t + n);
                    pv[k] = reinterpret_cast<const float *>(u)[at];
                    if (k < KSG) dv[k] = reinterpret_cast<const float *>(u + PLANE)[at];
                } else {
                    pv[k] = *reinterpret_cast<const bf8_t *>(u + bo[k] + t * 256);
                    dv[k] = *reinterpret_cast<const bf8_t *>(u + PLANE + bo[k] + t * 256);
                }
            }
            const float dxt = dxs[16 * t], dpt = dxs[PW + 16 * t];
#pragma unroll
            for (int a = 0; a < RT; ++a) {
                if (PART && a >= na) continue;
                float4_t va = float4_t{0.f, 0.f, 0.f, 0.f}, gg = va;
                if constexpr (F32) {
#pragma unroll
                    for (int k = 0; k < KS; ++k) {
                        va = __builtin_amdgcn_mfma_f32_16x16x4f32(A[a][k], pv[k], va, 0, 0, 0);
                        if (k < KSG)
                            gg = __builtin_amdgcn_mfma_f32_16x16x4f32(AG ? Ag[AG ? a : 0][k] : A[a][k],
                                                                      dv[k], gg, 0, 0, 0);
                    }
                } else {
                    // the small part products first
#pragma unroll
                    for (int k = SL::NI - 1; k >= 0; --k) {
                        va = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A[a][SL::av(k)], pv[SL::bv(k)],
                                                                     va, 0, 0, 0);
                        gg = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                            AG ? Ag[AG ? a : 0][SL::av(k)] : A[a][SL::av(k)], dv[SL::bv(k)], gg, 0,
                            0, 0);
                    }
                }
                if (t == PT - 1) {
                    load_a(nx.a, a, ao, NA, A[a]);
                    if (AG) load_a(nx.ag, a, ago, F32 ? KSG : NA, Ag[AG ? a : 0]);
                }
#pragma unroll
                for (int jj = 0; jj < 4; ++jj) {
                    const float fv = f[a][t][jj], xv = (TWO || SPLIT) ? x[a][t][jj] : fv;
                    sa[a][t][jj] += va[jj] * fv;
                    const float gf = gg[jj] * (SPLIT ? xv : fv);
                    cb1[a][t][jj] += dxt * gf;
                    cb2[a][t][jj] += dpt * gf;
                    if (TWO) {
                        sb[a][t][jj] += va[jj] * xv;
                        const float gh = gg[jj] * xv;
                        ca1[a][t][jj] += dxt * gh;
                        ca2[a][t][jj] += dpt * gh;
                    }
                }
                f[a][t] = load_f(nx.f, a, t);
                if (TWO || SPLIT) x[a][t] = load_f(nx.x, a, t);
            }
        }
    };

    if (e0 < e1) {
        load_unit(e0);
        colv = load_col(e0);
        coln = load_col(e0 + 64);
        {
            const Next nx = next_edge(e0);
#pragma unroll
            for (int a = 0; a < RT; ++a) {
                if (PART && a >= na) continue;
                load_a(nx.a, a, ao, NA, A[a]);
                if (AG) load_a(nx.ag, a, ago, F32 ? KSG : NA, Ag[AG ? a : 0]);
#pragma unroll
                for (int t = 0; t < PT; ++t) {
                    f[a][t] = load_f(nx.f, a, t);
                    if (TWO || SPLIT) x[a][t] = load_f(nx.x, a, t);
                }
            }
        }
        if (F32) {  // the rows past lmax, which the A operands take zero times
#pragma unroll
            for (int j = LM + 1; j < 4 * KS; ++j)
                reinterpret_cast<float *>(lds + he * PLANES)[fslot(j, hl)] = 0.f;
#pragma unroll
            for (int j = LM + 1 - DO; j < 4 * KSG; ++j)
                reinterpret_cast<float *>(lds + he * PLANES + PLANE)[fslot(j, hl)] = 0.f;
        } else if (NDG == 1) {  // the zero vectors
#pragma unroll
            for (int k = 0; k < 2; ++k)
                *reinterpret_cast<uint4_t *>(lds + he * PLANES + k * PLANE + (3 * PW + hl) * 16) =
                    uint4_t{0, 0, 0, 0};
        }
        for (int b = e0; b < e1; b += EG) {
            wave_sync();  // the pass before is read
            legendre();
            load_unit(b + EG);
            wave_sync();
            const int be = e1 - b < EG ? e1 - b : EG;
            for (int q = 0; q < be; ++q) edge(b + q, q);
        }
    }
    // S[i][r][plane][p]: planes (sa, cb1, cb2), with two slots (sa, ca1, ca2, sb, cb1, cb2)
    constexpr int NF = TWO ? 6 : 3;
    if constexpr (ES) {
        // every wave's sums of one plane in LDS, [wave][tile][64 lanes][4]; wave 0 adds them up
        float4_t *sum = reinterpret_cast<float4_t *>(smem);
        auto reduce = [&](float4_t (&v)[RT][PT]) {
            __syncthreads();
#pragma unroll
            for (int k = 0; k < RT * PT; ++k)
                sum[(wave * RT * PT + k) * 64 + lane] = v[k / PT][k % PT];
            __syncthreads();
            if (wave == 0) {
#pragma unroll
                for (int k = 0; k < RT * PT; ++k)
#pragma unroll
                    for (int w = 1; w < kSplitWaves; ++w)
                        v[k / PT][k % PT] += sum[(w * RT * PT + k) * 64 + lane];
            }
        };
        reduce(sa);
        reduce(cb1);
        reduce(cb2);
        if (TWO) {
            reduce(sb);
            reduce(ca1);
            reduce(ca2);
        }
        if (wave != 0) return;
    }
#pragma unroll
    for (int t = 0; t < PT; ++t) {
        const int p = p0 + 16 * t + n;
        if (p >= UV) continue;
#pragma unroll
        for (int a = 0; a < RT; ++a) {
            if (PART && a >= na) continue;
#pragma unroll
            for (int jj = 0; jj < 4; ++jj) {
                float *o = S + (i * R + 16 * (rt0 + a) + 4 * g + jj) * NF * (int64_t)UVs + p;
                o[0] = sa[a][t][jj];
                o[UVs] = TWO ? ca1[a][t][jj] : cb1[a][t][jj];
                o[2 * UVs] = TWO ? ca2[a][t][jj] : cb2[a][t][jj];
                if (TWO) {
                    o[3 * UVs] = sb[a][t][jj];
                    o[4 * UVs] = cb1[a][t][jj];
                    o[5 * UVs] = cb2[a][t][jj];
                }
            }
        }
    }
}

// Read-pattern ceiling of k_receiver_values: the same blocks in the same order, the same
// wave-uniform sender index per edge and the same 16-byte loads of the value tiles, with
// nothing computed from them but a running sum; sink receives a value only if that sum equals
// a constant no finite input sums to by chance, which keeps every load live.
template <int RT, int PT>
__global__ __launch_bounds__(64 * waves_for(false, RT, 1)) void k_gather_probe_values(
    int UV, int UVs, int R, int rt_first, int nchunks, int64_t N, const int32_t *__restrict__ row_ptr,
    const int32_t *__restrict__ col, const int32_t *__restrict__ order,
    const float *__restrict__ SF, float *__restrict__ sink)
{
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int NT = UVs / 16;
    int64_t i;
    int rg, ch;
    if (!recv_chunk_block(N, order, nchunks, rg, i, ch)) return;
    const int p0 = (ch * waves_for(false, RT, 1) + wave) * 16 * PT;
    if (p0 >= UV) return;
    const int rt0 = rt_first + rg * RT;
    const float *sfb = SF + ((int64_t)rt0 * NT + p0 / 16) * 256;
    const unsigned bytes = value_bytes(RT, NT, p0 / 16);
    const int64_t jstride = (int64_t)R * UVs;
    float4_t acc = float4_t{0.f, 0.f, 0.f, 0.f};
    const int e0 = row_ptr[i], e1 = row_ptr[i + 1];
    for (int e = e0; e < e1; ++e) {
        const int64_t j = __builtin_amdgcn_readfirstlane(col[e]);
        const __amdgpu_buffer_rsrc_t rs = rsrc(sfb + j * jstride, bytes);
#pragma unroll
        for (int a = 0; a < RT; ++a)
#pragma unroll
            for (int t = 0; t < PT; ++t)
                acc += bload16<float4_t>(rs, lane * 16u,
                                         value_offset(a, value_point_tile(PT, t, NT, p0 / 16), NT));
    }
    const float sum = acc[0] + acc[1] + acc[2] + acc[3];
    if (sum == -1.2345678e30f) sink[0] = sum;
}

// Tiles (rank x point) of all receivers, over those of a wave (eight, four of a single rank
// tile), below which a receiver's edges are split over the waves of a workgroup: with fewer the
// waves would not fill the 1024 SIMDs twice.
constexpr int64_t kSplitTiles = 2048;

struct Args {
    const Tabs<float> &tb;
    int64_t N;
    int R;
    const int32_t *row_ptr, *col, *order;
    const float *unit;
    const void *Rt, *Rtg;
    const float *SF, *SFf;
    float *S;
    hipStream_t s;
};

template <int LM, int RT, int PT, bool TWO, bool SPLIT, bool F32, bool ES, bool PART = false>
hipError_t receiver_rt(const Args &a, const RecvLaunch &l)
{
    if (l.rt != RT || l.pt != PT || (l.part && !PART)) return hipErrorInvalidValue;
    const Dims &d = a.tb.d;
    constexpr int ndg = rt_groups(LM), waves = ES ? kSplitWaves : waves_for(SPLIT, RT, ndg);
    const int chunk = 16 * PT * (ES ? 1 : waves), nchunks = (d.UV + chunk - 1) / chunk;
    const int64_t blocks = recv_blocks(a.N, (int64_t)l.groups * nchunks);
    if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    size_t lds = (size_t)waves * (F32 ? f32_wave_bytes(LM) : wave_bytes(ndg));
    const size_t sums = (size_t)kSplitWaves * RT * PT * 1024;
    if (ES && lds < sums) lds = sums;
    if (lds > (size_t)d.lds_max) return hipErrorNotSupported;
    hipLaunchKernelGGL((k_receiver_values<LM, RT, PT, TWO, SPLIT, ES, PART, F32>),
                       dim3((unsigned)blocks), dim3(64 * waves), lds, a.s, a.tb, a.R, l.first,
                       nchunks, a.N, a.row_ptr, a.col, a.order, a.unit, a.Rt, a.Rtg, a.SF, a.SFf,
                       a.S);
    return hipGetLastError();
}

template <int LM, bool TWO, bool SPLIT>
hipError_t receiver_lm(const Args &a)
{
    const int tiles = a.R / 16;
    constexpr bool half = TWO || SPLIT, F = receiver_values_f32(LM, 32, SPLIT);
    // Four waves of four degree groups take 100 KB of LDS, one workgroup per compute unit, and are
    // slower than two that do not share the edges (20 nodes, lmax 24, R = 48: 110 against 55 us).
    constexpr bool can_share = F || rt_groups(LM) < 4;
    const bool es = (can_share || tiles == 1) && a.N * tiles * (a.tb.d.UVs / 16) < kSplitTiles * (tiles == 1 ? 4 : 8);
    RecvLaunch l[2];
    const int n = recv_launches(tiles, half, es, l);
    if (tiles == 1)
        return es ? receiver_rt<LM, 1, 4, TWO, SPLIT, true, true>(a, l[0])
                  : receiver_rt<LM, 1, 4, TWO, SPLIT, true, false>(a, l[0]);
    if constexpr (can_share)
        if (es) return receiver_rt<LM, 2, 2, TWO, SPLIT, F, true, true>(a, l[0]);
    for (int k = 0; k < n; ++k) {
        hipError_t e = hipErrorInvalidValue;
        if constexpr (half) {
            if (l[k].rt == 1) e = receiver_rt<LM, 1, 4, TWO, SPLIT, F, false>(a, l[k]);
            if (l[k].rt == 2) e = receiver_rt<LM, 2, 2, TWO, SPLIT, F, false>(a, l[k]);
        } else {
            if (l[k].rt == 2) e = receiver_rt<LM, 2, 4, false, false, F, false>(a, l[k]);
            if (l[k].rt == 3) e = receiver_rt<LM, 3, 2, false, false, F, false>(a, l[k]);
            if (l[k].rt == 4) e = receiver_rt<LM, 4, 2, false, false, F, false>(a, l[k]);
        }
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace

hipError_t launch_receiver_values(const Tabs<float> &tb, int64_t N, int R, const int32_t *row_ptr,
                                  const int32_t *col, const int32_t *order, const float *unit,
                                  const void *Rt, const void *Rtg, const float *SF,
                                  const float *SFf, float *S, hipStream_t s)
{
    if (N == 0) return hipSuccess;
    if (R % 16 != 0 || !sender_mfma_supported(tb.d)) return hipErrorNotSupported;
    if (SFf && Rtg) return hipErrorInvalidValue;
    const Args a{tb, N, R, row_ptr, col, order, unit, Rt, Rtg, SF, SFf, S, s};
    switch (tb.d.lmax) {
#define CGTP_CASE(LMV)                                                                           \
    case LMV:                                                                                    \
        return SFf ? receiver_lm<LMV, true, false>(a)                                            \
                   : Rtg ? receiver_lm<LMV, false, true>(a) : receiver_lm<LMV, false, false>(a);
        CGTP_CASE(0) CGTP_CASE(1) CGTP_CASE(2) CGTP_CASE(3) CGTP_CASE(4) CGTP_CASE(5) CGTP_CASE(6)
        CGTP_CASE(7) CGTP_CASE(8) CGTP_CASE(9) CGTP_CASE(10) CGTP_CASE(11) CGTP_CASE(12)
        CGTP_CASE(13) CGTP_CASE(14) CGTP_CASE(15) CGTP_CASE(16) CGTP_CASE(17) CGTP_CASE(18)
        CGTP_CASE(19) CGTP_CASE(20) CGTP_CASE(21) CGTP_CASE(22) CGTP_CASE(23) CGTP_CASE(24)
#undef CGTP_CASE
    default: return hipErrorNotSupported;
    }
}

hipError_t launch_gather_probe_values(const Dims &d, int64_t N, int R, const int32_t *row_ptr,
                                      const int32_t *col, const int32_t *order, const float *SF,
                                      float *sink, hipStream_t s)
{
    if (R % 16 != 0) return hipErrorNotSupported;
    if (N == 0) return hipSuccess;
    RecvLaunch l[2];
    const int n = recv_launches(R / 16, false, false, l);
#define CGTP_CASE(RTV, PTV)                                                                      \
    case RTV: {                                                                                  \
        constexpr int waves = waves_for(false, RTV, 1), chunk = 16 * PTV * waves;                   \
        const int nchunks = (d.UV + chunk - 1) / chunk;                                          \
        const int64_t blocks = recv_blocks(N, (int64_t)l[k].groups * nchunks);                   \
        if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;                                  \
        hipLaunchKernelGGL((k_gather_probe_values<RTV, PTV>), dim3((unsigned)blocks),            \
                           dim3(64 * waves), 0, s, d.UV, d.UVs, R, l[k].first, nchunks, N,      \
                           row_ptr, col, order, SF, sink);                                       \
        break;                                                                                   \
    }
    for (int k = 0; k < n; ++k)
        switch (l[k].rt) { CGTP_CASE(1, 4) CGTP_CASE(2, 4) CGTP_CASE(3, 2) CGTP_CASE(4, 2) }
#undef CGTP_CASE
    return hipGetLastError();
}

}  // namespace cgtp
