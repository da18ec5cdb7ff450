// Device helpers shared by the libhfk kernels.
#pragma once

#include "hfk_internal.hpp"

namespace hfk {

constexpr double kPi = 3.14159265358979323846264338327950288;

// H(T) = erf(sqrt T) / sqrt T with H(0) = 2/sqrt(pi): the reduced Boys function
// (2/sqrt(pi)) F0(T).  Accurate library erf; used off the hot path (Schwarz bounds).
__device__ inline double erf_over_sqrt(double T)
{
    if (T < 1e-12) return kTwoOverSqrtPi * (1.0 - T / 3.0);
    const double s = sqrt(T);
    return erf(s) / s;
}

// Gaussian product of primitive pair ab = a*g + b of atoms i (at A) and j (at B, coordinates
// already centred): P = (a A + b B)/p, charge S = w_a w_b exp(-mu |A-B|^2) (pi/p)^(3/2), and
// p, mu, fa = a/p, fb = b/p.  With per-atom bases the exponents and weights come from the rows
// of atoms i and j.
struct PrimPair {
    double x, y, z, S, p, mu, fa, fb, ab2;
};
__device__ inline PrimPair prim_pair(const Basis &b, const BasisDev *__restrict__ bd, int64_t i, int64_t j, int ab,
                                     const double *A, const double *B)
{
    PrimPair w;
    const double dx = A[0] - B[0], dy = A[1] - B[1], dz = A[2] - B[2];
    w.ab2 = dx * dx + dy * dy + dz * dz;
    if (b.aexp) {
        const double ea = b.aexp[i * b.g + ab / b.g], eb = b.aexp[j * b.g + ab % b.g];
        w.p = ea + eb;
        w.mu = ea * eb / w.p;
        w.fa = ea / w.p;
        w.fb = eb / w.p;
        w.S = b.aw[i * b.g + ab / b.g] * b.aw[j * b.g + ab % b.g] * exp(-w.mu * w.ab2) * pow(kPi / w.p, 1.5);
    } else {
        w.p = bd->p[ab];
        w.mu = bd->mu[ab];
        w.fa = bd->fa[ab];
        w.fb = bd->fb[ab];
        w.S = b.w[ab / b.g] * b.w[ab % b.g] * exp(-w.mu * w.ab2) * bd->pi32[ab];
    }
    w.x = w.fa * A[0] + w.fb * B[0];
    w.y = w.fa * A[1] + w.fb * B[1];
    w.z = w.fa * A[2] + w.fb * B[2];
    return w;
}

// Schwarz bound of a pair: (ij|ij) = sum over the unordered primitive quartets, from a table of
// S, fb and p per primitive pair (tab[0 .. 3 g2)).  All primitive centres lie on the line A-B,
// P_ab - P_cd = (fb_ab - fb_cd) (B - A).
__device__ inline void pair_q_entry(const Basis &b, int64_t i, int64_t j, int ab, double r2, double *__restrict__ tab,
                                    double *bound = nullptr, double *bound0 = nullptr)
{
    const int x = ab / b.g, y = ab % b.g;
    const double ea = b.aexp ? b.aexp[i * b.g + x] : b.alpha[x], eb = b.aexp ? b.aexp[j * b.g + y] : b.alpha[y];
    const double ww = b.aexp ? b.aw[i * b.g + x] * b.aw[j * b.g + y] : b.w[x] * b.w[y];
    const double p = ea + eb, c = ww * pow(kPi / p, 1.5), s = c * exp(-(ea * eb / p) * r2);
    tab[ab] = s;
    tab[b.g2 + ab] = eb / p;
    tab[2 * b.g2 + ab] = p;
    if (bound) {
        // |S| p^(1/4), here and at distance zero
        const double p4 = sqrt(sqrt(p));
        *bound += fabs(s) * p4;
        *bound0 += fabs(c) * p4;
    }
}
// Lane l of `lanes`: its share of the sum.
__device__ inline double pair_q_sum(int g2, double r2, int l, int lanes, const double *__restrict__ tab)
{
    const double *S = tab, *f = tab + g2, *pp = f + g2;
    double s = 0.0;
    const int nc = g2 * (g2 + 1) / 2;
    for (int c = l; c < nc; c += lanes) {
        int ab = (int)((sqrtf(8.0f * (float)c + 1.0f) - 1.0f) * 0.5f);
        while (ab * (ab + 1) / 2 > c) --ab;
        while ((ab + 1) * (ab + 2) / 2 <= c) ++ab;
        const int cd = c - ab * (ab + 1) / 2;
        const double ss = S[ab] * S[cd];
        if (ss == 0.0) continue;
        const double df = f[ab] - f[cd], rho = pp[ab] * pp[cd] / (pp[ab] + pp[cd]);
        const double v = ss * sqrt(rho) * erf_over_sqrt(rho * (df * df * r2));
        s += ab == cd ? v : 2.0 * v;
    }
    return s;
}

__device__ inline int wave_max(int v)
{
#pragma unroll
    for (int w = 32; w > 0; w >>= 1) {
        const int o = __shfl_xor(v, w, 64);
        v = o > v ? o : v;
    }
    return v;
}

// Binary exponent e with u < 2^e of a primitive pair's bound (see term_limit).
__device__ inline short term_exponent(double u)
{
    if (!(u <= 1e300)) return (short)kTermAlways;
    if (!(u > 0.0)) return (short)kTermNever;
    int e;
    (void)frexp(u, &e);
    return (short)e;
}

// Bound u of a primitive pair with charge S, exponent sum p, mu and atoms r apart (grad: the
// derivative terms too).
__device__ inline double term_bound(double S, double p, double mu, double r, bool grad)
{
    const double sp = sqrt(p), u = fabs(S) * sqrt(sp);
    return grad ? u * fmax(1.0, fmax(sp, 2.0 * r * mu)) : u;
}

// Reciprocal square root in FP64: the hardware estimate (relative error ~5e-8) refined by
// one Newton step, y (1 + e/2) with e = 1 - x y^2, leaving ~1.5 e^2 ~ 4e-15.
__device__ inline double rsqrt_fp64(double x)
{
    const double y = __builtin_amdgcn_rsq(x);
    const double e = fma(-x * y, y, 1.0);
    return fma(y * e, 0.5, y);
}

__device__ inline float rsqrt_fp32(float x) { return __builtin_amdgcn_rsqf(x); }

__device__ inline double rsqrt_r(double x) { return rsqrt_fp64(x); }
__device__ inline float rsqrt_r(float x) { return rsqrt_fp32(x); }

// Far field of the gradient kernels: E(r) = 1/r and W(r) = E'(r)/r = -1/r^3 from x = r^2,
// scaled for the kernels' accumulators.  FP64: the estimate y of x^(-1/2) takes one Newton
// step folded into the product, e = y (x y^2 - 3) = -2 y1 (error ~1.5 (5e-8)^2), so E is carried
// times kE = -2 and W = e^3 = -8 y1^3 times kW = 8; the near-branch tables are scaled to match
// and the sums scaled back once per quartet.  FP32 has no Newton step: E = y, W = -y^3.
template <typename R> struct GradScale;
template <> struct GradScale<double> {
    static constexpr double kE = -2.0, kW = 8.0;
    static __device__ double e_far(double x)
    {
        const double y = __builtin_amdgcn_rsq(x);
        return y * fma(x, y * y, -3.0);
    }
    static __device__ double w_far(double e) { return e * e * e; }
};
template <> struct GradScale<float> {
    static constexpr float kE = 1.0f, kW = 1.0f;
    static __device__ float e_far(float x) { return rsqrt_fp32(x); }
    static __device__ float w_far(float e) { return -(e * e * e); }
};

// Table row of a lane below the switch radius, from r2 = |P-Q|^2 and rsh = rho/h:
// T' = r2 rsh on the grid of this precision.  Adding the rounding constant 1.5 2^52 (FP32:
// 1.5 2^23) in the FMA that forms T' rounds it to the nearest row, whose index is then read
// off the sum's encoding (no separate round and convert).  Returns the row's byte offset (rows
// of kRowLen values) and d = T' - row from one more FMA.
// The row needs no clamp: a caller takes this branch only for r2 < sw, where the switch
// radius^2 sw = kTswitch / rho and rsh come from the same rho (per-atom bases derive rsh
// from sw itself), so T' < kTswitch / h up to a few roundings and the row is at most
// kTswitch / h = 384 (FP32: 512), below the table's rows; r2 is a sum of squares, or in the
// expanded FP64 form below zero by rounding only (~1e-12 bohr^2), so the row is at least 0.
template <typename R, int kRowLen = BoysGrid<R>::stride>
__device__ inline unsigned boys_row(R r2, R rsh, R &d)
{
    using BG = BoysGrid<R>;
    constexpr unsigned kRowBytes = kRowLen * sizeof(R);
    static_assert(BG::rows > kTswitch * BG::inv_h, "rows up to kTswitch / h");
    if constexpr (sizeof(R) == 8) {
        constexpr double kRound = 6755399441055744.0;   // 1.5 * 2^52
        const double sum = fma(r2, rsh, kRound);
        d = fma(r2, rsh, -(sum - kRound));
        // the low 32 bits of the sum's encoding are the row
        return __umul24((unsigned)__double_as_longlong(sum), kRowBytes);
    } else {
        constexpr float kRound = 12582912.0f;           // 1.5 * 2^23
        const float sum = fmaf(r2, rsh, kRound);
        d = fmaf(r2, rsh, -(sum - kRound));
        // the sum is 1.5 2^23 + row, whose encoding is 0x4B400000 + row
        return (__float_as_uint(sum) - 0x4B400000u) * kRowBytes;
    }
}

// The row's polynomial at d (Horner).  FP64 rows are 48 bytes and FP32 rows 16 bytes, on
// 16-byte boundaries: three LDS reads and one.
template <typename R>
__device__ inline R boys_eval(const R *__restrict__ tab, unsigned off, R d)
{
    const R *c = (const R *)((const char *)tab + off);
    if constexpr (sizeof(R) == 8) {
        // degree-5 rows of 48 bytes on 16-byte boundaries: three LDS reads
        static_assert(BoysGrid<double>::order == 6 && BoysGrid<double>::stride == 6, "degree-5 rows");
        const double2 c01 = ((const double2 *)c)[0], c23 = ((const double2 *)c)[1], c45 = ((const double2 *)c)[2];
        R v = c45.y;
        v = v * d + c45.x;
        v = v * d + c23.y;
        v = v * d + c23.x;
        v = v * d + c01.y;
        v = v * d + c01.x;
        return v;
    } else {
        static_assert(BoysGrid<float>::order == 4 && BoysGrid<float>::stride == 4, "degree-3 rows of 16 bytes");
        const float4 r = *(const float4 *)c;
        return fmaf(fmaf(fmaf(r.w, d, r.z), d, r.y), d, r.x);
    }
}

// Value and derivative in d of a degree-7 FP64 row (kBoysOrderG coefficients) by joint
// Horner steps: p = p d + c_m, q = q d + p.
__device__ inline double boys_eval_d(const double *__restrict__ tab, unsigned off, double d, double &dp)
{
    static_assert(kBoysOrderG == 8, "degree-7 rows");
    const double *c = (const double *)((const char *)tab + off);
    double p = c[7], q = p;
    p = fma(p, d, c[6]);
    q = fma(q, d, p);
    p = fma(p, d, c[5]);
    q = fma(q, d, p);
    p = fma(p, d, c[4]);
    q = fma(q, d, p);
    p = fma(p, d, c[3]);
    q = fma(q, d, p);
    p = fma(p, d, c[2]);
    q = fma(q, d, p);
    p = fma(p, d, c[1]);
    q = fma(q, d, p);
    p = fma(p, d, c[0]);
    dp = q;
    return p;
}

// Wave-uniform tables read through the constant address space are fetched with scalar
// loads (they are never written while a kernel runs).
template <typename T> using cptr = const __attribute__((address_space(4))) T *;

// A value known to be the same in every lane, moved to scalar registers, so that what is
// derived from it (addresses, loop bounds, loads through cptr) stays out of the vector ones.
__device__ inline int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ inline long long uniform(long long v)
{
    const int lo = __builtin_amdgcn_readfirstlane((int)v), hi = __builtin_amdgcn_readfirstlane((int)(v >> 32));
    return ((long long)hi << 32) | (unsigned)lo;
}

// Block `at` of the numbering of bra groups: the last group g with goff[g] <= at, and within it
// ket-block-major over the group's bras (the last group holds what is left of the S bras).
__device__ inline void block_bra(cptr<long long> goff, int64_t ngroups, int gshift, int S, long long at, int &s,
                                 int &kblock)
{
    int64_t lo = 0, hi = ngroups - 1;
    while (lo < hi) {
        const int64_t mid = (lo + hi + 1) >> 1;
        if (goff[mid] <= at) lo = mid; else hi = mid - 1;
    }
    const int first = (int)(lo << gshift), left = S - first;
    const unsigned nb = left < (1 << gshift) ? left : 1 << gshift, local = (unsigned)(at - goff[lo]);
    kblock = (int)(local / nb);
    s = first + (int)(local % nb);
}

// Term masks of the quartet kernels.  Lane ab < G^2 holds the bra's exponent e_ab (kTermNone
// in the other lanes); kexp points at the maxima over the wave's kets of the G ket primitive
// pairs of one row cb.  need[d] has bit ab set if some ket primitive pair d' <= d of the row
// is not negligible beside bra primitive pair ab, so need[G-1] lists the bra primitive pairs
// with anything to do in the row, and the first d with the bit set is where the row's terms
// start: leading (tight) primitives fall away first, and the terms that stay are added in
// the order of the full sum.
template <int G> struct TermMask {
    using T = unsigned;
};
template <> struct TermMask<6> {
    using T = unsigned long long;
};
template <int G>
__device__ inline void term_masks(int ebra, cptr<int> kexp, int limit, typename TermMask<G>::T *need)
{
    using T = typename TermMask<G>::T;
    int e[G];
#pragma unroll
    for (int d = 0; d < G; ++d) e[d] = kexp[d];
    T m = 0;
#pragma unroll
    for (int d = 0; d < G; ++d) {
        m |= (T)__builtin_amdgcn_ballot_w64(ebra > limit - e[d]);
        need[d] = m;
    }
}
// The same over kets that lie in two blocks.
template <int G>
__device__ inline void term_masks(int ebra, cptr<int> kexp0, cptr<int> kexp1, int limit, typename TermMask<G>::T *need)
{
    using T = typename TermMask<G>::T;
    int e[G];
#pragma unroll
    for (int d = 0; d < G; ++d) e[d] = kexp0[d] > kexp1[d] ? kexp0[d] : kexp1[d];
    T m = 0;
#pragma unroll
    for (int d = 0; d < G; ++d) {
        m |= (T)__builtin_amdgcn_ballot_w64(ebra > limit - e[d]);
        need[d] = m;
    }
}
__device__ inline int term_first(unsigned m) { return __builtin_ctz(m); }
__device__ inline int term_first(unsigned long long m) { return __builtin_ctzll(m); }

// Calls body(integral_constant<ND>, ab) for every bra primitive pair ab listed in need, in
// ascending order, with ND >= the terms that pair needs of a row (its last ND): every count
// for G <= 4, every second one above (code size).
template <int ND> struct TermCount {
    static constexpr int value = ND;
};
template <int G, int ND, typename T, typename Body>
__device__ __attribute__((always_inline)) inline void term_dispatch(const T *need, int ab, Body &&body)
{
    constexpr int kStep = G <= 4 ? 1 : 2;
    if constexpr (ND - kStep < 1) {
        body(TermCount<ND>{}, ab);
    } else {
        // terms before the last ND - kStep: d < G - ND + kStep
        if ((need[G - ND + kStep - 1] >> ab) & 1)
            body(TermCount<ND>{}, ab);
        else
            term_dispatch<G, ND - kStep>(need, ab, body);
    }
}
template <int G, typename T, typename Body>
__device__ __attribute__((always_inline)) inline void for_terms(const T *need, Body &&body)
{
    for (T m = need[G - 1]; m; m &= m - 1) term_dispatch<G, G>(need, term_first(m), body);
}

// A uniform table at a 32-bit byte offset: the scalar load takes base and offset as they are.
// (The offset is hidden from the optimiser, which otherwise forms the 64-bit sum of its parts.)
template <typename R> __device__ inline cptr<R> at_bytes(cptr<R> base, unsigned bytes)
{
    asm("" : "+s"(bytes));
    return (cptr<R>)((cptr<char>)base + bytes);
}

// Ket table: one row per primitive pair cd, and within a row the values of a pair in 16-byte
// pieces, pair after pair: FP64 (Px, Py), (Pz, S) and a tail of |P|^2 (kQ) and kTswitch / p
// (kAtoms); FP32 (Px, Py, Pz, S) and a tail of kTswitch / p (kAtoms).  A lane's ket is two or three
// loads (FP32: one or two) of one buffer resource with the 64-bit part of the address in its
// base; an 8-byte load takes the texture addresser as long as a 16-byte one (16 cycles per
// wave), and a resource per value cost three scalar instructions each.  Offsets within a row
// stay below 2^31 for up to 2^31 / 48 pairs.
template <typename R, bool kQ, bool kAtoms> struct KetTable {
    static constexpr bool kDouble = sizeof(R) == 8;
    static constexpr int kTail = (kQ ? 1 : 0) + (kAtoms ? 1 : 0);
    static constexpr int kRow = (4 + kTail) * (int)sizeof(R);          // bytes of a row per pair
    static constexpr int kTailAt = 4 * (int)sizeof(R);                 // times pcap: where the tail starts

    static __device__ void store(R *tab, int64_t pcap, int cd, int64_t t, R x, R y, R z, R S, R q, R sw)
    {
        char *row = (char *)tab + (int64_t)cd * kRow * pcap;
        if constexpr (kDouble) {
            ((double2 *)row)[t] = make_double2(x, y);
            ((double2 *)(row + 16 * pcap))[t] = make_double2(z, S);
        } else {
            ((float4 *)row)[t] = make_float4(x, y, z, S);
        }
        R *tail = (R *)(row + (int64_t)kTailAt * pcap) + t * kTail;
        if constexpr (kQ) tail[0] = q;
        if constexpr (kAtoms) tail[kQ ? 1 : 0] = sw;
    }
    static __device__ void load(const R *tab, int64_t pcap, int cd, unsigned t, R &x, R &y, R &z, R &S, R &q, R &sw)
    {
        const __amdgpu_buffer_rsrc_t rc = __builtin_amdgcn_make_buffer_rsrc(
            (void *)((char *)const_cast<R *>(tab) + (int64_t)cd * kRow * pcap), (short)0, (int)(kRow * pcap), 0x00020000);
        const auto v = __builtin_amdgcn_raw_buffer_load_b128(rc, (int)(t * 16u), 0, 0);
        if constexpr (kDouble) {
            const double2 xy = __builtin_bit_cast(double2, v);
            const double2 zs = __builtin_bit_cast(
                double2, __builtin_amdgcn_raw_buffer_load_b128(rc, (int)(t * 16u), (int)(16 * pcap), 0));
            x = xy.x; y = xy.y; z = zs.x; S = zs.y;
            if constexpr (kTail == 2) {
                const double2 w = __builtin_bit_cast(
                    double2, __builtin_amdgcn_raw_buffer_load_b128(rc, (int)(t * 16u), (int)(32 * pcap), 0));
                q = w.x; sw = w.y;
            } else if constexpr (kTail == 1) {
                const double w = __builtin_bit_cast(
                    double, __builtin_amdgcn_raw_buffer_load_b64(rc, (int)(t * 8u), (int)(32 * pcap), 0));
                if constexpr (kQ) q = w; else sw = w;
            }
        } else {
            const float4 w = __builtin_bit_cast(float4, v);
            x = w.x; y = w.y; z = w.z; S = w.w;
            if constexpr (kAtoms)
                sw = __builtin_bit_cast(float,
                                        __builtin_amdgcn_raw_buffer_load_b32(rc, (int)(t * 4u), (int)(16 * pcap), 0));
        }
    }
};

// Pair index p = i(i+1)/2 + j (i >= j) back to (i, j).
__device__ inline void pair_of_index(int64_t p, int64_t &i, int64_t &j)
{
    int64_t r = (int64_t)((sqrt(8.0 * (double)p + 1.0) - 1.0) * 0.5);
    while (r * (r + 1) / 2 > p) --r;
    while ((r + 1) * (r + 2) / 2 <= p) ++r;
    i = r;
    j = p - r * (r + 1) / 2;
}

// Q band: floor((1 - log2 q) * bands per octave), clamped; larger Q -> smaller band.
__device__ inline int q_band(double q)
{
    const double x = (1.0 - log2(q)) * (double)kBandsPerOctave;
    if (!(x < (double)(kNumBands - 1))) return kNumBands - 1;
    return x < 0.0 ? 0 : (int)x;
}

// Lane permutation within rows of 16 lanes of a double (DPP moves of its halves).
template <int kCtrl>
__device__ inline double dpp_move(double v)
{
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_mov_dpp((int)b, kCtrl, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), kCtrl, 0xf, 0xf, true);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
__device__ inline double read_lane(double v, int lane)
{
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)b, lane), hi = __builtin_amdgcn_readlane((int)(b >> 32), lane);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// Wave-wide sum (64 lanes) of a double, the same in every lane: DPP within rows of 16 (swap of
// neighbours, of pairs, mirrored halves, mirrored row), then the four row sums.  No LDS
// permutes, of which a shuffle butterfly takes twelve.  Called with every lane active.
__device__ inline double wave_sum(double v)
{
    v += dpp_move<0xb1>(v);    // quad_perm [1, 0, 3, 2]
    v += dpp_move<0x4e>(v);    // quad_perm [2, 3, 0, 1]
    v += dpp_move<0x141>(v);   // row_half_mirror
    v += dpp_move<0x140>(v);   // row_mirror
    return (read_lane(v, 0) + read_lane(v, 16)) + (read_lane(v, 32) + read_lane(v, 48));
}

__device__ inline int lane_id() { return (int)__lane_id(); }

// Packs this wave's kets t = base + r * 64 + lane (r < sub <= kSubChunks) for which keep(t) holds
// into perm[0 .. count), as their distance from base (below 256), in ascending order (ballot +
// lane count, no atomics), and returns the wave-uniform count.
static_assert(kWave * kSubChunks <= 256, "distances fit a byte");
template <typename Keep>
__device__ inline int pack_kets(long long base, int lane, unsigned char *__restrict__ perm, Keep keep,
                                int sub = kSubChunks)
{
    int count = 0;
#pragma unroll
    for (int r = 0; r < kSubChunks; ++r) {
        if (r >= sub) break;
        const long long t = base + r * kWave + lane;
        const bool ok = keep(t);
        const unsigned long long mk = __builtin_amdgcn_ballot_w64(ok);
        if (ok)
            perm[count + (int)__builtin_amdgcn_mbcnt_hi((unsigned)(mk >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)mk, 0u))] =
                (unsigned char)(r * kWave + lane);
        count += (int)__popcll(mk);
    }
    __builtin_amdgcn_wave_barrier();
    return count;
}

}  // namespace hfk
