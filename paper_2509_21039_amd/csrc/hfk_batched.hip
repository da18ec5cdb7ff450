// Ragged batches of independent molecules in one persistent launch, forward Fock build and
// (optionally) the nuclear gradient fused into the same primitive loop.
//
// Pairs of every molecule are prepared in one pass and stored in (molecule, Q band) order;
// a bra's kets are the molecule's pairs up to its screen limit (t <= s keeps each quartet
// once).  Items of 256 kets are numbered molecule by molecule.  Workgroups fetch blocks from
// a global counter through a block table with two kinds of blocks:
//   owned:  all items of one molecule (molecules up to a tuned work bound), fetched first;
//   shared: up to bsz consecutive items of one molecule.
// A workgroup keeps the current molecule's whole two-electron matrix in LDS (lower
// triangle, the symmetrisation G = (F + F^T)/2 folded in: F_xy and F_yx land in the same
// slot) and its n x 3 gradient.  At the end of an owned block they are stored as they are
// (no other workgroup touches that molecule); at the end of a shared block they are added
// to the global accumulators with atomics.  Per primitive quartet the loop forms E(r) (the integral) and
// W(r) = E'(r)/r (its radial derivative) from the same r^2, so the forward result and the
// gradient come out of one pass over the quartets.
//
// Per-atom bases (kAtoms): pair bounds and tables come from the atom rows; the ket table's
// component 4 and a per-bra uniform array hold kTswitch / p, whose sum is the quartet's
// switch radius^2, and near steps derive rho from it (as in the single-molecule kernels).
#include <string.h>

#include <vector>

#include "hfk_device.hpp"
#include "hfk_boys.hpp"

namespace hfk {

struct BArgs {
    const DevHeader *hdr;
    const BasisDev *bd;
    const int *pk;
    const int *pl;
    const int *pm;
    const double *pq;
    const double *pd;
    const double *prim;
    const float *prim_f;
    const double *bra;
    const float *bra_f;
    const double *bip;      // per-atom bases: [pcap][g2] kTswitch / p of the bra pairs (and FP32)
    const float *bip_f;
    const double *kmu;      // per-atom gradient: [g2][pcap] ket mu and a/p
    const double *kfa;
    const long long *item_off;
    const int *lim;
    const short *bexp;      // [g2][pcap] term exponents of the bras
    const int *kexp;        // [64 kets][g2] maxima of the kets' exponents
    int tlim;               // term_limit(tau)
    const int *klo;
    const int *mol_n;
    const long long *mol_aoff;
    const long long *mol_doff;
    const long long *mol_toff;
    const double *xyz;
    const double *dens;
    double *facc;        // packed lower triangles, molecule m at mol_toff[m]
    double *gacc;        // [sum n][3]
    const long long *off_own;   // [nmol + 1] exclusive prefix of owned blocks per molecule
    const long long *off_sh;    // [nmol + 1] exclusive prefix of shared blocks per molecule
    const long long *mol_i0;    // [nmol] first item of each molecule
    const long long *mol_i1;    // [nmol] end of its items
    int nmol;
    unsigned long long *quartets;
    unsigned long long *next_block;
    int64_t pcap;
    double tau;
    int nmax;
};

static __device__ const BoysGrad64 kBoysB64 = make_boys_grad64();
static __device__ const BoysFloat kBoysB32 = make_boys_float(false);

template <typename R> struct BPrec;
template <> struct BPrec<double> {
    static __device__ const double *boys() { return kBoysB64.v; }
    static __device__ const double *prim(const BArgs &a) { return a.prim; }
    static __device__ const double *bra(const BArgs &a) { return a.bra; }
    static __device__ const double *bip(const BArgs &a) { return a.bip; }
    static __device__ const double *rsg(const BasisDev *bd) { return bd->rsg; }
};
template <> struct BPrec<float> {
    static __device__ const float *boys() { return kBoysB32.v; }
    static __device__ const float *prim(const BArgs &a) { return a.prim_f; }
    static __device__ const float *bra(const BArgs &a) { return a.bra_f; }
    static __device__ const float *bip(const BArgs &a) { return a.bip_f; }
    static __device__ const float *rsg(const BasisDev *bd) { return bd->rsg_f; }
};

__device__ inline int tri(int a, int b) { return a >= b ? a * (a + 1) / 2 + b : b * (b + 1) / 2 + a; }

// Last m in [0, nmol) with off[m] <= p: the molecule whose range of a prefix sum holds p
// (molecules with an empty range share their offset with the next one and are skipped).
__device__ inline int mol_of(const long long *__restrict__ off, int nmol, long long p)
{
    int lo = 0, hi = nmol - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (off[mid] <= p) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// ------------------------------------------------------------------ pair preparation

// Centroid of every molecule, one wave each.
__global__ __launch_bounds__(256) void k_b_mol(int nmol, const int *__restrict__ nm, const long long *__restrict__ aoff,
                                               const double *__restrict__ xyz, double *__restrict__ cent,
                                               unsigned long long *__restrict__ qmax)
{
    const int m = (int)((blockIdx.x * blockDim.x + threadIdx.x) / kWave), lane = threadIdx.x % kWave;
    if (m >= nmol) return;   // a whole wave
    double c[3] = {0, 0, 0};
    for (int i = lane; i < nm[m]; i += kWave)
        for (int d = 0; d < 3; ++d) c[d] += xyz[3 * (aoff[m] + i) + d];
    for (int d = 0; d < 3; ++d) {
        const double s = wave_sum(c[d]);
        if (lane == 0) cent[3 * m + d] = s / nm[m];
    }
    if (lane == 0) qmax[m] = 0;
}

// Schwarz bounds, TP lanes per pair, as in the single-molecule preparation: the primitive
// centres of a pair lie on the line A-B, and the lanes share its unordered primitive quartets.
// (One thread per pair took 56 us for 64 small molecules and 1.1 ms for 500 clusters.)
template <int TP>
__global__ __launch_bounds__(256) void k_b_pair_q(Basis b, int nmol, const long long *__restrict__ poff,
                                                  const long long *__restrict__ aoff, const double *__restrict__ xyz,
                                                  long long ptot, double *__restrict__ qout, int *__restrict__ mol,
                                                  unsigned long long *__restrict__ qmax)
{
    constexpr int PB = 256 / TP;
    extern __shared__ __attribute__((aligned(16))) double sm[];
    const int l = threadIdx.x % TP, pb = threadIdx.x / TP;
    double *tab = sm + (size_t)pb * 3 * b.g2;
    const long long p = (long long)blockIdx.x * PB + pb;
    const bool live = p < ptot;
    int m = 0;
    double r2 = 0.0;
    if (live) {
        m = mol_of(poff, nmol, p);
        int64_t i, j;
        pair_of_index(p - poff[m], i, j);
        i += aoff[m];
        j += aoff[m];
        const double dx = xyz[3 * i] - xyz[3 * j], dy = xyz[3 * i + 1] - xyz[3 * j + 1],
                     dz = xyz[3 * i + 2] - xyz[3 * j + 2];
        r2 = dx * dx + dy * dy + dz * dz;
        for (int ab = l; ab < b.g2; ab += TP) pair_q_entry(b, i, j, ab, r2, tab);
    }
    __syncthreads();
    double s = live ? pair_q_sum(b.g2, r2, l, TP, tab) : 0.0;
#pragma unroll
    for (int w = TP / 2; w > 0; w >>= 1) s += __shfl_xor(s, w, TP);
    if (live && l == 0) {
        const double q = sqrt(s);
        qout[p] = q;
        mol[p] = m;
        // most pairs are below the largest one met so far
        const unsigned long long bits = (unsigned long long)__double_as_longlong(q);
        if (bits > __hip_atomic_load(&qmax[m], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(&qmax[m], bits);
    }
}

template <int TP>
static void launch_b_pair_q(const Basis &b, int nmol, const long long *poff, const long long *aoff, const double *xyz,
                            long long ptot, double *q, int *mol, unsigned long long *qmax, hipStream_t st)
{
    constexpr int PB = 256 / TP;
    hipLaunchKernelGGL((k_b_pair_q<TP>), dim3((unsigned)((ptot + PB - 1) / PB)), dim3(256),
                       sizeof(double) * 3 * (size_t)b.g2 * PB, st, b, nmol, poff, aoff, xyz, ptot, q, mol, qmax);
}

// bucket_of holds the pair's molecule; it becomes its (molecule, band) bucket, or -1.
__global__ __launch_bounds__(256) void k_b_bucket_count(long long ptot, double tau,
                                                        const unsigned long long *__restrict__ qmax,
                                                        const double *__restrict__ q, int *__restrict__ bucket_of,
                                                        long long *__restrict__ cnt)
{
    const long long p = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= ptot) return;
    const int m = bucket_of[p];
    const double qm = __longlong_as_double((long long)qmax[m]);
    const double qp = q[p];
    int bk = -1;
    if (qp * qm >= tau && qp > 0.0) {
        bk = m * kNumBands + q_band(qp);
        atomicAdd((unsigned long long *)&cnt[bk], 1ULL);
    }
    bucket_of[p] = bk;
}

__global__ __launch_bounds__(256) void k_b_cursors(const long long *__restrict__ off, long long nb, int *__restrict__ cur,
                                                   DevHeader *__restrict__ hdr)
{
    const long long b = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (b < nb) cur[b] = (int)off[b];
    if (b == 0) {
        hdr->sig_pairs = (int)off[nb];
        hdr->quartets = 0;
    }
}

// Position of every significant pair (order within a bucket as the cursor hands out places).
__global__ __launch_bounds__(256) void k_b_slot(long long ptot, const int *__restrict__ bucket_of,
                                                int *__restrict__ cur, int *__restrict__ slot, int *__restrict__ pm)
{
    const long long p = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= ptot) return;
    const int bk = bucket_of[p];
    if (bk < 0) return;
    const int pos = atomicAdd(&cur[bk], 1);
    slot[pos] = (int)p;
    pm[pos] = bk / kNumBands;
}

// Tables of every significant pair at its position, for the precision of the build: one thread
// per (position, primitive pair), as in the single-molecule preparation, with 64 pad entries
// after the last pair and the maxima of the term exponents over every 64 positions.  (One
// thread per pair took 53 us for 64 small molecules and 1.0 ms for 500 clusters.)
struct BTables {
    const int *slot, *pm;
    int *pk, *pl;
    double *pq, *pd;
    void *prim, *bra, *bip;   // of the build's precision
    double *kmu, *kfa;
    short *bexp;              // [g2][pcap]
    int *kexp;                // [positions / 64][g2]
    bool grad;
};
template <typename R>
__global__ __launch_bounds__(256) void k_b_tables(Basis b, const BasisDev *__restrict__ bd,
                                                  const DevHeader *__restrict__ hdr,
                                                  const long long *__restrict__ poff,
                                                  const long long *__restrict__ aoff,
                                                  const long long *__restrict__ doff, const int *__restrict__ nm,
                                                  const double *__restrict__ cent, const double *__restrict__ xyz,
                                                  const double *__restrict__ dens, const double *__restrict__ q,
                                                  int64_t pcap, BTables T)
{
    const int S = hdr->sig_pairs;
    const int64_t at = (int64_t)blockIdx.x * 256;
    if (at >= (int64_t)S + 64) return;
    const int64_t pos = at + threadIdx.x;
    const int g2 = b.g2, ab = blockIdx.y;
    R *prim = (R *)T.prim, *bra = (R *)T.bra, *bip = (R *)T.bip;
    int e = kTermNever;
    if (pos < S) {
        const long long p = T.slot[pos];
        const int m = T.pm[pos];
        int64_t i, j;
        pair_of_index(p - poff[m], i, j);
        const double *c = cent + 3 * m;
        const int64_t gi = aoff[m] + i, gj = aoff[m] + j;
        const double A[3] = {xyz[3 * gi] - c[0], xyz[3 * gi + 1] - c[1], xyz[3 * gi + 2] - c[2]};
        const double B[3] = {xyz[3 * gj] - c[0], xyz[3 * gj + 1] - c[1], xyz[3 * gj + 2] - c[2]};
        const PrimPair w = prim_pair(b, bd, gi, gj, ab, A, B);
        if (ab == 0) {
            T.pk[pos] = (int)i;
            T.pl[pos] = (int)j;
            T.pq[pos] = q[p];
            T.pd[pos] = dens[doff[m] + i * nm[m] + j];
        }
        if (bip)
            KetTable<R, false, true>::store(prim, pcap, ab, pos, (R)w.x, (R)w.y, (R)w.z, (R)w.S, (R)0, (R)(kTswitch / w.p));
        else
            KetTable<R, false, false>::store(prim, pcap, ab, pos, (R)w.x, (R)w.y, (R)w.z, (R)w.S, (R)0, (R)0);
        // bra row: centre, charge and the charge weighted by mu and by the fractions
        // fa = a/p, fb = b/p of the primitive pair (the gradient's bra weights)
        const double fb = b.aexp ? 1.0 - w.fa : w.fb;
        const double row[kBBra] = {w.x, w.y, w.z, w.S, w.mu * w.S, w.fa * w.S, fb * w.S,
                                   w.fa * fb * w.S, fb * fb * w.S, 0.0, 0.0, 0.0};
        R *ba = bra + (pos * g2 + ab) * kBBra;
        for (int x = 0; x < kBBra; ++x) ba[x] = (R)row[x];
        if (bip) bip[pos * g2 + ab] = (R)(kTswitch / w.p);
        if (T.kmu) {
            T.kmu[(int64_t)ab * pcap + pos] = w.mu;
            T.kfa[(int64_t)ab * pcap + pos] = w.fa;
        }
        e = term_exponent(term_bound(w.S, w.p, w.mu, sqrt(w.ab2), T.grad));
        T.bexp[(int64_t)ab * pcap + pos] = (short)e;
    } else if (pos < (int64_t)S + 64) {
        if (ab == 0) {
            T.pk[pos] = 0;
            T.pl[pos] = 0;
            T.pq[pos] = 0.0;
            T.pd[pos] = 0.0;
        }
        if (bip)
            KetTable<R, false, true>::store(prim, pcap, ab, pos, (R)1e6, (R)1e6, (R)1e6, (R)0, (R)0, (R)1);
        else
            KetTable<R, false, false>::store(prim, pcap, ab, pos, (R)1e6, (R)1e6, (R)1e6, (R)0, (R)0, (R)1);
        if (T.kmu) {
            T.kmu[(int64_t)ab * pcap + pos] = 0.0;
            T.kfa[(int64_t)ab * pcap + pos] = 0.0;
        }
    }
    e = wave_max(e);
    if (threadIdx.x % kWave == 0) T.kexp[(pos / kWave) * g2 + ab] = e;
}

// Ket range of every bra s: kets t in [klo_s, lim_s), klo_s the first pair of its molecule,
// lim_s = min(s + 1, end of the molecule's band holding tau / Q_s).
__global__ __launch_bounds__(256) void k_b_limits(const DevHeader *__restrict__ hdr, double tau,
                                                  const double *__restrict__ pq, const int *__restrict__ pm,
                                                  const long long *__restrict__ boff, long long *__restrict__ nitems,
                                                  int *__restrict__ lims, int *__restrict__ klo, int64_t pcap)
{
    const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= pcap) return;
    long long ni = 0;
    if (s < hdr->sig_pairs) {
        const int m = pm[s];
        const long long start = boff[(long long)m * kNumBands];
        const double thr = tau / pq[s];
        long long bend;
        if (thr <= 0.0) {
            bend = boff[(long long)(m + 1) * kNumBands];
        } else {
            // band 0 is open-ended: a threshold above its edges still ends there
            const int bt = q_band(thr);
            bend = boff[(long long)m * kNumBands + bt + 1];
        }
        const long long lim = bend < s + 1 ? bend : s + 1;
        const long long cnt = lim > start ? lim - start : 0;
        ni = (cnt + kKetsPerItem - 1) / kKetsPerItem;
        lims[s] = (int)lim;
        klo[s] = (int)start;
    } else {
        lims[s] = 0;
        klo[s] = 0;
    }
    nitems[s] = ni;
}

// Block table of the quartet kernel.  Per molecule: its item range, and either one owned
// block (all its items; molecules with at most owned_bound unique quartets before the
// screen, P (P + 1) / 2 with P = n (n + 1) / 2) or ceil(items / bsz) shared blocks.
// bsz = block_items, or (0: automatic) total items / (8 x workgroups) clamped: at most
// 4 kBlockItems (big batches get fewer fetches and molecule switches), and at least
// kBlockItems for molecules of up to 32 items on average, which then are about a block each
// (200 molecules of up to 10 atoms: 261 us with 16, 278 with 4), a quarter of that for larger
// ones, whose blocks otherwise leave workgroups idle (64 molecules of up to 24 atoms: 503 us
// with 16, 370 with 4; 8 of up to 48: 522 and 429).  One workgroup, which also forms the
// blocks' prefix sums (a launch for each and three per prefix sum took 30 us).
constexpr int kBlockThreads = 1024;
__global__ __launch_bounds__(kBlockThreads) void k_b_blocks(DevHeader *__restrict__ hdr, int64_t nmol,
                                                  const int *__restrict__ nm, const long long *__restrict__ boff,
                                                  const long long *__restrict__ item_off, int block_items,
                                                  long long owned_bound, int groups, long long *__restrict__ mi0,
                                                  long long *__restrict__ mi1, long long *__restrict__ off_own,
                                                  long long *__restrict__ off_sh)
{
    __shared__ long long wsum[2][kBlockThreads / kWave];
    const int t = threadIdx.x, lane = t % kWave, wave = t / kWave;
    long long bsz = block_items;
    if (bsz <= 0) {
        const long long least = hdr->items <= 32 * nmol ? kBlockItems : kBlockItems / 4;
        bsz = hdr->items / (8LL * (long long)groups);
        bsz = bsz < least ? least : (bsz > 4 * kBlockItems ? 4 * kBlockItems : bsz);
    }
    long long base_own = 0, base_sh = 0;
    for (int64_t m0 = 0; m0 < nmol; m0 += kBlockThreads) {
        const int64_t m = m0 + t;
        long long own = 0, sh = 0;
        if (m < nmol) {
            const long long i0 = item_off[boff[m * kNumBands]], i1 = item_off[boff[(m + 1) * kNumBands]];
            mi0[m] = i0;
            mi1[m] = i1;
            const long long n = nm[m], P = n * (n + 1) / 2;
            const bool whole = owned_bound > 0 && P * (P + 1) / 2 <= owned_bound;
            own = whole && i1 > i0 ? 1 : 0;
            sh = whole ? 0 : (i1 - i0 + bsz - 1) / bsz;
        }
        long long x = own, y = sh;
#pragma unroll
        for (int o = 1; o < kWave; o <<= 1) {
            const long long u = __shfl_up(x, o, kWave), v = __shfl_up(y, o, kWave);
            if (lane >= o) {
                x += u;
                y += v;
            }
        }
        __syncthreads();
        if (lane == kWave - 1) {
            wsum[0][wave] = x;
            wsum[1][wave] = y;
        }
        __syncthreads();
        long long before_own = base_own, before_sh = base_sh;
        for (int w = 0; w < kBlockThreads / kWave; ++w) {
            if (w < wave) {
                before_own += wsum[0][w];
                before_sh += wsum[1][w];
            }
            base_own += wsum[0][w];
            base_sh += wsum[1][w];
        }
        if (m < nmol) {
            off_own[m] = before_own + x - own;
            off_sh[m] = before_sh + y - sh;
        }
    }
    if (t == 0) {
        off_own[nmol] = base_own;
        off_sh[nmol] = base_sh;
        hdr->bt_own = base_own;
        hdr->bt_sh = base_sh;
        hdr->bsz = bsz;
        hdr->tile = (int)bsz;
    }
}

// ------------------------------------------------------------------ fused quartet kernel

// Work within a block.  A block is a range of items of one molecule (all of them for an
// owned block).  Each item (bra s, 256 kets) is cut into four units of 64 kets, and the
// waves of the workgroup take consecutive shares of the block's units, each on its own: a wave
// walks its units in item order, keeps its bra's data while the bra stays the same, and folds its
// bra-side sums into LDS when the bra changes.  The waves meet only at the start and the
// end of a block (LDS cleared, then the molecule's accumulators written out), so a bra with
// few kets occupies one wave, not the workgroup.  The wave count per workgroup is set at
// launch (blockDim.x / 64): with a large molecule's triangle in LDS few workgroups fit on a
// CU, and wider ones keep the SIMDs supplied.
//
// Gradient contraction.  With P_ab = A + fb (B - A) and Q_cd = C + fd (D - C) (fa = a/p,
// fb = b/p, fc = c/q, fd = d/q), the separation splits into atom vectors,
//     P - Q = R_AC + fb R_BA - fd R_DC,   R_AC = A - C, R_BA = B - A, R_DC = D - C,
// so the W terms of the derivatives need only scalar sums of w = S_ab S_cd W(r) weighted by
// the fractions: per primitive quartet the lane adds S_cd E, mu_cd S_cd E, S_cd W, fd S_cd W,
// fc S_cd W and fc fd S_cd W (one FMA each), and once per bra primitive pair these are
// folded with the bra's weights (S, mu S, fa S, fb S, fa fb S, fb^2 S from the bra table).
// Every weighted sum is accumulated directly (no difference of two sums), so FP32 partial
// sums keep their relative accuracy.  Per kept quartet, with Gamma the density factor:
//   dA = Gamma [ -2 AB sum mu S S E + R_AC sum fa w + R_BA sum fa fb w - R_DC sum fa fd w ]
//   dB = Gamma [ +2 AB sum mu S S E + R_AC sum fb w + R_BA sum fb^2 w - R_DC sum fb fd w ]
//   dC = Gamma [ -2 CD sum mu_cd S S E - R_AC sum fc w - R_BA sum fc fb w + R_DC sum fc fd w ]
//   dD = -(dA + dB + dC)
template <int G, typename R, bool kGrad, bool kAtoms = false>
__global__ __launch_bounds__(kBatchMaxThreads) void k_batched(BArgs a)
{
    constexpr int G2 = G * G;
    extern __shared__ __attribute__((aligned(16))) double smem[];
    const int nmax = a.nmax;
    using BG = BoysGrid<R>;
    // the Boys table first (16-byte aligned rows), then the molecule's accumulators
    R *tHG = (R *)smem;
    double *Lt = (double *)(tHG + BG::table_len);  // [nmax (nmax+1) / 2]
    double *lg = Lt + nmax * (nmax + 1) / 2;                   // [3 nmax]
    const int nthr = (int)blockDim.x, tid = threadIdx.x, lane = tid % kWave;
    // the wave index through readfirstlane, so that everything derived from it (the unit
    // loop, the bra walk) is known to be wave-uniform and stays in scalar registers
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int nwaves = nthr / kWave;
    const int S = a.hdr->sig_pairs;
    const BasisDev *bd = a.bd;
    load_boys<R>(tHG, BPrec<R>::boys(), BG::table_len, tid, nthr);
    unsigned long long kept = 0;
    __shared__ long long blk_at;
    __shared__ int s_first;
    // blocks from a global counter through the block table: owned blocks first (whole
    // molecules), then shared blocks of bsz items, until both kinds are exhausted
    const long long bt_own = a.hdr->bt_own, bt_all = bt_own + a.hdr->bt_sh, bsz = a.hdr->bsz;
    const R *prim = BPrec<R>::prim(a);
    const cptr<R> rsg = (cptr<R>)BPrec<R>::rsg(bd);
    const cptr<double> cmu = (cptr<double>)bd->mu;
    const cptr<double> cfa = (cptr<double>)bd->fa;
    const cptr<double> cfb = (cptr<double>)bd->fb;
    for (;;) {
    __syncthreads();
    if (tid == 0) blk_at = (long long)atomicAdd(a.next_block, 1ULL);
    __syncthreads();
    const long long blk = blk_at;
    if (blk >= bt_all) break;
    const bool owned = blk < bt_own;
    const int mol = owned ? mol_of(a.off_own, a.nmol, blk) : mol_of(a.off_sh, a.nmol, blk - bt_own);
    long long m0 = a.mol_i0[mol];
    if (!owned) m0 += (blk - bt_own - a.off_sh[mol]) * bsz;
    const long long m1 = owned || m0 + bsz > a.mol_i1[mol] ? a.mol_i1[mol] : m0 + bsz;
    const int nm = a.mol_n[mol];
    const long long aoff = a.mol_aoff[mol], doff = a.mol_doff[mol], toff = a.mol_toff[mol];
    const int ntri = nm * (nm + 1) / 2;
    for (int x = tid; x < ntri; x += nthr) Lt[x] = 0.0;
    if (kGrad)
        for (int x = tid; x < 3 * nm; x += nthr) lg[x] = 0.0;
    if (tid == 0) {
        // the bra of item m0: the last s with item_off[s] <= m0
        int lo = 0, hi = S - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (a.item_off[mid] <= m0) lo = mid; else hi = mid - 1;
        }
        s_first = lo;
    }
    __syncthreads();
    {
    int s = s_first, curbra = -1;
    int bi = 0, bj = 0, lim = 0, klo = 0, ebra = kTermNone;
    double qs = 0.0, ds = 0.0;
    double jb = 0.0, gA[3] = {0, 0, 0}, gB[3] = {0, 0, 0};
    // folds this wave's bra-side sums into the LDS accumulators
    auto flush_bra = [&]() {
        const double w = wave_sum(jb);
        if (lane == 0 && w != 0.0) atomicAdd(&Lt[tri(bi, bj)], 4.0 * w);
        jb = 0.0;
        if (kGrad) {
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const double wa = wave_sum(gA[c]), wb = wave_sum(gB[c]);
                if (lane == 0) {
                    atomicAdd(&lg[3 * bi + c], wa);
                    atomicAdd(&lg[3 * bj + c], wb);
                }
                gA[c] = gB[c] = 0.0;
            }
        }
    };
    const long long nunits = (m1 - m0) * kUnitsPerItem;
    // consecutive units per wave: a bra's units mostly meet in one wave, which folds its sums
    // once; dealt out round-robin, a bra of ten units cost eight folds of seven wave sums
    const long long uend = nunits * (wave + 1) / nwaves;
    for (long long u = nunits * wave / nwaves; u < uend; ++u) {
        const long long m = m0 + u / kUnitsPerItem;
        while (a.item_off[s + 1] <= m) ++s;
        if (s != curbra) {
            if (curbra >= 0) flush_bra();
            curbra = s;
            // scalar loads: the bra's data stays in scalar registers
            bi = ((cptr<int>)a.pk)[s];
            bj = ((cptr<int>)a.pl)[s];
            qs = ((cptr<double>)a.pq)[s];
            ds = ((cptr<double>)a.pd)[s];
            lim = ((cptr<int>)a.lim)[s];
            klo = ((cptr<int>)a.klo)[s];
            ebra = lane < G2 ? (int)a.bexp[(int64_t)lane * a.pcap + s] : kTermNone;
        }
        const long long t0 = klo + (m - a.item_off[s]) * kKetsPerItem + (u % kUnitsPerItem) * kWave;
        if (t0 >= lim) continue;
        // the unit's 64 kets lie in one or two aligned blocks of 64
        const int kb0 = __builtin_amdgcn_readfirstlane((int)(t0 / kWave));
        const int kb1 = __builtin_amdgcn_readfirstlane((int)(((t0 + kWave < lim ? t0 + kWave : lim) - 1) / kWave));
        const cptr<int> kexp0 = (cptr<int>)(a.kexp + (int64_t)kb0 * G2), kexp1 = (cptr<int>)(a.kexp + (int64_t)kb1 * G2);
        const long long tk = t0 + lane;
        const bool valid = (tk < lim) && (qs * a.pq[tk] >= a.tau);
        const long long t = valid ? tk : S;   // lanes without a kept quartet read the first pad entry
        const cptr<R> bra = (cptr<R>)(BPrec<R>::bra(a) + (int64_t)s * kBBra * G2);
        const cptr<R> bipp = kAtoms ? (cptr<R>)(BPrec<R>::bip(a) + (int64_t)s * G2) : nullptr;
        const int k = a.pk[t], l = a.pl[t];

        // forward: eri; gradient: sX = sum mu_ab S S E, sZ = sum mu_cd S S E and the
        // fraction-weighted sums of w (names: weights of bra, then ket)
        R eri = R(0), sX = R(0), sZ = R(0);
        R wA = R(0), wAB = R(0), wB = R(0), wBB = R(0), wAD = R(0), wBD = R(0), wC = R(0), wCB = R(0), wCD = R(0);
#pragma unroll 1
        for (int cb = 0; cb < G; ++cb) {
            typename TermMask<G>::T need[G];
            term_masks<G>(ebra, kexp0 + cb * G, kexp1 + cb * G, a.tlim, need);
            if (!need[G - 1]) continue;
            R kx[G], ky[G], kz[G], ks[G], kp[G];
            R kms[G], kds[G], kcs[G], kcds[G];   // S_cd times mu_cd, fd, fc, fc fd
#pragma unroll
            for (int d = 0; d < G; ++d) {
                if (G <= 4 && !need[d]) continue;   // no bra primitive pair reads it
                R q;
                KetTable<R, false, kAtoms>::load(prim, a.pcap, cb * G + d, (unsigned)t, kx[d], ky[d], kz[d], ks[d], q, kp[d]);
            }
            if (kGrad) {
#pragma unroll
                for (int d = 0; d < G; ++d) {
                    if (G <= 4 && !need[d]) continue;
                    const int cd = cb * G + d;
                    double mu, fc;
                    if constexpr (kAtoms) {
                        mu = a.kmu[(int64_t)cd * a.pcap + t];
                        fc = a.kfa[(int64_t)cd * a.pcap + t];
                    } else {
                        mu = cmu[cd];
                        fc = cfa[cd];
                    }
                    const double fd = kAtoms ? 1.0 - fc : cfb[cd];
                    kms[d] = (R)mu * ks[d];
                    kcs[d] = (R)fc * ks[d];
                    kds[d] = (R)fd * ks[d];
                    kcds[d] = (R)(fc * fd) * ks[d];
                }
            }
            for_terms<G>(need, [&](auto nd, int ab) __attribute__((always_inline)) {
                constexpr int D0 = G - decltype(nd)::value;   // first term of the row
                // every scalar of this bra primitive in one batch of scalar loads:
                // Px Py Pz S mu*S fa*S fb*S fa*fb*S fb^2*S, and the switch data
                const cptr<R> bp = at_bytes<R>(bra, (unsigned)ab * (kBBra * sizeof(R)));
                R b[kGrad ? 9 : 4], u[4 * G], bsw = R(0);
#pragma unroll
                for (int c = 0; c < (kGrad ? 9 : 4); ++c) b[c] = bp[c];
                if constexpr (kAtoms) {
                    bsw = bipp[ab];
                    asm volatile("" ::"s"(bsw));
                } else {
                    const cptr<R> up =
                        at_bytes<R>(rsg, ((unsigned)ab * G2 + (unsigned)cb * G) * (unsigned)(4 * sizeof(R)));
#pragma unroll
                    for (int c = 4 * D0; c < 4 * G; ++c) u[c] = up[c];
#pragma unroll
                    for (int c = 4 * D0; c < 4 * G; ++c) asm volatile("" ::"s"(u[c]));
                }
                const R px = b[0], py = b[1], pz = b[2];
                R U = R(0), Y = R(0), X0 = R(0), X1 = R(0), Xc = R(0), Xcd = R(0);
                // every lane's separation and far-field E, W first (independent across d:
                // their reciprocal square roots issue back to back), then the near lanes
                // overwrite theirs from the table under exec masks
                R r2[G], E[G], W[G];
#pragma unroll
                for (int d = D0; d < G; ++d) {
                    const R dx = px - kx[d], dy = py - ky[d], dz = pz - kz[d];
                    r2[d] = dx * dx + dy * dy + dz * dz;
                    const R y = GradScale<R>::e_far(r2[d]);
                    E[d] = y;
                    W[d] = kGrad ? GradScale<R>::w_far(y) : R(0);
                }
#pragma unroll
                for (int d = D0; d < G; ++d) {
                    // switch radius^2 kTswitch / rho (per-atom bases: sum of the stored halves)
                    const R sw = kAtoms ? bsw + kp[d] : u[4 * d];
                    if (r2[d] < sw) {
                        // (rho/h, sqrt(rho/h), (rho/h)^(3/2)) from the table, or from sw
                        R q1, q2, q3;
                        if constexpr (kAtoms) {
                            q2 = rsqrt_r(sw) * R(BG::sqrt_sw_inv_h);
                            q1 = q2 * q2;
                            q3 = q1 * q2;
                        } else {
                            q1 = u[4 * d + 1];
                            q2 = u[4 * d + 2];
                            q3 = u[4 * d + 3];
                        }
                        // sqrt(h) H and h^(3/2) g at T' = T / h on the table grid
                        R dd;
                        const unsigned off = boys_row<R, BG::pair_stride>(r2[d], q1, dd);
                        if constexpr (sizeof(R) == 8) {
                            // degree-7 rows of H; g = 2 H': W on the grid is (2 kW / kE) dE/dd
                            double de;
                            E[d] = q2 * boys_eval_d(tHG, off, dd, de);
                            if constexpr (kGrad) W[d] = q3 * (R(2.0 * GradScale<R>::kW / GradScale<R>::kE) * de);
                        } else {
                            E[d] = q2 * boys_eval<R>(tHG, off, dd);
                            if constexpr (kGrad) W[d] = q3 * boys_eval<R>(tHG + BG::g_off, off, dd);
                        }
                    }
                }
#pragma unroll
                for (int d = D0; d < G; ++d) {
                    U = fma(ks[d], E[d], U);
                    if constexpr (kGrad) {
                        Y = fma(kms[d], E[d], Y);
                        X0 = fma(ks[d], W[d], X0);
                        X1 = fma(kds[d], W[d], X1);
                        Xc = fma(kcs[d], W[d], Xc);
                        Xcd = fma(kcds[d], W[d], Xcd);
                    }
                }
                eri = fma(b[3], U, eri);
                if constexpr (kGrad) {
                    sX = fma(b[4], U, sX);
                    sZ = fma(b[3], Y, sZ);
                    wA = fma(b[5], X0, wA);
                    wAB = fma(b[7], X0, wAB);
                    wB = fma(b[6], X0, wB);
                    wBB = fma(b[8], X0, wBB);
                    wAD = fma(b[5], X1, wAD);
                    wBD = fma(b[6], X1, wBD);
                    wC = fma(b[3], Xc, wC);
                    wCB = fma(b[6], Xc, wCB);
                    wCD = fma(b[3], Xcd, wCD);
                }
            });
        }
        {
            // back from the accumulators' scales (E times kE, W times kW)
            constexpr R iE = R(1) / GradScale<R>::kE, iW = R(1) / GradScale<R>::kW;
            eri *= iE;
            if (kGrad) {
                sX *= iE; sZ *= iE;
                wA *= iW; wAB *= iW; wB *= iW; wBB *= iW; wAD *= iW; wBD *= iW; wC *= iW; wCB *= iW; wCD *= iW;
            }
        }
        if (valid) {
            ++kept;
            double deg = 1.0;
            if (bi == bj) deg *= 0.5;
            if (k == l) deg *= 0.5;
            if (t == s) deg *= 0.5;
            const double v = (double)eri * deg;
            const double *Dm = a.dens + doff;
            const double Dik = Dm[bi * nm + k], Dil = Dm[bi * nm + l];
            const double Djk = Dm[bj * nm + k], Djl = Dm[bj * nm + l];
            const double dt = a.pd[t];
            jb = fma(dt, v, jb);
            atomicAdd(&Lt[tri(k, l)], 4.0 * ds * v);
            atomicAdd(&Lt[tri(bi, k)], -Djl * v);
            atomicAdd(&Lt[tri(bi, l)], -Djk * v);
            atomicAdd(&Lt[tri(bj, k)], -Dil * v);
            atomicAdd(&Lt[tri(bj, l)], -Dik * v);
            if (kGrad) {
                const double gam = deg * (4.0 * ds * dt - Dik * Djl - Dil * Djk);
                const double *xc = a.xyz + 3 * (aoff + k), *xd = a.xyz + 3 * (aoff + l);
                const cptr<double> A = (cptr<double>)a.xyz + 3 * (aoff + bi), B = (cptr<double>)a.xyz + 3 * (aoff + bj);
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    const double rac = A[c] - xc[c], rba = B[c] - A[c], rdc = xd[c] - xc[c];
                    const double GA = gam * (2.0 * rba * (double)sX + rac * (double)wA + rba * (double)wAB -
                                             rdc * (double)wAD);
                    const double GB = gam * (-2.0 * rba * (double)sX + rac * (double)wB + rba * (double)wBB -
                                             rdc * (double)wBD);
                    const double GC = gam * (2.0 * rdc * (double)sZ - rac * (double)wC - rba * (double)wCB +
                                             rdc * (double)wCD);
                    gA[c] += GA;
                    gB[c] += GB;
                    atomicAdd(&lg[3 * k + c], GC);
                    atomicAdd(&lg[3 * l + c], -(GA + GB + GC));
                }
            }
        }
    }
    if (curbra >= 0) flush_bra();
    }
    __syncthreads();
    if (owned) {
        // the molecule's only block: store the accumulators as they are
        for (int x = tid; x < ntri; x += nthr) a.facc[toff + x] = Lt[x];
        if (kGrad)
            for (int x = tid; x < 3 * nm; x += nthr) a.gacc[3 * aoff + x] = lg[x];
    } else {
        for (int x = tid; x < ntri; x += nthr) {
            const double v = Lt[x];
            if (v != 0.0) atomicAdd(&a.facc[toff + x], v);
        }
        if (kGrad) {
            for (int x = tid; x < 3 * nm; x += nthr) {
                const double v = lg[x];
                if (v != 0.0) atomicAdd(&a.gacc[3 * aoff + x], v);
            }
        }
    }
    }
    for (int off = 32; off > 0; off >>= 1) kept += __shfl_xor(kept, off, 64);
    if (lane == 0 && kept) atomicAdd(a.quartets, kept);
}

// G from the folded lower triangle, E2 = 1/2 sum D o G and the gradient, one block per molecule.
__global__ __launch_bounds__(256) void k_b_final(const int *__restrict__ mol_n, const long long *__restrict__ doff,
                                                 const long long *__restrict__ toff, const double *__restrict__ facc,
                                                 const double *__restrict__ dens, double *__restrict__ fock,
                                                 double *__restrict__ e2, const long long *__restrict__ aoff,
                                                 const double *__restrict__ gacc, double *__restrict__ d_xyz)
{
    __shared__ double red[256];
    const int m = blockIdx.x;
    const int n = mol_n[m];
    if (d_xyz)
        for (int x = threadIdx.x; x < 3 * n; x += 256) d_xyz[3 * aoff[m] + x] = gacc[3 * aoff[m] + x];
    const double *L = facc + toff[m];
    double e = 0.0;
    for (int x = threadIdx.x; x < n * n; x += 256) {
        const int i = x / n, j = x % n;
        const double v = i == j ? L[tri(i, i)] : 0.5 * L[tri(i, j)];
        fock[doff[m] + x] = v;
        e += dens[doff[m] + x] * v;
    }
    red[threadIdx.x] = e;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) e2[m] = 0.5 * red[0];
}

// ------------------------------------------------------------------ host side

template <int G, typename R, bool GR, bool AT>
static int bres(size_t smem, int threads)
{
    int nb = 0;
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_batched<G, R, GR, AT>, threads, smem) == hipSuccess
               ? nb
               : 0;
}

template <typename R, bool GR, bool AT>
static int bres_g(int g, size_t smem, int threads)
{
    switch (g) {
    case 1: return bres<1, R, GR, AT>(smem, threads);
    case 2: return bres<2, R, GR, AT>(smem, threads);
    case 3: return bres<3, R, GR, AT>(smem, threads);
    case 4: return bres<4, R, GR, AT>(smem, threads);
    case 5: return bres<5, R, GR, AT>(smem, threads);
    default: return bres<6, R, GR, AT>(smem, threads);
    }
}

// Workgroups of the batched kernel (`waves` waves each) that fit on one CU at once (0 if the
// runtime cannot tell).
int batched_resident_groups(int g, int prec, bool grad, bool atoms, int nmax, int waves)
{
    const size_t smem = batched_smem_bytes(nmax, prec);
    const int th = waves * kWave;
    if (prec == HFK_MIXED) {
        if (grad) return atoms ? bres_g<float, true, true>(g, smem, th) : bres_g<float, true, false>(g, smem, th);
        return atoms ? bres_g<float, false, true>(g, smem, th) : bres_g<float, false, false>(g, smem, th);
    }
    if (grad) return atoms ? bres_g<double, true, true>(g, smem, th) : bres_g<double, true, false>(g, smem, th);
    return atoms ? bres_g<double, false, true>(g, smem, th) : bres_g<double, false, false>(g, smem, th);
}

size_t batched_smem_bytes(int nmax, int prec)
{
    return sizeof(double) * ((size_t)nmax * (nmax + 1) / 2 + 3 * (size_t)nmax) +
           (prec == HFK_MIXED ? sizeof(float) * BoysGrid<float>::table_len
                              : sizeof(double) * BoysGrid<double>::table_len);
}

BLayout make_blayout(int64_t nmol, const int64_t *atom_off, int g, int with_grad, bool atoms)
{
    BLayout L;
    memset(&L, 0, sizeof(L));
    L.nmol = nmol;
    L.atoms = atoms;
    L.g = g;
    L.g2 = g * g;
    long long ptot = 0, ntot = 0, tri = 0, nmax = 0;
    for (int64_t m = 0; m < nmol; ++m) {
        const long long n = atom_off[m + 1] - atom_off[m];
        ptot += n * (n + 1) / 2;
        tri += n * (n + 1) / 2;
        ntot += n;
        nmax = n > nmax ? n : nmax;
    }
    L.ptot = ptot;
    L.ntot = ntot;
    L.tri = tri;
    L.nmax = (int)nmax;
    L.pcap = ((ptot + 63) / 64) * 64 + 64;
    size_t o = 0;
    auto take = [&](size_t bytes) {
        size_t at = o;
        o = (o + bytes + 255) & ~(size_t)255;
        return at;
    };
    const size_t PC = (size_t)L.pcap, g2 = (size_t)L.g2, NM = (size_t)nmol;
    const size_t NB = NM * kNumBands;
    L.hdr = take(sizeof(DevHeader));
    L.basis = take(sizeof(BasisDev));
    L.mol_n = take(sizeof(int) * NM);
    L.mol_aoff = take(sizeof(long long) * (NM + 1));
    L.mol_poff = take(sizeof(long long) * (NM + 1));
    L.mol_doff = take(sizeof(long long) * (NM + 1));
    L.mol_toff = take(sizeof(long long) * (NM + 1));
    L.cent = take(sizeof(double) * 3 * NM);
    L.qmax = take(sizeof(unsigned long long) * NM);
    L.q = take(sizeof(double) * (size_t)ptot);
    L.bucket_of = take(sizeof(int) * (size_t)ptot);
    L.bcnt = take(sizeof(long long) * NB);
    L.boff = take(sizeof(long long) * (NB + 1));
    L.bcur = take(sizeof(int) * NB);
    L.pk = take(sizeof(int) * PC);
    L.pl = take(sizeof(int) * PC);
    L.pm = take(sizeof(int) * PC);
    L.pq = take(sizeof(double) * PC);
    L.pd = take(sizeof(double) * PC);
    L.prim = take(sizeof(double) * (atoms ? 5 : 4) * g2 * PC);   // Px, Py, Pz, S (, kTswitch/p)
    L.prim_f = take(sizeof(float) * (atoms ? 5 : 4) * g2 * PC);
    if (atoms) {
        L.arow = take(sizeof(double) * 2 * (size_t)ntot * (size_t)g);
        L.bip = take(sizeof(double) * g2 * PC);
        L.bip_f = take(sizeof(float) * g2 * PC);
        if (with_grad) {
            L.kmu = take(sizeof(double) * g2 * PC);
            L.kfa = take(sizeof(double) * g2 * PC);
        }
    }
    L.bra = take(sizeof(double) * kBBra * g2 * PC);
    L.bra_f = take(sizeof(float) * kBBra * g2 * PC);
    L.nitems = take(sizeof(long long) * PC);
    L.bexp = take(sizeof(short) * (size_t)L.g2 * (size_t)L.pcap);
    L.kexp = take(sizeof(int) * (size_t)L.g2 * (size_t)(L.pcap / kWave + 4));
    L.lim = take(sizeof(int) * PC);
    L.klo = take(sizeof(int) * PC);
    L.item_off = take(sizeof(long long) * (PC + 1));
    const size_t scan_n = PC > NB ? PC : NB;
    L.scan_tmp = take(sizeof(long long) * ((scan_n + 1023) / 1024 + 1));
    L.facc = take(sizeof(double) * (size_t)tri);
    L.gacc = with_grad ? take(sizeof(double) * 3 * (size_t)ntot) : 0;
    L.mol_i0 = take(sizeof(long long) * NM);
    L.mol_i1 = take(sizeof(long long) * NM);
    L.off_own = take(sizeof(long long) * (NM + 1));
    L.off_sh = take(sizeof(long long) * (NM + 1));
    L.total = o;
    return L;
}

hipError_t upload_batch_tables(const BLayout &L, char *ws, const int64_t *atom_off_host, hipStream_t st)
{
    // the five tables lie one after another in the workspace: one copy of their staged image
    const int64_t nmol = L.nmol;
    std::vector<char> image(L.cent - L.mol_n);
    int *nm = (int *)image.data();
    auto table = [&](size_t at) { return (long long *)(image.data() + (at - L.mol_n)); };
    long long *aoff = table(L.mol_aoff), *poff = table(L.mol_poff), *doff = table(L.mol_doff), *toff = table(L.mol_toff);
    aoff[0] = poff[0] = doff[0] = toff[0] = 0;
    for (int64_t m = 0; m < nmol; ++m) {
        const long long n = atom_off_host[m + 1] - atom_off_host[m];
        nm[m] = (int)n;
        aoff[m + 1] = atom_off_host[m + 1];
        poff[m + 1] = poff[m] + n * (n + 1) / 2;
        doff[m + 1] = doff[m] + n * n;
        toff[m + 1] = toff[m] + n * (n + 1) / 2;
    }
    hipError_t e = hipMemcpyAsync(ws + L.mol_n, image.data(), image.size(), hipMemcpyHostToDevice, st);
    // the host image ends with this call: wait until the copy has consumed it
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    return e;
}

hipError_t launch_batched(const BLayout &L, const Basis &b, char *ws, const double *xyz, const double *dens, double tau,
                          int prec, double *fock, double *e2, double *d_xyz, int groups, const BatchedShape &shape,
                          hipStream_t st)
{
    const int64_t nmol = L.nmol;
    hipError_t e = hipSuccess;
    DevHeader *hdr = (DevHeader *)(ws + L.hdr);
    const BasisDev *bd = (const BasisDev *)(ws + L.basis);
    const int *d_n = (const int *)(ws + L.mol_n);
    const long long *d_aoff = (const long long *)(ws + L.mol_aoff);
    const long long *d_poff = (const long long *)(ws + L.mol_poff);
    const long long *d_doff = (const long long *)(ws + L.mol_doff);
    const long long *d_toff = (const long long *)(ws + L.mol_toff);
    double *cent = (double *)(ws + L.cent);
    unsigned long long *qmax = (unsigned long long *)(ws + L.qmax);
    const unsigned nbp = (unsigned)((L.ptot + 255) / 256);
    const long long NB = (long long)nmol * kNumBands;
    long long *bcnt = (long long *)(ws + L.bcnt);
    long long *boff = (long long *)(ws + L.boff);
    int *bcur = (int *)(ws + L.bcur);
    // header and basis constants, F's accumulators and the bucket counters cleared
    const HeaderInfo info{0, groups, prec, -1, 0, 0, 0};
    const bool grad = d_xyz != nullptr;
    // the gradient's accumulators follow F's
    const int64_t nacc = grad ? (int64_t)(L.gacc - L.facc) / 8 + 3 * L.ntot : L.tri;
    e = launch_prep_begin(b, (BasisDev *)(ws + L.basis), hdr, L.ntot, nullptr, info, (double *)(ws + L.facc), nacc,
                          bcnt, NB, st);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_b_mol, dim3((unsigned)((nmol + 3) / 4)), dim3(256), 0, st, (int)nmol, d_n, d_aoff, xyz, cent,
                       qmax);
    double *q = (double *)(ws + L.q);
    int *bucket = (int *)(ws + L.bucket_of);
    switch (b.g) {
    case 1: launch_b_pair_q<1>(b, (int)nmol, d_poff, d_aoff, xyz, L.ptot, q, bucket, qmax, st); break;
    case 2: launch_b_pair_q<4>(b, (int)nmol, d_poff, d_aoff, xyz, L.ptot, q, bucket, qmax, st); break;
    case 3: launch_b_pair_q<16>(b, (int)nmol, d_poff, d_aoff, xyz, L.ptot, q, bucket, qmax, st); break;
    default: launch_b_pair_q<64>(b, (int)nmol, d_poff, d_aoff, xyz, L.ptot, q, bucket, qmax, st); break;
    }
    hipLaunchKernelGGL(k_b_bucket_count, dim3(nbp), dim3(256), 0, st, L.ptot, tau, qmax, (const double *)q, bucket,
                       bcnt);
    e = launch_scan(bcnt, NB, boff, (long long *)(ws + L.scan_tmp), nullptr, st);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_b_cursors, dim3((unsigned)((NB + 255) / 256)), dim3(256), 0, st, boff, NB, bcur, hdr);
    // the pair of every position (the item counts' storage is free until the limits are computed)
    int *slot = (int *)(ws + L.nitems);
    hipLaunchKernelGGL(k_b_slot, dim3(nbp), dim3(256), 0, st, L.ptot, (const int *)bucket, bcur, slot,
                       (int *)(ws + L.pm));
    BTables T;
    T.slot = slot;
    T.pm = (const int *)(ws + L.pm);
    T.pk = (int *)(ws + L.pk);
    T.pl = (int *)(ws + L.pl);
    T.pq = (double *)(ws + L.pq);
    T.pd = (double *)(ws + L.pd);
    const bool mixed = prec == HFK_MIXED;
    T.prim = ws + (mixed ? L.prim_f : L.prim);
    T.bra = ws + (mixed ? L.bra_f : L.bra);
    T.bip = L.atoms ? ws + (mixed ? L.bip_f : L.bip) : nullptr;
    T.kmu = L.kmu ? (double *)(ws + L.kmu) : nullptr;
    T.kfa = L.kmu ? (double *)(ws + L.kfa) : nullptr;
    T.bexp = (short *)(ws + L.bexp);
    T.kexp = (int *)(ws + L.kexp);
    T.grad = grad;
    const dim3 tgrid((unsigned)((L.ptot + 64 + 255) / 256), (unsigned)L.g2);
    if (mixed)
        hipLaunchKernelGGL((k_b_tables<float>), tgrid, dim3(256), 0, st, b, bd, hdr, d_poff, d_aoff, d_doff, d_n, cent,
                           xyz, dens, (const double *)q, L.pcap, T);
    else
        hipLaunchKernelGGL((k_b_tables<double>), tgrid, dim3(256), 0, st, b, bd, hdr, d_poff, d_aoff, d_doff, d_n, cent,
                           xyz, dens, (const double *)q, L.pcap, T);
    const unsigned nbc = (unsigned)((L.pcap + 255) / 256);
    hipLaunchKernelGGL(k_b_limits, dim3(nbc), dim3(256), 0, st, hdr, tau, (const double *)(ws + L.pq),
                       (const int *)(ws + L.pm), boff, (long long *)(ws + L.nitems), (int *)(ws + L.lim),
                       (int *)(ws + L.klo), L.pcap);
    e = launch_scan((const long long *)(ws + L.nitems), L.pcap, (long long *)(ws + L.item_off),
                    (long long *)(ws + L.scan_tmp), &hdr->items, st);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_b_blocks, dim3(1), dim3(kBlockThreads), 0, st, hdr, (int64_t)nmol, d_n,
                       (const long long *)boff, (const long long *)(ws + L.item_off), shape.block_items,
                       shape.owned_bound, groups, (long long *)(ws + L.mol_i0), (long long *)(ws + L.mol_i1),
                       (long long *)(ws + L.off_own), (long long *)(ws + L.off_sh));
    BArgs a;
    a.hdr = hdr;
    a.bd = bd;
    a.pk = (const int *)(ws + L.pk);
    a.pl = (const int *)(ws + L.pl);
    a.pm = (const int *)(ws + L.pm);
    a.pq = (const double *)(ws + L.pq);
    a.pd = (const double *)(ws + L.pd);
    a.prim = (const double *)(ws + L.prim);
    a.prim_f = (const float *)(ws + L.prim_f);
    a.bra = (const double *)(ws + L.bra);
    a.bra_f = (const float *)(ws + L.bra_f);
    a.bip = L.atoms ? (const double *)(ws + L.bip) : nullptr;
    a.bip_f = L.atoms ? (const float *)(ws + L.bip_f) : nullptr;
    a.kmu = L.kmu ? (const double *)(ws + L.kmu) : nullptr;
    a.kfa = L.kmu ? (const double *)(ws + L.kfa) : nullptr;
    a.item_off = (const long long *)(ws + L.item_off);
    a.lim = (const int *)(ws + L.lim);
    a.bexp = (const short *)(ws + L.bexp);
    a.kexp = (const int *)(ws + L.kexp);
    a.tlim = term_limit(tau, prec);
    a.klo = (const int *)(ws + L.klo);
    a.mol_n = d_n;
    a.mol_aoff = d_aoff;
    a.mol_doff = d_doff;
    a.mol_toff = d_toff;
    a.xyz = xyz;
    a.dens = dens;
    a.facc = (double *)(ws + L.facc);
    a.gacc = grad ? (double *)(ws + L.gacc) : nullptr;
    a.quartets = &hdr->quartets;
    a.next_block = &hdr->next_block;
    a.off_own = (const long long *)(ws + L.off_own);
    a.off_sh = (const long long *)(ws + L.off_sh);
    a.mol_i0 = (const long long *)(ws + L.mol_i0);
    a.mol_i1 = (const long long *)(ws + L.mol_i1);
    a.nmol = (int)nmol;
    a.pcap = L.pcap;
    a.tau = tau;
    a.nmax = L.nmax;
    const size_t smem = batched_smem_bytes(L.nmax, prec);
    const int threads = (shape.waves == 8 ? 8 : 4) * kWave;
    profile_begin(st);
    if (grad && L.atoms && !L.kmu) return hipErrorInvalidValue;   // per-atom gradient tables missing
#define HFK_B_LAUNCH(GG, RR, GR)                                                                         \
    do {                                                                                                 \
        if (L.atoms)                                                                                     \
            hipLaunchKernelGGL((k_batched<GG, RR, GR, true>), dim3(groups), dim3(threads), smem, st, a); \
        else                                                                                             \
            hipLaunchKernelGGL((k_batched<GG, RR, GR, false>), dim3(groups), dim3(threads), smem, st, a); \
    } while (0)
    if (prec == HFK_MIXED) {
        if (grad) {
            switch (b.g) {
            case 1: HFK_B_LAUNCH(1, float, true); break;
            case 2: HFK_B_LAUNCH(2, float, true); break;
            case 3: HFK_B_LAUNCH(3, float, true); break;
            case 4: HFK_B_LAUNCH(4, float, true); break;
            case 5: HFK_B_LAUNCH(5, float, true); break;
            default: HFK_B_LAUNCH(6, float, true); break;
            }
        } else {
            switch (b.g) {
            case 1: HFK_B_LAUNCH(1, float, false); break;
            case 2: HFK_B_LAUNCH(2, float, false); break;
            case 3: HFK_B_LAUNCH(3, float, false); break;
            case 4: HFK_B_LAUNCH(4, float, false); break;
            case 5: HFK_B_LAUNCH(5, float, false); break;
            default: HFK_B_LAUNCH(6, float, false); break;
            }
        }
    } else {
        if (grad) {
            switch (b.g) {
            case 1: HFK_B_LAUNCH(1, double, true); break;
            case 2: HFK_B_LAUNCH(2, double, true); break;
            case 3: HFK_B_LAUNCH(3, double, true); break;
            case 4: HFK_B_LAUNCH(4, double, true); break;
            case 5: HFK_B_LAUNCH(5, double, true); break;
            default: HFK_B_LAUNCH(6, double, true); break;
            }
        } else {
            switch (b.g) {
            case 1: HFK_B_LAUNCH(1, double, false); break;
            case 2: HFK_B_LAUNCH(2, double, false); break;
            case 3: HFK_B_LAUNCH(3, double, false); break;
            case 4: HFK_B_LAUNCH(4, double, false); break;
            case 5: HFK_B_LAUNCH(5, double, false); break;
            default: HFK_B_LAUNCH(6, double, false); break;
            }
        }
    }
#undef HFK_B_LAUNCH
    profile_end(st);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_b_final, dim3((unsigned)nmol), dim3(256), 0, st, d_n, d_doff, d_toff,
                       (const double *)(ws + L.facc), dens, fock, e2, d_aoff, (const double *)a.gacc, d_xyz);
    return hipGetLastError();
}

}  // namespace hfk
