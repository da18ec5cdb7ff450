// Setup and pair preparation for the Fock build: basis constants, Boys table, Schwarz
// bounds, the Q-bucketed pair order and the work items of the quartet kernel.
#include <string.h>

#include "hfk_device.hpp"

namespace hfk {

// ------------------------------------------------------------------ setup

// First launch of a build: basis constants per primitive pair and quartet, header, centroid and
// bounding box of xyz if given (workgroup 0), and the clearing of F and of the bucket counters
// (the others).
// One launch in place of five: on small systems a launch costs more (4.5 us) than its work.
__global__ __launch_bounds__(256) void k_prep_begin(Basis b, BasisDev *__restrict__ bd, DevHeader *__restrict__ hdr,
                                                    int64_t n, const double *__restrict__ xyz, HeaderInfo info,
                                                    double *__restrict__ fzero, int64_t nf,
                                                    long long *__restrict__ cnt, int64_t ncnt)
{
    const int t = threadIdx.x;
    const int g = b.g, g2 = b.g2;
    if (blockIdx.x > 0) {
        const int64_t at = (int64_t)(blockIdx.x - 1) * blockDim.x + t, step = (int64_t)(gridDim.x - 1) * blockDim.x;
        for (int64_t x = at; x < g2 * g2; x += step) {
            const int ab = (int)x / g2, cd = (int)x % g2;
            const double p = b.alpha[ab / g] + b.alpha[ab % g];
            const double q = b.alpha[cd / g] + b.alpha[cd % g];
            const double rho = p * q / (p + q);
            if (cd == 0) {
                const double mu = b.alpha[ab / g] * b.alpha[ab % g] / p;
                bd->p[ab] = p;
                bd->mu[ab] = mu;
                bd->fa[ab] = b.alpha[ab / g] / p;
                bd->fb[ab] = b.alpha[ab % g] / p;
                bd->pi32[ab] = pow(kPi / p, 1.5);
            }
            bd->rho[x] = rho;
            bd->srho[x] = sqrt(rho);
            bd->rho_f[x] = (float)rho;
            bd->srho_f[x] = (float)sqrt(rho);
            const double r = rho * kBoysInvH, sr = sqrt(r), rf = rho * kBoysInvHF, srf = sqrt(rf);
            bd->rsn[3 * x] = kTswitch / rho;
            bd->rsn[3 * x + 1] = r;
            bd->rsn[3 * x + 2] = sr;
            bd->rsn_f[3 * x] = (float)(kTswitch / rho);
            bd->rsn_f[3 * x + 1] = (float)rf;
            bd->rsn_f[3 * x + 2] = (float)srf;
            bd->rsg[4 * x] = kTswitch / rho;
            bd->rsg[4 * x + 1] = r;
            bd->rsg[4 * x + 2] = sr;
            bd->rsg[4 * x + 3] = r * sr;
            bd->rsg_f[4 * x] = (float)(kTswitch / rho);
            bd->rsg_f[4 * x + 1] = (float)rf;
            bd->rsg_f[4 * x + 2] = (float)srf;
            bd->rsg_f[4 * x + 3] = (float)(rf * srf);
        }
        for (int64_t x = at; x < nf; x += step) fzero[x] = 0.0;
        for (int64_t x = at; x < ncnt; x += step) cnt[x] = 0;
        return;
    }
    // centroid and bounding box (block reductions)
    __shared__ double red[3][256], rmin[3][256], rmax[3][256];
    double s0 = 0, s1 = 0, s2 = 0;
    double lo[3] = {1e300, 1e300, 1e300}, hi[3] = {-1e300, -1e300, -1e300};
    for (int64_t i = t; xyz && i < n; i += blockDim.x) {
        s0 += xyz[3 * i];
        s1 += xyz[3 * i + 1];
        s2 += xyz[3 * i + 2];
        for (int c = 0; c < 3; ++c) {
            lo[c] = fmin(lo[c], xyz[3 * i + c]);
            hi[c] = fmax(hi[c], xyz[3 * i + c]);
        }
    }
    red[0][t] = s0; red[1][t] = s1; red[2][t] = s2;
    for (int c = 0; c < 3; ++c) {
        rmin[c][t] = lo[c];
        rmax[c][t] = hi[c];
    }
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (t < w) {
            for (int c = 0; c < 3; ++c) {
                red[c][t] += red[c][t + w];
                rmin[c][t] = fmin(rmin[c][t], rmin[c][t + w]);
                rmax[c][t] = fmax(rmax[c][t], rmax[c][t + w]);
            }
        }
        __syncthreads();
    }
    if (t == 0) {
        for (int c = 0; c < 3; ++c) {
            hdr->bmin[c] = rmin[c][0];
            hdr->bmax[c] = rmax[c][0];
        }
        hdr->qmax_bits = 0;
        hdr->sig_pairs = 0;
        hdr->items = 0;
        hdr->quartets = 0;
        hdr->max_bucket = 0;
        hdr->next_block = 0;
        hdr->centroid[0] = red[0][0] / (double)n;
        hdr->centroid[1] = red[1][0] / (double)n;
        hdr->centroid[2] = red[2][0] / (double)n;
        hdr->natoms = (int)n;
        hdr->strategy = info.strategy;
        hdr->groups = info.groups;
        hdr->precision = info.precision;
        hdr->variant = info.variant;
        hdr->tile = info.tile;
        hdr->group_bras = info.group_bras;
        hdr->ket_copies = info.ket_copies;
    }
}

hipError_t launch_prep_begin(const Basis &b, BasisDev *bd, DevHeader *hdr, int64_t n, const double *xyz,
                             const HeaderInfo &info, double *fzero, int64_t nf, long long *cnt, int64_t ncnt,
                             hipStream_t st)
{
    // the constants of one basis take a workgroup or a few; the clearing 4 KB a thread at most
    const int64_t work = (int64_t)b.g2 * b.g2 + (nf > ncnt ? nf : ncnt) / 4;
    const int64_t nb = 1 + (work + 255) / 256;
    hipLaunchKernelGGL(k_prep_begin, dim3((unsigned)(nb < 1024 ? nb : 1024)), dim3(256), 0, st, b, bd, hdr, n, xyz,
                       info, fzero, nf, cnt, ncnt);
    return hipGetLastError();
}

// ------------------------------------------------------------------ pairs

// Morton index of the cell holding point c inside the bounding box.
__device__ inline int morton_cell(const double *c, const DevHeader *__restrict__ hdr)
{
    constexpr int side = 1 << kCellBits;
    int code = 0;
    for (int d = 0; d < 3; ++d) {
        const double ext = hdr->bmax[d] - hdr->bmin[d];
        int u = ext > 0.0 ? (int)((c[d] - hdr->bmin[d]) / ext * side) : 0;
        u = u < 0 ? 0 : (u >= side ? side - 1 : u);
        for (int b = 0; b < kCellBits; ++b) code |= ((u >> b) & 1) << (3 * b + d);
    }
    return code;
}

// Schwarz bound of every pair i >= j: Q_ij = sqrt((ij|ij)) in FP64, TP lanes per pair.  All
// primitive centres lie on the line A-B, P_ab - P_cd = (fb_ab - fb_cd) (B - A), and the matrix
// (ab|cd) is symmetric, so the lanes share the g2 (g2 + 1) / 2 unordered primitive quartets,
// each S_ab S_cd sqrt(rho) H(rho |P-Q|^2) with the library's erf.  One thread per pair summed
// all g2^2 of them in a row: 43 us at 64 atoms and 627 us at 45 atoms with six primitives,
// however few pairs there are.  With one basis on every atom a pair whose bound
// U = sum |S_ab| p^(1/4) >= Q, times the largest U of any pair (the one at distance zero), is
// below tau can never be significant: its Q is left at zero (most pairs of a sparse system).
// Also the pair's bucket (Q band, spatial cell of its centre).
template <int TP>
__global__ __launch_bounds__(256) void k_pair_q(Basis b, DevHeader *__restrict__ hdr, int64_t n, double tau,
                                                const double *__restrict__ xyz, double *__restrict__ qout,
                                                int *__restrict__ bucket)
{
    constexpr int PB = 256 / TP;
    extern __shared__ __attribute__((aligned(16))) double sm[];
    __shared__ double red[256];
    const int l = threadIdx.x % TP, pb = threadIdx.x / TP;
    double *tab = sm + (size_t)pb * 3 * b.g2;
    const int64_t npair = n * (n + 1) / 2;
    const int64_t p = (int64_t)blockIdx.x * PB + pb;
    const bool live = p < npair;
    double r2 = 0.0, u = 0.0, u0 = 0.0;
    int64_t i = 0, j = 0;
    if (live) {
        pair_of_index(p, i, j);
        const double dx = xyz[3 * i] - xyz[3 * j], dy = xyz[3 * i + 1] - xyz[3 * j + 1],
                     dz = xyz[3 * i + 2] - xyz[3 * j + 2];
        r2 = dx * dx + dy * dy + dz * dz;
        for (int ab = l; ab < b.g2; ab += TP) pair_q_entry(b, i, j, ab, r2, tab, &u, &u0);
    }
#pragma unroll
    for (int w = TP / 2; w > 0; w >>= 1) {
        u += __shfl_xor(u, w, TP);
        u0 += __shfl_xor(u0, w, TP);
    }
    __syncthreads();
    double s = live && (b.aexp || !(u * u0 < tau)) ? pair_q_sum(b.g2, r2, l, TP, tab) : 0.0;
#pragma unroll
    for (int w = TP / 2; w > 0; w >>= 1) s += __shfl_xor(s, w, TP);
    const double q = sqrt(s);
    if (live && l == 0) {
        qout[p] = q;
        const double c[3] = {0.5 * (xyz[3 * i] + xyz[3 * j]), 0.5 * (xyz[3 * i + 1] + xyz[3 * j + 1]),
                             0.5 * (xyz[3 * i + 2] + xyz[3 * j + 2])};
        bucket[p] = q_band(q) * kNumCells + morton_cell(c, hdr);
    }
    // block max, then one atomic per block (positive doubles order like their bit patterns)
    red[threadIdx.x] = live ? q : 0.0;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (threadIdx.x < w) red[threadIdx.x] = fmax(red[threadIdx.x], red[threadIdx.x + w]);
        __syncthreads();
    }
    if (threadIdx.x == 0 && red[0] > 0.0)
        atomicMax(&hdr->qmax_bits, (unsigned long long)__double_as_longlong(red[0]));
}

template <int TP>
static void launch_pair_q(const Basis &b, DevHeader *hdr, int64_t n, double tau, const double *xyz, double *q,
                          int *bucket, hipStream_t st)
{
    constexpr int PB = 256 / TP;
    const int64_t np = n * (n + 1) / 2;
    hipLaunchKernelGGL((k_pair_q<TP>), dim3((unsigned)((np + PB - 1) / PB)), dim3(256),
                       sizeof(double) * 3 * (size_t)b.g2 * PB, st, b, hdr, n, tau, xyz, q, bucket);
}

// Counts the significant pairs of every bucket; the others' bucket becomes -1.
__global__ __launch_bounds__(256) void k_bucket_count(int64_t npair, double tau, const DevHeader *__restrict__ hdr,
                                                      const double *__restrict__ q, int *__restrict__ bucket_of,
                                                      long long *__restrict__ cnt)
{
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= npair) return;
    const double qmax = __longlong_as_double((long long)hdr->qmax_bits);
    const double qp = q[p];
    if (qp * qmax >= tau && qp > 0.0)
        atomicAdd((unsigned long long *)&cnt[bucket_of[p]], 1ULL);
    else
        bucket_of[p] = -1;
}

// Bucket offsets -> cursors (int) and the significant-pair total.
__global__ __launch_bounds__(256) void k_bucket_cursors(const long long *__restrict__ off, int *__restrict__ cur,
                                                        DevHeader *__restrict__ hdr)
{
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b < kNumBuckets) cur[b] = (int)off[b];
    if (b == 0) hdr->sig_pairs = (int)off[kNumBuckets];
}

// Writes the tables of every significant pair at its position x, holding pair slot[x]: atoms, Q,
// D_kl, the ket table {Px, Py, Pz, S, |P|^2} centred on the centroid (see KetTable) and the
// bra rows, for the precision of the build.  One thread per (position, primitive pair): the
// grid's y dimension is the primitive pair, so the table rows are written coalesced and the
// exponentials of a pair run side by side (one thread per pair took 24 us at 64 atoms and
// 81 us with six primitives).  With per-atom bases (bip != NULL) the ket table gains
// kTswitch / p as its last value and bip receives it per bra primitive pair: the two add up to kTswitch / rho of the quartet.  The 64
// positions after the last pair are padded with harmless entries (atom 0, zero weight, centres
// 1e6 bohr away), so that lanes past the last pair, or lanes pointed at the first pad entry,
// read defined memory and land in the far branch with a zero integral.  A wave also leaves the
// maximum of its 64 positions' term exponents, a workgroup that of its 256.
struct PairTables {
    const int *slot;
    int *posof;         // [npair] position of every significant pair
    int *pk, *pl;
    double *pq, *pd;
    double *prim;
    float *prim_f;
    double *bra;
    float *bra_f;
    double *bip;
    float *bip_f;
    double *kmu, *kfa;
    double *bgw;
    float *bgw_f;
    short *bexp;        // [g2][pcap]
    int *kexp64;        // [positions / 64][g2]
    int *kexp256;       // [positions / 256][g2]
    double *jzero;      // ket vectors to clear, [jcopies][pcap]
    int jcopies;
};
template <typename R>
__global__ __launch_bounds__(256) void k_pair_tables(Basis b, const BasisDev *__restrict__ bd,
                                                     const DevHeader *__restrict__ hdr, int64_t pcap,
                                                     const double *__restrict__ xyz, const double *__restrict__ dens,
                                                     const double *__restrict__ q, int64_t n, PairTables T)
{
    constexpr bool kDouble = sizeof(R) == 8;
    const int S = hdr->sig_pairs;
    const int64_t at = (int64_t)blockIdx.x * 256;
    if (at >= (int64_t)S + 64) return;
    const int64_t pos = at + threadIdx.x;
    const int g2 = b.g2, ab = blockIdx.y;
    R *prim = kDouble ? (R *)T.prim : (R *)T.prim_f;
    R *bra = kDouble ? (R *)T.bra : (R *)T.bra_f;
    R *bip = kDouble ? (R *)T.bip : (R *)T.bip_f;
    R *bgw = kDouble ? (R *)T.bgw : (R *)T.bgw_f;
    int e = kTermNever;
    if (pos < S) {
        const int64_t p = T.slot[pos];
        int64_t i, j;
        pair_of_index(p, i, j);
        const double c0 = hdr->centroid[0], c1 = hdr->centroid[1], c2 = hdr->centroid[2];
        const double A[3] = {xyz[3 * i] - c0, xyz[3 * i + 1] - c1, xyz[3 * i + 2] - c2};
        const double B[3] = {xyz[3 * j] - c0, xyz[3 * j + 1] - c1, xyz[3 * j + 2] - c2};
        const PrimPair w = prim_pair(b, bd, i, j, ab, A, B);
        const double px = w.x, py = w.y, pz = w.z, ps = w.S, mu = w.mu, fa = w.fa, p_ab = w.p, ab2 = w.ab2;
        const double p2 = px * px + py * py + pz * pz;
        if (ab == 0) {
            T.pk[pos] = (int)i;
            T.pl[pos] = (int)j;
            T.pq[pos] = q[p];
            T.pd[pos] = dens[i * n + j];
            T.posof[p] = (int)pos;
            for (int c = 0; c < T.jcopies; ++c) T.jzero[(int64_t)c * pcap + pos] = 0.0;
        }
        if (bip)
            KetTable<R, kDouble, true>::store(prim, pcap, ab, pos, (R)px, (R)py, (R)pz, (R)ps, (R)p2,
                                              (R)(kTswitch / p_ab));
        else
            KetTable<R, kDouble, false>::store(prim, pcap, ab, pos, (R)px, (R)py, (R)pz, (R)ps, (R)p2, (R)0);
        R *ba = bra + (pos * g2 + ab) * 8;
        ba[0] = (R)px; ba[1] = (R)py; ba[2] = (R)pz; ba[3] = (R)ps;
        ba[4] = (R)(-2.0 * px); ba[5] = (R)(-2.0 * py); ba[6] = (R)(-2.0 * pz); ba[7] = (R)p2;
        if (bip) bip[pos * g2 + ab] = (R)(kTswitch / p_ab);
        if (T.kmu) {
            // per-atom gradient: mu and a/p of every ket primitive pair
            T.kmu[(int64_t)ab * pcap + pos] = mu;
            T.kfa[(int64_t)ab * pcap + pos] = fa;
        }
        if (bgw) {
            // gradient: the bra weights mu S, fa S, fb S, fa fb S, fb^2 S of every primitive pair
            const double fbw = b.aexp ? 1.0 - fa : w.fb;
            const double row[kGW] = {mu * ps, fa * ps, fbw * ps, fa * fbw * ps, fbw * fbw * ps, 0.0, 0.0, 0.0};
            R *bw = bgw + (pos * g2 + ab) * kGW;
            for (int c = 0; c < kGW; ++c) bw[c] = (R)row[c];
        }
        e = term_exponent(term_bound(ps, p_ab, mu, sqrt(ab2), bgw != nullptr));
        T.bexp[(int64_t)ab * pcap + pos] = (short)e;
    } else if (pos < (int64_t)S + 64) {
        if (ab == 0) {
            T.pk[pos] = 0;
            T.pl[pos] = 0;
            T.pq[pos] = 0.0;
            T.pd[pos] = 0.0;
        }
        // kTswitch / p = 1: the switch radius stays far below the pad distance
        if (bip)
            KetTable<R, kDouble, true>::store(prim, pcap, ab, pos, (R)1e6, (R)1e6, (R)1e6, (R)0, (R)3e12, (R)1);
        else
            KetTable<R, kDouble, false>::store(prim, pcap, ab, pos, (R)1e6, (R)1e6, (R)1e6, (R)0, (R)3e12, (R)1);
        if (T.kmu) {
            T.kmu[(int64_t)ab * pcap + pos] = 0.0;
            T.kfa[(int64_t)ab * pcap + pos] = 0.0;
        }
    }
    __shared__ int emax[4];
    e = wave_max(e);
    if (threadIdx.x % 64 == 0) {
        emax[threadIdx.x / 64] = e;
        T.kexp64[(pos / 64) * g2 + ab] = e;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < 4; ++w) e = emax[w] > e ? emax[w] : e;
        T.kexp256[(int64_t)blockIdx.x * g2 + ab] = e;
    }
}

// New density on prepared tables: D_kl of every pair, and the accumulators of a build cleared.
__global__ __launch_bounds__(256) void k_new_density(DevHeader *__restrict__ hdr, int64_t n, int64_t pcap,
                                                     const double *__restrict__ dens, const int *__restrict__ pk,
                                                     const int *__restrict__ pl, double *__restrict__ pd,
                                                     double *__restrict__ fzero, int64_t nf,
                                                     double *__restrict__ jzero, int jcopies)
{
    const int64_t at = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, step = (int64_t)gridDim.x * blockDim.x;
    if (at == 0) {
        hdr->next_block = 0;
    }
    const int S = hdr->sig_pairs;
    for (int64_t x = at; x < nf; x += step) fzero[x] = 0.0;
    for (int64_t t = at; t < S; t += step) {
        pd[t] = dens[(int64_t)pk[t] * n + pl[t]];
        for (int c = 0; c < jcopies; ++c) jzero[(int64_t)c * pcap + t] = 0.0;
    }
}

// Order, ket ranges, items and blocks of a small system in one workgroup.  The general path
// counts 2^19 buckets through global memory and scans three times (twelve launches, 4 to 5 us
// each); here the buckets (kSmallBands bands, the last one open-ended, times kSmallCells cells:
// the top bits of the Morton code) are counted in LDS, and everything up to the block offsets
// follows from there.  Sixteen pairs a thread at most.
constexpr int kSmallThreads = 1024, kSmallPer = 16;
constexpr int64_t kSmallPairs = (int64_t)kSmallThreads * kSmallPer;
constexpr int kSmallBands = 24, kSmallCells = 512, kSmallBuckets = kSmallBands * kSmallCells;
static_assert(kSmallBuckets % kSmallThreads == 0, "whole bucket runs per thread");

// Exclusive prefix over the workgroup of one value per thread; total to every thread.
__device__ inline long long block_scan_1024(long long v, long long *__restrict__ wsum, long long &total)
{
    const int t = threadIdx.x, lane = t % kWave, wave = t / kWave;
    long long x = v;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const long long y = __shfl_up(x, o, kWave);
        if (lane >= o) x += y;
    }
    if (lane == kWave - 1) wsum[wave] = x;
    __syncthreads();
    long long before = 0;
    total = 0;
    for (int w = 0; w < kSmallThreads / kWave; ++w) {
        if (w < wave) before += wsum[w];
        total += wsum[w];
    }
    __syncthreads();
    return before + x - v;
}

__global__ __launch_bounds__(kSmallThreads) void k_order_small(
    DevHeader *__restrict__ hdr, int64_t n, double tau, const double *__restrict__ q, int *__restrict__ posof, int *__restrict__ slot, int item_kets, int gshift, int tile,
    int64_t ngroups, int *__restrict__ lims, long long *__restrict__ item_off, long long *__restrict__ goff)
{
    __shared__ int hist[kSmallBuckets];
    __shared__ int band_at[kSmallBands + 1];
    __shared__ long long wsum[kSmallThreads / kWave];
    __shared__ int gmax[kSmallPairs / kMinGroupBras + 1];
    const int t = threadIdx.x;
    const int npair = (int)(n * (n + 1) / 2);
    const double qmax = __longlong_as_double((long long)hdr->qmax_bits);
    for (int x = t; x < kSmallBuckets; x += kSmallThreads) hist[x] = 0;
    for (int64_t x = t; x < ngroups; x += kSmallThreads) gmax[x] = 0;
    __syncthreads();
    int bk[kSmallPer];
#pragma unroll
    for (int r = 0; r < kSmallPer; ++r) {
        const int p = r * kSmallThreads + t;
        bk[r] = -1;
        if (p < npair) {
            const double qp = q[p];
            const int b = posof[p], band = b / kNumCells, cell = b % kNumCells / (kNumCells / kSmallCells);
            if (qp * qmax >= tau && qp > 0.0) {
                bk[r] = (band < kSmallBands - 1 ? band : kSmallBands - 1) * kSmallCells + cell;
                atomicAdd(&hist[bk[r]], 1);
            } else {
                posof[p] = -1;
            }
        }
    }
    __syncthreads();
    // bucket offsets
    constexpr int kPer = kSmallBuckets / kSmallThreads;
    long long total;
    {
        int own[kPer], sum = 0;
        for (int x = 0; x < kPer; ++x) {
            own[x] = hist[t * kPer + x];
            sum += own[x];
        }
        int run = (int)block_scan_1024(sum, wsum, total);
        for (int x = 0; x < kPer; ++x) {
            hist[t * kPer + x] = run;
            if ((t * kPer + x) % kSmallCells == 0) band_at[(t * kPer + x) / kSmallCells] = run;
            run += own[x];
        }
        if (t == 0) band_at[kSmallBands] = (int)total;
    }
    __syncthreads();
    const int S = (int)total;
    // positions (order within a bucket as the cursor hands out places)
#pragma unroll
    for (int r = 0; r < kSmallPer; ++r)
        if (bk[r] >= 0) slot[atomicAdd(&hist[bk[r]], 1)] = r * kSmallThreads + t;
    __threadfence_block();
    __syncthreads();
    // ket ranges: consecutive bras per thread, so that the item offsets are one more scan
    const int per = (S + kSmallThreads - 1) / kSmallThreads;
    long long mine = 0;
    for (int x = 0; x < per; ++x) {
        const int s = t * per + x;
        if (s >= S) break;
        const double thr = tau / q[slot[s]];
        int bend = S;
        if (thr > 0.0) {
            // the band of the threshold finishes with the lane-level test; the first band and
            // the last one are open-ended
            const int bt = q_band(thr);
            bend = bt >= kSmallBands - 1 ? S : band_at[bt + 1];
        }
        const int lim = bend < s + 1 ? bend : s + 1;
        lims[s] = lim;
        const int ni = (lim + item_kets - 1) / item_kets;
        mine += ni;
        atomicMax(&gmax[s >> gshift], (ni + tile - 1) / tile);
    }
    long long items;
    long long run = block_scan_1024(mine, wsum, items);
    for (int x = 0; x < per; ++x) {
        const int s = t * per + x;
        if (s >= S) break;
        item_off[s] = run;
        run += (lims[s] + item_kets - 1) / item_kets;
    }
    __syncthreads();
    if (t == 0) {
        item_off[S] = items;
        long long nb = 0;
        for (int64_t x = 0; x < ngroups; ++x) {
            goff[x] = nb;
            const long long left = S - (x << gshift), gb = 1LL << gshift;
            nb += gmax[x] * (left < 0 ? 0 : (left < gb ? left : gb));
        }
        goff[ngroups] = nb;
        hdr->sig_pairs = S;
        hdr->items = items;
        hdr->blocks = nb;
    }
}

// Fixed pair order (deterministic strategy): every significant pair's index into its
// bucket's range (in any order), then each bucket's range sorted by pair index, so the
// bucketed order is a function of the inputs alone.
__global__ __launch_bounds__(256) void k_slot_fill(int64_t npair, const int *__restrict__ bucket_of,
                                                   int *__restrict__ cur, int *__restrict__ slot)
{
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= npair) return;
    const int bk = bucket_of[p];
    if (bk >= 0) slot[atomicAdd(&cur[bk], 1)] = (int)p;
}

__global__ __launch_bounds__(256) void k_bucket_max(const long long *__restrict__ off, DevHeader *__restrict__ hdr)
{
    __shared__ int red[256];
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    red[threadIdx.x] = b < kNumBuckets ? (int)(off[b + 1] - off[b]) : 0;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (threadIdx.x < w) red[threadIdx.x] = max(red[threadIdx.x], red[threadIdx.x + w]);
        __syncthreads();
    }
    if (threadIdx.x == 0) atomicMax(&hdr->max_bucket, red[0]);
}

__global__ __launch_bounds__(256) void k_slot_sort(const long long *__restrict__ off, int *__restrict__ slot)
{
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= kNumBuckets) return;
    const long long lo = off[b], hi = off[b + 1];
    // insertion sort of one bucket (buckets hold tens of pairs)
    for (long long x = lo + 1; x < hi; ++x) {
        const int v = slot[x];
        long long y = x - 1;
        while (y >= lo && slot[y] > v) {
            slot[y + 1] = slot[y];
            --y;
        }
        slot[y + 1] = v;
    }
}

// Ket range of every bra s (in bucketed order): kets t < lim_s with
// lim_s = min(s + 1, end of the band holding tau / Q_s); items of item_kets kets.
__global__ __launch_bounds__(256) void k_limits(const DevHeader *__restrict__ hdr, double tau,
                                                const double *__restrict__ pq,
                                                const long long *__restrict__ boff,
                                                long long *__restrict__ nitems, int *__restrict__ lims,
                                                int64_t pcap, int item_kets)
{
    const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t S = hdr->sig_pairs;
    if (s >= pcap) return;
    long long ni = 0;
    if (s < S) {
        const double thr = tau / pq[s];
        int64_t bend;
        if (thr <= 0.0) {
            bend = S;
        } else {
            // band 0 is open-ended (every Q above its lower edge), so a threshold above the
            // largest band edge still lands there; the lane-level test finishes the job
            const int bt = q_band(thr);
            bend = bt + 1 >= kNumBands ? S : boff[(bt + 1) * kNumCells];
        }
        const int64_t lim = bend < s + 1 ? bend : s + 1;
        ni = (lim + item_kets - 1) / item_kets;
        lims[s] = (int)lim;
    } else {
        lims[s] = 0;
    }
    nitems[s] = ni;
}

// ------------------------------------------------------------------ exclusive scan (int64)

constexpr int kScanBlock = 1024;

__global__ __launch_bounds__(kScanBlock) void k_scan_reduce(const long long *__restrict__ in, int64_t m,
                                                            long long *__restrict__ bsum)
{
    __shared__ long long red[kScanBlock];
    const int64_t i = (int64_t)blockIdx.x * kScanBlock + threadIdx.x;
    red[threadIdx.x] = i < m ? in[i] : 0;
    __syncthreads();
    for (int w = kScanBlock / 2; w > 0; w >>= 1) {
        if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) bsum[blockIdx.x] = red[0];
}

// Exclusive scan of the block sums in one block (nb <= 1024 * 16).
__global__ __launch_bounds__(kScanBlock) void k_scan_blocks(long long *__restrict__ bsum, int nb)
{
    __shared__ long long part[kScanBlock];
    const int t = threadIdx.x;
    const int per = (nb + kScanBlock - 1) / kScanBlock;
    long long s = 0;
    for (int i = 0; i < per; ++i) {
        const int x = t * per + i;
        if (x < nb) s += bsum[x];
    }
    part[t] = s;
    __syncthreads();
    for (int w = 1; w < kScanBlock; w <<= 1) {
        long long v = (t >= w) ? part[t - w] : 0;
        __syncthreads();
        part[t] += v;
        __syncthreads();
    }
    long long run = part[t] - s;
    for (int i = 0; i < per; ++i) {
        const int x = t * per + i;
        if (x < nb) {
            const long long v = bsum[x];
            bsum[x] = run;
            run += v;
        }
    }
}

__global__ __launch_bounds__(kScanBlock) void k_scan_final(const long long *__restrict__ in, int64_t m,
                                                           const long long *__restrict__ bsum,
                                                           long long *__restrict__ out,
                                                           long long *__restrict__ total)
{
    __shared__ long long part[kScanBlock];
    const int t = threadIdx.x;
    const int64_t i = (int64_t)blockIdx.x * kScanBlock + t;
    const long long v = i < m ? in[i] : 0;
    part[t] = v;
    __syncthreads();
    for (int w = 1; w < kScanBlock; w <<= 1) {
        long long u = (t >= w) ? part[t - w] : 0;
        __syncthreads();
        part[t] += u;
        __syncthreads();
    }
    const long long excl = bsum[blockIdx.x] + part[t] - v;
    if (i < m) out[i] = excl;
    if (i == m - 1) {
        out[m] = excl + v;
        if (total) *total = excl + v;
    }
}

hipError_t launch_scan(const long long *in, int64_t m, long long *out, long long *tmp, long long *total,
                       hipStream_t st)
{
    const int nb = (int)((m + kScanBlock - 1) / kScanBlock);
    hipLaunchKernelGGL(k_scan_reduce, dim3(nb), dim3(kScanBlock), 0, st, in, m, tmp);
    hipLaunchKernelGGL(k_scan_blocks, dim3(1), dim3(kScanBlock), 0, st, tmp, nb);
    hipLaunchKernelGGL(k_scan_final, dim3(nb), dim3(kScanBlock), 0, st, in, m, tmp, out, total);
    return hipGetLastError();
}

// ------------------------------------------------------------------ debug check of the density

__global__ void k_dchk_reset(DevHeader *hdr)
{
    hdr->dchk_asym = 0;
    hdr->dchk_max = 0;
    hdr->dchk_ratio = 0;
    hdr->dchk_bad = 0;
    hdr->dchk_mol = 0x7fffffff;
    hdr->dchk_badmol = 0x7fffffff;
}

// Non-negative doubles order like their bit patterns, so atomicMax on the patterns is a max.
__device__ inline void atomic_max_nonneg(unsigned long long *p, double v)
{
    atomicMax(p, (unsigned long long)__double_as_longlong(v));
}

// One matrix, any size: grid-stride over its entries, block maxima, then atomics.
__global__ __launch_bounds__(256) void k_dens_check(int64_t n, const double *__restrict__ D,
                                                    DevHeader *__restrict__ hdr)
{
    __shared__ double ra[256], rm[256];
    __shared__ unsigned long long rb[256];
    double asym = 0.0, mx = 0.0;
    unsigned long long bad = 0;
    const int64_t n2 = n * n;
    for (int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; x < n2; x += (int64_t)gridDim.x * blockDim.x) {
        const int64_t i = x / n, j = x - i * n;
        const double v = D[x];
        if (!isfinite(v)) {
            ++bad;
            continue;
        }
        mx = fmax(mx, fabs(v));
        const double w = D[j * n + i];
        if (isfinite(w)) asym = fmax(asym, fabs(v - w));
    }
    ra[threadIdx.x] = asym;
    rm[threadIdx.x] = mx;
    rb[threadIdx.x] = bad;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (threadIdx.x < w) {
            ra[threadIdx.x] = fmax(ra[threadIdx.x], ra[threadIdx.x + w]);
            rm[threadIdx.x] = fmax(rm[threadIdx.x], rm[threadIdx.x + w]);
            rb[threadIdx.x] += rb[threadIdx.x + w];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        atomic_max_nonneg(&hdr->dchk_asym, ra[0]);
        atomic_max_nonneg(&hdr->dchk_max, rm[0]);
        if (rb[0]) atomicAdd(&hdr->dchk_bad, rb[0]);
    }
}

// Many small matrices: one block per molecule (grid-stride over molecules), each judged
// against tol times its own largest entry.
__global__ __launch_bounds__(256) void k_dens_check_batched(int64_t nmol, const long long *__restrict__ doff,
                                                            const int *__restrict__ nmv,
                                                            const double *__restrict__ D, double tol,
                                                            DevHeader *__restrict__ hdr)
{
    __shared__ double ra[256], rm[256];
    __shared__ unsigned long long rb[256];
    for (int64_t m = blockIdx.x; m < nmol; m += gridDim.x) {
        const int64_t n = nmv[m];
        const double *Dm = D + doff[m];
        double asym = 0.0, mx = 0.0;
        unsigned long long bad = 0;
        for (int64_t x = threadIdx.x; x < n * n; x += blockDim.x) {
            const int64_t i = x / n, j = x - i * n;
            const double v = Dm[x];
            if (!isfinite(v)) {
                ++bad;
                continue;
            }
            mx = fmax(mx, fabs(v));
            const double w = Dm[j * n + i];
            if (isfinite(w)) asym = fmax(asym, fabs(v - w));
        }
        ra[threadIdx.x] = asym;
        rm[threadIdx.x] = mx;
        rb[threadIdx.x] = bad;
        __syncthreads();
        for (int w = 128; w > 0; w >>= 1) {
            if (threadIdx.x < w) {
                ra[threadIdx.x] = fmax(ra[threadIdx.x], ra[threadIdx.x + w]);
                rm[threadIdx.x] = fmax(rm[threadIdx.x], rm[threadIdx.x + w]);
                rb[threadIdx.x] += rb[threadIdx.x + w];
            }
            __syncthreads();
        }
        if (threadIdx.x == 0) {
            if (rb[0]) {
                atomicAdd(&hdr->dchk_bad, rb[0]);
                atomicMin(&hdr->dchk_badmol, (int)m);
            }
            const double a = ra[0], b = rm[0];
            if (a > tol * b) {
                atomicMin(&hdr->dchk_mol, (int)m);
                atomic_max_nonneg(&hdr->dchk_ratio, b > 0.0 ? a / b : a);
            }
        }
        __syncthreads();
    }
}

hipError_t launch_dens_check(DevHeader *hdr, int64_t n, const double *dens, hipStream_t st)
{
    hipLaunchKernelGGL(k_dchk_reset, dim3(1), dim3(1), 0, st, hdr);
    const int64_t nb = (n * n + 255) / 256;
    hipLaunchKernelGGL(k_dens_check, dim3((unsigned)(nb < 4096 ? nb : 4096)), dim3(256), 0, st, n, dens, hdr);
    return hipGetLastError();
}

hipError_t launch_dens_check_batched(DevHeader *hdr, int64_t nmol, const long long *mol_doff, const int *mol_n,
                                     const double *dens, double tol, hipStream_t st)
{
    hipLaunchKernelGGL(k_dchk_reset, dim3(1), dim3(1), 0, st, hdr);
    hipLaunchKernelGGL(k_dens_check_batched, dim3((unsigned)(nmol < 4096 ? nmol : 4096)), dim3(256), 0, st, nmol,
                       mol_doff, mol_n, dens, tol, hdr);
    return hipGetLastError();
}

// Blocks of every bra group: its bras (2^gshift, or what is left in the last one) times the
// largest block count among them (bras with fewer blocks leave empty slots, skipped by the
// kernels).
// One workgroup per group of bras: the largest block count of its bras (a block-wide max).
__global__ __launch_bounds__(256) void k_group_blocks(const DevHeader *__restrict__ hdr,
                                                      const long long *__restrict__ nitems, int64_t ngroups,
                                                      int gshift, int tile, long long *__restrict__ gcnt)
{
    __shared__ long long red[256];
    const int64_t g = blockIdx.x;   // the grid is exactly ngroups workgroups
    const int tid = threadIdx.x;
    const int64_t S = hdr->sig_pairs;
    const int64_t gb = (int64_t)1 << gshift;
    long long nb = 0;
    for (int64_t s = g * gb + tid; s < (g + 1) * gb && s < S; s += blockDim.x) {
        const long long b = (nitems[s] + tile - 1) / tile;
        nb = b > nb ? b : nb;
    }
    red[tid] = nb;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (tid < w) red[tid] = red[tid + w] > red[tid] ? red[tid + w] : red[tid];
        __syncthreads();
    }
    if (tid == 0) gcnt[g] = red[0] * (S - g * gb < gb ? S - g * gb : gb);
}

hipError_t launch_pairs(const Layout &L, const Basis &b, char *ws, const double *xyz, const double *dens,
                        double tau, int prec, const PairPlan &plan, hipStream_t st)
{
    DevHeader *hdr = (DevHeader *)(ws + L.hdr);
    BasisDev *bd = (BasisDev *)(ws + L.basis);
    const int64_t np = L.npair;
    const int bs = 256;
    const unsigned nbp = (unsigned)((np + bs - 1) / bs);
    long long *cnt = (long long *)(ws + L.bucket_cnt);
    long long *off = (long long *)(ws + L.bucket_off);
    int *cur = (int *)(ws + L.bucket_cur);
    double *q = (double *)(ws + L.q_unsorted);
    int *posof = (int *)(ws + L.bucket_of);
    const bool small = np <= kSmallPairs && !plan.fixed_order;
    const int ikets = item_kets(L);
    hipError_t e = launch_prep_begin(b, bd, hdr, L.n, xyz, plan.info, plan.fzero, plan.nf, cnt,
                                     small ? 0 : (int64_t)kNumBuckets, st);
    if (e != hipSuccess) return e;
    // lanes per pair: about three primitive quartets each
    switch (b.g) {
    case 1: launch_pair_q<1>(b, hdr, L.n, tau, xyz, q, posof, st); break;
    case 2: launch_pair_q<4>(b, hdr, L.n, tau, xyz, q, posof, st); break;
    case 3: launch_pair_q<16>(b, hdr, L.n, tau, xyz, q, posof, st); break;
    default: launch_pair_q<64>(b, hdr, L.n, tau, xyz, q, posof, st); break;
    }
    // the pair of every position (the item counts' storage is free until the limits are computed)
    int *slot = (int *)(ws + L.nitems);
    if (small) {
        hipLaunchKernelGGL(k_order_small, dim3(1), dim3(kSmallThreads), 0, st, hdr, L.n, tau, (const double *)q, posof, slot, ikets, L.gshift, L.tile, L.ngroups,
                           (int *)(ws + L.lim), (long long *)(ws + L.item_off), (long long *)(ws + L.goff));
    } else {
        hipLaunchKernelGGL(k_bucket_count, dim3(nbp), dim3(bs), 0, st, np, tau, hdr, (const double *)q, posof, cnt);
        e = launch_scan(cnt, kNumBuckets, off, (long long *)(ws + L.scan_tmp), nullptr, st);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(k_bucket_cursors, dim3((kNumBuckets + 255) / 256), dim3(256), 0, st, off, cur, hdr);
        if (plan.fixed_order) {
            hipLaunchKernelGGL(k_bucket_max, dim3((kNumBuckets + 255) / 256), dim3(256), 0, st, off, hdr);
            int hmax = 0;
            e = hipMemcpyAsync(&hmax, &hdr->max_bucket, sizeof(int), hipMemcpyDeviceToHost, st);
            if (e == hipSuccess) e = hipStreamSynchronize(st);
            if (e != hipSuccess) return e;
            if (hmax > kMaxFixedBucket) return hipErrorNotSupported;
        }
        hipLaunchKernelGGL(k_slot_fill, dim3(nbp), dim3(bs), 0, st, np, (const int *)posof, cur, slot);
        if (plan.fixed_order)
            hipLaunchKernelGGL(k_slot_sort, dim3((kNumBuckets + 255) / 256), dim3(256), 0, st, off, slot);
    }
    PairTables T;
    memset(&T, 0, sizeof(T));
    T.slot = slot;
    T.posof = posof;
    T.pk = (int *)(ws + L.pk);
    T.pl = (int *)(ws + L.pl);
    T.pq = (double *)(ws + L.pq);
    T.pd = (double *)(ws + L.pd);
    T.prim = (double *)(ws + L.prim);
    T.prim_f = (float *)(ws + L.prim_f);
    T.bra = (double *)(ws + L.bra);
    T.bra_f = (float *)(ws + L.bra_f);
    if (L.atoms) {
        T.bip = (double *)(ws + L.bip);
        T.bip_f = (float *)(ws + L.bip_f);
    }
    if (L.pmu) {
        T.kmu = (double *)(ws + L.pmu);
        T.kfa = (double *)(ws + L.pfa);
    }
    if (L.bgw) {
        T.bgw = (double *)(ws + L.bgw);
        T.bgw_f = (float *)(ws + L.bgw_f);
    }
    T.bexp = (short *)(ws + L.bexp);
    T.kexp64 = (int *)(ws + L.kexp64);
    T.kexp256 = (int *)(ws + L.kexp256);
    T.jzero = plan.jzero;
    T.jcopies = plan.jcopies;
    // np + 64 positions at most (64 pads after the last pair)
    const dim3 grid((unsigned)((np + 64 + 255) / 256), (unsigned)L.g2);
    if (prec == HFK_MIXED)
        hipLaunchKernelGGL((k_pair_tables<float>), grid, dim3(256), 0, st, b, (const BasisDev *)bd, hdr, L.pcap, xyz,
                           dens, (const double *)q, L.n, T);
    else
        hipLaunchKernelGGL((k_pair_tables<double>), grid, dim3(256), 0, st, b, (const BasisDev *)bd, hdr, L.pcap, xyz,
                           dens, (const double *)q, L.n, T);
    if (small) return hipGetLastError();
    hipLaunchKernelGGL(k_limits, dim3((unsigned)((L.pcap + 255) / 256)), dim3(256), 0, st, hdr, tau,
                       (const double *)(ws + L.pq), off, (long long *)(ws + L.nitems), (int *)(ws + L.lim),
                       L.pcap, ikets);
    e = launch_scan((const long long *)(ws + L.nitems), L.pcap, (long long *)(ws + L.item_off),
                    (long long *)(ws + L.scan_tmp), &hdr->items, st);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_group_blocks, dim3((unsigned)L.ngroups), dim3(256), 0, st, hdr,
                       (const long long *)(ws + L.nitems), L.ngroups, L.gshift, L.tile, (long long *)(ws + L.gcnt));
    return launch_scan((const long long *)(ws + L.gcnt), L.ngroups, (long long *)(ws + L.goff),
                       (long long *)(ws + L.scan_tmp), &hdr->blocks, st);
}

hipError_t launch_new_density(const Layout &L, char *ws, const double *dens, const PairPlan &plan, hipStream_t st)
{
    const int64_t work = plan.nf > L.npair ? plan.nf : L.npair;
    const int64_t nb = (work + 255) / 256;
    hipLaunchKernelGGL(k_new_density, dim3((unsigned)(nb < 2048 ? nb : 2048)), dim3(256), 0, st,
                       (DevHeader *)(ws + L.hdr), L.n, L.pcap, dens, (const int *)(ws + L.pk),
                       (const int *)(ws + L.pl), (double *)(ws + L.pd), plan.fzero, plan.nf, plan.jzero, plan.jcopies);
    return hipGetLastError();
}

}  // namespace hfk
