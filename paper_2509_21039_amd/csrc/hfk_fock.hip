// Forward Fock build on one GPU: the unique-quartet loop with the primitive contraction
// and the six-way scatter of the Hartree--Fock kernel (Background section, kernel
// listing), re-designed for CDNA4.
//
// Work decomposition.  Significant pairs are stored in Q-bucketed order (t = 0 .. S-1),
// so the kets kept by the screen for a bra s form a prefix t < lim_s (t <= s keeps each
// unordered quartet once; a lane-level test Q_s Q_t >= tau handles the partial bucket).
// An item is (bra s, up to four 64-lane chunks of consecutive kets per wave: 1024 kets with four
// waves; one chunk per wave on small systems, and on the smallest one chunk for all four).
// Persistent workgroups fetch blocks of items of one bra from a global counter (the cost per
// item varies with the bra's surroundings, and static ranges left a long tail of slow
// workgroups).  Blocks are numbered ket-block-major within groups of bras (1024 unless tuned),
// so the workgroups running together read the same kets, which then come from L2.  One ket per
// lane; the bra's primitive data are wave-uniform.  In the hybrid form the wave first packs the
// kets that pass the screen (ballot + lane count, order kept so loads stay coalesced) into full
// chunks.
//
// Accumulation (replacing one global FP64 atomic per update):
//   F_ij += 4 D_kl v   per-lane register, reduced across the wave when the bra changes
//   F_kl += 4 D_ij v   coalesced read-modify-write of a per-workgroup vector over kets
//                      (atomics into shared copies when per-workgroup ones exceed the budget)
//   F_ik, F_il, F_jk, F_jl -= ...   LDS atomics into copies of rows i and j of F, flushed
//                      to a per-workgroup copy of F (or with global atomics) once per bra
// and a final kernel sums the copies, symmetrises and forms E2.
//
// Deterministic strategy (kDet): the same arithmetic with every sum taken in a fixed order,
// so repeated builds agree bit for bit.  Blocks are dealt out by a static grid stride
// instead of the global counter and every workgroup owns its copy of F and of the ket
// vector.  Within a workgroup each wave stages its exchange updates (k, l, v) in LDS; at the
// end of every item the waves apply them to rows i and j one wave after the other (a wave's
// atomic adds within one instruction are applied by the LDS in a fixed lane order), and the
// F_ij partial sums of the four waves are added in wave order.  The final kernels sum the
// workgroup copies in workgroup order.
#include "hfk_device.hpp"
#include "hfk_boys.hpp"

namespace hfk {

struct FockArgs {
    const DevHeader *hdr;
    const BasisDev *bd;
    const int *pk;
    const int *pl;
    const double *pq;
    const double *pd;
    const double *prim;
    const float *prim_f;
    const double *bra;
    const float *bra_f;
    const double *bip;          // per-atom bases: [pcap][g2] kTswitch / p of the bra primitive pairs
    const float *bip_f;
    const long long *item_off;
    const long long *goff;      // [ngroups + 1] block offsets of the bra groups
    int64_t ngroups;
    int gshift;                 // log2 of the bras per group
    int tile;                   // items per block
    const int *lim;
    const short *bexp;          // [g2][pcap] term exponents of the bras
    const int *kexp;            // [ket block of a wave][g2] maxima of the kets' exponents
    int sub;                    // 64-ket chunks per wave of an item
    int nsplit;                 // waves that share a chunk's bra primitive pairs
    int last_first;             // blocks from the end of the numbering
    int tlim;                   // term_limit(tau)
    const double *dens;
    double *fpriv;
    double *jcol;       // [jcopies][pcap]
    unsigned long long *quartets;
    unsigned long long *next_block;
    int64_t pcap;
    double tau;
    int n;
    int strategy;
    int jcopies;        // ket vectors: one per workgroup if equal to the grid, else shared (atomics)
};

// Tables of the hybrid form (grid-scaled) and of the direct form.
static __device__ const BoysForward64 kBoys64 = make_boys_forward64();
static __device__ const BoysPlain64 kBoysPlain64 = make_boys_plain64();
static __device__ const BoysFloat kBoys32 = make_boys_float(false);
static __device__ const BoysFloat kBoysPlain32 = make_boys_float(true);

template <typename R> struct Prec;
template <> struct Prec<double> {
    static __device__ const double *boys(bool split) { return split ? kBoys64.v : kBoysPlain64.v; }
    static __device__ const double *prim(const FockArgs &a) { return a.prim; }
    static __device__ const double *bra(const FockArgs &a) { return a.bra; }
    static __device__ const double *bip(const FockArgs &a) { return a.bip; }
    static __device__ const double *rho(const BasisDev *bd) { return bd->rho; }
    static __device__ const double *srho(const BasisDev *bd) { return bd->srho; }
    static __device__ const double *rsn(const BasisDev *bd) { return bd->rsn; }
    static __device__ double rsqrt(double x) { return rsqrt_fp64(x); }
    // The hybrid kernel's FP64 accumulator carries -2 times the sum, which lets the Newton
    // step of the reciprocal square root fold into the product: with the hardware estimate
    // y, y1 = y (3 - x y^2) / 2 and -2 s y1 = (s y) (x y^2 - 3).  The far-field term of a
    // primitive quartet is returned as the two factors a = s y and b = x y^2 - 3 (three
    // operations after rsq; the accumulating FMA makes four), so that near lanes can replace
    // both before the one FMA that adds the term.
    static constexpr double kAccScale = -2.0;
    static __device__ void far_split(double s, double x, double &a, double &b)
    {
        const double y = __builtin_amdgcn_rsq(x);
        a = s * y;
        b = fma(x, y * y, -3.0);
    }
};
template <> struct Prec<float> {
    static __device__ const float *boys(bool split) { return split ? kBoys32.v : kBoysPlain32.v; }
    static __device__ const float *prim(const FockArgs &a) { return a.prim_f; }
    static __device__ const float *bra(const FockArgs &a) { return a.bra_f; }
    static __device__ const float *bip(const FockArgs &a) { return a.bip_f; }
    static __device__ const float *rho(const BasisDev *bd) { return bd->rho_f; }
    static __device__ const float *srho(const BasisDev *bd) { return bd->srho_f; }
    static __device__ const float *rsn(const BasisDev *bd) { return bd->rsn_f; }
    static __device__ float rsqrt(float x) { return rsqrt_fp32(x); }
    static constexpr float kAccScale = 1.0f;   // no Newton step in FP32
    static __device__ void far_split(float s, float x, float &a, float &b) { a = s; b = rsqrt_fp32(x); }
};

// Polynomial of the table row nearest to T (T below the switch, so the row exists).
template <typename R>
__device__ inline R boys_nearest_row(R T, const R *__restrict__ tab)
{
    using BG = BoysGrid<R>;
    const int k = (int)(T * R(BG::inv_h) + R(0.5));
    const R d = T - (R)k * R(BG::h);
    const R *c = tab + k * BG::stride;
    R v = c[BG::order - 1];
#pragma unroll
    for (int m = BG::order - 2; m >= 0; --m) v = v * d + c[m];
    return v;
}

// H(T) = erf(sqrt T)/sqrt T: table row below the switch, T^(-1/2) above it (both
// evaluated, one selected).
template <typename R>
__device__ inline R boys_h(R T, const R *__restrict__ tab)
{
    const R far = Prec<R>::rsqrt(fmax(T, R(1e-30)));
    const R Tc = fmin(T, R(kTswitch + 0.5));
    const R v = boys_nearest_row<R>(Tc, tab);
    return T < R(kTswitch) ? v : far;
}

// The lane's ket primitives are consumed in blocks of G (fixed c, all d), so only G of
// them occupy registers at a time; the bra primitive pair ab runs in the middle loop.

// Contracted (bra | ket) for one lane, every primitive quartet evaluated in place.
// (ab|cd) = S_ab S_cd sqrt(rho) H(rho |P - Q|^2).
template <int G, typename R>
__device__ inline R quartet_eri_direct(const R *__restrict__ lbra, const R *__restrict__ prim, int64_t pcap,
                                       int64_t t, const R *__restrict__ lrs, const R *__restrict__ tab)
{
    constexpr int G2 = G * G;
    R eri = R(0);
#pragma unroll 1
    for (int cb = 0; cb < G; ++cb) {
        R kx[G], ky[G], kz[G], ks[G];
#pragma unroll
        for (int d = 0; d < G; ++d) {
            R q, sw;
            KetTable<R, sizeof(R) == 8, false>::load(prim, pcap, cb * G + d, (unsigned)t, kx[d], ky[d], kz[d], ks[d], q,
                                                     sw);
        }
#pragma unroll 1
        for (int ab = 0; ab < G2; ++ab) {
            const R px = lbra[4 * ab], py = lbra[4 * ab + 1], pz = lbra[4 * ab + 2];
            R acc = R(0);
#pragma unroll
            for (int d = 0; d < G; ++d) {
                const int x = ab * G2 + cb * G + d;
                const R dx = px - kx[d], dy = py - ky[d], dz = pz - kz[d];
                const R r2 = dx * dx + dy * dy + dz * dz;
                const R h = boys_h<R>(r2 * lrs[2 * x], tab);
                acc += (ks[d] * lrs[2 * x + 1]) * h;
            }
            eri += lbra[4 * ab + 3] * acc;
        }
    }
    return eri;
}

// kAccScale sqrt(h) H(T) for a lane below the switch radius (the table is scaled to match).
template <typename R>
__device__ inline R boys_near(R r2, R rsh, const R *__restrict__ tab)
{
    R d;
    const unsigned off = boys_row<R>(r2, rsh, d);
    return boys_eval<R>(tab, off, d);
}

// Contracted (bra | ket), far field first: for one bra primitive pair a lane forms |P-Q|^2
// of its G ket primitive pairs and their far-field terms S_cd / |P-Q| (exact beyond the
// switch radius; the G reciprocal square roots issue back to back); then, under exec masks,
// lanes below the switch radius replace a term by S_cd sqrt(rho/h) * sqrt(h) H(T) from the
// grid table (a wave with no near lane, the common case once kets are spatially sorted, skips
// the table part, and only near lanes read the table from LDS); the terms are added last, in
// one branch-free run of FMAs.  Far values of near lanes (|P-Q|^2 may be zero or round
// below it) are discarded, never added.  Lanes without a kept quartet point at a pad entry
// (centres 1e6 bohr away, zero weight), so they are never near and add nothing.  Uniform data come through scalar loads issued together
// at the top of each bra primitive: (Px, Py, Pz, S, -2Px, -2Py, -2Pz, |P|^2) and, per
// primitive quartet, (switch radius^2, rho/h, sqrt(rho/h)).
// FP64 forms |P-Q|^2 as |P|^2 + |Q|^2 - 2 P.Q (4 operations; with centroid-centred
// coordinates the cancellation stays near 1e-13 bohr^2 absolute); FP32 subtracts the
// centres directly, which its precision needs.  The FP64 accumulator holds -2 times the sum
// (kAccScale; the near-branch table is scaled to match), which saves one operation in each
// Newton step of the reciprocal square root; the result is scaled back once per quartet.
// Per-atom bases (kAtoms): rho = p q / (p + q) differs per quartet, so the scalar combo
// table gives way to kTswitch / p of the bra (uniform, bip) and of the ket (last ket
// component): their sum is kTswitch / rho, the switch radius^2 itself, so the test costs
// one add; only the near branch needs sqrt(rho / h) = sqrt(kTswitch / h) / sqrt(that sum)
// (one reciprocal square root); the far field S_cd / |P-Q| does not depend on rho at all.
// Terms below the term screen (see term_limit) are left out: per row cb the wave forms the
// masks of the bra primitive pairs that still matter (one compare per ket primitive pair
// against the maxima over the wave's kets), walks only those and starts each row's run of
// terms at the first ket primitive pair that matters.  Kets of a wave come from one Q band,
// so they fall away together; a ket primitive pair that no bra primitive pair needs is not
// loaded either.  Measured (same card, without against with the screen): he512 FP64 59.8 ->
// 44.0 ms (44 of 81 terms left), he1024 mixed 195.6 -> 161.1 ms, 2016 atoms at 4 bohr 67.0 ->
// 55.6 ms, H/He 100 1.37 -> 1.08 ms, 45 atoms with six primitives 2.19 -> 1.83 ms.
template <int G, typename R, bool kAtoms = false>
__device__ inline R quartet_eri_hybrid(cptr<R> bra, const R *__restrict__ prim, int64_t pcap, unsigned t,
                                       cptr<R> rsn, const R *__restrict__ tab, int ebra, cptr<int> kexp, int tlim,
                                       cptr<R> bip = nullptr)
{
    constexpr int G2 = G * G;
    constexpr bool kExpand = sizeof(R) == 8;
    using TM = typename TermMask<G>::T;
    // FP32 with up to three primitives loads the next cb's ket data while it works on this one
    // (the kernel has registers to spare: he1024 mixed 209.6 -> 203.2 ms); FP64 would drop from
    // five to four waves per SIMD for it and run slower (he512 67.9 -> 73.5 ms), so it loads
    // each cb at its start
    constexpr bool kPrefetch = sizeof(R) == 4 && G <= 3;
    constexpr int kSlots = kPrefetch ? 2 : 1;
    R eri = R(0);
    R kx[kSlots][G], ky[kSlots][G], kz[kSlots][G], ks[kSlots][G], kq[kSlots][G], kp[kSlots][G];
    TM need[kSlots][G];
    auto load_cb = [&](int cbl, int slot) {
        term_masks<G>(ebra, kexp + cbl * G, tlim, need[slot]);
#pragma unroll
        for (int d = 0; d < G; ++d) {
            // no bra primitive pair reads it (prefetched rows are loaded whole: with a known
            // number of loads in flight the wait for one row leaves the next one's running)
            if (!kPrefetch && G <= 4 && !need[slot][d]) continue;
            KetTable<R, kExpand, kAtoms>::load(prim, pcap, cbl * G + d, t, kx[slot][d], ky[slot][d], kz[slot][d],
                                               ks[slot][d], kq[slot][d], kp[slot][d]);
        }
    };
    constexpr int kCbUnroll = kPrefetch ? G : 1;   // the slots must be compile-time indices
    if constexpr (kPrefetch) load_cb(0, 0);
#pragma unroll kCbUnroll
    for (int cb = 0; cb < G; ++cb) {
        const int cur = kPrefetch ? (cb & 1) : 0;
        if constexpr (kPrefetch) {
            if (cb + 1 < G) load_cb(cb + 1, cur ^ 1);
        } else {
            load_cb(cb, 0);
        }
        for_terms<G>(need[cur], [&](auto nd, int ab) __attribute__((always_inline)) {
            constexpr int D0 = G - decltype(nd)::value;   // first term of the row
            const cptr<R> bp = at_bytes<R>(bra, (unsigned)ab * (8 * sizeof(R)));
            R b[8];
#pragma unroll
            for (int c = 0; c < 8; ++c) b[c] = bp[c];
            R acc = R(0);
            R r2[G], fa[G], fb[G];
            auto far = [&](int d) __attribute__((always_inline)) {
                if (kExpand) {
                    r2[d] = fma(b[4], kx[cur][d], fma(b[5], ky[cur][d], fma(b[6], kz[cur][d], kq[cur][d] + b[7])));
                } else {
                    const R dx = b[0] - kx[cur][d], dy = b[1] - ky[cur][d], dz = b[2] - kz[cur][d];
                    r2[d] = dx * dx + dy * dy + dz * dz;
                }
                Prec<R>::far_split(ks[cur][d], r2[d], fa[d], fb[d]);
            };
            if constexpr (kAtoms) {
                const R bi = bip[ab];
                asm volatile("" ::"s"(bi));
#pragma unroll
                for (int d = D0; d < G; ++d) far(d);
#pragma unroll
                for (int d = D0; d < G; ++d) {
                    const R sw = bi + kp[cur][d];   // kTswitch / rho
                    if (r2[d] < sw) {
                        const R y = rsqrt_r(sw) * R(BoysGrid<R>::sqrt_sw_inv_h);   // sqrt(rho / h)
                        fa[d] = ks[cur][d] * y;
                        fb[d] = boys_near<R>(r2[d], y * y, tab);
                    }
                }
            } else {
                const cptr<R> up = at_bytes<R>(rsn, ((unsigned)ab * G2 + (unsigned)cb * G) * (unsigned)(3 * sizeof(R)));
                R u[3 * G];
#pragma unroll
                for (int c = 3 * D0; c < 3 * G; ++c) u[c] = up[c];
                // keep every uniform load in one batch at the top (not sunk into the branches)
#pragma unroll
                for (int c = 3 * D0; c < 3 * G; ++c) asm volatile("" ::"s"(u[c]));
#pragma unroll
                for (int d = D0; d < G; ++d) far(d);
#pragma unroll
                for (int d = D0; d < G; ++d) {
                    if (r2[d] < u[3 * d]) {
                        fa[d] = ks[cur][d] * u[3 * d + 2];
                        fb[d] = boys_near<R>(r2[d], u[3 * d + 1], tab);
                    }
                }
            }
#pragma unroll
            for (int d = D0; d < G; ++d) acc = fma(fa[d], fb[d], acc);
            eri = fma(b[3], acc, eri);
        });
    }
    return eri * (R(1) / Prec<R>::kAccScale);
}

// LDS carve-up of the quartet kernel (bytes, 16-byte aligned pieces).
template <typename R> struct FockSmem {
    static constexpr int kCombos = kMaxG2 * kMaxG2 / 16;                    // g <= 4 here: 256 combos
    static constexpr size_t tab_bytes = sizeof(R) * BoysGrid<R>::rows * BoysGrid<R>::stride;
    static constexpr size_t uni_bytes = 4 * sizeof(R) * 16 + 2 * sizeof(R) * kCombos;   // bra, (rho, srho)
    // deterministic strategy: per wave, kWaveKets staged updates (v, then k and l)
    static constexpr size_t stage_bytes = kWavesPerGroup * kWaveKets * (sizeof(double) + 2 * sizeof(int));
    // rows i and j of F, and (drows) of D; per wave, the packed kets of the hybrid form
    static size_t total(int n, bool split, bool det, bool drows, int nw)
    {
        return sizeof(double) * (drows ? 4 : 2) * (size_t)n + tab_bytes + (split ? (size_t)nw * kWaveKets : uni_bytes) +
               (det ? stage_bytes : 0);
    }
};
constexpr size_t kCuLds = (size_t)160 << 10;   // a CU's LDS

// LDS to count beside the carve-up.  FP64: the block counter's slot at the dynamic part's alignment;
// with it the runtime's occupancy query gives the same workgroups for every size from 100 to 6144
// atoms (three primitives).  With 256 bytes, 1303 to 1316 atoms were taken to hold three
// workgroups of four waves, not four, and ran eight waves (1303 at 4 bohr 11.7 ms for 11.4, at 6
// bohr 1.49 for 1.35).  FP32 keeps 256: exact, 1091 to 1105 atoms would run four waves without the
// rows of D, where eight with them are ahead (1092 at 4 bohr 4.99 ms and 4.52).
static size_t lds_beside(int prec) { return prec == HFK_MIXED ? 256 : 16; }

// Workgroups of nw waves that the LDS and the waves the registers allow (five per SIMD in FP64,
// six in FP32) leave a CU.
static int fock_groups(int64_t n, int prec, bool drows, int nw)
{
    const size_t need = (prec == HFK_MIXED ? FockSmem<float>::total((int)n, true, false, drows, nw)
                                           : FockSmem<double>::total((int)n, true, false, drows, nw)) +
                        lds_beside(prec);
    const int by_lds = (int)(kCuLds / need), by_waves = (prec == HFK_MIXED ? 24 : 20) / nw;
    return by_lds < by_waves ? by_lds : by_waves;
}

// Rows i and j of D in LDS too, for the hybrid form with up to three primitives outside the
// deterministic strategy, where no workgroup is lost for it: reading D_ik, D_il, D_jk and D_jl
// from memory takes 256 of the 600 texture-addresser cycles of 64 quartets (64 lanes, as many
// lines each).  300 atoms FP64 10.7 -> 10.4 ms, 512 mixed 23.1 -> 22.3; where the rows cost a
// workgroup (512 FP64: four per CU for five) 40.2 -> 42.5.
static bool fock_drows(int g, int64_t n, int prec, bool split, bool det, int nw)
{
    return g <= 3 && split && !det && fock_groups(n, prec, true, nw) >= fock_groups(n, prec, false, nw);
}

// Waves per SIMD the compiler has to leave room for where it ends just above the register
// count of one more by itself: FP64 per-atom bases with three primitives (97 VGPRs; 96 for five
// waves) and five or six primitives (130; 128 for four).
template <int G, typename R, bool kAtoms> constexpr int fock_waves()
{
    return sizeof(R) == 8 ? (G == 3 && kAtoms ? 5 : (G >= 5 && !kAtoms ? 4 : 1)) : 1;
}
// Widest workgroup: the hybrid form with up to three primitives (below 128 VGPRs).
template <int G, bool kSplit, bool kDet> constexpr int fock_max_threads()
{
    return kSplit && !kDet && G <= 3 ? 1024 : kGroupThreads;
}
template <int G, typename R, bool kSplit, bool kAtoms = false, bool kDet = false, bool kDRows = false>
__global__ __launch_bounds__((fock_max_threads<G, kSplit, kDet>()))
__attribute__((amdgpu_waves_per_eu(kDet ? 1 : fock_waves<G, R, kAtoms>()))) void k_fock(FockArgs a)
{
    constexpr int G2 = G * G;
    extern __shared__ __attribute__((aligned(16))) double smem[];
    const int n = a.n;
    // the table first, so its row addresses need no base register
    char *sp = (char *)smem;
    R *tab = (R *)sp;                       // Boys table (grid-scaled for the hybrid form)
    sp += FockSmem<R>::tab_bytes;
    double *rowi = (double *)sp;
    double *rowj = rowi + n;
    sp += sizeof(double) * 2 * (size_t)n;
    double2 *dij = (double2 *)sp;           // kDRows: (D_ic, D_jc)
    if (kDRows) sp += sizeof(double2) * (size_t)n;
    R *lbra = (R *)sp;                      // direct form: [G2][4] Px, Py, Pz, S of the current bra
    R *luni = lbra + 4 * 16;                // direct form: (rho, sqrt rho) per primitive quartet
    // deterministic strategy: staged exchange updates of each wave (the hybrid form has no
    // direct-form slots, so they start at the same place)
    double *stv = (double *)sp;                                   // [waves][kWaveKets] v
    int *stk = (int *)(stv + kWavesPerGroup * kWaveKets);         // [waves][kWaveKets] k
    int *stl = stk + kWavesPerGroup * kWaveKets;                  // [waves][kWaveKets] l
    __shared__ double jbs[kWavesPerGroup];
    const int tid = threadIdx.x, nthr = (int)blockDim.x, nw = nthr / kWave;
    const int wave = uniform(tid / kWave);
    const int lane = tid % kWave;
    // hybrid form: the packed kets of each wave, after the staged updates if there are any
    unsigned char *perm = (unsigned char *)(kDet ? (char *)(stl + kWavesPerGroup * kWaveKets) : sp) + wave * kWaveKets;
    const int gid = blockIdx.x, ng = gridDim.x;
    const int S = ((cptr<DevHeader>)a.hdr)->sig_pairs;
    const BasisDev *bd = a.bd;

    load_boys<R>(tab, Prec<R>::boys(kSplit), BoysGrid<R>::rows * BoysGrid<R>::stride, tid, nthr);
    if (!kSplit) {
        for (int x = tid; x < G2 * G2; x += nthr) {
            luni[2 * x] = Prec<R>::rho(bd)[x];
            luni[2 * x + 1] = Prec<R>::srho(bd)[x];
        }
    }
    cptr<R> crs = (cptr<R>)Prec<R>::rsn(bd);
    asm("" : "+s"(crs));   // a base of its own, not the table's place in the basis constants
    // a ket vector of the workgroup's own is cleared here, and added to without atomics unless
    // its waves meet on a ket
    const bool jown = a.jcopies >= ng, jshared = !jown || a.nsplit > 1;
    // waves that share a chunk each take every kWavesPerGroup-th bra primitive pair
    const bool myterms = lane < G2 && (a.nsplit == 1 || lane % kWavesPerGroup == wave);
    const int wkets = kWave * a.sub, ikets = (a.nsplit > 1 ? 1 : nw) * wkets;
    double *jcol = a.jcol + (int64_t)(gid % a.jcopies) * a.pcap;
    const bool priv = kDet || a.strategy == HFK_STRATEGY_PRIVATE;
    double *fp = priv ? a.fpriv + (int64_t)gid * n * n : a.fpriv;
    if (priv) {
        for (int64_t x = tid; x < (int64_t)n * n; x += nthr) fp[x] = 0.0;
    }
    if (jown) {
        for (int64_t x = tid; x < S; x += nthr) jcol[x] = 0.0;
    }
    __syncthreads();
    const R *prim = Prec<R>::prim(a);
    unsigned long long kept = 0;
    __shared__ long long blk_at;
    const long long NB = ((cptr<DevHeader>)a.hdr)->blocks;
    const cptr<long long> goff = (cptr<long long>)a.goff, item_off = (cptr<long long>)a.item_off;
    // blocks (bra group, ket block K, bra) fetched from a global counter until exhausted, or
    // dealt out by a static grid stride (deterministic strategy)
    for (long long it = 0;; ++it) {
    if (!kDet && tid == 0) blk_at = (long long)atomicAdd(a.next_block, 1ULL);
    __syncthreads();
    const long long blk = kDet ? (long long)gid + it * ng : uniform(blk_at);
    __syncthreads();
    if (blk >= NB) break;
    int s;
    long long m0, m1;
    {
        const long long at = a.last_first ? NB - 1 - blk : blk;
        int kb;
        block_bra(goff, a.ngroups, a.gshift, S, at, s, kb);
        const long long i1 = item_off[s + 1];
        m0 = item_off[s] + (long long)kb * a.tile;
        if (m0 >= i1) continue;   // this bra has fewer blocks than the group's longest
        m1 = m0 + a.tile < i1 ? m0 + a.tile : i1;
    }
    int cur = -1, bi = 0, bj = 0;
    double qs = 0.0, ds = 0.0, jb = 0.0;
    int lim = 0, ebra = kTermNone;

    for (long long m = m0; m <= m1; ++m) {
        if (m < m1) {
            while (item_off[s + 1] <= m) ++s;
        }
        if (m == m1 || s != cur) {
            if (cur >= 0) {
                // flush the finished bra: F_ij from the wave partial sums, then rows i, j
                const double w = wave_sum(jb);
                if constexpr (kDet) {
                    // the four wave sums in wave order
                    if (lane == 0) jbs[wave] = w;
                    __syncthreads();
                    if (tid == 0) {
                        double sw = jbs[0];
#pragma unroll
                        for (int wv = 1; wv < kWavesPerGroup; ++wv) sw += jbs[wv];
                        if (sw != 0.0) rowi[bj] += 4.0 * sw;
                    }
                } else {
                    if (lane == 0 && w != 0.0) atomicAdd(&rowi[bj], 4.0 * w);
                }
                jb = 0.0;
                __syncthreads();
                double *fi = fp + (int64_t)bi * n, *fj = fp + (int64_t)bj * n;
                if (priv) {
                    if (bi == bj) {
                        for (int c = tid; c < n; c += nthr) fi[c] += rowi[c] + rowj[c];
                    } else {
                        for (int c = tid; c < n; c += nthr) {
                            fi[c] += rowi[c];
                            fj[c] += rowj[c];
                        }
                    }
                } else {
                    for (int c = tid; c < n; c += nthr) {
                        const double vi = rowi[c], vj = rowj[c];
                        if (vi != 0.0) atomicAdd(&fi[c], vi);
                        if (vj != 0.0) atomicAdd(&fj[c], vj);
                    }
                }
                __syncthreads();
            }
            if (m == m1) break;
            const R *br = Prec<R>::bra(a) + (int64_t)s * 8 * G2;
            if (!kSplit && tid < 4 * G2) lbra[tid] = br[8 * (tid / 4) + tid % 4];
            // scalar loads: the bra's data stays in scalar registers
            bi = ((cptr<int>)a.pk)[s];
            bj = ((cptr<int>)a.pl)[s];
            for (int c = tid; c < n; c += nthr) {
                rowi[c] = 0.0;
                rowj[c] = 0.0;
                if constexpr (kDRows)
                    dij[c] = make_double2(a.dens[(int64_t)bi * n + c], a.dens[(int64_t)bj * n + c]);
            }
            __syncthreads();
            cur = s;
            qs = ((cptr<double>)a.pq)[s];
            ds = ((cptr<double>)a.pd)[s];
            lim = ((cptr<int>)a.lim)[s];
            if (kSplit) ebra = myterms ? (int)a.bexp[(int64_t)lane * a.pcap + s] : kTermNone;
        }
        const long long wbase = (m - item_off[s]) * ikets + (a.nsplit > 1 ? 0 : wave * wkets);
        if constexpr (!kDet) {
            if (wbase >= lim) continue;
        }
        const cptr<int> kexp = (cptr<int>)(a.kexp + (int)(wbase / wkets) * G2);
        // one 64-lane chunk: ket t per lane (valid: kept by the screen), scatter of v
        // (deterministic strategy: the exchange updates are staged at position `slot`)
        auto chunk = [&](int t, bool valid, int slot) {
            R eri;
            if (kSplit)
                eri = quartet_eri_hybrid<G, R, kAtoms>(
                    (cptr<R>)(Prec<R>::bra(a) + (int64_t)s * 8 * G2), prim, a.pcap, (unsigned)t, crs, tab,
                    ebra, kexp, a.tlim, kAtoms ? (cptr<R>)(Prec<R>::bip(a) + (int64_t)s * G2) : nullptr);
            else
                eri = quartet_eri_direct<G, R>(lbra, prim, a.pcap, t, luni, tab);
            const int k = a.pk[t], l = a.pl[t];
            double deg = 1.0;
            if (bi == bj) deg *= 0.5;
            if (k == l) deg *= 0.5;
            if (t == s) deg *= 0.5;
            const double v = valid ? (double)eri * deg : 0.0;
            jb = fma(a.pd[t], v, jb);
            if (valid) {
                if (a.nsplit == 1 || wave == 0) ++kept;
                if (jshared)
                    atomicAdd(&jcol[t], 4.0 * ds * v);
                else
                    jcol[t] += 4.0 * ds * v;
                if constexpr (kDet) {
                    stv[wave * kWaveKets + slot] = v;
                    stk[wave * kWaveKets + slot] = k;
                    stl[wave * kWaveKets + slot] = l;
                } else {
                    double2 Dk, Dl;
                    if constexpr (kDRows) {
                        Dk = dij[k];
                        Dl = dij[l];
                    } else {
                        const double *Di = a.dens + (int64_t)bi * n;
                        const double *Dj = a.dens + (int64_t)bj * n;
                        Dk = make_double2(Di[k], Dj[k]);
                        Dl = make_double2(Di[l], Dj[l]);
                    }
                    atomicAdd(&rowi[k], -Dl.y * v);
                    atomicAdd(&rowi[l], -Dk.y * v);
                    atomicAdd(&rowj[k], -Dl.x * v);
                    atomicAdd(&rowj[l], -Dk.x * v);
                }
            }
        };
        if constexpr (kDet) {
            int nvalid = 0;
            if (wbase < lim) {
                nvalid = pack_kets(wbase, lane, perm, [&](long long t) { return t < lim && qs * a.pq[t] >= a.tau; });
                for (int c0 = 0; c0 < nvalid; c0 += kWave) {
                    const bool valid = c0 + lane < nvalid;
                    chunk(valid ? (int)wbase + perm[c0 + lane] : S, valid, c0 + lane);
                }
            }
            // every wave's updates are staged; apply them wave after wave
            __syncthreads();
            const double *Di = a.dens + (int64_t)bi * n;
            const double *Dj = a.dens + (int64_t)bj * n;
            for (int wv = 0; wv < kWavesPerGroup; ++wv) {
                if (wave == wv) {
                    for (int e = lane; e < nvalid; e += kWave) {
                        const double v = stv[wave * kWaveKets + e];
                        const int k = stk[wave * kWaveKets + e], l = stl[wave * kWaveKets + e];
                        atomicAdd(&rowi[k], -Dj[l] * v);
                        atomicAdd(&rowi[l], -Dj[k] * v);
                        atomicAdd(&rowj[k], -Di[l] * v);
                        atomicAdd(&rowj[l], -Di[k] * v);
                    }
                }
                __syncthreads();
            }
        } else if (kSplit) {
            // keep the screened kets of this wave's 256, in order, packed into full chunks
            const int nvalid = pack_kets(wbase, lane, perm,
                                         [&](long long t) { return t < lim && qs * a.pq[t] >= a.tau; }, a.sub);
            if (nvalid == 0) continue;
            for (int c0 = 0; c0 < nvalid; c0 += kWave) {
                const bool valid = c0 + lane < nvalid;
                chunk(valid ? (int)wbase + perm[c0 + lane] : S, valid, 0);   // S: first pad entry
            }
            __builtin_amdgcn_wave_barrier();
        } else {
            for (int c = 0; c < a.sub; ++c) {
                const long long t0 = wbase + c * kWave;
                if (t0 >= lim) break;
                const long long t = t0 + lane;   // < S + 64 <= pcap: padded tables
                chunk((int)t, t < lim && qs * a.pq[t] >= a.tau, 0);
            }
        }
    }
    }
    // survivors: one atomic per wave
    for (int off = 32; off > 0; off >>= 1) kept += __shfl_xor(kept, off, 64);
    if (lane == 0 && kept) atomicAdd(a.quartets, kept);
}

// ------------------------------------------------------------------ final reduction

__global__ __launch_bounds__(256) void k_sum_private(const double *__restrict__ fpriv, int groups, int64_t n2,
                                                     double *__restrict__ fsum)
{
    const int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (x >= n2) return;
    double s = 0.0;
    for (int gph = 0; gph < groups; ++gph) s += fpriv[(int64_t)gph * n2 + x];
    fsum[x] = s;
}

// Sum of the copies of the ket-side Coulomb vector, left in copy 0 (many copies only).
__global__ __launch_bounds__(256) void k_jcol_sum(const DevHeader *__restrict__ hdr, double *__restrict__ jcol,
                                                  int copies, int64_t pcap)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= hdr->sig_pairs) return;
    double s = 0.0;
    for (int c = 0; c < copies; ++c) s += jcol[(int64_t)c * pcap + t];
    jcol[t] = s;
}

// G = (F + F^T)/2 with the ket-side Coulomb terms of the pair (i, j) (each pair is one
// position), and the workgroups' partial sums of D o G; a single workgroup writes E2 itself.
// One or two launches: copying F, adding the ket terms, symmetrising and summing took four of
// 4.5 us.  (Summing the partials in the workgroup that ends last needs a device-wide fence in
// every workgroup, which made the kernel 16 us at 64 atoms.)
constexpr int kFinishPer = 4;
template <int kThreads>
__global__ __launch_bounds__(kThreads) void k_finish(const double *__restrict__ F, const double *__restrict__ jcol,
                                                     int copies, int64_t pcap, const int *__restrict__ posof,
                                                     const double *__restrict__ dens, int n,
                                                     double *__restrict__ fock, double *__restrict__ part,
                                                     double *__restrict__ e2)
{
    __shared__ double red[kThreads];
    const int n2 = n * n, at = blockIdx.x * kThreads * kFinishPer + threadIdx.x;
    double e = 0.0;
#pragma unroll
    for (int r = 0; r < kFinishPer; ++r) {
        const int x = at + r * kThreads;
        if (x < n2) {
            const int i = x / n, j = x - i * n;
            const int hi = i > j ? i : j, lo = i > j ? j : i;
            const int t = posof[(int64_t)hi * (hi + 1) / 2 + lo];
            double J = 0.0;
            if (t >= 0) {
#pragma unroll 8
                for (int c = 0; c < copies; ++c) J += jcol[(int64_t)c * pcap + t];
            }
            const double gv = i == j ? F[x] + J : 0.5 * (F[x] + F[(int64_t)j * n + i] + J);
            fock[x] = gv;
            e += dens[x] * gv;
        }
    }
    red[threadIdx.x] = e;
    __syncthreads();
    for (int w = kThreads / 2; w > 0; w >>= 1) {
        if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        if (gridDim.x == 1)
            *e2 = 0.5 * red[0];
        else
            part[blockIdx.x] = red[0];
    }
}

// E2 = 1/2 sum of the partials (one block, fixed order).
__global__ __launch_bounds__(256) void k_energy(const double *__restrict__ part, int nb, double *__restrict__ e2)
{
    __shared__ double red[256];
    double s = 0.0;
    for (int b = threadIdx.x; b < nb; b += 256) s += part[b];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) *e2 = 0.5 * red[0];
}

template <int G, typename R> using FockKernel = void (*)(FockArgs);

// The kernel of a build: the direct form keeps a bra's primitive data in LDS slots sized for
// g <= 4; per-atom bases and the deterministic strategy run the hybrid form only.
template <int G, typename R>
static FockKernel<G, R> fock_kernel(bool split, bool atoms, bool det, bool drows)
{
    (void)drows;
    (void)split;
    if (det) return atoms ? k_fock<G, R, true, true, true> : k_fock<G, R, true, false, true>;
    if constexpr (G <= 3) {
        if (drows) return atoms ? k_fock<G, R, true, true, false, true> : k_fock<G, R, true, false, false, true>;
    }
    if (atoms) return k_fock<G, R, true, true>;
    if constexpr (G <= 4) {
        if (!split) return k_fock<G, R, false>;
    }
    return k_fock<G, R, true>;
}

template <int G, typename R>
static hipError_t launch_fock_t(const FockArgs &a, int groups, int nw, int variant, bool atoms, hipStream_t st)
{
    const bool det = a.strategy == HFK_STRATEGY_DETERMINISTIC;
    const bool split = G > 4 || variant != 0 || atoms || det;
    const bool drows = fock_drows(G, a.n, sizeof(R) == 8 ? HFK_FP64 : HFK_MIXED, split, det, nw);
    const size_t smem = FockSmem<R>::total(a.n, split, det, drows, nw);
    profile_begin(st);
    hipLaunchKernelGGL((fock_kernel<G, R>(split, atoms, det, drows)), dim3(groups), dim3(nw * kWave), smem, st, a);
    profile_end(st);
    return hipGetLastError();
}

template <int G, typename R>
static int resident_t(bool split, bool atoms, bool det, int64_t n, int nw)
{
    split = split || G > 4;
    const bool drows = fock_drows(G, n, sizeof(R) == 8 ? HFK_FP64 : HFK_MIXED, split, det, nw);
    const size_t smem = FockSmem<R>::total((int)n, split, det, drows, nw);
    int nb = 0;
    const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
        &nb, reinterpret_cast<const void *>(fock_kernel<G, R>(split, atoms, det, drows)), nw * kWave, smem);
    return e == hipSuccess ? nb : 0;
}

// Workgroups of the quartet kernel that fit on one CU at once (registers and LDS); 0 if
// the runtime cannot tell.  Persistent workgroups beyond this would only queue.
int fock_resident_groups(int g, int prec, int variant, int64_t n, bool atoms, bool det, int nw)
{
    const bool split = variant != 0 || atoms || det;
    if (prec == HFK_MIXED) {
        switch (g) {
        case 1: return resident_t<1, float>(split, atoms, det, n, nw);
        case 2: return resident_t<2, float>(split, atoms, det, n, nw);
        case 3: return resident_t<3, float>(split, atoms, det, n, nw);
        case 4: return resident_t<4, float>(split, atoms, det, n, nw);
        case 5: return resident_t<5, float>(split, atoms, det, n, nw);
        default: return resident_t<6, float>(split, atoms, det, n, nw);
        }
    }
    switch (g) {
    case 1: return resident_t<1, double>(split, atoms, det, n, nw);
    case 2: return resident_t<2, double>(split, atoms, det, n, nw);
    case 3: return resident_t<3, double>(split, atoms, det, n, nw);
    case 4: return resident_t<4, double>(split, atoms, det, n, nw);
    case 5: return resident_t<5, double>(split, atoms, det, n, nw);
    default: return resident_t<6, double>(split, atoms, det, n, nw);
    }
}

// The LDS rows of F grow with the atoms, and with four waves sharing them fewer and fewer waves
// fit on a CU (12 at 2016 atoms): wider workgroups share a pair of rows among more waves, and are
// taken where more waves then fit.  FP64 at 4 bohr, ms with four waves and with eight: 1303 atoms
// 11.4 / 11.7 (16 waves a CU either way, four lose less at the end of a block), 1400 (12 and 16)
// 16.0 / 13.6, 2016 33.8 / 29.9; mixed 1092 4.99 / 4.52, 2016 24.9 / 16.3.  With eight and with
// sixteen, thinly spread (7 bohr): FP64 3400 6.5 / 7.2 (16 waves either way), 3813 on 10.9 / 8.7,
// 6144 27.1 / 21.6; mixed 4300 9.0 / 10.5, 4500 14.3 / 11.2; per-atom bases 3800 19.1 / 14.7.
// Below 1 ms the last blocks show: mixed 1092 atoms at 6 bohr 0.78 ms with four, 0.81 with eight.
// Widths that the four SIMDs don't share evenly lose on both sides (2016 atoms: five waves 31.1,
// six 37.8).
int fock_waves_per_group(int g, int prec, int variant, int64_t n, bool atoms, bool det)
{
    if (g > 3 || det || (variant == 0 && !atoms)) return kWavesPerGroup;
    int best = kWavesPerGroup;
    for (const int nw : {8, 16})
        if (nw * fock_groups(n, prec, false, nw) > best * fock_groups(n, prec, false, best)) best = nw;
    return best;
}

PairPlan fock_plan(const Layout &L, char *ws, int strategy, int prec, int variant)
{
    PairPlan p;
    const int copies = effective_copies(L);
    p.info = HeaderInfo{strategy, L.groups, prec, variant, L.tile, 1 << L.gshift, copies};
    p.fixed_order = strategy == HFK_STRATEGY_DETERMINISTIC;
    // workgroups clear their own copies; shared ones are cleared before the launch
    p.fzero = strategy == HFK_STRATEGY_ATOMIC ? (double *)(ws + L.fpriv) : nullptr;
    p.nf = p.fzero ? L.n * L.n : 0;
    p.jzero = copies < L.groups ? (double *)(ws + L.jcol) : nullptr;
    p.jcopies = p.jzero ? copies : 0;
    return p;
}

hipError_t launch_fock(const Layout &L, const Basis &b, char *ws, const double *dens, double tau, int prec,
                       int strategy, int variant, double *fock, double *e2, hipStream_t st)
{
    DevHeader *hdr = (DevHeader *)(ws + L.hdr);
    FockArgs a;
    a.hdr = hdr;
    a.bd = (const BasisDev *)(ws + L.basis);
    a.pk = (const int *)(ws + L.pk);
    a.pl = (const int *)(ws + L.pl);
    a.pq = (const double *)(ws + L.pq);
    a.pd = (const double *)(ws + L.pd);
    a.prim = (const double *)(ws + L.prim);
    a.prim_f = (const float *)(ws + L.prim_f);
    a.bra = (const double *)(ws + L.bra);
    a.bra_f = (const float *)(ws + L.bra_f);
    a.bip = L.atoms ? (const double *)(ws + L.bip) : nullptr;
    a.bip_f = L.atoms ? (const float *)(ws + L.bip_f) : nullptr;
    a.item_off = (const long long *)(ws + L.item_off);
    a.lim = (const int *)(ws + L.lim);
    a.bexp = (const short *)(ws + L.bexp);
    a.kexp = (const int *)(ws + (L.sub == kSubChunks ? L.kexp256 : L.kexp64));
    a.sub = L.sub;
    a.nsplit = L.nsplit;
    a.last_first = L.sub == kSubChunks ? 0 : 1;
    a.tlim = term_limit(tau, prec);
    a.goff = (const long long *)(ws + L.goff);
    a.ngroups = L.ngroups;
    a.gshift = L.gshift;
    a.tile = L.tile;
    a.dens = dens;
    a.fpriv = (double *)(ws + L.fpriv);
    a.jcol = (double *)(ws + L.jcol);
    a.quartets = &hdr->quartets;
    a.next_block = &hdr->next_block;
    a.pcap = L.pcap;
    a.tau = tau;
    a.n = (int)L.n;
    a.strategy = strategy;
    a.jcopies = effective_copies(L);
    const int64_t n2 = L.n * L.n;
    const unsigned nb2 = (unsigned)((n2 + 255) / 256);
    hipError_t err = hipSuccess;
    const int g = b.g;
    const bool at = L.atoms;
    if (prec == HFK_MIXED) {
        switch (g) {
        case 1: err = launch_fock_t<1, float>(a, L.groups, L.nw, variant, at, st); break;
        case 2: err = launch_fock_t<2, float>(a, L.groups, L.nw, variant, at, st); break;
        case 3: err = launch_fock_t<3, float>(a, L.groups, L.nw, variant, at, st); break;
        case 4: err = launch_fock_t<4, float>(a, L.groups, L.nw, variant, at, st); break;
        case 5: err = launch_fock_t<5, float>(a, L.groups, L.nw, 1, at, st); break;
        default: err = launch_fock_t<6, float>(a, L.groups, L.nw, 1, at, st); break;
        }
    } else {
        switch (g) {
        case 1: err = launch_fock_t<1, double>(a, L.groups, L.nw, variant, at, st); break;
        case 2: err = launch_fock_t<2, double>(a, L.groups, L.nw, variant, at, st); break;
        case 3: err = launch_fock_t<3, double>(a, L.groups, L.nw, variant, at, st); break;
        case 4: err = launch_fock_t<4, double>(a, L.groups, L.nw, variant, at, st); break;
        case 5: err = launch_fock_t<5, double>(a, L.groups, L.nw, 1, at, st); break;
        default: err = launch_fock_t<6, double>(a, L.groups, L.nw, 1, at, st); break;
        }
    }
    if (err != hipSuccess) return err;
    const double *F = a.fpriv;
    if (strategy == HFK_STRATEGY_PRIVATE || strategy == HFK_STRATEGY_DETERMINISTIC) {
        double *fsum = (double *)(ws + L.fsum);
        hipLaunchKernelGGL(k_sum_private, dim3(nb2), dim3(256), 0, st, a.fpriv, L.groups, n2, fsum);
        F = fsum;
    }
    int copies = a.jcopies;
    if (copies > 16) {
        // both triangles of G would read every copy
        hipLaunchKernelGGL(k_jcol_sum, dim3((unsigned)((L.pcap + 255) / 256)), dim3(256), 0, st, hdr, a.jcol, copies,
                           L.pcap);
        copies = 1;
    }
    double *part = (double *)(ws + L.e2part);
    const int *posof = (const int *)(ws + L.bucket_of);
    if (n2 <= 1024 * kFinishPer) {
        hipLaunchKernelGGL((k_finish<1024>), dim3(1), dim3(1024), 0, st, F, (const double *)a.jcol, copies, L.pcap, posof,
                           dens, a.n, fock, part, e2);
    } else {
        const unsigned nb = (unsigned)((n2 + 256 * kFinishPer - 1) / (256 * kFinishPer));
        hipLaunchKernelGGL((k_finish<256>), dim3(nb), dim3(256), 0, st, F, (const double *)a.jcol, copies, L.pcap, posof,
                           dens, a.n, fock, part, e2);
        hipLaunchKernelGGL(k_energy, dim3(1), dim3(256), 0, st, (const double *)part, (int)nb, e2);
    }
    return hipGetLastError();
}

}  // namespace hfk
