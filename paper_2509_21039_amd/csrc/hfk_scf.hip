// Closed-shell self-consistent field around the two-electron build: the loop on either side
// of the paper's kernel (which computes the electron-repulsion term of the Fock operator).
//
//   H = T + V (one-electron integrals of contracted s functions, kernels below)
//   X = S^(-1/2) (symmetric orthogonalisation)
//   repeat: G = G(D) (the screened two-electron build), F = H + G,
//           E = 1/2 sum D o (H + F) + E_nn,
//           e = X (F D S - S D F) X (the commutator in the orthonormal basis),
//           F_x = DIIS extrapolation over the last kDiisMax (F, e),
//           eigenvectors C' of X F_x X, C = X C', D = 2 C_occ C_occ^T (Aufbau)
//   until |E - E_prev| < e_tol and max |e| < d_tol.
//
// The integral kernels and the two-electron build are this library's.  Up to kSmallScf atoms
// the dense products and the symmetric eigenproblems are one-workgroup kernels of this library
// too; above that they go to rocBLAS and rocSOLVER, whose scratch comes from the caller's
// workspace.  Matrices are n x n FP64 with leading dimension n; every one that is
// symmetric reads the same in either storage order, and the products are taken column-major.
#include <math.h>
#include <stdio.h>
#include <string.h>

#include <algorithm>
#include <vector>

#include <rocblas/rocblas.h>
#include <rocsolver/rocsolver.h>

#include "hfk_device.hpp"
#include "hfk_scf.hpp"

namespace hfk {

// ------------------------------------------------------------------ one-electron integrals

// S and H = T + V for every i >= j (written to both triangles).  For primitives a (atom i)
// and b (atom j): p = a + b, mu = a b / p, K = w_a w_b exp(-mu R^2),
//   S_ab = K (pi/p)^(3/2),  T_ab = mu (3 - 2 mu R^2) S_ab,
//   V_ab = - sum_C Z_C K (2 pi / p) F0(p |P - C|^2),  F0(t) = (sqrt(pi)/2) erf(sqrt t)/sqrt t.
// A primitive product whose K (2 pi / p) is below 1e-17 skips the nucleus loop: its term is
// at most 1e-17 times the total nuclear charge (F0 <= 1).
// Sixteen lanes share a pair: lane l takes every sixteenth (primitive product, nucleus) term, and
// the lanes' sums are added in a fixed order (one thread per pair took 122 us at 36 atoms).
constexpr int kOneLanes = 16;
__global__ __launch_bounds__(256) void k_one_electron(int64_t n, int g, const double *__restrict__ xyz,
                                                      const double *__restrict__ Z,
                                                      const double *__restrict__ aexp,
                                                      const double *__restrict__ aw, double *__restrict__ S,
                                                      double *__restrict__ H)
{
    const int64_t npair = n * (n + 1) / 2;
    const int64_t q = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / kOneLanes;
    const int l = threadIdx.x % kOneLanes;
    const bool live = q < npair;
    int64_t i = 0, j = 0;
    double s = 0.0, t = 0.0, v = 0.0;
    if (live) {
        pair_of_index(q, i, j);
        const double A[3] = {xyz[3 * i], xyz[3 * i + 1], xyz[3 * i + 2]};
        const double B[3] = {xyz[3 * j], xyz[3 * j + 1], xyz[3 * j + 2]};
        const double r2 =
            (A[0] - B[0]) * (A[0] - B[0]) + (A[1] - B[1]) * (A[1] - B[1]) + (A[2] - B[2]) * (A[2] - B[2]);
        for (int a = 0; a < g; ++a)
            for (int c = 0; c < g; ++c) {
                const double ea = aexp[i * g + a], eb = aexp[j * g + c];
                const double p = ea + eb, mu = ea * eb / p;
                const double K = aw[i * g + a] * aw[j * g + c] * exp(-mu * r2);
                const double sab = K * pow(kPi / p, 1.5);
                s += sab;
                t += mu * (3.0 - 2.0 * mu * r2) * sab;
                const double kv = K * (2.0 * kPi / p);
                if (fabs(kv) < 1e-17) continue;
                const double P[3] = {(ea * A[0] + eb * B[0]) / p, (ea * A[1] + eb * B[1]) / p,
                                     (ea * A[2] + eb * B[2]) / p};
                double vz = 0.0;
                for (int64_t cc = l; cc < n; cc += kOneLanes) {
                    const double dx = P[0] - xyz[3 * cc], dy = P[1] - xyz[3 * cc + 1], dz = P[2] - xyz[3 * cc + 2];
                    vz += Z[cc] * erf_over_sqrt(p * (dx * dx + dy * dy + dz * dz));
                }
                v -= kv * 0.5 * sqrt(kPi) * vz;
            }
    }
#pragma unroll
    for (int w = kOneLanes / 2; w > 0; w >>= 1) v += __shfl_xor(v, w, kOneLanes);
    if (live && l == 0) {
        S[i * n + j] = S[j * n + i] = s;
        H[i * n + j] = H[j * n + i] = t + v;
    }
}

// E_nn = sum_{A > B} Z_A Z_B / R_AB (one block, fixed order).
__global__ __launch_bounds__(256) void k_enuc(int64_t n, const double *__restrict__ xyz, const double *__restrict__ Z,
                                              double *__restrict__ out)
{
    __shared__ double red[256];
    double e = 0.0;
    for (int64_t a = threadIdx.x; a < n; a += 256)
        for (int64_t b = 0; b < a; ++b) {
            const double dx = xyz[3 * a] - xyz[3 * b], dy = xyz[3 * a + 1] - xyz[3 * b + 1],
                         dz = xyz[3 * a + 2] - xyz[3 * b + 2];
            e += Z[a] * Z[b] / sqrt(dx * dx + dy * dy + dz * dz);
        }
    red[threadIdx.x] = e;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) *out = red[0];
}

// ------------------------------------------------------------------ small dense helpers

// W(:, k) = U(:, k) / sqrt(s_k) (column-major).
__global__ __launch_bounds__(256) void k_scale_cols(int64_t n, const double *__restrict__ U,
                                                    const double *__restrict__ s, double *__restrict__ W)
{
    const int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (x < n * n) W[x] = U[x] / sqrt(s[x / n]);
}

__global__ __launch_bounds__(256) void k_add(int64_t m, const double *__restrict__ a, const double *__restrict__ b,
                                             double *__restrict__ c)
{
    const int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (x < m) c[x] = a[x] + b[x];
}

// Out = A - A^T.
__global__ __launch_bounds__(256) void k_antisym(int64_t n, const double *__restrict__ A, double *__restrict__ out)
{
    const int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (x >= n * n) return;
    const int64_t r = x % n, c = x / n;
    out[x] = A[x] - A[r * n + c];
}

// The numbers the host needs after each build, in one launch of 3 + kDiisMax blocks, each a
// fixed-order block reduction (so repeated runs agree bit for bit):
//   out[0] = <D, H>, out[1] = <D, F>, out[2] = max |e|,
//   out[3 + k] = <e, e_k> for every history slot k set in `filled` (0 for the others).
__global__ __launch_bounds__(256) void k_scf_scalars(int64_t n2, const double *__restrict__ D,
                                                     const double *__restrict__ H, const double *__restrict__ F,
                                                     const double *__restrict__ e, const double *__restrict__ hist,
                                                     unsigned filled, double *__restrict__ out)
{
    __shared__ double red[256];
    const int q = blockIdx.x;   // uniform over the block: an early return keeps every barrier whole
    const bool mx = q == 2;
    const double *a = q < 2 ? D : e;
    const double *b = q == 0 ? H : (q == 1 ? F : (q == 2 ? e : hist + (int64_t)(q - 3) * n2));
    if (q >= 3 && !((filled >> (q - 3)) & 1u)) {
        if (threadIdx.x == 0) out[q] = 0.0;
        return;
    }
    double v = 0.0;
    for (int64_t x = threadIdx.x; x < n2; x += 256) v = mx ? fmax(v, fabs(a[x])) : fma(a[x], b[x], v);
    red[threadIdx.x] = v;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (threadIdx.x < w)
            red[threadIdx.x] = mx ? fmax(red[threadIdx.x], red[threadIdx.x + w]) : red[threadIdx.x] + red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[q] = red[0];
}

__global__ void k_clear_info(int *__restrict__ info) { *info = 0; }

struct Coefs {
    double c[kDiisMax];
    int slot[kDiisMax];
    int m;
};

// out = sum_i c_i F[slot_i] (the DIIS combination).
__global__ __launch_bounds__(256) void k_lincomb(int64_t n2, Coefs cf, const double *__restrict__ hist,
                                                 double *__restrict__ out)
{
    const int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (x >= n2) return;
    double s = 0.0;
    for (int i = 0; i < cf.m; ++i) s += cf.c[i] * hist[(int64_t)cf.slot[i] * n2 + x];
    out[x] = s;
}

// ------------------------------------------------------------------ small systems in one workgroup

// Up to kSmallScf atoms the dense part of an iteration is two launches of one workgroup with its
// matrices in LDS: the error matrix with the scalars the host needs, and the extrapolation, the
// eigenproblem and the density.  The libraries' route is some 60 launches per iteration (the
// eigensolver's reduction alone 35 of them at 36 atoms, 0.9 ms in all): per SCF 12 atoms 5.3 ms, in
// one workgroup 1.3; 36 atoms 14.0 and 3.6; 48 23.7 and 6.7; 63 33.9 and 11.8.  The limit is what
// the kernels are laid out for (three matrices of 64 rows take 100 KB of LDS); larger systems were
// not tried in one workgroup.  The eigenproblem is solved by cyclic Jacobi rotations, n/2
// disjoint ones at a time (round-robin pairing), which suits one workgroup: a round is one
// division-and-root chain and one pass over 2 x 2 blocks.  Its start is the last eigenvectors,
// so that few sweeps remain once the density settles.
constexpr int kSmallScf = 64;
constexpr int kScfThreads = 1024;

// Row length in LDS: odd, so that a column's elements fall in different banks.
__host__ __device__ inline int scf_ld(int n) { return n | 1; }

__device__ inline void lds_load(double *__restrict__ dst, const double *__restrict__ src, int n)
{
    const int ld = scf_ld(n);
    for (int x = threadIdx.x; x < n * n; x += kScfThreads) dst[x / n * ld + x % n] = src[x];
}

// C = op(A) B in LDS (op: transpose if ta), two by two elements per thread; C is neither A nor B.
// Ends with a barrier.
__device__ inline void lds_gemm(double *__restrict__ C, const double *__restrict__ A, const double *__restrict__ B,
                                int n, bool ta)
{
    const int ld = scf_ld(n), h = (n + 1) / 2;
    for (int x = threadIdx.x; x < h * h; x += kScfThreads) {
        const int r0 = x / h * 2, c0 = x % h * 2, r1 = r0 + 1 < n ? r0 + 1 : r0, c1 = c0 + 1 < n ? c0 + 1 : c0;
        double s00 = 0.0, s01 = 0.0, s10 = 0.0, s11 = 0.0;
#pragma unroll 4
        for (int k = 0; k < n; ++k) {
            const double a0 = ta ? A[k * ld + r0] : A[r0 * ld + k], a1 = ta ? A[k * ld + r1] : A[r1 * ld + k];
            const double b0 = B[k * ld + c0], b1 = B[k * ld + c1];
            s00 = fma(a0, b0, s00);
            s01 = fma(a0, b1, s01);
            s10 = fma(a1, b0, s10);
            s11 = fma(a1, b1, s11);
        }
        C[r0 * ld + c0] = s00;
        if (c1 != c0) C[r0 * ld + c1] = s01;
        if (r1 != r0) C[r1 * ld + c0] = s10;
        if (c1 != c0 && r1 != r0) C[r1 * ld + c1] = s11;
    }
    __syncthreads();
}

// Sum (or maximum) of one value per thread, in a fixed order, the same in every thread.
__device__ inline double block_reduce(double v, bool mx, double *__restrict__ red)
{
    const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
#pragma unroll
    for (int w = kWave / 2; w > 0; w >>= 1) {
        const double o = __shfl_xor(v, w, kWave);
        v = mx ? fmax(v, o) : v + o;
    }
    __syncthreads();
    if (lane == 0) red[wave] = v;
    __syncthreads();
    double r = red[0];
    for (int w = 1; w < kScfThreads / kWave; ++w) r = mx ? fmax(r, red[w]) : r + red[w];
    return r;
}

// Round-robin pairing of m (even) indices: in round r slot 0 holds (m - 1, r) and slot k
// ((r + k) mod (m - 1), (r - k) mod (m - 1)), so that every two meet once in m - 1 rounds.  A
// slot's two indices step by one from round to round (no division in the loop).
struct JacobiSlot {
    int a, b;
};
__device__ inline JacobiSlot jacobi_slot(int k, int m)
{
    return JacobiSlot{k == 0 ? m - 1 : k, k == 0 ? 0 : m - 1 - k};
}
__device__ inline void jacobi_step(JacobiSlot &s, int m)
{
    if (s.a < m - 1) s.a = s.a + 1 == m - 1 ? 0 : s.a + 1;
    s.b = s.b + 1 == m - 1 ? 0 : s.b + 1;
}

// 1/sqrt(x) and 1/x to FP64 accuracy: the hardware estimates and two Newton steps.
__device__ inline double rsqrt_full(double x)
{
    double y = __builtin_amdgcn_rsq(x);
#pragma unroll
    for (int i = 0; i < 2; ++i) y = fma(0.5 * y, fma(-x * y, y, 1.0), y);
    return y;
}
__device__ inline double rcp_full(double x)
{
    double y = __builtin_amdgcn_rcp(x);
#pragma unroll
    for (int i = 0; i < 2; ++i) y = fma(y, fma(-x, y, 1.0), y);
    return y;
}

// Diagonalises the symmetric A in place and accumulates the rotations into V (V -> V J).
// Elements below 2^-54 of the norm are left; a sweep whose rotations all had a tangent below
// 1e-8 is the last one (convergence is quadratic: what remains is below 1e-16 of the norm).  The
// matrix is scaled by a power of two meanwhile.  Returns false for a matrix with a non-finite
// element, or after 40 sweeps.
__device__ inline bool lds_jacobi(double *__restrict__ A, double *__restrict__ V, int n, double2 *__restrict__ cs,
                                  double *__restrict__ red)
{
    const int ld = scf_ld(n), m = n + (n & 1), np = m / 2, t = threadIdx.x;
    __shared__ int turned;
    double v = 0.0;
    for (int x = t; x < n * n; x += kScfThreads) v += fabs(A[x / n * ld + x % n]);
    const double norm = block_reduce(v, false, red);
    if (!(norm <= 1e300)) return false;
    if (n == 1 || norm == 0.0) return true;
    int ex;
    (void)frexp(norm, &ex);
    __syncthreads();
    for (int x = t; x < n * n; x += kScfThreads) A[x / n * ld + x % n] = ldexp(A[x / n * ld + x % n], -ex);
    const double tiny = ldexp(norm, -ex) / n * 0x1p-54;
    // this thread's tasks: 2 x 2 blocks (I, J) of A, rotated from both sides, then (row i, J) of
    // V, rotated from the right
    constexpr int kTasks = (kSmallScf / 2 * (kSmallScf / 2) + kSmallScf * (kSmallScf / 2)) / kScfThreads;
    const int na = np * np, all = na + n * np;
    int ti[kTasks], tj[kTasks];
#pragma unroll
    for (int k = 0; k < kTasks; ++k) {
        const int x = t + k * kScfThreads, y = x < na ? x : x - na;
        ti[k] = x < all ? y / np : -1;
        tj[k] = y % np;
    }
    bool done = false;
    for (int sweep = 0; sweep < 40 && !done; ++sweep) {
        __syncthreads();
        if (t == 0) turned = 0;
        JacobiSlot own = jacobi_slot(t, m), si[kTasks], sj[kTasks];
#pragma unroll
        for (int k = 0; k < kTasks; ++k) {
            si[k] = jacobi_slot(ti[k], m);
            sj[k] = jacobi_slot(tj[k], m);
        }
        __syncthreads();
        for (int r = 0; r < m - 1; ++r) {
            if (t < np) {
                const int p = own.a < own.b ? own.a : own.b, q = own.a < own.b ? own.b : own.a;
                double c = 1.0, s = 0.0;
                if (q < n) {
                    const double apq = A[p * ld + q], d = A[q * ld + q] - A[p * ld + p];
                    if (fabs(apq) > tiny) {
                        // tangent of the smaller angle: 2 apq / (d +- sqrt(d^2 + 4 apq^2))
                        const double w = fma(d, d, 4.0 * apq * apq), root = w * rsqrt_full(w);
                        const double tn = 2.0 * apq * rcp_full(d >= 0.0 ? d + root : d - root);
                        c = rsqrt_full(fma(tn, tn, 1.0));
                        s = tn * c;
                        if (fabs(tn) > 1e-8) turned = 1;
                    }
                }
                cs[t] = make_double2(c, s);
                jacobi_step(own, m);
            }
            __syncthreads();
#pragma unroll
            for (int k = 0; k < kTasks; ++k) {
                if (ti[k] < 0) continue;
                const double2 cj = cs[tj[k]];
                const int u = sj[k].a < sj[k].b ? sj[k].a : sj[k].b, w = sj[k].a < sj[k].b ? sj[k].b : sj[k].a;
                jacobi_step(sj[k], m);
                if (t + k * kScfThreads < na) {
                    const double2 ci = cs[ti[k]];
                    const int p = si[k].a < si[k].b ? si[k].a : si[k].b, q = si[k].a < si[k].b ? si[k].b : si[k].a;
                    jacobi_step(si[k], m);
                    if (ci.y == 0.0 && cj.y == 0.0) continue;
                    const bool hq = q < n, hw = w < n;
                    const double pu = A[p * ld + u], pw = hw ? A[p * ld + w] : 0.0;
                    const double qu = hq ? A[q * ld + u] : 0.0, qw = hq && hw ? A[q * ld + w] : 0.0;
                    // columns u, w, then rows p, q
                    const double pu1 = cj.x * pu - cj.y * pw, pw1 = cj.y * pu + cj.x * pw;
                    const double qu1 = cj.x * qu - cj.y * qw, qw1 = cj.y * qu + cj.x * qw;
                    const bool diag = ti[k] == tj[k];   // the rotated element is zero by construction
                    A[p * ld + u] = ci.x * pu1 - ci.y * qu1;
                    if (hw) A[p * ld + w] = diag ? 0.0 : ci.x * pw1 - ci.y * qw1;
                    if (hq) A[q * ld + u] = diag ? 0.0 : ci.y * pu1 + ci.x * qu1;
                    if (hq && hw) A[q * ld + w] = ci.y * pw1 + ci.x * qw1;
                } else {
                    if (cj.y == 0.0) continue;
                    const double x0 = V[ti[k] * ld + u], x1 = V[ti[k] * ld + w];
                    V[ti[k] * ld + u] = cj.x * x0 - cj.y * x1;
                    V[ti[k] * ld + w] = cj.y * x0 + cj.x * x1;
                }
            }
            __syncthreads();
        }
        done = !turned;
    }
    __syncthreads();
    for (int k = t; k < n; k += kScfThreads) A[k * ld + k] = ldexp(A[k * ld + k], ex);
    return done;
}

// Rank of every eigenvalue (ascending, ties by place), into rank[0 .. n).
__device__ inline void lds_ranks(const double *__restrict__ A, int n, int *__restrict__ rank)
{
    const int ld = scf_ld(n);
    for (int k = threadIdx.x; k < n; k += kScfThreads) {
        const double v = A[k * ld + k];
        int r = 0;
        for (int x = 0; x < n; ++x) {
            const double o = A[x * ld + x];
            r += o < v || (o == v && x < k);
        }
        rank[k] = r;
    }
    __syncthreads();
}

// X = S^(-1/2), and for the host: out[0] = E_nn (already there), out[1] and out[2] the smallest
// and largest eigenvalue of S, out[3] = 1 if the eigenproblem failed.
__global__ __launch_bounds__(kScfThreads) void k_small_invsqrt(int n, const double *__restrict__ S,
                                                               double *__restrict__ X, double *__restrict__ out)
{
    extern __shared__ __attribute__((aligned(16))) double sm[];
    __shared__ double2 cs[kSmallScf / 2];
    __shared__ double red[kScfThreads / kWave];
    const int ld = scf_ld(n), t = threadIdx.x;
    double *A = sm, *V = sm + n * ld;
    lds_load(A, S, n);
    for (int x = t; x < n * n; x += kScfThreads) V[x / n * ld + x % n] = x / n == x % n ? 1.0 : 0.0;
    __syncthreads();
    const bool ok = lds_jacobi(A, V, n, cs, red);
    __syncthreads();
    for (int x = t; x < n * n; x += kScfThreads) {
        const int i = x / n, j = x % n;
        double s = 0.0;
        for (int k = 0; k < n; ++k) s = fma(V[i * ld + k] / sqrt(A[k * ld + k]), V[j * ld + k], s);
        X[x] = s;
    }
    if (t == 0) {
        double lo = A[0], hi = A[0];
        for (int k = 1; k < n; ++k) {
            lo = fmin(lo, A[k * ld + k]);
            hi = fmax(hi, A[k * ld + k]);
        }
        out[1] = lo;
        out[2] = hi;
        out[3] = ok ? 0.0 : 1.0;
    }
}

// F = H + G, the error e = X (F D S - S D F) X, both into their history slots, and the numbers
// the host needs (as k_scf_scalars, with the last eigenproblem's status at out[3 + kDiisMax]).
__global__ __launch_bounds__(kScfThreads) void k_small_error(int n, const double *__restrict__ H,
                                                             const double *__restrict__ G,
                                                             const double *__restrict__ D,
                                                             const double *__restrict__ S,
                                                             const double *__restrict__ X, double *__restrict__ F,
                                                             double *__restrict__ hF, double *__restrict__ hE, int slot,
                                                             unsigned filled, const int *__restrict__ info,
                                                             double *__restrict__ out)
{
    extern __shared__ __attribute__((aligned(16))) double sm[];
    __shared__ double red[kScfThreads / kWave];
    const int ld = scf_ld(n), n2 = n * n, t = threadIdx.x;
    double *B1 = sm, *B2 = B1 + n * ld, *B3 = B2 + n * ld;
    double dh = 0.0, df = 0.0;
    for (int x = t; x < n2; x += kScfThreads) {
        const double h = H[x], f = h + G[x], d = D[x];
        F[x] = f;
        hF[(int64_t)slot * n2 + x] = f;
        B1[x / n * ld + x % n] = f;
        B3[x / n * ld + x % n] = d;
        dh = fma(d, h, dh);
        df = fma(d, f, df);
    }
    __syncthreads();
    lds_gemm(B2, B1, B3, n, false);          // F D
    lds_load(B3, S, n);
    __syncthreads();
    lds_gemm(B1, B2, B3, n, false);          // F D S
    lds_load(B3, X, n);
    for (int x = t; x < n2; x += kScfThreads) {
        const int i = x / n, j = x % n;
        B2[i * ld + j] = B1[i * ld + j] - B1[j * ld + i];
    }
    __syncthreads();
    lds_gemm(B1, B2, B3, n, false);
    lds_gemm(B2, B3, B1, n, false);          // X (F D S - S D F) X
    double mx = 0.0;
    for (int x = t; x < n2; x += kScfThreads) {
        const double e = B2[x / n * ld + x % n];
        hE[(int64_t)slot * n2 + x] = e;
        mx = fmax(mx, fabs(e));
    }
    dh = block_reduce(dh, false, red);
    df = block_reduce(df, false, red);
    mx = block_reduce(mx, true, red);
    for (int k = 0; k < kDiisMax; ++k) {
        double v = 0.0;
        if ((filled >> k) & 1u) {
            for (int x = t; x < n2; x += kScfThreads) {
                const double e = B2[x / n * ld + x % n];
                v = fma(e, k == slot ? e : hE[(int64_t)k * n2 + x], v);
            }
        }
        v = block_reduce(v, false, red);
        if (t == 0) out[3 + k] = v;
    }
    if (t == 0) {
        out[0] = dh;
        out[1] = df;
        out[2] = mx;
        out[3 + kDiisMax] = (double)*info;
    }
}

// Orbitals of Fx = sum_i c_i F[slot_i]: A = X Fx X in the basis of the last eigenvectors V
// (warm; else of the identity), eigenvalues ascending into eps, V the eigenvectors (columns in
// that order), and with dens the density 2 C_occ C_occ^T of C = X V.
__global__ __launch_bounds__(kScfThreads) void k_small_orbitals(int n, Coefs cf, const double *__restrict__ hist,
                                                                const double *__restrict__ X,
                                                                double *__restrict__ Vg, bool warm, int nocc,
                                                                double *__restrict__ dens, double *__restrict__ eps,
                                                                int *__restrict__ info)
{
    extern __shared__ __attribute__((aligned(16))) double sm[];
    __shared__ double2 cs[kSmallScf / 2];
    __shared__ double red[kScfThreads / kWave];
    __shared__ int rank[kSmallScf];
    const int ld = scf_ld(n), n2 = n * n, t = threadIdx.x;
    double *B1 = sm, *B2 = B1 + n * ld, *B3 = B2 + n * ld;
    for (int x = t; x < n2; x += kScfThreads) {
        double s = 0.0;
        for (int i = 0; i < cf.m; ++i) s += cf.c[i] * hist[(int64_t)cf.slot[i] * n2 + x];
        B1[x / n * ld + x % n] = s;
        B3[x / n * ld + x % n] = X[x];
    }
    __syncthreads();
    lds_gemm(B2, B1, B3, n, false);
    lds_gemm(B1, B3, B2, n, false);          // X Fx X
    if (warm) {
        lds_load(B3, Vg, n);
        __syncthreads();
        lds_gemm(B2, B1, B3, n, false);
        lds_gemm(B1, B3, B2, n, true);       // V^T X Fx X V
    } else {
        for (int x = t; x < n2; x += kScfThreads) B3[x / n * ld + x % n] = x / n == x % n ? 1.0 : 0.0;
    }
    // the rotations take the matrix as symmetric: leave it exactly so
    for (int x = t; x < n2; x += kScfThreads) {
        const int i = x / n, j = x % n;
        B2[i * ld + j] = 0.5 * (B1[i * ld + j] + B1[j * ld + i]);
    }
    __syncthreads();
    const bool ok = lds_jacobi(B2, B3, n, cs, red);
    __syncthreads();
    lds_ranks(B2, n, rank);
    for (int k = t; k < n; k += kScfThreads) eps[rank[k]] = B2[k * ld + k];
    for (int x = t; x < n2; x += kScfThreads) Vg[x / n * n + rank[x % n]] = B3[x / n * ld + x % n];
    if (t == 0) *info = ok ? 0 : 1;
    if (!dens) return;
    __syncthreads();
    lds_load(B2, X, n);
    __syncthreads();
    lds_gemm(B1, B2, B3, n, false);          // C = X V, columns not yet in order
    for (int x = t; x < n2; x += kScfThreads) {
        const int i = x / n, j = x % n;
        double s = 0.0;
        for (int k = 0; k < n; ++k)
            if (rank[k] < nocc) s = fma(B1[i * ld + k], B1[j * ld + k], s);
        dens[x] = 2.0 * s;
    }
}

static size_t small_scf_lds(int64_t n) { return sizeof(double) * 3 * (size_t)n * (size_t)scf_ld((int)n); }

// ------------------------------------------------------------------ layout

ScfLayout make_scf_layout(size_t base, int64_t n)
{
    ScfLayout L;
    size_t o = base;
    auto take = [&](size_t bytes) {
        const size_t at = o;
        o = (o + bytes + 255) & ~(size_t)255;
        return at;
    };
    const size_t n2 = (size_t)n * (size_t)n * sizeof(double);
    L.S = take(n2);
    L.H = take(n2);
    L.X = take(n2);
    L.F = take(n2);
    L.G = take(n2);
    L.Fx = take(n2);
    L.A = take(n2);
    L.C = take(n2);
    L.T1 = take(n2);
    L.T2 = take(n2);
    L.eps = take(sizeof(double) * (size_t)n);
    L.evw = take(sizeof(double) * (size_t)n);
    L.info = take(sizeof(int));
    L.scal = take(sizeof(double) * 32);
    L.Z = take(sizeof(double) * (size_t)n);
    L.diisF = take(n2 * kDiisMax);
    L.diisE = take(n2 * kDiisMax);
    // the eigensolver's scratch grows like n^2 (checked against the library's own query)
    L.rocws_bytes = 4 * n2 + ((size_t)64 << 20);
    L.rocws = take(L.rocws_bytes);
    L.total = o;
    return L;
}

// ------------------------------------------------------------------ the loop

namespace {

struct Ctx {
    rocblas_handle h = nullptr;   // the calling thread's handle for the current device
    hipStream_t st = nullptr;
    int64_t n = 0;
    char *msg = nullptr;
    size_t msglen = 0;
};

// One rocBLAS handle per calling thread and device, created on the first SCF call and kept
// for the life of the thread: creating one per call cost time on every call, and handles are
// not shared between threads.  Each call sets its stream and its workspace before any use.
// The handles are never destroyed (so teardown order at process exit does not matter).
rocblas_handle thread_handle()
{
    thread_local std::vector<rocblas_handle> handles;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0) return nullptr;
    if ((int)handles.size() <= dev) handles.resize(dev + 1, nullptr);
    if (!handles[dev] && rocblas_create_handle(&handles[dev]) != rocblas_status_success) handles[dev] = nullptr;
    return handles[dev];
}

hfk_status say(Ctx &c, hfk_status s, const char *what)
{
    snprintf(c.msg, c.msglen, "%s", what);
    return s;
}

unsigned blocks(int64_t m) { return (unsigned)((m + 255) / 256); }

// C = op(A) op(B) (column-major n x n, inner dimension k).
bool gemm(Ctx &c, bool ta, bool tb, rocblas_int k, const double *A, const double *B, double *C, double alpha = 1.0)
{
    const double beta = 0.0;
    const rocblas_int n = (rocblas_int)c.n;
    return rocblas_dgemm(c.h, ta ? rocblas_operation_transpose : rocblas_operation_none,
                         tb ? rocblas_operation_transpose : rocblas_operation_none, n, n, k, &alpha, A,
                         ta ? k : n, B, tb ? n : k, &beta, C, n) == rocblas_status_success;
}

// Orbitals of Fx: A = X Fx X, eigenpairs (eps ascending, vectors in A), C = X A, and when
// dens is given D = 2 C_occ C_occ^T.
hfk_status diagonalise(Ctx &c, const ScfLayout &SL, char *ws, const double *Fx, int nocc, double *dens)
{
    double *X = (double *)(ws + SL.X), *A = (double *)(ws + SL.A), *C = (double *)(ws + SL.C);
    double *T1 = (double *)(ws + SL.T1);
    if (!gemm(c, false, false, (rocblas_int)c.n, Fx, X, T1) || !gemm(c, false, false, (rocblas_int)c.n, X, T1, A))
        return say(c, HFK_EHIP, "dgemm failed");
    if (rocsolver_dsyevd(c.h, rocblas_evect_original, rocblas_fill_lower, (rocblas_int)c.n, A, (rocblas_int)c.n,
                         (double *)(ws + SL.eps), (double *)(ws + SL.evw), (rocblas_int *)(ws + SL.info)) !=
        rocblas_status_success)
        return say(c, HFK_EHIP, "dsyevd failed");
    if (!gemm(c, false, false, (rocblas_int)c.n, X, A, C)) return say(c, HFK_EHIP, "dgemm failed");
    if (dens) {
        // D = 2 C(:, 0:nocc) C(:, 0:nocc)^T
        const double two = 2.0, zero = 0.0;
        const rocblas_int n = (rocblas_int)c.n;
        if (rocblas_dgemm(c.h, rocblas_operation_none, rocblas_operation_transpose, n, n, (rocblas_int)nocc, &two, C,
                          n, C, n, &zero, dens, n) != rocblas_status_success)
            return say(c, HFK_EHIP, "dgemm failed");
    }
    return HFK_OK;
}

// The status the last symmetric eigensolve left in the workspace (waits for the stream):
// a positive value means it did not converge, as with a matrix that holds NaN or Inf.
hfk_status info_status(Ctx &c, int info)
{
    if (info == 0) return HFK_OK;
    snprintf(c.msg, c.msglen, "the symmetric eigenproblem did not converge (info = %d)", info);
    return HFK_EHIP;
}

hfk_status solver_info(Ctx &c, char *ws, const ScfLayout &SL)
{
    int info = 0;
    if (hipMemcpyAsync(&info, ws + SL.info, sizeof(int), hipMemcpyDeviceToHost, c.st) != hipSuccess ||
        hipStreamSynchronize(c.st) != hipSuccess)
        return say(c, HFK_EHIP, "eigensolver status copy failed");
    return info_status(c, info);
}

// Solves the (m+1) x (m+1) DIIS system by Gaussian elimination with partial pivoting;
// false if it is singular.
bool diis_solve(const std::vector<double> &B, int m, std::vector<double> &coef)
{
    const int N = m + 1;
    std::vector<double> M((size_t)N * (N + 1));
    for (int i = 0; i < N; ++i) {
        for (int j = 0; j < N; ++j) M[i * (N + 1) + j] = (i < m && j < m) ? B[i * kDiisMax + j] : (i == m && j == m ? 0.0 : -1.0);
        M[i * (N + 1) + N] = i == m ? -1.0 : 0.0;
    }
    for (int col = 0; col < N; ++col) {
        int piv = col;
        for (int r = col + 1; r < N; ++r)
            if (fabs(M[r * (N + 1) + col]) > fabs(M[piv * (N + 1) + col])) piv = r;
        if (fabs(M[piv * (N + 1) + col]) < 1e-300) return false;
        if (piv != col)
            for (int k = 0; k <= N; ++k) std::swap(M[col * (N + 1) + k], M[piv * (N + 1) + k]);
        for (int r = 0; r < N; ++r) {
            if (r == col) continue;
            const double f = M[r * (N + 1) + col] / M[col * (N + 1) + col];
            for (int k = col; k <= N; ++k) M[r * (N + 1) + k] -= f * M[col * (N + 1) + k];
        }
    }
    coef.assign(m, 0.0);
    for (int i = 0; i < m; ++i) coef[i] = M[i * (N + 1) + N] / M[i * (N + 1) + i];
    return true;
}

}  // namespace

hfk_status run_scf(const Layout &L, const Basis &b, char *ws, const ScfLayout &SL, const double *xyz,
                   const double *charges_host, int nocc, double tau, int prec, int strat, int max_iter,
                   double e_tol, double d_tol, double *dens, bool use_guess, double *eps_out, ScfResult *res,
                   hipStream_t st, char *msg, size_t msglen)
{
    Ctx c;
    c.st = st;
    c.n = L.n;
    c.msg = msg;
    c.msglen = msglen;
    const int64_t n = L.n, n2 = n * n;
    const bool small = n <= kSmallScf;
    const unsigned lds = (unsigned)(small ? small_scf_lds(n) : 0);
    if (!small) c.h = thread_handle();
    if (!small && !c.h) return say(c, HFK_EHIP, "rocblas_create_handle failed");
    if (!small) {
        if (rocblas_set_stream(c.h, st) != rocblas_status_success)
            return say(c, HFK_EHIP, "rocblas_set_stream failed");
        (void)rocblas_set_pointer_mode(c.h, rocblas_pointer_mode_host);
        // the library scratch comes from the workspace: its own size query first (with the
        // real buffers, which a query does not touch)
        size_t need = 0;
        const double one = 1.0, zero = 0.0;
        const rocblas_int ni = (rocblas_int)n;
        double *qa = (double *)(ws + SL.A), *qb = (double *)(ws + SL.T1), *qc = (double *)(ws + SL.T2);
        (void)rocblas_start_device_memory_size_query(c.h);
        (void)rocsolver_dsyevd(c.h, rocblas_evect_original, rocblas_fill_lower, ni, qa, ni, (double *)(ws + SL.eps),
                               (double *)(ws + SL.evw), (rocblas_int *)(ws + SL.info));
        (void)rocblas_dgemm(c.h, rocblas_operation_none, rocblas_operation_none, ni, ni, ni, &one, qa, ni, qb, ni, &zero,
                            qc, ni);
        if (rocblas_stop_device_memory_size_query(c.h, &need) != rocblas_status_success)
            return say(c, HFK_EHIP, "rocblas memory size query failed");
        if (need > SL.rocws_bytes) return say(c, HFK_ENOMEM, "linear-algebra scratch exceeds its workspace share");
        if (rocblas_set_workspace(c.h, ws + SL.rocws, SL.rocws_bytes) != rocblas_status_success)
            return say(c, HFK_EHIP, "rocblas_set_workspace failed");
    }
    double *S = (double *)(ws + SL.S), *H = (double *)(ws + SL.H), *X = (double *)(ws + SL.X);
    double *F = (double *)(ws + SL.F), *G = (double *)(ws + SL.G), *Fx = (double *)(ws + SL.Fx);
    double *A = (double *)(ws + SL.A), *T1 = (double *)(ws + SL.T1), *T2 = (double *)(ws + SL.T2);
    double *Z = (double *)(ws + SL.Z), *scal = (double *)(ws + SL.scal), *eps = (double *)(ws + SL.eps);
    double *hF = (double *)(ws + SL.diisF), *hE = (double *)(ws + SL.diisE);
    hipError_t e = hipMemcpyAsync(Z, charges_host, sizeof(double) * n, hipMemcpyHostToDevice, st);
    if (e != hipSuccess) return say(c, HFK_EHIP, "charges copy failed");
    hipLaunchKernelGGL(k_one_electron, dim3(blocks(kOneLanes * (n * (n + 1) / 2))), dim3(256), 0, st, n, b.g, xyz, Z, b.aexp,
                       b.aw, S, H);
    hipLaunchKernelGGL(k_enuc, dim3(1), dim3(256), 0, st, n, xyz, Z, scal);
    if ((e = hipGetLastError()) != hipSuccess) return say(c, HFK_EHIP, "integral launch failed");
    double enn = 0.0;
    hfk_status s_ok = HFK_OK;
    int *info_dev = (int *)(ws + SL.info);
    bool warm = false;
    int solves = 0;
    // one workgroup: orbitals of the combination cf of `hist`, from the last eigenvectors, and
    // from the identity every eighth time (the rotations' rounding does not pile up)
    auto small_orbitals = [&](const Coefs &cf, const double *hist, double *out_dens) {
        hipLaunchKernelGGL(k_small_orbitals, dim3(1), dim3(kScfThreads), lds, st, (int)n, cf, hist, (const double *)X, A,
                           warm, nocc, out_dens, eps, info_dev);
        warm = ++solves % 8 != 0;
    };
    Coefs self;
    memset(&self, 0, sizeof(self));
    self.c[0] = 1.0;
    self.m = 1;
    if (small) {
        hipLaunchKernelGGL(k_small_invsqrt, dim3(1), dim3(kScfThreads), lds, st, (int)n, (const double *)S, X, scal);
        double sv[4];
        if (hipGetLastError() != hipSuccess ||
            hipMemcpyAsync(sv, scal, sizeof(sv), hipMemcpyDeviceToHost, st) != hipSuccess ||
            hipStreamSynchronize(st) != hipSuccess)
            return say(c, HFK_EHIP, "overlap eigenvalue copy failed");
        enn = sv[0];
        if (sv[3] != 0.0) return info_status(c, (int)sv[3]);
        if (!(sv[1] > 1e-12 * sv[2])) return say(c, HFK_EUNSUPPORTED, "overlap matrix is (nearly) singular");
        if (!use_guess) small_orbitals(self, H, dens);
    } else {
    if (hipMemcpyAsync(&enn, scal, sizeof(double), hipMemcpyDeviceToHost, st) != hipSuccess ||
        hipStreamSynchronize(st) != hipSuccess)
        return say(c, HFK_EHIP, "nuclear repulsion copy failed");

    // X = S^(-1/2) = U s^(-1/2) U^T
    if (hipMemcpyAsync(A, S, sizeof(double) * n2, hipMemcpyDeviceToDevice, st) != hipSuccess)
        return say(c, HFK_EHIP, "copy failed");
    if (rocsolver_dsyevd(c.h, rocblas_evect_original, rocblas_fill_lower, (rocblas_int)n, A, (rocblas_int)n, eps,
                         (double *)(ws + SL.evw), (rocblas_int *)(ws + SL.info)) != rocblas_status_success)
        return say(c, HFK_EHIP, "dsyevd failed");
    {
        std::vector<double> s(n);
        if (hipMemcpyAsync(s.data(), eps, sizeof(double) * n, hipMemcpyDeviceToHost, st) != hipSuccess ||
            hipStreamSynchronize(st) != hipSuccess)
            return say(c, HFK_EHIP, "eigenvalue copy failed");
        if ((s_ok = solver_info(c, ws, SL)) != HFK_OK) return s_ok;
        if (!(s[0] > 1e-12 * s[n - 1])) return say(c, HFK_EUNSUPPORTED, "overlap matrix is (nearly) singular");
    }
    hipLaunchKernelGGL(k_scale_cols, dim3(blocks(n2)), dim3(256), 0, st, n, A, eps, T1);
    if (!gemm(c, false, true, (rocblas_int)n, T1, A, X)) return say(c, HFK_EHIP, "dgemm failed");

    if (!use_guess && (s_ok = diagonalise(c, SL, ws, H, nocc, dens)) != HFK_OK) return s_ok;
    }
    if (small && use_guess) {
        // no eigenproblem has been solved yet: its status reads as success
        hipLaunchKernelGGL(k_clear_info, dim3(1), dim3(1), 0, st, info_dev);
    }

    std::vector<double> B((size_t)kDiisMax * kDiisMax, 0.0);
    std::vector<int> age(kDiisMax, -1);   // iteration that filled each slot, -1 empty
    double e_old = 0.0, E = 0.0;
    bool have_old = false, conv = false;
    int it = 0;
    double *e2tmp = scal + 1;
    const PairPlan plan = fock_plan(L, ws, strat, prec, 1);
    for (it = 1; it <= max_iter; ++it) {
        // G(D), F = H + G
        // the pairs, their order and tables depend on the geometry only: later builds take the
        // new density on the tables of the first
        hipError_t ef = it == 1 ? launch_pairs(L, b, ws, xyz, dens, tau, prec, plan, st)
                                : launch_new_density(L, ws, dens, plan, st);
        if (ef == hipSuccess) ef = launch_fock(L, b, ws, dens, tau, prec, strat, 1, G, e2tmp, st);
        if (ef != hipSuccess) return say(c, HFK_EHIP, "Fock build failed");
        // e = X (F D S - S D F) X into the history slot of the oldest entry
        int slot = 0;
        for (int k = 0; k < kDiisMax; ++k)
            if (age[k] < age[slot]) slot = k;
        double *ek = hE + (int64_t)slot * n2;
        age[slot] = it;
        unsigned filled = 0;
        for (int k = 0; k < kDiisMax; ++k)
            if (age[k] >= 0) filled |= 1u << k;
        if (small) {
            hipLaunchKernelGGL(k_small_error, dim3(1), dim3(kScfThreads), lds, st, (int)n, (const double *)H,
                               (const double *)G, (const double *)dens, (const double *)S, (const double *)X, F, hF, hE,
                               slot, filled, (const int *)info_dev, scal + 8);
        } else {
        hipLaunchKernelGGL(k_add, dim3(blocks(n2)), dim3(256), 0, st, n2, H, G, F);
        if (!gemm(c, false, false, (rocblas_int)n, F, dens, T1) || !gemm(c, false, false, (rocblas_int)n, T1, S, T2))
            return say(c, HFK_EHIP, "dgemm failed");
        hipLaunchKernelGGL(k_antisym, dim3(blocks(n2)), dim3(256), 0, st, n, T2, T1);
        if (!gemm(c, false, false, (rocblas_int)n, T1, X, T2) || !gemm(c, false, false, (rocblas_int)n, X, T2, ek))
            return say(c, HFK_EHIP, "dgemm failed");
        if (hipMemcpyAsync(hF + (int64_t)slot * n2, F, sizeof(double) * n2, hipMemcpyDeviceToDevice, st) != hipSuccess)
            return say(c, HFK_EHIP, "copy failed");
        // E = 1/2 (<D, H> + <D, F>) + E_nn, max |e| and the new row of the DIIS matrix, read
        // back with one wait
        hipLaunchKernelGGL(k_scf_scalars, dim3(3 + kDiisMax), dim3(256), 0, st, n2, dens, H, F, ek, hE, filled,
                           scal + 8);
        }
        // with the status of the last eigensolve: the one whose orbitals gave this density
        double sc[4 + kDiisMax];
        int info = 0;
        if (hipGetLastError() != hipSuccess ||
            hipMemcpyAsync(sc, scal + 8, sizeof(sc), hipMemcpyDeviceToHost, st) != hipSuccess ||
            (!small && hipMemcpyAsync(&info, ws + SL.info, sizeof(int), hipMemcpyDeviceToHost, st) != hipSuccess) ||
            hipStreamSynchronize(st) != hipSuccess)
            return say(c, HFK_EHIP, "scalar copy failed");
        if (small) info = (int)sc[3 + kDiisMax];
        if ((s_ok = info_status(c, info)) != HFK_OK) return s_ok;
        E = 0.5 * (sc[0] + sc[1]) + enn;
        const double emax = sc[2];
        for (int k = 0; k < kDiisMax; ++k)
            if (age[k] >= 0) B[slot * kDiisMax + k] = B[k * kDiisMax + slot] = sc[3 + k];
        if (have_old && fabs(E - e_old) < e_tol && emax < d_tol) {
            conv = true;
            break;
        }
        // the last build allowed: its density is the one whose energy is E (no further
        // eigensolve, which could also leave a failed solve behind the returned density)
        if (it == max_iter) break;
        // DIIS over the filled slots (oldest first), else F itself
        std::vector<int> order;
        for (int k = 0; k < kDiisMax; ++k)
            if (age[k] >= 0) order.push_back(k);
        std::sort(order.begin(), order.end(), [&](int x, int y) { return age[x] < age[y]; });
        const double *Fuse = F;
        Coefs use = self;
        if (order.size() >= 2) {
            const int m = (int)order.size();
            std::vector<double> Bm((size_t)kDiisMax * kDiisMax, 0.0), coef;
            for (int i = 0; i < m; ++i)
                for (int j = 0; j < m; ++j) Bm[i * kDiisMax + j] = B[order[i] * kDiisMax + order[j]];
            if (diis_solve(Bm, m, coef)) {
                Coefs cf;
                cf.m = m;
                for (int i = 0; i < m; ++i) {
                    cf.c[i] = coef[i];
                    cf.slot[i] = order[i];
                }
                use = cf;
                Fuse = Fx;
                if (!small) hipLaunchKernelGGL(k_lincomb, dim3(blocks(n2)), dim3(256), 0, st, n2, cf, hF, Fx);
            }
        }
        if (small)
            small_orbitals(use, Fuse == F ? (const double *)F : (const double *)hF, dens);
        else if ((s_ok = diagonalise(c, SL, ws, Fuse, nocc, dens)) != HFK_OK)
            return s_ok;
        e_old = E;
        have_old = true;
    }
    if (it > max_iter) it = max_iter;
    // orbital energies of the final F (the density stays the one that built it)
    if (small)
        small_orbitals(self, F, nullptr);
    else if ((s_ok = diagonalise(c, SL, ws, F, nocc, nullptr)) != HFK_OK)
        return s_ok;
    if (eps_out && hipMemcpyAsync(eps_out, eps, sizeof(double) * n, hipMemcpyDeviceToDevice, st) != hipSuccess)
        return say(c, HFK_EHIP, "eigenvalue copy failed");
    if (hipStreamSynchronize(st) != hipSuccess) return say(c, HFK_EHIP, "stream sync failed");
    if ((s_ok = solver_info(c, ws, SL)) != HFK_OK) return s_ok;
    res->energy = E;
    res->iterations = it;
    res->converged = conv ? 1 : 0;
    return HFK_OK;
}

}  // namespace hfk
