// FP64 symmetric eigensolver of the projector stage (Sec. 3: the projectors
// of the scheme it cites come from the singular triplets of one matrix per
// sector of the cut; here they are taken from a symmetric eigenproblem, the
// Gram matrix Y Y^T or the Jordan-Wielandt matrix [[0, Y], [Y^T, 0]]).
//
// Four steps, each one launch over every matrix of a cut:
//   1. Householder tridiagonalisation T = Q^T A Q (Q = H_0 ... H_{n-3},
//      H_k = I - tau_k v_k v_k^T).  The rows of a matrix are spread over the
//      workgroups of one job, cyclically (row i on workgroup i mod G), and
//      stay in registers for the whole reduction.  The rank-2 update of
//      column k, A -= v w^T + w v^T, is applied lazily: each workgroup applies
//      it to its own rows in the pass of column k+1 that also forms
//      p = tau A v, so one column costs one exchange between the job's
//      workgroups (its p slices and the next row, through global memory).
//      The jobs of a launch sit on disjoint workgroups, each job on the
//      workgroups of one XCD where it fits.
//   2. All eigenvalues by multisection: counts on a grid common to all, then
//      one wavefront per eigenvalue, its 64 lanes evaluating Sturm counts of T
//      at 64 points of the current interval, about 7 passes to 2 ulp.
//   3. Eigenvectors of T for the kept eigenvalues from the twisted
//      factorisation of T - lam I (two recurrences at once, no iteration), a
//      workgroup each.  Eigenvalues closer than 1e-3 ||T|| form a cluster,
//      gone through in order by one wavefront: each vector has the earlier
//      ones projected out, and if less than half of it is left (a degenerate
//      value) it comes from inverse iteration instead (tridiagonal LU with
//      partial pivoting, two solves from a fixed pseudo-random start,
//      reorthogonalised in every solve).  What is left of the products of
//      close vectors is taken out in one pass over all (polish_kernel).
//   4. Back-transformation z <- Q z through the stored reflectors, a vector
//      in the registers of one wavefront (four above n = 704).
// The matrix is scaled by a power of two (exact) so that its largest entry
// is in [1, 2); eigenvalues are returned unscaled.
#include <algorithm>
#include <array>
#include <cfloat>
#include <cmath>
#include <cstring>
#include <map>
#include <mutex>
#include <set>
#include <vector>

#include "internal.hpp"

namespace symten {
namespace {

constexpr int kEigThreads = 256;                 // bisection: four eigenvalues per workgroup
constexpr int kEigWaves = kEigThreads / 64;
constexpr int kSpinLimit = 1 << 21;     // polls of an exchange before it gives up

__host__ __device__ inline int v_stride(int n) { return (n + 63) & ~63; }

struct TridJob {
    const double* A;                   // n x n, column-major (ld lda), both triangles
    int n, lda, G;                     // order, leading dim, workgroups
    double *d, *e, *e2, *tau, *V, *scale;   // outputs (scaled by *scale; e2: coupling2 of e); V: reflector k in row k, stride v_stride(n),
                                       // zeros outside its entries k+1 .. n-1
    double* xbuf;                      // exchange area (xbuf_doubles), filled with kEmpty
    int* status;                       // set to 1 if an exchange gave up
    int variant;                       // index into kTridVariants
};

// Wavefront reductions on DPP lane moves (no LDS round trips): within
// rows of 16 lanes by quad permutations and row mirrors, across rows by the
// row broadcasts of lanes 15 and 31, so that lane 63 holds the result, which
// every lane then reads.  Lanes a DPP move has no source for contribute 0
// (the identity of both reductions below, since max is taken of |x| >= 0 or
// of values whose identity the caller supplies as 0).
template <int CTRL, int ROWS>
__device__ inline double dpp_move(double x) {
    const uint64_t u = __builtin_bit_cast(uint64_t, x);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, CTRL, ROWS, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), CTRL, ROWS, 0xF, false);
    return __builtin_bit_cast(double, ((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo);
}
__device__ inline double lane63(double x) {
    const uint64_t u = __builtin_bit_cast(uint64_t, x);
    const uint32_t lo = __builtin_amdgcn_readlane((int)(uint32_t)u, 63);
    const uint32_t hi = __builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), 63);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
__device__ inline double wave_sum(double x) {
    x += dpp_move<0xB1, 0xF>(x);    // quad_perm [1,0,3,2]
    x += dpp_move<0x4E, 0xF>(x);    // quad_perm [2,3,0,1]
    x += dpp_move<0x141, 0xF>(x);   // row_half_mirror
    x += dpp_move<0x140, 0xF>(x);   // row_mirror: every lane holds its row's sum
    x += dpp_move<0x142, 0xA>(x);   // row_bcast:15 into rows 1, 3
    x += dpp_move<0x143, 0xC>(x);   // row_bcast:31 into rows 2, 3
    return lane63(x);
}
// maximum of values >= 0
__device__ inline double wave_max(double x) {
    x = fmax(x, dpp_move<0xB1, 0xF>(x));
    x = fmax(x, dpp_move<0x4E, 0xF>(x));
    x = fmax(x, dpp_move<0x141, 0xF>(x));
    x = fmax(x, dpp_move<0x140, 0xF>(x));
    x = fmax(x, dpp_move<0x142, 0xA>(x));
    x = fmax(x, dpp_move<0x143, 0xC>(x));
    return lane63(x);
}
// Sum (or max) over the workgroup of NW waves, in a fixed order; every
// thread gets it.
template <int NW>
__device__ double block_sum(double x, double* red) {
    x = wave_sum(x);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = x;
    __syncthreads();
    double s = 0.0;
#pragma unroll
    for (int i = 0; i < NW; ++i) s += red[i];
    __syncthreads();
    return s;
}
template <int NW>
__device__ double block_max(double x, double* red) {
    x = wave_max(x);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = x;
    __syncthreads();
    double s = 0.0;
#pragma unroll
    for (int i = 0; i < NW; ++i) s = fmax(s, red[i]);
    __syncthreads();
    return s;
}

// Sums of four per-lane values over the wavefront: the rows share the two
// widest exchange steps (v_permlane32_swap / v_permlane16_swap trade halves
// between two registers, so adding the pair sums both rows at once), then
// each 16-lane group finishes one row with DPP moves: 21 instructions against
// 72 for four separate sums.  Lane group q = lane / 16 gets the sum of row
// reduced_row(q).
constexpr int kRowGroup = 4, kColGroup = 3;
template <bool W32>
__device__ inline void swap_halves(double& x, double& y) {
    const uint64_t a = __builtin_bit_cast(uint64_t, x), b = __builtin_bit_cast(uint64_t, y);
    uint64_t l, h;
    if constexpr (W32) {
        const auto lo = __builtin_amdgcn_permlane32_swap((uint32_t)a, (uint32_t)b, false, false);
        const auto hi = __builtin_amdgcn_permlane32_swap((uint32_t)(a >> 32), (uint32_t)(b >> 32), false, false);
        l = ((uint64_t)(uint32_t)hi[0] << 32) | (uint32_t)lo[0];
        h = ((uint64_t)(uint32_t)hi[1] << 32) | (uint32_t)lo[1];
    } else {
        const auto lo = __builtin_amdgcn_permlane16_swap((uint32_t)a, (uint32_t)b, false, false);
        const auto hi = __builtin_amdgcn_permlane16_swap((uint32_t)(a >> 32), (uint32_t)(b >> 32), false, false);
        l = ((uint64_t)(uint32_t)hi[0] << 32) | (uint32_t)lo[0];
        h = ((uint64_t)(uint32_t)hi[1] << 32) | (uint32_t)lo[1];
    }
    x = __builtin_bit_cast(double, l);
    y = __builtin_bit_cast(double, h);
}
__device__ inline double four_sums(const double (&x)[kRowGroup]) {
    double y0 = x[0], t0 = x[1], y1 = x[2], t1 = x[3];
    swap_halves<true>(y0, t0);
    swap_halves<true>(y1, t1);
    y0 += t0;   // lanes 0..31: row 0, 32..63: row 1
    y1 += t1;
    swap_halves<false>(y0, y1);
    double z = y0 + y1;   // 16-lane groups: rows 0, 2, 1, 3
    z += dpp_move<0xB1, 0xF>(z);
    z += dpp_move<0x4E, 0xF>(z);
    z += dpp_move<0x141, 0xF>(z);
    z += dpp_move<0x140, 0xF>(z);
    return z;
}
__device__ inline int reduced_row(int group) { return 2 * (group & 1) + (group >> 1); }

// Exchange between the workgroups of a job.  Every value has a slot of its
// own in an area filled with kEmpty, written once; readers poll the slots
// themselves, so there is no counter, no barrier between workgroups and no
// wait for a store.  kEmpty is a signalling NaN: every exchanged value is the
// result of an FP64 operation, which never is one.  Readers use agent-scope
// loads, which are served by L2 and not by a compute unit's L1.  While all
// workgroups of a job run on one XCD (same XCC_ID register), a store that
// reaches that XCD's L2 is enough; otherwise stores are agent-scope too.
// Measured per exchange of 696 values among 32 workgroups of one XCD: 1.0 us
// (1.6 us with an atomic counter and plain loads); 3136 values among 128
// workgroups over all XCDs: 2.1 us (3.5 us with the counter).  Polls are
// bounded: after kSpinLimit of them the workgroup records the failure and
// waits no more, so the launch always ends.
constexpr uint64_t kEmpty = 0xFFF4DEADBEEF5A5Aull;
// The job's pointers come out of memory, so their address space is stated:
// flat accesses would count as LDS accesses too, and every LDS wait would wait
// for the exchange.  32-bit offsets from a wavefront-uniform base keep an
// address in one register.
#ifdef __HIP_DEVICE_COMPILE__
#define GLOBAL_MEM __attribute__((address_space(1)))
#define LOCAL_MEM __attribute__((address_space(3)))
#else
#define GLOBAL_MEM
#define LOCAL_MEM
#endif
typedef GLOBAL_MEM uint64_t gu64;
typedef GLOBAL_MEM double gf64;
template <class P>
__device__ inline P* at8(P* base, uint32_t idx) {
    return (P*)((GLOBAL_MEM char*)base + 8 * idx);
}
template <bool LOCAL>
__device__ inline void put_x(gu64* base, uint32_t idx, double v) {
    __hip_atomic_store(at8(base, idx), __builtin_bit_cast(uint64_t, v), __ATOMIC_RELAXED,
                       LOCAL ? __HIP_MEMORY_SCOPE_WORKGROUP : __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline void put_x(gu64* base, uint32_t idx, double v, bool local) {
    if (local) put_x<true>(base, idx, v);
    else put_x<false>(base, idx, v);
}
__device__ inline uint64_t get_x(gu64* base, uint32_t idx) {
    return __hip_atomic_load(at8(base, idx), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// 1/x and 1/sqrt(x) of a normal, positive x: the hardware's approximation and
// two Newton steps
__device__ inline double rcp_newton(double x) {
    double r = __builtin_amdgcn_rcp(x);
    r = fma(r, fma(-x, r, 1.0), r);
    return fma(r, fma(-x, r, 1.0), r);
}
__device__ inline double rsq_newton(double x) {
    double y = __builtin_amdgcn_rsq(x);
    y = fma(0.5 * y, fma(-x * y, y, 1.0), y);
    return fma(0.5 * y, fma(-x * y, y, 1.0), y);
}
// Householder vector of a column with leading entry alpha and squared norm
// xn2 of the rest: beta, tau and the factor of the rest.  A rest below
// 2^-480 of the scaled matrix counts as zero.
__device__ inline void householder(double alpha, double xn2, double& beta, double& tau, double& scal) {
    beta = alpha;
    tau = scal = 0.0;
    if (xn2 > 0x1p-960) {
        const double h2 = fma(alpha, alpha, xn2), y = rsq_newton(h2);
        double h = h2 * y;
        h = fma(0.5 * y, fma(-h, h, h2), h);
        beta = -copysign(h, alpha);
        tau = fma(fabs(alpha), y, 1.0);                       // (beta - alpha) / beta
        scal = copysign(rcp_newton(fabs(alpha) + h), alpha);  // 1 / (alpha - beta)
    }
}
// Square of an off-diagonal entry of T as the Sturm counts take it: never
// zero, so that a product that comes out as exactly zero does not end the
// sequence (entries of T are at most 2^13, so 2^-100 is no change of T).
__device__ inline double coupling2(double e) { return fmax(e * e, 0x1p-200); }

__global__ void fill_empty_kernel(uint64_t* __restrict__ d, int64_t n) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        d[i] = kEmpty;
}

// Step 1 for one workgroup g of a job.  The matrix stays in registers: the
// NW waves form WR row groups of WC waves; wave (wr, wc) holds, for its RW
// rows i = g + G (wr + WR s), the columns j = lane + 64 (wc + WC c), c < CW
// (the last RL rows in LDS where the registers do not take them all), and the
// entries of v and w at those columns.  Thread tid owns the columns
// j = tid + T q of the column vectors.  Per column k:
//  (a) the Householder vector from the column, each thread its entries, and
//      {w, v} to every wave through LDS;
//  (b) one pass over the rows i > k that applies the pending rank-2 update of
//      column k-1 and forms p_i = tau (row_i . v); the owner of row k+1
//      publishes it;
//  (c) every thread polls its entries of p and of row k+1;
//  (d) w = p - (tau/2)(p.v) v is the pending update, and row k+1 with it the
//      next column.
// It is bound by this serial chain, not by arithmetic or memory.  At n = 696
// (29 workgroups of one XCD) a column takes 2.5 us: 0.7 us of exchange, 0.5 us
// for the pass, the rest the four LDS rounds (two sums, two broadcasts); the
// reduction 1.74 ms.  With the rows in LDS and an atomic counter as barrier
// the pass read and wrote 150 KB of LDS per column, and the reduction took
// 3.5 ms.  At n = 2624 (175 workgroups over all XCDs) 6 us per column, 16 ms;
// there the exchange is bound by the reads that pass the L2s (1.4 TB/s), so
// slots of finished columns are not polled (20 ms with them).  Four waves per
// workgroup where the registers allow it (n <= 704): eight read the {w, v}
// pairs twice as often.
template <int T, int WC, int CW, int RW, int RL = 0>
struct Trid {
    static constexpr int NW = T / 64, WR = NW / WC, R = RW * WR;
    static constexpr int RR = RW - RL;                  // rows of a wave in registers; RL in LDS
    static constexpr int NP = 64 * WC * CW;             // columns, padded
    static constexpr int PQ = (CW + WR - 1) / WR;       // columns exchanged per thread
    static constexpr int NQ = T * PQ;                   // exchanged columns, padded to threads
    static constexpr bool SOLO = R >= NP;               // the job has one workgroup: no exchange
    // LDS, in doubles: p (one workgroup: the raw p and row k+1 too) and the
    // next column; {v, w} of the own rows (and a slot per lane for the rest);
    // {w, v} of all columns; sums and partial row sums
    static constexpr int LP = 0, LX = LP + NQ, LOWN = LX + NQ, LVW = LOWN + 2 * (R + 64),
                         LRAW = LVW + (WR > 1 ? 2 * NQ : 0), LRED = LRAW + (SOLO ? 2 * NP : 0), LPART = LRED + 2 * NW,
                         LFAIL = LPART + (WC > 1 ? NW * (RW + 3) : 0), LROW = LFAIL + 2, LDS = LROW + WR * RL * NP;
    static_assert(WC * WR == NW, "waves form a grid");
    static_assert(256 * R <= 65536 && R + 64 < 65536, "places are 16 bits");

    static __device__ __forceinline__ void columns(const TridJob& J, const int g, double* sm, double (&a)[RR][CW],
                                                   const double sc, const bool local) {
        const int n = J.n, G = SOLO ? 1 : J.G, ldv = v_stride(n);
        const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
        const int wc = w % WC, wr = w / WC;
        double* part_s = sm + LPART;
        double* rows = sm + LROW + wr * RL * NP + lane + 64 * wc;   // this lane's entries of the LDS rows
        const int gr = (G * R + 15) & ~15, region = gr + NP;   // per column: p slices, then row k+1
        gu64* reg = (gu64*)J.xbuf + ((2 * G + 15) & ~15);
        const gf64* A = (const gf64*)J.A;
        gf64 *V = (gf64*)J.V, *Jd = (gf64*)J.d, *Je = (gf64*)J.e, *Jtau = (gf64*)J.tau;
        auto* failed = (LOCAL_MEM volatile int*)(sm + LFAIL);
        // sum over the workgroup's threads, in a fixed order
        auto put_sum = [&](double x, int at) {
            x = wave_sum(x);
            if (lane == 0) sm[at + w] = x;
        };
        auto get_sum = [&](int at) {
            double x = 0.0;
#pragma unroll
            for (int q = 0; q < NW; ++q) x += sm[at + q];
            return x;
        };
        // this thread's exchanged columns: x the next column, v, w; place:
        // their p slot and, above it, their place among the own rows
        double x[PQ], vq[PQ], wq[PQ];
        uint32_t place[PQ];
        double part = 0.0;
#pragma unroll
        for (int q = 0; q < PQ; ++q) {
            const int j = tid + T * q, jc = min(j, n - 1), r = jc / G;
            x[q] = j < n ? A[j] * sc : 0.0;   // column 0
            const double y = j >= 2 ? x[q] : 0.0;
            part = fma(y, y, part);
            vq[q] = wq[q] = 0.0;
            place[q] = ((jc - r * G) * R + r) | (j < n && jc - r * G == g ? (r % WR) * RW + r / WR : R + lane) << 16;
        }
        for (int j = tid; j < 2 * (R + 64); j += T) sm[LOWN + j] = 0.0;   // column -1 leaves no update
        double v[CW], vA[CW], wA[CW];   // v of column k; v and w of column k-1
#pragma unroll
        for (int c = 0; c < CW; ++c) v[c] = vA[c] = wA[c] = 0.0;
        int own = G > 1 ? 1 : 0, own_r = G > 1 ? 0 : 1;   // workgroup and local row of row k+1
        int own_k = 0;                                    // workgroup that stores column k
#pragma unroll 1
        for (int k = 0; k + 1 < n; ++k) {
            __asm__("" : "+s"(reg), "+s"(V));   // scalar bases: no per-lane address carried round the loop
            // (a) Householder vector of column k
#pragma unroll
            for (int q = 0; q < PQ; ++q) sm[LX + tid + T * q] = x[q];
            put_sum(part, LRED + NW);
            __syncthreads();
            const double dk = sm[LX + k], alpha = sm[LX + k + 1], xn2 = get_sum(LRED + NW);
            double beta, tau, scal;
            householder(alpha, xn2, beta, tau, scal);
#pragma unroll
            for (int q = 0; q < PQ; ++q) vq[q] = tid + T * q > k + 1 && (T * (q + 1) <= NP || tid + T * q < NP)
                                                     ? x[q] * scal
                                                     : (tid + T * q == k + 1 ? 1.0 : 0.0);
            const int c_lo = max(k + 1 - 64 * wc, 0) / (64 * WC);   // columns j > k: slots c >= c_lo
            if constexpr (WR > 1) {
#pragma unroll
                for (int q = 0; q < PQ; ++q)
                    *(double2*)(sm + LVW + 2 * (tid + T * q)) = make_double2(wq[q], vq[q]);
                __syncthreads();
#pragma unroll
                for (int c0 = 0; c0 < CW; c0 += kColGroup) {
                    if (c0 + kColGroup > c_lo) {
#pragma unroll
                        for (int c = c0; c < c0 + kColGroup && c < CW; ++c) {
                            const double2 wv = *(const double2*)(sm + LVW + 2 * (lane + 64 * (wc + WC * c)));
                            vA[c] = v[c];
                            wA[c] = wv.x;
                            v[c] = wv.y;
                        }
                    }
                }
            } else {
#pragma unroll
                for (int c = 0; c < CW; ++c) {
                    vA[c] = v[c];
                    wA[c] = wq[c];
                    v[c] = vq[c];
                }
            }
            if (SOLO || g == own_k) {
#pragma unroll
                for (int q = 0; q < PQ; ++q)
                    if (64 * w + T * q < ldv) *at8(V, tid + T * q) = vq[q];
                if (tid == 0) {
                    Jd[k] = dk;
                    Je[k] = beta;
                    ((gf64*)J.e2)[k] = coupling2(beta);
                    Jtau[k] = tau;
                }
            }
            V += ldv;
            // (b) own rows i > k: slots s >= s_lo
            const int s_lo = (max(own_r + (g < own ? 1 : 0) - wr, 0) + WR - 1) / WR;
#pragma unroll
            for (int s0 = 0; s0 < RW; s0 += kRowGroup) {
                if (s0 + kRowGroup > s_lo) {
                    double vu[kRowGroup], wu[kRowGroup], acc[kRowGroup];
#pragma unroll
                    for (int u = 0; u < kRowGroup; ++u) {
                        acc[u] = 0.0;
                        if (s0 + u < RW) {
                            const double2 t = *(const double2*)(sm + LOWN + 2 * (wr * RW + s0 + u));
                            vu[u] = t.x;
                            wu[u] = t.y;
                        }
                    }
#pragma unroll
                    for (int c0 = 0; c0 < CW; c0 += kColGroup) {
                        if (c0 + kColGroup > c_lo) {
#pragma unroll
                            for (int c = c0; c < c0 + kColGroup && c < CW; ++c) {
#pragma unroll
                                for (int u = 0; u < kRowGroup && s0 + u < RW; ++u) {
                                    double y = s0 + u < RR ? a[min(s0 + u, RR - 1)][c]
                                                           : rows[(s0 + u - RR) * NP + 64 * WC * c];
                                    y = fma(-vu[u], wA[c], y);
                                    y = fma(-wu[u], vA[c], y);
                                    if (s0 + u < RR) a[min(s0 + u, RR - 1)][c] = y;
                                    else rows[(s0 + u - RR) * NP + 64 * WC * c] = y;
                                    acc[u] = fma(y, v[c], acc[u]);
                                }
                            }
                        }
                    }
                    const double z = four_sums(acc);
                    const int s = s0 + reduced_row(lane >> 4);
                    if ((lane & 15) == 0 && s < RW) {
                        if constexpr (WC > 1) part_s[w * (RW + 3) + s] = z;
                        else if constexpr (SOLO) sm[LRAW + wr + WR * s] = tau * z;
                        else put_x(reg, g * R + wr + WR * s, tau * z, local);
                    }
                }
            }
            if (g == own && own_r % WR == wr) {   // publish row k+1
                const int sp = own_r / WR;
                if constexpr (RL > 0)
                    if (sp >= RR) {
#pragma unroll
                        for (int c = 0; c < CW; ++c)
                            put_x(reg + gr, lane + 64 * (wc + WC * c), rows[(sp - RR) * NP + 64 * WC * c], local);
                    }
#pragma unroll
                for (int s = 0; s < RR; ++s) {
                    if (s == sp) {
                        if (SOLO) {
#pragma unroll
                            for (int c = 0; c < CW; ++c) sm[LRAW + NP + lane + 64 * (wc + WC * c)] = a[s][c];
                        } else if (local) {
#pragma unroll
                            for (int c = 0; c < CW; ++c) put_x<true>(reg + gr, lane + 64 * (wc + WC * c), a[s][c]);
                        } else {
#pragma unroll
                            for (int c = 0; c < CW; ++c) put_x<false>(reg + gr, lane + 64 * (wc + WC * c), a[s][c]);
                        }
                    }
                }
            }
            if constexpr (WC > 1) {
                __syncthreads();
                if (tid < R) {   // local row tid = (row group tid % WR, slot tid / WR)
                    double y = 0.0;
#pragma unroll
                    for (int q = 0; q < WC; ++q) y += part_s[((tid % WR) * WC + q) * (RW + 3) + tid / WR];
                    put_x(reg, g * R + tid, tau * y, local);
                }
            }
            // (c) this thread's columns of p and of row k+1
            double pr[PQ], rr[PQ];
            if constexpr (SOLO) {
                __syncthreads();
#pragma unroll
                for (int q = 0; q < PQ; ++q) {
                    pr[q] = sm[LRAW + min(tid + T * q, NP - 1)];
                    rr[q] = sm[LRAW + NP + min(tid + T * q, NP - 1)];
                }
            } else {
                // slots of a wave without a column in k+1 .. n-1 are left out
                uint64_t pu[PQ], ru[PQ];
#pragma unroll
                for (int q = 0; q < PQ; ++q) pu[q] = ru[q] = 0;
                for (int polls = 0;;) {
                    bool empty = false;
#pragma unroll
                    for (int q = 0; q < PQ; ++q) {
                        if (T * q + 64 * w + 63 > k && T * q + 64 * w < n) {
                            pu[q] = get_x(reg, place[q] & 0xffff);
                            ru[q] = get_x(reg + gr, tid + T * q);
                        }
                    }
#pragma unroll
                    for (int q = 0; q < PQ; ++q)
                        empty |= (pu[q] == kEmpty && (unsigned)(tid + T * q - k - 1) < (unsigned)(n - k - 1)) ||
                                 ru[q] == kEmpty;
                    if (!__any(empty) || *failed) break;
                    if (++polls > kSpinLimit) {
                        *failed = 1;
                        break;
                    }
                }
#pragma unroll
                for (int q = 0; q < PQ; ++q) {
                    pr[q] = __builtin_bit_cast(double, pu[q]);
                    rr[q] = __builtin_bit_cast(double, ru[q]);
                }
                reg += region;
            }
            part = 0.0;
#pragma unroll
            for (int q = 0; q < PQ; ++q) {
                pr[q] = (unsigned)(tid + T * q - k - 1) < (unsigned)(n - k - 1) ? pr[q] : 0.0;
                part = fma(pr[q], vq[q], part);
                sm[LP + tid + T * q] = pr[q];
            }
            put_sum(part, LRED);
            __syncthreads();
            // (d) w, the pending update, and the next column
            const double c2 = 0.5 * tau * get_sum(LRED), w1 = sm[LP + k + 1] - c2;   // (v's entry k+1 is 1)
            part = 0.0;
#pragma unroll
            for (int q = 0; q < PQ; ++q) {
                wq[q] = fma(-c2, vq[q], pr[q]);
                x[q] = fma(-vq[q], w1, rr[q]) - wq[q];
                // (row k+1 is zero at j >= n; a thread beyond the padded columns read another's entry)
                const double y = tid + T * q >= k + 3 && (T * (q + 1) <= NP || tid + T * q < NP) ? x[q] : 0.0;
                part = fma(y, y, part);
                *(double2*)(sm + LOWN + 2 * (place[q] >> 16)) = make_double2(vq[q], wq[q]);
            }
            if (++own == G) {
                own = 0;
                ++own_r;
            }
            if (++own_k == G) own_k = 0;
        }
        if (g == 0) {
#pragma unroll
            for (int q = 0; q < PQ; ++q)
                if (tid + T * q == n - 1) Jd[n - 1] = x[q];
        }
    }

    static __device__ __forceinline__ void job(const TridJob& J, const int g, double* sm) {
        const int n = J.n, G = SOLO ? 1 : J.G;
        const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
        const int wc = w % WC, wr = w / WC;
        double* red = sm + LRED;
        volatile int* failed = (volatile int*)(sm + LFAIL);
        const gf64* A = (const gf64*)J.A;
        if (tid == 0) *failed = 0;
        double a[RR][CW];
        double* rows = sm + LROW + wr * RL * NP + lane + 64 * wc;
        double mx = 0.0;
#pragma unroll
        for (int s = 0; s < RW; ++s) {
            const int i = g + G * (wr + WR * s);
#pragma unroll
            for (int c = 0; c < CW; ++c) {
                const int j = lane + 64 * (wc + WC * c);
                const double y = (i < n && j < n) ? A[j + (int64_t)i * J.lda] : 0.0;   // row i = column i
                if (s < RR) a[min(s, RR - 1)][c] = y;
                else rows[(s - RR) * NP + 64 * WC * c] = y;
                mx = fmax(mx, fabs(y));
            }
        }
        __syncthreads();
        mx = block_max<NW>(mx, red);
        bool local = true;
        if constexpr (!SOLO) {
            gu64* x0 = (gu64*)J.xbuf;
            if (tid == 0) {
                unsigned xcc;
                __asm__ volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(xcc));
                put_x<false>(x0, g, mx + 0.0);
                put_x<false>(x0, G + g, (double)xcc);
            }
            double gm = 0.0, first = 0.0, last = 0.0;   // largest entry; 64 - smallest and 1 + largest id
            for (int t = tid; t < 2 * G; t += T) {
                uint64_t u = get_x(x0, t);
                for (int polls = 0; u == kEmpty && !*failed; u = get_x(x0, t))
                    if (++polls > kSpinLimit) *failed = 1;
                const double x = __builtin_bit_cast(double, u);
                if (t < G) gm = fmax(gm, x);
                else {
                    first = fmax(first, 64.0 - x);
                    last = fmax(last, 1.0 + x);
                }
            }
            mx = block_max<NW>(gm, red);
            first = block_max<NW>(first, red);
            last = block_max<NW>(last, red);
            local = first + last == 65.0;   // every workgroup of the job on one XCD
        }
        const double sc = mx > 0.0 && isfinite(mx) ? ldexp(1.0, -ilogb(mx)) : 1.0;
        if (g == 0 && tid == 0) *J.scale = sc;
#pragma unroll
        for (int s = 0; s < RW; ++s)
#pragma unroll
            for (int c = 0; c < CW; ++c) {
                if (s < RR) a[min(s, RR - 1)][c] *= sc;
                else rows[(s - RR) * NP + 64 * WC * c] *= sc;
            }
        columns(J, g, sm, a, sc, local);
        __syncthreads();
        if (tid == 0 && *failed) *J.status = 1;
    }
};

// Register shapes of a job: (threads, waves across the columns, column slots
// per lane, rows per wave, of them in LDS).  A variant takes orders up to
// 64 WC CW; a workgroup holds RW waves / WC rows.  256-thread variants hold
// whole rows per wave (no LDS round for a row sum); beyond n = 704 their
// vectors and rows no longer fit the registers of four waves, and eight waves
// share the columns.  RW is set so that a job of the variant's largest order
// fits one XCD's 32 compute units up to n = 1024 (its exchange costs half of
// one over all XCDs: 3.6 us per column at n = 1024, 4.6 us at 1100), above
// that by the registers: more rows spill (n = 2624 with 15 rows all in
// registers: 32.9 ms in all, with four of them in LDS 24.2 ms).  bmap[b] =
// (job, rank) of workgroup b; job < 0: idle workgroup.  Dynamic LDS:
// tridiag_lds.
struct TridVariant {
    int T, WC, CW, RW, RL;
    int nmax() const { return 64 * WC * CW; }
    int rows() const { return RW * (T / 64 / WC); }
};
const TridVariant kTridVariants[] = {
    {256, 1, 2, 32, 0}, {256, 1, 3, 12, 0}, {256, 1, 4, 8, 0},  {256, 1, 6, 6, 0}, {256, 1, 8, 5, 0}, {256, 1, 11, 6, 0},
    {512, 2, 8, 8, 0},  {512, 4, 6, 12, 0}, {512, 8, 4, 20, 0}, {512, 8, 6, 15, 4}, {512, 8, 7, 13, 3},
    {512, 1, 6, 4, 0}, {512, 2, 6, 6, 0}};
constexpr int kTridVariantsN = 11;   // chosen by the order alone
constexpr int kTridWide = 6;         // first 512-thread variant
// Two more of 512 threads for orders that have 256-thread variants, so that
// jobs of both kinds share a launch (cooperative launches run one after
// another): the smaller jobs then end with the larger ones instead of after them
// (SU(2) move, f32, orders up to 1024:
// 3.85 ms in two launches, 2.40 ms in one).
constexpr int kTridJoint = kTridVariantsN, kTridJointN = 2;

__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) void tridiag_kernel(
    const TridJob* __restrict__ jobs, const int2* __restrict__ bmap) {
    const int2 bm = bmap[blockIdx.x];
    if (bm.x < 0) return;
    const TridJob J = jobs[bm.x];
    extern __shared__ double sm[];
    switch (J.variant) {
        case 0: Trid<256, 1, 2, 32>::job(J, bm.y, sm); break;
        case 1: Trid<256, 1, 3, 12>::job(J, bm.y, sm); break;
        case 2: Trid<256, 1, 4, 8>::job(J, bm.y, sm); break;
        case 3: Trid<256, 1, 6, 6>::job(J, bm.y, sm); break;
        case 4: Trid<256, 1, 8, 5>::job(J, bm.y, sm); break;
        default: Trid<256, 1, 11, 6>::job(J, bm.y, sm); break;
    }
}
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) void tridiag_wide_kernel(
    const TridJob* __restrict__ jobs, const int2* __restrict__ bmap) {
    const int2 bm = bmap[blockIdx.x];
    if (bm.x < 0) return;
    const TridJob J = jobs[bm.x];
    extern __shared__ double sm[];
    switch (J.variant) {
        case 6: Trid<512, 2, 8, 8>::job(J, bm.y, sm); break;
        case 7: Trid<512, 4, 6, 12>::job(J, bm.y, sm); break;
        case 8: Trid<512, 8, 4, 20>::job(J, bm.y, sm); break;
        case 9: Trid<512, 8, 6, 15, 4>::job(J, bm.y, sm); break;
        case 10: Trid<512, 8, 7, 13, 3>::job(J, bm.y, sm); break;
        case 11: Trid<512, 1, 6, 4>::job(J, bm.y, sm); break;
        default: Trid<512, 2, 6, 6>::job(J, bm.y, sm); break;
    }
}

// Step 1 for a Jordan-Wielandt matrix [[0, Y], [Y^T, 0]] (FP64 moves).  With
// its states in the order u_0, v_0, u_1, v_1, ... the reduction above keeps the
// zero blocks: column 2i (state u_i) has entries on the v side only, its
// reflector acts on v_i .. , p = tau M v lives on the u side, so p . v = 0,
// w = p, and T has a zero diagonal (the Golub-Kahan form of Y).  Held as such
// it takes Y and Y^T (2 m^2 values instead of 4 m^2 for the joint matrix) and
// one sum per column.  Column 2i+1 (state v_i) mirrors it: reflector on
// u_(i+1) .., p on the v side.
struct BidJob {
    const double* Y;                   // nu x nv, column-major (ld ldy)
    int nu, nv, ldy, G, variant;
    double *d, *e, *e2, *scale;        // T of order nu + nv, scaled by *scale
    double *V[2], *tau[2];             // reflectors and factors of the v side (0) and the u side (1)
    double* xbuf;                      // exchange area (bid_xbuf_doubles), filled with kEmpty
    int* status;
};
// Columns of T that are formed (the last one without an exchange); the rest of
// the states (of the longer side) are decoupled zeros.
__host__ __device__ inline int bid_columns(int nu, int nv) { return nu > nv ? 2 * nv : 2 * nu - 1; }

// One workgroup of a job: rows i = g + G (wr + WR s) of Y (lanes along v) and
// of Y^T (lanes along u), both in registers.  Per column h (i = h / 2, side
// s = h & 1; "here" the reflector's side, "there" the other one):
//  (a) the reflector, each thread its entries; {w, v} here to every wave;
//  (b) the owner publishes the next column as its rows hold it, which is
//      before the updates of columns h-1 and h;
//  (c) one pass over the rows > i there: the updates of columns h-2 and h-1,
//      then p = tau row . v;
//  (d) every thread polls p and the next column and applies the two updates.
// Row scalars of a pass are the pairs that (a) of column h-1 shared.  Bound
// like the symmetric reduction by its serial chain, two LDS rounds and one
// exchange per column: 2.4 us per column at m = 696 (29 workgroups of one XCD).
template <int WC, int CW, int RW>
struct Bid {
    static constexpr int T = 512, NW = T / 64, WR = NW / WC, R = RW * WR;
    static constexpr int NP = 64 * WC * CW;
    static constexpr int PQ = (CW + WR - 1) / WR, NQ = T * PQ;
    static constexpr bool SOLO = R >= NP;
    // LDS, in doubles: the next column; {w, v} of both sides; one workgroup:
    // raw p and next column; sums; partial row sums
    static constexpr int PAIRS = 2 * (NQ > NP + R ? NQ : NP + R);
    static constexpr int LX = 0, LVW = LX + NQ, LRAW = LVW + 2 * PAIRS, LRED = LRAW + (SOLO ? 2 * NP : 0),
                         LPART = LRED + NW, LFAIL = LPART + (WC > 1 ? NW * (RW + 3) : 0), LDS = LFAIL + 2;

    struct State {
        const BidJob& J;
        double* sm;
        gu64* reg;
        double sc;
        double x[PQ], part;            // the column here, its squared norm below the leading entry (this thread's share)
        double wq[2][PQ], vq[2][PQ];   // w and v per side at this thread's columns (0: v side)
        double v[2][CW];               // v per side at this lane's columns
        uint32_t place[PQ];
        int g, G, region, gr, own_r, own;   // row i + s of the side here: workgroup own, local row own_r
        bool local;
    };

    template <int S>
    static __device__ __forceinline__ void column(State& z, const int i, const bool last, double (&a)[RW][CW],
                                                  double (&at)[RW][CW]) {
        // a: rows there (lanes here); at: rows here (lanes there)
        const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
        const int wc = w % WC, wr = w / WC;
        double* sm = z.sm;
        const int n = S ? z.J.nu : z.J.nv, no = S ? z.J.nv : z.J.nu;   // entries here, there
        const int L = i + S;                                         // leading entry here
        auto* failed = (LOCAL_MEM volatile int*)(sm + LFAIL);
        // (a)
#pragma unroll
        for (int q = 0; q < PQ; ++q) sm[LX + tid + T * q] = z.x[q];
        const double ps = wave_sum(z.part);
        if (lane == 0) sm[LRED + w] = ps;
        __syncthreads();
        double xn2 = 0.0;
#pragma unroll
        for (int q = 0; q < NW; ++q) xn2 += sm[LRED + q];
        double beta, tau, scal;
        householder(sm[LX + L], xn2, beta, tau, scal);
#pragma unroll
        for (int q = 0; q < PQ; ++q) {
            const int j = tid + T * q;
            z.vq[S][q] = j > L && (T * (q + 1) <= NP || j < NP) ? z.x[q] * scal : (j == L ? 1.0 : 0.0);
            *(double2*)(sm + LVW + S * PAIRS + 2 * j) = make_double2(z.wq[S][q], z.vq[S][q]);
        }
        __syncthreads();
        const int ldv = v_stride(n);
        if (SOLO || z.g == z.own) {   // the owner of row L here stores the reflector
            gf64* V = (gf64*)z.J.V[S] + (size_t)i * ldv;
#pragma unroll
            for (int q = 0; q < PQ; ++q)
                if (64 * w + T * q < ldv) *at8(V, tid + T * q) = z.vq[S][q];
            if (tid == 0) {
                ((gf64*)z.J.tau[S])[i] = tau;
                ((gf64*)z.J.e)[2 * i + S] = beta;
                ((gf64*)z.J.e2)[2 * i + S] = coupling2(beta);
            }
        }
        if (last) return;
        // (b) row L here holds the next column
        if ((SOLO || z.g == z.own) && z.own_r % WR == wr) {
            const int sp = z.own_r / WR;
#pragma unroll
            for (int s = 0; s < RW; ++s) {
                if (s == sp) {
                    if (SOLO) {
#pragma unroll
                        for (int c = 0; c < CW; ++c) sm[LRAW + NP + lane + 64 * (wc + WC * c)] = at[s][c];
                    } else if (z.local) {
#pragma unroll
                        for (int c = 0; c < CW; ++c) put_x<true>(z.reg + z.gr, lane + 64 * (wc + WC * c), at[s][c]);
                    } else {
#pragma unroll
                        for (int c = 0; c < CW; ++c) put_x<false>(z.reg + z.gr, lane + 64 * (wc + WC * c), at[s][c]);
                    }
                }
            }
        }
        // (c)
        const int c_lo = max(L - 64 * wc, 0) / (64 * WC);
        double vA[CW], wA[CW];
#pragma unroll
        for (int c = 0; c < CW; ++c) {
            const double2 t = *(const double2*)(sm + LVW + S * PAIRS + 2 * (lane + 64 * (wc + WC * c)));
            vA[c] = z.v[S][c];
            wA[c] = t.x;
            z.v[S][c] = t.y;
        }
        // rows > i there: local rows >= rmin
        const int ri = S ? z.own_r : z.own_r, rmin = S ? (z.g < z.own ? ri + 1 : ri) : (z.g <= z.own ? ri + 1 : ri);
        const int s_lo = (max(rmin - wr, 0) + WR - 1) / WR;
        double* part_s = sm + LPART;
#pragma unroll
        for (int s0 = 0; s0 < RW; s0 += kRowGroup) {
            if (s0 + kRowGroup > s_lo) {
                double vu[kRowGroup], wu[kRowGroup], acc[kRowGroup];
#pragma unroll
                for (int u = 0; u < kRowGroup; ++u) {
                    acc[u] = 0.0;
                    if (s0 + u < RW) {
                        const double2 t = *(const double2*)(sm + LVW + (1 - S) * PAIRS +
                                                            2 * (z.g + z.G * (wr + WR * (s0 + u))));
                        wu[u] = t.x;   // w of column h-2, v of column h-1
                        vu[u] = t.y;
                    }
                }
#pragma unroll
                for (int c0 = 0; c0 < CW; c0 += kColGroup) {
                    if (c0 + kColGroup > c_lo) {
#pragma unroll
                        for (int c = c0; c < c0 + kColGroup && c < CW; ++c) {
#pragma unroll
                            for (int u = 0; u < kRowGroup && s0 + u < RW; ++u) {
                                double y = a[s0 + u][c];
                                y = fma(-wu[u], vA[c], y);
                                y = fma(-vu[u], wA[c], y);
                                a[s0 + u][c] = y;
                                acc[u] = fma(y, z.v[S][c], acc[u]);
                            }
                        }
                    }
                }
                const double t = four_sums(acc);
                const int s = s0 + reduced_row(lane >> 4);
                if ((lane & 15) == 0 && s < RW) {
                    if constexpr (WC > 1) part_s[w * (RW + 3) + s] = t;
                    else if constexpr (SOLO) sm[LRAW + wr + WR * s] = tau * t;
                    else put_x(z.reg, z.g * R + wr + WR * s, tau * t, z.local);
                }
            }
        }
        if constexpr (WC > 1) {
            __syncthreads();
            if (tid < R) {
                double y = 0.0;
#pragma unroll
                for (int q = 0; q < WC; ++q) y += part_s[((tid % WR) * WC + q) * (RW + 3) + tid / WR];
                put_x(z.reg, z.g * R + tid, tau * y, z.local);
            }
        }
        // (d)
        double pr[PQ], rr[PQ];
        if constexpr (SOLO) {
            __syncthreads();
#pragma unroll
            for (int q = 0; q < PQ; ++q) {
                pr[q] = sm[LRAW + min(tid + T * q, NP - 1)];
                rr[q] = sm[LRAW + NP + min(tid + T * q, NP - 1)];
            }
        } else {
            uint64_t pu[PQ], ru[PQ];
#pragma unroll
            for (int q = 0; q < PQ; ++q) pu[q] = ru[q] = 0;
            for (int polls = 0;;) {
                bool empty = false;
#pragma unroll
                for (int q = 0; q < PQ; ++q) {
                    if (T * q + 64 * w + 63 > i && T * q + 64 * w < no) {
                        pu[q] = get_x(z.reg, z.place[q]);
                        ru[q] = get_x(z.reg + z.gr, tid + T * q);
                    }
                }
#pragma unroll
                for (int q = 0; q < PQ; ++q)
                    empty |= (pu[q] == kEmpty && (unsigned)(tid + T * q - i - 1) < (unsigned)(no - i - 1)) ||
                             ru[q] == kEmpty;
                if (!__any(empty) || *failed) break;
                if (++polls > kSpinLimit) {
                    *failed = 1;
                    break;
                }
            }
#pragma unroll
            for (int q = 0; q < PQ; ++q) {
                pr[q] = __builtin_bit_cast(double, pu[q]);
                rr[q] = __builtin_bit_cast(double, ru[q]);
            }
            z.reg += z.region;
        }
        const double wl = sm[LVW + S * PAIRS + 2 * L];   // w of column h-1 at row L here
        z.part = 0.0;
#pragma unroll
        for (int q = 0; q < PQ; ++q) {
            const int j = tid + T * q;
            const double p = (unsigned)(j - i - 1) < (unsigned)(no - i - 1) ? pr[q] : 0.0;
            z.wq[1 - S][q] = p;
            z.x[q] = fma(-wl, z.vq[1 - S][q], rr[q]) - p;
            const double y = j >= i + 2 && (T * (q + 1) <= NP || j < NP) ? z.x[q] : 0.0;
            z.part = fma(y, y, z.part);
        }
        if (S == 0) {   // row i + 1 comes next
            if (++z.own == z.G) {
                z.own = 0;
                ++z.own_r;
            }
        }
    }

    static __device__ __forceinline__ void job(const BidJob& J, const int g, double* sm) {
        const int nu = J.nu, nv = J.nv, G = SOLO ? 1 : J.G, N = nu + nv;
        const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
        const int wc = w % WC, wr = w / WC;
        auto* failed = (LOCAL_MEM volatile int*)(sm + LFAIL);
        const gf64* Y = (const gf64*)J.Y;
        if (tid == 0) *failed = 0;
        for (int j = tid; j < 2 * PAIRS; j += T) sm[LVW + j] = 0.0;
        if (g == 0) {
            gf64 *d = (gf64*)J.d, *e = (gf64*)J.e, *e2 = (gf64*)J.e2;
            for (int j = tid; j < N; j += T) {
                d[j] = 0.0;
                if (j >= bid_columns(nu, nv)) {
                    e[j] = 0.0;
                    e2[j] = coupling2(0.0);
                }
            }
        }
        double au[RW][CW], av[RW][CW];   // rows of Y, rows of Y^T
        double mx = 0.0;
#pragma unroll
        for (int s = 0; s < RW; ++s) {
            const int i = g + G * (wr + WR * s);
#pragma unroll
            for (int c = 0; c < CW; ++c) {
                const int j = lane + 64 * (wc + WC * c);
                au[s][c] = i < nu && j < nv ? Y[i + (int64_t)j * J.ldy] : 0.0;
                av[s][c] = i < nv && j < nu ? Y[j + (int64_t)i * J.ldy] : 0.0;
                mx = fmax(mx, fmax(fabs(au[s][c]), fabs(av[s][c])));
            }
        }
        __syncthreads();
        mx = block_max<NW>(mx, sm + LRED);
        bool local = true;
        if constexpr (!SOLO) {
            gu64* x0 = (gu64*)J.xbuf;
            if (tid == 0) {
                unsigned xcc;
                __asm__ volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(xcc));
                put_x<false>(x0, g, mx + 0.0);
                put_x<false>(x0, G + g, (double)xcc);
            }
            double gm = 0.0, first = 0.0, lastx = 0.0;   // largest entry; 64 - smallest and 1 + largest id
            for (int t = tid; t < 2 * G; t += T) {
                uint64_t u = get_x(x0, t);
                for (int polls = 0; u == kEmpty && !*failed; u = get_x(x0, t))
                    if (++polls > kSpinLimit) *failed = 1;
                const double x = __builtin_bit_cast(double, u);
                if (t < G) gm = fmax(gm, x);
                else {
                    first = fmax(first, 64.0 - x);
                    lastx = fmax(lastx, 1.0 + x);
                }
            }
            mx = block_max<NW>(gm, sm + LRED);
            first = block_max<NW>(first, sm + LRED);
            lastx = block_max<NW>(lastx, sm + LRED);
            local = first + lastx == 65.0;   // every workgroup of the job on one XCD
        }
        const double sc = mx > 0.0 && isfinite(mx) ? ldexp(1.0, -ilogb(mx)) : 1.0;
        if (g == 0 && tid == 0) *(gf64*)J.scale = sc;
#pragma unroll
        for (int s = 0; s < RW; ++s)
#pragma unroll
            for (int c = 0; c < CW; ++c) {
                au[s][c] *= sc;
                av[s][c] *= sc;
            }
        State z{J, sm};
        z.g = g;
        z.G = G;
        z.gr = (G * R + 15) & ~15;
        z.region = z.gr + NP;
        z.reg = (gu64*)J.xbuf + ((2 * G + 15) & ~15);
        z.local = local;
        z.own = z.own_r = 0;
        z.part = 0.0;
#pragma unroll
        for (int q = 0; q < PQ; ++q) {
            const int j = tid + T * q, r = min(j, NP - 1) / G;
            z.place[q] = min((min(j, NP - 1) - r * G) * R + r, G * R - 1);
            z.x[q] = j < nv ? Y[(int64_t)j * J.ldy] * sc : 0.0;   // row 0 of Y
            const double y = j >= 1 ? z.x[q] : 0.0;
            z.part = fma(y, y, z.part);
            z.wq[0][q] = z.wq[1][q] = z.vq[0][q] = z.vq[1][q] = 0.0;
        }
#pragma unroll
        for (int c = 0; c < CW; ++c) z.v[0][c] = z.v[1][c] = 0.0;
        const int H = bid_columns(nu, nv);
#pragma unroll 1
        for (int h = 0; h < H; h += 2) {
            __asm__("" : "+s"(z.reg));
            column<0>(z, h >> 1, h + 1 == H, au, av);
            if (h + 1 < H) column<1>(z, h >> 1, h + 2 == H, av, au);
        }
        __syncthreads();
        if (tid == 0 && *failed) *J.status = 1;
    }
};

// Register shapes: (waves across the columns, column slots per lane, rows of Y
// and of Y^T per wave), sides up to 64 WC CW.  Up to 768 a job fits one XCD.
struct BidVariant {
    int WC, CW, RW;
    int nmax() const { return 64 * WC * CW; }
    int rows() const { return RW * (8 / WC); }
};
const BidVariant kBidVariants[] = {{1, 2, 16}, {2, 2, 8}, {2, 3, 6}, {4, 2, 10}, {4, 3, 12}, {8, 2, 16}, {8, 3, 12}, {8, 4, 9}};
constexpr int kBidVariantsN = sizeof(kBidVariants) / sizeof(kBidVariants[0]);
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) void bidiag_kernel(
    const BidJob* __restrict__ jobs, const int2* __restrict__ bmap) {
    const int2 bm = bmap[blockIdx.x];
    if (bm.x < 0) return;
    const BidJob J = jobs[bm.x];
    extern __shared__ double sm[];
    switch (J.variant) {
        case 0: Bid<1, 2, 16>::job(J, bm.y, sm); break;
        case 1: Bid<2, 2, 8>::job(J, bm.y, sm); break;
        case 2: Bid<2, 3, 6>::job(J, bm.y, sm); break;
        case 3: Bid<4, 2, 10>::job(J, bm.y, sm); break;
        case 4: Bid<4, 3, 12>::job(J, bm.y, sm); break;
        case 5: Bid<8, 2, 16>::job(J, bm.y, sm); break;
        case 6: Bid<8, 3, 12>::job(J, bm.y, sm); break;
        default: Bid<8, 4, 9>::job(J, bm.y, sm); break;
    }
}

struct BisJob {
    const double *d, *e, *e2, *scale;
    double* w;      // n eigenvalues, ascending, unscaled
    double* range;  // lower end, upper end and norm (NaN: T is not finite) of the spectrum's interval
    int* count;     // eigenvalues below grid points 1 .. points of the interval
    int n, points;
    int half;       // > 0: spectrum +-, the `half` largest are found, the rest mirrored or zero
};

// Number of eigenvalues of T below x: sign changes of the leading principal
// minors p_i = (d_i - x) p_{i-1} - e2_{i-1} p_{i-2}, which carries the same
// kind of relative errors in d_i - x and e2 as the quotients p_i / p_{i-1}, but
// needs no division: 24 + 18 instructions per eight steps, where a reciprocal
// with a Newton step and the guard of the quotient took twice the time per
// step.  T is wave-uniform and comes through the scalar cache (d and e^2 in LDS
// took two broadcast reads per step).  The pair is scaled back every eight
// steps: entries of T are below 2^13 and coupling2 is at least 2^-200, so
// eight steps stay within the exponents.  With three to thirteen wavefronts per
// SIMD the instructions bound it: all values of the seven matrices of a move at
// D = 6, chi = 64 (3.3e3 in all) 393 -> 175 us in FP32, 775 -> 329 us in FP64,
// of the sixteen at D = 8, chi = 200 6.9 -> 2.3 ms, with the grid below.
#ifdef __HIP_DEVICE_COMPILE__
#define UNIFORM_MEM __attribute__((address_space(4)))
#else
#define UNIFORM_MEM
#endif
typedef UNIFORM_MEM const double cf64;
__device__ inline uint32_t high_word(double x) { return (uint32_t)(__builtin_bit_cast(uint64_t, x) >> 32); }
__device__ inline int sturm_count(cf64* d, cf64* e2, int n, double x) {
    double p0 = 1.0, p1 = d[0] - x;
    uint32_t signs = high_word(p1) >> 31;   // bit 0: the last minor's sign
    int cnt = (int)signs, i = 1;
    auto step = [&](double di, double ei) {
        const double p2 = fma(di - x, p1, -(ei * p0));
        p0 = p1;
        p1 = p2;
        signs = signs << 1 | high_word(p2) >> 31;
    };
    for (; i + 8 <= n; i += 8) {
        double D[8], E[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            D[u] = d[i + u];
            E[u] = e2[i + u - 1];
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) step(D[u], E[u]);
        cnt += __popc((signs ^ signs >> 1) & 0xff);
        const int ex = 1023 - (int)max(high_word(p0) >> 20 & 0x7ff, high_word(p1) >> 20 & 0x7ff);
        p0 = __builtin_amdgcn_ldexp(p0, ex);
        p1 = __builtin_amdgcn_ldexp(p1, ex);
    }
    for (; i < n; ++i) {
        step(d[i], e2[i - 1]);
        cnt += (signs ^ signs >> 1) & 1;
    }
    return cnt;
}

// Step 2, first part: counts at equally spaced points of the interval, 64 per
// wave; bmap[b] = (job, first group of 64 points).  They serve all eigenvalues
// of the job: with 8 points per eigenvalue (kGridShare) each starts from an
// interval two multisection passes small, for an eighth of one pass.
constexpr int kGridShare = 8;
__host__ __device__ inline int grid_points(int n) { return 64 * ((n + kGridShare - 1) / kGridShare); }
__global__ __launch_bounds__(kEigThreads) void bisect_grid_kernel(const BisJob* __restrict__ jobs,
                                                                   const int2* __restrict__ bmap) {
    const int2 bm = bmap[blockIdx.x];
    const BisJob J = jobs[bm.x];
    const int n = J.n;
    __shared__ double red[kEigWaves];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    double lo = INFINITY, hi = -INFINITY, bad = 0.0;
    for (int i = tid; i < n; i += kEigThreads) {
        const double di = J.d[i];
        const double el = i > 0 ? fabs(J.e[i - 1]) : 0.0, er = i + 1 < n ? fabs(J.e[i]) : 0.0;
        lo = fmin(lo, di - el - er);
        hi = fmax(hi, di + el + er);
        if (!isfinite(di + el + er)) bad = 1.0;
    }
    // (block_max is a maximum of values >= 0: of the distances from an entry)
    const double d0 = J.d[0];
    lo = d0 - block_max<kEigWaves>(d0 - fmin(lo, d0), red);
    hi = d0 + block_max<kEigWaves>(fmax(hi, d0) - d0, red);
    // NaN or Inf in the matrix: no counts, NaN for every eigenvalue
    const double tnorm = block_max<kEigWaves>(bad, red) > 0.0 ? NAN : fmax(fabs(lo), fabs(hi));
    lo -= 4.0 * DBL_EPSILON * tnorm * n;
    hi += 4.0 * DBL_EPSILON * tnorm * n;
    const int t = (bm.y + wave) * 64 + lane;
    if (tnorm > 0.0 && (bm.y + wave) * 64 < J.points)
        J.count[t] = sturm_count((cf64*)J.d, (cf64*)J.e2, n, lo + (hi - lo) * (double)(t + 1) / (double)(J.points + 1));
    if (bm.y == 0 && tid == 0) {
        J.range[0] = lo;
        J.range[1] = hi;
        J.range[2] = tnorm;
    }
}

// Second part.  bmap[b] = (job, first index); wave q of the workgroup finds the
// eigenvalue of index first + q (ascending): its interval from the grid's
// counts, then passes of 64 counts each, about 7, to 2 ulp.
__global__ __launch_bounds__(kEigThreads) void bisect_kernel(const BisJob* __restrict__ jobs,
                                                              const int2* __restrict__ bmap) {
    const int2 bm = bmap[blockIdx.x];
    const BisJob J = jobs[bm.x];
    const int n = J.n;
    const int lane = threadIdx.x & 63, j = __builtin_amdgcn_readfirstlane(bm.y + (int)(threadIdx.x >> 6));
    if (j >= n) return;
    const double lo = J.range[0], hi = J.range[1], tnorm = J.range[2];
    const double eps = DBL_EPSILON;
    const bool mirror = J.half > 0;
    double a = lo, b = hi;
    if (!(tnorm > 0.0)) {   // T = 0, or not finite
        a = b = tnorm;
    } else {
        // first grid point with more than j eigenvalues below it
        int first = 0, len = J.points;
        while (len > 0) {
            const int step = (len + 63) >> 6, at = min(lane * step + step - 1, len - 1);   // last of the lane's part
            const unsigned long long above = __ballot(J.count[first + at] > j);
            if (!above) {
                first += len;
                break;
            }
            const int c = __ffsll((long long)above) - 1;
            first += c * step;
            len = min(step, len - c * step);
            if (step == 1) break;
        }
        const double h = hi - lo, np = (double)(J.points + 1);
        if (first > 0) a = lo + h * (double)first / np;
        if (first < J.points) b = lo + h * (double)(first + 1) / np;
        for (int pass = 0; pass < 64; ++pass) {
            const double x = a + (b - a) * (double)(lane + 1) / 65.0;
            const int cnt = sturm_count((cf64*)J.d, (cf64*)J.e2, n, x);
            const unsigned long long above = __ballot(cnt > j);
            const int m = above ? __ffsll((long long)above) - 1 : 64;
            const double xm1 = __shfl(x, m > 0 ? m - 1 : 0, 64);
            const double xm = __shfl(x, m < 64 ? m : 63, 64);
            const double na = m > 0 ? xm1 : a, nb = m < 64 ? xm : b;
            const bool stuck = na == a && nb == b;
            a = na;
            b = nb;
            if (stuck || b - a <= fmax(2.0 * eps * fmax(fabs(a), fabs(b)), eps * tnorm)) break;
        }
    }
    // the mirrored values: their places, and zeros between the two halves
    if (mirror && j == n - 1)
        for (int i = J.half + lane; i < n - J.half; i += 64) J.w[i] = 0.0;
    if (lane == 0) {
        const double x = 0.5 * (a + b) / *J.scale;
        J.w[j] = x;
        if (mirror) J.w[n - 1 - j] = -x;
    }
}

// Inverse iteration solves per eigenvector: from a random start, the first
// solve leaves an error of about |lambda error| / gap, the second one at
// rounding level (eigenvalues from the multisection are accurate to
// 2 eps ||T||).
constexpr int kInvIters = 2;

struct VecJob {
    const double *d, *e, *scale, *w;   // w: eigenvalues ascending, unscaled
    double* Zt;                        // n x kv eigenvectors of T (column j: j-th largest)
    double* Zp;                        // the same after polish_kernel
    double* work;                      // 5 n per cluster slot
    int n, kv;
};
struct VecCluster {
    int job, first, count, pad;        // eigenvalue ranks first .. first+count-1 (descending)
    int64_t woff;                      // offset of its 5 n doubles of LU work space
};

__device__ inline double start_entry(int i, int m) {
    // fixed pseudo-random start vector entries in (-1, 1) (a 32-bit integer hash)
    uint32_t h = (uint32_t)i * 0x9E3779B1u ^ ((uint32_t)m + 0x7F4A7C15u) * 0x85EBCA77u;
    h ^= h >> 15;
    h *= 0x2C1B3C6Du;
    h ^= h >> 12;
    h *= 0x297A2D39u;
    h ^= h >> 15;
    return ((double)h + 0.5) / 2147483648.0 - 1.0;
}

// Step 3, every kept eigenvalue on a workgroup of its own: the eigenvector
// straight from the twisted factorisation of T - lam I.  Wave 0
// runs the top-down recurrence D+_i = (d_i - lam) - e_{i-1}^2 / D+_{i-1},
// wave 1 the bottom-up one D-_i = (d_i - lam) - e_i^2 / D-_{i+1} at the same
// time; the twist r minimises |gamma_i| = |D+_i + D-_i - (d_i - lam)| (ties:
// the lower index); then z_r = 1, z_i = -e_i z_{i+1} / D+_i above r and
// z_i = -e_{i-1} z_{i-1} / D-_i below it, normalised.  Its residual is
// |gamma_r| / ||z||, which an eigenvalue accurate to 2 eps ||T|| keeps at
// rounding level (no iteration).  Dynamic LDS: d, e, D+, D-, z (5 n).
__global__ __launch_bounds__(128) void twist_kernel(const VecJob* __restrict__ jobs,
                                                     const int2* __restrict__ bmap) {
    const int2 bm = bmap[blockIdx.x];   // (job, rank of the eigenvalue, descending)
    const VecJob J = jobs[bm.x];
    const int n = J.n, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    extern __shared__ double sm[];
    double *d = sm, *e = sm + n, *dp = sm + 2 * n, *dm = sm + 3 * n, *z = sm + 4 * n;
    __shared__ double red_v[2];
    __shared__ int red_i[2];
    for (int i = tid; i < n; i += 128) {
        d[i] = J.d[i];
        e[i] = i + 1 < n ? J.e[i] : 0.0;
    }
    __syncthreads();
    double tl = 0.0, em = 0.0;
    for (int i = tid; i < n; i += 128) {
        tl = fmax(tl, fabs(d[i]) + (i > 0 ? fabs(e[i - 1]) : 0.0) + fabs(e[i]));
        em = fmax(em, e[i] * e[i]);
    }
    tl = wave_max(tl);
    em = wave_max(em);
    if (lane == 0) red_v[wave] = tl;
    __syncthreads();
    const double tnorm = fmax(red_v[0], red_v[1]);
    __syncthreads();
    const int jr = bm.y;
    double* zo = J.Zt + (size_t)jr * n;
    if (n == 1 || tnorm == 0.0) {   // T = 0: the unit vectors
        for (int i = tid; i < n; i += 128) zo[i] = i == jr ? 1.0 : 0.0;
        return;
    }
    const double lam = J.w[n - 1 - jr] * *J.scale;
    // pivots below this are raised to it (keeping the sign): never zero
    const double piv = DBL_MIN * fmax(1.0, em) / DBL_EPSILON;
    auto guard = [&](double q) { return fabs(q) < piv ? (q < 0.0 ? -piv : piv) : q; };
    auto rcp = [&](double q) {
        const double r0 = __builtin_amdgcn_rcp(q);
        return fma(r0, fma(-q, r0, 1.0), r0);
    };
    if (lane == 0 && wave == 0) {
        double q = guard(d[0] - lam);
        dp[0] = q;
        double dn = d[1], ep = e[0];
        for (int i = 1; i < n; ++i) {
            const double a = dn - lam, e2 = ep * ep;
            if (i + 1 < n) {
                dn = d[i + 1];
                ep = e[i];
            }
            q = guard(a - e2 * rcp(q));
            dp[i] = q;
        }
    } else if (lane == 0 && wave == 1) {
        double q = guard(d[n - 1] - lam);
        dm[n - 1] = q;
        double dn = d[n - 2], ep = e[n - 2];
        for (int i = n - 2; i >= 0; --i) {
            const double a = dn - lam, e2 = ep * ep;
            if (i > 0) {
                dn = d[i - 1];
                ep = e[i - 1];
            }
            q = guard(a - e2 * rcp(q));
            dm[i] = q;
        }
    }
    __syncthreads();
    // twist: argmin |gamma| (lowest index on ties)
    double bv = INFINITY;
    int bi = n;
    for (int i = tid; i < n; i += 128) {
        const double g = fabs(dp[i] + dm[i] - (d[i] - lam));
        if (g < bv) {
            bv = g;
            bi = i;
        }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const double ov = __shfl_xor(bv, o, 64);
        const int oi = __shfl_xor(bi, o, 64);
        if (ov < bv || (ov == bv && oi < bi)) {
            bv = ov;
            bi = oi;
        }
    }
    if (lane == 0) {
        red_v[wave] = bv;
        red_i[wave] = bi;
    }
    __syncthreads();
    const int r = (red_v[1] < red_v[0] || (red_v[1] == red_v[0] && red_i[1] < red_i[0])) ? red_i[1] : red_i[0];
    // ratios in parallel, then the two product chains at once, wave 0 upwards
    // from r, wave 1 downwards: each lane multiplies a run of consecutive
    // ratios, the runs' products are scanned across the lanes, and each lane
    // goes through its run again
    for (int i = tid; i < n; i += 128) {
        if (i < r) z[i] = -e[i] / dp[i];
        else if (i > r) z[i] = -e[i - 1] / dm[i];
        else z[i] = 1.0;
    }
    __syncthreads();
    {
        const int len = wave == 0 ? r : n - 1 - r;      // ratios of this wave's chain
        const int step = wave == 0 ? -1 : 1;
        const int run = (len + 63) / 64, f0 = min(lane * run, len), f1 = min(f0 + run, len);
        double prod = 1.0;
        for (int f = f0; f < f1; ++f) prod *= z[r + step * (f + 1)];
        double before = __shfl_up(prod, 1, 64);
        if (lane == 0) before = 1.0;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const double up = __shfl_up(before, o, 64);
            if (lane >= o) before *= up;
        }
        // (the product of a run by itself may overflow where the vector's
        // entries do not, with couplings far below rounding: then one lane
        // multiplies in order)
        const bool scanned = !__any(!isfinite(before));
        if (!scanned) before = 1.0;
        for (int f = scanned ? f0 : 0, end = scanned ? f1 : (lane == 0 ? len : 0); f < end; ++f) {
            before *= z[r + step * (f + 1)];
            z[r + step * (f + 1)] = before;
        }
    }
    __syncthreads();
    double part = 0.0;
    for (int i = tid; i < n; i += 128) part += z[i] * z[i];
    part = wave_sum(part);
    if (lane == 0) red_v[wave] = part;
    __syncthreads();
    const double inv = 1.0 / sqrt(red_v[0] + red_v[1]);
    for (int i = tid; i < n; i += 128) zo[i] = z[i] * inv;
}

// Step 3 for eigenvalues closer than the clustering bound: one wavefront per
// cluster goes through its members' vectors (from twist_kernel) in order and
// projects the earlier ones out; unless little is left (a value degenerate
// with an earlier one) that is the vector, else it comes from inverse
// iteration.  There lane 0 runs the recurrences of the LU factorisation and
// the solves, carrying the values each step depends on in registers; the
// whole wave does the vector operations.  INLDS: the factors (5 n doubles)
// in LDS after z, d, e, else in the job's work space.
template <bool INLDS>
__global__ __launch_bounds__(64) void cluster_kernel(const VecJob* __restrict__ jobs,
                                                      const VecCluster* __restrict__ clusters) {
    const VecCluster C = clusters[blockIdx.x];
    const VecJob J = jobs[C.job];
    const int n = J.n, lane = threadIdx.x;
    extern __shared__ double sm[];
    double *z = sm, *d = sm + n, *e = sm + 2 * n;
    double *dl = INLDS ? sm + 3 * n : J.work + C.woff, *du = dl + n, *du2 = dl + 2 * n, *rdd = dl + 3 * n,
           *piv = dl + 4 * n;
    double tl = 0.0;
    for (int i = lane; i < n; i += 64) {
        d[i] = J.d[i];
        e[i] = i + 1 < n ? J.e[i] : 0.0;
    }
    __syncthreads();
    for (int i = lane; i < n; i += 64)
        tl = fmax(tl, fabs(d[i]) + (i > 0 ? fabs(e[i - 1]) : 0.0) + fabs(e[i]));
    const double tnorm = wave_max(tl);
    if (n == 1 || tnorm == 0.0) return;             // the unit vectors stand
    const double small = DBL_EPSILON * tnorm;
    const double sc = *J.scale;
    for (int m = 1; m < C.count; ++m) {             // the first vector stands
        const int jr = C.first + m;                 // rank (descending)
        const double lam = J.w[n - 1 - jr] * sc;    // scaled eigenvalue
        double* zo = J.Zt + (size_t)jr * n;
        for (int i = lane; i < n; i += 64) z[i] = zo[i];
        for (int q = 0; q < m; ++q) {
            const double* y = J.Zt + (size_t)(C.first + q) * n;
            double pq = 0.0;
            for (int i = lane; i < n; i += 64) pq += y[i] * z[i];
            const double dot = wave_sum(pq);
            for (int i = lane; i < n; i += 64) z[i] -= dot * y[i];
        }
        double part = 0.0;
        for (int i = lane; i < n; i += 64) part += z[i] * z[i];
        const double left = wave_sum(part);
        if (left >= 0.25) {
            const double inv = 1.0 / sqrt(left);
            for (int i = lane; i < n; i += 64) zo[i] = z[i] * inv;
            __threadfence_block();
            __syncthreads();   // later members of the cluster read this vector
            continue;
        }
        __syncthreads();
        if (lane == 0) {
            // LU with partial pivoting of T - lam I (LAPACK's tridiagonal
            // scheme; row interchanges recorded in piv, tiny pivots raised
            // to eps ||T||, reciprocals of the pivots kept).  The entries of
            // the next step are loaded one step ahead.
            double cd = d[0] - lam, cu = e[0];
            double sub = e[0], dnx = d[1], enx = n > 2 ? e[1] : 0.0;
            for (int i = 0; i + 1 < n; ++i) {
                const double s0 = sub;
                double nd = dnx - lam, nu = enx;
                sub = enx;
                dnx = i + 2 < n ? d[i + 2] : 0.0;
                enx = i + 3 < n ? e[i + 2] : 0.0;
                if (fabs(cd) >= fabs(s0)) {
                    if (fabs(cd) < small) cd = cd < 0.0 ? -small : small;
                    const double r0 = __builtin_amdgcn_rcp(cd);
                    const double r = fma(r0, fma(-cd, r0, 1.0), r0);
                    const double f = s0 * r;
                    dl[i] = f;
                    du[i] = cu;
                    du2[i] = 0.0;
                    rdd[i] = r;
                    piv[i] = 0.0;
                    nd -= f * cu;
                } else {
                    const double r0 = __builtin_amdgcn_rcp(s0);
                    const double r = fma(r0, fma(-s0, r0, 1.0), r0);
                    const double f = cd * r;
                    dl[i] = f;
                    rdd[i] = r;
                    du[i] = nd;
                    du2[i] = nu;
                    piv[i] = 1.0;
                    nd = cu - f * nd;
                    nu = -f * nu;
                }
                cd = nd;
                cu = nu;
            }
            if (fabs(cd) < small) cd = cd < 0.0 ? -small : small;
            rdd[n - 1] = 1.0 / cd;
        }
        for (int i = lane; i < n; i += 64) z[i] = start_entry(i, jr);
        __syncthreads();
        for (int it = 0; it < kInvIters; ++it) {
            if (lane == 0) {
                // L U y = P z in place: forward with the interchanges ...
                double zi = z[0];
                double zn = z[1], pv = piv[0], f = dl[0];
                for (int i = 0; i + 1 < n; ++i) {
                    const double zn0 = zn, pv0 = pv, f0 = f;
                    if (i + 2 < n) {
                        zn = z[i + 2];
                        pv = piv[i + 1];
                        f = dl[i + 1];
                    }
                    if (pv0 == 0.0) {
                        z[i] = zi;
                        zi = zn0 - f0 * zi;
                    } else {
                        z[i] = zn0;
                        zi = zi - f0 * zn0;
                    }
                }
                // ... then back substitution
                double z1 = zi * rdd[n - 1];
                z[n - 1] = z1;
                double z2 = 0.0;
                double zc_in = z[n - 2], u1 = du[n - 2], u2 = du2[n - 2], rr = rdd[n - 2];
                for (int i = n - 2; i >= 0; --i) {
                    const double a0 = zc_in, a1 = u1, a2 = u2, a3 = rr;
                    if (i > 0) {
                        zc_in = z[i - 1];
                        u1 = du[i - 1];
                        u2 = du2[i - 1];
                        rr = rdd[i - 1];
                    }
                    const double zc = (a0 - a1 * z1 - a2 * z2) * a3;
                    z[i] = zc;
                    z2 = z1;
                    z1 = zc;
                }
            }
            __syncthreads();
            // against the cluster's earlier vectors
            for (int q = 0; q < m; ++q) {
                const double* y = J.Zt + (size_t)(C.first + q) * n;
                double part = 0.0;
                for (int i = lane; i < n; i += 64) part += y[i] * z[i];
                const double dot = wave_sum(part);
                for (int i = lane; i < n; i += 64) z[i] -= dot * y[i];
            }
            double mx = 0.0;
            for (int i = lane; i < n; i += 64) mx = fmax(mx, fabs(z[i]));
            mx = wave_max(mx);
            const double inv = mx > 0.0 ? 1.0 / mx : 1.0;
            double part = 0.0;
            for (int i = lane; i < n; i += 64) {
                const double v = z[i] * inv;
                z[i] = v;
                part += v * v;
            }
            const double r = 1.0 / sqrt(wave_sum(part));
            for (int i = lane; i < n; i += 64) z[i] *= r;
            __syncthreads();
        }
        for (int i = lane; i < n; i += 64) zo[i] = z[i];
        __threadfence_block();
        __syncthreads();   // later members of the cluster read this vector
    }
}

// Vectors of eigenvalues a gap g ||T|| apart are orthogonal to about eps / g,
// 2e-13 at the 1e-3 where clusters end: each gives up half of its product with
// every other kept vector that is less than 1e-2 ||T|| away (all products
// before any change), which leaves them orthogonal to rounding.  Those vectors
// are a run of ranks lo .. hi-1 around its own.  (Three neighbours on either
// side are not enough beside a multiplet: 4.7e-13 at order 200, now 1e-14;
// 12.5 -> 13.2 us in the FP32 move at D = 6, chi = 64, 19 -> 21 us in FP64.)  A
// wave takes a product, the products wait in LDS (kv doubles, dynamic), then
// every thread subtracts at its own entries.
__global__ __launch_bounds__(kEigThreads) void polish_kernel(const VecJob* __restrict__ jobs,
                                                              const int2* __restrict__ bmap) {
    const int2 bm = bmap[blockIdx.x];
    const VecJob J = jobs[bm.x];
    const int n = J.n, jr = bm.y, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    extern __shared__ double dot[];
    const double near = 1e-2 * fmax(fabs(J.w[0]), fabs(J.w[n - 1])), wj = J.w[n - 1 - jr];
    auto is_near = [&](int i) { return i >= 0 && i < J.kv && fabs(J.w[n - 1 - i] - wj) < near; };
    int lo = jr, hi = jr + 1;
    for (int c = 64; c == 64; lo -= c) c = __popcll(__ballot(is_near(lo - 1 - lane)));
    for (int c = 64; c == 64; hi += c) c = __popcll(__ballot(is_near(hi + lane)));
    const double* z = J.Zt + (size_t)jr * n;
    for (int i = lo + wave; i < hi; i += kEigWaves) {
        const double* y = J.Zt + (size_t)i * n;
        double part = 0.0;
        for (int r = lane; r < n; r += 64) part = fma(y[r], z[r], part);
        part = wave_sum(part);
        if (lane == 0) dot[i - lo] = i == jr ? 0.0 : 0.5 * part;
    }
    __syncthreads();
    for (int r = tid; r < n; r += kEigThreads) {
        const double* y = J.Zt + (size_t)lo * n + r;
        double x = z[r];
#pragma unroll 4
        for (int i = 0; i < hi - lo; ++i) x = fma(-dot[i], y[(size_t)i * n], x);
        J.Zp[(size_t)jr * n + r] = x;
    }
}

struct BackJob {
    const double *V, *tau, *Zt;   // reflectors; vectors of T (column j at Zt + j ldt)
    double* Z;                    // column j at Z + j ldz, n entries
    int n, count, ldt, ldz;       // entries, reflectors, strides
    // entry j of the vector is row_of(j) of T's: all rows, or the u (side 0)
    // or v (side 1) states of a Jordan-Wielandt matrix, `other` the size of
    // the other side (their order alternates until one side ends)
    int side, other;
    __device__ int row_of(int j) const { return side < 0 ? j : (j < other + 1 - side ? 2 * j + side : other + j); }
};

// Step 4.  NW waves per eigenvector (bmap[b] = (job, vector)), which stays in
// registers: lane entries i = tid + 64 NW q, q < SL.  The reflectors are read
// straight from memory (L2: all vectors go through them at about the same
// time), kBackAhead of them ahead; each costs one dot product, one wavefront
// sum and one update, so the dependent chain of the sum bounds it: 0.3 us per
// reflector at n = 696 with one wave.  The loads are global ones without
// conditions, at most 63 in flight where the registers allow it (flat loads
// under a test per slot were each waited for with all the others: the vectors
// of a move at D = 6, chi = 64 292 us, now 213 us; D = 8, chi = 200 2.24 and
// 2.16 ms).  One wave while a vector's entries and the reflectors ahead fit its
// registers; beyond that four waves, whose partial sums meet in LDS.
template <int NW, int SL>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(1, 1))) void backtr_kernel(const BackJob* __restrict__ jobs,
                                                          const int2* __restrict__ bmap) {
    const int2 bm = bmap[blockIdx.x];
    const BackJob J = jobs[bm.x];
    const int n = J.n, ldv = v_stride(n), tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    __shared__ double red[2][NW];
    constexpr int kBackAhead = SL <= 4 ? 12 : (SL <= 8 ? 7 : (NW > 1 ? 8 : 5));
    double z[SL], v[kBackAhead][SL], tj[kBackAhead];
    const double* zt = J.Zt + (size_t)bm.y * J.ldt;
#pragma unroll
    for (int q = 0; q < SL; ++q) {
        const int i = tid + 64 * NW * q;
        z[q] = i < n ? zt[J.row_of(i)] : 0.0;
    }
    // slots past the reflector's end read its last entries and leave z at 0
    uint32_t off[SL];
    double keep[SL];
#pragma unroll
    for (int q = 0; q < SL; ++q) {
        const int first = 64 * (wave + NW * q);
        off[q] = min(first, ldv - 64) + lane;
        keep[q] = first < ldv ? 1.0 : 0.0;
    }
    auto load = [&](int j, double (&vj)[SL], double& t) {
        const gf64* row = (const gf64*)J.V + (size_t)max(j, 0) * ldv;
        t = ((cf64*)J.tau)[max(j, 0)];
#pragma unroll
        for (int q = 0; q < SL; ++q) vj[q] = *at8(row, off[q]);
    };
#pragma unroll
    for (int u = 0; u < kBackAhead; ++u) load(J.count - 1 - u, v[u], tj[u]);
    int par = 0;
    for (int j0 = J.count - 1; j0 >= 0; j0 -= kBackAhead) {
#pragma unroll
        for (int u = 0; u < kBackAhead; ++u) {
            double part = 0.0, part2 = 0.0;
#pragma unroll
            for (int q = 0; q < SL; q += 2) {
                part += v[u][q] * z[q];
                if (q + 1 < SL) part2 += v[u][q + 1] * z[q + 1];
            }
            part = wave_sum(part + part2);
            if constexpr (NW > 1) {
                if (lane == 0) red[par][wave] = part;
                __syncthreads();
                part = 0.0;
#pragma unroll
                for (int q = 0; q < NW; ++q) part += red[par][q];
                par ^= 1;
            }
            const double f = j0 >= u ? part * tj[u] : 0.0;
#pragma unroll
            for (int q = 0; q < SL; ++q) z[q] = fma(-(f * keep[q]), v[u][q], z[q]);
            load(j0 - u - kBackAhead, v[u], tj[u]);
        }
    }
#pragma unroll
    for (int q = 0; q < SL; ++q) {
        const int i = tid + 64 * NW * q;
        if (i < n) J.Z[(size_t)bm.y * J.ldz + i] = z[q];
    }
}
// Shapes of the back-transformation by the largest order of a launch.
struct BackShape {
    int nmax, threads;
    const void* fn;
};
const BackShape kBackShapes[] = {
    {128, 64, (const void*)backtr_kernel<1, 2>},   {256, 64, (const void*)backtr_kernel<1, 4>},
    {512, 64, (const void*)backtr_kernel<1, 8>},   {704, 64, (const void*)backtr_kernel<1, 11>},
    {1024, 256, (const void*)backtr_kernel<4, 4>}, {2048, 256, (const void*)backtr_kernel<4, 8>},
    {3328, 256, (const void*)backtr_kernel<4, 13>}};

struct DevInfo {
    int lds = 0, cus = 0;
};
DevInfo dev_info() {
    static std::mutex mu;
    static std::map<int, DevInfo> cache;
    int dev = 0;
    HIPCHK(hipGetDevice(&dev));
    std::lock_guard<std::mutex> lk(mu);
    auto it = cache.find(dev);
    if (it != cache.end()) return it->second;
    DevInfo di;
    int lds = 0, cus = 0;
    HIPCHK(hipDeviceGetAttribute(&lds, hipDeviceAttributeMaxSharedMemoryPerBlock, dev));
    HIPCHK(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
    di.lds = std::min(lds, 160 * 1024) - 4096;   // room for the kernels' static shared variables
    di.cus = cus;
    cache[dev] = di;
    return di;
}

// Variant and workgroups of a job of order n (G = 0: it does not fit).
size_t tridiag_lds(const TridVariant& v) {   // Trid::LDS
    const int nw = v.T / 64, wr = nw / v.WC, nq = v.T * ((v.CW + wr - 1) / wr), np = v.nmax();
    return 8 * (size_t)(2 * nq + 2 * (v.rows() + 64) + (wr > 1 ? 2 * nq : 0) + (v.rows() >= np ? 2 * np : 0) + 2 * nw +
                        (v.WC > 1 ? nw * (v.RW + 3) : 0) + 2 + wr * v.RL * np);
}
void tridiag_shape(int n, const DevInfo& di, int& variant, int& G, bool joint = false) {
    const int end = joint ? kTridJoint + kTridJointN : kTridVariantsN;
    variant = joint ? kTridJoint : 0;
    G = 0;
    if (n <= 0) return;
    while (variant < end && kTridVariants[variant].nmax() < n) ++variant;
    if (variant == end) return;
    const TridVariant& v = kTridVariants[variant];
    const int g = (n + v.rows() - 1) / v.rows();
    // the vector steps hold T and its factorisations (5 n) in LDS
    if (g > di.cus || tridiag_lds(v) > (size_t)di.lds || 40LL * n > di.lds) return;
    G = g;
}

size_t bid_lds(const BidVariant& v) {   // Bid::LDS
    const int wr = 8 / v.WC, nq = 512 * ((v.CW + wr - 1) / wr), np = v.nmax();
    return 8 * (size_t)(nq + 4 * std::max(nq, np + v.rows()) + (v.rows() >= np ? 2 * np : 0) + 8 +
                        (v.WC > 1 ? 8 * (v.RW + 3) : 0) + 2);
}
void bid_shape(int ru, int rd, const DevInfo& di, int& variant, int& G) {
    variant = G = 0;
    const int m = std::max(ru, rd);
    if (std::min(ru, rd) <= 0) return;
    while (variant < kBidVariantsN && kBidVariants[variant].nmax() < m) ++variant;
    if (variant == kBidVariantsN) return;
    const BidVariant& v = kBidVariants[variant];
    const int g = (m + v.rows() - 1) / v.rows();
    if (g > di.cus || bid_lds(v) > (size_t)di.lds || 40LL * (ru + rd) > di.lds) return;
    G = g;
}

// Dynamic LDS limits of the solver's kernels, raised once per device.
void set_lds_limits(const DevInfo& di) {
    static std::mutex mu;
    static std::set<int> done;
    int dev = 0;
    HIPCHK(hipGetDevice(&dev));
    std::lock_guard<std::mutex> lk(mu);
    if (done.count(dev)) return;
    const char* names[] = {"tridiag", "tridiag_wide", "bidiag", "cluster", "cluster", "twist"};
    const void* fns[] = {(const void*)tridiag_kernel, (const void*)tridiag_wide_kernel, (const void*)bidiag_kernel,
                         (const void*)cluster_kernel<true>, (const void*)cluster_kernel<false>,
                         (const void*)twist_kernel};
    for (int i = 0; i < 6; ++i) {
        const hipError_t e = hipFuncSetAttribute(fns[i], hipFuncAttributeMaxDynamicSharedMemorySize, di.lds);
        if (e != hipSuccess)
            fail(SYMTEN_E_HIP, std::string("eigh: dynamic LDS limit of the ") + names[i] + " kernel: " +
                                   hipGetErrorString(e));
    }
    done.insert(dev);
}

// Doubles of a job's exchange area: maxima and XCC ids, then per column the
// p slices of its workgroups and the published row.
size_t bid_xbuf_doubles(int ru, int rd, const BidVariant& v, int G) {
    const size_t gr = ((size_t)G * v.rows() + 15) & ~(size_t)15;
    return (((size_t)2 * G + 15) & ~(size_t)15) + (size_t)bid_columns(ru, rd) * (v.nmax() + gr);
}
size_t xbuf_doubles(int n, const TridVariant& v, int G) {
    const size_t npad = v.nmax(), gr = ((size_t)G * v.rows() + 15) & ~(size_t)15;
    return (((size_t)2 * G + 15) & ~(size_t)15) + (size_t)n * (npad + gr);
}

}  // namespace

struct EighWork {
    std::vector<EighProblem> probs;
    std::vector<BufferPtr> keep;
    std::vector<double*> d, e, e2, scale, w;
    std::vector<std::array<double*, 2>> tau, V;   // Jordan-Wielandt: v side, u side
    int* status = nullptr;               // one per problem
};

bool eigh_fits(int n) {
    int R, G;
    tridiag_shape(n, dev_info(), R, G);
    return G > 0;
}

bool eigh_jw_fits(int ru, int rd) {
    int v, G;
    bid_shape(ru, rd, dev_info(), v, G);
    return G > 0;
}

int eigh_problems(const EighWork& wk) { return (int)wk.probs.size(); }

int eigh_max_order() {
    const DevInfo di = dev_info();
    int lo = 1, hi = 1 << 16;   // largest n that fits (fits is monotone in n)
    int R, G;
    while (lo < hi) {
        const int mid = (lo + hi + 1) / 2;
        tridiag_shape(mid, di, R, G);
        if (G > 0) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

std::shared_ptr<EighWork> eigh_values(const std::vector<EighProblem>& probs, hipStream_t s) {
    auto wk = std::make_shared<EighWork>();
    wk->probs = probs;
    const int np = (int)probs.size();
    if (np == 0) return wk;
    const DevInfo di = dev_info();
    std::vector<int> Vs(np), Gs(np);
    auto jw = [&](int p) { return probs[p].rd > 0; };
    auto xbuf_of = [&](int p) {
        return jw(p) ? bid_xbuf_doubles(probs[p].ru, probs[p].rd, kBidVariants[Vs[p]], Gs[p])
                     : xbuf_doubles(probs[p].n, kTridVariants[Vs[p]], Gs[p]);
    };
    for (int p = 0; p < np; ++p) {
        const EighProblem& P = probs[p];
        const int n = P.n;
        if (n < 1 || !P.A || !P.w || (jw(p) ? P.ru < 1 || P.ru + P.rd != n || P.lda < P.ru : P.lda < n))
            fail(SYMTEN_E_INVAL, "eigh: bad problem");
        if (jw(p)) bid_shape(P.ru, P.rd, di, Vs[p], Gs[p]);
        else tridiag_shape(n, di, Vs[p], Gs[p]);
        if (Gs[p] == 0) fail(SYMTEN_E_CAPACITY, "eigh: matrix of order " + std::to_string(n) + " exceeds the registers of the chip");
    }
    // ---- launches of step 1: jobs by size, packed into launches of at most
    // one workgroup per compute unit, Jordan-Wielandt jobs and jobs of 512 and of
    // 256 threads in launches of their own
    auto kind = [&](int p) { return jw(p) ? 2 : (Vs[p] >= kTridWide ? 1 : 0); };
    auto pack = [&] {
        std::vector<int> order(np);
        for (int p = 0; p < np; ++p) order[p] = p;
        std::stable_sort(order.begin(), order.end(), [&](int a, int b) {
            return kind(a) != kind(b) ? kind(a) > kind(b) : Gs[a] > Gs[b];
        });
        // largest first, each into the first launch of its kind with room
        std::vector<std::vector<int>> out;
        std::vector<int> used;
        for (int p : order) {
            size_t l = 0;
            while (l < out.size() && (kind(out[l][0]) != kind(p) || used[l] + Gs[p] > di.cus)) ++l;
            if (l == out.size()) {
                out.emplace_back();
                used.push_back(0);
            }
            out[l].push_back(p);
            used[l] += Gs[p];
        }
        return out;
    };
    std::vector<std::vector<int>> launches = pack();
    {   // all in 512-thread variants if that saves a launch
        bool kinds[3] = {false, false, false};
        for (int p = 0; p < np; ++p) kinds[kind(p)] = true;
        if (kinds[0] && kinds[1]) {
            const std::vector<int> v0 = Vs, g0 = Gs;
            bool fits = true;
            for (int p = 0; p < np; ++p)
                if (kind(p) == 0) {
                    tridiag_shape(probs[p].n, di, Vs[p], Gs[p], true);
                    fits = fits && Gs[p] > 0;
                }
            std::vector<std::vector<int>> joint;
            if (fits) joint = pack();
            if (fits && joint.size() < launches.size()) {
                launches = std::move(joint);
            } else {
                Vs = v0;
                Gs = g0;
            }
        }
    }
    size_t doubles = 0, xdoubles = 0;
    for (int p = 0; p < np; ++p) {
        const EighProblem& P = probs[p];
        const int n = P.n;
        xdoubles += xbuf_of(p);
        doubles += 3 * (size_t)n + 1;
        doubles += jw(p) ? ((size_t)P.ru + P.rd) + (size_t)std::min(P.ru, P.rd) * (v_stride(P.ru) + v_stride(P.rd))
                         : (size_t)n + (size_t)n * v_stride(n);
    }
    doubles += xdoubles;
    BufferPtr buf = device_alloc(8 * doubles + 8 * (size_t)np * 2);
    BufferPtr ibuf = device_alloc(sizeof(int) * (size_t)np);
    launch_fill_zero(ibuf->ptr, sizeof(int) * (int64_t)np, s);
    wk->keep = {buf, ibuf};
    wk->status = (int*)ibuf->ptr;
    std::vector<TridJob> tj(np);
    std::vector<BidJob> gj(np);
    // the exchange areas first (each a multiple of 16 doubles, so each
    // starts on a 128-byte line of the pool's aligned block), then the rest
    double* q = (double*)buf->ptr;
    hipLaunchKernelGGL(fill_empty_kernel, dim3((unsigned)std::min<size_t>((xdoubles + 255) / 256, 4096)), dim3(256), 0,
                       s, (uint64_t*)buf->ptr, (int64_t)xdoubles);
    HIPCHK(hipGetLastError());
    std::vector<double*> xb(np);
    for (int p = 0; p < np; ++p) {
        xb[p] = q;
        q += xbuf_of(p);
    }
    for (int p = 0; p < np; ++p) {
        const EighProblem& P = probs[p];
        const int n = P.n;
        std::array<double*, 2> V{}, tau{};
        if (jw(p)) {
            const int m = std::min(P.ru, P.rd);
            V[0] = q; q += (size_t)m * v_stride(P.rd);
            V[1] = q; q += (size_t)m * v_stride(P.ru);
            tau[0] = q; q += P.rd;
            tau[1] = q; q += P.ru;
        } else {
            V[0] = q; q += (size_t)n * v_stride(n);
            tau[0] = q; q += n;
        }
        double* d = q; q += n;
        double* e = q; q += n;
        double* e2 = q; q += n;
        double* scale = q; q += 1;
        int* status = P.status ? P.status : wk->status + p;
        if (jw(p)) gj[p] = BidJob{P.A, P.ru, P.rd, P.lda, Gs[p], Vs[p], d, e, e2, scale, {V[0], V[1]}, {tau[0], tau[1]}, xb[p], status};
        else tj[p] = TridJob{P.A, n, P.lda, Gs[p], d, e, e2, tau[0], V[0], scale, xb[p], status, Vs[p]};
        wk->d.push_back(d);
        wk->e.push_back(e);
        wk->e2.push_back(e2);
        wk->tau.push_back(tau);
        wk->V.push_back(V);
        wk->scale.push_back(scale);
        wk->w.push_back(P.w);
    }
    // a job that fits one XCD (cus / 8 workgroups) takes blocks b = x (mod 8) of
    // one XCD x
    const int per_xcd = std::max(1, di.cus / 8);
    const size_t lds_bytes = (size_t)di.lds;
    set_lds_limits(di);
    std::vector<BufferPtr> descs;
    for (auto& L : launches) {
        // slots per XCD: slot t of XCD x is block x + 8 t
        std::vector<std::vector<int2>> xcd(8);
        std::vector<int2> spill;
        for (int p : L) {
            int best = -1;
            if (Gs[p] <= per_xcd)
                for (int x = 0; x < 8; ++x)
                    if ((int)xcd[x].size() + Gs[p] <= per_xcd && (best < 0 || xcd[x].size() < xcd[best].size()))
                        best = x;
            for (int r = 0; r < Gs[p]; ++r) {
                if (best >= 0) xcd[best].push_back(make_int2(p, r));
                else spill.push_back(make_int2(p, r));
            }
        }
        for (auto& sp : spill) {   // jobs wider than an XCD: the emptiest XCDs first
            int x = 0;
            for (int y = 1; y < 8; ++y)
                if (xcd[y].size() < xcd[x].size()) x = y;
            xcd[x].push_back(sp);
        }
        size_t depth = 0;
        for (auto& v : xcd) depth = std::max(depth, v.size());
        std::vector<int2> bmap(8 * depth, make_int2(-1, 0));
        for (int x = 0; x < 8; ++x)
            for (size_t t = 0; t < xcd[x].size(); ++t) bmap[x + 8 * t] = xcd[x][t];
        // the job descriptors and the block map in one upload
        const int kd = kind(L[0]);
        const size_t jb = (kd == 2 ? sizeof(BidJob) : sizeof(TridJob)) * np, mb = sizeof(int2) * bmap.size();
        std::vector<char> host(jb + mb);
        std::memcpy(host.data(), kd == 2 ? (const void*)gj.data() : (const void*)tj.data(), jb);
        std::memcpy(host.data() + jb, bmap.data(), mb);
        BufferPtr db;
        upload_async(db, host.data(), host.size(), s);
        descs.push_back(db);
        const void* djobs = db->ptr;
        const int2* dmap = (const int2*)((const char*)db->ptr + jb);
        void* args[] = {(void*)&djobs, (void*)&dmap};
        // Householder reduction (FP64): 4/3 n^3, of Y to its Golub-Kahan form
        // 4 (m n^2 - n^3 / 3), n <= m
        int64_t flops = 0;
        for (int p : L) {
            const int64_t n = kd == 2 ? std::min(probs[p].ru, probs[p].rd) : probs[p].n,
                          m = kd == 2 ? std::max(probs[p].ru, probs[p].rd) : 0;
            flops += kd == 2 ? 4 * (m * n * n - n * n * n / 3) : 4 * n * n * n / 3;
        }
        const void* fn[] = {(const void*)tridiag_kernel, (const void*)tridiag_wide_kernel, (const void*)bidiag_kernel};
        profile_launch(kd == 2 ? "eigh_bidiag" : "eigh_tridiag", flops, flops, 0, s, [&] {
            HIPCHK(hipLaunchCooperativeKernel(fn[kd], dim3((unsigned)bmap.size()), dim3(kd ? 512 : 256), args,
                                              (unsigned)lds_bytes, s));
        });
    }
    // ---- step 2: 64 points of the grid, then one eigenvalue, per wave; four
    // waves per workgroup
    {
        size_t points = 0;
        for (int p = 0; p < np; ++p) points += grid_points(probs[p].n);
        BufferPtr grid = device_alloc(8 * 3 * (size_t)np + sizeof(int) * points);
        double* range = (double*)grid->ptr;
        int* count = (int*)(range + 3 * (size_t)np);
        std::vector<BisJob> bj(np);
        std::vector<int2> gmap, bmap;
        for (int p = 0; p < np; ++p) {
            const int n = probs[p].n, half = jw(p) ? std::min(probs[p].ru, probs[p].rd) : 0;
            const int pts = grid_points(n);
            bj[p] = BisJob{wk->d[p], wk->e[p], wk->e2[p], wk->scale[p], probs[p].w, range + 3 * p, count, n, pts, half};
            count += pts;
            for (int t = 0; t < pts / 64; t += kEigWaves) gmap.push_back(make_int2(p, t));
            for (int j = half ? n - half : 0; j < n; j += kEigWaves) bmap.push_back(make_int2(p, j));
        }
        Tables tab;
        const size_t oj = tab.add(bj), og = tab.add(gmap), ob = tab.add(bmap);
        tab.send(s);
        profile_launch("eigh_bisect", 0, 0, 0, s, [&] {
            hipLaunchKernelGGL(bisect_grid_kernel, dim3((unsigned)gmap.size()), dim3(kEigThreads), 0, s,
                               tab.at<BisJob>(oj), tab.at<int2>(og));
            HIPCHK(hipGetLastError());
            hipLaunchKernelGGL(bisect_kernel, dim3((unsigned)bmap.size()), dim3(kEigThreads), 0, s,
                               tab.at<BisJob>(oj), tab.at<int2>(ob));
            HIPCHK(hipGetLastError());
        });
    }
    for (auto& b : descs) wk->keep.push_back(b);
    return wk;
}

void eigh_status(const EighWork& wk, hipStream_t s) {
    const int np = (int)wk.probs.size();
    if (np == 0) return;
    std::vector<int> st(np);
    HIPCHK(hipMemcpyAsync(st.data(), wk.status, sizeof(int) * np, hipMemcpyDeviceToHost, s));
    HIPCHK(hipStreamSynchronize(s));
    for (int v : st)
        if (v) fail(SYMTEN_E_HIP, "eigh: the workgroups of a tridiagonalisation did not meet");
}

void eigh_vectors(EighWork& wk, const std::vector<int>& kv, const std::vector<double*>& Z,
                  const std::vector<const double*>& w_host, hipStream_t s) {
    const int np = (int)wk.probs.size();
    if ((int)kv.size() != np || (int)Z.size() != np || (int)w_host.size() != np)
        fail(SYMTEN_E_INVAL, "eigh_vectors: one entry per problem");
    // clusters of close eigenvalues (descending), from the host copy of w
    std::vector<VecCluster> cl;
    size_t ztot = 0, worktot = 0;
    int nvec = 0, nmax = 0, ncmax = 0, kmax = 0;
    for (int p = 0; p < np; ++p) {
        const int n = wk.probs[p].n, k = kv[p];
        if (k < 0 || k > n) fail(SYMTEN_E_INVAL, "eigh_vectors: vector count out of range");
        if (k == 0) continue;
        const double* w = w_host[p];
        const double tn = std::max(std::fabs(w[0]), std::fabs(w[n - 1]));
        const double ortol = 1e-3 * tn;
        nvec += k;
        nmax = std::max(nmax, n);
        kmax = std::max(kmax, k);
        int j = 0;
        while (j < k) {
            int c = 1;
            while (j + c < k && w[n - 1 - (j + c - 1)] - w[n - 1 - (j + c)] <= ortol) ++c;
            if (c > 1) {
                cl.push_back(VecCluster{p, j, c, 0, (int64_t)worktot});
                worktot += 5 * (size_t)n;
                ncmax = std::max(ncmax, n);
            }
            j += c;
        }
        ztot += (size_t)n * k;
    }
    if (nvec == 0) return;
    BufferPtr zt = device_alloc(8 * 2 * ztot);   // as they come, then polished
    BufferPtr work = device_alloc(8 * std::max<size_t>(worktot, 1));
    std::vector<VecJob> vj(np);
    std::vector<BackJob> bj;
    std::vector<int2> bmap, tmap;   // (problem, vector), (back-transformation, vector)
    size_t zo = 0;
    int nbmax = 0;
    for (int p = 0; p < np; ++p) {
        const EighProblem& P = wk.probs[p];
        const int n = P.n;
        double *zr = (double*)zt->ptr + zo, *z = zr + ztot;
        vj[p] = VecJob{wk.d[p], wk.e[p], wk.scale[p], wk.w[p], zr, z, (double*)work->ptr, n, kv[p]};
        for (int c = 0; c < kv[p]; ++c) bmap.push_back(make_int2(p, c));
        const int first = (int)bj.size();
        if (P.rd > 0) {   // the u and the v entries go back on their own
            const int H = bid_columns(P.ru, P.rd);
            bj.push_back(BackJob{wk.V[p][1], wk.tau[p][1], z, Z[p], P.ru, H / 2, n, n, 0, P.rd});
            bj.push_back(BackJob{wk.V[p][0], wk.tau[p][0], z, Z[p] ? Z[p] + P.ru : nullptr, P.rd, (H + 1) / 2, n, n, 1, P.ru});
        } else {
            bj.push_back(BackJob{wk.V[p][0], wk.tau[p][0], z, Z[p], n, n - 1, n, n, -1, 0});
        }
        for (int b = first; b < (int)bj.size() && kv[p] > 0; ++b) {
            nbmax = std::max(nbmax, bj[b].n);
            for (int c = 0; c < kv[p]; ++c) tmap.push_back(make_int2(b, c));
        }
        zo += (size_t)n * kv[p];
    }
    const size_t b1 = sizeof(VecJob) * np, b2 = sizeof(VecCluster) * cl.size(), b3 = sizeof(BackJob) * bj.size(),
                 b4 = sizeof(int2) * bmap.size(), b5 = sizeof(int2) * tmap.size();
    std::vector<char> host(b1 + b2 + b3 + b4 + b5);
    std::memcpy(host.data(), vj.data(), b1);
    std::memcpy(host.data() + b1, cl.data(), b2);
    std::memcpy(host.data() + b1 + b2, bj.data(), b3);
    std::memcpy(host.data() + b1 + b2 + b3, bmap.data(), b4);
    std::memcpy(host.data() + b1 + b2 + b3 + b4, tmap.data(), b5);
    BufferPtr db;
    upload_async(db, host.data(), host.size(), s);
    const char* base = (const char*)db->ptr;
    const DevInfo di = dev_info();
    set_lds_limits(di);
    const BackShape* bs = nullptr;
    for (auto& x : kBackShapes)
        if (!bs && x.nmax >= nbmax) bs = &x;
    if (!bs || 40 * (size_t)nmax > (size_t)di.lds) fail(SYMTEN_E_CAPACITY, "eigh: vectors exceed the registers or LDS");
    const VecJob* dvj = (const VecJob*)base;
    const int2* dmap = (const int2*)(base + b1 + b2 + b3);
    profile_launch("eigh_twist", 0, 0, 0, s, [&] {
        hipLaunchKernelGGL(twist_kernel, dim3((unsigned)nvec), dim3(128), 40 * (size_t)nmax, s, dvj, dmap);
        HIPCHK(hipGetLastError());
    });
    if (!cl.empty())
        profile_launch("eigh_cluster", 0, 0, 0, s, [&] {
            const VecCluster* dcl = (const VecCluster*)(base + b1);
            if (64 * (size_t)ncmax <= (size_t)di.lds)
                hipLaunchKernelGGL(cluster_kernel<true>, dim3((unsigned)cl.size()), dim3(64), 64 * (size_t)ncmax, s,
                                   dvj, dcl);
            else
                hipLaunchKernelGGL(cluster_kernel<false>, dim3((unsigned)cl.size()), dim3(64), 24 * (size_t)ncmax, s,
                                   dvj, dcl);
            HIPCHK(hipGetLastError());
        });
    profile_launch("eigh_polish", 0, 0, 0, s, [&] {
        hipLaunchKernelGGL(polish_kernel, dim3((unsigned)nvec), dim3(kEigThreads), 8 * (size_t)kmax, s, dvj, dmap);
        HIPCHK(hipGetLastError());
    });
    int64_t bflops = 0;   // back-transformation: 2 n^2 per vector
    for (auto& t : tmap) bflops += 2 * (int64_t)bj[t.x].n * bj[t.x].n;
    profile_launch("eigh_backtr", bflops, bflops, 0, s, [&] {
        const BackJob* dbj = (const BackJob*)(base + b1 + b2);
        const int2* dtmap = dmap + bmap.size();
        void* args[] = {(void*)&dbj, (void*)&dtmap};
        HIPCHK(hipLaunchKernel(bs->fn, dim3((unsigned)tmap.size()), dim3((unsigned)bs->threads), args, 0, s));
    });
    wk.keep.push_back(zt);
    wk.keep.push_back(work);
    wk.keep.push_back(db);
}

}  // namespace symten
