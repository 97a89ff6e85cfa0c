// Pressure solver of Karp et al. (arXiv 2207.07098), Sec. II-B: restarted
// GMRES preconditioned by an overlapping additive Schwarz method with a
// coarse-grid solve of 10 P-CG iterations (the hybrid Schwarz scheme of
// Lottes & Fischer cited there).
//
//  * Local solves: every element extended by one node layer across each
//    face that has a neighbour, on the box [-1, N+1]^3 of local indices
//    (edge and corner points of the extension carry no data); the operator
//    on the box is the separable approximation
//    M_t x M_s x K_r + M_t x K_s x M_r + K_t x M_s x M_r from 1D stiffness K
//    and lumped mass M of the neighbour-element-neighbour line (mean edge
//    lengths), solved by fast diagonalisation: per direction K S = M S Lambda
//    (host, once), then u = S (Lambda_r + Lambda_s + Lambda_t)^-1 S^T r with
//    three tensor contractions each way on matrix cores (one element per
//    wave, the box gathered through a map built at bind time), in the
//    precision of the vectors (FP32 tables for the inner FP32 solves).
//  * Additive combination with counting weights (1 / number of subdomains
//    holding the node): the boxes are stored whole and summed node by node.
//  * Coarse grid: the N = 1 operator on the element vertices (its own
//    context), trilinear interpolation P and restriction P^T (summed in the
//    local-solve gather when both parts run), 10 Jacobi-PCG iterations from
//    zero on the assembled operator (sem_coarse.hip).
//  * Flexible GMRES(m) (the coarse PCG makes the preconditioner nonlinear):
//    Arnoldi with classical Gram-Schmidt twice, the second projection of
//    each new vector delayed to the next step (two sweeps over the basis
//    per step, each compiled for the exact basis size and streamed with
//    non-temporal accesses), Givens rotations on the host, FP64 sums
//    throughout; or FP64 refinement around FP32-vector GMRES, whose 16-bit
//    operator steps down to FP32 when its corrections stall.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <array>
#include <cfloat>
#include <chrono>
#include <cmath>
#include <cstring>
#include <map>
#include <memory>
#include <type_traits>
#include <unordered_map>

#include "sem_coarse.h"
#include "sem_internal.h"
#include "sem_reduce.h"
#include "sem_threads.h"

using namespace sem;

namespace {

constexpr int kGmBlock = 256;
constexpr int kGmGrid = 2048;
constexpr int kGmMaxVec = 32;            // basis vectors in one multi-dot
// coef[] slots: single-vector sums at 0.., the sums of a delayed step at
// kGmD.. (2 * kGmMaxVec + 3 values); in the host's copy also that step's
// scalars at kGmScal..
constexpr int kGmD = kGmMaxVec + 2, kGmScal = kGmD + 2 * kGmMaxVec + 4;
constexpr int kGmCoef = kGmScal + 4;

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

unsigned gm_grid(int64_t n) {
    const int64_t g = (n + kGmBlock - 1) / kGmBlock;
    return (unsigned)std::max<int64_t>(1, std::min<int64_t>(g, kGmGrid));
}

__device__ double gm_block_sum(double v, double *red) {
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        const double o = __shfl_xor(v, off, 64);
        v += ((lane ^ off) < (int)blockDim.x - wv * 64) ? o : 0.0;
    }
    __syncthreads();
    if (lane == 0) red[wv] = v;
    __syncthreads();
    double s = 0.0;
    for (int q = 0; q < nw; ++q) s += red[q];
    return s;
}

__device__ __forceinline__ int64_t gm_interior(int64_t n_bnd, int64_t e, int i, int j, int k, int N) {
    const int nm = N - 1;
    return n_bnd + e * (int64_t)(nm * nm * nm) + ((k - 1) * nm + (j - 1)) * nm + (i - 1);
}

__device__ __forceinline__ int gm_ring(int i, int j, int N) {
    if (j == 0) return i;
    if (j == N) return N + 1 + 2 * (N - 1) + i;
    return N + 1 + 2 * (j - 1) + (i == 0 ? 0 : 1);
}

__device__ __forceinline__ int gm_bpos(int i, int j, int k, int n1) {
    const int N = n1 - 1, C = n1 * n1;
    if (k == 0) return i + n1 * j;
    if (k == N) return C + (N - 1) * 4 * N + i + n1 * j;
    return C + (k - 1) * 4 * N + gm_ring(i, j, N);
}

// Solver index of local point (i,j,k) of element e, or -1 on a Dirichlet node.
__device__ __forceinline__ int64_t gm_node(const int32_t *bmap, int64_t n_bnd, int64_t e, int i,
                                           int j, int k, int N, int nb) {
    if (i == 0 || i == N || j == 0 || j == N || k == 0 || k == N) {
        const int32_t m = bmap[e * nb + gm_bpos(i, j, k, N + 1)];
        return m < 0 ? -1 : (int64_t)m;
    }
    return gm_interior(n_bnd, e, i, j, k, N);
}

// The local solves compute in the precision of the vectors they act on:
// FP64 for the FP64 GMRES, FP32 (tables rounded once at bind time) for the
// FP32 inner solves of the refinement, whose corrections the FP64 outer
// residual judges.
template <typename VT>
struct FdmParams {
    const VT *r;              // residual (unique, solver order; FP64 or FP32)
    VT *o;                    // [E][BoxStore::SIZE] local solutions
    const int32_t *at;        // [NE][NE^2] storage position of a box point or -1
    const VT *S;              // [E][3][NE][NE] eigenvectors S[a][m]
    const VT *lam;            // [E][3][NE]
    const int32_t *fmap;      // [E][NE][NE^2] box gather map: solver index or -1
    int64_t E;
    // coarse restriction fused into the gather (b0 null: not done here)
    const uint16_t *own;      // [E][NE^2] bit c: box point (a, b, c) is an owned node of e
    double *b0;               // coarse right-hand side, summed atomically
    const int32_t *cmap;      // [E][8] coarse index of each element corner or -1
    const double *xi;         // GLL nodes [N+1]
};

// Storage of an element's local solution: the values of its interior points
// (solver order of the element interior), of its boundary points (order of the
// element map), then of the six extension planes (p + n1 q each), so that the
// sum reads contiguous runs; edges and corners of the extension carry no data.
// Padded to multiples of 64 bytes of FP64.
template <int NE>
struct BoxStore {
    static constexpr int N = NE - 3, N1 = N + 1, NI = (N - 1) * (N - 1) * (N - 1),
                         NB = N1 * N1 * N1 - NI, F2 = N1 * N1, SIZE = (NI + NB + 6 * F2 + 7) / 8 * 8;
    // position of box point (a, b, c), -1 for the edges and corners
    static __device__ int at(int a, int b, int c) {
        const int i = a - 1, j = b - 1, k = c - 1;
        const bool oi = i < 0 || i > N, oj = j < 0 || j > N, ok = k < 0 || k > N;
        if (oi + oj + ok > 1) return -1;
        if (oi) return NI + NB + (i < 0 ? 0 : 1) * F2 + j + N1 * k;
        if (oj) return NI + NB + (j < 0 ? 2 : 3) * F2 + i + N1 * k;
        if (ok) return NI + NB + (k < 0 ? 4 : 5) * F2 + i + N1 * j;
        if (i == 0 || i == N || j == 0 || j == N || k == 0 || k == N) return NI + gm_bpos(i, j, k, N1);
        return ((k - 1) * (N - 1) + (j - 1)) * (N - 1) + i - 1;
    }
};

// Box gather map of every element, built once when the workspace is bound
// (with the storage positions at[c][a + NE b] of a box):
// fmap[e][c][a + NE b] = solver index of box point (a, b, c) (own points
// through the element's map, one-layer extension through the face map),
// -1 where the box holds no data (edges and corners of the extension).
template <int NE>
__global__ void __launch_bounds__((NE * NE + 63) / 64 * 64)
k_fdm_map(const int32_t *__restrict__ ghost, const int32_t *__restrict__ bmap,
          const uint8_t *__restrict__ owner, int64_t E, int64_t n_bnd, int nb,
          int32_t *__restrict__ fmap, uint16_t *__restrict__ own, int32_t *__restrict__ at) {
    constexpr int C = NE * NE, N = NE - 3, n1 = NE - 2;
    const int64_t e = blockIdx.x;
    const int t = threadIdx.x;
    if (t >= C || e >= E) return;
    if (e == 0)
        for (int c = 0; c < NE; ++c) at[c * C + t] = BoxStore<NE>::at(t % NE, t / NE, c);
    const int i = t % NE - 1, j = t / NE - 1;
    // owned own points of the column: interior points, and on the element
    // boundary the first copy of a non-Dirichlet node
    uint32_t mask = 0;
    if (i >= 0 && i <= N && j >= 0 && j <= N)
        for (int k = 0; k <= N; ++k) {
            const bool bnd = i == 0 || i == N || j == 0 || j == N || k == 0 || k == N;
            bool take = true;
            if (bnd) {
                const int b = gm_bpos(i, j, k, N + 1);
                take = bmap[e * nb + b] >= 0 && owner[e * nb + b];
            }
            if (take) mask |= 1u << (k + 1);
        }
    own[(size_t)e * C + t] = (uint16_t)mask;
    for (int c = 0; c < NE; ++c) {
        const int k = c - 1;
        const int oi = (i < 0 || i > N), oj = (j < 0 || j > N), ok = (k < 0 || k > N);
        int64_t g = -1;
        if (oi + oj + ok == 0) {
            g = gm_node(bmap, n_bnd, e, i, j, k, N, nb);
        } else if (oi + oj + ok == 1) {
            int f, p, q;
            if (oi) { f = i < 0 ? 0 : 1; p = j; q = k; }
            else if (oj) { f = j < 0 ? 2 : 3; p = i; q = k; }
            else { f = k < 0 ? 4 : 5; p = i; q = j; }
            g = ghost[((size_t)e * 6 + f) * n1 * n1 + p + n1 * q];
        }
        fmap[((size_t)e * NE + c) * C + t] = (int32_t)g;
    }
}

// Fast-diagonalisation solve on matrix cores, one element per wave.
//
// Each of the six contractions (S_t^T, S_s^T, S_r^T, then S_r, S_s, S_t) is a
// NE x NE by NE x NE^2 product: 16x16x4 MFMAs with the matrix padded to 16
// rows as operand A (lane: row lane % 16, column 4 s + lane / 16 in step s)
// and 16 lines of the box per tile as operand B (lane: line lane % 16).  The
// box is gathered straight into operand layout for the t-direction, passes
// through one LDS buffer whenever the contracted direction changes ([index to
// be contracted next][line], with pitches that keep the transposing writes
// free of bank conflicts), and the r-direction's forward result is already the
// operand of its backward pass (result row = the next contraction index; FP32
// results lie at row 4 (lane / 16) + register, FP64 ones at 4 register + lane
// / 16, and the operand A follows).  One wave per workgroup: its LDS
// operations stay in order, so there are no workgroup barriers.
//
// What bounds it at NE = 10 in FP64: 126 MFMAs of 64 cycles per element (54% of
// the kernel's SIMD cycles; 10 of 16 rows are used) and about 1150 vector
// instructions (34%), which share the issue of three waves per SIMD; 1.9 GB of
// maps, tables and box values at 48^3 are 0.3 ms.  0.78 ms there.  A lane that
// held a column of the box and took every product on the vector ALUs read
// one LDS operand per FMA, four times what LDS delivers, and added the result
// with 99 million atomics: 2.02 ms (21x18x16, NE = 9 in FP32: 78 -> 33 us).  A
// persistent form with the next element's map in flight kept 20 more
// registers alive and spilled 54 of them at three waves (1.35 ms).
template <int NE, typename VT>
struct FdmShape {
    static constexpr int C = NE * NE, T = (C + 15) / 16, KS = (NE + 3) / 4;
    // Row pitch of the LDS buffer where a line's results go to row hi ([hi][lo
    // + NE row]) and to row lo ([lo][row + NE hi]): for NE = 5..16 the smallest
    // values that cost the fewest LDS cycles over the writes and reads of a pass
    // with 16 (FP64) or 32 (FP32) lanes served per cycle, found by a search over
    // 34 pitches (tests/test_lds_pitches.py repeats it; NE = 10 in FP64: 168 and
    // 168 cycles, none lost to conflicts; a pitch of 112 for both: 198 and 563,
    // and 62% of the LDS cycles counted as conflicts).
    static constexpr int kHi64[12] = {37, 38, 55, 72, 89, 106, 123, 156, 173, 206, 239, 256};
    static constexpr int kLo64[12] = {33, 41, 49, 65, 81, 105, 129, 145, 177, 201, 225, 257};
    static constexpr int kHi32[12] = {25, 48, 80, 80, 112, 112, 144, 156, 176, 208, 240, 272};
    static constexpr int kLo32[12] = {45, 39, 81, 85, 82, 105, 146, 149, 174, 211, 231, 275};
    static constexpr int PHI = sizeof(VT) == 8 ? kHi64[NE - 5] : kHi32[NE - 5];
    static constexpr int PLO = sizeof(VT) == 8 ? kLo64[NE - 5] : kLo32[NE - 5];
    static constexpr int ROWS = NE * (PHI > PLO ? PHI : PLO);
    static_assert(PHI >= C && PLO >= C, "a row holds all lines");
};

typedef double gm_d4 __attribute__((ext_vector_type(4)));
typedef float gm_f4 __attribute__((ext_vector_type(4)));
template <typename T> struct GmAcc;
template <> struct GmAcc<double> {
    using type = gm_d4;
    static constexpr int QMUL = 1, RMUL = 4;        // result row = QMUL (lane / 16) + RMUL reg
    static __device__ __forceinline__ gm_d4 mma(double a, double b, gm_d4 c) {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
};
template <> struct GmAcc<float> {
    using type = gm_f4;
    static constexpr int QMUL = 4, RMUL = 1;
    static __device__ __forceinline__ gm_f4 mma(float a, float b, gm_f4 c) {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
};

// 1 / x to rounding for positive normal x (the hardware estimate and Newton
// steps; a division adds scaling for the ends of the exponent range).  The FP32
// tables are scaled so that every sum it is used on is normal.
__device__ __forceinline__ double gm_inverse(double x) {
    double y = __builtin_amdgcn_rcp(x);
    y = fma(fma(-x, y, 1.0), y, y);
    return fma(fma(-x, y, 1.0), y, y);
}
__device__ __forceinline__ float gm_inverse(float x) {
    const float y = __builtin_amdgcn_rcpf(x);
    return fmaf(fmaf(-x, y, 1.0f), y, y);
}

// Waves per SIMD the register budget allows for: operands and results of all
// tiles are live at once (NE = 10: 7 tiles).
template <int NE, typename VT>
struct FdmOcc {
    static constexpr int value =
        sizeof(VT) == 8 ? (NE <= 8 ? 5 : (NE <= 10 ? 3 : (NE <= 12 ? 2 : 1)))
                        : (NE <= 8 ? 5 : (NE <= 10 ? 4 : (NE <= 12 ? 3 : (NE <= 14 ? 2 : 1))));
};

template <int NE, typename VT>
__global__ void __attribute__((amdgpu_flat_work_group_size(64, 64),
                               amdgpu_waves_per_eu(FdmOcc<NE, VT>::value)))
k_fdm(FdmParams<VT> P) {
    using Sh = FdmShape<NE, VT>;
    using A = GmAcc<VT>;
    using Acc = typename A::type;
    constexpr int C = Sh::C, T = Sh::T, KS = Sh::KS;
    constexpr int NR = A::RMUL == 4 ? KS : 4;       // result registers that hold rows < NE
    constexpr int QS = (3 * C + 63) / 64;
    // + 64: results of padded rows and lines, and what the last tile's reads
    // of the last row go beyond it
    __shared__ VT buf[Sh::ROWS + 64];
    __shared__ VT Sl[3 * C];
    __shared__ VT lams[3][NE];
    __shared__ double phi[2][NE];                   // coarse shape functions at the box points
    const int64_t e = blockIdx.x;
    const int lane = threadIdx.x, j = lane & 15, q = lane >> 4;
    // ---- gather map, eigenvectors and eigenvalues of the element
    int32_t idx[T][KS];
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            const int col = 16 * t + j, k = 4 * s + q;
            const bool ok = col < C && k < NE;
            const int32_t m = __builtin_nontemporal_load(
                P.fmap + ((size_t)e * NE + (k < NE ? k : NE - 1)) * C + (col < C ? col : C - 1));
            idx[t][s] = ok ? m : -1;
        }
    VT sr[QS];
#pragma unroll
    for (int x = 0; x < QS; ++x)
        sr[x] = __builtin_nontemporal_load(P.S + (size_t)e * 3 * C + min(lane + 64 * x, 3 * C - 1));
    const VT lr0 = P.lam[(size_t)e * 3 * NE + min(lane, 3 * NE - 1)];
    int32_t corner = -1;                            // of the lane's element corner (lane < 8)
    uint32_t own[T];
    if (P.b0) {
        corner = P.cmap[e * 8 + (lane & 7)];
#pragma unroll
        for (int t = 0; t < T; ++t) {
            const int col = 16 * t + j;
            const uint32_t m = P.own[(size_t)e * C + (col < C ? col : C - 1)];
            own[t] = col < C ? m : 0u;
        }
        if (lane < NE) {
            const bool in = lane >= 1 && lane <= NE - 2;
            const double x = P.xi[in ? lane - 1 : 0];
            phi[0][lane] = in ? 0.5 * (1.0 - x) : 0.0;
            phi[1][lane] = in ? 0.5 * (1.0 + x) : 0.0;
        }
    }
    wave_lds_sync();
    VT v[T][KS];
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            const VT x = P.r[idx[t][s] >= 0 ? idx[t][s] : 0];
            v[t][s] = idx[t][s] >= 0 ? x : VT(0);
        }
#pragma unroll
    for (int x = 0; x < QS; ++x)
        if (lane + 64 * x < 3 * C) Sl[lane + 64 * x] = sr[x];
    if (lane < 3 * NE) lams[lane / NE][lane % NE] = lr0;
    wave_lds_sync();
    // ---- P^T r over the element's owned points: the t-shape functions on the
    // lane's points, then the r and s ones, one wave sum per corner
    if (P.b0) {
        double cs[8] = {};
        double p0[KS], p1[KS];
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            const int k = 4 * s + q, kc = k < NE ? k : NE - 1;   // phi is zero at NE - 1
            p0[s] = phi[0][kc];
            p1[s] = phi[1][kc];
        }
#pragma unroll
        for (int t = 0; t < T; ++t) {
            const int col = 16 * t + j, a = col % NE, b = col / NE;
            double x0 = 0.0, x1 = 0.0;
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                const double vc = ((own[t] >> (4 * s + q)) & 1u) ? (double)v[t][s] : 0.0;
                x0 += p0[s] * vc;
                x1 += p1[s] * vc;
            }
            const int bc = b < NE ? b : NE - 1;
            const double fa0 = phi[0][a], fa1 = phi[1][a], fb0 = phi[0][bc], fb1 = phi[1][bc];
            const double y[4] = {fb0 * x0, fb1 * x0, fb0 * x1, fb1 * x1};
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                cs[2 * u] += fa0 * y[u];
                cs[2 * u + 1] += fa1 * y[u];
            }
        }
        // corner u's sum from lane 63 to lane u: one atomic instruction
        double mine = 0.0;
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const double sum = wave_total(cs[u]);
            mine = lane == u ? sum : mine;
        }
        if (lane < 8 && corner >= 0) unsafeAtomicAdd(P.b0 + corner, mine);
    }
    // ---- contractions.  Line (lo, hi) of a tile; the LDS positions of its
    // results for the next direction: w1 = [hi][lo + NE row], w2 = [lo][row + NE hi]
    Acc acc[T];
    // S_d^T (row = mode, contracted over points) or S_d (row = point)
    const int jc = j < NE ? j : NE - 1;
    auto contract = [&](int d, bool forward) {
        VT a[KS];
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            const int k = 4 * s + q, kc = k < NE ? k : NE - 1;
            const VT x = Sl[d * C + (forward ? kc * NE + jc : jc * NE + kc)];
            a[s] = j < NE && k < NE ? x : VT(0);
        }
#pragma unroll
        for (int t = 0; t < T; ++t) acc[t] = Acc{0, 0, 0, 0};
#pragma unroll
        for (int s = 0; s < KS; ++s)
#pragma unroll
            for (int t = 0; t < T; ++t) acc[t] = A::mma(a[s], v[t][s], acc[t]);
    };
    auto put = [&](bool by_hi) {
#pragma unroll
        for (int t = 0; t < T; ++t) {
            const int col = 16 * t + j, lo = col % NE, hi = col / NE;
            const int base = by_hi ? hi * Sh::PHI + lo : lo * Sh::PLO + NE * hi;
            const int step = by_hi ? NE : 1;
#pragma unroll
            for (int r = 0; r < NR; ++r) {
                const int row = A::QMUL * q + A::RMUL * r;
                buf[col < C && row < NE ? base + step * row : Sh::ROWS + lane] = acc[t][r];
            }
        }
        wave_lds_sync();
    };
    auto get = [&](bool by_hi) {
        const int pitch = by_hi ? Sh::PHI : Sh::PLO;
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            const int k = 4 * s + q, kc = k < NE ? k : NE - 1;   // operand A is zero beyond NE
#pragma unroll
            for (int t = 0; t < T; ++t) v[t][s] = buf[kc * pitch + 16 * t + j];
        }
        wave_lds_sync();
    };
    contract(2, true);                              // t forward: lines (a, b)
    put(true);
    get(true);
    contract(1, true);                              // s forward: lines (a, m_t)
    put(false);
    get(false);
    contract(0, true);                              // r forward: lines (m_s, m_t)
    {
        const VT cut = VT(1e-13) * (lams[0][NE - 1] + lams[1][NE - 1] + lams[2][NE - 1]);
        VT lr[NR], aR[NR];                          // S_r in the order of the result rows
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            const int row = A::QMUL * q + A::RMUL * r, rc = row < NE ? row : NE - 1;
            lr[r] = lams[0][rc];
            const VT x = Sl[jc * NE + rc];
            aR[r] = j < NE && row < NE ? x : VT(0);
        }
        Acc in[T];
#pragma unroll
        for (int t = 0; t < T; ++t) {
            const int col = 16 * t + j, lo = col % NE, hi = col / NE < NE ? col / NE : NE - 1;
            const VT ls = lams[1][lo] + lams[2][hi];
            // a zero sum only for an element without any neighbour or
            // Dirichlet face (its constant mode): pseudo-inverse
#pragma unroll
            for (int r = 0; r < NR; ++r) {
                const VT lsum = lr[r] + ls;
                in[t][r] = acc[t][r] * (lsum > cut ? gm_inverse(lsum) : VT(0));
            }
        }
#pragma unroll
        for (int t = 0; t < T; ++t) acc[t] = Acc{0, 0, 0, 0};
#pragma unroll
        for (int r = 0; r < NR; ++r)                // r backward, straight from the registers
#pragma unroll
            for (int t = 0; t < T; ++t) acc[t] = A::mma(aR[r], in[t][r], acc[t]);
    }
    put(false);                                     // lines (m_s, m_t), rows a
    get(false);
    contract(1, false);                             // s backward: lines (a, m_t)
    put(true);
    get(true);
    // storage positions, on their way during the last contraction
    int32_t at[T][NR];
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            const int col = 16 * t + j, row = A::QMUL * q + A::RMUL * r;
            at[t][r] = P.at[(row < NE ? row : 0) * C + (col < C ? col : 0)];
        }
    contract(2, false);                             // t backward: lines (a, b), rows c
    VT *o = P.o + (size_t)e * BoxStore<NE>::SIZE;
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            const int col = 16 * t + j, row = A::QMUL * q + A::RMUL * r;
            if (col < C && row < NE && at[t][r] >= 0) o[at[t][r]] = acc[t][r];
        }
}

template <typename VT>
struct CoarseParams {
    const VT *r;              // fine residual
    double *b0;               // coarse right-hand side
    const int32_t *cmap;      // [E][8] coarse solver index or -1
    const uint8_t *owner;     // [E][n_b] 1 on the first copy of each boundary node
    const int32_t *bmap;      // [E][n_b] element-boundary map
    const double *xi;         // GLL nodes [N+1]
    int64_t E, n_bnd;
    int nb;
};

// Restriction on its own (the coarse part without the local solves): one
// 64-lane workgroup per element, N1 known at compile time so that each lane's
// points are unrolled and their loads are in flight together.  Every unique
// node is handled by exactly one local copy: element-interior points and, on
// element boundaries, the copy that comes first in the node's copy list
// (owner flag, built on the host).  b0[corner c of e] += sum over owned points of phi_c(x) r[g].
template <int N1, typename VT>
__global__ void __launch_bounds__(64) k_restrict_e(CoarseParams<VT> P) {
    constexpr int N = N1 - 1, NP = N1 * N1 * N1, Q = (NP + 63) / 64;
    const int64_t e = blockIdx.x;
    double acc[8] = {};
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const int l = threadIdx.x + 64 * q;
        if (l < NP) {
            const int i = l % N1, j = (l / N1) % N1, k = l / (N1 * N1);
            const bool bnd = i == 0 || i == N || j == 0 || j == N || k == 0 || k == N;
            int64_t g;
            bool take;
            if (bnd) {
                const int b = gm_bpos(i, j, k, N1);
                const int32_t m = P.bmap[e * P.nb + b];
                take = m >= 0 && P.owner[e * P.nb + b];
                g = m & 0x7fffffff;
            } else {
                g = gm_interior(P.n_bnd, e, i, j, k, N);
                take = true;
            }
            if (take) {
                const double rv = (double)P.r[g];
                const double wi[2] = {0.5 * (1.0 - P.xi[i]), 0.5 * (1.0 + P.xi[i])};
                const double wj[2] = {0.5 * (1.0 - P.xi[j]), 0.5 * (1.0 + P.xi[j])};
                const double wk[2] = {0.5 * (1.0 - P.xi[k]), 0.5 * (1.0 + P.xi[k])};
#pragma unroll
                for (int c = 0; c < 8; ++c) acc[c] += wi[c & 1] * wj[(c >> 1) & 1] * wk[(c >> 2) & 1] * rv;
            }
        }
    }
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        double sum = acc[c];
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off, 64);
        acc[c] = sum;
    }
    if (threadIdx.x == 0)
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            const int32_t gc = P.cmap[e * 8 + c];
            if (gc >= 0) atomicAdd(P.b0 + gc, acc[c]);
        }
}

// Sum of the overlapping local solutions and the coarse correction:
//   z[g] = (sum of the box values that map to g) / (their number) + (P x0)[g],
// 0 on Dirichlet nodes, in a fixed order.  The local solves leave each box
// whole (o); adding them with atomics instead cost 0.7 ms at 48^3 (99 million,
// resolved beyond the L2s), a cleared vector and 0.27 ms of combination.
// 0.41 ms there for 1.6 GB (counted): the scattered list loads set the pace
// (every extension value loaded at its interior point, six mostly idle loads
// per point: 0.54 ms).
// One element per wave; it sums
//   * its interior nodes: the element's own value and, on the layer next to a
//     face with a neighbour, the value of the neighbour's extension plane, at a
//     position that is linear in the face coordinates (NbrFace): no index list;
//   * the boundary nodes that appear in it first (a contiguous range of the
//     solver order): a list of storage positions built at bind time (k_sum_count,
//     k_sum_fill, k_sum_sort), the element's own copy in front, which also
//     places the node for P.
// Positions have 32 bits: the smallest mesh with more (48.8 million elements at
// N = 2) needs 315 GB of workspaces, beyond the card's memory.
struct NbrFace {
    int32_t e;                // neighbour across the face or -1
    int32_t base, sp, sq;     // its storage position of face point (p, q): base + p sp + q sq
};

template <typename VT>
struct SumParams {
    const VT *o;              // [E][BoxStore::SIZE] local solutions, or null (no local part)
    VT *z;
    VT *clear;                // cleared on the boundary nodes (the vector that the
                              // operator adds to next), or null
    const double *x0;         // coarse solution, or null (no coarse part)
    const int32_t *cmap;      // [E][8] coarse index of each element corner or -1
    const double *xi;         // GLL nodes [N+1]
    const NbrFace *nbr;       // [E][6]
    const uint32_t *off, *pos;  // lists of the boundary nodes
    const int32_t *bpos2l;    // local index of an element's boundary point
    const int32_t *first;     // [E + 1] first boundary node that an element owns
    int64_t E, n_bnd;
};

template <int NE, typename VT>
__global__ void __launch_bounds__(kGmBlock) k_fdm_sum(SumParams<VT> P) {
    using St = BoxStore<NE>;
    constexpr int N = St::N, N1 = St::N1, NM = N - 1, NI = St::NI, NF = NM * NM;
    constexpr int QI = (NI + 63) / 64, QF = (NF + 63) / 64, W = kGmBlock / 64;
    constexpr int64_t B = St::SIZE;
    __shared__ double phi[2][N1];                     // shape functions at the nodes
    __shared__ uint16_t b2l[St::NB];
    __shared__ double zs[W][NI];                      // interior sums of the wave's element
    for (int x = threadIdx.x; x < St::NB; x += kGmBlock) b2l[x] = (uint16_t)P.bpos2l[x];
    if (threadIdx.x < N1) {
        const double x = P.xi[threadIdx.x];
        phi[0][threadIdx.x] = 0.5 * (1.0 - x);
        phi[1][threadIdx.x] = 0.5 * (1.0 + x);
    }
    __syncthreads();
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int64_t e = (int64_t)blockIdx.x * W + wv;
    if (e >= P.E) return;
    const int32_t g0 = P.first[e], g1 = P.first[e + 1];
    int32_t nbe[6];
#pragma unroll
    for (int f = 0; f < 6; ++f) nbe[f] = P.nbr[e * 6 + f].e;
    // interior points: the element's own values, then every face's layer of
    // the neighbour's extension plane, one lane per face point
    double *zb = zs[wv];
    if (P.o) {
        VT own[QI], ext[6][QF];
#pragma unroll
        for (int u = 0; u < QI; ++u) own[u] = P.o[e * B + min(lane + 64 * u, NI - 1)];
#pragma unroll
        for (int f = 0; f < 6; ++f) {
            const NbrFace nf = P.nbr[e * 6 + f];
#pragma unroll
            for (int u = 0; u < QF; ++u) {
                const int t = min(lane + 64 * u, NF - 1), p = t % NM + 1, q = t / NM + 1;
                ext[f][u] = P.o[nf.e >= 0 ? (int64_t)nf.e * B + nf.base + p * nf.sp + q * nf.sq : e * B];
            }
        }
#pragma unroll
        for (int u = 0; u < QI; ++u)
            if (lane + 64 * u < NI) zb[lane + 64 * u] = (double)own[u];
        wave_lds_sync();
#pragma unroll
        for (int f = 0; f < 6; ++f) {
            if (nbe[f] < 0) continue;
            constexpr int s[3] = {1, NM, NM * NM};
            const int d = f / 2, sp = s[d == 0 ? 1 : 0], sq = s[d == 2 ? 1 : 2];
#pragma unroll
            for (int u = 0; u < QF; ++u) {
                const int t = lane + 64 * u;
                if (t < NF) zb[(f % 2 ? (NM - 1) * s[d] : 0) + t % NM * sp + t / NM * sq] += (double)ext[f][u];
            }
            wave_lds_sync();
        }
    }
    double xc[8];
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        const int32_t gc = P.cmap[e * 8 + c];
        xc[c] = (P.x0 && gc >= 0) ? P.x0[gc] : 0.0;
    }
    auto coarse = [&](int i, int j, int k) {
        double r[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) r[c] = phi[0][i] * xc[2 * c] + phi[1][i] * xc[2 * c + 1];
        return phi[0][k] * (phi[0][j] * r[0] + phi[1][j] * r[1]) +
               phi[1][k] * (phi[0][j] * r[2] + phi[1][j] * r[3]);
    };
    // boundary nodes: two per lane and pass, the first four positions of their
    // lists requested together (a pass waits for off, pos and the values in turn)
    constexpr int U = 2, V = 4;
    for (int32_t ga = g0 + lane; ga < g1; ga += 64 * U) {
        uint32_t lo[U], hi[U], own[U];
        uint32_t at[U][V];
        double sum[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int32_t g = ga + 64 * u < g1 ? ga + 64 * u : ga;
            lo[u] = P.off[g];
            hi[u] = P.off[g + 1];
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int t = 0; t < V; ++t)
                at[u][t] = lo[u] < hi[u] ? P.pos[lo[u] + t < hi[u] ? lo[u] + t : lo[u]] : 0u;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            own[u] = at[u][0];
            sum[u] = 0.0;
            if (P.o) {
                VT v[V];
#pragma unroll
                for (int t = 0; t < V; ++t) v[t] = P.o[at[u][t]];
#pragma unroll
                for (int t = 0; t < V; ++t)
                    if (lo[u] + t < hi[u]) sum[u] += (double)v[t];
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (ga + 64 * u >= g1) break;
            double z = 0.0;
            if (lo[u] < hi[u]) {                      // else a Dirichlet node: 0
                if (P.o) {
                    for (uint32_t t = lo[u] + V; t < hi[u]; ++t) sum[u] += (double)P.o[P.pos[t]];
                    z = sum[u] * (1.0 / (double)(hi[u] - lo[u]));
                }
                if (P.x0) {
                    const int l = b2l[(int)(own[u] - (uint32_t)(e * B)) - NI];
                    z += coarse(l % N1, l / N1 % N1, l / St::F2);
                }
            }
            P.z[ga + 64 * u] = (VT)z;
            if (P.clear) P.clear[ga + 64 * u] = VT(0);
        }
    }
#pragma unroll
    for (int u = 0; u < QI; ++u) {
        const int l = lane + 64 * u;
        if (l >= NI) break;
        const int x[3] = {l % NM + 1, (l / NM) % NM + 1, l / (NM * NM) + 1};
        double z = 0.0;
        if (P.o) {
            int cnt = 1;
#pragma unroll
            for (int f = 0; f < 6; ++f) cnt += x[f / 2] == (f % 2 ? N - 1 : 1) && nbe[f] >= 0;
            z = zb[l] * (1.0 / cnt);
        }
        if (P.x0) z += coarse(x[0], x[1], x[2]);
        P.z[P.n_bnd + e * NI + l] = (VT)z;
    }
}

// Lists of the storage positions of every boundary node: counts, then
// positions (in any order), then each list in ascending order with its first
// element point in front.  `cur` starts at zero for both.
__global__ void __launch_bounds__(kGmBlock) k_sum_count(int64_t npoints, int64_t n_bnd,
                                                        const int32_t *__restrict__ fmap,
                                                        uint32_t *__restrict__ cur) {
    for (int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; x < npoints;
         x += (int64_t)gridDim.x * blockDim.x) {
        const int32_t g = fmap[x];
        if (g >= 0 && g < n_bnd) atomicAdd(cur + g, 1u);
    }
}

template <int NE>
__global__ void __launch_bounds__(kGmBlock) k_sum_fill(int64_t npoints, int64_t n_bnd,
                                                       const int32_t *__restrict__ fmap,
                                                       const int32_t *__restrict__ at,
                                                       const uint32_t *__restrict__ off,
                                                       uint32_t *__restrict__ cur,
                                                       uint32_t *__restrict__ pos) {
    constexpr int B = NE * NE * NE;
    for (int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; x < npoints;
         x += (int64_t)gridDim.x * blockDim.x) {
        const int32_t g = fmap[x];
        if (g >= 0 && g < n_bnd)
            pos[off[g] + atomicAdd(cur + g, 1u)] = (uint32_t)(x / B) * BoxStore<NE>::SIZE + at[x % B];
    }
}

template <int NE>
__global__ void __launch_bounds__(kGmBlock) k_sum_sort(int64_t n_bnd, const uint32_t *__restrict__ off,
                                                       uint32_t *__restrict__ pos) {
    const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= n_bnd) return;
    const uint32_t lo = off[g], hi = off[g + 1];
    for (uint32_t t = lo + 1; t < hi; ++t) {
        const uint32_t x = pos[t];
        uint32_t u = t;
        for (; u > lo && pos[u - 1] > x; --u) pos[u] = pos[u - 1];
        pos[u] = x;
    }
    for (uint32_t t = lo; t < hi; ++t) {
        const uint32_t x = pos[t];
        if ((int)(x % (uint32_t)BoxStore<NE>::SIZE) < BoxStore<NE>::NI + BoxStore<NE>::NB) {
            for (uint32_t u = t; u > lo; --u) pos[u] = pos[u - 1];
            pos[lo] = x;
            break;
        }
    }
}

// out[i] = sum over blocks of part[i][b] for i = blockIdx.x: one workgroup per
// value (a single workgroup that took the values in turn needed 20 us for 40
// values of 700 blocks, this form 4 us).
__global__ void __launch_bounds__(kGmBlock) k_gm_finish(int nblocks,
                                                        const double *__restrict__ part,
                                                        double *__restrict__ out,
                                                        double *__restrict__ host) {
    __shared__ double red[kGmBlock / 64];
    const double *p = part + (size_t)blockIdx.x * nblocks;
    double s = 0.0;
    for (int b = threadIdx.x; b < nblocks; b += kGmBlock) s += p[b];
    s = wave_sum63(s);
    if ((threadIdx.x & 63) == 63) red[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        s = red[0];
#pragma unroll
        for (int w = 1; w < kGmBlock / 64; ++w) s += red[w];
        out[blockIdx.x] = s;
        if (host) host[blockIdx.x] = s;       // pinned: read after an event, no copy
    }
}

// part[blk] = v . v over the block's share (any alignment of v)
template <typename T>
__global__ void __launch_bounds__(kGmBlock) k_gm_norm2(int64_t n, const T *__restrict__ v,
                                                       double *__restrict__ part) {
    __shared__ double red[kGmBlock / 64];
    double acc = 0.0;
    for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < n;
         q += (int64_t)gridDim.x * blockDim.x) {
        const double x = (double)v[q];
        acc += x * x;
    }
    acc = gm_block_sum(acc, red);
    if (threadIdx.x == 0) part[blockIdx.x] = acc;
}

// The Gram-Schmidt kernels below are instantiated for the exact number L of
// basis vectors, so that the loads of all L vectors at a point are issued
// together; each lane takes two consecutive points per step (one 16-byte
// load per FP64 vector).  The bases and w are workspace arrays, aligned to
// 256 bytes with a leading dimension ld that is a multiple of 32 values.
template <typename T> struct PairOf;
template <> struct PairOf<double> { using type = double2; };
template <> struct PairOf<float> { using type = float2; };

// Block sums of acc[0..M) into part[i][blk]: every wave sums its lanes, one
// barrier, then one lane per value adds the waves' sums.
template <int M>
__device__ __forceinline__ void gm_store_sums(const double *acc, double *part) {
    constexpr int NW = kGmBlock / 64;
    __shared__ double red[NW][M];
    const int wv = threadIdx.x >> 6;
#pragma unroll
    for (int i = 0; i < M; ++i) {
        const double sum = wave_sum63(acc[i]);
        if ((threadIdx.x & 63) == 63) red[wv][i] = sum;
    }
    __syncthreads();
    if (threadIdx.x < M) {
        double s = red[0][threadIdx.x];
#pragma unroll
        for (int w = 1; w < NW; ++w) s += red[w][threadIdx.x];
        part[(size_t)threadIdx.x * gridDim.x + blockIdx.x] = s;
    }
}

// The basis sweeps stream every vector once per pass (the basis exceeds
// the caches at the sizes that matter): non-temporal loads and stores.
template <typename T>
struct NtPair {
    typedef T type __attribute__((ext_vector_type(2)));
};
template <typename T>
__device__ __forceinline__ typename NtPair<T>::type gm_ld(const T *base, int64_t p) {
    return __builtin_nontemporal_load(reinterpret_cast<const typename NtPair<T>::type *>(base) + p);
}
template <typename T>
__device__ __forceinline__ void gm_st(typename NtPair<T>::type v, T *base, int64_t p) {
    __builtin_nontemporal_store(v, reinterpret_cast<typename NtPair<T>::type *>(base) + p);
}

// part[i][blk] = X_i . v (i < L), part[L][blk] = v . v
template <int L, typename T>
__global__ void __launch_bounds__(kGmBlock) k_gm_dots(int64_t n, int64_t ld,
                                                      const T *__restrict__ X,
                                                      const T *__restrict__ v,
                                                      double *__restrict__ part) {
    double acc[L + 1];
#pragma unroll
    for (int i = 0; i <= L; ++i) acc[i] = 0.0;
    const int64_t np = n >> 1, stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < np; p += stride) {
        const auto vp = gm_ld(v, p);
        const double v0 = (double)vp.x, v1 = (double)vp.y;
#pragma unroll
        for (int i = 0; i < L; ++i) {
            const auto xp = gm_ld(X + i * ld, p);
            acc[i] += (double)xp.x * v0 + (double)xp.y * v1;
        }
        acc[L] += v0 * v0 + v1 * v1;
    }
    if ((n & 1) && blockIdx.x == 0 && threadIdx.x == 0) {   // odd length: last point
        const double vq = (double)v[n - 1];
#pragma unroll
        for (int i = 0; i < L; ++i) acc[i] += (double)X[i * ld + n - 1] * vq;
        acc[L] += vq * vq;
    }
    gm_store_sums<L + 1>(acc, part);
}

// x += sum_{i<L} y_i Z_i at the end of a cycle (y = coef[0..L)), summed in
// the order of i; exact L so that all loads of a point are in flight
// together, basis pairs streamed non-temporally (x may be only 8-byte
// aligned: scalar accesses).
template <int L, typename T>
__global__ void __launch_bounds__(kGmBlock) k_gm_xupd(int64_t n, int64_t ld,
                                                      const T *__restrict__ Z,
                                                      const double *__restrict__ y,
                                                      T *__restrict__ x) {
    double c[L];
#pragma unroll
    for (int i = 0; i < L; ++i) c[i] = y[i];
    const int64_t np = n >> 1, stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < np; p += stride) {
        double s0 = (double)x[2 * p], s1 = (double)x[2 * p + 1];
#pragma unroll
        for (int i = 0; i < L; ++i) {
            const auto zp = gm_ld(Z + i * ld, p);
            s0 += c[i] * (double)zp.x;
            s1 += c[i] * (double)zp.y;
        }
        x[2 * p] = (T)s0;
        x[2 * p + 1] = (T)s1;
    }
    if ((n & 1) && blockIdx.x == 0 && threadIdx.x == 0) {   // odd length: last point
        double s = (double)x[n - 1];
#pragma unroll
        for (int i = 0; i < L; ++i) s += c[i] * (double)Z[i * ld + n - 1];
        x[n - 1] = (T)s;
    }
}

// Arnoldi with delayed reorthogonalisation (classical Gram-Schmidt twice,
// the second projection of each new vector done during the next step).
// At step j the basis V_0..V_{L-1} (L = j) is final and slot j holds the
// once-projected, roughly normalised vector vt; w = A z with z the search
// direction computed from vt.  One sweep forms all inner products
//   part[.][blk] = [ X_i . vt (i < L), X_i . w (i < L), vt.vt, vt.w, w.w ].
template <int L, typename T>
__global__ void __launch_bounds__(kGmBlock) k_gm_dots2(int64_t n, int64_t ld,
                                                       const T *__restrict__ X,
                                                       const T *__restrict__ vt,
                                                       const T *__restrict__ w,
                                                       double *__restrict__ part) {
    constexpr int M = 2 * L + 3;
    double acc[M];
#pragma unroll
    for (int i = 0; i < M; ++i) acc[i] = 0.0;
    const int64_t np = n >> 1, stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < np; p += stride) {
        const auto vp = gm_ld(vt, p);
        const auto wp = gm_ld(w, p);
        const double v0 = (double)vp.x, v1 = (double)vp.y, w0 = (double)wp.x, w1 = (double)wp.y;
#pragma unroll
        for (int i = 0; i < L; ++i) {
            const auto xp = gm_ld(X + i * ld, p);
            const double x0 = (double)xp.x, x1 = (double)xp.y;
            acc[i] += x0 * v0 + x1 * v1;
            acc[L + i] += x0 * w0 + x1 * w1;
        }
        acc[2 * L] += v0 * v0 + v1 * v1;
        acc[2 * L + 1] += v0 * w0 + v1 * w1;
        acc[2 * L + 2] += w0 * w0 + w1 * w1;
    }
    if ((n & 1) && blockIdx.x == 0 && threadIdx.x == 0) {   // odd length: last point
        const double v0 = (double)vt[n - 1], w0 = (double)w[n - 1];
#pragma unroll
        for (int i = 0; i < L; ++i) {
            const double x0 = (double)X[i * ld + n - 1];
            acc[i] += x0 * v0;
            acc[L + i] += x0 * w0;
        }
        acc[2 * L] += v0 * v0;
        acc[2 * L + 1] += v0 * w0;
        acc[2 * L + 2] += w0 * w0;
    }
    gm_store_sums<M>(acc, part);
}

// Scalars of the delayed step from the sums d = [q (L), p (L), r, s, t]
// (q = X^T vt, p = X^T w, r = vt.vt, s = vt.w, t = w.w):
//   beta = |vt - X q| = sqrt(r - |q|^2)   (X orthonormal)
//   h    = (s - q.p) / beta               (w against the final vector)
//   c    = 1 / |w - X p - h v|, |.|^2 = t - |p|^2 - h^2, or 1/|w| where that
//          difference is not safely positive (any positive scale is exact
//          here: the next step measures the stored vector).
__device__ __forceinline__ void gm_delayed_scalars(const double *q, const double *pv, int L,
                                                   double r, double s, double t, double &beta,
                                                   double &h, double &c) {
    double qq = 0.0, qp = 0.0, pp = 0.0;
    for (int i = 0; i < L; ++i) {
        qq += q[i] * q[i];
        qp += q[i] * pv[i];
        pp += pv[i] * pv[i];
    }
    const double b2 = r - qq;
    beta = b2 > 0.0 ? sqrt(b2) : 0.0;
    h = beta > 0.0 ? (s - qp) / beta : 0.0;
    const double est = t - pp - h * h;
    c = est > 1e-4 * t ? 1.0 / sqrt(est) : (t > 0.0 ? 1.0 / sqrt(t) : 0.0);
}

// The sweep that closes step j: the final basis vector and the next
// once-projected one,
//   v   = (vt - X q) / beta           (stored over vt),
//   out = (w - X p - h v) * c          (the next slot),
// with q, p, r, s, t from d and beta, h, c as above (block 0 stores d and
// them for the host).
template <int L, typename T>
__global__ void __launch_bounds__(kGmBlock) k_gm_update2(int64_t n, int64_t ld,
                                                         const T *__restrict__ X,
                                                         const double *__restrict__ d,
                                                         T *__restrict__ vt,
                                                         const T *__restrict__ w,
                                                         T *__restrict__ out,
                                                         double *__restrict__ host) {
    double q[L], pv[L];
#pragma unroll
    for (int i = 0; i < L; ++i) {
        q[i] = d[i];
        pv[i] = d[L + i];
    }
    double beta, h, c;
    gm_delayed_scalars(q, pv, L, d[2 * L], d[2 * L + 1], d[2 * L + 2], beta, h, c);
    const double ib = beta > 0.0 ? 1.0 / beta : 0.0;
    if (blockIdx.x == 0) {                    // pinned host memory
        if (threadIdx.x < 2 * L + 3) host[kGmD + threadIdx.x] = d[threadIdx.x];
        if (threadIdx.x == 0) {
            host[kGmScal] = beta;
            host[kGmScal + 1] = h;
            host[kGmScal + 2] = c;
        }
    }
    const int64_t np = n >> 1, stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < np; p += stride) {
        const auto vp = gm_ld(vt, p);
        const auto wp = gm_ld(w, p);
        double a0 = (double)vp.x, a1 = (double)vp.y, b0 = (double)wp.x, b1 = (double)wp.y;
#pragma unroll
        for (int i = 0; i < L; ++i) {
            const auto xp = gm_ld(X + i * ld, p);
            const double x0 = (double)xp.x, x1 = (double)xp.y;
            a0 -= q[i] * x0;
            a1 -= q[i] * x1;
            b0 -= pv[i] * x0;
            b1 -= pv[i] * x1;
        }
        typename NtPair<T>::type v, o;
        v.x = (T)(a0 * ib);
        v.y = (T)(a1 * ib);
        o.x = (T)((b0 - h * (double)v.x) * c);
        o.y = (T)((b1 - h * (double)v.y) * c);
        gm_st<T>(v, vt, p);
        gm_st<T>(o, out, p);
    }
    if ((n & 1) && blockIdx.x == 0 && threadIdx.x == 0) {
        double a = (double)vt[n - 1], b = (double)w[n - 1];
#pragma unroll
        for (int i = 0; i < L; ++i) {
            const double x = (double)X[i * ld + n - 1];
            a -= q[i] * x;
            b -= pv[i] * x;
        }
        const T v = (T)(a * ib);
        vt[n - 1] = v;
        out[n - 1] = (T)((b - h * (double)v) * c);
    }
}

// First Arnoldi step of a cycle, from coef[0] = p = V_0 . w and coef[1] = w.w:
// out = (w - p V_0) * c with c = 1/sqrt(w.w - p^2) (V_0 has norm one).  Where
// that difference is not safely positive, c = 1/|w| instead (0 for w = 0).
// Block 0 stores p, w.w and c for the host.
template <typename T>
__global__ void __launch_bounds__(kGmBlock) k_gm_first(int64_t n, const T *__restrict__ V0,
                                                       const double *__restrict__ coef,
                                                       const T *__restrict__ w, T *__restrict__ out,
                                                       double *__restrict__ host) {
    using P = typename PairOf<T>::type;
    const double pv = coef[0], ww = coef[1], est = ww - pv * pv;
    const double c = est > 1e-4 * ww ? 1.0 / sqrt(est) : (ww > 0.0 ? 1.0 / sqrt(ww) : 0.0);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        host[0] = pv;
        host[1] = ww;
        host[kGmScal + 2] = c;
    }
    const int64_t np = n >> 1, stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < np; p += stride) {
        const P wp = reinterpret_cast<const P *>(w)[p], xp = reinterpret_cast<const P *>(V0)[p];
        P o;
        o.x = (T)(((double)wp.x - pv * (double)xp.x) * c);
        o.y = (T)(((double)wp.y - pv * (double)xp.y) * c);
        reinterpret_cast<P *>(out)[p] = o;
    }
    if ((n & 1) && blockIdx.x == 0 && threadIdx.x == 0)
        out[n - 1] = (T)(((double)w[n - 1] - pv * (double)V0[n - 1]) * c);
}

// r = b - w (b without w) and part[blk] = r . r in one pass (any alignment).
template <typename T>
__global__ void __launch_bounds__(kGmBlock) k_gm_resid(int64_t n, const T *__restrict__ b,
                                                       const T *__restrict__ w, T *__restrict__ r,
                                                       double *__restrict__ part) {
    __shared__ double red[kGmBlock / 64];
    double sum = 0.0;
    for (int64_t q = (int64_t)blockIdx.x * kGmBlock + threadIdx.x; q < n;
         q += (int64_t)gridDim.x * kGmBlock) {
        const T rq = w ? (T)((double)b[q] - (double)w[q]) : b[q];
        r[q] = rq;
        sum += (double)rq * (double)rq;
    }
    sum = gm_block_sum(sum, red);
    if (threadIdx.x == 0) part[blockIdx.x] = sum;
}

// dst = src * sc
template <typename TS, typename TD>
__global__ void k_gm_scale(int64_t n, const TS *__restrict__ src, TD *__restrict__ dst, double sc) {
    for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < n;
         q += (int64_t)gridDim.x * blockDim.x)
        dst[q] = (TD)((double)src[q] * sc);
}

// Cyclic Jacobi eigenvalue method for a symmetric n x n matrix A (row
// major, destroyed): eigenvalues in lam, eigenvectors in the columns of V.
void jacobi_eigen(int n, std::vector<double> &A, std::vector<double> &V, std::vector<double> &lam) {
    V.assign((size_t)n * n, 0.0);
    for (int i = 0; i < n; ++i) V[(size_t)i * n + i] = 1.0;
    for (int sweep = 0; sweep < 100; ++sweep) {
        double off = 0.0, tot = 0.0;
        for (int i = 0; i < n; ++i)
            for (int j = 0; j < n; ++j) {
                const double a2 = A[(size_t)i * n + j] * A[(size_t)i * n + j];
                tot += a2;
                if (i != j) off += a2;
            }
        if (off <= 1e-30 * tot) break;
        for (int p = 0; p < n; ++p)
            for (int q = p + 1; q < n; ++q) {
                const double apq = A[(size_t)p * n + q];
                if (apq == 0.0) continue;
                const double app = A[(size_t)p * n + p], aqq = A[(size_t)q * n + q];
                const double theta = (aqq - app) / (2.0 * apq);
                const double t = (theta >= 0 ? 1.0 : -1.0) / (std::fabs(theta) + std::sqrt(theta * theta + 1.0));
                const double cs = 1.0 / std::sqrt(t * t + 1.0), sn = t * cs;
                for (int k = 0; k < n; ++k) {           // rotate columns p, q
                    const double akp = A[(size_t)k * n + p], akq = A[(size_t)k * n + q];
                    A[(size_t)k * n + p] = cs * akp - sn * akq;
                    A[(size_t)k * n + q] = sn * akp + cs * akq;
                }
                for (int k = 0; k < n; ++k) {           // rotate rows p, q
                    const double apk = A[(size_t)p * n + k], aqk = A[(size_t)q * n + k];
                    A[(size_t)p * n + k] = cs * apk - sn * aqk;
                    A[(size_t)q * n + k] = sn * apk + cs * aqk;
                }
                for (int k = 0; k < n; ++k) {
                    const double vkp = V[(size_t)k * n + p], vkq = V[(size_t)k * n + q];
                    V[(size_t)k * n + p] = cs * vkp - sn * vkq;
                    V[(size_t)k * n + q] = sn * vkp + cs * vkq;
                }
            }
    }
    // ascending eigenvalues, vectors reordered with them
    std::vector<int> ord(n);
    for (int i = 0; i < n; ++i) ord[i] = i;
    std::sort(ord.begin(), ord.end(),
              [&](int p, int q) { return A[(size_t)p * n + p] < A[(size_t)q * n + q]; });
    std::vector<double> Vs((size_t)n * n);
    lam.resize(n);
    for (int c = 0; c < n; ++c) {
        lam[c] = A[(size_t)ord[c] * n + ord[c]];
        for (int r = 0; r < n; ++r) Vs[(size_t)r * n + c] = V[(size_t)r * n + ord[c]];
    }
    V.swap(Vs);
}

}  // namespace

struct sem_gmres_s {
    sem_ctx ctx = nullptr;           // fine problem (Poisson, FP64)
    sem_ctx coarse = nullptr;        // N = 1 problem on the element vertices
    int m = 30;                      // restart length
    int NE = 0;                      // N + 3
    int64_t ld = 0;                  // leading dimension of the bases (values)
    // host-built preconditioner data
    std::vector<double> S, lam;      // [E][3][NE][NE], [E][3][NE]
    std::vector<int32_t> ghost;      // [E][6][(N+1)^2]
    std::vector<int32_t> cmap;       // [E][8]
    std::vector<NbrFace> nbr;        // [E][6]
    int64_t nfaces = 0;              // faces with a neighbour
    std::vector<uint8_t> owner;      // [E][n_b] first copy of each boundary node
    // device
    char *ws = nullptr;
    size_t ws_bytes = 0;
    size_t coarse_ws = 0;
    CoarsePlan cplan;                // assembled coarse operator and its solve
    double *dS = nullptr, *dlam = nullptr, *dxi = nullptr;
    float *dS32 = nullptr, *dlam32 = nullptr;   // FP32 copies (reduced precisions only)
    int32_t *dghost = nullptr, *dcmap = nullptr;
    uint8_t *downer = nullptr;
    int32_t *dfmap = nullptr;
    uint16_t *down = nullptr;
    NbrFace *dnbr = nullptr;
    uint32_t *doff = nullptr, *dpos = nullptr;   // storage positions of the boundary nodes
    int32_t *dat = nullptr;          // storage positions of a box
    int32_t *dfirst = nullptr;       // [E + 1] first boundary node that an element owns
    std::vector<int32_t> first;
    double *o = nullptr;             // local solutions (FP32 ones use the first half)
    double *b0 = nullptr, *x0 = nullptr;
    bool b0_clear = false;           // b0 is zero when queued work has run
    double *V = nullptr, *Z = nullptr, *w = nullptr, *r = nullptr;
    double *part = nullptr, *coef = nullptr;
    float *rhs32 = nullptr, *d32 = nullptr;
    // pinned: the values of coef that the host reads, as in coef, and behind
    // them the coefficients of a cycle's end on their way to the device
    double *host = nullptr;
    hipEvent_t event = nullptr;
    std::string err;
};

static sem_status gfail(sem_gmres g, sem_status st, const std::string &m) {
    if (g) g->err = m;
    return fail(nullptr, st, m);
}

// Face f = 2d + side of element e in local coordinates: its corner with face
// coordinates (p, q) in {0, 1}^2 (face coordinates: the two other local
// directions in increasing order).
static int face_corner(int f, int p, int q) {
    const int d = f / 2, side = f % 2;
    int ijk[3];
    ijk[d] = side;
    ijk[d == 0 ? 1 : 0] = p;
    ijk[d == 2 ? 1 : 2] = q;
    return ijk[0] + 2 * ijk[1] + 4 * ijk[2];
}

// Host set-up of the local solves: face neighbours and their orientation
// from the corner (vertex) ids, the extension maps, element lengths, 1D
// operators and their generalised eigendecompositions.
static sem_status build_local(sem_gmres G) {
    sem_ctx c = G->ctx;
    const int N = c->N, n1 = N + 1, NE = N + 3, F2 = n1 * n1;
    const int64_t E = c->E;
    // faces by their sorted vertex ids
    std::map<std::array<int64_t, 4>, std::vector<std::pair<int64_t, int>>> faces;
    for (int64_t e = 0; e < E; ++e)
        for (int f = 0; f < 6; ++f) {
            std::array<int64_t, 4> k;
            for (int t = 0; t < 4; ++t) k[t] = c->corners[e * 8 + face_corner(f, t & 1, t >> 1)];
            std::sort(k.begin(), k.end());
            faces[k].push_back({e, f});
        }
    std::vector<int64_t> nbr(E * 6, -1);
    std::vector<int> nbr_face(E * 6, -1);
    for (auto &kv : faces) {
        if (kv.second.size() == 2) {
            auto a = kv.second[0], b = kv.second[1];
            nbr[a.first * 6 + a.second] = b.first;
            nbr_face[a.first * 6 + a.second] = b.second;
            nbr[b.first * 6 + b.second] = a.first;
            nbr_face[b.first * 6 + b.second] = a.second;
        } else if (kv.second.size() > 2) {
            return gfail(G, SEM_ERR_MESH, "a face is shared by more than two elements");
        }
    }
    // element lengths: mean of the four edges along each local direction
    std::vector<double> L(E * 3, 0.0);
    for (int64_t e = 0; e < E; ++e) {
        const double *X = c->corner_xyz.data() + e * 24;
        auto dist = [&](int c0, int c1) {
            double s = 0;
            for (int d = 0; d < 3; ++d) s += (X[d * 8 + c1] - X[d * 8 + c0]) * (X[d * 8 + c1] - X[d * 8 + c0]);
            return std::sqrt(s);
        };
        for (int p = 0; p < 2; ++p)
            for (int q = 0; q < 2; ++q) {
                L[e * 3 + 0] += 0.25 * dist(0 + 2 * p + 4 * q, 1 + 2 * p + 4 * q);
                L[e * 3 + 1] += 0.25 * dist(p + 0 + 4 * q, p + 2 + 4 * q);
                L[e * 3 + 2] += 0.25 * dist(p + 2 * q + 0, p + 2 * q + 4);
            }
    }
    // extension maps
    G->ghost.assign(E * 6 * F2, -1);
    auto node_of = [&](int64_t e, int i, int j, int k) -> int64_t {
        if (i == 0 || i == N || j == 0 || j == N || k == 0 || k == N) {
            int b;
            {   // boundary position of (i, j, k): plane 0, ring planes, plane N
                const int C = n1 * n1;
                if (k == 0) b = i + n1 * j;
                else if (k == N) b = C + (N - 1) * 4 * N + i + n1 * j;
                else {
                    int rg;
                    if (j == 0) rg = i;
                    else if (j == N) rg = N + 1 + 2 * (N - 1) + i;
                    else rg = N + 1 + 2 * (j - 1) + (i == 0 ? 0 : 1);
                    b = C + (k - 1) * 4 * N + rg;
                }
            }
            const int32_t m = c->bmap[(size_t)e * c->nb + b];
            return m < 0 ? -1 : (int64_t)m;
        }
        const int nm = N - 1;
        return c->n_bnd + e * (int64_t)(nm * nm * nm) + ((k - 1) * nm + (j - 1)) * nm + (i - 1);
    };
    std::vector<double> lens_nb(E * 6, -1.0);
    G->nbr.assign(E * 6, NbrFace{-1, 0, 0, 0});
    for (int64_t e = 0; e < E; ++e)
        for (int f = 0; f < 6; ++f) {
            const int64_t n = nbr[e * 6 + f];
            if (n < 0) continue;
            G->nfaces += 1;
            // corners (0,0), (1,0), (0,1) of e's face in n's local frame
            int loc[3][3];
            const int pq[3][2] = {{0, 0}, {1, 0}, {0, 1}};
            for (int t = 0; t < 3; ++t) {
                const int64_t vid = c->corners[e * 8 + face_corner(f, pq[t][0], pq[t][1])];
                int cn = -1;
                for (int q = 0; q < 8; ++q)
                    if (c->corners[n * 8 + q] == vid) cn = q;
                if (cn < 0) return gfail(G, SEM_ERR_MESH, "inconsistent face neighbour");
                loc[t][0] = (cn & 1) * N;
                loc[t][1] = ((cn >> 1) & 1) * N;
                loc[t][2] = ((cn >> 2) & 1) * N;
            }
            int dP[3], dQ[3], ax = -1;
            for (int d = 0; d < 3; ++d) {
                dP[d] = (loc[1][d] - loc[0][d]) / N;
                dQ[d] = (loc[2][d] - loc[0][d]) / N;
                if (dP[d] == 0 && dQ[d] == 0) ax = d;
            }
            if (ax < 0) return gfail(G, SEM_ERR_MESH, "degenerate face orientation");
            const int inward = loc[0][ax] == 0 ? 1 : -1;
            lens_nb[e * 6 + f] = L[n * 3 + ax];
            // the neighbour's extension plane over this face (BoxStore)
            NbrFace &nf = G->nbr[e * 6 + f];
            nf.e = (int32_t)n;
            nf.base = c->np + (2 * ax + (inward == 1 ? 0 : 1)) * F2;
            const int d1 = ax == 0 ? 1 : 0, d2 = ax == 2 ? 1 : 2;
            nf.base += loc[0][d1] + n1 * loc[0][d2];
            nf.sp = dP[d1] + n1 * dP[d2];
            nf.sq = dQ[d1] + n1 * dQ[d2];
            for (int q = 0; q < n1; ++q)
                for (int p = 0; p < n1; ++p) {
                    int x[3];
                    for (int d = 0; d < 3; ++d) x[d] = loc[0][d] + p * dP[d] + q * dQ[d];
                    x[ax] += inward;
                    const int64_t g = node_of(n, x[0], x[1], x[2]);
                    G->ghost[(e * 6 + f) * F2 + p + n1 * q] = (int32_t)g;
                }
        }
    // 1D operators and eigendecompositions
    std::vector<double> Khat((size_t)n1 * n1, 0.0);
    for (int i = 0; i < n1; ++i)
        for (int j = 0; j < n1; ++j) {
            double s = 0;
            for (int q = 0; q < n1; ++q) s += c->D[q * n1 + i] * c->rho[q] * c->D[q * n1 + j];
            Khat[(size_t)i * n1 + j] = s;
        }
    G->S.assign((size_t)E * 3 * NE * NE, 0.0);
    G->lam.assign((size_t)E * 3 * NE, 0.0);
    host_ranges(E, [&](int64_t e0, int64_t e1) {
        std::vector<double> Kl((size_t)(3 * N + 1) * (3 * N + 1)), Ml(3 * N + 1);
        std::vector<double> A((size_t)NE * NE), Vv, lm;
        std::vector<double> Ke((size_t)NE * NE), Me(NE);
        for (int64_t e = e0; e < e1; ++e)
            for (int d = 0; d < 3; ++d) {
                const double h[3] = {lens_nb[e * 6 + 2 * d], L[e * 3 + d], lens_nb[e * 6 + 2 * d + 1]};
                std::fill(Kl.begin(), Kl.end(), 0.0);
                std::fill(Ml.begin(), Ml.end(), 0.0);
                const int nl = 3 * N + 1;
                for (int el = 0; el < 3; ++el) {
                    if (!(h[el] > 0)) continue;
                    for (int i = 0; i < n1; ++i) {
                        Ml[el * N + i] += 0.5 * h[el] * c->rho[i];
                        for (int j = 0; j < n1; ++j)
                            Kl[(size_t)(el * N + i) * nl + el * N + j] += 2.0 / h[el] * Khat[(size_t)i * n1 + j];
                    }
                }
                bool keep[32];
                for (int a = 0; a < NE; ++a) keep[a] = true;
                if (!(h[0] > 0)) keep[0] = false;
                if (!(h[2] > 0)) keep[NE - 1] = false;
                if (c->face_bc[e * 6 + 2 * d]) keep[0] = keep[1] = false;
                if (c->face_bc[e * 6 + 2 * d + 1]) keep[NE - 2] = keep[NE - 1] = false;
                for (int a = 0; a < NE; ++a) {
                    Me[a] = keep[a] ? Ml[N - 1 + a] : 1.0;
                    for (int b = 0; b < NE; ++b)
                        Ke[(size_t)a * NE + b] = (keep[a] && keep[b]) ? Kl[(size_t)(N - 1 + a) * nl + N - 1 + b]
                                                                      : (a == b ? 1.0 : 0.0);
                }
                // K S = M S Lambda via the symmetric M^-1/2 K M^-1/2
                for (int a = 0; a < NE; ++a)
                    for (int b = 0; b < NE; ++b)
                        A[(size_t)a * NE + b] = Ke[(size_t)a * NE + b] / std::sqrt(Me[a] * Me[b]);
                jacobi_eigen(NE, A, Vv, lm);
                double *S = G->S.data() + ((size_t)e * 3 + d) * NE * NE;
                for (int a = 0; a < NE; ++a)
                    for (int mo = 0; mo < NE; ++mo)
                        S[(size_t)a * NE + mo] = keep[a] ? Vv[(size_t)a * NE + mo] / std::sqrt(Me[a]) : 0.0;
                // modes living on dropped points get no weight: zero eigenvector rows there
                double *lmb = G->lam.data() + ((size_t)e * 3 + d) * NE;
                for (int mo = 0; mo < NE; ++mo) lmb[mo] = lm[mo];
            }
    });
    return SEM_OK;
}

// BoxStore::SIZE at run time.
static int64_t box_size(int n1) { return (n1 * n1 * n1 + 6 * n1 * n1 + 7) / 8 * 8; }

// What host allocations throw does not cross the C interface: `report` makes a
// status of its message.
template <typename F, typename R>
static sem_status no_throw(F call, R report) {
    try {
        return call();
    } catch (const std::exception &e) {
        return report(SEM_ERR_OOM, std::string("host memory: ") + e.what());
    }
}

static sem_status create(sem_ctx c, int restart, sem_gmres G) {
    G->ctx = c;
    G->m = restart;
    G->NE = c->N + 3;
    G->ld = (int64_t)(align256(8 * (size_t)c->n_unique) / 8);
    // the coarse problem: N = 1 on the same connectivity
    sem_mesh m0;
    m0.num_elements = c->E;
    m0.corner_ids = c->corners.data();
    m0.face_bc = c->face_bc.data();
    m0.num_vertices = c->num_vertices;
    m0.vertex_xyz = nullptr;
    sem_options o0{SEM_PREC_BIT(SEM_FP64), 0};
    sem_status st = sem_setup(&m0, 1, &o0, &G->coarse);
    if (st) {
        const std::string msg = std::string("coarse grid: ") + sem_last_error(nullptr);
        return fail(c, st, msg);
    }
    st = sem_workspace_size(G->coarse, &G->coarse_ws);
    if (st) return fail(c, st, "coarse grid workspace");
    coarse_pattern(G->coarse, G->cplan);
    st = build_local(G);
    if (st) return st;
    // the first copy of every element-boundary node owns it
    G->owner.assign((size_t)c->E * c->nb, 0);
    // (boundary nodes are numbered by first appearance, so an element owns a
    // contiguous range of them)
    G->first.assign((size_t)c->E + 1, 0);
    for (int64_t g = 0; g < c->n_bnd; ++g) {
        const int32_t own = c->csr_idx[c->csr_off[g]];
        G->owner[own] = 1;
        G->first[own / c->nb + 1] += 1;
    }
    for (int64_t e = 0; e < c->E; ++e) G->first[e + 1] += G->first[e];
    // coarse index of every element corner (Dirichlet: -1)
    G->cmap.assign(c->E * 8, -1);
    for (int64_t e = 0; e < c->E; ++e)
        for (int q = 0; q < 8; ++q) {
            // at N = 1 every point is a boundary point; position b = local index
            const int32_t v = G->coarse->bmap[(size_t)e * G->coarse->nb + q];
            G->cmap[e * 8 + q] = v < 0 ? -1 : v;
        }
    return SEM_OK;
}

extern "C" sem_status sem_gmres_create(sem_ctx c, int restart, sem_gmres *out) {
    if (!c || !out) return fail(c, SEM_ERR_INVALID, "null argument");
    *out = nullptr;
    if (!c->geometry_ready || c->corner_xyz.empty())
        return fail(c, SEM_ERR_STATE, "geometry not set");
    if (!c->solver || !c->L.r64) return fail(c, SEM_ERR_STATE, "context set up without solver vectors");
    if (c->N < 2 || c->N > 13) return fail(c, SEM_ERR_UNSUPPORTED, "the Schwarz solves need 2 <= N <= 13");
    if (restart < 1 || restart > kGmMaxVec - 1)
        return fail(c, SEM_ERR_INVALID, "restart must be in 1.." + std::to_string(kGmMaxVec - 1));
    if (c->helm) return fail(c, SEM_ERR_UNSUPPORTED, "the pressure solver is for the Poisson operator");
    if (c->E > (int64_t)UINT32_MAX / box_size(c->n1))
        return fail(c, SEM_ERR_UNSUPPORTED, "more local-solve values than 32 bits count");
    struct Free {
        void operator()(sem_gmres g) const { sem_gmres_free(g); }
    };
    auto build = [&]() -> sem_status {
        std::unique_ptr<sem_gmres_s, Free> g(new sem_gmres_s());
        const sem_status st = create(c, restart, g.get());
        if (!st) *out = g.release();
        return st;
    };
    return no_throw(build, [&](sem_status st, const std::string &m) { return fail(c, st, m); });
}

extern "C" void sem_gmres_free(sem_gmres G) {
    if (!G) return;
    sem_free(G->coarse);
    if (G->event) (void)hipEventDestroy(G->event);
    if (G->host) (void)hipHostFree(G->host);
    delete G;
}

extern "C" const char *sem_gmres_last_error(sem_gmres G) { return G ? G->err.c_str() : ""; }

static size_t gm_layout(sem_gmres G, size_t *off) {
    sem_ctx c = G->ctx;
    const int64_t E = c->E, NE = G->NE, n1 = c->n1;
    size_t o = 0;
    auto take = [&](size_t b) {
        const size_t r = o;
        o += align256(b);
        return r;
    };
    off[0] = take(G->coarse_ws);
    // the coarse context's partial sums, which only its own CG would use, give
    // their place to other arrays while it lasts
    size_t spare = G->coarse->L.partials, spare_end = spare + kPartialsBytes;
    auto take_spare = [&](size_t b) {
        if (spare + align256(b) > spare_end) return take(b);
        const size_t r = spare;
        spare += align256(b);
        return off[0] + r;
    };
    off[1] = take(8 * (size_t)E * 3 * NE * NE);       // S
    off[2] = take(8 * (size_t)E * 3 * NE);            // lambda
    off[4] = take(4 * (size_t)E * 8);                 // coarse map
    off[5] = take(sizeof(NbrFace) * (size_t)E * 6);   // neighbour faces
    off[6] = take(8 * 16);                            // xi
    // Local solutions, live from k_fdm to k_fdm_sum of one application only.
    // Two arrays lie in the same place: the ghost map, read while the box maps
    // are built, and r, read between a residual and the first application of
    // the cycle that it starts.
    off[3] = off[13] = off[7] = take(8 * (size_t)E * box_size(n1));
    off[8] = take(8 * (size_t)G->coarse->n_unique);   // b0
    off[9] = take(8 * (size_t)G->coarse->n_unique);   // x0
    off[10] = take(8 * (size_t)G->ld * (G->m + 1));   // V
    off[11] = take(8 * (size_t)G->ld * G->m);         // Z
    off[12] = take(8 * (size_t)c->n_unique);          // w, FP32 vectors in its first half
    off[14] = take_spare(8 * (size_t)kGmGrid * (2 * kGmMaxVec + 3));   // partial sums, at most 2 L + 3 per block
    off[15] = take(8 * kGmCoef);
    // the FP32 inner right-hand side, read before the cycle's first operator
    off[16] = off[12] + 4 * (size_t)c->n_unique;
    off[17] = take(4 * (size_t)c->n_unique);          // FP32 inner correction
    off[18] = take((size_t)E * c->nb);                // owner flags
    off[19] = take(4 * (size_t)E * NE * NE * NE);    // box gather map
    off[20] = take(2 * (size_t)E * NE * NE);         // owned-point masks of the box columns
    // FP32 eigenvector tables for the inner solves of the refinement
    const bool low = (c->precisions & ~SEM_PREC_BIT(SEM_FP64)) != 0;
    off[21] = take(low ? 4 * (size_t)E * 3 * NE * NE : 0);
    off[22] = take(low ? 4 * (size_t)E * 3 * NE : 0);
    off[23] = take_spare(coarse_bytes(G->cplan));
    // position lists of the boundary nodes: at most every element-boundary
    // point and the rim of the extension plane over every face with a neighbour
    off[24] = take(4 * ((size_t)c->n_bnd + 1));
    off[25] = take(4 * ((size_t)E * c->nb + (size_t)G->nfaces * 4 * c->N));
    off[26] = take(4 * (size_t)NE * NE * NE);         // storage positions of a box
    off[27] = take(4 * ((size_t)E + 1));              // first owned boundary node
    return o;
}

extern "C" sem_status sem_gmres_workspace_size(sem_gmres G, size_t *bytes) {
    if (!G || !bytes) return gfail(G, SEM_ERR_INVALID, "null argument");
    size_t off[28];
    *bytes = gm_layout(G, off);
    return SEM_OK;
}

// Position lists of the boundary nodes from the box gather maps (the counts
// are summed on the host; the local solutions' array holds them meanwhile).
template <int NE>
static hipError_t build_positions(sem_gmres G, hipStream_t s) {
    sem_ctx c = G->ctx;
    const int64_t nb = c->n_bnd, np = c->E * NE * NE * NE;
    uint32_t *cur = reinterpret_cast<uint32_t *>(G->o);
    uint32_t *off = G->doff, *pos = G->dpos;
    const dim3 gp(gm_grid(np)), gn((unsigned)((nb + kGmBlock - 1) / kGmBlock)), t(kGmBlock);
    std::vector<uint32_t> cnt(nb), hoff(nb + 1);
    hipError_t e = launch_fill32(reinterpret_cast<float *>(cur), nb, 0.0f, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_sum_count, gp, t, 0, s, np, nb, (const int32_t *)G->dfmap, cur);
    e = hipMemcpyAsync(cnt.data(), cur, 4 * (size_t)nb, hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) return e;
    hoff[0] = 0;
    for (int64_t g = 0; g < nb; ++g) hoff[g + 1] = hoff[g] + cnt[g];
    e = hipMemcpyAsync(off, hoff.data(), 4 * hoff.size(), hipMemcpyHostToDevice, s);
    if (e == hipSuccess) e = launch_fill32(reinterpret_cast<float *>(cur), nb, 0.0f, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_sum_fill<NE>, gp, t, 0, s, np, nb, (const int32_t *)G->dfmap,
                       (const int32_t *)G->dat, (const uint32_t *)off, cur, pos);
    hipLaunchKernelGGL(k_sum_sort<NE>, gn, t, 0, s, nb, (const uint32_t *)off, pos);
    e = hipGetLastError();
    return e == hipSuccess ? hipStreamSynchronize(s) : e;   // hoff is a temporary
}

static sem_status bind_workspace(sem_gmres G, void *dev, size_t bytes, sem_stream stream) {
    size_t off[28];
    const size_t need = gm_layout(G, off);
    if (bytes < need)
        return gfail(G, SEM_ERR_OOM, "workspace of " + std::to_string(bytes) + " bytes, need " +
                                         std::to_string(need));
    if ((uintptr_t)dev & 255) return gfail(G, SEM_ERR_INVALID, "workspace not 256-byte aligned");
    sem_ctx c = G->ctx;
    hipStream_t s = (hipStream_t)stream;
    char *w = static_cast<char *>(dev);
    if (!G->host)
        SEM_HIP(c, hipHostMalloc((void **)&G->host, 8 * (kGmCoef + kGmMaxVec),
                                 hipHostMallocMapped | hipHostMallocCoherent));
    if (!G->event) SEM_HIP(c, hipEventCreateWithFlags(&G->event, hipEventDisableTiming));
    G->ws = w;
    G->ws_bytes = bytes;
    sem_status st = sem_bind_workspace(G->coarse, w + off[0], G->coarse_ws, stream);
    if (st) return gfail(G, st, std::string("coarse grid: ") + sem_last_error(G->coarse));
    // coarse geometry: the element corners ([E][3][8] = [E][3][2][2][2])
    st = sem_set_geometry(G->coarse, c->corner_xyz.data(), stream);
    if (st) return gfail(G, st, std::string("coarse grid: ") + sem_last_error(G->coarse));
    G->dS = reinterpret_cast<double *>(w + off[1]);
    G->dlam = reinterpret_cast<double *>(w + off[2]);
    G->dghost = reinterpret_cast<int32_t *>(w + off[3]);
    G->dcmap = reinterpret_cast<int32_t *>(w + off[4]);
    G->dnbr = reinterpret_cast<NbrFace *>(w + off[5]);
    G->dxi = reinterpret_cast<double *>(w + off[6]);
    G->o = reinterpret_cast<double *>(w + off[7]);
    G->doff = reinterpret_cast<uint32_t *>(w + off[24]);
    G->dpos = reinterpret_cast<uint32_t *>(w + off[25]);
    G->dat = reinterpret_cast<int32_t *>(w + off[26]);
    G->dfirst = reinterpret_cast<int32_t *>(w + off[27]);
    SEM_HIP(c, hipMemcpyAsync(G->dfirst, G->first.data(), 4 * G->first.size(), hipMemcpyHostToDevice, s));
    G->b0 = reinterpret_cast<double *>(w + off[8]);
    G->x0 = reinterpret_cast<double *>(w + off[9]);
    G->V = reinterpret_cast<double *>(w + off[10]);
    G->Z = reinterpret_cast<double *>(w + off[11]);
    G->w = reinterpret_cast<double *>(w + off[12]);
    G->r = reinterpret_cast<double *>(w + off[13]);
    G->part = reinterpret_cast<double *>(w + off[14]);
    G->coef = reinterpret_cast<double *>(w + off[15]);
    G->rhs32 = reinterpret_cast<float *>(w + off[16]);
    G->d32 = reinterpret_cast<float *>(w + off[17]);
    G->downer = reinterpret_cast<uint8_t *>(w + off[18]);
    G->dfmap = reinterpret_cast<int32_t *>(w + off[19]);
    G->down = reinterpret_cast<uint16_t *>(w + off[20]);
    G->b0_clear = false;
    SEM_HIP(c, coarse_bind(G->coarse, G->cplan, w + off[23], G->b0, G->x0, s));
    G->b0_clear = true;
    SEM_HIP(c, hipMemcpyAsync(G->dS, G->S.data(), 8 * G->S.size(), hipMemcpyHostToDevice, s));
    SEM_HIP(c, hipMemcpyAsync(G->dlam, G->lam.data(), 8 * G->lam.size(), hipMemcpyHostToDevice, s));
    G->dS32 = G->dlam32 = nullptr;
    if (off[22] > off[21]) {
        G->dS32 = reinterpret_cast<float *>(w + off[21]);
        G->dlam32 = reinterpret_cast<float *>(w + off[22]);
        // rounded once; the copies are synchronous (the host buffers are
        // temporaries).  The eigenvalues are scaled by a power of two of the
        // element's largest sum, half of which goes with S_r in either direction:
        // sums from element lengths above 1e19 or below 1e-18 leave FP32's
        // normal range, outside which the hardware's reciprocal estimate is 0
        // or infinite
        const size_t C = (size_t)G->NE * G->NE, NE = G->NE;
        std::vector<float> s32(G->S.size()), l32(G->lam.size());
        host_ranges(c->E, [&](int64_t e0, int64_t e1) {
            for (int64_t e = e0; e < e1; ++e) {
                const double *lam = G->lam.data() + (size_t)e * 3 * NE, *S = G->S.data() + (size_t)e * 3 * C;
                const double top = lam[NE - 1] + lam[2 * NE - 1] + lam[3 * NE - 1];
                const int ex = top > 0.0 && top <= DBL_MAX ? std::ilogb(top) / 2 : 0;
                const double fl = std::ldexp(1.0, -2 * ex), fs = std::ldexp(1.0, -ex);
                for (size_t q = 0; q < 3 * NE; ++q) l32[(size_t)e * 3 * NE + q] = (float)(lam[q] * fl);
                for (size_t q = 0; q < 3 * C; ++q)
                    s32[(size_t)e * 3 * C + q] = (float)(q < C ? S[q] * fs : S[q]);
            }
        });
        SEM_HIP(c, hipMemcpyAsync(G->dS32, s32.data(), 4 * s32.size(), hipMemcpyHostToDevice, s));
        SEM_HIP(c, hipMemcpyAsync(G->dlam32, l32.data(), 4 * l32.size(), hipMemcpyHostToDevice, s));
        SEM_HIP(c, hipStreamSynchronize(s));
    }
    SEM_HIP(c, hipMemcpyAsync(G->dghost, G->ghost.data(), 4 * G->ghost.size(), hipMemcpyHostToDevice, s));
    SEM_HIP(c, hipMemcpyAsync(G->dcmap, G->cmap.data(), 4 * G->cmap.size(), hipMemcpyHostToDevice, s));
    SEM_HIP(c, hipMemcpyAsync(G->dnbr, G->nbr.data(), sizeof(NbrFace) * G->nbr.size(),
                              hipMemcpyHostToDevice, s));
    SEM_HIP(c, hipMemcpyAsync(G->downer, G->owner.data(), G->owner.size(), hipMemcpyHostToDevice, s));
    SEM_HIP(c, hipMemcpyAsync(G->dxi, c->xi, 8 * c->n1, hipMemcpyHostToDevice, s));
    // box gather maps from the element and face maps
#define SEM_FMAP(ne)                                                                            \
    case ne:                                                                                    \
        hipLaunchKernelGGL(k_fdm_map<ne>, dim3((unsigned)c->E), dim3(((ne) * (ne) + 63) / 64 * 64), 0, \
                           s, (const int32_t *)G->dghost, dptr<int32_t>(c, c->L.bmap),        \
                           (const uint8_t *)G->downer, c->E, c->n_bnd, c->nb, G->dfmap, G->down, G->dat); \
        break;
    switch (G->NE) {
        SEM_FMAP(5) SEM_FMAP(6) SEM_FMAP(7) SEM_FMAP(8) SEM_FMAP(9) SEM_FMAP(10) SEM_FMAP(11)
        SEM_FMAP(12) SEM_FMAP(13) SEM_FMAP(14) SEM_FMAP(15) SEM_FMAP(16)
        default: return gfail(G, SEM_ERR_UNSUPPORTED, "order");
    }
#undef SEM_FMAP
    SEM_HIP(c, hipGetLastError());
    hipError_t pe = hipErrorInvalidValue;
#define SEM_POS(ne)                                                                              \
    case ne: pe = build_positions<ne>(G, s); break;
    switch (G->NE) {
        SEM_POS(5) SEM_POS(6) SEM_POS(7) SEM_POS(8) SEM_POS(9) SEM_POS(10) SEM_POS(11) SEM_POS(12)
        SEM_POS(13) SEM_POS(14) SEM_POS(15) SEM_POS(16)
        default: break;
    }
#undef SEM_POS
    SEM_HIP(c, pe);
    SEM_HIP(c, hipStreamSynchronize(s));
    return SEM_OK;
}

extern "C" sem_status sem_gmres_bind_workspace(sem_gmres G, void *dev, size_t bytes,
                                               sem_stream stream) {
    if (!G || !dev) return gfail(G, SEM_ERR_INVALID, "null argument");
    return no_throw([&]() { return bind_workspace(G, dev, bytes, stream); },
                    [&](sem_status st, const std::string &m) { return gfail(G, st, m); });
}

// z from the local solutions (o null: without them) and the coarse solution.
template <typename VT>
static sem_status combine(sem_gmres G, const VT *o, bool coarse, VT *z, VT *clear, hipStream_t s) {
    sem_ctx c = G->ctx;
    SumParams<VT> P{o, z, clear, coarse ? G->x0 : nullptr, G->dcmap, G->dxi, G->dnbr,
                       G->doff, G->dpos,
                       dptr<int32_t>(c, c->L.bpos2l), G->dfirst, c->E, c->n_bnd};
    const dim3 g((unsigned)((c->E + kGmBlock / 64 - 1) / (kGmBlock / 64))), t(kGmBlock);
#define SEM_SUM(ne)                                                       \
    case ne:                                                              \
        hipLaunchKernelGGL((k_fdm_sum<ne, VT>), g, t, 0, s, P);        \
        break;
    switch (G->NE) {
        SEM_SUM(5) SEM_SUM(6) SEM_SUM(7) SEM_SUM(8) SEM_SUM(9) SEM_SUM(10) SEM_SUM(11) SEM_SUM(12)
        SEM_SUM(13) SEM_SUM(14) SEM_SUM(15) SEM_SUM(16)
        default: return gfail(G, SEM_ERR_UNSUPPORTED, "order");
    }
#undef SEM_SUM
    SEM_HIP(c, hipGetLastError());
    return SEM_OK;
}

// z = M^-1 r: parts & 1 local Schwarz solves, parts & 2 coarse grid; the
// boundary block of `clear`, if given, is cleared on the way.  r and
// z are FP64 or FP32 vectors; the local solves compute in the vectors'
// precision, the coarse grid in FP64 either way.
template <typename VT>
static sem_status precondition(sem_gmres G, const VT *r, VT *z, unsigned parts, hipStream_t s,
                               VT *clear = nullptr) {
    sem_ctx c = G->ctx;
    const bool local = parts & SEM_PC_SCHWARZ, coarse = parts & SEM_PC_COARSE;
    // with both parts the coarse restriction is summed in the local-solve
    // kernel's gather (the residual is read once)
    const bool fused = local && coarse;
    // the local solutions in the vectors' precision (FP32 ones use the first
    // half of the FP64 array)
    VT *o = reinterpret_cast<VT *>(G->o);
    constexpr bool f32 = std::is_same<VT, float>::value;
    // The coarse solve leaves b0 cleared for the next restriction.  A call that
    // ends with an error in between leaves it filled: cleared here then.
    if (coarse) {
        if (!G->b0_clear) SEM_HIP(c, launch_fill(G->b0, G->coarse->n_unique, 0.0, s));
        G->b0_clear = false;
    }
    if (local) {
        const VT *S, *lam;
        if constexpr (f32) {
            if (!G->dS32) return gfail(G, SEM_ERR_STATE, "no FP32 tables: no reduced precision at set-up");
            S = G->dS32;
            lam = G->dlam32;
        } else {
            S = G->dS;
            lam = G->dlam;
        }
        FdmParams<VT> P{r,       o, G->dat, S, lam, G->dfmap, c->E,
                        G->down, fused ? G->b0 : nullptr, G->dcmap, G->dxi};
#define SEM_FDM(ne)                                                                          \
    case ne:                                                                                 \
        hipLaunchKernelGGL((k_fdm<ne, VT>), dim3((unsigned)c->E), dim3(64), 0, s, P);        \
        break;
        switch (G->NE) {
            SEM_FDM(5) SEM_FDM(6) SEM_FDM(7) SEM_FDM(8) SEM_FDM(9) SEM_FDM(10) SEM_FDM(11)
            SEM_FDM(12) SEM_FDM(13) SEM_FDM(14) SEM_FDM(15) SEM_FDM(16)
            default: return gfail(G, SEM_ERR_UNSUPPORTED, "order");
        }
#undef SEM_FDM
        SEM_HIP(c, hipGetLastError());
    }
    if (coarse) {
        CoarseParams<VT> C{r,       G->b0, G->dcmap, G->downer, dptr<int32_t>(c, c->L.bmap), G->dxi,
                           c->E, c->n_bnd, c->nb};
#define SEM_RESTRICT(n1)                                                                    \
    case n1:                                                                                \
        hipLaunchKernelGGL((k_restrict_e<n1, VT>), dim3((unsigned)c->E), dim3(64), 0, s, C); \
        break;
        if (!fused) switch (c->n1) {
            SEM_RESTRICT(3) SEM_RESTRICT(4) SEM_RESTRICT(5) SEM_RESTRICT(6) SEM_RESTRICT(7)
            SEM_RESTRICT(8) SEM_RESTRICT(9) SEM_RESTRICT(10) SEM_RESTRICT(11) SEM_RESTRICT(12)
            SEM_RESTRICT(13) SEM_RESTRICT(14)
            default: return gfail(G, SEM_ERR_UNSUPPORTED, "order");
        }
#undef SEM_RESTRICT
        SEM_HIP(c, hipGetLastError());
        // 10 Jacobi-PCG iterations from zero on the coarse operator (which
        // leave b0 cleared for the next application)
        SEM_HIP(c, coarse_solve(G->cplan, s));
        G->b0_clear = true;
    }
    return combine<VT>(G, local ? o : nullptr, coarse, z, clear, s);
}

extern "C" sem_status sem_gmres_precondition(sem_gmres G, const double *r, double *z,
                                             unsigned parts, sem_stream stream) {
    if (!G || !r || !z) return gfail(G, SEM_ERR_INVALID, "null argument");
    if (!G->ws) return gfail(G, SEM_ERR_STATE, "no workspace bound");
    if (!(parts & (SEM_PC_SCHWARZ | SEM_PC_COARSE)) || (parts & ~3u))
        return gfail(G, SEM_ERR_INVALID, "parts must name SEM_PC_SCHWARZ and/or SEM_PC_COARSE");
    hipStream_t s = (hipStream_t)stream;
    const sem_status st = precondition<double>(G, r, z, parts, s);
    if (st || !(parts & SEM_PC_COARSE)) return st;
    CgState cs;
    SEM_HIP(G->ctx, hipMemcpyAsync(&cs, coarse_result(G->cplan), sizeof(cs), hipMemcpyDeviceToHost, s));
    SEM_HIP(G->ctx, hipStreamSynchronize(s));
    if (cs.status == CG_NONFINITE)
        return gfail(G, SEM_ERR_NAN, "coarse solve: FP64 PCG met a non-finite value");
    return SEM_OK;
}

// y = A x with the operator of precision prec (FP64 vectors for SEM_FP64,
// FP32 otherwise; atomic summation into a cleared boundary block)
template <typename T>
static sem_status apply_A(sem_gmres G, int prec, const T *x, T *y, hipStream_t s) {
    sem_ctx c = G->ctx;
    if (std::is_same<T, double>::value) SEM_HIP(c, launch_fill((double *)y, c->n_bnd, 0.0, s));
    else SEM_HIP(c, launch_fill32((float *)y, c->n_bnd, 0.0f, s));
    SEM_HIP(c, launch_ax(c, prec, x, y, 0, OUT_ATOMIC, nullptr, nullptr, c->tile[prec], s));
    return SEM_OK;
}

// Grid of a reduction kernel: the workgroups that are resident at once on
// the device (no partial second wave), at most one per kGmBlock entries and
// at most kGmGrid (the size of the partial-sum buffer).
template <typename K>
static unsigned resident_grid(K kern, int &per_cu, int ncu, int64_t n) {
    if (per_cu == 0) {
        int nb = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, kern, kGmBlock, 0) != hipSuccess || nb < 1)
            nb = 1;
        per_cu = nb;
    }
    const int64_t need = (n + kGmBlock - 1) / kGmBlock;
    return (unsigned)std::max<int64_t>(1, std::min<int64_t>({need, (int64_t)per_cu * ncu, (int64_t)kGmGrid}));
}

#define SEM_GM_CASES(M)                                                                      \
    M(1) M(2) M(3) M(4) M(5) M(6) M(7) M(8) M(9) M(10) M(11) M(12) M(13) M(14) M(15) M(16)    \
    M(17) M(18) M(19) M(20) M(21) M(22) M(23) M(24) M(25) M(26) M(27) M(28) M(29) M(30) M(31)

// coef[i] = X_i . v (i < L), coef[L] = v.v; also in host[0..L] if given
template <int L, typename T>
struct GmDots {
    static hipError_t run(sem_gmres G, const T *X, const T *v, double *host, hipStream_t s) {
        static int per_cu = 0;
        const int64_t n = G->ctx->n_unique;
        const unsigned g = resident_grid(k_gm_dots<L, T>, per_cu, G->ctx->num_cus, n / 2);
        hipLaunchKernelGGL((k_gm_dots<L, T>), dim3(g), dim3(kGmBlock), 0, s, n, G->ld, X, v, G->part);
        hipLaunchKernelGGL(k_gm_finish, dim3(L + 1), dim3(kGmBlock), 0, s, (int)g,
                           (const double *)G->part, G->coef, host);
        return hipGetLastError();
    }
};

// x += Z y, y = coef[0..L)
template <int L, typename T>
struct GmXupd {
    static hipError_t run(sem_gmres G, const T *Z, T *x, hipStream_t s) {
        static int per_cu = 0;
        const int64_t n = G->ctx->n_unique;
        const unsigned g = resident_grid(k_gm_xupd<L, T>, per_cu, G->ctx->num_cus, n / 2);
        hipLaunchKernelGGL((k_gm_xupd<L, T>), dim3(g), dim3(kGmBlock), 0, s, n, G->ld, Z,
                           (const double *)G->coef, x);
        return hipGetLastError();
    }
};

// coef[kGmD..] = [X^T vt (L), X^T w (L), vt.vt, vt.w, w.w]
template <int L, typename T>
struct GmDots2 {
    static hipError_t run(sem_gmres G, const T *X, const T *vt, const T *w, hipStream_t s) {
        static int per_cu = 0;
        const int64_t n = G->ctx->n_unique;
        const unsigned g = resident_grid(k_gm_dots2<L, T>, per_cu, G->ctx->num_cus, n / 2);
        hipLaunchKernelGGL((k_gm_dots2<L, T>), dim3(g), dim3(kGmBlock), 0, s, n, G->ld, X, vt, w,
                           G->part);
        hipLaunchKernelGGL(k_gm_finish, dim3(2 * L + 3), dim3(kGmBlock), 0, s, (int)g,
                           (const double *)G->part, G->coef + kGmD, (double *)nullptr);
        return hipGetLastError();
    }
};

// vt <- final basis vector, out <- next once-projected vector (from coef[kGmD..]);
// all of them and beta, h, c to the host
template <int L, typename T>
struct GmUpdate2 {
    static hipError_t run(sem_gmres G, const T *X, T *vt, const T *w, T *out, hipStream_t s) {
        static int per_cu = 0;
        const int64_t n = G->ctx->n_unique;
        const unsigned g = resident_grid(k_gm_update2<L, T>, per_cu, G->ctx->num_cus, n / 2);
        hipLaunchKernelGGL((k_gm_update2<L, T>), dim3(g), dim3(kGmBlock), 0, s, n, G->ld, X,
                           (const double *)(G->coef + kGmD), vt, w, out, G->host);
        return hipGetLastError();
    }
};

// Op<l, T>::run(args...) for the basis size l in 1..kGmMaxVec-1
template <template <int, typename> class Op, typename T, typename... A>
static hipError_t gm_dispatch(int l, A... a) {
    switch (l) {
#define SEM_GM_CASE(L) \
    case L: return Op<L, T>::run(a...);
        SEM_GM_CASES(SEM_GM_CASE)
#undef SEM_GM_CASE
        default: return hipErrorInvalidValue;
    }
}

// What the host reads -- Gram-Schmidt sums, norms -- is written to pinned
// memory by the kernel that forms it: gm_mark after that kernel, gm_wait before
// reading (work queued in between runs on).
static sem_status gm_mark(sem_gmres G, hipStream_t s) {
    SEM_HIP(G->ctx, hipEventRecord(G->event, s));
    return SEM_OK;
}
static sem_status gm_wait(sem_gmres G) {
    SEM_HIP(G->ctx, hipEventSynchronize(G->event));
    return SEM_OK;
}

// *out = v.v (FP64 sum; v of any alignment)
template <typename T>
static sem_status gm_norm2(sem_gmres G, const T *v, double *out, hipStream_t s) {
    static int per_cu = 0;
    const int64_t n = G->ctx->n_unique;
    const unsigned g = resident_grid(k_gm_norm2<T>, per_cu, G->ctx->num_cus, n);
    hipLaunchKernelGGL(k_gm_norm2<T>, dim3(g), dim3(kGmBlock), 0, s, n, v, G->part);
    hipLaunchKernelGGL(k_gm_finish, dim3(1), dim3(kGmBlock), 0, s, (int)g, (const double *)G->part,
                       G->coef, G->host);
    SEM_HIP(G->ctx, hipGetLastError());
    sem_status e = gm_mark(G, s);
    if (!e) e = gm_wait(G);
    *out = G->host[0];
    return e;
}

// First Arnoldi step of a cycle (V_0 final, no vector awaiting its second
// projection): see k_gm_first.
template <typename T>
static hipError_t gm_first_step(sem_gmres G, const T *V0, const T *w, T *out, hipStream_t s) {
    static int per_cu = 0;
    const int64_t n = G->ctx->n_unique;
    hipError_t e = GmDots<1, T>::run(G, V0, w, nullptr, s);
    if (e != hipSuccess) return e;
    const unsigned g = resident_grid(k_gm_first<T>, per_cu, G->ctx->num_cus, n / 2);
    hipLaunchKernelGGL(k_gm_first<T>, dim3(g), dim3(kGmBlock), 0, s, n, V0, (const double *)G->coef, w,
                       out, G->host);
    return hipGetLastError();
}

// r = b - A x in T vectors; returns ||r|| in *rn.
template <typename T>
static sem_status residual(sem_gmres G, int prec, const T *b, const T *x, T *r, T *w, bool x_zero,
                           double *rn, hipStream_t s) {
    static int per_cu = 0;
    sem_ctx c = G->ctx;
    const int64_t n = c->n_unique;
    if (!x_zero) {
        sem_status e = apply_A<T>(G, prec, x, w, s);
        if (e) return e;
    }
    const unsigned g = resident_grid(k_gm_resid<T>, per_cu, c->num_cus, n);
    hipLaunchKernelGGL(k_gm_resid<T>, dim3(g), dim3(kGmBlock), 0, s, n, b,
                       x_zero ? (const T *)nullptr : (const T *)w, r, G->part);
    hipLaunchKernelGGL(k_gm_finish, dim3(1), dim3(kGmBlock), 0, s, (int)g, (const double *)G->part,
                       G->coef, G->host);
    SEM_HIP(c, hipGetLastError());
    sem_status e = gm_mark(G, s);
    if (!e) e = gm_wait(G);
    if (e) return e;
    *rn = std::sqrt(G->host[0]);
    return SEM_OK;
}

// Flexible GMRES(m) cycles on A x = b in T vectors (operator precision
// prec) until ||b - A x|| <= atol (recurrence estimate within a cycle, true
// residual at its end) or max_iter steps in all.  V, Z, w, r live in the
// solver's basis arrays (FP32 vectors use the first half of each slot).  b may
// lie in the second half of w and r among the local solutions: with one_cycle
// neither is read once the first application has started.
// Returns SEM_OK when converged, SEM_ERR_NOT_CONVERGED at the cap; *res_out
// is the last true residual norm.  one_cycle (inner solves of the
// refinement): a single cycle from x = 0 that stops on the recurrence
// estimate alone -- a residual recomputed in FP32 carries a rounding floor
// of about eps_32 ||A|| ||x||, which on ill-conditioned meshes exceeds the
// inner tolerance, so the FP64 outer residual judges the correction.
template <typename T>
static sem_status fgmres(sem_gmres G, int prec, const T *b, T *x, bool x_zero, double atol,
                         int64_t max_iter, sem_solve_info *info, double *res_out, hipStream_t s,
                         bool one_cycle = false) {
    sem_ctx c = G->ctx;
    const int64_t n = c->n_unique, ld = G->ld;
    const unsigned grid = gm_grid(n);
    const int m = G->m;
    T *V = reinterpret_cast<T *>(G->V), *Z = reinterpret_cast<T *>(G->Z);
    T *w = reinterpret_cast<T *>(G->w), *r = reinterpret_cast<T *>(G->r);
    if (x_zero) {
        if (std::is_same<T, double>::value) SEM_HIP(c, launch_fill((double *)x, n, 0.0, s));
        else SEM_HIP(c, launch_fill32((float *)x, n, 0.0f, s));
    }
    double beta = 0.0;
    sem_status e = residual<T>(G, prec, b, x, r, w, x_zero, &beta, s);
    if (e) return e;
    *res_out = beta;
    if (!std::isfinite(beta)) return gfail(G, SEM_ERR_NAN, "non-finite residual");
    if (beta <= atol) return SEM_OK;
    std::vector<double> H((size_t)(m + 1) * m), Hr((size_t)(m + 1) * m), hs(m), cs(m), sn(m),
        g(m + 1), y(m);
    for (;;) {
        const double inv = 1.0 / beta;                 // V_0 = r / beta
        hipLaunchKernelGGL((k_gm_scale<T, T>), dim3(grid), dim3(kGmBlock), 0, s, n, (const T *)r, V, inv);
        std::fill(H.begin(), H.end(), 0.0);
        std::fill(g.begin(), g.end(), 0.0);
        g[0] = beta;
        std::fill(Hr.begin(), Hr.end(), 0.0);
        // Column k of the Hessenberg matrix is complete once the vector in
        // slot k+1 has had its second projection (during step k+1, or in a
        // closing sweep): then it is rotated into H and g.
        auto rotate = [&](int k) {
            for (int i = 0; i <= k + 1; ++i) H[(size_t)i * m + k] = Hr[(size_t)i * m + k];
            for (int i = 0; i < k; ++i) {
                const double a = H[(size_t)i * m + k], bq = H[(size_t)(i + 1) * m + k];
                H[(size_t)i * m + k] = cs[i] * a + sn[i] * bq;
                H[(size_t)(i + 1) * m + k] = -sn[i] * a + cs[i] * bq;
            }
            const double a = H[(size_t)k * m + k], bq = H[(size_t)(k + 1) * m + k];
            const double den = std::hypot(a, bq);
            cs[k] = den > 0 ? a / den : 1.0;
            sn[k] = den > 0 ? bq / den : 0.0;
            H[(size_t)k * m + k] = den;
            H[(size_t)(k + 1) * m + k] = 0.0;
            g[k + 1] = -sn[k] * g[k];
            g[k] = cs[k] * g[k];
        };
        // vector in slot k+1 = (beta v_{k+1} + V q) / c_k: add its second
        // projection to column k (hs[k] = 1/c_k) and complete the column
        auto complete = [&](int k, const double *q, double beta_k) {
            for (int i = 0; i <= k; ++i) Hr[(size_t)i * m + k] += q[i] * hs[k];
            Hr[(size_t)(k + 1) * m + k] = beta_k * hs[k];
            rotate(k);
        };
        // residual norm if the provisional column k were complete
        auto estimate = [&](int k) {
            double col[kGmMaxVec + 1];
            for (int i = 0; i <= k; ++i) col[i] = Hr[(size_t)i * m + k];
            col[k + 1] = hs[k];                          // provisional h_{k+1,k}
            for (int i = 0; i < k; ++i) {
                const double a = col[i], bq = col[i + 1];
                col[i] = cs[i] * a + sn[i] * bq;
                col[i + 1] = -sn[i] * a + cs[i] * bq;
            }
            const double den = std::hypot(col[k], col[k + 1]);
            return den > 0 ? std::fabs(col[k + 1] / den * g[k]) : std::fabs(g[k]);
        };
        // z_j = M^-1 v_j and w = A z_j
        auto expand = [&](int j) -> sem_status {
            T *Zj = Z + (size_t)j * ld;
            sem_status st = precondition<T>(G, V + (size_t)j * ld, Zj, SEM_PC_SCHWARZ | SEM_PC_COARSE, s, w);
            if (st) return st;
            SEM_HIP(c, launch_ax(c, prec, Zj, w, 0, OUT_ATOMIC, nullptr, nullptr, c->tile[prec], s));
            return SEM_OK;
        };
        // a non-finite step: whatever is queued has ended before the return
        auto nan_step = [&]() {
            (void)hipStreamSynchronize(s);
            return gfail(G, SEM_ERR_NAN, "non-finite Arnoldi vector");
        };
        int jdone = 0;
        bool ahead = false;                              // step j's expansion is queued
        double est0 = beta, est1 = beta;                 // estimates of the last two steps
        for (int j = 0; j < m; ++j) {
            T *Vj = V + (size_t)j * ld, *Vn = V + (size_t)(j + 1) * ld;
            if (!ahead && (e = expand(j))) return e;
            if (j == 0) {
                SEM_HIP(c, gm_first_step<T>(G, V, w, Vn, s));
            } else {
                SEM_HIP(c, (gm_dispatch<GmDots2, T>(j, G, (const T *)V, (const T *)Vj, (const T *)w, s)));
                SEM_HIP(c, (gm_dispatch<GmUpdate2, T>(j, G, (const T *)V, Vj, (const T *)w, Vn, s)));
            }
            e = gm_mark(G, s);
            if (e) return e;
            // The next expansion needs none of the numbers that the host waits
            // for, so it is queued before the wait, unless this step is
            // expected to be the cycle's last (the reduction of the step
            // before, once more, would reach atol): the read-back and some
            // twenty launches, 30 to 56 us a step on small meshes, are hidden.
            ahead = j + 1 < m && info->iterations + 1 < max_iter &&
                    (j == 0 || est1 * std::min(1.0, est1 / est0) > atol);
            if (ahead && (e = expand(j + 1))) return e;
            e = gm_wait(G);
            if (e) return e;
            if (j == 0) {
                const double *d0 = G->host, cc = G->host[kGmScal + 2];
                if (!std::isfinite(d0[0]) || !std::isfinite(d0[1]) || !std::isfinite(cc)) return nan_step();
                Hr[0] = d0[0];
                hs[0] = cc > 0 ? 1.0 / cc : 0.0;
            } else {
                const int L = j;
                const double *d = G->host + kGmD, *sc = G->host + kGmScal;
                for (int q = 0; q < 2 * L + 3; ++q)
                    if (!std::isfinite(d[q])) return nan_step();
                complete(j - 1, d, sc[0]);               // q = d[0..L), beta = sc[0]
                if (sc[0] == 0.0) {                      // the vector lies in span(V): done
                    jdone = j;
                    info->rel_residual = std::fabs(g[j]);
                    break;
                }
                for (int q = 0; q < L; ++q) Hr[(size_t)q * m + j] = d[L + q];
                Hr[(size_t)j * m + j] = sc[1];
                hs[j] = sc[2] > 0 ? 1.0 / sc[2] : 0.0;
            }
            info->iterations += 1;
            jdone = j + 1;
            const double est = estimate(j);
            info->rel_residual = est;
            est0 = est1;
            est1 = est;
            if (est <= atol || info->iterations >= max_iter || j + 1 == m || hs[j] == 0) {
                // closing sweep: second projection of the vector in slot j+1
                double q[kGmMaxVec + 1] = {}, beta_j = 0.0;
                if (hs[j] > 0) {
                    SEM_HIP(c, (gm_dispatch<GmDots, T>(j + 1, G, (const T *)V, (const T *)Vn, G->host, s)));
                    e = gm_mark(G, s);
                    if (!e) e = gm_wait(G);
                    if (e) return e;
                    std::copy(G->host, G->host + j + 2, q);
                    double qq = 0.0;
                    for (int i = 0; i <= j; ++i) qq += q[i] * q[i];
                    const double b2 = q[j + 1] - qq;
                    if (!std::isfinite(b2)) return gfail(G, SEM_ERR_NAN, "non-finite Arnoldi vector");
                    beta_j = b2 > 0 ? std::sqrt(b2) : 0.0;
                    q[j + 1] = 0.0;
                }
                complete(j, q, beta_j);
                info->rel_residual = std::fabs(g[j + 1]);
                break;
            }
        }
        // y = H^-1 g (upper triangular), x += Z y
        for (int i = jdone - 1; i >= 0; --i) {
            double sum = g[i];
            for (int k = i + 1; k < jdone; ++k) sum -= H[(size_t)i * m + k] * y[k];
            y[i] = sum / H[(size_t)i * m + i];
        }
        std::copy(y.begin(), y.begin() + jdone, G->host + kGmCoef);
        SEM_HIP(c, hipMemcpyAsync(G->coef, G->host + kGmCoef, 8 * jdone, hipMemcpyHostToDevice, s));
        SEM_HIP(c, (gm_dispatch<GmXupd, T>(jdone, G, (const T *)Z, x, s)));
        if (one_cycle) {
            *res_out = std::fabs(g[jdone]);
            return SEM_OK;
        }
        e = residual<T>(G, prec, b, x, r, w, false, &beta, s);
        if (e) return e;
        *res_out = beta;
        if (!std::isfinite(beta)) return gfail(G, SEM_ERR_NAN, "non-finite residual");
        if (beta <= atol) return SEM_OK;
        if (info->iterations >= max_iter) return SEM_ERR_NOT_CONVERGED;
        info->restarts += 1;
    }
}

extern "C" sem_status sem_gmres_solve(sem_gmres G, const double *b, double *x,
                                      const sem_solve_options *opts, sem_solve_info *info,
                                      sem_stream stream) {
    sem_solve_info dummy;
    if (!info) info = &dummy;
    std::memset(info, 0, sizeof(*info));
    if (!G || !b || !x) return info->status = gfail(G, SEM_ERR_INVALID, "null argument");
    if (!G->ws) return info->status = gfail(G, SEM_ERR_STATE, "no workspace bound");
    sem_ctx c = G->ctx;
    if (c->helm) return info->status = gfail(G, SEM_ERR_UNSUPPORTED, "Poisson operator only");
    sem_solve_options o;
    if (opts) o = *opts; else sem_default_solve_options(&o);
    if (!(o.tol > 0) || o.max_iter < 1) return info->status = gfail(G, SEM_ERR_INVALID, "bad tolerance or cap");
    const int prec = (int)o.precision;
    if (prec < 0 || prec >= kNumPrec || !((c->precisions >> prec) & 1u))
        return info->status = gfail(G, SEM_ERR_UNSUPPORTED, "precision not configured at setup");
    hipStream_t s = (hipStream_t)stream;
    const int64_t n = c->n_unique;
    auto t0 = std::chrono::steady_clock::now();
    auto done = [&](sem_status st) {
        info->seconds = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
        info->rel_residual = info->true_rel_residual;
        if (st == SEM_ERR_NOT_CONVERGED && G->err.empty()) G->err = "iteration cap reached";
        return info->status = st;
    };
    double bn = 0.0;
    {
        double bb = 0.0;
        sem_status e = gm_norm2<double>(G, b, &bb, s);
        if (e) return done(e);
        bn = std::sqrt(bb);
    }
    if (!std::isfinite(bn)) return done(gfail(G, SEM_ERR_NAN, "non-finite right-hand side"));
    if (bn == 0.0) {
        SEM_HIP(c, launch_fill(x, n, 0.0, s));
        info->true_rel_residual = 0.0;
        return done(SEM_OK);
    }
    double res = 0.0;
    if (prec == SEM_FP64) {
        const sem_status st = fgmres<double>(G, SEM_FP64, b, x, o.zero_guess != 0, o.tol * bn,
                                             o.max_iter, info, &res, s);
        info->true_rel_residual = res / bn;
        return done(st);
    }
    // FP64 iterative refinement around FP32-vector GMRES with the operator
    // of precision prec: r = b - A x (FP64), inner A d = r / ||r|| to
    // inner_tol, x += ||r|| d.  Two corrections in a row that do not halve
    // the FP64 residual mean the operator's accuracy is reached: a 16-bit
    // operator then gives way to the FP32 one (when configured), which
    // gives way to FP64 GMRES from the current x.
    if (o.zero_guess) SEM_HIP(c, launch_fill(x, n, 0.0, s));
    double prev = INFINITY, prev2 = INFINITY;
    int cur = prec, since = 0;            // inner precision, steps since it was set
    for (int outer = 0;; ++outer, ++since) {
        double rn = 0.0;
        // FP64 residual into G->r
        sem_status e = residual<double>(G, SEM_FP64, b, x, G->r, G->w, false, &rn, s);
        if (e) return done(e);
        info->true_rel_residual = rn / bn;
        info->outer_iterations = outer;
        if (!std::isfinite(rn)) return done(gfail(G, SEM_ERR_NAN, "non-finite residual"));
        if (rn <= o.tol * bn) return done(SEM_OK);
        const bool stalled = since >= 2 && rn > 0.5 * prev2;
        if (stalled && cur != SEM_FP32 && ((c->precisions >> SEM_FP32) & 1u) &&
            outer < o.max_outer && info->iterations < o.max_iter) {
            cur = SEM_FP32;                    // 16-bit accuracy reached: FP32 operator
            since = 0;
            prev = prev2 = INFINITY;
        } else if (stalled || outer >= o.max_outer || info->iterations >= o.max_iter) {
            info->fallback = stalled ? SEM_FALLBACK_STAGNATION : SEM_FALLBACK_OUTER_CAP;
            const int64_t before = info->iterations;
            const sem_status st = fgmres<double>(G, SEM_FP64, b, x, false, o.tol * bn,
                                                 o.max_iter, info, &res, s);
            info->fallback_iterations = info->iterations - before;
            info->true_rel_residual = res / bn;
            return done(st);
        }
        prev2 = prev;
        prev = rn;
        // inner right-hand side r / ||r|| in FP32
        const double inv = 1.0 / rn;
        hipLaunchKernelGGL((k_gm_scale<double, float>), dim3(gm_grid(n)), dim3(kGmBlock), 0, s, n,
                           (const double *)G->r, G->rhs32, inv);
        SEM_HIP(c, hipGetLastError());
        double rin = 0.0;
        if (cur != prec) ++info->fp32_outer;
        e = fgmres<float>(G, cur, G->rhs32, G->d32, true, o.inner_tol, o.max_iter, info, &rin,
                          s, true);
        if (e != SEM_OK && e != SEM_ERR_NOT_CONVERGED) return done(e);
        // x += ||r|| d
        SEM_HIP(c, launch_ir_update(c, x, G->d32, nullptr, 0, s, rn));
    }
}
