// Coarse-grid solver of the pressure preconditioner (see sem_coarse.h).
//
// The N = 1 problem is small (one unknown per element vertex), so its ten
// PCG iterations are bound by launches and reductions, not by bytes.  The
// element-based CG took five kernels per iteration with atomics in the
// operator, in a captured graph on a stream of its own, and one host round
// trip per application.  Here the operator is assembled once (27 entries per
// row on a structured mesh), so that w = A p is a gather: no atomics, no
// cleared vector, a fixed summation order, and
//  * up to 1024 rows: one workgroup does everything, one row per lane, the
//    row's entries in registers and p in LDS (three barriers per iteration);
//  * up to 32768 rows of at most 28 entries: PCG with a single reduction, one
//    kernel per iteration, four lanes to a row;
//  * above: two kernels per iteration, one lane to a row.
// Each workgroup sums the partial sums of the preceding kernel itself and takes
// the scalar CG step; workgroup 0 leaves the new state in the slot of this
// (half) iteration, which only the next kernel reads, so no launch is spent on
// a reduction.
// Nothing waits on the host.
// GPU time of one application (8^3 elements, 729 rows; 21x18x16, 7106 rows;
// 48^3, 117,649 rows): 29 / 68 / 155 us, as element-based CG 260 / 250 / 500 us
// and a host round trip.  The kernels of the two larger forms, one kernel and
// two per iteration: 3375 rows 68 and 97 us, 15625 rows 74 and 100, 24389 rows
// 89 and 102, 35937 rows 113 and 104 (32 bytes per neighbour instead of 8; at
// 117,649 rows 26.6 us an iteration instead of 15.4), hence the limit.  The
// one-workgroup form does not gain from the single reduction (28.8 us either
// way).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "sem_coarse.h"
#include "sem_reduce.h"
#include "sem_threads.h"

namespace sem {

namespace {

constexpr int kCsBlock = 256;
constexpr int kCsOneRows = 1024, kCsOneWidth = 27;   // limits of the one-workgroup solve
constexpr int kCsStates = 2 * kCoarseIterations;
// Single-reduction form over several workgroups: entries per lane (of the four
// that share a row) and the rows up to which it is used.
constexpr int kStepSlots = 7;
constexpr int64_t kStepRows = 32768;

size_t a256(size_t x) { return (x + 255) & ~(size_t)255; }

struct CsArgs {
    int64_t n, ld;
    int width;
    const int32_t *idx;
    const double *val, *dinv;
    double *b, *x, *r, *z, *w, *p;
    double *partA, *partB;        // [blocks][3], [blocks][2]
    CgState *st;                  // [kCsStates]
    int nblocks;
    struct CsRow *q0, *q1;        // single-reduction form: rows before and after a step
};

// What a neighbour needs to form u = M^-1 r of a row after the step: one
// gather of 32 bytes.
struct __align__(32) CsRow {
    double r, w, s, dinv;
};

// Sums of NV values over the workgroup (whole waves), one barrier; a barrier
// must lie between two sums through the same `red`.
template <int NV>
__device__ __forceinline__ void cs_block_sum(double (&v)[NV], double (*red)[16]) {
    const int wv = threadIdx.x >> 6, nw = blockDim.x >> 6;
#pragma unroll
    for (int a = 0; a < NV; ++a) v[a] = wave_sum63(v[a]);
    if ((threadIdx.x & 63) == 63)
#pragma unroll
        for (int a = 0; a < NV; ++a) red[a][wv] = v[a];
    __syncthreads();
#pragma unroll
    for (int a = 0; a < NV; ++a) {
        double s = 0.0;
        for (int q = 0; q < nw; ++q) s += red[a][q];
        v[a] = s;
    }
}

// This lane's share of the packed partials of all workgroups (fixed order).
template <int NV>
__device__ __forceinline__ void cs_load_partials(const double *part, int nblocks, double (&v)[NV]) {
#pragma unroll
    for (int a = 0; a < NV; ++a) v[a] = 0.0;
    for (int q = threadIdx.x; q < nblocks; q += kCsBlock)
#pragma unroll
        for (int a = 0; a < NV; ++a) v[a] += part[(size_t)q * NV + a];
}

__device__ __forceinline__ void cs_init(CgState &s) {
    s = CgState{};
    s.tol2 = 1e-28;               // (1e-14)^2 relative to b.b
    s.max_iter = kCoarseIterations;
}

// Entry values of the assembled operator: row g sums, over its element
// copies in ascending order, the element matrix of the trilinear basis.
__global__ void k_cs_assemble(int64_t n, int64_t ld, int width, const int32_t *__restrict__ idx,
                              const int32_t *__restrict__ off, const int32_t *__restrict__ copies,
                              const int32_t *__restrict__ bmap, const uint8_t *__restrict__ bdir,
                              const double *__restrict__ G, const double *__restrict__ D,
                              double *__restrict__ val) {
    const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= n) return;
    for (int s = 0; s < width; ++s) val[s * ld + g] = 0.0;
    if (bdir[g]) return;
    for (int32_t q = off[g]; q < off[g + 1]; ++q) {
        const int64_t e = copies[q] >> 3;
        const int c = copies[q] & 7;
        for (int c2 = 0; c2 < 8; ++c2) {
            const int32_t m = bmap[e * 8 + c2];
            if (m < 0) continue;
            double a = 0.0;
            for (int p = 0; p < 8; ++p) {
                const int x[3] = {p & 1, (p >> 1) & 1, p >> 2};
                double gc[3], g2[3];
                for (int d = 0; d < 3; ++d) {
                    // derivative of the corner's shape function along d at p
                    const int same = p ^ c, same2 = p ^ c2, rest = 7 & ~(1 << d);
                    gc[d] = (same & rest) ? 0.0 : D[x[d] * 2 + ((c >> d) & 1)];
                    g2[d] = (same2 & rest) ? 0.0 : D[x[d] * 2 + ((c2 >> d) & 1)];
                }
                double f[6];
                for (int t = 0; t < 6; ++t) f[t] = G[goff(8, e, x[2], x[0] + 2 * x[1], t, 2)];
                a += gc[0] * (f[0] * g2[0] + f[3] * g2[1] + f[4] * g2[2]) +
                     gc[1] * (f[3] * g2[0] + f[1] * g2[1] + f[5] * g2[2]) +
                     gc[2] * (f[4] * g2[0] + f[5] * g2[1] + f[2] * g2[2]);
            }
            for (int s = 0; s < width; ++s)
                if (idx[s * ld + g] == m) {
                    val[s * ld + g] += a;
                    break;
                }
        }
    }
}

// The whole solve in one workgroup.
__global__ void __launch_bounds__(kCsOneRows) k_cs_one(CsArgs P) {
    __shared__ double ps[kCsOneRows];
    __shared__ double redA[2][16], redB[2][16];
    const int i = threadIdx.x;
    const bool on = i < P.n;
    double v[kCsOneWidth];
    uint32_t id[(kCsOneWidth + 1) / 2];      // columns, two to a register
#pragma unroll
    for (int s = 0; s < kCsOneWidth; ++s) {
        const bool take = on && s < P.width;
        v[s] = take ? P.val[(size_t)s * P.ld + i] : 0.0;
        const uint32_t c = take ? (uint32_t)P.idx[(size_t)s * P.ld + i] : 0u;
        id[s / 2] = (s & 1) ? id[s / 2] | (c << 16) : c;
    }
    const double b = on ? P.b[i] : 0.0, d = on ? P.dinv[i] : 0.0;
    if (on) P.b[i] = 0.0;
    CgState S;
    cs_init(S);
    double r = b, p = d * r, x = 0.0;
    {
        double t[2] = {r * p, r * r};
        cs_block_sum<2>(t, redB);
        cg_finish_begin(S, t[0], t[1], t[1]);
    }
    for (int it = 0; it < kCoarseIterations && !S.done; ++it) {
        ps[i] = p;
        __syncthreads();
        double w = 0.0;
#pragma unroll
        for (int s = 0; s < kCsOneWidth; ++s) w += v[s] * ps[(id[s / 2] >> (16 * (s & 1))) & 0xffffu];
        double t1[1] = {p * w};
        cs_block_sum<1>(t1, redA);
        cg_finish_ax(S, t1[0]);
        if (S.done) break;
        x += S.alpha * p;
        r -= S.alpha * w;
        const double z = d * r;
        double t2[2] = {r * r, r * z};
        cs_block_sum<2>(t2, redB);
        cg_finish_update(S, t2[0], t2[1]);
        p = z + S.beta * p;
    }
    if (on) P.x[i] = S.status == CG_NONFINITE ? __builtin_nan("") : x;
    if (i == 0) {
        P.st[kCsStates - 1].status = S.status;
        P.st[kCsStates - 1].done = S.done;
    }
}

// Scalars of the single-reduction form (Chronopoulos and Gear) from gamma =
// r.u, delta = u.A u and r.r of the current residual, u = M^-1 r: beta as
// usual, p.A p = delta - beta^2 (p.A p)' with (p.A p)' of the step before.
__device__ __forceinline__ void cs_scalars(CgState &S, bool first, double gamma, double delta,
                                           double rr) {
    if (first) {
        cs_init(S);
        cg_finish_begin(S, gamma, rr, rr);
        if (!S.done) cg_finish_ax(S, delta);
        return;
    }
    const double before = S.pAp;
    cg_finish_update(S, rr, gamma);
    if (!S.done) cg_finish_ax(S, delta - S.beta * S.beta * before);
}

// The single-reduction form over several workgroups, one kernel per iteration
// and one before.  kStepInit: w = A u for r = b; the others sum the partials
// of the kernel before, step, and form w = A u of the new residual, of which
// every row computes its neighbours' u itself, u_j = dinv_j (r_j - alpha (w_j +
// beta s_j)), from the old rows (two buffers in turn).  kStepLast only needs x.
// Four lanes share a row, kStepSlots entries each, so that all loads of a row
// are requested at once, before the sums: the kernel is a chain of three loads
// and a sum, 256 lanes to 64 rows.
enum { kStepInit, kStepFirst, kStepNext, kStepLast };
template <int MODE>
__global__ void __launch_bounds__(kCsBlock) k_cs_step(CsArgs P, int it) {
    __shared__ double red[3][16];
    __shared__ CgState sh;
    const int sub = threadIdx.x & 3;
    const int64_t i = (int64_t)blockIdx.x * (kCsBlock / 4) + (threadIdx.x >> 2);
    const bool on = i < P.n;
    const CsRow *old = (it & 1) ? P.q1 : P.q0;
    CsRow *next = MODE == kStepInit ? P.q0 : ((it & 1) ? P.q0 : P.q1);
    int stopped = 0;
    double t[3] = {0.0, 0.0, 0.0};
    if constexpr (MODE == kStepNext || MODE == kStepLast) stopped = P.st[it - 1].done;
    if (MODE != kStepInit && !stopped)
        cs_load_partials<3>((it & 1) ? P.partB : P.partA, P.nblocks, t);
    double a[kStepSlots];
    CsRow nb[kStepSlots], me{0.0, 0.0, 0.0, 0.0};
    double p = 0.0, x = 0.0;
    const bool matrix = MODE != kStepLast;
    if (on && !stopped) {
        if constexpr (MODE == kStepInit) {
            me.r = P.b[i];
            me.dinv = P.dinv[i];
        } else {
            me = old[i];
            if constexpr (MODE != kStepFirst) {
                p = P.p[i];
                x = P.x[i];
            }
        }
        if (matrix) {
            int j[kStepSlots];
#pragma unroll
            for (int s = 0; s < kStepSlots; ++s) {
                const int c = sub + 4 * s;
                j[s] = c < P.width ? P.idx[(size_t)c * P.ld + i] : (int)i;
                a[s] = c < P.width ? P.val[(size_t)c * P.ld + i] : 0.0;
            }
#pragma unroll
            for (int s = 0; s < kStepSlots; ++s) {
                if constexpr (MODE == kStepInit) nb[s] = CsRow{P.b[j[s]], 0.0, 0.0, P.dinv[j[s]]};
                else nb[s] = old[j[s]];
            }
        }
    }
    double alpha = 0.0, beta = 0.0;
    if constexpr (MODE != kStepInit) {
        if (!stopped) cs_block_sum<3>(t, red);
        if (threadIdx.x == 0) {
            if (MODE != kStepFirst) sh = P.st[it - 1];
            if (!stopped) cs_scalars(sh, MODE == kStepFirst, t[0], t[1], t[2]);
            if (blockIdx.x == 0) {
                P.st[it] = sh;
                if (MODE == kStepLast) P.st[kCsStates - 1] = sh;
            }
        }
        __syncthreads();
        if (MODE == kStepFirst && on && sub == 0) P.b[i] = 0.0;
        if (sh.done) {
            if (on && sub == 0 && !stopped) {
                if (sh.status == CG_NONFINITE) P.x[i] = __builtin_nan("");
                else if (MODE == kStepFirst) P.x[i] = 0.0;
            }
            return;
        }
        alpha = sh.alpha;
        beta = sh.beta;
    }
    // this row's step
    const double u0 = me.dinv * me.r;
    if constexpr (MODE != kStepInit) {
        p = u0 + beta * p;
        if (on && sub == 0) {
            P.x[i] = x + alpha * p;
            if (matrix) P.p[i] = p;
        }
        if (!matrix) return;
        me.s = me.w + beta * me.s;
        me.r -= alpha * me.s;
    }
    const double u = me.dinv * me.r;
    double w = 0.0;
    if (on)
#pragma unroll
        for (int s = 0; s < kStepSlots; ++s)
            w += a[s] * (nb[s].dinv * (nb[s].r - alpha * (nb[s].w + beta * nb[s].s)));
    w += dpp_mov<0xb1>(w);                   // quad_perm [1,0,3,2]
    w += dpp_mov<0x4e>(w);                   // quad_perm [2,3,0,1]
    me.w = w;
    if (on && sub == 0) next[i] = me;
    const bool lead = on && sub == 0;
    double g[3] = {lead ? me.r * u : 0.0, lead ? w * u : 0.0, lead ? me.r * me.r : 0.0};
    __syncthreads();                         // red: the first sum has been read
    cs_block_sum<3>(g, red);
    double *part = MODE == kStepInit || (it & 1) ? P.partA : P.partB;
    if (threadIdx.x == 0)
#pragma unroll
        for (int c = 0; c < 3; ++c) part[(size_t)blockIdx.x * 3 + c] = g[c];
}

// First half of iteration `it`: the scalar step after the residual update,
// p = z + beta p, w = A p = A z + beta w, and the partial sums of p.w (with
// r.z and r.r in the first iteration).  A z does not need beta, so the row's
// entries and neighbours are on their way while the sums are formed.
template <bool FIRST>
__global__ void __launch_bounds__(kCsBlock) k_cs_dir(CsArgs P, int it) {
    __shared__ double red[3][16];
    __shared__ CgState sh;
    const int64_t i = (int64_t)blockIdx.x * kCsBlock + threadIdx.x;
    const bool on = i < P.n;
    int stopped = 0;
    double t2[2] = {0.0, 0.0};
    if constexpr (!FIRST) {
        stopped = P.st[2 * it - 2].done;
        if (!stopped) cs_load_partials<2>(P.partB, P.nblocks, t2);
    }
    double az = 0.0, zi = 0.0, bi = 0.0, pi = 0.0, wi = 0.0;
    if (on && !stopped) {
        for (int s0 = 0; s0 < P.width; s0 += kCoarseUnroll) {
            int j[kCoarseUnroll];
            double a[kCoarseUnroll], zj[kCoarseUnroll];
#pragma unroll
            for (int s = 0; s < kCoarseUnroll; ++s) {
                j[s] = P.idx[(size_t)(s0 + s) * P.ld + i];
                a[s] = P.val[(size_t)(s0 + s) * P.ld + i];
            }
#pragma unroll
            for (int s = 0; s < kCoarseUnroll; ++s)
                zj[s] = FIRST ? P.dinv[j[s]] * P.b[j[s]] : P.z[j[s]];
#pragma unroll
            for (int s = 0; s < kCoarseUnroll; ++s) az += a[s] * zj[s];
        }
        if (FIRST) {
            bi = P.b[i];
            zi = P.dinv[i] * bi;
        } else {
            zi = P.z[i];
            pi = P.p[i];
            wi = P.w[i];
        }
    }
    double beta = 0.0;
    if constexpr (!FIRST) {
        if (!stopped) cs_block_sum<2>(t2, red);
        if (threadIdx.x == 0) {
            sh = P.st[2 * it - 2];
            if (!stopped) cg_finish_update(sh, t2[0], t2[1]);
            if (blockIdx.x == 0) P.st[2 * it - 1] = sh;
        }
        __syncthreads();
        if (sh.done) {
            if (!stopped && sh.status == CG_NONFINITE && on) P.x[i] = __builtin_nan("");
            return;
        }
        beta = sh.beta;
    }
    pi = zi + beta * pi;
    wi = az + beta * wi;
    if (on) {
        P.p[i] = pi;
        P.w[i] = wi;
    }
    if constexpr (FIRST) {
        double t[3] = {pi * wi, bi * pi, bi * bi};
        cs_block_sum<3>(t, red);
        if (threadIdx.x == 0)
#pragma unroll
            for (int a = 0; a < 3; ++a) P.partA[(size_t)blockIdx.x * 3 + a] = t[a];
    } else {
        double t[1] = {pi * wi};
        cs_block_sum<1>(t, red);
        if (threadIdx.x == 0) P.partA[blockIdx.x] = t[0];
    }
}

// Second half: alpha, x += alpha p, r -= alpha w, z = dinv r and the partial
// sums of r.r and r.z (the last iteration only needs x).  The first iteration
// starts from x = 0, r = b and clears b for the next application.
template <bool FIRST>
__global__ void __launch_bounds__(kCsBlock) k_cs_update(CsArgs P, int it) {
    __shared__ double red[3][16];
    __shared__ CgState sh;
    const int64_t i = (int64_t)blockIdx.x * kCsBlock + threadIdx.x;
    const bool on = i < P.n, last = it == kCoarseIterations - 1;
    constexpr int NV = FIRST ? 3 : 1;
    double t[NV] = {};
    const int stopped = FIRST ? 0 : P.st[2 * it - 1].done;
    if (!stopped) cs_load_partials<NV>(P.partA, P.nblocks, t);
    double ri = 0.0, wi = 0.0, pi = 0.0, di = 0.0, xi = 0.0;
    if (on && !stopped) {
        ri = FIRST ? P.b[i] : P.r[i];
        wi = P.w[i];
        pi = P.p[i];
        di = P.dinv[i];
        if (!FIRST) xi = P.x[i];
    }
    if (!stopped) cs_block_sum<NV>(t, red);
    if (threadIdx.x == 0) {
        if constexpr (FIRST) {
            cs_init(sh);
            cg_finish_begin(sh, t[1], t[2], t[2]);
            if (!sh.done) cg_finish_ax(sh, t[0]);
        } else {
            sh = P.st[2 * it - 1];
            if (!stopped) cg_finish_ax(sh, t[0]);
        }
        if (blockIdx.x == 0) {
            P.st[2 * it] = sh;
            if (last) P.st[kCsStates - 1] = sh;
        }
    }
    __syncthreads();
    if (FIRST && on) P.b[i] = 0.0;
    if (sh.done) {
        if (on && !stopped) {
            if (sh.status == CG_NONFINITE) P.x[i] = __builtin_nan("");
            else if (FIRST) P.x[i] = 0.0;
        }
        return;
    }
    if (on) P.x[i] = xi + sh.alpha * pi;
    if (last) return;
    ri -= sh.alpha * wi;
    const double zi = di * ri;
    if (on) {
        P.r[i] = ri;
        P.z[i] = zi;
    }
    double u[2] = {ri * ri, ri * zi};
    cs_block_sum<2>(u, red);
    if (threadIdx.x == 0) {
        P.partB[(size_t)blockIdx.x * 2] = u[0];
        P.partB[(size_t)blockIdx.x * 2 + 1] = u[1];
    }
}

int cs_blocks(int64_t n) { return (int)((n + kCsBlock - 1) / kCsBlock); }
int cs_step_blocks(int64_t n) { return (int)((n + kCsBlock / 4 - 1) / (kCsBlock / 4)); }
bool cs_step_form(const CoarsePlan &p) { return p.n <= kStepRows && p.width <= 4 * kStepSlots; }

}  // namespace

void coarse_pattern(sem_ctx c, CoarsePlan &plan) {
    const int64_t n = c->n_unique;
    plan.n = n;
    plan.ld = (int64_t)(a256(4 * (size_t)n) / 4);
    std::vector<std::vector<int32_t>> rows(n);
    host_ranges(n, [&](int64_t g0, int64_t g1) {
        for (int64_t g = g0; g < g1; ++g) {
            if (c->bdir[g]) continue;
            std::vector<int32_t> &r = rows[g];
            r.reserve(64);
            for (int32_t q = c->csr_off[g]; q < c->csr_off[g + 1]; ++q) {
                const int64_t e = c->csr_idx[q] / 8;
                for (int c2 = 0; c2 < 8; ++c2) {
                    const int32_t m = c->bmap[(size_t)e * 8 + c2];
                    if (m >= 0) r.push_back(m);
                }
            }
            std::sort(r.begin(), r.end());
            r.erase(std::unique(r.begin(), r.end()), r.end());
        }
    });
    size_t w = 1;
    for (auto &r : rows) w = std::max(w, r.size());
    plan.width = (int)((w + kCoarseUnroll - 1) / kCoarseUnroll) * kCoarseUnroll;
    plan.ids.assign((size_t)plan.width * plan.ld, 0);
    for (int s = 0; s < plan.width; ++s)
        for (int64_t g = 0; g < n; ++g)
            plan.ids[(size_t)s * plan.ld + g] =
                (size_t)s < rows[g].size() ? rows[g][s] : (int32_t)g;
}

static size_t layout(const CoarsePlan &p, size_t (&off)[7]) {
    size_t o = 0;
    auto take = [&](size_t bytes) {
        const size_t at = o;
        o += a256(bytes);
        return at;
    };
    off[0] = take(4 * (size_t)p.width * p.ld);
    off[1] = take(8 * (size_t)p.width * p.ld);
    const bool step = cs_step_form(p);
    // p, and r, z, w or the two buffers of rows
    off[5] = take(8 * (size_t)p.n);
    for (int q = 0; q < 3; ++q) off[2 + q] = take((step ? (q < 2 ? sizeof(CsRow) : 0) : 8) * (size_t)p.n);
    off[6] = take(8 * (step ? 6 * (size_t)cs_step_blocks(p.n) : 5 * (size_t)cs_blocks(p.n)) +
                  sizeof(CgState) * kCsStates + 256);
    return o;
}

size_t coarse_bytes(const CoarsePlan &p) {
    size_t off[7];
    return layout(p, off);
}

hipError_t coarse_bind(sem_ctx c, CoarsePlan &p, char *ws, double *b, double *x, hipStream_t s) {
    size_t off[7];
    layout(p, off);
    p.idx = reinterpret_cast<int32_t *>(ws + off[0]);
    p.val = reinterpret_cast<double *>(ws + off[1]);
    p.r = reinterpret_cast<double *>(ws + off[2]);
    p.z = reinterpret_cast<double *>(ws + off[3]);
    p.w = reinterpret_cast<double *>(ws + off[4]);
    p.p = reinterpret_cast<double *>(ws + off[5]);
    p.state = reinterpret_cast<CgState *>(ws + off[6]);
    p.part = reinterpret_cast<double *>(ws + off[6] + a256(sizeof(CgState) * kCsStates));
    p.dinv = dptr<double>(c, c->L.dinv64);
    p.b = b;
    p.x = x;
    hipError_t e = hipMemcpyAsync(p.idx, p.ids.data(), 4 * p.ids.size(), hipMemcpyHostToDevice, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_cs_assemble, dim3((unsigned)cs_blocks(p.n)), dim3(kCsBlock), 0, s, p.n,
                       p.ld, p.width, (const int32_t *)p.idx, dptr<int32_t>(c, c->L.csr_off),
                       dptr<int32_t>(c, c->L.csr_idx), dptr<int32_t>(c, c->L.bmap),
                       dptr<uint8_t>(c, c->L.bdir), dptr<double>(c, c->L.G[0]),
                       dptr<double>(c, c->L.dhat64), p.val);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    return launch_fill(b, p.n, 0.0, s);
}

hipError_t coarse_solve(const CoarsePlan &p, hipStream_t s) {
    const bool step = cs_step_form(p);
    const int nb = step ? cs_step_blocks(p.n) : cs_blocks(p.n);
    CsArgs A{p.n, p.ld, p.width, p.idx, p.val, p.dinv, p.b, p.x, p.r, p.z, p.w, p.p,
             p.part, p.part + 3 * (size_t)nb, p.state, nb,
             reinterpret_cast<CsRow *>(p.r), reinterpret_cast<CsRow *>(p.z)};
    if (p.n <= kCsOneRows && p.width <= kCsOneWidth) {
        hipLaunchKernelGGL(k_cs_one, dim3(1), dim3((unsigned)((p.n + 63) / 64 * 64)), 0, s, A);
        return hipGetLastError();
    }
    const dim3 g((unsigned)nb), t(kCsBlock);
    if (step) {
        hipLaunchKernelGGL(k_cs_step<kStepInit>, g, t, 0, s, A, 0);
        hipLaunchKernelGGL(k_cs_step<kStepFirst>, g, t, 0, s, A, 0);
        for (int it = 1; it + 1 < kCoarseIterations; ++it)
            hipLaunchKernelGGL(k_cs_step<kStepNext>, g, t, 0, s, A, it);
        hipLaunchKernelGGL(k_cs_step<kStepLast>, g, t, 0, s, A, kCoarseIterations - 1);
        return hipGetLastError();
    }
    for (int it = 0; it < kCoarseIterations; ++it) {
        if (it == 0) {
            hipLaunchKernelGGL(k_cs_dir<true>, g, t, 0, s, A, it);
            hipLaunchKernelGGL(k_cs_update<true>, g, t, 0, s, A, it);
        } else {
            hipLaunchKernelGGL(k_cs_dir<false>, g, t, 0, s, A, it);
            hipLaunchKernelGGL(k_cs_update<false>, g, t, 0, s, A, it);
        }
    }
    return hipGetLastError();
}

const CgState *coarse_result(const CoarsePlan &p) { return p.state + (kCsStates - 1); }

}  // namespace sem
