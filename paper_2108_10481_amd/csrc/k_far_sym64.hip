// Far field, matrix-free, FP64, with every unordered triangle pair evaluated
// once for both directions, as k_far_sym.hip does in FP32 (same sums, forms,
// scaled coordinates and partial slots; see there).  Everything is FP64 and on
// the VALU: the FP64 matrix instructions of this chip share the vector unit
// (one v_mfma_f64_16x16x4 and 32 independent FMAs take 261 cycles together, 118
// and 158 apart), so the squared distances are the subtracted form.
//
// Work: tiles of 64 Morton-consecutive triangles, an item (a, b, z), a <= b, is the
// pairs of tile range a x tile range b that meet in the steps of part z, done by
// one block of four wavefronts.  For a tile pair (I, J) lane l of every wavefront
// holds target t = 64 I + l; in step k it meets source s = 64 J + ((l + k) mod 64)
// (on a diagonal tile I == J only the steps and lanes that meet each unordered
// pair once: 1 <= k <= 31, and k = 32 on the lower half of the lanes).  Wavefront
// w takes the steps k = w + 4 (z + Z i).  The target's sums stay in its lane; the
// sums of the source side are held by the lane that meets the source and move 4 Z
// lanes down after every step.  Tile J's records are staged once per block in LDS
// (one array per field: the rotated reads hit distinct banks), about 1.3 reads
// per point pair.  The layout of k_far_sym.hip (rows broadcast from LDS, 6.7 reads
// per pair) was tried first: the LDS was 50% busy, the wavefronts waited for it
// 38% of the time and taking 12% of the arithmetic out changed nothing.
//
// Bound: the FP64 vector rate (an FP64 instruction measures 5.2 cycles per
// wavefront at this load, v_rsq_f64 18): 36 (direct) and 47 (second kind)
// instructions per unordered point pair against 2 x 55 issue slots of the kernel
// that evaluates each ordered pair.  Measured per product, before and now:
// direct 320 triangles 163 -> 50 us, 5780 1.90 -> 0.91 ms, 20480 21.2 -> 10.8 ms;
// Juffer 12500 9.97 -> 4.87 ms.
#include <algorithm>

#include "far.h"
#include "fp64.h"

namespace pbm {

constexpr int kS64Batch = 2;
constexpr int kS64Waves = 4, kS64Tile = 64;
typedef double f64x2 __attribute__((ext_vector_type(2)));

struct alignas(16) S64Cols {
    double y[6][3][kS64Tile];    // Y_q
    double n[4][kS64Tile];       // n_s, O_s
    double w[6][4][kS64Tile];    // the source point's four weights
    double curl[3][kS64Tile];    // C_s
    double cen[3][kS64Tile];     // centroid
    int id[3][kS64Tile];
    // targets: what a step uses once (in registers these spilled)
    double tcen[3][kS64Tile], tcurl[3][kS64Tile];
};
struct alignas(16) S64Lds {
    S64Cols c;
    double out[kS64Waves][16][kS64Tile];
    int item;
};

// the target of a lane, relative to its tile's centre, and its sums
struct S64Target {
    double x[6], y[6], z[6], n[3], o, b1[6], b2[6];
    double a1[6], a2[6], W[3];
};

// One step: the 36 point pairs of the lane's target and source j: adds the
// target's sums to t and the source's to acc1, acc2, accW.  Forms and factoring as
// sym_block (k_far_sym.hip).
template <int FORM, bool K0, bool NEAR, bool LOC>
__device__ __forceinline__ void s64_step(const SymCoef<double> &cf, const S64Cols &C, int lane, int j, bool live, S64Target &t,
                                         double (&acc1)[6], double (&acc2)[6], double (&accW)[3])
{
    const double nsx = C.n[0][j], nsy = C.n[1][j], nsz = C.n[2][j], os = C.n[3][j];
    auto dns_of = [&](int p) { return fma(t.x[p], nsx, fma(t.y[p], nsy, fma(t.z[p], nsz, -os))); };
    double rc = 0.0, ec = 1.0;   // LOC: centroid distance and its exponential
    if (LOC) {
        const double dx = C.tcen[0][lane] - C.cen[0][j], dy = C.tcen[1][lane] - C.cen[1][j],
                     dz = C.tcen[2][lane] - C.cen[2][j];
        double c2[1] = {dx * dx + dy * dy + dz * dz}, ci[1];
        rsqrt3_n<1>(c2, ci);
        rc = c2[0] *= ci[0];
        exp2neg_n<1>(c2);
        ec = c2[0];
    }
    double P[6], Q[6];
    double gs = 0.0, nn = 0.0;
#pragma unroll
    for (int p = 0; p < 6; ++p) P[p] = Q[p] = 0.0;
    if (FORM >= 1) {
        nn = t.n[0] * nsx + t.n[1] * nsy + t.n[2] * nsz;
#pragma unroll
        for (int p = 0; p < 6; ++p) Q[p] = dns_of(p) * t.b2[p];
    }
#pragma unroll
    for (int q = 0; q < 6; ++q) {
        const double yx = C.y[q][0][j], yy = C.y[q][1][j], yz = C.y[q][2][j];
        const double w0 = C.w[q][0][j], w1 = C.w[q][1][j], w2 = C.w[q][2][j], w3 = C.w[q][3][j];
        const double dnt = fma(-yx, t.n[0], fma(-yy, t.n[1], fma(-yz, t.n[2], t.o)));
        const double tq = dnt * w2, nb = nn * w3;   // FORM >= 1
        double S1 = 0.0, S2 = 0.0, s1 = 0.0, s2 = 0.0;
        // kS64Batch target points at a time, every step of their pairs together, so
        // that their dependent chains (reciprocal root, exponential) overlap
#pragma unroll
        for (int p0 = 0; p0 < 6; p0 += kS64Batch) {
            constexpr int N = kS64Batch;
            double r2[N], ri[N], e[N];
#pragma unroll
            for (int i = 0; i < N; ++i) {
                const double dx = t.x[p0 + i] - yx, dy = t.y[p0 + i] - yy, dz = t.z[p0 + i] - yz;
                r2[i] = dx * dx + dy * dy + dz * dz;
            }
            rsqrt3_n<N>(r2, ri);
            if (NEAR) {
#pragma unroll
                for (int i = 0; i < N; ++i) ri[i] = live ? ri[i] : 0.0;   // every kernel value is then zero
            }
            if (!K0) {
                if (LOC) {
#pragma unroll
                    for (int i = 0; i < N; ++i) e[i] = fma(-r2[i], ri[i], rc);
                    exp2near_n<N>(e);
#pragma unroll
                    for (int i = 0; i < N; ++i) e[i] *= ec;
                } else {
#pragma unroll
                    for (int i = 0; i < N; ++i) e[i] = r2[i] * ri[i];
                    exp2neg_n<N>(e);
                }
            }
#pragma unroll
            for (int i = 0; i < N; ++i) {
                const int p = p0 + i;
                const double ri2 = ri[i] * ri[i], R3 = ri[i] * ri2;
                const double gy = K0 ? ri[i] : e[i] * ri[i];
                const double E = K0 ? R3 : e[i] * fma(cf.kap, ri2, R3);
                if (FORM == 0) {
                    P[p] = fma(w0, R3, P[p]);
                    t.a1[p] = fma(w1, ri[i], t.a1[p]);
                    Q[p] = fma(w2, E, Q[p]);
                    t.a2[p] = fma(w3, gy, t.a2[p]);
                    S1 = fma(t.b1[p], R3, S1);
                    s1 = fma(t.b2[p], ri[i], s1);
                    S2 = fma(t.b1[p], E, S2);
                    s2 = fma(t.b2[p], gy, s2);
                } else {
                    const double ww = rule_w(p) * rule_w(q);
                    double k, vv, kt, dd;
                    if (FORM == 3) {
                        k = kt = E;
                        vv = dd = gy;
                    } else if (FORM == 1) {
                        k = fma(cf.bK, E, R3);
                        vv = fma(cf.bV, gy, ri[i]);
                        kt = fma(cf.bT, E, R3);
                        dd = fma(cf.bD, gy, ri[i]);
                    } else {
                        k = fma(cf.bK, E, cf.aK * R3);
                        vv = fma(cf.bV, gy, cf.aV * ri[i]);
                        kt = fma(cf.bT, E, cf.aT * R3);
                        dd = fma(cf.bD, gy, cf.aD * ri[i]);
                    }
                    P[p] = fma(w0, k, P[p]);
                    t.a1[p] = fma(w1, vv, t.a1[p]);
                    t.a2[p] = fma(tq, kt, fma(nb, gy, t.a2[p]));
                    S1 = fma(t.b1[p], k, S1);
                    s1 = fma(t.b2[p], vv, s1);
                    s2 = fma(Q[p], kt, s2);
                    S2 = fma(t.b1[p], gy, S2);
                    gs = fma(ww, dd, gs);
                }
            }
        }
        acc1[q] = fma(cf.cV, s1, fma(-cf.cK * dnt, S1, acc1[q]));
        acc2[q] = FORM == 0 ? fma(cf.cD, s2, fma(-cf.cT * dnt, S2, acc2[q])) : fma(cf.kD * nn, S2, fma(-cf.cT, s2, acc2[q]));
        // keeps the next source points' LDS reads behind these pairs: hoisted all
        // together they took 92 registers and the sums spilled
        asm volatile("" ::: "memory");
    }
#pragma unroll
    for (int p = 0; p < 6; ++p) {
        const double dns = dns_of(p);
        t.a1[p] = fma(dns, P[p], t.a1[p]);
        if (FORM == 0) t.a2[p] = fma(dns, Q[p], t.a2[p]);
    }
    if (FORM >= 1) {
        const double gc = cf.cD * gs;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            t.W[c] = fma(gc, C.curl[c][j], t.W[c]);
            accW[c] = fma(gc, C.tcurl[c][lane], accW[c]);
        }
    }
}

// the steps k = k0, k0 + dk, .. of one tile pair: returns the step after the last
// (lane l then holds the sums of source (l + k) mod 64)
template <int FORM, bool K0, bool NEAR, bool LOC>
__device__ __forceinline__ int s64_steps(const SymCoef<double> &cf, const S64Cols &C, int lane, int k0, int dk, bool diag,
                                         const int (&tv)[3], S64Target &t, double (&acc1)[6], double (&acc2)[6],
                                         double (&accW)[3])
{
    const int kend = NEAR && diag ? 33 : 64;
    int k = k0;
#pragma unroll 1
    for (; k < kend; k += dk) {
        const int j = (lane + k) & 63;
        bool live = true;
        if (NEAR) {
            live = (tv[0] >= 0) & (C.id[0][j] >= 0) & (!diag | ((k >= 1) & ((k < 32) | (lane < 32))));
#pragma unroll
            for (int v = 0; v < 3; ++v)
#pragma unroll
                for (int u = 0; u < 3; ++u) live = live & (tv[v] != C.id[u][j]);
        }
        s64_step<FORM, K0, NEAR, LOC>(cf, C, lane, j, live, t, acc1, acc2, accW);
        // the source sums move dk lanes down: lane l next meets source l + k + dk
        const int from = (lane + dk) & 63;
#pragma unroll
        for (int q = 0; q < 6; ++q) {
            acc1[q] = __shfl(acc1[q], from);
            acc2[q] = __shfl(acc2[q], from);
        }
        if (FORM >= 1) {
#pragma unroll
            for (int c = 0; c < 3; ++c) accW[c] = __shfl(accW[c], from);
        }
    }
    return k;
}

// the wavefronts' 16 values of 64 triangles, summed in wavefront order onto (add) or
// into the slot o (16 values per triangle) of triangles s0..
__device__ __forceinline__ void s64_flush(const S64Lds &L, int tid, int s0, int T, double *__restrict__ o, bool add)
{
    const int s = s0 + (tid & 63), m = tid >> 6;   // values 4 m .. 4 m + 3
    if (s >= T) return;
    f64x2 *so = (f64x2 *)(o + (size_t)s * 16 + 4 * m);
    f64x2 v0 = add ? so[0] : f64x2{0.0, 0.0}, v1 = add ? so[1] : f64x2{0.0, 0.0};
#pragma unroll
    for (int w = 0; w < kS64Waves; ++w) {
        v0 += f64x2{L.out[w][4 * m][tid & 63], L.out[w][4 * m + 1][tid & 63]};
        v1 += f64x2{L.out[w][4 * m + 2][tid & 63], L.out[w][4 * m + 3][tid & 63]};
    }
    so[0] = v0;
    so[1] = v1;
}

// Item (a, b, z) of one mesh by one block; part holds the 2 nr Z slots
template <int FORM, bool K0>
__device__ __forceinline__ void s64_item(const SymCoef<double> &cf, const int32_t *__restrict__ tri,
                                         const double *__restrict__ stat, const double *__restrict__ tiles,
                                         const double *__restrict__ dyn, int T, int rt, int nr, int Z, int a, int b, int z,
                                         double *__restrict__ part, S64Lds &L)
{
    const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int ntile = (T + kS64Tile - 1) / kS64Tile;
    const int I0 = a * rt, I1 = min(ntile, I0 + rt);
    const int J0 = b * rt, J1 = min(ntile, J0 + rt);
    for (int I = I0; I < I1; ++I) {
        const double *tI = tiles + kTileRec * (size_t)I;
        const double c[3] = {tI[0], tI[1], tI[2]};
        S64Target t;
        int tv[3];
        {
            const int s = min(kS64Tile * I + lane, T - 1);
            const bool in = kS64Tile * I + lane < T;   // past the end: the last triangle with zero weights
            const double *ts = stat + (size_t)s * kStat, *td = dyn + (size_t)s * kDyn;
#pragma unroll
            for (int p = 0; p < 6; ++p) {
                t.x[p] = (ts[3 * p] - c[0]) * cf.s;
                t.y[p] = (ts[3 * p + 1] - c[1]) * cf.s;
                t.z[p] = (ts[3 * p + 2] - c[2]) * cf.s;
                t.b1[p] = in ? td[p] : 0.0;
                t.b2[p] = in ? td[6 + p] : 0.0;
                t.a1[p] = t.a2[p] = 0.0;
            }
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                t.n[k] = ts[18 + k];
                if (w == 0) {   // read after the barriers below
                    L.c.tcen[k][lane] = (ts[37 + k] - c[k]) * cf.s;
                    L.c.tcurl[k][lane] = in ? td[12 + k] : 0.0;
                }
                t.W[k] = 0.0;
                tv[k] = in ? tri[3 * s + k] : -1;
            }
            t.o = t.x[0] * t.n[0] + t.y[0] * t.n[1] + t.z[0] * t.n[2];
        }
        for (int J = a == b ? I : J0; J < J1; ++J) {
            const double *tJ = tiles + kTileRec * (size_t)J;
            // stage tile J: thread = (source, quarter of its record)
            {
                const int sj = min(kS64Tile * J + lane, T - 1);
                const bool in = kS64Tile * J + lane < T;
                const double *ss = stat + (size_t)sj * kStat, *sd = dyn + (size_t)sj * kDyn;
                if (w < 3) {
#pragma unroll
                    for (int k = 0; k < 2; ++k) {
                        const int q = 2 * w + k;
#pragma unroll
                        for (int m = 0; m < 3; ++m) L.c.y[q][m][lane] = (ss[3 * q + m] - c[m]) * cf.s;
                        const double b1 = in ? sd[q] : 0.0, b2 = in ? sd[6 + q] : 0.0;
                        L.c.w[q][0][lane] = cf.cK * b1;
                        L.c.w[q][1][lane] = cf.cV * b2;
                        L.c.w[q][2][lane] = cf.cT * (FORM == 0 ? b1 : b2);
                        L.c.w[q][3][lane] = FORM == 0 ? cf.cD * b2 : cf.kD * b1;
                    }
                } else {
                    double o = 0.0;
#pragma unroll
                    for (int k = 0; k < 3; ++k) {
                        L.c.n[k][lane] = ss[18 + k];
                        o = fma((ss[k] - c[k]) * cf.s, ss[18 + k], o);
                        L.c.cen[k][lane] = (ss[37 + k] - c[k]) * cf.s;
                        if (FORM >= 1) L.c.curl[k][lane] = in ? sd[12 + k] : 0.0;
                        L.c.id[k][lane] = in ? tri[3 * sj + k] : -1;
                    }
                    L.c.n[3][lane] = o;
                }
            }
            __syncthreads();
            // triangles that share a vertex are in tiles whose bounding spheres meet
            const double dx = tJ[0] - c[0], dy = tJ[1] - c[1], dz = tJ[2] - c[2], reach = 1.001 * (tI[3] + tJ[3]);
            const bool near = dx * dx + dy * dy + dz * dz < reach * reach;
            constexpr bool kLoc = FORM == 0 && !K0;   // the other forms have no registers for it (spills: 5.3 against 5.1 ms)
            const bool loc = kLoc && (tI[4] + tJ[4]) * cf.s < kExpNear;
            double acc1[6], acc2[6], accW[3] = {0.0, 0.0, 0.0};
#pragma unroll
            for (int q = 0; q < 6; ++q) acc1[q] = acc2[q] = 0.0;
            const int k0 = w + kS64Waves * z, dk = kS64Waves * Z;
            int k;
            if (near) k = s64_steps<FORM, K0, true, false>(cf, L.c, lane, k0, dk, I == J, tv, t, acc1, acc2, accW);
            else if (loc) k = s64_steps<FORM, K0, false, kLoc>(cf, L.c, lane, k0, dk, false, tv, t, acc1, acc2, accW);
            else k = s64_steps<FORM, K0, false, false>(cf, L.c, lane, k0, dk, false, tv, t, acc1, acc2, accW);
            const int j = (lane + k) & 63;
#pragma unroll
            for (int q = 0; q < 6; ++q) {
                L.out[w][q][j] = acc1[q];
                L.out[w][6 + q][j] = acc2[q];
            }
#pragma unroll
            for (int m = 0; m < 3; ++m) L.out[w][12 + m][j] = accW[m];
            L.out[w][15][j] = 0.0;
            __syncthreads();
            s64_flush(L, tid, kS64Tile * J, T, part + (size_t)((Z + z) * nr + a) * T * 16, I != I0);
        }
        __syncthreads();   // the last source flush is read
#pragma unroll
        for (int p = 0; p < 6; ++p) {
            L.out[w][p][lane] = t.a1[p];
            L.out[w][6 + p][lane] = t.a2[p];
        }
#pragma unroll
        for (int k = 0; k < 3; ++k) L.out[w][12 + k][lane] = t.W[k];
        L.out[w][15][lane] = 0.0;
        __syncthreads();
        s64_flush(L, tid, kS64Tile * I, T, part + (size_t)(z * nr + b) * T * 16, false);
        __syncthreads();   // and this one
    }
}

__device__ __forceinline__ int s64_next_item(int *__restrict__ next, S64Lds &L)
{
    __syncthreads();   // the previous item's number is read and its LDS consumed
    if (threadIdx.x == 0) L.item = atomicAdd(next, 1);
    __syncthreads();
    return __builtin_amdgcn_readfirstlane(L.item);
}

template <int FORM, bool K0>
__global__ __launch_bounds__(64 * kS64Waves, 2) void k_far_sym64(int T, int rt, int nr, int Z, SymCoef<double> cf,
                                                              const int32_t *__restrict__ tri,
                                                              const double *__restrict__ stat,
                                                              const double *__restrict__ tiles,
                                                              const double *__restrict__ dyn,
                                                              const int4 *__restrict__ items, int nitems,
                                                              int *__restrict__ next, double *__restrict__ part,
                                                              DevCtl ctl)
{
    __shared__ S64Lds lds;
    if (ctl_skip(ctl)) return;   // uniform: every wavefront leaves
    for (;;) {
        const int i = s64_next_item(next, lds);
        if (i >= nitems) return;
        const int4 it = items[i];
        s64_item<FORM, K0>(cf, tri, stat, tiles, dyn, T, rt, nr, Z, it.y, it.z, it.w, part, lds);
    }
}

template <int FORM, bool K0>
__global__ __launch_bounds__(64 * kS64Waves, 2) void k_far_sym64_batch(const FarReq<double> *__restrict__ reqs,
                                                                    const int4 *__restrict__ items, int nitems,
                                                                    int *__restrict__ next)
{
    __shared__ S64Lds lds;
    for (;;) {
        const int i = s64_next_item(next, lds);
        if (i >= nitems) return;
        const int4 it = items[i];
        const FarReq<double> &rq = reqs[it.x];
        if (rq.skip && *rq.skip) continue;
        s64_item<FORM, K0>(rq.sc, rq.tri, rq.stat64, rq.tiles, rq.dyn, rq.T, rq.rt, rq.nr, rq.nz, it.y, it.z, it.w, rq.part, lds);
    }
}

static const void *sym64_kernel(int form, bool k0)
{
    const void *k = nullptr;
#define SYM_ADDR(KF) k = reinterpret_cast<const void *>(&KF);
    SYM_PICK(k_far_sym64, form, k0, SYM_ADDR)
    return k;
}

static const void *sym64_batch_kernel(int form, bool k0)
{
    const void *k = nullptr;
    SYM_PICK(k_far_sym64_batch, form, k0, SYM_ADDR)
    return k;
}

int sym64_blocks(int nitems, int form, bool k0) { return resident_blocks(sym64_kernel(form, k0), 64 * kS64Waves, nitems); }
int sym64_batch_blocks(int form, bool k0, int n) { return resident_blocks(sym64_batch_kernel(form, k0), 64 * kS64Waves, n); }

void launch_far_sym64(DevMesh &d)
{
    SymCoef<double> cf;
    const int form = sym_coef(d, cf);
    const bool k0 = d.far_k0;
    const int nb = d.sym_blocks[sym_form_index(form)];
#define SYM_RUN(KF)                                                                                              \
    hipLaunchKernelGGL(KF, dim3(nb), dim3(64 * kS64Waves), 0, d.stream, d.hm.T, d.sym_rt, d.sym_nr, d.sym_nz, cf, d.tri,   \
                       d.stat64, d.sym_tiles, d.dyn64, d.sym_items, d.sym_nitems, d.sym_next, (double *)d.part,  \
                       d.ctl);
    SYM_PICK(k_far_sym64, form, k0, SYM_RUN)
    HIPCHECK(hipGetLastError());
}

void launch_far_sym64_batch(int form, bool k0, const void *reqs, const int4 *items, int n, int nblocks, int *next,
                            hipStream_t s)
{
    if (n == 0) return;
    launch_sym_reset(s, next);
#define SYM_RUNB(KF) \
    hipLaunchKernelGGL(KF, dim3(nblocks), dim3(64 * kS64Waves), 0, s, (const FarReq<double> *)reqs, items, n, next);
    SYM_PICK(k_far_sym64_batch, form, k0, SYM_RUNB)
    HIPCHECK(hipGetLastError());
}

}  // namespace pbm
