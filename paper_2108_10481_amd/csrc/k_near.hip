// Near field: Sauter-Schwab quadrature of every ordered triangle pair that
// shares a vertex (Numerical discretization; S. Sauter and C. Schwab, Boundary
// Element Methods, Springer 2011, sec. 5.2), assembly of the four near-field
// vertex blocks of the chosen formulation (mass terms included), and the
// block-diagonal preconditioner (Preconditioning, Algebraic preconditioners).
// Everything here is FP64 in every precision mode.
#include <mutex>
#include <vector>

#include "fp64.h"
#include "pbm_internal.h"

namespace pbm {

// Reference triangle {0 <= u2 <= u1 <= 1}, chi(u) = P0 + u1 (P1 - P0) + u2 (P2 - P1),
// barycentrics (1 - u1, u1 - u2, u2), surface element 2|T| du.  The unit
// hypercube (xi, a, b, c) is split into regions mapped onto the pair of
// reference triangles with Jacobians that cancel the 1/r singularity.
struct SSPoint { double u1, u2, v1, v2, jac; };

static SSPoint ss_map(int cas, int r, double xi, double a, double b, double c)
{
    SSPoint m;
    if (cas == 3) {          // identical triangles: 6 regions
        m.jac = xi * xi * xi * a * a * b;
        switch (r) {
        case 0: m.u1 = xi; m.u2 = xi * (1 - a + a * b); m.v1 = xi * (1 - a * b * c); m.v2 = xi * (1 - a); break;
        case 1: m.u1 = xi * (1 - a * b * c); m.u2 = xi * (1 - a); m.v1 = xi; m.v2 = xi * (1 - a + a * b); break;
        case 2: m.u1 = xi; m.u2 = xi * a * (1 - b + b * c); m.v1 = xi * (1 - a * b); m.v2 = xi * a * (1 - b); break;
        case 3: m.u1 = xi * (1 - a * b); m.u2 = xi * a * (1 - b); m.v1 = xi; m.v2 = xi * a * (1 - b + b * c); break;
        case 4: m.u1 = xi * (1 - a * b * c); m.u2 = xi * a * (1 - b * c); m.v1 = xi; m.v2 = xi * a * (1 - b); break;
        default: m.u1 = xi; m.u2 = xi * a * (1 - b); m.v1 = xi * (1 - a * b * c); m.v2 = xi * a * (1 - b * c); break;
        }
    } else if (cas == 2) {   // common edge P0-P1 (u2 = 0 on both): 5 regions
        m.jac = xi * xi * xi * a * a * (r == 0 ? 1.0 : b);
        switch (r) {
        case 0: m.u1 = xi; m.u2 = xi * a * c; m.v1 = xi * (1 - a * b); m.v2 = xi * a * (1 - b); break;
        case 1: m.u1 = xi; m.u2 = xi * a; m.v1 = xi * (1 - a * b * c); m.v2 = xi * a * b * (1 - c); break;
        case 2: m.u1 = xi * (1 - a * b); m.u2 = xi * a * (1 - b); m.v1 = xi; m.v2 = xi * a * b * c; break;
        case 3: m.u1 = xi * (1 - a * b * c); m.u2 = xi * a * b * (1 - c); m.v1 = xi; m.v2 = xi * a; break;
        default: m.u1 = xi * (1 - a * b * c); m.u2 = xi * a * (1 - b * c); m.v1 = xi; m.v2 = xi * a * b; break;
        }
    } else {                 // common vertex P0: 2 regions
        m.jac = xi * xi * xi * b;
        if (r == 0) { m.u1 = xi; m.u2 = xi * a; m.v1 = xi * b; m.v2 = xi * b * c; }
        else { m.u1 = xi * b; m.u2 = xi * b * c; m.v1 = xi; m.v2 = xi * a; }
    }
    return m;
}

// The rule's points, the same for every pair of a case: u1, u2, v1, v2, then the
// nine weights w lambda_k(u) mu_l(v) (Jacobian included), padded to 16 doubles
// (two 64-byte scalar loads).  Cases in the order identical, edge, vertex.
constexpr int kSSRec = 16;
constexpr int kMaxSS = 8;                          // singular_order
constexpr int kSSRegions[4] = {0, 2, 5, 6};        // by shared vertices
struct SSTable {
    const double *pts = nullptr;
    int first[4] = {}, count[4] = {};              // by shared vertices
};

// Device table of order n on the current device: built at its first use and kept
// until the process ends (13 n^4 records of 128 bytes, 426 KB at order 4)
static SSTable ss_table(int n)
{
    constexpr int kMaxDevices = 64;
    static std::mutex mu;
    static SSTable tab[kMaxDevices][kMaxSS + 1];
    int dev = -1;
    HIPCHECK(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) fail(PB_E_DEVICE, "device index out of range for the quadrature tables");
    std::lock_guard<std::mutex> lk(mu);
    SSTable &t = tab[dev][n];
    if (t.pts) return t;
    std::vector<double> x(n), w(n), rec;
    gauss_legendre01(n, x.data(), w.data());
    SSTable s;
    for (int cas = 3; cas >= 1; --cas) {
        s.first[cas] = (int)(rec.size() / kSSRec);
        for (int r = 0; r < kSSRegions[cas]; ++r)
            for (int i0 = 0; i0 < n; ++i0)
                for (int i1 = 0; i1 < n; ++i1)
                    for (int i2 = 0; i2 < n; ++i2)
                        for (int i3 = 0; i3 < n; ++i3) {
                            const SSPoint m = ss_map(cas, r, x[i0], x[i1], x[i2], x[i3]);
                            const double W = w[i0] * w[i1] * w[i2] * w[i3] * m.jac;
                            const double lx[3] = {1.0 - m.u1, m.u1 - m.u2, m.u2};
                            const double ly[3] = {1.0 - m.v1, m.v1 - m.v2, m.v2};
                            double q[kSSRec] = {m.u1, m.u2, m.v1, m.v2};
                            for (int k = 0; k < 3; ++k)
                                for (int l = 0; l < 3; ++l) q[4 + 3 * k + l] = W * lx[k] * ly[l];
                            rec.insert(rec.end(), q, q + kSSRec);
                        }
        s.count[cas] = (int)(rec.size() / kSSRec) - s.first[cas];
    }
    void *p = nullptr;
    HIPCHECK(hipMalloc(&p, sizeof(double) * rec.size()));
    const hipError_t e = hipMemcpy(p, rec.data(), sizeof(double) * rec.size(), hipMemcpyHostToDevice);
    if (e != hipSuccess) (void)hipFree(p);
    HIPCHECK(e);
    s.pts = (const double *)p;
    return t = s;
}

// Local vertex order: shared vertices first.  Identical: stored order.  Edge:
// the test triangle is rotated so the shared edge is (0,1) in its own cyclic
// order; the trial triangle lists the same two vertices in the same order
// then its free vertex.  Vertex: both rotated so the shared vertex is first.
// The stored (outward) normals are kept whatever the local order.
__device__ inline int ss_order(int t, int s, const int *tv, const int *sv, int *pt, int *ps)
{
    pt[0] = ps[0] = 0; pt[1] = ps[1] = 1; pt[2] = ps[2] = 2;
    if (t == s) return 3;
    int ns = 0, kt[3] = {0, 0, 0}, ks[3] = {0, 0, 0};
    for (int k = 0; k < 3; ++k)
        for (int l = 0; l < 3; ++l)
            if (tv[k] == sv[l]) { kt[ns] = k; ks[ns] = l; ++ns; }
    if (ns == 2) {
        int k0 = kt[0], k1 = kt[1];
        if ((k0 + 1) % 3 != k1) { int tmp = k0; k0 = k1; k1 = tmp; }
        pt[0] = k0; pt[1] = k1; pt[2] = 3 - k0 - k1;
        for (int l = 0; l < 3; ++l) {
            if (sv[l] == tv[k0]) ps[0] = l;
            if (sv[l] == tv[k1]) ps[1] = l;
        }
        ps[2] = 3 - ps[0] - ps[1];
    } else if (ns == 1) {
        for (int m = 0; m < 3; ++m) { pt[m] = (kt[0] + m) % 3; ps[m] = (ks[0] + m) % 3; }
    }
    return ns;
}

// An ordered pair (t, s): vertex ids in quadrature order and x - y = A + u1 e1 + u2 e2
// - v1 f1 - v2 f2 at the point (u, v)
struct SSPair {
    int p, t, s, pt[3], ps[3];
    double A[3], e1[3], e2[3], f1[3], f2[3], ns[3];
};
struct SSData {
    const int32_t *pair_t, *pair_s, *tri;
    const double *xyz, *geo;
    double kl, kappa;
    double *out;
};

__device__ __forceinline__ void ss_load(const SSData &D, int p, SSPair &q)
{
    q.p = p;
    q.t = D.pair_t[p];
    q.s = D.pair_s[p];
    int tv[3], sv[3];
    for (int k = 0; k < 3; ++k) { tv[k] = D.tri[3 * q.t + k]; sv[k] = D.tri[3 * q.s + k]; }
    (void)ss_order(q.t, q.s, tv, sv, q.pt, q.ps);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const double P0 = D.xyz[3 * tv[q.pt[0]] + c], P1 = D.xyz[3 * tv[q.pt[1]] + c], P2 = D.xyz[3 * tv[q.pt[2]] + c];
        const double Q0 = D.xyz[3 * sv[q.ps[0]] + c], Q1 = D.xyz[3 * sv[q.ps[1]] + c], Q2 = D.xyz[3 * sv[q.ps[2]] + c];
        q.A[c] = P0 - Q0;
        q.e1[c] = P1 - P0; q.e2[c] = P2 - P1;
        q.f1[c] = Q1 - Q0; q.f2[c] = Q2 - Q1;
        q.ns[c] = D.geo[(size_t)q.s * kGeo + 18 + c];
    }
}

// One point's record cur (13 values) into the sums of V (aL[0], aY[0]) and K.  RANGE
// 0: every kappa log2(e) r of a near pair is at most kExpSmall, 8 instead of 15
// instructions for its exponential; 2: some may pass 2^30, past which exp2neg_n's
// exponent wraps, and are cut off at 2000 (2^-2000 = 0).  Identical triangles (CASE
// 3) lie in one plane: d.n = 0, K = 0, only V is summed.
template <int CASE, int RANGE, int NK>
__device__ __forceinline__ void ss_add(const SSPair &q, const double (&cur)[13], double kl, double kappa, double (&aL)[NK][9],
                                       double (&aY)[NK][9])
{
    double d[3];
#pragma unroll
    for (int c = 0; c < 3; ++c)
        d[c] = fma(cur[0], q.e1[c], fma(cur[1], q.e2[c], fma(-cur[2], q.f1[c], fma(-cur[3], q.f2[c], q.A[c]))));
    const double r2[1] = {d[0] * d[0] + d[1] * d[1] + d[2] * d[2]};
    double ri[1], ek[1];
    rsqrt3_n<1>(r2, ri);
    ek[0] = kl * r2[0] * ri[0];
    if (RANGE == 2) ek[0] = fmin(ek[0], 2000.0);
    if (RANGE == 0) exp2small_n<1>(ek);
    else exp2neg_n<1>(ek);
    const double gL = ri[0], gY = ek[0] * ri[0];
    double fL = 0.0, fY = 0.0;
    if (CASE != 3) {
        const double dn = d[0] * q.ns[0] + d[1] * q.ns[1] + d[2] * q.ns[2];
        const double ri2 = gL * gL, ri3 = gL * ri2;
        fL = dn * ri3;
        fY = dn * (ek[0] * fma(kappa, ri2, ri3));
    }
#pragma unroll
    for (int v = 0; v < 9; ++v) {
        aL[0][v] = fma(cur[4 + v], gL, aL[0][v]);
        aY[0][v] = fma(cur[4 + v], gY, aY[0][v]);
        if (CASE != 3) {
            aL[NK - 1][v] = fma(cur[4 + v], fL, aL[NK - 1][v]);
            aY[NK - 1][v] = fma(cur[4 + v], fY, aY[NK - 1][v]);
        }
    }
}

// out[36 p + 4 (3 a + b) + op], op = V_L, K_L, V_Y, K_Y (the four values that one
// vertex pair's row needs lie together); a, b local vertex ids of t and s in stored
// order
template <int CASE, int NK>
__device__ __forceinline__ void ss_store(const SSData &D, const SSPair &q, const double (&aL)[NK][9], const double (&aY)[NK][9])
{
    const double scale = D.geo[(size_t)q.t * kGeo + 21] * D.geo[(size_t)q.s * kGeo + 21] / kPi;   // (2|t|)(2|s|) / (4 pi)
    double *o = D.out + (size_t)q.p * 36;
#pragma unroll
    for (int k = 0; k < 3; ++k)
#pragma unroll
        for (int l = 0; l < 3; ++l) {
            double4 v;
            v.x = aL[0][3 * k + l] * scale;
            v.y = CASE == 3 ? 0.0 : aL[NK - 1][3 * k + l] * scale;
            v.z = aY[0][3 * k + l] * scale;
            v.w = CASE == 3 ? 0.0 : aY[NK - 1][3 * k + l] * scale;
            *(double4 *)(o + 4 * (3 * q.pt[k] + q.ps[l])) = v;
        }
}

// One lane per ordered pair (t, s): the WAVES wavefronts of a block hold the same
// 64 pairs of one case (CASE shared vertices) and take a part of the rule's points
// each, which are then uniform across the wavefront: a point and its nine weights
// come through scalar loads and feed the vector unit as scalar operands, and the
// 36 sums need no reduction across lanes, only over the wavefronts (LDS).
// Bound: the FP64 vector rate, 75 instructions per point and pair (68 in RANGE 0; 39
// and 32 for identical triangles); with a group of lanes per pair (points, weights
// and basis formed by every lane, 36 butterfly reductions) it was about 130.
// Refresh of a 24500-triangle matrix-free handle (all of the near field): 1.67 ->
// 0.81 ms (0.71 with k_near_slots as it is below).
template <int CASE, int RANGE, int WAVES>
__device__ __forceinline__ void ss_pairs(const SSData &D, int first, int count, const int32_t *__restrict__ idx,
                                         const double *__restrict__ pts, int npts, double (*__restrict__ red)[18][64])
{
    const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int item = first + lane;
    const bool active = item < count;   // lanes past the end repeat the last pair and do not store
    SSPair q;
    ss_load(D, idx[active ? item : count - 1], q);
    constexpr int NK = CASE == 3 ? 1 : 2;   // V alone, or V and K, per kernel
    double aL[NK][9], aY[NK][9];
#pragma unroll
    for (int o = 0; o < NK; ++o)
#pragma unroll
        for (int v = 0; v < 9; ++v) aL[o][v] = aY[o][v] = 0.0;
    using CD = const __attribute__((address_space(4))) double *;
    const int i0 = (int)((long long)npts * w / WAVES), i1 = (int)((long long)npts * (w + 1) / WAVES);
    CD rec = (CD)(pts + (size_t)i0 * kSSRec);
    double cur[13];
#pragma unroll
    for (int k = 0; k < 13; ++k) cur[k] = rec[k];
    for (int i = i0; i < i1; ++i) {
        // the next point's record is loaded while this one is summed
        CD nxt = rec + (i + 1 < i1 ? kSSRec : 0);
        double nx[13];
#pragma unroll
        for (int k = 0; k < 13; ++k) nx[k] = nxt[k];
        rec = nxt;
        ss_add<CASE, RANGE, NK>(q, cur, D.kl, D.kappa, aL, aY);
#pragma unroll
        for (int k = 0; k < 13; ++k) cur[k] = nx[k];
    }
    // the wavefronts' sums, in order, onto the first wavefront's: Laplace, then Yukawa
    auto join = [&](double (&a)[NK][9]) {
        __syncthreads();
        if (w > 0) {
#pragma unroll
            for (int o = 0; o < NK; ++o)
#pragma unroll
                for (int v = 0; v < 9; ++v) red[w - 1][9 * o + v][lane] = a[o][v];
        }
        __syncthreads();
        if (w == 0) {
#pragma unroll
            for (int o = 0; o < NK; ++o)
#pragma unroll
                for (int v = 0; v < 9; ++v)
                    for (int u = 0; u < WAVES - 1; ++u) a[o][v] += red[u][9 * o + v][lane];
        }
    };
    join(aL);
    join(aY);
    if (w == 0 && active) ss_store<CASE, NK>(D, q, aL, aY);
}

// All pairs in one launch, blocks of 64 pairs of one case: identical, edge, then
// vertex pairs (fewest, with the most points, first)
struct SSRange { int first, count, blocks, npts; const double *pts; };
template <int RANGE, int WAVES>
__global__ __launch_bounds__(64 * WAVES) void k_near_ss(SSRange r3, SSRange r2, SSRange r1, const int32_t *__restrict__ idx,
                                                        SSData D)
{
    __shared__ double red[WAVES - 1][18][64];
    int b = blockIdx.x;
    if (b < r3.blocks) {
        ss_pairs<3, RANGE, WAVES>(D, 64 * b, r3.count, idx + r3.first, r3.pts, r3.npts, red);
        return;
    }
    b -= r3.blocks;
    if (b < r2.blocks) {
        ss_pairs<2, RANGE, WAVES>(D, 64 * b, r2.count, idx + r2.first, r2.pts, r2.npts, red);
        return;
    }
    b -= r2.blocks;
    ss_pairs<1, RANGE, WAVES>(D, 64 * b, r1.count, idx + r1.first, r1.pts, r1.npts, red);
}

// One wavefront per ordered pair, a lane per point, and a reduction over the lanes:
// where the pairs are too few to give every SIMD blocks of 64, a pair's chain of
// points is cut into 64.  The block's wavefronts have pairs of one case and share
// the records of 64 points in LDS (read by each from the caches they took 2.5 times
// the time of the arithmetic).
constexpr int kSSWaves = 4;    // sk, si cover 13 (of 16) values of 64 points with 256 threads
constexpr int kSSRow = 68;     // rows 8 banks apart
template <int CASE, int RANGE>
__device__ __forceinline__ void ss_pair_wave(const SSData &D, int first, int count, const int32_t *__restrict__ idx,
                                             const double *__restrict__ pts, int npts, double (*__restrict__ L)[kSSRow])
{
    const int tid = threadIdx.x, lane = tid & 63;
    const int item = first + __builtin_amdgcn_readfirstlane(tid >> 6);
    SSPair q;
    ss_load(D, idx[min(item, count - 1)], q);   // past the end: the last pair, not stored
    constexpr int NK = CASE == 3 ? 1 : 2;
    double aL[NK][9], aY[NK][9];
#pragma unroll
    for (int o = 0; o < NK; ++o)
#pragma unroll
        for (int v = 0; v < 9; ++v) aL[o][v] = aY[o][v] = 0.0;
    const int si = tid >> 2, sk = 4 * (tid & 3);   // staging: a quarter of point si's record
    for (int i0 = 0; i0 < npts; i0 += 64) {
        const double2 *rec = (const double2 *)(pts + (size_t)min(i0 + si, npts - 1) * kSSRec + sk);
        const double2 u = rec[0], v = rec[1];
        __syncthreads();   // the previous points are read
        L[sk][si] = u.x;
        if (sk < 12) {
            L[sk + 1][si] = u.y;
            L[sk + 2][si] = v.x;
            L[sk + 3][si] = v.y;
        }
        __syncthreads();
        if (i0 + lane < npts) {
            double cur[13];
#pragma unroll
            for (int k = 0; k < 13; ++k) cur[k] = L[k][lane];
            ss_add<CASE, RANGE, NK>(q, cur, D.kl, D.kappa, aL, aY);
        }
    }
#pragma unroll
    for (int o = 0; o < NK; ++o)
#pragma unroll
        for (int v = 0; v < 9; ++v)
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) {
                aL[o][v] += __shfl_xor(aL[o][v], off);
                aY[o][v] += __shfl_xor(aY[o][v], off);
            }
    if (lane == 0 && item < count) ss_store<CASE, NK>(D, q, aL, aY);
}

// blocks of kSSWaves pairs of one case
template <int RANGE>
__global__ __launch_bounds__(64 * kSSWaves) void k_near_ss_wave(SSRange r3, SSRange r2, SSRange r1,
                                                                const int32_t *__restrict__ idx, SSData D)
{
    __shared__ double L[13][kSSRow];
    int b = blockIdx.x;
    if (b < r3.blocks) {
        ss_pair_wave<3, RANGE>(D, kSSWaves * b, r3.count, idx + r3.first, r3.pts, r3.npts, L);
        return;
    }
    b -= r3.blocks;
    if (b < r2.blocks) {
        ss_pair_wave<2, RANGE>(D, kSSWaves * b, r2.count, idx + r2.first, r2.pts, r2.npts, L);
        return;
    }
    b -= r2.blocks;
    ss_pair_wave<1, RANGE>(D, kSSWaves * b, r1.count, idx + r1.first, r1.pts, r1.npts, L);
}

// Pair indices 0..n-1 grouped by the number of shared vertices: identical,
// then edge, then vertex pairs; count[c] pairs share c vertices.
void ss_group(const std::vector<int32_t> &tri, int n, const int32_t *t, const int32_t *s, std::vector<int32_t> &idx,
              int count[4])
{
    std::vector<int32_t> by[4];
    for (int i = 0; i < n; ++i) {
        int c = 0;
        for (int a = 0; a < 3; ++a)
            for (int b = 0; b < 3; ++b) c += tri[3 * t[i] + a] == tri[3 * s[i] + b];
        if (t[i] == s[i]) c = 3;
        by[std::min(c, 3)].push_back(i);
    }
    idx.clear();
    for (int c = 3; c >= 1; --c) idx.insert(idx.end(), by[c].begin(), by[c].end());
    for (int c = 0; c < 4; ++c) count[c] = (int)by[c].size();
    if (count[0]) fail(PB_E_INVALID_ARG, "pair does not share a vertex");
}

static void launch_ss(DevMesh &d, const int count[4], const int32_t *idx, const int32_t *pt, const int32_t *ps,
                      double *out, int order)
{
    if (count[1] + count[2] + count[3] == 0) return;
    if (order < 1 || order > kMaxSS) fail(PB_E_INVALID_ARG, "singular_order must be in [1, 8]");
    const SSTable tab = ss_table(order);
    SSRange r[4];
    int blocks = 0, first = 0;
    for (int c = 3; c >= 1; --c) {
        r[c] = SSRange{first, count[c], (count[c] + 63) / 64, tab.count[c], tab.pts + (size_t)tab.first[c] * kSSRec};
        first += count[c];
        blocks += r[c].blocks;
    }
    const double kl = d.prm.kappa * 1.4426950408889634;
    // a near pair's points are at most two longest edges apart
    const double reach = 2.0 * d.max_edge * kl;
    const int range = reach <= kExpSmall ? 0 : reach < 1073741824.0 ? 1 : 2;
    const SSData D{pt, ps, d.tri, d.xyz, d.geo, kl, d.prm.kappa, out};
#define SS_PICK(KERNEL0, KERNEL1, KERNEL2, grid, threads)                                                                \
    if (range == 0) hipLaunchKernelGGL((KERNEL0), dim3(grid), dim3(threads), 0, d.stream, r[3], r[2], r[1], idx, D);     \
    else if (range == 1) hipLaunchKernelGGL((KERNEL1), dim3(grid), dim3(threads), 0, d.stream, r[3], r[2], r[1], idx, D); \
    else hipLaunchKernelGGL((KERNEL2), dim3(grid), dim3(threads), 0, d.stream, r[3], r[2], r[1], idx, D)
    // A wavefront per pair costs 4.5 ns a pair for its reduction and about 10 ps a pair
    // and n^4 point; blocks of 64 pairs a chain of 0.29 us per n^4 until they fill the
    // device.  The lines meet at 28000 n^4 / (437 + n^4) pairs; below 20000 a wavefront
    // per pair was the faster one everywhere.  Refresh in us, wavefront / block, at
    // 980, 4100, 9300 and 16580 pairs (80 .. 1280 triangles): n = 2 46 / 47, 68 / 53;
    // 4 56 / 100, 83 / 108, 121 / 111; 6 101 / 326, 144 / 336, 245 / 350, 398 / 390;
    // 8 272 / 1221, 302 / 1265, 565 / 1264, 945 / 1233 (with a group of lanes per pair
    // n = 8 took 708, 715, 995, 1289).  Eight wavefronts share a block's pairs while
    // four leave compute units idle: n = 6, 25940 pairs in 406 blocks 435 / 655 us,
    // 50900 in 796 779 / 756; n = 3 82 / 79 in 406.
    const double n4 = (double)order * order * order * order;
    if (first < 20000.0 * n4 / (437.0 + n4)) {
        blocks = 0;
        for (int c = 3; c >= 1; --c) blocks += r[c].blocks = (count[c] + kSSWaves - 1) / kSSWaves;
        SS_PICK(k_near_ss_wave<0>, k_near_ss_wave<1>, k_near_ss_wave<2>, blocks, 64 * kSSWaves);
    } else if (blocks < (order >= 4 ? 512 : 256)) {
        SS_PICK((k_near_ss<0, 8>), (k_near_ss<1, 8>), (k_near_ss<2, 8>), blocks, 512);
    } else {
        SS_PICK((k_near_ss<0, 4>), (k_near_ss<1, 4>), (k_near_ss<2, 4>), blocks, 256);
    }
#undef SS_PICK
    HIPCHECK(hipGetLastError());
}

void launch_near_field(DevMesh &d)
{
    launch_ss(d, d.ss_count, d.ss_idx, d.pair_t, d.pair_s, d.pairblk, d.opt.singular_order);
}

void launch_pair_blocks_subset(DevMesh &d, int n, const int32_t *t_sorted, const int32_t *s_sorted,
                               const int32_t *idx, const int count[4], double *out)
{
    (void)n;
    launch_ss(d, count, idx, t_sorted, s_sorted, out, d.opt.singular_order);
}

// Near-field vertex blocks (mass terms included) of the chosen formulation.
// One thread per nonzero slot (i, j) sums, in the fixed order row i visits
// them, the contributions of the near pairs (t containing i as local vertex k,
// s containing j as local vertex l); the slot is owned by one thread, so there
// is no atomic and the result is deterministic.
struct NearCoef {
    double kappa;
    FormCoef f;                // the formulation's block coefficients
};

// per pair: sum of its 3 x 3 V_L and V_Y entries (the hypersingular curl part)
__global__ void k_pair_sums(int64_t npair, const double *__restrict__ blk, double *__restrict__ sums)
{
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= npair) return;
    const double *B = blk + p * 36;
    double SL = 0.0, SY = 0.0;
    for (int a = 0; a < 9; ++a) { SL += B[4 * a]; SY += B[4 * a + 2]; }
    sums[2 * p] = SL;
    sums[2 * p + 1] = SY;
}

// The values of one nonzero (i, j): its contributions in slot order.  Bound: the
// caches, a chain of loads (code, pair, block) per contribution at scattered
// pairs.  The four values of a contribution lie together (with one 3 x 3 block per
// operator each was in a cache line of its own), and kSlotBatch contributions are
// loaded before the first is added, in their order.  24500 triangles, direct: one
// by one 167 us, in batches 116, with the values together 66; 10580, Juffer: 128,
// 103, 73 us.
constexpr int kSlotBatch = 4;
template <int FAMILY>
__global__ __launch_bounds__(256) void k_near_slots(int64_t nnz, NearCoef cf, const int32_t *__restrict__ slot_ptr,
                                                    const uint32_t *__restrict__ slot_code,
                                                    const int32_t *__restrict__ pair_t, const int32_t *__restrict__ pair_s,
                                                    const int32_t *__restrict__ pair_rev, const double *__restrict__ geo,
                                                    const double *__restrict__ blk, const double *__restrict__ sums,
                                                    double *__restrict__ N, double *__restrict__ Mval)
{
    const int64_t slot = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (slot >= nnz) return;
    const FormCoef &f = cf.f;
    double n11 = 0.0, n12 = 0.0, n21 = 0.0, n22 = 0.0, mass = 0.0;
    const int c1 = slot_ptr[slot + 1];
    for (int c0 = slot_ptr[slot]; c0 < c1; c0 += kSlotBatch) {
        uint32_t code[kSlotBatch];
        int t[kSlotBatch], s[kSlotBatch], rev[kSlotBatch];
        double4 q[kSlotBatch];   // V_L, K_L, V_Y, K_Y
        double dL[kSlotBatch], dY[kSlotBatch], tL[kSlotBatch], tY[kSlotBatch];
#pragma unroll
        for (int u = 0; u < kSlotBatch; ++u) code[u] = slot_code[min(c0 + u, c1 - 1)];   // the last again past the end
#pragma unroll
        for (int u = 0; u < kSlotBatch; ++u) {
            const int p = (int)(code[u] >> 4), kl = 3 * (int)((code[u] >> 2) & 3) + (int)(code[u] & 3);
            t[u] = pair_t[p];
            s[u] = pair_s[p];
            if (FAMILY != 0) rev[u] = pair_rev[p];
            q[u] = *(const double4 *)(blk + (size_t)p * 36 + 4 * kl);
        }
        if (FAMILY != 0) {   // row 2: D and T (Neumann trace equations)
#pragma unroll
            for (int u = 0; u < kSlotBatch; ++u) {
                const int p = (int)(code[u] >> 4), k = (code[u] >> 2) & 3, l = code[u] & 3;
                const double *gt = geo + (size_t)t[u] * kGeo, *gs = geo + (size_t)s[u] * kGeo;
                const double *R = blk + (size_t)rev[u] * 36 + 4 * (3 * l + k);
                const double nn = gt[18] * gs[18] + gt[19] * gs[19] + gt[20] * gs[20];
                const double cc = gt[22 + 3 * k] * gs[22 + 3 * l] + gt[23 + 3 * k] * gs[23 + 3 * l] +
                                  gt[24 + 3 * k] * gs[24 + 3 * l];
                // D: curl_k . curl_l V + kappa^2 (n_t . n_s) V, by parts; T = K^T
                dL[u] = cc * sums[2 * (size_t)p];
                dY[u] = cc * sums[2 * (size_t)p + 1] + cf.kappa * cf.kappa * nn * q[u].z;
                tL[u] = R[1];
                tY[u] = R[3];
            }
        }
#pragma unroll
        for (int u = 0; u < kSlotBatch; ++u) {
            if (c0 + u >= c1) break;
            const int k = (code[u] >> 2) & 3, l = code[u] & 3;
            const double mss = (s[u] == t[u]) ? geo[(size_t)t[u] * kGeo + 21] / 12.0 * (k == l ? 2.0 : 1.0) : 0.0;
            mass += mss;
            // row 1: K and V (Dirichlet trace equations)
            n11 += f.mass[0][0] * mss + f.aL[0][0] * q[u].y + f.aY[0][0] * q[u].w;
            n12 += f.mass[0][1] * mss + f.aL[0][1] * q[u].x + f.aY[0][1] * q[u].z;
            if (FAMILY == 0) {
                n21 += f.mass[1][0] * mss + f.aL[1][0] * q[u].y + f.aY[1][0] * q[u].w;
                n22 += f.mass[1][1] * mss + f.aL[1][1] * q[u].x + f.aY[1][1] * q[u].z;
            } else {
                n21 += f.mass[1][0] * mss + f.aL[1][0] * dL[u] + f.aY[1][0] * dY[u];
                n22 += f.mass[1][1] * mss + f.aL[1][1] * tL[u] + f.aY[1][1] * tY[u];
            }
        }
    }
    N[slot] = n11;
    N[nnz + slot] = n12;
    N[2 * nnz + slot] = n21;
    N[3 * nnz + slot] = n22;
    if (Mval) Mval[slot] = mass;
}

// per-vertex analytic inverse of [[A11_ii, A12_ii], [A21_ii, A22_ii]]; every
// diagonal entry comes from pairs sharing vertex i, i.e. from the near field.
__global__ void k_block_diag(int V, int enabled, const int32_t *__restrict__ diag, const double *__restrict__ N,
                             int64_t nnz, double *__restrict__ pinv)
{
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= V) return;
    double *o = pinv + 4 * (size_t)i;
    if (!enabled) { o[0] = 1.0; o[1] = 0.0; o[2] = 0.0; o[3] = 1.0; return; }
    const int sl = diag[i];
    const double a = N[sl], b = N[nnz + sl], c = N[2 * nnz + sl], e = N[3 * nnz + sl];
    const double det = a * e - b * c;
    o[0] = e / det; o[1] = -b / det; o[2] = -c / det; o[3] = a / det;
}

// ------------------------------------------------ mass preconditioners
// blockdiag(aM, bM)^-1 (Eqs. prec:mass, prec:mass:scaled), M the P1 mass
// matrix.  M^-1 is applied as a fixed-degree Chebyshev iteration on the
// Jacobi-scaled mass matrix D^-1 M (Y. Saad, Iterative Methods for Sparse
// Linear Systems, 2nd ed., sec. 12.3): for P1 triangles every element's
// generalised eigenvalues against its diagonal are 2, 1/2, 1/2, so the
// spectrum of D^-1 M lies in [1/2, 2] on any mesh (element-by-element bound)
// and each step reduces the error by 1/3 at least.  kChebSteps steps give a
// fixed linear operator within 2 (1/3)^20 = 6e-10 of M^-1; no reductions, so
// it is capturable like every other part of an iteration.
constexpr int kChebSteps = 20;
constexpr double kChebTheta = 1.25, kChebDelta = 0.75;   // centre and half-width of [1/2, 2]

__global__ void k_mass_diag(int V, const int32_t *__restrict__ diag, const double *__restrict__ Mval,
                            double *__restrict__ Mdinv)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < V) Mdinv[i] = 1.0 / Mval[diag[i]];
}

// systems s < nvec of 2V entries (both halves use M); x = 0, r = in, d = D^-1 r / theta
__global__ void k_cheb_init(int V, const double *__restrict__ Mdinv, const double *__restrict__ in,
                            double *__restrict__ x, double *__restrict__ r, double *__restrict__ dv, DevCtl ctl)
{
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= 2 * V || ctl_skip(ctl)) return;
    const size_t o = (size_t)blockIdx.y * 2 * V + e;
    const int i = e < V ? e : e - V;
    const double v = in[o];
    x[o] = 0.0;
    r[o] = v;
    dv[o] = v * Mdinv[i] * (1.0 / kChebTheta);
}

// x += d; r -= M d; d' = c1 d + c2 D^-1 r
__global__ void k_cheb_step(int V, const int32_t *__restrict__ row_ptr, const int32_t *__restrict__ col,
                            const double *__restrict__ Mval, const double *__restrict__ Mdinv, double c1, double c2,
                            double *__restrict__ x, double *__restrict__ r, const double *__restrict__ dv,
                            double *__restrict__ dn, DevCtl ctl)
{
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= 2 * V || ctl_skip(ctl)) return;
    const size_t base = (size_t)blockIdx.y * 2 * V + (e < V ? 0 : V);
    const int i = e < V ? e : e - V;
    const size_t o = base + i;
    double md = 0.0;
    for (int sl = row_ptr[i]; sl < row_ptr[i + 1]; ++sl) md += Mval[sl] * dv[base + col[sl]];
    const double rv = r[o] - md;
    x[o] += dv[o];
    r[o] = rv;
    dn[o] = c1 * dv[o] + c2 * Mdinv[i] * rv;
}

// out = (x + d) scaled by 1/a (first half) and 1/b (second half)
__global__ void k_cheb_final(int V, double sa, double sb, const double *__restrict__ x, const double *__restrict__ dv,
                             double *__restrict__ out, DevCtl ctl)
{
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= 2 * V || ctl_skip(ctl)) return;
    const size_t o = (size_t)blockIdx.y * 2 * V + e;
    out[o + ctl_off(ctl)] = (x[o] + dv[o]) * (e < V ? sa : sb);
}

void mass_precond(DevMesh &d, int nvec, const double *in, double *out, const DevCtl &ctl)
{
    double sa = 1.0, sb = 1.0;
    if (d.prm.preconditioner == PB_SCALED_MASS) {
        sa = 1.0 / (1.0 + d.prm.eps_out / d.prm.eps_in);
        sb = 1.0 / (1.0 + d.prm.eps_in / d.prm.eps_out);
    }
    mass_precond(d, nvec, in, out, ctl, sa, sb);
}

void mass_precond(DevMesh &d, int nvec, const double *in, double *out, const DevCtl &ctl, double sa, double sb)
{
    const int V = d.hm.V;
    if (nvec < 1 || nvec > kMassBatch) fail(PB_E_INVALID_ARG, "mass preconditioner batch size");
    const size_t n = 2 * (size_t)V * kMassBatch;
    double *x = d.cheb, *r = d.cheb + n, *dv[2] = {d.cheb + 2 * n, d.cheb + 3 * n};
    const dim3 g((unsigned)((2 * V + 255) / 256), (unsigned)nvec), b(256);
    hipLaunchKernelGGL(k_cheb_init, g, b, 0, d.stream, V, d.Mdinv, in, x, r, dv[0], ctl);
    const double s1 = kChebTheta / kChebDelta;
    double rho = 1.0 / s1;
    int cur = 0;
    for (int k = 1; k < kChebSteps; ++k, cur ^= 1) {
        const double rn = 1.0 / (2.0 * s1 - rho);
        hipLaunchKernelGGL(k_cheb_step, g, b, 0, d.stream, V, d.row_ptr, d.col, d.Mval, d.Mdinv, rn * rho,
                           2.0 * rn / kChebDelta, x, r, dv[cur], dv[cur ^ 1], ctl);
        rho = rn;
    }
    hipLaunchKernelGGL(k_cheb_final, g, b, 0, d.stream, V, sa, sb, x, dv[cur], out, ctl);
    HIPCHECK(hipGetLastError());
}

void launch_near_values(DevMesh &d, const FormCoef &f, const double *blk, const double *sums, double *N,
                        double *Mval)
{
    NearCoef cf;
    cf.kappa = d.prm.kappa;
    cf.f = f;
    const int64_t nnz = d.nnz();
    const dim3 g((unsigned)((nnz + 255) / 256)), b(256);
    if (f.family == 0)
        hipLaunchKernelGGL(k_near_slots<0>, g, b, 0, d.stream, nnz, cf, d.slot_ptr, d.slot_code, d.pair_t, d.pair_s,
                           d.pair_rev, d.geo, blk, sums, N, Mval);
    else
        hipLaunchKernelGGL(k_near_slots<1>, g, b, 0, d.stream, nnz, cf, d.slot_ptr, d.slot_code, d.pair_t, d.pair_s,
                           d.pair_rev, d.geo, blk, sums, N, Mval);
    HIPCHECK(hipGetLastError());
}

void launch_near_field_fast(DevMesh &d)
{
    launch_ss(d, d.ss_count, d.ss_idx, d.pair_t, d.pair_s, d.pairblkP, calderon_fast_order(d.opt));
    const int64_t np = d.npair();
    hipLaunchKernelGGL(k_pair_sums, dim3((unsigned)((np + 255) / 256)), dim3(256), 0, d.stream, np, d.pairblkP,
                       d.pair_sumsP);
    HIPCHECK(hipGetLastError());
}

// near-field values of the formulation (and of a Calderon preconditioner's
// operator P when it is not A), mass matrix, block-diagonal preconditioner
void launch_near_assemble(DevMesh &d)
{
    const int V = d.hm.V;
    const int64_t np = d.npair();
    if (d.fm.family == 1)
        hipLaunchKernelGGL(k_pair_sums, dim3((unsigned)((np + 255) / 256)), dim3(256), 0, d.stream, np, d.pairblk,
                           d.pair_sums);
    launch_near_values(d, d.fm, d.pairblk, d.pair_sums, d.N, d.Mval);
    if (d.NP) {
        if (d.pairblkP) launch_near_values(d, d.fmP, d.pairblkP, d.pair_sumsP, d.NP, nullptr);
        else launch_near_values(d, d.fmP, d.pairblk, d.pair_sums, d.NP, nullptr);
    }
    if (d.Mval)
        hipLaunchKernelGGL(k_mass_diag, dim3((V + 255) / 256), dim3(256), 0, d.stream, V, d.diag_slot, d.Mval,
                           d.Mdinv);
    hipLaunchKernelGGL(k_block_diag, dim3((V + 255) / 256), dim3(256), 0, d.stream, V,
                       d.prm.preconditioner == PB_BLOCK_DIAG ? 1 : 0, d.diag_slot, d.N, d.nnz(), d.pinv);
    HIPCHECK(hipGetLastError());
}

}  // namespace pbm
