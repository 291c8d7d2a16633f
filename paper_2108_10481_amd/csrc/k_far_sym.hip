// Far field, matrix-free, FP32, with every unordered triangle pair evaluated
// once (the kernel values G(x, y) = G(y, x) and the kernel factors of the
// four operators serve both (target t <- source s) and (s <- t); Numerical
// discretization: regular quadrature of the pairs sharing no vertex).
//
// Work: tiles of 64 Morton-consecutive triangles, tile ranges of `rt` tiles;
// an item (a, b), a <= b, is the pairs of triangles of range a x range b
// (I <= J when a == b) and is done by one block of four wavefronts.  For a tile
// pair (I, J) wavefront w holds the 16 target triangles 64 I + 16 w + r and
// walks the 64 sources of J in four groups of 16 columns: lane l has the column
// l mod 16 and the rows 4 (l / 16) + v, v = 0..3, the result layout of
// v_mfma_f32_16x16x4, for every one of the 36 point pairs.
//
// The squared distances of a 16 x 16 block of point pairs are one matrix
// instruction: r^2 = |X|^2 - 2 X.Y + |Y|^2 is (X, 1).(-2Y, |Y|^2) with |X|^2 as
// the accumulator's start, which takes the six vector instructions of the
// subtracted form off the VALU, the unit that bounds this kernel; so are the
// normal components d.n_s = X.n_s - O_s and d.n_t = O_t - Y.n_t (O: a
// triangle's plane offset; the points of a flat triangle lie in its plane).
// The points enter relative to the centre of tile J, subtracted in FP64 and then
// rounded, so their own rounding is that of a tile's size and not of the mesh's;
// the terms that cancel cost at most 81 roundings of r^2 (kSymApart, far.h).  Tile
// pairs that are not apart take the subtracted form (NEAR), and only they can hold
// pairs that share a vertex.
//
// Coordinates (points and the plane offsets) are used scaled by s = kappa
// log2(e), with the coefficients of sym_coef: then exp(-kappa r) = exp2(-r')
// with r' = r2' / sqrt(r2') and no multiply for the argument.  Unscreened
// meshes (far_k0: K0) keep their coordinates and skip the exponential:
// e = 1, so the Yukawa kernels are the Laplace ones.
//
// Bound: VALU issue.  A point pair of the direct form costs 6 instructions for
// the kernel values, two transcendentals and 8 fused multiply-adds into the sums
// (16.3 executed with everything outside, by counters), the issue slots are 91%
// taken.  Measured per product, before (a lane per target triangle, the source
// sums rotating through the wavefront, r^2 subtracted on the VALU) and now:
// 81920 triangles direct 80.4 -> 69.5 ms, Juffer 108 -> 86 ms; 20480 triangles
// Juffer 6.97 -> 5.98 ms; against the FP64 operator at 20480 triangles the error
// went from 1.2e-8 / 5.5e-8 (direct / Juffer) to 0.6e-8 / 0.7e-8, the input
// rounding of global coordinates being gone; on spheres of 20480 triangles graded
// towards a pole, edges 1 : 24, 1 : 240, 1 : 1900, the largest error of an entry went
// from 2.5e-6, 8.2e-6, 4.0e-5 to 3.4e-7, 7.0e-7, 5.4e-6 (direct).  Three wavefronts per SIMD (168
// registers, spilling) gained 3% on the direct form at 81920 triangles, lost 2%
// at 20480 and 10% on Juffer.
//
// Output: per triangle, one 16-value partial (6 + 6 point sums, 3 curl sums)
// per target-side item (slot b, the source range) and one per source-side
// item (slot nr + a, the target range): every slot is written by exactly one
// item, so no atomics and a fixed summation order.  k_far_sym_finish adds a
// triangle's slots in FP64 (nr + 1 for each part of the items) and projects them as
// k_far_finish does.
#include <algorithm>
#include <map>
#include <mutex>

#include "far.h"

namespace pbm {

constexpr int kSymWaves = 4;   // wavefronts per block, 16 rows of the target tile each
// LDS of one block: the columns (sources of tile J) and per wavefront the rows
// (its 16 targets), relative to tile J's centre
struct SymCols {
    f32x4 bq[6][64];      // (-2 Y_q, |Y_q|^2)
    f32x4 bn[64];         // (n_s, -O_s)
    f32x4 w[6][64];       // the source point's four weights (sym_cols)
    f32x4 curl[64];       // C_s
    int id[3][64];        // vertex ids (NEAR)
};
struct SymRows {
    float x2[6][16];      // |X_p|^2
    float x[6][3][16];    // X_p (NEAR)
    float o[16];          // O_t
    float d[16][16];      // the dynamic record: b1 6, b2 6, C 3
};
struct SymLds {
    SymCols c;
    SymRows r[kSymWaves];
    f32x4 out[kSymWaves][64][4];   // source-side sums of each wavefront's rows
    int item;
};

// sum over the 16 lanes of a row, in every lane of it
template <int CTRL>
__device__ __forceinline__ float dpp_add(float x)
{
    return x + __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), CTRL, 0xf, 0xf, true));
}
__device__ __forceinline__ float row_sum(float x)
{
    return dpp_add<0x121>(dpp_add<0x122>(dpp_add<0x124>(dpp_add<0x128>(x))));   // row_ror 8, 4, 2, 1
}

// One wavefront's 16 targets against one group of 16 sources (columns col0..):
// adds to its targets' sums a1, a2, W and returns the sources' sums over its rows
// (value m of column l mod 16 in row m / 4's component m mod 4).
//   A[p] = (X_p, 1), A2 = (n_t / 2, 0): the matrix operands of the targets
//   live[v] (NEAR): the pair of row v and the lane's column is summed here
// FORM 0 (direct): Laplace row kL K_L + vL V_L, Yukawa row kY K_Y + vY V_Y with
// R3 = r^-3, E = e (r^-3 + kappa r^-2): the double-layer sums of target point p
// over the source points (P, Q) take d.n_s once per triangle pair, those of
// source point q over the target points (S1, S2) d.n_t once per source point.
// FORM 1, 3, 4: row 1 = K and V, row 2 = T and D, each operator's two kernels
// joined in one value per point pair: L + b Y with the factor a taken out (FORM
// 1), Y alone (FORM 3: no Laplace term), a L + b Y (FORM 4: some operator
// without a Laplace term).  T's normal factors are per point and go with the
// weights; its target side carries d.n_t b2 per source point, its source side
// d.n_s b2_t per target point (wt).
template <int FORM, bool K0, bool NEAR>
__device__ __forceinline__ void sym_block(const SymCoef<float> &cf, const SymCols &C, const SymRows &R, int col0, int lane,
                                          const float (&A)[6], float A2, const bool (&live)[4], f32x4 (&a1)[6],
                                          f32x4 (&a2)[6], f32x4 (&W)[3], f32x4 &src)
{
    const int lc = col0 + (lane & 15), g = lane >> 4, r0 = 4 * g;
    const f32x4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
    const float bn = ((const float *)&C.bn[lc])[g];
    f32x4 P[6], Q[6];   // FORM 0: Q the Yukawa double layer; else Q = d.n_s b2_t
    f32x4 gs = zero, nn = zero;
#pragma unroll
    for (int p = 0; p < 6; ++p) P[p] = Q[p] = zero;
    if (FORM >= 1) {
        nn = 2.0f * mfma4(A2, bn, zero);   // n_t . n_s
#pragma unroll
        for (int p = 0; p < 6; ++p) Q[p] = mfma4(A[p], bn, zero) * *(const f32x4 *)&R.d[6 + p][r0];
    }
    float acc[16];
#pragma unroll
    for (int q = 0; q < 6; ++q) {
        const float b = ((const float *)&C.bq[q][lc])[g];
        const f32x4 w = C.w[q][lc];
        const f32x4 dnt = mfma4(A2, b, *(const f32x4 *)&R.o[r0]);
        f32x4 yq = zero;
        if (NEAR) yq = C.bq[q][lc];
        f32x4 S1 = zero, S2 = zero;
        f32x4 tq = zero, nb = zero;
        if (FORM >= 1) {
            tq = dnt * w[2];
            nb = nn * w[3];
        }
        float s1 = 0.0f, s2 = 0.0f;
#pragma unroll
        for (int p = 0; p < 6; ++p) {
            f32x4 r2;
            if (NEAR) {
                const f32x4 xx = *(const f32x4 *)&R.x[p][0][r0], xy = *(const f32x4 *)&R.x[p][1][r0],
                            xz = *(const f32x4 *)&R.x[p][2][r0];
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const float dx = fmaf(0.5f, yq[0], xx[v]), dy = fmaf(0.5f, yq[1], xy[v]),
                                dz = fmaf(0.5f, yq[2], xz[v]);
                    r2[v] = dx * dx + dy * dy + dz * dz;
                }
            } else {
                r2 = mfma4(A[p], b, *(const f32x4 *)&R.x2[p][r0]);
            }
            const f32x4 t1 = *(const f32x4 *)&R.d[p][r0], t2 = *(const f32x4 *)&R.d[6 + p][r0];
            const float ww = float(rule_w(p) * rule_w(q));
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                float ri = rsqrt_r(r2[v]);
                if (NEAR) ri = live[v] ? ri : 0.0f;   // every kernel value of the pair is then zero
                const float ri2 = ri * ri, R3 = ri * ri2;
                const float e = K0 ? 1.0f : __builtin_amdgcn_exp2f(-(r2[v] * ri));
                const float gy = K0 ? ri : e * ri;
                const float E = K0 ? R3 : e * fmaf(cf.kap, ri2, R3);
                if (FORM == 0) {
                    P[p][v] = fmaf(w[0], R3, P[p][v]);
                    a1[p][v] = fmaf(w[1], ri, a1[p][v]);
                    Q[p][v] = fmaf(w[2], E, Q[p][v]);
                    a2[p][v] = fmaf(w[3], gy, a2[p][v]);
                    S1[v] = fmaf(t1[v], R3, S1[v]);
                    s1 = fmaf(t2[v], ri, s1);
                    S2[v] = fmaf(t1[v], E, S2[v]);
                    s2 = fmaf(t2[v], gy, s2);
                } else {
                    float k, vv, kt, dd;
                    if (FORM == 3) {
                        k = kt = E;
                        vv = dd = gy;
                    } else if (FORM == 1) {
                        k = fmaf(cf.bK, E, R3);
                        vv = fmaf(cf.bV, gy, ri);
                        kt = fmaf(cf.bT, E, R3);
                        dd = fmaf(cf.bD, gy, ri);
                    } else {
                        k = fmaf(cf.bK, E, cf.aK * R3);
                        vv = fmaf(cf.bV, gy, cf.aV * ri);
                        kt = fmaf(cf.bT, E, cf.aT * R3);
                        dd = fmaf(cf.bD, gy, cf.aD * ri);
                    }
                    P[p][v] = fmaf(w[0], k, P[p][v]);
                    a1[p][v] = fmaf(w[1], vv, a1[p][v]);
                    a2[p][v] = fmaf(tq[v], kt, fmaf(nb[v], gy, a2[p][v]));
                    S1[v] = fmaf(t1[v], k, S1[v]);
                    s1 = fmaf(t2[v], vv, s1);
                    s2 = fmaf(Q[p][v], kt, s2);
                    S2[v] = fmaf(t1[v], gy, S2[v]);
                    gs[v] = fmaf(ww, dd, gs[v]);
                }
            }
        }
        float k1 = 0.0f, k2 = 0.0f;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            k1 = fmaf(dnt[v], S1[v], k1);
            k2 = fmaf(FORM == 0 ? dnt[v] : nn[v], S2[v], k2);
        }
        if (FORM == 0) {
            acc[q] = fmaf(cf.cV, s1, -cf.cK * k1);
            acc[6 + q] = fmaf(cf.cD, s2, -cf.cT * k2);
        } else {
            acc[q] = fmaf(cf.cV, s1, -cf.cK * k1);
            acc[6 + q] = fmaf(cf.kD, k2, -cf.cT * s2);
        }
        // row data stay in LDS: without this the compiler hoists all 18 row vectors
        // of the p loop out of the q loop and spills
        asm volatile("" ::: "memory");
    }
    acc[12] = acc[13] = acc[14] = acc[15] = 0.0f;
#pragma unroll
    for (int p = 0; p < 6; ++p) {
        const f32x4 dns = mfma4(A[p], bn, zero);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            a1[p][v] = fmaf(dns[v], P[p][v], a1[p][v]);
            if (FORM == 0) a2[p][v] = fmaf(dns[v], Q[p][v], a2[p][v]);
        }
    }
    if (FORM >= 1) {
        const f32x4 cs = C.curl[lc];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const f32x4 ct = *(const f32x4 *)&R.d[12 + c][r0];
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const float gc = cf.cD * gs[v];
                W[c][v] = fmaf(gc, cs[c], W[c][v]);
                acc[12 + c] = fmaf(gc, ct[v], acc[12 + c]);
            }
        }
    }
    src = lane_rows_sum(acc);
}

// Staging of one column (source triangle sj, zero weights unless `in`) per lane,
// relative to the centre c of its tile: wavefronts 0..2 two points each,
// wavefront 3 the rest
template <int FORM, typename IP, typename DP, typename RP>
__device__ __forceinline__ void sym_cols(const SymCoef<float> &cf, SymCols &C, int w, int lane, int sj, bool in,
                                         const double (&c)[3], IP __restrict__ tri, DP __restrict__ stat, RP __restrict__ dyn)
{
    const double s = cf.s;
    const auto ss = stat + (size_t)sj * kStat;
    const auto sd = dyn + (size_t)sj * kDyn;
    if (w < 3) {
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int q = 2 * w + k;
            const double yx = (ss[3 * q] - c[0]) * s, yy = (ss[3 * q + 1] - c[1]) * s, yz = (ss[3 * q + 2] - c[2]) * s;
            C.bq[q][lane] = f32x4{(float)(-2.0 * yx), (float)(-2.0 * yy), (float)(-2.0 * yz),
                                  (float)(yx * yx + yy * yy + yz * yz)};
            const float b1 = in ? sd[q] : 0.0f, b2 = in ? sd[6 + q] : 0.0f;
            // FORM 0: the weights of R3, 1/r, E, e/r; else those of K, V, T and D's normal part
            C.w[q][lane] = FORM == 0 ? f32x4{cf.cK * b1, cf.cV * b2, cf.cT * b1, cf.cD * b2}
                                     : f32x4{cf.cK * b1, cf.cV * b2, cf.cT * b2, cf.kD * b1};
        }
    } else {
        const double nx = ss[18], ny = ss[19], nz = ss[20];
        const double os = (ss[21] - (c[0] * nx + c[1] * ny + c[2] * nz)) * s;
        C.bn[lane] = f32x4{(float)nx, (float)ny, (float)nz, (float)-os};
        if (FORM >= 1) C.curl[lane] = in ? f32x4{sd[12], sd[13], sd[14], 0.0f} : f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        C.id[0][lane] = in ? tri[3 * sj] : -1;
        C.id[1][lane] = in ? tri[3 * sj + 1] : -1;
        C.id[2][lane] = in ? tri[3 * sj + 2] : -1;
    }
}

// ... and of a wavefront's 16 rows (records ts, td of the lane's row l mod 16, zero
// weights unless `in`): A, A2 the matrix operands
template <typename DP, typename RP>
__device__ __forceinline__ void sym_rows(const SymCoef<float> &cf, SymRows &R, int lane, bool in, const double (&c)[3],
                                         DP ts, RP td, float (&A)[6], float &A2)
{
    const int g = lane >> 4, li = lane & 15;
    const double s = cf.s;
#pragma unroll
    for (int p = 0; p < 6; ++p) {
        const double cg = g == 0 ? c[0] : g == 1 ? c[1] : c[2];
        const float xs = (float)((ts[3 * p + (g < 3 ? g : 2)] - cg) * s);
        A[p] = g < 3 ? xs : 1.0f;
        if (g < 3) R.x[p][g][li] = xs;
    }
    A2 = g < 3 ? 0.5f * (float)ts[18 + (g < 3 ? g : 2)] : 0.0f;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const int p = g + 4 * k;
        if (p < 6) {
            const double x = (ts[3 * p] - c[0]) * s, y = (ts[3 * p + 1] - c[1]) * s, z = (ts[3 * p + 2] - c[2]) * s;
            R.x2[p][li] = (float)(x * x + y * y + z * z);
        } else if (p == 6) {
            R.o[li] = (float)((ts[21] - (c[0] * ts[18] + c[1] * ts[19] + c[2] * ts[20])) * s);
        }
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) R.d[4 * g + k][li] = in ? td[4 * g + k] : 0.0f;
}

// Tile records (kTileRec): centre of the bounding box of the tile's (at most 64)
// triangles' vertices, the largest distance of a vertex from it and of a
// quadrature point from its triangle's centroid.  One wavefront per tile.
__global__ __launch_bounds__(64) void k_sym_tiles(int T, const double *__restrict__ xyz, const int32_t *__restrict__ tri,
                                                  double *__restrict__ tiles)
{
    const int t = min(kSymTile * (int)blockIdx.x + (int)threadIdx.x, T - 1);
    double lo[3], hi[3], p[3][3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const double *x = xyz + 3 * (size_t)tri[3 * (size_t)t + k];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            p[k][c] = x[c];
            lo[c] = k == 0 ? x[c] : fmin(lo[c], x[c]);
            hi[c] = k == 0 ? x[c] : fmax(hi[c], x[c]);
        }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1)
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            lo[c] = fmin(lo[c], __shfl_xor(lo[c], off));
            hi[c] = fmax(hi[c], __shfl_xor(hi[c], off));
        }
    double r2 = 0.0, h2 = 0.0;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        double d2 = 0.0, e2 = 0.0;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const double d = p[k][c] - 0.5 * (lo[c] + hi[c]), e = p[k][c] - (p[0][c] + p[1][c] + p[2][c]) / 3.0;
            d2 += d * d;
            e2 += e * e;
        }
        r2 = fmax(r2, d2);
        h2 = fmax(h2, e2);
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        r2 = fmax(r2, __shfl_xor(r2, off));
        h2 = fmax(h2, __shfl_xor(h2, off));
    }
    if (threadIdx.x == 0) {
        double *o = tiles + kTileRec * (size_t)blockIdx.x;
#pragma unroll
        for (int c = 0; c < 3; ++c) o[c] = 0.5 * (lo[c] + hi[c]);
        o[3] = sqrt(r2);
        // the points' offsets from the centroid are 1 - 3 b = 0.7253 (outer orbit) of
        // the vertices' at most
        o[4] = (1.0 - 3.0 * kRuleB) * sqrt(h2);
    }
}

// Row tile I against nk column tiles by one block: tile_of(k) the k-th, src_slot(k,
// sj, cl) where its triangle sj (column cl) takes its 16 sums (null: nowhere),
// row_slot(t) where triangle t of I takes its
template <int FORM, bool K0, typename IP, typename DP, typename RP, typename TileOf, typename SrcSlot, typename RowSlot>
__device__ __forceinline__ void sym_row(const SymCoef<float> &cf, IP __restrict__ tri, DP __restrict__ stat,
                                        DP __restrict__ tiles, RP __restrict__ dyn, int T, int I, int nk, TileOf tile_of,
                                        SrcSlot src_slot, RowSlot row_slot, SymLds &L)
{
    const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int g = lane >> 4, li = lane & 15;
    SymRows &R = L.r[w];
    const f32x4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
    const int t = 64 * I + 16 * w + li;      // the lane's target triangle as an operand row
    const int tc = min(t, T - 1);
    const auto ts = stat + (size_t)tc * kStat;
    const auto td = dyn + (size_t)tc * kDyn;
    f32x4 a1[6], a2[6], W[3];
#pragma unroll
    for (int p = 0; p < 6; ++p) a1[p] = a2[p] = zero;
    W[0] = W[1] = W[2] = zero;
    for (int k = 0; k < nk; ++k) {
        const int J = tile_of(k);
        const double cx = tiles[kTileRec * (size_t)J], cy = tiles[kTileRec * (size_t)J + 1], cz = tiles[kTileRec * (size_t)J + 2];
        const double c[3] = {cx, cy, cz};
        const int sj = 64 * J + lane;
        sym_cols<FORM>(cf, L.c, w, lane, min(sj, T - 1), sj < T, c, tri, stat, dyn);
        float A[6], A2;
        sym_rows(cf, R, lane, t < T, c, ts, td, A, A2);
        __syncthreads();
        // well separated: |X| |Y| stays of the order of r^2
        const double dx = tiles[kTileRec * (size_t)I] - cx, dy = tiles[kTileRec * (size_t)I + 1] - cy, dz = tiles[kTileRec * (size_t)I + 2] - cz;
        const double reach = kSymApart * (tiles[kTileRec * (size_t)I + 3] + tiles[kTileRec * (size_t)J + 3]);
        const bool near = dx * dx + dy * dy + dz * dz < reach * reach;
        if (!near) {
            const bool live[4] = {true, true, true, true};
            for (int cb = 0; cb < 4; ++cb) {
                f32x4 src;
                sym_block<FORM, K0, false>(cf, L.c, R, 16 * cb, lane, A, A2, live, a1, a2, W, src);
                L.out[w][16 * cb + li][g] = src;
            }
        } else {
            int tv[4][3];
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int tr = 64 * I + 16 * w + 4 * g + v, trc = min(tr, T - 1);
#pragma unroll
                for (int k = 0; k < 3; ++k) tv[v][k] = tr < T ? tri[3 * trc + k] : -1;
            }
            for (int cb = 0; cb < 4; ++cb) {
                f32x4 src = zero;
                if (I != J || cb >= w) {   // uniform: below the diagonal every pair has been met
                    const int j0 = L.c.id[0][16 * cb + li], j1 = L.c.id[1][16 * cb + li], j2 = L.c.id[2][16 * cb + li];
                    bool live[4];
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        bool m = (j0 >= 0) & (tv[v][0] >= 0);
#pragma unroll
                        for (int k = 0; k < 3; ++k) m = m & (tv[v][k] != j0) & (tv[v][k] != j1) & (tv[v][k] != j2);
                        if (I == J) m = m & (16 * w + 4 * g + v < 16 * cb + li);
                        live[v] = m;
                    }
                    sym_block<FORM, K0, true>(cf, L.c, R, 16 * cb, lane, A, A2, live, a1, a2, W, src);
                }
                L.out[w][16 * cb + li][g] = src;
            }
        }
        __syncthreads();
        // the four wavefronts' source-side sums, in order, onto the slot (the item's
        // earlier target tiles came before)
        {
            const int cl = tid >> 2, m = tid & 3, sj = 64 * J + cl;
            float *o = sj < T ? src_slot(k, sj, cl) : nullptr;
            if (o) {
                f32x4 *so = (f32x4 *)o + m;
                f32x4 v = zero;
#pragma unroll
                for (int u = 0; u < kSymWaves; ++u) v += L.out[u][cl][m];
                *so = v;
            }
        }
    }
    // target-side sums over the 16 columns of each row of lanes
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        float o[16];
#pragma unroll
        for (int p = 0; p < 6; ++p) {
            o[p] = row_sum(a1[p][v]);
            o[6 + p] = row_sum(a2[p][v]);
        }
#pragma unroll
        for (int k = 0; k < 3; ++k) o[12 + k] = FORM == 0 ? 0.0f : row_sum(W[k][v]);
        o[15] = 0.0f;
        const int tr = 64 * I + 16 * w + 4 * g + v;
        if (li == 0 && tr < T) {
            f32x4 *fo = (f32x4 *)row_slot(tr);
#pragma unroll
            for (int k = 0; k < 4; ++k) fo[k] = f32x4{o[4 * k], o[4 * k + 1], o[4 * k + 2], o[4 * k + 3]};
        }
    }
}

// Item (a, b, z) of one mesh by one block: part z of nz takes the column groups
// 4 z / nz .. 4 (z + 1) / nz of every tile (PARTS; else nz = 1); part holds the 2 nr nz slots.  sym_row's work
// written out: through the shared functions the compiler issues the staging loads
// later, 8% of a product of 1620 triangles (direct 103 us against 93, second kind
// 122 against 114; 1% either way at 20480).
template <int FORM, bool K0, bool PARTS, typename IP, typename DP, typename RP>
__device__ __forceinline__ void sym_item(const SymCoef<float> &cf, IP __restrict__ tri, DP __restrict__ stat,
                                         DP __restrict__ tiles, RP __restrict__ dyn, int T, int rt, int nr, int nz, int a, int b, int z,
                                         float *__restrict__ part, SymLds &L)
{
    const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int g = lane >> 4, li = lane & 15;
    const int ntile = (T + 63) / 64;
    const int cb0 = PARTS ? 4 * z / nz : 0, cb1 = PARTS ? 4 * (z + 1) / nz : 4;
    const int I0 = a * rt, I1 = min(ntile, I0 + rt);
    const int J0 = b * rt, J1 = min(ntile, J0 + rt);
    SymRows &R = L.r[w];
    const f32x4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
    for (int I = I0; I < I1; ++I) {
        const int t = 64 * I + 16 * w + li;      // the lane's target triangle as an operand row
        const int tc = min(t, T - 1);
        const auto ts = stat + (size_t)tc * kStat;
        const auto td = dyn + (size_t)tc * kDyn;
        f32x4 a1[6], a2[6], W[3];
#pragma unroll
        for (int p = 0; p < 6; ++p) a1[p] = a2[p] = zero;
        W[0] = W[1] = W[2] = zero;
        for (int J = a == b ? I : J0; J < J1; ++J) {
            const double cx = tiles[kTileRec * (size_t)J], cy = tiles[kTileRec * (size_t)J + 1], cz = tiles[kTileRec * (size_t)J + 2];
            const double c[3] = {cx, cy, cz};
            const double s = cf.s;
            // columns: wavefronts 0..2 two points each, wavefront 3 the rest
            {
                const int sj = min(64 * J + lane, T - 1);
                const bool in = 64 * J + lane < T;   // past the end: the last triangle with zero weights
                const auto ss = stat + (size_t)sj * kStat;
                const auto sd = dyn + (size_t)sj * kDyn;
                if (w < 3) {
#pragma unroll
                    for (int k = 0; k < 2; ++k) {
                        const int q = 2 * w + k;
                        const double yx = (ss[3 * q] - cx) * s, yy = (ss[3 * q + 1] - cy) * s, yz = (ss[3 * q + 2] - cz) * s;
                        L.c.bq[q][lane] = f32x4{(float)(-2.0 * yx), (float)(-2.0 * yy), (float)(-2.0 * yz),
                                                (float)(yx * yx + yy * yy + yz * yz)};
                        const float b1 = in ? sd[q] : 0.0f, b2 = in ? sd[6 + q] : 0.0f;
                        // FORM 0: the weights of R3, 1/r, E, e/r; else those of K, V, T and D's normal part
                        L.c.w[q][lane] = FORM == 0 ? f32x4{cf.cK * b1, cf.cV * b2, cf.cT * b1, cf.cD * b2}
                                                   : f32x4{cf.cK * b1, cf.cV * b2, cf.cT * b2, cf.kD * b1};
                    }
                } else {
                    const double nx = ss[18], ny = ss[19], nz = ss[20];
                    const double os = (ss[21] - (cx * nx + cy * ny + cz * nz)) * s;
                    L.c.bn[lane] = f32x4{(float)nx, (float)ny, (float)nz, (float)-os};
                    if (FORM >= 1) L.c.curl[lane] = in ? f32x4{sd[12], sd[13], sd[14], 0.0f} : zero;
                    L.c.id[0][lane] = in ? tri[3 * sj] : -1;
                    L.c.id[1][lane] = in ? tri[3 * sj + 1] : -1;
                    L.c.id[2][lane] = in ? tri[3 * sj + 2] : -1;
                }
            }
            // rows of this wavefront
            float A[6], A2;
#pragma unroll
            for (int p = 0; p < 6; ++p) {
                const double cg = g == 0 ? c[0] : g == 1 ? c[1] : c[2];
                const float xs = (float)((ts[3 * p + (g < 3 ? g : 2)] - cg) * s);
                A[p] = g < 3 ? xs : 1.0f;
                if (g < 3) R.x[p][g][li] = xs;
            }
            A2 = g < 3 ? 0.5f * (float)ts[18 + (g < 3 ? g : 2)] : 0.0f;
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const int p = g + 4 * k;
                if (p < 6) {
                    const double x = (ts[3 * p] - cx) * s, y = (ts[3 * p + 1] - cy) * s, z = (ts[3 * p + 2] - cz) * s;
                    R.x2[p][li] = (float)(x * x + y * y + z * z);
                } else if (p == 6) {
                    R.o[li] = (float)((ts[21] - (cx * ts[18] + cy * ts[19] + cz * ts[20])) * s);
                }
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) R.d[4 * g + k][li] = t < T ? td[4 * g + k] : 0.0f;
            __syncthreads();
            // well separated: |X| |Y| stays of the order of r^2
            const double dx = tiles[kTileRec * (size_t)I] - cx, dy = tiles[kTileRec * (size_t)I + 1] - cy, dz = tiles[kTileRec * (size_t)I + 2] - cz;
            const double reach = kSymApart * (tiles[kTileRec * (size_t)I + 3] + tiles[kTileRec * (size_t)J + 3]);
            const bool near = dx * dx + dy * dy + dz * dz < reach * reach;
            if (!near) {
                const bool live[4] = {true, true, true, true};
                for (int cb = cb0; cb < cb1; ++cb) {
                    f32x4 src;
                    sym_block<FORM, K0, false>(cf, L.c, R, 16 * cb, lane, A, A2, live, a1, a2, W, src);
                    L.out[w][16 * cb + li][g] = src;
                }
            } else {
                int tv[4][3];
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int tr = 64 * I + 16 * w + 4 * g + v, trc = min(tr, T - 1);
#pragma unroll
                    for (int k = 0; k < 3; ++k) tv[v][k] = tr < T ? tri[3 * trc + k] : -1;
                }
                for (int cb = cb0; cb < cb1; ++cb) {
                    f32x4 src = zero;
                    if (I != J || cb >= w) {   // uniform: below the diagonal every pair has been met
                        const int j0 = L.c.id[0][16 * cb + li], j1 = L.c.id[1][16 * cb + li], j2 = L.c.id[2][16 * cb + li];
                        bool live[4];
#pragma unroll
                        for (int v = 0; v < 4; ++v) {
                            bool m = (j0 >= 0) & (tv[v][0] >= 0);
#pragma unroll
                            for (int k = 0; k < 3; ++k) m = m & (tv[v][k] != j0) & (tv[v][k] != j1) & (tv[v][k] != j2);
                            if (I == J) m = m & (16 * w + 4 * g + v < 16 * cb + li);
                            live[v] = m;
                        }
                        sym_block<FORM, K0, true>(cf, L.c, R, 16 * cb, lane, A, A2, live, a1, a2, W, src);
                    }
                    L.out[w][16 * cb + li][g] = src;
                }
            }
            __syncthreads();
            // the four wavefronts' source-side sums, in order, onto the slot (the item's
            // earlier target tiles came before)
            {
                const int cl = tid >> 2, k = tid & 3, sj = 64 * J + cl;
                if (sj < T) {
                    f32x4 *so = (f32x4 *)(part + ((size_t)((PARTS ? (nz + z) * nr : nr) + a) * T + sj) * 16) + k;
                    f32x4 v = I == I0 ? zero : *so;
                    if (!PARTS || (cl >> 4 >= cb0 && cl >> 4 < cb1))   // the other parts' columns: zero
#pragma unroll
                        for (int u = 0; u < kSymWaves; ++u) v += L.out[u][cl][k];
                    *so = v;
                }
            }
        }
        // target-side sums over the 16 columns of each row of lanes
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            float o[16];
#pragma unroll
            for (int p = 0; p < 6; ++p) {
                o[p] = row_sum(a1[p][v]);
                o[6 + p] = row_sum(a2[p][v]);
            }
#pragma unroll
            for (int k = 0; k < 3; ++k) o[12 + k] = FORM == 0 ? 0.0f : row_sum(W[k][v]);
            o[15] = 0.0f;
            const int tr = 64 * I + 16 * w + 4 * g + v;
            if (li == 0 && tr < T) {
                f32x4 *fo = (f32x4 *)(part + ((size_t)((PARTS ? z * nr : 0) + b) * T + tr) * 16);
#pragma unroll
                for (int k = 0; k < 4; ++k) fo[k] = f32x4{o[4 * k], o[4 * k + 1], o[4 * k + 2], o[4 * k + 3]};
            }
        }
    }
}

// the next item of a queue, for the whole block
__device__ __forceinline__ int sym_next_item(int *__restrict__ next, SymLds &L)
{
    __syncthreads();   // the previous item's number is read and its LDS consumed
    if (threadIdx.x == 0) L.item = atomicAdd(next, 1);
    __syncthreads();
    return __builtin_amdgcn_readfirstlane(L.item);
}

// One mesh: each block takes items (heaviest first) from a device counter
// until the list is done.
template <int FORM, bool K0>
__global__ __launch_bounds__(64 * kSymWaves, 2) void k_far_sym(int T, int rt, int nr, int nz, SymCoef<float> cf,
                                                              const int32_t *__restrict__ tri,
                                                              const double *__restrict__ stat,
                                                              const double *__restrict__ tiles,
                                                              const float *__restrict__ dyn,
                                                              const int4 *__restrict__ items, int nitems,
                                                              int *__restrict__ next, float *__restrict__ part,
                                                              DevCtl ctl)
{
    __shared__ SymLds lds;
    if (ctl_skip(ctl)) return;   // uniform: every wavefront leaves
    for (;;) {
        const int i = sym_next_item(next, lds);
        if (i >= nitems) return;
        const int4 it = items[i];
        sym_item<FORM, K0, false>(cf, tri, stat, tiles, dyn, T, rt, nr, 1, it.y, it.z, 0, part, lds);
    }
}

// ... with items in parts (meshes of few items).  A kernel of its own: the part's
// bounds as variables cost the direct form of k_far_sym registers (70.2 against 69.2
// ms at 81920 triangles).
template <int FORM, bool K0>
__global__ __launch_bounds__(64 * kSymWaves, 2) void k_far_sym_parts(int T, int rt, int nr, int nz, SymCoef<float> cf,
                                                              const int32_t *__restrict__ tri,
                                                              const double *__restrict__ stat,
                                                              const double *__restrict__ tiles,
                                                              const float *__restrict__ dyn,
                                                              const int4 *__restrict__ items, int nitems,
                                                              int *__restrict__ next, float *__restrict__ part,
                                                              DevCtl ctl)
{
    __shared__ SymLds lds;
    if (ctl_skip(ctl)) return;   // uniform: every wavefront leaves
    for (;;) {
        const int i = sym_next_item(next, lds);
        if (i >= nitems) return;
        const int4 it = items[i];
        sym_item<FORM, K0, true>(cf, tri, stat, tiles, dyn, T, rt, nr, nz, it.y, it.z, it.w, part, lds);
    }
}

// Several meshes (batched requests): items {request, a, b}; a request whose
// stop flag is set contributes nothing.
template <int FORM, bool K0>
__global__ __launch_bounds__(64 * kSymWaves, 2) void k_far_sym_batch(const FarReq<float> *__restrict__ reqs,
                                                                    const int4 *__restrict__ items, int nitems,
                                                                    int *__restrict__ next)
{
    __shared__ SymLds lds;
    for (;;) {
        const int i = sym_next_item(next, lds);
        if (i >= nitems) return;
        const int4 it = items[i];
        const FarReq<float> &rq = reqs[it.x];
        if (rq.skip && *rq.skip) continue;
        sym_item<FORM, K0, true>(rq.sc, rq.tri, rq.stat64, rq.tiles, rq.dyn, rq.T, rq.rt, rq.nr, rq.nz, it.y, it.z, it.w, rq.part,
                             lds);
    }
}

// Listed pairs of tiles (the treecode's direct part): item {row tile I, first and
// end entry, slot}, entry {column tile J, slot or -1}.  The item's slot takes I's
// sums over its entries, an entry's slot those of its column tile (-1: dropped,
// that tile meets I through proxies).
template <int FORM, bool K0>
__global__ __launch_bounds__(64 * kSymWaves, 2) void k_sym_list(int T, SymCoef<float> cf, const int32_t *__restrict__ tri,
                                                               const double *__restrict__ stat,
                                                               const double *__restrict__ tiles,
                                                               const float *__restrict__ dyn,
                                                               const int4 *__restrict__ items,
                                                               const int2 *__restrict__ entries,
                                                               float *__restrict__ slots, DevCtl ctl)
{
    __shared__ SymLds lds;
    if (ctl_skip(ctl)) return;
    const int4 it = items[blockIdx.x];
    sym_row<FORM, K0>(cf, tri, stat, tiles, dyn, T, it.x, it.z - it.y, [&](int k) { return entries[it.y + k].x; },
                      [&](int k, int sj, int cl) {
                          const int slot = entries[it.y + k].y;
                          return slot < 0 ? nullptr : slots + ((size_t)slot * kSymTile + cl) * 16;
                      },
                      [&](int tr) { return slots + ((size_t)it.w * kSymTile + tr - kSymTile * it.x) * 16; }, lds);
}

// kFinishLanes lanes per triangle over its (nr + 1) nz slots, then the test
// projection of k_far_finish (sym_finish_group, far.h)
template <typename R>
__global__ __launch_bounds__(256) void k_far_sym_finish(int T, int rt, int nr, int nz, int family, int swap,
                                                          const double *__restrict__ geo,
                                                          const R *__restrict__ part,
                                                          double *__restrict__ triout, DevCtl ctl)
{
    if (ctl_skip(ctl)) return;
    const int t = (int)((blockIdx.x * (size_t)blockDim.x + threadIdx.x) / kFinishLanes);
    const int l = threadIdx.x % kFinishLanes;
    sym_finish_group<R>(t, l, t < T, T, rt, nr, nz, family, swap, geo, part, triout);   // the group agrees on t < T
}

__global__ void k_sym_set(int *p, int v) { *p = v; }

// ------------------------------------------------------------------ host

// Ranges of rt tiles: at most 320 ranges (51000 items) in FP32, kSym64Ranges in
// FP64, whose slots are twice as large.  In FP32 an item's four column groups are
// dealt to nz parts while there are fewer than 400 (per product in one part / now:
// 320 triangles second kind 75 / 51 us, 720 76 / 65, 1280 direct 74 / 69, 1620 94 /
// 89; up to 512 parts: 1280 76).  In FP64 an item (64 steps of 36 point
// pairs per lane, 16 for each wavefront) is cut into nz parts where the items
// are few for the 512 resident blocks: into two below 2048 items, further below
// 600 (measured per product, 1620 triangles / 351 items: 2 parts 138 us, 8 172 us,
// 16 226 us; 3380 triangles / 1431 items: 1 part 444 us, 2 416 us).  parts
// false: items stay whole (no room for the parts' slots under a memory budget).
SymSplit sym_split(int T, bool fp32, bool parts)
{
    const int most = fp32 ? 320 : kSym64Ranges, ntile = (T + kSymTile - 1) / kSymTile;
    SymSplit s;
    s.rt = std::max(1, (ntile + most - 1) / most);
    s.nr = (ntile + s.rt - 1) / s.rt;
    const int n = s.nr * (s.nr + 1) / 2;
    if (!parts) return s;
    if (fp32) {
        while (s.nz < 4 && n * s.nz < 400) s.nz *= 2;
    } else {
        while (s.nz < 16 && n * s.nz < (s.nz == 1 ? 2048 : 600)) s.nz *= 2;
    }
    return s;
}

// Items {request, a, b, part}; larger ones come first, among equal ones those near
// the diagonal, whose tiles touch and take longer, so that the list ends with the
// lightest.
void sym_items(int T, const SymSplit &s, int request, std::vector<int4> &items)
{
    const int ntile = (T + kSymTile - 1) / kSymTile, rt = s.rt;
    std::vector<std::pair<int, int4>> w;
    for (int k = 0; k < s.nr; ++k)
        for (int a = 0; a + k < s.nr; ++a) {
            const int b = a + k;
            const int na = std::min(ntile, (a + 1) * rt) - a * rt, nb = std::min(ntile, (b + 1) * rt) - b * rt;
            const int pairs = a == b ? na * (na + 1) / 2 : na * nb;
            for (int z = 0; z < s.nz; ++z) w.push_back({pairs, make_int4(request, a, b, z)});
        }
    std::stable_sort(w.begin(), w.end(), [](const std::pair<int, int4> &x, const std::pair<int, int4> &y) {
        return x.first > y.first;
    });
    items.clear();
    for (auto &e : w) items.push_back(e.second);
}

static const void *sym_kernel(int form, bool k0)
{
    const void *k = nullptr;
#define SYM_ADDR(KF) k = reinterpret_cast<const void *>(&KF);
    SYM_PICK(k_far_sym, form, k0, SYM_ADDR)
    return k;
}

static const void *sym_batch_kernel(int form, bool k0)
{
    const void *k = nullptr;
    SYM_PICK(k_far_sym_batch, form, k0, SYM_ADDR)
    return k;
}

// as many blocks as are resident at once, or one per item if fewer.  The resident
// number is a constant of the kernel and the device; asked once, since a handle's
// creation needs it for several kernels.
int resident_blocks(const void *kernel, int threads, int nitems)
{
    static std::mutex mu;
    static std::map<std::pair<const void *, int>, long long> known;   // kernel, device
    int dev = 0;
    HIPCHECK(hipGetDevice(&dev));
    std::lock_guard<std::mutex> lock(mu);
    long long &n = known[{kernel, dev}];
    if (n == 0) {
        int ncu = 0, per_cu = 0;
        HIPCHECK(hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev));
        HIPCHECK(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, threads, 0));
        n = (long long)std::max(ncu, 1) * std::max(per_cu, 1);
    }
    return (int)std::max(1LL, std::min(n, (long long)nitems));
}

int sym_blocks(bool fp32, int nitems, int form, bool k0)
{
    return fp32 ? resident_blocks(sym_kernel(form, k0), 64 * kSymWaves, nitems) : sym64_blocks(nitems, form, k0);
}
int sym_batch_blocks_for(bool fp32, int form, bool k0, int n)
{
    return fp32 ? resident_blocks(sym_batch_kernel(form, k0), 64 * kSymWaves, n) : sym64_batch_blocks(form, k0, n);
}

void launch_sym_tiles(DevMesh &d)
{
    hipLaunchKernelGGL(k_sym_tiles, dim3((d.hm.T + kSymTile - 1) / kSymTile), dim3(64), 0, d.stream, d.hm.T, d.xyz, d.tri,
                       d.sym_tiles);
    HIPCHECK(hipGetLastError());
}

void launch_sym_reset(hipStream_t s, int *next) { hipLaunchKernelGGL(k_sym_set, dim3(1), dim3(1), 0, s, next, 0); }

void launch_far_sym(DevMesh &d)
{
    SymCoef<float> cf;
    const int form = sym_coef(d, cf);
    const bool k0 = d.far_k0;
    const int nb = d.sym_blocks[sym_form_index(form)];
#define SYM_RUN(KF)                                                                                             \
    hipLaunchKernelGGL(KF, dim3(nb), dim3(64 * kSymWaves), 0, d.stream, d.hm.T, d.sym_rt, d.sym_nr, d.sym_nz, cf, d.tri,  \
                       d.stat64, d.sym_tiles, d.dyn32, d.sym_items, d.sym_nitems, d.sym_next, (float *)d.part,  \
                       d.ctl);
    if (d.sym_nz > 1) {
        SYM_PICK(k_far_sym_parts, form, k0, SYM_RUN)
    } else {
        SYM_PICK(k_far_sym, form, k0, SYM_RUN)
    }
    HIPCHECK(hipGetLastError());
}

void launch_sym_list(DevMesh &d, const int4 *items, int nitems, const int2 *entries, const double *tiles, float *slots)
{
    SymCoef<float> cf;
    const int form = sym_coef(d, cf);
    const bool k0 = d.far_k0;
#define SYM_RUN_LIST(KF)                                                                                           \
    hipLaunchKernelGGL(KF, dim3(nitems), dim3(64 * kSymWaves), 0, d.stream, d.hm.T, cf, d.tri, d.stat64, tiles, d.dyn32, \
                       items, entries, slots, d.ctl);
    SYM_PICK(k_sym_list, form, k0, SYM_RUN_LIST)
    HIPCHECK(hipGetLastError());
}

void launch_far_sym_finish(DevMesh &d)
{
    const int T = d.hm.T;
    const FormCoef &f = d.fm;
    const int swap = f.family == 0 && laplace_row(f) == 1;
    const dim3 grid((unsigned)(((size_t)T * kFinishLanes + 255) / 256)), block(256);
    if (d.prm.precision == PB_FP64)
        hipLaunchKernelGGL(k_far_sym_finish<double>, grid, block, 0, d.stream, T, d.sym_rt, d.sym_nr, d.sym_nz, f.family, swap,
                           d.geo, (const double *)d.part, d.triout, d.ctl);
    else
        hipLaunchKernelGGL(k_far_sym_finish<float>, grid, block, 0, d.stream, T, d.sym_rt, d.sym_nr, d.sym_nz, f.family, swap,
                           d.geo, (const float *)d.part, d.triout, d.ctl);
    HIPCHECK(hipGetLastError());
}

// batched requests: one queue per kernel form and screening of {request, a, b} items
void launch_far_sym_batch(int form, bool k0, const void *reqs, const int4 *items, int n, int nblocks, int *next,
                          hipStream_t s)
{
    if (n == 0) return;
    launch_sym_reset(s, next);
#define SYM_RUNB(KF) \
    hipLaunchKernelGGL(KF, dim3(nblocks), dim3(64 * kSymWaves), 0, s, (const FarReq<float> *)reqs, items, n, next);
    SYM_PICK(k_far_sym_batch, form, k0, SYM_RUNB)
    HIPCHECK(hipGetLastError());
}

}  // namespace pbm
