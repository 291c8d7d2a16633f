// Geometry, charge-to-surface projections (Eq. sources), reaction potential
// (Eq. phireac_bie) and the charge-inside-surface check.
#include <algorithm>
#include <mutex>
#include <type_traits>

#include "fp64.h"
#include "pbm_internal.h"

namespace pbm {

// One thread per (Morton-sorted) triangle: area, outward unit normal, surface
// curls of the three P1 hats, the six regular quadrature points, and the
// FP64 / FP32 source-target records used by the far-field kernels.
__global__ void k_geometry(int T, const double *__restrict__ xyz, const int32_t *__restrict__ tri,
                           double *__restrict__ geo, double *__restrict__ stat64, float *__restrict__ stat32)
{
    int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= T) return;
    double P[3][3];
    for (int k = 0; k < 3; ++k) {
        int v = tri[3 * t + k];
        for (int c = 0; c < 3; ++c) P[k][c] = xyz[3 * v + c];
    }
    double e1[3], e2[3];
    for (int c = 0; c < 3; ++c) { e1[c] = P[1][c] - P[0][c]; e2[c] = P[2][c] - P[0][c]; }
    double cr[3] = {e1[1] * e2[2] - e1[2] * e2[1], e1[2] * e2[0] - e1[0] * e2[2], e1[0] * e2[1] - e1[1] * e2[0]};
    double len = sqrt(cr[0] * cr[0] + cr[1] * cr[1] + cr[2] * cr[2]);
    double area = 0.5 * len;
    double n[3] = {cr[0] / len, cr[1] / len, cr[2] / len};
    double *g = geo + (size_t)t * kGeo;
    double *s64 = stat64 + (size_t)t * kStat;
    float *s32 = stat32 + (size_t)t * kStat;
#pragma unroll
    for (int p = 0; p < 6; ++p) {
        double x[3];
        for (int c = 0; c < 3; ++c)
            x[c] = rule_bary(p, 0) * P[0][c] + rule_bary(p, 1) * P[1][c] + rule_bary(p, 2) * P[2][c];
        double yn = x[0] * n[0] + x[1] * n[1] + x[2] * n[2];
        for (int c = 0; c < 3; ++c) {
            g[3 * p + c] = x[c];
            s64[3 * p + c] = x[c];
            s32[3 * p + c] = (float)x[c];
        }
        s64[21 + p] = yn;
        s32[21 + p] = (float)yn;
    }
    for (int c = 0; c < 3; ++c) {
        g[18 + c] = n[c];
        s64[18 + c] = n[c];
        s32[18 + c] = (float)n[c];
    }
    g[21] = area;
    // curl of hat k: n x grad(lambda_k) = -(P_{k+2} - P_{k+1}) / (2 |t|)
    for (int k = 0; k < 3; ++k) {
        int a = (k + 1) % 3, b = (k + 2) % 3;
        for (int c = 0; c < 3; ++c) g[22 + 3 * k + c] = -(P[b][c] - P[a][c]) / (2.0 * area);
    }
    g[31] = 0.0;
    s64[27] = area;
    s32[27] = (float)area;
    for (int i = 0; i < 9; ++i) {
        s64[28 + i] = g[22 + i];
        s32[28 + i] = (float)g[22 + i];
    }
    // centroid (the one-point rule of fast Calderon's preconditioner)
    for (int c = 0; c < 3; ++c) {
        const double m = (P[0][c] + P[1][c] + P[2][c]) / 3.0;
        s64[37 + c] = m;
        s32[37 + c] = (float)m;
    }
}

void launch_geometry(DevMesh &d)
{
    int T = d.hm.T;
    hipLaunchKernelGGL(k_geometry, dim3((T + 255) / 256), dim3(256), 0, d.stream, T, d.xyz, d.tri, d.geo,
                       d.stat64, d.stat32);
    HIPCHECK(hipGetLastError());
}

// ------------------------------------------------------------------ sources
// One thread per quadrature point and chunk of charges (grid.y): phi_D and phi_N of
// Eq. sources without the 1/(4 pi eps_in) factor, f[c][2][6 T].  Charges are read
// with uniform (scalar) loads, two at a time.  Bound: the FP64 vector rate, 19
// instructions per point and charge (a division by the square root took about 50);
// 40500 triangles, 2000 charges: the projections and the potential below together
// went from 2.40 to 0.83 ms, host copies included.
__global__ __launch_bounds__(256) void k_source_field(int T, int nq, int chunk, const double *__restrict__ geo,
                                                      const double *__restrict__ qb, double *__restrict__ f)
{
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= 6 * T) return;
    int t = i / 6, p = i - 6 * t;
    const double *g = geo + (size_t)t * kGeo;
    double x = g[3 * p], y = g[3 * p + 1], z = g[3 * p + 2];
    double nx = g[18], ny = g[19], nz = g[20];
    const double *qx = qb, *qy = qb + nq, *qz = qb + 2 * nq, *qq = qb + 3 * nq;
    double sD = 0.0, sN = 0.0;
    const int j0 = blockIdx.y * chunk, j1 = min(nq, j0 + chunk);
    auto add = [&](int j, auto n) {
        constexpr int N = decltype(n)::value;
        double r2[N], ri[N], dn[N];
#pragma unroll
        for (int k = 0; k < N; ++k) {
            const double dx = x - qx[j + k], dy = y - qy[j + k], dz = z - qz[j + k];
            r2[k] = dx * dx + dy * dy + dz * dz;
            dn[k] = dx * nx + dy * ny + dz * nz;
        }
        rsqrt3_n<N>(r2, ri);
#pragma unroll
        for (int k = 0; k < N; ++k) {
            const double a = qq[j + k] * ri[k];
            sD += a;
            sN = fma(-dn[k] * (ri[k] * ri[k]), a, sN);
        }
    };
    int j = j0;
    for (; j + 1 < j1; j += 2) add(j, std::integral_constant<int, 2>());
    if (j < j1) add(j, std::integral_constant<int, 1>());
    double *o = f + (size_t)blockIdx.y * 12 * T;
    o[i] = sD;
    o[(size_t)6 * T + i] = sN;
}

// per-triangle P1 test projection of point values (summed over the C chunks of
// charges): out[t][k] = |t| sum_p w_p lambda_k(p) f[t][p] * scale
__global__ void k_project2(int T, int C, const double *__restrict__ geo, const double *__restrict__ f, double scale,
                           double *__restrict__ triout)
{
    int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= T) return;
    double area = geo[(size_t)t * kGeo + 21];
    for (int h = 0; h < 2; ++h) {
        double fp[6];
#pragma unroll
        for (int p = 0; p < 6; ++p) {
            fp[p] = 0.0;
            for (int c = 0; c < C; ++c) fp[p] += f[((size_t)c * 2 + h) * 6 * T + 6 * (size_t)t + p];
        }
        for (int k = 0; k < 3; ++k) {
            double s = 0.0;
#pragma unroll
            for (int p = 0; p < 6; ++p) s += rule_w(p) * rule_bary(p, k) * fp[p];
            triout[6 * (size_t)t + 3 * h + k] = s * area * scale;
        }
    }
}

// per-vertex gather of triangle contributions in fixed incidence order
__global__ void k_gather_tri(int V, const int32_t *__restrict__ inc_ptr, const int32_t *__restrict__ inc_tk,
                             const double *__restrict__ triout, double *__restrict__ y)
{
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= V) return;
    double a = 0.0, b = 0.0;
    for (int e = inc_ptr[i]; e < inc_ptr[i + 1]; ++e) {
        int tk = inc_tk[e];
        int t = tk >> 2, k = tk & 3;
        a += triout[6 * (size_t)t + k];
        b += triout[6 * (size_t)t + 3 + k];
    }
    y[i] = a;
    y[V + i] = b;
}

void launch_rhs(DevMesh &d, int nq, const double *qbuf, double *b)
{
    int T = d.hm.T, V = d.hm.V;
    // chunks of charges while the points alone give less than about 8 wavefronts per
    // SIMD, of at least 16 charges; their values go to the far field's partial sums,
    // which hold at least 16 T doubles per source chunk
    int C = std::max(1, std::min({8192 / ((6 * T + 63) / 64), nq / 16, d.S}));
    const int chunk = (nq + C - 1) / C;
    C = (nq + chunk - 1) / chunk;
    double *f = C > 1 ? (double *)d.part : d.fpts;
    hipLaunchKernelGGL(k_source_field, dim3((6 * T + 255) / 256, C), dim3(256), 0, d.stream, T, nq, chunk, d.geo, qbuf, f);
    hipLaunchKernelGGL(k_project2, dim3((T + 255) / 256), dim3(256), 0, d.stream, T, C, d.geo, f,
                       kInv4Pi / d.prm.eps_in, d.triout);
    hipLaunchKernelGGL(k_gather_tri, dim3((V + 255) / 256), dim3(256), 0, d.stream, V, d.inc_ptr, d.inc_tk,
                       d.triout, b);
    HIPCHECK(hipGetLastError());
}

// right-hand side of the formulation from [<phi_i, varphi_D>; <phi_i, varphi_N>], in place
__global__ void k_rhs_combine(int V, double d1, double n1, double d2, double n2, double *__restrict__ b)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= V) return;
    const double bD = b[i], bN = b[V + i];
    b[i] = d1 * bD + n1 * bN;
    b[V + i] = d2 * bD + n2 * bN;
}

void formulation_rhs(DevMesh &d, int nq, const double *qbuf, double *b)
{
    launch_rhs(d, nq, qbuf, b);
    const FormCoef &f = d.fm;
    const int V = d.hm.V;
    hipLaunchKernelGGL(k_rhs_combine, dim3((V + 255) / 256), dim3(256), 0, d.stream, V, f.rhsD[0], f.rhsN[0],
                       f.rhsD[1], f.rhsN[1], b);
    HIPCHECK(hipGetLastError());
}

// --------------------------------------------------------- reaction potential
// One wavefront per 64 points and chunk of source triangles: a lane per point, the
// triangles through scalar loads.  Sums G(x_k, y) b2 - dG/dn_y(x_k, y) b1 with the
// Laplace kernel (no 4 pi), where b1 = w|s| phi(y), b2 = w|s| dphi(y) are the FP64
// dynamic records of the traces; d.n is the same for a triangle's six points.
// Bound: the FP64 vector rate, 16 instructions per pair; with a block per point
// and the lanes over the sources every block read all records again (36 GB of
// cache traffic at 40500 triangles and 2000 points).
__global__ __launch_bounds__(256) void k_reaction(int T, int npts, int C, int chunk, const double *__restrict__ pts,
                                                  const double *__restrict__ stat, const double *__restrict__ dyn,
                                                  double *__restrict__ part)
{
    const int id = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int c = id % C, k = (id / C) * 64 + ((int)threadIdx.x & 63);
    if ((id / C) * 64 >= npts) return;
    const int kc = min(k, npts - 1);
    const double x = point_cut(pts[3 * kc]), y = point_cut(pts[3 * kc + 1]), z = point_cut(pts[3 * kc + 2]);
    const int s0 = c * chunk, s1 = min(T, s0 + chunk);
    using CD = const __attribute__((address_space(4))) double *;
    double acc = 0.0;
    for (int s = s0; s < s1; ++s) {
        CD st = (CD)(stat + (size_t)s * kStat), dy = (CD)(dyn + (size_t)s * kDyn);
        double r2[6], ri[6], dn = 0.0, a = 0.0;
#pragma unroll
        for (int q = 0; q < 6; ++q) {
            const double dx = x - st[3 * q], dyy = y - st[3 * q + 1], dz = z - st[3 * q + 2];
            r2[q] = dx * dx + dyy * dyy + dz * dz;
            if (q == 0) dn = dx * st[18] + dyy * st[19] + dz * st[20];
        }
        rsqrt3_n<6>(r2, ri);
#pragma unroll
        for (int q = 0; q < 6; ++q) {
            acc = fma(ri[q], dy[6 + q], acc);
            a = fma(ri[q] * (ri[q] * ri[q]), dy[q], a);
        }
        acc = fma(-dn, a, acc);
    }
    if (k < npts) part[(size_t)k * C + c] = acc;
}

// out[k] = (sum over chunks of part[k C + c]) / (4 pi): one wavefront per point
__global__ __launch_bounds__(256) void k_reaction_finish(int npts, int C, const double *__restrict__ part,
                                                         double *__restrict__ out)
{
    const int k = blockIdx.x * 4 + ((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (k >= npts) return;
    double s = 0.0;
    for (int c = lane; c < C; c += 64) s += part[(size_t)k * C + c];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);
    if (lane == 0) out[k] = s * kInv4Pi;
}

// Fixed-shape tree reduction -> deterministic partials.
constexpr int kRedBlock = 256;

__device__ inline double block_sum(double v, double *sh)
{
    sh[threadIdx.x] = v;
    __syncthreads();
    for (int s = kRedBlock / 2; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) sh[threadIdx.x] += sh[threadIdx.x + s];
        __syncthreads();
    }
    double r = sh[0];
    __syncthreads();
    return r;
}

// The potential at few points of a small mesh: a block per point, its lanes over the
// quadrature points, in one launch.  Bound: latency; the chunks of k_reaction are
// chains of eight triangles behind scalar loads, and their sums a launch of their
// own.  Potentials at 1 / 200 points, copies included, in us, by k_reaction and so:
// 80 triangles 44 / 45 and 39 / 40, 320 46 / 46.5 and 42 / 44, 500 47 / 47.5 and 43.5 /
// 45.5; a block per point at 720 45.7 / 46.6 against 46.5 / 47, at 1620 54 / 55 against
// 49 / 50.
constexpr int kPointTriangles = 768, kPointPoints = 512;
__global__ __launch_bounds__(kRedBlock) void k_reaction_point(int T, const double *__restrict__ pts,
                                                              const double *__restrict__ stat,
                                                              const double *__restrict__ dyn, double *__restrict__ out)
{
    __shared__ double sh[kRedBlock];
    const int k = blockIdx.x;
    const double x = point_cut(pts[3 * k]), y = point_cut(pts[3 * k + 1]), z = point_cut(pts[3 * k + 2]);
    double acc = 0.0;
    for (int i = threadIdx.x; i < 6 * T; i += kRedBlock) {
        const int s = i / 6, q = i - 6 * s;
        const double *st = stat + (size_t)s * kStat, *dy = dyn + (size_t)s * kDyn;
        const double dx = x - st[3 * q], dyy = y - st[3 * q + 1], dz = z - st[3 * q + 2];
        const double r2[1] = {dx * dx + dyy * dyy + dz * dz};
        double ri[1];
        rsqrt3_n<1>(r2, ri);
        const double dn = dx * st[18] + dyy * st[19] + dz * st[20];
        acc = fma(ri[0], dy[6 + q], fma(-dn * (ri[0] * (ri[0] * ri[0])), dy[q], acc));
    }
    const double tot = block_sum(acc, sh);
    if (threadIdx.x == 0) out[k] = tot * kInv4Pi;
}

// Solid angle subtended by each triangle at point k (Van Oosterom-Strackee);
// the sum is 4 pi for points inside a closed outward-oriented surface.
__global__ __launch_bounds__(kRedBlock) void k_solid_angle(int T, int chunk, const double *__restrict__ pts,
                                                           const double *__restrict__ xyz,
                                                           const int32_t *__restrict__ tri, double *__restrict__ part)
{
    __shared__ double sh[kRedBlock];
    int k = blockIdx.x, c = blockIdx.y;
    double x = pts[3 * k], y = pts[3 * k + 1], z = pts[3 * k + 2];
    int s0 = c * chunk, s1 = min(T, s0 + chunk);
    double acc = 0.0;
    for (int s = s0 + threadIdx.x; s < s1; s += kRedBlock) {
        double a[3], b[3], e[3];
        for (int m = 0; m < 3; ++m) {
            a[m] = xyz[3 * tri[3 * s] + m] - (m == 0 ? x : m == 1 ? y : z);
            b[m] = xyz[3 * tri[3 * s + 1] + m] - (m == 0 ? x : m == 1 ? y : z);
            e[m] = xyz[3 * tri[3 * s + 2] + m] - (m == 0 ? x : m == 1 ? y : z);
        }
        double la = sqrt(a[0] * a[0] + a[1] * a[1] + a[2] * a[2]);
        double lb = sqrt(b[0] * b[0] + b[1] * b[1] + b[2] * b[2]);
        double le = sqrt(e[0] * e[0] + e[1] * e[1] + e[2] * e[2]);
        double det = a[0] * (b[1] * e[2] - b[2] * e[1]) - a[1] * (b[0] * e[2] - b[2] * e[0]) +
                     a[2] * (b[0] * e[1] - b[1] * e[0]);
        double ab = a[0] * b[0] + a[1] * b[1] + a[2] * b[2];
        double ae = a[0] * e[0] + a[1] * e[1] + a[2] * e[2];
        double be = b[0] * e[0] + b[1] * e[1] + b[2] * e[2];
        acc += 2.0 * atan2(det, la * lb * le + ab * le + ae * lb + be * la);
    }
    double tot = block_sum(acc, sh);
    if (threadIdx.x == 0) part[(size_t)k * gridDim.y + c] = tot;
}

static int red_chunks(int T) { return T < 4096 ? 1 : (T + 4095) / 4096; }

// Source chunks of the reaction potential at npts points: about four wavefronts
// per SIMD, chunks of at least 8 triangles, and at most the allocation-free entry
// point's scratch for the partial sums (a function of T and npts alone, so both
// entry points sum alike)
int reaction_chunks(int T, int npts)
{
    if (T <= kPointTriangles && npts <= kPointPoints) return 1;   // k_reaction_point
    const int waves = (npts + 63) / 64;
    const int most = std::max(1, (int)(kNoAllocScratchDoubles / (size_t)npts));
    return std::max(1, std::min({4096 / waves, T / 8, most}));
}

// part: npts x reaction_chunks partial sums; out: npts potentials
void launch_reaction(DevMesh &d, int npts, const double *pts, double *part, double *out)
{
    const int T = d.hm.T, C = reaction_chunks(T, npts), chunk = (T + C - 1) / C;
    if (T <= kPointTriangles && npts <= kPointPoints) {
        hipLaunchKernelGGL(k_reaction_point, dim3(npts), dim3(kRedBlock), 0, d.stream, T, pts, d.stat64, d.dyn64, out);
        HIPCHECK(hipGetLastError());
        return;
    }
    const long long waves = (long long)((npts + 63) / 64) * C;
    hipLaunchKernelGGL(k_reaction, dim3((unsigned)((waves + 3) / 4)), dim3(256), 0, d.stream, T, npts, C, chunk, pts,
                       d.stat64, d.dyn64, part);
    hipLaunchKernelGGL(k_reaction_finish, dim3((npts + 3) / 4), dim3(256), 0, d.stream, npts, C, part, out);
    HIPCHECK(hipGetLastError());
}

void launch_inside_test(DevMesh &d, int nq, const double *qpts, double *out_part)
{
    int T = d.hm.T, C = red_chunks(T);
    int chunk = (T + C - 1) / C;
    hipLaunchKernelGGL(k_solid_angle, dim3(nq, C), dim3(kRedBlock), 0, d.stream, T, chunk, qpts, d.xyz, d.tri,
                       out_part);
    HIPCHECK(hipGetLastError());
}

int reduction_chunks(int T) { return red_chunks(T); }

// ------------------------------------------- reaction potential, no allocation
// Partial sums (point x source chunk) of pb_mesh_reaction_potential_noalloc
// live in this file-scope array: one copy per device, held until the process
// ends.  Host code never uses the array's name as an address; it uses the
// device address resolved once per device by noalloc_scratch().
static __device__ __align__(256) double scratch[kNoAllocScratchDoubles];

static double *noalloc_scratch()
{
    constexpr int kMaxDevices = 64;
    static std::mutex mu;
    static double *addr[kMaxDevices] = {};
    int dev = -1;
    HIPCHECK(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) fail(PB_E_DEVICE, "device index out of range for the scratch table");
    std::lock_guard<std::mutex> lk(mu);
    if (!addr[dev]) {
        void *p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p)
            fail(PB_E_DEVICE, std::string("hipGetSymbolAddress(scratch): ") + hipGetErrorString(e));
        addr[dev] = (double *)p;
    }
    return addr[dev];
}

void reaction_potential_noalloc(DevMesh &d, const double *traces, int npts, const double *pts, double *out,
                                hipStream_t stream)
{
    const int C = red_chunks(d.hm.T);
    if ((size_t)npts * (size_t)C > kNoAllocScratchDoubles)
        fail(PB_E_INVALID_ARG, "npts x source chunks (" + std::to_string((size_t)npts * C) +
                                   ") exceeds the scratch of " + std::to_string(kNoAllocScratchDoubles) + " doubles");
    double *part = noalloc_scratch();
    struct StreamSwap {
        DevMesh &d;
        hipStream_t keep;
        StreamSwap(DevMesh &dm, hipStream_t s) : d(dm), keep(dm.stream) { if (s) d.stream = s; }
        ~StreamSwap() { d.stream = keep; }
    } swap(d, stream);
    launch_source_prep(d, traces, false);
    launch_reaction(d, npts, pts, part, out);
}

}  // namespace pbm
