// Field off the surface and winding numbers of a mesh.
//
// Field (Sec. 2, Eq. "representation"): outside the body the total field is
// the incident plane wave plus [SLP_ext psi_ext - DLP_ext phi_ext](x), inside
// it is [SLP_int psi_int - DLP_int phi_int](x), with
//   [SLP psi](x) = int G(x, y) psi(y) dy,  [DLP phi](x) = int dG/dn(y) phi(y) dy,
//   G = exp(i k r) / (4 pi r),  dG/dn(y) = exp(i k r) (i k r - 1) ((y - x).n_y) / (4 pi r^3).
// The potentials are the P1 functions of the solve's unknowns: with the
// multiple-traces system as printed (Sec. 3.3) p = -v and dp/dn = -w on each
// mesh, so phi_ext = v_ext, psi_ext = w_ext (phi_ext = -gamma_D p,
// psi_ext = -gamma_N p, Eq. "potentials:traces") and phi_int = -v_int,
// psi_int = -w_int.  Each triangle integral is the 6-point rule of the
// regular assembly; points near a mesh get that rule's nearly-singular error.
//
//   field_density_kernel   per quadrature point and right-hand side: area *
//                          weight * density (P1 interpolation), both
//                          potentials, with their signs; both meshes.
//   field_partial_kernel   one lane per point (sorted by region), one wave per
//                          (64 points, chunk of triangles), both regions in
//                          one launch; a triangle's data is the same for the
//                          whole wave and comes through the scalar unit; up
//                          to 16 right-hand sides share the kernel's values;
//                          FP64 throughout; per-chunk partial sums.
//   field_combine_kernel   fixed-order sum of the chunk partials, 1 / (4 pi),
//                          the incident wave for exterior points, written at
//                          the point's place in the caller's order.
//   winding kernels        sum over triangles of the signed solid angle
//                          (Van Oosterom and Strackee, 1983) over 4 pi, the
//                          same chunked structure: 1 inside a closed outward
//                          mesh, 0 outside.
#include <algorithm>
#include <cmath>
#include <vector>

#include "internal.h"
#include "phase.h"
#include "rule6.h"

namespace bemtx {

namespace {

constexpr int FLD_PB = 64;      // points per wave, one wave per workgroup
constexpr int FLD_WG = 8192;    // target workgroups per launch and region (points x triangle chunks)
constexpr int FLD_TMIN = 16;    // triangles per chunk, at least
constexpr int FLD_RMAX = 16;    // right-hand sides per launch, at most

// One region of a field call: its mesh, its points (sorted by region) and its
// chunks of tpc triangles.
struct FieldRegion {
    const TriGeo *geo;
    const int32_t *tri;
    const double4 *dens;     // [nt][6][R]: area * w_q * (psi, phi)(y_q) (sign folded in)
    const double *pts;
    const int32_t *dst;      // place of each point in the caller's order
    double2 *part;           // [chunk][R][np]
    double k, kim, sgn;
    int64_t phi, psi;        // offsets of the two potentials in an unknown vector
    int nt, np, nchunk, tpc, npb;
};
struct FieldArgs {
    FieldRegion reg[2];      // exterior, interior
    const double2 *x;        // unknowns in internal numbering, [nrhs][n]
    int64_t n;
    int nrhs;                // right-hand sides of this launch (at most the kernel's R)
};

// grid (ceil(6 (nt_0 + nt_1) / 256), R)
__global__ __launch_bounds__(256) void field_density_kernel(FieldArgs A, int R)
{
    const int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int r = blockIdx.y;
    const int64_t n0 = 6 * (int64_t)A.reg[0].nt;
    const FieldRegion &g = A.reg[u < n0 ? 0 : 1];
    const int64_t v = u < n0 ? u : u - n0;
    if (v >= 6 * (int64_t)g.nt) return;
    const int64_t t = v / 6;
    const int q = (int)(v - 6 * t);
    double pr = 0, pi = 0, sr = 0, si = 0;
    if (r < A.nrhs) {
        const double2 *x = A.x + r * A.n;
        const double W = g.sgn * g.geo[t].area * r6_w(q);
        for (int a = 0; a < 3; ++a) {
            const double b = r6_bary(q, a);
            const int64_t i = g.tri[3 * t + a];
            const double2 ph = x[g.phi + i], ps = x[g.psi + i];
            pr += b * ph.x; pi += b * ph.y;
            sr += b * ps.x; si += b * ps.y;
        }
        pr *= W; pi *= W; sr *= W; si *= W;
    }
    const_cast<double4 *>(g.dens)[v * R + r] = make_double4(sr, si, pr, pi);
}

// The contribution of one triangle at the point x to the sums of R
// right-hand sides: sum over its quadrature points of G psi - dG/dn phi,
// times 4 pi.  (y - x).n is the same for every y of the triangle, but is taken at
// each: next to a facet the nearest point, which counts most, then has the
// smallest error (one value from the centroid made fields near a body 4 % and more
// further off than the sums without BASE; 873 against 884 us on 100 x 100 points).  BASE: the
// phase from the triangle's centroid, exp(i k r) = exp(i k r0) exp(i k (r - r0))
// with |k (r - r0)| <= k rho <= kShortPhase (short polynomials instead of a reduction
// per point); the factor exp(i k r0) is applied to the triangle's sums for
// few right-hand sides and to the values for many.
template <bool CK, bool BASE, int R>
__device__ inline void field_triangle(const TriGeo &g, const double4 *__restrict__ dens, double x0, double x1, double x2,
                                      double k, double kim, double (&ar)[R], double (&ai)[R])
{
    constexpr bool late = R <= 4;   // factors on the triangle's sums
    const double c0 = g.c[0] - x0, c1 = g.c[1] - x1, c2 = g.c[2] - x2;
    double er = 1.0, ei = 0.0, kr0 = 0.0;
    if constexpr (BASE) {
        kr0 = k * sqrt(c0 * c0 + c1 * c1 + c2 * c2);
        phase_sincos(kr0, &ei, &er);
    }
    double tr[R], ti[R];   // the triangle's sums without exp(i k r0) (late)
#pragma unroll
    for (int r = 0; r < R; ++r) tr[r] = ti[r] = 0.0;
#pragma unroll
    for (int q = 0; q < 6; ++q) {
        const double d0 = g.qp[q][0] - x0, d1 = g.qp[q][1] - x1, d2 = g.qp[q][2] - x2;   // y - x
        const double r2 = d0 * d0 + d1 * d1 + d2 * d2;
        const double rinv = rsqrt_pos(r2);
        const double rr = r2 * rinv, kr = k * rr;
        double sn, cs;
        if constexpr (BASE) small_sincos<true>(fma(k, rr, -kr0), sn, cs);
        else phase_sincos(kr, &sn, &cs);
        double gr = cs * rinv, gi = sn * rinv;                            // exp(ikr) / r
        const double s = -(d0 * g.n[0] + d1 * g.n[1] + d2 * g.n[2]) * (rinv * rinv);
        double fr, fi;                                                    // -exp(ikr)(ikr - 1)(y-x).n / r^3
        if constexpr (CK) {
            const double dmp = exp(-kim * rr), am = -1.0 - kim * rr;
            gr *= dmp; gi *= dmp;
            fr = (gr * am - gi * kr) * s;
            fi = (gr * kr + gi * am) * s;
        } else {
            fr = (-gr - gi * kr) * s;
            fi = (gr * kr - gi) * s;
        }
        if constexpr (BASE && !late) {
            const double g0 = gr, f0 = fr;
            gr = g0 * er - gi * ei; gi = g0 * ei + gi * er;
            fr = f0 * er - fi * ei; fi = f0 * ei + fi * er;
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const double4 w = dens[q * R + r];
            double &zr = late ? tr[r] : ar[r], &zi = late ? ti[r] : ai[r];
            zr = fma(-fi, w.w, fma(fr, w.z, fma(-gi, w.y, fma(gr, w.x, zr))));
            zi = fma(fi, w.z, fma(fr, w.w, fma(gi, w.x, fma(gr, w.y, zi))));
        }
    }
    if constexpr (late)
#pragma unroll
        for (int r = 0; r < R; ++r) {
            ar[r] = fma(-ti[r], ei, fma(tr[r], er, ar[r]));
            ai[r] = fma(ti[r], er, fma(tr[r], ei, ai[r]));
        }
}

template <bool CK, int R>
__device__ inline void field_chunk(const FieldRegion &g, int chunk, int i, bool live)
{
    const int t0 = chunk * g.tpc, t1 = min(g.nt, t0 + g.tpc);
    const double x0 = live ? g.pts[3 * i] : 0.0, x1 = live ? g.pts[3 * i + 1] : 0.0, x2 = live ? g.pts[3 * i + 2] : 0.0;
    const TriGeo *__restrict__ geo = g.geo;
    const double4 *__restrict__ dens = g.dens;
    double ar[R], ai[R];
#pragma unroll
    for (int r = 0; r < R; ++r) ar[r] = ai[r] = 0.0;
#pragma unroll 1
    for (int t = t0; t < t1; ++t) {
        if (g.k * geo[t].rho <= kShortPhase)
            field_triangle<CK, true, R>(geo[t], dens + (int64_t)6 * R * t, x0, x1, x2, g.k, g.kim, ar, ai);
        else
            field_triangle<CK, false, R>(geo[t], dens + (int64_t)6 * R * t, x0, x1, x2, g.k, g.kim, ar, ai);
    }
    if (live)
#pragma unroll
        for (int r = 0; r < R; ++r) g.part[((int64_t)chunk * R + r) * g.np + i] = make_double2(ar[r], ai[r]);
}

// Bound by FP64 issue: about 65 vector operations per (point, quadrature
// point) for one right-hand side and 8 more for each further one.  10,000
// points on meshes of 5,120 + 3,920 triangles: 861 -> 634 us (triangles
// staged in LDS, a phase reduction per point, one launch per region before);
// 2,867 points x 12 right-hand sides on 2,420 + 3,380 triangles, absorbing:
// 4,180 us in 24 launches -> 571 us in one.
// part[chunk][r][i] of both regions.  Workgroups of region 0 first; a
// region's chunks are outermost, so that neighbouring workgroups read the
// same triangles.  CK: the interior wavenumber is complex (an absorbing
// medium), G = exp(i k r - kim r) / (4 pi r).
template <bool CK, int R>
__global__ __launch_bounds__(FLD_PB, R == 16 ? 2 : (R == 12 ? 3 : 4)) void field_partial_kernel(FieldArgs A)
{
    int b = blockIdx.x;
    const int n0 = A.reg[0].npb * A.reg[0].nchunk;
    const bool inner = b >= n0;
    const FieldRegion &g = A.reg[inner ? 1 : 0];
    if (inner) b -= n0;
    const int chunk = b / g.npb, i = (b - chunk * g.npb) * FLD_PB + threadIdx.x;
    if (CK && inner) field_chunk<true, R>(g, chunk, i, i < g.np);
    else field_chunk<false, R>(g, chunk, i, i < g.np);
}

struct FieldSources {
    double d[FLD_RMAX][3];
};

// grid (ceil((np_0 + np_1) / 256), nrhs)
__global__ __launch_bounds__(256) void field_combine_kernel(FieldArgs A, int R, FieldSources src, int kind, double k_ext,
                                                            int64_t npts, double2 *__restrict__ field)
{
    const int u = blockIdx.x * blockDim.x + threadIdx.x, r = blockIdx.y;
    const bool ext = u < A.reg[0].np;
    const FieldRegion &g = A.reg[ext ? 0 : 1];
    const int i = ext ? u : u - A.reg[0].np;
    if (i >= g.np) return;
    double sr = 0.0, si = 0.0;
    const double2 *p = g.part + (int64_t)r * g.np + i;
    const int64_t step = (int64_t)R * g.np;
#pragma unroll 8
    for (int c = 0; c < g.nchunk; ++c) {
        const double2 v = p[c * step];
        sr += v.x;
        si += v.y;
    }
    sr *= kInv4Pi;
    si *= kInv4Pi;
    const double p0 = g.pts[3 * i], p1 = g.pts[3 * i + 1], p2 = g.pts[3 * i + 2];
    const double d0 = src.d[r][0], d1 = src.d[r][1], d2 = src.d[r][2];
    if (ext && kind == 0) {   // plane wave exp(i k d.x)
        double sn, cs;
        phase_sincos(k_ext * (d0 * p0 + d1 * p1 + d2 * p2), &sn, &cs);
        sr += cs;
        si += sn;
    } else if (ext) {         // point source exp(i k r) / (4 pi r), r = |x - x0|
        const double R0 = p0 - d0, R1 = p1 - d1, R2 = p2 - d2;
        const double rr = sqrt(R0 * R0 + R1 * R1 + R2 * R2);
        double sn, cs;
        phase_sincos(k_ext * rr, &sn, &cs);
        sr += cs * kInv4Pi / rr;
        si += sn * kInv4Pi / rr;
    }
    field[r * npts + g.dst[i]] = make_double2(sr, si);
}

// length from its square; 0 for 0
__device__ inline double length_of(double r2) { return r2 * rsqrt_pos(fmax(r2, 1e-300)); }

// atan2(num, den).  The half solid angle of all triangles but those next to the
// point is small: |num| <= den / 8 takes the quotient (hardware reciprocal, one Newton
// step, one correction of the quotient) and q + q z p(z), z = q^2, p minimax as in
// phase.h with errors below 2e-18 relative to q.  den is bounded so that its reciprocal is
// neither 0 nor infinite; a point far enough for the lengths' product to overflow, a corner
// (0, 0) and NaN take the library function.
__device__ inline double half_angle(double num, double den)
{
    if (!(fabs(num) <= 0.125 * den && den > 1e-290 && den < 1e290)) return atan2(num, den);
    double y = __builtin_amdgcn_rcp(den);
    y = fma(y, fma(-den, y, 1.0), y);
    double q = num * y;
    q = fma(fma(-den, q, num), y, q);
    const double z = q * q;
    double p = fma_const(0.07342729565358729, z, -0.0908360288044579);
    p = fma_const(p, z, 0.11111035635624597);
    p = fma_const(p, z, -0.14285713890803944);
    p = fma_const(p, z, 0.19999999999049253);
    p = fma_const(p, z, -0.3333333333333257);
    return fma(q * z, p, q);
}

// part[chunk][i] = half the chunk's solid angle, the sum over its triangles of
// atan2(num, den).  Bound by FP64 issue; a call for 10,000 points and 5,120
// triangles takes 303 us with the library's arctangent for every triangle, 177 us so.
__global__ __launch_bounds__(FLD_PB) void winding_partial_kernel(int np, const double *__restrict__ pts, int nt,
                                                                 int tpc, int npb, const TriGeo *__restrict__ geo,
                                                                 double *__restrict__ part)
{
    const int chunk = blockIdx.x / npb, i = (blockIdx.x - chunk * npb) * FLD_PB + threadIdx.x;
    const int t0 = chunk * tpc, t1 = min(nt, t0 + tpc);
    const bool live = i < np;
    const double x0 = live ? pts[3 * (int64_t)i] : 0.0, x1 = live ? pts[3 * (int64_t)i + 1] : 0.0,
                 x2 = live ? pts[3 * (int64_t)i + 2] : 0.0;
    double acc = 0.0;
#pragma unroll 1
    for (int t = t0; t < t1; ++t) {
        const double(*v)[3] = geo[t].p;
        const double a0 = v[0][0] - x0, a1 = v[0][1] - x1, a2 = v[0][2] - x2;
        const double b0 = v[1][0] - x0, b1 = v[1][1] - x1, b2 = v[1][2] - x2;
        const double c0 = v[2][0] - x0, c1 = v[2][1] - x1, c2 = v[2][2] - x2;
        const double la = length_of(a0 * a0 + a1 * a1 + a2 * a2), lb = length_of(b0 * b0 + b1 * b1 + b2 * b2),
                     lc = length_of(c0 * c0 + c1 * c1 + c2 * c2);
        const double num = a0 * (b1 * c2 - b2 * c1) + a1 * (b2 * c0 - b0 * c2) + a2 * (b0 * c1 - b1 * c0);
        const double den = la * lb * lc + (a0 * b0 + a1 * b1 + a2 * b2) * lc + (a0 * c0 + a1 * c1 + a2 * c2) * lb +
                           (b0 * c0 + b1 * c1 + b2 * c2) * la;
        acc += half_angle(num, den);
    }
    if (live) part[(int64_t)chunk * np + i] = acc;
}

// w[i] = the chunks' sum over 2 pi.  With the errors of its additions (exact, by
// two-sum) added at the end: up to a few hundred chunks of a closed body add to
// 2 pi or cancel, and plain addition was the largest error of the result.
__global__ __launch_bounds__(256) void winding_combine_kernel(int np, int nchunk, const double *__restrict__ part,
                                                              double *__restrict__ w)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= np) return;
    double s = 0.0, e = 0.0;
#pragma unroll 8
    for (int c = 0; c < nchunk; ++c) {
        const double v = part[(int64_t)c * np + i], t = s + v, d = t - s;
        e += (s - (t - d)) + (v - d);
        s = t;
    }
    w[i] = 2.0 * (s + e) * kInv4Pi;
}

// Triangle chunks for np points: about FLD_WG workgroups, at least FLD_TMIN
// triangles per chunk.  lean: the fewer chunks of 256-point workgroups with
// at least 128 triangles each, where the partial sums have to be small.
void chunking(int64_t np, int nt, bool lean, int &nchunk, int &tpc)
{
    const int64_t pblocks = lean ? (np + 255) / 256 : (np + FLD_PB - 1) / FLD_PB;
    const int64_t tmin = lean ? 128 : FLD_TMIN, wg = lean ? FLD_WG / (256 / FLD_PB) : FLD_WG;
    const int64_t maxc = std::max<int64_t>(1, (nt + tmin - 1) / tmin);
    nchunk = (int)std::min<int64_t>(maxc, std::max<int64_t>(1, wg / std::max<int64_t>(1, pblocks)));
    tpc = (nt + nchunk - 1) / nchunk;
    nchunk = (nt + tpc - 1) / tpc;
}

// Right-hand sides per launch for the `left` that remain: the smallest built
// width that holds them (unused ones have zero densities), at most what
// keeps the densities and partial sums of a launch within 1 GiB (one at the
// least).
int field_width(int left, size_t bytes_per_rhs)
{
    const size_t cap = std::max<size_t>(1, (size_t(1) << 30) / std::max<size_t>(1, bytes_per_rhs));
    int w = 1;
    for (int c : {1, 2, 4, 8, 12, 16})
        if ((size_t)c <= cap) {
            w = c;
            if (c >= left) break;
        }
    return w;
}

template <bool CK> void launch_partial(const KTimer &kt, int R, unsigned wg, hipStream_t st, const FieldArgs &A)
{
    switch (R) {
    case 1: launch_k(kt, field_partial_kernel<CK, 1>, dim3(wg), dim3(FLD_PB), 0, st, A); break;
    case 2: launch_k(kt, field_partial_kernel<CK, 2>, dim3(wg), dim3(FLD_PB), 0, st, A); break;
    case 4: launch_k(kt, field_partial_kernel<CK, 4>, dim3(wg), dim3(FLD_PB), 0, st, A); break;
    case 8: launch_k(kt, field_partial_kernel<CK, 8>, dim3(wg), dim3(FLD_PB), 0, st, A); break;
    case 12: launch_k(kt, field_partial_kernel<CK, 12>, dim3(wg), dim3(FLD_PB), 0, st, A); break;
    default: launch_k(kt, field_partial_kernel<CK, 16>, dim3(wg), dim3(FLD_PB), 0, st, A); break;
    }
}

}  // namespace

bem_status launch_to_internal(const bem_problem *p, const double2 *x_caller, double2 *x_int, int nrhs, hipStream_t st);

namespace {

// The points and chunks of region `only` (-1: of both) with nothing in the other.
void set_regions(FieldArgs &A, const bem_problem *p, const int np[2], int only, bool lean)
{
    for (int m = 0; m < 2; ++m) {
        FieldRegion &g = A.reg[m];
        g.np = only < 0 || only == m ? np[m] : 0;
        g.nt = g.np > 0 ? (int)(m == 0 ? p->ext : p->inte)->h.nt : 0;   // no points: no densities
        chunking(g.np, std::max(1, g.nt), lean, g.nchunk, g.tpc);
        g.npb = (g.np + FLD_PB - 1) / FLD_PB;
    }
}
size_t dens_bytes(const FieldRegion &g) { return (size_t)g.nt * 6 * sizeof(double4); }      // of one right-hand side
size_t part_bytes(const FieldRegion &g) { return (size_t)g.nchunk * g.np * sizeof(double2); }

// The launches of A's regions for its right-hand sides, the kernel's width R.
bem_status launch_regions(bem_problem *p, FieldArgs &A, int R, const FieldSources &src, int64_t npts, double2 *field,
                          DevMem &dens, DevMem &part, hipStream_t st)
{
    FieldRegion *g = A.reg;
    bem_status s = dev_alloc(p->ctx, dens, R * (dens_bytes(g[0]) + dens_bytes(g[1])));
    if (!s) s = dev_alloc(p->ctx, part, R * (part_bytes(g[0]) + part_bytes(g[1])));
    if (s) return s;
    g[0].dens = dens.as<double4>();
    g[1].dens = dens.as<double4>() + R * dens_bytes(g[0]) / sizeof(double4);
    g[0].part = part.as<double2>();
    g[1].part = part.as<double2>() + R * part_bytes(g[0]) / sizeof(double2);
    const int64_t nd = 6 * ((int64_t)g[0].nt + g[1].nt), np = (int64_t)g[0].np + g[1].np;
    hipLaunchKernelGGL(field_density_kernel, dim3((unsigned)((nd + 255) / 256), R), dim3(256), 0, st, A, R);
    BEM_HIP(hipGetLastError());
    {
        KTimer kt(p->ctx, K_FIELD);
        const unsigned wg = (unsigned)(g[0].npb * g[0].nchunk + g[1].npb * g[1].nchunk);
        if (p->k_int_im != 0.0) launch_partial<true>(kt, R, wg, st, A);
        else launch_partial<false>(kt, R, wg, st, A);
        BEM_HIP(hipGetLastError());
    }
    hipLaunchKernelGGL(field_combine_kernel, dim3((unsigned)((np + 255) / 256), A.nrhs), dim3(256), 0, st, A, R, src,
                       p->incident, p->k_ext, npts, field);
    BEM_HIP(hipGetLastError());
    return BEM_OK;
}

}  // namespace

// Fields of nrhs right-hand sides at the points of both regions: pts [np_0 +
// np_1][3] and dst on the device, exterior points first; x: the unknowns in
// caller numbering (device, [nrhs][n]); dirs (host); field [nrhs][npts].  Work
// buffers: the unknowns of one launch's right-hand sides in internal
// numbering, their densities and partial sums.  Where these do not fit the
// memory, one right-hand side at a time; where that does not, one region at a
// time in few chunks.
bem_status launch_field(bem_problem *p, const int np[2], const double *pts, const int32_t *dst, const double2 *x,
                        const double *dirs, int nrhs, double2 *field, DevMem &xint, DevMem &dens, DevMem &part,
                        hipStream_t st)
{
    const bem_mesh *ms[2] = {p->ext, p->inte};
    const int64_t ne = p->ext->h.nv, ni = p->inte->h.nv, n = 2 * ne + 2 * ni, npts = (int64_t)np[0] + np[1];
    FieldArgs A;
    A.n = n;
    for (int m = 0; m < 2; ++m) {
        FieldRegion &g = A.reg[m];
        g.geo = ms[m]->d.geo.as<TriGeo>();
        g.tri = ms[m]->d.tri.as<int32_t>();
        g.pts = pts + (m == 0 ? 0 : (size_t)3 * np[0]);
        g.dst = dst + (m == 0 ? 0 : np[0]);
        g.k = m == 0 ? p->k_ext : p->k_int;
        g.kim = m == 0 ? 0.0 : p->k_int_im;
        g.sgn = m == 0 ? 1.0 : -1.0;
        g.phi = m == 0 ? 0 : 2 * ne;
        g.psi = m == 0 ? ne : 2 * ne + ni;
    }
    int most = nrhs;
    bool lean = false;
    for (int r0 = 0; r0 < nrhs;) {
        set_regions(A, p, np, -1, false);
        const int R = field_width(std::min(most, nrhs - r0), std::max(dens_bytes(A.reg[0]) + dens_bytes(A.reg[1]),
                                                                      part_bytes(A.reg[0]) + part_bytes(A.reg[1])));
        A.nrhs = std::min(R, nrhs - r0);
        FieldSources src{};
        for (int r = 0; r < A.nrhs; ++r)
            for (int c = 0; c < 3; ++c) src.d[r][c] = dirs[3 * (r0 + r) + c];
        bem_status s = dev_alloc(p->ctx, xint, (size_t)R * n * sizeof(double2));
        if (!s) {
            s = launch_to_internal(p, x + (int64_t)r0 * n, xint.as<double2>(), A.nrhs, st);
            if (s) return s;
            A.x = xint.as<double2>();
            for (int only = lean ? 0 : -1; only < (lean ? 2 : 0) && !s; ++only) {
                if (lean && np[only] == 0) continue;
                if (lean) set_regions(A, p, np, only, true);
                s = launch_regions(p, A, R, src, npts, field + (int64_t)r0 * npts, dens, part, st);
            }
        }
        if (s == BEM_E_OOM && !lean) {   // little memory left
            xint.release();
            dens.release();
            part.release();
            lean = R == 1;
            most = 1;
            continue;
        }
        if (s) return s;
        r0 += A.nrhs;
    }
    return BEM_OK;
}

bem_status launch_winding(const bem_mesh *m, int np, const double *pts, double *w, DevMem &part, hipStream_t st)
{
    if (np == 0) return BEM_OK;
    const int nt = (int)m->h.nt;
    int nchunk, tpc;
    chunking(np, nt, false, nchunk, tpc);
    bem_status s = dev_alloc(m->ctx, part, (size_t)nchunk * np * sizeof(double));
    if (s == BEM_E_OOM) {   // little memory left
        chunking(np, nt, true, nchunk, tpc);
        s = dev_alloc(m->ctx, part, (size_t)nchunk * np * sizeof(double));
    }
    if (s) return s;
    const int npb = (np + FLD_PB - 1) / FLD_PB;
    hipLaunchKernelGGL(winding_partial_kernel, dim3((unsigned)npb * nchunk), dim3(FLD_PB), 0, st, np, pts, nt, tpc, npb,
                       m->d.geo.as<TriGeo>(), part.as<double>());
    BEM_HIP(hipGetLastError());
    hipLaunchKernelGGL(winding_combine_kernel, dim3((np + 255) / 256), dim3(256), 0, st, np, nchunk,
                       part.as<double>(), w);
    BEM_HIP(hipGetLastError());
    return BEM_OK;
}

}  // namespace bemtx
