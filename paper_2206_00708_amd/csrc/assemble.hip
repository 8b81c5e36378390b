// Galerkin P1 assembly of the Helmholtz boundary integral operators
// V (kernel G), K (dG/dn_y), T (dG/dn_x) and D (hypersingular, integrated by
// parts) on one triangle mesh, G(x,y) = exp(i k |x-y|) / (4 pi |x-y|)
// (Sec. 2.1, Sec. 2.4), in FP64 on gfx950.
//
//   geometry_kernel   per-triangle table: the six points of the order-four
//                     rule, unit normal and plane, area, P1 surface curls,
//                     vertices.
//   regular_tiles     triangle pairs that share no vertex, order-four rule
//                     (6 x 6 points, Sec. 5.1).  One workgroup per unordered
//                     pair of locality blocks (16 x 16 triangles), one
//                     triangle pair per thread; V, K, T and the scalar sum of
//                     G are reduced in registers, D follows from them
//                     (curl.curl S - k^2 n.n V).  The 9 entries of each pair
//                     are summed per vertex slot through LDS in a fixed order
//                     (runs of slot-sorted corners) and the block-pair tile
//                     is written once.  Because the
//                     regular rule is symmetric in (x, y), the tile of
//                     (b1, b2) also provides (b2, b1): V, D transpose to
//                     themselves and K, T into each other.
//   gather_tiles      dense entries (i, j) and (j, i) = one fixed-order sum
//                     of the tile entries of the blocks containing i and j.
//   singular_pairs    ordered pairs sharing 3 / 2 / 1 vertices: Sauter-Schwab
//                     regularising maps of [0,1]^4 with ng^4 Gauss points per
//                     region (6 / 5 / 2 regions); 16 lanes per pair, or a wave.
//   near_scatter      adds the singular contributions of each touched entry
//                     in a fixed order.
// Every entry is produced by a fixed sequence of additions, so the result is
// bitwise reproducible run to run.
#include <cmath>

#include "dpp.h"
#include "internal.h"
#include "phase.h"
#include "rule6.h"

namespace bemtx {

namespace {


__device__ inline double dot3(const double *a, const double *b) { return a[0] * b[0] + a[1] * b[1] + a[2] * b[2]; }

}  // namespace

__global__ void geometry_kernel(const double *__restrict__ xyz, const int32_t *__restrict__ tri, int nt,
                                TriGeo *__restrict__ geo, TriGeoF *__restrict__ geof)
{
    int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= nt) return;
    TriGeo g;
    for (int a = 0; a < 3; ++a)
        for (int c = 0; c < 3; ++c) g.p[a][c] = xyz[3 * (int64_t)tri[3 * t + a] + c];
    double e1[3], e2[3];
    for (int c = 0; c < 3; ++c) { e1[c] = g.p[1][c] - g.p[0][c]; e2[c] = g.p[2][c] - g.p[0][c]; }
    double cr[3] = {e1[1] * e2[2] - e1[2] * e2[1], e1[2] * e2[0] - e1[0] * e2[2], e1[0] * e2[1] - e1[1] * e2[0]};
    double len = sqrt(dot3(cr, cr));
    g.area = 0.5 * len;
    for (int c = 0; c < 3; ++c) g.n[c] = cr[c] / len;
    g.off = dot3(g.n, g.p[0]);
    for (int a = 0; a < 3; ++a)
        for (int c = 0; c < 3; ++c) g.curl[a][c] = (g.p[(a + 1) % 3][c] - g.p[(a + 2) % 3][c]) / len;
#pragma unroll
    for (int q = 0; q < 6; ++q)
        for (int c = 0; c < 3; ++c)
            g.qp[q][c] = r6_bary(q, 0) * g.p[0][c] + r6_bary(q, 1) * g.p[1][c] + r6_bary(q, 2) * g.p[2][c];
    for (int c = 0; c < 3; ++c) g.c[c] = (g.p[0][c] + g.p[1][c] + g.p[2][c]) / 3.0;
    g.rho = 0.0;
    for (int q = 0; q < 6; ++q) {
        const double e[3] = {g.qp[q][0] - g.c[0], g.qp[q][1] - g.c[1], g.qp[q][2] - g.c[2]};
        g.rho = fmax(g.rho, sqrt(dot3(e, e)));
    }
    geo[t] = g;
    TriGeoF f;
    for (int c = 0; c < 3; ++c) f.c[c] = (g.p[0][c] + g.p[1][c] + g.p[2][c]) / 3.0;
    for (int q = 0; q < 6; ++q)
        for (int c = 0; c < 3; ++c) f.dq[q][c] = (float)(g.qp[q][c] - f.c[c]);
    for (int c = 0; c < 3; ++c) f.n[c] = (float)g.n[c];
    f.area = (float)g.area;
    for (int a = 0; a < 3; ++a)
        for (int c = 0; c < 3; ++c) f.curl[a][c] = (float)g.curl[a][c];
    f.rho = (float)(g.rho * (1.0 + 1e-6));   // not below the FP64 radius
    geof[t] = f;
}

// ------------------------------------------------------------ regular pairs

struct TileArgs {
    const TriGeo *geo;
    const int32_t *tri;
    const int32_t *blk_start;
    const int32_t *blk_nslot;
    const uint8_t *slot_off;    // [nb][SLOT_OFF_LD] first slot-major rank of each slot
    const uint8_t *slot_rank;   // [nb][3 * BT] slot-major rank of each corner
    const SlotPlaces *slot_place;   // [nb][SMAX]
    int32_t nb;
    double k;
    double kim;            // imaginary part of the wavenumber (read by the absorbing instantiation only)
    double2 *scratch;      // [tile of the strip][SMAX*SMAX][op]
    int32_t b0, nrow;      // first tile row of the strip, rows
};

// tiles of assembly strip s: rows b in [strip_b[s], strip_b[s + 1]), nb - b each
inline int64_t strip_tiles(const MeshData &h, int s)
{
    int64_t n = 0;
    for (int b = h.strip_b[s]; b < h.strip_b[s + 1]; ++b) n += h.nb - b;
    return n;
}

// The tiles (b1, b2), b1 <= b2, of a strip's rows b0 .. b0 + nrow - 1: row i of the grid holds row i
// of the strip, nb - b0 - i tiles, and after it row nrow - 1 - i, so that all rows of the grid are of one
// length; a middle row fills the first part of its grid row only (false past its end).
inline dim3 tile_grid(int nb, int b0, int nrow) { return dim3(2 * (nb - b0) - (nrow - 1), (nrow + 1) / 2); }
template <class TA> __device__ inline bool tile_of(const TA &A, int &b1, int &b2)
{
    const int i = blockIdx.y, x = blockIdx.x, len = A.nb - A.b0 - i;
    b1 = A.b0 + (x < len ? i : A.nrow - 1 - i);
    b2 = b1 + (x < len ? x : x - len);
    return x < len || A.nrow - 1 - i > i;
}

// the blocks of a tile: first triangle, triangles and slots of each
struct TileBlocks {
    int b1, b2, s1, n1, s2, n2, ns1, ns2;
    int64_t at;   // the tile's place in the scratch: row by row from the strip's first
    template <class TA> __device__ TileBlocks(const TA &A, int b1_, int b2_) : b1(b1_), b2(b2_)
    {
        s1 = A.blk_start[b1];
        n1 = A.blk_start[b1 + 1] - s1;
        s2 = A.blk_start[b2];
        n2 = A.blk_start[b2 + 1] - s2;
        ns1 = A.blk_nslot[b1];
        ns2 = A.blk_nslot[b2];
        const int64_t i = b1 - A.b0;
        at = i * (A.nb - A.b0) - i * (i - 1) / 2 + (b2 - b1);
    }
};

// A tile's tables come to LDS by loads that are all in flight at once: a
// triangle's members by eight threads, then one 32-bit word per thread of
// the corners' vertices and the slot tables, in the order of TileSlots.  (One
// loop per table waits for memory in each of its turns, and at two or three
// workgroups per compute unit nothing hides that: 10,242 + 7,842 vertices
// FP64 60.2 -> 54.2 ms, mixed 37.3 -> 35.4 ms, with the tile numbers from the
// grid in place of a square root.)
struct TileSlots {
    int32_t vtx[2 * 3 * BT];        // corners' vertices
    uint8_t r1[3 * BT];             // rank of each test corner
    SlotPlaces w2[SMAX];
    uint8_t o1[SLOT_OFF_LD];        // see tile_slot_sums
};

constexpr int TW_R1 = 6 * BT, TW_W2 = TW_R1 + 3 * BT / 4, TW_O1 = TW_W2 + SMAX * (int)sizeof(SlotPlaces) / 4,
              TW_END = TW_O1 + SLOT_OFF_LD / 4;
static_assert(TW_END <= 256 && offsetof(TileSlots, r1) == 4 * TW_R1 && offsetof(TileSlots, w2) == 4 * TW_W2 &&
                  offsetof(TileSlots, o1) == 4 * TW_O1,
              "one word per thread");

template <class TA> __device__ inline uint32_t tile_slots_word(const TA &A, const TileBlocks &B, int tid)
{
    // one load for all; vertices of triangles past a block's last repeat its last
    const uint32_t *p = reinterpret_cast<const uint32_t *>(A.tri) + 3 * B.s1;
    int i = min(tid, 3 * B.n1 - 1);
    if (tid >= 3 * BT) { p = reinterpret_cast<const uint32_t *>(A.tri) + 3 * B.s2; i = min(tid - 3 * BT, 3 * B.n2 - 1); }
    if (tid >= TW_R1) { p = reinterpret_cast<const uint32_t *>(A.slot_rank) + B.b1 * (3 * BT / 4); i = tid - TW_R1; }
    if (tid >= TW_W2) { p = reinterpret_cast<const uint32_t *>(A.slot_place + (int64_t)B.b2 * SMAX); i = tid - TW_W2; }
    if (tid >= TW_O1) {
        p = reinterpret_cast<const uint32_t *>(A.slot_off) + B.b1 * (SLOT_OFF_LD / 4);
        i = min(tid, TW_END - 1) - TW_O1;
    }
    return p[i];
}

// The pair (test triangle t1, trial triangle t2) has a place in the tile and shares no vertex.
__device__ inline bool tile_pair_active(const TileSlots &S, const TileBlocks &B, int t1, int t2)
{
    bool active = t1 < B.n1 && t2 < B.n2;
    if (active) {
        for (int a = 0; a < 3; ++a)
            for (int b = 0; b < 3; ++b) active = active && (S.vtx[3 * t1 + a] != S.vtx[3 * BT + 3 * t2 + b]);
    }
    return active;
}

// Per-slot sums of the 9 entries of every triangle pair of the tile:
// entry (q1, q2) adds the entries (a, b) of every pair whose test triangle
// has slot q1 at corner a and trial triangle slot q2 at corner b.  The
// corners of each block are ranked in slot-major order (the order of the
// block's slot lists, built on the host), so that the corners of a slot
// form a run of consecutive ranks.  The sum separates over the two blocks:
//   trial side: P[op][rank1(u)][q2] = sum over the run of trial slot q2 of
//      the entries of test corner u = (t1, a);
//   test side: entry (q1, q2) = sum over the run of test slot q1 of the P
//      rows, written to out[4 * e + op] (tile layout [entry][op]).
// Both sides add in run order, i.e. in slot-list order.
//
// A wave holds the pairs of four test triangles, so the trial side needs no
// other wave: it goes through the wave's own four staged rows (one per test
// triangle), one (operator, test corner) at a time, ordered by the LDS queue
// alone.  The P rows of all operators are kept together, so the workgroup meets
// once before the test side, whose items load the operators' rows independently.
// Rows of SMAX entries for four operators would leave room for one workgroup per
// compute unit: they are S4 entries where the trial block has that few slots
// (16 triangles of a compact patch have 13 to 17), else D follows V, K and T in a
// second pass over the same rows.
// The kernel is bound by VALU issue, so the places of a run are turned into LDS
// addresses once per tile and serve every operator; places past a run's end
// point at an entry that holds zero, and are added like the others.
constexpr int SROW = 3 * BT + 1;        // staged row: one entry per trial corner, then the zero entry
constexpr int ST_WAVE = 4 * SROW;       // staged rows of one wave
constexpr int S4 = 18;                  // trial slots up to which P holds four operators
constexpr int p_op(int row) { return 3 * BT * row + 1; }   // P rows of one operator, then the zero entry
constexpr int P_LEN = std::max(3 * p_op(SMAX), 4 * p_op(S4));
constexpr int SLOT_IT1 = (SMAX + 15) / 16;   // trial-side items per lane (16 slots x 4 rows at a time)

// Orders the wave's LDS accesses before and after it for the compiler; the
// LDS serves one wave's accesses in the order they are issued.
__device__ inline void wave_lds_order()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// The places of a run's m entries as byte offsets (m = 0: no run), the others
// at an entry that holds zero.  most: the longest run among the lanes that
// load together, so that they take the same branches.
struct RunPlaces {
    int at[LMAX], m, most;
    __device__ void set_length(int len)
    {
        m = len;
        most = __any(m > 6) ? LMAX : (__any(m > 4) ? 6 : 4);
    }
};

// the entries of a run in `base`, loaded at once, and their sum in run order
template <class C2> struct RunValues {
    C2 x[LMAX];
    __device__ void load(const C2 *base, const RunPlaces &p)
    {
        const char *b = reinterpret_cast<const char *>(base);
        auto get = [&](int v) { x[v] = *reinterpret_cast<const C2 *>(b + p.at[v]); };
#pragma unroll
        for (int v = 0; v < 4; ++v) get(v);
        if (p.most > 4) {
#pragma unroll
            for (int v = 4; v < 6; ++v) get(v);
            if (p.most > 6)
#pragma unroll
                for (int v = 6; v < LMAX; ++v) get(v);
        }
    }
    __device__ C2 sum(const RunPlaces &p) const
    {
        C2 s = x[0];
#pragma unroll
        for (int v = 1; v < 4; ++v) { s.x += x[v].x; s.y += x[v].y; }
        if (p.most > 4) {
#pragma unroll
            for (int v = 4; v < 6; ++v) { s.x += x[v].x; s.y += x[v].y; }
            if (p.most > 6)
#pragma unroll
                for (int v = 6; v < LMAX; ++v) { s.x += x[v].x; s.y += x[v].y; }
        }
        return s;
    }
};

// The slot sums of one tile.  entry(op, a, b): this thread's entry of
// operator op at corners (a, b) (called with constants once unrolled, for
// threads whose pair has a place in the tile only).  st: the workgroup's
// staged rows (ST_WAVE entries per wave); P: P_LEN entries.  o1, r1: first
// slot-major rank of each test slot and rank of each test corner; w2: per trial
// slot the places of its corners in a staged row and their number (SlotPlaces).
template <class C2, class Entry>
__device__ inline void tile_slot_sums(int tid, int n1, int n2, int ns1, int ns2, const uint8_t *o1, const uint8_t *r1,
                                      const SlotPlaces *w2, C2 *st, C2 *P, C2 *out, Entry entry)
{
    constexpr int EB = sizeof(C2);
    const int lane = tid & 63, wave = tid >> 6;
    const int t1 = tid >> 4, t2 = tid & 15;
    const bool staged = t1 < n1 && t2 < n2;
    if (lane < 4) st[wave * ST_WAVE + lane * SROW + 3 * BT] = C2{0, 0};
    const bool four = ns2 <= S4;
    const int prow = four ? S4 : SMAX, pop = p_op(prow);
    if (tid < (four ? 4 : 3)) P[tid * pop + pop - 1] = C2{0, 0};
    // A row is staged corner by corner in the order of the trial triangles (neighbouring lanes write
    // neighbouring places).  Trial-side items of this lane: row (test triangle) lane / 16, slots
    // lane % 16 and so on by 16 (neighbouring lanes write neighbouring sums)
    C2 *const mine = st + wave * ST_WAVE + (t1 & 3) * SROW + t2;
    const int row = lane >> 4, ti = 4 * wave + row;
    const int row_at = EB * (wave * ST_WAVE + row * SROW);
    RunPlaces run1[SLOT_IT1];
    int pr[3];
#pragma unroll
    for (int j = 0; j < SLOT_IT1; ++j) {
        const int q2 = (lane & 15) + 16 * j;
        const SlotPlaces w = w2[min(q2, SMAX - 1)];
        run1[j].set_length(q2 < ns2 && ti < n1 ? (int)(w.n & 255u) : 0);
#pragma unroll
        for (int v = 0; v < LMAX; ++v) run1[j].at[v] = row_at + EB * (int)(w.at[v >> 2] >> (8 * (v & 3)) & 255u);
    }
#pragma unroll
    for (int a = 0; a < 3; ++a) pr[a] = (ti < n1 ? r1[3 * ti + a] : 0) * prow + (lane & 15);
    // test-side items (q1, q2) of this thread: tid, tid + 256, ..; the places of the first before the barrier
    const float inv = 1.0f / (float)ns2;
    RunPlaces run2;
    int item;
    auto place = [&](int it) {
        const int q1 = (int)(((float)it + 0.5f) * inv), q2 = it - q1 * ns2;
        const int s0 = o1[q1];
        run2.set_length(o1[q1 + 1] - s0);
#pragma unroll
        for (int v = 0; v < LMAX; ++v) run2.at[v] = EB * (v < run2.m ? (s0 + v) * prow + q2 : pop - 1);
        item = 4 * (q1 * SMAX + q2);
    };
    auto test_side = [&](int op0, int nop) {   // operators op0 .. op0 + nop - 1 from the P rows 0 .. nop - 1
#pragma unroll 1
        for (int it = tid;;) {
            if (it < ns1 * ns2) {
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (q < nop) {
                        RunValues<C2> r;
                        r.load(P + q * pop, run2);
                        out[item + op0 + q] = r.sum(run2);
                    }
            }
            it += 256;
            if (it >= ns1 * ns2) break;
            place(it);
        }
    };
    auto stage = [&](int op, int a) {
        if (staged)
#pragma unroll
            for (int b = 0; b < 3; ++b) mine[BT * b] = entry(op, a, b);
    };
    stage(0, 0);
#pragma unroll
    for (int op = 0; op < 4; ++op) {
        if (op == 3 && !four) {
            place(tid < ns1 * ns2 ? tid : 0);
            __syncthreads();
            test_side(0, 3);
            __syncthreads();
        }
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            RunValues<C2> r[SLOT_IT1];
            wave_lds_order();
#pragma unroll
            for (int j = 0; j < SLOT_IT1; ++j)
                if (16 * j < ns2) r[j].load(st, run1[j]);
            wave_lds_order();
            if (a < 2) stage(op, a + 1);
            else if (op < 3) stage(op + 1, 0);
#pragma unroll
            for (int j = 0; j < SLOT_IT1; ++j)
                if (16 * j < ns2 && run1[j].m > 0) P[(op == 3 && !four ? 0 : op) * pop + pr[a] + 16 * j] = r[j].sum(run1[j]);
        }
    }
    place(tid < ns1 * ns2 ? tid : 0);
    __syncthreads();
    if (four) test_side(0, 4);
    else test_side(3, 1);
}

// The 6-point rule applied to six values g_0 .. g_5 with the P1 functions:
// sum over q of w_q lambda_b(q) g_q for b = 0..2.  With the two orbits'
// barycentric coordinates (a, a, 1 - 2a) it is, up to the factor kR6G,
//   h_b + kR6H (h_0 + h_1 + h_2) + kR6S (g_3 + g_4 + g_5),  h_b = g_b + kR6C g_{b+3}:
// two operations per value instead of three.
constexpr double kR6G = kW1 * (1.0 - 3.0 * kA1);
constexpr double kR6C = kW2 * (1.0 - 3.0 * kA2) / kR6G;
constexpr double kR6H = kW1 * kA1 / kR6G;
constexpr double kR6S = kW2 * kA2 / kR6G - kR6H * kR6C;
template <class R> struct Rule6Const {
    static constexpr R G = kR6G, C = kR6C, H = kR6H, S = kR6S;
};
// (Mixed operators against FP64 ones, 10,242 + 7,842 vertices: V 5.0e-8, K and T 6.1e-8, D 9.4e-8; 5.7e-8, 8.7e-8 and
// 9.2e-8 with correctly rounded 1 / r and the plain weights.)  In FP32 the constants' own rounding would put errors up to 9e-8 on the orbits' weights, the same for all
// pairs; C, H and S are the floats within 6 ulps, with their G, that leave the least: 3e-9, the weights' sum exact.
template <> struct Rule6Const<float> {
    static constexpr double G = kR6G * 1.000000060973267;
    static constexpr float C = -1.0566645860671997f, H = -1.3199776411056519f, S = -1.5281931161880493f;
};
template <class R> struct Rule6Sum {
    using Q = Rule6Const<R>;
    R h[3], s;
    __device__ void add(int b, R g0, R g1)   // g_b and g_{b+3}, b = 0, 1, 2 in this order
    {
        h[b] = g0 + Q::C * g1;
        s = b == 0 ? g1 : s + g1;
    }
    __device__ void finish()
    {
        const R m = Q::H * (h[0] + h[1] + h[2]) + Q::S * s;
#pragma unroll
        for (int b = 0; b < 3; ++b) h[b] += m;
    }
};

// A triangle's table in LDS: TriGeo up to its vertices, padded to an odd number of 16-byte units (19): the 16
// trial triangles a wave reads at once then fall on distinct LDS banks.
struct alignas(16) TileGeo {
    double qp[6][3], n[3], off, area, c[3], rho, curl[3][3];
    double pad[2];
};
static_assert(sizeof(TileGeo) == (TRI_TILE + 2) * sizeof(double) && offsetof(TriGeo, p) == TRI_TILE * sizeof(double) &&
                  offsetof(TileGeo, curl) == offsetof(TriGeo, curl),
              "LDS tables of the tile kernels");

// 6 x 6 point pairs of one regular triangle pair (x on X, y on Y): the 3 x 3
// element sums of V (kernel G), K (dG/dn_y), T (dG/dn_x) and the scalar sum
// of G, unscaled (times area_X area_Y / (4 pi) later).  K and T use that
// (y - x).n_y is the same for every y on the plane of Y and (x - y).n_x for
// every x on the plane of X: one factor per test point and one per trial
// point.  BASE: phase from the per-pair base (see the caller; 1 up to 1, 2 up
// to kShortPhase radian off it), whose factor exp(i k r0) is applied to the sums.  CK:
// complex wavenumber k + i kim; the damping exp(-kim r) has the same base.
template <bool CK, int BASE>
__device__ inline void pair_quadrature(const TileGeo &X, const TileGeo &Y, double k, double kim, double (&vr)[9],
                                       double (&vi)[9], double (&kr)[9], double (&ki)[9], double (&tr)[9],
                                       double (&ti)[9], double &sr, double &si)
{
    const double ny0 = Y.n[0], ny1 = Y.n[1], ny2 = Y.n[2];
    const double ey0 = Y.off;
    double e0r = 1.0, e0i = 0.0, kr0 = 0.0, mr0 = 0.0;
    if constexpr (BASE) {
        const double c0 = X.c[0] - Y.c[0], c1 = X.c[1] - Y.c[1], c2 = X.c[2] - Y.c[2];
        const double r0 = sqrt(c0 * c0 + c1 * c1 + c2 * c2);
        kr0 = k * r0;
        phase_sincos(kr0, &e0i, &e0r);
        if constexpr (CK) {
            mr0 = kim * r0;
            const double dmp = exp(-mr0);
            e0r *= dmp;
            e0i *= dmp;
        }
    }
    double dtq[6];   // (x - y).n_x
    {
        const double nx0 = X.n[0], nx1 = X.n[1], nx2 = X.n[2];
        const double ex0 = X.off;
#pragma unroll
        for (int q = 0; q < 6; ++q) dtq[q] = ex0 - (nx0 * Y.qp[q][0] + nx1 * Y.qp[q][1] + nx2 * Y.qp[q][2]);
    }
#pragma unroll
    for (int p = 0; p < 6; ++p) {
        const double x0 = X.qp[p][0], x1 = X.qp[p][1], x2 = X.qp[p][2];
        const double dkp = ey0 - (ny0 * x0 + ny1 * x1 + ny2 * x2);   // (y - x).n_y
        Rule6Sum<double> hvr, hvi, hkr, hki, htr, hti;
#pragma unroll
        for (int b = 0; b < 3; ++b) {
            double gr[2], gi[2], fr[2], fi[2];
#pragma unroll
            for (int o = 0; o < 2; ++o) {
                const int q = b + 3 * o;
                const double d0 = x0 - Y.qp[q][0], d1 = x1 - Y.qp[q][1], d2 = x2 - Y.qp[q][2];
                const double r2 = d0 * d0 + d1 * d1 + d2 * d2;
                const double rinv = rsqrt_pos(r2);
                const double r = r2 * rinv;
                const double kr_ = k * r;
                double sn, cs;
                if constexpr (BASE) {
                    small_sincos<BASE == 2>(fma(k, r, -kr0), sn, cs);
                } else {
                    phase_sincos(kr_, &sn, &cs);
                }
                gr[o] = cs * rinv; gi[o] = sn * rinv;              // exp(ikr)/r
                const double rinv2 = rinv * rinv;
                if constexpr (CK) {                                // exp(ikr)(ikr-1)/r^3
                    const double mr_ = kim * r, am = -1.0 - mr_;
                    double dmp;
                    if constexpr (BASE) dmp = small_exp<BASE == 2>(fma(-kim, r, mr0));
                    else dmp = exp(-mr_);
                    gr[o] *= dmp; gi[o] *= dmp;
                    fr[o] = (gr[o] * am - gi[o] * kr_) * rinv2;
                    fi[o] = (gr[o] * kr_ + gi[o] * am) * rinv2;
                } else {
                    fr[o] = (-gr[o] - gi[o] * kr_) * rinv2;
                    fi[o] = (gr[o] * kr_ - gi[o]) * rinv2;
                }
            }
            hvr.add(b, gr[0], gr[1]); hvi.add(b, gi[0], gi[1]);
            hkr.add(b, fr[0], fr[1]); hki.add(b, fi[0], fi[1]);
            htr.add(b, fr[0] * dtq[b], fr[1] * dtq[b + 3]); hti.add(b, fi[0] * dtq[b], fi[1] * dtq[b + 3]);
        }
        hvr.finish(); hvi.finish(); hkr.finish(); hki.finish(); htr.finish(); hti.finish();
        const double wp = p < 3 ? kW1 : kW2;
        const double ap = p < 3 ? kA1 : kA2;
        const int pc = p < 3 ? p : p - 3;            // corner carrying 1 - 2a
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const double W = kR6G * wp * (a == pc ? 1.0 - 2.0 * ap : ap);
            const double Wk = W * dkp;
#pragma unroll
            for (int b = 0; b < 3; ++b) {
                vr[3 * a + b] += W * hvr.h[b]; vi[3 * a + b] += W * hvi.h[b];
                kr[3 * a + b] += Wk * hkr.h[b]; ki[3 * a + b] += Wk * hki.h[b];
                tr[3 * a + b] += W * htr.h[b]; ti[3 * a + b] += W * hti.h[b];
            }
        }
    }
    const double scale = X.area * Y.area * kInv4Pi;
    if constexpr (BASE) {
        const double er = scale * e0r, ei = scale * e0i;
        auto turn = [&](double &re, double &im) {
            const double x = re;
            re = x * er - im * ei;
            im = x * ei + im * er;
        };
#pragma unroll
        for (int e = 0; e < 9; ++e) {
            turn(vr[e], vi[e]);
            turn(kr[e], ki[e]);
            turn(tr[e], ti[e]);
        }
    } else {
#pragma unroll
        for (int e = 0; e < 9; ++e) {
            vr[e] *= scale; vi[e] *= scale; kr[e] *= scale; ki[e] *= scale; tr[e] *= scale; ti[e] *= scale;
        }
    }
    // sum G over the point pairs: the P1 functions sum to one at every point,
    // so the sum over a, b of the V entries is that sum
    sr = 0.0;
    si = 0.0;
#pragma unroll
    for (int e = 0; e < 9; ++e) { sr += vr[e]; si += vi[e]; }
}

struct TileArgsF {
    const TriGeoF *geof;
    const int32_t *tri;
    const int32_t *blk_start;
    const int32_t *blk_nslot;
    const uint8_t *slot_off;    // [nb][SLOT_OFF_LD] first slot-major rank of each slot
    const uint8_t *slot_rank;   // [nb][3 * BT] slot-major rank of each corner
    const SlotPlaces *slot_place;   // [nb][SMAX]
    int32_t nb;
    double k;
    double kim;            // imaginary part of the wavenumber (read by the absorbing instantiation only)
    float2 *scratch;       // [tile of the strip][SMAX*SMAX][op]
    int32_t b0, nrow;      // first tile row of the strip, rows
};

// CK: complex wavenumber k + i kim (an absorbing medium), G = exp(i k r - kim r) / (4 pi r);
// the real-k instantiation is the one the benchmarks time.
template <bool CK>
__global__ __launch_bounds__(256, 2) void regular_tiles_kernel(TileArgs A)
{
    __shared__ TileGeo geo[2 * BT];      // the test block's triangles, then the trial block's
    __shared__ TileSlots S;
    __shared__ double2 st[4][ST_WAVE];   // each wave's staged rows
    __shared__ double2 P[P_LEN];         // test-corner rank x trial slot partial sums

    int b1, b2;
    if (!tile_of(A, b1, b2)) return;
    const TileBlocks B(A, b1, b2);
    const int tid = threadIdx.x, t1 = tid >> 4, t2 = tid & 15;
    {
        constexpr int GN = (TRI_TILE + 7) / 8;
        const int t = tid >> 3;   // (triangles past a block's last repeat its last)
        const double *src = reinterpret_cast<const double *>(
            A.geo + (t < BT ? B.s1 + min(t, B.n1 - 1) : B.s2 + min(t - BT, B.n2 - 1)));
        double g[GN];
#pragma unroll
        for (int i = 0; i < GN; ++i) g[i] = src[min((tid & 7) + 8 * i, TRI_TILE - 1)];
        const uint32_t w = tile_slots_word(A, B, tid);
#pragma unroll
        for (int i = 0; i < GN; ++i)
            if ((tid & 7) + 8 * i < TRI_TILE) reinterpret_cast<double *>(geo + t)[(tid & 7) + 8 * i] = g[i];
        if (tid < TW_END) reinterpret_cast<uint32_t *>(&S)[tid] = w;
    }
    __syncthreads();
    const double k = A.k;
    const double k2r = CK ? k * k - A.kim * A.kim : k * k, k2i = 2.0 * k * A.kim;
    const TileGeo &X = geo[t1], &Y = geo[BT + t2];
    const bool active = tile_pair_active(S, B, t1, t2);
    double vr[9], vi[9], kr[9], ki[9], tr[9], ti[9], sr = 0.0, si = 0.0;
#pragma unroll
    for (int e = 0; e < 9; ++e) { vr[e] = vi[e] = kr[e] = ki[e] = tr[e] = ti[e] = 0.0; }
    // Phase by a per-pair base where k (rho_X + rho_Y) <= 1 for every pair of
    // the wave: with r0 the centroid distance, |k (r - r0)| <= 1 for every
    // point pair, so exp(i k r) = exp(i k r0) exp(i k (r - r0)) takes one
    // reduced sin/cos per pair and short polynomials per point pair (shorter
    // ones up to kShortPhase).  The choice is the wave's, so that its lanes run one
    // of the three forms.
    // Complex k: the damping's exponent is held to the same bounds (2,252 + 1,692 vertices with an absorbing
    // interior: 3.32 -> 3.18 ms against the library's exp and the full reduction at every point).
    const double spread = active ? (CK ? fmax(k, A.kim) : k) * (X.rho + Y.rho) : 0.0;
    const int base = __any(spread > 1.0) ? 0 : (__any(spread > kShortPhase) ? 1 : 2);
    if (active) {
        if (base == 2) pair_quadrature<CK, 2>(X, Y, k, A.kim, vr, vi, kr, ki, tr, ti, sr, si);
        else if (base == 1) pair_quadrature<CK, 1>(X, Y, k, A.kim, vr, vi, kr, ki, tr, ti, sr, si);
        else pair_quadrature<CK, 0>(X, Y, k, A.kim, vr, vi, kr, ki, tr, ti, sr, si);
    }

    const double nn = X.n[0] * Y.n[0] + X.n[1] * Y.n[1] + X.n[2] * Y.n[2];
    tile_slot_sums(tid, B.n1, B.n2, B.ns1, B.ns2, S.o1, S.r1, S.w2, &st[0][0], P,
                   A.scratch + B.at * (4 * SMAX * SMAX),
                   [&](int op, int a, int b) {
                       const int e = 3 * a + b;
                       if (op == 0) return make_double2(vr[e], vi[e]);
                       if (op == 1) return make_double2(kr[e], ki[e]);
                       if (op == 2) return make_double2(tr[e], ti[e]);
                       const double cc = X.curl[a][0] * Y.curl[b][0] + X.curl[a][1] * Y.curl[b][1] + X.curl[a][2] * Y.curl[b][2];
                       if constexpr (CK)   // complex k^2
                           return make_double2(cc * sr - nn * (k2r * vr[e] - k2i * vi[e]), cc * si - nn * (k2r * vi[e] + k2i * vr[e]));
                       else
                           return make_double2(cc * sr - k2r * nn * vr[e], cc * si - k2r * nn * vi[e]);
                   });
}

// The point pairs of one regular triangle pair in FP32.  The phase k|x - y|
// is split per triangle pair: with d0 the FP64 centroid difference and r0 =
// |d0|, exp(i k r) = exp(i k r0) exp(i k D), where exp(i k r0) is evaluated
// once in FP64 and applied to the sums, and D = r - r0 = e.(2 d0 + e) / (r +
// r0), e = (x - c_x) - (y - c_y), is small and accurate in FP32; FP32 alone
// would lose about k r * 6e-8 of phase.  1 / r is the hardware estimate (1 ulp) with a
// Newton step, since it enters K and T three times (their errors 8.4e-8 -> 6.1e-8;
// 10,242 + 7,842 vertices 33.7 -> 34.1 ms); the quotient in D takes the
// hardware reciprocal, whose error meets the small phase k D only.  SMALL: |k D| and, CK, |kim D| <= 1
// at every point pair.  CK: the damping exp(-kim r) splits like the phase, exp(-kim r0) in
// FP64 per pair and exp(-kim D) in FP32 per point; where kim D is not small, both
// go to each value (exp(-kim D) / r^3 alone can leave the range of FP32).
template <bool CK, bool SMALL>
__device__ inline void pair_quadrature_f32(const TriGeoF &X, const TriGeoF &Y, double k, double kim, float (&vr)[9],
                                           float (&vi)[9], float (&kr)[9], float (&ki)[9], float (&tr)[9],
                                           float (&ti)[9], float &sr, float &si)
{
    const double d00 = X.c[0] - Y.c[0], d01 = X.c[1] - Y.c[1], d02 = X.c[2] - Y.c[2];
    const double r0 = sqrt(d00 * d00 + d01 * d01 + d02 * d02);
    double s0, c0;
    phase_sincos(k * r0, &s0, &c0);
    if constexpr (CK) {
        const double dm0 = exp(-kim * r0);
        s0 *= dm0;
        c0 *= dm0;
    }
    constexpr bool EACH = CK && !SMALL;   // the pair's factor on the values instead of the sums
    const float e0r = (float)c0, e0i = (float)s0;
    const float kf = (float)k, kimf = (float)kim;
    const float f00 = (float)d00, f01 = (float)d01, f02 = (float)d02, r0f = (float)r0;
    const float ny0 = Y.n[0], ny1 = Y.n[1], ny2 = Y.n[2];
    const float dk0 = (float)-(d00 * ny0 + d01 * ny1 + d02 * ny2);
    float dtq[6];   // (x - y).n_x: the same for every x on the plane of X
    {
        const float nx0 = X.n[0], nx1 = X.n[1], nx2 = X.n[2];
        const float dt0 = (float)(d00 * nx0 + d01 * nx1 + d02 * nx2);
#pragma unroll
        for (int q = 0; q < 6; ++q) dtq[q] = dt0 - (nx0 * Y.dq[q][0] + nx1 * Y.dq[q][1] + nx2 * Y.dq[q][2]);
    }
#pragma unroll 1
    for (int p = 0; p < 6; ++p) {
        const float x0 = X.dq[p][0], x1 = X.dq[p][1], x2 = X.dq[p][2];
        const float dkp = dk0 - (ny0 * x0 + ny1 * x1 + ny2 * x2);   // (y - x).n_y
        Rule6Sum<float> hvr, hvi, hkr, hki, htr, hti;
#pragma unroll
        for (int b = 0; b < 3; ++b) {
            float gr[2], gi[2], fr[2], fi[2];
#pragma unroll
            for (int o = 0; o < 2; ++o) {
                const int q = b + 3 * o;
                const float q0 = x0 - Y.dq[q][0], q1 = x1 - Y.dq[q][1], q2 = x2 - Y.dq[q][2];   // e
                const float d0 = f00 + q0, d1 = f01 + q1, d2 = f02 + q2;                         // x - y
                const float r2 = d0 * d0 + d1 * d1 + d2 * d2;
                const float ri = __builtin_amdgcn_rsqf(r2);
                const float rinv = fmaf(0.5f * ri, fmaf(-r2 * ri, ri, 1.f), ri);
                const float r = r2 * rinv;
                const float num = q0 * (f00 + d0) + q1 * (f01 + d1) + q2 * (f02 + d2);
                const float dr = num * __builtin_amdgcn_rcpf(r + r0f);
                float sd, cd;
                if constexpr (SMALL) small_sincos_f32(kf * dr, sd, cd);
                else sincosf(kf * dr, &sd, &cd);
                if constexpr (EACH) {
                    const float dd = expf(-kimf * dr), x = cd;
                    cd = (e0r * x - e0i * sd) * dd;
                    sd = (e0r * sd + e0i * x) * dd;
                }
                gr[o] = cd * rinv; gi[o] = sd * rinv;              // exp(ik(r - r0))/r
                const float kr_ = kf * r, rinv2 = rinv * rinv;
                if constexpr (CK) {
                    const float am = -1.f - kimf * r;
                    if constexpr (!EACH) {
                        const float dd = expf(-kimf * dr);
                        gr[o] *= dd; gi[o] *= dd;
                    }
                    fr[o] = (gr[o] * am - gi[o] * kr_) * rinv2;
                    fi[o] = (gr[o] * kr_ + gi[o] * am) * rinv2;
                } else {
                    fr[o] = (-gr[o] - gi[o] * kr_) * rinv2;
                    fi[o] = (gr[o] * kr_ - gi[o]) * rinv2;
                }
            }
            hvr.add(b, gr[0], gr[1]); hvi.add(b, gi[0], gi[1]);
            hkr.add(b, fr[0], fr[1]); hki.add(b, fi[0], fi[1]);
            htr.add(b, fr[0] * dtq[b], fr[1] * dtq[b + 3]); hti.add(b, fi[0] * dtq[b], fi[1] * dtq[b + 3]);
        }
        hvr.finish(); hvi.finish(); hkr.finish(); hki.finish(); htr.finish(); hti.finish();
        constexpr double G = Rule6Const<float>::G;
        const float wo = p < 3 ? (float)(G * kW1 * kA1) : (float)(G * kW2 * kA2);
        const float wc = p < 3 ? (float)(G * kW1 * (1.0 - 2.0 * kA1)) : (float)(G * kW2 * (1.0 - 2.0 * kA2));
        const int pc = p < 3 ? p : p - 3;   // corner carrying 1 - 2a
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const float W = a == pc ? wc : wo, Wk = W * dkp;
#pragma unroll
            for (int b = 0; b < 3; ++b) {
                vr[3 * a + b] += W * hvr.h[b]; vi[3 * a + b] += W * hvi.h[b];
                kr[3 * a + b] += Wk * hkr.h[b]; ki[3 * a + b] += Wk * hki.h[b];
                tr[3 * a + b] += W * htr.h[b]; ti[3 * a + b] += W * hti.h[b];
            }
        }
    }
    const float scale = X.area * Y.area * (float)kInv4Pi, er = EACH ? scale : scale * e0r, ei = EACH ? 0.f : scale * e0i;
    auto turn = [&](float &re, float &im) {
        const float x = re;
        re = x * er - im * ei;
        im = x * ei + im * er;
    };
#pragma unroll
    for (int e = 0; e < 9; ++e) {
        turn(vr[e], vi[e]);
        turn(kr[e], ki[e]);
        turn(tr[e], ti[e]);
    }
    // the sum of G over the point pairs is the sum of the V entries (the P1 functions sum to one)
#pragma unroll
    for (int e = 0; e < 9; ++e) { sr += vr[e]; si += vi[e]; }
}

// Mixed-precision form of the regular-pair tile: FP32 arithmetic (the phase
// in FP64 once per triangle pair), complex64 tiles.
template <bool CK>
__global__ __launch_bounds__(256, 3) void regular_tiles_f32_kernel(TileArgsF A)
{
    __shared__ TriGeoF geo[2 * BT];      // the test block's triangles, then the trial block's
    __shared__ TileSlots S;
    __shared__ float2 st[4][ST_WAVE];    // each wave's staged rows
    __shared__ float2 P[P_LEN];          // test-corner rank x trial slot partial sums

    int b1, b2;
    if (!tile_of(A, b1, b2)) return;
    const TileBlocks B(A, b1, b2);
    const int tid = threadIdx.x, t1 = tid >> 4, t2 = tid & 15;
    {
        constexpr int GW = sizeof(TriGeoF) / sizeof(double), GN = (GW + 7) / 8;
        const int t = tid >> 3;   // (triangles past a block's last repeat its last)
        const double *src = reinterpret_cast<const double *>(
            A.geof + (t < BT ? B.s1 + min(t, B.n1 - 1) : B.s2 + min(t - BT, B.n2 - 1)));
        double g[GN];
#pragma unroll
        for (int i = 0; i < GN; ++i) g[i] = src[min((tid & 7) + 8 * i, GW - 1)];
        const uint32_t w = tile_slots_word(A, B, tid);
#pragma unroll
        for (int i = 0; i < GN; ++i)
            if ((tid & 7) + 8 * i < GW) reinterpret_cast<double *>(geo + t)[(tid & 7) + 8 * i] = g[i];
        if (tid < TW_END) reinterpret_cast<uint32_t *>(&S)[tid] = w;
    }
    __syncthreads();
    const float kf = (float)A.k;
    const float k2r = CK ? (float)(A.k * A.k - A.kim * A.kim) : kf * kf, k2i = (float)(2.0 * A.k * A.kim);
    const TriGeoF &X = geo[t1], &Y = geo[BT + t2];
    const bool active = tile_pair_active(S, B, t1, t2);
    float vr[9], vi[9], kr[9], ki[9], tr[9], ti[9], sr = 0.f, si = 0.f;
#pragma unroll
    for (int e = 0; e < 9; ++e) { vr[e] = vi[e] = kr[e] = ki[e] = tr[e] = ti[e] = 0.f; }
    // |k (r - r0)| <= 1, and the damping's exponent alike, at every point pair of every pair of the wave
    const bool tame = !__any(active && (CK ? fmaxf(kf, (float)A.kim) : kf) * (X.rho + Y.rho) > 1.f);
    if (active) {
        if (tame) pair_quadrature_f32<CK, true>(X, Y, A.k, A.kim, vr, vi, kr, ki, tr, ti, sr, si);
        else pair_quadrature_f32<CK, false>(X, Y, A.k, A.kim, vr, vi, kr, ki, tr, ti, sr, si);
    }
    const float nn = X.n[0] * Y.n[0] + X.n[1] * Y.n[1] + X.n[2] * Y.n[2];
    tile_slot_sums(tid, B.n1, B.n2, B.ns1, B.ns2, S.o1, S.r1, S.w2, &st[0][0], P,
                   A.scratch + B.at * (4 * SMAX * SMAX),
                   [&](int op, int a, int b) {
                       const int e = 3 * a + b;
                       if (op == 0) return make_float2(vr[e], vi[e]);
                       if (op == 1) return make_float2(kr[e], ki[e]);
                       if (op == 2) return make_float2(tr[e], ti[e]);
                       const float cc = X.curl[a][0] * Y.curl[b][0] + X.curl[a][1] * Y.curl[b][1] + X.curl[a][2] * Y.curl[b][2];
                       if constexpr (CK)   // complex k^2
                           return make_float2(cc * sr - nn * (k2r * vr[e] - k2i * vi[e]), cc * si - nn * (k2r * vi[e] + k2i * vr[e]));
                       else
                           return make_float2(cc * sr - k2r * nn * vr[e], cc * si - k2r * nn * vi[e]);
                   });
}

// The contributions to dense entry (i, j) of the tiles of one strip (tile
// rows [b0, b1), tile t at (t - tile_base) in the scratch): every tile
// (min(bi, bj), max(bi, bj)) of the blocks bi, bj containing i and j whose
// first block lies in the strip, in membership order (memberships of i,
// then of j).  The same terms with the roles of i and j exchanged make up
// entry (j, i): V and D are the same numbers, K and T exchange (the tile of
// (bj, bi) read from the other side).  So one sum gives both entries, and a
// strip reads each tile entry once.  The strip of the smallest membership
// of i and j is the first to reach (i, j) and writes it; later strips add
// their share (strips run in order on one stream).
//
// Entries a strip reaches have i or j in its row list R (the vertices with a
// membership in its blocks) and both at or after lo (the first vertex with a
// membership at or after b0).  Two launches cover them as unordered pairs:
//   RR: i = R[a], j = R[b] for a <= b (16 x 16 chunks of R; workgroups whose
//       row chunk comes after their column chunk return at once);
//   RO: i in R, j in [lo, nv) outside R (16 rows of R x 16 columns).
// A workgroup of 256 threads holds a 16 x 16 block: it writes (i, j) along
// rows (consecutive j), stages the sums in LDS and writes (j, i) along rows
// j (consecutive i of R).
template <class C2>
__device__ inline bool strip_sum(int i, int j, int nb, int b0, int b1, int64_t tile_base, const int32_t *memb_ptr,
                                 const int32_t *memb, const C2 *scratch, C2 (&acc)[4], bool &first)
{
    using R = decltype(C2::x);
    const int pi0 = memb_ptr[i], pi1 = memb_ptr[i + 1];
    const int pj0 = memb_ptr[j], pj1 = memb_ptr[j + 1];
    R vx = 0, vy = 0, kx = 0, ky = 0, tx = 0, ty = 0, dx = 0, dy = 0;
    bool any = false;
    for (int p = pi0; p < pi1; ++p) {
        const int mi = memb[p], bi = mi >> 8, si = mi & 255;
        for (int q = pj0; q < pj1; ++q) {
            const int mj = memb[q], bj = mj >> 8, sj = mj & 255;
            const int lo_b = bi < bj ? bi : bj, hi_b = bi < bj ? bj : bi;
            if (lo_b < b0 || lo_b >= b1) continue;
            any = true;
            const int64_t tile = (int64_t)lo_b * nb - (int64_t)lo_b * (lo_b - 1) / 2 + (hi_b - lo_b) - tile_base;
            const C2 *tl = scratch + tile * (4 * SMAX * SMAX);
            if (bi <= bj) {
                const int e = si * SMAX + sj;
                const C2 a0 = tl[4 * e], a1 = tl[4 * e + 1], a2 = tl[4 * e + 2], a3 = tl[4 * e + 3];
                vx += a0.x; vy += a0.y; kx += a1.x; ky += a1.y;
                tx += a2.x; ty += a2.y; dx += a3.x; dy += a3.y;
            } else {
                // tile of (bj, bi): test side is j; K and T swap under transposition
                const int e = sj * SMAX + si;
                const C2 a0 = tl[4 * e], a1 = tl[4 * e + 1], a2 = tl[4 * e + 2], a3 = tl[4 * e + 3];
                vx += a0.x; vy += a0.y; kx += a2.x; ky += a2.y;
                tx += a1.x; ty += a1.y; dx += a3.x; dy += a3.y;
            }
        }
    }
    acc[0] = C2{vx, vy};
    acc[1] = C2{kx, ky};
    acc[2] = C2{tx, ty};
    acc[3] = C2{dx, dy};
    first = min(memb[pi0] >> 8, memb[pj0] >> 8) >= b0;   // lists ascend by block
    return any;
}

// (i, j) of the four operators: written by the first strip to reach it, added to by later ones
template <class C2>
__device__ inline void strip_put(C2 *const (&op)[4], int64_t o, const C2 (&v)[4], bool first)
{
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        if (first) {
            op[k][o] = v[k];
        } else {
            const C2 x = op[k][o];
            op[k][o] = C2{x.x + v[k].x, x.y + v[k].y};
        }
    }
}

template <class C2, bool RR>
__global__ __launch_bounds__(256) void gather_strip_kernel(int nv, int nb, int b0, int b1, int64_t tile_base, int lo,
                                                           const int32_t *__restrict__ rows, int nrows,
                                                           const int32_t *__restrict__ memb_ptr,
                                                           const int32_t *__restrict__ memb,
                                                           const C2 *__restrict__ scratch, C2 *__restrict__ V,
                                                           C2 *__restrict__ K, C2 *__restrict__ T, C2 *__restrict__ D)
{
    __shared__ C2 sv[4][16][17];
    __shared__ uint8_t sflag[16][17];   // bit 0: a contribution, bit 1: first strip to reach the entry
    if (RR && blockIdx.x > blockIdx.y) return;
    C2 *const op[4] = {V, K, T, D};
    const int64_t ld = op_ld(nv);
    const int tid = threadIdx.x, ra = tid >> 4, cb = tid & 15;
    // (i, j): i = R[16 blockIdx.x + ra], j = R[16 blockIdx.y + cb] (RR) or lo + 16 blockIdx.y + cb (RO)
    const int ai = 16 * (int)blockIdx.x + ra, aj = 16 * (int)blockIdx.y + cb;
    bool ok = ai < nrows && (RR ? (aj < nrows && (blockIdx.x < blockIdx.y || ra <= cb)) : lo + aj < nv);
    int i = 0, j = 0;
    if (ok) {
        i = rows[ai];
        j = RR ? rows[aj] : lo + aj;
        if (!RR)   // columns in R are the RR launch's
            for (int p = memb_ptr[j]; p < memb_ptr[j + 1] && ok; ++p) {
                const int bj = memb[p] >> 8;
                ok = bj < b0 || bj >= b1;
            }
    }
    C2 acc[4];
    bool first = false, any = false;
    if (ok) {
        any = strip_sum(i, j, nb, b0, b1, tile_base, memb_ptr, memb, scratch, acc, first);
        if (first || any) strip_put(op, (int64_t)i * ld + j, acc, first);
    }
    // (j, i) from the same sums, through LDS: V, D as they are, K and T exchanged
#pragma unroll
    for (int k = 0; k < 4; ++k) sv[k][ra][cb] = acc[k];
    sflag[ra][cb] = (uint8_t)((ok && any ? 1 : 0) | (ok && first && i != j ? 2 : 0) | (ok && i != j ? 4 : 0));
    __syncthreads();
    const int rb = tid >> 4, ca = tid & 15;   // row j of column block rb, column i of row block ca
    const int f = sflag[ca][rb];
    if (f & 4) {
        const int aj2 = 16 * (int)blockIdx.y + rb, ai2 = 16 * (int)blockIdx.x + ca;
        const int jj = RR ? rows[aj2] : lo + aj2, ii = rows[ai2];
        if (f & 3) {
            const C2 w[4] = {sv[0][ca][rb], sv[2][ca][rb], sv[1][ca][rb], sv[3][ca][rb]};
            strip_put(op, (int64_t)jj * ld + ii, w, (f & 2) != 0);
        }
    }
}

// the padding columns [nv, op_ld(nv)) of every row of the four operators: zero
template <class C2>
__global__ void zero_padding_kernel(int nv, C2 *__restrict__ V, C2 *__restrict__ K, C2 *__restrict__ T, C2 *__restrict__ D)
{
    const int pad = (int)(op_ld(nv) - nv);
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (pad == 0 || t >= (int64_t)nv * pad) return;
    const int64_t o = (t / pad) * op_ld(nv) + nv + t % pad;
    V[o] = C2{0, 0};
    K[o] = C2{0, 0};
    T[o] = C2{0, 0};
    D[o] = C2{0, 0};
}

// ----------------------------------------------------------- singular pairs

constexpr int SING_WIDE_MAX = 8192;   // pairs up to which the longer ones take a whole wave (singular_pairs_kernel)

struct GLTab {
    double x[NG_MAX], w[NG_MAX];
};

// Sauter-Schwab regions on the reference triangle {0 <= s2 <= s1 <= 1}.
__device__ inline void ss_map(int kind, int reg, double xi, double e1, double e2, double e3, double &x0, double &x1,
                              double &y0, double &y1, double &jac)
{
    const double xi3 = xi * xi * xi;
    if (kind == 3) {
        jac = xi3 * e1 * e1 * e2;
        const double a = xi, b = xi * (1.0 - e1 + e1 * e2), c = xi * (1.0 - e1 * e2 * e3), d = xi * (1.0 - e1);
        const double f = xi * e1 * (1.0 - e2 + e2 * e3), g = xi * (1.0 - e1 * e2), h = xi * e1 * (1.0 - e2);
        const double m = xi * e1 * (1.0 - e2 * e3);
        switch (reg) {
        case 0: x0 = a; x1 = b; y0 = c; y1 = d; break;
        case 1: x0 = c; x1 = d; y0 = a; y1 = b; break;
        case 2: x0 = a; x1 = f; y0 = g; y1 = h; break;
        case 3: x0 = g; x1 = h; y0 = a; y1 = f; break;
        case 4: x0 = c; x1 = m; y0 = a; y1 = h; break;
        default: x0 = a; x1 = h; y0 = c; y1 = m; break;
        }
    } else if (kind == 2) {
        jac = xi3 * e1 * e1 * (reg == 0 ? 1.0 : e2);
        switch (reg) {
        case 0: x0 = xi; x1 = xi * e1 * e3; y0 = xi * (1.0 - e1 * e2); y1 = xi * e1 * (1.0 - e2); break;
        case 1: x0 = xi; x1 = xi * e1; y0 = xi * (1.0 - e1 * e2 * e3); y1 = xi * e1 * e2 * (1.0 - e3); break;
        case 2: x0 = xi * (1.0 - e1 * e2); x1 = xi * e1 * (1.0 - e2); y0 = xi; y1 = xi * e1 * e2 * e3; break;
        case 3: x0 = xi * (1.0 - e1 * e2 * e3); x1 = xi * e1 * e2 * (1.0 - e3); y0 = xi; y1 = xi * e1; break;
        default: x0 = xi * (1.0 - e1 * e2 * e3); x1 = xi * e1 * (1.0 - e2 * e3); y0 = xi; y1 = xi * e1 * e2; break;
        }
    } else {
        jac = xi3 * e2;
        if (reg == 0) { x0 = xi; x1 = xi * e1; y0 = xi * e2; y1 = xi * e2 * e3; }
        else { x0 = xi * e2; x1 = xi * e2 * e3; y0 = xi; y1 = xi * e1; }
    }
}

// One ordered singular pair on LPP lanes: 16 take the ng^2 points of the last
// two coordinates among them; 64 also split the first coordinate.  Sums over
// the lanes by DPP.  out: [pair][corner pair][V, K, T, D].
template <bool CK, int LPP>
__device__ inline void singular_pair(const TriGeo *__restrict__ geo, const SingPair *__restrict__ pairs, int pid, int ng,
                                     const GLTab &gl, double k, double kim, double2 *__restrict__ out)
{
    const int lane = threadIdx.x & (LPP - 1);
    const SingPair sp = pairs[pid];
    const TriGeo &X = geo[sp.tau];
    const TriGeo &Y = geo[sp.sig];
    int px[3], py[3];
    for (int r = 0; r < 3; ++r) { px[r] = (sp.perm >> (2 * r)) & 3; py[r] = (sp.perm >> (6 + 2 * r)) & 3; }
    // x - y = xs0 ax0 + xs1 ax1 - ys0 ay0 - ys1 ay1: the first reference corner is shared
    double ax[2][3], ay[2][3];
    for (int c = 0; c < 3; ++c) {
        const double x0 = X.p[px[0]][c], x1 = X.p[px[1]][c], x2 = X.p[px[2]][c];
        const double y0 = Y.p[py[0]][c], y1 = Y.p[py[1]][c], y2 = Y.p[py[2]][c];
        ax[0][c] = x1 - x0; ax[1][c] = x2 - x1;
        ay[0][c] = y1 - y0; ay[1][c] = y2 - y1;
    }
    const double nx[3] = {X.n[0], X.n[1], X.n[2]}, ny[3] = {Y.n[0], Y.n[1], Y.n[2]};
    const int kind = sp.kind;
    const int nreg = kind == 3 ? 6 : (kind == 2 ? 5 : 2);
    double vr[9], vi[9], kr[9], ki[9], tr[9], ti[9];
#pragma unroll
    for (int e = 0; e < 9; ++e) { vr[e] = vi[e] = kr[e] = ki[e] = tr[e] = ti[e] = 0.0; }
    const int ng2 = ng * ng;
    for (int inner = lane & 15; inner < ng2; inner += 16) {
        const int i2 = inner / ng, i3 = inner - i2 * ng;
        const double e2 = gl.x[i2], e3 = gl.x[i3], w23 = gl.w[i2] * gl.w[i3];
        for (int reg = 0; reg < nreg; ++reg)
            for (int i0 = lane >> 4; i0 < ng; i0 += LPP / 16)
                for (int i1 = 0; i1 < ng; ++i1) {
                    const double xi = gl.x[i0], e1 = gl.x[i1];
                    double xs0, xs1, ys0, ys1, jac;
                    ss_map(kind, reg, xi, e1, e2, e3, xs0, xs1, ys0, ys1, jac);
                    const double wt = gl.w[i0] * gl.w[i1] * w23 * jac;
                    // both points by the same operations (left to itself, the compiler fuses the difference into one
                    // of the two): the regions come in pairs with x and y exchanged, and in K and T of a coincident
                    // pair, whose (x - y).n is rounding alone, the two cancel if d changes its sign exactly
                    double d[3];
                    for (int c = 0; c < 3; ++c)
                        d[c] = fma(xs1, ax[1][c], xs0 * ax[0][c]) - fma(ys1, ay[1][c], ys0 * ay[0][c]);
                    const double r2 = d[0] * d[0] + d[1] * d[1] + d[2] * d[2];
                    const double rinv = rsqrt_pos(r2);
                    const double r = r2 * rinv, kr_ = k * r;
                    double sn, cs;
                    phase_sincos(kr_, &sn, &cs);
                    double gr = cs * rinv * wt, gi = sn * rinv * wt;
                    const double rinv2 = rinv * rinv;
                    double fr, fi;
                    if constexpr (CK) {
                        const double dmp = exp(-kim * r), am = -1.0 - kim * r;
                        gr *= dmp; gi *= dmp;
                        fr = (gr * am - gi * kr_) * rinv2;
                        fi = (gr * kr_ + gi * am) * rinv2;
                    } else {
                        fr = (-gr - gi * kr_) * rinv2;
                        fi = (gr * kr_ - gi) * rinv2;
                    }
                    const double dk = -(d[0] * ny[0] + d[1] * ny[1] + d[2] * ny[2]);
                    const double dt = d[0] * nx[0] + d[1] * nx[1] + d[2] * nx[2];
                    const double gkr = fr * dk, gki = fi * dk, gtr = fr * dt, gti = fi * dt;
                    const double phx[3] = {1.0 - xs0, xs0 - xs1, xs1}, phy[3] = {1.0 - ys0, ys0 - ys1, ys1};
#pragma unroll
                    for (int a = 0; a < 3; ++a)
#pragma unroll
                        for (int b = 0; b < 3; ++b) {
                            const double ph = phx[a] * phy[b];
                            vr[3 * a + b] += ph * gr; vi[3 * a + b] += ph * gi;
                            kr[3 * a + b] += ph * gkr; ki[3 * a + b] += ph * gki;
                            tr[3 * a + b] += ph * gtr; ti[3 * a + b] += ph * gti;
                        }
                }
    }
    // over the lanes of the pair, into its last lane
    auto total = [](double v) { return LPP == 64 ? wsum63(v) : rsum15(v); };
#pragma unroll
    for (int e = 0; e < 9; ++e) {
        vr[e] = total(vr[e]); vi[e] = total(vi[e]);
        kr[e] = total(kr[e]); ki[e] = total(ki[e]);
        tr[e] = total(tr[e]); ti[e] = total(ti[e]);
    }
    if (lane != LPP - 1) return;
    // the sum of G over the points: the P1 functions of each side sum to one
    // at every point, so it is the sum of the nine V entries
    double sr = 0.0, si = 0.0;
#pragma unroll
    for (int e = 0; e < 9; ++e) { sr += vr[e]; si += vi[e]; }
    const double scale = 4.0 * X.area * Y.area * kInv4Pi;
    const double nn = nx[0] * ny[0] + nx[1] * ny[1] + nx[2] * ny[2];
    double2 *o = out + (int64_t)pid * 36;
#pragma unroll
    for (int ra = 0; ra < 3; ++ra)
#pragma unroll
        for (int rb = 0; rb < 3; ++rb) {
            const int a = px[ra], b = py[rb];        // own corners
            const int e = 3 * a + b, re = 3 * ra + rb;
            const double cc = X.curl[a][0] * Y.curl[b][0] + X.curl[a][1] * Y.curl[b][1] + X.curl[a][2] * Y.curl[b][2];
            const double Vr = vr[re] * scale, Vi = vi[re] * scale;
            o[4 * e] = make_double2(Vr, Vi);
            o[4 * e + 1] = make_double2(kr[re] * scale, ki[re] * scale);
            o[4 * e + 2] = make_double2(tr[re] * scale, ti[re] * scale);
            if constexpr (CK) {
                const double k2r = k * k - kim * kim, k2i = 2.0 * k * kim;
                o[4 * e + 3] = make_double2(cc * sr * scale - nn * (k2r * Vr - k2i * Vi),
                                            cc * si * scale - nn * (k2r * Vi + k2i * Vr));
            } else {
                o[4 * e + 3] = make_double2(cc * sr * scale - k * k * nn * Vr, cc * si * scale - k * k * nn * Vi);
            }
        }
}

// The first nwide pairs (4 per workgroup) take a whole wave each, the others
// (16 per workgroup) 16 lanes.  On meshes whose pairs leave most SIMDs with
// one wave or none, the coincident and edge pairs (96 and 80 points per lane
// on 16 lanes, against 32 of a vertex pair) are the wide ones, since the kernel
// then takes the time of its longest pair (162 vertices, 4,300 pairs: 67 ->
// 33 us); larger meshes fill the device with 16 lanes per pair and sum over
// fewer lanes.
template <bool CK>
__global__ __launch_bounds__(256, 2) void singular_pairs_kernel(const TriGeo *__restrict__ geo,
                                                             const SingPair *__restrict__ pairs, int npairs, int nwide,
                                                             int ng, GLTab gl, double k, double kim,
                                                             double2 *__restrict__ out)
{
    const int bw = (nwide + 3) / 4, b = blockIdx.x;
    if (b < bw) {
        const int pid = 4 * b + (threadIdx.x >> 6);
        if (pid < nwide) singular_pair<CK, 64>(geo, pairs, pid, ng, gl, k, kim, out);
    } else {
        const int pid = nwide + 16 * (b - bw) + (threadIdx.x >> 4);
        if (pid < npairs) singular_pair<CK, 16>(geo, pairs, pid, ng, gl, k, kim, out);
    }
}

// Add the singular contributions (FP64) to their dense entries (fixed order):
// a thread per entry and operator, so that four neighbours read a
// contribution's 64 bytes together, four contributions in flight (a thread per
// entry waited out the latency of one after the other: 23 us on the smallest
// meshes).
template <class C2>
__global__ __launch_bounds__(256) void near_scatter_kernel(int nv, int nnear, const int32_t *__restrict__ ni,
                                                           const int32_t *__restrict__ nj,
                                                           const int32_t *__restrict__ nptr,
                                                           const int32_t *__restrict__ nsrc,
                                                           const double2 *__restrict__ contrib, C2 *__restrict__ V,
                                                           C2 *__restrict__ K, C2 *__restrict__ T, C2 *__restrict__ D)
{
    using R = decltype(C2::x);
    const int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t e = u >> 2;
    const int op = (int)u & 3;
    if (e >= nnear) return;
    double sx = 0, sy = 0;
    const int q1 = nptr[e + 1];
#pragma unroll 4
    for (int q = nptr[e]; q < q1; ++q) {
        const double2 c = contrib[4 * (int64_t)nsrc[q] + op];   // nsrc: pair * 9 + corner pair
        sx += c.x;
        sy += c.y;
    }
    C2 *dst = (op == 0 ? V : op == 1 ? K : op == 2 ? T : D) + (int64_t)ni[e] * op_ld(nv) + nj[e];
    const C2 x = *dst;
    *dst = C2{(R)((double)x.x + sx), (R)((double)x.y + sy)};
}

// ------------------------------------------------------------- launchers

bem_status launch_geometry(const bem_mesh *m, hipStream_t st)
{
    const int nt = (int)m->h.nt;
    hipLaunchKernelGGL(geometry_kernel, dim3((nt + 255) / 256), dim3(256), 0, st, m->d.xyz.as<double>(),
                       m->d.tri.as<int32_t>(), nt, m->d.geo.as<TriGeo>(), m->d.geof.as<TriGeoF>());
    BEM_HIP(hipGetLastError());
    return BEM_OK;
}

// tile scratch of one mesh: two strips' tiles (or one when the mesh has a
// single strip); entry size 16 B (complex128) or 8 B (complex64)
size_t tile_scratch_bytes(const bem_mesh *m, size_t entry_bytes)
{
    const MeshData &h = m->h;
    const int ns = (int)h.strip_b.size() - 1;
    int64_t most = 0;
    for (int s = 0; s < ns; ++s) most = std::max(most, strip_tiles(h, s));
    return (size_t)(ns > 1 ? 2 : 1) * (size_t)most * 4 * SMAX * SMAX * entry_bytes;
}

// Regular-pair assembly strip by strip: the tiles of strip s into half s % 2
// of the scratch on the main stream; its gather into the operators on the
// context's gather stream, which overlaps the next strip's tiles.  The main
// stream reuses a half once the gather of two strips before is done, and
// waits for the last gather before returning.  A mesh of one strip has
// nothing to overlap: all of it goes to `st`, without the events between streams.
bem_status launch_regular(const bem_mesh *m, double k, double kim, bool fp32, void *scratch, void *ops[4], hipStream_t st)
{
    bem_ctx *ctx = m->ctx;
    const MeshData &h = m->h;
    const int64_t nb = h.nb;
    const int nv = (int)h.nv;
    const int ns = (int)h.strip_b.size() - 1;
    const size_t eb = fp32 ? sizeof(float2) : sizeof(double2);
    int64_t most = 0;
    for (int s = 0; s < ns; ++s) most = std::max(most, strip_tiles(h, s));
    const size_t half = (size_t)most * 4 * SMAX * SMAX * eb;
    const bool one = ns == 1;
    if (!one && !ctx->gather) BEM_HIP(hipStreamCreateWithFlags(&ctx->gather, hipStreamNonBlocking));
    hipStream_t gs = one ? st : ctx->gather;
    // events (kept by the context, so that no event is destroyed while a wait on it is queued): [0] main-stream
    // work before the assembly, [1 + b] tiles of half b done, [3 + b] its gather done
    hipEvent_t *ev = ctx->strip_ev;
    if (!one) {
        for (int q = 0; q < 5; ++q)
            if (!ev[q]) BEM_HIP(hipEventCreateWithFlags(&ev[q], hipEventDisableTiming));
        BEM_HIP(hipEventRecord(ev[0], st));
        BEM_HIP(hipStreamWaitEvent(gs, ev[0], 0));   // the operator blocks may have served earlier main-stream work
    }
    if ((int64_t)op_ld(nv) > nv) {
        const int64_t npad = (int64_t)nv * (op_ld(nv) - nv);
        const dim3 gz((unsigned)((npad + 255) / 256));
        if (!fp32)
            hipLaunchKernelGGL(zero_padding_kernel<double2>, gz, dim3(256), 0, gs, nv, static_cast<double2 *>(ops[0]),
                               static_cast<double2 *>(ops[1]), static_cast<double2 *>(ops[2]), static_cast<double2 *>(ops[3]));
        else
            hipLaunchKernelGGL(zero_padding_kernel<float2>, gz, dim3(256), 0, gs, nv, static_cast<float2 *>(ops[0]),
                               static_cast<float2 *>(ops[1]), static_cast<float2 *>(ops[2]), static_cast<float2 *>(ops[3]));
        BEM_HIP(hipGetLastError());
    }
    for (int s = 0; s < ns; ++s) {
        const int b0 = h.strip_b[s], b1 = h.strip_b[s + 1], hb = s % 2;
        const int64_t t0 = b0 * nb - (int64_t)b0 * (b0 - 1) / 2;
        char *buf = static_cast<char *>(scratch) + hb * half;
        if (s >= 2) BEM_HIP(hipStreamWaitEvent(st, ev[3 + hb], 0));
        {
            KTimer kt(ctx, K_REGULAR);
            const dim3 grid = tile_grid((int)nb, b0, b1 - b0);
            if (!fp32) {
                TileArgs A;
                A.geo = m->d.geo.as<TriGeo>();
                A.tri = m->d.tri.as<int32_t>();
                A.blk_start = m->d.blk_start.as<int32_t>();
                A.blk_nslot = m->d.blk_nslot.as<int32_t>();
                A.slot_off = m->d.slot_off.as<uint8_t>();
                A.slot_rank = m->d.slot_rank.as<uint8_t>();
                A.slot_place = m->d.slot_place.as<SlotPlaces>();
                A.nb = (int32_t)nb;
                A.k = k;
                A.kim = kim;
                A.scratch = reinterpret_cast<double2 *>(buf);
                A.b0 = b0;
                A.nrow = b1 - b0;
                if (kim != 0.0)
                    launch_k(kt, regular_tiles_kernel<true>, grid, dim3(256), 0, st, A);
                else
                    launch_k(kt, regular_tiles_kernel<false>, grid, dim3(256), 0, st, A);
            } else {
                TileArgsF A;
                A.geof = m->d.geof.as<TriGeoF>();
                A.tri = m->d.tri.as<int32_t>();
                A.blk_start = m->d.blk_start.as<int32_t>();
                A.blk_nslot = m->d.blk_nslot.as<int32_t>();
                A.slot_off = m->d.slot_off.as<uint8_t>();
                A.slot_rank = m->d.slot_rank.as<uint8_t>();
                A.slot_place = m->d.slot_place.as<SlotPlaces>();
                A.nb = (int32_t)nb;
                A.k = k;
                A.kim = kim;
                A.scratch = reinterpret_cast<float2 *>(buf);
                A.b0 = b0;
                A.nrow = b1 - b0;
                if (kim != 0.0)
                    launch_k(kt, regular_tiles_f32_kernel<true>, grid, dim3(256), 0, st, A);
                else
                    launch_k(kt, regular_tiles_f32_kernel<false>, grid, dim3(256), 0, st, A);
            }
        }
        BEM_HIP(hipGetLastError());
        if (!one) {
            BEM_HIP(hipEventRecord(ev[1 + hb], st));
            BEM_HIP(hipStreamWaitEvent(gs, ev[1 + hb], 0));
        }
        const int r0 = h.strip_rptr[s], nr = h.strip_rptr[s + 1] - r0, lo = h.strip_lo[s];
        const int32_t *rows = m->d.strip_rows.as<int32_t>() + r0;
        const unsigned cr = (unsigned)((nr + 15) / 16);
        const dim3 ga(cr, cr), gb(cr, (unsigned)((nv - lo + 15) / 16));
#define GATHER_ARGS(C2)                                                                                              \
    nv, (int)nb, b0, b1, t0, lo, rows, nr, m->d.memb_ptr.as<int32_t>(), m->d.memb.as<int32_t>(),                    \
        reinterpret_cast<const C2 *>(buf), static_cast<C2 *>(ops[0]), static_cast<C2 *>(ops[1]),                     \
        static_cast<C2 *>(ops[2]), static_cast<C2 *>(ops[3])
        if (nr > 0) {   // (every strip has rows: its blocks have vertices)
            KTimer kt(ctx, K_GATHER);
            if (!fp32) {
                launch_k(kt, gather_strip_kernel<double2, true>, ga, dim3(256), 0, gs, GATHER_ARGS(double2));
                KTimer kt2(ctx, K_GATHER);
                launch_k(kt2, gather_strip_kernel<double2, false>, gb, dim3(256), 0, gs, GATHER_ARGS(double2));
            } else {
                launch_k(kt, gather_strip_kernel<float2, true>, ga, dim3(256), 0, gs, GATHER_ARGS(float2));
                KTimer kt2(ctx, K_GATHER);
                launch_k(kt2, gather_strip_kernel<float2, false>, gb, dim3(256), 0, gs, GATHER_ARGS(float2));
            }
        }
#undef GATHER_ARGS
        BEM_HIP(hipGetLastError());
        if (!one) BEM_HIP(hipEventRecord(ev[3 + hb], gs));
    }
    if (!one) BEM_HIP(hipStreamWaitEvent(st, ev[3 + (ns - 1) % 2], 0));   // gathers run in order: the last covers all
    return BEM_OK;
}

bem_status launch_singular(const bem_mesh *m, double k, double kim, int ng, const double *glx, const double *glw, bool fp32,
                           double2 *contrib, void *ops[4], hipStream_t st)
{
    GLTab gl;
    for (int i = 0; i < NG_MAX; ++i) { gl.x[i] = i < ng ? glx[i] : 0.0; gl.w[i] = i < ng ? glw[i] : 0.0; }
    const int np = (int)m->h.sing.size();
    if (np > 0) {
        KTimer kt(m->ctx, K_SINGULAR);
        const int nwide = np <= SING_WIDE_MAX ? m->h.nsing_kind[3] + m->h.nsing_kind[2] : 0;   // (sorted by kind: 3, 2, 1)
        const dim3 grid((nwide + 3) / 4 + (np - nwide + 15) / 16);
        auto kernel = kim != 0.0 ? singular_pairs_kernel<true> : singular_pairs_kernel<false>;
        launch_k(kt, kernel, grid, dim3(256), 0, st, m->d.geo.as<TriGeo>(), m->d.sing.as<SingPair>(), np, nwide, ng, gl, k,
                 kim, contrib);
        BEM_HIP(hipGetLastError());
    }
    const int nn = (int)m->h.near_i.size();
    if (nn > 0) {
        KTimer kt(m->ctx, K_NEAR);
        const int nv = (int)m->h.nv;
        if (!fp32)
            launch_k(kt, near_scatter_kernel<double2>, dim3((unsigned)((4 * (int64_t)nn + 255) / 256)), dim3(256), 0, st, nv, nn,
                     m->d.near_i.as<int32_t>(), m->d.near_j.as<int32_t>(), m->d.near_ptr.as<int32_t>(),
                     m->d.near_src.as<int32_t>(), (const double2 *)contrib, static_cast<double2 *>(ops[0]),
                     static_cast<double2 *>(ops[1]), static_cast<double2 *>(ops[2]), static_cast<double2 *>(ops[3]));
        else
            launch_k(kt, near_scatter_kernel<float2>, dim3((unsigned)((4 * (int64_t)nn + 255) / 256)), dim3(256), 0, st, nv, nn,
                     m->d.near_i.as<int32_t>(), m->d.near_j.as<int32_t>(), m->d.near_ptr.as<int32_t>(),
                     m->d.near_src.as<int32_t>(), (const double2 *)contrib, static_cast<float2 *>(ops[0]),
                     static_cast<float2 *>(ops[1]), static_cast<float2 *>(ops[2]), static_cast<float2 *>(ops[3]));
        BEM_HIP(hipGetLastError());
    }
    return BEM_OK;
}

}  // namespace bemtx
