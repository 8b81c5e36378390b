// Tables of the sparse inverse-mass apply (the mass-matrix preconditioner of
// Sec. 3.3 applied without forming M^-1).
//
// z = M^-1 y is computed by Chebyshev iteration on the Jacobi-scaled P1 mass
// matrix: every eigenvalue of diag(M)^-1 M lies in [1/2, 2] (each element
// matrix (A/12)[[2,1,1],[1,2,1],[1,1,2]] scaled by its diagonal has the
// eigenvalues 2, 1/2, 1/2, and the Rayleigh quotient of the sum lies between
// those of its terms), so k steps reduce the error by 4 3^-k on any mesh.
// One kernel launch takes s steps on overlapping patches: a patch owns a
// compact cluster of vertices and holds every vertex within s edges of them; after t steps the iterate is exact (to rounding) on the
// vertices within s - t edges, so after s steps on the owned ones.  The
// patch's vertices are listed by distance from the owned range, so that the
// rows updated at step t are a prefix of the list.
#include <algorithm>
#include <atomic>
#include <vector>

#include "internal.h"

namespace bemtx {

namespace {

// one patch: its owned vertices and every vertex within s edges of them
struct Patch {
    std::vector<int32_t> vert, cnt, rptr, col;
    std::vector<double> dinv, val;
};

// Owned sets: compact clusters of at most `own` vertices, grown breadth-first
// from the lowest unassigned vertex over unassigned neighbours (a compact
// set has the shortest rings around it).  Deterministic.
std::vector<std::vector<int32_t>> clusters(const Csr &M, int own)
{
    const int32_t nv = (int32_t)M.nrows;
    std::vector<char> taken(nv, 0);
    std::vector<std::vector<int32_t>> out;
    for (int32_t seed = 0; seed < nv; ++seed) {
        if (taken[seed]) continue;
        std::vector<int32_t> c{seed};
        taken[seed] = 1;
        for (size_t q = 0; q < c.size() && (int)c.size() < own; ++q)
            for (int32_t e = M.ptr[c[q]]; e < M.ptr[c[q] + 1] && (int)c.size() < own; ++e) {
                const int32_t u = M.col[e];
                if (!taken[u]) {
                    taken[u] = 1;
                    c.push_back(u);
                }
            }
        std::sort(c.begin(), c.end());
        out.push_back(std::move(c));
    }
    return out;
}

// (a patch of more than lmax vertices: the vertices only)
void build_patch(const Csr &M, const std::vector<int32_t> &owned, int s, int lmax, std::vector<int32_t> &dist,
                 std::vector<int32_t> &loc, Patch &P)
{
    P.vert.clear();
    for (int32_t v : owned) {
        dist[v] = 0;
        P.vert.push_back(v);
    }
    size_t front = 0;
    for (int d = 1; d <= s; ++d) {   // breadth-first rings; each ring in ascending vertex order
        const size_t end = P.vert.size();
        std::vector<int32_t> ring;
        for (size_t q = front; q < end; ++q) {
            const int32_t v = P.vert[q];
            for (int32_t e = M.ptr[v]; e < M.ptr[v + 1]; ++e) {
                const int32_t u = M.col[e];
                if (dist[u] < 0) {
                    dist[u] = d;
                    ring.push_back(u);
                }
            }
        }
        std::sort(ring.begin(), ring.end());
        P.vert.insert(P.vert.end(), ring.begin(), ring.end());
        front = end;
    }
    const int32_t L = (int32_t)P.vert.size();
    if (L > lmax) {
        for (int32_t v : P.vert) dist[v] = -1;
        return;
    }
    for (int32_t l = 0; l < L; ++l) loc[P.vert[l]] = l;
    P.cnt.assign(s + 1, 0);
    for (int32_t l = 0; l < L; ++l) P.cnt[dist[P.vert[l]]]++;
    for (int d = 1; d <= s; ++d) P.cnt[d] += P.cnt[d - 1];   // cnt[d] = vertices within d edges
    P.dinv.assign(L, 0.0);
    P.rptr.assign(L + 1, 0);
    P.col.clear();
    P.val.clear();
    for (int32_t l = 0; l < L; ++l) {
        const int32_t v = P.vert[l];
        double diag = 0.0;
        for (int32_t e = M.ptr[v]; e < M.ptr[v + 1]; ++e)
            if (M.col[e] == v) diag += M.val[e];
        P.dinv[l] = 1.0 / diag;
        if (dist[v] < s)   // rows read only at the steps that update them
            for (int32_t e = M.ptr[v]; e < M.ptr[v + 1]; ++e) {
                P.col.push_back(loc[M.col[e]]);
                P.val.push_back(M.val[e]);
            }
        P.rptr[l + 1] = (int32_t)P.col.size();
    }
    for (int32_t v : P.vert) {
        dist[v] = -1;
        loc[v] = -1;
    }
}

}  // namespace

bem_status cheb_tables(const Csr M[2], int s, ChebTables &T)
{
    T.s = s;
    // Rows are the same in every patch, so their width is looked at first.
    for (int m = 0; m < 2; ++m)
        for (int64_t v = 0; v < M[m].nrows; ++v)
            if (M[m].ptr[v + 1] - M[m].ptr[v] > CHEB_WMAX)
                return set_error(BEM_E_MESH, "inverse-mass rows wider than the kernel's limit "
                                             "(a vertex with more than 15 neighbours)");
    // Owned vertices per patch: halved until the largest patch fits the kernel's register and LDS budget.  A patch
    // that does not fit ends its try at once.  (Steps of an eighth find larger patches, 448 owned for 10,242 + 8,002
    // vertices: 64 runs 436 -> 317 us per launch, but one run, whose launch takes as long as its largest patch, 18.3 ->
    // 20.2 us.)
    for (int own = CHEB_OWN_MAX; own >= 32; own /= 2) {
        std::atomic<bool> over{false};
        std::vector<Patch> patches;
        std::vector<int32_t> pm;
        for (int m = 0; m < 2 && !over; ++m) {
            const int32_t nv = (int32_t)M[m].nrows;
            const std::vector<std::vector<int32_t>> cl = clusters(M[m], own);
            const int32_t np = (int32_t)cl.size();
            T.nparts[m] = np;
            const size_t first = patches.size();
            patches.resize(first + np);
            pm.insert(pm.end(), np, m);
            parallel_for(np, 1, [&](int64_t a, int64_t b) {
                std::vector<int32_t> dist(nv, -1), loc(nv, -1);
                for (int64_t q = a; q < b && !over; ++q) {
                    build_patch(M[m], cl[q], s, CHEB_LMAX, dist, loc, patches[first + q]);
                    if (patches[first + q].vert.size() > (size_t)CHEB_LMAX) over = true;
                }
            });
        }
        if (over) continue;
        int lmax = 0;
        for (const Patch &P : patches) lmax = std::max(lmax, (int)P.vert.size());
        T.own = own;
        T.lmax = lmax;
        T.pmesh.assign(pm.begin(), pm.end());
        const int32_t np = (int32_t)patches.size();
        T.vbeg.assign(np + 1, 0);
        for (int32_t q = 0; q < np; ++q) T.vbeg[q + 1] = T.vbeg[q] + (int32_t)patches[q].vert.size();
        T.cnt.resize((size_t)np * (s + 1));
        T.vert.resize(T.vbeg[np]);
        T.dinv.resize(T.vbeg[np]);
        // the rows as ELL blocks per patch, [q][local row], for the kernel, which keeps a row's entries in
        // registers for all steps of a launch: w columns beside the diagonal, padded with zero entries on the
        // row's own vertex, and w + 1 values, the diagonal first
        int w = 1;
        for (int m = 0; m < 2; ++m)
            for (int64_t v = 0; v < M[m].nrows; ++v) w = std::max(w, M[m].ptr[v + 1] - M[m].ptr[v] - 1);
        T.ell_w = w;
        T.ecol.resize((size_t)w * T.vert.size());
        T.eval.resize((size_t)(w + 1) * T.vert.size());
        parallel_for(np, 1, [&](int64_t q0, int64_t q1) {
            for (int64_t q = q0; q < q1; ++q) {
                const Patch &P = patches[q];
                const int32_t vb = T.vbeg[q], L = (int32_t)P.vert.size();
                std::copy(P.cnt.begin(), P.cnt.end(), T.cnt.begin() + q * (s + 1));
                std::copy(P.vert.begin(), P.vert.end(), T.vert.begin() + vb);
                std::copy(P.dinv.begin(), P.dinv.end(), T.dinv.begin() + vb);
                uint16_t *ec = T.ecol.data() + (size_t)w * vb;
                double *ev = T.eval.data() + (size_t)(w + 1) * vb;
                std::fill(ev, ev + (size_t)(w + 1) * L, 0.0);
                for (int32_t l = 0; l < L; ++l) {
                    int e = 0;
                    for (int32_t k = P.rptr[l]; k < P.rptr[l + 1]; ++k) {
                        if (P.col[k] == l) {
                            ev[l] += P.val[k];
                            continue;
                        }
                        ec[(size_t)e * L + l] = (uint16_t)P.col[k];
                        ev[(size_t)(e + 1) * L + l] = P.val[k];
                        ++e;
                    }
                    for (; e < w; ++e) ec[(size_t)e * L + l] = (uint16_t)l;
                }
            }
        });
        return BEM_OK;
    }
    return set_error(BEM_E_MESH, "inverse-mass patches exceed the kernel's limit");
}

}  // namespace bemtx
