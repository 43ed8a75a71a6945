// geometry.hip -- the median-dual geometry loop over tets and its reverse.
//
// Inside a tet (p, q, r, s) the dual face between the cells of p and q joins
// the edge midpoint, the centroids of the faces pqr and pqs and the tet
// centroid; its area vector is half the cross product of that quadrilateral's
// diagonals, (x_r + x_s - x_p - x_q) x (x_s - x_r) / 24, pointing from p to q
// when (p, q, r, s) has the tet's orientation.  Each vertex owns a quarter of
// the tet's volume.  These are the edge weights and node volumes that the edge
// loops read (the per-edge data of the edge loops, Sec. 4); computing them on
// the device, and their reverse, lets the flux adjoint's weight sensitivities
// reach the node coordinates.
//
// Two forms.  Scatter: one thread per tet adds its six face vectors and four
// volume quarters (or, in reverse, its four x-bar shares) to HBM with FP64
// atomics.  Gather: no atomics, fixed summation orders, the same bits on every
// run.  The forward gather walks the tets around each edge from coordinates
// staged in LDS (ring form, below), the gather reverse the edges around each
// node (link form, at the end).  Where a mesh does not fit them, per-tet results
// go to a scratch buffer that one thread per edge or node then sums over its
// incident tets.  The loop runs once per mesh (or once per design step for the
// reverse).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "kernels.hpp"

namespace opf {
namespace gpu {
namespace {

// Local edge k: vertices (a, b) and the completing pair (r, s) such that
// (a, b, r, s) is an even permutation of (0, 1, 2, 3).
constexpr int kTetEdge[6][4] = {{0, 1, 2, 3}, {0, 2, 3, 1}, {0, 3, 1, 2},
                                   {1, 2, 0, 3}, {1, 3, 2, 0}, {2, 3, 0, 1}};

__device__ __forceinline__ void cross3(const double *a, const double *b, double *c)
{
    c[0] = a[1] * b[2] - a[2] * b[1];
    c[1] = a[2] * b[0] - a[0] * b[2];
    c[2] = a[0] * b[1] - a[1] * b[0];
}

__device__ __forceinline__ void tet_x(const TetArrays &a, const int *g, double period, double x[4][3])
{
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
        for (int d = 0; d < 3; ++d) x[v][d] = a.x[d][g[v]];
    if (period > 0.0) {
        const double ip = 1.0 / period;
#pragma unroll
        for (int v = 1; v < 4; ++v)
#pragma unroll
            for (int d = 0; d < 3; ++d) x[v][d] -= period * rint((x[v][d] - x[0][d]) * ip);
    }
}

// +1 if edge e runs from node na to node nb, else -1 (the map guarantees it
// is one of the two).
__device__ __forceinline__ double orient(const int2 *e2n, int e, int na)
{
    return e2n[e].x == na ? 1.0 : -1.0;
}

__global__ __launch_bounds__(256) void k_geometry(int T, TetArrays a, double period)
{
    const int t = (int)blockIdx.x * 256 + (int)threadIdx.x;
    if (t >= T) return;
    int g[4], ed[6];
#pragma unroll
    for (int v = 0; v < 4; ++v) g[v] = a.t2n[4 * t + v];
#pragma unroll
    for (int k = 0; k < 6; ++k) ed[k] = a.t2e[6 * t + k];
    double x[4][3];
    tet_x(a, g, period, x);
#pragma unroll
    for (int k = 0; k < 6; ++k) {
        const int p = kTetEdge[k][0], q = kTetEdge[k][1], r = kTetEdge[k][2], s = kTetEdge[k][3];
        double u[3], v[3], c[3];
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            u[d] = x[r][d] + x[s][d] - x[p][d] - x[q][d];
            v[d] = x[s][d] - x[r][d];
        }
        cross3(u, v, c);
        const double sg = orient(a.e2n, ed[k], g[p]) * (1.0 / 24.0);
#pragma unroll
        for (int d = 0; d < 3; ++d) unsafeAtomicAdd(a.w[d] + ed[k], sg * c[d]);
    }
    double e1[3], e2[3], e3[3], c[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        e1[d] = x[1][d] - x[0][d];
        e2[d] = x[2][d] - x[0][d];
        e3[d] = x[3][d] - x[0][d];
    }
    cross3(e2, e3, c);
    const double q4 = (e1[0] * c[0] + e1[1] * c[1] + e1[2] * c[2]) * (1.0 / 24.0);
#pragma unroll
    for (int v = 0; v < 4; ++v) unsafeAtomicAdd(a.vol + g[v], q4);
}

__global__ __launch_bounds__(256) void k_geometry_adj(int T, TetArrays a, double period)
{
    const int t = (int)blockIdx.x * 256 + (int)threadIdx.x;
    if (t >= T) return;
    int g[4], ed[6];
#pragma unroll
    for (int v = 0; v < 4; ++v) g[v] = a.t2n[4 * t + v];
#pragma unroll
    for (int k = 0; k < 6; ++k) ed[k] = a.t2e[6 * t + k];
    double x[4][3], xb[4][3];
    tet_x(a, g, period, x);
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
        for (int d = 0; d < 3; ++d) xb[v][d] = 0.0;
    // face vector c = u x v / 24: ubar = v x cbar / 24, vbar = cbar x u / 24
#pragma unroll
    for (int k = 0; k < 6; ++k) {
        const int p = kTetEdge[k][0], q = kTetEdge[k][1], r = kTetEdge[k][2], s = kTetEdge[k][3];
        const double sg = orient(a.e2n, ed[k], g[p]) * (1.0 / 24.0);
        double u[3], v[3], cb[3], ub[3], vb[3];
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            u[d] = x[r][d] + x[s][d] - x[p][d] - x[q][d];
            v[d] = x[s][d] - x[r][d];
            cb[d] = sg * a.w[d][ed[k]];
        }
        cross3(v, cb, ub);
        cross3(cb, u, vb);
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            xb[p][d] -= ub[d];
            xb[q][d] -= ub[d];
            xb[r][d] += ub[d] - vb[d];
            xb[s][d] += ub[d] + vb[d];
        }
    }
    // volume V = e1 . (e2 x e3) / 6 with e_k = x_k - x_0, a quarter to each vertex
    const double Vb = 0.25 * (a.vol[g[0]] + a.vol[g[1]] + a.vol[g[2]] + a.vol[g[3]]) * (1.0 / 6.0);
    double e1[3], e2[3], e3[3], c1[3], c2[3], c3[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        e1[d] = x[1][d] - x[0][d];
        e2[d] = x[2][d] - x[0][d];
        e3[d] = x[3][d] - x[0][d];
    }
    cross3(e2, e3, c1);
    cross3(e3, e1, c2);
    cross3(e1, e2, c3);
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        xb[1][d] += Vb * c1[d];
        xb[2][d] += Vb * c2[d];
        xb[3][d] += Vb * c3[d];
        xb[0][d] -= Vb * (c1[d] + c2[d] + c3[d]);
    }
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
        for (int d = 0; d < 3; ++d) unsafeAtomicAdd(a.xbar[d] + g[v], xb[v][d]);
}

// ---------------------------------------------------------- gather form -- */
//
// Phase 1, one thread per tet (tets in the order of the incidence lists, so
// the map reads coalesce): the tet's results go to the scratch buffer as one
// record per tet.  Phase 2, one thread per edge or node: the sum over its
// incident tets, in list order; the tets around an edge or a node are close
// in that order, so their records share cache lines.

// record of tet t: the signed face vector of local edge k / 24 at
// scratch[18 t + 3k + d]; the volume determinant / 24 at scratch[18 T + t] (an
// array of its own, so that the per-node sums read 16 tets per cache line)
__global__ __launch_bounds__(256) void k_tet_forward(int T, TetArrays a, double period)
{
    const int t = (int)blockIdx.x * 256 + (int)threadIdx.x;
    if (t >= T) return;
    int g[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) g[v] = a.t2n[4 * t + v];
    double x[4][3];
    tet_x(a, g, period, x);
    double *rec = a.scratch + (size_t)t * 18;
#pragma unroll
    for (int k = 0; k < 6; ++k) {
        const int p = kTetEdge[k][0], q = kTetEdge[k][1], r = kTetEdge[k][2], s = kTetEdge[k][3];
        double u[3], v[3], c[3];
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            u[d] = x[r][d] + x[s][d] - x[p][d] - x[q][d];
            v[d] = x[s][d] - x[r][d];
        }
        cross3(u, v, c);
        const double sg = (a.t2e[6 * t + k] < 0 ? -1.0 : 1.0) * (1.0 / 24.0);
#pragma unroll
        for (int d = 0; d < 3; ++d) rec[3 * k + d] = sg * c[d];
    }
    double e1[3], e2[3], e3[3], c[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        e1[d] = x[1][d] - x[0][d];
        e2[d] = x[2][d] - x[0][d];
        e3[d] = x[3][d] - x[0][d];
    }
    cross3(e2, e3, c);
    a.scratch[(size_t)18 * T + t] = (e1[0] * c[0] + e1[1] * c[1] + e1[2] * c[2]) * (1.0 / 24.0);
}

// The sums below walk a list in order; they fetch kSumAhead entries at a
// time (these loops are latency-bound) and add them in list order.
constexpr int kSumAhead = 4;

// w[e] += sum over the tets around e of their face vector of e
__global__ __launch_bounds__(256) void k_edge_sum_faces(TetArrays a)
{
    const int e = (int)blockIdx.x * 256 + (int)threadIdx.x;
    if (e >= a.E) return;
    double acc[3] = {0.0, 0.0, 0.0};
    const int end = a.e2t_off[e + 1];
    for (int j = a.e2t_off[e]; j < end; j += kSumAhead) {
        double r[kSumAhead][3];
#pragma unroll
        for (int u = 0; u < kSumAhead; ++u) {
            // past the end of the list: re-read its first entry (always valid)
            const int tk = a.e2t[j + u < end ? j + u : j];
            const double *rec = a.scratch + (size_t)(tk >> 3) * 18 + 3 * (tk & 7);
#pragma unroll
            for (int d = 0; d < 3; ++d) r[u][d] = rec[d];
        }
#pragma unroll
        for (int u = 0; u < kSumAhead; ++u)
#pragma unroll
            for (int d = 0; d < 3; ++d)
                if (j + u < end) acc[d] += r[u][d];
    }
#pragma unroll
    for (int d = 0; d < 3; ++d) a.w[d][e] = (a.write_w ? 0.0 : a.w[d][e]) + acc[d];
}

// vol[i] += sum over the tets around i of a quarter of their volume
__global__ __launch_bounds__(256) void k_node_sum_vol(int T, TetArrays a)
{
    const int i = (int)blockIdx.x * 256 + (int)threadIdx.x;
    if (i >= a.N) return;
    const double *det = a.scratch + (size_t)18 * T;
    double acc = 0.0;
    const int end = a.n2t_off[i + 1];
    for (int j = a.n2t_off[i]; j < end; j += kSumAhead) {
        double r[kSumAhead];
#pragma unroll
        for (int u = 0; u < kSumAhead; ++u) {
            r[u] = det[a.n2t[j + u < end ? j + u : j] >> 2];
        }
#pragma unroll
        for (int u = 0; u < kSumAhead; ++u)
            if (j + u < end) acc += r[u];
    }
    a.vol[i] = (a.write_vol ? 0.0 : a.vol[i]) + acc;
}

// The reverse of one tet at coordinates x (unwrapped): its x-bar shares xb
// from the signed weight adjoints cb[k] = +-wbar / 24 of its six local edges
// and the sum vbs of its vertices' volume adjoints (a quarter of the volume
// to each vertex).  Face c = u x v / 24: ubar = v x cbar, vbar = cbar x u.
__device__ __forceinline__ void tet_shares(const double (&x)[4][3], const double (&cb)[6][3],
                                           double vbs, double (&xb)[4][3])
{
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
        for (int d = 0; d < 3; ++d) xb[v][d] = 0.0;
#pragma unroll
    for (int k = 0; k < 6; ++k) {
        const int p = kTetEdge[k][0], q = kTetEdge[k][1], r = kTetEdge[k][2], s = kTetEdge[k][3];
        double u[3], v[3], ub[3], vb[3];
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            u[d] = x[r][d] + x[s][d] - x[p][d] - x[q][d];
            v[d] = x[s][d] - x[r][d];
        }
        cross3(v, cb[k], ub);
        cross3(cb[k], u, vb);
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            xb[p][d] -= ub[d];
            xb[q][d] -= ub[d];
            xb[r][d] += ub[d] - vb[d];
            xb[s][d] += ub[d] + vb[d];
        }
    }
    // volume V = e1 . (e2 x e3) / 6 with e_k = x_k - x_0
    const double Vb = 0.25 * vbs * (1.0 / 6.0);
    double e1[3], e2[3], e3[3], c1[3], c2[3], c3[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        e1[d] = x[1][d] - x[0][d];
        e2[d] = x[2][d] - x[0][d];
        e3[d] = x[3][d] - x[0][d];
    }
    cross3(e2, e3, c1);
    cross3(e3, e1, c2);
    cross3(e1, e2, c3);
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        xb[1][d] += Vb * c1[d];
        xb[2][d] += Vb * c2[d];
        xb[3][d] += Vb * c3[d];
        xb[0][d] -= Vb * (c1[d] + c2[d] + c3[d]);
    }
}

// the six weight adjoints of tet t, read from their interleaved copy wT
__device__ __forceinline__ void tet_wbar(const TetArrays &a, int t, double (&cb)[6][3])
{
#pragma unroll
    for (int k = 0; k < 6; ++k) {
        const int ew = a.t2e[6 * t + k], ed = ew & 0x7fffffff;
        const double sg = (ew < 0 ? -1.0 : 1.0) * (1.0 / 24.0);
#pragma unroll
        for (int d = 0; d < 3; ++d) cb[k][d] = sg * a.wT[3 * (size_t)ed + d];
    }
}

// wT[3 e + d] = wbar[d][e]: one 24-byte record per edge for the tets' gathers
__global__ __launch_bounds__(256) void k_interleave_w(TetArrays a)
{
    const int e = (int)blockIdx.x * 256 + (int)threadIdx.x;
    if (e >= a.E) return;
#pragma unroll
    for (int d = 0; d < 3; ++d) a.wT[3 * (size_t)e + d] = a.w[d][e];
}

// the share of x-bar of tet t at its local vertex v: 3 doubles at the
// (tet, vertex) pair's slot in the node-major list n2t
__device__ __forceinline__ void put_shares(const TetArrays &a, int t, const double (&xb)[4][3])
{
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        double *rec = a.scratch + (size_t)3 * a.n2t_pos[4 * t + v];
#pragma unroll
        for (int d = 0; d < 3; ++d) rec[d] = xb[v][d];
    }
}

__global__ __launch_bounds__(256) void k_tet_reverse(int T, TetArrays a, double period)
{
    const int t = (int)blockIdx.x * 256 + (int)threadIdx.x;
    if (t >= T) return;
    int g[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) g[v] = a.t2n[4 * t + v];
    double x[4][3], xb[4][3], cb[6][3];
    tet_x(a, g, period, x);
    tet_wbar(a, t, cb);
    tet_shares(x, cb, a.vol[g[0]] + a.vol[g[1]] + a.vol[g[2]] + a.vol[g[3]], xb);
    put_shares(a, t, xb);
}

// xbar[i] += sum over the tets around i of their share at i: one contiguous
// run of records per node
__global__ __launch_bounds__(256) void k_node_sum_xbar(TetArrays a)
{
    const int i = (int)blockIdx.x * 256 + (int)threadIdx.x;
    if (i >= a.N) return;
    double acc[3] = {0.0, 0.0, 0.0};
    const int end = a.n2t_off[i + 1];
    for (int j = a.n2t_off[i]; j < end; j += kSumAhead) {
        double r[kSumAhead][3];
#pragma unroll
        for (int u = 0; u < kSumAhead; ++u) {
            const double *rec = a.scratch + (size_t)3 * (j + u < end ? j + u : j);
#pragma unroll
            for (int d = 0; d < 3; ++d) r[u][d] = rec[d];
        }
#pragma unroll
        for (int u = 0; u < kSumAhead; ++u)
#pragma unroll
            for (int d = 0; d < 3; ++d)
                if (j + u < end) acc[d] += r[u][d];
    }
#pragma unroll
    for (int d = 0; d < 3; ++d) a.xbar[d][i] += acc[d];
}

// ------------------------------------------------------------ ring form -- */
//
// The forward gather without per-tet records.  One workgroup per chunk of KG
// consecutive nodes stages the coordinates of its nodes and of its halo (the
// other vertices of the tets around its edges) in LDS; then one thread per
// edge of the chunk walks the tets around its edge in list order.  Around edge
// (a, b), tet (a, b, r, s) gives the face (x_r + x_s - x_a - x_b) x (x_s - x_r)
// / 24 (the formula above with p = a, q = b) and the determinant
// (x_b - x_a) . ((x_r - x_a) x (x_s - x_a)), six times the tet's volume; every
// difference is taken from x_a (wrapped to its nearest image in a periodic
// box).  The edge's weight gets the sum of its faces, and the sum of its
// determinants goes to edge_det; a node's volume is then the sum over its
// edges of edge_det / 72: a tet lies around three of its edges at each vertex,
// and each vertex owns a quarter of its volume.  Fixed orders throughout: the
// same bits on every run.

__device__ __forceinline__ void geo_diff(const double *x, const double *a, bool wrap, double period,
                                         double ip, double *d)
{
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        d[k] = x[k] - a[k];
        if (wrap) d[k] -= period * rint(d[k] * ip);
    }
}

// LDS rows: plane of (x, y) pairs, then plane of z (L rows each).
__device__ __forceinline__ void geo_get(const double *X, int L, uint32_t l, double *x)
{
    const double2 xy = reinterpret_cast<const double2 *>(X)[l];
    x[0] = xy.x;
    x[1] = xy.y;
    x[2] = X[2 * L + l];
}

// The edges of a chunk go in batches of kGeoThreads, one per thread (workgroup
// blockIdx.y of gridDim.y taking every gridDim.y-th batch); each batch's ring
// entries (one contiguous run) are first copied to LDS by the
// whole workgroup, so that the walks read LDS only.  Around edge (a, b) with
// chain c_0 .. c_k and d_i = x_(c_i) - x_a, tet i contributes
// (d_(i-1) + d_i - d_b) x (d_i - d_(i-1)) / 24 = (2 d_(i-1) x d_i
// - d_b x (d_i - d_(i-1))) / 24 to the face and d_b . (d_(i-1) x d_i) to the
// determinant sum; summed over the chain, the d_b terms telescope to
// d_b x (d_k - d_0), zero on a closed ring.  One vertex and one cross product
// per tet.
__global__ __launch_bounds__(kGeoThreads) void k_geo_rings(TetArrays a, double period)
{
    extern __shared__ __align__(16) unsigned char smem[];
    double *X = reinterpret_cast<double *>(smem);
    uint32_t *R32 = reinterpret_cast<uint32_t *>(smem + (size_t)a.L * 24);
    const uint16_t *R16 = reinterpret_cast<const uint16_t *>(R32);
    const uint32_t *ring32 = reinterpret_cast<const uint32_t *>(a.ring);
    const int L = a.L, KG = a.KG, c = (int)blockIdx.x, t = (int)threadIdx.x;
    const int v0 = c * KG, nown = min(KG, a.N - v0);
    const int h0 = a.halo_off[c], nh = a.halo_off[c + 1] - h0;
    const int2 ce = a.chunk_e[c];
    // the words of a batch: whole 4-byte words covering its entries, kGeoPre
    // per thread at most; the next batch's are loaded while this one computes
    uint32_t pre[kGeoPre];
    auto fetch = [&](int b0, int &q0, int &nq) {
        const int eb = ce.x + b0, nb = min(kGeoThreads, ce.y - b0);
        const int wb = a.ring_off[eb], we = a.ring_off[eb + nb];
        q0 = wb >> 1;
        nq = ((we + 1) >> 1) - q0;
#pragma unroll
        for (int u = 0; u < kGeoPre; ++u) {
            const int j = t + u * kGeoThreads;
            if (j < nq) pre[u] = ring32[q0 + j];
        }
    };
    const int first = (int)blockIdx.y * kGeoThreads, step = (int)gridDim.y * kGeoThreads;
    if (first >= ce.y) return;
    int q0 = 0, nq = 0;
    fetch(first, q0, nq);
    for (int l = t; l < nown + nh; l += kGeoThreads) {
        const bool own = l < nown;
        const int g = own ? v0 + l : a.halo[h0 + l - nown];
        const int row = own ? l : KG + l - nown;
        reinterpret_cast<double2 *>(X)[row] = make_double2(a.x[0][g], a.x[1][g]);
        X[2 * L + row] = a.x[2][g];
    }
    const bool wrap = period > 0.0;
    const double ip = wrap ? 1.0 / period : 0.0;
    for (int b0 = first; b0 < ce.y; b0 += step) {
        const int nb = min(kGeoThreads, ce.y - b0), eb = ce.x + b0;
        const int sh = 2 * q0;  // entry o of this batch sits at R16[o - sh]
        const bool act = t < nb;
        const int e = eb + t;
        int o0 = 0, o1 = 0;
        double w0[3] = {0.0, 0.0, 0.0};
        if (act) {
            o0 = a.ring_off[e] - sh;
            o1 = a.ring_off[e + 1] - sh;
            if (!a.write_w)
#pragma unroll
                for (int d = 0; d < 3; ++d) w0[d] = a.w[d][e];
        }
        __syncthreads();  // coordinates staged; the last batch's entries read
#pragma unroll
        for (int u = 0; u < kGeoPre; ++u) {
            const int j = t + u * kGeoThreads;
            if (j < nq) R32[j] = pre[u];
        }
        __syncthreads();
        if (b0 + step < ce.y) fetch(b0 + step, q0, nq);
        if (!act) continue;
        double xa[3], xb[3], db[3], d0[3], dp[3];
        geo_get(X, L, R16[o0], xa);
        geo_get(X, L, R16[o0 + 1], xb);
        geo_diff(xb, xa, wrap, period, ip, db);
        geo_get(X, L, R16[o0 + 2], d0);
        geo_diff(d0, xa, wrap, period, ip, d0);
#pragma unroll
        for (int d = 0; d < 3; ++d) dp[d] = d0[d];
        double C[3] = {0.0, 0.0, 0.0};
        for (int j = o0 + 3; j < o1; ++j) {
            double xn[3], dn[3], cr[3];
            geo_get(X, L, R16[j], xn);
            geo_diff(xn, xa, wrap, period, ip, dn);
            cross3(dp, dn, cr);
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                C[d] += cr[d];
                dp[d] = dn[d];
            }
        }
        double ds[3], corr[3];
#pragma unroll
        for (int d = 0; d < 3; ++d) ds[d] = dp[d] - d0[d];
        cross3(db, ds, corr);
#pragma unroll
        for (int d = 0; d < 3; ++d) a.w[d][e] = w0[d] + (2.0 * C[d] - corr[d]) * (1.0 / 24.0);
        a.edge_det[e] = db[0] * C[0] + db[1] * C[1] + db[2] * C[2];
    }
}

// Volumes, one workgroup per chunk: the determinant sums of the edges at its
// nodes go to LDS (its own edge range, coalesced, then the edges it shares
// with lower chunks, vsec), and each node adds those of its edges in the
// order of its slot list vloc: vol (+)= sum / 72.
__global__ __launch_bounds__(kGeoVolThreads) void k_geo_vol(TetArrays a)
{
    extern __shared__ __align__(16) unsigned char smem[];
    double *D = reinterpret_cast<double *>(smem);
    const int c = (int)blockIdx.x, t = (int)threadIdx.x;
    const int v0 = c * a.KG, nown = min(a.KG, a.N - v0);
    const int2 ce = a.chunk_e[c];
    const int s0 = a.vsec_off[c], ns = a.vsec_off[c + 1] - s0;
    for (int j = t; j < ce.y; j += kGeoVolThreads) D[j] = a.edge_det[ce.x + j];
    for (int j = t; j < ns; j += kGeoVolThreads) D[ce.y + j] = a.edge_det[a.vsec[s0 + j]];
    __syncthreads();
    for (int l = t; l < nown; l += kGeoVolThreads) {
        const int i = v0 + l;
        const double vi = a.write_vol ? 0.0 : a.vol[i];
        double acc = 0.0;
        const int end = a.vloc_off[i + 1];
        for (int j = a.vloc_off[i]; j < end; ++j) acc += D[a.vloc[j]];
        a.vol[i] = vi + acc * (1.0 / 72.0);
    }
}

// ------------------------------------------------------------ link form -- */
//
// The reverse without per-tet records.  Where the tets around edge (a, b) close
// a ring, its weight is the sum of c_(i-1) x c_i / 12 over the ring (the terms
// in a and b cancel), so only the ring's vertices see it: vertex c_i gets
// wbar x (c_(i-1) - c_(i+1)) / 12.  A node thus sums over the edges of its link
// (the edges in whose ring it stands, 36 on average) the edge's adjoint crossed
// with the difference of the two vertices next to it.  Those two, r and s, are
// also the apexes of the two tets (a, b, r, v) and (a, b, v, s) on the two sides
// of the triangle (a, b, v), whose volumes change with v by (a x b + b x r +
// r x a) / 6 and -(a x b + b x s + s x a) / 6 (all from v); a tet's volume
// adjoint is a quarter of the sum over its vertices, so the a x b terms of the
// two add up to (volbar_r - volbar_s) / 24 (a x b), and the other terms are
// those of the tets' other link edges.  One workgroup per chunk stages the
// coordinates, volume adjoints and edge adjoints its nodes need in LDS, then
// kLinkSplit threads per node walk its entries and add their sums in a fixed
// order: the same bits on every run.
// Against per-tet records (every tet's shares written, then summed per node:
// 11.7 GB moved on the 160^3 box for 1.8 GB it needs) the 1M-node box takes 237 us
// instead of 730.  What bounds it now is the staging: 20 cache lines per node
// go from L2 to the CUs (2.5 GB, about 10 TB/s), since a chunk's edges share
// their lines with those of its neighbours; without the edge adjoints it takes
// 190 us, without the walk 225.  Larger chunks (76 KB of LDS, two workgroups per
// CU) and smaller ones (38 KB, four) are 1-3 % slower; 512-node chunks that take
// their edges in slices of 1024 halve those lines but wait at each slice
// (718 us).  All loads are issued before the first wait: one dependent trip each
// for offsets, indices and data.
constexpr int kLinkAhead = 10;  // entries of a thread fetched before the staging
constexpr int kLinkBatch = 4;   // edge adjoints of a thread in flight together

template <bool WRAP, bool VOL>
__device__ __forceinline__ void link_walk(const TetArrays &a, const double2 *XY, const double2 *ZV,
                                          const double2 *W01, const double *W2, int e0, int v, int j0,
                                          int j1, const uint32_t (&pre)[kLinkAhead], double period,
                                          double (&out)[3])
{
    const double ip = WRAP ? 1.0 / period : 0.0;
    const double2 vxy = XY[v], vzv = ZV[v];
    const double xv[3] = {vxy.x, vxy.y, vzv.x};
    // row l relative to v
    auto from_v = [&](uint32_t l, double *d, double &vb) {
        const double2 xy = XY[l], zv = ZV[l];
        const double x[3] = {xy.x, xy.y, zv.x};
        geo_diff(x, xv, WRAP, period, ip, d);
        vb = zv.y;
    };
    double sw[3] = {0.0, 0.0, 0.0}, sv[3] = {0.0, 0.0, 0.0};
    auto entry = [&](uint32_t en) {
        const uint32_t slot = en & 0xfffu;
        const double2 w01 = W01[slot];
        const double wb[3] = {w01.x, w01.y, W2[slot]};
        double dr[3], ds[3], d[3], c[3], vr, vs;
        from_v((en >> 12) & 0x3ffu, dr, vr);
        from_v(en >> 22, ds, vs);
#pragma unroll
        for (int k = 0; k < 3; ++k) d[k] = dr[k] - ds[k];
        cross3(wb, d, c);
#pragma unroll
        for (int k = 0; k < 3; ++k) sw[k] += c[k];
        if constexpr (VOL) {
            const uint32_t ab = a.lk_ends[e0 + slot];
            double da[3], db[3], un;
            from_v(ab & 0xffffu, da, un);
            from_v(ab >> 16, db, un);
            cross3(da, db, c);
#pragma unroll
            for (int k = 0; k < 3; ++k) sv[k] += (vr - vs) * c[k];
        }
    };
#pragma unroll
    for (int i = 0; i < kLinkAhead; ++i)
        if (j0 + i * kLinkSplit < j1) entry(pre[i]);
    for (int j = j0 + kLinkAhead * kLinkSplit; j < j1; j += kLinkSplit) entry(a.lk_ent[j]);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        out[k] = sw[k] * (1.0 / 12.0);
        if constexpr (VOL) out[k] += sv[k] * (1.0 / 24.0);
    }
}

__global__ __launch_bounds__(kLinkThreads, 6) void k_link_reverse(TetArrays a, double period)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const int c = xcd_map((int)blockIdx.x, (int)gridDim.x), t = (int)threadIdx.x;
    const int v0 = a.lk_node[c], nown = a.lk_node[c + 1] - v0;
    const int h0 = a.lk_halo_off[c], rows = nown + a.lk_halo_off[c + 1] - h0;
    const int e0 = a.lk_edge_off[c], ne = a.lk_edge_off[c + 1] - e0;
    double2 *XY = reinterpret_cast<double2 *>(smem), *ZV = XY + rows, *W01 = ZV + rows;
    double *W2 = reinterpret_cast<double *>(W01 + ne);
    const int v = t / kLinkSplit, part = t % kLinkSplit;
    const bool act = v < nown;
    const int j0 = act ? a.lk_ent_off[v0 + v] + part : 0, j1 = act ? a.lk_ent_off[v0 + v + 1] : 0;
    uint32_t pre[kLinkAhead];
#pragma unroll
    for (int i = 0; i < kLinkAhead; ++i) pre[i] = j0 + i * kLinkSplit < j1 ? a.lk_ent[j0 + i * kLinkSplit] : 0u;
    // coordinates, then edge adjoints: the first of both in flight together
    const double r0 = a.x[0][v0], r1 = a.x[1][v0], r2 = a.x[2][v0], vb0 = a.vol[v0];
    int e[kLinkBatch];
    auto ids = [&](int b) {
#pragma unroll
        for (int i = 0; i < kLinkBatch; ++i) e[i] = a.lk_edge[e0 + min(b + i * kLinkThreads, ne - 1)];
    };
    if (ne > 0) ids(t);
    int need = 0;
    auto row = [&](int l, double x, double y, double z, double vb) {
        XY[l] = make_double2(x, y);
        ZV[l] = make_double2(z, vb);
        // differences need no wrap where every row is within a quarter period of
        // the first; the volume part is zero where all volume adjoints are equal
        const double far = fmax(fabs(x - r0), fmax(fabs(y - r1), fabs(z - r2)));
        need |= (period > 0.0 && !(far <= 0.25 * period) ? 1 : 0) | (vb - vb0 == 0.0 ? 0 : 2);
    };
    auto node = [&](int l) { return l < nown ? v0 + l : a.lk_halo[h0 + l - nown]; };
    const int g0 = node(min(t, rows - 1));
    const double x0 = a.x[0][g0], y0 = a.x[1][g0], z0 = a.x[2][g0], q0 = a.vol[g0];
    for (int b = t; b < ne; b += kLinkThreads * kLinkBatch) {
        double w[kLinkBatch][3];
#pragma unroll
        for (int i = 0; i < kLinkBatch; ++i)
#pragma unroll
            for (int d = 0; d < 3; ++d) w[i][d] = a.w[d][e[i]];
        if (b == t && t < rows) row(t, x0, y0, z0, q0);
#pragma unroll
        for (int i = 0; i < kLinkBatch; ++i) {
            const int j = b + i * kLinkThreads;
            if (j < ne) {
                W01[j] = make_double2(w[i][0], w[i][1]);
                W2[j] = w[i][2];
            }
        }
        if (b + kLinkThreads * kLinkBatch < ne) ids(b + kLinkThreads * kLinkBatch);
    }
    if (t >= ne && t < rows) row(t, x0, y0, z0, q0);
    for (int l = t + kLinkThreads; l < rows; l += kLinkThreads) {
        const int g = node(l);
        row(l, a.x[0][g], a.x[1][g], a.x[2][g], a.vol[g]);
    }
    constexpr int NW = kLinkThreads / 64;
    __shared__ int needs[NW];
    const int any = (__any(need & 1) ? 1 : 0) | (__any(need & 2) ? 2 : 0);
    if ((t & 63) == 0) needs[t >> 6] = any;
    __syncthreads();
    int all = 0;
#pragma unroll
    for (int i = 0; i < NW; ++i) all |= needs[i];
    const bool wrap = all & 1, vol = all & 2;
    double s[3];
    const int vr = act ? v : 0;
    if (vol) {
        if (wrap) link_walk<true, true>(a, XY, ZV, W01, W2, e0, vr, j0, j1, pre, period, s);
        else link_walk<false, true>(a, XY, ZV, W01, W2, e0, vr, j0, j1, pre, period, s);
    } else {
        if (wrap) link_walk<true, false>(a, XY, ZV, W01, W2, e0, vr, j0, j1, pre, period, s);
        else link_walk<false, false>(a, XY, ZV, W01, W2, e0, vr, j0, j1, pre, period, s);
    }
#pragma unroll
    for (int k = 0; k < 3; ++k)
#pragma unroll
        for (int o = 1; o < kLinkSplit; o <<= 1) s[k] += __shfl_xor(s[k], o, kLinkSplit);
    if (act && part < 3) {
        const double add = part == 0 ? s[0] : part == 1 ? s[1] : s[2];
        double *xb = part == 0 ? a.xbar[0] : part == 1 ? a.xbar[1] : a.xbar[2];
        xb[v0 + v] += add;
    }
}

// Workgroups per chunk of the ring kernel, each taking every so many batches and
// staging the chunk's coordinates for itself: as many as bring the launch to 1024
// workgroups, at most 8 (a chunk has about 7 batches).  One, two, four and eight
// per chunk: 16 chunks (8,000 nodes) 31, 22, 18 and 17 us with the volumes, 178
// chunks 37, 30, 28 and 28, 512 chunks 49, 47, 48 and 49, 1000 chunks 82, 79, 86
// and 98, 1954 chunks 153, 157, 170 and 196.
int ring_groups(int nchunk)
{
    return std::min(8, (1024 + nchunk - 1) / nchunk);
}

}  // namespace

int launch_geometry(bool adjoint, bool gather, int T, const TetArrays &a, double period,
                    hipStream_t st)
{
    if (T <= 0) return 0;
    if (gather) {
        const dim3 gt((T + 255) / 256), ge((a.E + 255) / 256), gn((a.N + 255) / 256);
        if (adjoint && a.lk_ent) {
            if (a.lk_lds > 65536) {
                const hipError_t e = hipFuncSetAttribute(
                    reinterpret_cast<const void *>(k_link_reverse),
                    hipFuncAttributeMaxDynamicSharedMemorySize, a.lk_lds);
                if (e != hipSuccess) return (int)e;
            }
            hipLaunchKernelGGL(k_link_reverse, dim3(a.lk_chunks), dim3(kLinkThreads), a.lk_lds, st, a,
                               period);
        } else if (adjoint) {
            hipLaunchKernelGGL(k_interleave_w, ge, dim3(256), 0, st, a);
            hipLaunchKernelGGL(k_tet_reverse, gt, dim3(256), 0, st, T, a, period);
            hipLaunchKernelGGL(k_node_sum_xbar, gn, dim3(256), 0, st, a);
        } else if (a.ring) {
            const size_t lds = geo_ring_lds(a.L, a.RB);
            if (lds > 65536) {
                const hipError_t e = hipFuncSetAttribute(
                    reinterpret_cast<const void *>(k_geo_rings),
                    hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
                if (e != hipSuccess) return (int)e;
            }
            hipLaunchKernelGGL(k_geo_rings, dim3(a.nchunk, ring_groups(a.nchunk)), dim3(kGeoThreads), lds, st, a, period);
            hipLaunchKernelGGL(k_geo_vol, dim3(a.nchunk), dim3(kGeoVolThreads),
                               (size_t)a.DV * sizeof(double), st, a);
        } else {
            hipLaunchKernelGGL(k_tet_forward, gt, dim3(256), 0, st, T, a, period);
            hipLaunchKernelGGL(k_edge_sum_faces, ge, dim3(256), 0, st, a);
            hipLaunchKernelGGL(k_node_sum_vol, gn, dim3(256), 0, st, T, a);
        }
        return (int)hipGetLastError();
    }
    const int grid = (T + 255) / 256;
    if (adjoint)
        hipLaunchKernelGGL(k_geometry_adj, dim3(grid), dim3(256), 0, st, T, a, period);
    else
        hipLaunchKernelGGL(k_geometry, dim3(grid), dim3(256), 0, st, T, a, period);
    return (int)hipGetLastError();
}

}  // namespace gpu
}  // namespace opf
