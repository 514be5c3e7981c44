// The Q1 hexahedral operator of the finite-element case study (Section IV),
// on the structured n^3 grid, computed from the element coefficients on the
// device: a matrix-free product and a device assembly of the same operator
// in CSR.
//
// -div(sigma grad u) + c u with trilinear hexahedra of side h = 1/(n-1), one
// coefficient sigma_e per element.  Between two nodes that differ in d
// coordinates (d = 0..3) an element contributes sigma_e h Khat(d) +
// c h^3 Mhat(d), with Khat = (1/3, 0, -1/12, -1/12) and Mhat(d) =
// (1/3)^(3-d) (1/6)^d (tensor products of the 1-D linear element).  Entry
// a_ij sums these over the elements containing both nodes; node i's 27
// neighbours are the offsets {-1, 0, 1}^3 inside the grid.
//
// Node id = x + n y + n^2 z (x fastest), element id the same with n - 1;
// sigma is an (n-1)^3 FP64 array in element order.  The assembly and the product
// on small grids take one thread per node (a workgroup covers 64 consecutive
// nodes of an x-line), the 8 surrounding coefficients read once per node and the
// row's 27 entries formed from their sub-box sums (q1_row); the product on
// others marches along z (k_q1_march).  Either way the row's 27 products are
// added in ascending column order (separate multiply and add), the same
// order as the assembled row, so q1_apply equals the sequential product of
// the matrix q1_assemble writes, bit for bit.
#include <algorithm>
#include <cmath>
#include <cstdint>

#include "context.hpp"

namespace jpcg {

struct Q1Coef {
    double hk[4];   // h Khat(d)
    double chm[4];  // c h^3 Mhat(d)
};

static Q1Coef q1_coef(int n, double c)
{
    const double h = 1.0 / (double)(n - 1);
    const double khat[4] = {1.0 / 3.0, 0.0, -1.0 / 12.0, -1.0 / 12.0};
    const double mhat[4] = {1.0 / 27.0, 1.0 / 54.0, 1.0 / 108.0, 1.0 / 216.0};
    Q1Coef q;
    for (int d = 0; d < 4; ++d) {
        q.hk[d] = h * khat[d];
        q.chm[d] = c * (h * h * h) * mhat[d];
    }
    return q;
}

// Row i's CSR start: rows are z-major, and a node at coordinate t has
// cnt(t) = 3 - [t == 0] - [t == n - 1] neighbours along that axis, so the
// entries before it are C(z) S^2 + cnt(z) (C(y) S + cnt(y) C(x)) with
// S = 3n - 2 and C(t) = sum_{u<t} cnt(u).
__device__ __forceinline__ int q1_cnt(int t, int n) { return 3 - (t == 0) - (t == n - 1); }
__device__ __forceinline__ long long q1_cum(int t, int n) { return t == 0 ? 0 : (t == n ? 3LL * n - 2 : 3LL * t - 1); }

// The 27 entries of node i's row, offset o = 9 (dz + 1) + 3 (dy + 1) + (dx + 1)
// (ascending column order).  Along each axis the neighbour at -1 shares the
// element below the node (slot 0), +1 the one above (slot 1), 0 both; the
// shared elements' coefficient sum and count are sums over a sub-box of the
// 2 x 2 x 2 elements, formed axis by axis once per node, and
// a = h Khat(d) sum(sigma) + c h^3 Mhat(d) count.
__device__ __forceinline__ void q1_row(const double (&sg)[2][2][2], const double (&in)[2][2][2], const Q1Coef& q,
                                       double (&a)[27])
{
#pragma clang fp contract(off)
    double sx[2][2][3], cx[2][2][3];
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int v = 0; v < 2; ++v) {
            sx[u][v][0] = sg[u][v][0];
            sx[u][v][1] = sg[u][v][1];
            sx[u][v][2] = sg[u][v][0] + sg[u][v][1];
            cx[u][v][0] = in[u][v][0];
            cx[u][v][1] = in[u][v][1];
            cx[u][v][2] = in[u][v][0] + in[u][v][1];
        }
    double sy[2][3][3], cy[2][3][3];
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int kx = 0; kx < 3; ++kx) {
            sy[u][0][kx] = sx[u][0][kx];
            sy[u][1][kx] = sx[u][1][kx];
            sy[u][2][kx] = sx[u][0][kx] + sx[u][1][kx];
            cy[u][0][kx] = cx[u][0][kx];
            cy[u][1][kx] = cx[u][1][kx];
            cy[u][2][kx] = cx[u][0][kx] + cx[u][1][kx];
        }
    // Slot choice per offset: -1 -> 0, +1 -> 1, 0 -> 2 (both).
    constexpr int kSlot[3] = {0, 2, 1};
#pragma unroll
    for (int o = 0; o < 27; ++o) {
        const int ix = o % 3, iy = (o / 3) % 3, iz = o / 9;
        const int kx = kSlot[ix], ky = kSlot[iy], kz = kSlot[iz];
        const double ss = kz == 2 ? sy[0][ky][kx] + sy[1][ky][kx] : sy[kz][ky][kx];
        const double cc = kz == 2 ? cy[0][ky][kx] + cy[1][ky][kx] : cy[kz][ky][kx];
        const int d = (ix != 1) + (iy != 1) + (iz != 1);
        a[o] = fma(q.hk[d], ss, q.chm[d] * cc);
    }
}

// Coefficients of the 8 elements around node (x, y, z): sg = sigma (0 outside
// the grid), in = 1 inside, 0 outside.
__device__ __forceinline__ void q1_elements(const double* __restrict__ sigma, int n, int x, int y, int z,
                                            double (&sg)[2][2][2], double (&in)[2][2][2])
{
    const int m = n - 1;
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const int ez = z - 1 + a, ey = y - 1 + b, ex = x - 1 + e;
                const bool ok = ez >= 0 && ez < m && ey >= 0 && ey < m && ex >= 0 && ex < m;
                sg[a][b][e] = ok ? sigma[((size_t)ez * m + ey) * m + ex] : 0.0;
                in[a][b][e] = ok ? 1.0 : 0.0;
            }
}

// Grid (ceil(n / 64), n, n) of 64-thread workgroups: thread x of workgroup
// (bx, y, z) is node (64 bx + x, y, z), so no index is divided.
constexpr int kQ1X = 64;

__global__ __launch_bounds__(kQ1X) void k_q1_apply(int n, Q1Coef q, const double* __restrict__ sigma,
                                                   const double* __restrict__ xv, double* __restrict__ yv)
{
#pragma clang fp contract(off)
    const int x = blockIdx.x * kQ1X + threadIdx.x, y = blockIdx.y, z = blockIdx.z;
    if (x >= n) return;
    const int nn = n * n;
    const int i = x + n * y + nn * z;
    double sg[2][2][2], in[2][2][2];
    q1_elements(sigma, n, x, y, z, sg, in);
    // Neighbour offsets clamped into the grid (a neighbour outside reads the
    // node itself and its term is selected away), so the 27 loads issue
    // together without branches.
    const int ox[3] = {x > 0 ? -1 : 0, 0, x < n - 1 ? 1 : 0};
    const int oy[3] = {y > 0 ? -n : 0, 0, y < n - 1 ? n : 0};
    const int oz[3] = {z > 0 ? -nn : 0, 0, z < n - 1 ? nn : 0};
    const bool vx[3] = {x > 0, true, x < n - 1}, vy[3] = {y > 0, true, y < n - 1}, vz[3] = {z > 0, true, z < n - 1};
    double xs[27];
#pragma unroll
    for (int o = 0; o < 27; ++o) xs[o] = xv[i + ox[o % 3] + oy[(o / 3) % 3] + oz[o / 9]];
    double a[27];
    q1_row(sg, in, q, a);
    double acc = 0.0;
#pragma unroll
    for (int o = 0; o < 27; ++o) {
        const double t = a[o] * xs[o];
        acc = acc + ((vx[o % 3] && vy[(o / 3) % 3] && vz[o / 9]) ? t : 0.0);
    }
    yv[i] = acc;
}

// The same product marching along z.  A wave's lanes hold two neighbouring nodes
// each of one or more x-lines (2 L nodes of a line in L lanes) and walk the
// planes of their share of the grid: a plane's three lines per node are read
// once and added to the rows of the plane below, of their own plane and of the
// plane above, which is the ascending column order; an element layer's sums
// serve the two planes it lies between, and a line's neighbours in x come from
// the lanes beside.  What lies outside the grid is a node of value 0 with
// elements of coefficient 0, whose terms are zeros and change no sum.
//
// What bounds it: the double-precision adds and multiplies (about 110 a node).
// With a node per lane and 35 loads for each, the vector-memory address path
// took 34.4 us at 128^3 (50 MB); 15.7 as it is, 6 loads of 16 bytes a plane for
// two nodes (16.9 with the mass terms formed in each plane and the ends of longer
// lines in every case).
struct Q1March {
    int n, lanes;   // lanes of a line
    int chunks;     // of 2 * lanes nodes per line
    int lines;      // lines per workgroup
    int ygroups;    // of lines
    int planes;     // per workgroup
    int G;
};
constexpr int kQ1BS = 256;

struct alignas(8) Q1Pair {
    double x, y;
};

// Entries `at` and at + 1 of a line of `len`, from the pair read at min(at, len - 2);
// 0 where `ok` is false or the line has ended.
__device__ __forceinline__ void q1_pick(const Q1Pair& d, int at, int len, bool ok, double& a, double& b)
{
    a = ok && at < len ? (at == len - 1 ? d.y : d.x) : 0.0;
    b = ok && at < len - 1 ? d.y : 0.0;
}

// The neighbour lane's value (the wave shifted by one lane), `edge` at the ends of the wave.
__device__ __forceinline__ double q1_from_left(double v, double edge)
{
    const int lo = __builtin_amdgcn_update_dpp(__double2loint(edge), __double2loint(v), 0x138, 0xf, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(__double2hiint(edge), __double2hiint(v), 0x138, 0xf, 0xf, false);
    return __hiloint2double(hi, lo);
}
__device__ __forceinline__ double q1_from_right(double v, double edge)
{
    const int lo = __builtin_amdgcn_update_dpp(__double2loint(edge), __double2loint(v), 0x130, 0xf, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(__double2hiint(edge), __double2hiint(v), 0x130, 0xf, 0xf, false);
    return __hiloint2double(hi, lo);
}

// An element layer around a lane's two nodes: [line below, above, both][element
// left of the first node, between, right of the second, sums at the first and
// the second].
struct Q1Layer {
    double s[3][5];
};

// CHUNKS: a line goes on past the lanes.
template <bool CHUNKS>
__global__ __launch_bounds__(kQ1BS, 3) void k_q1_march(Q1March g, Q1Coef q, const double* __restrict__ sigma,
                                                    const double* __restrict__ xv, double* __restrict__ yv)
{
#pragma clang fp contract(off)
    const int n = g.n, m = n - 1;
    int L = xcd_logical_block((int)blockIdx.x, g.G);
    const int chunk = CHUNKS ? L % g.chunks : 0;
    if (CHUNKS) L /= g.chunks;
    const int yg = L % g.ygroups, z0 = (L / g.ygroups) * g.planes, z1 = min(z0 + g.planes, n);
    const int l = threadIdx.x % g.lanes, y = yg * g.lines + (int)threadIdx.x / g.lanes;
    const int x = 2 * (chunk * g.lanes + l);
    const bool in_y = y < n;
    // Where a line goes on past the lanes, its ends read one entry more.
    const bool first = l == 0, last = l == g.lanes - 1;

    // Loads are sent a plane ahead, from addresses inside the arrays whatever the
    // lane, and looked at when the plane's turn comes.
    const int xa = min(x, n - 2), ea = min(x, m - 2), side = first ? max(x - 1, 0) : min(x + 2, n - 1);
    const bool beside = CHUNKS && (first ? x > 0 : last && x + 2 < n);
    struct Plane {
        Q1Pair v[3];  // lines y - 1, y, y + 1
        double e[3];  // an end lane's neighbour beyond
    };
    auto load_plane = [&](int z, Plane& p) {
        const double* plane = xv + (size_t)min(max(z, 0), n - 1) * n * n;
#pragma unroll
        for (int b = 0; b < 3; ++b) {
            const unsigned line = (unsigned)min(max(y + b - 1, 0), n - 1) * (unsigned)n;
            p.v[b] = *(const Q1Pair*)(plane + line + (unsigned)xa);
            p.e[b] = 0.0;
            if (CHUNKS) p.e[b] = plane[line + (unsigned)side];
        }
    };
    struct Elements {
        Q1Pair v[2];  // lines y - 1, y
        double e[2];
    };
    auto load_elements = [&](int z, Elements& t) {
        const double* plane = sigma + (size_t)min(max(z, 0), m - 1) * m * m;
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const unsigned line = (unsigned)min(max(y + b - 1, 0), m - 1) * (unsigned)m;
            t.v[b] = *(const Q1Pair*)(plane + line + (unsigned)ea);
            t.e[b] = 0.0;
            if (CHUNKS) t.e[b] = plane[line + (unsigned)min(max(x - 1, 0), m - 1)];
        }
    };
    auto layer_of = [&](const Elements& t, int z, Q1Layer& s) {
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const int yy = y + b - 1;
            const bool ok = z >= 0 && z < m && yy >= 0 && yy < m;
            q1_pick(t.v[b], x, m, ok, s.s[b][1], s.s[b][2]);
            const double left = q1_from_left(s.s[b][2], 0.0);
            s.s[b][0] = first ? (ok && beside && x - 1 < m ? t.e[b] : 0.0) : left;
            s.s[b][3] = s.s[b][0] + s.s[b][1];
            s.s[b][4] = s.s[b][1] + s.s[b][2];
        }
#pragma unroll
        for (int k = 0; k < 5; ++k) s.s[2][k] = s.s[0][k] + s.s[1][k];
    };
    // Elements per offset: an axis along which the neighbour differs shares
    // one element, the others as many as there are around the node.
    const double cy = (double)((y > 0) + (y < m));
    const double cx[2] = {(double)((x > 0) + (x < m)), (double)((x + 1 > 0) + (x + 1 < m))};
    // chm * count per plane offset and line offset: for offsets -1 and 1 in x, and
    // for 0 at either node.
    struct Mass {
        double edge[2], centre[2][2];
    };
    auto mass_of = [&](int dz, double cz, Mass& t) {
#pragma unroll
        for (int dy = 0; dy < 2; ++dy) {
            const double cyz = dy == 0 ? cz * cy : cz;
            t.edge[dy] = q.chm[dz + dy + 1] * cyz;
#pragma unroll
            for (int u = 0; u < 2; ++u) t.centre[dy][u] = q.chm[dz + dy] * (cyz * cx[u]);
        }
    };
    Mass beside_plane, own_plane;
    mass_of(1, 1.0, beside_plane);
    // The nine terms of one plane for the lane's nodes: lines iy, offsets ix.
    constexpr int kSlot[3] = {0, 2, 1};
    auto add = [&](const double (&v)[3][4], const Q1Layer& s, int dz, const Mass& t, double (&acc)[2]) {
#pragma unroll
        for (int iy = 0; iy < 3; ++iy) {
            const int dy = iy != 1, by = kSlot[iy];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const double a0 = fma(q.hk[dz + dy + 1], s.s[by][u], t.edge[dy]);
                const double a1 = fma(q.hk[dz + dy], s.s[by][3 + u], t.centre[dy][u]);
                const double a2 = fma(q.hk[dz + dy + 1], s.s[by][1 + u], t.edge[dy]);
                acc[u] = acc[u] + a0 * v[iy][u];
                acc[u] = acc[u] + a1 * v[iy][u + 1];
                acc[u] = acc[u] + a2 * v[iy][u + 2];
            }
        }
    };

    double low[2], mid[2] = {0.0, 0.0}, high[2] = {0.0, 0.0};  // rows of planes p - 1, p, p + 1
    Plane next;
    Elements elems;
    Q1Layer below, above = {};  // element layers p - 1 and p
    load_plane(z0 - 1, next);
    load_elements(z0 - 1, elems);
    for (int p = z0 - 1; p <= z1; ++p) {
        double v[3][4];
#pragma unroll
        for (int b = 0; b < 3; ++b) {
            const int yy = y + b - 1;
            const bool ok = p >= 0 && p < n && yy >= 0 && yy < n;
            q1_pick(next.v[b], x, n, ok, v[b][1], v[b][2]);
            const double left = q1_from_left(v[b][2], 0.0), right = q1_from_right(v[b][1], 0.0);
            const double beyond = ok && beside ? next.e[b] : 0.0;
            v[b][0] = first ? beyond : left;
            v[b][3] = last ? beyond : right;
        }
        below = above;
        layer_of(elems, p, above);
        if (p < z1) {
            load_plane(p + 1, next);
            load_elements(p + 1, elems);
        }
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            low[u] = mid[u];
            mid[u] = high[u];
            high[u] = 0.0;
        }
        if (p > z0) {
            add(v, below, 1, beside_plane, low);
            double* out = yv + ((size_t)(p - 1) * n + y) * n + x;
            if (in_y && x < n) out[0] = low[0];
            if (in_y && x + 1 < n) out[1] = low[1];
        }
        if (p >= z0 && p < z1) {
            Q1Layer both;
#pragma unroll
            for (int b = 0; b < 3; ++b)
#pragma unroll
                for (int k = 0; k < 5; ++k) both.s[b][k] = below.s[b][k] + above.s[b][k];
            mass_of(0, (double)((p > 0) + (p < m)), own_plane);
            add(v, both, 0, own_plane, mid);
        }
        if (p + 1 < z1) add(v, above, 1, beside_plane, high);
    }
}

// From this many nodes per edge on the march is the faster one (64-node lines in
// 32 lanes; a share's planes come one after the other): 16^3 4.1 us against 2.9,
// 48^3 5.2 against 4.6, 51^3 5.3 against 5.7, 64^3 5.6 against 6.9, 80^3 10.8
// against 15.8, 150^3 39 against 70.
constexpr int kQ1MarchMin = 50;

// Planes per workgroup: as many workgroups as give each SIMD its three waves in
// one round, as a share reads two planes beyond its own (128^3: 17.7 us; with
// waves for 1.5, 2, 4 and 6 per SIMD 20.4, 17.2, 18.1 and 19.6; 150^3 39 against 54,
// 43, 43 and 43).
static Q1March q1_march(int n)
{
    constexpr int kWaves = 3 * 4 * 256;
    Q1March g{};
    g.n = n;
    g.lanes = 64;
    if (n <= g.lanes) g.lanes /= 2;
    g.chunks = (n + 2 * g.lanes - 1) / (2 * g.lanes);
    g.lines = kQ1BS / g.lanes;
    g.ygroups = (n + g.lines - 1) / g.lines;
    const long long waves = (long long)g.chunks * g.ygroups * (kQ1BS / kWave);
    g.planes = (int)std::max(1LL, std::min<long long>(n, (waves * n + kWaves - 1) / kWaves));
    g.G = g.chunks * g.ygroups * ((n + g.planes - 1) / g.planes);
    return g;
}

__global__ __launch_bounds__(kQ1X) void k_q1_assemble(int n, Q1Coef q, const double* __restrict__ sigma,
                                                      int* __restrict__ rowptr, int* __restrict__ col,
                                                      double* __restrict__ val)
{
    const int x = blockIdx.x * kQ1X + threadIdx.x, y = blockIdx.y, z = blockIdx.z;
    if (x >= n) return;
    const int nn = n * n;
    const int i = x + n * y + nn * z;
    const long long S = 3LL * n - 2;
    long long k = q1_cum(z, n) * S * S + q1_cnt(z, n) * (q1_cum(y, n) * S + q1_cnt(y, n) * q1_cum(x, n));
    rowptr[i] = (int)k;
    if (i == n * nn - 1) rowptr[i + 1] = (int)(S * S * S);
    double sg[2][2][2], in[2][2][2];
    q1_elements(sigma, n, x, y, z, sg, in);
    double a[27];
    q1_row(sg, in, q, a);
#pragma unroll
    for (int o = 0; o < 27; ++o) {
        const int dx = o % 3 - 1, dy = (o / 3) % 3 - 1, dz = o / 9 - 1;
        const int zz = z + dz, yy = y + dy, xx = x + dx;
        if (zz < 0 || zz >= n || yy < 0 || yy >= n || xx < 0 || xx >= n) continue;
        col[k] = i + dx + n * dy + nn * dz;
        val[k] = a[o];
        ++k;
    }
}

static bool q1_size_ok(int n)
{
    if (n < 2) return false;
    const long long S = 3LL * n - 2;
    return S * S * S < (1LL << 31) && (long long)n * n * n < (1LL << 31);
}

}  // namespace jpcg

using namespace jpcg;

extern "C" {

int q1_apply(int32_t n_edge, double c, const double* sigma, const double* x, double* y, void* stream)
{
    if (!sigma || !x || !y || x == y || !jpcg::q1_size_ok(n_edge) || !(c >= 0.0)) return CG_EINVAL;
    try {
        // The zeros that stand for what lies outside would not cancel an
        // infinite c.
        if (n_edge >= kQ1MarchMin && std::isfinite(c)) {
            const Q1March g = q1_march(n_edge);
            const auto march = g.chunks > 1 ? k_q1_march<true> : k_q1_march<false>;
            march<<<g.G, kQ1BS, 0, (hipStream_t)stream>>>(g, q1_coef(n_edge, c), sigma, x, y);
        } else {
            const dim3 grid((n_edge + kQ1X - 1) / kQ1X, n_edge, n_edge);
            k_q1_apply<<<grid, kQ1X, 0, (hipStream_t)stream>>>(n_edge, q1_coef(n_edge, c), sigma, x, y);
        }
        JPCG_HIP(hipGetLastError());
        return 0;
    } catch (const HipError&) {
        return CG_EHIP;
    }
}

int q1_assemble(int32_t n_edge, double c, const double* sigma, int32_t* rowptr, int32_t* col, double* val,
                void* stream)
{
    if (!sigma || !rowptr || !col || !val || !jpcg::q1_size_ok(n_edge) || !(c >= 0.0)) return CG_EINVAL;
    try {
        const dim3 grid((n_edge + kQ1X - 1) / kQ1X, n_edge, n_edge);
        k_q1_assemble<<<grid, kQ1X, 0, (hipStream_t)stream>>>(n_edge, q1_coef(n_edge, c), sigma, rowptr, col, val);
        JPCG_HIP(hipGetLastError());
        return 0;
    } catch (const HipError&) {
        return CG_EHIP;
    }
}

}  // extern "C"
