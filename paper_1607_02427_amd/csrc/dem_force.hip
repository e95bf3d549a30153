// Pair force, torque, energy and virial of rounded polytopes.
//
// Sec. II, Eq. 1 (3D): U_ij sums the WCA potential over every edge-edge
// pair, every (vertex of i, face of j) pair and every (vertex of j, face of
// i) pair; Eq. 2 (2D): over every (vertex of i, edge of j) and (vertex of j,
// edge of i) pair; each at the nearest points of the two features.  The
// potential is WCA (Eq. 3-4) with sigma_ij = r_i + r_j; the force acts along
// the nearest-point line and the torque on each particle comes from its own
// interaction point.  Nearly parallel edges interact at the midpoints of
// their overlap (Sec. II, paragraph on parallel edges).
//
// Mapping to gfx950:
//  1. k_pairs: each unordered pair of the half list once, in two stages.
//     The separation stage (4 lanes per pair, 16 in small systems, 1 in
//     large ones) loads
//     the pair, drops it beyond R_i + R_j + r_cut, and tests each body's
//     vertices against the other's supporting planes; a pair separated by
//     more than r_cut has no feature pair inside the cutoff.  The rest queue
//     in LDS for the feature stage (8 or 16 lanes per pair):
//     a per-feature prefilter keeps only vertices, edges and faces within
//     reach of the other body and not wholly beyond one of its supporting
//     planes, every remaining feature pair of Eq. 1/2 gets a cheap
//     conservative test (plane distance and bounding circle for
//     vertex-face; bounding spheres, then the distance of the two lines, for
//     edge-edge; bounding spheres for vertex-edge), and the survivors are
//     compacted into a per-pair LDS queue so the exact nearest-point and WCA
//     work runs on dense lanes, those of the wavefront's other pairs
//     included.  The group reduces force, both torques and
//     energy in a fixed order; a pair with a feature pair inside the cutoff
//     writes one record into each particle's row slot (FP32 records in FP32
//     mode; every sum over pairs is FP64) and sets the slot's bit in the
//     particle's written-slot mask.
//  2. k_gather: each particle sums the records of its written slots in slot
//     order (deterministic) into F, tau, U_i and W_i and clears its mask,
//     optionally fused with the closing kick of the integrator.  Where
//     steps are not folded, k_replica_tail then closes the step of each
//     replica (thermostat half steps, budget, rebuilds).
// FP32 mode does the geometry in FP32 from FP64 pair offsets rounded once;
// problems within 1% of the cutoff, segment pairs that are nearly parallel
// (sin^2 < 1e-2) and terms whose force line passes close to a centre are
// redone in FP64, because FP32 cannot resolve them (steep force near the
// cutoff; closest points ill-conditioned, error ~ eps / sin^2; a torque that
// is a small fraction of |lever| |f|).
#include <algorithm>
#include <type_traits>

#include "dem_internal.h"
#include "dem_listbuild.h"

namespace dem {
namespace {

template <typename T>
struct V3 {
    T x, y, z;
};
template <typename T>
__device__ inline V3<T> v3(T a, T b, T c) { return {a, b, c}; }
template <typename T>
__device__ inline V3<T> operator+(V3<T> a, V3<T> b) { return {a.x + b.x, a.y + b.y, a.z + b.z}; }
template <typename T>
__device__ inline V3<T> operator-(V3<T> a, V3<T> b) { return {a.x - b.x, a.y - b.y, a.z - b.z}; }
template <typename T>
__device__ inline V3<T> operator*(T s, V3<T> a) { return {s * a.x, s * a.y, s * a.z}; }
template <typename T>
__device__ inline T dot(V3<T> a, V3<T> b) { return a.x * b.x + a.y * b.y + a.z * b.z; }
template <typename T>
__device__ inline V3<T> cross(V3<T> a, V3<T> b)
{
    return {a.y * b.z - a.z * b.y, a.z * b.x - a.x * b.z, a.x * b.y - a.y * b.x};
}
template <typename T>
__device__ inline V3<T> xyz(const Vec4<T> &a) { return {a.x, a.y, a.z}; }
template <typename T>
__device__ inline T clamp01(T t) { return t < T(0) ? T(0) : (t > T(1) ? T(1) : t); }
template <typename T, typename U>
__device__ inline V3<T> cvt(V3<U> a) { return {(T)a.x, (T)a.y, (T)a.z}; }

template <typename T>
struct M3 {
    T m[9];
};
template <typename T>
__device__ inline V3<T> mul(const M3<T> &R, V3<T> v)
{
    return {R.m[0] * v.x + R.m[1] * v.y + R.m[2] * v.z, R.m[3] * v.x + R.m[4] * v.y + R.m[5] * v.z,
            R.m[6] * v.x + R.m[7] * v.y + R.m[8] * v.z};
}
template <typename T>
__device__ inline V3<T> mulT(const M3<T> &R, V3<T> v)
{
    return {R.m[0] * v.x + R.m[3] * v.y + R.m[6] * v.z, R.m[1] * v.x + R.m[4] * v.y + R.m[7] * v.z,
            R.m[2] * v.x + R.m[5] * v.y + R.m[8] * v.z};
}

// q / d for 0 <= q < 2^16 and 1 <= d <= 64 with a precomputed 1/d: the
// fractional part of (q + 1/2)/d lies in [1/(2d), 1 - 1/(2d)], far from the
// rounding error of one FP32 multiply, so truncation is exact.
__device__ inline int qdiv(int q, float inv_d) { return (int)(((float)q + 0.5f) * inv_d); }

// Signed distance of v beyond a plane (unit normal, offset).
template <typename T>
__device__ inline T plane_gap(const Vec4<T> &pl, V3<T> v)
{
    return dot(xyz(pl), v) - pl.w;
}

// Nearest point of the closed segment a + t u (t in [0,1]) to p.
template <typename T>
__device__ inline V3<T> seg_point(V3<T> p, V3<T> a, V3<T> u, T inv_uu)
{
    return a + clamp01(dot(p - a, u) * inv_uu) * u;
}

// Nearest point of a face of shape S to p, both in S's body frame: the
// projection if it is inside the closed polygon (in-plane half-spaces for
// convex faces, crossing number for concave ones), else the nearest point of
// the face's own boundary edges.  fi is the face's packed loop range, which
// the FP64 redo reads from the FP32 table in LDS.  The loops take kU loop
// entries at a time with no branch between them, so their loads are issued
// together; entries past the last repeat it, which changes neither the test
// nor the strict minimum.
template <typename T>
__device__ inline V3<T> face_point(const ShapeTab<T> &S, int f, int fi, V3<T> p)
{
    constexpr int kU = sizeof(T) == 8 ? 2 : 4;
    const Vec4<T> nf = S.fn[f];
    const V3<T> n = xyz(nf);
    const T sd = dot(n, p) - nf.w;
    const int k0 = face_first(fi), k1 = face_end(fi);
    bool inside;
    if (face_convex(fi)) {
        inside = true;
        for (int k = k0; k < k1; k += kU) {
#pragma unroll
            for (int u = 0; u < kU; ++u) {
                const Vec4<T> l = S.ln[k + u < k1 ? k + u : k1 - 1];
                inside &= dot(xyz(l), p) >= l.w;
            }
        }
    } else {
        const V3<T> e1 = v3<T>(S.fe1[f][0], S.fe1[f][1], S.fe1[f][2]);
        const V3<T> e2 = cross(n, e1);
        const V3<T> o = xyz(S.lv[k0]);
        const T px = dot(p - o, e1), py = dot(p - o, e2);
        inside = false;
        for (int k = k0; k < k1; ++k) {
            const int kn = (k + 1 < k1) ? k + 1 : k0;
            const T ax = S.lxy[k][0], ay = S.lxy[k][1], bx = S.lxy[kn][0], by = S.lxy[kn][1];
            if ((ay > py) != (by > py)) {
                const T xc = ax + (py - ay) * (bx - ax) / (by - ay);
                if (px < xc) inside = !inside;
            }
        }
    }
    if (inside) return p - sd * n;
    T best = T(3.0e38);
    V3<T> q = p;
    for (int k = k0; k < k1; k += kU) {
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const int ku = k + u < k1 ? k + u : k1 - 1;
            const Vec4<T> a4 = S.lv[ku];
            const V3<T> a = xyz(a4);
            const V3<T> c = seg_point(p, a, xyz(S.lv[ku + 1 < k1 ? ku + 1 : k0]) - a, a4.w);
            const V3<T> d = p - c;
            const T d2 = dot(d, d);
            if (d2 < best) {
                best = d2;
                q = c;
            }
        }
    }
    return q;
}

// Minimum image of d = x_j - x_i, |d| <= L (positions in [0, L]): d - L rint(d / L)
// without its division, from which it differs only where |d| is within
// rounding of L/2, far beyond any interaction.
__device__ inline double min_image_near(double d, double L)
{
    const double h = 0.5 * L;
    return d > h ? d - L : (d < -h ? d + L : d);
}

// Hamilton product a b of quaternions (w, x, y, z), and the rotation of v by
// a unit quaternion q = (w, u): v + 2 w (u x v) + 2 u x (u x v).
__device__ inline void qmul(const double a[4], const double b[4], double o[4])
{
    o[0] = a[0] * b[0] - a[1] * b[1] - a[2] * b[2] - a[3] * b[3];
    o[1] = a[0] * b[1] + a[1] * b[0] + a[2] * b[3] - a[3] * b[2];
    o[2] = a[0] * b[2] - a[1] * b[3] + a[2] * b[0] + a[3] * b[1];
    o[3] = a[0] * b[3] + a[1] * b[2] - a[2] * b[1] + a[3] * b[0];
}
__device__ inline V3<double> qrot(const double q[4], V3<double> v)
{
    const V3<double> u = v3<double>(q[1], q[2], q[3]);
    const V3<double> c = cross(u, v);
    return v + (2.0 * q[0]) * c + 2.0 * cross(u, c);
}

// Set bits of m in the lanes below this one (the hardware's masked bit
// count: no lane mask is held in registers).
__device__ inline int popc_below(unsigned long long m)
{
    return (int)__builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
}

constexpr int kWaves = kPairWaves;  // waves per block
constexpr int kQueue = 128;        // survivor queue entries per pair
// Problem k of a solve round adds into partial sum k % kVirt, whatever the
// number of lanes per pair, and the partial sums are combined by one fixed
// tree: the result of a pair is the same bit for bit with 8 or 16 lanes.
constexpr int kVirt = 16;

// Reciprocal: the hardware FP32 estimate (1 ulp), exact division in FP64.
__device__ inline float rcp(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ inline double rcp(double x) { return 1.0 / x; }

__device__ inline unsigned plane_bits(float w) { return __float_as_uint(w); }
__device__ inline unsigned plane_bits(double w) { return (unsigned)__double_as_longlong(w); }
__device__ inline void set_plane_bits(float &w, unsigned m) { w = __uint_as_float(m); }
__device__ inline void set_plane_bits(double &w, unsigned m) { w = __longlong_as_double((long long)m); }

template <typename T>
struct alignas(16) PairLds {
    // j's vertices in i's frame and i's in j's; w: the supporting planes of
    // the other body that the vertex lies more than r_cut beyond (bit p:
    // plane p), as bits (plane_bits)
    Vec4<T> vj[DEM_MAX_VERTS];
    Vec4<T> vi[DEM_MAX_VERTS];
    // features that can reach the other body (conservative prefilter), by index
    unsigned char vi_near[DEM_MAX_VERTS], vj_near[DEM_MAX_VERTS];
    unsigned char ei_near[DEM_MAX_EDGES], ej_near[DEM_MAX_EDGES];
    unsigned char fi_near[DEM_MAX_FACES], fj_near[DEM_MAX_FACES];
    unsigned short queue[kQueue];
    // the pair's list lengths, for the lanes of other groups that cull its
    // problems
    int nA, nB, nfj, nfi, nej;
    float inv_fj, inv_fi, inv_ej;
};

// Feature-cell form of the feature search (one per lane group, beside its
// PairLds): the cell masks of i's edges (edges of j within reach of each,
// 3D), and the prefix of the problem counts over the near entries (i's
// vertices, j's vertices, i's edges), which numbers the pair's problems.
struct alignas(16) PairFc {
    unsigned eib[DEM_MAX_EDGES];
    unsigned short pf[2 * DEM_MAX_VERTS + DEM_MAX_EDGES + 2];
};

// The masks of the shape-local feature cell of shape S (its cells at
// `cells`) that holds point p, given in S's frame; zero outside the grid.
template <typename T, int DIM>
__device__ inline uint2 fc_lookup(const uint2 *__restrict__ cells, const ShapeTab<T> &S, V3<T> p)
{
    const int g = S.fc_g;
    const int ix = (int)floor((p.x - S.fc_lo) * S.fc_ih);
    const int iy = (int)floor((p.y - S.fc_lo) * S.fc_ih);
    const int iz = DIM == 3 ? (int)floor((p.z - S.fc_lo) * S.fc_ih) : 0;
    if (ix < 0 || ix >= g || iy < 0 || iy >= g || iz < 0 || iz >= (DIM == 3 ? g : 1)) return make_uint2(0u, 0u);
    return cells[(iz * g + iy) * g + ix];
}

// Index of the r-th set bit of m (r < popcount(m)).
__device__ inline int nth_bit(unsigned m, int r)
{
    for (int k = 0; k < r; ++k) m &= m - 1u;
    return __builtin_ctz(m);
}

// Closest points of segments p1 + s d1 and p2 + t d2 (s, t in [0,1]) with
// a = |d1|^2, e = |d2|^2 and their reciprocals ia, ie given.
// Non-parallel: the clamped line solution (Ericson, Real-Time Collision
// Detection, 2005, Sec. 5.1.9) with the cross-product form of its
// denominator.  Nearly parallel (|d1 x d2|^2 < par_s2 a e): each point is
// the midpoint of its segment's overlap with the other segment's
// projection, or the facing endpoint.  Returns |d1 x d2|^2.
template <typename T>
__device__ inline T seg_seg(V3<T> p1, V3<T> d1, T a, T ia, V3<T> p2, V3<T> d2, T e, T ie, T par_s2, V3<T> &P,
                            V3<T> &Q)
{
    const V3<T> r = p1 - p2;
    const T b = dot(d1, d2), c = dot(d1, r), f = dot(d2, r);
    const V3<T> cr = cross(d1, d2);
    const T den = dot(cr, cr);
    T s, t;
    if (den < par_s2 * a * e) {
        const T t0 = -c * ia, t1 = (b - c) * ia;
        T lo = fmax(T(0), fmin(t0, t1)), hi = fmin(T(1), fmax(t0, t1));
        s = (lo <= hi) ? T(0.5) * (lo + hi) : (fmax(t0, t1) < T(0) ? T(0) : T(1));
        const T u0 = f * ie, u1 = (f + b) * ie;
        lo = fmax(T(0), fmin(u0, u1));
        hi = fmin(T(1), fmax(u0, u1));
        t = (lo <= hi) ? T(0.5) * (lo + hi) : (fmax(u0, u1) < T(0) ? T(0) : T(1));
    } else {
        s = clamp01((b * f - c * e) * rcp(den));
        t = (b * s + f) * ie;
        if (t < T(0)) {
            t = T(0);
            s = clamp01(-c * ia);
        } else if (t > T(1)) {
            t = T(1);
            s = clamp01((b - c) * ia);
        }
    }
    P = p1 + s * d1;
    Q = p2 + t * d2;
    return den;
}

// The feature-pair problems of one particle pair, restricted to the
// features that passed the prefilter: family A pairs near vertices of i
// with near faces (2D: edges) of j, family B near vertices of j with near
// faces (edges) of i, family C near edges of i with near edges of j (3D).
// Problem q decodes to list positions by an exact small division.
template <typename T, int DIM, bool FC = false>
struct Problem {
    const ShapeTab<T> &Si, &Sj;
    const PairLds<T> &W;
    const M3<T> &Rr;
    V3<T> t;
    int nA, nB;
    int nfj, nfi, nej;            // list lengths used as divisors
    float inv_fj, inv_fi, inv_ej;
    // feature cells: nA, nB the near vertices of i and of j, nfj all near
    // entries (with i's near edges); problem q belongs to the entry e with
    // pf[e] <= q < pf[e + 1] and is the (q - pf[e])-th feature of its mask.
    // In both numberings the cull and the solves take the problem's code
    // fam << 10 | x << 5 | y (fc_code, pack).
    const PairFc *F = nullptr;

    __device__ int fc_code(int q) const
    {
        {
            int lo = 0, hi = nfj;
            while (hi - lo > 1) {
                const int mid = (lo + hi) >> 1;
                if ((int)F->pf[mid] <= q) lo = mid;
                else hi = mid;
            }
            const int r = q - (int)F->pf[lo];
            unsigned m;
            int fam, x;
            if (lo < nA) {
                fam = 0;
                x = W.vi_near[lo];
                m = plane_bits(W.vi[x].w);
            } else if (lo < nA + nB) {
                fam = 1;
                x = W.vj_near[lo - nA];
                m = plane_bits(W.vj[x].w);
            } else {
                fam = 2;
                x = W.ei_near[lo - nA - nB];
                m = F->eib[x];
            }
            return fam << 10 | x << 5 | nth_bit(m, r);
        }
    }

    // the queue holds codes fam << 10 | x << 5 | y (the cull forms them: a
    // solve step then decodes its problem without LDS loads)
    __device__ static void decode(int code, int &fam, int &x, int &y)
    {
        fam = code >> 10;
        x = (code >> 5) & 31;
        y = code & 31;
    }

    // code of problem q of the plane-prefilter numbering: vertex x of i
    // against face (2D: edge) y of j for q < nA, vertex x of j against face
    // y of i for q < nA + nB, edge x of i against edge y of j after that
    __device__ int pack(int q) const
    {
        int fam, x, y;
        if (q < nA) {
            const int ax = qdiv(q, inv_fj);
            fam = 0;
            x = W.vi_near[ax];
            y = (DIM == 3) ? W.fj_near[q - ax * nfj] : W.ej_near[q - ax * nfj];
        } else if (q < nA + nB) {
            const int qq = q - nA, bx = qdiv(qq, inv_fi);
            fam = 1;
            x = W.vj_near[bx];
            y = (DIM == 3) ? W.fi_near[qq - bx * nfi] : W.ei_near[qq - bx * nfi];
        } else {
            const int qq = q - nA - nB, ex = qdiv(qq, inv_ej);
            fam = 2;
            x = W.ei_near[ex];
            y = W.ej_near[qq - ex * nej];
        }
        return fam << 10 | x << 5 | y;
    }

    // conservative cull: false if no point of the two features can be within rc
    __device__ bool candidate(int q, T rc) const
    {
        int fam, x, y;
        decode(q, fam, x, y);
        const ShapeTab<T> &S = fam == 0 ? Sj : Si;  // the face's (2D: edge's) owner
        if (DIM == 3) {
            if (fam < 2) {  // vertex against face, in the face owner's frame
                const V3<T> pt = xyz(fam == 0 ? W.vi[x] : W.vj[x]);
                const Vec4<T> nf = S.fn[y], fc = S.fc[y];
                const T sd = dot(xyz(nf), pt) - nf.w;
                const V3<T> dc = pt - xyz(fc);
                const T lim = fc.w + rc;
                return fabs(sd) < rc && dot(dc, dc) < lim * lim;
            }
            // edge against edge: bounding spheres of the two segments, then,
            // unless they are close to parallel, the distance between their
            // lines (a lower bound of the segments' distance)
            const V3<T> a = xyz(W.vj[Sj.e[y][0]]), d2 = xyz(W.vj[Sj.e[y][1]]) - a;
            const Vec4<T> em = Si.em[x];
            const V3<T> dm = xyz(em) - (a + T(0.5) * d2);
            const T lim = em.w + Sj.em[y].w + rc;
            if (!(dot(dm, dm) < lim * lim)) return false;
            const V3<T> d1 = xyz(Si.ed[x]);
            const V3<T> n = cross(d1, d2);
            const T nn = dot(n, n);
            const T rn = dot(xyz(em) - a, n);
            return !(nn > T(1e-4) * Si.ea[x].w * dot(d2, d2) && rn * rn > T(1.001) * rc * rc * nn);
        } else {  // vertex against edge, in the edge owner's frame
            const Vec4<T> em = S.em[y];
            const V3<T> dm = xyz(fam == 0 ? W.vi[x] : W.vj[x]) - xyz(em);
            const T lim = em.w + rc;
            return dot(dm, dm) < lim * lim;
        }
    }

    // exact nearest points: P on i and rho = P - Q, in i's frame; for edge
    // pairs also sin^2 of their angle (1 otherwise)
    __device__ int solve(int q, T par_s2, V3<T> &P, V3<T> &rho, T &sin2, int &ex, int &ey) const
    {
        int fam, x, y;
        decode(q, fam, x, y);
        ex = x;
        ey = y;
        sin2 = T(1);
        if (fam < 2) {
            // both vertex families in one path, the operands selected, so a
            // wavefront that holds both runs the face search once
            const ShapeTab<T> &S = fam == 0 ? Sj : Si;
            const V3<T> pt = xyz(fam == 0 ? W.vi[x] : W.vj[x]);
            V3<T> c;
            if (DIM == 3) {
                c = face_point(S, y, S.fi[y], pt);
            } else {
                const Vec4<T> ed = S.ed[y];
                c = seg_point(pt, xyz(S.ea[y]), xyz(ed), ed.w);
            }
            if (fam == 0) {
                P = xyz(Si.v[x]);
                rho = mul(Rr, pt - c);  // offset formed in j's frame, then rotated
            } else {
                P = c;
                rho = P - pt;
            }
        } else {
            const V3<T> b0 = xyz(W.vj[Sj.e[y][0]]);
            const V3<T> d2 = xyz(W.vj[Sj.e[y][1]]) - b0;
            const Vec4<T> a = Si.ea[x], d1 = Si.ed[x];
            const T e = Sj.ea[y].w, ie = Sj.ed[y].w;
            V3<T> Q;
            const T den = seg_seg(xyz(a), xyz(d1), a.w, d1.w, b0, d2, e, ie, par_s2, P, Q);
            sin2 = den * d1.w * ie;
            rho = P - Q;
        }
        return fam;
    }
};

template <typename T>
struct Acc {
    V3<T> F, Ti, Tj;
    T U;
};

// WCA (Eq. 3-4) at interaction point P on i with offset rho = P - Q.
template <typename T>
__device__ inline int add_wca(Acc<T> &A, V3<T> P, V3<T> rho, V3<T> t, T sig2, T rc2, T eps)
{
    const T r2 = dot(rho, rho);
    if (!(r2 < rc2)) return 0;
    const T ir2 = rcp(r2);
    const T s2 = sig2 * ir2;
    const T s6 = s2 * s2 * s2;
    const T h = T(2) * s6 - T(1);
    const T u = eps * h * h;  // 4 eps (s12 - s6) + eps without the cancellation of the shift
    const T fr = T(24) * eps * s6 * h * ir2;
    const V3<T> f = fr * rho;
    A.F = A.F + f;
    A.Ti = A.Ti + cross(P, f);
    A.Tj = A.Tj + cross(f, (P - rho) - t);  // lever of Q about j's centre (at t), force -f
    A.U += u;
    return 1;
}

// The wavefront's groups' counts n (scalar: the same in every lane), laid end
// to end: their total, and which group item c falls in and where that
// group's items begin.
template <int N>
struct Spans {
    int n[N];
    __device__ explicit Spans(const int (&count)[N])
    {
#pragma unroll
        for (int h = 0; h < N; ++h) n[h] = __builtin_amdgcn_readfirstlane(count[h]);
    }
    __device__ int total() const
    {
        int t = 0;
#pragma unroll
        for (int h = 0; h < N; ++h) t += n[h];
        return t;
    }
    __device__ void find(int c, int &g, int &begin) const
    {
        int run = 0;
        g = begin = 0;
#pragma unroll
        for (int h = 1; h < N; ++h) {
            run += n[h - 1];
            const bool past = c >= run;
            g = past ? h : g;
            begin = past ? run : begin;
        }
    }
    __device__ int begin_of(int g) const
    {
        int run = 0, o = 0;
#pragma unroll
        for (int h = 1; h < N; ++h) {
            run += n[h - 1];
            o = g >= h ? run : o;
        }
        return o;
    }
};

// Sum over the GL lanes of a group of the lanes' two partial sums (a, b):
// partial sum s of the kVirt canonical ones is a of lane s (s < GL) or b of
// lane s - GL; the tree pairs s with s + 8 first, then halves.
template <int GL, typename T>
__device__ inline T group_sum(T a, T b)
{
    T v = GL == kVirt ? a : a + b;
    for (int off = (GL == kVirt ? kVirt / 2 : GL / 2); off > 0; off >>= 1) v += __shfl_xor(v, off, GL);
    return v;
}

__device__ inline void wave_sync_lds()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Appends this lane's item to its group's list when keep is set; returns
// the group's new length.  All 64 lanes must call it together.
__device__ inline int group_append(bool keep, unsigned char *list, int len, int item, unsigned long long gmask)
{
    const unsigned long long m = __ballot(keep);
    if (keep) list[len + popc_below(m & gmask)] = (unsigned char)item;
    return len + __popcll(m & gmask);
}

// Whether FP32 cannot resolve a feature-pair problem, which is then redone
// in FP64 (refine_pair) from the FP64 positions and orientations.  P is the
// nearest point on i, rho = P - Q, t is j's centre, all in i's frame.
//  * Within 1% of the cutoff: the force is a steep function of the distance
//    (dF/dr = 72 eps / r_cut^2) and an isolated contact there has nothing to
//    hide behind.
//  * Nearly parallel edges (sin^2 < 1e-2): their closest points are
//    ill-conditioned (error ~ eps / sin^2), and the error reaches the lever.
//  * A force line that passes close to either centre (the angle between
//    rho and the lever P, or Q - t, has sin^2 < 1e-2): the term's torque is
//    then a small fraction of |lever| |f|, while the rounding of the pair
//    offset to FP32 turns the force's direction by about 1e-6, an error of
//    1e-6 |lever| |f| that would dominate it.  Bodies touching along the
//    line of their centres (a vertex on its symmetry axis, a face contact
//    centred under the other body) have zero torque this way.
template <typename T, int DIM>
__device__ inline bool fp32_unresolved(int fam, T r2, T rc2, T rc, T sin2, V3<T> P, V3<T> rho, V3<T> t)
{
    if (sizeof(T) != 4) return false;
    if (r2 > T(0.99) * rc2 && r2 < T(1.0001) * rc2) return true;
    if (DIM == 3 && fam == 2 && sin2 < T(1e-2) && r2 < T(1.0001) * rc2 + T(1e-3) * rc) return true;
    if (!(r2 < rc2)) return false;
    const V3<T> ci = cross(P, rho);
    const V3<T> lj = (P - rho) - t;
    const V3<T> cj = cross(lj, rho);
    const T k2 = T(1e-2) * r2;
    return dot(ci, ci) < k2 * dot(P, P) || dot(cj, cj) < k2 * dot(lj, lj);
}

// FP64 redo of one FP32 feature-pair problem and of its WCA terms, added to
// A: family 0 is vertex x of i against face (2D: edge) y of j, family 1
// vertex x of j against face (edge) y of i, family 2 edge x of i against
// edge y of j.  It is used where FP32 cannot resolve the answer: within 1%
// of the cutoff, where the force is a steep function of the distance
// (dF/dr = 72 eps / r_cut^2 there), and for nearly parallel edges, whose
// closest points are ill-conditioned (error ~ eps / sin).  Returns 1 if the
// pair is inside the cutoff.  Face loop ranges are read from the FP32 tables
// Ti, Tj in LDS, coordinates from the FP64 tables Di, Dj.
template <typename T, int DIM>
__device__ int refine_pair(const double *box, double eps, double par_s2, const PartRec64 &ri, const PartRec64 &rj,
                           const ShapeTab<T> &Ti, const ShapeTab<T> &Tj, const ShapeTab<double> &Di,
                           const ShapeTab<double> &Dj, int fam, int x, int y, double sig, Acc<T> &A)
{
    // the pair's transform as quaternions, which keeps few values live:
    // qr = conj(q_i) q_j takes j's body frame to i's, td = conj(q_i) d is
    // j's centre in i's frame
    const double qi[4] = {ri.qw, -ri.qx, -ri.qy, -ri.qz};
    const double qj[4] = {rj.qw, rj.qx, rj.qy, rj.qz};
    double qr[4];
    qmul(qi, qj, qr);
    const double qrc[4] = {qr[0], -qr[1], -qr[2], -qr[3]};
    const V3<double> dd = v3<double>(min_image_near(rj.x - ri.x, box[0]), min_image_near(rj.y - ri.y, box[1]),
                                     DIM == 3 ? min_image_near(rj.z - ri.z, box[2]) : 0.0);
    const V3<double> td = qrot(qi, dd);
    V3<double> P, rho;
    if (fam < 2) {
        // one path for both vertex families: i's vertex in j's frame, or j's
        // in i's
        const bool A0 = fam == 0;
        const ShapeTab<double> &D = A0 ? Dj : Di;
        const ShapeTab<T> &F = A0 ? Tj : Ti;
        const V3<double> vx = xyz(A0 ? Di.v[x] : Dj.v[x]);
        double qs[4];
        for (int k = 0; k < 4; ++k) qs[k] = A0 ? qrc[k] : qr[k];
        const V3<double> rv = qrot(qs, A0 ? vx - td : vx);
        const V3<double> pt = A0 ? rv : td + rv;
        V3<double> c;
        if (DIM == 3) {
            c = face_point(D, y, F.fi[y], pt);
        } else {
            const Vec4<double> ed = D.ed[y];
            c = seg_point(pt, xyz(D.ea[y]), xyz(ed), ed.w);
        }
        if (A0) {
            P = vx;
            rho = qrot(qr, pt - c);
        } else {
            P = c;
            rho = P - pt;
        }
    } else {
        const Vec4<double> a = Di.ea[x], d1 = Di.ed[x], b = Dj.ea[y], db = Dj.ed[y];
        const V3<double> b0 = td + qrot(qr, xyz(b));
        const V3<double> d2 = qrot(qr, xyz(db));
        V3<double> Q;
        seg_seg(xyz(a), xyz(d1), a.w, d1.w, b0, d2, b.w, db.w, par_s2, P, Q);
        rho = P - Q;
    }
    const double rc = kWcaCut * sig;
    Acc<double> B;
    B.F = B.Ti = B.Tj = v3<double>(0, 0, 0);
    B.U = 0.0;
    const int hit = add_wca(B, P, rho, td, sig * sig, rc * rc, eps);
    if (hit) {
        A.F = A.F + cvt<T>(B.F);
        A.Ti = A.Ti + cvt<T>(B.Ti);
        A.Tj = A.Tj + cvt<T>(B.Tj);
        A.U += (T)B.U;
    }
    return hit;
}

// The current replica of a pair-kernel block, staged in LDS beside its
// shape tables: SysParams' block from box to wide, then its lists.
struct alignas(16) RepLds {
    double box[3], eps, par_s2;
    double R[DEM_MAX_SHAPES], rad[DEM_MAX_SHAPES], wide;
    int r, sbase, np, poff, first_tile, ncmp, last, pad;
};
static_assert(offsetof(RepLds, r) == kPairConst * sizeof(double), "copied from SysParams as it is");

// What a workgroup reads of replica r before it can request anything else.
struct RepHead {
    int np, first, poff, sbase, n_shapes;
};
template <bool UNITS>
__device__ inline RepHead rep_head(const SysParams *reps, const ListPtrs &l, int r)
{
    return {l.flags[r * FLAG_COUNT + FLAG_NPAIRS], UNITS ? l.cunit[r] : l.tile_start[r], reps[r].poff, reps[r].sbase,
            reps[r].n_shapes};
}

// A pair entry in LDS: 16 bytes as it is in the pair list, or, with a lane per
// pair in the separation stage (64 to a tile, 72 in a wavefront's queue), 8:
// 24 bits for each particle slot and 8 for each row slot (255: none).
template <int SL>
using QueueEnt = std::conditional_t<SL == 1, unsigned long long, int4>;
__device__ inline void put_ent(int4 &q, int4 e) { q = e; }
__device__ inline int4 get_ent(int4 q) { return q; }
__device__ inline void put_ent(unsigned long long &q, int4 e)
{
    q = (unsigned)(e.x & 0xffffff) | (unsigned)(e.z & 0xff) << 24 |
        (unsigned long long)((unsigned)(e.y & 0xffffff) | (unsigned)(e.w & 0xff) << 24) << 32;
}
__device__ inline int4 get_ent(unsigned long long q)
{
    const unsigned a = (unsigned)q, b = (unsigned)(q >> 32);
    const int z = (int)(a >> 24), w = (int)(b >> 24);
    return make_int4((int)(a & 0xffffffu), (int)(b & 0xffffffu), z == 255 ? -1 : z, w == 255 ? -1 : w);
}
// Stages replica r: its shape tables and parameters, and the pair entries of
// `tile`, the first tile the block takes of it, into each wavefront's entry
// slots (nxt, kPP of them).  Every thread of the block calls it together.
// All of it is requested at once, so a block waits for one round trip
// before its first particle records.  UNITS: the block walks force units of
// the replica's compacted pairs (split form) instead of its pair tiles, and
// reads its entries itself.
template <typename T, bool UNITS, int kPP, typename QE>
__device__ void stage_replica(const SysParams *reps, const ListPtrs &l, const ShapeTab<T> *gtab, ShapeTab<T> *tab,
                              RepLds &rl, int r, const RepHead &hd, int tile, QE *nxt)
{
    __syncthreads();
    int tid = threadIdx.x;  // (formed here, not held across the caller's loop)
    asm volatile("" : "+v"(tid));
    int4 ent = make_int4(0, 0, 0, 0);
    const bool fetch = !UNITS && (tid & 63) < kPP;
    if (fetch) {  // (entries past the last repeat it; a replica with a tile has a pair)
        const int q = ((tile - hd.first) * kWaves + (tid >> 6)) * kPP + (tid & 63);
        ent = l.pairs[hd.poff + (q < hd.np ? q : hd.np - 1)];
    }
    constexpr int kC = kPairConst / 2;
    const bool cst = tid >= 64 * kWaves - kC;
    uint4 c = make_uint4(0, 0, 0, 0);
    if (cst) c = reinterpret_cast<const uint4 *>(reps[r].box)[tid - (64 * kWaves - kC)];
    // 16-byte words (the tables are 16-byte aligned and sized), up to two
    // loads per thread in flight before their stores
    constexpr int kU = 2;
    const int n16 = hd.n_shapes * (int)(sizeof(ShapeTab<T>) / 16);
    const uint4 *src = reinterpret_cast<const uint4 *>(gtab + hd.sbase);
    uint4 *dst = reinterpret_cast<uint4 *>(tab);
    for (int w0 = tid; w0 < n16; w0 += kU * blockDim.x) {
        uint4 v[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const int w = w0 + u * (int)blockDim.x;
            v[u] = w < n16 ? src[w] : make_uint4(0, 0, 0, 0);
        }
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const int w = w0 + u * (int)blockDim.x;
            if (w < n16) dst[w] = v[u];
        }
    }
    if (fetch) put_ent(nxt[tid & 63], ent);
    if (cst) reinterpret_cast<uint4 *>(rl.box)[tid - (64 * kWaves - kC)] = c;
    if (threadIdx.x == 0) {  // (one thread: the LDS addresses stay scalar)
        rl.r = r;
        rl.sbase = hd.sbase;
        rl.np = hd.np;
        rl.poff = hd.poff;
        rl.first_tile = hd.first;
        rl.ncmp = UNITS ? l.ccount[r] : 0;
    }
    __syncthreads();
}

// j's body frame in i's, R_i^T R_j (rows of R are body axes in space).
template <typename T>
__device__ inline M3<T> rel_rotation(const M3<T> &Ri, const M3<T> &Rj)
{
    M3<T> Rr;
    for (int a = 0; a < 3; ++a)
        for (int c = 0; c < 3; ++c)
            Rr.m[3 * a + c] = Ri.m[a] * Rj.m[c] + Ri.m[3 + a] * Rj.m[3 + c] + Ri.m[6 + a] * Rj.m[6 + c];
    return Rr;
}

// The pair that a lane group works on in the feature stage (in LDS; lanes of
// other groups that take its problems read it too).
template <typename T>
struct alignas(16) PairGeo {
    int4 ent;    // i, j, slot of j in row i, slot of i in row j (-1: none)
    int si, sj;
    T rc, sig2;  // cutoff and sigma^2 of the pair
    T Rr[9];     // R_i^T R_j: j's body frame in i's
    T t[3];      // R_i^T d: j's centre in i's frame
    T Ri[9];     // R_i, body to space
    T d[3];      // minimum-image x_j - x_i
};
// The separation stage takes SL lanes per pair, so a wavefront settles
// 64 / SL pairs at a time whatever the feature stage's lane count; a tile
// is kPairWaves * 64 / SL pairs.  The pairs it keeps wait in the
// wavefront's LDS queue until it holds one for each of its groups: one
// separation tile adds at most 64 / SL entries to fewer than one per
// feature-stage group already waiting.
constexpr int queue_slots(int sep, int lanes) { return 64 / sep + 64 / lanes; }
// What waits in the queue: the pair with its transform (PairGeo), so a
// feature round starts without a round trip (0.8 to 1.1 us of a small
// system's launch), with 16 lanes per pair and for planar shapes in FP32;
// otherwise the pair's entry alone, and the round loads the two records
// again and forms the transform anew, which leaves the LDS for the pooled
// solve (8 lanes in 3D) or for a second workgroup per CU (FP64).  The force
// kernel of the split form reads entries.
template <typename T>
__host__ __device__ constexpr bool parked(int dim, int lanes, int sep, int stage)
{
    return sizeof(T) == 4 && stage == kFused && sep != 1 && (lanes == 16 || dim == 2);
}
// Per wavefront: problems of each group's pair, and those its queue holds.
template <int kGroups>
struct alignas(16) WaveCtl {
    int tot[kGroups], cnt[kGroups];
};
// Whether the wavefront's 64 lanes share the solves of all its pairs (their
// results pass through LDS), and how many results LDS holds at a time: half
// a wavefront's with a lane per pair in the separation stage, so that three
// workgroups share a CU (FP32).  Not with 8 lanes in 2D, where pairs have few
// problems, nor in FP64: the 8 lanes of a pair add its results up one after
// the other, twice as many each as with 16 and twice as wide as in FP32, which
// costs more than the sharing saves where pairs have many (8000 cubes packed
// face to face 331 us a step pooled, 177 not; in a fluid of volume fraction 0.4
// 37.8 and 36.0; 8000 icosahedra in a gas 40.3 and 42.1, but those take 16),
// and the results' LDS left one workgroup a CU with the feature cells (those
// cubes 498 and 209).
template <typename T>
__host__ __device__ constexpr bool pooled(int dim, int lanes) { return lanes == 16 || (dim == 3 && sizeof(T) == 4); }
__host__ __device__ constexpr int pool_results(int sep) { return sep == 1 ? 32 : 64; }

// One block of 4 waves takes a contiguous range of tiles (256 / SL pairs of
// one replica each, 16, 64 or 256; wave w takes pairs (64 / SL) w .. (64 /
// SL)(w + 1) - 1 of a tile in the first stage).
// Blocks are dealt round-robin to the 8 XCDs, so block b runs on XCD b % 8:
// XCD x gets the x-th eighth of the tiles, and pairs of neighbouring
// particles share its L2.  The tables of the block's current replica live
// in LDS and are restaged when its range crosses into the next replica.
//
// A pair passes two stages.  The first loads it and tests it against the
// bound R_i + R_j + r_cut and against the supporting planes of both bodies:
// when every vertex of one body lies more than r_cut beyond a supporting
// plane of the other, the two inner bodies are farther apart than r_cut, no
// feature pair of Eq. 1/2 is inside the cutoff, and the pair's record is
// zero (SL lanes per pair, 64 / SL pairs per wavefront).  The other live pairs
// wait in the wave's LDS queue; whenever it holds one for each group of the
// second stage (GL lanes per pair; or the range or the replica ends) that
// stage runs the feature prefilter, the per-problem cull and the exact
// solves on them, so the costly stage runs on full waves.  A pair's result
// does not depend on which group or round takes it.
// Work counter of one lane; the uncounted kernel keeps none (registers).
template <bool ON>
struct Tally {
    unsigned v = 0;
    __device__ void add(unsigned x) { v += x; }
    __device__ unsigned get() const { return v; }
};
template <>
struct Tally<false> {
    __device__ void add(unsigned) {}
    __device__ unsigned get() const { return 0; }
};

// OCC wavefronts per SIMD, one build for each precision and form
// (pair_occ): the kernel is latency-bound, so more resident waves overlap
// more round trips, as many as the registers (168 at 3) and a workgroup's
// LDS allow.  The uncounted variants fit without spilling because the
// feature stage reads the pair's transform from LDS (the queue where pairs
// wait with it, parked(), else the group's own slot) instead of holding it.
template <typename T, int DIM, int GL, bool COUNT, int OCC, int SL, int STAGE, bool FC>
__global__ void __launch_bounds__(64 * kWaves, OCC) k_pairs(BatchParams b, const SysParams *__restrict__ reps, StatePtrs s,
                                                          ListPtrs l, const PartRec<T> *__restrict__ prec,
                                                          const PartRec64 *__restrict__ rec64,
                                                          SlotRec<T> *__restrict__ rec, const ShapeTab<T> *__restrict__ gtab,
                                                          const ShapeTab<double> *__restrict__ gtab64,
                                                          unsigned long long *stats)
{
    static_assert(GL == 8 || GL == 16, "8 or 16 lanes per pair");
    static_assert(OCC >= 2 && OCC <= 4, "2 to 4 wavefronts per SIMD");
    static_assert(SL == 1 || SL == 4 || SL == 16, "1, 4 or 16 lanes per pair in the separation stage");
    static_assert(SL != 1 || (GL == 8 && STAGE == kFused), "a lane per pair: with 8 lanes in the feature stage");
    static_assert(STAGE >= kFused && STAGE <= kForces, "fused, search or forces");
    constexpr bool kSearch = STAGE == kSearchOnly;  // first stage only: compact the pairs it keeps
    constexpr bool kForce = STAGE == kForces;       // second stage only, on the compacted pairs
    constexpr int kSepLanes = SL;
    constexpr int kPairsPerWave = 64 / SL;
    constexpr int kGL = GL;                                    // lanes per particle pair
    constexpr int kGroups = 64 / kGL;                         // pairs per wave in the feature stage
    constexpr int kTile = kWaves * kPairsPerWave;             // pairs per block tile
    constexpr int kQCap = queue_slots(SL, kGL);
    constexpr int kVP = (DEM_MAX_VERTS + kSepLanes - 1) / kSepLanes;  // vertices per lane in the separation test
    constexpr int kSets = kVirt / kGL;                        // partial sums per lane
    extern __shared__ __align__(16) unsigned char smem[];
    const size_t orl = b.tab_slots * sizeof(ShapeTab<T>);
    ShapeTab<T> *tab = reinterpret_cast<ShapeTab<T> *>(smem);
    RepLds &rl = *reinterpret_cast<RepLds *>(smem + orl);
    PairLds<T> *pls = reinterpret_cast<PairLds<T> *>(smem + orl + sizeof(RepLds));
    PairGeo<T> *geo = reinterpret_cast<PairGeo<T> *>(pls + kWaves * kGroups);
    constexpr bool kPark = parked<T>(DIM, GL, SL, STAGE);
    constexpr int kGeo = kPark ? kQCap : kGroups;  // pairs with transforms per wavefront
    constexpr int kEnt = kPark ? 0 : kQCap;        // entries without
    WaveCtl<kGroups> *ctl = reinterpret_cast<WaveCtl<kGroups> *>(geo + kWaves * kGeo);
    QueueEnt<SL> *qall = reinterpret_cast<QueueEnt<SL> *>(ctl + kWaves);
    // results of one pooled solve step, one per lane
    constexpr bool kPool = pooled<T>(DIM, GL);
    constexpr int kRes = pool_results(SL);
    constexpr bool kSeq = GL == 16;  // the prefilter takes both bodies' vertices (faces) in one sequence
    Acc<T> *pres = reinterpret_cast<Acc<T> *>(qall + kWaves * kEnt);
    // the feature-cell form's per-group prefix and edge masks
    PairFc *pfc = reinterpret_cast<PairFc *>(reinterpret_cast<unsigned char *>(pres) +
                                             (kPool ? kWaves * kRes * sizeof(Acc<T>) : 0));

    const int lane = __lane_id();
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // the pair entries of this wavefront's next separation tile
    // (the search kernel has no feature stage: its slots follow the scan's words)
    QueueEnt<SL> *nxt = (kSearch ? reinterpret_cast<QueueEnt<SL> *>(reinterpret_cast<int *>(pls) + 64 * kWaves)
                                 : reinterpret_cast<QueueEnt<SL> *>(reinterpret_cast<unsigned char *>(pfc) +
                                                                    (FC ? kWaves * kGroups * sizeof(PairFc) : 0))) +
                        wid * kPairsPerWave;
    const int grp = lane / kGL, sub = lane % kGL;
    const unsigned long long gmask = ((kGL == 64) ? ~0ull : ((1ull << kGL) - 1)) << (kGL * grp);
    PairLds<T> &W = pls[wid * kGroups + grp];
    QueueEnt<SL> *qb = qall + wid * kEnt;
    WaveCtl<kGroups> &wc = ctl[wid];
    PairGeo<T> *wgeo = geo + wid * kGeo;
    const size_t N = (size_t)b.N;
    // requested with the tile count, not after it: a single system's values,
    // and a batch's first guess
    RepHead hd = rep_head<kForce>(reps, l, 0);
    const int ntiles = l.tile_start[b.nrep];
    const unsigned stamp = (unsigned)l.gflags[G_STAMP];
    const int G = gridDim.x, per = G >> 3;
    // the force kernel's units: kWaves * kGroups compacted pairs of one
    // replica, so each wavefront takes one feature round
    const int *first = kForce ? l.cunit : l.tile_start;
    const int nunits = kForce ? l.cunit[b.nrep] : ntiles;
    // XCD x (block b runs on XCD b % 8) takes the x-th eighth of the units;
    // its q-th block (q = b / 8) a contiguous share of them, or, when the
    // eighth holds fewer units than the XCD has blocks, unit q: the blocks
    // launched first take the work, and no unit waits for the grid's last
    // blocks to be dispatched
    const int xcd = blockIdx.x & 7, q = blockIdx.x >> 3;
    const int us = (int)((long long)nunits * xcd / 8), un = (int)((long long)nunits * (xcd + 1) / 8) - us;
    int t0, t1;
    if (q >= per) {  // (grids are multiples of 8; none is left over)
        t0 = t1 = 0;
    } else if (un >= per) {
        t0 = us + (int)((long long)un * q / per);
        t1 = us + (int)((long long)un * (q + 1) / per);
    } else {
        t0 = us + (q < un ? q : un);
        t1 = us + (q < un ? q + 1 : un);
    }
    const T grow = T(1.00001);
    Tally<COUNT> c_pairs, c_feat, c_in, c_near, c_ee, c_ref, c_sep, c_pv;

    int r = 0, r_end = 0;
    if (t0 < t1) {  // replica of the first tile: the last r with tile_start[r] <= t0
        int lo = 0, hi = b.nrep;
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (first[mid] <= t0) lo = mid;
            else hi = mid;
        }
        r = lo;
        r_end = first[r + 1];
        if (b.nrep > 1) hd = rep_head<kForce>(reps, l, r);
        stage_replica<T, kForce, kPairsPerWave>(reps, l, gtab, tab, rl, r, hd, t0, nxt);
    }
    int head = 0, tail = 0;  // queue positions, the same in every lane of the wave
    int tt = t0;
    for (;;) {
        const bool done = tt >= t1;
        const bool restage = !done && tt >= r_end;
        const int pending = tail - head;
        if (!kSearch && (pending >= kGroups || (pending > 0 && (kForce || done || restage)))) {
            // ---- second stage: group g takes queue entry head + g ----
            const int take = pending < kGroups ? pending : kGroups;
            const bool live = grp < take;
            const int h0 = head;  // the round's first entry
            head += take;
            auto geo_of = [&](int g) -> PairGeo<T> & { return wgeo[kPark ? (h0 + g) % kQCap : g]; };
            PairGeo<T> &G = geo_of(grp);
            const M3<T> &Rr = *reinterpret_cast<const M3<T> *>(G.Rr);
            int4 ent = make_int4(0, 0, 0, 0);
            int si = 0, sj = 0;
            V3<T> t = v3<T>(0, 0, 0);
            T sig2 = T(0), rc = T(0), Bi = T(0), Bj = T(0);
            if constexpr (kPark) {
                if (live) {
                    si = G.si;
                    sj = G.sj;
                    t = v3<T>(G.t[0], G.t[1], G.t[2]);
                    rc = G.rc;
                    sig2 = G.sig2;
                    Bi = (T)rl.R[si] + rc;
                    Bj = (T)rl.R[sj] + rc;
                }
            } else {
                // (groups without a pair repeat the last one's loads and drop it)
                ent = get_ent(qb[(h0 + (live ? grp : take - 1)) % kQCap]);
                const PartRec<T> ri = prec[ent.x];
                const PartRec<T> rj = prec[ent.y];
                M3<T> Ri, Rj;
                for (int k = 0; k < 9; ++k) {
                    Ri.m[k] = ri.R[k];
                    Rj.m[k] = rj.R[k];
                }
                const double dx = min_image_near(rj.x - ri.x, rl.box[0]);
                const double dy = min_image_near(rj.y - ri.y, rl.box[1]);
                const double dz = (DIM == 3) ? min_image_near(rj.z - ri.z, rl.box[2]) : 0.0;
                si = ri.sid;
                sj = rj.sid;
                const M3<T> Rrel = rel_rotation(Ri, Rj);
                t = mulT(Ri, v3<T>((T)dx, (T)dy, (T)dz));
                const double sigd = rl.rad[si] + rl.rad[sj];
                sig2 = (T)(sigd * sigd);
                rc = (T)(kWcaCut * sigd);
                Bi = (T)rl.R[si] + rc;
                Bj = (T)rl.R[sj] + rc;
                if (sub == 0) {
                    // the transform is read from LDS where it is used, which
                    // keeps registers free for the solves and the FP64 redo
                    G.ent = ent;
                    G.si = si;
                    G.sj = sj;
                    G.rc = rc;
                    G.sig2 = sig2;
                    for (int k = 0; k < 9; ++k) {
                        G.Rr[k] = Rrel.m[k];
                        G.Ri[k] = Ri.m[k];
                    }
                    G.t[0] = t.x;
                    G.t[1] = t.y;
                    G.t[2] = t.z;
                    G.d[0] = (T)dx;
                    G.d[1] = (T)dy;
                    G.d[2] = (T)dz;
                }
                wave_sync_lds();
            }
            const ShapeTab<T> &Si = tab[si];
            const ShapeTab<T> &Sj = tab[sj];
            const T par_s2 = (T)rl.par_s2;
            const T eps = (T)rl.eps;
            const T rc2 = rc * rc;
            const T rcm = rc * T(1.0001);  // the cull keeps pairs FP32 may place just outside the cutoff

            // Feature prefilter (conservative): a vertex, edge or face can touch
            // the other body only if it lies within R_other + r_cut of that body's
            // centre, widened by the edge half length or the face's bounding
            // radius, and if it is not wholly more than r_cut beyond one of
            // the other body's supporting planes (for an edge or a face: all
            // its vertices beyond the same plane).  One lane per feature;
            // survivors are listed by index.
            int cvj = 0, cvi = 0, cei = 0, cej = 0, cfi = 0, cfj = 0;
            int fc_total = 0;
            PairFc &Fc = pfc[FC ? wid * kGroups + grp : 0];
            const T thr = rcm + T(1e-5) * (Bi + Bj);
            // What bounds it is the chain of LDS reads and dependent terms of
            // each pass.  With 16 lanes, both bodies' vertices, and both
            // bodies' faces, are taken in one sequence (kSeq), so that a pass
            // has few idle lanes: of two cubes, 16 vertices and 12 faces each
            // fill one pass (216 cubes 12.8 us against 13.5, 1000 tetrahedra
            // 14.5 against 15.1).  Edges, of which bodies have more than 8,
            // and 8 lanes per pair take a pass of each body at once, whose
            // chains overlap (262,144 octahedra 338 us against 354 in one
            // sequence).
            auto vertex = [&](bool has, bool of_j, int vk) {
                if (!has) return false;
                const ShapeTab<T> &A = of_j ? Sj : Si;
                const ShapeTab<T> &B = of_j ? Si : Sj;
                const V3<T> u = xyz(A.v[vk]);
                const V3<T> vj = t + mul(Rr, u), vi = mulT(Rr, u - t);
                const V3<T> v = v3<T>(of_j ? vj.x : vi.x, of_j ? vj.y : vi.y, of_j ? vj.z : vi.z);
                const T lim = of_j ? Bi : Bj;
                const int nsep = B.nsep;
                unsigned mb = 0;
#pragma unroll 4
                for (int p = 0; p < nsep; ++p) mb |= (plane_gap(B.sp[p], v) > thr ? 1u : 0u) << p;
                Vec4<T> v4 = {v.x, v.y, v.z, T(0)};
                set_plane_bits(v4.w, mb);
                (of_j ? W.vj : W.vi)[vk] = v4;
                return mb == 0 && dot(v, v) < grow * lim * lim;
            };
            auto edge = [&](bool has, bool of_i, int e) {
                if (!has) return false;
                const ShapeTab<T> &A = of_i ? Si : Sj;
                const Vec4<T> *vs = of_i ? W.vi : W.vj;
                const Vec4<T> em = A.em[e], a = vs[A.e[e][0]], b = vs[A.e[e][1]];
                const V3<T> di = xyz(em) - t, dj = T(0.5) * (xyz(a) + xyz(b));
                const V3<T> d = v3<T>(of_i ? di.x : dj.x, of_i ? di.y : dj.y, of_i ? di.z : dj.z);
                const T lim = (of_i ? Bj : Bi) + em.w;
                return (plane_bits(a.w) & plane_bits(b.w)) == 0 && dot(d, d) < grow * lim * lim;
            };
            const V3<T> ti = DIM == 3 ? -(T)1 * mulT(Rr, t) : t;  // i's centre in j's frame
            auto face = [&](bool has, bool of_i, int f) {
                if (!has) return false;
                const ShapeTab<T> &A = of_i ? Si : Sj;
                const Vec4<T> *vs = of_i ? W.vi : W.vj;
                const Vec4<T> fc = A.fc[f];
                const V3<T> d = v3<T>(fc.x - (of_i ? t.x : ti.x), fc.y - (of_i ? t.y : ti.y), fc.z - (of_i ? t.z : ti.z));
                const T lim = (of_i ? Bj : Bi) + fc.w;
                const int fi = A.fi[f];
                unsigned all = ~0u;
#pragma unroll 4
                for (int k = face_first(fi); k < face_end(fi); ++k) all &= plane_bits(vs[A.floop[k]].w);
                return all == 0 && dot(d, d) < grow * lim * lim;
            };
            // na features of the first body and nb of the second: near ones
            // listed by index
            auto list = [&](auto one, auto near, int na, int nb, int most, unsigned char *la, unsigned char *lb, int &ca, int &cb) {
                constexpr bool seq = decltype(one)::value;
                for (int x0 = 0; x0 < (seq ? 2 : 1) * most; x0 += kGL) {
                    const int x = x0 + sub;
                    if constexpr (seq) {
                        const bool first = x < na;
                        const int k = first ? x : x - na;
                        const bool hit = near(live && x < na + nb, first, k);
                        ca = group_append(hit && first, la, ca, k, gmask);
                        cb = group_append(hit && !first, lb, cb, k, gmask);
                        if (__ballot(live && x0 + kGL < na + nb) == 0) break;
                    } else {
                        const bool ha = near(live && x < na, true, x), hb = near(live && x < nb, false, x);
                        ca = group_append(ha, la, ca, x, gmask);
                        cb = group_append(hb, lb, cb, x, gmask);
                        if (__ballot(live && (x0 + kGL < na || x0 + kGL < nb)) == 0) break;
                    }
                }
            };
            list(std::integral_constant<bool, kSeq>(), vertex, Sj.nv, Si.nv, DEM_MAX_VERTS, W.vj_near, W.vi_near, cvj, cvi);
            wave_sync_lds();
            list(std::false_type(), edge, Si.ne, Sj.ne, DEM_MAX_EDGES, W.ei_near, W.ej_near, cei, cej);
            if (DIM == 3)
                list(std::integral_constant<bool, kSeq>(), face, Si.nf, Sj.nf, DEM_MAX_FACES, W.fi_near, W.fj_near, cfi, cfj);
            wave_sync_lds();
            if constexpr (FC) {
                // Shape-local feature cells narrow the near sets per feature:
                // a near vertex keeps only the other body's near faces (2D:
                // edges) listed by the cell it lies in, a near edge of i only
                // j's near edges listed by the cell of its midpoint.
                unsigned mfi = 0u, mfj = 0u, mei = 0u, mej = 0u;
                for (int k = sub; k < cfi; k += kGL) mfi |= 1u << W.fi_near[k];
                for (int k = sub; k < cfj; k += kGL) mfj |= 1u << W.fj_near[k];
                for (int k = sub; k < cei; k += kGL) mei |= 1u << W.ei_near[k];
                for (int k = sub; k < cej; k += kGL) mej |= 1u << W.ej_near[k];
                for (int off = 1; off < kGL; off <<= 1) {
                    mfi |= __shfl_xor(mfi, off, kGL);
                    mfj |= __shfl_xor(mfj, off, kGL);
                    mei |= __shfl_xor(mei, off, kGL);
                    mej |= __shfl_xor(mej, off, kGL);
                }
                const unsigned tj = DIM == 3 ? mfj : mej, ti = DIM == 3 ? mfi : mei;
                const uint2 *celli = l.fcells + (size_t)(rl.sbase + si) * kFcCells;
                const uint2 *cellj = l.fcells + (size_t)(rl.sbase + sj) * kFcCells;
                for (int k = sub; k < cvi; k += kGL) {
                    const int x = W.vi_near[k];
                    set_plane_bits(W.vi[x].w, fc_lookup<T, DIM>(cellj, Sj, xyz(W.vi[x])).x & tj);
                }
                for (int k = sub; k < cvj; k += kGL) {
                    const int x = W.vj_near[k];
                    set_plane_bits(W.vj[x].w, fc_lookup<T, DIM>(celli, Si, xyz(W.vj[x])).x & ti);
                }
                if (DIM == 3)
                    for (int k = sub; k < cei; k += kGL) {
                        const int e = W.ei_near[k];
                        const V3<T> m = T(0.5) * (xyz(W.vi[Si.e[e][0]]) + xyz(W.vi[Si.e[e][1]]));
                        Fc.eib[e] = fc_lookup<T, DIM>(cellj, Sj, m).y & mej;
                    }
                wave_sync_lds();
                // problem counts of the near entries (i's vertices, j's
                // vertices, i's edges in 3D) and their prefix, GL at a time
                const int nent = cvi + cvj + (DIM == 3 ? cei : 0);
                if (sub == 0) Fc.pf[0] = 0;
                for (int k0 = 0; k0 < nent; k0 += kGL) {
                    const int k = k0 + sub;
                    int c = 0;
                    if (k < nent)
                        c = __popc(k < cvi ? plane_bits(W.vi[W.vi_near[k]].w)
                                           : (k < cvi + cvj ? plane_bits(W.vj[W.vj_near[k - cvi]].w)
                                                            : Fc.eib[W.ei_near[k - cvi - cvj]]));
                    for (int off = 1; off < kGL; off <<= 1) {
                        const int u = __shfl_up(c, off, kGL);
                        if (sub >= off) c += u;
                    }
                    if (k < nent) Fc.pf[k + 1] = (unsigned short)(fc_total + c);
                    fc_total += __shfl(c, kGL - 1, kGL);
                }
                wave_sync_lds();
            }

            Problem<T, DIM, FC> P{Si, Sj, W, Rr, t, 0, 0, 1, 1, 1, 1.f, 1.f, 1.f};
            int total;
            if (FC) {
                P.nA = cvi;
                P.nB = cvj;
                P.nfj = cvi + cvj + (DIM == 3 ? cei : 0);
                P.F = &Fc;
                total = fc_total;
            } else if (DIM == 3) {
                P.nA = cvi * cfj;
                P.nB = cvj * cfi;
                total = P.nA + P.nB + cei * cej;
                P.nfj = cfj;
                P.nfi = cfi;
            } else {
                P.nA = cvi * cej;
                P.nB = cvj * cei;
                total = P.nA + P.nB;
                P.nfj = cej;
                P.nfi = cei;
            }
            P.nej = cej;
            P.inv_fj = 1.0f / (float)(P.nfj > 0 ? P.nfj : 1);
            P.inv_fi = 1.0f / (float)(P.nfi > 0 ? P.nfi : 1);
            P.inv_ej = 1.0f / (float)(P.nej > 0 ? P.nej : 1);
            if (!live) total = 0;
            if (sub == 0 && live) c_feat.add(total);

            Acc<T> A0, A1;  // partial sums kVirt-canonical: sub and sub + GL
            A0.F = A0.Ti = A0.Tj = A1.F = A1.Ti = A1.Tj = v3<T>(0, 0, 0);
            A0.U = A1.U = T(0);
            // Where some pair has more problems than two steps of its own
            // group would cull (and none so many that its queue could fill
            // up before its last candidate), the problems of all the
            // wavefront's pairs are shared out over its 64 lanes: lane c
            // takes the c-th of the pairs' concatenated problems, so the
            // cull takes as many steps as the problems need and not as the
            // busiest pair's; survivors are appended to their pair's queue
            // in problem order.  With fewer, sharing costs more than the
            // steps it saves (216 cubes, 16 lanes: 0.9 us of 14).
            const bool share = __ballot(total > 2 * kGL) != 0 && __ballot(total > kQueue - kVirt) == 0;
            int count = 0;
            for (int qb = 0;; qb += kGL) {
                bool last = share;
                if (share) {
                    if (sub == 0) {
                        W.nA = P.nA;
                        W.nB = P.nB;
                        W.nfj = P.nfj;
                        W.nfi = P.nfi;
                        W.nej = P.nej;
                        W.inv_fj = P.inv_fj;
                        W.inv_fi = P.inv_fi;
                        W.inv_ej = P.inv_ej;
                        wc.tot[grp] = total;
                        wc.cnt[grp] = 0;
                    }
                    wave_sync_lds();
                    const Spans<kGroups> probs(wc.tot);
                    const int nprob = probs.total();
                    for (int c0 = 0; c0 < nprob; c0 += 64) {
                        const int c = c0 + lane;
                        const bool has = c < nprob;
                        int g, og;
                        probs.find(c, g, og);
                        PairLds<T> &Wg = pls[wid * kGroups + g];
                        const PairGeo<T> &Gg = geo_of(g);
                        const Problem<T, DIM, FC> Pg{tab[Gg.si], tab[Gg.sj], Wg,
                                                     *reinterpret_cast<const M3<T> *>(Gg.Rr), t, Wg.nA, Wg.nB, Wg.nfj,
                                                     Wg.nfi, Wg.nej, Wg.inv_fj, Wg.inv_fi, Wg.inv_ej,
                                                     &pfc[FC ? wid * kGroups + g : 0]};
                        int qc = 0;
                        bool keep = false;
                        if (has) {
                            qc = FC ? Pg.fc_code(c - og) : Pg.pack(c - og);
                            keep = Pg.candidate(qc, Gg.rc * T(1.0001));
                        }
                        // survivors of this pair in earlier steps, in this
                        // step below this lane, and in this step altogether
                        const unsigned long long m = __ballot(keep);
                        const int s0 = og > c0 ? og - c0 : 0;  // the pair's first lane
                        const unsigned long long mg = m & (~0ull << s0);
                        const int before = wc.cnt[g] + popc_below(mg);
                        if (keep) Wg.queue[before] = (unsigned short)qc;
                        // (the pair's last lane of this step leaves its count)
                        if (has && (lane == 63 || c + 1 == og + wc.tot[g])) wc.cnt[g] = before + (keep ? 1 : 0);
                        wave_sync_lds();
                    }
                    count = wc.cnt[grp];
                } else {
                    const int q = qb + sub;
                    const bool has = q < total;
                    last = __ballot(has) == 0;
                    if (!last) {
                        const int qc = has ? (FC ? P.fc_code(q) : P.pack(q)) : 0;
                        const bool keep = has && P.candidate(qc, rcm);
                        const unsigned long long m = __ballot(keep);
                        if (keep) W.queue[count + popc_below(m & gmask)] = (unsigned short)qc;
                        count += __popcll(m & gmask);
                    }
                }
                // rounds end at the same problems for any lane count and any
                // other pairs in the wavefront: a pair's queue is checked
                // after each kVirt of its candidates, and only a pair whose
                // queue is nearly full (or every pair, after its last
                // candidate) solves it at that point
                const bool full = !share && (qb + kGL) % kVirt == 0 && count > kQueue - kVirt;
                if (last || __ballot(full) != 0) {
                    const bool mine = last || full;  // this pair solves its queue now
                    wave_sync_lds();
                    if constexpr (kPool) {
                        // The round's problems of all the wavefront's pairs
                        // are shared out over its 64 lanes, so a pair with
                        // many problems no longer holds up the others; each
                        // result goes through LDS to the lane that owns its
                        // partial sum (problem k: lane k mod 16 of the pair's
                        // group) and is added there in problem order, the
                        // order of the unpooled steps, so every pair shape
                        // gives the same bits.
                        if (sub == 0) wc.cnt[grp] = mine ? count : 0;
                        wave_sync_lds();
                        const Spans<kGroups> left(wc.cnt);
                        const int nleft = left.total();
                        const int o_lo = left.begin_of(grp), o_hi = o_lo + wc.cnt[grp];  // this lane's own pair
                        Acc<T> *res = pres + wid * kRes;
                        for (int c0 = 0; c0 < nleft; c0 += 64) {
                            const int c = c0 + lane;
                            Acc<T> A;
                            A.F = A.Ti = A.Tj = v3<T>(0, 0, 0);
                            A.U = T(0);
                            if (c < nleft) {
                                int g, og;
                                left.find(c, g, og);
                                const PairLds<T> &Wg = pls[wid * kGroups + g];
                                const PairGeo<T> &Gg = geo_of(g);
                                const int gi = Gg.si, gj = Gg.sj;
                                const ShapeTab<T> &Sgi = tab[gi];
                                const ShapeTab<T> &Sgj = tab[gj];
                                const V3<T> tg = v3<T>(Gg.t[0], Gg.t[1], Gg.t[2]);
                                const Problem<T, DIM, FC> Pg{Sgi, Sgj, Wg, *reinterpret_cast<const M3<T> *>(Gg.Rr), tg,
                                                             0, 0, 1, 1, 1, 1.f, 1.f, 1.f};
                                const T gsig2 = Gg.sig2, grc = Gg.rc;
                                const T grc2 = grc * grc;
                                V3<T> Pt, rho;
                                T sin2;
                                int e, gf;
                                const int fam = Pg.solve(Wg.queue[c - og], par_s2, Pt, rho, sin2, e, gf);
                                c_near.add(fam < 2 ? 1 : 0);
                                c_ee.add(fam == 2 ? 1 : 0);
                                const T r2 = dot(rho, rho);
                                const bool redo = fp32_unresolved<T, DIM>(fam, r2, grc2, grc, sin2, Pt, rho, tg);
                                if (redo) {
                                    c_ref.add(1);
                                    c_in.add(refine_pair<T, DIM>(rl.box, rl.eps, rl.par_s2, rec64[Gg.ent.x], rec64[Gg.ent.y],
                                                                Sgi, Sgj, gtab64[rl.sbase + gi], gtab64[rl.sbase + gj], fam,
                                                                e, gf, rl.rad[gi] + rl.rad[gj], A));
                                } else {
                                    c_in.add(add_wca(A, Pt, rho, tg, gsig2, grc2, eps));
                                }
                            }
                            // this lane's partial sums: problems k of its pair
                            // with k mod 16 = sub (8 lanes: and sub + 8) that
                            // fall in this step, kRes of the step at a time
#pragma unroll
                            for (int p0 = 0; p0 < 64; p0 += kRes) {
                                if (kRes == 64 || (lane & ~(kRes - 1)) == p0) res[lane & (kRes - 1)] = A;
                                wave_sync_lds();
                                const int b0 = c0 + p0, hi = o_hi < b0 + kRes ? o_hi : b0 + kRes;
                                int k = (o_lo > b0 ? o_lo : b0) - o_lo;
                                k += (sub - k % kGL + kGL) % kGL;
                                for (; o_lo + k < hi; k += kGL) {
                                    const Acc<T> &B = res[o_lo + k - b0];
                                    Acc<T> &S = (kSets == 1 || k % kVirt < kGL) ? A0 : A1;
                                    S.F = S.F + B.F;
                                    S.Ti = S.Ti + B.Ti;
                                    S.Tj = S.Tj + B.Tj;
                                    S.U += B.U;
                                }
                                wave_sync_lds();
                            }
                        }
                    } else
                    for (int m = 0;; ++m) {
                        const int k = m * kGL + sub;
                        const bool w = mine && k < count;
                        if (__ballot(w) == 0) break;
                        if (w) {
                            Acc<T> A;
                            A.F = A.Ti = A.Tj = v3<T>(0, 0, 0);
                            A.U = T(0);
                            V3<T> Pt, rho;
                            T sin2;
                            int e, g;
                            const int fam = P.solve(W.queue[k], par_s2, Pt, rho, sin2, e, g);
                            c_near.add(fam < 2 ? 1 : 0);
                            c_ee.add(fam == 2 ? 1 : 0);
                            const T r2 = dot(rho, rho);
                            const bool redo = fp32_unresolved<T, DIM>(fam, r2, rc2, rc, sin2, Pt, rho, t);
                            if (redo) {
                                c_ref.add(1);
                                c_in.add(refine_pair<T, DIM>(rl.box, rl.eps, rl.par_s2, rec64[G.ent.x], rec64[G.ent.y], Si, Sj,
                                                            gtab64[rl.sbase + si], gtab64[rl.sbase + sj], fam, e, g, rl.rad[si] + rl.rad[sj], A));
                            } else {
                                c_in.add(add_wca(A, Pt, rho, t, sig2, rc2, eps));
                            }
                            Acc<T> &S = (kSets == 1 || (m & 1) == 0) ? A0 : A1;
                            S.F = S.F + A.F;
                            S.Ti = S.Ti + A.Ti;
                            S.Tj = S.Tj + A.Tj;
                            S.U += A.U;
                        }
                    }
                    if (mine) count = 0;
                    wave_sync_lds();
                }
                if (last) break;
            }
            // group reduction (every lane of the group gets the sums); rotate to
            // the space frame and write both row slots, one record per lane
            const T F0 = group_sum<kGL>(A0.F.x, A1.F.x), F1 = group_sum<kGL>(A0.F.y, A1.F.y),
                    F2 = group_sum<kGL>(A0.F.z, A1.F.z);
            const T I0 = group_sum<kGL>(A0.Ti.x, A1.Ti.x), I1 = group_sum<kGL>(A0.Ti.y, A1.Ti.y),
                    I2 = group_sum<kGL>(A0.Ti.z, A1.Ti.z);
            const T J0 = group_sum<kGL>(A0.Tj.x, A1.Tj.x), J1 = group_sum<kGL>(A0.Tj.y, A1.Tj.y),
                    J2 = group_sum<kGL>(A0.Tj.z, A1.Tj.z);
            const T U = group_sum<kGL>(A0.U, A1.U);
            if (live && sub < 2) {  // lane 0 writes i's slot, lane 1 j's
                const int4 ent = G.ent;
                const int i = ent.x, j = ent.y;
                M3<T> Ri;
                for (int k = 0; k < 9; ++k) Ri.m[k] = G.Ri[k];
                const V3<T> dv = v3<T>(G.d[0], G.d[1], G.d[2]);
                const V3<T> Fs = mul(Ri, v3<T>(F0, F1, F2));
                const bool js = sub == 1;
                const V3<T> Ts = mul(Ri, js ? v3<T>(J0, J1, J2) : v3<T>(I0, I1, I2));
                const T sg = js ? T(-1) : T(1);
                const int slot = js ? ent.w : ent.z;
                if (slot >= 0) {
                    SlotRec<T> w;
                    w.F[0] = sg * Fs.x;
                    w.F[1] = sg * Fs.y;
                    w.F[2] = sg * Fs.z;
                    w.U = U;
                    w.tq[0] = Ts.x;
                    w.tq[1] = Ts.y;
                    w.tq[2] = Ts.z;
                    w.d[0] = sg * dv.x;
                    w.d[1] = sg * dv.y;
                    w.d[2] = sg * dv.z;
                    w.pad1 = T(0);
                    set_stamp(w, stamp);
                    const int pi = js ? j : i;
                    rec[(size_t)slot * N + pi] = w;
                    atomicOr(&l.smask[(size_t)(slot >> 5) * N + pi], 1u << (slot & 31));
                }
            }
            continue;
        }
        if (done) break;
        if (restage) {
            do {
                ++r;
                r_end = first[r + 1];
            } while (tt >= r_end);
            stage_replica<T, kForce, kPairsPerWave>(reps, l, gtab, tab, rl, r, rep_head<kForce>(reps, l, r), tt, nxt);
        }
        if constexpr (kForce) {
            // ---- unit tt: this wave's kGroups compacted pairs, one lane each ----
            // (uniform over the wave: the queue positions stay scalar)
            const int base = __builtin_amdgcn_readfirstlane((tt - rl.first_tile) * (kWaves * kGroups) + wid * kGroups);
            const int left = __builtin_amdgcn_readfirstlane(rl.ncmp) - base;
            const int n = left < 0 ? 0 : (left > kGroups ? kGroups : left);
            head = tail = 0;  // the queue is empty between units
            if (lane < n) put_ent(qb[lane], l.cpairs[rl.poff + base + lane]);
            tail = n;
            wave_sync_lds();
            ++tt;
            continue;
        }
        // ---- first stage on tile tt: SL lanes per pair ----
        // (lane indices formed here, not held across the feature stage: an
        // empty asm keeps the compiler from hoisting them out of the loop)
        int lane1 = lane;
        asm volatile("" : "+v"(lane1));
        const int grp1 = lane1 / kSepLanes, sub1 = lane1 % kSepLanes;
        const int q = (tt - rl.first_tile) * kTile + wid * kPairsPerWave + grp1;
        // The entry was fetched while the tile before this one was worked
        // on (or while the tables were staged), so a tile waits for one
        // round trip, the particle records (position, rotation and shape in
        // one line each), not two; lanes past the replica's last pair work
        // on that pair and drop it.
        const int4 ent = get_ent(nxt[grp1]);
        const int i = ent.x, j = ent.y;
        const PartRec<T> ri = prec[i];
        const PartRec<T> rj = prec[j];
        const bool more = !kForce && tt + 1 < t1 && tt + 1 < r_end;
        int4 ent1 = make_int4(0, 0, 0, 0);
        if (more && lane1 < kPairsPerWave) {
            const int q1 = (tt + 1 - rl.first_tile) * kTile + wid * kPairsPerWave + lane1;
            ent1 = l.pairs[rl.poff + (q1 < rl.np ? q1 : rl.np - 1)];
        }
        M3<T> Ri, Rj;
        for (int k = 0; k < 9; ++k) {
            Ri.m[k] = ri.R[k];
            Rj.m[k] = rj.R[k];
        }
        const double dx = min_image_near(rj.x - ri.x, rl.box[0]);
        const double dy = min_image_near(rj.y - ri.y, rl.box[1]);
        const double dz = (DIM == 3) ? min_image_near(rj.z - ri.z, rl.box[2]) : 0.0;
        const int si = ri.sid, sj = rj.sid;
        const double bound = rl.R[si] + rl.R[sj] + kWcaCut * (rl.rad[si] + rl.rad[sj]);
        bool live = q < rl.np && dx * dx + dy * dy + dz * dz < bound * bound;
        if (live && tab[si].ne == 0 && tab[sj].ne == 0 && tab[si].nf == 0 && tab[sj].nf == 0) {
            // two points (spheres, disks): the central WCA term of their
            // centres, in FP64, written here; no separation test, no
            // feature stage (no contraction: every kernel variant rounds the
            // term alike)
#pragma clang fp contract(off)
            c_pairs.add(sub1 == 0 ? 1 : 0);
            const double sig = rl.rad[si] + rl.rad[sj], rc = kWcaCut * sig;
            const double r2 = dx * dx + dy * dy + dz * dz;
            c_in.add(sub1 == 0 && r2 < rc * rc ? 1 : 0);
            if (sub1 < 2 && r2 < rc * rc) {  // lane 0 writes i's slot, lane 1 j's (a lane per pair: both)
                const double ir2 = 1.0 / r2, s2 = sig * sig * ir2, s6 = s2 * s2 * s2, h = 2.0 * s6 - 1.0;
                const double fr = 24.0 * rl.eps * s6 * h * ir2;  // force on i along x_i - x_j
                for (int side = 0; side < (SL == 1 ? 2 : 1); ++side) {
                    const bool js = SL == 1 ? side == 1 : sub1 == 1;
                    const double sg = js ? 1.0 : -1.0;
                    SlotRec<T> w;
                    w.F[0] = (T)(sg * fr * dx);
                    w.F[1] = (T)(sg * fr * dy);
                    w.F[2] = (T)(sg * fr * dz);
                    w.U = (T)(rl.eps * h * h);
                    w.tq[0] = w.tq[1] = w.tq[2] = T(0);
                    w.d[0] = (T)(-sg * dx);
                    w.d[1] = (T)(-sg * dy);
                    w.d[2] = (T)(-sg * dz);
                    w.pad1 = T(0);
                    set_stamp(w, stamp);
                    const int slot = js ? ent.w : ent.z;
                    const int pi = js ? ent.y : ent.x;
                    if (slot >= 0) {
                        rec[(size_t)slot * N + pi] = w;
                        atomicOr(&l.smask[(size_t)(slot >> 5) * N + pi], 1u << (slot & 31));
                    }
                }
            }
            live = false;
        }
        bool need = false;
        if (__ballot(live) != 0) {
            const ShapeTab<T> &Si = tab[si];
            const ShapeTab<T> &Sj = tab[sj];
            const M3<T> Rr = rel_rotation(Ri, Rj);
            const V3<T> t = mulT(Ri, v3<T>((T)dx, (T)dy, (T)dz));
            const T rc = (T)(kWcaCut * (rl.rad[si] + rl.rad[sj]));
            const T Bi = (T)rl.R[si] + rc, Bj = (T)rl.R[sj] + rc;
            // separation beyond which no feature pair can be inside the
            // cutoff, with room for the rounding of the transformed vertices
            const T thr = rc * T(1.0001) + T(1e-5) * (Bi + Bj);
            bool sep;
            if constexpr (kSepLanes == 1) {
                // A lane takes the whole pair: each supporting plane's normal
                // is carried into the other body's frame and the body's
                // lowest vertex along it found, and only for the planes that
                // can separate at all: the other body's centre must lie thr
                // plus its inner radius beyond (one to three planes of an
                // octahedron's eight).  Four lanes per pair repeat the
                // transform and test every plane: 262,144 octahedra, 430
                // instructions for 16 pairs against about 600 for 64.
                sep = false;
                auto side = [&](const ShapeTab<T> &A, const ShapeTab<T> &B, bool of_i, V3<T> c) {
                    const T lim = thr + B.rin;
                    unsigned cand = 0u;
                    const int ns = live && !sep ? A.nsep : 0;
#pragma unroll 4
                    for (int p = 0; p < ns; ++p) cand |= (plane_gap(A.sp[p], c) > lim ? 1u : 0u) << p;
                    while (__ballot(cand != 0u) != 0ull) {
                        const int p = cand != 0u ? __builtin_ctz(cand) : 0;
                        const Vec4<T> pl = A.sp[p];
                        const V3<T> m = of_i ? mulT(Rr, xyz(pl)) : mul(Rr, xyz(pl));
                        T lo = T(3.0e38);
                        const int nv = cand != 0u ? B.nv : 0;
#pragma unroll 4
                        for (int v = 0; v < nv; ++v) lo = fmin(lo, dot(m, xyz(B.v[v])));
                        c_pv.add(nv);
                        sep |= cand != 0u && plane_gap(pl, c) + lo > thr;
                        cand = sep ? 0u : cand & (cand - 1u);
                    }
                };
                side(Si, Sj, true, t);
                side(Sj, Si, false, T(-1) * mulT(Rr, t));
            } else {
                // bit p of bi (bj): every vertex of j (i) this lane holds lies
                // more than thr beyond supporting plane p of i (j); no early exit
                // and one group reduction at the end, so the plane loads of
                // successive planes overlap, and one loop for both bodies, so
                // theirs do (1000 tetrahedra 14.0 us, one body after the other
                // 14.5).  VP vertices of each body per lane,
                // as few as the replica's shapes need: with VP for
                // DEM_MAX_VERTS throughout, half of the plane tests of bodies
                // with 8 vertices or fewer were made on empty slots.
                unsigned bi = 0, bj = 0;
                auto planes = [&](auto vp) {
                    constexpr int VP = decltype(vp)::value;
                    V3<T> wj[VP], wi[VP];  // this lane's vertices: j's in i's frame, i's in j's frame
                    bool hj[VP], hi[VP];
#pragma unroll
                    for (int p = 0; p < VP; ++p) {
                        const int k = p * kSepLanes + sub1;
                        hj[p] = live && k < Sj.nv;
                        hi[p] = live && k < Si.nv;
                        wj[p] = t + mul(Rr, xyz(Sj.v[k]));
                        wi[p] = mulT(Rr, xyz(Si.v[k]) - t);
                    }
                    const int nsi = live ? Si.nsep : 0, nsj = live ? Sj.nsep : 0;
#pragma unroll 2
                    for (int p = 0; p < (nsi > nsj ? nsi : nsj); ++p) {
                        const bool oi = p < nsi, oj = p < nsj;
                        const Vec4<T> pi = Si.sp[oi ? p : 0], pj = Sj.sp[oj ? p : 0];
                        bool ai = oi, aj = oj;
#pragma unroll
                        for (int v = 0; v < VP; ++v) {
                            ai &= !hj[v] || plane_gap(pi, wj[v]) > thr;
                            aj &= !hi[v] || plane_gap(pj, wi[v]) > thr;
                            c_pv.add((oi && hj[v] ? 1 : 0) + (oj && hi[v] ? 1 : 0));
                        }
                        bi |= (ai ? 1u : 0u) << p;
                        bj |= (aj ? 1u : 0u) << p;
                    }
                };
                if (kSepLanes == 4 && rl.wide == 0.0) planes(std::integral_constant<int, kSepLanes == 4 ? 2 : 1>());
                else planes(std::integral_constant<int, kVP>());
                for (int off = 1; off < kSepLanes; off <<= 1) {
                    bi &= __shfl_xor(bi, off, kSepLanes);
                    bj &= __shfl_xor(bj, off, kSepLanes);
                }
                sep = (bi | bj) != 0;
            }
            need = live && !sep;
            if (sub1 == 0 && live) {
                c_pairs.add(1);
                c_sep.add(sep ? 1 : 0);
            }
            // queue the pairs that need the feature stage, one entry per group
            const unsigned long long m = __ballot(need && sub1 == 0);
            if constexpr (kSearch) {
                // or, in the split form, append them to the replica's compacted pairs
                if (m != 0) {
                    int at = 0;
                    if (lane == 0) at = atomicAdd(&l.ccount[rl.r], (int)__popcll(m));
                    at = __shfl(at, 0);
                    if (need && sub1 == 0) l.cpairs[rl.poff + at + popc_below(m)] = ent;
                }
            } else if (need && sub1 == 0) {
                const int at = (tail + popc_below(m)) % kQCap;
                if constexpr (kPark) {
                    PairGeo<T> &e = wgeo[at];
                    const double sigd = rl.rad[si] + rl.rad[sj];
                    e.ent = ent;
                    e.si = si;
                    e.sj = sj;
                    e.rc = rc;
                    e.sig2 = (T)(sigd * sigd);
                    for (int k = 0; k < 9; ++k) {
                        e.Rr[k] = Rr.m[k];
                        e.Ri[k] = Ri.m[k];
                    }
                    e.t[0] = t.x;
                    e.t[1] = t.y;
                    e.t[2] = t.z;
                    e.d[0] = (T)dx;
                    e.d[1] = (T)dy;
                    e.d[2] = (T)dz;
                } else {
                    put_ent(qb[at], ent);
                }
            }
            tail += __popcll(m);
        }
        if (more && lane1 < kPairsPerWave) put_ent(nxt[lane1], ent1);
        wave_sync_lds();  // the queue entries are visible to every lane
        ++tt;
    }
    if constexpr (kSearch || kForce) {
        // the last workgroup to finish: after the search, the force units
        // of each replica; after the forces, the counts back to zero for
        // the next evaluation (every workgroup has read them by then)
        __syncthreads();
        if (threadIdx.x == 0) {
            __threadfence();
            rl.last = atomicAdd(&l.ctick[kSearch ? 0 : 1], 1) == (int)gridDim.x - 1 ? 1 : 0;
        }
        __syncthreads();
        if (rl.last) {
            if constexpr (kSearch) {
                const int per_unit = kWaves * (64 / b.pair_lanes);
                for (int q = threadIdx.x; q < b.nrep; q += blockDim.x) {
                    const int c = __hip_atomic_load(&l.ccount[q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    l.cunit[q] = (c + per_unit - 1) / per_unit;
                }
                __syncthreads();
                int *part = reinterpret_cast<int *>(pls);  // LDS the search does not use
                const int total = lb::block_scan<64 * kWaves>(l.cunit, l.cunit, b.nrep, part);
                if (threadIdx.x == 0) l.cunit[b.nrep] = total;
            } else {
                for (int q = threadIdx.x; q < b.nrep; q += blockDim.x) l.ccount[q] = 0;
            }
            if (threadIdx.x == 0) l.ctick[kSearch ? 0 : 1] = 0;
        }
    }
    if (COUNT && stats) {
        // The counters go to one of kStatBanks copies by workgroup, one line
        // each, added up when they are read; the workgroup's lanes are
        // summed in LDS first and a zero is not added.  One copy alone
        // serialised 8 atomics per wavefront on one line across the XCDs
        // (5003 FP64 L-prisms: 295 us per counted launch against 68
        // uncounted; 72 with the banks).
        // in the order of Stat, ST_LAUNCHES left out
        const unsigned cnt[8] = {c_pairs.get(), c_feat.get(), c_in.get(), c_near.get(), c_ref.get(), c_ee.get(),
                                 c_sep.get(), c_pv.get()};
        static_assert(ST_LAUNCHES == 3 && ST_PLANETESTS == 8, "counter k is word k, or k + 1 from ST_LAUNCHES on");
        // A wavefront's sums take 32 bits: the 2^31 pairs a handle can hold are
        // spread over 256 CUs of four wavefronts at least, and a pair of
        // bodies of 16 vertices and 20 planes makes 640 plane tests, 1.3e9 a
        // wavefront.  (A workgroup's could pass 2^32; adding 64-bit words per
        // lane instead costs 2 us of 96 on those L-prisms.)
        unsigned *sum = reinterpret_cast<unsigned *>(smem);  // the tables are done with; 8 words per wavefront
        __syncthreads();
        if (threadIdx.x < 8 * kWaves) sum[threadIdx.x] = 0u;
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 8; ++k)
            if (cnt[k] != 0u) atomicAdd(&sum[8 * wid + k], cnt[k]);
        __syncthreads();
        unsigned long long *bank = stats + (size_t)(blockIdx.x % kStatBanks) * kStatStride;
        if (threadIdx.x < 8) {
            unsigned long long v = 0ull;
#pragma unroll
            for (int w = 0; w < kWaves; ++w) v += sum[8 * w + threadIdx.x];
            if (v != 0ull) atomicAdd(&bank[threadIdx.x + (threadIdx.x >= ST_LAUNCHES ? 1 : 0)], v);
            if (blockIdx.x == 0 && threadIdx.x == 0) atomicAdd(&bank[ST_LAUNCHES], 1ull);
        }
    }
}

__device__ inline void body_torque(const double q[4], double tx, double ty, double tz, double out[3])
{
    double R[9];
    quat_to_rot(q[0], q[1], q[2], q[3], R);
    out[0] = R[0] * tx + R[3] * ty + R[6] * tz;
    out[1] = R[1] * tx + R[4] * ty + R[7] * tz;
    out[2] = R[2] * tx + R[5] * ty + R[8] * tz;
}

// Per-particle sums of the row-slot records, optionally fused with the
// closing kick.  One block per chunk, so a block belongs to one replica.
// Each particle's row is split over kGatherLanes lanes (lane l takes slots
// l, l + kGatherLanes, ... in order) and combined by a fixed butterfly, so
// the result does not depend on scheduling.  With the kick and a thermostat
// each block writes its chunk's kinetic partials, for the next kick-drift
// (folded steps) or k_replica_tail.  A replica with no budget left is
// skipped.  The kick's form carries the row workgroups and the step's words,
// and so takes 171 registers in FP32 and 181 in FP64 (3D): two wavefronts per
// SIMD.  Built for three it spills 20 and 68 bytes a lane, which is faster
// only where two leave a second round short, and in FP32 alone (160,000
// spheres 52.4 -> 51.6 us a step; 64,000 28.5 -> 29.0, 160,000 in FP64 58.0 ->
// 59.6; 262,144 octahedra 445 -> 452).
// written row slots a lane loads together in the gather (a record is 48
// bytes in FP32, 96 in FP64; about a quarter of a row's slots are written)
template <typename T>
constexpr int gather_batch() { return 4; }
static_assert(kGatherLanes == 1, "the gather walks a particle's written-slot bits in one lane");

// Adds one row-slot record to a particle's sums: F, tau, U_i = 1/2 sum U_ij
// and W_i = 1/2 sum r_ij (x) F_ij with r_ij = -d.
template <typename T>
__device__ inline void add_slot(double acc[16], const SlotRec<T> &w)
{
    const double f[3] = {(double)w.F[0], (double)w.F[1], (double)w.F[2]};
    for (int a = 0; a < 3; ++a) {
        acc[a] += f[a];
        acc[3 + a] += (double)w.tq[a];
    }
    acc[6] += 0.5 * (double)w.U;
    const double d[3] = {(double)w.d[0], (double)w.d[1], (double)w.d[2]};
    for (int a = 0; a < 3; ++a)
        for (int c = 0; c < 3; ++c) acc[7 + 3 * a + c] -= 0.5 * d[a] * f[c];
}

// Workgroups of a step's gather beyond its chunk workgroups carry the
// neighbour rows of the step's list build (one wavefront per 4 particles;
// each takes every nrole-th group of the replicas that rebuild), from the
// cells the kick-drift filled.  The pair kernel is done with the rows in
// place; the gather workgroups read records, not rows.
constexpr int kRowWorkgroups = 2048;
inline int row_workgroups(const BatchParams &b) { return pad8(std::min(b.nchunk * (kChunk / lb::kNbrPer), kRowWorkgroups)); }

// The replicas that rebuild are found 64 at a time (one lane each); the
// groups of each are dealt over the role workgroups, starting at a
// replica-dependent workgroup so that small replicas spread out too.
template <int DIM>
__device__ void step_rows(const BatchParams &b, const SysParams *reps, const StatePtrs &s, const ListPtrs &l,
                          lb::RowBuf &buf, int first)
{
    const int nrole = (int)gridDim.x - first, me = xcd_block((int)blockIdx.x - first, nrole);
    for (int r0 = 0; r0 < b.nrep; r0 += 64) {
        const int rl = r0 + (int)__lane_id();
        const bool bld = rl < b.nrep && lb::building(LISTS_STEP, rl, reps[rl], l.flags + rl * FLAG_COUNT);
        for (unsigned long long m = __ballot(bld); m != 0ull; m &= m - 1ull) {
            const int r = r0 + __builtin_ctzll(m);
            const SysParams &p = reps[r];
            int32_t *fl = l.flags + r * FLAG_COUNT;
            const int g0 = p.off / lb::kNbrPer, ng = (p.n + lb::kNbrPer - 1) / lb::kNbrPer;
            for (int k = (me + nrole - (int)(((long long)r * 977) % nrole)) % nrole; k < ng; k += nrole)
                lb::nbr_rows<DIM>(b, p, s, l, fl, g0 + k, buf);
        }
    }
}

// A replica's step is done: its budget and count (from left and done), and
// its rebuild flags moved on to the next step.
__device__ inline void step_done(int32_t *fl, int32_t *gflags, int built, int trigger, int nbuilds, int64_t left,
                                 int64_t done, int64_t *budget, int64_t *steps)
{
    *budget = left - 1;
    *steps = done + 1;
    if (built != 0) {  // this step's lists are built: count them
        fl[FLAG_REBUILD] = 0;
        fl[FLAG_NBUILDS] = nbuilds + 1;
        atomicSub(&gflags[G_ANY], 1);
    }
    if (trigger != 0) {  // the next step rebuilds
        fl[FLAG_TRIGGER] = 0;
        fl[FLAG_REBUILD] = 1;
        atomicAdd(&gflags[G_ANY], 1);
    }
}

template <typename T, int DIM, bool KICK>
__global__ void __launch_bounds__(kGatherBlock) k_gather(BatchParams b, const SysParams *reps, StatePtrs s, OutPtrs o,
                                                      ListPtrs l, const SlotRec<T> *__restrict__ rec, double *ke_part,
                                                      double *thermo, int64_t *budget, int64_t *steps)
{
    const int G = KICK ? pad8(b.nchunk) : (int)gridDim.x;  // chunk workgroups
    if (KICK && (int)blockIdx.x >= G) {
        __shared__ lb::RowBuf rbuf;
        if (l.gflags[G_NOW] != 0) step_rows<DIM>(b, reps, s, l, rbuf, G);
        return;
    }
    constexpr int kB = gather_batch<T>();
    const int sub = threadIdx.x % kGatherLanes;
    const int cb = xcd_block(blockIdx.x, G);  // this block's chunk
    const int i = cb * kGatherPer + threadIdx.x / kGatherLanes;
    if (KICK && blockIdx.x == 0 && threadIdx.x == 0) l.gflags[G_FILL] = l.gflags[G_NOW];  // whether pair entries are to be written
    // what depends on the slot alone is requested with the replica's
    // parameters instead of after them (the state only within the length
    // of its arrays).  The records are those of the rows the pair kernel
    // used; a build in this step has already written the next rows, so the
    // written slots are bounded by the row capacity, not the new row length.
    const int nw = slot_words(b.cap);
    uint32_t mw[kRowMax / 32];  // slots written since the last gather, 32 per word
#pragma unroll
    for (int wd = 0; wd < kRowMax / 32; ++wd) mw[wd] = (i < b.N && wd < nw) ? l.smask[(size_t)wd * b.N + i] : 0u;
    double sv[3] = {0.0, 0.0, 0.0}, sL[3] = {0.0, 0.0, 0.0}, sq[4] = {1.0, 0.0, 0.0, 0.0};
    int ssid = 0;
    if (KICK && i < b.nstate) {
        ssid = s.sid[i];
        sv[0] = s.vx[i];
        sv[1] = s.vy[i];
        sL[2] = s.Lz[i];
        if (DIM == 3) {
            sv[2] = s.vz[i];
            sL[0] = s.Lx[i];
            sL[1] = s.Ly[i];
            sq[0] = s.qw[i];
            sq[1] = s.qx[i];
            sq[2] = s.qy[i];
            sq[3] = s.qz[i];
        }
    }
    const unsigned stamp = (unsigned)l.gflags[G_STAMP];  // records of this evaluation only
    const int r = chunk_replica(b, l.chunk_rep, cb);
    if (r < 0) return;
    const SysParams &p = reps[r];
    // the step's words, requested with the replica's parameters; one thread
    // per replica (the lead) moves them on at the end
    const int32_t *cfl = l.flags + r * FLAG_COUNT;
    const double *cth = thermo + r * TH_COUNT;
    const bool active = KICK && cfl[FLAG_ACTIVE] != 0;
    const int built = KICK ? cfl[FLAG_BUILD] : 0, commit = KICK ? cfl[FLAG_CLOSE] : 0, trigger = KICK ? cfl[FLAG_TRIGGER] : 0;
    double st[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    int64_t left = 0, done = 0;
    int nbuilds = 0;
    if (KICK) {
        st[0] = cth[TH_S_XI];
        st[1] = cth[TH_S_ETA];
        st[2] = cth[TH_S_SB];
        st[3] = cth[TH_S_SA];
        st[4] = cth[TH_S_XI_B];
        st[5] = cth[TH_S_ETA_B];
        left = budget[r];
        done = steps[r];
        nbuilds = cfl[FLAG_NBUILDS];
    }
    // This step's build has its pair entries to write; folded, the step's
    // bookkeeping too (nothing written here is used by another workgroup of
    // this kernel).
    auto lead = [&]() {
        if (!KICK || threadIdx.x != 0 || cb != p.off / kChunk) return;
        int32_t *fl = l.flags + r * FLAG_COUNT;
        fl[FLAG_FILL] = built;
        if (!b.fold) return;
        if (commit != 0) {
            double *th = thermo + r * TH_COUNT;
            th[TH_XI] = st[0];
            th[TH_ETA] = st[1];
            th[TH_SB] = st[2];
            th[TH_SA] = st[3];
            th[TH_XI_B] = st[4];
            th[TH_ETA_B] = st[5];
            th[TH_OPEN] = 1.0;
        }
        fl[FLAG_PEND] = active && p.ensemble == DEM_NVT ? 1 : 0;
        if (active) step_done(fl, l.gflags, built, trigger, nbuilds, left, done, &budget[r], &steps[r]);
    };
    if (KICK && !active) {
        lead();
        return;
    }
    const bool npt = KICK && p.ensemble == DEM_NPT;
    const bool nvt = KICK && (p.ensemble == DEM_NVT || npt);
    const size_t N = (size_t)b.N;
    const bool mine = i >= p.off && i < p.off + p.n;
    double acc[16];
    for (int c = 0; c < 16; ++c) acc[c] = 0.0;  // F[3], T[3], U, W[9]
    if (mine) {
        // only the slots written since the last gather, whose words are
        // cleared for the next evaluation; ascending, so they are added in
        // row order.  Loads go in batches: every load of a batch is issued
        // before any of its sums, so the batch's round trips overlap.
        // (Batches that run on over the words were slower: 5.7 -> 6.8 us
        // per launch on 4096 cubes.)
#pragma unroll
        for (int wd = 0; wd < kRowMax / 32; ++wd) {
            uint32_t bits = mw[wd];
            if (bits == 0u) continue;
            l.smask[(size_t)wd * N + i] = 0u;
            while (bits != 0u) {
                SlotRec<T> w[kB];
                bool h[kB];
#pragma unroll
                for (int u = 0; u < kB; ++u) {
                    h[u] = bits != 0u;
                    const int k = 32 * wd + (h[u] ? __builtin_ctz(bits) : 0);
                    w[u] = h[u] ? rec[(size_t)k * N + i] : SlotRec<T>{};
                    bits &= bits - 1u;
                }
                __builtin_amdgcn_sched_barrier(0);  // keep the loads ahead of the sums
#pragma unroll
                for (int u = 0; u < kB; ++u)
                    if (h[u] && slot_stamp(w[u]) == stamp) add_slot(acc, w[u]);
            }
        }
    }
    for (int off = 1; off < kGatherLanes; off <<= 1)
        for (int c = 0; c < 16; ++c) acc[c] += __shfl_xor(acc[c], off, kGatherLanes);
    double kt = 0.0, kr = 0.0, tw = 0.0;
    if (mine && sub == 0) {
        double *F = acc, *Tq = acc + 3;
        if (DIM == 2) {
            F[2] = 0.0;
            Tq[0] = Tq[1] = 0.0;
        }
        o.Fx[i] = F[0];
        o.Fy[i] = F[1];
        o.Fz[i] = F[2];
        o.Tx[i] = Tq[0];
        o.Ty[i] = Tq[1];
        o.Tz[i] = Tq[2];
        o.U[i] = acc[6];
        for (int c = 0; c < 9; ++c) o.W[(size_t)c * b.wstride + i] = acc[7 + c];
        if (KICK) {
            const int sid = ssid;
            const double hm = 0.5 * p.dt / p.mass[sid];
            double v[3] = {sv[0] + hm * F[0], sv[1] + hm * F[1], 0.0};
            if (npt) {  // the kick's exact flow with the barostat's friction
                const double *th = thermo + r * TH_COUNT;
                const double damp = th[TH_DAMP], fk = th[TH_FK] / p.mass[sid];
                for (int a = 0; a < DIM; ++a) v[a] = sv[a] * damp + fk * F[a];
            }
            s.vx[i] = v[0];
            s.vy[i] = v[1];
            double L[3] = {0.0, 0.0, 0.0};
            if (DIM == 3) {
                if (!npt) v[2] = sv[2] + hm * F[2];
                s.vz[i] = v[2];
                double tb[3];
                body_torque(sq, Tq[0], Tq[1], Tq[2], tb);
                L[0] = sL[0] + 0.5 * p.dt * tb[0];
                L[1] = sL[1] + 0.5 * p.dt * tb[1];
                L[2] = sL[2] + 0.5 * p.dt * tb[2];
                s.Lx[i] = L[0];
                s.Ly[i] = L[1];
                s.Lz[i] = L[2];
            } else {
                L[2] = sL[2] + 0.5 * p.dt * Tq[2];
                s.Lz[i] = L[2];
            }
            if (nvt) {
                kt = 0.5 * p.mass[sid] * (v[0] * v[0] + v[1] * v[1] + v[2] * v[2]);
                for (int a = 0; a < 3; ++a)
                    if (p.inertia[sid][a] > 0.0) kr += 0.5 * L[a] * L[a] / p.inertia[sid][a];
            }
            if (npt) tw = acc[7] + acc[11] + (DIM == 3 ? acc[15] : 0.0);
        }
    }
    lead();
    if (!nvt) return;
    static_assert(kGatherBlock == 64, "one wavefront per workgroup");
    kt = wave_sum(kt);
    kr = wave_sum(kr);
    if (npt) tw = wave_sum(tw);
    if (threadIdx.x == 0) {
        put_kinetic(ke_part, b.N, cb, kt, kr, tw);
    }
}

// The end of a step for each replica where the steps are not folded (one
// block per replica slot, after k_gather): the thermostat's closing half
// step and the next step's opening half step from the kinetic energy after
// the closing kick (the gather's partial sums per chunk, added in chunk
// order), the step budget and count, and the list-rebuild transitions.  A
// kernel of its own, so the partial sums are visible without a device-wide
// fence in every gather block.  Workgroups beyond the replica slots carry
// the end of the step's list build (lb::fill_step).
__global__ void __launch_bounds__(kGatherBlock) k_replica_tail(BatchParams b, SysParams *reps, ListPtrs l,
                                                               const double *ke_part, double *thermo, int64_t *budget,
                                                               int64_t *steps)
{
    if ((int)blockIdx.x >= b.nrep) {
        static_assert(kGatherBlock == 64, "one wavefront per workgroup");
        __shared__ int part[kGatherBlock];
        lb::fill_step(b, reps, l, (int)blockIdx.x - b.nrep, (int)gridDim.x - b.nrep, part);
        return;
    }
    const int r = blockIdx.x;
    int32_t *fl = l.flags + r * FLAG_COUNT;
    double *th = thermo + r * TH_COUNT;
    // the slot's step values are requested together with its parameters
    // (the thermostat slots exist for every replica slot)
    const int64_t left = budget[r];
    const int32_t rebuilt = fl[FLAG_REBUILD];
    const double xi0 = th[TH_XI], eta0 = th[TH_ETA];
    SysParams &p = reps[r];
    if (!p.live || p.n == 0 || left <= 0) return;
    if (p.ensemble == DEM_NPT) {
        // closing of this step: barostat half step (K_trans after the
        // closing kick, the virial of this step's forces, this step's box),
        // thermostat half step; opening of the next: thermostat, barostat;
        // then the next step's kick and drift factors and its box
        const int nblk = (p.n + kChunk - 1) / kChunk;
        const int c0 = p.off / kChunk;
        double at = 0.0, ar = 0.0, aw = 0.0;
#pragma unroll 8
        for (int c = threadIdx.x; c < nblk; c += blockDim.x) {
            at += ke_part[kKePer * (c0 + c)];
            ar += ke_part[kKePer * (c0 + c) + 1];
            aw += ke_part[kKePer * (c0 + c) + 2];
        }
        double Kt2 = 2.0 * wave_sum(at);
        const double Kr2 = 2.0 * wave_sum(ar);
        const double trW = wave_sum(aw);
        if (threadIdx.x == 0) {
            double xi = xi0, eta = eta0, veps = th[TH_VEPS];
            baro_half(p, Kt2, trW, veps);
            double K2 = Kt2 + Kr2;
            const double sb = nh_half_npt(p, xi, eta, K2, veps);
            Kt2 *= sb * sb;
            th[TH_XI_B] = xi;
            th[TH_ETA_B] = eta;
            th[TH_VEPS_B] = veps;
            th[TH_SB] = sb;
            const double sa = nh_half_npt(p, xi, eta, K2, veps);
            Kt2 *= sa * sa;
            baro_half(p, Kt2, trW, veps);
            th[TH_XI] = xi;
            th[TH_ETA] = eta;
            th[TH_VEPS] = veps;
            th[TH_SA] = sa;
            th[TH_OPEN] = 1.0;
            npt_factors(p, veps, th);
            if (rebuilt != 0)  // this step's lists were built in this step's box
                for (int a = 0; a < 3; ++a) p.box_build[a] = p.box[a];
            double box[3];
            for (int a = 0; a < 3; ++a) {
                th[TH_BOXN + a] = p.box[a];
                box[a] = p.box[a] * th[TH_GROW];
            }
            set_box(p, box, fl);
        }
    }
    if (p.ensemble == DEM_NVT) {
        const double K = kinetic_total(p, ke_part, b.N);
        if (threadIdx.x == 0) {
            const NhStep s = nh_step(p, xi0, eta0, 0.0, 0.0, K, true);
            th[TH_XI_B] = s.xi_b;
            th[TH_ETA_B] = s.eta_b;
            th[TH_SB] = s.sb;
            th[TH_XI] = s.xi;
            th[TH_ETA] = s.eta;
            th[TH_SA] = s.sa;
            th[TH_OPEN] = 1.0;
        }
    }
    if (threadIdx.x == 0)
        step_done(fl, l.gflags, rebuilt, fl[FLAG_TRIGGER], fl[FLAG_NBUILDS], left, steps[r], &budget[r], &steps[r]);
}

template <typename T>
__global__ void k_rotations(BatchParams b, const SysParams *reps, StatePtrs s, ListPtrs l, PartRec<T> *rot,
                            PartRec64 *rec64)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const int c = i / kChunk;
    if (c >= b.nchunk) return;
    const int r = l.chunk_rep[c];
    if (r < 0 || i >= reps[r].off + reps[r].n) return;
    double R[9];
    quat_to_rot(s.qw[i], s.qx[i], s.qy[i], s.qz[i], R);
    // the pair kernel's minimum image reaches one box: a position that the
    // caller has left outside the box is taken as its image inside
    const double *box = reps[r].box;
    auto inside = [](double x, double L) { return x >= 0.0 && x <= L ? x : x - L * floor(x / L); };
    PartRec<T> rc;
    rc.x = inside(s.x[i], box[0]);
    rc.y = inside(s.y[i], box[1]);
    rc.z = b.dim == 3 ? inside(s.z[i], box[2]) : 0.0;
    for (int k = 0; k < 9; ++k) rc.R[k] = (T)R[k];
    rc.sid = s.sid[i];
    rot[i] = rc;
    if (sizeof(T) == 4) rec64[i] = PartRec64{rc.x, rc.y, rc.z, s.qw[i], s.qx[i], s.qy[i], s.qz[i], 0.0};
}

template <typename T, int DIM, int GL, int OCC, int SL, int STAGE, bool FC>
void pairs_t(const Launch &L, unsigned long long *stats, hipStream_t stream);

// The compiled shapes: 8 or 16 lanes per pair with the 4-lane separation
// stage, 16 lanes with the 16-lane one; in the split form, the search kernel
// (4-lane separation stage, kSearchOcc wavefronts per SIMD) and then the
// force kernel at 8 or 16 lanes.  Each feature stage with the supporting-
// plane prefilter or with the shape-local feature cells (FC).
// One build serves shapes that ask for 2 and for 3 wavefronts per SIMD.  In
// FP32 it is for 3 (168 registers): a build for 2 was no faster on any of
// eight workloads and, where it takes more than 168 registers, slower (8
// lanes, 262,144 octahedra: 698 us against 536).  In FP64 it is for 2: the
// LDS of a workgroup lets a CU hold two, whatever the registers.  So is the
// FC feature stage, which does not fit 168 registers.
template <typename T, bool FC>
constexpr int pair_occ() { return FC || sizeof(T) == 8 ? 2 : 3; }
template <typename T, int DIM, bool FC>
void pairs_form(const Launch &L, unsigned long long *stats, hipStream_t stream)
{
    const bool g8 = L.b.pair_lanes == 8;
    constexpr int O = pair_occ<T, FC>();
    if (L.b.pair_split) {
        pairs_t<T, DIM, 16, kSearchOcc, 4, kSearchOnly, false>(L, stats, stream);
        g8 ? pairs_t<T, DIM, 8, O, 4, kForces, FC>(L, stats, stream) : pairs_t<T, DIM, 16, O, 4, kForces, FC>(L, stats, stream);
    } else if (L.b.pair_sep == 16)
        pairs_t<T, DIM, 16, O, 16, kFused, FC>(L, stats, stream);
    else if (!FC && DIM == 3 && L.b.pair_sep == 1)
        pairs_t<T, 3, 8, O, 1, kFused, false>(L, stats, stream);
    else
        g8 ? pairs_t<T, DIM, 8, O, 4, kFused, FC>(L, stats, stream) : pairs_t<T, DIM, 16, O, 4, kFused, FC>(L, stats, stream);
}

template <typename T, int DIM>
void pairs_shape(const Launch &L, unsigned long long *stats, hipStream_t stream)
{
    if (L.b.feature_cells) pairs_form<T, DIM, true>(L, stats, stream);
    else pairs_form<T, DIM, false>(L, stats, stream);
}

template <typename T, int DIM, int GL, int OCC, int SL, int STAGE, bool FC>
void pairs_t(const Launch &L, unsigned long long *stats, hipStream_t stream)
{
    const size_t sh = pair_kernel_lds(sizeof(T) == 4 ? DEM_FP32 : DEM_FP64, DIM, L.b.tab_slots, GL, SL, STAGE, FC ? 1 : 0);
    const int grid = STAGE == kSearchOnly ? L.b.search_blocks : L.b.pair_blocks;
    const auto rot = reinterpret_cast<const PartRec<T> *>(L.f.rot);
    const auto rec = reinterpret_cast<SlotRec<T> *>(L.f.rec);
    const auto tab = reinterpret_cast<const ShapeTab<T> *>(L.f.tab);
    const auto tab64 = reinterpret_cast<const ShapeTab<double> *>(L.f.tab64);
    if (stats)
        k_pairs<T, DIM, GL, true, OCC, SL, STAGE, FC><<<grid, 64 * kWaves, sh, stream>>>(L.b, L.reps, L.s, L.l, rot,
                                                                                      L.f.rec64, rec, tab, tab64, stats);
    else
        k_pairs<T, DIM, GL, false, OCC, SL, STAGE, FC><<<grid, 64 * kWaves, sh, stream>>>(L.b, L.reps, L.s, L.l, rot,
                                                                                       L.f.rec64, rec, tab, tab64, nullptr);
}

template <typename T, int DIM>
void gather_t(const Launch &L, bool kick, hipStream_t stream)
{
    const SlotRec<T> *rec = reinterpret_cast<const SlotRec<T> *>(L.f.rec);
    if (kick) {
        k_gather<T, DIM, true><<<pad8(L.b.nchunk) + row_workgroups(L.b), kGatherBlock, 0, stream>>>(
            L.b, L.reps, L.s, L.o, L.l, rec, L.ke_part, L.thermo, L.budget, L.steps);
        if (!L.b.fold)
            k_replica_tail<<<L.b.nrep + std::min(L.b.nchunk * lb::kFillParts, kFillWorkgroups), kGatherBlock, 0, stream>>>(
                L.b, const_cast<SysParams *>(L.reps), L.l, L.ke_part, L.thermo, L.budget, L.steps);
    }
    else
        k_gather<T, DIM, false><<<pad8(L.b.nchunk), kGatherBlock, 0, stream>>>(L.b, L.reps, L.s, L.o, L.l, rec, L.ke_part,
                                                                     L.thermo, L.budget, L.steps);
}

}  // namespace

void launch_rotations(const Launch &L, hipStream_t stream)
{
    if (L.b.nchunk == 0) return;
    const int nb = blocks_for(L.b.nchunk * kChunk);
    if (L.precision == DEM_FP32)
        k_rotations<float><<<nb, kBlock, 0, stream>>>(L.b, L.reps, L.s, L.l, reinterpret_cast<PartRec<float> *>(L.f.rot),
                                                      L.f.rec64);
    else
        k_rotations<double><<<nb, kBlock, 0, stream>>>(L.b, L.reps, L.s, L.l, reinterpret_cast<PartRec<double> *>(L.f.rot),
                                                       L.f.rec64);
}

void launch_pairs(const Launch &L, unsigned long long *stats, hipStream_t stream)
{
    if (L.b.nchunk == 0) return;
    if (L.precision == DEM_FP32) {
        if (L.b.dim == 3) pairs_shape<float, 3>(L, stats, stream);
        else pairs_shape<float, 2>(L, stats, stream);
    } else {
        if (L.b.dim == 3) pairs_shape<double, 3>(L, stats, stream);
        else pairs_shape<double, 2>(L, stats, stream);
    }
}

void launch_gather(const Launch &L, bool kick, hipStream_t stream)
{
    if (L.b.nchunk == 0) return;
    if (L.precision == DEM_FP32) {
        if (L.b.dim == 3) gather_t<float, 3>(L, kick, stream);
        else gather_t<float, 2>(L, kick, stream);
    } else {
        if (L.b.dim == 3) gather_t<double, 3>(L, kick, stream);
        else gather_t<double, 2>(L, kick, stream);
    }
}

size_t pair_kernel_lds(int precision, int dim, int tab_slots, int lanes, int sep, int stage, int fc)
{
    const bool f32 = precision == DEM_FP32;
    const int groups = 64 / lanes;
    const size_t w = f32 ? sizeof(ShapeTab<float>) : sizeof(ShapeTab<double>);
    const size_t pl = f32 ? sizeof(PairLds<float>) : sizeof(PairLds<double>);
    const size_t pg = f32 ? sizeof(PairGeo<float>) : sizeof(PairGeo<double>);
    const size_t qe = sep == 1 ? sizeof(QueueEnt<1>) : sizeof(QueueEnt<4>);
    const int slots = queue_slots(sep, lanes);
    const bool park = f32 ? parked<float>(dim, lanes, sep, stage) : parked<double>(dim, lanes, sep, stage);
    const size_t queue = park ? slots * pg : groups * pg + slots * qe;
    const size_t ctl = lanes == 8 ? sizeof(WaveCtl<8>) : sizeof(WaveCtl<4>);
    const size_t acc = !(f32 ? pooled<float>(dim, lanes) : pooled<double>(dim, lanes))
                           ? 0
                           : pool_results(sep) * (f32 ? sizeof(Acc<float>) : sizeof(Acc<double>));
    const size_t en = kWaves * (64 / sep) * qe;  // entry slots
    if (stage == kSearchOnly)  // tables, replica, and the last workgroup's scan
        return en + (size_t)tab_slots * w + sizeof(RepLds) + sizeof(int) * 64 * kWaves;
    return en + (size_t)tab_slots * w + sizeof(RepLds) +
           kWaves * (groups * pl + ctl + queue + acc + (fc ? groups * sizeof(PairFc) : 0));
}

namespace {
template <typename T, int DIM, int STAGE, bool FC>
hipError_t pair_occupancy(int *per_cu, size_t lds, int lanes, int sep)
{
    const int t = 64 * kWaves;
    auto occ = [&](auto kernel) { return hipOccupancyMaxActiveBlocksPerMultiprocessor(per_cu, kernel, t, lds); };
    constexpr int O = pair_occ<T, FC>();
    if constexpr (STAGE == kSearchOnly) {
        return occ(k_pairs<T, DIM, 16, false, kSearchOcc, 4, kSearchOnly, false>);
    } else {
        if constexpr (STAGE == kFused)
        {
            if (sep == 16) return occ(k_pairs<T, DIM, 16, false, O, 16, STAGE, FC>);
            if (sep == 1 && !FC && DIM == 3) return occ(k_pairs<T, 3, 8, false, O, 1, STAGE, false>);
        }
        return lanes == 8 ? occ(k_pairs<T, DIM, 8, false, O, 4, STAGE, FC>) : occ(k_pairs<T, DIM, 16, false, O, 4, STAGE, FC>);
    }
}

template <typename T, int DIM>
hipError_t pair_occupancy_stage(int *per_cu, size_t lds, int lanes, int sep, int stage, int fc)
{
    if (stage == kSearchOnly) return pair_occupancy<T, DIM, kSearchOnly, false>(per_cu, lds, lanes, sep);
    if (stage == kForces)
        return fc ? pair_occupancy<T, DIM, kForces, true>(per_cu, lds, lanes, sep)
                  : pair_occupancy<T, DIM, kForces, false>(per_cu, lds, lanes, sep);
    return fc ? pair_occupancy<T, DIM, kFused, true>(per_cu, lds, lanes, sep)
              : pair_occupancy<T, DIM, kFused, false>(per_cu, lds, lanes, sep);
}
}  // namespace

int pair_blocks_resident(int precision, int dim, int tab_slots, int lanes, int sep, int stage, int fc)
{
    const size_t lds = pair_kernel_lds(precision, dim, tab_slots, lanes, sep, stage, fc);
    int per_cu = 0, cus = 0, dev = 0;
    hipError_t e;
    if (precision == DEM_FP32)
        e = dim == 3 ? pair_occupancy_stage<float, 3>(&per_cu, lds, lanes, sep, stage, fc)
                     : pair_occupancy_stage<float, 2>(&per_cu, lds, lanes, sep, stage, fc);
    else
        e = dim == 3 ? pair_occupancy_stage<double, 3>(&per_cu, lds, lanes, sep, stage, fc)
                     : pair_occupancy_stage<double, 2>(&per_cu, lds, lanes, sep, stage, fc);
    if (e != hipSuccess || hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
        return 512;
    // LDS is handed out in granules of 1280 bytes (measured: three workgroups
    // of 53,589 bytes share a CU, three of 54,101 do not), which the runtime's
    // count leaves out; a grid of more blocks than fit would run in two rounds
    const size_t granule = 1280, held = (size_t)163840 / ((lds + granule - 1) / granule * granule);
    per_cu = std::min(per_cu, (int)held);
    return std::max(8, per_cu * cus);
}

}  // namespace dem
