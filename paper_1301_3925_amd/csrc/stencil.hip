// AD-LBR stencil construction on the GPU: one thread per grid point.
//
// 2D (Section 2): Lagrange's reduction of Z^2 for the metric of D, sign fix
// of Corollary 2, superbase (e, f, -e-f), weights of Lemma 1.
// 3D (Section 2): greedy D-reduced basis (Definition 2), Proposition
// (MakeObtuse), Selling's decomposition.
//
// Every decision (rounding of a projection coefficient, a norm comparison,
// a sign test) is an FP64 operation on products of exact integer
// coefficients with the tensor entries, in a fixed order, and this file is
// compiled with -ffp-contract=off: the integer offsets are therefore a
// deterministic function of the FP64 tensor, reproducible on any IEEE
// machine that evaluates the same expressions.
//
// The 2D metric is Q = adj(D) = det(D) D^{-1}, a positive multiple of the
// paper's M = det(D)^{1/2} D^{-1} (eq. (DM)); reduced and obtuse bases do not
// change under positive scaling, and <e^perp, D f^perp> = <e, Q f> gives the
// Lemma 1 weights from the same products.
#include <type_traits>

#include "common.h"

namespace adlbr {
namespace {

constexpr int kMaxIter = 200;

// Both reductions run first on lattice vectors whose integer components are
// held as doubles: products and sums of components within +-2^24 stay below
// 2^53, so they are exact, and neither integer multiplies (a quarter of the
// rate here) nor conversions remain in the scalar products.  A point whose
// reduction leaves that range is reduced again, from the start, in 64-bit
// integers.  The coefficients are the same numbers either way, hence so is
// every decision taken from them.
constexpr double kExact = 16777216.0;

// a * b + c on components (exact, see above)
__device__ __forceinline__ double mad(double a, double b, double c) { return __builtin_fma(a, b, c); }
__device__ __forceinline__ ll mad(ll a, ll b, ll c) { return a * b + c; }

// The rounded coefficient as a component, and whether it (or a component made
// with it) stays in the exact range; 64-bit integers have no range to leave.
template <typename I> __device__ __forceinline__ I coef(double r) {
    if constexpr (std::is_same_v<I, double>) return r;
    else return (ll)r;
}
__device__ __forceinline__ bool exact(double x) { return fabs(x) <= kExact; }  // not for NaN
__device__ __forceinline__ bool exact(ll) { return true; }

// ------------------------------------------------------------------- 2D --
struct Form2 {
    double xx, xy, yy;
};

template <typename I> struct V2T {
    I x, y;
};
typedef V2T<ll> V2;

template <typename I> __device__ __forceinline__ double form2(const Form2 &q, V2T<I> a, V2T<I> b) {
    const I cxx = a.x * b.x;
    const I cxy = mad(a.x, b.y, a.y * b.x);
    const I cyy = a.y * b.y;
    return ((double)cxx * q.xx + (double)cxy * q.xy) + (double)cyy * q.yy;
}

// Lagrange: repeat (e, f) := (f, e - Round(<e,f>/<f,f>) f) while |e| > |f|
// (a vector's norm is formed once and moves with it).  Iterations used, -1
// past kMaxIter, -2 when the exact range is left.
template <typename I> __device__ int reduce_pair2(const Form2 &q, V2T<I> &e, V2T<I> &f) {
    double nf = form2(q, f, f);
    for (int it = 1; it <= kMaxIter; ++it) {
        const I k = coef<I>(round(form2(q, e, f) / nf));
        const V2T<I> g{mad(-k, f.x, e.x), mad(-k, f.y, e.y)};
        if (!exact(k) || !exact(g.x) || !exact(g.y)) return -2;
        e = f;
        f = g;
        const double ne = nf;
        nf = form2(q, f, f);
        if (!(ne > nf)) return it;
    }
    return -1;
}

template <typename TD, typename TW>
__global__ void k_stencil2d(const TD *__restrict__ D, long long N, int16_t *__restrict__ off,
                            TW *__restrict__ w, int32_t *status) {
    const long long z = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (z >= N) return;
    const double dxx = (double)D[z], dxy = (double)D[N + z], dyy = (double)D[2 * N + z];
    int st = 0;
    V2 s[3] = {{0, 0}, {0, 0}, {0, 0}};
    double g[3] = {0.0, 0.0, 0.0};
    const bool finite = isfinite(dxx) && isfinite(dxy) && isfinite(dyy);
    if (!finite || !(dxx > 0.0) || !(dyy > 0.0) || !(dxx * dyy - dxy * dxy > 0.0)) {
        st |= ADLBR_ST_NOT_SPD;
    } else {
        const Form2 q{dyy, -dxy, dxx};
        V2 e{1, 0}, f{0, 1};
        V2T<double> ed{1, 0}, fd{0, 1};
        int red = reduce_pair2<double>(q, ed, fd);
        if (red == -2) {
            red = reduce_pair2<ll>(q, e, f);  // left the exact range: again in 64 bits
        } else {
            e = V2{(ll)ed.x, (ll)ed.y};
            f = V2{(ll)fd.x, (ll)fd.y};
        }
        if (red < 0) st |= ADLBR_ST_ITER;
        if (form2(q, e, f) > 0.0) f = V2{-f.x, -f.y};
        s[0] = e;
        s[1] = f;
        s[2] = V2{-e.x - f.x, -e.y - f.y};
        // gamma(+-s_i) = -1/2 <s_{i+1}, Q s_{i+2}>
        for (int i = 0; i < 3; ++i) {
            double v = -0.5 * form2(q, s[(i + 1) % 3], s[(i + 2) % 3]);
            if (v < 0.0) {
                st |= ADLBR_ST_CLAMPED;
                v = 0.0;
            }
            g[i] = v;
        }
        for (int i = 0; i < 3; ++i)
            if (s[i].x > 32767 || s[i].x < -32767 || s[i].y > 32767 || s[i].y < -32767)
                st |= ADLBR_ST_RANGE;
    }
    if (st & (ADLBR_ST_NOT_SPD | ADLBR_ST_RANGE | ADLBR_ST_ITER)) {
        for (int i = 0; i < 3; ++i) {
            s[i] = V2{0, 0};
            g[i] = 0.0;
        }
    }
    for (int i = 0; i < 3; ++i) {
        off[(2 * i) * N + z] = (int16_t)s[i].x;
        off[(2 * i + 1) * N + z] = (int16_t)s[i].y;
        w[i * N + z] = (TW)g[i];
    }
    report(status, z, st);
}

// ------------------------------------------------------------------- 3D --
struct Form3 {
    double xx, yy, zz, xy, xz, yz;
};

// Lattice vectors with integer components of type I (double first, see
// kExact).
template <typename I> struct V3T {
    I x, y, z;
};
typedef V3T<ll> V3;

template <typename I>
__device__ __forceinline__ double form3(const Form3 &q, const V3T<I> &a, const V3T<I> &b) {
    const I cxx = a.x * b.x, cyy = a.y * b.y, czz = a.z * b.z;
    const I cxy = mad(a.x, b.y, a.y * b.x);
    const I cxz = mad(a.x, b.z, a.z * b.x);
    const I cyz = mad(a.y, b.z, a.z * b.y);
    return (((((double)cxx * q.xx + (double)cyy * q.yy) + (double)czz * q.zz) +
             (double)cxy * q.xy) + (double)cxz * q.xz) + (double)cyz * q.yz;
}

// out = y - k x; false when k or the result leaves the exact range.
template <typename I>
__device__ __forceinline__ bool v3_axpy(I k, const V3T<I> &x, const V3T<I> &y, V3T<I> &out) {
    out = V3T<I>{mad(-k, x.x, y.x), mad(-k, x.y, y.y), mad(-k, x.z, y.z)};
    return exact(k) && exact(out.x) && exact(out.y) && exact(out.z);
}

template <typename T> __device__ __forceinline__ void swap_if(bool c, T &a, T &b) {
    const T x = a, y = b;
    a = c ? y : x;
    b = c ? x : y;
}

// component by component: a choice between whole vectors is taken by address,
// which puts them in scratch memory
template <typename I> __device__ __forceinline__ void swap_if(bool c, V3T<I> &a, V3T<I> &b, double &na, double &nb) {
    swap_if(c, a.x, b.x);
    swap_if(c, a.y, b.y);
    swap_if(c, a.z, b.z);
    swap_if(c, na, nb);
}

// Lagrange on the pair of norms ne, nf (kept with their vectors): iterations
// used, -1 past kMaxIter, -2 when the exact range is left.
template <typename I>
__device__ int reduce_pair3(const Form3 &q, V3T<I> &e, V3T<I> &f, double &ne, double &nf) {
    for (int it = 1; it <= kMaxIter; ++it) {
        V3T<I> g;
        if (!v3_axpy<I>(coef<I>(round(form3(q, e, f) / nf)), f, e, g)) return -2;
        e = f;
        ne = nf;
        f = g;
        nf = form3(q, f, f);
        if (!(ne > nf)) return it;
    }
    return -1;
}

template <typename I> __device__ __forceinline__ double max_abs(const V3T<I> &v) {
    return fmax(fmax(fabs((double)v.x), fabs((double)v.y)), fabs((double)v.z));
}

// Greedy reduction: sort by norm (stable), reduce the first two with
// Lagrange, replace the third by its offset from the closest vector of the
// plane lattice of the first two (searched among round(y) + {-1,0,1}^2,
// first minimum in i-major order), until the third is not shorter than the
// second.  1: reduced; 0: past kMaxIter; -2: the exact range is left.
//
// The nine candidates' norms follow from the centre's by the pair's Gram
// entries to within rounding: all forms involved are bounded by
// T = m^2 sum|q| (m the largest component of any candidate), each rounds by
// at most 11 eps T, and an estimate adds nine of them, so 1024 eps T covers
// its distance to the norm as form3 rounds it.  When one estimate is that far
// below the others it is the minimum, and no candidate but it is formed;
// otherwise (ties, extreme anisotropy, and always in 64-bit integers, whose
// forms may overflow) all nine are compared.
template <typename I> __device__ int greedy3(const Form3 &q, V3T<I> b[3]) {
    const double qs = (fabs(q.xx) + fabs(q.yy) + fabs(q.zz)) +
                      2.0 * ((fabs(q.xy) + fabs(q.xz)) + fabs(q.yz));
    double n0 = form3(q, b[0], b[0]), n1 = form3(q, b[1], b[1]), n2 = form3(q, b[2], b[2]);
    for (int it = 0; it < kMaxIter; ++it) {
        // stable insertion sort of three vectors by squared norm
        swap_if(n0 > n1, b[0], b[1], n0, n1);
        const bool low = n1 > n2;
        swap_if(low, b[1], b[2], n1, n2);
        swap_if(low && n0 > n1, b[0], b[1], n0, n1);
        const int rp = reduce_pair3<I>(q, b[0], b[1], n0, n1);
        if (rp == -2) return -2;
        if (rp < 0) return 0;
        const double g12 = form3(q, b[0], b[1]);
        const double p1 = form3(q, b[0], b[2]), p2 = form3(q, b[1], b[2]);
        const double det = n0 * n1 - g12 * g12;
        const double y1 = (p1 * n1 - p2 * g12) / det;
        const double y2 = (p2 * n0 - p1 * g12) / det;
        const I c1 = coef<I>(round(y1)), c2 = coef<I>(round(y2));
        V3T<I> t, v;
        bool clear = false;  // b[2] is settled by the estimates
        if constexpr (std::is_same_v<I, double>) {
            if (!v3_axpy<I>(c1, b[0], b[2], t) || !v3_axpy<I>(c2, b[1], t, v)) return -2;
            const double nv = form3(q, v, v), d1 = form3(q, v, b[0]), d2 = form3(q, v, b[1]);
            const double m = (max_abs(v) + max_abs(b[0])) + max_abs(b[1]);
            const double margin = (1024.0 * 2.220446049250313e-16) * (m * m) * qs;
            double low1 = INFINITY, low2 = INFINITY;  // the two smallest estimates
            int at = 0;
#pragma unroll
            for (int k = 0; k < 9; ++k) {
                const double i = (double)(k / 3 - 1), j = (double)(k % 3 - 1);
                const double e = ((nv - 2.0 * (i * d1 + j * d2)) + (i * i * n0 + j * j * n1)) +
                                 2.0 * (i * j) * g12;
                low2 = fmin(low2, fmax(low1, e));
                at = e < low1 ? k : at;
                low1 = fmin(low1, e);
            }
            clear = low2 - low1 > margin;
            if (clear && at == 4) {
                b[2] = v;
                n2 = nv;
            } else if (clear) {
                if (!v3_axpy<I>(c1 + (I)(at / 3 - 1), b[0], b[2], t) ||
                    !v3_axpy<I>(c2 + (I)(at % 3 - 1), b[1], t, v))
                    return -2;
                b[2] = v;
                n2 = form3(q, v, v);
            }
        }
        if (!clear) {
            double best = INFINITY;
            V3T<I> bv = b[2];
            for (int i = -1; i <= 1; ++i)
                for (int j = -1; j <= 1; ++j) {
                    if (!v3_axpy<I>(c1 + (I)i, b[0], b[2], t) || !v3_axpy<I>(c2 + (I)j, b[1], t, v))
                        return -2;
                    const double nc = form3(q, v, v);
                    if (nc < best) {
                        best = nc;
                        bv = v;
                    }
                }
            b[2] = bv;
            n2 = form3(q, bv, bv);
        }
        if (n2 >= n1) return 1;
    }
    return 0;
}

template <typename I> __device__ __forceinline__ V3T<I> cross3(const V3T<I> &a, const V3T<I> &b) {
    return V3T<I>{mad(a.y, b.z, -(a.z * b.y)), mad(a.z, b.x, -(a.x * b.z)),
                  mad(a.x, b.y, -(a.y * b.x))};
}

template <typename I> __device__ __forceinline__ V3T<I> signed3(const V3T<I> &a, bool neg) {
    return V3T<I>{neg ? -a.x : a.x, neg ? -a.y : a.y, neg ? -a.z : a.z};
}

// Proposition (MakeObtuse): order the reduced basis so that
// |<b1,b2>| <= |<b1,b3>| <= |<b2,b3>| (first such permutation in
// lexicographic order), make <b1,b3>, <b2,b3> <= 0 by sign flips, and pick
// one of the two superbases of eq. (3DSuperBase).  Three products decide it
// all: a form is symmetric and changes sign exactly with either vector.
template <typename I> __device__ void obtuse_superbase3(const Form3 &q, const V3T<I> r[3], V3T<I> e[4]) {
    const double g01 = form3(q, r[0], r[1]), g02 = form3(q, r[0], r[2]), g12 = form3(q, r[1], r[2]);
    const double a01 = fabs(g01), a02 = fabs(g02), a12 = fabs(g12);
    // the six permutations (b1, b2, b3) with their products (ij, ik, jk)
    V3T<I> b1 = r[0], b2 = r[1], b3 = r[2];
    double ij = g01, ik = g02, jk = g12;
    const auto take = [&](const V3T<I> &x, const V3T<I> &y, const V3T<I> &z, double xy, double xz,
                          double yz) {
        b1 = x;
        b2 = y;
        b3 = z;
        ij = xy;
        ik = xz;
        jk = yz;
    };
    if (a01 <= a02 && a02 <= a12) {
    } else if (a02 <= a01 && a01 <= a12) {
        take(r[0], r[2], r[1], g02, g01, g12);
    } else if (a01 <= a12 && a12 <= a02) {
        take(r[1], r[0], r[2], g01, g12, g02);
    } else if (a12 <= a01 && a01 <= a02) {
        take(r[1], r[2], r[0], g12, g01, g02);
    } else if (a02 <= a12 && a12 <= a01) {
        take(r[2], r[0], r[1], g02, g12, g01);
    } else if (a12 <= a02 && a02 <= a01) {
        take(r[2], r[1], r[0], g12, g02, g01);
    }
    const bool f1 = ik > 0.0, f2 = jk > 0.0;
    b1 = signed3(b1, f1);
    b2 = signed3(b2, f2);
    const bool first = (f1 != f2 ? -ij : ij) <= 0.0;
    // first: (b1, b2, b3, -b1-b2-b3), otherwise (-b1, b2, b1+b3, -b2-b3)
    const I s = first ? 0 : 1, t = first ? 1 : 0;
    e[0] = signed3(b1, !first);
    e[1] = b2;
    e[2] = V3T<I>{mad(s, b1.x, b3.x), mad(s, b1.y, b3.y), mad(s, b1.z, b3.z)};
    e[3] = V3T<I>{mad(-t, b1.x, -b2.x) - b3.x, mad(-t, b1.y, -b2.y) - b3.y,
                  mad(-t, b1.z, -b2.z) - b3.z};
}

// Slots and weights from a reduced basis: Selling's decomposition on the
// obtuse superbase, pair (i,j) -> slot e_k x e_l, weight -1/2 <e_i, D e_j>.
// A slot beyond +-32767 sets ADLBR_ST_RANGE.
template <typename I> __device__ __forceinline__ int selling3(const Form3 &q, const V3T<I> r[3], int cs[6][3], double g[6]) {
    V3T<I> e[4];
    obtuse_superbase3<I>(q, r, e);
    constexpr int pairs[6][4] = {{0, 1, 2, 3}, {0, 2, 1, 3}, {0, 3, 1, 2},
                                 {1, 2, 0, 3}, {1, 3, 0, 2}, {2, 3, 0, 1}};
    int st = 0;
#pragma unroll
    for (int k = 0; k < 6; ++k) {
        const V3T<I> c = cross3(e[pairs[k][2]], e[pairs[k][3]]);
        double v = -0.5 * form3(q, e[pairs[k][0]], e[pairs[k][1]]);
        if (v < 0.0) {
            st |= ADLBR_ST_CLAMPED;
            v = 0.0;
        }
        g[k] = v;
        if (!(c.x >= -32767 && c.x <= 32767 && c.y >= -32767 && c.y <= 32767 && c.z >= -32767 &&
              c.z <= 32767))
            st |= ADLBR_ST_RANGE;
        cs[k][0] = (int)c.x;
        cs[k][1] = (int)c.y;
        cs[k][2] = (int)c.z;
    }
    return st;
}

// A first offset that no stencil has: the point is left to the 64-bit pass.
constexpr int16_t kRedo = -32768;

// The stencils of a 3D field.  WIDE = false: every point whose reduction
// stays in the exact range; the first offset of any other is set to kRedo.
// WIDE = true, a launch of its own: those points, in 64-bit integers.  Apart,
// the common pass needs neither the wide registers nor scratch memory.  Bound
// by FP64 arithmetic (about 100 scalar products a point) and its chains at 5
// waves a SIMD.  160^3: 1107 us with integer components, nine candidates each
// time and arrays that the compiler placed in LDS (one wave a SIMD);
// 261 + 9 us in this form.
template <typename TD, typename TW, bool WIDE>
__global__ __launch_bounds__(256) void k_stencil3d(const TD *__restrict__ D, long long N,
                                                   int16_t *__restrict__ off,
                                                   TW *__restrict__ w, int32_t *status) {
    typedef std::conditional_t<WIDE, ll, double> I;
    const long long z = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (z >= N) return;
    if (WIDE && off[z] != kRedo) return;
    // input planes xx, xy, xz, yy, yz, zz
    const double a = (double)D[z], xy = (double)D[N + z], xz = (double)D[2 * N + z];
    const double b = (double)D[3 * N + z], yz = (double)D[4 * N + z], c = (double)D[5 * N + z];
    int st = 0;
    int cs[6][3];
    double g[6];
    bool ok = isfinite(a) && isfinite(b) && isfinite(c) && isfinite(xy) && isfinite(xz) &&
              isfinite(yz);
    ok = ok && a > 0.0 && a * b - xy * xy > 0.0;
    ok = ok && (a * (b * c - yz * yz) - xy * (xy * c - yz * xz) + xz * (xy * yz - b * xz)) > 0.0;
    int red = 0;
    const Form3 q{a, b, c, xy, xz, yz};
    V3T<I> r[3] = {{1, 0, 0}, {0, 1, 0}, {0, 0, 1}};
    if (ok) red = greedy3<I>(q, r);
    if (red == 1) st |= selling3<I>(q, r, cs, g);
    else if (!ok) st |= ADLBR_ST_NOT_SPD;
    else if (red != -2) st |= ADLBR_ST_ITER;
    if (red != 1 || (st & ADLBR_ST_RANGE)) {
#pragma unroll
        for (int k = 0; k < 6; ++k) {
            cs[k][0] = cs[k][1] = cs[k][2] = 0;
            g[k] = 0.0;
        }
        if (red == -2) cs[0][0] = kRedo;
    }
#pragma unroll
    for (int k = 0; k < 6; ++k) {
#pragma unroll
        for (int c2 = 0; c2 < 3; ++c2) off[(3 * k + c2) * N + z] = (int16_t)cs[k][c2];
        // the weights may take the tensor's place, which the 64-bit pass reads
        if (red != -2) w[k * N + z] = (TW)g[k];
    }
    report(status, z, st);
}

template <typename TD, typename TW>
void launch_stencil(int dim, const void *D, long long N, int16_t *off, void *w, int32_t *status,
                    hipStream_t s) {
    const unsigned nb = (unsigned)((N + 255) / 256);
    if (dim == 2) {
        hipLaunchKernelGGL((k_stencil2d<TD, TW>), dim3(nb), dim3(256), 0, s, (const TD *)D, N, off,
                           (TW *)w, status);
        return;
    }
    hipLaunchKernelGGL((k_stencil3d<TD, TW, false>), dim3(nb), dim3(256), 0, s, (const TD *)D, N,
                       off, (TW *)w, status);
    hipLaunchKernelGGL((k_stencil3d<TD, TW, true>), dim3(nb), dim3(256), 0, s, (const TD *)D, N,
                       off, (TW *)w, status);
}

}  // namespace
}  // namespace adlbr

using namespace adlbr;

extern "C" int adlbr_build_stencils(const adlbr_grid *g, const void *D, int D_dtype,
                                    int16_t *offsets, void *weights, int w_dtype,
                                    int32_t *status, void *stream) {
    clear_error();
    GridInfo gi;
    int rc = check_grid(g, &gi);
    if (rc) return rc;
    if (!D || !offsets || !weights || !status) {
        set_error("adlbr_build_stencils: null pointer argument");
        return ADLBR_E_INVALID;
    }
    if ((D_dtype != ADLBR_F64 && D_dtype != ADLBR_F32) ||
        (w_dtype != ADLBR_F64 && w_dtype != ADLBR_F32)) {
        set_error("adlbr_build_stencils: D and weights must be ADLBR_F64 or ADLBR_F32");
        return ADLBR_E_INVALID;
    }
    hipStream_t s = as_stream(stream);
    hipLaunchKernelGGL(k_status_init, dim3(1), dim3(1), 0, s, status);
    if (D_dtype == ADLBR_F64 && w_dtype == ADLBR_F64)
        launch_stencil<double, double>(gi.dim, D, gi.N, offsets, weights, status, s);
    else if (D_dtype == ADLBR_F64)
        launch_stencil<double, float>(gi.dim, D, gi.N, offsets, weights, status, s);
    else if (w_dtype == ADLBR_F64)
        launch_stencil<float, double>(gi.dim, D, gi.N, offsets, weights, status, s);
    else
        launch_stencil<float, float>(gi.dim, D, gi.N, offsets, weights, status, s);
    hipLaunchKernelGGL(k_status_final, dim3(1), dim3(1), 0, s, status);
    ADLBR_LAUNCH_CHECK();
    return ADLBR_OK;
}
