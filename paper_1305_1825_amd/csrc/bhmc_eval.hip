// Treecode evaluation kernels for one expansion order p (compiled once per p
// with -DBHMC_P=p, so every recurrence index below is a compile-time constant
// and the Taylor coefficients live in registers).
//
// Traversal (Sec. 3.2).  A workgroup evaluates the potential at a few targets
// at once.  The MAC traversal runs breadth first: the frontier of one level
// sits in LDS, every lane classifies one cell for the targets that reached it,
// and a scan of the lanes' counts hands out slots in the far list, the near list
// and the next frontier, so the order of every list, and therefore every sum, is
// deterministic.
// Far cells are evaluated lane-per-cell in the harmonic form of the expansion
// of eq. 3.3 (below); near leaves are flattened
// into (leaf, slot) pairs read from the leaf-ordered pool, so the lanes of a
// wave read consecutive slots.
//
// Exclusion.  The mover i and its image are taken out of the source set: a
// frontier entry carries two bits telling whether its cell holds them (the
// bits follow the digits of their keys down the tree).  At most one far cell
// per (target, excluded source) can hold one of them; those cells go to a list
// of their own and are evaluated less the expansion of the excluded source.
#include "bhmc_dev.hpp"
#include "bhmc_internal.hpp"

#include <algorithm>

#ifndef BHMC_P
#error "compile once per expansion order with -DBHMC_P=<p>"
#endif

#define BHMC_CAT2(a, b) a##b
#define BHMC_CAT(a, b) BHMC_CAT2(a, b)
#define BHMC_NS BHMC_CAT(eval_p, BHMC_P)

namespace bhmc {
namespace BHMC_NS {

constexpr int P = BHMC_P;
constexpr int NTERM = (P + 1) * (P + 2) * (P + 3) / 6;
constexpr int MSTR = (NTERM + 3) & ~3;  // moment row stride (32-byte rows)

// ------------------------------------------------------------ index tables
constexpr int cmindex(int n1, int n2, int n3) {
    int s = n1 + n2 + n3;
    return s * (s + 1) * (s + 2) / 6 + (s - n1) * (s - n1 + 1) / 2 + (s - n1 - n2);
}

struct TEnt { int n1, n2, n3, s, x1, y1, z1, x2, y2, z2; };
template <int N>
struct TTab { TEnt e[N]; };

// entries of every multi-index up to order PP, in the graded order above
template <int PP>
constexpr TTab<(PP + 1) * (PP + 2) * (PP + 3) / 6> make_tab() {
    TTab<(PP + 1) * (PP + 2) * (PP + 3) / 6> t{};
    int k = 0;
    for (int s = 0; s <= PP; ++s)
        for (int n1 = s; n1 >= 0; --n1)
            for (int n2 = s - n1; n2 >= 0; --n2) {
                const int n3 = s - n1 - n2;
                TEnt e{};
                e.n1 = n1; e.n2 = n2; e.n3 = n3; e.s = s;
                e.x1 = n1 >= 1 ? cmindex(n1 - 1, n2, n3) : -1;
                e.y1 = n2 >= 1 ? cmindex(n1, n2 - 1, n3) : -1;
                e.z1 = n3 >= 1 ? cmindex(n1, n2, n3 - 1) : -1;
                e.x2 = n1 >= 2 ? cmindex(n1 - 2, n2, n3) : -1;
                e.y2 = n2 >= 2 ? cmindex(n1, n2 - 2, n3) : -1;
                e.z2 = n3 >= 2 ? cmindex(n1, n2, n3 - 2) : -1;
                t.e[k++] = e;
            }
    return t;
}
constexpr auto TT = make_tab<P>();
// one order more for the field, dT_n/dR_k = (n_k + 1) T_{n + e_k}; the first
// NTERM entries coincide with TT
constexpr int NTERM1 = (P + 2) * (P + 3) * (P + 4) / 6;
constexpr auto TT1 = make_tab<P + 1>();

struct MiTab { int v[3 * NTERM]; };
constexpr MiTab make_mi() {
    MiTab m{};
    for (int k = 0; k < NTERM; ++k) { m.v[3 * k] = TT.e[k].n1; m.v[3 * k + 1] = TT.e[k].n2; m.v[3 * k + 2] = TT.e[k].n3; }
    return m;
}
__constant__ MiTab c_mi = make_mi();

// (n1, n2, n3) of term k packed as n1 | n2 << 8 | n3 << 16; workgroups keep a
// copy of this table in LDS, so runtime term indices read it there
__device__ __forceinline__ uint32_t mi_code(int k) {
    return (uint32_t)c_mi.v[3 * k] | ((uint32_t)c_mi.v[3 * k + 1] << 8) | ((uint32_t)c_mi.v[3 * k + 2] << 16);
}

// d^n by repeated multiplication (x, then y, then z), as the moments are built
__device__ __forceinline__ double mono(uint32_t code, double dx, double dy, double dz) {
    const int n1 = (int)(code & 255u), n2 = (int)((code >> 8) & 255u), n3 = (int)(code >> 16);
    double v = 1.0;
    for (int e = 0; e < n1; ++e) v *= dx;
    for (int e = 0; e < n2; ++e) v *= dy;
    for (int e = 0; e < n3; ++e) v *= dz;
    return v;
}

// ------------------------------------------------------------ far field
// T_n(R) by eq. 3.4 with T_0 = 1/|R|:
//   T_n = -[ (2s-1)/s sum_i R_i T_{n-e_i} + (s-1)/s sum_i T_{n-2e_i} ] / |R|^2.
template <int K, int N>
__device__ __forceinline__ void t_step(double (&T)[N], double Rx, double Ry, double Rz, double ir2) {
    constexpr TEnt e = TT1.e[K];
    double f = 0.0, g = 0.0;
    if constexpr (e.x1 >= 0) f = Rx * T[e.x1];
    if constexpr (e.y1 >= 0) f = fma(Ry, T[e.y1], f);
    if constexpr (e.z1 >= 0) f = fma(Rz, T[e.z1], f);
    if constexpr (e.x2 >= 0) g = T[e.x2];
    if constexpr (e.y2 >= 0) g += T[e.y2];
    if constexpr (e.z2 >= 0) g += T[e.z2];
    constexpr double A = (2.0 * e.s - 1.0) / e.s;
    constexpr double B = (e.s - 1.0) / e.s;
    if constexpr (e.s >= 2) T[K] = -fma(A, f, B * g) * ir2;
    else T[K] = -(A * f) * ir2;
}

// Moment rows are read through pointers qualified with their address space:
// global (HBM) rows then compile to global loads and LDS rows to LDS loads, each
// waited for by its own counter, so several of a row's loads are in flight at
// once.  Through a generic pointer they become flat loads, each waited for in
// full before the next is issued.
using GRow = const __attribute__((address_space(1))) double*;
using LRow = const __attribute__((address_space(3))) double*;
__device__ __forceinline__ GRow grow(const double* p) { return (GRow)p; }
__device__ __forceinline__ LRow lrow(const double* p) { return (LRow)p; }

// An FP64 add to HBM through a global-qualified pointer: the compiler then knows
// it cannot write LDS, so LDS loads stay free to move across it.
using GDbl = __attribute__((address_space(1))) double*;
__device__ __forceinline__ void gatomic_add(double* p, double v) { __builtin_amdgcn_global_atomic_fadd_f64((GDbl)p, v); }

// The same for single records of the tree in HBM: cell geometry, cell header,
// a source, a slot's source index, a tracking entry.
using GInt = const __attribute__((address_space(1))) int*;
__device__ __forceinline__ double4 gload(const double4* p) {
    const GRow q = (GRow)(const double*)p;
    return make_double4(q[0], q[1], q[2], q[3]);
}
__device__ __forceinline__ int4 gload(const int4* p) {
    const GInt q = (GInt)(const int*)p;
    return make_int4(q[0], q[1], q[2], q[3]);
}
__device__ __forceinline__ int2 gload(const int2* p) {
    const GInt q = (GInt)(const int*)p;
    return make_int2(q[0], q[1]);
}
__device__ __forceinline__ int gload(const int* p) { return *(GInt)p; }

// The descriptor fields that the traversals use per lane, held in scalar registers.  Read
// from the workgroup's copy in LDS where they are used, they are vector values to the
// compiler, which keeps dozens of them in vector registers across the whole round.
__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ long long uni(long long v) {
    return (long long)(((uint64_t)(uint32_t)uni((int)(v >> 32)) << 32) | (uint32_t)uni((int)v));
}
__device__ __forceinline__ double uni(double v) { return __longlong_as_double(uni(__double_as_longlong(v))); }
template <class T>
__device__ __forceinline__ T* uni(T* v) { return (T*)uni((long long)v); }

struct RepU {
    const Rep& d;
    double4* cgeo; int4* cm; double* H; double* M; float* M32; double4* pool4; int* pidx; double4* src; int2* track;
    uint32_t* spill;
    long long spill_words;
    double theta2, reach2, ovl2, tau2, l_B, a, a2, gamma, Qc;
    int n, nsrc, ncell, pool, n0, images, geom, nline, fcap, spill_regions;
    const double *line_t, *line_c;
    __device__ __forceinline__ explicit RepU(const Rep& r)
        : d(r), cgeo(uni(r.cgeo)), cm(uni(r.cm)), H(uni(r.H)), M(uni(r.M)), M32(uni(r.M32)), pool4(uni(r.pool4)),
          pidx(uni(r.pidx)), src(uni(r.src)), track(uni(r.track)), spill(uni(r.spill)), spill_words(uni(r.spill_words)),
          theta2(uni(r.theta2)), reach2(uni(r.reach2)), ovl2(uni(r.ovl2)), tau2(uni(r.tau2)), l_B(uni(r.l_B)), a(uni(r.a)), a2(uni(r.a2)),
          gamma(uni(r.gamma)), Qc(uni(r.Qc)), n(uni(r.n)), nsrc(uni(r.nsrc)), ncell(uni(r.ncell)), pool(uni(r.pool)),
          n0(uni(r.n0)), images(uni(r.images)), geom(uni(r.geom)), nline(uni(r.nline)), fcap(uni(r.fcap)),
          spill_regions(uni(r.spill_regions)), line_t(r.line_t), line_c(r.line_c) {}
    __device__ __forceinline__ operator const Rep&() const { return d; }
};

// ------------------------------------------------------------ harmonic form of the expansion
// Up to order p the sum of eq. 3.3 over the C(p + 3, 3) Cartesian terms is, degree by
// degree, sum_j q_j P_l(cos psi_j) |d_j|^l / |X|^(l + 1) (d_j = y_j - c, X = x - c), and
// by the addition theorem of the Legendre polynomials that is a sum over the (p + 1)^2
// solid harmonics:
//   phi(x) = sum_{l <= p} sum_{m <= l} [Hc_lm Re A_lm(X) + Hs_lm Im A_lm(X)] / |X|^(2l + 1),
//   A_lm(v) = (v_x + i v_y)^m a_lm(v_z, |v|^2),  a_mm = 1, a_{m+1,m} = v_z,
//   a_lm = v_z a_{l-1,m} - beta_lm |v|^2 a_{l-2,m},  beta_lm = ((l-1)^2 - m^2) / ((2l-1)(2l-3)),
//   H_lm = N_lm sum_j q_j A_lm(d_j),  N_lm = (2 - [m = 0]) ((2l-1)!!)^2 / ((l + m)! (l - m)!)
// (a_lm is P_l^m without its (1 - z^2)^(m/2), scaled to leading coefficient one).  The
// value is the one of the Cartesian sum up to rounding; it reads (p + 1)^2 coefficients
// instead of C(p + 3, 3) (36 for 56 at p = 5, 81 for 165 at p = 8) and costs 5 FP64
// instructions per (l, m) instead of 8 per Cartesian term, with no T_n held in registers:
// 90 FP64 instructions a cell at p = 5 where the Cartesian form took about 450.  The far
// cells were bound by the issue of those (32 of the 104 us of a round of eight moves on the
// 10^4-ion colloid, 212 of 390 us in the sweep of 256 replicas at theta = 0.3, p = 5; now 21
// and 73).
// Row of a cell: the (c, s) pairs of m = 1..p (l = m..p each), the p + 1 coefficients of
// m = 0, the centre.
constexpr int NH = (P + 1) * (P + 1);
constexpr int NPAIR = (P + 1) * (P + 2) / 2;
constexpr int HCEN = NH;                   // centre at [NH], [NH + 1], [NH + 2]
constexpr int HSTR = (NH + 3 + 1) & ~1;    // row stride, 16-byte rows

// place of the (l, m) coefficient (of its c part for m >= 1; the s part follows it)
constexpr int hplace(int l, int m) {
    if (m == 0) return NH - (P + 1) + l;
    int o = 0;
    for (int k = 1; k < m; ++k) o += 2 * (P + 1 - k);
    return o + 2 * (l - m);
}
constexpr double hbeta(int l, int m) {
    return l < m + 2 ? 0.0 : (double)((l - 1) * (l - 1) - m * m) / (double)((2 * l - 1) * (2 * l - 3));
}
constexpr double hnorm(int l, int m) {
    double v = m == 0 ? 1.0 : 2.0;
    for (int k = 1; k <= l; ++k) v *= (double)(2 * k - 1) * (double)(2 * k - 1);
    for (int k = 2; k <= l + m; ++k) v /= (double)k;
    for (int k = 2; k <= l - m; ++k) v /= (double)k;
    return v;
}

// sum_{lm} H_lm A_lm(X) / |X|^(2l+1) at X = (x, y, z): with w = 1 / |X|^2, u = z w and
// zeta = (x + i y) w, each a_lm / |X|^(2(l-m)) obeys the recurrence above in (u, w), and the
// powers of zeta come in by Horner's rule from m = p down.  The row is loaded in one or two
// runs of columns ahead of their use (as many loads in flight as registers allow), and the
// scheduling boundaries keep the compiler from computing every column's factors first.
constexpr int kHRun = 64;  // doubles of a row held in registers at once
constexpr int hsplit() {   // columns m >= hsplit() are the first run
    if (NH <= kHRun) return 0;
    int m = P;
    while (m > 0 && hplace(m, m) + 2 * (P + 1 - m) > NH / 2 + P) --m;
    return m + 1;
}
constexpr int kHSplit = hsplit();

// column m of the recurrence: qc, qs = sum_l H_lm a_lm / |X|^(2(l-m)); h is the row from place base on
template <int M, int N>
__device__ __forceinline__ void far_column(const double (&h)[N], int base, double u, double w, double& qc, double& qs) {
    constexpr int pl = hplace(M, M), st = M ? 2 : 1;
    qc = h[pl - base];
    qs = M ? h[pl + 1 - base] : 0.0;
    double a0 = 1.0, a1 = u;
#pragma unroll
    for (int l = M + 1; l <= P; ++l) {
        if (l > M + 1) {
            const double bw = hbeta(l, M) * w;
            const double a2 = l == M + 2 ? fma(u, a1, -bw) : fma(u, a1, -bw * a0);
            a0 = a1; a1 = a2;
        }
        qc = fma(h[pl + st * (l - M) - base], a1, qc);
        if (M) qs = fma(h[pl + st * (l - M) + 1 - base], a1, qs);
    }
}

// One target's place in a cell's expansion, and its sum so far.
struct FarAt { double u, w, zx, zy, ir, a, b; };
__device__ __forceinline__ void far_at(FarAt& f, double x, double y, double z) {
    const double r2 = x * x + y * y + z * z;
    f.ir = rsqrt_nr(r2);
    f.w = f.ir * f.ir; f.u = z * f.w; f.zx = x * f.w; f.zy = y * f.w;
    f.a = 0.0; f.b = 0.0;
}

template <int M, int LAST, int NT, int N>
__device__ __forceinline__ void far_columns(const double (&h)[N], int base, FarAt (&f)[NT]) {
    if constexpr (M >= LAST) {
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            double qc, qs;
            far_column<M>(h, base, f[t].u, f[t].w, qc, qs);
            if constexpr (M == P) {
                f[t].a = qc; f[t].b = qs;
            } else {
                const double ta = fma(f[t].b, f[t].zy, fma(f[t].a, f[t].zx, qc));
                if constexpr (M > 0) f[t].b = fma(f[t].b, f[t].zx, fma(-f[t].a, f[t].zy, qs));
                f[t].a = ta;
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        far_columns<M - 1, LAST>(h, base, f);
    }
}

// Values at NT targets of an expansion row, its own centre included; the row is read once.
template <int NT, class HP>
__device__ __forceinline__ void far_rows(HP __restrict__ H, const double (&tx)[NT], const double (&ty)[NT],
                                         const double (&tz)[NT], double (&v)[NT]) {
    // the columns of the first run take places 0 .. n1 - 1 (m = 1 .. p lie in this order in the
    // row, so a first run of the columns m >= kHSplit is the tail of the pairs)
    constexpr int lo = kHSplit ? hplace(kHSplit, kHSplit) : 0;         // first place of the first run
    constexpr int n1 = (kHSplit ? NH - (P + 1) : NH) - lo;
    const double cx = H[HCEN], cy = H[HCEN + 1], cz = H[HCEN + 2];
    FarAt f[NT];
    {
        double h[n1];
#pragma unroll
        for (int k = 0; k < n1; ++k) h[k] = H[lo + k];
#pragma unroll
        for (int t = 0; t < NT; ++t) far_at(f[t], tx[t] - cx, ty[t] - cy, tz[t] - cz);
        __builtin_amdgcn_sched_barrier(0);
        far_columns<P, kHSplit>(h, lo, f);
    }
    if constexpr (kHSplit > 0) {
        // the columns below the split: their pairs at places 0 .. lo - 1, then those of m = 0
        double h[NH];
#pragma unroll
        for (int k = 0; k < lo; ++k) h[k] = H[k];
#pragma unroll
        for (int k = NH - (P + 1); k < NH; ++k) h[k] = H[k];
        __builtin_amdgcn_sched_barrier(0);
        far_columns<kHSplit - 1, 0>(h, 0, f);
    }
#pragma unroll
    for (int t = 0; t < NT; ++t) v[t] = f[t].ir * f[t].a;
}
template <class HP>
__device__ __forceinline__ double far_row(HP H, double tx, double ty, double tz) {
    const double x[1] = {tx}, y[1] = {ty}, z[1] = {tz};
    double v[1];
    far_rows<1>(H, x, y, z, v);
    return v[0];
}

// Tables of the regular harmonics for terms picked at run time, copied to LDS: beta_lm
// at [l * (P + 1) + m], and per pair (l, m) its norm and l | m << 8 | place << 16.
struct HTab {
    double beta[(P + 1) * (P + 1)];
    double norm[NPAIR];
    uint32_t lm[NPAIR];
};
constexpr HTab make_htab() {
    HTab t{};
    int k = 0;
    for (int l = 0; l <= P; ++l)
        for (int m = 0; m <= P; ++m) {
            t.beta[l * (P + 1) + m] = m <= l ? hbeta(l, m) : 0.0;
            if (m > l) continue;
            t.norm[k] = hnorm(l, m);
            t.lm[k] = (uint32_t)l | ((uint32_t)m << 8) | ((uint32_t)hplace(l, m) << 16);
            ++k;
        }
    return t;
}
__constant__ HTab c_htab = make_htab();

__device__ __forceinline__ void fill_htab(HTab& t) {
    for (int k = threadIdx.x; k < (P + 1) * (P + 1); k += blockDim.x) t.beta[k] = c_htab.beta[k];
    for (int k = threadIdx.x; k < NPAIR; k += blockDim.x) { t.norm[k] = c_htab.norm[k]; t.lm[k] = c_htab.lm[k]; }
}

// A_lm(d) for l, m picked at run time.
__device__ __forceinline__ void reg_pair(const HTab& T, int l, int m, double dx, double dy, double dz, double& c,
                                         double& s) {
    double cr = 1.0, ci = 0.0;
    for (int e = 0; e < m; ++e) {
        const double t = fma(cr, dx, -(ci * dy));
        ci = fma(cr, dy, ci * dx);
        cr = t;
    }
    const double r2 = dx * dx + dy * dy + dz * dz;
    double a0 = 0.0, a1 = 1.0;
    for (int k = m + 1; k <= l; ++k) {
        const double a2 = fma(dz, a1, -(T.beta[k * (P + 1) + m] * r2) * a0);
        a0 = a1; a1 = a2;
    }
    c = cr * a1;
    s = ci * a1;
}

// q N_lm A_lm(d) for every place of a row (c and s parts).
__device__ __forceinline__ void reg_row(double dx, double dy, double dz, double q, double* row) {
    const double r2 = dx * dx + dy * dy + dz * dz;
    double cr = q, ci = 0.0;
#pragma unroll
    for (int m = 0; m <= P; ++m) {
        if (m > 0) {
            const double t = fma(cr, dx, -(ci * dy));
            ci = fma(cr, dy, ci * dx);
            cr = t;
        }
        double a0 = 0.0, a1 = 1.0;
#pragma unroll
        for (int l = m; l <= P; ++l) {
            if (l == m + 1) { a0 = 1.0; a1 = dz; }
            if (l > m + 1) {
                const double a2 = fma(dz, a1, -(hbeta(l, m) * r2) * a0);
                a0 = a1; a1 = a2;
            }
            const double v = hnorm(l, m) * a1;
            row[hplace(l, m)] = v * cr;
            if (m > 0) row[hplace(l, m) + 1] = v * ci;
        }
    }
}

// The coefficients of pair k of cell c, and a source of charge q at offset d added to them.
struct HPair { double c, s; };
__device__ __forceinline__ HPair hpair_load(const RepU& R, const HTab& T, int c, int k) {
    const uint32_t code = T.lm[k];
    const GRow h = grow(R.H + (size_t)c * HSTR + (code >> 16));
    return HPair{h[0], (code & 0xFF00u) ? h[1] : 0.0};
}
__device__ __forceinline__ void hpair_store(const RepU& R, const HTab& T, int c, int k, double hc, double hs) {
    const uint32_t code = T.lm[k];
    double* h = R.H + (size_t)c * HSTR + (code >> 16);
    h[0] = hc;
    if (code & 0xFF00u) h[1] = hs;
}
__device__ __forceinline__ void hpair_add(const HTab& T, int k, double dx, double dy, double dz, double q, double& hc,
                                          double& hs) {
    const uint32_t code = T.lm[k];
    double c, s;
    reg_pair(T, (int)(code & 255u), (int)((code >> 8) & 255u), dx, dy, dz, c, s);
    const double w = q * T.norm[k];
    hc = fma(w, c, hc);
    hs = fma(w, s, hs);
}

// A row's coefficients from the Cartesian moments: H_lm = N_lm sum_n A_lm,n M^n with the
// monomial coefficients of A_lm, a sparse table (term, coefficient) per row place.
constexpr int hrow_terms() {  // how many (place, term) coefficients are not zero
    int n = 0;
    for (int l = 0; l <= P; ++l)
        for (int m = 0; m <= l; ++m)
            for (int t = m; t <= l; t += 2)            // powers of x and y together
                for (int b = 0; b <= t; ++b) n += (m == 0 ? (b % 2 == 0) : 1);
    return n;
}
constexpr int HROWT = hrow_terms();
struct HRows {
    int start[NH + 1];
    int term[HROWT];
    double coef[HROWT];
};
// Coefficients of A_lm by its recurrence over dense polynomials of one degree: place of
// x^a y^b z^c is cmindex(a, b, c).
constexpr HRows make_hrows() {
    HRows t{};
    int n = 0;
    // rows in the order of their places: m = 1..p (c, s alternating in l), then m = 0
    for (int mm = 1; mm <= P + 1; ++mm) {
        const int m = mm <= P ? mm : 0;
        // polynomials of the last two degrees, index by (a, b): c = l - a - b
        double A[3][2][(P + 1) * (P + 1)] = {};
        // (x + i y)^m
        double binom = 1.0;
        for (int b = 0; b <= m; ++b) {
            const double sgn = (b % 4 == 0 || b % 4 == 1) ? 1.0 : -1.0;
            A[m % 3][b % 2][(m - b) * (P + 1) + b] = sgn * binom;
            binom = binom * (double)(m - b) / (double)(b + 1);
        }
        for (int l = m; l <= P; ++l) {
            if (l > m) {
                for (int part = 0; part < 2; ++part)
                    for (int k = 0; k < (P + 1) * (P + 1); ++k) A[l % 3][part][k] = A[(l + 2) % 3][part][k];  // z A_{l-1}
                if (l >= m + 2)
                    for (int part = 0; part < 2; ++part)
                        for (int a = 0; a <= l - 2; ++a)
                            for (int b = 0; a + b <= l - 2; ++b) {
                                const double v = A[(l + 1) % 3][part][a * (P + 1) + b] * hbeta(l, m);
                                if (v == 0.0) continue;
                                A[l % 3][part][(a + 2) * (P + 1) + b] -= v;
                                A[l % 3][part][a * (P + 1) + b + 2] -= v;
                                A[l % 3][part][a * (P + 1) + b] -= v;
                            }
            }
            for (int part = 0; part < (m == 0 ? 1 : 2); ++part) {
                t.start[hplace(l, m) + part] = n;
                for (int a = 0; a <= l; ++a)
                    for (int b = 0; a + b <= l; ++b) {
                        const double v = A[l % 3][part][a * (P + 1) + b];
                        if (v == 0.0) continue;
                        t.term[n] = cmindex(a, b, l - a - b);
                        t.coef[n] = hnorm(l, m) * v;
                        ++n;
                    }
            }
        }
    }
    t.start[NH] = n;
    return t;
}
__device__ const HRows c_hrows = make_hrows();

// sum_n T_n M^n in the Cartesian form, each T_n folded into the sum as soon as it exists.  LEAN:
// the moments are read two at a time where they are used, for registers, instead of all ahead.
template <bool LEAN, int K, class MP>
__device__ __forceinline__ void cart_rec(double (&T)[NTERM], double Rx, double Ry, double Rz, double ir2,
                                         MP __restrict__ Mc, double& acc) {
    if constexpr (K < NTERM) {
        if constexpr (K > 0) t_step<K>(T, Rx, Ry, Rz, ir2);
        acc = fma(T[K], Mc[K], acc);
        if constexpr (LEAN && K % 2 == 1) __builtin_amdgcn_sched_barrier(0);
        cart_rec<LEAN, K + 1>(T, Rx, Ry, Rz, ir2, Mc, acc);
    }
}
template <bool LEAN, class MP>
__device__ __forceinline__ double cart_eval(double Rx, double Ry, double Rz, MP Mc) {
    double T[NTERM];
    T[0] = rsqrt_nr(Rx * Rx + Ry * Ry + Rz * Rz);
    double acc = 0.0;
    cart_rec<LEAN, 0>(T, Rx, Ry, Rz, T[0] * T[0], Mc, acc);
    return acc;
}

// The same in single precision from the single-precision moments: T_n by eq. 3.4 in
// FP32 and sum_n T_n M^n accumulated in FP32 per cell (the caller adds the cell's value
// to an FP64 sum).
template <int K>
__device__ __forceinline__ void t_step_f(float (&T)[NTERM], float Rx, float Ry, float Rz, float ir2) {
    constexpr TEnt e = TT.e[K];
    float f = 0.0f, g = 0.0f;
    if constexpr (e.x1 >= 0) f = Rx * T[e.x1];
    if constexpr (e.y1 >= 0) f = fmaf(Ry, T[e.y1], f);
    if constexpr (e.z1 >= 0) f = fmaf(Rz, T[e.z1], f);
    if constexpr (e.x2 >= 0) g = T[e.x2];
    if constexpr (e.y2 >= 0) g += T[e.y2];
    if constexpr (e.z2 >= 0) g += T[e.z2];
    constexpr float A = (float)((2.0 * e.s - 1.0) / e.s);
    constexpr float B = (float)((e.s - 1.0) / e.s);
    if constexpr (e.s >= 2) T[K] = -fmaf(A, f, B * g) * ir2;
    else T[K] = -(A * f) * ir2;
}

template <int K>
__device__ __forceinline__ void far_rec_f(float (&T)[NTERM], float Rx, float Ry, float Rz, float ir2,
                                          const __attribute__((address_space(1))) float* __restrict__ Mc, float& acc) {
    if constexpr (K < NTERM) {
        if constexpr (K > 0) t_step_f<K>(T, Rx, Ry, Rz, ir2);
        acc = fmaf(T[K], Mc[K], acc);
        far_rec_f<K + 1>(T, Rx, Ry, Rz, ir2, Mc, acc);
    }
}

__device__ __forceinline__ double far_eval_f(double Rx, double Ry, double Rz, const float* M32row) {
    const float rx = (float)Rx, ry = (float)Ry, rz = (float)Rz;
    const float r2 = rx * rx + ry * ry + rz * rz;
    float T[NTERM];
    T[0] = __builtin_amdgcn_rsqf(r2);
    T[0] = T[0] * fmaf(-0.5f * r2 * T[0], T[0], 1.5f);  // one Newton step
    const float ir2 = T[0] * T[0];
    float acc = 0.0f;
    far_rec_f<0>(T, rx, ry, rz, ir2, (const __attribute__((address_space(1))) float*)M32row, acc);
    return (double)acc;
}

// Kernels with far cells are instantiated twice: F32 = false for handles without a replica that
// keeps M32, whose registers the FP32 recurrence (every T_n of eq. 3.4 at once) would otherwise set.
// That recurrence is run once for each target of a move either way: from order 5 on a lane takes one
// target (one after the other in a lane against a lane each: 400 moves of 6,000 ions, p = 10, 18.1 and
// 13.8 ms, p = 6 4.00 and 3.73 ms), below it both (p = 2: 2.39 and 2.50 ms). One move at a time at p = 5:
// 400 moves of 2,000 ions 7.1 and 6.7 ms, 256 replicas, 1,000 moves each, 25.4 and 25.9 ms.
// A 256-thread workgroup has twice the far cells a lane and gains from a higher order on: its rounds from
// 9 (both and apart: 256 replicas, 1,000 moves at p = 5 14.3 and 15.8 ms, p = 8 30.2 and 32.8, p = 9 49.6
// and 49.8, p = 10 64.1 and 60.6; 400 moves of 2,000 ions at p = 8 5.0 and 5.0, p = 10 12.8 and 11.7), one
// move at a time from 8 (500 moves at p = 5 14.0 and 14.4 ms, p = 7 19.8 and 20.2, p = 8 24.8 and 24.9,
// p = 9 30.9 and 30.3; 400 moves of 2,000 ions at p = 8 10.9 and 9.9).
template <int BLOCK>
constexpr bool kF32Apart = P > (BLOCK > 256 ? 4 : 7);
template <int BLOCK>
constexpr bool kF32RoundsApart = P > (BLOCK > 256 ? 4 : 8);
// Values at the two targets of a move (F32: single precision where a lane takes both).
template <bool F32>
__device__ __forceinline__ void far_value2(const RepU& R, int c, const double (&tx)[2], const double (&ty)[2],
                                           const double (&tz)[2], double (&v)[2]) {
    if (F32 && R.M32) {
        const double4 g = gload(R.cgeo + c);
        v[0] = far_eval_f(g.x - tx[0], g.y - ty[0], g.z - tz[0], R.M32 + (size_t)c * MSTR);
        __builtin_amdgcn_sched_barrier(0);  // one recurrence's T_n in registers at a time
        v[1] = far_eval_f(g.x - tx[1], g.y - ty[1], g.z - tz[1], R.M32 + (size_t)c * MSTR);
        return;
    }
    far_rows<2>(grow(R.H + (size_t)c * HSTR), tx, ty, tz, v);
}

// sum_{s <= p} P_s(cos psi) |d|^s / |R|^(s+1), psi the angle between d and -R: the
// expansion of eq. 3.3 of one unit point source at c + d seen from c - R, order by
// order equal to sum_{|n| <= p} T_n(R) d^n.  With A_s = P_s(cos psi) |d|^s |R|^s,
// (s + 1) A_{s+1} = (2s + 1) (-d.R) A_s - s |d|^2 |R|^2 A_{s-1}.
__device__ __forceinline__ double point_expansion(double Rx, double Ry, double Rz, double dx, double dy, double dz) {
    const double r2 = Rx * Rx + Ry * Ry + Rz * Rz;
    const double ir = rsqrt_nr(r2);
    const double irr = ir * ir;
    const double c1 = -(dx * Rx + dy * Ry + dz * Rz);
    const double c2 = (dx * dx + dy * dy + dz * dz) * r2;
    double a0 = 1.0, a1 = c1;
    double sc = ir;               // |R|^-(2s+1)
    double v = a0 * sc;
    if (P >= 1) { sc *= irr; v = fma(a1, sc, v); }
#pragma unroll
    for (int s = 1; s < P; ++s) {
        const double a2 = fma((2.0 * s + 1.0) / (s + 1.0) * c1, a1, -((double)s / (s + 1.0) * c2) * a0);
        a0 = a1; a1 = a2;
        sc *= irr;
        v = fma(a1, sc, v);
    }
    return v;
}

// A double read from another lane of the same 16-lane row by a DPP control
// (two 32-bit moves), no memory traffic; every control used here has a source
// lane inside the row for every lane.
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_mov_dpp((int)b, CTRL, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), CTRL, 0xF, 0xF, true);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// Reduce-scatter over the 16 lanes of a row: before, every lane holds x[0..15];
// after, x[0] of lane l holds the row's sum of x[i(l)], with
// i(l) = b3 << 3 | (b0 ^ b2) << 2 | (b1 ^ b2) << 1 | b2 for the bits b_j of l in
// its row.  Four exchange stages with the partners l ^ 8, l ^ 1, l ^ 2 and
// l ^ 7 (DPP row_ror:8, two quad permutations, row_half_mirror); at each stage
// a lane keeps the half of its values that its partner does not keep and adds
// the partner's copy of that half.  15 exchanges instead of the 64 of sixteen
// row sums, and every lane ends with a distinct index.
template <int CTRL, int M>
__device__ __forceinline__ void rs_stage(double (&x)[16], bool up) {
#pragma unroll
    for (int j = 0; j < M / 2; ++j) {
        const double lo = x[j], hi = x[j + M / 2];
        x[j] = (up ? hi : lo) + dpp_f64<CTRL>(up ? lo : hi);
    }
}
__device__ __forceinline__ int rs_index(int l) {
    return (((l >> 3) & 1) << 3) | (((l ^ (l >> 2)) & 1) << 2) | ((((l >> 1) ^ (l >> 2)) & 1) << 1) | ((l >> 2) & 1);
}
__device__ __forceinline__ double row_reduce_scatter16(double (&x)[16], int l) {
    rs_stage<0x128, 16>(x, (l >> 3) & 1);
    rs_stage<0xB1, 8>(x, (l ^ (l >> 2)) & 1);
    rs_stage<0x4E, 4>(x, ((l >> 1) ^ (l >> 2)) & 1);
    rs_stage<0x141, 2>(x, (l >> 2) & 1);
    return x[0];
}
// Row sums of four values by the first two stages above and two plain sums:
// every lane gets the sum of value b3 << 1 | (b0 ^ b2), so lanes 0, 1, 8 and 9
// of the row hold the sums of a, b, c and d.
__device__ __forceinline__ double row_sum4_scatter(double a, double b, double c, double d, int l) {
    const bool u1 = (l >> 3) & 1;
    const double s0 = (u1 ? c : a) + dpp_f64<0x128>(u1 ? a : c);
    const double s1 = (u1 ? d : b) + dpp_f64<0x128>(u1 ? b : d);
    const bool u2 = (l ^ (l >> 2)) & 1;
    double v = (u2 ? s1 : s0) + dpp_f64<0xB1>(u2 ? s0 : s1);
    v += dpp_f64<0x4E>(v);
    v += dpp_f64<0x141>(v);
    return v;
}

// ------------------------------------------------------------ traversal state
constexpr uint32_t kCellMask = 0xFFFFFFu;
constexpr uint32_t kFlagIon = 1u << 28, kFlagImg = 1u << 29;

// base + the lanes below this one in the ballot b: two instructions, the addition with them
__device__ __forceinline__ int rank_below(uint64_t b, int base) {
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(b >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)b, (uint32_t)base));
}

// An opened cell's eight frontier entries (header ne for its first child; two 16-byte
// stores where the frontier is in LDS, whose places are multiples of eight); the children
// on the movers' root paths (digit dig_i, dig_k of 0..7, or -1) get their flag bits after.
__device__ __forceinline__ void put_children(uint32_t* lds, uint32_t* hbm, uint32_t ne, int dig_i, uint32_t bit_i,
                                             int dig_k, uint32_t bit_k) {
    if (hbm) {
#pragma unroll
        for (int d = 0; d < 8; ++d) hbm[d] = (ne + (uint32_t)d) | (d == dig_i ? bit_i : 0u) | (d == dig_k ? bit_k : 0u);
        return;
    }
    const uint32_t v[8] = {ne, ne + 1u, ne + 2u, ne + 3u, ne + 4u, ne + 5u, ne + 6u, ne + 7u};
    __builtin_memcpy(__builtin_assume_aligned(lds, 16), v, 16);
    __builtin_memcpy(__builtin_assume_aligned(lds + 4, 16), v + 4, 16);
    if (dig_i >= 0) lds[dig_i] |= bit_i;
    if (dig_k >= 0) lds[dig_k] |= bit_k;
}

// Frontier region of this workgroup in HBM (null if none): a level whose frontier
// outgrows its LDS capacity continues there, and so do the levels after it.
__device__ __forceinline__ uint32_t* spill_region(uint32_t* spill, int regions, long long words) {
    return (spill && (int)blockIdx.x < regions) ? spill + (size_t)blockIdx.x * (size_t)words : nullptr;
}

template <int NTG, int BLOCK>
struct Trav {
    static constexpr int FCAP = 4096;
    static constexpr int FARCAP = 1024 + BLOCK;
    static constexpr int NEARCAP = 512 + BLOCK;
    static constexpr int OVLCAP = 256;
    static constexpr int NW = BLOCK / 64;
    static constexpr int OWNCAP = 2048;  // slots of the near leaves listed one by one
    // the lists, free once the traversal has ended: then the commit's table of harmonics
    static constexpr int LISTWORDS = 2 * FCAP + FARCAP + 3 * NEARCAP + 1;
    static constexpr int HROWS = (LISTWORDS / 2) / NH;
    union {
        struct {
            alignas(16) uint32_t front[2][FCAP];
            uint32_t farl[FARCAP];
            uint32_t nearl[NEARCAP];
            int near_base[NEARCAP];
            int near_pre[NEARCAP + 1];       // slot counts, then their exclusive prefix
        };
        double hrow[HROWS][NH];
    };
    uint16_t near_own[OWNCAP];       // near list entry of each of its slots
    uint32_t flagl[2 * NTG];
    double tx[NTG], ty[NTG], tz[NTG];
    int ex_i[NTG], ex_k[NTG];
    uint64_t kx_i[NTG], kx_k[NTG];
    double4 es_i[NTG], es_k[NTG];
    uint32_t ovl[OVLCAP];
    int n_ovl, ovl_t, ovl_ex;
    int near_tot;                    // slot total of the near leaves, from a one-wave scan
    int err, overlap, coincide;
    uint64_t wcnt[2][NW];            // per-wave packed list counts, double buffered
    uint64_t wsum[NW + 1];
    double red[NW][NTG];
    double res[NTG];
    uint32_t mi[NTERM];              // multi-index of each term, packed (mi_code)
    HTab ht;                         // tables of the regular harmonics
};

template <int NTG, int BLOCK>
__device__ __forceinline__ void fill_mi(Trav<NTG, BLOCK>& S) {
    for (int k = threadIdx.x; k < NTERM; k += BLOCK) S.mi[k] = mi_code(k);
    fill_htab(S.ht);
}

template <int NTG>
__device__ __forceinline__ void add_to(double (&acc)[NTG], int t, double v) {
#pragma unroll
    for (int k = 0; k < NTG; ++k)
        if (k == t) acc[k] += v;
}

// Value at (x, y, z) of far cell c without the excluded sources it holds (a flagged cell):
// its value less their own expansions about its centre, in FP64 also where the other far
// cells are taken in single precision (then from the moments, which that replica's commits
// repair in place of its expansion rows).  Out of line: a traversal has a few of these per
// target, and the far loop keeps its registers.
template <bool F32>
__device__ __attribute__((noinline)) double flagged_value(const Rep& R, int c, double x, double y, double z, bool ion,
                                                          double4 si, bool img, double4 sk) {
    const double4 g = gload(R.cgeo + c);
    double v;
    if (F32 && R.M32) v = cart_eval<false>(g.x - x, g.y - y, g.z - z, grow(R.M + (size_t)c * MSTR));
    else v = far_row(grow(R.H + (size_t)c * HSTR), x, y, z);
    if (ion) v -= si.w * point_expansion(g.x - x, g.y - y, g.z - z, si.x - g.x, si.y - g.y, si.z - g.z);
    if (img) v -= sk.w * point_expansion(g.x - x, g.y - y, g.z - z, sk.x - g.x, sk.y - g.y, sk.z - g.z);
    return v;
}

// Prefix counts of a chunk's lists over its N <= 16 (part, wave) counts, four 16-bit fields
// each (no field overflows: a chunk has at most 1024 entries).  Every 16-lane row scans a copy
// of the counts by DPP, a 32-bit add a step for two fields, and a wave reads its own place and
// the totals from there into scalar registers; summing the counts in every thread took about
// 100 vector instructions a chunk.
template <int N>
struct ChunkScan {
    uint32_t lo, hi;
    __device__ __forceinline__ explicit ChunkScan(const uint64_t* cnt) {
        static_assert(N <= 16, "a row of lanes holds the counts");
        const int j = lane_id() & 15;
        const uint64_t v = j < N ? cnt[j] : 0ull;
        lo = (uint32_t)v; hi = (uint32_t)(v >> 32);
#define BHMC_SCAN_STEP(CTRL)                                                              \
        lo += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)lo, CTRL, 0xF, 0xF, false);   \
        hi += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)hi, CTRL, 0xF, 0xF, false);
        BHMC_SCAN_STEP(0x111) BHMC_SCAN_STEP(0x112) BHMC_SCAN_STEP(0x114) BHMC_SCAN_STEP(0x118)  // row_shr 1, 2, 4, 8
#undef BHMC_SCAN_STEP
    }
    // counts of the first k places (k uniform), packed as the counts are
    __device__ __forceinline__ uint64_t before(int k) const {
        if (k == 0) return 0ull;
        return ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)hi, k - 1) << 32) |
               (uint32_t)__builtin_amdgcn_readlane((int)lo, k - 1);
    }
};

// The near list entry of flattened slot f: the last j with pre[j] <= f.
__device__ __forceinline__ int near_search(const int* pre, int near_n, int f) {
    int lo = 0, hi = near_n - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (pre[mid] <= f) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// The same for every slot at once, where they fit: each entry writes its number to its
// slots, so a slot finds it in one read instead of a search of dependent reads.  Entries of more
// than 64 slots on average (leaf capacities in use are 8 to 32) are left to the search: a lane
// would write an entry's slots one after another, all of them where a system is one leaf.
__device__ __forceinline__ bool near_listed(int near_n, int total, int cap) { return total <= cap && total <= 64 * near_n; }
template <int BLOCK>
__device__ __forceinline__ void near_list(uint16_t* own, const int* pre, int near_n, int total, int cap) {
    if (!near_listed(near_n, total, cap)) return;  // uniform
    for (int j = threadIdx.x; j < near_n; j += BLOCK) {
        const int end = j + 1 < near_n ? pre[j + 1] : total;
        for (int f = pre[j]; f < end; ++f) own[f] = (uint16_t)j;
    }
}

// Exclusive scan of the near leaves' slot counts (in place in near_pre).  Up to
// 64 leaves (the usual case) the first wave scans them by shuffles and one
// barrier publishes the result; beyond that, block scans of BLOCK at a time.
template <int NTG, int BLOCK>
__device__ int near_scan(Trav<NTG, BLOCK>& S, int near_n) {
    if (near_n <= 64) {  // uniform
        if (threadIdx.x < 64) {
            const int j = threadIdx.x;
            const int v = j < near_n ? S.near_pre[j] : 0;
            int x = v;
#pragma unroll
            for (int off = 1; off < 64; off <<= 1) {
                const int y = __shfl_up(x, off, 64);
                if (j >= off) x += y;
            }
            if (j < near_n) S.near_pre[j] = x - v;
            if (j == 63) S.near_tot = x;
        }
        __syncthreads();
        return S.near_tot;
    }
    int carry = 0;
    for (int base = 0; base < near_n; base += BLOCK) {
        const int j = base + threadIdx.x;
        const int v = j < near_n ? S.near_pre[j] : 0;
        uint64_t tot;
        const uint64_t ex = block_exscan<BLOCK>((uint64_t)v, S.wsum, tot);
        if (j < near_n) S.near_pre[j] = carry + (int)ex;
        carry += (int)tot;
        __syncthreads();
    }
    return carry;
}

// squared distance from a point to the closed cube of centre g and half side g.w
__device__ __forceinline__ double box_dist2(double4 g, double x, double y, double z) {
    double ax = fabs(x - g.x) - g.w, ay = fabs(y - g.y) - g.w, az = fabs(z - g.z) - g.w;
    ax = ax > 0.0 ? ax : 0.0; ay = ay > 0.0 ? ay : 0.0; az = az > 0.0 ? az : 0.0;
    return ax * ax + ay * ay + az * az;
}

// Hard-core check below cells the traversal took as far: descend every cell
// whose cube comes within tau (plus a rounding margin) of the target.
template <int NTG, int BLOCK>
__device__ void overlap_below_far(const RepU& R, Trav<NTG, BLOCK>& S, int* cnt2) {
    using TS = Trav<NTG, BLOCK>;
    const int t = S.ovl_t;
    const double x = S.tx[t], y = S.ty[t], z = S.tz[t];
    const double reach2 = R.reach2;
    // n_ovl counts every insert attempt; entries past OVLCAP were never stored
    int cur = 0, fs = S.n_ovl < TS::OVLCAP ? S.n_ovl : TS::OVLCAP;
    for (int j = threadIdx.x; j < fs; j += BLOCK) S.front[0][j] = S.ovl[j];
    while (fs > 0) {
        if (threadIdx.x == 0) cnt2[cur ^ 1] = 0;
        __syncthreads();
        for (int j = threadIdx.x; j < fs; j += BLOCK) {
            const int c = (int)S.front[cur][j];
            if (c < 0 || c >= R.ncell) { S.err = kErrOvlLeaf; continue; }
            const int4 m = R.cm[c];
            if (m.y >= 0 && m.y + 8 > R.ncell) { S.err = kErrChildLink; continue; }
            if (m.y < 0) {
                if (m.x < 0 || m.z < 0 || m.z + m.x > R.pool) { S.err = kErrOvlLeaf; continue; }
                for (int k = 0; k < m.x; ++k) {
                    const int sid = R.pidx[m.z + k];
                    if (sid >= R.n || sid == S.ovl_ex) continue;
                    const double4 s = R.pool4[m.z + k];
                    const double dx = x - s.x, dy = y - s.y, dz = z - s.z;
                    if (dx * dx + dy * dy + dz * dz <= R.tau2) S.overlap = 1;
                }
            } else {
                for (int d = 0; d < 8; ++d) {
                    const int ch = m.y + d;
                    if (R.cm[ch].x == 0) continue;
                    if (box_dist2(R.cgeo[ch], x, y, z) <= reach2) {
                        const int slot = atomicAdd(&cnt2[cur ^ 1], 1);
                        if (slot < TS::FCAP) S.front[cur ^ 1][slot] = (uint32_t)ch;
                        else S.err = kErrStack;
                    }
                }
            }
        }
        __syncthreads();
        fs = cnt2[cur ^ 1];
        if (fs > TS::FCAP) fs = TS::FCAP;
        cur ^= 1;
        __syncthreads();
    }
}

// ------------------------------------------------------------ the move traversal
// The two targets of a move (the mover's old and new position) exclude the
// same two sources, so they share every frontier entry: a cell with a 2-bit
// mask of the targets for which it is still open (bits 24-25), a 2-bit mask of
// the targets summing every source below it directly by the N_0 rule (bits
// 26-27) and the two exclusion flags.  Each target takes exactly the decisions
// of its own traversal.  A lane reads a far cell's row once and evaluates both
// targets from it, and likewise near sources.
constexpr int kMaskSh = 24, kDirSh = 26;

template <bool F32, int BLOCK>
__device__ __forceinline__ void far_pass_mc(const RepU& R, Trav<2, BLOCK>& S, int far_n, int nflag,
                                            double (&acc)[2]) {
    const int t = (int)(threadIdx.x & 1);
    if (F32 && kF32Apart<BLOCK> && R.M32) {
        for (int j2 = threadIdx.x; j2 < 2 * far_n; j2 += BLOCK) {
            const uint32_t e = S.farl[j2 >> 1];
            if (!((e >> (kMaskSh + t)) & 1u)) continue;
            const int c = (int)(e & kCellMask);
            if (c >= R.ncell) { S.err = kErrFarCell; continue; }
            const double4 g = gload(R.cgeo + c);
            add_to<2>(acc, t, far_eval_f(g.x - S.tx[t], g.y - S.ty[t], g.z - S.tz[t], R.M32 + (size_t)c * MSTR));
        }
    } else {
        for (int j = threadIdx.x; j < far_n; j += BLOCK) {
            const uint32_t e = S.farl[j];
            const int c = (int)(e & kCellMask);
            if (c >= R.ncell) { S.err = kErrFarCell; continue; }
            const double tx[2] = {S.tx[0], S.tx[1]}, ty[2] = {S.ty[0], S.ty[1]}, tz[2] = {S.tz[0], S.tz[1]};
            double v[2];
            far_value2<F32 && !kF32Apart<BLOCK>>(R, c, tx, ty, tz, v);
            acc[0] += ((e >> kMaskSh) & 1u) ? v[0] : 0.0;
            acc[1] += ((e >> kMaskSh) & 2u) ? v[1] : 0.0;
        }
    }
    // the cells holding an excluded source, less what it adds: a lane per target
    for (int j2 = threadIdx.x; j2 < 2 * nflag; j2 += BLOCK) {
        const uint32_t e = S.flagl[j2 >> 1];
        if (!((e >> (kMaskSh + t)) & 1u)) continue;
        const int c = (int)(e & kCellMask);
        if (c >= R.ncell) { S.err = kErrFarCell; continue; }
        add_to<2>(acc, t, flagged_value<F32>(R, c, S.tx[t], S.ty[t], S.tz[t], e & kFlagIon, S.es_i[0], e & kFlagImg,
                                        S.es_k[0]));
    }
}

// Near leaves of both targets.  For the new position (the overlap target),
// every ion other than the mover within tau is an overlap.
template <int BLOCK>
__device__ __forceinline__ void near_pass_mc(const RepU& R, Trav<2, BLOCK>& S, int near_n, int total,
                                             double (&acc)[2]) {
    const int n_ion = R.n;
    const bool listed = near_listed(near_n, total, Trav<2, BLOCK>::OWNCAP);  // uniform
    for (int f = threadIdx.x; f < total; f += BLOCK) {
        const int lo = listed ? (int)S.near_own[f] : near_search(S.near_pre, near_n, f);
        const uint32_t e = S.nearl[lo];
        const uint32_t mask = (e >> kMaskSh) & 3u;
        const int slot = S.near_base[lo] + (f - S.near_pre[lo]);
        const double4 s = gload(R.pool4 + slot);
        int sid = -1;
        if ((e & (kFlagIon | kFlagImg)) || (mask & 2u)) {
            sid = gload(R.pidx + slot);
            if (((e & kFlagIon) && sid == S.ex_i[0]) || ((e & kFlagImg) && sid == S.ex_k[0])) continue;
        }
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            if (!((mask >> t) & 1u)) continue;
            const double dx = S.tx[t] - s.x, dy = S.ty[t] - s.y, dz = S.tz[t] - s.z;
            const double d2 = dx * dx + dy * dy + dz * dz;
            if (t == 1 && sid < n_ion && sid != S.ovl_ex && d2 <= R.tau2) S.overlap = 1;
            if (d2 == 0.0) { S.coincide = 1; continue; }
            add_to<2>(acc, t, s.w * rsqrt_nr(d2));
        }
    }
}

// Breadth-first MAC traversal (Sec. 3.2) of the two targets of a move from
// the fs0 entries of level level0 in front[0].  A level is taken BLOCK entries at a
// time: every lane classifies one, and ballots and one barrier hand out places in the
// far, near and flagged lists and the next frontier in the order of the entries, so
// every list, and with it every sum, is the same from run to run.  Full lists are
// evaluated on the way, what is left at the end.  A frontier lives in LDS up to lcap
// entries; a level that outgrows them moves to the workgroup's HBM region, what it has
// written so far first, and the levels after it stay there.  hook(level) is called once
// a level.  On return res[0..1] are the potentials (the same in every thread); S.err is
// 0 or the check that failed (kErrFrontier: no room for a frontier, kErrStack: another
// list; then res is not set); S.overlap: an ion other than the mover within tau of the
// new position; S.coincide: a source at a target.
template <bool F32, int BLOCK, class Hook>
__device__ int traverse_mc(const RepU& R, Trav<2, BLOCK>& S, int* cnt2, Hook&& hook, int fs0, int level0,
                           double (&res)[2]) {
    using TS = Trav<2, BLOCK>;
    res[0] = res[1] = 0.0;
    constexpr int NW = TS::NW;
    const int tid = threadIdx.x, lane = lane_id(), w = wave_id();
    double acc[2] = {0.0, 0.0};
    int cur = 0, fs = fs0, far_n = 0, near_n = 0, nflag = 0, buf = 0;
    bool failed = false, frontier_full = false;
    uint32_t* const gfr = spill_region(R.spill, R.spill_regions, R.spill_words);
    const int gcap = gfr ? (int)(R.spill_words / 2 < 0x7FFFFFFF ? R.spill_words / 2 : 0x7FFFFFFF) : 0;
    const int lcap = R.fcap < TS::FCAP ? R.fcap : TS::FCAP;
    bool rg = false, wg = false;
    int level = level0;
    for (; fs > 0 && !failed; ++level) {
        int next_n = 0;
        for (int base = 0; base < fs; base += BLOCK) {
            if (far_n > TS::FARCAP - BLOCK) {
                __syncthreads();
                far_pass_mc<F32, BLOCK>(R, S, far_n, 0, acc);
                far_n = 0;
                __syncthreads();
            }
            if (near_n > TS::NEARCAP - BLOCK) {
                __syncthreads();
                const int total = near_scan<2, BLOCK>(S, near_n);
                near_list<BLOCK>(S.near_own, S.near_pre, near_n, total, TS::OWNCAP);
                __syncthreads();
                near_pass_mc<BLOCK>(R, S, near_n, total, acc);
                near_n = 0;
                __syncthreads();
            }
            const int j = base + tid;
            const bool valid = j < fs;
            const uint32_t e = valid ? (rg ? gfr[(size_t)cur * gcap + j] : S.front[cur][j]) : 0u;
            const int c = (int)(e & kCellMask);
            const int fi = (e & kFlagIon) ? 1 : 0, fk = (e & kFlagImg) ? 1 : 0;
            const uint32_t open = (e >> kMaskSh) & 3u, dir = (e >> kDirSh) & 3u;
            int4 m = make_int4(0, -1, 0, 0);
            double4 g = make_double4(0.0, 0.0, 0.0, 0.0);
            if (valid && c < R.ncell) { m = gload(R.cm + c); g = gload(R.cgeo + c); }
            // once per level, in the shadow of the loads just issued
            if (base == 0) hook(level);
            uint32_t farb = 0, nearb = 0, copen = 0, cdir = 0;
            if (valid && c >= R.ncell) {
                S.err = kErrFrontCell;
            } else if (valid) {
                const int np = m.x - fi - fk;
                if (m.y >= 0 && m.y + 8 > R.ncell) {
                    S.err = kErrChildLink;
                } else if (np > 0) {
                    // both targets' tests side by side, then the decisions as bit masks
                    const double dx0 = g.x - S.tx[0], dy0 = g.y - S.ty[0], dz0 = g.z - S.tz[0];
                    const double dx1 = g.x - S.tx[1], dy1 = g.y - S.ty[1], dz1 = g.z - S.tz[1];
                    const double d20 = dx0 * dx0 + dy0 * dy0 + dz0 * dz0;
                    const double d21 = dx1 * dx1 + dy1 * dy1 + dz1 * dz1;
                    const double h2 = 3.0 * (g.w * g.w);
                    const uint32_t mac = (h2 <= R.theta2 * d20 ? 1u : 0u) | (h2 <= R.theta2 * d21 ? 2u : 0u);
                    const bool internal = m.y >= 0;
                    const uint32_t live = open & ~dir;
                    farb = live & mac & (np >= R.n0 ? 3u : 0u);
                    const uint32_t rest = live & ~farb;
                    copen = rest & ((np > R.n0 && internal) ? 3u : 0u);
                    nearb = (rest & ~copen & (internal ? 0u : 3u)) | (dir & (internal ? 0u : 3u));
                    cdir = (rest & ~copen & (internal ? 3u : 0u)) | (dir & (internal ? 3u : 0u));
                    if ((farb & 2u) && d21 <= R.ovl2 && S.ovl_t == 1 && box_dist2(g, S.tx[1], S.ty[1], S.tz[1]) <= R.reach2) {
                        const int slot = atomicAdd(&S.n_ovl, 1);
                        if (slot < TS::OVLCAP) S.ovl[slot] = (uint32_t)c; else S.err = kErrStack;
                    }
                }
            }
            const bool flagged = (fi | fk) != 0;
            const bool kf = farb && !flagged, kg = farb && flagged, kn = nearb != 0, ks = (copen | cdir) != 0;
            const uint64_t bf = __ballot(kf), bn = __ballot(kn), bs = __ballot(ks), bg = __ballot(kg);
            if (lane == 0)
                S.wcnt[buf][w] = (uint64_t)__popcll(bf) | ((uint64_t)__popcll(bn) << 16) |
                                 ((uint64_t)__popcll(bs) << 32) | ((uint64_t)__popcll(bg) << 48);
            __syncthreads();
            const ChunkScan<NW> scan(S.wcnt[buf]);
            const uint64_t before = scan.before(uni(w)), tot = scan.before(NW);
            buf ^= 1;
            const int tf = (int)(tot & 0xffff), tn = (int)((tot >> 16) & 0xffff);
            const int ts = (int)((tot >> 32) & 0xffff), tg = (int)(tot >> 48);
            if (nflag + tg > 4) {  // uniform
                failed = true;
                break;
            }
            if (next_n + 8 * ts > (wg ? gcap : lcap)) {  // uniform
                if (wg || next_n + 8 * ts > gcap) {
                    failed = frontier_full = true;
                    break;
                }
                for (int k = tid; k < next_n; k += BLOCK) gfr[(size_t)(cur ^ 1) * gcap + k] = S.front[cur ^ 1][k];
                wg = true;
            }
            const uint32_t flags = e & (kFlagIon | kFlagImg);
            if (kf) S.farl[rank_below(bf, far_n + (int)(before & 0xffff))] = (uint32_t)c | (farb << kMaskSh);
            if (kg) S.flagl[rank_below(bg, nflag + (int)(before >> 48))] = (uint32_t)c | (farb << kMaskSh) | flags;
            if (kn) {
                const int o = rank_below(bn, near_n + (int)((before >> 16) & 0xffff));
                S.nearl[o] = (uint32_t)c | (nearb << kMaskSh) | flags;
                S.near_base[o] = m.z;
                S.near_pre[o] = m.x;
                if (m.x < 0 || m.z < 0 || m.z + m.x > R.pool) { S.near_pre[o] = 0; S.err = kErrNearSlots; }
            }
            if (ks) {
                const int o = next_n + 8 * rank_below(bs, (int)((before >> 32) & 0xffff));
                const int dig_i = fi ? key_digit(S.kx_i[0], level + 1) : -1;
                const int dig_k = fk ? key_digit(S.kx_k[0], level + 1) : -1;
                const uint32_t masks = (copen << kMaskSh) | (cdir << kDirSh);
                put_children(&S.front[cur ^ 1][wg ? 0 : o], wg ? gfr + (size_t)(cur ^ 1) * gcap + o : nullptr,
                             (uint32_t)m.y | masks, dig_i, kFlagIon, dig_k, kFlagImg);
            }
            far_n += tf; near_n += tn; nflag += tg; next_n += 8 * ts;
        }
        __syncthreads();  // the next level reads what this one wrote
        cur ^= 1;
        fs = next_n;
        rg = wg;
    }
    if (failed) {
        if (tid == 0) S.err = frontier_full ? kErrFrontier : kErrStack;
        __syncthreads();
        return level;
    }
    const int total = near_scan<2, BLOCK>(S, near_n);
    near_list<BLOCK>(S.near_own, S.near_pre, near_n, total, TS::OWNCAP);
    far_pass_mc<F32, BLOCK>(R, S, far_n, nflag, acc);
    __syncthreads();  // publishes near_own
    near_pass_mc<BLOCK>(R, S, near_n, total, acc);
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const double sum = wave_sum(acc[k]);
        if (lane == 0) S.red[w][k] = sum;
    }
    __syncthreads();
    if (S.ovl_t >= 0 && S.n_ovl > 0 && S.err == 0) overlap_below_far<2, BLOCK>(R, S, cnt2);
    // every thread sums the wave sums itself, in the same order
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        double sum = 0.0;
        for (int ww = 0; ww < NW; ++ww) sum += S.red[ww][k];
        res[k] = sum;
    }
    return level;
}

// What a unit source at sc adds to the potential at (x, y, z) through the tree when
// the traversal keeps it as an ordinary source (N_0 = 0): walk its root path from the
// top; the first cell passing the MAC takes it through its expansion, otherwise its
// leaf takes it directly.  bad is set (and 0 returned) where a link is broken.
__device__ __forceinline__ double walk_value(const Rep& R, double4 sc, double x, double y, double z, int& bad) {
    const uint64_t key = morton_key(R, sc.x, sc.y, sc.z);
    int c = 0;
    for (int level = 0; level < kMaxLevels; ++level) {
        if (c < 0 || c >= R.ncell) break;
        const double4 g = R.cgeo[c];
        const double dx = g.x - x, dy = g.y - y, dz = g.z - z;
        const double d2 = dx * dx + dy * dy + dz * dz;
        if (3.0 * (g.w * g.w) <= R.theta2 * d2) return point_expansion(dx, dy, dz, sc.x - g.x, sc.y - g.y, sc.z - g.z);
        const int link = R.cm[c].y;
        if (link < 0) {
            const double ex = x - sc.x, ey = y - sc.y, ez = z - sc.z;
            return rsqrt_nr(ex * ex + ey * ey + ez * ez);
        }
        if (link + 8 > R.ncell) break;
        c = link + key_digit(key, level + 1);
    }
    bad = 1;
    return 0.0;
}

// ------------------------------------------------------------ one Monte Carlo move
constexpr int kMaxPathCells = 4 * kMaxLevels;
constexpr int kLineContrib = 16;  // old and new position of up to 8 line images of the mover
constexpr int kPowCells = 24;  // longer path-cell lists build their monomials by repeated products
constexpr int kDrawBatch = 64;  // trial moves drawn ahead at once, one per lane of the first wave

struct McShared {
    int path[4][kMaxLevels];  // root paths: ion old, ion new, image old, image new
    double4 path_geo[4][kMaxLevels];  // geometry of each path cell, read with its link
    int plen[4];
    int fs0, level0;          // where the move traversal starts
    uint64_t key[4];
    double4 contrib[4];       // (position, charge) of the four contributions
    double alpha;             // the move's Metropolis uniform
    // commit state gathered while the traversal runs
    int2 tr[2];               // tracking (leaf cell, slot) of the ion and of its image
    int4 lm_old[2];           // (count, link, base, cap) of their leaves
    int4 lm_new[2];           // same for the leaves of their new positions
    int last_pidx[2];         // source in the last slot of each old leaf
    double4 last_pool[2];     // and its (x, y, z, q)
    int self_pidx[2];         // source found at the tracked slot (must be the mover)
    int pf_stage[2];
    // distinct cells of the four root paths with the contributions they take
    int nlist;
    int list_cell[kMaxPathCells];
    int list_mask[kMaxPathCells];   // bit jj: contribution jj applies; bit 4: internal cell
    int list_lev[kMaxPathCells];
    double4 list_geo[kMaxPathCells];
    int ok;
    int err;
    int cnt2[2];
    // the next trial moves (index, dx, dy, dz, alpha), and the next mover's ion and image as
    // loaded while the current move's traversal runs
    int dr_i[kDrawBatch];
    double dr_d[kDrawBatch][4];
    double4 nx_si, nx_mo;
    // powers 0..p of each contribution's offset from each of the first kPowCells list cells,
    // per axis: d^n = x^n1 y^n2 z^n3 by two products
    double pw[kPowCells][4][3][P + 1];
    // the mover's line images (multiple-image model): old (2m) and new (2m + 1) position and
    // charge of line image m, the root paths of both, descended beside the traversal; for each
    // old one and each target the first path cell passing the MAC (level, or -1: its leaf sums
    // it directly; and its geometry); each new leaf's count and capacity
    double4 lpos[kLineContrib];
    double4 lmac_geo[kLineContrib / 2][2];
    uint64_t lkey[kLineContrib];
    int lpath[kLineContrib][kMaxLevels];
    int lplen[kLineContrib];
    int lmac[kLineContrib / 2][2];
    int lcnt[kLineContrib / 2], lcap[kLineContrib / 2];
    int lnext[kLineContrib];  // next level of each line path; -1 before its position is read
};

struct MoveOut { double dE; int reason; int accepted; int stop; int detail; };

constexpr double kInf = __builtin_huge_val();

// One stage of the commit prefetch for old source j (0: ion, 1: image).
__device__ __forceinline__ void prefetch_stage(const RepU& R, McShared& MS, int j, int s) {
    const int stage = MS.pf_stage[j];
    if (stage == 0) {
        const int2 t = gload(R.track + s);
        MS.tr[j] = t;
        MS.pf_stage[j] = (t.x >= 0 && t.x < R.ncell) ? 1 : 9;
    } else if (stage == 1) {
        const int4 m = gload(R.cm + MS.tr[j].x);
        MS.lm_old[j] = m;
        const bool sane = m.y < 0 && m.x >= 1 && m.z >= 0 && m.z + m.x <= R.pool && m.x <= m.w &&
                          MS.tr[j].y >= 0 && MS.tr[j].y < m.x;
        MS.pf_stage[j] = sane ? 2 : 9;
    } else if (stage == 2) {
        const int4 m = MS.lm_old[j];
        MS.last_pidx[j] = gload(R.pidx + m.z + m.x - 1);
        MS.last_pool[j] = gload(R.pool4 + m.z + m.x - 1);
        MS.self_pidx[j] = gload(R.pidx + m.z + MS.tr[j].y);
        MS.pf_stage[j] = 3;
    }
}

// ------------------------------------------------------------ line images of the mover
// The multiple-image model gives each ion M line-image sources (2n + m n + i) besides
// its Kelvin image.  A move keeps the mover's own line images in its traversal as
// ordinary sources.  Beside the traversal, lanes of an otherwise idle wave descend the
// root paths of their old and new positions (line_step), noting for each old one the
// first cell that passes the MAC for each target; afterwards each is taken back out of
// both potentials where the traversal met it (line_corrections), every leaf an accepted
// move fills is checked in commit order, and the line images are moved after the ion and
// its image, in source order, by the local modification of Sec. 3.3 (lines_commit).

// One step of line contribution j's root path (j = 2m: old position of line image m,
// 2m + 1: new), as the ion's own paths descend.
__device__ __forceinline__ void line_step(const Rep& R, McShared& MS, const double* tx, const double* ty,
                                          const double* tz, int j, int level, int i) {
    const int c = MS.lpath[j][level];
    const bool cok = c >= 0 && c < R.ncell;
    const bool old = (j & 1) == 0;
    int4 m = make_int4(0, -1, 0, 0);
    double4 g = make_double4(0.0, 0.0, 0.0, 0.0);
    if (cok) {
        m = gload(R.cm + c);
        if (old) g = gload(R.cgeo + c);
    }
    if (!cok || (m.y >= 0 && m.y + 8 > R.ncell)) {
        MS.err = kErrPathCell;
        MS.lplen[j] = level + 1;
        MS.lpath[j][level] = 0;
        return;
    }
    if (old) {
        const int mm = j >> 1;
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            if (MS.lmac[mm][t] >= 0) continue;
            const double dx = g.x - tx[t], dy = g.y - ty[t], dz = g.z - tz[t];
            const double d2 = dx * dx + dy * dy + dz * dz;
            if (3.0 * (g.w * g.w) <= R.theta2 * d2) { MS.lmac[mm][t] = level; MS.lmac_geo[mm][t] = g; }
        }
    }
    if (m.y >= 0 && level + 1 < kMaxLevels) {
        MS.lpath[j][level + 1] = m.y + key_digit(MS.lkey[j], level + 1);
        return;
    }
    if (m.y >= 0) MS.err = kErrPathDepth;
    MS.lplen[j] = level + 1;
    if (!old) {
        MS.lcnt[j >> 1] = m.x;
        MS.lcap[j >> 1] = m.w;
        if (m.z < 0 || m.x < 0 || m.z + m.w > R.pool) MS.err = kErrCommitLeaf;
    } else if (gload(R.track + (2 * R.n + (j >> 1) * R.n + i)).x != c) {
        MS.err = kErrCommitSlot;  // the tracked leaf must be the one the old position's key leads to
    }
}

// Up to nsteps steps of line contribution j = tl's root path, its position read (old) or
// placed as the build places it from the new Kelvin image (new) on the first call.  The
// lane's state lives in LDS, so nothing of it stays in registers across the traversal.
__device__ __attribute__((noinline)) void line_lane_steps(const Rep& R, McShared& MS, const double* tx,
                                                          const double* ty, const double* tz, int tl, int i,
                                                          int nsteps) {
    int level = MS.lnext[tl];
    if (level < 0) {
        const int m = tl >> 1;
        double4 p;
        if (tl & 1) {
            const double4 k = MS.contrib[3];
            p = make_double4(R.line_t[m] * k.x, R.line_t[m] * k.y, R.line_t[m] * k.z, R.line_c[m] * k.w);
        } else {
            p = gload(R.src + (2 * R.n + m * R.n + i));
        }
        MS.lpos[tl] = p;
        MS.lkey[tl] = morton_key(R, p.x, p.y, p.z);
        level = 0;
    }
    for (int k = 0; k < nsteps && MS.lplen[tl] == 0 && level < kMaxLevels; ++k) line_step(R, MS, tx, ty, tz, tl, level++, i);
    MS.lnext[tl] = level;
}

// What the mover's own line images added to the potential at target t, from the paths
// descended beside the traversal: line image m through the expansion of the first cell of
// its root path that passes the MAC, else directly at its leaf.  Lanes 2m + t of every
// wave compute it, so each wave holds the sums without a barrier.
__device__ __attribute__((noinline)) void line_corrections(const Rep& R, const McShared& MS, double& c0, double& c1) {
    const int lane = lane_id(), t = lane & 1, m = lane >> 1;
    double v = 0.0;
    if (m < R.nline) {
        const double4 sc = MS.lpos[2 * m], x = MS.contrib[t];
        const int l = MS.lmac[m][t];
        if (l >= 0) {
            const double4 g = MS.lmac_geo[m][t];
            v = sc.w * point_expansion(g.x - x.x, g.y - x.y, g.z - x.z, sc.x - g.x, sc.y - g.y, sc.z - g.z);
        } else {
            const double ex = x.x - sc.x, ey = x.y - sc.y, ez = x.z - sc.z;
            v = sc.w * rsqrt_nr(ex * ex + ey * ey + ez * ez);
        }
    }
    c0 = wave_sum(t == 0 ? v : 0.0);
    c1 = wave_sum(t == 1 ? v : 0.0);
}

// Would the 2 + M insertions of this move (ion, Kelvin image, line images in source
// order) overflow a leaf?  Each new leaf is checked with the counts the earlier ones
// leave behind.
__device__ __forceinline__ int fit_old_leaf(const McShared& MS, int k) {
    return k == 0 ? MS.tr[0].x : (k == 1 ? MS.tr[1].x : MS.lpath[2 * (k - 2)][MS.lplen[2 * (k - 2)] - 1]);
}
__device__ __forceinline__ int fit_new_leaf(const McShared& MS, int k) {
    return k < 2 ? MS.path[2 * k + 1][MS.plen[2 * k + 1] - 1] : MS.lpath[2 * (k - 2) + 1][MS.lplen[2 * (k - 2) + 1] - 1];
}
__device__ __attribute__((noinline)) bool lines_fit(const Rep& R, const McShared& MS) {
    for (int k = 0; k < 2 + R.nline; ++k) {
        const int lo = fit_old_leaf(MS, k), ln = fit_new_leaf(MS, k);
        if (ln == lo) continue;
        int c = k < 2 ? MS.lm_new[k].x : MS.lcnt[k - 2];
        const int cap = k < 2 ? MS.lm_new[k].w : MS.lcap[k - 2];
        for (int e = 0; e < k; ++e) {
            const int eo = fit_old_leaf(MS, e), en = fit_new_leaf(MS, e);
            if (en == eo) continue;
            if (en == ln) c += 1;
            if (eo == ln) c -= 1;
        }
        if (c + 1 > cap) return false;
    }
    return true;
}

// Distinct cells of the 2M line paths, built in the frontier buffer (free after the
// traversal): bit j of a cell's mask = contribution j applies; kLineInternal = not a leaf.
struct LineList {
    int nlist;
    int cell[kLineContrib * kMaxLevels];
    uint32_t mask[kLineContrib * kMaxLevels];
    uint8_t lev[kLineContrib * kMaxLevels];
    int row0[kLineContrib];  // first table row of each path
    int pad;
};
static_assert(sizeof(LineList) % 8 == 0, "the table of harmonics follows the list");
constexpr uint32_t kLineInternal = 1u << 16;

template <int BLOCK>
__device__ __forceinline__ LineList& line_list(Trav<2, BLOCK>& S) {
    static_assert(sizeof(LineList) <= sizeof(S.front), "the line-path cell list must fit the frontier buffer");
    return *reinterpret_cast<LineList*>(&S.front[0][0]);
}
// the table of the line paths' harmonics after it, in the rest of the list space
template <int BLOCK>
constexpr int kLineRows = (int)((sizeof(Trav<2, BLOCK>::hrow) - sizeof(LineList)) / (8 * NH));

// Move one line image between leaf index arrays (or rewrite its slot) from the current
// state in HBM; false on a broken index.
__device__ __forceinline__ bool line_slot_move(const RepU& R, int s, int lo, int ln, double4 pn) {
    const int2 tr = R.track[s];
    const int4 mo = R.cm[lo];
    if (tr.x != lo || mo.y >= 0 || tr.y < 0 || tr.y >= mo.x || mo.z < 0 || mo.z + mo.x > R.pool) return false;
    if (ln != lo) {
        const int last = mo.x - 1, k = tr.y;
        const int4 mn = R.cm[ln];
        if (mn.y >= 0 || mn.x < 0 || mn.x + 1 > mn.w || mn.z < 0 || mn.z + mn.w > R.pool) return false;
        if (k != last) {
            const int moved = R.pidx[mo.z + last];
            if (moved < 0 || moved >= R.nsrc) return false;
            R.pool4[mo.z + k] = R.pool4[mo.z + last];
            R.pidx[mo.z + k] = moved;
            R.track[moved] = make_int2(lo, k);
        }
        R.cm[lo].x = last;
        R.pool4[mn.z + mn.x] = pn;
        R.pidx[mn.z + mn.x] = s;
        R.track[s] = make_int2(ln, mn.x);
        R.cm[ln].x = mn.x + 1;
    } else {
        R.pool4[mo.z + tr.y] = pn;
    }
    R.src[s] = pn;
    return true;
}

// After the ion and its image: the line images' slot moves (one lane each when no two
// of them touch a common leaf, else one lane in source order), beside them the distinct
// cells of their 2M root paths, then every thread repairs those cells' moments and counts,
// applying to each cell, in order, old line image 0 (-), new line image 0 (+), old 1 ...
template <bool F32, int BLOCK>
__device__ __forceinline__ void lines_commit(const RepU& R, Trav<2, BLOCK>& S, McShared& MS, int i) {
    LineList& LL = line_list(S);
    const int tid = threadIdx.x, M = R.nline, nc = 2 * M;
    const bool cart = F32 && R.M32;  // uniform
    double* const rowtab = (double*)((char*)&LL + sizeof(LineList));
    int rows = 0;
    for (int j = 0; j < nc; ++j) rows += MS.lplen[j];
    const bool use_rows = !cart && rows <= kLineRows<BLOCK>;
    if (tid == 0) LL.nlist = 0;  // the list space held the ion's and its image's table until now
    __syncthreads();
    if (wave_id() == 0) {
        const int m = lane_id();
        int lo = -1, ln = -1;
        if (m < M) {
            lo = MS.lpath[2 * m][MS.lplen[2 * m] - 1];
            ln = MS.lpath[2 * m + 1][MS.lplen[2 * m + 1] - 1];
        }
        bool clash = false;
        for (int e = 0; e < M; ++e) {
            const int eo = __shfl(lo, e, 64), en = __shfl(ln, e, 64);
            if (m < M && e != m && (eo == lo || eo == ln || en == lo || en == ln)) clash = true;
        }
        if (__ballot(clash) == 0) {
            if (m < M && !line_slot_move(R, 2 * R.n + m * R.n + i, lo, ln, MS.lpos[2 * m + 1])) MS.err = kErrCommitSlot;
        } else if (m == 0) {
            for (int k = 0; k < M; ++k) {
                const int ko = MS.lpath[2 * k][MS.lplen[2 * k] - 1], kn = MS.lpath[2 * k + 1][MS.lplen[2 * k + 1] - 1];
                if (!line_slot_move(R, 2 * R.n + k * R.n + i, ko, kn, MS.lpos[2 * k + 1])) { MS.err = kErrCommitSlot; break; }
            }
        }
    } else {
        for (int it = tid - 64; it < nc * kMaxLevels; it += BLOCK - 64) {
            const int j = it / kMaxLevels, l = it % kMaxLevels;
            if (l >= MS.lplen[j]) continue;
            const int c = MS.lpath[j][l];
            bool owner = true;
            for (int jj = 0; jj < j; ++jj)
                if (l < MS.lplen[jj] && MS.lpath[jj][l] == c) owner = false;
            if (!owner) continue;
            uint32_t mask = l < MS.lplen[j] - 1 ? kLineInternal : 0u;
            for (int jj = j; jj < nc; ++jj)
                if (l < MS.lplen[jj] && MS.lpath[jj][l] == c) mask |= 1u << jj;
            const int slot = atomicAdd(&LL.nlist, 1);
            LL.cell[slot] = c;
            LL.mask[slot] = mask;
            LL.lev[slot] = (uint8_t)l;
        }
        if (use_rows)
            for (int it = tid - 64; it < nc * kMaxLevels; it += BLOCK - 64) {
                const int j = it / kMaxLevels, l = it % kMaxLevels;
                if (l >= MS.lplen[j]) continue;
                int r0 = 0;
                for (int jj = 0; jj < j; ++jj) r0 += MS.lplen[jj];
                if (l == 0) LL.row0[j] = r0;
                const int c = MS.lpath[j][l];
                const double4 sp = MS.lpos[j], g = gload(R.cgeo + c);
                reg_row(sp.x - g.x, sp.y - g.y, sp.z - g.z, (j & 1) ? sp.w : -sp.w, rowtab + (r0 + l) * NH);
            }
    }
    __syncthreads();
    if (use_rows) {
        for (int it = tid; it < LL.nlist * NH; it += BLOCK) {
            const int li = it / NH, k = it % NH;
            const int c = LL.cell[li], l = LL.lev[li];
            const uint32_t mask = LL.mask[li];
            double* const hp = R.H + (size_t)c * HSTR + k;
            double h = *(GRow)hp;
            for (uint32_t rest = mask & 0xFFFFu; rest; rest &= rest - 1u) h += rowtab[(LL.row0[__builtin_ctz(rest)] + l) * NH + k];
            *hp = h;
            const int dc = __popc(mask & 0xAAAAu) - __popc(mask & 0x5555u);
            if (k == 0 && (mask & kLineInternal) && dc != 0) R.cm[c].x += dc;
        }
    } else if (!cart) {
        for (int it = tid; it < LL.nlist * NPAIR; it += BLOCK) {
            const int li = it / NPAIR, k = it % NPAIR;
            const int c = LL.cell[li];
            const uint32_t mask = LL.mask[li];
            const double4 g = gload(R.cgeo + c);
            const HPair hp = hpair_load(R, S.ht, c, k);
            double hc = hp.c, hs = hp.s;
            for (int j = 0; j < nc; ++j) {
                if (!(mask & (1u << j))) continue;
                const double4 sp = MS.lpos[j];
                hpair_add(S.ht, k, sp.x - g.x, sp.y - g.y, sp.z - g.z, (j & 1) ? sp.w : -sp.w, hc, hs);
            }
            hpair_store(R, S.ht, c, k, hc, hs);
            const int dc = __popc(mask & 0xAAAAu) - __popc(mask & 0x5555u);
            if (k == 0 && (mask & kLineInternal) && dc != 0) R.cm[c].x += dc;
        }
    }
    if (cart) {  // the moments and their single-precision copy, where the far field reads that
        for (int it = tid; it < LL.nlist * NTERM; it += BLOCK) {
            const int li = it / NTERM, k = it % NTERM;
            const int c = LL.cell[li];
            const uint32_t mask = LL.mask[li];
            const double4 g = R.cgeo[c];
            double mk = R.M[(size_t)c * MSTR + k];
            for (int j = 0; j < nc; ++j) {
                if (!(mask & (1u << j))) continue;
                const double4 sp = MS.lpos[j];
                const double v = mono(S.mi[k], sp.x - g.x, sp.y - g.y, sp.z - g.z);
                mk = (j & 1) ? mk + sp.w * v : mk - sp.w * v;
            }
            R.M[(size_t)c * MSTR + k] = mk;
            R.M32[(size_t)c * MSTR + k] = (float)mk;
            const int dc = __popc(mask & 0xAAAAu) - __popc(mask & 0x5555u);
            if (k == 0 && (mask & kLineInternal) && dc != 0) R.cm[c].x += dc;
        }
    }
    __syncthreads();
}

// Local modification of Sec. 3.3 for an accepted move.  Thread 0 moves the
// ion and then its image between leaf index arrays (delete = the last entry
// fills the hole; add = append) from the state gathered during the
// traversal; the other threads repair the moments and counts of the distinct
// cells of the four root paths, applying to each cell, in order, the old ion
// (-), the new ion (+), the old image (-) and the new image (+).
template <bool F32, int BLOCK>
__device__ __forceinline__ void commit(const RepU& R, Trav<2, BLOCK>& S, McShared& MS, int i) {
    const int tid = threadIdx.x;
    const bool imgs = R.images != 0;
    const bool cart = F32 && R.M32;  // uniform: the Cartesian moments are repaired, not the expansion rows
    const int nps = imgs ? 4 : 2;
    int row0[4], rows = 0;  // first table row of each root path
#pragma unroll
    for (int jj = 0; jj < 4; ++jj) { row0[jj] = rows; rows += jj < nps ? MS.plen[jj] : 0; }
    const bool use_rows = !cart && rows <= Trav<2, BLOCK>::HROWS;
    const bool use_pw = cart && MS.nlist <= kPowCells;
    if (use_rows) {  // the harmonics of every path entry, a lane each, in the traversal's list space
        for (int r = tid; r < rows; r += BLOCK) {
            const int jj = (r >= row0[1] ? 1 : 0) + (nps > 2 ? (r >= row0[2] ? 1 : 0) + (r >= row0[3] ? 1 : 0) : 0);
            const double4 sc = MS.contrib[jj], g = MS.path_geo[jj][r - row0[jj]];
            reg_row(sc.x - g.x, sc.y - g.y, sc.z - g.z, (jj & 1) ? sc.w : -sc.w, S.hrow[r]);
        }
        __syncthreads();
    }
    if (use_pw) {
        for (int it = tid; it < MS.nlist * 12; it += BLOCK) {
            const int li = it / 12, r = it % 12, jj = r / 3, ax = r % 3;
            const double4 s = MS.contrib[jj], g = MS.list_geo[li];
            const double d = ax == 0 ? s.x - g.x : (ax == 1 ? s.y - g.y : s.z - g.z);
            double v = 1.0;
            MS.pw[li][jj][ax][0] = 1.0;
            for (int e = 1; e <= P; ++e) { v *= d; MS.pw[li][jj][ax][e] = v; }
        }
        __syncthreads();
    }
    if (tid == 0) {
        // leaf states: cell, base, count of up to four leaves, followed through the moves
        int lc[4], lb[4], ln[4];
        int nl = 0;
        auto find = [&](int cell, int base, int count) {
            for (int k = 0; k < nl; ++k)
                if (lc[k] == cell) return k;
            lc[nl] = cell; lb[nl] = base; ln[nl] = count;
            return nl++;
        };
        const int a = find(MS.tr[0].x, MS.lm_old[0].z, MS.lm_old[0].x);
        const int b = find(MS.path[1][MS.plen[1] - 1], MS.lm_new[0].z, MS.lm_new[0].x);
        int img_slot = imgs ? MS.tr[1].y : -1;
        const int K = R.n + i;
        const double4 ion_new = MS.contrib[1];
        if (a != b) {
            const int k = MS.tr[0].y, last = ln[a] - 1;
            const int moved = MS.last_pidx[0];
            if (k != last) {
                R.pool4[lb[a] + k] = MS.last_pool[0];
                R.pidx[lb[a] + k] = moved;
                if (moved >= 0 && moved < R.nsrc) R.track[moved] = make_int2(lc[a], k);
                else MS.err = kErrCommitSource;
                if (moved == K) img_slot = k;
            }
            ln[a] = last;
            R.cm[lc[a]].x = last;
            const int pos = ln[b];
            R.pool4[lb[b] + pos] = ion_new;
            R.pidx[lb[b] + pos] = i;
            R.track[i] = make_int2(lc[b], pos);
            ln[b] = pos + 1;
            R.cm[lc[b]].x = pos + 1;
        } else {
            R.pool4[lb[a] + MS.tr[0].y] = ion_new;
        }
        R.src[i] = ion_new;
        if (imgs) {
            const int c_old = MS.tr[1].x;
            const int touched = (c_old == lc[a] || c_old == lc[b]);
            const int cc = find(c_old, MS.lm_old[1].z, MS.lm_old[1].x);
            const int dd = find(MS.path[3][MS.plen[3] - 1], MS.lm_new[1].z, MS.lm_new[1].x);
            const double4 img_new = MS.contrib[3];
            if (cc != dd) {
                const int last = ln[cc] - 1;
                int moved;
                double4 mv;
                if (!touched) {
                    moved = MS.last_pidx[1];
                    mv = MS.last_pool[1];
                } else {  // the ion's move changed this leaf: read its last entry again
                    moved = R.pidx[lb[cc] + last];
                    mv = R.pool4[lb[cc] + last];
                }
                if (img_slot != last) {
                    R.pool4[lb[cc] + img_slot] = mv;
                    R.pidx[lb[cc] + img_slot] = moved;
                    if (moved >= 0 && moved < R.nsrc) R.track[moved] = make_int2(lc[cc], img_slot);
                    else MS.err = kErrCommitSource;
                }
                ln[cc] = last;
                R.cm[lc[cc]].x = last;
                const int pos = ln[dd];
                R.pool4[lb[dd] + pos] = img_new;
                R.pidx[lb[dd] + pos] = K;
                R.track[K] = make_int2(lc[dd], pos);
                ln[dd] = pos + 1;
                R.cm[lc[dd]].x = pos + 1;
            } else {
                R.pool4[lb[cc] + img_slot] = img_new;
            }
            R.src[K] = img_new;
        }
    }
    // expansion rows and counts of the distinct path cells: one coefficient of a cell per item, a
    // table read per contribution; a list of paths longer than the table forms the harmonics of
    // each (l, m) pair where it needs them
    if (use_rows) {
        for (int it = tid; it < MS.nlist * NH; it += BLOCK) {
            const int li = it / NH, k = it % NH;
            const int c = MS.list_cell[li], mask = MS.list_mask[li], l = MS.list_lev[li];
            double* const hp = R.H + (size_t)c * HSTR + k;
            double h = *(GRow)hp;
#pragma unroll
            for (int jj = 0; jj < 4; ++jj) h += (mask & (1 << jj)) ? S.hrow[row0[jj] + l][k] : 0.0;
            *hp = h;
            const int dc = __popc(mask & 10) - __popc(mask & 5);
            if (k == 0 && (mask & 16) && dc != 0) R.cm[c].x += dc;
        }
    } else if (!cart) {
        for (int it = tid; it < MS.nlist * NPAIR; it += BLOCK) {
            const int li = it / NPAIR, k = it % NPAIR;
            const int c = MS.list_cell[li], mask = MS.list_mask[li];
            const double4 g = MS.list_geo[li];
            const HPair hp = hpair_load(R, S.ht, c, k);
            double hc = hp.c, hs = hp.s;
            for (int jj = 0; jj < 4; ++jj) {
                if (!(mask & (1 << jj))) continue;
                const double4 s = MS.contrib[jj];
                hpair_add(S.ht, k, s.x - g.x, s.y - g.y, s.z - g.z, (jj & 1) ? s.w : -s.w, hc, hs);
            }
            hpair_store(R, S.ht, c, k, hc, hs);
            const int dc = __popc(mask & 10) - __popc(mask & 5);
            if (k == 0 && (mask & 16) && dc != 0) R.cm[c].x += dc;
        }
    }
    if (!cart) {
        __syncthreads();
        return;
    }
    // the moments and their single-precision copy: all loads first, then stores
    const int items = MS.nlist * NTERM;
    constexpr int G = 4;
    for (int base = tid; base < items; base += G * BLOCK) {
        double mk[G];
#pragma unroll
        for (int u = 0; u < G; ++u) {
            const int it = base + u * BLOCK;
            if (it < items) {
                const int li = it / NTERM, k = it % NTERM;
                mk[u] = R.M[(size_t)MS.list_cell[li] * MSTR + k];
            }
        }
#pragma unroll
        for (int u = 0; u < G; ++u) {
            const int it = base + u * BLOCK;
            if (it >= items) continue;
            const int li = it / NTERM, k = it % NTERM;
            const int c = MS.list_cell[li], mask = MS.list_mask[li];
            const double4 g = MS.list_geo[li];
            double m = mk[u];
#pragma unroll
            for (int jj = 0; jj < 4; ++jj) {
                if (!(mask & (1 << jj))) continue;
                const double4 s = MS.contrib[jj];
                double v;
                if (use_pw) {
                    const uint32_t code = S.mi[k];
                    v = MS.pw[li][jj][0][code & 255u] * MS.pw[li][jj][1][(code >> 8) & 255u] *
                        MS.pw[li][jj][2][code >> 16];
                } else {
                    v = mono(S.mi[k], s.x - g.x, s.y - g.y, s.z - g.z);
                }
                m = (jj & 1) ? m + s.w * v : m - s.w * v;
            }
            R.M[(size_t)c * MSTR + k] = m;
            R.M32[(size_t)c * MSTR + k] = (float)m;
            const int dc = __popc(mask & 10) - __popc(mask & 5);
            if (k == 0 && (mask & 16) && dc != 0) R.cm[c].x += dc;
        }
    }
    __syncthreads();
}

// mode 0: evaluate; 1: Metropolis with alpha, commit if accepted;
// 2: commit unless rejected by a wall or an overlap.
//
// si and mo are the mover's ion and image as stored (mo unused without images);
// inext >= 0 names the next move's ion, whose sources one lane loads into
// MS.nx_si / MS.nx_mo during the traversal (valid if the ion is not i).
template <int BLOCK, bool LINES, bool F32>
__device__ __forceinline__ MoveOut one_move(const RepU& R, Trav<2, BLOCK>& S, McShared& MS, int i, double4 si,
                            double4 mo, double rx, double ry, double rz, double alpha, int mode, int inext) {
    static_assert(BLOCK >= 256, "the path descents, the commit prefetch and the next mover's load run on "
                                "the last three waves");
    const int tid = threadIdx.x;
    MoveOut out{kInf, 0, 0, 0, 0};
    const bool imgs = R.images != 0;
    const int nps = imgs ? 4 : 2;
    if (outside(R, rx, ry, rz)) { out.reason = 1; return out; }
    if (tid < 4) {
        // lane j sets up contribution j (old ion, new ion, old image, new image) and its key,
        // the four side by side; lane 0 then writes the targets' state
        const int j = tid;
        double4 cj;
        if (j == 0) cj = si;
        else if (j == 1) cj = make_double4(rx, ry, rz, si.w);
        else if (j == 2) cj = mo;
        else cj = imgs ? kelvin(R, rx, ry, rz, si.w) : make_double4(0, 0, 0, 0);
        const uint64_t kj = (j < 2 || imgs) ? morton_key(R, cj.x, cj.y, cj.z) : 0;
        MS.key[j] = kj;
        MS.contrib[j] = cj;
        const uint32_t klo = (uint32_t)kj, khi = (uint32_t)(kj >> 32);
        const uint64_t kio = (uint64_t)(uint32_t)__shfl((int)klo, 0, 64) |
                             ((uint64_t)(uint32_t)__shfl((int)khi, 0, 64) << 32);
        const uint64_t kmo = (uint64_t)(uint32_t)__shfl((int)klo, 2, 64) |
                             ((uint64_t)(uint32_t)__shfl((int)khi, 2, 64) << 32);
        if (j == 0) {
            S.tx[0] = si.x; S.ty[0] = si.y; S.tz[0] = si.z;
            S.tx[1] = rx; S.ty[1] = ry; S.tz[1] = rz;
            for (int t = 0; t < 2; ++t) {
                S.ex_i[t] = i; S.ex_k[t] = imgs ? R.n + i : -1;
                S.kx_i[t] = kio; S.kx_k[t] = kmo;
                S.es_i[t] = si; S.es_k[t] = mo;
            }
            S.ovl_t = 1; S.ovl_ex = i; S.n_ovl = 0;
            S.err = 0; S.overlap = 0; S.coincide = 0;
            // The root holds both targets, so the MAC never takes it (theta < 1): it is opened
            // for both whenever it is split and holds more than N_0 sources besides the two
            // excluded ones.  Then the traversal starts from its children, cells 1..8 in digit
            // order.
            const int np_root = R.nsrc - 1 - (imgs ? 1 : 0);
            if (R.ncell > 1 && np_root > R.n0) {
                const int di = key_digit(kio, 1), dk = imgs ? key_digit(kmo, 1) : -1;
                for (int d = 0; d < 8; ++d)
                    S.front[0][d] = (uint32_t)(1 + d) | (3u << kMaskSh) | (d == di ? kFlagIon : 0u) |
                                    (d == dk ? kFlagImg : 0u);
                MS.fs0 = 8;
                MS.level0 = 1;
            } else {
                S.front[0][0] = (3u << kMaskSh) | kFlagIon | (imgs ? kFlagImg : 0u);
                MS.fs0 = 1;
                MS.level0 = 0;
            }
            MS.alpha = alpha;
            MS.err = 0;
            MS.nlist = 0;
        }
    }
    // work beside the traversal runs on the last waves, which have no frontier entries to
    // classify on most levels, each task on a wave of its own (divergent lanes of one wave
    // would wait for their loads one after another): the root-path descents on lanes 0-3 of
    // the last wave, the commit prefetch on lanes 0-1 of the wave before it, and the next
    // mover's load on lane 0 of the wave before that
    const int th = tid - (BLOCK - 64), tp = tid - (BLOCK - 128);
    if (th >= 0 && th < 4) { MS.path[th][0] = 0; MS.plen[th] = 0; }
    if (tp == 0 || tp == 1) MS.pf_stage[tp] = (tp == 1 && !imgs) ? 3 : 0;
    int my_level = 0;  // the next level of this lane's root path
    // the line images' root paths (multiple-image model) on lanes 16 .. 16 + 2M - 1 of the
    // wave that loads the next mover
    {
        const int tl = tid - (BLOCK - 192) - 16;
        if (LINES && tl >= 0 && tl < 2 * R.nline) {
            MS.lpath[tl][0] = 0;
            MS.lplen[tl] = 0;
            MS.lnext[tl] = -1;
            if (!(tl & 1)) { MS.lmac[tl >> 1][0] = -1; MS.lmac[tl >> 1][1] = -1; }
        }
    }
    __syncthreads();
    // one step of a root path: descend by the key's digit, or stop at the leaf
    auto step = [&](int pj, int level) {
        const int c = MS.path[pj][level];
        const bool cok = c >= 0 && c < R.ncell;
        const int link = cok ? gload(R.cm + c).y : -1;
        if (cok) MS.path_geo[pj][level] = gload(R.cgeo + c);
        if (c < 0 || c >= R.ncell || (link >= 0 && link + 8 > R.ncell)) {
            MS.err = kErrPathCell;
            MS.plen[pj] = level + 1;
            MS.path[pj][level] = 0;
        } else if (link >= 0 && level + 1 < kMaxLevels) {
            MS.path[pj][level + 1] = link + key_digit(MS.key[pj], level + 1);
        } else {
            if (link >= 0) MS.err = kErrPathDepth;
            MS.plen[pj] = level + 1;
            if (pj & 1) {  // a new position's leaf: its slot state for the commit
                const int4 m = gload(R.cm + c);
                MS.lm_new[pj >> 1] = m;
                if (m.y >= 0 || m.z < 0 || m.x < 0 || m.z + m.w > R.pool) MS.err = kErrCommitLeaf;
            }
        }
    };
    // the root paths descend two levels, and the commit state two stages, per traversal level;
    // the next mover's sources are loaded on the first level
    auto hook = [&](int level) {
        if (th >= 0 && th < nps)
            for (int k = 0; k < 2 && MS.plen[th] == 0 && my_level < kMaxLevels; ++k) step(th, my_level++);
        if (tp == 0 || tp == 1)
            for (int k = 0; k < 2; ++k) prefetch_stage(R, MS, tp, tp == 0 ? i : R.n + i);
        if (tp == -64 && level == MS.level0 && inext >= 0) {
            MS.nx_si = R.src[inext];
            MS.nx_mo = imgs ? R.src[R.n + inext] : make_double4(0, 0, 0, 0);
        }
        if (LINES && tid - (BLOCK - 192) - 16 >= 0 && tid - (BLOCK - 192) - 16 < 2 * R.nline)
            line_lane_steps(R, MS, S.tx, S.ty, S.tz, tid - (BLOCK - 192) - 16, i, 2);
    };
    double pot[2];
    const int levels = traverse_mc<F32, BLOCK>(R, S, MS.cnt2, hook, MS.fs0, MS.level0, pot);
    (void)levels;
    if (S.err) {
        out.stop = (S.err == kErrStack || S.err == kErrFrontier) ? -7 : -8;
        out.detail = S.err;
        __syncthreads();
        return out;
    }
    if (th >= 0 && th < nps) {
        while (MS.plen[th] == 0 && my_level < kMaxLevels) step(th, my_level++);
        if (MS.plen[th] == 0) { MS.err = kErrPathDepth; MS.plen[th] = 1; MS.path[th][0] = 0; }
    }
    if (tp == 0 || tp == 1) {
        const int s = tp == 0 ? i : R.n + i;
        for (int k = 0; k < 3 && MS.pf_stage[tp] < 3; ++k) prefetch_stage(R, MS, tp, s);
        if (MS.pf_stage[tp] != 3) MS.err = kErrCommitSlot;
    }
    {
        const int tl = tid - (BLOCK - 192) - 16;
        if (LINES && tl >= 0 && tl < 2 * R.nline) {
            line_lane_steps(R, MS, S.tx, S.ty, S.tz, tl, i, kMaxLevels);
            if (MS.lplen[tl] == 0) { MS.err = kErrPathDepth; MS.lplen[tl] = 1; MS.lpath[tl][0] = 0; }
        }
    }
    __syncthreads();
    if (MS.err) { out.stop = -8; out.detail = MS.err; __syncthreads(); return out; }
    // distinct cells of the root paths (any order: each cell's updates are applied by one thread set)
    for (int it = tid; it < nps * kMaxLevels; it += BLOCK) {
        const int j = it / kMaxLevels, l = it % kMaxLevels;
        if (l >= MS.plen[j]) continue;
        const int c = MS.path[j][l];
        bool owner = true;
        for (int jj = 0; jj < j; ++jj)
            if (l < MS.plen[jj] && MS.path[jj][l] == c) owner = false;
        if (!owner) continue;
        int mask = l < MS.plen[j] - 1 ? 16 : 0;
        for (int jj = j; jj < nps; ++jj)
            if (l < MS.plen[jj] && MS.path[jj][l] == c) mask |= 1 << jj;
        const int slot = atomicAdd(&MS.nlist, 1);
        MS.list_cell[slot] = c;
        MS.list_mask[slot] = mask;
        MS.list_lev[slot] = l;
        MS.list_geo[slot] = MS.path_geo[j][l];
    }
    const double po = pot[0], pn = pot[1];
    if (S.overlap || S.coincide) { out.reason = 2; __syncthreads(); return out; }
    double lc0 = 0.0, lc1 = 0.0;  // what the mover's own line images added at the two targets
    if (LINES && R.nline > 0) line_corrections(R, MS, lc0, lc1);
    // the move's positions and alpha come back from LDS: no registers held across the traversal
    const double4 so = MS.contrib[0], sn = MS.contrib[1];
    const double q = so.w, l = R.l_B;
    double dE = LINES && R.nline > 0 ? l * q * ((pn - lc1) - (po - lc0)) : l * q * (pn - po);
    if (R.geom == 1) {
        const double rn2 = sn.x * sn.x + sn.y * sn.y + sn.z * sn.z;
        const double ro2 = so.x * so.x + so.y * so.y + so.z * so.z;
        if (imgs) dE += 0.5 * l * R.gamma * R.a * q * q * (1.0 / (rn2 - R.a2) - 1.0 / (ro2 - R.a2));
        // own line images: c_m q_K at t_m r_K, |r - t_m r_K| = (r^2 - t_m a^2) / |r|
        if (LINES)
            for (int m = 0; m < R.nline; ++m)
                dE += 0.5 * l * R.line_c[m] * R.gamma * R.a * q * q *
                      (1.0 / (rn2 - R.line_t[m] * R.a2) - 1.0 / (ro2 - R.line_t[m] * R.a2));
        if (R.Qc != 0.0) dE += l * R.Qc * q * (1.0 / sqrt(rn2) - 1.0 / sqrt(ro2));
    }
    out.dE = dE;
    bool acc = false;
    if (mode == 1) acc = dE <= 0.0 || MS.alpha <= exp(-dE);
    else if (mode == 2) acc = true;
    if (!acc) { __syncthreads(); return out; }
    if (tid == BLOCK - 1) {  // a thread with no path-cell item above
        // the tracked leaves must be the leaves the old positions' keys lead to,
        // and the tracked slots must hold the movers
        bool sane = MS.tr[0].x == MS.path[0][MS.plen[0] - 1] && MS.self_pidx[0] == i;
        if (imgs) sane = sane && MS.tr[1].x == MS.path[2][MS.plen[2] - 1] && MS.self_pidx[1] == R.n + i;
        sane = sane && MS.last_pidx[0] >= 0 && MS.last_pidx[0] < R.nsrc;
        bool ok = sane;
        if (sane) {
            const int cio = MS.tr[0].x, cin = MS.path[1][MS.plen[1] - 1];
            if (cin != cio && MS.lm_new[0].x + 1 > MS.lm_new[0].w) ok = false;
            if (imgs) {
                const int cmo = MS.tr[1].x, cmn = MS.path[3][MS.plen[3] - 1];
                if (cmn != cmo) {
                    int c = MS.lm_new[1].x;
                    if (cin != cio) { if (cmn == cin) c += 1; if (cmn == cio) c -= 1; }
                    if (c + 1 > MS.lm_new[1].w) ok = false;
                }
            }
        } else {
            MS.err = kErrCommitSlot;
        }
        if (LINES && R.nline > 0 && ok && !lines_fit(R, MS)) ok = false;  // every insertion of the move, in commit order
        MS.ok = ok;
    }
    __syncthreads();
    if (MS.err) { out.stop = -8; out.detail = MS.err; __syncthreads(); return out; }
    if (!MS.ok) { out.stop = -6; __syncthreads(); return out; }
    commit<F32, BLOCK>(R, S, MS, i);
    if (LINES && R.nline > 0 && !MS.err) lines_commit<F32, BLOCK>(R, S, MS, i);
    if (MS.err) { out.stop = -8; out.detail = MS.err; }
    out.accepted = 1;
    return out;
}

// ------------------------------------------------------------ kernels
constexpr int kMcBlock = 512;      // a single chain: the widest traversal per move
constexpr int kMcBlockBatch = 256; // replicas: two workgroups per CU hide each other's latency

__device__ __forceinline__ void load_rep(Rep& dst, const Rep* src) {
    constexpr int W = (int)(sizeof(Rep) / 8);
    static_assert(sizeof(Rep) % 8 == 0, "Rep is copied as 8-byte words");
    const uint64_t* a = (const uint64_t*)src;
    uint64_t* b = (uint64_t*)&dst;
    for (int k = threadIdx.x; k < W; k += blockDim.x) b[k] = a[k];
}

// Persistent Metropolis kernel: each workgroup takes replicas from the queue
// and advances its chain from move_next to move_end (Sec. 2 steps 1-3 with the
// treecode energy change and the local adjustment of Sec. 3.3).  A replica
// whose accepted move would overflow a leaf index array stops before that
// move with mc_status = ECAPACITY; the host rebuilds it and resumes.
template <int BLOCK, bool LINES, bool F32>
__global__ void __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(2))) k_mc(Rep* reps, McArgs A) {
    __shared__ Trav<2, BLOCK> S;
    __shared__ McShared MS;
    __shared__ Rep Rs;
    __shared__ int s_r;
    const int tid = threadIdx.x;
    fill_mi(S);  // published by the first barrier below
    for (;;) {
        if (tid == 0) {
            const int qi = atomicAdd(A.queue, 1);
            s_r = qi < A.nlist ? A.list[qi] : -1;
        }
        __syncthreads();
        const int r = s_r;
        if (r < 0) break;
        load_rep(Rs, reps + r);
        __syncthreads();
        const RepU R(Rs);
        long long m = uni(Rs.move_next);
        const long long m0 = m, mend = uni(Rs.move_end);
        const bool imgs = R.images != 0;
        long long st_moves = 0, st_acc = 0, st_wall = 0, st_ovl = 0, st_met = 0;
        int status = 0, detail = 0;
        int prev_i = -1;
        bool have_nx = false;  // MS.nx_si / nx_mo hold this move's sources as of the last move
        for (; m < mend; ++m) {
            const int b = (int)((m - m0) & (kDrawBatch - 1));
            if (b == 0) {
                // the first wave draws the next kDrawBatch moves, one per lane
                if (tid < kDrawBatch && m + tid < mend) {
                    const Draw d = draw_move(A.seed, (uint32_t)r, (uint64_t)(m + tid), Rs.n, A.step);
                    MS.dr_i[tid] = d.i;
                    MS.dr_d[tid][0] = d.dx; MS.dr_d[tid][1] = d.dy; MS.dr_d[tid][2] = d.dz;
                    MS.dr_d[tid][3] = d.alpha;
                }
                __syncthreads();
            }
            const int i = MS.dr_i[b];
            const int inext = (b + 1 < kDrawBatch && m + 1 < mend) ? MS.dr_i[b + 1] : -1;
            // the last move changed only its own ion and image
            const bool use_nx = have_nx && i != prev_i;
            const double4 si = use_nx ? MS.nx_si : Rs.src[i];
            const double4 mo = use_nx ? MS.nx_mo : (imgs ? Rs.src[Rs.n + i] : make_double4(0, 0, 0, 0));
            const MoveOut o = one_move<BLOCK, LINES, F32>(R, S, MS, i, si, mo, si.x + MS.dr_d[b][0], si.y + MS.dr_d[b][1],
                                              si.z + MS.dr_d[b][2], MS.dr_d[b][3], 1, inext);
            // a move outside the walls returns before its traversal, so before the load
            have_nx = inext >= 0 && o.reason != 1;
            prev_i = i;
            if (o.stop) { status = o.stop; detail = o.detail; break; }
            ++st_moves;
            if (o.accepted) ++st_acc;
            else if (o.reason == 1) ++st_wall;
            else if (o.reason == 2) ++st_ovl;
            else ++st_met;
            if (A.accept && tid == 0) A.accept[m - A.move_base] = (uint8_t)o.accepted;
            __syncthreads();
        }
        if (tid == 0) {
            Rep* g = reps + r;
            g->move_next = m;
            g->mc_status = status;
            if (detail) g->err_detail = detail;
            g->stats[0] += st_moves; g->stats[1] += st_acc; g->stats[2] += st_wall;
            g->stats[3] += st_ovl; g->stats[4] += st_met;
        }
        __syncthreads();
    }
}

template <bool LINES, bool F32>
__global__ void __launch_bounds__(kMcBlock) k_move(Rep* reps, int r, MoveIO in, MoveIO* io) {
    __shared__ Trav<2, kMcBlock> S;
    __shared__ McShared MS;
    __shared__ Rep Rs;
    fill_mi(S);
    load_rep(Rs, reps + r);
    __syncthreads();
    const int i = in.i;
    const double4 si = Rs.src[i];
    const double4 mo = Rs.images ? Rs.src[Rs.n + i] : make_double4(0, 0, 0, 0);
    const MoveOut o = one_move<kMcBlock, LINES, F32>(RepU(Rs), S, MS, i, si, mo, in.rn[0], in.rn[1], in.rn[2], 0.0,
                                         in.mode == 0 ? 0 : 2, -1);
    if (threadIdx.x == 0) {
        io->dE = o.dE;
        io->reason = o.reason;
        io->status = o.stop;
        if (o.detail) reps[r].err_detail = o.detail;
    }
}

#include "bhmc_moves.hpp"

#include "bhmc_group.hpp"

// Pair terms of a target with its own image y inside a far cell: with
// D_n = (y - c)^n, v = sum_{|n|<=p} T_n D_n, F_k = sum_{|m|<=p+1} m_k T_m D_{m-e_k}
// (the image's part of the target's field) and G_k = sum_{|n|<=p} n_k T_n D_{n-e_k}
// (the image's own gradient of v).
template <int K>
__device__ __forceinline__ void flag_rec(double (&T)[NTERM1], double (&D)[NTERM], double Rx, double Ry, double Rz,
                                         double ir2, double dx, double dy, double dz, double& v, double (&F)[3],
                                         double (&G)[3]) {
    if constexpr (K < NTERM1) {
        constexpr TEnt e = TT1.e[K];
        if constexpr (K > 0) t_step<K>(T, Rx, Ry, Rz, ir2);
        if constexpr (K < NTERM) {
            if constexpr (K == 0) D[0] = 1.0;
            else if constexpr (e.n1 >= 1) D[K] = D[e.x1] * dx;
            else if constexpr (e.n2 >= 1) D[K] = D[e.y1] * dy;
            else D[K] = D[e.z1] * dz;
            v = fma(T[K], D[K], v);
            if constexpr (e.x1 >= 0) G[0] = fma((double)e.n1 * T[K], D[e.x1], G[0]);
            if constexpr (e.y1 >= 0) G[1] = fma((double)e.n2 * T[K], D[e.y1], G[1]);
            if constexpr (e.z1 >= 0) G[2] = fma((double)e.n3 * T[K], D[e.z1], G[2]);
        }
        if constexpr (e.x1 >= 0) F[0] = fma((double)e.n1 * T[K], D[e.x1], F[0]);
        if constexpr (e.y1 >= 0) F[1] = fma((double)e.n2 * T[K], D[e.y1], F[1]);
        if constexpr (e.z1 >= 0) F[2] = fma((double)e.n3 * T[K], D[e.z1], F[2]);
        flag_rec<K + 1>(T, D, Rx, Ry, Rz, ir2, dx, dy, dz, v, F, G);
    }
}

// The far cell that holds a target's own image in its traversal (found by k_grad;
// one thread per ion): the image's pair terms with the target, taken through that
// cell's expansion, come back out of the target's potential, field and energy term
// and out of the image's source-side gradient.  Kept apart from k_grad because it
// holds every monomial of the image and T up to order p + 1 at once.
__global__ void __launch_bounds__(256) k_gflag(Rep* reps, int r, const int* fcell, double4* G, double4* Gt,
                                               double* eterm) {
    const Rep& R = reps[r];
    const int ion = blockIdx.x * blockDim.x + threadIdx.x;
    if (ion >= R.n || !R.images) return;
    const int c = fcell[ion];
    if (c < 0) return;
    if (c >= R.ncell) { reps[r].err_detail = kErrFlagCell; return; }
    const double4 g = R.cgeo[c];
    const double4 x = R.src[ion];
    const double4 y = R.src[R.n + ion];
    const double Rx = g.x - x.x, Ry = g.y - x.y, Rz = g.z - x.z;
    double T[NTERM1], D[NTERM];
    T[0] = rsqrt_nr(Rx * Rx + Ry * Ry + Rz * Rz);
    const double ir2 = T[0] * T[0];
    double v = 0.0, F[3] = {0.0, 0.0, 0.0}, Gk[3] = {0.0, 0.0, 0.0};
    flag_rec<0>(T, D, Rx, Ry, Rz, ir2, y.x - g.x, y.y - g.y, y.z - g.z, v, F, Gk);
    const double half_lB = 0.5 * R.l_B, wq = half_lB * x.w;
    double4 gt = Gt[ion];
    gt.x += wq * (y.w * F[0]);
    gt.y += wq * (y.w * F[1]);
    gt.z += wq * (y.w * F[2]);
    gt.w -= half_lB * (y.w * v);
    Gt[ion] = gt;
    eterm[ion] -= 0.5 * x.w * (y.w * v);
    double4 gs = G[R.n + ion];
    gs.x -= wq * y.w * Gk[0];
    gs.y -= wq * y.w * Gk[1];
    gs.z -= wq * y.w * Gk[2];
    gs.w -= wq * v;
    G[R.n + ion] = gs;
}

// The target's own line images (multiple-image model; one thread per ion, after
// k_gflag): k_grad kept them in the ion's traversal as ordinary sources, so each pair
// term of the ion with one of them comes back out where the traversal met it -- through
// the expansion of the first cell of the line image's root path that passes the MAC,
// else directly at its leaf -- from the ion's potential, field and energy term and from
// the line image's source-side gradient.  The ion's energy with its own line images,
// 1/2 q sum_m c_m q_K / |r - t_m r_K|, joins its energy term (its gradient is k_chain's).
__global__ void __launch_bounds__(256) k_gline(Rep* reps, int r, double4* G, double4* Gt, double* eterm) {
    const Rep& R = reps[r];
    const int ion = blockIdx.x * blockDim.x + threadIdx.x;
    if (ion >= R.n || R.nline <= 0) return;
    const double4 x = R.src[ion];
    const double half_lB = 0.5 * R.l_B, wq = half_lB * x.w;
    double4 gt = Gt[ion];
    double e = eterm[ion];
    for (int m = 0; m < R.nline; ++m) {
        const int s = 2 * R.n + m * R.n + ion;
        const double4 y = R.src[s];
        const uint64_t key = morton_key(R, y.x, y.y, y.z);
        int c = 0, far = -1;
        bool leaf = false;
        double4 g = make_double4(0.0, 0.0, 0.0, 0.0);
        for (int level = 0; level < kMaxLevels; ++level) {
            if (c < 0 || c >= R.ncell) break;
            g = R.cgeo[c];
            const double dx = g.x - x.x, dy = g.y - x.y, dz = g.z - x.z;
            if (3.0 * (g.w * g.w) <= R.theta2 * (dx * dx + dy * dy + dz * dz)) { far = c; break; }
            const int link = R.cm[c].y;
            if (link < 0) { leaf = true; break; }
            if (link + 8 > R.ncell) break;
            c = link + key_digit(key, level + 1);
        }
        double v, F[3] = {0.0, 0.0, 0.0}, Gk[3] = {0.0, 0.0, 0.0};
        if (far >= 0) {
            const double Rx = g.x - x.x, Ry = g.y - x.y, Rz = g.z - x.z;
            double T[NTERM1], D[NTERM];
            T[0] = rsqrt_nr(Rx * Rx + Ry * Ry + Rz * Rz);
            v = 0.0;
            flag_rec<0>(T, D, Rx, Ry, Rz, T[0] * T[0], y.x - g.x, y.y - g.y, y.z - g.z, v, F, Gk);
        } else if (leaf) {
            // 1/|x - y|: -d/dx = d/dy = (x - y) / |x - y|^3
            const double ex = x.x - y.x, ey = x.y - y.y, ez = x.z - y.z;
            const double ir = rsqrt_nr(ex * ex + ey * ey + ez * ez), ir3 = ir * ir * ir;
            v = ir;
            F[0] = Gk[0] = ex * ir3; F[1] = Gk[1] = ey * ir3; F[2] = Gk[2] = ez * ir3;
        } else {
            reps[r].err_detail = kErrPathCell;
            v = __builtin_nan("");
        }
        gt.x += wq * (y.w * F[0]);
        gt.y += wq * (y.w * F[1]);
        gt.z += wq * (y.w * F[2]);
        gt.w -= half_lB * (y.w * v);
        e -= 0.5 * x.w * (y.w * v);
        double4 gs = G[s];
        gs.x -= wq * y.w * Gk[0];
        gs.y -= wq * y.w * Gk[1];
        gs.z -= wq * y.w * Gk[2];
        gs.w -= wq * v;
        G[s] = gs;
    }
    const double r2 = x.x * x.x + x.y * x.y + x.z * x.z;
    for (int m = 0; m < R.nline; ++m) e += 0.5 * x.w * (R.line_c[m] * R.gamma * R.a * x.w / (r2 - R.line_t[m] * R.a2));
    Gt[ion] = gt;
    eterm[ion] = e;
}

// Step 3, one thread per ion: both roles of the ion, its image mapped back
// by the chain rule through q_K = gamma a q / |r| and r_K = a^2 r / |r|^2,
// and the exact self-image and central-charge terms.
__global__ void __launch_bounds__(256) k_chain(const Rep* reps, int r, const double4* G, const double4* Gt,
                                               double* dEdr, double* dEdq) {
    const Rep& R = reps[r];
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= R.n) return;
    const double4 si = R.src[i];
    const double x = si.x, y = si.y, z = si.z, q = si.w;
    const double4 a = Gt[i], b = G[i];
    double gx = a.x + b.x, gy = a.y + b.y, gz = a.z + b.z, gq = a.w + b.w;
    const double l = R.l_B;
    const double r2 = x * x + y * y + z * z;
    if (R.images) {
        // a line image sits at t_m r_K with charge c_m q_K: its gradient joins the Kelvin image's
        double4 h = G[R.n + i];
        for (int m = 0; m < R.nline; ++m) {
            const double4 hm = G[2 * R.n + m * R.n + i];
            h.x += R.line_t[m] * hm.x; h.y += R.line_t[m] * hm.y; h.z += R.line_t[m] * hm.z;
            h.w += R.line_c[m] * hm.w;
        }
        const double rn = sqrt(r2);
        const double ir2 = 1.0 / r2, ir4 = ir2 * ir2;
        const double rh = x * h.x + y * h.y + z * h.z;
        gx += R.a2 * (h.x * ir2 - 2.0 * x * rh * ir4);
        gy += R.a2 * (h.y * ir2 - 2.0 * y * rh * ir4);
        gz += R.a2 * (h.z * ir2 - 2.0 * z * rh * ir4);
        const double c = -R.gamma * R.a * q / (r2 * rn);
        gx += h.w * c * x; gy += h.w * c * y; gz += h.w * c * z;
        gq += h.w * R.gamma * R.a / rn;
        const double den = r2 - R.a2;
        const double cs = -l * R.gamma * R.a * q * q / (den * den);
        gx += cs * x; gy += cs * y; gz += cs * z;
        gq += l * R.gamma * R.a * q / den;
        // the ion's energy with its own line images, 1/2 l_B c_m gamma a q^2 / (r^2 - t_m a^2)
        for (int m = 0; m < R.nline; ++m) {
            const double dm = r2 - R.line_t[m] * R.a2;
            const double cl = -l * R.line_c[m] * R.gamma * R.a * q * q / (dm * dm);
            gx += cl * x; gy += cl * y; gz += cl * z;
            gq += l * R.line_c[m] * R.gamma * R.a * q / dm;
        }
    }
    if (R.geom == 1 && R.Qc != 0.0) {
        const double rn = sqrt(r2);
        const double ir3 = 1.0 / (r2 * rn);
        gx += -l * R.Qc * q * x * ir3; gy += -l * R.Qc * q * y * ir3; gz += -l * R.Qc * q * z * ir3;
        gq += l * R.Qc / rn;
    }
    dEdr[3 * (size_t)i] = gx; dEdr[3 * (size_t)i + 1] = gy; dEdr[3 * (size_t)i + 2] = gz;
    dEdq[i] = gq;
}

__global__ void __launch_bounds__(256) k_zero(double* p, size_t n) {
    for (size_t k = blockIdx.x * (size_t)blockDim.x + threadIdx.x; k < n; k += (size_t)gridDim.x * blockDim.x)
        p[k] = 0.0;
}

template <bool LINES, bool F32>
void start_mc(hipStream_t s, Rep* reps, const McArgs& a, int grid, int wide) {
    if (wide) hipLaunchKernelGGL((k_mc<kMcBlock, LINES, F32>), dim3(grid), dim3(kMcBlock), 0, s, reps, a);
    else hipLaunchKernelGGL((k_mc<kMcBlockBatch, LINES, F32>), dim3(grid), dim3(kMcBlockBatch), 0, s, reps, a);
}
void run_mc(hipStream_t s, Rep* reps, const McArgs& a, int grid, int wide) {
    // handles with line images or a single-precision far field take the instantiations with
    // their steps; the others keep the registers of the plain kernel
    if (a.lines) {
        if (a.far32) start_mc<true, true>(s, reps, a, grid, wide);
        else start_mc<true, false>(s, reps, a, grid, wide);
    } else {
        if (a.far32) start_mc<false, true>(s, reps, a, grid, wide);
        else start_mc<false, false>(s, reps, a, grid, wide);
    }
}
template <bool F32>
void start_mcb(hipStream_t s, Rep* reps, const McArgs& a, int grid, int wide) {
    if (wide) hipLaunchKernelGGL((k_mcb<kMcBlock, F32>), dim3(grid), dim3(kMcBlock), 0, s, reps, a);
    else hipLaunchKernelGGL((k_mcb<kMcBlockBatch, F32>), dim3(grid), dim3(kMcBlockBatch), 0, s, reps, a);
}
void run_mcb(hipStream_t s, Rep* reps, const McArgs& a, int grid, int wide) {
    if (a.far32) start_mcb<true>(s, reps, a, grid, wide);
    else start_mcb<false>(s, reps, a, grid, wide);
}
void run_move(hipStream_t s, Rep* reps, int r, const MoveIO& in, MoveIO* io, int lines, int far32) {
    const dim3 grid(1), block(kMcBlock);
    if (lines) {
        if (far32) hipLaunchKernelGGL((k_move<true, true>), grid, block, 0, s, reps, r, in, io);
        else hipLaunchKernelGGL((k_move<true, false>), grid, block, 0, s, reps, r, in, io);
    } else {
        if (far32) hipLaunchKernelGGL((k_move<false, true>), grid, block, 0, s, reps, r, in, io);
        else hipLaunchKernelGGL((k_move<false, false>), grid, block, 0, s, reps, r, in, io);
    }
}
// Line images of the multiple-image model (one thread per ion, after k_energy): an
// ion's own line images stay in its traversal as sources, so each is taken back out of
// its potential and energy term where the traversal met it (walk_value).  The ion's
// energy with its own line images, 1/2 q sum_m c_m q_K / |r - t_m r_K|, is added.
__global__ void __launch_bounds__(256) k_eline(Rep* reps, int r, double* phi, double* eterm) {
    const Rep& R = reps[r];
    const int ion = blockIdx.x * blockDim.x + threadIdx.x;
    if (ion >= R.n) return;
    const double4 si = R.src[ion];
    double sub = 0.0;
    for (int m = 0; m < R.nline; ++m) {
        const double4 sc = R.src[2 * R.n + m * R.n + ion];
        int bad = 0;
        double v = walk_value(R, sc, si.x, si.y, si.z, bad);
        if (bad) { reps[r].err_detail = kErrPathCell; v = __builtin_nan(""); }
        sub += sc.w * v;
    }
    const double r2 = si.x * si.x + si.y * si.y + si.z * si.z;
    double self = 0.0;  // own line images: c_m q_K at t_m r_K, |r - t_m r_K| = (r^2 - t_m a^2) / r
    for (int m = 0; m < R.nline; ++m) self += R.line_c[m] * R.gamma * R.a * si.w / (r2 - R.line_t[m] * R.a2);
    if (phi) phi[ion] -= sub;
    eterm[ion] += 0.5 * si.w * (self - sub);
}

// Ions per group of the energy traversal: 16 once that fills the chip, fewer (more workgroups)
// for small systems; 4 only as long as all its workgroups run at once (energy_groups_per_cu on
// each of 256 CUs: up to 2,048 ions in FP64 from order 4 on, 4,096 in single precision up to order 4).
// (2,500 ions, p = 4: 52 us in groups of 4, where the last 113 of 625 run alone.)
// Measured with 4 / 8 / 16: 500 ions 39 / 44 / 53 us, 2,000 43 / 47 / 61,
// 4,500 92 / 79 / 85, 10,000 176 / 139 / 147, 30,000 474 / 326 / 280, 100,000 1558 / 1068 / 898.
// Single precision, 2,500 ions (p = 4, theta = 0.5, leaf 8): 51.5 us in groups of 8 with two
// workgroups a CU, 42.4 in groups of 4 with four.
int energy_group_log2(int n, int far32) {
    return n >= 16384 ? 4 : (n > 4 * 256 * energy_groups_per_cu(far32 != 0) ? 3 : 2);
}

void run_energy(hipStream_t s, Rep* reps, int r, int n, double* phi, double* eterm, int max_grid, int nline, int far32) {
    const int lg = energy_group_log2(n, far32);
    int grid = (n + (1 << lg) - 1) >> lg;
    if (max_grid > 0 && grid > max_grid) grid = max_grid;
    if (far32) hipLaunchKernelGGL(k_energy<true>, dim3(grid), dim3(kGroupBlock), 0, s, reps, r, lg, phi, eterm);
    else if (kEnergyTwice && n >= kEnergyW3Min)
        hipLaunchKernelGGL((k_energy<false, kEnergyTwice ? 3 : 2>), dim3(grid), dim3(kGroupBlock), 0, s, reps, r, lg, phi, eterm);
    else hipLaunchKernelGGL(k_energy<false>, dim3(grid), dim3(kGroupBlock), 0, s, reps, r, lg, phi, eterm);
    if (nline > 0) hipLaunchKernelGGL(k_eline, dim3((n + 255) / 256), dim3(256), 0, s, reps, r, phi, eterm);
}
void run_grad(hipStream_t s, Rep* reps, int r, const GradWork& w, double* dEdr, double* dEdq, double* eterm,
              int max_grid) {
    // L and G are adjacent in the workspace
    const size_t nz = (size_t)(w.G - (double4*)w.L) * 4 + 4 * (size_t)w.nsrc;
    hipLaunchKernelGGL(k_zero, dim3((unsigned)std::min<size_t>(4096, (nz + 255) / 256)), dim3(256), 0, s, w.L, nz);
    int ggrid = (w.n + kGT - 1) / kGT;
    if (max_grid > 0 && ggrid > max_grid) ggrid = max_grid;
    hipLaunchKernelGGL(k_grad, dim3(ggrid), dim3(kGroupBlock), 0, s, reps, r, w.L, w.G, w.Gt, eterm, w.fcell);
    hipLaunchKernelGGL(k_gflag, dim3((w.n + 255) / 256), dim3(256), 0, s, reps, r, (const int*)w.fcell, w.G,
                       w.Gt, eterm);
    if (w.nline > 0)
        hipLaunchKernelGGL(k_gline, dim3((w.n + 255) / 256), dim3(256), 0, s, reps, r, w.G, w.Gt, eterm);
    hipLaunchKernelGGL(k_adj_down, dim3((w.nsrc + 255) / 256), dim3(256), 0, s, (const Rep*)reps, r,
                       (const double*)w.L, w.G);
    hipLaunchKernelGGL(k_chain, dim3((w.n + 255) / 256), dim3(256), 0, s, (const Rep*)reps, r,
                       (const double4*)w.G, (const double4*)w.Gt, dEdr, dEdq);
}

// Expansion rows from the moments: one thread per (cell, row place).
__global__ void __launch_bounds__(256) k_expand(Rep* reps, const int* list) {
    const Rep& R = reps[list ? list[blockIdx.y] : blockIdx.y];
    if (R.status) return;
    const long long items = (long long)R.ncell * HSTR;
    for (long long it = blockIdx.x * 256ll + threadIdx.x; it < items; it += (long long)gridDim.x * 256) {
        const int c = (int)(it / HSTR), k = (int)(it % HSTR);
        double v = 0.0;
        if (k < NH) {
            const double* M = R.M + (size_t)c * MSTR;
            for (int e = c_hrows.start[k]; e < c_hrows.start[k + 1]; ++e) v = fma(c_hrows.coef[e], M[c_hrows.term[e]], v);
        } else if (k < NH + 3) {
            const double4 g = R.cgeo[c];
            v = k == HCEN ? g.x : (k == HCEN + 1 ? g.y : g.z);
        }
        R.H[(size_t)c * HSTR + k] = v;
    }
}

void run_expand(hipStream_t s, int nrep, Rep* reps, const int* list, int max_ncell) {
    const long long blocks = ((long long)max_ncell * HSTR + 255) / 256;
    hipLaunchKernelGGL(k_expand, dim3((unsigned)std::max(1ll, std::min(blocks, 8192ll)), nrep), dim3(256), 0, s, reps,
                       list);
}

// Phase timers of the batched kernel (a build with -DBHMC_PHASE_TIMERS): ticks of the
// constant clock per phase, then rounds and moves; reset after reading if asked.
int read_phases(unsigned long long* out, int n, int reset) {
#ifdef BHMC_PHASE_TIMERS
    unsigned long long v[kNumPhases];
    if (hipMemcpyFromSymbol(v, HIP_SYMBOL(g_phase), sizeof(v)) != hipSuccess) return -1;
    for (int k = 0; k < n && k < kNumPhases; ++k) out[k] = v[k];
    if (reset) {
        for (int k = 0; k < kNumPhases; ++k) v[k] = 0;
        if (hipMemcpyToSymbol(HIP_SYMBOL(g_phase), v, sizeof(v)) != hipSuccess) return -1;
    }
    return kNumPhases;
#else
    (void)out; (void)n; (void)reset;
    return 0;
#endif
}

const EvalOps kOps = {run_mc, run_mcb, kBM, run_expand, run_move, run_energy, run_grad, read_phases};

}  // namespace BHMC_NS

const EvalOps* BHMC_CAT(eval_ops_p, BHMC_P)() { return &BHMC_NS::kOps; }

}  // namespace bhmc
