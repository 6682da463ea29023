// asm_kernels.hip -- element-by-element assembly into CSR on gfx950.
//
// Section 4.2 / Listing 1 of the paper: an outer loop over elements and an
// inner loop over Gauss points and node pairs accumulating the elemental
// matrix from shape functions and the Jacobian weight, then a scatter into
// CSR.  Section 4.3 packs elements so that a SIMD unit processes several at
// once.  gfx950 form:
//
//   * matrix operators of a HEX08 mesh: owner groups (k_own), each CSR row
//     computed whole by one work-group and written once (k_own_copies: those of
//     another type's mesh in an order of poor locality);
//   * matrix operators of the other meshes and the element-vector passes:
//     blocks of <= 64 spatially compact elements of one type, a block's row
//     images (or nodal sums) to its own place in a work array, and a gather
//     that adds them row by row (k_part, k_vec);
//   * without the work array, or asked for by the upload (as the serving
//     runtime does), the coloured form (k_assemble): the CSR rows a block
//     touches live in an LDS image, initialised from HBM (or zero for the
//     first block to touch a row) and written back once; blocks of one colour
//     share no node, so a launch per (colour, element type) needs no atomics
//     in HBM.
// In all three the nodal fields are staged in LDS (structure of arrays, so that
// lanes reading different nodes hit different banks), a TET04, PYR05 or PEN06
// element is one lane, a HEX08 block two waves of 4 matrix rows each (under
// 256 registers a wave, so that two share each SIMD), and the sums in LDS run
// conflict-free in an order that the plan fixes: results are bitwise
// reproducible.
//
// Precision: FP64, or (mixed) FP32 Gauss-point products and elemental sums
// with the Jacobian, det J, J^-1 and the CSR accumulation in FP64.
#include <algorithm>
#include <cstring>
#include <type_traits>

#include "internal.h"
#include "plan.h"

namespace feasm {
namespace {

constexpr int OP_MOM = FE_OP_MOMENTUM, OP_SCA = FE_OP_SCALAR, OP_POI = FE_OP_POISSON;
// element-vector passes of the explicit step (no matrix): residual + lumped
// mass, pressure gradient, divergence right-hand side
constexpr int OP_RES = kOpResidual, OP_GRD = kOpGradient, OP_DIV = kOpDivergence, OP_SRS = kOpScalarResidual;

// Trilinear hexahedron, 2x2x2 Gauss rule (points xi fastest, weights 1).
struct Hex {
    static constexpr int NEN = 8, NG = 8;
    static constexpr double kG = 0.57735026918962576451;   // 1/sqrt(3)
    __host__ __device__ static constexpr int sx(int a) { return ((a & 3) == 1 || (a & 3) == 2) ? 1 : -1; }
    __host__ __device__ static constexpr int sy(int a) { return (a & 3) >= 2 ? 1 : -1; }
    __host__ __device__ static constexpr int sz(int a) { return a >= 4 ? 1 : -1; }
    __host__ __device__ static constexpr double gp(int g, int d) { return ((g >> d) & 1) ? kG : -kG; }
    __host__ __device__ static constexpr double w(int) { return 1.0; }
    __host__ __device__ static constexpr double N(int g, int a)
    {
        return 0.125 * (1.0 + sx(a) * gp(g, 0)) * (1.0 + sy(a) * gp(g, 1)) * (1.0 + sz(a) * gp(g, 2));
    }
    static constexpr bool kRolled = true, kSparse = false;
    __host__ __device__ static constexpr double dN(int g, int a, int j)
    {
        return j == 0 ? 0.125 * sx(a) * (1.0 + sy(a) * gp(g, 1)) * (1.0 + sz(a) * gp(g, 2))
             : j == 1 ? 0.125 * sy(a) * (1.0 + sx(a) * gp(g, 0)) * (1.0 + sz(a) * gp(g, 2))
                      : 0.125 * sz(a) * (1.0 + sx(a) * gp(g, 0)) * (1.0 + sy(a) * gp(g, 1));
    }
};

// Shape-function values and reference gradients at the Gauss points of an
// element type, for the rolled Gauss loop (read from constant memory).
template <class EL> struct RefTables {
    double N[EL::NG][EL::NEN];        // N[g][a]
    double dN[EL::NG][EL::NEN][3];    // dN[g][a][j]
};

template <class EL> constexpr RefTables<EL> make_tables()
{
    RefTables<EL> t{};
    for (int g = 0; g < EL::NG; ++g)
        for (int a = 0; a < EL::NEN; ++a) {
            t.N[g][a] = EL::N(g, a);
            for (int j = 0; j < 3; ++j) t.dN[g][a][j] = EL::dN(g, a, j);
        }
    return t;
}

__constant__ RefTables<Hex> kHexTab = make_tables<Hex>();

// Linear tetrahedron, 4-point degree-2 rule (weights 1/24).
struct Tet {
    static constexpr int NEN = 4, NG = 4;
    static constexpr bool kRolled = false, kSparse = true;
    __device__ static constexpr double Nv(int g, int a) { return N(g, a); }
    __device__ static constexpr double dNv(int g, int a, int j) { return dN(g, a, j); }
    static constexpr double kA = 0.13819660112501051518;   // (5 - sqrt5)/20
    static constexpr double kB = 0.58541019662496845446;   // 1 - 3a
    __host__ __device__ static constexpr double w(int) { return 1.0 / 24.0; }
    __host__ __device__ static constexpr double N(int g, int a) { return a == g ? kB : kA; }
    __host__ __device__ static constexpr double dN(int, int a, int j) { return a == 0 ? -1.0 : (a == j + 1 ? 1.0 : 0.0); }
};

// Linear prism: triangle (0,0),(1,0),(0,1) x zeta in [-1,1], nodes 0-2 at
// zeta = -1 and 3-5 above them; N_a = L_i (1 -+ zeta)/2 with the barycentric
// L = (1-xi-eta, xi, eta).  Rule: the degree-2 triangle points (1/6,1/6),
// (2/3,1/6), (1/6,2/3) x Gauss-Legendre +-1/sqrt3 (point g: triangle point
// g % 3, zeta side g / 3), weights 1/6.
struct Pen {
    static constexpr int NEN = 6, NG = 6;
    static constexpr bool kRolled = true, kSparse = false;
    // dN(g, a, j) is zero at every point
    __host__ __device__ static constexpr bool zero(int a, int j) { return j < 2 && a % 3 != 0 && a % 3 != j + 1; }
    static constexpr double kG = 0.57735026918962576451;
    __host__ __device__ static constexpr double px(int g) { return g % 3 == 1 ? 2.0 / 3.0 : 1.0 / 6.0; }
    __host__ __device__ static constexpr double py(int g) { return g % 3 == 2 ? 2.0 / 3.0 : 1.0 / 6.0; }
    __host__ __device__ static constexpr double pz(int g) { return g >= 3 ? kG : -kG; }
    __host__ __device__ static constexpr double bary(int i, int g)
    {
        return i == 0 ? 1.0 - px(g) - py(g) : i == 1 ? px(g) : py(g);
    }
    __host__ __device__ static constexpr double side(int a) { return a >= 3 ? 1.0 : -1.0; }
    __host__ __device__ static constexpr double w(int) { return 1.0 / 6.0; }
    __host__ __device__ static constexpr double N(int g, int a)
    {
        return bary(a % 3, g) * 0.5 * (1.0 + side(a) * pz(g));
    }
    __host__ __device__ static constexpr double dN(int g, int a, int j)
    {
        // d bary / d xi = (-1, 1, 0), d bary / d eta = (-1, 0, 1)
        return j == 2 ? 0.5 * side(a) * bary(a % 3, g)
                      : (a % 3 == 0 ? -1.0 : (a % 3 == j + 1 ? 1.0 : 0.0)) * 0.5 * (1.0 + side(a) * pz(g));
    }
};

// Pyramid on the base [-1,1]^2 at zeta = 0 (nodes 0-3 at (-,-), (+,-), (+,+),
// (-,+)) with the apex, node 4, at (0,0,1).  Rational basis, m = 1 - zeta:
// N_a = (m + sx xi)(m + sy eta) / (4m), N_4 = zeta.  Rule: conical product,
// (xi, eta) = m (+-1/sqrt3, +-1/sqrt3) and zeta at the 2-point Gauss-Jacobi
// nodes for the weight (1-zeta)^2 on [0,1], 1/3 -+ sqrt10/15, with weights
// 1/6 +- sqrt10/48 (point g: xi side bit 0, eta side bit 1, zeta node bit 2).
struct Pyr {
    static constexpr int NEN = 5, NG = 8;
    static constexpr bool kRolled = true, kSparse = false;
    static constexpr double kG = 0.57735026918962576451;    // 1/sqrt(3)
    static constexpr double kR = 3.16227766016837933200;    // sqrt(10)
    __host__ __device__ static constexpr double pz(int g) { return (g & 4) ? 1.0 / 3.0 + kR / 15.0 : 1.0 / 3.0 - kR / 15.0; }
    __host__ __device__ static constexpr double pm(int g) { return 1.0 - pz(g); }
    __host__ __device__ static constexpr double px(int g) { return ((g & 1) ? kG : -kG) * pm(g); }
    __host__ __device__ static constexpr double py(int g) { return ((g & 2) ? kG : -kG) * pm(g); }
    __host__ __device__ static constexpr double sx(int a) { return (a == 1 || a == 2) ? 1.0 : -1.0; }
    __host__ __device__ static constexpr double sy(int a) { return a >= 2 ? 1.0 : -1.0; }
    __host__ __device__ static constexpr double w(int g) { return (g & 4) ? 1.0 / 6.0 - kR / 48.0 : 1.0 / 6.0 + kR / 48.0; }
    __host__ __device__ static constexpr double N(int g, int a)
    {
        return a == 4 ? pz(g) : (pm(g) + sx(a) * px(g)) * (pm(g) + sy(a) * py(g)) / (4.0 * pm(g));
    }
    __host__ __device__ static constexpr double dN(int g, int a, int j)
    {
        return a == 4 ? (j == 2 ? 1.0 : 0.0)
             : j == 0 ? sx(a) * (pm(g) + sy(a) * py(g)) / (4.0 * pm(g))
             : j == 1 ? sy(a) * (pm(g) + sx(a) * px(g)) / (4.0 * pm(g))
                      : (sx(a) * sy(a) * px(g) * py(g) - pm(g) * pm(g)) / (4.0 * pm(g) * pm(g));
    }
};

__constant__ RefTables<Pen> kPenTab = make_tables<Pen>();
__constant__ RefTables<Pyr> kPyrTab = make_tables<Pyr>();

struct KArgs {
    const double *X;
    const int32_t *blk_elem_ptr, *blk_node_ptr, *blk_nodes, *blk_rdesc, *blk_rowstart, *color_blk;
    const uint8_t *blk_nphase, *elem_off, *elem_phase;
    const uint16_t *elem_lnode;
    int64_t N, E;
    int off_stride;           // bytes of elem_off per element
    int form;                 // residual pass: FE_FORM_* operator variants
    const double *u, *rho, *mu, *Y, *p;
    double dt, Dk;
    double *values, *rhs;
    double *blk_mindet;       // [nblk] per-block smallest det J
    long long *blk_bad;       // [nblk] per-block first bad element (mesh index) or -1
    int blk_offset;
};

template <int OP> struct OpTraits;
template <> struct OpTraits<FE_OP_MOMENTUM> { static constexpr int NF = 8, NRHS = 3; };
template <> struct OpTraits<FE_OP_SCALAR> { static constexpr int NF = 8, NRHS = 1; };
template <> struct OpTraits<FE_OP_POISSON> { static constexpr int NF = 7, NRHS = 1; };
template <> struct OpTraits<kOpResidual> { static constexpr int NF = 8, NRHS = 4; };    // r_x, r_y, r_z, lumped mass
template <> struct OpTraits<kOpGradient> { static constexpr int NF = 4, NRHS = 3; };    // x, y, z, p
template <> struct OpTraits<kOpDivergence> { static constexpr int NF = 7, NRHS = 1; };
template <> struct OpTraits<kOpScalarResidual> { static constexpr int NF = 8, NRHS = 2; };   // r, lumped mass

// Waves per element block: a HEX08 element's 8 rows are split between two
// waves (4 rows each) so that a wave needs <= 256 registers and two blocks'
// waves share each SIMD; a TET04 element stays on one lane.
template <class EL> struct Split { static constexpr int W = EL::NEN == 8 ? 2 : 1; };

__device__ inline void lds_add(double *p, double v)
{
    __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

template <class EL> __device__ inline double RefN(int g, int a);
template <class EL> __device__ inline double RefdN(int g, int a, int j);
template <> __device__ inline double RefN<Hex>(int g, int a) { return kHexTab.N[g][a]; }
template <> __device__ inline double RefdN<Hex>(int g, int a, int j) { return kHexTab.dN[g][a][j]; }
template <> __device__ inline double RefN<Tet>(int g, int a) { return Tet::N(g, a); }
template <> __device__ inline double RefdN<Tet>(int g, int a, int j) { return Tet::dN(g, a, j); }
template <> __device__ inline double RefN<Pen>(int g, int a) { return kPenTab.N[g][a]; }
template <> __device__ inline double RefdN<Pen>(int g, int a, int j) { return kPenTab.dN[g][a][j]; }
template <> __device__ inline double RefN<Pyr>(int g, int a) { return kPyrTab.N[g][a]; }
template <> __device__ inline double RefdN<Pyr>(int g, int a, int j) { return kPyrTab.dN[g][a][j]; }

// Whether d = dN(g, a, j) counts (a compile-time answer: its table may be read
// at run time).
template <class EL> __device__ constexpr bool has_dN(int a, int j, double d)
{
    if constexpr (EL::NEN == 6) return !EL::zero(a, j);
    else return !EL::kSparse || d != 0.0;
}

// FP64 Poisson matrices of the types with an element on one lane: the entries
// on and above the diagonal are summed, the others are theirs (PEN06: 63 of 108
// products a point; with the zeros above 57^3 takes 113 us instead of 126).
template <class EL, int OP, class Q, int RA>
constexpr bool kSymmetric = OP == OP_POI && RA == EL::NEN && sizeof(Q) == 8;

// One Gauss point for rows [a0, a0 + RA) of the elemental matrix.
// Geometry in FP64 (from the LDS-staged nodal data), products in Q.
//   MOM/SCA: A_ab += N_a s_b + wk grad N_a . grad N_b,
//            s_b = rho dV (N_b / dt + u . grad N_b), wk = mu dV or rho D dV;
//            B_a += rho dV / dt N_a f, f = u (MOM) or Y (SCA).
//   POI    : A_ab += dV grad N_a . grad N_b,
//            B_a += dV / dt grad N_a . (rho u).
// Geometry of one element kept in registers for the Gauss loop: HEX08 the
// trilinear coefficients c1..c7 of x(xi), the other types the node coordinates.
template <class EL> struct Geo { double v[EL::NEN == 8 ? 7 : EL::NEN][3]; };

template <class EL>
__device__ __forceinline__ void load_geo(const double *nd, int T, const int (&ln)[EL::NEN], Geo<EL> &G)
{
    constexpr int NEN = EL::NEN;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        double x[NEN];
#pragma unroll
        for (int a = 0; a < NEN; ++a) x[a] = nd[i * T + ln[a]];
        if (NEN == 8) {
#pragma unroll
            for (int m = 1; m < 8; ++m) {
                double sum = 0.0;
#pragma unroll
                for (int a = 0; a < 8; ++a) {
                    const int sx = Hex::sx(a), sy = Hex::sy(a), sz = Hex::sz(a);
                    const int sgn = m == 1 ? sx : m == 2 ? sy : m == 3 ? sz : m == 4 ? sx * sy
                                  : m == 5 ? sy * sz : m == 6 ? sx * sz : sx * sy * sz;
                    sum = sgn > 0 ? sum + x[a] : sum - x[a];
                }
                G.v[m - 1][i] = 0.125 * sum;
            }
        } else {
#pragma unroll
            for (int a = 0; a < NEN; ++a) G.v[a][i] = x[a];
        }
    }
}

// A Jacobian's determinant (returned) and inverse.
__device__ __forceinline__ double invert_jacobian(const double (&J)[3][3], double (&Ji)[3][3])
{
    const double c00 = J[1][1] * J[2][2] - J[1][2] * J[2][1];
    const double c01 = J[1][2] * J[2][0] - J[1][0] * J[2][2];
    const double c02 = J[1][0] * J[2][1] - J[1][1] * J[2][0];
    const double det = J[0][0] * c00 + J[0][1] * c01 + J[0][2] * c02;
    const double id = 1.0 / det;
    Ji[0][0] = c00 * id;
    Ji[1][0] = c01 * id;
    Ji[2][0] = c02 * id;
    Ji[0][1] = (J[0][2] * J[2][1] - J[0][1] * J[2][2]) * id;
    Ji[1][1] = (J[0][0] * J[2][2] - J[0][2] * J[2][0]) * id;
    Ji[2][1] = (J[0][1] * J[2][0] - J[0][0] * J[2][1]) * id;
    Ji[0][2] = (J[0][1] * J[1][2] - J[0][2] * J[1][1]) * id;
    Ji[1][2] = (J[0][2] * J[1][0] - J[0][0] * J[1][2]) * id;
    Ji[2][2] = (J[0][0] * J[1][1] - J[0][1] * J[1][0]) * id;
    return det;
}

// Jacobian of the map at Gauss point g, its determinant (returned) and inverse.
template <class EL>
__device__ __forceinline__ double jacobian_inverse(int g, const Geo<EL> &GE, double (&Ji)[3][3])
{
    constexpr int NEN = EL::NEN;
    const auto &geo = GE.v;
    double J[3][3];
    if (NEN == 8) {
        // x(xi) = c0 + c1 xi + c2 eta + c3 zeta + c4 xi eta + c5 eta zeta + c6 xi zeta
        //         + c7 xi eta zeta (geo[m-1] = c_m): each Jacobian column is 3 FMAs.
        const double xi = (g & 1) ? Hex::kG : -Hex::kG;
        const double et = (g & 2) ? Hex::kG : -Hex::kG;
        const double ze = (g & 4) ? Hex::kG : -Hex::kG;
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            J[i][0] = geo[0][i] + et * geo[3][i] + ze * geo[5][i] + (et * ze) * geo[6][i];
            J[i][1] = geo[1][i] + xi * geo[3][i] + ze * geo[4][i] + (xi * ze) * geo[6][i];
            J[i][2] = geo[2][i] + et * geo[4][i] + xi * geo[5][i] + (xi * et) * geo[6][i];
        }
    } else {
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                double s = 0.0;
#pragma unroll
                for (int a = 0; a < NEN; ++a) {
                    const double d = RefdN<EL>(g, a, j);
                    if (has_dN<EL>(a, j, d)) s += geo[a][i] * d;
                }
                J[i][j] = s;
            }
    }
    return invert_jacobian(J, Ji);
}

// One Gauss point of an element-vector pass for rows [A0, A0 + RA), FP64,
// from the physical gradients dN and dV = w det J:
//   OP_RES: B_i[a] -= dV (rho N_a (u . grad u_i) + mu grad N_a . grad u_i), i < 3,
//           B_3[a] += dV rho N_a (lumped mass); form FE_FORM_FULL_STRESS adds
//           mu (d u_j / d x_i)(d N_a / d x_j) (the viscous term 2 mu eps(u)),
//           FE_FORM_EMAC adds rho N_a (div u) u_i (Eq. (1)'s convective form
//           at the Gauss point);
//   OP_GRD: B_j[a] += dV N_a (grad p)_j;
//   OP_DIV: B_0[a] += dV / dt grad N_a . (rho u);
//   OP_SRS: B_0[a] -= dV rho (N_a (u . grad Y) + D grad N_a . grad Y),
//           B_1[a] += dV rho N_a (Y in slot 7, D = Dk).
// Fields in LDS: x, y, z, then u_x, u_y, u_z, rho, mu (OP_GRD: p in slot 3).
template <class EL, int OP, int RA, int A0>
__device__ __forceinline__ void element_vector_point(int g, const double *nd, int T, const int (&ln)[EL::NEN],
                                                     const double (&dN)[EL::NEN][3], double dV,
                                                     double (&B)[OpTraits<OP>::NRHS][RA], double inv_dt,
                                                     int form, double Dk)
{
    constexpr int NEN = EL::NEN;
    if constexpr (OP == OP_SRS) {
        double rg = 0.0, ug[3] = {0.0, 0.0, 0.0}, gy[3] = {0.0, 0.0, 0.0};
#pragma unroll
        for (int b = 0; b < NEN; ++b) {
            const double Nb = RefN<EL>(g, b), yb = nd[7 * T + ln[b]];
            rg += Nb * nd[6 * T + ln[b]];
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                ug[i] += Nb * nd[(3 + i) * T + ln[b]];
                gy[i] += dN[b][i] * yb;
            }
        }
        const double adv = ug[0] * gy[0] + ug[1] * gy[1] + ug[2] * gy[2], w = dV * rg;
#pragma unroll
        for (int r = 0; r < RA; ++r) {
            const int a = A0 + r;
            const double Na = RefN<EL>(g, a);
            const double dif = dN[a][0] * gy[0] + dN[a][1] * gy[1] + dN[a][2] * gy[2];
            B[0][r] -= w * (Na * adv + Dk * dif);
            B[1][r] += w * Na;
        }
    } else if constexpr (OP == OP_GRD) {
        double gp[3] = {0.0, 0.0, 0.0};
#pragma unroll
        for (int b = 0; b < NEN; ++b) {
            const double pb = nd[3 * T + ln[b]];
#pragma unroll
            for (int j = 0; j < 3; ++j) gp[j] += dN[b][j] * pb;
        }
#pragma unroll
        for (int r = 0; r < RA; ++r) {
            const double wn = dV * RefN<EL>(g, A0 + r);
#pragma unroll
            for (int j = 0; j < 3; ++j) B[j][r] += wn * gp[j];
        }
    } else {
        double rg = 0.0, mg = 0.0, ug[3] = {0.0, 0.0, 0.0}, gu[3][3] = {};
#pragma unroll
        for (int b = 0; b < NEN; ++b) {
            const double Nb = RefN<EL>(g, b);
            rg += Nb * nd[6 * T + ln[b]];
            if (OP == OP_RES) mg += Nb * nd[7 * T + ln[b]];
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                const double ub = nd[(3 + i) * T + ln[b]];
                ug[i] += Nb * ub;
                if (OP == OP_RES) {
#pragma unroll
                    for (int j = 0; j < 3; ++j) gu[i][j] += dN[b][j] * ub;   // d u_i / d x_j
                }
            }
        }
        if constexpr (OP == OP_RES) {
            const bool full = (form & FE_FORM_FULL_STRESS) != 0, emac = (form & FE_FORM_EMAC) != 0;
            const double divu = gu[0][0] + gu[1][1] + gu[2][2];
#pragma unroll
            for (int r = 0; r < RA; ++r) {
                const int a = A0 + r;
                const double wr = dV * rg * RefN<EL>(g, a), wm = dV * mg;
#pragma unroll
                for (int i = 0; i < 3; ++i) {
                    double adv = ug[0] * gu[i][0] + ug[1] * gu[i][1] + ug[2] * gu[i][2];
                    double vis = dN[a][0] * gu[i][0] + dN[a][1] * gu[i][1] + dN[a][2] * gu[i][2];
                    if (full) vis += dN[a][0] * gu[0][i] + dN[a][1] * gu[1][i] + dN[a][2] * gu[2][i];
                    if (emac) adv += divu * ug[i];
                    B[i][r] -= wr * adv + wm * vis;
                }
                B[3][r] += wr;
            }
        } else {
            const double f0 = rg * ug[0], f1 = rg * ug[1], f2 = rg * ug[2], w = dV * inv_dt;
#pragma unroll
            for (int r = 0; r < RA; ++r) {
                const int a = A0 + r;
                B[0][r] += w * (dN[a][0] * f0 + dN[a][1] * f1 + dN[a][2] * f2);
            }
        }
    }
}

template <class EL, int OP, class Q, int RA, int A0, class FT>
__device__ __forceinline__ void gauss_point(int g, const Geo<EL> &GE, const double *nd, const FT *nf, int T,
                                            const int (&ln)[EL::NEN],
                                            Q (&A)[RA][EL::NEN], Q (&B)[OpTraits<OP>::NRHS][RA], double &mindet,
                                            double inv_dt, double Dk, int form)
{
    constexpr int NEN = EL::NEN;
    double Ji[3][3];
    const double det = jacobian_inverse<EL>(g, GE, Ji);
    mindet = fmin(mindet, det);
    // physical gradients grad N_a = J^-T grad_ref N_a (all nodes: needed for columns)
    Q dN[NEN][3];
#pragma unroll
    for (int a = 0; a < NEN; ++a)
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            double s = 0.0;
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                const double d = RefdN<EL>(g, a, j);
                if (has_dN<EL>(a, j, d)) s += Ji[j][i] * d;
            }
            dN[a][i] = Q(s);
        }
    if constexpr (OP >= OP_RES) {
        element_vector_point<EL, OP, RA, A0>(g, nd, T, ln, dN, EL::w(g) * det, B, inv_dt, form, Dk);
    } else {
        // nf: the fields after x, y, z (u_x, u_y, u_z, rho, mu / Y), interpolated
        // in their staged precision FT
        FT rg = 0, fg = 0, ug0 = 0, ug1 = 0, ug2 = 0;
#pragma unroll
        for (int a = 0; a < NEN; ++a) {
            const FT Na = FT(RefN<EL>(g, a));
            rg += Na * nf[3 * T + ln[a]];
            ug0 += Na * nf[0 * T + ln[a]];
            ug1 += Na * nf[1 * T + ln[a]];
            ug2 += Na * nf[2 * T + ln[a]];
            if (OP != OP_POI) fg += Na * nf[4 * T + ln[a]];
        }
        const double dV = EL::w(g) * det;
        if (OP == OP_POI) {
            const Q qdV = Q(dV), qi = Q(inv_dt);
            const Q f0 = Q(rg * ug0), f1 = Q(rg * ug1), f2 = Q(rg * ug2);
#pragma unroll
            for (int r = 0; r < RA; ++r) {
                const int a = A0 + r;
                const Q G0 = qdV * dN[a][0], G1 = qdV * dN[a][1], G2 = qdV * dN[a][2];
#pragma unroll
                for (int b = kSymmetric<EL, OP, Q, RA> ? r : 0; b < NEN; ++b)
                    A[r][b] += G0 * dN[b][0] + G1 * dN[b][1] + G2 * dN[b][2];
                B[0][r] += qi * (G0 * f0 + G1 * f1 + G2 * f2);
            }
        } else {
            const Q w1 = Q(dV) * Q(rg);
            const Q wk = (OP == OP_MOM) ? Q(dV) * Q(fg) : Q(dV) * (Q(rg) * Q(Dk));   // fg = mu (MOM) or Y (SCA)
            const Q qi = Q(inv_dt);
            const Q qu0 = Q(ug0), qu1 = Q(ug1), qu2 = Q(ug2);
            Q s[NEN];
#pragma unroll
            for (int b = 0; b < NEN; ++b)
                s[b] = w1 * (Q(RefN<EL>(g, b)) * qi + (qu0 * dN[b][0] + qu1 * dN[b][1] + qu2 * dN[b][2]));
#pragma unroll
            for (int r = 0; r < RA; ++r) {
                const int a = A0 + r;
                const Q Na = Q(RefN<EL>(g, a));
                const Q G0 = wk * dN[a][0], G1 = wk * dN[a][1], G2 = wk * dN[a][2];
#pragma unroll
                for (int b = 0; b < NEN; ++b) A[r][b] += Na * s[b] + (G0 * dN[b][0] + G1 * dN[b][1] + G2 * dN[b][2]);
                const Q wn = w1 * Na * qi;
                if (OP == OP_MOM) {
                    B[0][r] += wn * qu0;
                    B[1][r] += wn * qu1;
                    B[2][r] += wn * qu2;
                } else {
                    B[0][r] += wn * Q(fg);
                }
            }
        }
    }
}

// All Gauss points of one element for rows [A0, A0 + RA).  ln is taken by
// value: the loop makes its copy opaque at every point so that the nodal
// field reads are re-issued from LDS instead of being hoisted into registers.
template <class EL> struct Rows { int v[EL::NEN]; };

template <class EL, int OP, class Q, int RA, int A0, class FT = double>
__device__ __forceinline__ void gauss_loop(const Geo<EL> &GE, const double *nd, const FT *nf, int T, Rows<EL> rows,
                                           Q (&A)[RA][EL::NEN], Q (&B)[OpTraits<OP>::NRHS][RA], double &mindet,
                                           double inv_dt, double Dk, int form)
{
    constexpr int NEN = EL::NEN, NG = EL::NG;
    int ln[NEN];
#pragma unroll
    for (int a = 0; a < NEN; ++a) ln[a] = rows.v[a];
    if (EL::kRolled) {
#pragma unroll 1
        for (int g = 0; g < NG; ++g) {
#pragma unroll
            for (int a = 0; a < NEN; ++a) asm volatile("" : "+v"(ln[a]));
            gauss_point<EL, OP, Q, RA, A0, FT>(g, GE, nd, nf, T, ln, A, B, mindet, inv_dt, Dk, form);
        }
    } else {
#pragma unroll
        for (int g = 0; g < NG; ++g)
            gauss_point<EL, OP, Q, RA, A0, FT>(g, GE, nd, nf, T, ln, A, B, mindet, inv_dt, Dk, form);
    }
    if constexpr (kSymmetric<EL, OP, Q, RA>) {
#pragma unroll
        for (int r = 1; r < RA; ++r)
#pragma unroll
            for (int b = 0; b < r; ++b) A[r][b] = A[b][r];
    }
}

// gauss_loop of FE_OP_SCALAR for NS scalars at once (HEX08, rows 0-3): the points'
// geometry, gradients and s_b are computed once, and each scalar's sums are
// formed as gauss_point forms them.  Y_k in slot 7 + k, diffusivity D[k].
template <int NS, class Q, class FT>
__device__ __forceinline__ void scalars_loop(const Geo<Hex> &GE, const double *nd, const FT *nf, int T, Rows<Hex> rows,
                                             Q (&A)[NS][4][8], Q (&B)[NS][1][4], double &mindet, double inv_dt,
                                             const double (&D)[kOwnScalars])
{
    int ln[8];
#pragma unroll
    for (int a = 0; a < 8; ++a) ln[a] = rows.v[a];
#pragma unroll 1
    for (int g = 0; g < Hex::NG; ++g) {
#pragma unroll
        for (int a = 0; a < 8; ++a) asm volatile("" : "+v"(ln[a]));
        double Ji[3][3];
        const double det = jacobian_inverse<Hex>(g, GE, Ji);
        mindet = fmin(mindet, det);
        Q dN[8][3];
#pragma unroll
        for (int a = 0; a < 8; ++a)
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                double s = 0.0;
#pragma unroll
                for (int j = 0; j < 3; ++j) s += Ji[j][i] * RefdN<Hex>(g, a, j);
                dN[a][i] = Q(s);
            }
        FT rg = 0, ug0 = 0, ug1 = 0, ug2 = 0, fg[NS] = {};
#pragma unroll
        for (int a = 0; a < 8; ++a) {
            const FT Na = FT(RefN<Hex>(g, a));
            rg += Na * nf[3 * T + ln[a]];
            ug0 += Na * nf[0 * T + ln[a]];
            ug1 += Na * nf[1 * T + ln[a]];
            ug2 += Na * nf[2 * T + ln[a]];
#pragma unroll
            for (int k = 0; k < NS; ++k) fg[k] += Na * nf[(4 + k) * T + ln[a]];
        }
        const double dV = Hex::w(g) * det;
        const Q w1 = Q(dV) * Q(rg), qi = Q(inv_dt);
        const Q qu0 = Q(ug0), qu1 = Q(ug1), qu2 = Q(ug2);
        Q s[8];
#pragma unroll
        for (int b = 0; b < 8; ++b)
            s[b] = w1 * (Q(RefN<Hex>(g, b)) * qi + (qu0 * dN[b][0] + qu1 * dN[b][1] + qu2 * dN[b][2]));
#pragma unroll
        for (int k = 0; k < NS; ++k) {
            const Q wk = Q(dV) * (Q(rg) * Q(D[k]));
#pragma unroll
            for (int a = 0; a < 4; ++a) {
                const Q Na = Q(RefN<Hex>(g, a));
                const Q G0 = wk * dN[a][0], G1 = wk * dN[a][1], G2 = wk * dN[a][2];
#pragma unroll
                for (int b = 0; b < 8; ++b)
                    A[k][a][b] += Na * s[b] + (G0 * dN[b][0] + G1 * dN[b][1] + G2 * dN[b][2]);
                const Q wn = w1 * Na * qi;
                B[k][0][a] += wn * Q(fg[k]);
            }
        }
    }
}

// One work-group = one block of <= 64 elements = W waves.  Lane l computes
// rows [a0, a0 + RA) of element l mod 64 with a0 = (l / 64) * RA.
// The block body of every assembly and element-vector pass: block
// color_blk[blk_offset + wg] of the launch.  FORM >= 0 fixes the residual
// pass's operator variants at compile time; -1 reads them from the arguments.
template <class EL, int OP, class Q, int FORM>
__device__ __forceinline__ void assemble_block(const KArgs &k, int wg)
{
    constexpr int NEN = EL::NEN, NG = EL::NG, W = Split<EL>::W, RA = NEN / W, NT = 64 * W;
    constexpr int NF = OpTraits<OP>::NF, NRHS = OpTraits<OP>::NRHS;
    constexpr bool VEC = OP >= OP_RES;       // element-vector pass: no row image
    extern __shared__ double lds[];

    const int blk = k.color_blk[k.blk_offset + wg];
    const int e0 = k.blk_elem_ptr[blk], ne = k.blk_elem_ptr[blk + 1] - e0;
    const int n0 = k.blk_node_ptr[blk], T = k.blk_node_ptr[blk + 1] - n0;
    const int tid = threadIdx.x;
    const int el = tid & 63, wv = tid >> 6, a0 = wv * RA;
    const int64_t N = k.N;

    double *nd = lds;                        // [NF][T] nodal fields
    double *rimg = nd + NF * T;              // [NRHS][T] rhs image
    int *rdesc = (int *)(rimg + NRHS * T);   // [T] row descriptors
    double *img = (double *)(rdesc + T + (T & 1));   // 8-byte aligned row image (matrix passes)

    // Element data that depends only on the block: issue these loads first.
    const bool act = el < ne;
    const int e = e0 + (act ? el : 0);
    int ln[NEN];
#pragma unroll
    for (int a = 0; a < NEN; ++a) ln[a] = k.elem_lnode[(int64_t)a * k.E + e];
    // in-row offsets of this lane's rows: a multiple of 4 bytes from a 4-byte
    // boundary (off_stride is a multiple of 4, a0 * NEN is 0 or 32), padded
    // to whole words inside the element's slot
    constexpr int kOffWords = (RA * NEN + 3) / 4;
    uint32_t offw[kOffWords];
    if constexpr (!VEC) {
        const uint32_t *op = (const uint32_t *)(k.elem_off + (int64_t)e * k.off_stride + a0 * NEN);
#pragma unroll
        for (int q = 0; q < kOffWords; ++q) offw[q] = op[q];
    }
    const int ph = act ? (int)k.elem_phase[e] : -1;

    // 1. stage, one touched row per lane: nodal fields, rhs and the row's
    //    previous partial sums (zero for the first writer) into LDS.  Two
    //    dependent load rounds: the block's row tables, then fields + values.
    constexpr int kRowBatch = 32;   // columns loaded per batch (rows are <= 255)
    for (int t = tid; t < T; t += NT) {
        const int g = k.blk_nodes[n0 + t];
        const int rd = k.blk_rdesc[n0 + t];
        const int r0 = VEC ? 0 : k.blk_rowstart[n0 + t];   // matrix passes: the row in CSR
        const int len = VEC ? 0 : (rd >> 16) & 0xff, base = rd & 0xffff;
        const bool first = rd < 0;
        double f[NF + NRHS];
        f[0] = k.X[g];
        f[1] = k.X[N + g];
        f[2] = k.X[2 * N + g];
        if constexpr (OP == OP_GRD) {
            f[3] = k.p[g];
        } else {
            f[3] = k.u[g];
            f[4] = k.u[N + g];
            f[5] = k.u[2 * N + g];
            f[6] = k.rho[g];
            if (OP == OP_MOM || OP == OP_RES) f[7] = k.mu[g];
            if (OP == OP_SCA || OP == OP_SRS) f[7] = k.Y[g];
        }
#pragma unroll
        for (int r = 0; r < NRHS; ++r) f[NF + r] = first ? 0.0 : k.rhs[r * N + g];
        // matrix passes: the row's previous values, loaded before the LDS
        // writes below so that the loads overlap them
        double v[kRowBatch];
        if constexpr (!VEC) {
#pragma unroll
            for (int q = 0; q < kRowBatch; ++q) v[q] = (!first && q < len) ? k.values[r0 + q] : 0.0;
        }
#pragma unroll
        for (int q = 0; q < NF; ++q) nd[q * T + t] = f[q];
#pragma unroll
        for (int r = 0; r < NRHS; ++r) rimg[r * T + t] = f[NF + r];
        rdesc[t] = rd;
        if constexpr (!VEC) {
#pragma unroll
            for (int q = 0; q < kRowBatch; ++q)
                if (q < len) img[base + q] = v[q];
            for (int q = kRowBatch; q < len; ++q) img[base + q] = first ? 0.0 : k.values[r0 + q];
        }
    }
    __syncthreads();

    // 3. elemental matrix rows of this lane
    Q A[RA][NEN];
    Q B[NRHS][RA];
#pragma unroll
    for (int r = 0; r < RA; ++r) {
#pragma unroll
        for (int b = 0; b < NEN; ++b) A[r][b] = Q(0);
#pragma unroll
        for (int q = 0; q < NRHS; ++q) B[q][r] = Q(0);
    }
    double mindet = __builtin_huge_val();
    const double inv_dt = 1.0 / k.dt;
    Geo<EL> GE;
    load_geo<EL>(nd, T, ln, GE);
    // the row range is a compile-time constant in each branch (wave-uniform)
    {
        Rows<EL> rows;
#pragma unroll
        for (int a = 0; a < NEN; ++a) rows.v[a] = ln[a];
        const int form = FORM >= 0 ? FORM : k.form;
        if (W == 1 || wv == 0)
            gauss_loop<EL, OP, Q, RA, 0>(GE, nd, nd + 3 * T, T, rows, A, B, mindet, inv_dt, k.Dk, form);
        else
            gauss_loop<EL, OP, Q, RA, (RA % NEN)>(GE, nd, nd + 3 * T, T, rows, A, B, mindet, inv_dt, k.Dk, form);
    }
    // this lane's rows of the element, selected without dynamic indexing
    int lr[RA];
#pragma unroll
    for (int r = 0; r < RA; ++r) {
        // arithmetic blend (a select of two loads would become one load at a
        // computed address and push ln[] to scratch)
        const int hi = (W == 1) ? 0 : wv;
        lr[r] = ln[r] + hi * (ln[(RA + r) % NEN] - ln[r]);
    }

    // 4. scatter into the LDS images: wave by wave, then phase by phase, then
    //    in (a, b) order -- no two lanes of one instruction hit one address.
    int base[RA];
#pragma unroll
    for (int r = 0; r < RA; ++r) base[r] = VEC ? 0 : rdesc[lr[r]] & 0xffff;
    const int nph = k.blk_nphase[blk];
#pragma unroll
    for (int w = 0; w < W; ++w) {
        if (wv == w) {
            for (int p = 0; p < nph; ++p) {
                if (ph == p) {
#pragma unroll
                    for (int r = 0; r < RA; ++r) {
                        if constexpr (!VEC) {
#pragma unroll
                            for (int b = 0; b < NEN; ++b) {
                                const int idx = r * NEN + b;
                                const int off = (offw[idx >> 2] >> (8 * (idx & 3))) & 0xff;
                                lds_add(&img[base[r] + off], (double)A[r][b]);
                            }
                        }
#pragma unroll
                        for (int q = 0; q < NRHS; ++q) lds_add(&rimg[q * T + lr[r]], (double)B[q][r]);
                    }
                }
            }
        }
        if (W > 1) __syncthreads();
    }

    // status: per-block smallest det J and first non-positive element
    if (wv == 0) {
        double md = act ? mindet : __builtin_huge_val();
        long long bad = (act && !(mindet > 0.0)) ? (long long)e : (long long)0x7fffffffffffffffLL;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            md = fmin(md, __shfl_xor(md, o));
            const long long ob = __shfl_xor(bad, o);
            bad = ob < bad ? ob : bad;
        }
        if (el == 0) {
            k.blk_mindet[blk] = md;
            k.blk_bad[blk] = bad == 0x7fffffffffffffffLL ? -1 : bad;
        }
    }
    __syncthreads();

    // 5. write back, one touched row per lane (LDS reads batched ahead of the
    //    stores)
    for (int t = tid; t < T && !VEC; t += NT) {
        const int rd = rdesc[t];
        const int64_t r0 = k.blk_rowstart[n0 + t];
        const int len = (rd >> 16) & 0xff, base = rd & 0xffff;
        double v[kRowBatch];
#pragma unroll
        for (int q = 0; q < kRowBatch; ++q)
            if (q < len) v[q] = img[base + q];
#pragma unroll
        for (int q = 0; q < kRowBatch; ++q)
            if (q < len) k.values[r0 + q] = v[q];
        for (int q = kRowBatch; q < len; ++q) k.values[r0 + q] = img[base + q];
    }
    for (int t = tid; t < T; t += NT) {
        const int g = k.blk_nodes[n0 + t];
#pragma unroll
        for (int r = 0; r < NRHS; ++r) k.rhs[r * N + g] = rimg[r * T + t];
    }
}

template <class EL, int OP, class Q>
__global__ void __launch_bounds__(64 * Split<EL>::W, 2) k_assemble(KArgs k)
{
    assemble_block<EL, OP, Q, -1>(k, blockIdx.x);
}

// Batched coloured assembly (the serving runtime): one launch runs the same
// (colour, type) launch of several meshes.  Work-group w belongs to entry j
// with wgs[j] <= w < wgs[j + 1] (a handful of entries: a linear scan); the
// entry's kernel arguments are ks[slot[j]], its blocks color_blk[first[j] +
// w - wgs[j]].  Each block runs the code of k_assemble, so a mesh's results
// do not depend on what shares the launch.
struct AsmBatch {
    int n;
    int slot[kMaxBatch];
    int first[kMaxBatch];
    int wgs[kMaxBatch + 1];
};
// The device table's slot: KArgs, then (meshes that assemble by blocks with a
// gather) GatherArgs.
constexpr size_t kGatherArgsAt = 256;
static_assert(sizeof(KArgs) <= kGatherArgsAt);

template <class EL, int OP>
__global__ void __launch_bounds__(64 * Split<EL>::W, 2) k_bat_assemble(const KArgs *__restrict__ ks, AsmBatch B)
{
    int j = 0;
    while (j + 1 < B.n && (int)blockIdx.x >= B.wgs[j + 1]) ++j;
    // read in place (its blk_offset is 0): a copy would hold every field live
    const KArgs &k = *(const KArgs *)((const char *)ks + (size_t)B.slot[j] * kKArgsBytes);
    assemble_block<EL, OP, double, -1>(k, B.first[j] + (int)blockIdx.x - B.wgs[j]);
}

// The momentum residual pass with its operator variants (FE_FORM_* bits)
// fixed at compile time.
template <class EL, int FORM>
__global__ void __launch_bounds__(64 * Split<EL>::W, 2) k_residual(KArgs k)
{
    assemble_block<EL, OP_RES, double, FORM>(k, blockIdx.x);
}

// ---- HEX08 by sums over one direction at a time ------------------------------
// The trilinear basis and its 2x2x2 rule are products of the two-point rule of
// a line, L0, L1 = (1 -+ t)/2 at t = -+1/sqrt3, so interpolating to the points
// and adding up over them go direction by direction: 3 operations per pair of
// values and direction instead of 8 products per point and field.
constexpr double kHexP = 0.5 * (1.0 + Hex::kG);   // L0 at the first point = L1 at the second

// Values at the ends of a line (a, b) -> at its two points.
__device__ __forceinline__ void line_points(double a, double b, double &p0, double &p1)
{
    const double d = a - b;
    p0 = fma(kHexP, d, b);
    p1 = fma(-kHexP, d, a);
}
// Sums over a line's two points (p0, p1) weighted with L0 and L1 (the
// transpose of line_points, which is symmetric).
__device__ __forceinline__ void line_nodes(double p0, double p1, double &a, double &b) { line_points(p0, p1, a, b); }

// Local node of tensor position (ix, iy, iz).
__host__ __device__ constexpr int hex_node(int ix, int iy, int iz) { return 4 * iz + (iy ? (ix ? 2 : 3) : ix); }

// A nodal field on the slab of Gauss points zeta = z: its values (f) and zeta
// derivatives (h) at the four lines (ix, iy).
__device__ __forceinline__ void hex_slab(const double *f, const int (&ln)[8], double z, double (&v)[2][2],
                                         double (&h)[2][2])
{
#pragma unroll
    for (int ix = 0; ix < 2; ++ix)
#pragma unroll
        for (int iy = 0; iy < 2; ++iy) {
            const double a = f[ln[hex_node(ix, iy, 0)]], b = f[ln[hex_node(ix, iy, 1)]];
            h[ix][iy] = 0.5 * (b - a);
            v[ix][iy] = fma(z, h[ix][iy], 0.5 * (a + b));
        }
}
// Lines (ix, iy) -> the slab's points (gx, gy).
__device__ __forceinline__ void hex_points(const double (&v)[2][2], double (&p)[2][2])
{
    double t[2][2];
#pragma unroll
    for (int iy = 0; iy < 2; ++iy) line_points(v[0][iy], v[1][iy], t[0][iy], t[1][iy]);
#pragma unroll
    for (int gx = 0; gx < 2; ++gx) line_points(t[gx][0], t[gx][1], p[gx][0], p[gx][1]);
}
// Reference gradient of a field on the slab: d/dxi at (gy), d/deta at (gx),
// d/dzeta at (gx, gy).
struct SlabGrad {
    double x[2], y[2], z[2][2];
};
__device__ __forceinline__ void hex_grad(const double (&v)[2][2], const double (&h)[2][2], SlabGrad &g)
{
    line_points(0.5 * (v[1][0] - v[0][0]), 0.5 * (v[1][1] - v[0][1]), g.x[0], g.x[1]);
    line_points(0.5 * (v[0][1] - v[0][0]), 0.5 * (v[1][1] - v[1][0]), g.y[0], g.y[1]);
    hex_points(h, g.z);
}
// Cofactors C of the Jacobian at the slab's point (gx, gy): C[j] = det J times
// the physical gradient of reference coordinate j; det J is returned.
__device__ __forceinline__ double hex_cofactors(const SlabGrad (&X)[3], int gx, int gy, double (&C)[3][3])
{
    double c0[3], c1[3], c2[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        c0[i] = X[i].x[gy];
        c1[i] = X[i].y[gx];
        c2[i] = X[i].z[gx][gy];
    }
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const int j = (i + 1) % 3, k = (i + 2) % 3;
        C[0][i] = c1[j] * c2[k] - c1[k] * c2[j];
        C[1][i] = c2[j] * c0[k] - c2[k] * c0[j];
        C[2][i] = c0[j] * c1[k] - c0[k] * c1[j];
    }
    return c0[0] * C[0][0] + c0[1] * C[0][1] + c0[2] * C[0][2];
}

// Sums over a line's two points weighted with L_a L_b: s[0] both ends at the
// first node, s[1] one at each, s[2] both at the second.
__device__ __forceinline__ void line_pairs(double p0, double p1, double (&s)[3])
{
    constexpr double Q = 1.0 - kHexP;
    s[0] = fma(kHexP * kHexP, p0, (Q * Q) * p1);
    s[1] = (kHexP * Q) * (p0 + p1);
    s[2] = fma(Q * Q, p0, (kHexP * kHexP) * p1);
}

// The matrix rows of the four nodes with iz = AZ of one HEX08 element, FP64
// (the terms of gauss_point), and their right-hand sides.  Every term is a
// coefficient at a Gauss point (the mass m, the convection c_l, the diffusion
// D_jl on reference coordinates) times a product of line functions of row and
// column, so a term is first added up over zeta with its weights for the two
// column layers bz, then over the lines of xi and eta: ~1,900 operations per
// four rows against ~3,000 for products formed at every point.  t1 .. t8 are
// the terms by which of row and column carries a derivative in xi or eta:
// t1 none, t2 column xi, t3 row xi, t4 column eta, t5 row eta, t6 both xi,
// t7 both eta, t8 row xi and column eta (and, D being symmetric, row eta and
// column xi).  One slab of points after the other in a rolled loop.
template <int OP, int AZ>
__device__ __forceinline__ void hex_matrix(const double *nd, const double *nf, int T, const int (&ln0)[8],
                                           double (&A)[4][8], double (&B)[OpTraits<OP>::NRHS][4], double &mindet,
                                           double inv_dt, double Dk)
{
    constexpr bool POI = OP == OP_POI;
    constexpr int NS = POI ? 0 : OpTraits<OP>::NRHS;   // right-hand sides from a source
    int ln[8];
#pragma unroll
    for (int a = 0; a < 8; ++a) ln[a] = ln0[a];
    double t1[2][2][2] = {}, t2[2][2][2] = {}, t3[2][2] = {}, t4[2][2][2] = {}, t5[2][2] = {}, t6[2][2] = {},
           t7[2][2] = {}, t8[2][2][2] = {};
    double rs[NS ? NS : 1][2][2] = {}, rx[2] = {}, ry[2] = {}, rz[2][2] = {};
#pragma unroll 1
    for (int gz = 0; gz < 2; ++gz) {
        const double z = gz ? Hex::kG : -Hex::kG;
#pragma unroll
        for (int a = 0; a < 8; ++a) asm volatile("" : "+v"(ln[a]));   // fields are read again, not kept
        // weights of the rows' layer and of the two column layers
        const double Lb[2] = {0.5 * (1.0 - z), 0.5 * (1.0 + z)};
        const double La = Lb[AZ], da = AZ ? 0.5 : -0.5;
        SlabGrad X[3];
        double v[2][2], h[2][2], up[3][2][2], rp[2][2], mp[2][2];
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            hex_slab(nd + i * T, ln, z, v, h);
            hex_grad(v, h, X[i]);
        }
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            hex_slab(nf + i * T, ln, z, v, h);
            hex_points(v, up[i]);
        }
        hex_slab(nf + 3 * T, ln, z, v, h);
        hex_points(v, rp);
        if constexpr (!POI) {
            hex_slab(nf + 4 * T, ln, z, v, h);
            hex_points(v, mp);   // mu or Y
        }
#pragma unroll
        for (int gx = 0; gx < 2; ++gx)
#pragma unroll
            for (int gy = 0; gy < 2; ++gy) {
                double C[3][3];
                const double det = hex_cofactors(X, gx, gy, C);
                mindet = fmin(mindet, det);
                const double r = rp[gx][gy];
                const double k = (POI ? 1.0 : OP == OP_MOM ? mp[gx][gy] : r * Dk) / det;
                double c[3];   // rho det J times the velocity's reference components
#pragma unroll
                for (int j = 0; j < 3; ++j)
                    c[j] = r * (C[j][0] * up[0][gx][gy] + C[j][1] * up[1][gx][gy] + C[j][2] * up[2][gx][gy]);
                auto D = [&](int j, int l) { return k * (C[j][0] * C[l][0] + C[j][1] * C[l][1] + C[j][2] * C[l][2]); };
                const double dzz = da * D(2, 2), dxz = D(0, 2), dyz = D(1, 2), dxy = D(0, 1);
                const double dxx = La * D(0, 0), dyy = La * D(1, 1);
                const double m = POI ? 0.0 : La * (r * det * inv_dt);
#pragma unroll
                for (int bz = 0; bz < 2; ++bz) {
                    const double db = bz ? 0.5 : -0.5;
                    if constexpr (POI) {
                        if (bz == 0) t1[0][gx][gy] += dzz;
                        t2[bz][gx][gy] += (da * Lb[bz]) * dxz;
                        t4[bz][gx][gy] += (da * Lb[bz]) * dyz;
                    } else {
                        t1[bz][gx][gy] += Lb[bz] * m + db * (La * c[2] + dzz);
                        t2[bz][gx][gy] += Lb[bz] * (La * c[0] + da * dxz);
                        t4[bz][gx][gy] += Lb[bz] * (La * c[1] + da * dyz);
                    }
                    t6[bz][gy] += Lb[bz] * dxx;
                    t7[bz][gx] += Lb[bz] * dyy;
                    t8[bz][gx][gy] += (La * Lb[bz]) * dxy;
                }
                t3[gx][gy] += La * dxz;
                t5[gx][gy] += La * dyz;
                if constexpr (POI) {
                    rx[gy] += La * c[0];
                    ry[gx] += La * c[1];
                    rz[gx][gy] += c[2];
                } else {
#pragma unroll
                    for (int q = 0; q < NS; ++q)
                        rs[q][gx][gy] += m * (OP == OP_MOM ? up[q][gx][gy] : mp[gx][gy]);
                }
            }
    }
    // over xi and eta, one column layer at a time.  sx, sy: -+1/2, the
    // derivatives of the line functions.
#pragma unroll
    for (int bz = 0; bz < 2; ++bz) {
        const double db = bz ? 0.5 : -0.5;
        double a1[3][3], a2[2][3], a3[2][3], a4[3][2], a5[3][2], a6[3], a7[3], a8[2][2];
        {
            double w[3][2];
#pragma unroll
            for (int gy = 0; gy < 2; ++gy) {
                double q[3];
                if constexpr (POI) line_pairs(db * t1[0][0][gy], db * t1[0][1][gy], q);
                else line_pairs(t1[bz][0][gy], t1[bz][1][gy], q);
#pragma unroll
                for (int x = 0; x < 3; ++x) w[x][gy] = q[x];
            }
#pragma unroll
            for (int x = 0; x < 3; ++x) line_pairs(w[x][0], w[x][1], a1[x]);
        }
        {
            double w[2][2], u[2][2];
#pragma unroll
            for (int gy = 0; gy < 2; ++gy) {
                line_nodes(t2[bz][0][gy], t2[bz][1][gy], w[0][gy], w[1][gy]);
                line_nodes(db * t3[0][gy], db * t3[1][gy], u[0][gy], u[1][gy]);
            }
#pragma unroll
            for (int x = 0; x < 2; ++x) {
                line_pairs(w[x][0], w[x][1], a2[x]);
                line_pairs(u[x][0], u[x][1], a3[x]);
            }
        }
        {
            double w[2][2], u[2][2];
#pragma unroll
            for (int gx = 0; gx < 2; ++gx) {
                line_nodes(t4[bz][gx][0], t4[bz][gx][1], w[gx][0], w[gx][1]);
                line_nodes(db * t5[gx][0], db * t5[gx][1], u[gx][0], u[gx][1]);
            }
#pragma unroll
            for (int y = 0; y < 2; ++y) {
                double q[3];
                line_pairs(w[0][y], w[1][y], q);
#pragma unroll
                for (int x = 0; x < 3; ++x) a4[x][y] = q[x];
                line_pairs(u[0][y], u[1][y], q);
#pragma unroll
                for (int x = 0; x < 3; ++x) a5[x][y] = q[x];
            }
        }
        line_pairs(t6[bz][0], t6[bz][1], a6);
        line_pairs(t7[bz][0], t7[bz][1], a7);
        {
            double w[2][2];
#pragma unroll
            for (int gx = 0; gx < 2; ++gx) line_nodes(t8[bz][gx][0], t8[bz][gx][1], w[gx][0], w[gx][1]);
#pragma unroll
            for (int y = 0; y < 2; ++y) line_nodes(w[0][y], w[1][y], a8[0][y], a8[1][y]);
        }
#pragma unroll
        for (int ax = 0; ax < 2; ++ax)
#pragma unroll
            for (int ay = 0; ay < 2; ++ay)
#pragma unroll
                for (int bx = 0; bx < 2; ++bx)
#pragma unroll
                    for (int by = 0; by < 2; ++by) {
                        const double sxa = ax ? 0.5 : -0.5, sxb = bx ? 0.5 : -0.5, sya = ay ? 0.5 : -0.5,
                                     syb = by ? 0.5 : -0.5;
                        const int x = ax + bx, y = ay + by;
                        double e = a1[x][y];
                        e += sxb * a2[ax][y];
                        e += sxa * a3[bx][y];
                        e += syb * a4[x][ay];
                        e += sya * a5[x][by];
                        e += (sxa * sxb) * a6[y];
                        e += (sya * syb) * a7[x];
                        e += (sxa * syb) * a8[bx][ay];
                        e += (sya * sxb) * a8[ax][by];
                        A[hex_node(ax, ay, 0)][hex_node(bx, by, bz)] = e;
                    }
    }
    if constexpr (POI) {
        const double da = (AZ ? 0.5 : -0.5) * inv_dt;
        double nx[2], ny[2], w[2][2], n[2][2];
        line_nodes(rx[0], rx[1], nx[0], nx[1]);
        line_nodes(ry[0], ry[1], ny[0], ny[1]);
#pragma unroll
        for (int gx = 0; gx < 2; ++gx) line_nodes(rz[gx][0], rz[gx][1], w[gx][0], w[gx][1]);
#pragma unroll
        for (int y = 0; y < 2; ++y) line_nodes(w[0][y], w[1][y], n[0][y], n[1][y]);
#pragma unroll
        for (int ax = 0; ax < 2; ++ax)
#pragma unroll
            for (int ay = 0; ay < 2; ++ay)
                B[0][hex_node(ax, ay, 0)] =
                    da * n[ax][ay] + inv_dt * ((ax ? 0.5 : -0.5) * nx[ay] + (ay ? 0.5 : -0.5) * ny[ax]);
    } else {
#pragma unroll
        for (int q = 0; q < NS; ++q) {
            double w[2][2];
#pragma unroll
            for (int gx = 0; gx < 2; ++gx) line_nodes(rs[q][gx][0], rs[q][gx][1], w[gx][0], w[gx][1]);
#pragma unroll
            for (int y = 0; y < 2; ++y) {
                double n0, n1;
                line_nodes(w[0][y], w[1][y], n0, n1);
                B[q][hex_node(0, y, 0)] = n0;
                B[q][hex_node(1, y, 0)] = n1;
            }
        }
    }
}

// ---- owner assembly of the matrix operators ---------------------------------
// HEX08.  One work-group owns a group of consecutive CSR rows and computes every
// element contribution to them, so each row is written once and never read
// back, in a single launch (no colours).  Steps:
//   1. stage the group's touched nodes' fields in LDS (owned rows first);
//      zero the owned rows' image and right-hand sides;
//   2. one task per lane: rows 0-3 of its element, rotated so that the rows
//      the group owns lie on its first face (FP64: hex_matrix; mixed: the
//      FP32 Gauss loop);
//   3. wavefront after wavefront (a barrier between them), add the owned rows
//      into LDS, local row after local row: the plan deals the tasks so that
//      one instruction's lanes hold distinct rows, mostly in one step, and the
//      order of the sums is fixed.  (Phases of tasks without a common row
//      over the whole group, ten of them with a barrier each, took 5.2 of a
//      group's 22 us on 101^3 HEX08.)
//   4. write the rows (contiguous in CSR) and right-hand sides once.
// Bound by FP64 arithmetic and the staging before it (10 and 5 of a group's 22
// us, two groups to a CU).  Whole calls, Gauss point after Gauss point with
// phases -> direction by direction and wavefront after wavefront: momentum 10^3
// 45 -> 33 us, 72^3 251 -> 164, 128^3 1250 -> 840; Poisson 128^3 1020 -> 694;
// mixed (Gauss points kept, so that its FP32 results stay the same) momentum
// 128^3 884 -> 830.
struct OArgs {
    const double *X;
    const int32_t *rowptr;
    const int4 *groups;
    const int32_t *node_ptr, *nodes, *elem;
    const uint8_t *nphase, *off, *phase;
    const uint16_t *ln;
    int ln_stride, off_stride;
    int64_t N;
    const double *u, *rho, *mu, *Y;   // Y [scalars][N]
    double dt, D[kOwnScalars];
    int64_t nnz;
    double *values, *rhs;             // [scalars][nnz], [scalars][N]
    double *g_mindet;
    long long *g_bad;
};

// Work-groups are dispatched round-robin over MI355X's 8 XCDs (work-group b
// on XCD b % 8), each with its own L2.  xcd_item maps work-group b of a
// G-group launch to item i so that every XCD takes one contiguous range of
// items (a bijection of [0, G)).  Consecutive owner groups cover neighbouring
// rows and share halo nodes, so their cache lines of the nodal fields are then
// fetched once into that XCD's L2 instead of once into each of several.
constexpr int kAsmXcds = 8;
__device__ inline int xcd_item(int b, int G)
{
    const int q = G / kAsmXcds, rem = G % kAsmXcds, x = b % kAsmXcds, slot = b / kAsmXcds;
    return x * q + (x < rem ? x : rem) + slot;
}

// A group's smallest det J and first element with det J <= 0 (or -1), by its
// NT threads.
template <int NT>
__device__ __forceinline__ void group_status(double md, bool is_bad, long long elem, double *mindet, long long *first_bad)
{
    constexpr long long kNone = 0x7fffffffffffffffLL;
    __shared__ double smd[NT / 64];
    __shared__ long long sbad[NT / 64];
    const int tid = threadIdx.x;
    long long bad = is_bad ? elem : kNone;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        md = fmin(md, __shfl_xor(md, o));
        const long long ob = __shfl_xor(bad, o);
        bad = ob < bad ? ob : bad;
    }
    if ((tid & 63) == 0) {
        smd[tid >> 6] = md;
        sbad[tid >> 6] = bad;
    }
    __syncthreads();
    if (tid == 0) {
#pragma unroll
        for (int w = 1; w < NT / 64; ++w) {
            md = fmin(md, smd[w]);
            bad = sbad[w] < bad ? sbad[w] : bad;
        }
        *mindet = md;
        *first_bad = bad == kNone ? -1 : bad;
    }
}

// NS: scalars at once (mixed FE_OP_SCALAR): the staging and the points' FP64
// geometry, half of a pass, serve all of them: five scalars as 3 + 2 on 72^3 HEX08
// 741 -> 569 us for the call (474 MB), the same results to the bit.
// FP64, whose sums of one scalar fill the registers, takes them one by one.
template <int OP, class Q, int NS = 1>
__global__ void __launch_bounds__(kOwnTasks, 2) k_own(OArgs k)
{
    constexpr int NEN = 8, RA = 4;
    constexpr int NF = OpTraits<OP>::NF + NS - 1, NRHS = OpTraits<OP>::NRHS;
    static_assert(NS == 1 || (OP == OP_SCA && sizeof(Q) == 4 && NS <= kOwnScalars));
    extern __shared__ double lds[];
    const int gi = xcd_item(blockIdx.x, gridDim.x);   // this work-group's group
    const int4 gd = k.groups[gi];   // first task, tasks, first row, rows
    const int tid = threadIdx.x;
    const int r0 = gd.z, nr = gd.w;
    const int n0 = k.node_ptr[gi], T = k.node_ptr[gi + 1] - n0;
    const int64_t v0 = k.rowptr[r0];
    const int L = (int)(k.rowptr[r0 + nr] - v0);
    const int64_t N = k.N;
    // Fields of the touched nodes: x, y, z in FP64 (the geometry is FP64 in
    // both modes), the others in the quadrature's precision (the mixed mode
    // interpolates them in FP32, which halves their LDS traffic).
    using FT = Q;
    double *nd = lds;                   // [3][T] coordinates
    FT *nf = (FT *)(nd + 3 * T);        // [NF - 3][T] u_x, u_y, u_z, rho, mu / Y
    double *img = nd + 3 * T + ((NF - 3) * T * (int)sizeof(FT) + 7) / 8;   // [L] the owned rows
    double *rimg = img + L;             // [NRHS][nr] their right-hand sides

    // task data first: its loads overlap the staging below
    const bool live = tid < gd.y;
    const int64_t t = gd.x + (live ? tid : 0);
    int ln[NEN];
    {
        const uint16_t *lp = k.ln + t * k.ln_stride;
#pragma unroll
        for (int a = 0; a < NEN; ++a) ln[a] = lp[a];
    }
    constexpr int kOffWords = (RA * NEN + 3) / 4;
    uint32_t offw[kOffWords];
    {
        const uint32_t *op = (const uint32_t *)(k.off + t * k.off_stride);
#pragma unroll
        for (int q = 0; q < kOffWords; ++q) offw[q] = op[q];
    }
    const int ph = live ? (int)k.phase[t] : -1;
    const int64_t elem = k.elem[t];

    // 1. stage
    for (int q = tid; q < T; q += kOwnTasks) {
        const int g = k.nodes[n0 + q];
        double f[NF];
        f[0] = k.X[g];
        f[1] = k.X[N + g];
        f[2] = k.X[2 * N + g];
        f[3] = k.u[g];
        f[4] = k.u[N + g];
        f[5] = k.u[2 * N + g];
        f[6] = k.rho[g];
        if constexpr (NF > 7) f[7] = OP == OP_MOM ? k.mu[g] : k.Y[g];
#pragma unroll
        for (int c = 1; c < NS; ++c) f[7 + c] = k.Y[c * N + g];
#pragma unroll
        for (int c = 0; c < 3; ++c) nd[c * T + q] = f[c];
#pragma unroll
        for (int c = 3; c < NF; ++c) nf[(c - 3) * T + q] = FT(f[c]);
    }
    for (int q = tid; q < L; q += kOwnTasks) img[q] = 0.0;
    for (int q = tid; q < NRHS * nr; q += kOwnTasks) rimg[q] = 0.0;
    __syncthreads();

    // 2. this lane's rows
    Q A[NS][RA][NEN];
    Q B[NS][NRHS][RA];
#pragma unroll
    for (int c = 0; c < NS; ++c)
#pragma unroll
        for (int r = 0; r < RA; ++r) {
#pragma unroll
            for (int b = 0; b < NEN; ++b) A[c][r][b] = Q(0);
#pragma unroll
            for (int q = 0; q < NRHS; ++q) B[c][q][r] = Q(0);
        }
    double mindet = __builtin_huge_val();
    if constexpr (sizeof(Q) == 8) {
        if (live) hex_matrix<OP, 0>(nd, nf, T, ln, A[0], B[0], mindet, 1.0 / k.dt, k.D[0]);
    } else if (live) {
        Geo<Hex> GE;
        load_geo<Hex>(nd, T, ln, GE);
        Rows<Hex> rows;
#pragma unroll
        for (int a = 0; a < NEN; ++a) rows.v[a] = ln[a];
        if constexpr (NS > 1) scalars_loop<NS>(GE, nd, nf, T, rows, A, B, mindet, 1.0 / k.dt, k.D);
        else gauss_loop<Hex, OP, Q, RA, 0, FT>(GE, nd, nf, T, rows, A[0], B[0], mindet, 1.0 / k.dt, k.D[0], 0);
    }
    int base[RA];
#pragma unroll
    for (int r = 0; r < RA; ++r) base[r] = ln[r] < nr ? (int)(k.rowptr[r0 + ln[r]] - v0) : -1;

    const int nph = k.nphase[gi];
#pragma unroll
    for (int c = 0; c < NS; ++c) {
        if (c > 0) {
            __syncthreads();
            for (int q = tid; q < L; q += kOwnTasks) img[q] = 0.0;
            for (int q = tid; q < NRHS * nr; q += kOwnTasks) rimg[q] = 0.0;
            __syncthreads();
        }
        // 3. wavefront after wavefront
#pragma unroll 1
        for (int w = 0; w < kOwnTasks / 64; ++w) {
            if ((tid >> 6) == w) {
                for (int p = 0; p < nph; ++p) {
                    if (ph != p) continue;
#pragma unroll
                    for (int r = 0; r < RA; ++r) {
                        if (base[r] < 0) continue;   // a row another group owns
#pragma unroll
                        for (int b = 0; b < NEN; ++b) {
                            const int idx = r * NEN + b;
                            const int o = (offw[idx >> 2] >> (8 * (idx & 3))) & 0xff;
                            lds_add(&img[base[r] + o], (double)A[c][r][b]);
                        }
#pragma unroll
                        for (int q = 0; q < NRHS; ++q) lds_add(&rimg[q * nr + ln[r]], (double)B[c][q][r]);
                    }
                }
            }
            __syncthreads();
        }

        // 4. write the owned rows and right-hand sides once
        for (int q = tid; q < L; q += kOwnTasks) k.values[c * k.nnz + v0 + q] = img[q];
        for (int q = tid; q < NRHS * nr; q += kOwnTasks) {
            const int h = q / nr, i = q - h * nr;
            k.rhs[(c * NRHS + h) * N + r0 + i] = rimg[q];
        }
    }
    group_status<kOwnTasks>(live ? mindet : __builtin_huge_val(), live && !(mindet > 0.0), elem, k.g_mindet + gi,
                            k.g_bad + gi);
}

// The owner assembly of the other types, for meshes in an order of poor
// locality (plan.h, max_images): a lane takes all rows of its element.  Their
// nodes lie in many elements (24 for a Kuhn tetrahedron's), so that phases with
// a barrier each would be as many: each wavefront adds into its own copy of the
// rows, phases within the wavefront, and the copies are summed in their order.
template <class EL, int OP, class Q>
__global__ void __launch_bounds__(kOwnTasks, 2) k_own_copies(OArgs k)
{
    constexpr int NEN = EL::NEN, NC = kOwnTasks / 64;
    constexpr int NF = OpTraits<OP>::NF, NRHS = OpTraits<OP>::NRHS;
    extern __shared__ double lds[];
    const int gi = xcd_item(blockIdx.x, gridDim.x);   // this work-group's group
    const int4 gd = k.groups[gi];   // first task, tasks, first row, rows
    const int tid = threadIdx.x;
    const int r0 = gd.z, nr = gd.w;
    const int n0 = k.node_ptr[gi], T = k.node_ptr[gi + 1] - n0;
    const int64_t v0 = k.rowptr[r0];
    const int L = (int)(k.rowptr[r0 + nr] - v0);
    const int64_t N = k.N;
    using FT = Q;
    double *nd = lds;                   // [3][T] coordinates
    FT *nf = (FT *)(nd + 3 * T);        // [NF - 3][T] u_x, u_y, u_z, rho, mu / Y
    double *imgs = nd + 3 * T + ((NF - 3) * T * (int)sizeof(FT) + 7) / 8;   // [NC][L] the owned rows
    double *rimgs = imgs + NC * L;      // [NC][NRHS][nr] their right-hand sides
    double *img = imgs + (tid >> 6) * L, *rimg = rimgs + (tid >> 6) * NRHS * nr;

    const bool live = tid < gd.y;
    const int64_t t = gd.x + (live ? tid : 0);
    Rows<EL> rows;
    {
        const uint16_t *lp = k.ln + t * k.ln_stride;
#pragma unroll
        for (int a = 0; a < NEN; ++a) rows.v[a] = lp[a];
    }
    constexpr int kOffWords = (NEN * NEN + 3) / 4;
    uint32_t offw[kOffWords];
    {
        const uint32_t *op = (const uint32_t *)(k.off + t * k.off_stride);
#pragma unroll
        for (int q = 0; q < kOffWords; ++q) offw[q] = op[q];
    }
    const int ph = live ? (int)k.phase[t] : -1;
    for (int q = tid; q < T; q += kOwnTasks) {
        const int g = k.nodes[n0 + q];
        double f[NF];
        f[0] = k.X[g];
        f[1] = k.X[N + g];
        f[2] = k.X[2 * N + g];
        f[3] = k.u[g];
        f[4] = k.u[N + g];
        f[5] = k.u[2 * N + g];
        f[6] = k.rho[g];
        if constexpr (NF > 7) f[7] = OP == OP_MOM ? k.mu[g] : k.Y[g];
#pragma unroll
        for (int c = 0; c < 3; ++c) nd[c * T + q] = f[c];
#pragma unroll
        for (int c = 3; c < NF; ++c) nf[(c - 3) * T + q] = FT(f[c]);
    }
    for (int q = tid; q < NC * L; q += kOwnTasks) imgs[q] = 0.0;
    for (int q = tid; q < NC * NRHS * nr; q += kOwnTasks) rimgs[q] = 0.0;
    __syncthreads();

    Q A[NEN][NEN];
    Q B[NRHS][NEN];
#pragma unroll
    for (int r = 0; r < NEN; ++r) {
#pragma unroll
        for (int b = 0; b < NEN; ++b) A[r][b] = Q(0);
#pragma unroll
        for (int q = 0; q < NRHS; ++q) B[q][r] = Q(0);
    }
    double mindet = __builtin_huge_val();
    if (live) {
        Geo<EL> GE;
        load_geo<EL>(nd, T, rows.v, GE);
        gauss_loop<EL, OP, Q, NEN, 0, FT>(GE, nd, nf, T, rows, A, B, mindet, 1.0 / k.dt, k.D[0], 0);
    }
    int base[NEN];
#pragma unroll
    for (int r = 0; r < NEN; ++r) base[r] = rows.v[r] < nr ? (int)(k.rowptr[r0 + rows.v[r]] - v0) : -1;
    const int nph = k.nphase[gi];
    for (int p = 0; p < nph; ++p) {
        if (ph != p) continue;
#pragma unroll
        for (int r = 0; r < NEN; ++r) {
            if (base[r] < 0) continue;   // a row another group owns
#pragma unroll
            for (int b = 0; b < NEN; ++b) {
                const int idx = r * NEN + b;
                const int o = (offw[idx >> 2] >> (8 * (idx & 3))) & 0xff;
                lds_add(&img[base[r] + o], (double)A[r][b]);
            }
#pragma unroll
            for (int q = 0; q < NRHS; ++q) lds_add(&rimg[q * nr + rows.v[r]], (double)B[q][r]);
        }
    }
    __syncthreads();
    for (int q = tid; q < L; q += kOwnTasks) {
        double v = imgs[q];
#pragma unroll
        for (int c = 1; c < NC; ++c) v += imgs[c * L + q];
        k.values[v0 + q] = v;
    }
    for (int q = tid; q < NRHS * nr; q += kOwnTasks) {
        const int h = q / nr, i = q - h * nr;
        double v = rimgs[q];
#pragma unroll
        for (int c = 1; c < NC; ++c) v += rimgs[c * NRHS * nr + q];
        k.rhs[h * N + r0 + i] = v;
    }
    group_status<kOwnTasks>(live ? mindet : __builtin_huge_val(), live && !(mindet > 0.0), k.elem[t], k.g_mindet + gi,
                            k.g_bad + gi);
}

template <int OP>
void launch_own_op(const OArgs &k, int64_t G, size_t lds, bool mixed, hipStream_t s)
{
    if (mixed) hipLaunchKernelGGL((k_own<OP, float>), dim3((unsigned)G), dim3(kOwnTasks), lds, s, k);
    else hipLaunchKernelGGL((k_own<OP, double>), dim3((unsigned)G), dim3(kOwnTasks), lds, s, k);
}

template <class EL>
void launch_own_copies(const OArgs &k, int op, int64_t G, size_t lds, bool mixed, hipStream_t s)
{
    const dim3 grid((unsigned)G), block(kOwnTasks);
    switch (op) {
    case OP_MOM:
        if (mixed) hipLaunchKernelGGL((k_own_copies<EL, OP_MOM, float>), grid, block, lds, s, k);
        else hipLaunchKernelGGL((k_own_copies<EL, OP_MOM, double>), grid, block, lds, s, k);
        break;
    case OP_SCA:
        if (mixed) hipLaunchKernelGGL((k_own_copies<EL, OP_SCA, float>), grid, block, lds, s, k);
        else hipLaunchKernelGGL((k_own_copies<EL, OP_SCA, double>), grid, block, lds, s, k);
        break;
    default:
        if (mixed) hipLaunchKernelGGL((k_own_copies<EL, OP_POI, float>), grid, block, lds, s, k);
        else hipLaunchKernelGGL((k_own_copies<EL, OP_POI, double>), grid, block, lds, s, k);
        break;
    }
}

void launch_own(const OArgs &k, int op, int scalars, int64_t G, size_t lds, bool mixed, hipStream_t s)
{
    switch (op) {
    case OP_MOM: launch_own_op<OP_MOM>(k, G, lds, mixed, s); break;
    case OP_SCA:
        if (scalars == 3) hipLaunchKernelGGL((k_own<OP_SCA, float, 3>), dim3((unsigned)G), dim3(kOwnTasks), lds, s, k);
        else if (scalars == 2) hipLaunchKernelGGL((k_own<OP_SCA, float, 2>), dim3((unsigned)G), dim3(kOwnTasks), lds, s, k);
        else launch_own_op<OP_SCA>(k, G, lds, mixed, s);
        break;
    default: launch_own_op<OP_POI>(k, G, lds, mixed, s); break;
    }
}

// ---- status word -----------------------------------------------------------------
// Per-block status (smallest det J, first bad mesh element or -1) and where its
// reduction goes: a device word, or the caller's pinned host word, which saves
// the copy (4 us) a call would wait for.
struct StatusArgs {
    const double *mindet;
    const long long *bad;
    int64_t n;
    AsmStatus *out;
};

// One group of NT threads reduces st, eight loads in flight per thread.
template <int NT>
__device__ __forceinline__ void reduce_status(const StatusArgs &st)
{
    constexpr long long kNone = 0x7fffffffffffffffLL;
    __shared__ double sd[NT / 64];
    __shared__ long long sb[NT / 64];
    double md = __builtin_huge_val();
    long long b = kNone;
    const int t = threadIdx.x;
    for (int64_t i = t; i < st.n; i += 4 * NT) {
        double m4[4];
        long long b4[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int64_t ii = i + u * NT < st.n ? i + u * NT : i;
            m4[u] = st.mindet[ii];
            b4[u] = st.bad[ii];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            md = fmin(md, m4[u]);
            if (b4[u] >= 0 && b4[u] < b) b = b4[u];
        }
    }
    const auto wave = [&] {
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            md = fmin(md, __shfl_xor(md, o));
            const long long ob = __shfl_xor(b, o);
            b = ob < b ? ob : b;
        }
    };
    wave();
    if (t % 64 == 0) {
        sd[t / 64] = md;
        sb[t / 64] = b;
    }
    __syncthreads();
    if (t >= 64) return;
    md = t < NT / 64 ? sd[t] : __builtin_huge_val();
    b = t < NT / 64 ? sb[t] : kNone;
    wave();
    if (t == 0) {
        unsigned long long u;
        __builtin_memcpy(&u, &md, 8);
        st.out->min_det_key = u;
        st.out->first_bad = b == kNone ? -1 : b;
    }
}

// ---- matrix operators by element blocks, in one launch per element type ----------
// TET04, PEN06, PYR05 and hybrid meshes.  A block's row images start from zero
// and go, whole, to the block's own place in a work array, its right-hand
// sides to another; k_part_gather then writes each CSR row once, the sum of
// its images in block order.  No colours, no row is read back, no element is
// computed twice, and the order of every sum is fixed by the plan.  FT:
// precision of the staged fields after x, y, z (FP32 for the mixed mode on
// meshes of one type).
//
// Bound by latency, in the blocks (a 64-TET04 momentum block: staging 5 us, sums
// 4 us, of 11) as in the gather, with 8-12 blocks to a CU; PEN06 half by FP64
// arithmetic.  Whole calls, owner groups (each element computed by every group
// that owns one of its rows: 1.6x) -> blocks, momentum / Poisson: TET04 45^3
// cubes 114 / 88 -> 91 / 76 us, 90^3 657 / 467 -> 525 / 428; PEN06 57^3 194 / 164
// -> 156 / 121; PYR05 40^3 189 / 158 -> 130 / 118.  Coloured blocks (40 launches)
// -> blocks: hybrid 64^3 816 / 750 -> 223 / 184, 20^3 745 / 700 -> 83 / 74 (outputs
// allocated by the call; into given ones 5 to 30 us less, before as after).  A HEX08 mesh stays with owner
// groups: k_part takes 0.42 ns per HEX08 element (65 k of the hybrid mesh) before
// its gather, k_own as much in all (101^3).
struct PartArgs {
    const int32_t *img_ptr;   // [blocks + 1]
    double *img, *sums;       // row images, [NRHS][VT] right-hand sides
    int64_t VT;
};

template <class EL, int OP, class Q, class FT>
__device__ __forceinline__ void part_block(const KArgs &k, const PartArgs &pa, int blk)
{
    constexpr int NEN = EL::NEN, W = Split<EL>::W, RA = NEN / W, NT = 64 * W;
    constexpr int NF = OpTraits<OP>::NF, NRHS = OpTraits<OP>::NRHS;
    extern __shared__ double lds[];
    const int e0 = k.blk_elem_ptr[blk], ne = k.blk_elem_ptr[blk + 1] - e0;
    const int n0 = k.blk_node_ptr[blk], T = k.blk_node_ptr[blk + 1] - n0;
    const int i0 = pa.img_ptr[blk], L = pa.img_ptr[blk + 1] - i0;
    const int tid = threadIdx.x, el = tid & 63, wv = tid >> 6;
    const int64_t N = k.N;
    double *nd = lds;                                    // [3][T] coordinates
    FT *nf = (FT *)(nd + 3 * T);                         // [NF - 3][T] u_x, u_y, u_z, rho, mu / Y
    double *rimg = nd + 3 * T + ((NF - 3) * T * (int)sizeof(FT) + 7) / 8;   // [NRHS][T]
    double *img = rimg + NRHS * T;                       // [L]
    int *rbase = (int *)(img + L);                       // [T] row images' places in img
    const bool act = el < ne;
    const int e = e0 + (act ? el : 0);
    int ln[NEN];
#pragma unroll
    for (int a = 0; a < NEN; ++a) ln[a] = k.elem_lnode[(int64_t)a * k.E + e];
    constexpr int kOffWords = (RA * NEN + 3) / 4;
    uint32_t offw[kOffWords];
    {
        const uint32_t *op = (const uint32_t *)(k.elem_off + (int64_t)e * k.off_stride + wv * RA * NEN);
#pragma unroll
        for (int q = 0; q < kOffWords; ++q) offw[q] = op[q];
    }
    const int ph = act ? (int)k.elem_phase[e] : -1, nph = k.blk_nphase[blk];
    for (int t = tid; t < T; t += NT) {
        const int g = k.blk_nodes[n0 + t];
        rbase[t] = k.blk_rdesc[n0 + t] & 0xffff;
        double f[NF];
        f[0] = k.X[g];
        f[1] = k.X[N + g];
        f[2] = k.X[2 * N + g];
        f[3] = k.u[g];
        f[4] = k.u[N + g];
        f[5] = k.u[2 * N + g];
        f[6] = k.rho[g];
        if constexpr (NF > 7) f[7] = OP == OP_MOM ? k.mu[g] : k.Y[g];
#pragma unroll
        for (int c = 0; c < 3; ++c) nd[c * T + t] = f[c];
#pragma unroll
        for (int c = 3; c < NF; ++c) nf[(c - 3) * T + t] = FT(f[c]);
#pragma unroll
        for (int r = 0; r < NRHS; ++r) rimg[r * T + t] = 0.0;
    }
    for (int t = tid; t < L; t += NT) img[t] = 0.0;
    __syncthreads();

    Q A[RA][NEN];
    Q B[NRHS][RA];
#pragma unroll
    for (int r = 0; r < RA; ++r) {
#pragma unroll
        for (int b = 0; b < NEN; ++b) A[r][b] = Q(0);
#pragma unroll
        for (int q = 0; q < NRHS; ++q) B[q][r] = Q(0);
    }
    double mindet = __builtin_huge_val();
    const double inv_dt = 1.0 / k.dt;
    if constexpr (NEN == 8 && sizeof(Q) == 8) {
        if (wv == 0) hex_matrix<OP, 0>(nd, nf, T, ln, A, B, mindet, inv_dt, k.Dk);
        else hex_matrix<OP, 1>(nd, nf, T, ln, A, B, mindet, inv_dt, k.Dk);
    } else {
        Geo<EL> GE;
        load_geo<EL>(nd, T, ln, GE);
        Rows<EL> rows;
#pragma unroll
        for (int a = 0; a < NEN; ++a) rows.v[a] = ln[a];
        if (W == 1 || wv == 0) gauss_loop<EL, OP, Q, RA, 0, FT>(GE, nd, nf, T, rows, A, B, mindet, inv_dt, k.Dk, 0);
        else gauss_loop<EL, OP, Q, RA, (RA % NEN), FT>(GE, nd, nf, T, rows, A, B, mindet, inv_dt, k.Dk, 0);
    }
    int lr[RA], base[RA];   // this lane's rows
#pragma unroll
    for (int r = 0; r < RA; ++r) {
        lr[r] = W == 1 ? ln[r] : ln[r] + wv * (ln[(RA + r) % NEN] - ln[r]);   // (a select would go through scratch)
        base[r] = rbase[lr[r]];
    }
#pragma unroll
    for (int w = 0; w < W; ++w) {
        if (wv == w) {
            for (int p = 0; p < nph; ++p) {
                if (ph != p) continue;
#pragma unroll
                for (int r = 0; r < RA; ++r) {
#pragma unroll
                    for (int b = 0; b < NEN; ++b) {
                        const int idx = r * NEN + b;
                        const int o = (offw[idx >> 2] >> (8 * (idx & 3))) & 0xff;
                        lds_add(&img[base[r] + o], (double)A[r][b]);
                    }
#pragma unroll
                    for (int q = 0; q < NRHS; ++q) lds_add(&rimg[q * T + lr[r]], (double)B[q][r]);
                }
            }
        }
        if (W > 1) __syncthreads();
    }
    if (wv == 0) {
        double md = act ? mindet : __builtin_huge_val();
        long long bad = (act && !(mindet > 0.0)) ? (long long)e : (long long)0x7fffffffffffffffLL;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            md = fmin(md, __shfl_xor(md, o));
            const long long ob = __shfl_xor(bad, o);
            bad = ob < bad ? ob : bad;
        }
        if (el == 0) {
            k.blk_mindet[blk] = md;
            k.blk_bad[blk] = bad == 0x7fffffffffffffffLL ? -1 : bad;
        }
    }
    __syncthreads();
    for (int t = tid; t < L; t += NT) pa.img[i0 + t] = img[t];
    for (int t = tid; t < T; t += NT)
#pragma unroll
        for (int r = 0; r < NRHS; ++r) pa.sums[r * pa.VT + n0 + t] = rimg[r * T + t];
}

template <class EL, int OP, class Q, class FT>
__global__ void __launch_bounds__(64 * Split<EL>::W, 2) k_part(KArgs k, PartArgs pa)
{
    part_block<EL, OP, Q, FT>(k, pa, k.color_blk[k.blk_offset + xcd_item(blockIdx.x, gridDim.x)]);
}

// 8 lanes per CSR row: lane l adds entries l, l + 8, l + 16 and l + 24 of two
// of the row's images at a time (8 loads in flight), in block order, lane r
// right-hand side r.  The places of eight images are read by the eight lanes
// at once and handed round, so that a row waits for three loads in a chain
// (its pointers, its places, its images): 43 -> 27 us on 57^3 PEN06 (195 k rows,
// 110 MB) against 16 lanes that each read every place themselves.  Each XCD takes one contiguous range
// of rows, as of blocks in k_part; the first group reduces the status word
// meanwhile (the seven after it only keep the XCDs' ranges).
constexpr int kGatherLanes = 8;
constexpr int kGatherStatus = 8;   // leading groups
constexpr int kGatherRows = 256 / kGatherLanes;
inline int64_t gather_groups(int64_t N) { return (N + kGatherRows - 1) / kGatherRows + kGatherStatus; }
struct GatherArgs {
    int64_t N;
    const int32_t *rowptr, *ptr, *slot, *place;
    PartArgs pa;
    double *values, *rhs;
    StatusArgs st;
};

// Group `item` of the rows.
template <int NRHS>
__device__ __forceinline__ void part_gather(int item, int64_t N, const int32_t *__restrict__ rowptr,
                                            const int32_t *__restrict__ ptr, const int32_t *__restrict__ slot,
                                            const int32_t *__restrict__ place, const PartArgs &pa,
                                            double *__restrict__ values, double *__restrict__ rhs)
{
    const int64_t i = (int64_t)item * kGatherRows + threadIdx.x / kGatherLanes;
    const int lane = threadIdx.x % kGatherLanes;
    if (i >= N) return;
    const int r0 = rowptr[i], len = rowptr[i + 1] - r0;
    const int q0 = ptr[i], q1 = ptr[i + 1];
    double b = 0.0;
    for (int j0 = 0; j0 < len; j0 += 4 * kGatherLanes) {
        double s[4] = {0.0, 0.0, 0.0, 0.0};
        int j[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            j[v] = j0 + v * kGatherLanes + lane;
            if (j[v] >= len) j[v] = 0;
        }
        for (int q = q0; q < q1; q += kGatherLanes) {
            const int qi = q + lane < q1 ? q + lane : q;
            const int pl = place[qi], sl = slot[qi];
            const int n = q1 - q < kGatherLanes ? q1 - q : kGatherLanes;
            for (int u = 0; u < n; u += 2) {
                const bool two = u + 1 < n;
                const double *w0 = pa.img + __shfl(pl, u, kGatherLanes);
                const double *w1 = pa.img + __shfl(pl, two ? u + 1 : u, kGatherLanes);
                double x0[4], x1[4];
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    x0[v] = w0[j[v]];
                    x1[v] = w1[j[v]];
                }
                if (j0 == 0) {
                    const int t0 = __shfl(sl, u, kGatherLanes), t1 = __shfl(sl, two ? u + 1 : u, kGatherLanes);
                    if (lane < NRHS) {
                        b += pa.sums[lane * pa.VT + t0];
                        if (two) b += pa.sums[lane * pa.VT + t1];
                    }
                }
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    s[v] += x0[v];
                    if (two) s[v] += x1[v];
                }
            }
        }
#pragma unroll
        for (int v = 0; v < 4; ++v)
            if (j0 + v * kGatherLanes + lane < len) values[r0 + j0 + v * kGatherLanes + lane] = s[v];
    }
    if (lane < NRHS) rhs[lane * N + i] = b;
}

template <int NRHS>
__global__ void __launch_bounds__(256) k_part_gather(GatherArgs g)
{
    if (blockIdx.x < kGatherStatus) {
        if (blockIdx.x == 0) reduce_status<256>(g.st);
        return;
    }
    part_gather<NRHS>(xcd_item(blockIdx.x - kGatherStatus, gridDim.x - kGatherStatus), g.N, g.rowptr, g.ptr, g.slot,
                      g.place, g.pa, g.values, g.rhs);
}

// The same for several meshes at once (the serving runtime's hybrid requests):
// one launch per element type and one for the gathers, as k_bat_assemble.  Each
// request's sums are those of its launches alone.  A launch per request and
// type leaves most of the chip idle on small meshes: a saturated server then
// spent 0.27 / 0.39 / 0.58 ms per request of 4^3 / 8^3 / 12^3 cells, in these
// common launches 0.20 / 0.30 / 0.48 (colour by colour 0.19 / 0.32-0.39 / 0.56).
// The momentum kernel of hexahedra holds its arguments by pointer and spills 43
// registers, the one alone 16; the times are with that.
template <class EL, int OP>
__global__ void __launch_bounds__(64 * Split<EL>::W, 2) k_bat_part(const char *__restrict__ table, AsmBatch B)
{
    int j = 0;
    while (j + 1 < B.n && (int)blockIdx.x >= B.wgs[j + 1]) ++j;
    const char *const entry = table + (size_t)B.slot[j] * kKArgsBytes;
    const KArgs &k = *(const KArgs *)entry;
    const GatherArgs &g = *(const GatherArgs *)(entry + kGatherArgsAt);
    part_block<EL, OP, double, double>(k, g.pa, k.color_blk[B.first[j] + (int)blockIdx.x - B.wgs[j]]);
}

template <int NRHS>
__global__ void __launch_bounds__(256) k_bat_part_gather(const char *__restrict__ table, AsmBatch B)
{
    int j = 0;
    while (j + 1 < B.n && (int)blockIdx.x >= B.wgs[j + 1]) ++j;
    const GatherArgs &g = *(const GatherArgs *)(table + (size_t)B.slot[j] * kKArgsBytes + kGatherArgsAt);
    const int item = (int)blockIdx.x - B.wgs[j] - kGatherStatus;
    if (item < 0) {
        if (item == -kGatherStatus) reduce_status<256>(g.st);
        return;
    }
    part_gather<NRHS>(item, g.N, g.rowptr, g.ptr, g.slot, g.place, g.pa, g.values, g.rhs);
}

template <class EL, int OP>
void launch_part_op(const AsmLaunch &L, KArgs k, const PartArgs &pa, bool mixed, bool hybrid, hipStream_t s)
{
    k.blk_offset = L.first;
    const dim3 grid(L.count), block(64 * Split<EL>::W);
    // (a HEX08 block is one of a hybrid mesh: a mesh of HEX08 takes k_own)
    if (!mixed) hipLaunchKernelGGL((k_part<EL, OP, double, double>), grid, block, L.lds[OP], s, k, pa);
    else if (hybrid || EL::NEN == 8) hipLaunchKernelGGL((k_part<EL, OP, float, double>), grid, block, L.lds[OP], s, k, pa);
    else if constexpr (EL::NEN != 8) hipLaunchKernelGGL((k_part<EL, OP, float, float>), grid, block, L.lds[OP], s, k, pa);
}

template <class EL>
void launch_part(const AsmLaunch &L, const KArgs &k, const PartArgs &pa, int op, bool mixed, bool hybrid, hipStream_t s)
{
    switch (op) {
    case OP_MOM: launch_part_op<EL, OP_MOM>(L, k, pa, mixed, hybrid, s); break;
    case OP_SCA: launch_part_op<EL, OP_SCA>(L, k, pa, mixed, hybrid, s); break;
    default: launch_part_op<EL, OP_POI>(L, k, pa, mixed, hybrid, s); break;
    }
}

constexpr int kStatusThreads = 1024;
__global__ void __launch_bounds__(kStatusThreads) k_asm_status(StatusArgs st)
{
    reduce_status<kStatusThreads>(st);
}

template <class EL, int OP, class Q>
void launch_one(const AsmLaunch &L, KArgs k, hipStream_t s)
{
    k.blk_offset = L.first;
    hipLaunchKernelGGL((k_assemble<EL, OP, Q>), dim3(L.count), dim3(64 * Split<EL>::W), L.lds[OP], s, k);
}

template <class EL, int FORM>
void launch_residual(const AsmLaunch &L, KArgs k, hipStream_t s)
{
    k.blk_offset = L.first;
    hipLaunchKernelGGL((k_residual<EL, FORM>), dim3(L.count), dim3(64 * Split<EL>::W), L.lds[OP_RES], s, k);
}

template <class EL>
void launch_type(const AsmLaunch &L, const KArgs &k, int op, bool mixed, hipStream_t s)
{
    switch (op) {
    case OP_MOM: mixed ? launch_one<EL, OP_MOM, float>(L, k, s) : launch_one<EL, OP_MOM, double>(L, k, s); break;
    case OP_SCA: mixed ? launch_one<EL, OP_SCA, float>(L, k, s) : launch_one<EL, OP_SCA, double>(L, k, s); break;
    case OP_POI: mixed ? launch_one<EL, OP_POI, float>(L, k, s) : launch_one<EL, OP_POI, double>(L, k, s); break;
    // element-vector passes are FP64 only
    case OP_RES:
        switch (k.form) {
        case 0: launch_residual<EL, 0>(L, k, s); break;
        case 1: launch_residual<EL, 1>(L, k, s); break;
        case 2: launch_residual<EL, 2>(L, k, s); break;
        default: launch_residual<EL, 3>(L, k, s); break;
        }
        break;
    case OP_GRD: launch_one<EL, OP_GRD, double>(L, k, s); break;
    case OP_SRS: launch_one<EL, OP_SRS, double>(L, k, s); break;
    default: launch_one<EL, OP_DIV, double>(L, k, s); break;
    }
}

// ---- element-vector passes: HEX08
// An element-vector pass on one HEX08 element (FP64; the terms of
// element_vector_point, fields in LDS as there): per component a source s
// tested with N_a and a flux q tested with the reference gradient of N_a.
// One slab of four points after the other (a rolled loop: both unrolled do
// not fit 256 registers).
template <int OP, int FORM>
__device__ __forceinline__ void hex_vector(const double *nd, int T, const int (&ln0)[8],
                                           double (&B)[OpTraits<OP>::NRHS][8], double &mindet, double inv_dt, double Dk)
{
    constexpr int NRHS = OpTraits<OP>::NRHS;
    constexpr int NQ = OP == OP_RES ? 3 : OP == OP_GRD ? 0 : 1;       // components with a flux
    constexpr int NS = OP == OP_DIV ? 0 : NRHS;                       // components with a source
    constexpr int NG = OP == OP_RES ? 3 : OP == OP_DIV ? 0 : 1;       // fields whose gradient is needed
    constexpr bool FULL = (FORM & FE_FORM_FULL_STRESS) != 0, EMAC = (FORM & FE_FORM_EMAC) != 0;
    int ln[8];
#pragma unroll
    for (int a = 0; a < 8; ++a) ln[a] = ln0[a];
#pragma unroll 1
    for (int gz = 0; gz < 2; ++gz) {
        const double z = gz ? Hex::kG : -Hex::kG;
#pragma unroll
        for (int a = 0; a < 8; ++a) asm volatile("" : "+v"(ln[a]));   // fields are read again, not kept
        SlabGrad X[3], G[NG ? NG : 1];
        double up[3][2][2], rp[2][2], mp[2][2], v[2][2], h[2][2];
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            hex_slab(nd + i * T, ln, z, v, h);
            hex_grad(v, h, X[i]);
        }
        if constexpr (OP != OP_GRD) {
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                hex_slab(nd + (3 + i) * T, ln, z, v, h);
                if constexpr (OP == OP_RES) hex_grad(v, h, G[i]);
                hex_points(v, up[i]);
            }
            hex_slab(nd + 6 * T, ln, z, v, h);
            hex_points(v, rp);
        }
        if constexpr (OP == OP_RES) {
            hex_slab(nd + 7 * T, ln, z, v, h);
            hex_points(v, mp);
        }
        if constexpr (OP == OP_GRD || OP == OP_SRS) {
            hex_slab(nd + (OP == OP_GRD ? 3 : 7) * T, ln, z, v, h);
            hex_grad(v, h, G[0]);
        }
        double s[NS ? NS : 1][2][2], q0[NQ ? NQ : 1][2] = {}, q1[NQ ? NQ : 1][2] = {}, q2[NQ ? NQ : 1][2][2];
#pragma unroll
        for (int gx = 0; gx < 2; ++gx)
#pragma unroll
            for (int gy = 0; gy < 2; ++gy) {
                double C[3][3];
                const double det = hex_cofactors(X, gx, gy, C);
                mindet = fmin(mindet, det);
                double uh[3];   // det J times the velocity's reference components
                if constexpr (OP != OP_GRD) {
#pragma unroll
                    for (int j = 0; j < 3; ++j)
                        uh[j] = C[j][0] * up[0][gx][gy] + C[j][1] * up[1][gx][gy] + C[j][2] * up[2][gx][gy];
                }
                if constexpr (OP == OP_GRD) {
#pragma unroll
                    for (int i = 0; i < 3; ++i)
                        s[i][gx][gy] = C[0][i] * G[0].x[gy] + C[1][i] * G[0].y[gx] + C[2][i] * G[0].z[gx][gy];
                } else if constexpr (OP == OP_DIV) {
                    const double w = rp[gx][gy] * inv_dt;
                    q0[0][gy] += w * uh[0];
                    q1[0][gx] += w * uh[1];
                    q2[0][gx][gy] = w * uh[2];
                } else {
                    const double r = rp[gx][gy];
                    // viscosity (or rho D) over det J
                    const double k = (OP == OP_RES ? mp[gx][gy] : r * Dk) / det;
                    double D[3][3];   // k C C^T: flux j = sum_l D[j][l] d/dxi_l
                    if constexpr (!FULL) {
#pragma unroll
                        for (int j = 0; j < 3; ++j)
#pragma unroll
                            for (int l = j; l < 3; ++l)
                                D[j][l] = D[l][j] = k * (C[j][0] * C[l][0] + C[j][1] * C[l][1] + C[j][2] * C[l][2]);
                    }
                    double gp[3][3], div = 0.0;   // det J times du_i / dx_j
                    if constexpr (OP == OP_RES && (FULL || EMAC)) {
#pragma unroll
                        for (int i = 0; i < 3; ++i)
#pragma unroll
                            for (int j = 0; j < 3; ++j)
                                gp[i][j] = C[0][j] * G[i].x[gy] + C[1][j] * G[i].y[gx] + C[2][j] * G[i].z[gx][gy];
                        div = gp[0][0] + gp[1][1] + gp[2][2];
                    }
#pragma unroll
                    for (int i = 0; i < NG; ++i) {
                        const double g0 = G[i].x[gy], g1 = G[i].y[gx], g2 = G[i].z[gx][gy];
                        double adv = uh[0] * g0 + uh[1] * g1 + uh[2] * g2;
                        if constexpr (EMAC) adv += div * up[i][gx][gy];
                        s[i][gx][gy] = -r * adv;
                        double f[3];
                        if constexpr (FULL) {
                            double t[3];
#pragma unroll
                            for (int j = 0; j < 3; ++j) t[j] = k * (gp[i][j] + gp[j][i]);
#pragma unroll
                            for (int j = 0; j < 3; ++j) f[j] = C[j][0] * t[0] + C[j][1] * t[1] + C[j][2] * t[2];
                        } else {
#pragma unroll
                            for (int j = 0; j < 3; ++j) f[j] = D[j][0] * g0 + D[j][1] * g1 + D[j][2] * g2;
                        }
                        q0[i][gy] -= f[0];
                        q1[i][gx] -= f[1];
                        q2[i][gx][gy] = -f[2];
                    }
                    s[NG][gx][gy] = r * det;   // lumped mass
                }
            }
        // to the nodes: the slab's share of (ix, iy, iz)
        const double L[2] = {0.5 * (1.0 - z), 0.5 * (1.0 + z)};
#pragma unroll
        for (int c = 0; c < NRHS; ++c) {
            double n0[2] = {}, n1[2] = {};   // xi flux by iy (halved at ix), eta flux by ix
            if (c < NQ) {
                line_nodes(q0[c < NQ ? c : 0][0], q0[c < NQ ? c : 0][1], n0[0], n0[1]);
                line_nodes(q1[c < NQ ? c : 0][0], q1[c < NQ ? c : 0][1], n1[0], n1[1]);
            }
#pragma unroll
            for (int iz = 0; iz < 2; ++iz) {
                double t[2][2], w[2][2];
#pragma unroll
                for (int gx = 0; gx < 2; ++gx) {
                    double m[2];
#pragma unroll
                    for (int gy = 0; gy < 2; ++gy) {
                        m[gy] = c < NS ? L[iz] * s[c < NS ? c : 0][gx][gy] : 0.0;
                        if (c < NQ) m[gy] += (iz ? 0.5 : -0.5) * q2[c < NQ ? c : 0][gx][gy];
                    }
                    line_nodes(m[0], m[1], t[gx][0], t[gx][1]);
                }
#pragma unroll
                for (int iy = 0; iy < 2; ++iy) line_nodes(t[0][iy], t[1][iy], w[0][iy], w[1][iy]);
#pragma unroll
                for (int ix = 0; ix < 2; ++ix)
#pragma unroll
                    for (int iy = 0; iy < 2; ++iy) {
                        double x = w[ix][iy];
                        if (c < NQ) x += L[iz] * ((ix ? 0.5 : -0.5) * n0[iy] + (iy ? 0.5 : -0.5) * n1[ix]);
                        B[c][hex_node(ix, iy, iz)] += x;
                    }
            }
        }
    }
}

// ---- element-vector passes in one launch per element type ---------------------
// One wave = one block of <= 64 elements, one element per lane.  The block's
// fields are staged in LDS, the lanes add their vectors into the LDS sums of
// the block's nodes in phase order, and the sums go to the block's own places
// of a work array (no other block writes them, so no colours); k_vec_gather
// then adds each node's block sums in block order.  The order of every sum is
// fixed by the plan.
template <class EL, int OP, int FORM>
__global__ void __launch_bounds__(64, 2) k_vec(KArgs k, double *__restrict__ work, int64_t VT)
{
    constexpr int NEN = EL::NEN, NF = OpTraits<OP>::NF, NRHS = OpTraits<OP>::NRHS;
    extern __shared__ double lds[];
    const int blk = k.color_blk[k.blk_offset + xcd_item(blockIdx.x, gridDim.x)];
    const int e0 = k.blk_elem_ptr[blk], ne = k.blk_elem_ptr[blk + 1] - e0;
    const int n0 = k.blk_node_ptr[blk], T = k.blk_node_ptr[blk + 1] - n0;
    const int lane = threadIdx.x;
    const int64_t N = k.N;
    double *nd = lds, *sums = nd + NF * T;   // [NF][T] fields, [NRHS][T] sums
    const bool act = lane < ne;
    const int e = e0 + (act ? lane : 0);
    int ln[NEN];
#pragma unroll
    for (int a = 0; a < NEN; ++a) ln[a] = k.elem_lnode[(int64_t)a * k.E + e];
    const int ph = act ? (int)k.elem_phase[e] : -1, nph = k.blk_nphase[blk];
    for (int t = lane; t < T; t += 64) {
        const int g = k.blk_nodes[n0 + t];
        double f[NF];
        f[0] = k.X[g];
        f[1] = k.X[N + g];
        f[2] = k.X[2 * N + g];
        if constexpr (OP == OP_GRD) {
            f[3] = k.p[g];
        } else {
            f[3] = k.u[g];
            f[4] = k.u[N + g];
            f[5] = k.u[2 * N + g];
            f[6] = k.rho[g];
            if constexpr (OP == OP_RES) f[7] = k.mu[g];
            if constexpr (OP == OP_SRS) f[7] = k.Y[g];
        }
#pragma unroll
        for (int q = 0; q < NF; ++q) nd[q * T + t] = f[q];
#pragma unroll
        for (int r = 0; r < NRHS; ++r) sums[r * T + t] = 0.0;
    }
    __syncthreads();
    double B[NRHS][NEN];
#pragma unroll
    for (int r = 0; r < NRHS; ++r)
#pragma unroll
        for (int a = 0; a < NEN; ++a) B[r][a] = 0.0;
    double mindet = __builtin_huge_val();
    if constexpr (NEN == 8) {
        hex_vector<OP, FORM>(nd, T, ln, B, mindet, 1.0 / k.dt, k.Dk);
    } else {
        Geo<EL> GE;
        load_geo<EL>(nd, T, ln, GE);
        Rows<EL> rows;
#pragma unroll
        for (int a = 0; a < NEN; ++a) rows.v[a] = ln[a];
        double A[NEN][NEN];   // unused: no matrix
        gauss_loop<EL, OP, double, NEN, 0>(GE, nd, nd + 3 * T, T, rows, A, B, mindet, 1.0 / k.dt, k.Dk, FORM);
    }
    for (int p = 0; p < nph; ++p)
        if (ph == p) {
#pragma unroll
            for (int a = 0; a < NEN; ++a)
#pragma unroll
                for (int r = 0; r < NRHS; ++r) lds_add(&sums[r * T + ln[a]], B[r][a]);
        }
    double md = act ? mindet : __builtin_huge_val();
    long long bad = (act && !(mindet > 0.0)) ? (long long)e : (long long)0x7fffffffffffffffLL;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        md = fmin(md, __shfl_xor(md, o));
        const long long ob = __shfl_xor(bad, o);
        bad = ob < bad ? ob : bad;
    }
    if (lane == 0) {
        k.blk_mindet[blk] = md;
        k.blk_bad[blk] = bad == 0x7fffffffffffffffLL ? -1 : bad;
    }
    __syncthreads();
    for (int t = lane; t < T; t += 64)
#pragma unroll
        for (int r = 0; r < NRHS; ++r) work[r * VT + n0 + t] = sums[r * T + t];
}

// out[r][i] = node i's block sums in block order, one thread per node, four
// places at a time, so that their loads are in flight together.  (Nodes of
// one block only, ~40 %, written by k_vec itself instead: the scattered
// stores cost k_vec 6 us on 101^3 HEX08 and saved 3.5 us here.)  The first
// group reduces the status word meanwhile.
template <int NRHS>
__global__ void __launch_bounds__(256) k_vec_gather(int64_t N, int64_t VT, const int32_t *__restrict__ ptr,
                                                    const int32_t *__restrict__ slot,
                                                    const double *__restrict__ work, double *__restrict__ out,
                                                    StatusArgs st)
{
    if (blockIdx.x == 0) {
        reduce_status<256>(st);
        return;
    }
    const int64_t i = (int64_t)(blockIdx.x - 1) * 256 + threadIdx.x;
    if (i >= N) return;
    double s[NRHS];
#pragma unroll
    for (int r = 0; r < NRHS; ++r) s[r] = 0.0;
    const int q0 = ptr[i], q1 = ptr[i + 1];
    for (int q = q0; q < q1; q += 4) {
        int t[4];
        double w[4][NRHS];
#pragma unroll
        for (int j = 0; j < 4; ++j) t[j] = slot[q + j < q1 ? q + j : q];
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int r = 0; r < NRHS; ++r) w[j][r] = work[r * VT + t[j]];
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (q + j < q1) {
#pragma unroll
                for (int r = 0; r < NRHS; ++r) s[r] += w[j][r];
            }
    }
#pragma unroll
    for (int r = 0; r < NRHS; ++r) out[r * N + i] = s[r];
}

template <class EL, int OP, int FORM>
void launch_vec_op(const AsmLaunch &L, KArgs k, double *work, int64_t VT, hipStream_t s)
{
    k.blk_offset = L.first;
    hipLaunchKernelGGL((k_vec<EL, OP, FORM>), dim3(L.count), dim3(64), L.lds[OP], s, k, work, VT);
}

template <class EL>
void launch_vec(const AsmLaunch &L, const KArgs &k, int op, double *work, int64_t VT, hipStream_t s)
{
    switch (op) {
    case OP_RES:
        switch (k.form) {
        case 0: launch_vec_op<EL, OP_RES, 0>(L, k, work, VT, s); break;
        case 1: launch_vec_op<EL, OP_RES, 1>(L, k, work, VT, s); break;
        case 2: launch_vec_op<EL, OP_RES, 2>(L, k, work, VT, s); break;
        default: launch_vec_op<EL, OP_RES, 3>(L, k, work, VT, s); break;
        }
        break;
    case OP_GRD: launch_vec_op<EL, OP_GRD, 0>(L, k, work, VT, s); break;
    case OP_SRS: launch_vec_op<EL, OP_SRS, 0>(L, k, work, VT, s); break;
    default: launch_vec_op<EL, OP_DIV, 0>(L, k, work, VT, s); break;
    }
}

// ---- momentum operator with the full-stress viscous term: 3x3 blocks ------
// Eq. (1)'s viscous term -div(2 mu eps(u)) tested with N_a e_i couples the
// velocity components.  Row (a, i), column (b, k) of the element matrix:
//   delta_ik (M_ab / dt + C_ab + K_ab [+ E_ab]) [+ T_ab[i][k]],
//   T_ab[i][k] = sum_g dV mu_g (dN_a / dx_k)(dN_b / dx_i)   (FE_FORM_FULL_STRESS),
//   E_ab = sum_g dV rho_g (div u)_g N_a N_b                  (FE_FORM_EMAC),
// with M, C, K those of the scalar momentum operator.
//
// One lane per (element, row) task, one work-group per group of whole rows,
// each block row written to HBM once, contiguously.  A group
//   1. stages its nodes' fields in LDS;
//   2. some Gauss points at a time: one lane per (element, point) writes what
//      its tasks share to LDS: grad N_b and s_b = rho dV (N_b / dt + u . grad N_b
//      [+ (div u) N_b]) of every node b, mu dV and rho dV u / dt; then every
//      task adds the points to its 8 block columns in registers (grad N_a .
//      grad N_b is the trace of the full-stress block: one sum more a column);
//   3. adds the columns into the rows' image in LDS, a row's tasks at once:
//      the plan orders each task's columns so that they never meet;
//   4. writes the rows.
// The order of every sum is fixed.  Bound by LDS (32 doubles a task and point, the
// items of ~85 elements a group of 256 tasks) and FP64 arithmetic, 41 of 135 us,
// at two waves a SIMD.  FE_FORM_FULL_STRESS | EMAC on 40^3 HEX08 (134 MB of blocks):
// 135 us against 206 with each task computing its element's points from global
// memory, 390 registers, and a row's tasks adding one after the other (8 x 75
// LDS additions with 8 lanes active).  Whole calls, form 3: 64^3 HEX08 840 -> 512
// us, 30^3 cubes TET04 218 -> 141, 40^3 PEN06 272 -> 187, 30^3 PYR05 370 -> 235,
// hybrid 32^3 286 -> 236.  Groups of 64 or 128 tasks share an element's points
// among fewer (194 and 175 us).
struct BArgs {
    const double *X;
    const uint8_t *etype;
    const int32_t *rowptr;
    const uint32_t *task_meta, *task_perm;
    const uint8_t *task_cols;
    const int4 *wdesc, *wlists;
    const int32_t *wave_elem, *wave_node;
    const uint16_t *wave_ln;
    int class_end[4];   // of several types: see RowPlan
    const int32_t *conn, *alone_elem;   // each task alone
    const uint16_t *alone_meta;
    int stride;
    int64_t N;
    const double *u, *rho, *mu;
    double inv_dt;
    double *values, *rhs;
    double *w_mindet;
    long long *w_bad;
};

// Meshes of several types: eight nodes and points, those that a type lacks zero.
struct AnyElement {
    static constexpr int NEN = 8, NG = 8;
};

// Doubles of one (element, point) item: [8]{grad N_b, s_b}, mu dV, rho dV u / dt,
// padded so that 16 lanes' 16-byte accesses fall on distinct banks.
constexpr int kItemNodes = 32, kItem = 38;
// Doubles of a staged node: x, y, z, u_x, u_y, u_z, rho, mu, padded alike.  Node by
// node, so that an element's reads take one address a node and constant offsets
// (field by field, the 64 addresses of a HEX08 element went to scratch).
constexpr int kBlockNode = 10;

// Shape functions: {d N_b / d xi, N_b} of node b at point g, and the weights, of
// TET04, PYR05, PEN06 and HEX08; zero where the type lacks them.
struct ItemTable {
    double v[4][8][8][4], w[4][8];
};
template <class EL> constexpr void fill_items(ItemTable &t, int type)
{
    for (int g = 0; g < EL::NG; ++g) {
        t.w[type][g] = EL::w(g);
        for (int b = 0; b < EL::NEN; ++b) {
            for (int j = 0; j < 3; ++j) t.v[type][g][b][j] = EL::dN(g, b, j);
            t.v[type][g][b][3] = EL::N(g, b);
        }
    }
}
constexpr ItemTable make_items()
{
    ItemTable t{};
    fill_items<Tet>(t, 0);
    fill_items<Pyr>(t, 1);
    fill_items<Pen>(t, 2);
    fill_items<Hex>(t, 3);
    return t;
}
__constant__ ItemTable kItems = make_items();
__device__ constexpr int item_type(int nen) { return nen == 8 ? 3 : nen - 4; }
__device__ __forceinline__ int item_points(int type) { return type == 0 ? Tet::NG : type == 2 ? Pen::NG : 8; }

// Node b's reference gradient and shape function at point g.  Several types: read
// anew from LDS for each use (the opaque 0), not kept in registers.
template <class EL>
__device__ __forceinline__ void shape(int g, int b, const double2 *tab, double (&d)[3], double &N)
{
    if constexpr (std::is_same<EL, AnyElement>::value) {
        int again = 0;
        asm volatile("" : "+v"(again));
        const double2 t0 = tab[again + 2 * b], t1 = tab[again + 2 * b + 1];
        d[0] = t0.x;
        d[1] = t0.y;
        d[2] = t1.x;
        N = t1.y;
    } else {
        N = RefN<EL>(g, b);
#pragma unroll
        for (int j = 0; j < 3; ++j) d[j] = RefdN<EL>(g, b, j);
    }
}

// The item of point g of an element whose nodes' fields start at nd + ln[b] in
// LDS; returns det J.  g is the wave's, so one type's shape functions are scalar
// operands; of several types they are the lane's, tab in LDS, wg the weight.
// One node's loads at a time (sched_barrier): the block sums hold most of the
// registers.
template <class EL, bool EMAC>
__device__ __forceinline__ double block_item(int g, const double *nd, const int (&ln)[8], const double2 *tab, double wg,
                                             double inv_dt, double *out)
{
    constexpr int NEN = EL::NEN;
    [[maybe_unused]] double gu[3][3] = {};
    double J[3][3] = {}, Ji[3][3], rg = 0.0, mg = 0.0, ag[3] = {0.0, 0.0, 0.0}, div = 0.0;
#pragma unroll
    for (int b = 0; b < NEN; ++b) {
        const double *f = nd + ln[b];
        double d[3], N;
        shape<EL>(g, b, tab, d, N);
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            const double x = f[i], u = f[3 + i];
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                J[i][j] += x * d[j];
                if (EMAC) gu[i][j] += u * d[j];
            }
            ag[i] += N * u;
        }
        rg += N * f[6];
        mg += N * f[7];
        __builtin_amdgcn_sched_barrier(0);
    }
    const double det = invert_jacobian(J, Ji);
    if constexpr (EMAC)
#pragma unroll
        for (int i = 0; i < 3; ++i) div += Ji[0][i] * gu[i][0] + Ji[1][i] * gu[i][1] + Ji[2][i] * gu[i][2];
    const double dV = wg * det, w1 = dV * rg, c0 = w1 * (inv_dt + div);
    double c[3];   // w1 u in reference directions
#pragma unroll
    for (int j = 0; j < 3; ++j) c[j] = w1 * (ag[0] * Ji[j][0] + ag[1] * Ji[j][1] + ag[2] * Ji[j][2]);
#pragma unroll
    for (int b = 0; b < NEN; ++b) {
        double d[3], N;
        shape<EL>(g, b, tab, d, N);
        double2 o0, o1;
        o0.x = Ji[0][0] * d[0] + Ji[1][0] * d[1] + Ji[2][0] * d[2];
        o0.y = Ji[0][1] * d[0] + Ji[1][1] * d[1] + Ji[2][1] * d[2];
        o1.x = Ji[0][2] * d[0] + Ji[1][2] * d[1] + Ji[2][2] * d[2];
        o1.y = c0 * N + c[0] * d[0] + c[1] * d[1] + c[2] * d[2];
        *(double2 *)(out + 4 * b) = o0;
        *(double2 *)(out + 4 * b + 2) = o1;
        __builtin_amdgcn_sched_barrier(0);
    }
    out[kItemNodes] = dV * mg;
#pragma unroll
    for (int i = 0; i < 3; ++i) out[kItemNodes + 1 + i] = w1 * ag[i] * inv_dt;
    return det;
}

// double2 of a kernel's table in LDS: [types][NG][NS]{d N_b / d xi, N_b}, or one
// type's [NG][NS] N_b.
constexpr int item_table(int nen, int ng, bool any) { return any ? 4 * 128 : (nen * ng + 1) / 2; }

template <class EL, int FORM, int NT>
__device__ __forceinline__ void block_group(const BArgs &k, int wi)
{
    constexpr bool FULL = (FORM & FE_FORM_FULL_STRESS) != 0, EMAC = (FORM & FE_FORM_EMAC) != 0;
    constexpr bool ANY = std::is_same<EL, AnyElement>::value;
    constexpr int NS = EL::NEN, NG = EL::NG;
    constexpr int NV = FULL ? 9 : 1;   // values of a block kept in the image
    extern __shared__ double2 lds2[];
    double *lds = (double *)lds2;
    const int4 wd = k.wdesc[wi], wl = k.wlists[wi];
    const int tid = threadIdx.x, ne = wl.y, T = wl.w;
    const int64_t N = k.N;
    double *nd = lds;                       // [T] nodes
    double2 *tab = (double2 *)(nd + kBlockNode * T);
    double *items = (double *)(tab + item_table(EL::NEN, EL::NG, ANY));   // [points][ne] items
    const int r0 = wd.z, nr = wd.w;
    const int64_t v0 = k.rowptr[r0];
    const int L = (int)(k.rowptr[r0 + nr] - v0);
    const int64_t t = wd.x + (tid < wd.y ? tid : 0);
    uint32_t meta = tid < wd.y ? k.task_meta[t] : kRowNoTask;
    const bool live = meta != kRowNoTask;
    const uint32_t perm = live ? k.task_perm[t] : 0x88888888u;
    const bool row_first = live && (meta & kRowFirstTask) != 0;
    meta = live ? meta & ~kRowFirstTask : 0u;
    const uint64_t cols = *(const uint64_t *)(k.task_cols + 8 * t);
    const int le = meta & 255, a = meta >> 8 & 7, rl = meta >> 11 & 255, round = live ? (int)(meta >> 19) : -1;
    const int ro = (int)(k.rowptr[r0 + rl] - v0);
    __shared__ int nround;   // rounds of the group's rows
    if (tid == 0) nround = 0;
    // this lane's element in the item passes
    // (a wave's lanes take one point)
    const int np = row_points(ne, NT), wpp = (ne + 63) / 64, wv = __builtin_amdgcn_readfirstlane(tid / 64);
    const int gi = ne > 0 ? wv / wpp : NG, ie = ne > 0 ? (wv - gi * wpp) * 64 + tid % 64 : 0;
    const bool item = gi < np && ie < ne;
    const int64_t lel = wl.x + (item ? ie : 0);
    const int e = ne > 0 ? k.wave_elem[lel] : 0;
    int ln[8];
    {
        const uint4 q = ne > 0 ? *(const uint4 *)(k.wave_ln + 8 * lel) : uint4{0, 0, 0, 0};
        const uint32_t w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
        for (int b = 0; b < 8; ++b) ln[b] = kBlockNode * (int)(w[b / 2] >> (16 * (b % 2)) & 0xffff);
    }
    // type (of several) of the item's and of the task's element
    [[maybe_unused]] int type = 0, ttype = 0;
    if constexpr (ANY) {
        type = ne > 0 ? item_type(k.etype[e]) : 0;
        ttype = ne > 0 ? item_type(k.etype[k.wave_elem[wl.x + le]]) : 0;
    }
    if constexpr (ANY)
        for (int q = tid; q < item_table(NS, NG, ANY); q += NT) tab[q] = ((const double2 *)&kItems.v[0][0][0][0])[q];
    else
        for (int q = tid; q < NG * NS; q += NT) ((double *)tab)[q] = kItems.v[item_type(NS)][q / NS][q % NS][3];
    for (int q = tid; q < T; q += NT) {
        const int g = k.wave_node[wl.z + q];
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            nd[kBlockNode * q + i] = k.X[i * N + g];
            nd[kBlockNode * q + 3 + i] = k.u[i * N + g];
        }
        nd[kBlockNode * q + 6] = k.rho[g];
        nd[kBlockNode * q + 7] = k.mu[g];
    }
    __syncthreads();

    // FULL: A without s_b, which S sums; else S sums both
    double A[NS][9], S[NS], B[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        S[s] = 0.0;
#pragma unroll
        for (int q = 0; q < 9; ++q) A[s][q] = 0.0;
    }
    int at[NS];   // slot s's node in an item
#pragma unroll
    for (int s = 0; s < NS; ++s) at[s] = 4 * (int)(perm >> (4 * s) & 7);
    double mindet = __builtin_huge_val();
#pragma unroll 1
    for (int g0 = 0; g0 < NG; g0 += np) {
        const int g = g0 + gi;
        if (item && g < NG) {
            double *out = items + kItem * (gi * ne + ie);
            if constexpr (ANY) {
                // a point that the type lacks adds zero
                if (g >= item_points(type))
                    for (int q = 0; q < kItemNodes + 4; ++q) out[q] = 0.0;
                else
                    mindet = fmin(mindet, block_item<EL, EMAC>(g, nd, ln, tab + 128 * type + 16 * g,
                                                                      kItems.w[type][g], k.inv_dt, out));
            } else {
                mindet = fmin(mindet, block_item<EL, EMAC>(g, nd, ln, tab, EL::w(g), k.inv_dt, out));
            }
        }
        __syncthreads();
#pragma unroll 1
        for (int p = 0; p < np && g0 + p < NG; ++p) {
            const double *it = items + kItem * (p * ne + le);
            const double wm = it[kItemNodes],
                         Na = ANY ? tab[128 * ttype + 2 * (NS * (g0 + p) + a) + 1].y
                                  : ((const double *)tab)[NS * (g0 + p) + a];
            double da[3];
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                da[i] = wm * it[4 * a + i];
                B[i] += Na * it[kItemNodes + 1 + i];
            }
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                const double2 x = *(const double2 *)(it + at[s]), y = *(const double2 *)(it + at[s] + 2);
                const double d[3] = {x.x, x.y, y.x};
                S[s] += Na * y.y;
                if constexpr (FULL) {
#pragma unroll
                    for (int i = 0; i < 3; ++i)
#pragma unroll
                        for (int kk = 0; kk < 3; ++kk) A[s][3 * i + kk] += da[kk] * d[i];
                } else {
                    S[s] += da[0] * d[0] + da[1] * d[1] + da[2] * d[2];
                }
                if (s % 2) __builtin_amdgcn_sched_barrier(0);   // two slots' loads in flight, as above
            }
        }
        __syncthreads();
    }

    // the rows' image, over the fields and items
    double *img = lds;            // [NV L] block values of the group's rows
    double *rt = lds + NV * L;    // [3][NT] the tasks' right-hand sides
    int *rows = (int *)(rt + 3 * NT), *first = rows + NT;   // [NT] the tasks' rows; the rows' first tasks
    for (int j = tid; j < NV * L; j += NT) img[j] = 0.0;
#pragma unroll
    for (int i = 0; i < 3; ++i) rt[i * NT + tid] = B[i];
    rows[tid] = live ? rl : -1;
    first[tid] = NT;
    if constexpr (FULL) {
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            S[s] += A[s][0] + A[s][4] + A[s][8];
#pragma unroll
            for (int i = 0; i < 3; ++i) A[s][4 * i] += S[s];
        }
    }
    if (round >= 0) atomicMax(&nround, round + 1);
    __syncthreads();
    if (row_first) first[rl] = tid;
    for (int p = 0; p < nround; ++p) {
        if (round == p) {
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                if ((perm >> (4 * s) & 8) == 0) {
                    double *dst = img + NV * (ro + (int)((cols >> (8 * s)) & 0xff));
#pragma unroll
                    for (int q = 0; q < NV; ++q) lds_add(dst + q, FULL ? A[s][q] : S[s]);
                }
            }
        }
        __syncthreads();   // a row's rounds may lie in two wavefronts
    }
    double *vout = k.values + 9 * v0;
    for (int j = tid; j < 9 * L; j += NT) {
        if constexpr (FULL) vout[j] = img[j];
        else vout[j] = (j % 9) % 4 == 0 ? img[j / 9] : 0.0;
    }
    if (tid < nr) {
        double b[3] = {0.0, 0.0, 0.0};
        // (not the lanes past the group's tasks: 12 us for a group's last row of 15^3 TET04 cubes)
        for (int j = first[tid]; j < wd.y && (rows[j] == tid || rows[j] < 0); ++j)
            if (rows[j] == tid) {
#pragma unroll
                for (int i = 0; i < 3; ++i) b[i] += rt[i * NT + j];
            }
#pragma unroll
        for (int i = 0; i < 3; ++i) k.rhs[i * N + r0 + tid] = b[i];
    }
    // status: the group's smallest det J and first element with det J <= 0
    constexpr long long kNone = 0x7fffffffffffffffLL;
    __shared__ double sd[NT / 64];
    __shared__ long long sb[NT / 64];
    double md = mindet;
    long long bad = !(mindet > 0.0) ? (long long)e : kNone;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        md = fmin(md, __shfl_xor(md, o));
        const long long ob = __shfl_xor(bad, o);
        bad = ob < bad ? ob : bad;
    }
    if (tid % 64 == 0) {
        sd[tid / 64] = md;
        sb[tid / 64] = bad;
    }
    __syncthreads();
    if (tid == 0) {
#pragma unroll
        for (int w = 1; w < NT / 64; ++w) {
            md = fmin(md, sd[w]);
            bad = sb[w] < bad ? sb[w] : bad;
        }
        k.w_mindet[wi] = md;
        k.w_bad[wi] = bad == kNone ? -1 : bad;
    }
}

template <class EL, int FORM, int NT>
__global__ void __launch_bounds__(NT, 2) k_block(BArgs k)
{
    block_group<EL, FORM, NT>(k, xcd_item(blockIdx.x, gridDim.x));
}

// Several types: the groups of several types, the longest, first, then those of
// one type, type after type; one launch, since with one each the chip waits for
// the last groups of every type (hybrid 10^3: 91 us against 51).
template <int FORM, int NT>
__global__ void __launch_bounds__(NT, 2) k_block_types(BArgs k)
{
    // each type's groups over all XCDs
    const int b = blockIdx.x;
    int c = 0, first = 0;
    while (c < 4 && b >= k.class_end[c]) first = k.class_end[c++];
    const int wi = first + xcd_item(b - first, (c < 4 ? k.class_end[c] : (int)gridDim.x) - first);
    switch (c) {
    case 0: block_group<AnyElement, FORM, NT>(k, wi); break;
    case 1: block_group<Hex, FORM, NT>(k, wi); break;
    case 2: block_group<Pyr, FORM, NT>(k, wi); break;
    case 3: block_group<Pen, FORM, NT>(k, wi); break;
    default: block_group<Tet, FORM, NT>(k, wi); break;
    }
}

// The other form (plan.h, RowForm): one lane per task, which computes its
// element's points itself from global memory, one wavefront per group of whole
// rows, added into LDS one task of a row after the other.  Bound by the chain
// of those additions (8 x 75 with 8 lanes active for HEX08) and by its 390
// registers, one wavefront a SIMD.
// Element e's block row a: S[b] (the scalar part, times the identity) and
// T[b][3i + k] (the full-stress coupling), and the right-hand side B[i].
template <class EL, int FORM>
__device__ __forceinline__ void block_row(const BArgs &k, int64_t e, int a, double (&S)[8], double (&T)[8][9],
                                          double (&B)[3], double &mindet)
{
    constexpr int NEN = EL::NEN, NG = EL::NG;
    constexpr bool FULL = (FORM & FE_FORM_FULL_STRESS) != 0, EMAC = (FORM & FE_FORM_EMAC) != 0;
    const int64_t N = k.N;
    int c[NEN];
#pragma unroll
    for (int b = 0; b < NEN; ++b) c[b] = k.conn[e * k.stride + b];
    double xl[3 * NEN], ul[3][NEN], rl[NEN], ml[NEN];
#pragma unroll
    for (int b = 0; b < NEN; ++b) {
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            xl[i * NEN + b] = k.X[i * N + c[b]];
            ul[i][b] = k.u[i * N + c[b]];
        }
        rl[b] = k.rho[c[b]];
        ml[b] = k.mu[c[b]];
    }
    int ln[NEN];
#pragma unroll
    for (int b = 0; b < NEN; ++b) ln[b] = b;
    Geo<EL> GE;
    load_geo<EL>(xl, NEN, ln, GE);
#pragma unroll 1
    for (int g = 0; g < NG; ++g) {
        double Ji[3][3];
        const double det = jacobian_inverse<EL>(g, GE, Ji);
        mindet = fmin(mindet, det);
        double dN[NEN][3];
#pragma unroll
        for (int b = 0; b < NEN; ++b)
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                double s = 0.0;
#pragma unroll
                for (int j = 0; j < 3; ++j) s += Ji[j][i] * RefdN<EL>(g, b, j);
                dN[b][i] = s;
            }
        // the task's own row a (a runtime index: read from the tables, not
        // from the register array)
        double dNa[3];
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            double s = 0.0;
#pragma unroll
            for (int j = 0; j < 3; ++j) s += Ji[j][i] * RefdN<EL>(g, a, j);
            dNa[i] = s;
        }
        const double Na = RefN<EL>(g, a);
        const double dV = EL::w(g) * det;
        double rg = 0.0, mg = 0.0, ag[3] = {0.0, 0.0, 0.0}, diva = 0.0;
#pragma unroll
        for (int b = 0; b < NEN; ++b) {
            const double Nb = RefN<EL>(g, b);
            rg += Nb * rl[b];
            mg += Nb * ml[b];
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                ag[i] += Nb * ul[i][b];
                if (EMAC) diva += dN[b][i] * ul[i][b];
            }
        }
        const double w1 = dV * rg, wm = dV * mg, wa = w1 * Na;
#pragma unroll
        for (int b = 0; b < NEN; ++b) {
            const double Nb = RefN<EL>(g, b);
            const double gg = dNa[0] * dN[b][0] + dNa[1] * dN[b][1] + dNa[2] * dN[b][2];
            const double agb = ag[0] * dN[b][0] + ag[1] * dN[b][1] + ag[2] * dN[b][2];
            double sv = wa * (Nb * k.inv_dt + agb) + wm * gg;
            if (EMAC) sv += wa * diva * Nb;
            S[b] += sv;
            if (FULL) {
#pragma unroll
                for (int i = 0; i < 3; ++i)
#pragma unroll
                    for (int kk = 0; kk < 3; ++kk) T[b][3 * i + kk] += wm * dNa[kk] * dN[b][i];
            }
        }
#pragma unroll
        for (int i = 0; i < 3; ++i) B[i] += wa * ag[i] * k.inv_dt;
    }
}

template <int FORM>
__global__ void __launch_bounds__(64) k_block_alone(BArgs k)
{
    extern __shared__ double lds[];
    const int wi = xcd_item(blockIdx.x, gridDim.x);   // this wave's row range
    const int4 wd = k.wdesc[wi];   // first task, tasks, first row, rows
    const int lane = threadIdx.x;
    const int r0 = wd.z, nr = wd.w;
    const int64_t v0 = k.rowptr[r0];
    const int nimg = 9 * (int)(k.rowptr[r0 + nr] - v0);
    double *img = lds;            // [nimg] block values of the wave's rows
    double *rimg = lds + nimg;    // [3][64] their right-hand sides
    for (int j = lane; j < nimg; j += 64) img[j] = 0.0;
#pragma unroll
    for (int i = 0; i < 3; ++i) rimg[i * 64 + lane] = 0.0;

    const bool live = lane < wd.y;
    const int64_t t = wd.x + (live ? lane : 0);
    const int64_t e = k.alone_elem[t];
    const int meta = k.alone_meta[t];
    const int a = meta & 15, ph = live ? (meta >> 4) : -1;
    const int nen = k.etype ? (int)k.etype[e] : k.stride;
    const uint64_t cols = *(const uint64_t *)(k.task_cols + 8 * t);
    const int row = k.conn[e * k.stride + a];
    const int ro = (int)(k.rowptr[row] - v0), rl = row - r0;
    double S[8], T[8][9], B[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int b = 0; b < 8; ++b) {
        S[b] = 0.0;
#pragma unroll
        for (int q = 0; q < 9; ++q) T[b][q] = 0.0;
    }
    double mindet = __builtin_huge_val();
    if (live) {
        switch (nen) {
        case 8: block_row<Hex, FORM>(k, e, a, S, T, B, mindet); break;
        case 6: block_row<Pen, FORM>(k, e, a, S, T, B, mindet); break;
        case 5: block_row<Pyr, FORM>(k, e, a, S, T, B, mindet); break;
        default: block_row<Tet, FORM>(k, e, a, S, T, B, mindet); break;
        }
    }
    __syncthreads();
    // phases: a row's tasks one after the other in element order; the tasks
    // of one phase hold distinct rows, so no two lanes add to one address
    int nph = ph + 1;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) nph = max(nph, __shfl_xor(nph, o));
    for (int p = 0; p < nph; ++p) {
        if (ph == p) {
#pragma unroll
            for (int b = 0; b < 8; ++b) {
                if (b < nen) {
                    double *dst = img + 9 * (ro + (int)((cols >> (8 * b)) & 0xff));
#pragma unroll
                    for (int i = 0; i < 3; ++i)
#pragma unroll
                        for (int kk = 0; kk < 3; ++kk)
                            lds_add(dst + 3 * i + kk, (i == kk ? S[b] : 0.0) + T[b][3 * i + kk]);
                }
            }
#pragma unroll
            for (int i = 0; i < 3; ++i) lds_add(&rimg[i * 64 + rl], B[i]);
        }
    }
    __syncthreads();
    // each value and right-hand side entry written once, contiguously
    double *vout = k.values + 9 * v0;
    for (int j = lane; j < nimg; j += 64) vout[j] = img[j];
    if (lane < nr) {
#pragma unroll
        for (int i = 0; i < 3; ++i) k.rhs[i * k.N + r0 + lane] = rimg[i * 64 + lane];
    }
    group_status<64>(live ? mindet : __builtin_huge_val(), live && !(mindet > 0.0), e, k.w_mindet + wi, k.w_bad + wi);
}

template <class EL, int NT>
void launch_block_lanes(const BArgs &k, const DevRowPlan &r, int form, hipStream_t s)
{
    constexpr bool ANY = std::is_same<EL, AnyElement>::value;
    const size_t nv = (form & FE_FORM_FULL_STRESS) ? 9 : 1;
    const size_t work = (size_t)(kBlockNode * r.max_nodes + 2 * item_table(EL::NEN, EL::NG, ANY) + kItem * r.max_items);
    const size_t image = (size_t)(nv * (r.max_img / 9) + 4 * NT);
    const size_t lds = std::max(work, image) * sizeof(double);
    const dim3 grid((unsigned)r.n_waves), blk(NT);
    if constexpr (ANY) {
        switch (form) {
        case 0: hipLaunchKernelGGL((k_block_types<0, NT>), grid, blk, lds, s, k); break;
        case 1: hipLaunchKernelGGL((k_block_types<1, NT>), grid, blk, lds, s, k); break;
        case 2: hipLaunchKernelGGL((k_block_types<2, NT>), grid, blk, lds, s, k); break;
        default: hipLaunchKernelGGL((k_block_types<3, NT>), grid, blk, lds, s, k); break;
        }
    } else {
        switch (form) {
        case 0: hipLaunchKernelGGL((k_block<EL, 0, NT>), grid, blk, lds, s, k); break;
        case 1: hipLaunchKernelGGL((k_block<EL, 1, NT>), grid, blk, lds, s, k); break;
        case 2: hipLaunchKernelGGL((k_block<EL, 2, NT>), grid, blk, lds, s, k); break;
        default: hipLaunchKernelGGL((k_block<EL, 3, NT>), grid, blk, lds, s, k); break;
        }
    }
}
template <class EL>
void launch_block(const BArgs &k, const DevRowPlan &r, int form, hipStream_t s)
{
    if (r.lanes == kRowTasks) launch_block_lanes<EL, kRowTasks>(k, r, form, s);
    // (small HEX08 meshes take each task alone)
    else if constexpr (!std::is_same<EL, Hex>::value) launch_block_lanes<EL, kRowTasksSmall>(k, r, form, s);
}

// ---- boundary assembly: equilibrium wall model ---------------------------
// The wall law (Reichardt, kappa = 0.41) at exchange distance delta: u_tau
// from U = u_tau u+(delta u_tau / nu) by a fixed number of Newton steps from
// the laminar guess sqrt(nu U / delta); traction -rho u_tau^2 u_t / |u_t|
// with u_t the tangential part of the interpolated velocity.
constexpr double kWallKappa = 0.41;
constexpr int kWallNewton = 16;

__device__ double wall_utau(double U, double nu, double delta)
{
    if (!(U > 0.0)) return 0.0;
    double ut = sqrt(nu * U / delta);
    for (int k = 0; k < kWallNewton; ++k) {
        const double yp = delta * ut / nu;
        const double e1 = exp(-yp / 11.0), e3 = exp(-yp / 3.0);
        const double up = log(1.0 + kWallKappa * yp) / kWallKappa + 7.8 * (1.0 - e1 - yp / 11.0 * e3);
        const double du = 1.0 / (1.0 + kWallKappa * yp) + 7.8 * (e1 / 11.0 - e3 / 11.0 + yp * e3 / 33.0);
        ut -= (ut * up - U) / (up + yp * du);
        if (ut <= 0.0) ut = 1e-300;
    }
    return ut;
}

// Four lanes per face, one per Gauss point (3-point rule on triangles: the
// fourth lane adds nothing; 2x2 Gauss on quadrilaterals): each lane forms
// its point's w |x_s x x_t| N_a t, the quad of lanes sums them in the fixed
// order (q0 + q1) + (q2 + q3) and its first lane writes the face's part.
__global__ void __launch_bounds__(64) k_wall_faces(int64_t F, const uint8_t *fnen, const int32_t *fconn,
                                                   const double *X, int64_t N, const double *u, const double *rho,
                                                   const double *mu, double delta, double *part)
{
    const int64_t t = (int64_t)blockIdx.x * 64 + threadIdx.x;
    const int64_t f = t >> 2;
    const int q = (int)(t & 3);
    const bool live = f < F;                  // whole quads are live or not (64 = 16 quads)
    const int64_t fs = live ? f : 0;
    const int nn = fnen[fs];
    int c[4];
#pragma unroll
    for (int a = 0; a < 4; ++a) c[a] = fconn[4 * fs + a];
    double P[4][3] = {};
    const double g = 0.57735026918962576451;
    if (live && !(nn == 3 && q == 3)) {
        double Nq[4], ds[4], dt[4], w;
        if (nn == 3) {
            const double s = q == 1 ? 2.0 / 3.0 : 1.0 / 6.0, tt = q == 2 ? 2.0 / 3.0 : 1.0 / 6.0;
            Nq[0] = 1.0 - s - tt; Nq[1] = s; Nq[2] = tt; Nq[3] = 0.0;
            ds[0] = -1.0; ds[1] = 1.0; ds[2] = 0.0; ds[3] = 0.0;
            dt[0] = -1.0; dt[1] = 0.0; dt[2] = 1.0; dt[3] = 0.0;
            w = 1.0 / 6.0;
        } else {
            const double s = (q & 1) ? g : -g, tt = (q & 2) ? g : -g;
#pragma unroll
            for (int a = 0; a < 4; ++a) {
                const double cx = (a == 1 || a == 2) ? 1.0 : -1.0, cy = a >= 2 ? 1.0 : -1.0;
                Nq[a] = 0.25 * (1.0 + cx * s) * (1.0 + cy * tt);
                ds[a] = 0.25 * cx * (1.0 + cy * tt);
                dt[a] = 0.25 * cy * (1.0 + cx * s);
            }
            w = 1.0;
        }
        double xs[3] = {}, xt[3] = {}, ug[3] = {}, rg = 0.0, mg = 0.0;
#pragma unroll
        for (int a = 0; a < 4; ++a) {
            if (a >= nn) break;
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                const double xi = X[i * N + c[a]];
                xs[i] += ds[a] * xi;
                xt[i] += dt[a] * xi;
                ug[i] += Nq[a] * u[i * N + c[a]];
            }
            rg += Nq[a] * rho[c[a]];
            mg += Nq[a] * mu[c[a]];
        }
        const double nv[3] = {xs[1] * xt[2] - xs[2] * xt[1], xs[2] * xt[0] - xs[0] * xt[2],
                              xs[0] * xt[1] - xs[1] * xt[0]};
        const double a2 = nv[0] * nv[0] + nv[1] * nv[1] + nv[2] * nv[2];
        if (a2 > 0.0) {
            const double area = sqrt(a2);
            const double un = (ug[0] * nv[0] + ug[1] * nv[1] + ug[2] * nv[2]) / a2;
            const double ut[3] = {ug[0] - un * nv[0], ug[1] - un * nv[1], ug[2] - un * nv[2]};
            const double U = sqrt(ut[0] * ut[0] + ut[1] * ut[1] + ut[2] * ut[2]);
            if (U > 0.0) {
                const double tau = wall_utau(U, mg / rg, delta);
                const double fac = -w * area * rg * tau * tau / U;
#pragma unroll
                for (int a = 0; a < 4; ++a)
#pragma unroll
                    for (int i = 0; i < 3; ++i) P[a][i] = fac * Nq[a] * ut[i];
            }
        }
    }
    // (q0 + q1) + (q2 + q3): xor 1 pairs q0/q1 and q2/q3, xor 2 then adds the pairs
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            double v = P[a][i];
            v += __shfl_xor(v, 1);
            v += __shfl_xor(v, 2);
            P[a][i] = v;
        }
    if (live && q == 0) {
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
            for (int i = 0; i < 3; ++i) part[(4 * f + a) * 3 + i] = P[a][i];
    }
}

// One thread per wall node: its face entries summed in their fixed order.
__global__ void __launch_bounds__(256) k_wall_gather(int64_t W, const int32_t *nodes, const int32_t *ptr,
                                                     const int32_t *ent, const double *part, int64_t N, double *out)
{
    const int64_t w = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (w >= W) return;
    double s0 = 0.0, s1 = 0.0, s2 = 0.0;
    for (int32_t k = ptr[w]; k < ptr[w + 1]; ++k) {
        const double *p = part + (int64_t)ent[k] * 3;
        s0 += p[0];
        s1 += p[1];
        s2 += p[2];
    }
    const int64_t i = nodes[w];
    out[i] += s0;
    out[N + i] += s1;
    out[2 * N + i] += s2;
}

__global__ void __launch_bounds__(256) k_zero(int64_t n, double *x)
{
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) x[i] = 0.0;
}

}  // namespace

hipError_t launch_wall_traction(const DevMesh &m, const DevWall &w, const double *u, const double *rho,
                                const double *mu, double *out, bool zero_first, hipStream_t s)
{
    if (zero_first) {
        const int64_t n = 3 * m.N;
        const int64_t nb = std::min<int64_t>((n + 255) / 256, 2048);
        hipLaunchKernelGGL(k_zero, dim3((unsigned)std::max<int64_t>(nb, 1)), dim3(256), 0, s, n, out);
    }
    if (w.F == 0) return hipGetLastError();
    hipLaunchKernelGGL(k_wall_faces, dim3((unsigned)((4 * w.F + 63) / 64)), dim3(64), 0, s, w.F, w.nen, w.conn, m.X,
                       m.N, u, rho, mu, w.delta, w.part);
    hipLaunchKernelGGL(k_wall_gather, dim3((unsigned)((w.W + 255) / 256)), dim3(256), 0, s, w.W, w.nodes, w.ptr,
                       w.ent, w.part, m.N, out);
    return hipGetLastError();
}

namespace {

// The coloured kernels' arguments for one operator pass.
KArgs make_kargs(const AsmArgs &a)
{
    const DevMesh &m = *a.m;
    KArgs k{};
    k.X = m.X;
    k.blk_elem_ptr = m.blk_elem_ptr;
    k.blk_node_ptr = m.blk_node_ptr;
    k.blk_nodes = m.blk_nodes;
    k.blk_rdesc = m.blk_rdesc;
    k.blk_rowstart = m.blk_rowstart;
    k.color_blk = m.color_blk;
    k.blk_nphase = m.blk_nphase;
    k.elem_off = m.elem_off;
    k.elem_phase = m.elem_phase;
    k.elem_lnode = m.elem_lnode;
    k.N = m.N;
    k.E = m.E;
    k.u = a.u;
    k.rho = a.rho;
    k.mu = a.mu;
    k.Y = a.Y;
    k.p = a.p;
    k.dt = a.dt;
    k.Dk = a.Dk;
    k.values = a.values;
    k.rhs = a.rhs;
    // status scratch lives right after the AsmStatus word: per-block (or,
    // owner assembly, per-group) smallest det J, then first bad element, each
    // sized for the larger of the two counts
    const int64_t nstat = std::max<int64_t>(m.nblk, m.own_G);
    k.blk_mindet = (double *)(a.status + 1);
    k.blk_bad = (long long *)(k.blk_mindet + nstat);
    k.off_stride = m.off_stride;
    k.form = a.form;
    return k;
}

template <class EL>
void launch_bat_part(int op, const AsmBatch &B, const char *table, size_t lds, hipStream_t s)
{
    if (op == OP_MOM)
        hipLaunchKernelGGL((k_bat_part<EL, OP_MOM>), dim3(B.wgs[B.n]), dim3(64 * Split<EL>::W), lds, s, table, B);
    else
        hipLaunchKernelGGL((k_bat_part<EL, OP_POI>), dim3(B.wgs[B.n]), dim3(64 * Split<EL>::W), lds, s, table, B);
}

template <class EL>
void launch_bat(int op, const AsmBatch &B, const KArgs *ks, size_t lds, hipStream_t s)
{
    if (op == OP_MOM)
        hipLaunchKernelGGL((k_bat_assemble<EL, OP_MOM>), dim3(B.wgs[B.n]), dim3(64 * Split<EL>::W), lds, s, ks, B);
    else
        hipLaunchKernelGGL((k_bat_assemble<EL, OP_POI>), dim3(B.wgs[B.n]), dim3(64 * Split<EL>::W), lds, s, ks, B);
}

}  // namespace

// The gather of one operator pass by blocks.
static GatherArgs make_gather(const AsmArgs &a, const KArgs &k)
{
    const DevMesh &m = *a.m;
    return GatherArgs{m.N, m.rowptr, m.node_slot_ptr, m.node_slot, m.node_img,
                      PartArgs{m.blk_img_ptr, a.img_work, a.img_work + m.img_total, m.vec_T}, a.values, a.rhs,
                      StatusArgs{k.blk_mindet, k.blk_bad, m.nblk, a.status_out ? a.status_out : a.status}};
}

void fill_kargs(const AsmArgs &a, void *out)
{
    KArgs k = make_kargs(a);
    memset(out, 0, kKArgsBytes);
    if (a.img_work) {
        k.color_blk = a.m->vec_blk;
        const GatherArgs g = make_gather(a, k);
        memcpy((char *)out + kGatherArgsAt, &g, sizeof g);
    }
    memcpy(out, &k, sizeof(KArgs));
}

// launch_assemble_batch of meshes that assemble by blocks with a gather.
static hipError_t launch_part_batch(const AsmArgs *a, const int *slot, int n, const char *table, hipStream_t s)
{
    static_assert(kGatherArgsAt + sizeof(GatherArgs) <= kKArgsBytes, "the device table's slot size");
    const int op = a[0].op;
    for (int nen : {8, 6, 5, 4}) {
        AsmBatch B{};
        size_t lds = 0;
        for (int i = 0; i < n; ++i)
            for (const AsmLaunch &L : a[i].m->vec_launches) {
                if (L.nen != nen) continue;
                B.slot[B.n] = slot[i];
                B.first[B.n] = L.first;
                B.wgs[B.n + 1] = B.wgs[B.n] + L.count;
                lds = std::max(lds, L.lds[op]);
                ++B.n;
            }
        if (B.n == 0) continue;
        switch (nen) {
        case 8: launch_bat_part<Hex>(op, B, table, lds, s); break;
        case 6: launch_bat_part<Pen>(op, B, table, lds, s); break;
        case 5: launch_bat_part<Pyr>(op, B, table, lds, s); break;
        default: launch_bat_part<Tet>(op, B, table, lds, s); break;
        }
        const hipError_t err = hipGetLastError();
        if (err != hipSuccess) return err;
    }
    AsmBatch B{};
    for (int i = 0; i < n; ++i) {
        B.slot[i] = slot[i];
        B.wgs[i + 1] = B.wgs[i] + (int)gather_groups(a[i].m->N);
    }
    B.n = n;
    if (op == OP_MOM) hipLaunchKernelGGL(k_bat_part_gather<3>, dim3(B.wgs[n]), dim3(256), 0, s, table, B);
    else hipLaunchKernelGGL(k_bat_part_gather<1>, dim3(B.wgs[n]), dim3(256), 0, s, table, B);
    return hipGetLastError();
}

hipError_t launch_assemble_batch(const AsmArgs *a, const int *slot, int n, const void *kargs_d, hipStream_t s)
{
    if (n < 1 || n > kMaxBatch) return hipErrorInvalidValue;
    const int op = a[0].op;
    if (op != OP_MOM && op != OP_POI) return hipErrorInvalidValue;
    size_t nl = 0;
    for (int i = 0; i < n; ++i) {
        if (a[i].op != op || a[i].m->own_G > 0 || (a[i].img_work != nullptr) != (a[0].img_work != nullptr))
            return hipErrorInvalidValue;
        nl = std::max(nl, a[i].m->launches.size());
    }
    if (a[0].img_work) return launch_part_batch(a, slot, n, (const char *)kargs_d, s);
    const KArgs *ks = (const KArgs *)kargs_d;
    // launch li of every mesh, one launch per element type; launch li + 1
    // after it, so each mesh keeps its own colour order
    for (size_t li = 0; li < nl; ++li) {
        for (int nen : {8, 6, 5, 4}) {
            AsmBatch B{};
            size_t lds = 0;
            for (int i = 0; i < n; ++i) {
                const std::vector<AsmLaunch> &Ls = a[i].m->launches;
                if (li >= Ls.size() || Ls[li].nen != nen || Ls[li].count == 0) continue;
                B.slot[B.n] = slot[i];
                B.first[B.n] = Ls[li].first;
                B.wgs[B.n + 1] = B.wgs[B.n] + Ls[li].count;
                lds = std::max(lds, Ls[li].lds[op]);
                ++B.n;
            }
            if (B.n == 0) continue;
            switch (nen) {
            case 8: launch_bat<Hex>(op, B, ks, lds, s); break;
            case 6: launch_bat<Pen>(op, B, ks, lds, s); break;
            case 5: launch_bat<Pyr>(op, B, ks, lds, s); break;
            default: launch_bat<Tet>(op, B, ks, lds, s); break;
            }
            const hipError_t err = hipGetLastError();
            if (err != hipSuccess) return err;
        }
    }
    // each mesh's status word from its per-block scratch (as launch_assemble)
    for (int i = 0; i < n; ++i) {
        const KArgs k = make_kargs(a[i]);
        hipLaunchKernelGGL(k_asm_status, dim3(1), dim3(kStatusThreads), 0, s,
                           StatusArgs{k.blk_mindet, k.blk_bad, a[i].m->nblk,
                                      a[i].status_out ? a[i].status_out : a[i].status});
    }
    return hipGetLastError();
}

hipError_t launch_assemble(const AsmArgs &a, bool mixed, hipStream_t s)
{
    const DevMesh &m = *a.m;
    if (a.op < 0 || a.op >= kNumOps) return hipErrorInvalidValue;
    KArgs k = make_kargs(a);
    AsmStatus *const out = a.status_out ? a.status_out : a.status;
    if (a.scalars != 1 && (a.scalars < 1 || a.scalars > kOwnScalars || a.op != OP_SCA || !mixed || m.own_G <= 0 || m.nen != 8))
        return hipErrorInvalidValue;
    if (a.op < OP_RES && m.own_G > 0) {
        // matrix operators of a HEX08 mesh, or another in poor order: the owner
        // assembly, one launch
        OArgs o{};
        o.X = m.X;
        o.rowptr = m.rowptr;
        o.groups = m.own_groups;
        o.node_ptr = m.own_node_ptr;
        o.nodes = m.own_nodes;
        o.elem = m.own_elem;
        o.nphase = m.own_nphase;
        o.ln = m.own_ln;
        o.off = m.own_off;
        o.phase = m.own_phase;
        o.ln_stride = m.own_ln_stride;
        o.off_stride = m.own_off_stride;
        o.N = m.N;
        o.u = a.u;
        o.rho = a.rho;
        o.mu = a.mu;
        o.Y = a.Y;
        o.dt = a.dt;
        o.D[0] = a.Dk;
        for (int c = 1; c < a.scalars; ++c) o.D[c] = a.D_next[c - 1];
        o.nnz = m.nnz;
        o.values = a.values;
        o.rhs = a.rhs;
        o.g_mindet = k.blk_mindet;
        o.g_bad = k.blk_bad;
        const int nf = a.op == OP_POI ? 7 : 8, nrhs = a.op == OP_MOM ? 3 : 1;
        const int copies = m.nen == 8 ? 1 : kOwnTasks / 64;
        // x, y, z in FP64, the other fields in the quadrature's precision
        const size_t fb = mixed ? sizeof(float) : sizeof(double);
        const size_t fields = 3 * (size_t)m.own_max_nodes + ((nf - 4 + a.scalars) * (size_t)m.own_max_nodes * fb + 7) / 8;
        const size_t lds = (fields + (size_t)copies * (m.own_max_img + nrhs * m.own_max_rows)) * sizeof(double);
        switch (m.nen) {
        case 8: launch_own(o, a.op, a.scalars, m.own_G, lds, mixed, s); break;
        case 6: launch_own_copies<Pen>(o, a.op, m.own_G, lds, mixed, s); break;
        case 5: launch_own_copies<Pyr>(o, a.op, m.own_G, lds, mixed, s); break;
        case 4: launch_own_copies<Tet>(o, a.op, m.own_G, lds, mixed, s); break;
        default: return hipErrorInvalidValue;
        }
        const hipError_t err = hipGetLastError();
        if (err != hipSuccess) return err;
        if (!a.want_status) return hipSuccess;
        hipLaunchKernelGGL(k_asm_status, dim3(1), dim3(kStatusThreads), 0, s,
                           StatusArgs{k.blk_mindet, k.blk_bad, m.own_G, out});
        return hipGetLastError();
    }
    if (a.op < OP_RES && a.img_work && m.img_total > 0) {
        // matrix operators of the other meshes: by blocks, then the gather
        k.color_blk = m.vec_blk;
        const GatherArgs g = make_gather(a, k);
        for (const AsmLaunch &L : m.vec_launches) {
            switch (L.nen) {
            case 8: launch_part<Hex>(L, k, g.pa, a.op, mixed, m.hybrid, s); break;
            case 6: launch_part<Pen>(L, k, g.pa, a.op, mixed, m.hybrid, s); break;
            case 5: launch_part<Pyr>(L, k, g.pa, a.op, mixed, m.hybrid, s); break;
            case 4: launch_part<Tet>(L, k, g.pa, a.op, mixed, m.hybrid, s); break;
            default: return hipErrorInvalidValue;
            }
            const hipError_t err = hipGetLastError();
            if (err != hipSuccess) return err;
        }
        const dim3 grid((unsigned)gather_groups(m.N)), block(256);
        if (a.op == OP_MOM) hipLaunchKernelGGL(k_part_gather<3>, grid, block, 0, s, g);
        else hipLaunchKernelGGL(k_part_gather<1>, grid, block, 0, s, g);
        return hipGetLastError();
    }
    if (a.op >= OP_RES && a.vec_work) {
        // element-vector passes: one launch per element type, then the gather
        k.color_blk = m.vec_blk;
        for (const AsmLaunch &L : m.vec_launches) {
            switch (L.nen) {
            case 8: launch_vec<Hex>(L, k, a.op, a.vec_work, m.vec_T, s); break;
            case 6: launch_vec<Pen>(L, k, a.op, a.vec_work, m.vec_T, s); break;
            case 5: launch_vec<Pyr>(L, k, a.op, a.vec_work, m.vec_T, s); break;
            case 4: launch_vec<Tet>(L, k, a.op, a.vec_work, m.vec_T, s); break;
            default: return hipErrorInvalidValue;
            }
            const hipError_t err = hipGetLastError();
            if (err != hipSuccess) return err;
        }
        const dim3 grid((unsigned)((m.N + 255) / 256) + 1), block(256);
        const StatusArgs st{k.blk_mindet, k.blk_bad, m.nblk, out};
        switch (a.op) {
        case OP_RES: hipLaunchKernelGGL(k_vec_gather<4>, grid, block, 0, s, m.N, m.vec_T, m.node_slot_ptr, m.node_slot, a.vec_work, a.rhs, st); break;
        case OP_GRD: hipLaunchKernelGGL(k_vec_gather<3>, grid, block, 0, s, m.N, m.vec_T, m.node_slot_ptr, m.node_slot, a.vec_work, a.rhs, st); break;
        case OP_SRS: hipLaunchKernelGGL(k_vec_gather<2>, grid, block, 0, s, m.N, m.vec_T, m.node_slot_ptr, m.node_slot, a.vec_work, a.rhs, st); break;
        default: hipLaunchKernelGGL(k_vec_gather<1>, grid, block, 0, s, m.N, m.vec_T, m.node_slot_ptr, m.node_slot, a.vec_work, a.rhs, st); break;
        }
        return hipGetLastError();
    }
    // one launch per (colour, element type), in the planned order
    for (const AsmLaunch &L : m.launches) {
        if (L.count == 0) continue;
        switch (L.nen) {
        case 8: launch_type<Hex>(L, k, a.op, mixed, s); break;
        case 6: launch_type<Pen>(L, k, a.op, mixed, s); break;
        case 5: launch_type<Pyr>(L, k, a.op, mixed, s); break;
        case 4: launch_type<Tet>(L, k, a.op, mixed, s); break;
        default: return hipErrorInvalidValue;
        }
        const hipError_t err = hipGetLastError();
        if (err != hipSuccess) return err;
    }
    if (!a.want_status) return hipSuccess;
    hipLaunchKernelGGL(k_asm_status, dim3(1), dim3(kStatusThreads), 0, s,
                       StatusArgs{k.blk_mindet, k.blk_bad, m.nblk, out});
    return hipGetLastError();
}

hipError_t launch_assemble_block(const DevMesh &m, const DevRowPlan &r, int form, double dt, const double *u,
                                 const double *rho, const double *mu, double *values, double *rhs,
                                 AsmStatus *status, hipStream_t s)
{
    if (r.n_waves <= 0) return hipErrorInvalidValue;
    BArgs k{};
    k.X = m.X;
    k.etype = r.etype;
    k.rowptr = m.rowptr;
    k.task_meta = r.task_meta;
    k.task_perm = r.task_perm;
    k.task_cols = r.task_cols;
    k.wdesc = r.wdesc;
    k.wlists = r.wlists;
    k.wave_elem = r.wave_elem;
    k.wave_node = r.wave_node;
    k.wave_ln = r.wave_ln;
    k.N = m.N;
    k.u = u;
    k.rho = rho;
    k.mu = mu;
    k.inv_dt = 1.0 / dt;
    k.values = values;
    k.rhs = rhs;
    k.w_mindet = r.w_mindet;
    k.w_bad = r.w_bad;
    if (r.lanes != kRowTasks && (r.lanes != kRowTasksSmall || (r.nen == 8 && !r.alone))) return hipErrorInvalidValue;
    for (int c = 0; c < 4; ++c) k.class_end[c] = r.class_end[c];
    if (r.alone) {
        k.conn = r.conn;
        k.stride = r.stride;
        k.alone_elem = r.alone_elem;
        k.alone_meta = r.alone_meta;
        const size_t lds = (size_t)(r.max_img + 3 * 64) * sizeof(double);
        const dim3 grid((unsigned)r.n_waves), blk(64);
        switch (form) {
        case 0: hipLaunchKernelGGL(k_block_alone<0>, grid, blk, lds, s, k); break;
        case 1: hipLaunchKernelGGL(k_block_alone<1>, grid, blk, lds, s, k); break;
        case 2: hipLaunchKernelGGL(k_block_alone<2>, grid, blk, lds, s, k); break;
        default: hipLaunchKernelGGL(k_block_alone<3>, grid, blk, lds, s, k); break;
        }
    } else switch (r.nen) {
    case 8: launch_block<Hex>(k, r, form, s); break;
    case 6: launch_block<Pen>(k, r, form, s); break;
    case 5: launch_block<Pyr>(k, r, form, s); break;
    case 4: launch_block<Tet>(k, r, form, s); break;
    default: launch_block<AnyElement>(k, r, form, s); break;
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_asm_status, dim3(1), dim3(kStatusThreads), 0, s,
                       StatusArgs{r.w_mindet, r.w_bad, r.n_waves, status});
    return hipGetLastError();
}

}  // namespace feasm
