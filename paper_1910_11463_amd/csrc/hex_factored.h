// Device functions of the factored block-scaled operator of a structured hex
// mesh (see hex_offdiag in amg_solve.hip for the derivation).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace pair {

struct HexDir {
    double kap[3];
    int in;
};

// sqrt 2 as stored, and its reciprocal: W^{-1} has to invert the W and the
// eigenvalues of the stored value.  (The double nearest to 1 / sqrt 2 is one step up;
// the two roundings then add up in every element: 4.2e-15 of |psi| on 16^3 elements
// and 9.7e-15 on 32^3, uniform, S2, against 1.4e-15 and 1.2e-15 so.)
constexpr double kHexS2 = 1.4142135623730950488;
constexpr double kHexC = 1.0 / kHexS2;

// The eigenvalues sigma_t + kap_x lam_ex + kap_y lam_ey + kap_z lam_0 (lam =
// 2 +- i sqrt2) of an element's diagonal block in the Kronecker-sum basis:
// real part mr, imaginary parts mi, and 1 / |.|^2.  (A tile sweep divides one of
// the four per lane and forms its own.)
struct HexDen {
    double mr, mi[2][2], inv[2][2];
};

__device__ __forceinline__ HexDen hex_den(double sig, const HexDir& dr) {
    HexDen d;
    d.mr = sig + 2.0 * (dr.kap[0] + dr.kap[1] + dr.kap[2]);
#pragma unroll
    for (int ex = 0; ex < 2; ++ex)
#pragma unroll
        for (int ey = 0; ey < 2; ++ey) {
            d.mi[ex][ey] = kHexS2 * ((ex ? -dr.kap[0] : dr.kap[0]) + (ey ? -dr.kap[1] : dr.kap[1]) + dr.kap[2]);
            d.inv[ex][ey] = 1.0 / (d.mr * d.mr + d.mi[ex][ey] * d.mi[ex][ey]);
        }
    return d;
}

// y = [sigma_t I + T_x (+) T_y (+) T_z]^{-1} g with the element's eigenvalues from
// hex_den.
__device__ __forceinline__ void hex_kron_solve(const HexDen& dn, const HexDir& dr, const double gv[8], double y[8]) {
    constexpr double kS2 = kHexS2;
    constexpr double kC = 0.5 * kHexC;
    const int sx = dr.in & 1, sy = (dr.in >> 1) & 1, sz = (dr.in >> 2) & 1;
    // W^{-1} along z (row 0: 1/2 on the inflow-side node, -i C on both)
    double ur[2][2], ui[2][2];
#pragma unroll
    for (int ax = 0; ax < 2; ++ax)
#pragma unroll
        for (int ay = 0; ay < 2; ++ay) {
            const double lo = gv[ax + 2 * ay], hi = gv[ax + 2 * ay + 4];
            ur[ax][ay] = 0.5 * (sz ? hi : lo);
            ui[ax][ay] = -kC * (lo + hi);
        }
    // along y: both eigen-indices (row 1 is the conjugate of row 0)
    double vr[2][2], vi[2][2];
#pragma unroll
    for (int ax = 0; ax < 2; ++ax) {
        const double hr = 0.5 * (sy ? ur[ax][1] : ur[ax][0]), hi = 0.5 * (sy ? ui[ax][1] : ui[ax][0]);
        const double sr = ur[ax][0] + ur[ax][1], si = ui[ax][0] + ui[ax][1];
        vr[ax][0] = hr + kC * si; vi[ax][0] = hi - kC * sr;
        vr[ax][1] = hr - kC * si; vi[ax][1] = hi + kC * sr;
    }
    // along x
    double gr[2][2], gi[2][2];
#pragma unroll
    for (int ey = 0; ey < 2; ++ey) {
        const double hr = 0.5 * (sx ? vr[1][ey] : vr[0][ey]), hi = 0.5 * (sx ? vi[1][ey] : vi[0][ey]);
        const double sr = vr[0][ey] + vr[1][ey], si = vi[0][ey] + vi[1][ey];
        gr[0][ey] = hr + kC * si; gi[0][ey] = hi - kC * sr;
        gr[1][ey] = hr - kC * si; gi[1][ey] = hi + kC * sr;
    }
    // divide by sigma_t + kap_x lam_ex + kap_y lam_ey + kap_z lam_0, lam = 2 +- i sqrt2
    const double mr = dn.mr;
    double zr[2][2], zi[2][2];
#pragma unroll
    for (int ex = 0; ex < 2; ++ex)
#pragma unroll
        for (int ey = 0; ey < 2; ++ey) {
            const double mi = dn.mi[ex][ey];
            const double inv = dn.inv[ex][ey];
            zr[ex][ey] = (gr[ex][ey] * mr + gi[ex][ey] * mi) * inv;
            zi[ex][ey] = (gi[ex][ey] * mr - gr[ex][ey] * mi) * inv;
        }
    // W along x (column 0: 1 on the inflow-side node, -1 + i sqrt2 on the other)
    double pr[2][2], pi[2][2];
#pragma unroll
    for (int ey = 0; ey < 2; ++ey) {
        const double sr = zr[0][ey] + zr[1][ey], si = zi[0][ey] + zi[1][ey];
        const double dre = zr[0][ey] - zr[1][ey], dim = zi[0][ey] - zi[1][ey];
        const double orr = -sr - kS2 * dim, oi = -si + kS2 * dre;
        pr[0][ey] = sx ? orr : sr; pi[0][ey] = sx ? oi : si;
        pr[1][ey] = sx ? sr : orr; pi[1][ey] = sx ? si : oi;
    }
    // along y
    double qr[2][2], qi[2][2];
#pragma unroll
    for (int ax = 0; ax < 2; ++ax) {
        const double sr = pr[ax][0] + pr[ax][1], si = pi[ax][0] + pi[ax][1];
        const double dre = pr[ax][0] - pr[ax][1], dim = pi[ax][0] - pi[ax][1];
        const double orr = -sr - kS2 * dim, oi = -si + kS2 * dre;
        qr[ax][0] = sy ? orr : sr; qi[ax][0] = sy ? oi : si;
        qr[ax][1] = sy ? sr : orr; qi[ax][1] = sy ? si : oi;
    }
    // along z, real part doubled
#pragma unroll
    for (int ax = 0; ax < 2; ++ax)
#pragma unroll
        for (int ay = 0; ay < 2; ++ay) {
            const double same = 2.0 * qr[ax][ay];
            const double other = -2.0 * (qr[ax][ay] + kS2 * qi[ax][ay]);
            y[ax + 2 * ay] = sz ? other : same;
            y[ax + 2 * ay + 4] = sz ? same : other;
        }
}

// y = D_e^{-1} A_eU x_U from the upwind neighbours' face values v_d[t] (t the
// node index with bit d removed; zero where the face is on the inflow boundary),
// with the element's eigenvalues from hex_den.
__device__ __forceinline__ void hex_face_solve_den(const HexDen& dn, const HexDir& dr, const double v0[4],
                                                   const double v1[4], const double v2[4], double y[8]) {
    // g = sum_d -kap_d M1^{-1}[a_d][s_d] v_d
    double al[3][2];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const int sd = (dr.in >> d) & 1;
        al[d][0] = sd == 0 ? -4.0 * dr.kap[d] : 2.0 * dr.kap[d];
        al[d][1] = sd == 1 ? -4.0 * dr.kap[d] : 2.0 * dr.kap[d];
    }
    double gv[8];
#pragma unroll
    for (int a = 0; a < 8; ++a) {
        const int ax = a & 1, ay = (a >> 1) & 1, az = a >> 2;
        gv[a] = al[0][ax] * v0[ay + 2 * az] + al[1][ay] * v1[ax + 2 * az] + al[2][az] * v2[ax + 2 * ay];
    }
    hex_kron_solve(dn, dr, gv, y);
}

__device__ __forceinline__ void hex_face_solve(double sig, const HexDir& dr, const double v0[4],
                                               const double v1[4], const double v2[4], double y[8]) {
    hex_face_solve_den(hex_den(sig, dr), dr, v0, v1, v2, y);
}

__device__ __forceinline__ HexDir load_hex_dir(uint32_t m, const double* __restrict__ kap,
                                               const int32_t* __restrict__ inflow) {
    HexDir d;
    d.kap[0] = kap[3 * m];
    d.kap[1] = kap[3 * m + 1];
    d.kap[2] = kap[3 * m + 2];
    d.in = inflow[m];
    return d;
}

__device__ __forceinline__ void load8(const double* __restrict__ p, double v[8]) {
    const double2* q = reinterpret_cast<const double2*>(p);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const double2 t = q[i];
        v[2 * i] = t.x;
        v[2 * i + 1] = t.y;
    }
}

__device__ __forceinline__ void store8(double* __restrict__ p, const double v[8]) {
    double2* q = reinterpret_cast<double2*>(p);
#pragma unroll
    for (int i = 0; i < 4; ++i) q[i] = make_double2(v[2 * i], v[2 * i + 1]);
}

}  // namespace pair
