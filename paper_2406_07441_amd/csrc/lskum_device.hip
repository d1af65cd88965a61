// Device kernels of the MI355X implicit LSKUM solver (gfx950, wave64).
//
// One iteration (Section 4, Algorithm 3, with the colour sweeps of
// Algorithms 6-7):
//   k_qgrad<...>   x (1 + m)        q-derivatives, eq. (16): first-order pass and
//                                   m inner passes; the optional limiter is
//                                   applied in the last pass
//   k_residual[_tiled]<...>         LSKUM residual eq. (11), (15); local time
//                                   step and scalar diagonal eq. (25), (34)-(35);
//                                   per-point linearisation data for the sweeps
//   k_norm_partial, k_norm_comp     density residual norm per component and the
//                                   convergence test
//   k_sweep<...>   x C colours      forward sweep, eq. (27) first line
//   k_sweep<...>   x C colours      backward sweep, eq. (27) second line
//   k_update                        U += dU and the q-variables of eq. (14)
//
// Mapping: LANES consecutive lanes share a point and split its neighbour
// loop, combining partial sums with cross-lane shuffles in a fixed order;
// points of a block are contiguous (storage order, or colour order in the
// sweeps); block ids are remapped so that consecutive point ranges stay on one
// XCD (each XCD has its own L2).  All per-point sums run in CSR neighbour
// order.  The per-point 4x4 algebra is not a dense contraction, so no matrix
// cores are used.
#include "lskum_internal.h"
#include "lskum_math.h"

#include <cmath>

namespace lskum {

namespace {

constexpr int kBlock = 256;
constexpr double kInvSqrtPi = 0.56418958354775628694807945156077;
constexpr int8_t kWall = 0, kInterior = 1, kOuter = 2;

// Frame points (wall, and outer points under the kinetic far field) split
// their stencil along the tangent t and the normal n = (-t_y, t_x): t+, t-
// and one normal half -- the fluid side (dn > 0, the n- split) at a wall, the
// inner side (dn < 0, the n+ split) at an outer point, whose normal points
// out of the domain.
__device__ __forceinline__ bool in_normal_split(int8_t ty, double dn) {
    return ty == kWall ? dn > 0.0 : dn < 0.0;
}

// Workgroups are dispatched round-robin over the 8 XCDs.  Give XCD x the
// contiguous range of logical blocks [x*per + min(x, rem), ...) so that
// neighbouring point ranges share an L2.
__device__ __forceinline__ int xcd_block(int b, int nb) {
    const int x = b & 7, r = b >> 3;
    const int per = nb >> 3, rem = nb & 7;
    return x * per + (x < rem ? x : rem) + r;
}

// A point takes part in an iteration while its component is active.
__device__ __forceinline__ bool live(const int32_t* __restrict__ comp,
                                     const int32_t* __restrict__ active, int64_t p) {
    return active[comp ? comp[p] : 0] != 0;
}

// Projections onto a wall frame, evaluated without contraction so that split
// membership (the sign of da) is decided exactly as a plain multiply-add would.
__device__ __forceinline__ double dot_nc(double ax, double ay, double bx, double by) {
#pragma clang fp contract(off)
    double r = ax * bx;
    double s = ay * by;
    return r + s;
}

struct Prim {
    double rho, u1, u2, p, sb, isb, rhoE;  // sb = sqrt(beta), isb = 1/sqrt(beta)
};

// Primitive state of a (reconstructed) q vector, eq. (14) inverted:
// beta = -q4/2, u = (q2, q3)/(2 beta), rho = exp(q1 + beta |u|^2) beta^(-1/(gamma-1)),
// p = rho/(2 beta).  Division free: with r = 1/sqrt(beta), 1/(2 beta) = r^2/2 and,
// for gamma = 1.4, beta^(-5/2) = r^5.
__device__ __forceinline__ Prim prim_from_q(const D4& q, double inv_gm1, bool g14) {
    Prim w;
    const double beta = -0.5 * q.w;
    const double r = rsqrt(beta);
    const double i2b = 0.5 * r * r;
    w.u1 = q.y * i2b;
    w.u2 = q.z * i2b;
    const double usq = w.u1 * w.u1 + w.u2 * w.u2;
    const double e = exp_fast(q.x + beta * usq);
    const double r2 = r * r;
    w.rho = g14 ? e * (r2 * r2 * r) : e * exp(-inv_gm1 * log(beta));
    w.p = w.rho * i2b;
    w.sb = beta * r;
    w.isb = r;
    w.rhoE = w.p * inv_gm1 + 0.5 * w.rho * usq;
    return w;
}

// Kinetic split flux G_d^sg of a primitive state along the unit direction (dx, dy)
// (half-range moments of the Maxwellian, eq. 3-6).
__device__ __forceinline__ void split_flux(const Prim& w, double dx, double dy, double sg,
                                           double G[4]) {
    const double ud = w.u1 * dx + w.u2 * dy;
    const double S = ud * w.sb;
    double er, g;
    erf_exp(S, er, g);
    const double A = 0.5 * (1.0 + sg * er);
    const double B = g * (0.5 * kInvSqrtPi) * w.isb;
    const double mass = w.rho * (ud * A + sg * B);
    const double pA = w.p * A;
    G[0] = mass;
    G[1] = pA * dx + w.u1 * mass;
    G[2] = pA * dy + w.u2 * mass;
    G[3] = (w.rhoE + w.p) * ud * A + sg * (w.rhoE + 0.5 * w.p) * B;
}

// ---------------------------------------------------------------------------
// Geometry precompute (once per cloud).
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(kBlock) k_precompute(int64_t n, const D2* __restrict__ xy,
                                                       const D2* __restrict__ frame,
                                                       const int8_t* __restrict__ type,
                                                       const int32_t* __restrict__ off,
                                                       const int32_t* __restrict__ idx,
                                                       PointGeom* __restrict__ geom,
                                                       D4* __restrict__ lsq,
                                                       unsigned long long* __restrict__ counts) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    const D2 r0 = xy[p];
    const int8_t ty = type[p];
    const D2 t = frame[p];
    double sxx = 0, syy = 0, sxy = 0, rmin2 = INFINITY;
    // split sums: a = split direction, b = transverse
    double saa[4] = {0, 0, 0, 0}, sbb[4] = {0, 0, 0, 0}, sab[4] = {0, 0, 0, 0};
    int cnt[4] = {0, 0, 0, 0};
    const int32_t e0 = off[p], e1 = off[p + 1];
    for (int32_t e = e0; e < e1; ++e) {
        const D2 ri = xy[idx[e]];
        const double dx = ri.x - r0.x, dy = ri.y - r0.y;
        sxx += dx * dx;
        syy += dy * dy;
        sxy += dx * dy;
        const double d2 = dx * dx + dy * dy;
        rmin2 = d2 < rmin2 ? d2 : rmin2;
        if (ty != kInterior) {
            const double ds = dot_nc(dx, dy, t.x, t.y);
            const double dn = dot_nc(dx, dy, -t.y, t.x);
            if (ds != 0.0) {
                const int k = ds < 0.0 ? 0 : 1;
                saa[k] += ds * ds; sbb[k] += dn * dn; sab[k] += ds * dn; ++cnt[k];
            }
            if (in_normal_split(ty, dn)) {
                saa[2] += dn * dn; sbb[2] += ds * ds; sab[2] += ds * dn; ++cnt[2];
            }
        } else {
            if (dx != 0.0) {
                const int k = dx < 0.0 ? 0 : 1;
                saa[k] += dx * dx; sbb[k] += dy * dy; sab[k] += dx * dy; ++cnt[k];
            }
            if (dy != 0.0) {
                const int k = dy < 0.0 ? 2 : 3;
                saa[k] += dy * dy; sbb[k] += dx * dx; sab[k] += dx * dy; ++cnt[k];
            }
        }
    }
    PointGeom g;
    const double det = sxx * syy - sxy * sxy;
    if (!(det > 1e-12 * sxx * syy)) {
        atomicAdd(&counts[0], 1ull);  // singular full stencil
        lsq[p] = {0, 0, 0, sqrt(rmin2)};
    } else {
        lsq[p] = {syy / det, -sxy / det, sxx / det, sqrt(rmin2)};
    }
    const int nsplit = ty == kInterior ? 4 : 3;
    double cb[4] = {0, 0, 0, 0}, cab[4] = {0, 0, 0, 0};
    for (int k = 0; k < nsplit; ++k) {
        const double dk = saa[k] * sbb[k] - sab[k] * sab[k];
        if (cnt[k] < 2 || !(dk > 1e-12 * saa[k] * sbb[k])) {
            // degenerate half stencil: contributes 0 (counted for the points
            // that always take part; outer splits only with the far field)
            if (ty != kOuter) atomicAdd(&counts[1], 1ull);
            continue;
        }
        cb[k] = sbb[k] / dk;
        cab[k] = -sab[k] / dk;
    }
    // LS_k(1): the weight sums, with the weights exactly as the kernels form them
    double ls1[4] = {0, 0, 0, 0};
    {
        for (int32_t e = e0; e < e1; ++e) {
            const D2 ri = xy[idx[e]];
            const double dx = ri.x - r0.x, dy = ri.y - r0.y;
            if (ty != kInterior) {
                const double ds = dot_nc(dx, dy, t.x, t.y);
                const double dn = dot_nc(dx, dy, -t.y, t.x);
                if (ds != 0.0) {
                    const int k = ds < 0.0 ? 0 : 1;
                    ls1[k] += cb[k] * ds + cab[k] * dn;
                }
                if (in_normal_split(ty, dn)) ls1[2] += cb[2] * dn + cab[2] * ds;
            } else {
                if (dx != 0.0) {
                    const int k = dx < 0.0 ? 0 : 1;
                    ls1[k] += cb[k] * dx + cab[k] * dy;
                }
                if (dy != 0.0) {
                    const int k = dy < 0.0 ? 2 : 3;
                    ls1[k] += cb[k] * dy + cab[k] * dx;
                }
            }
        }
    }
    for (int k = 0; k < 4; ++k) g.split[k] = {cb[k], cab[k]};
    g.ls1 = {ls1[0], ls1[1], ls1[2], ls1[3]};
    geom[p] = g;
}

// Free stream: rho 1, p 1/gamma, velocity M (cos a, sin a); wall points keep
// the tangential velocity only.
__global__ void __launch_bounds__(kBlock) k_free_stream(int64_t n, const int8_t* __restrict__ type,
                                                        const D2* __restrict__ frame, double gamma,
                                                        const int32_t* __restrict__ comp,
                                                        const double* __restrict__ vinf,
                                                        D4* __restrict__ U) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    const int k = comp ? comp[p] : 0;
    double u1 = vinf[2 * k], u2 = vinf[2 * k + 1];
    if (type[p] == kWall) {
        const D2 t = frame[p];
        const double ut = u1 * t.x + u2 * t.y;
        u1 = ut * t.x;
        u2 = ut * t.y;
    }
    const double rho = 1.0, pr = 1.0 / gamma;
    U[p] = {rho, rho * u1, rho * u2, pr / (gamma - 1.0) + 0.5 * rho * (u1 * u1 + u2 * u2)};
}

// q-variables of eq. (14) from U.
__device__ __forceinline__ D4 q_of_U(const D4& u, double gamma, double inv_gm1, bool& bad) {
    const double rho = u.x;
    const double irho = 1.0 / rho;
    const double u1 = u.y * irho, u2 = u.z * irho;
    const double usq = u1 * u1 + u2 * u2;
    const double p = (gamma - 1.0) * (u.w - 0.5 * rho * usq);
    bad = !(rho > 0.0) || !(p > 0.0);
    const double beta = 0.5 * rho / p;
    return {log(rho) + inv_gm1 * log(beta) - beta * usq, 2.0 * beta * u1, 2.0 * beta * u2,
            -2.0 * beta};
}

__global__ void __launch_bounds__(kBlock) k_q_from_U(int64_t n, double gamma,
                                                     const D4* __restrict__ U, D4* __restrict__ q,
                                                     int32_t* __restrict__ flags) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    bool bad;
    q[p] = q_of_U(U[p], gamma, 1.0 / (gamma - 1.0), bad);
    if (bad) flags[0] = 1;
}

// Cross-lane moves by data-parallel primitives (vector instructions; shuffles
// go through LDS): xor 1 and 2 within a quad, the mirror of 8 lanes, which
// takes a quad's lanes to the other quad's, and lane l of 16 to l + 8.
constexpr int kDppXor1 = 0xB1, kDppXor2 = 0x4E, kDppMirror8 = 0x141, kDppRotate8 = 0x128;
constexpr int kDppQuad1 = 0x55, kDppQuad2 = 0xAA;  // broadcast of a quad's lane 1, 2

template <int CTRL>
__device__ __forceinline__ float dpp(float v) {
    return __int_as_float(
        __builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}
template <int CTRL>
__device__ __forceinline__ double dpp(double v) {
    return __hiloint2double(
        __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xf, 0xf, true),
        __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xf, 0xf, true));
}

// Sums of four values over a point's LANES (4, 8, 16) lanes, scattered: lane l
// gets the sum of value l % 4.  Sixteen lanes come as (first, rest), a lane's
// first entry and the sum of its others, and add up in the order of eight
// lanes: entry l, then l + 8, l + 16, l + 24.  Lists of up to 32 entries thus
// give the same bits with either, and with 32 lanes, where the second half's
// entries first join the first half's lanes (from_second_half).
template <int LANES, class T>
__device__ __forceinline__ T scatter_sum(T a[4], const T rest[4], int lane) {
    if constexpr (LANES == 16) {
        const bool low = lane < 8;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const T other = dpp<kDppRotate8>(rest[v]);
            const T f = dpp<kDppRotate8>(a[v]);
            a[v] += f;
            a[v] += low ? rest[v] : other;
            a[v] += low ? other : rest[v];
        }
    }
#pragma unroll
    for (int v = 0; v < 4; ++v)
        if (LANES >= 8) a[v] += dpp<kDppMirror8>(a[v]);
    const bool hi = lane & 2, odd = lane & 1;
    T x0 = hi ? a[2] : a[0], x1 = hi ? a[3] : a[1];
    x0 += dpp<kDppXor2>(hi ? a[0] : a[2]);
    x1 += dpp<kDppXor2>(hi ? a[1] : a[3]);
    return (odd ? x1 : x0) + dpp<kDppXor1>(odd ? x0 : x1);
}

// For the first 16 of 32 lanes, the value that lane + 16 holds (rows of 16
// lanes change places two by two).
__device__ __forceinline__ int from_second_half(int v) {
    return __builtin_amdgcn_permlane16_swap(v, v, false, false)[1];
}
__device__ __forceinline__ float from_second_half(float v) {
    return __int_as_float(from_second_half(__float_as_int(v)));
}
__device__ __forceinline__ double from_second_half(double v) {
    return __hiloint2double(from_second_half(__double2hiint(v)),
                            from_second_half(__double2loint(v)));
}

// ---------------------------------------------------------------------------
// q-derivatives (eq. 16): first-order pass and Jacobi inner passes, with the
// optional limiter fused into the last pass.
//
// Venkatakrishnan's limiter on the q~ reconstruction (an addition: the paper
// names no limiter).  Per point and component, phi = min over neighbours of
//   (d1^2 + eps^2 + 2 d1 d2) / (d1^2 + 2 d2^2 + d1 d2 + eps^2),
// d2 = -(dx qx + dy qy)/2 the reconstruction increment toward the neighbour,
// d1 the largest (d2 > 0) or smallest (d2 < 0) neighbour difference,
// eps^2 = (K h)^3 with h the nearest-neighbour distance, and phi <= 1.
// With A = d1^2 + eps^2 and d1 d2 >= 0 the ratio is >= 1 for |d2| <= |d1|/2
// and falls with |d2| beyond (its derivative in d2 > 0 has the sign of
// d1 A - 4 A d2 - 4 d1 d2^2 <= 0 there; d2 < 0 is the mirror image), so
// min(1, ratio) is non-increasing in |d2| on each side: the minimum over the
// neighbours is the ratio at the largest positive and the most negative d2.
// The walk therefore only keeps the extremes of dx qx + dy qy, and the ratio
// is formed twice per component.  The limited derivatives phi * (qx, qy) go
// to qxl, qyl; the unlimited ones of that pass to qx_out, qy_out only when
// those are given (a query of the derivatives: the residual reads qxl, qyl).
//
// LANES consecutive lanes share one point and split its neighbours; the LS
// right-hand sides, the neighbour extrema and the limiter minimum are
// combined with cross-lane shuffles.
// ---------------------------------------------------------------------------
template <int LANES>
__device__ __forceinline__ double lane_sum(double v) {
#pragma unroll
    for (int o = LANES / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// The limiter factor of one component from the walk's extremes tlo <= 0 <=
// thi of dx qx + dy qy (d2 = -t/2): the ratio at d2 = -tlo/2 with d1 = dmax
// and at d2 = -thi/2 with d1 = dmin, and 1.
__device__ __forceinline__ double venkat_phi(double tlo, double thi, double dmax, double dmin,
                                             double eps2) {
    double phi = 1.0;
    if (tlo < 0.0) {
        const double d2 = -0.5 * tlo, d1 = dmax;
        const double nu = d1 * d1 + eps2 + 2.0 * d1 * d2;
        const double de = d1 * d1 + 2.0 * d2 * d2 + d1 * d2 + eps2;
        phi = fmin(phi, nu / de);
    }
    if (thi > 0.0) {
        const double d2 = -0.5 * thi, d1 = dmin;
        const double nu = d1 * d1 + eps2 + 2.0 * d1 * d2;
        const double de = d1 * d1 + 2.0 * d2 * d2 + d1 * d2 + eps2;
        phi = fmin(phi, nu / de);
    }
    return fmax(phi, 0.0);
}

// Neighbour data of the q-derivative sums: position, q and (defect
// correction passes) the current derivatives.
struct QNbr {
    D2 r;
    D4 q, gx, gy;
};

template <bool INNER>
__device__ __forceinline__ QNbr load_qnbr(int32_t i, const D2* __restrict__ xy,
                                          const D4* __restrict__ q, const D4* __restrict__ qx,
                                          const D4* __restrict__ qy) {
    QNbr nb{xy[i], q[i], {}, {}};
    if (INNER) {
        nb.gx = qx[i];
        nb.gy = qy[i];
    }
    return nb;
}

constexpr int kDxyCache = 8;  // limiter: LDS slots per thread for neighbour offsets

// Four workgroups per CU: the limited pass fits 128 VGPRs (four wavefronts
// per SIMD), which measured faster than three wavefronts without the bound.
template <bool INNER, bool LIMIT, int LANES>
__global__ void __launch_bounds__(kBlock, 4) k_qgrad(
    int64_t n, double K, const D2* __restrict__ xy, const int32_t* __restrict__ off,
    const int32_t* __restrict__ idx, const D4* __restrict__ lsq,
    const int32_t* __restrict__ comp, const int32_t* __restrict__ active,
    const D4* __restrict__ q, const D4* __restrict__ qx_in, const D4* __restrict__ qy_in,
    D4* __restrict__ qx_out, D4* __restrict__ qy_out, D4* __restrict__ qxl,
    D4* __restrict__ qyl) {
    const int64_t gt = (int64_t)xcd_block(blockIdx.x, gridDim.x) * blockDim.x + threadIdx.x;
    const int64_t p = gt / LANES;
    const int lane = (int)(gt % LANES);
    if (p >= n || !live(comp, active, p)) return;  // uniform over the lanes of a point
    const D2 r0 = xy[p];
    const D4 q0 = q[p];
    const double qv[4] = {q0.x, q0.y, q0.z, q0.w};
    D4 gx0{}, gy0{};
    if (INNER) {
        gx0 = qx_in[p];
        gy0 = qy_in[p];
    }
    double bx[4] = {0, 0, 0, 0}, by[4] = {0, 0, 0, 0};
    double dmax[4] = {0, 0, 0, 0}, dmin[4] = {0, 0, 0, 0};
    // both neighbour walks are software-pipelined: indices two entries ahead,
    // neighbour data one entry ahead of the one being used; past the end the
    // last entry is re-read (in bounds) and not used
    // with the limiter, a lane keeps the offsets of its first kDxyCache
    // entries in LDS for the second walk
    __shared__ D2 dxy_cache[LIMIT ? kDxyCache * kBlock : 1];
    const int32_t e0 = off[p], e1 = off[p + 1], last = e1 - 1;
    if (e0 + lane < e1) {
        int32_t e = e0 + lane;
        int32_t i_next = idx[min(e + LANES, last)];
        QNbr cur = load_qnbr<INNER>(idx[e], xy, q, qx_in, qy_in);
        for (int k = 0; e < e1; e += LANES, ++k) {
            const int32_t i_after = idx[min(e + 2 * LANES, last)];
            const QNbr nxt = load_qnbr<INNER>(i_next, xy, q, qx_in, qy_in);
            const double dx = cur.r.x - r0.x, dy = cur.r.y - r0.y;
            if (LIMIT && k < kDxyCache) dxy_cache[k * kBlock + threadIdx.x] = {dx, dy};
            const D4 qi = cur.q;
            double dq[4] = {qi.x - qv[0], qi.y - qv[1], qi.z - qv[2], qi.w - qv[3]};
            if (LIMIT) {
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    dmax[v] = fmax(dmax[v], dq[v]);
                    dmin[v] = fmin(dmin[v], dq[v]);
                }
            }
            if (INNER) {
                const D4 gxi = cur.gx, gyi = cur.gy;
                dq[0] -= 0.5 * (dx * (gxi.x - gx0.x) + dy * (gyi.x - gy0.x));
                dq[1] -= 0.5 * (dx * (gxi.y - gx0.y) + dy * (gyi.y - gy0.y));
                dq[2] -= 0.5 * (dx * (gxi.z - gx0.z) + dy * (gyi.z - gy0.z));
                dq[3] -= 0.5 * (dx * (gxi.w - gx0.w) + dy * (gyi.w - gy0.w));
            }
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                bx[v] += dx * dq[v];
                by[v] += dy * dq[v];
            }
            cur = nxt;
            i_next = i_after;
        }
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        bx[v] = lane_sum<LANES>(bx[v]);
        by[v] = lane_sum<LANES>(by[v]);
    }
    const D4 L = lsq[p];
    double gx[4], gy[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        gx[v] = L.x * bx[v] + L.y * by[v];
        gy[v] = L.y * bx[v] + L.z * by[v];
    }
    if (lane == 0 && (!LIMIT || qx_out)) {  // the limited pass writes them on request only
        qx_out[p] = {gx[0], gx[1], gx[2], gx[3]};
        qy_out[p] = {gy[0], gy[1], gy[2], gy[3]};
    }
    if (!LIMIT) return;
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
        for (int o = LANES / 2; o > 0; o >>= 1) {
            dmax[v] = fmax(dmax[v], __shfl_xor(dmax[v], o, 64));
            dmin[v] = fmin(dmin[v], __shfl_xor(dmin[v], o, 64));
        }
    const double kh = K * L.w;
    const double eps2 = kh * kh * kh;
    double tlo[4] = {0, 0, 0, 0}, thi[4] = {0, 0, 0, 0};  // extremes of dx qx + dy qy
    int k = 0;
    for (int32_t e = e0 + lane; e < e1; e += LANES, ++k) {
        double dx, dy;
        if (k < kDxyCache) {  // written by this thread in the first walk
            const D2 d = dxy_cache[k * kBlock + threadIdx.x];
            dx = d.x;
            dy = d.y;
        } else {
            const D2 ri = xy[idx[e]];
            dx = ri.x - r0.x;
            dy = ri.y - r0.y;
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const double t = dx * gx[v] + dy * gy[v];
            tlo[v] = fmin(tlo[v], t);
            thi[v] = fmax(thi[v], t);
        }
    }
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
        for (int o = LANES / 2; o > 0; o >>= 1) {
            tlo[v] = fmin(tlo[v], __shfl_xor(tlo[v], o, 64));
            thi[v] = fmax(thi[v], __shfl_xor(thi[v], o, 64));
        }
    if (lane == 0) {
        double phi[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) phi[v] = venkat_phi(tlo[v], thi[v], dmax[v], dmin[v], eps2);
        qxl[p] = {phi[0] * gx[0], phi[1] * gx[1], phi[2] * gx[2], phi[3] * gx[3]};
        qyl[p] = {phi[0] * gy[0], phi[1] * gy[1], phi[2] * gy[2], phi[3] * gy[3]};
    }
}

// The same q-derivative pass with the neighbour gathers staged in LDS.  Tile
// b holds the points tile_pts[b kQTile ...] (-1 past its end: kQTile
// consecutive points, or a block of kQTileJ points by kQTileK rows of a cloud
// stored row by row); the host lists the union of their neighbours
// (tile_idx[tile_off[b] ...], sorted) and gives every CSR entry its
// neighbour's position in that list (lnbr).  The block
// first copies position, q (and the current derivatives) of the listed
// points into LDS -- runs of consecutive indices, so mostly coalesced --
// then every neighbour read of the sums comes from LDS: a point's 24
// neighbour records are shared with the tile's other points instead of being
// gathered 24 times from the caches.  Four lanes per point, each summing
// its neighbours in the order of k_qgrad<INNER, LIMIT, 4>; the compiler may
// contract the products differently, so the two forms can differ in the
// last bits.
// The lanes' sums and extremes are scattered (data-parallel moves), lane v
// getting component v's: it forms and stores that component's derivatives,
// and the limiter's two divisions run for four components at once; the second
// walk needs all components in every lane and gets them by quad broadcasts.
// Both passes at 2,621,440 points: 553 us with all-lane sums by shuffles (which
// go through LDS), lane 0 doing the limiter and a runtime stride of the staged
// arrays; 454 us without; 418 us with the least-squares inverse in an array of
// its own instead of a 160-byte record.  The limited pass then issues vector
// instructions for 171 us of its time.
static_assert(kQTile * 4 == kBlock, "a q-derivative tile is one point per four lanes");
constexpr int kLnPre = 8;  // list positions per lane held in registers (a whole stencil of <= 32)

template <int C>
__device__ __forceinline__ double quad_bcast(double v) {  // component C's value, held by lane C
    return dpp<C * 0x55>(v);
}

// fmax and fmin as the one instruction they are.  The functions' operands are
// first brought to a canonical form (an instruction each) wherever the
// compiler cannot see that they are no signalling NaNs, as after a branch or a
// cross-lane move; the instruction treats NaNs as the functions do.
__device__ __forceinline__ double max_f64(double a, double b) {
    double r;
    asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
__device__ __forceinline__ double min_f64(double a, double b) {
    double r;
    asm("v_min_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

// The largest / smallest of four values over a quad, scattered as scatter_sum.
template <bool MAX>
__device__ __forceinline__ double scatter_extreme(const double a[4], int lane) {
    auto pick = [](double x, double y) { return MAX ? max_f64(x, y) : min_f64(x, y); };
    const bool hi = lane & 2, odd = lane & 1;
    const double x0 = pick(hi ? a[2] : a[0], dpp<kDppXor2>(hi ? a[0] : a[2]));
    const double x1 = pick(hi ? a[3] : a[1], dpp<kDppXor2>(hi ? a[1] : a[3]));
    return pick(odd ? x1 : x0, dpp<kDppXor1>(odd ? x0 : x1));
}

// S: stride of the staged arrays, at least the cloud's longest list (tile_stride).
template <bool INNER, bool LIMIT, int S>
__global__ void __launch_bounds__(kBlock, 4) k_qgrad_tiled(
    double K, const D2* __restrict__ xy, const int32_t* __restrict__ off,
    const int32_t* __restrict__ tile_pts, const uint16_t* __restrict__ lnbr,
    const int32_t* __restrict__ tile_off,
    const int32_t* __restrict__ tile_idx, const D4* __restrict__ lsq,
    const int32_t* __restrict__ comp, const int32_t* __restrict__ active,
    const D4* __restrict__ q, const D4* __restrict__ qx_in, const D4* __restrict__ qy_in,
    D4* __restrict__ qx_out, D4* __restrict__ qy_out, D4* __restrict__ qxl,
    D4* __restrict__ qyl) {
    // arrays of component pairs: the lanes of a wave read consecutive list
    // positions, so 16-byte reads fall in distinct banks, and the fixed stride
    // makes the arrays' offsets immediate operands
    __shared__ D2 s_nb[(INNER ? 7 : 3) * S];  // (x, y), q, then q_x, q_y
    const int tile = xcd_block(blockIdx.x, gridDim.x);
    // the point's own data and its first list positions are requested before
    // the staging, so their latency overlaps it
    const int64_t p = tile_pts[(int64_t)tile * kQTile + threadIdx.x / 4];
    const int lane = threadIdx.x % 4;
    const bool inb = p >= 0;
    D2 r0{};
    D4 q0{}, gx0{}, gy0{}, L{};
    int32_t e0 = 0, e1 = 0;
    if (inb) {
        r0 = xy[p];
        q0 = q[p];
        e0 = off[p];
        e1 = off[p + 1];
        L = lsq[p];
        if (INNER) {
            gx0 = qx_in[p];
            gy0 = qy_in[p];
        }
    }
    int lpre[kLnPre];
#pragma unroll
    for (int k = 0; k < kLnPre; ++k) {
        const int32_t e = e0 + lane + 4 * k;
        lpre[k] = e < e1 ? lnbr[e] : 0;
    }
    const int32_t h0 = tile_off[tile], nh = tile_off[tile + 1] - h0;
    for (int32_t k = threadIdx.x; k < nh; k += kBlock) {
        const int32_t i = tile_idx[h0 + k];
        const D4 qi = q[i];
        s_nb[k] = xy[i];
        s_nb[S + k] = {qi.x, qi.y};
        s_nb[2 * S + k] = {qi.z, qi.w};
        if (INNER) {
            const D4 gx = qx_in[i], gy = qy_in[i];
            s_nb[3 * S + k] = {gx.x, gx.y};
            s_nb[4 * S + k] = {gx.z, gx.w};
            s_nb[5 * S + k] = {gy.x, gy.y};
            s_nb[6 * S + k] = {gy.z, gy.w};
        }
    }
    __syncthreads();
    if (!inb || !live(comp, active, p)) return;  // uniform over the lanes of a point
    const double qv[4] = {q0.x, q0.y, q0.z, q0.w};
    double bx[4] = {0, 0, 0, 0}, by[4] = {0, 0, 0, 0};
    double dmax[4] = {0, 0, 0, 0}, dmin[4] = {0, 0, 0, 0};
    // a lane takes entries e0 + lane, e0 + lane + 4, ... in order: the first
    // kLnPre from registers, any further ones from memory
    auto first_walk = [&](int li) {
        const D2 r = s_nb[li], qa = s_nb[S + li], qb = s_nb[2 * S + li];
        const double dx = r.x - r0.x, dy = r.y - r0.y;
        double dq[4] = {qa.x - qv[0], qa.y - qv[1], qb.x - qv[2], qb.y - qv[3]};
        if (LIMIT) {
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                dmax[v] = max_f64(dmax[v], dq[v]);
                dmin[v] = min_f64(dmin[v], dq[v]);
            }
        }
        if (INNER) {
            const D2 xa = s_nb[3 * S + li], xb = s_nb[4 * S + li];
            const D2 ya = s_nb[5 * S + li], yb = s_nb[6 * S + li];
            dq[0] -= 0.5 * (dx * (xa.x - gx0.x) + dy * (ya.x - gy0.x));
            dq[1] -= 0.5 * (dx * (xa.y - gx0.y) + dy * (ya.y - gy0.y));
            dq[2] -= 0.5 * (dx * (xb.x - gx0.z) + dy * (yb.x - gy0.z));
            dq[3] -= 0.5 * (dx * (xb.y - gx0.w) + dy * (yb.y - gy0.w));
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            bx[v] += dx * dq[v];
            by[v] += dy * dq[v];
        }
    };
#pragma unroll
    for (int k = 0; k < kLnPre; ++k)
        if (e0 + lane + 4 * k < e1) first_walk(lpre[k]);
    for (int32_t e = e0 + lane + 4 * kLnPre; e < e1; e += 4) first_walk(lnbr[e]);
    // component `lane` from here on
    const double sx = scatter_sum<4>(bx, bx, lane), sy = scatter_sum<4>(by, by, lane);
    const double gx = L.x * sx + L.y * sy, gy = L.y * sx + L.z * sy;
    auto component = [lane](D4* f, int64_t i) { return reinterpret_cast<double*>(f + i) + lane; };
    if (!LIMIT || qx_out) {  // the limited pass writes them on request only
        *component(qx_out, p) = gx;
        *component(qy_out, p) = gy;
    }
    if (!LIMIT) return;
    const double hi = scatter_extreme<true>(dmax, lane), lo = scatter_extreme<false>(dmin, lane);
    const double kh = K * L.w;
    const double eps2 = kh * kh * kh;
    const double ax[4] = {quad_bcast<0>(gx), quad_bcast<1>(gx), quad_bcast<2>(gx), quad_bcast<3>(gx)};
    const double ay[4] = {quad_bcast<0>(gy), quad_bcast<1>(gy), quad_bcast<2>(gy), quad_bcast<3>(gy)};
    double tlo[4] = {0, 0, 0, 0}, thi[4] = {0, 0, 0, 0};  // extremes of dx qx + dy qy
    auto second_walk = [&](int li) {
        const D2 r = s_nb[li];
        const double dx = r.x - r0.x, dy = r.y - r0.y;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const double t = dx * ax[v] + dy * ay[v];
            tlo[v] = min_f64(tlo[v], t);
            thi[v] = max_f64(thi[v], t);
        }
    };
#pragma unroll
    for (int k = 0; k < kLnPre; ++k)
        if (e0 + lane + 4 * k < e1) second_walk(lpre[k]);
    for (int32_t e = e0 + lane + 4 * kLnPre; e < e1; e += 4) second_walk(lnbr[e]);
    const double phi = venkat_phi(scatter_extreme<false>(tlo, lane),
                                  scatter_extreme<true>(thi, lane), hi, lo, eps2);
    *component(qxl, p) = phi * gx;
    *component(qyl, p) = phi * gy;
}

// Unsplit Euler flux Jacobian product A_d(U) dU along unit direction d
// (eq. 2 differentiated by hand): with u_d' = ((dm . d) - u_d drho)/rho and
// p' = (gamma-1)(dE - u . dm + |u|^2 drho / 2),
//   (dm . d, dm u_d + m u_d' + p' d, (dE + p') u_d + (E + p) u_d');
// FD = true: the flux difference G_d(U + dU) - G_d(U) instead.
template <bool FD>
__device__ __forceinline__ void unsplit_jvp(const D4& u, const double dv[4], double dx, double dy,
                                            double gm1, double J[4]) {
    if (FD) {
        const double a0 = u.x + dv[0], a1 = u.y + dv[1], a2 = u.z + dv[2], a3 = u.w + dv[3];
        const double ua = (a1 * dx + a2 * dy) / a0, ub = (u.y * dx + u.z * dy) / u.x;
        const double pa = gm1 * (a3 - 0.5 * (a1 * a1 + a2 * a2) / a0);
        const double pb = gm1 * (u.w - 0.5 * (u.y * u.y + u.z * u.z) / u.x);
        J[0] = (a1 * dx + a2 * dy) - (u.y * dx + u.z * dy);
        J[1] = (a1 * ua + pa * dx) - (u.y * ub + pb * dx);
        J[2] = (a2 * ua + pa * dy) - (u.z * ub + pb * dy);
        J[3] = (a3 + pa) * ua - (u.w + pb) * ub;
        return;
    }
    const double irho = 1.0 / u.x, u1 = u.y * irho, u2 = u.z * irho;
    const double ud = u1 * dx + u2 * dy;
    const double p = gm1 * (u.w - 0.5 * u.x * (u1 * u1 + u2 * u2));
    const double dmd = dv[1] * dx + dv[2] * dy;
    const double udd = (dmd - ud * dv[0]) * irho;
    const double pd = gm1 * (dv[3] - (u1 * dv[1] + u2 * dv[2]) + 0.5 * (u1 * u1 + u2 * u2) * dv[0]);
    J[0] = dmd;
    J[1] = dv[1] * ud + u.y * udd + pd * dx;
    J[2] = dv[2] * ud + u.z * udd + pd * dy;
    J[3] = (dv[3] + pd) * ud + (u.w + p) * udd;
}

// Neighbour data of one stencil pair of the residual.
struct Nbr {
    D2 r;
    D4 q, gx, gy;
};

__device__ __forceinline__ Nbr load_nbr(int32_t i, const D2* __restrict__ xy,
                                        const D4* __restrict__ q, const D4* __restrict__ qx,
                                        const D4* __restrict__ qy) {
    return {xy[i], q[i], qx[i], qy[i]};
}

// 1/sqrt(x) for x > 0; for x <= 0, infinite or NaN the split fluxes end as NaN
// with this as with a guarded function, so it has no guard (four instructions
// fewer of ten).
__device__ __forceinline__ double rsqrt_pos(double x) {
    const double y = __builtin_amdgcn_rsq(x);
    const double e = fma(-x * y, y, 1.0);
    return fma(y * e, fma(e, 0.375, 0.5), y);
}

// 1/sqrt(x) and, in r2, 1/x: both from the seed y and e = 1 - x y^2, where e is that
// of the rounded y^2, so 1/x = y^2/(1 - e) is within one unit in the last place.
// (The square of the first is off by up to 2, and velocity, density and pressure
// would all take that over.)
__device__ __forceinline__ double rsqrt_recip_pos(double x, double& r2) {
    const double y = __builtin_amdgcn_rsq(x);
    const double y2 = y * y;
    const double e = fma(-x, y2, 1.0);
    r2 = fma(y2, fma(e, e, e), y2);
    return fma(y * e, fma(e, 0.375, 0.5), y);
}

// v for s < 0, -v for s > 0 (the sign of the split that offset s lies in)
__device__ __forceinline__ double flip_by(double v, double s) {
    const uint64_t sign = (uint64_t)1 << 63;
    return __longlong_as_double((int64_t)((uint64_t)__double_as_longlong(v) ^
                                          (~(uint64_t)__double_as_longlong(s) & sign)));
}

// erf and exp of S; the code of the unit range lies in the path's order and the
// outer range's beside it (as the frame and general-gamma paths do elsewhere):
// 2,621,440 points, residual 637 us with them in turn, 617 so, and 1% less for an
// iteration at M 1.2 too.
__device__ __forceinline__ void unit_or_outer(double S, double t, const PolyLead& lead, double& er,
                                              double& g) {  // g scaled by e^(1/2)
    if (__builtin_expect(t < 1.0, 1)) {
        erf_exp_unit(S, t, lead, er, g);
    } else {  // fast flow (or a non-physical state)
        erf_exp_outer(S, t, er, g);
        g *= 1.0 / kExpHalf;
    }
}

// One end of a stencil pair: the weighted sum of its split fluxes along the
// two split directions of the point,
//   sum_d w_d G_d^{sg_d},   d = x, y (interior) or t, n (frame points),
// from a reconstructed q vector.  The primitive state is that of prim_from_q;
// with A_d = (1 + sg_d erf S_d)/2, B_d = exp(-S_d^2)/(2 sqrt(pi beta)) and
//   P = sum_d w_d u_d A_d,   Q = sum_d w_d sg_d B_d,   F = P + Q,
// the mass term is rho F, the momentum term sum_d w_d p A_d d + u rho F and
// the energy term (rhoE + p) P + (rhoE + p/2) Q = p ((1/(gamma-1) + 1/2 +
// beta |u|^2) F + P/2), since rhoE = p (1/(gamma-1) + beta |u|^2).  The two
// directions share everything but A, B: 18 instructions after the functions
// where two separate fluxes took about 60.  hw_d = w_d/2 and hs_d = sg_d w_d/2.
// Written in explicit fused steps with contraction off, so that both ends of a
// pair round alike (a uniform field's residual is exactly zero).
// The energy term from beta |u|^2 (from a q vector), or with RHO_E from rho E (of a
// conserved state): (rho E + p/2) F + p P/2.
template <bool FRAME, bool RHO_E>
__device__ __forceinline__ D4 weighted_flux(double rho, double p, double r, double u1, double u2,
                                            double ua, double ub, double en, double era, double ga,
                                            double erb, double gb, const D2& t, double hwa,
                                            double hsa, double hwb, double hsb, double inv_gm1) {
#pragma clang fp contract(off)
    const double aa = fma(hsa, era, hwa), ab = fma(hsb, erb, hwb);  // w A
    const double P = fma(ua, aa, ub * ab);
    const double F = fma(fma(hsa, ga, hsb * gb), r * (kInvSqrtPi * kExpHalf), P);
    const double M = rho * F;
    const double pa = FRAME ? fma(aa, t.x, -(ab * t.y)) : aa;
    const double pb = FRAME ? fma(aa, t.y, ab * t.x) : ab;
    return {M, fma(p, pa, u1 * M), fma(p, pb, u2 * M),
            RHO_E ? fma(fma(0.5, p, en), F, 0.5 * p * P)
                  : p * fma((inv_gm1 + 0.5) + en, F, 0.5 * P)};
}

template <bool FRAME, bool G14>
__device__ __forceinline__ D4 end_sum(const D4& q, const D2& t, double hwa, double hsa,
                                      double hwb, double hsb, double inv_gm1,
                                      const PolyLead& lead) {
#pragma clang fp contract(off)
    const double beta = -0.5 * q.w;
    double r2;
    const double r = rsqrt_recip_pos(beta, r2), i2b = 0.5 * r2;
    const double u1 = q.y * i2b, u2 = q.z * i2b;
    const double sb = beta * r;  // sqrt(beta)
    const double ua = FRAME ? fma(u1, t.x, u2 * t.y) : u1;
    const double ub = FRAME ? fma(u2, t.x, -(u1 * t.y)) : u2;
    const double Sa = ua * sb, Sb = ub * sb;
    const double ta = Sa * Sa, tb = Sb * Sb;
    const double bu = FRAME ? beta * fma(u1, u1, u2 * u2) : ta + tb;
    double era, ga, erb, gb;
    unit_or_outer(Sa, ta, lead, era, ga);
    unit_or_outer(Sb, tb, lead, erb, gb);
    const double lr = q.x + bu;  // log rho + log(beta)/(gamma - 1)
    const double rho = G14 ? exp_lead(lr, lead) * (r2 * r2 * r)
                           : exp_lead(fma(-inv_gm1, log(beta), lr), lead);
    return weighted_flux<FRAME, false>(rho, rho * i2b, r, u1, u2, ua, ub, bu, era, ga, erb, gb, t, hwa, hsa,
                                hwb, hsb, inv_gm1);
}

// q~ = q - (dx q_x + dy q_y)/2 from hx = -dx/2, hy = -dy/2 (eq. 15).  G14 rounds
// twice at q's magnitude, one instruction less per component: with the corrected
// 1/beta of end_sum the residual is still nearer to its exact value than with one
// rounding here and r^2 there.
template <bool G14>
__device__ __forceinline__ D4 reconstruct(const D4& q, const D4& gx, const D4& gy, double hx,
                                          double hy) {
    if (!G14)
        return {q.x + fma(hy, gy.x, hx * gx.x), q.y + fma(hy, gy.y, hx * gx.y),
                q.z + fma(hy, gy.z, hx * gx.z), q.w + fma(hy, gy.w, hx * gx.w)};
    return {fma(hy, gy.x, fma(hx, gx.x, q.x)), fma(hy, gy.y, fma(hx, gx.y, q.y)),
            fma(hy, gy.z, fma(hx, gx.z, q.z)), fma(hy, gy.w, fma(hx, gx.w, q.w))};
}

// Everything a residual launch reads and writes.
struct ResidualArgs {
    int64_t n;
    double gamma;
    const double* cfl;
    const D2* xy;
    const D2* frame;
    const int8_t* type;
    const int32_t* off;
    const int32_t* idx;
    const D4* lsq;
    const PointGeom* geom;
    const int32_t* comp;
    const int32_t* active;
    const int32_t* tile_pts;  // the LDS tiles of lskum_tiles.h (tiled kernel only)
    const uint16_t* lnbr;
    const int32_t* tile_off;
    const int32_t* tile_idx;
    const D4* U;
    const D4* q;
    const D4* qx;
    const D4* qy;
    D4* R;
    double* Dg;
    D4* jv0;
    F4* jv0f;
    F4* jv2f;
    float* Df;
    double* rr_out;
    int32_t* flags;
    int variant, fd;
    D4* dUio;
    F4* dUfio;
    D4* Rs;
    const int32_t* colour;
    int sweep0, farfield;
    const double* vinf;
};

// A residual sum and whether one of its q~ had beta <= 0.
struct ResidualSum {
    double x, y, z, w;
    bool bad;
};

// One (point, neighbour) pair of the residual sum (eq. 11), added to R: from the q~
// at both ends their primitive states and the split flux differences of every split
// the neighbour at offset (dx, dy) lies in (x+-/y+- at interior points, t+-/n- at a
// wall), weighted by the point's split coefficients coef[k * stride].  A split that
// the neighbour is not in has weight zero.
template <bool FRAME, bool G14>
__device__ __forceinline__ void pair_add(double dx, double dy, const D4& qti, const D4& qt0,
                                         const D2& t, int8_t ty, const D2* coef, int stride,
                                         double inv_gm1, const PolyLead& lead, ResidualSum& R) {
#pragma clang fp contract(off)
    double da = dx, db = dy;
    if (FRAME) {
        da = dot_nc(dx, dy, t.x, t.y);
        db = dot_nc(dx, dy, -t.y, t.x);
    }
    const bool in_a = da != 0.0, in_b = FRAME ? in_normal_split(ty, db) : db != 0.0;
    if (!in_a && !in_b) return;
    const D2 ca = coef[da < 0.0 ? 0 : stride];
    const D2 cb = coef[FRAME || db < 0.0 ? 2 * stride : 3 * stride];
    const double wa = 0.5 * fma(ca.x, da, ca.y * db), wb = 0.5 * fma(cb.x, db, cb.y * da);
    const double hwa = in_a ? wa : 0.0, hwb = in_b ? wb : 0.0;
    const double hsa = flip_by(hwa, da), hsb = flip_by(hwb, db);
    R.bad |= !(qti.w < 0.0) || !(qt0.w < 0.0);
    const D4 ci = end_sum<FRAME, G14>(qti, t, hwa, hsa, hwb, hsb, inv_gm1, lead);
    const D4 c0 = end_sum<FRAME, G14>(qt0, t, hwa, hsa, hwb, hsb, inv_gm1, lead);
    R.x += ci.x - c0.x;
    R.y += ci.y - c0.y;
    R.z += ci.z - c0.z;
    R.w += ci.w - c0.w;
}

// The walk of a lane over its entries of a point's list, compiled apart for
// interior and frame points (a wavefront of interior points then holds no
// registers for frames) and for gamma = 1.4: W<FRAME, G14>.
template <class Walk>
__device__ __forceinline__ ResidualSum residual_walks(int8_t ty, bool g14, Walk walk) {
    if (__builtin_expect(g14, 1)) {
        if (__builtin_expect(ty == kInterior, 1)) return walk(std::false_type{}, std::true_type{});
        return walk(std::true_type{}, std::true_type{});
    }
    if (ty == kInterior) return walk(std::false_type{}, std::false_type{});
    return walk(std::true_type{}, std::false_type{});
}

// Sum over the lanes of a point, by every lane; SUB neighbouring threads hold
// the same sums of a lane.
template <int LANES, int SUB = 1>
__device__ __forceinline__ void residual_lane_sum(ResidualSum& R) {
#pragma unroll
    for (int o = LANES / 2; o > 0; o >>= 1) {
        R.x += __shfl_xor(R.x, o * SUB, 64);
        R.y += __shfl_xor(R.y, o * SUB, 64);
        R.z += __shfl_xor(R.z, o * SUB, 64);
        R.w += __shfl_xor(R.w, o * SUB, 64);
    }
#pragma unroll
    for (int o = LANES * SUB / 2; o > 0; o >>= 1) R.bad |= __shfl_xor((int)R.bad, o, 64) != 0;
}

// The contributions of SUB neighbouring threads added to R in thread order, by
// each of them.
template <int SUB>
__device__ __forceinline__ void add_in_turn(ResidualSum& R, const ResidualSum& c) {
    static_assert(SUB == 2 || SUB == 4);
    auto turn = [&](auto ctrl) {
        constexpr int C = decltype(ctrl)::value;
        R.x += dpp<C>(c.x);
        R.y += dpp<C>(c.y);
        R.z += dpp<C>(c.z);
        R.w += dpp<C>(c.w);
    };
    if constexpr (SUB == 2) {
        turn(std::integral_constant<int, 0xA0>{});  // quad_perm 0 0 2 2
        turn(std::integral_constant<int, 0xF5>{});  // 1 1 3 3
    } else {
        turn(std::integral_constant<int, 0x00>{});
        turn(std::integral_constant<int, 0x55>{});
        turn(std::integral_constant<int, 0xAA>{});
        turn(std::integral_constant<int, 0xFF>{});
    }
    R.bad |= c.bad;
}

// ---------------------------------------------------------------------------
// Residual (eq. 11 with the q~ reconstruction of eq. 15), local time step,
// scalar diagonal (eq. 25, 34-35) and the sweep linearisation data.
// ---------------------------------------------------------------------------
// The kernel's arguments, and loads and stores through pointers among them,
// for code after a long loop: the arguments are read from the kernel-argument
// segment again (a second look that the compiler does not merge with the
// first), where holding them through the loop would spill scalar registers
// into vector lanes and cost a vector instruction for each one's way back.
typedef const __attribute__((address_space(4))) ResidualArgs KernArgs;

__device__ __forceinline__ KernArgs& reread_args() {
    auto* k = (KernArgs*)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(k));
    return *k;
}

template <class T>
struct Raw { using type = T; };
template <>
struct Raw<D4> { typedef double type __attribute__((ext_vector_type(4))); };
template <>
struct Raw<D2> { typedef double type __attribute__((ext_vector_type(2))); };
template <>
struct Raw<F4> { typedef float type __attribute__((ext_vector_type(4))); };

template <class T>
__device__ __forceinline__ T gload(const T* p, int64_t i) {
    using V = typename Raw<T>::type;
    const V v = *(const __attribute__((address_space(1))) V*)(p + i);
    return __builtin_bit_cast(T, v);
}
template <class T>
__device__ __forceinline__ void gstore(T* p, int64_t i, const T& v) {
    using V = typename Raw<T>::type;
    *(__attribute__((address_space(1))) V*)(p + i) = __builtin_bit_cast(V, v);
}

// What follows a point's sum over its neighbours: wall tangency, the far
// field's ghost, R and its square, linearisation data, time step, diagonal and
// the forward sweep's first colour phase.
template <bool MIXED>
__device__ __forceinline__ void residual_finish(int64_t p, int8_t ty, const ResidualSum& sum,
                                                double inv_gm1, bool g14) {
    KernArgs& A = reread_args();
    double Rp[4] = {sum.x, sum.y, sum.z, sum.w};
    const bool bad = sum.bad;
    const D2 t = gload(A.frame, p);
    const bool part = ty != kOuter || A.farfield;  // outer points: kinetic far field only
    if (ty == kWall) {  // drop the normal-momentum component
        const double nx = -t.y, ny = t.x;
        const double mn = Rp[1] * nx + Rp[2] * ny;
        Rp[1] -= mn * nx;
        Rp[2] -= mn * ny;
    }
    if (ty == kOuter && A.farfield) {
        // kinetic far field: the n- half (molecules entering the domain)
        // from a free-stream ghost one nearest-neighbour distance outside,
        // (G_n-(U_inf) - G_n-(U_0)) / h with the point's own q
        const int k = A.comp ? gload(A.comp, p) : 0;
        const double v1 = gload(A.vinf, 2 * k), v2 = gload(A.vinf, 2 * k + 1);
        Prim wf;
        wf.rho = 1.0;
        wf.u1 = v1;
        wf.u2 = v2;
        wf.p = 1.0 / A.gamma;
        wf.sb = sqrt(0.5 * A.gamma);
        wf.isb = 1.0 / wf.sb;
        wf.rhoE = wf.p * inv_gm1 + 0.5 * (v1 * v1 + v2 * v2);
        const Prim w0 = prim_from_q(gload(A.q, p), inv_gm1, g14);
        double Gf[4], G0[4];
        split_flux(wf, -t.y, t.x, -1.0, Gf);
        split_flux(w0, -t.y, t.x, -1.0, G0);
        const double ih = 1.0 / gload(A.lsq, p).w;
#pragma unroll
        for (int v = 0; v < 4; ++v) Rp[v] += (Gf[v] - G0[v]) * ih;
    }
    gstore(A.rr_out, p, ty != kOuter ? Rp[0] * Rp[0] : 0.0);
    gstore(A.R, p, D4{Rp[0], Rp[1], Rp[2], Rp[3]});

    // linearisation data at the current state, local time step, diagonal
    const D4 u = gload(A.U, p);
    const double rho = u.x, irho = 1.0 / rho;
    const double u1 = u.y * irho, u2 = u.z * irho;
    const double usq = u1 * u1 + u2 * u2;
    const double pr = (A.gamma - 1.0) * (u.w - 0.5 * rho * usq);
    const double beta = 0.5 * rho / pr;
    const D4 j0 = {rho, u1, u2, pr};
    const double a = sqrt(A.gamma * pr / rho);
    const double hn = gload(A.lsq, p).w;  // nearest-neighbour distance
    const D4 ls1 = gload(&A.geom[p].ls1, 0);
    const double dt = gload(A.cfl, A.comp ? gload(A.comp, p) : 0) * hn / (sqrt(usq) + a);
    double Dp = 1.0 / dt;
    if (A.variant == 0) {
        // Anandhanarayanan et al.: split Jacobians -> +-rho(A+-) I (eq. 34-35)
        if (ty == kWall) {
            const double ut = u1 * t.x + u2 * t.y, un = -u1 * t.y + u2 * t.x;
            Dp -= ls1.x * fmax(ut + a, 0.0);
            Dp += ls1.y * fmax(a - ut, 0.0);
            Dp += ls1.z * fmax(a - un, 0.0);
        } else if (ty != kOuter) {
            Dp -= ls1.x * fmax(u1 + a, 0.0);
            Dp += ls1.y * fmax(a - u1, 0.0);
            Dp -= ls1.z * fmax(u2 + a, 0.0);
            Dp += ls1.w * fmax(a - u2, 0.0);
        } else if (A.farfield) {
            // t+, t-, n+ of the stencil and the ghost's n- half, whose
            // single weight is 1/h (its increment is zero)
            const double ut = u1 * t.x + u2 * t.y, un = -u1 * t.y + u2 * t.x;
            Dp -= ls1.x * fmax(ut + a, 0.0);
            Dp += ls1.y * fmax(a - ut, 0.0);
            Dp -= ls1.z * fmax(un + a, 0.0);
            Dp += fmax(a - un, 0.0) / hn;
        }
    } else {
        // Manish et al.: A+- = (A +- rho(A) I)/2, rho(A) = |u_d| + a (eq. 29-33); the
        // A part, S_0 = -1/2 sum_k LS_k(1) A_k dU_0, is taken with the previous
        // iteration's increment onto the forward right-hand side A.R - S (eq. 36-38)
        double dv[4] = {0, 0, 0, 0};
        if (MIXED) {
            const F4 d = gload(A.dUfio, p);
            dv[0] = d.x; dv[1] = d.y; dv[2] = d.z; dv[3] = d.w;
        } else {
            const D4 d = gload(A.dUio, p);
            dv[0] = d.x; dv[1] = d.y; dv[2] = d.z; dv[3] = d.w;
        }
        double Sv[4] = {0, 0, 0, 0}, Ja[4], Jb[4];
        double ca = 0.0, cb = 0.0;
        if (ty == kWall) {
            const double ut = u1 * t.x + u2 * t.y, un = -u1 * t.y + u2 * t.x;
            Dp -= 0.5 * (fabs(ut) + a) * (ls1.x - ls1.y);
            Dp += 0.5 * (fabs(un) + a) * ls1.z;
            if (A.fd) {
                unsplit_jvp<true>(u, dv, t.x, t.y, A.gamma - 1.0, Ja);
                unsplit_jvp<true>(u, dv, -t.y, t.x, A.gamma - 1.0, Jb);
            } else {
                unsplit_jvp<false>(u, dv, t.x, t.y, A.gamma - 1.0, Ja);
                unsplit_jvp<false>(u, dv, -t.y, t.x, A.gamma - 1.0, Jb);
            }
            ca = ls1.x + ls1.y;
            cb = ls1.z;
        } else if (ty == kOuter && A.farfield) {
            const double ut = u1 * t.x + u2 * t.y, un = -u1 * t.y + u2 * t.x;
            Dp -= 0.5 * (fabs(ut) + a) * (ls1.x - ls1.y);
            Dp -= 0.5 * (fabs(un) + a) * ls1.z;
            if (A.fd) {
                unsplit_jvp<true>(u, dv, t.x, t.y, A.gamma - 1.0, Ja);
                unsplit_jvp<true>(u, dv, -t.y, t.x, A.gamma - 1.0, Jb);
            } else {
                unsplit_jvp<false>(u, dv, t.x, t.y, A.gamma - 1.0, Ja);
                unsplit_jvp<false>(u, dv, -t.y, t.x, A.gamma - 1.0, Jb);
            }
            ca = ls1.x + ls1.y;
            cb = ls1.z;
        } else if (ty != kOuter) {
            Dp -= 0.5 * (fabs(u1) + a) * (ls1.x - ls1.y);
            Dp -= 0.5 * (fabs(u2) + a) * (ls1.z - ls1.w);
            if (A.fd) {
                unsplit_jvp<true>(u, dv, 1.0, 0.0, A.gamma - 1.0, Ja);
                unsplit_jvp<true>(u, dv, 0.0, 1.0, A.gamma - 1.0, Jb);
            } else {
                unsplit_jvp<false>(u, dv, 1.0, 0.0, A.gamma - 1.0, Ja);
                unsplit_jvp<false>(u, dv, 0.0, 1.0, A.gamma - 1.0, Jb);
            }
            ca = ls1.x + ls1.y;
            cb = ls1.z + ls1.w;
        }
        if (part)
#pragma unroll
            for (int v = 0; v < 4; ++v) Sv[v] = -0.5 * (ca * Ja[v] + cb * Jb[v]);
        gstore(A.Rs, p, D4{Rp[0] - Sv[0], Rp[1] - Sv[1], Rp[2] - Sv[2], Rp[3] - Sv[3]});
        if (A.sweep0)
#pragma unroll
            for (int v = 0; v < 4; ++v) Sv[v] = Rp[v] - Sv[v];
    }
    if (MIXED) {
        // erf and exp of the fp32 sweeps, formed in double precision
        const double sb = sqrt(beta), sx = u1 * sb, sy = u2 * sb;
        D4 j2;
        erf_exp(sx, j2.x, j2.y);
        erf_exp(sy, j2.z, j2.w);
        gstore(A.jv0f, p, F4{(float)j0.x, (float)j0.y, (float)j0.z, (float)j0.w});
        gstore(A.jv2f, p, F4{(float)j2.x, (float)j2.y, (float)j2.z, (float)j2.w});
        gstore(A.Df, p, (float)Dp);
    } else {
        gstore(A.jv0, p, j0);
        gstore(A.Dg, p, Dp);
    }
    // the forward sweep's first colour phase: its points have no lower
    // neighbours, dU* = -R / D (R - S for the Manish variant), in the
    // sweep precision, by the reciprocal of D
    if (A.sweep0 && gload(A.colour, p) == 0) {
        double rs[4] = {Rp[0], Rp[1], Rp[2], Rp[3]};
        if (A.variant != 0) {
            const D4 r2 = gload(A.Rs, p);
            rs[0] = r2.x; rs[1] = r2.y; rs[2] = r2.z; rs[3] = r2.w;
        }
        if (MIXED) {
            float o[4] = {0.f, 0.f, 0.f, 0.f};
            if (part) {
                const float iD = 1.0f / (float)Dp;
#pragma unroll
                for (int v = 0; v < 4; ++v) o[v] = -((float)rs[v] + 0.0f) * iD;
                if (ty == kWall) {
                    const float nx = (float)(-t.y), ny = (float)t.x;
                    const float mn = o[1] * nx + o[2] * ny;
                    o[1] -= mn * nx;
                    o[2] -= mn * ny;
                }
            }
            gstore(A.dUfio, p, F4{o[0], o[1], o[2], o[3]});
        } else {
            double o[4] = {0, 0, 0, 0};
            if (part) {
                const double iD = 1.0 / Dp;
#pragma unroll
                for (int v = 0; v < 4; ++v) o[v] = -(rs[v] + 0.0) * iD;
                if (ty == kWall) {
                    const double nx = -t.y, ny = t.x;
                    const double mn = o[1] * nx + o[2] * ny;
                    o[1] -= mn * nx;
                    o[2] -= mn * ny;
                }
            }
            gstore(A.dUio, p, D4{o[0], o[1], o[2], o[3]});
        }
    }
    if (bad || !(rho > 0.0) || !(pr > 0.0)) gstore(A.flags, 0, 1);
}

// Direct gathers, where residual_form does not take tiles.  LANES consecutive lanes
// share one point: each takes every LANES-th neighbour, the four residual sums are
// combined with cross-lane shuffles and the first lane finishes the point.
// Software pipeline (interior points, gamma 1.4): neighbour indices two
// entries ahead; the next neighbour's data is requested as soon as this one's
// has gone into q~, and arrives during the flux evaluation; past the end the
// last entry is re-read (in bounds), unused.
template <bool MIXED, int LANES>
__global__ void __launch_bounds__(kBlock) k_residual(ResidualArgs A) {
    const int64_t gt = (int64_t)xcd_block(blockIdx.x, gridDim.x) * blockDim.x + threadIdx.x;
    const int64_t p = gt / LANES;
    const int lane = (int)(gt % LANES);
    const double inv_gm1 = 1.0 / (A.gamma - 1.0);
    const bool g14 = A.gamma == 1.4;
    const PolyLead lead = poly_lead();
    __shared__ D2 s_coef[4 * kBlock];  // each lane writes and reads its own copy
    if (p >= A.n || !live(A.comp, A.active, p)) return;
    const int8_t ty = A.type[p];
    ResidualSum sum{};
    if (ty != kOuter || A.farfield) {
        const D2 r0 = A.xy[p];
        const D4 q0 = A.q[p], gx0 = A.qx[p], gy0 = A.qy[p];
        D2* coef = s_coef + threadIdx.x;
        const PointGeom& G = A.geom[p];
#pragma unroll
        for (int k = 0; k < 4; ++k) coef[k * kBlock] = G.split[k];
        const int32_t e1 = A.off[p + 1], last = e1 - 1;
        const int32_t eb = A.off[p] + lane;
        sum = residual_walks(ty, g14, [&](auto frame, auto is14) __attribute__((always_inline)) {
            ResidualSum R{};
            constexpr bool FRAME = decltype(frame)::value, G14 = decltype(is14)::value;
            constexpr bool PIPE = !FRAME && G14;
            const D2 t = FRAME ? A.frame[p] : D2{1.0, 0.0};
            int32_t e = eb;
            if (e >= e1) return R;
            int32_t i_next = A.idx[min(e + LANES, last)];
            Nbr nb = load_nbr(A.idx[e], A.xy, A.q, A.qx, A.qy);
            for (; e < e1; e += LANES) {
                const double dx = nb.r.x - r0.x, dy = nb.r.y - r0.y;
                const double hx = -0.5 * dx, hy = -0.5 * dy;
                const D4 qti = reconstruct<G14>(nb.q, nb.gx, nb.gy, hx, hy);
                const D4 qt0 = reconstruct<G14>(q0, gx0, gy0, hx, hy);
                if (PIPE) {
                    nb = load_nbr(i_next, A.xy, A.q, A.qx, A.qy);
                    i_next = A.idx[min(e + 2 * LANES, last)];
                    __builtin_amdgcn_sched_barrier(0);
                }
                pair_add<FRAME, G14>(dx, dy, qti, qt0, t, ty, coef, kBlock, inv_gm1, lead, R);
                if (!PIPE) {
                    nb = load_nbr(i_next, A.xy, A.q, A.qx, A.qy);
                    i_next = A.idx[min(e + 2 * LANES, last)];
                }
            }
            return R;
        });
    }
    residual_lane_sum<LANES>(sum);
    if (lane == 0) residual_finish<MIXED>(p, ty, sum, inv_gm1, g14);
}

// The same with the neighbours staged in LDS, on the tiles of the
// q-derivative passes: a block of kQTile points, LANES lanes each, copies
// position, q and derivatives of the tile's listed points once (112 bytes
// each, about 2.5 listed points per point) and every pair reads its neighbour
// there.  S is the stride of the staged arrays, at least the longest list of
// the cloud.  SUB neighbouring threads form one lane: they evaluate the next SUB
// pairs of its walk together and add them in the walk's order.  The lanes' sums
// meet in LDS, and the first wavefront finishes the tile's points, one per lane.
// The arithmetic and the order of the sums are those of k_residual.
// Bound by vector instruction issue: about 280 per pair in the loop and 310 with
// staging and the points' ends, after sharing the two directions' work (end_sum), 430
// before.  2,621,440 points, two lanes per point: 854 us with separate fluxes per
// direction, 615 us now (FP64); a bound of four wavefronts per SIMD spills 56 bytes
// and takes 1,055 us.
template <bool MIXED, int LANES, int S, int SUB>
__global__ void __launch_bounds__(kQTile * LANES * SUB) k_residual_tiled(ResidualArgs A) {
    __shared__ D2 s_nb[7 * S];  // (x, y), q, q_x, q_y in pairs of components
    __shared__ D2 s_coef[4 * kQTile];
    const int tile = xcd_block(blockIdx.x, gridDim.x);
    constexpr int kThreads = kQTile * LANES * SUB, kStep = LANES * SUB;
    const int pt = threadIdx.x / kStep, sub = threadIdx.x % SUB, lane = threadIdx.x / SUB % LANES;
    const int64_t p = A.tile_pts[(int64_t)tile * kQTile + pt];
    const double inv_gm1 = 1.0 / (A.gamma - 1.0);
    const bool g14 = A.gamma == 1.4;
    const PolyLead lead = poly_lead();
    // the point's own data is requested before the staging
    const bool on = p >= 0 && live(A.comp, A.active, p);
    int8_t ty = kOuter;
    D2 r0{};
    D4 q0{}, gx0{}, gy0{};
    int32_t eb = 0, e1 = 0;
    if (on) {
        ty = A.type[p];
        r0 = A.xy[p];
        q0 = A.q[p];
        gx0 = A.qx[p];
        gy0 = A.qy[p];
        eb = A.off[p] + lane;
        e1 = A.off[p + 1];
        for (int k = threadIdx.x % kStep; k < 4; k += kStep)
            s_coef[k * kQTile + pt] = A.geom[p].split[k];
    }
    // a pointer of its own, so that the loop holds it and not its neighbours among the arguments
    auto* lnbr = (const __attribute__((address_space(1))) uint16_t*)A.lnbr;
    asm volatile("" : "+s"(lnbr));
    int li = eb < e1 ? lnbr[min(eb + LANES * sub, e1 - 1)] : 0;
    const int32_t h0 = A.tile_off[tile], nh = A.tile_off[tile + 1] - h0;
    for (int32_t k = threadIdx.x; k < nh; k += kThreads) {
        const int32_t i = A.tile_idx[h0 + k];
        const D4 a = A.q[i], b = A.qx[i], c = A.qy[i];
        s_nb[k] = A.xy[i];
        s_nb[S + k] = {a.x, a.y};
        s_nb[2 * S + k] = {a.z, a.w};
        s_nb[3 * S + k] = {b.x, b.y};
        s_nb[4 * S + k] = {b.z, b.w};
        s_nb[5 * S + k] = {c.x, c.y};
        s_nb[6 * S + k] = {c.z, c.w};
    }
    __syncthreads();
    ResidualSum sum{};
    if (on && (ty != kOuter || A.farfield)) {
        const D2* coef = s_coef + pt;
        sum = residual_walks(ty, g14, [&](auto frame, auto is14) __attribute__((always_inline)) {
            ResidualSum R{};
            constexpr bool FRAME = decltype(frame)::value, G14 = decltype(is14)::value;
            const D2 t = FRAME ? A.frame[p] : D2{1.0, 0.0};
            for (int32_t e = eb; e < e1; e += kStep) {
                const D2 r = s_nb[li], qa = s_nb[S + li], qb = s_nb[2 * S + li];
                const D2 xa = s_nb[3 * S + li], xb = s_nb[4 * S + li];
                const D2 ya = s_nb[5 * S + li], yb = s_nb[6 * S + li];
                li = lnbr[min(e + kStep + LANES * sub, e1 - 1)];  // the next entry's position
                const double dx = r.x - r0.x, dy = r.y - r0.y;
                const double hx = -0.5 * dx, hy = -0.5 * dy;
                const D4 qti = reconstruct<G14>({qa.x, qa.y, qb.x, qb.y}, {xa.x, xa.y, xb.x, xb.y},
                                           {ya.x, ya.y, yb.x, yb.y}, hx, hy);
                const D4 qt0 = reconstruct<G14>(q0, gx0, gy0, hx, hy);
                if constexpr (SUB == 1) {
                    pair_add<FRAME, G14>(dx, dy, qti, qt0, t, ty, coef, kQTile, inv_gm1, lead, R);
                } else {
                    ResidualSum one{};
                    if (e + LANES * sub < e1)
                        pair_add<FRAME, G14>(dx, dy, qti, qt0, t, ty, coef, kQTile, inv_gm1, lead,
                                             one);
                    add_in_turn<SUB>(R, one);
                }
            }
            return R;
        });
    }
    residual_lane_sum<LANES, SUB>(sum);
    if (LANES > 1) {
        // hand the sums to the first wavefront through the staging area
        __syncthreads();
        double* s_R = reinterpret_cast<double*>(s_nb);
        int32_t* s_bad = reinterpret_cast<int32_t*>(s_nb + 2 * kQTile);
        int32_t* s_p = s_bad + kQTile;
        if (threadIdx.x % kStep == 0) {
            s_R[pt] = sum.x;
            s_R[kQTile + pt] = sum.y;
            s_R[2 * kQTile + pt] = sum.z;
            s_R[3 * kQTile + pt] = sum.w;
            s_bad[pt] = sum.bad ? 1 : 0;
            s_p[pt] = on ? (int32_t)p : -1;
        }
        __syncthreads();
        const int t = threadIdx.x;
        if (t >= kQTile || s_p[t] < 0) return;
        sum = {s_R[t], s_R[kQTile + t], s_R[2 * kQTile + t], s_R[3 * kQTile + t], s_bad[t] != 0};
        residual_finish<MIXED>(s_p[t], gload(reread_args().type, s_p[t]), sum, inv_gm1, g14);
    } else if (on) {
        residual_finish<MIXED>(p, ty, sum, inv_gm1, g14);
    }
}

// Residual norm of each component in two deterministic stages: one block
// per reduction chunk sums R_rho^2 over the chunk's points, then one thread
// wavefront per component adds its chunks: res = sqrt(sum) / (non-outer count).
// A component whose norm is not finite is retired as failed; one that reaches
// tol_abs (> 0) is retired as converged.
__global__ void __launch_bounds__(kBlock) k_norm_partial(const double* __restrict__ rr,
                                                         const int32_t* __restrict__ chunk_start,
                                                         const int32_t* __restrict__ chunk_comp,
                                                         const int32_t* __restrict__ active,
                                                         double* __restrict__ partial) {
    __shared__ double red[kBlock / 64];
    const int c = blockIdx.x;
    if (!active[chunk_comp[c]]) return;  // uniform over the block
    double s = 0.0;
    // unrolled so that the loads are issued together; the additions keep their order
#pragma unroll 4
    for (int64_t p = chunk_start[c] + threadIdx.x; p < chunk_start[c + 1]; p += blockDim.x)
        s += rr[p];
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
        for (int w = 0; w < kBlock / 64; ++w) t += red[w];
        partial[c] = t;
    }
}

__global__ void __launch_bounds__(64) k_norm_comp(const double* __restrict__ partial,
                                                  const int32_t* __restrict__ comp_chunk_off,
                                                  const double* __restrict__ inv_active,
                                                  const double* __restrict__ tol_abs,
                                                  int32_t* __restrict__ active,
                                                  int32_t* __restrict__ status,
                                                  int32_t* __restrict__ iters,
                                                  double* __restrict__ res_last,
                                                  double* __restrict__ out) {
    const int k = blockIdx.x;  // one wavefront per component
    if (!active[k]) return;
    double t = 0.0;
    // unrolled so that the loads are issued together; the additions keep their order
#pragma unroll 8
    for (int c = comp_chunk_off[k] + threadIdx.x; c < comp_chunk_off[k + 1]; c += 64) t += partial[c];
    for (int o = 32; o > 0; o >>= 1) t += __shfl_xor(t, o, 64);
    if (threadIdx.x != 0) return;
    const double res = sqrt(t) * inv_active[k];
    out[k] = res;
    res_last[k] = res;
    iters[k] += 1;
    if (!(res <= 1e300)) {
        status[k] = -1;
        active[k] = 0;
    } else if (tol_abs[k] > 0.0 && res <= tol_abs[k]) {
        status[k] = 1;
        active[k] = 0;
    }
}

__global__ void k_reset_components(int ncomp, int32_t* __restrict__ active,
                                   int32_t* __restrict__ status, int32_t* __restrict__ iters) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= ncomp) return;
    active[k] = 1;
    status[k] = 0;
    iters[k] = 0;
}

// ---------------------------------------------------------------------------
// Split-flux Jacobian-vector products for the sweeps.
// ---------------------------------------------------------------------------
// Half the split weight and its signed copy, (w/2, sg w/2), from a list
// entry's weight and its negative-offset bit (sg = +1 when set).
__device__ __forceinline__ double signed_half(double hw, uint8_t cd, int neg_bit) {
    const uint64_t flip = (uint64_t)((~(uint32_t)cd >> neg_bit) & 1u) << 63;
    return __longlong_as_double((int64_t)((uint64_t)__double_as_longlong(hw) ^ flip));
}
__device__ __forceinline__ float signed_half(float hw, uint8_t cd, int neg_bit) {
    return __uint_as_float(__float_as_uint(hw) ^ (((~(uint32_t)cd >> neg_bit) & 1u) << 31));
}

// The reciprocal of rho p (one for 1/rho and 1/p) and 1/sqrt(beta) of a
// physical state: hardware seeds refined to double precision without the
// guards of a division; the fp32 sweeps use the seeds (about 1 ulp).
__device__ __forceinline__ double recip_pos(double x) {
    double y = __builtin_amdgcn_rcp(x);
    y = fma(fma(-x, y, 1.0), y, y);
    return fma(fma(-x, y, 1.0), y, y);
}
__device__ __forceinline__ float recip_pos(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ __forceinline__ float rsqrt_pos(float x) { return __builtin_amdgcn_rsqf(x); }

// Adds sum_d w_d A_d(U_i) dU_i over the two split directions of the point to
// acc (d = x, y, or t, n of a frame point): the exact tangent of the weighted
// split fluxes of weighted_flux (the paper's exact Jacobian-vector product).
// With rho', u', p' from dU, beta' = (rho' - 2 beta p')/(2p) and
// h = beta'/(2 beta), differentiating F_d = u_d A_d + sg_d B_d leaves
//   F_d' = u_d' A_d - h sg_d B_d
// (the terms in S_d' cancel), and A_d' = sg_d exp(-S_d^2) S_d'/sqrt(pi),
// S_d' = sqrt(beta) (u_d' + h u_d).  With P = sum w u_d A_d, P' = sum w u_d' A_d,
// Q = sum w sg_d B_d, X_d = w A_d':
//   mass      rho' F + rho F',  F = P + Q, F' = P' - h Q
//   momentum  sum_d (p' w A_d + p X_d) d + u_i' rho F + u_i mass
//   energy    E' F + p' (P + Q/2) + (rhoE + p/2) F' + (p/2) (P' + sum_d u_d X_d)
// About 130 instructions in double precision, erf and exp included; two
// separate directions took about 160 with erf and exp gathered.
// ga, gb are exp(-S^2), scaled by e^(1/2) in double precision (erf_exp_unit).
template <bool FRAME, class T>
__device__ __forceinline__ void weighted_jvp(const Vec4<T>& a, const Vec4<T>& d, T irho, T beta,
                                             T isb, T sb, T ua, T ub, T era, T ga, T erb, T gb,
                                             T tx, T ty, T hwa, T hsa, T hwb, T hsb, T gm1,
                                             T inv_gm1, T acc[4]) {
    constexpr T kC = T(std::is_same_v<T, double> ? kInvSqrtPi * kExpHalf : kInvSqrtPi);
    const T u1d = (d.y - a.y * d.x) * irho, u2d = (d.z - a.z * d.x) * irho;
    const T hu2 = T(0.5) * (a.y * a.y + a.z * a.z);
    const T pd = gm1 * (d.w - d.x * hu2 - a.x * (a.y * u1d + a.z * u2d));
    const T h = (d.x - (T(2) * beta) * pd) * (T(0.5) * irho);
    const T uad = FRAME ? u1d * tx + u2d * ty : u1d, ubd = FRAME ? u2d * tx - u1d * ty : u2d;
    const T aa = hsa * era + hwa, ab = hsb * erb + hwb;  // w A
    const T Ga = hsa * ga, Gb = hsb * gb;
    const T P = ua * aa + ub * ab, Pd = uad * aa + ubd * ab;
    const T Q = (Ga + Gb) * (isb * kC);
    const T c = T(2) * kC * sb;
    const T Xa = Ga * c * (uad + h * ua), Xb = Gb * c * (ubd + h * ub);
    const T F = P + Q, Fd = Pd - h * Q;
    const T m = d.x * F + a.x * Fd, rF = a.x * F;
    const T va = pd * aa + a.w * Xa, vb = pd * ab + a.w * Xb;
    const T hE = a.w * (inv_gm1 + T(0.5)) + a.x * hu2;
    acc[0] += m;
    acc[1] += (FRAME ? va * tx - vb * ty : va) + u1d * rF + a.y * m;
    acc[2] += (FRAME ? va * ty + vb * tx : vb) + u2d * rF + a.z * m;
    acc[3] += d.w * F + pd * (P + T(0.5) * Q) + hE * Fd +
              (T(0.5) * a.w) * (Pd + ua * Xa + ub * Xb);
}

// Weighted split fluxes of a conserved state, for the flux differences of
// eq. (28).
template <bool FRAME>
__device__ __forceinline__ D4 state_flux(const D4& u, const D2& t, double hwa, double hsa,
                                         double hwb, double hsb, double gm1, double inv_gm1,
                                         const PolyLead& lead) {
#pragma clang fp contract(off)
    const double irho = recip_pos(u.x);
    const double u1 = u.y * irho, u2 = u.z * irho;
    const double usq = fma(u1, u1, u2 * u2);
    const double p = gm1 * fma(-0.5 * u.x, usq, u.w);
    const double beta = 0.5 * u.x * recip_pos(p);
    const double r = rsqrt_pos(beta);
    const double sb = beta * r;
    const double ua = FRAME ? fma(u1, t.x, u2 * t.y) : u1;
    const double ub = FRAME ? fma(u2, t.x, -(u1 * t.y)) : u2;
    const double Sa = ua * sb, Sb = ub * sb;
    double era, ga, erb, gb;
    unit_or_outer(Sa, Sa * Sa, lead, era, ga);
    unit_or_outer(Sb, Sb * Sb, lead, erb, gb);
    // rho E as it is: formed again from p it cost the differences a tenth more rounding error
    return weighted_flux<FRAME, true>(u.x, p, r, u1, u2, ua, ub, u.w, era, ga, erb, gb, t, hwa, hsa,
                                      hwb, hsb, inv_gm1);
}

// Split weights and bits of the sweep-list entries of the colour-sorted point
// q (thread per q): for interior points the x split (a) and y split (b) the
// neighbour falls in; for frame points the t split (a) and the normal split
// (b): n- on the fluid side of a wall point, n+ on the inner side of an outer
// point (used under the kinetic far field) -- membership and weights exactly
// as the residual forms them.
__global__ void __launch_bounds__(kBlock) k_sweep_weights(int64_t n,
                                                          const int32_t* __restrict__ col_perm,
                                                          const D2* __restrict__ xy,
                                                          const D2* __restrict__ frame,
                                                          const int8_t* __restrict__ type,
                                                          const PointGeom* __restrict__ geom,
                                                          const int32_t* __restrict__ off,
                                                          const int32_t* __restrict__ idx,
                                                          D2* __restrict__ w,
                                                          F2* __restrict__ wf,
                                                          uint8_t* __restrict__ code) {
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= n) return;
    const int32_t p = col_perm[q];
    const int8_t ty = type[p];
    const D2 r0 = xy[p], t = frame[p];
    const PointGeom& G = geom[p];
    for (int32_t e = off[q]; e < off[q + 1]; ++e) {
        const D2 ri = xy[idx[e]];
        const double dx = ri.x - r0.x, dy = ri.y - r0.y;
        uint8_t cd = 0;
        double wa = 0.0, wb = 0.0;
        if (ty != kInterior) {
            const double ds = dot_nc(dx, dy, t.x, t.y);
            const double dn = dot_nc(dx, dy, -t.y, t.x);
            cd |= kSwWall;
            if (ds != 0.0) {
                const D2 cc = ds < 0.0 ? G.split[0] : G.split[1];
                cd |= kSwA | (ds < 0.0 ? kSwNegA : 0);
                wa = cc.x * ds + cc.y * dn;
            }
            if (in_normal_split(ty, dn)) {
                cd |= kSwB | (dn < 0.0 ? kSwNegB : 0);
                wb = G.split[2].x * dn + G.split[2].y * ds;
            }
        } else {
            if (dx != 0.0) {
                const D2 cc = dx < 0.0 ? G.split[0] : G.split[1];
                cd |= kSwA | (dx < 0.0 ? kSwNegA : 0);
                wa = cc.x * dx + cc.y * dy;
            }
            if (dy != 0.0) {
                const D2 cc = dy < 0.0 ? G.split[2] : G.split[3];
                cd |= kSwB | (dy < 0.0 ? kSwNegB : 0);
                wb = cc.x * dy + cc.y * dx;
            }
        }
        w[e] = {wa, wb};
        wf[e] = {(float)wa, (float)wb};
        code[e] = cd;
    }
}

// Contribution sum_k w_i^k A_k(U_i) dU_i of neighbour i to point p's sweep
// sum (eq. 22-27) from the entry's weights and split bits: interior points
// use the x and y split the neighbour falls in, frame points the t split and
// the normal split (n- at a wall, n+ at a far-field outer point) in the frame
// t of point p.  A split that the neighbour is not in has weight zero.
// The double-precision sweeps gather (rho, u1, u2, p) and dU of a neighbour,
// 64 bytes, and form erf and exp of S; the fp32 sweeps gather those too (16
// bytes more, formed in double precision by the residual kernel).
template <bool FRAME, class T, int MODE>
__device__ __forceinline__ void sweep_entry(uint8_t cd, const D2& t, const W2<T>& w, int32_t i,
                                            const Vec4<T>* __restrict__ jv0,
                                            const Vec4<T>* __restrict__ jv2,
                                            const D4* __restrict__ U,
                                            const Vec4<T>* __restrict__ dU, T gm1, T inv_gm1,
                                            const PolyLead& lead, T acc[4]) {
    const Vec4<T> d = dU[i];
    const T hwa = T(0.5) * w.x, hwb = T(0.5) * w.y;
    const T hsa = signed_half(hwa, cd, 1), hsb = signed_half(hwb, cd, 3);
    if constexpr (MODE == 1) {
        const D4 u = U[i];
        const D4 v = {u.x + d.x, u.y + d.y, u.z + d.z, u.w + d.w};
        const D4 f1 = state_flux<FRAME>(v, t, hwa, hsa, hwb, hsb, gm1, inv_gm1, lead);
        const D4 f0 = state_flux<FRAME>(u, t, hwa, hsa, hwb, hsb, gm1, inv_gm1, lead);
        acc[0] += f1.x - f0.x;
        acc[1] += f1.y - f0.y;
        acc[2] += f1.z - f0.z;
        acc[3] += f1.w - f0.w;
    } else {
        const Vec4<T> a = jv0[i];
        Vec4<T> k{};
        if constexpr (std::is_same_v<T, float>) k = jv2[i];
        const T rp = recip_pos(a.x * a.w);
        const T irho = a.w * rp, beta = T(0.5) * a.x * (a.x * rp);
        const T isb = rsqrt_pos(beta), sb = beta * isb;
        const T tx = T(t.x), ty = T(t.y);
        const T ua = FRAME ? a.y * tx + a.z * ty : a.y, ub = FRAME ? a.z * tx - a.y * ty : a.z;
        if constexpr (std::is_same_v<T, double>) {
            const T Sa = ua * sb, Sb = ub * sb;
            unit_or_outer(Sa, Sa * Sa, lead, k.x, k.y);
            unit_or_outer(Sb, Sb * Sb, lead, k.z, k.w);
        } else if (FRAME) {  // frame directions: erf/exp at the neighbour state are formed here
            erf_exp(ua * sb, k.x, k.y);
            erf_exp(ub * sb, k.z, k.w);
        }
        weighted_jvp<FRAME>(a, d, irho, beta, isb, sb, ua, ub, k.x, k.y, k.z, k.w, tx, ty, hwa, hsa,
                            hwb, hsb, gm1, inv_gm1, acc);
    }
}

// One colour phase of a sweep (eq. 27).  FWD: dU*_0 = -(R_0 + sum_lower w A dU*) / D_0;
// backward: dU_0 = dU*_0 - (sum_upper w A dU) / D_0.  MODE 0 exact tangent,
// 1 flux difference.  T is the arithmetic of the products and increments.
// LANES consecutive lanes share one point: each walks every LANES-th entry of
// the point's lower (forward) or upper (backward) list.  From four lanes on,
// the partial sums are scattered so that lane v finishes component v, its own
// data requested with the list entries; below, lane 0 finishes the point.  The
// phase's points are the colour-sorted positions [start, start + count) and
// their lists one contiguous block.
// Bound by the bytes gathered at 2,621,440 points (each phase re-reads the
// records of the colours around its points) and by the dependent loads of a
// phase at small ones.  Forward sweep, eight lanes, FP64: 600 us with erf and
// exp of S gathered beside the state and lane 0 finishing a point, 446 us now;
// 163,840 points 78 and 66 us; flux differences there 111 and 78 us; 640,000
// points in mixed precision 145 and 119 us.
template <class T, bool FWD, int MODE, int LANES>
__global__ void __launch_bounds__(kBlock, MODE == 1 || LANES >= 16 ? 4 : 5) k_sweep(
    int32_t start, int32_t count, const int32_t* __restrict__ col_perm,
    const D2* __restrict__ frame, const int8_t* __restrict__ type,
    const int32_t* __restrict__ loff, const int32_t* __restrict__ lidx,
    const W2<T>* __restrict__ lw, const uint8_t* __restrict__ lcode,
    const int32_t* __restrict__ qcomp, const int32_t* __restrict__ active,
    const Vec4<T>* __restrict__ jv0, const Vec4<T>* __restrict__ jv2,
    const D4* __restrict__ U, const D4* __restrict__ R,
    const T* __restrict__ Dg, Vec4<T>* __restrict__ dU, double gamma, int farfield) {
    constexpr bool SCATTER = LANES >= 4;
    const int gt = xcd_block(blockIdx.x, gridDim.x) * blockDim.x + threadIdx.x;
    const int pt = gt / LANES, lane = gt % LANES;
    if (pt >= count) return;  // uniform over the lanes of a point
    // A phase is short and latency-bound, so its loads are ordered to form as
    // few dependent levels as possible: q-indexed offsets and permutation;
    // then the point's own record and the list entries together; then the
    // neighbours' data.  Nothing waits on the point type before the list walk
    // (an outer point's products are formed and discarded).
    const int32_t q = start + pt;
    const int32_t p = col_perm[q];
    const int32_t e0 = loff[q], e1 = loff[q + 1];
    const int32_t k = qcomp ? qcomp[q] : 0;
    if (!qcomp && !active[0]) return;  // beside the loads above, not before them
    // the lane's first list entry, then the point's own record
    int32_t e = e0 + lane;
    uint8_t cd = 0;
    W2<T> w = {T(0), T(0)};
    int32_t i = 0;
    if (e < e1) {
        cd = lcode[e];
        w = lw[e];
        i = lidx[e];
    }
    const int v = lane & 3;
    T own = T(0), dg = T(1);
    int8_t ty = kInterior;
    if (SCATTER) {
        ty = type[p];
        dg = Dg[p];
        own = FWD ? T(reinterpret_cast<const double*>(R + p)[v])
                  : reinterpret_cast<const T*>(dU + p)[v];
    }
    // retired component of a batch (uniform per point): looked up beside the
    // loads above, not before them
    if (qcomp && !active[k]) return;
    const T gm1 = T(gamma - 1.0), inv_gm1 = T(1.0 / (gamma - 1.0));
    const PolyLead lead = poly_lead<T>();
    T acc[4] = {T(0), T(0), T(0), T(0)};
    T first[4] = {T(0), T(0), T(0), T(0)};  // sixteen lanes: the first entry's part
    while (e < e1) {
        // the next entry is requested before this one's neighbour data is used;
        // past the end the last entry is re-read (in bounds) and not used
        const int32_t en = e + LANES;
        const int32_t ec = en < e1 ? en : e1 - 1;
        const uint8_t cdn = lcode[ec];
        const W2<T> wn = lw[ec];
        const int32_t in = lidx[ec];
        if (__builtin_expect(cd & kSwWall, 0))
            sweep_entry<true, T, MODE>(cd, frame[p], w, i, jv0, jv2, U, dU, gm1, inv_gm1, lead, acc);
        else
            sweep_entry<false, T, MODE>(cd, D2{1.0, 0.0}, w, i, jv0, jv2, U, dU, gm1, inv_gm1, lead,
                                        acc);
        if constexpr (LANES == 16)
            if (e < e0 + LANES) {
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    first[c] = acc[c];
                    acc[c] = T(0);
                }
            }
        cd = cdn;
        w = wn;
        i = in;
        e = en;
    }
    // lists of at most 32 entries: one each (in the loop's form all the same; cut
    // down to one pass, the compiler lays out more code, and a phase takes longer)
    if constexpr (LANES == 32)
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            first[c] = acc[c];
            acc[c] = from_second_half(acc[c]);
        }
    if constexpr (SCATTER) {
        const T sum = LANES >= 16 ? scatter_sum<16>(first, acc, lane & 15)
                                  : scatter_sum<LANES>(acc, first, lane);
        T out = FWD ? -(own + sum) / dg : own - sum / dg;
        if (ty == kOuter && !farfield) {
            if (!FWD) return;
            out = T(0);
        }
        if (ty == kWall) {
            const D2 t = frame[p];
            const T nx = T(-t.y), ny = T(t.x);
            const T mn = dpp<kDppQuad1>(out) * nx + dpp<kDppQuad2>(out) * ny;
            out -= v == 1 ? mn * nx : (v == 2 ? mn * ny : T(0));
        }
        if (lane < 4) reinterpret_cast<T*>(dU + p)[v] = out;
    } else {
        if constexpr (LANES == 2)
#pragma unroll
            for (int c = 0; c < 4; ++c) acc[c] += dpp<kDppXor1>(acc[c]);
        if (lane != 0) return;
        ty = type[p];
        dg = Dg[p];
        Vec4<T> o;
        if (FWD) {
            const D4 r = R[p];
            o = {T(r.x), T(r.y), T(r.z), T(r.w)};
        } else {
            o = dU[p];
        }
        if (ty == kOuter && !farfield) {
            if (FWD) dU[p] = {T(0), T(0), T(0), T(0)};
            return;
        }
        const T iD = T(1) / dg;
        T out[4] = {o.x - acc[0] * iD, o.y - acc[1] * iD, o.z - acc[2] * iD, o.w - acc[3] * iD};
        if (FWD) {
            out[0] = -(o.x + acc[0]) * iD;
            out[1] = -(o.y + acc[1]) * iD;
            out[2] = -(o.z + acc[2]) * iD;
            out[3] = -(o.w + acc[3]) * iD;
        }
        if (ty == kWall) {
            const D2 t = frame[p];
            const T nx = T(-t.y), ny = T(t.x);
            const T mn = out[1] * nx + out[2] * ny;
            out[1] -= mn * nx;
            out[2] -= mn * ny;
        }
        dU[p] = {out[0], out[1], out[2], out[3]};
    }
}

// U += dU (Section 3) and the q-variables of the new state (eq. 14).
template <class T>
__global__ void __launch_bounds__(kBlock) k_update(int64_t n, double gamma, D4* __restrict__ U,
                                                   const Vec4<T>* __restrict__ dU,
                                                   const int32_t* __restrict__ comp,
                                                   const int32_t* __restrict__ active,
                                                   D4* __restrict__ q, int32_t* __restrict__ flags) {
    const int64_t p = (int64_t)xcd_block(blockIdx.x, gridDim.x) * blockDim.x + threadIdx.x;
    if (p >= n || !live(comp, active, p)) return;
    D4 u = U[p];
    const Vec4<T> d = dU[p];
    u.x += (double)d.x;
    u.y += (double)d.y;
    u.z += (double)d.z;
    u.w += (double)d.w;
    U[p] = u;
    bool bad;
    q[p] = q_of_U(u, gamma, 1.0 / (gamma - 1.0), bad);
    if (bad) flags[0] = 1;
}

// Explicit iteration (the paper's explicit LSKUM solver): U <- U - dt R with
// the implicit scheme's local time step dt = CFL rmin / (|u| + a) at the
// current state, then the next q-variables.  Outer points keep their state
// unless the kinetic far field gives them a residual.
__global__ void __launch_bounds__(kBlock) k_explicit_update(
    int64_t n, double gamma, const double* __restrict__ cfl, const int8_t* __restrict__ type,
    const D4* __restrict__ lsq, const int32_t* __restrict__ comp,
    const int32_t* __restrict__ active, const D4* __restrict__ R, D4* __restrict__ U,
    D4* __restrict__ q, int32_t* __restrict__ flags, int farfield) {
    const int64_t p = (int64_t)xcd_block(blockIdx.x, gridDim.x) * blockDim.x + threadIdx.x;
    if (p >= n || !live(comp, active, p) || (type[p] == kOuter && !farfield)) return;
    D4 u = U[p];
    const double rho = u.x, irho = 1.0 / rho;
    const double u1 = u.y * irho, u2 = u.z * irho;
    const double usq = u1 * u1 + u2 * u2;
    const double pr = (gamma - 1.0) * (u.w - 0.5 * rho * usq);
    const double a = sqrt(gamma * pr / rho);
    const double dt = cfl[comp ? comp[p] : 0] * lsq[p].w / (sqrt(usq) + a);
    const D4 r = R[p];
    u.x -= dt * r.x;
    u.y -= dt * r.y;
    u.z -= dt * r.z;
    u.w -= dt * r.w;
    U[p] = u;
    bool bad;
    q[p] = q_of_U(u, gamma, 1.0 / (gamma - 1.0), bad);
    if (bad) flags[0] = 1;
}

// Pressure force on the closed wall polygon of each component (one block per
// component): sum over edges (a, b) of -(p_mid - p_inf) * |e| * (edge normal
// pointing out of the body), orient = +1 for a counter-clockwise polygon.
__global__ void __launch_bounds__(kBlock) k_forces(const int32_t* __restrict__ wall,
                                                   const int32_t* __restrict__ wall_off,
                                                   const double* __restrict__ orient_k,
                                                   const D2* __restrict__ xy, const D4* __restrict__ U,
                                                   double gamma, double* __restrict__ out) {
    __shared__ double rx[kBlock / 64], ry[kBlock / 64];
    const int k = blockIdx.x;
    const int64_t w0 = wall_off[k], m = wall_off[k + 1] - w0;
    const double orient = orient_k[k];
    double fx = 0.0, fy = 0.0;
    const double pinf = 1.0 / gamma;
    for (int64_t j = threadIdx.x; j < m; j += blockDim.x) {
        const int32_t a = wall[w0 + j], b = wall[w0 + (j + 1 == m ? 0 : j + 1)];
        const D4 ua = U[a], ub = U[b];
        const double pa = (gamma - 1.0) * (ua.w - 0.5 * (ua.y * ua.y + ua.z * ua.z) / ua.x);
        const double pb = (gamma - 1.0) * (ub.w - 0.5 * (ub.y * ub.y + ub.z * ub.z) / ub.x);
        const double pm = 0.5 * (pa + pb) - pinf;
        const D2 ra = xy[a], rb = xy[b];
        const double ex = rb.x - ra.x, ey = rb.y - ra.y;
        fx -= pm * (orient * ey);
        fy -= pm * (-orient * ex);
    }
    for (int o = 32; o > 0; o >>= 1) {
        fx += __shfl_xor(fx, o, 64);
        fy += __shfl_xor(fy, o, 64);
    }
    if ((threadIdx.x & 63) == 0) {
        rx[threadIdx.x >> 6] = fx;
        ry[threadIdx.x >> 6] = fy;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double sx = 0, sy = 0;
        for (int w = 0; w < kBlock / 64; ++w) {
            sx += rx[w];
            sy += ry[w];
        }
        out[2 * k] = sx;
        out[2 * k + 1] = sy;
    }
}

__global__ void __launch_bounds__(kBlock) k_soa_to_aos(const double* __restrict__ soa,
                                                       D4* __restrict__ aos, int64_t n) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    aos[p] = {soa[p], soa[n + p], soa[2 * n + p], soa[3 * n + p]};
}

template <class T>
__global__ void __launch_bounds__(kBlock) k_aos_to_soa(const Vec4<T>* __restrict__ aos,
                                                       double* __restrict__ soa, int64_t n) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    const Vec4<T> v = aos[p];
    soa[p] = (double)v.x;
    soa[n + p] = (double)v.y;
    soa[2 * n + p] = (double)v.z;
    soa[3 * n + p] = (double)v.w;
}

__global__ void k_clear_flags(int32_t* flags) {
    if (threadIdx.x < 4) flags[threadIdx.x] = 0;
}

inline unsigned grid_for(int64_t n) { return (unsigned)((n + kBlock - 1) / kBlock); }

}  // namespace

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------
hipError_t launch_precompute(Cloud& c, hipStream_t st) {
    unsigned long long* d_cnt = nullptr;
    hipError_t e = hipMalloc((void**)&d_cnt, 2 * sizeof(unsigned long long));
    if (e != hipSuccess) return e;
    unsigned long long h[2] = {0, 0};
    e = hipMemsetAsync(d_cnt, 0, 2 * sizeof(unsigned long long), st);
    if (e == hipSuccess && c.n > 0) {
        hipLaunchKernelGGL(k_precompute, dim3(grid_for(c.n)), dim3(kBlock), 0, st, c.n, c.xy,
                           c.frame, c.type, c.off, c.idx, c.geom, c.lsq, d_cnt);
        e = hipGetLastError();
    }
    if (e == hipSuccess) e = hipMemcpyAsync(h, d_cnt, sizeof(h), hipMemcpyDeviceToHost, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    (void)hipFree(d_cnt);
    if (e != hipSuccess) return e;
    c.n_degenerate = (int64_t)h[1];
    if (h[0]) return hipErrorInvalidValue;  // singular full stencil, reported by the caller
    return hipSuccess;
}

hipError_t launch_sweep_weights(Cloud& c, hipStream_t st) {
    if (c.n > 0) {
        hipLaunchKernelGGL(k_sweep_weights, dim3(grid_for(c.n)), dim3(kBlock), 0, st, c.n,
                           c.col_perm, c.xy, c.frame, c.type, c.geom, c.lo_off, c.lo_idx, c.lo_w,
                           c.lo_wf, c.lo_code);
        hipLaunchKernelGGL(k_sweep_weights, dim3(grid_for(c.n)), dim3(kBlock), 0, st, c.n,
                           c.col_perm, c.xy, c.frame, c.type, c.geom, c.up_off, c.up_idx, c.up_w,
                           c.up_wf, c.up_code);
    }
    return hipGetLastError();
}

hipError_t launch_free_stream(State& s) {
    const Cloud& c = *s.cloud;
    hipLaunchKernelGGL(k_free_stream, dim3(grid_for(c.n)), dim3(kBlock), 0, s.stream, c.n, c.type,
                       c.frame, s.prm.gamma, c.comp, s.vinf, s.U);
    return hipGetLastError();
}

hipError_t launch_q_from_U(State& s) {
    const Cloud& c = *s.cloud;
    hipLaunchKernelGGL(k_q_from_U, dim3(grid_for(c.n)), dim3(kBlock), 0, s.stream, c.n,
                       s.prm.gamma, s.U, s.q, s.flags);
    return hipGetLastError();
}

template <int LANES>
static void qgrad_lanes(State& s, bool keep) {
    const Cloud& c = *s.cloud;
    const dim3 g(grid_for(c.n * LANES)), b(kBlock);
    const double K = s.prm.limiter_k;
    const int m = s.prm.inner_iters;
    const bool lim = s.prm.limiter != 0;
    // pass 0 (first order), then m inner passes; the limiter rides on the last
    if (m == 0 && lim)
        hipLaunchKernelGGL((k_qgrad<false, true, LANES>), g, b, 0, s.stream, c.n, K, c.xy, c.off,
                           c.idx, c.lsq, c.comp, s.active, s.q, nullptr, nullptr,
                           keep ? s.qx[0] : nullptr, keep ? s.qy[0] : nullptr, s.qxl, s.qyl);
    else
        hipLaunchKernelGGL((k_qgrad<false, false, LANES>), g, b, 0, s.stream, c.n, K, c.xy, c.off,
                           c.idx, c.lsq, c.comp, s.active, s.q, nullptr, nullptr, s.qx[0],
                           s.qy[0], nullptr, nullptr);
    int cur = 0;
    for (int it = 0; it < m; ++it) {
        if (it == m - 1 && lim)
            hipLaunchKernelGGL((k_qgrad<true, true, LANES>), g, b, 0, s.stream, c.n, K, c.xy,
                               c.off, c.idx, c.lsq, c.comp, s.active, s.q, s.qx[cur], s.qy[cur],
                               keep ? s.qx[1 - cur] : nullptr, keep ? s.qy[1 - cur] : nullptr,
                               s.qxl, s.qyl);
        else
            hipLaunchKernelGGL((k_qgrad<true, false, LANES>), g, b, 0, s.stream, c.n, K, c.xy,
                               c.off, c.idx, c.lsq, c.comp, s.active, s.q, s.qx[cur], s.qy[cur],
                               s.qx[1 - cur], s.qy[1 - cur], nullptr, nullptr);
        cur = 1 - cur;
    }
    s.qsel = cur;
}

// Tiled passes (LDS-staged neighbours): block = tile, staged arrays of stride
// S.
template <int S>
static void qgrad_tiled(State& s, bool keep) {
    const Cloud& c = *s.cloud;
    const dim3 g((unsigned)c.ntile), b(kBlock);
    const double K = s.prm.limiter_k;
    const int m = s.prm.inner_iters;
    const bool lim = s.prm.limiter != 0;
    if (m == 0 && lim)
        hipLaunchKernelGGL((k_qgrad_tiled<false, true, S>), g, b, 0, s.stream, K, c.xy, c.off,
                           c.tile_pts, c.lnbr, c.tile_off, c.tile_idx, c.lsq,
                           c.comp, s.active, s.q, nullptr, nullptr, keep ? s.qx[0] : nullptr,
                           keep ? s.qy[0] : nullptr, s.qxl, s.qyl);
    else
        hipLaunchKernelGGL((k_qgrad_tiled<false, false, S>), g, b, 0, s.stream, K, c.xy, c.off,
                           c.tile_pts, c.lnbr, c.tile_off, c.tile_idx, c.lsq,
                           c.comp, s.active, s.q, nullptr, nullptr, s.qx[0], s.qy[0], nullptr,
                           nullptr);
    int cur = 0;
    for (int it = 0; it < m; ++it) {
        if (it == m - 1 && lim)
            hipLaunchKernelGGL((k_qgrad_tiled<true, true, S>), g, b, 0, s.stream, K, c.xy, c.off,
                               c.tile_pts, c.lnbr, c.tile_off, c.tile_idx, c.lsq,
                               c.comp, s.active, s.q, s.qx[cur], s.qy[cur],
                               keep ? s.qx[1 - cur] : nullptr, keep ? s.qy[1 - cur] : nullptr,
                               s.qxl, s.qyl);
        else
            hipLaunchKernelGGL((k_qgrad_tiled<true, false, S>), g, b, 0, s.stream, K, c.xy, c.off,
                               c.tile_pts, c.lnbr, c.tile_off, c.tile_idx, c.lsq,
                               c.comp, s.active, s.q, s.qx[cur], s.qy[cur], s.qx[1 - cur],
                               s.qy[1 - cur], nullptr, nullptr);
        cur = 1 - cur;
    }
    s.qsel = cur;
}

hipError_t launch_q_derivatives(State& s, bool keep_unlimited) {
    if (s.qgrad_tiled && s.cloud->ntile > 0) {
        switch (tile_stride(s.cloud->tile_hmax)) {
            case kTileStride: qgrad_tiled<kTileStride>(s, keep_unlimited); break;
            case kTileStride4: qgrad_tiled<kTileStride4>(s, keep_unlimited); break;
            case kTileStride3: qgrad_tiled<kTileStride3>(s, keep_unlimited); break;
            default: qgrad_tiled<kQTileMax>(s, keep_unlimited);
        }
        return hipGetLastError();
    }
    switch (s.qgrad_lanes) {
        case 1: qgrad_lanes<1>(s, keep_unlimited); break;
        case 2: qgrad_lanes<2>(s, keep_unlimited); break;
        case 8: qgrad_lanes<8>(s, keep_unlimited); break;
        default: qgrad_lanes<4>(s, keep_unlimited); break;
    }
    return hipGetLastError();
}

// In colour order the first forward phase (no lower neighbours) is done by the
// residual kernel and the first backward phase (no upper neighbours: dU = dU*)
// is skipped.
static int fused_first_colour(const State& s) { return s.prm.order == 0 && s.prm.scheme == 0; }

template <bool MIXED, int LANES>
static void residual_lanes(State& s, bool in_step) {
    const Cloud& c = *s.cloud;
    const ResidualArgs A{c.n,        s.prm.gamma, s.cfl,      c.xy,
                         c.frame,    c.type,      c.off,      c.idx,
                         c.lsq,      c.geom,      c.comp,     s.active,   c.tile_pts,
                         c.lnbr,     c.tile_off,  c.tile_idx, s.U,
                         s.q,        s.prm.limiter ? s.qxl : s.qx[s.qsel],
                         s.prm.limiter ? s.qyl : s.qy[s.qsel], s.R,
                         s.D,        s.jv0,       s.jv0f,
                         s.jv2f,     s.Df,        s.rr,       s.flags,
                         s.prm.variant, s.prm.jvp_mode, s.dU, s.dUf,
                         s.Rs,       c.colour,    in_step && fused_first_colour(s),
                         s.prm.farfield, s.vinf};
    const ResidualForm form = residual_form(s);
    if (!form.tiled) {
        hipLaunchKernelGGL((k_residual<MIXED, LANES>), dim3(grid_for(c.n * LANES)), dim3(kBlock), 0,
                           s.stream, A);
        return;
    }
    const dim3 g((unsigned)c.ntile), b(kQTile * LANES * form.sub);
    if constexpr (LANES == 2) {
        if (form.sub == 4) {
            hipLaunchKernelGGL((k_residual_tiled<MIXED, 2, kTileStride, 4>), g, b, 0, s.stream, A);
            return;
        }
        if (form.sub == 2) {
            hipLaunchKernelGGL((k_residual_tiled<MIXED, 2, kTileStride, 2>), g, b, 0, s.stream, A);
            return;
        }
    }
    hipLaunchKernelGGL((k_residual_tiled<MIXED, LANES, kTileStride, 1>), g, b, 0, s.stream, A);
}

template <bool MIXED>
static void residual_t(State& s, bool in_step) {
    switch (s.residual_lanes) {
        case 1: residual_lanes<MIXED, 1>(s, in_step); break;
        case 2: residual_lanes<MIXED, 2>(s, in_step); break;
        case 8: residual_lanes<MIXED, 8>(s, in_step); break;
        default: residual_lanes<MIXED, 4>(s, in_step); break;
    }
}

hipError_t launch_residual(State& s, int slot, bool in_step) {
    (void)slot;
    if (s.prm.precision == 1)
        residual_t<true>(s, in_step);
    else
        residual_t<false>(s, in_step);
    return hipGetLastError();
}

hipError_t launch_norm(State& s, int slot) {
    const Cloud& c = *s.cloud;
    hipLaunchKernelGGL(k_norm_partial, dim3(c.nchunk), dim3(kBlock), 0, s.stream, s.rr,
                       c.chunk_start, c.chunk_comp, s.active, s.partial);
    hipLaunchKernelGGL(k_norm_comp, dim3(c.ncomp), dim3(64), 0, s.stream, s.partial,
                       c.comp_chunk_off, c.comp_inv_active, s.tol_abs, s.active, s.status, s.iters,
                       s.res_last, s.res_hist + (size_t)slot * c.ncomp);
    return hipGetLastError();
}

hipError_t launch_reset_components(State& s) {
    const Cloud& c = *s.cloud;
    hipLaunchKernelGGL(k_reset_components, dim3((c.ncomp + 63) / 64), dim3(64), 0, s.stream,
                       c.ncomp, s.active, s.status, s.iters);
    return hipGetLastError();
}

// The phases of a sweep as ranges of the colour-sorted points: one per
// colour (Algorithm 6), or per (point type, colour) with wall, interior and
// outer points in turn (Algorithm 5); colours ascending forward, descending
// backward.
static std::vector<std::pair<int32_t, int32_t>> sweep_phases(const State& s, bool forward) {
    const Cloud& c = *s.cloud;
    std::vector<std::pair<int32_t, int32_t>> ph;
    const int C = c.ncolour;
    if (s.prm.order == 0) {
        for (int k = fused_first_colour(s) ? 1 : 0; k < C; ++k) {
            const int col = forward ? k : C - 1 - k;
            ph.emplace_back(c.h_col_off[col], c.h_col_off[col + 1] - c.h_col_off[col]);
        }
        return ph;
    }
    for (int g = 0; g < 3; ++g)
        for (int k = 0; k < C; ++k) {
            const int col = forward ? k : C - 1 - k;
            const int32_t a = c.h_grp_off[3 * col + g], b = c.h_grp_off[3 * col + g + 1];
            ph.emplace_back(a, b - a);
        }
    return ph;
}

// The sweep-list weights in the sweep arithmetic's precision.
template <class T>
static const W2<T>* list_weights(const D2* w, const F2* wf) {
    if constexpr (std::is_same_v<T, float>) return wf;
    else return w;
}

constexpr int64_t kThinPhase = 160 * 1024;  // threads: two or three wavefronts on every SIMD

template <class T, int MODE, int LANES>
static void sweep_lanes(State& s, bool forward, const Vec4<T>* jv0, const Vec4<T>* jv2,
                        const T* Dg, Vec4<T>* dU) {
    const Cloud& c = *s.cloud;
    for (const auto& [start, cnt] : sweep_phases(s, forward)) {
        if (!cnt) continue;
        // one wavefront to a block while a phase has two or three for a SIMD at most:
        // they spread over the CUs, where four to a block wait on one another's gathers
        // (iteration with 256 and 64 threads: 1,024 points 95.2 and 89.9 us, 80,000
        // points 158.5 and 154.1, 163,840 points, 146,000 threads, 209.7 and 207.6;
        // 215,040 points, 191,000 threads, 210.4 and 211.7; 360,000 points in mixed
        // precision 281 and 285)
        const int64_t threads = (int64_t)cnt * LANES;
        const int block = threads <= kThinPhase ? 64 : kBlock;
        const dim3 g((unsigned)((threads + block - 1) / block)), b(block);
        if (forward)
            hipLaunchKernelGGL((k_sweep<T, true, MODE, LANES>), g, b, 0, s.stream, start, cnt,
                               c.col_perm, c.frame, c.type, c.lo_off, c.lo_idx,
                               list_weights<T>(c.lo_w, c.lo_wf), c.lo_code, c.qcomp, s.active,
                               jv0, jv2, s.U, s.prm.variant ? s.Rs : s.R, Dg, dU,
                               s.prm.gamma, s.prm.farfield);
        else
            hipLaunchKernelGGL((k_sweep<T, false, MODE, LANES>), g, b, 0, s.stream, start, cnt,
                               c.col_perm, c.frame, c.type, c.up_off, c.up_idx,
                               list_weights<T>(c.up_w, c.up_wf), c.up_code, c.qcomp, s.active,
                               jv0, jv2, s.U, s.R, Dg, dU, s.prm.gamma, s.prm.farfield);
    }
}

template <class T, int MODE>
static void sweep_t(State& s, bool forward, const Vec4<T>* jv0, const Vec4<T>* jv2,
                    const T* Dg, Vec4<T>* dU) {
    switch (s.sweep_lanes) {
        case 1: sweep_lanes<T, MODE, 1>(s, forward, jv0, jv2, Dg, dU); break;
        case 2: sweep_lanes<T, MODE, 2>(s, forward, jv0, jv2, Dg, dU); break;
        case 8: sweep_lanes<T, MODE, 8>(s, forward, jv0, jv2, Dg, dU); break;
        case 16: sweep_lanes<T, MODE, 16>(s, forward, jv0, jv2, Dg, dU); break;
        case 32: sweep_lanes<T, MODE, 32>(s, forward, jv0, jv2, Dg, dU); break;
        default: sweep_lanes<T, MODE, 4>(s, forward, jv0, jv2, Dg, dU); break;
    }
}

template <class T>
__global__ void __launch_bounds__(kBlock) k_zero4(int64_t n, Vec4<T>* __restrict__ v) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p < n) v[p] = {T(0), T(0), T(0), T(0)};
}

hipError_t launch_sweep_dir(State& s, bool forward) {
    const Cloud& c = *s.cloud;
    // Algorithm 5 reads increments of points not yet visited in the forward
    // sweep: they start the sweep at zero (a kernel, so that graphs replay it)
    if (forward && s.prm.order == 1) {
        if (s.prm.precision == 1)
            hipLaunchKernelGGL(k_zero4<float>, dim3(grid_for(c.n)), dim3(kBlock), 0, s.stream, c.n,
                               s.dUf);
        else
            hipLaunchKernelGGL(k_zero4<double>, dim3(grid_for(c.n)), dim3(kBlock), 0, s.stream,
                               c.n, s.dU);
    }
    if (s.prm.precision == 1)
        sweep_t<float, 0>(s, forward, s.jv0f, (const F4*)s.jv2f, s.Df, s.dUf);
    else if (s.prm.jvp_mode == 1)
        sweep_t<double, 1>(s, forward, s.jv0, (const D4*)nullptr, s.D, s.dU);
    else
        sweep_t<double, 0>(s, forward, s.jv0, (const D4*)nullptr, s.D, s.dU);
    return hipGetLastError();
}

hipError_t launch_sweeps(State& s) {
    hipError_t e = launch_sweep_dir(s, true);
    if (e != hipSuccess) return e;
    return launch_sweep_dir(s, false);
}

hipError_t launch_explicit_update(State& s) {
    const Cloud& c = *s.cloud;
    hipLaunchKernelGGL(k_explicit_update, dim3(grid_for(c.n)), dim3(kBlock), 0, s.stream, c.n,
                       s.prm.gamma, s.cfl, c.type, c.lsq, c.comp, s.active, s.R, s.U, s.q,
                       s.flags, s.prm.farfield);
    return hipGetLastError();
}

hipError_t launch_update(State& s) {
    const Cloud& c = *s.cloud;
    if (s.prm.precision == 1)
        hipLaunchKernelGGL(k_update<float>, dim3(grid_for(c.n)), dim3(kBlock), 0, s.stream, c.n,
                           s.prm.gamma, s.U, s.dUf, c.comp, s.active, s.q, s.flags);
    else
        hipLaunchKernelGGL(k_update<double>, dim3(grid_for(c.n)), dim3(kBlock), 0, s.stream, c.n,
                           s.prm.gamma, s.U, s.dU, c.comp, s.active, s.q, s.flags);
    return hipGetLastError();
}

hipError_t launch_forces(State& s) {
    const Cloud& c = *s.cloud;
    hipLaunchKernelGGL(k_forces, dim3(c.ncomp), dim3(kBlock), 0, s.stream, c.wall_list,
                       c.wall_off, c.comp_orient, c.xy, s.U, s.prm.gamma, s.fsum);
    return hipGetLastError();
}

hipError_t launch_soa_to_aos(const double* soa, D4* aos, int64_t n, hipStream_t st) {
    if (n) hipLaunchKernelGGL(k_soa_to_aos, dim3(grid_for(n)), dim3(kBlock), 0, st, soa, aos, n);
    return hipGetLastError();
}

hipError_t launch_aos_to_soa(const D4* aos, double* soa, int64_t n, hipStream_t st) {
    if (n)
        hipLaunchKernelGGL(k_aos_to_soa<double>, dim3(grid_for(n)), dim3(kBlock), 0, st, aos, soa, n);
    return hipGetLastError();
}

hipError_t launch_aosf_to_soa(const F4* aos, double* soa, int64_t n, hipStream_t st) {
    if (n)
        hipLaunchKernelGGL(k_aos_to_soa<float>, dim3(grid_for(n)), dim3(kBlock), 0, st, aos, soa, n);
    return hipGetLastError();
}

hipError_t launch_clear_flags(int32_t* flags, hipStream_t st) {
    hipLaunchKernelGGL(k_clear_flags, dim3(1), dim3(64), 0, st, flags);
    return hipGetLastError();
}

__global__ void k_fill(int n, double v, double* __restrict__ out) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k < n) out[k] = v;
}

// The allocation-free residual's launches around the common ones: what a state
// keeps per component, then the field as points with its q-variables; at the end
// the residual as components with its norm and flag.  Eight launches in all: at
// 40,250 points 43 us, and 53 with the fifteen that a state's own calls would take.
__global__ void k_scratch_begin(int nc, double cfl, double v1, double v2, double* __restrict__ cfls,
                                double* __restrict__ tol_abs, double* __restrict__ vinf,
                                int32_t* __restrict__ active, int32_t* __restrict__ status,
                                int32_t* __restrict__ iters, int32_t* __restrict__ flags) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k < 4) flags[k] = 0;
    if (k >= nc) return;
    cfls[k] = cfl;
    tol_abs[k] = 0.0;
    vinf[2 * k] = v1;
    vinf[2 * k + 1] = v2;
    active[k] = 1;
    status[k] = 0;
    iters[k] = 0;
}

__global__ void __launch_bounds__(kBlock) k_load_field(int64_t n, double gamma,
                                                       const double* __restrict__ soa,
                                                       D4* __restrict__ U, D4* __restrict__ q,
                                                       int32_t* __restrict__ flags) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    const D4 u = {soa[p], soa[n + p], soa[2 * n + p], soa[3 * n + p]};
    U[p] = u;
    bool bad;
    q[p] = q_of_U(u, gamma, 1.0 / (gamma - 1.0), bad);
    if (bad) flags[0] = 1;
}

__global__ void __launch_bounds__(kBlock) k_residual_out(int64_t n, const D4* __restrict__ R,
                                                         const double* __restrict__ res,
                                                         const int32_t* __restrict__ flags,
                                                         double* __restrict__ soa,
                                                         double* __restrict__ out) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p == 0) {
        out[0] = res[0];
        out[1] = flags[0] ? 1.0 : 0.0;
    }
    if (p >= n) return;
    const D4 v = R[p];
    soa[p] = v.x;
    soa[n + p] = v.y;
    soa[2 * n + p] = v.z;
    soa[3 * n + p] = v.w;
}

hipError_t launch_scratch_begin(State& s, double v1, double v2, const double* U) {
    const Cloud& c = *s.cloud;
    hipLaunchKernelGGL(k_scratch_begin, dim3((c.ncomp + 63) / 64), dim3(64), 0, s.stream, c.ncomp,
                       s.prm.cfl, v1, v2, s.cfl, s.tol_abs, s.vinf, s.active, s.status, s.iters,
                       s.flags);
    hipLaunchKernelGGL(k_load_field, dim3(grid_for(c.n)), dim3(kBlock), 0, s.stream, c.n,
                       s.prm.gamma, U, s.U, s.q, s.flags);
    return hipGetLastError();
}

hipError_t launch_residual_out(State& s, double* R, double* out) {
    const int64_t n = R ? s.cloud->n : 0;
    hipLaunchKernelGGL(k_residual_out, dim3(std::max(grid_for(n), 1u)), dim3(kBlock), 0, s.stream, n,
                       s.R, s.res_hist, s.flags, R, out);
    return hipGetLastError();
}

hipError_t reset_cfl(State& s) {
    const int nc = s.cloud->ncomp;
    hipLaunchKernelGGL(k_fill, dim3((nc + 255) / 256), dim3(256), 0, s.stream, nc, s.prm.cfl,
                       s.cfl);
    return hipGetLastError();
}

hipError_t clear_increment(State& s, int64_t p0, int64_t n) {
    if (n <= 0) return hipSuccess;
    hipError_t e = hipMemsetAsync(s.dU + p0, 0, n * sizeof(D4), s.stream);
    if (e == hipSuccess) e = hipMemsetAsync(s.dUf + p0, 0, n * sizeof(F4), s.stream);
    return e;
}

}  // namespace lskum
