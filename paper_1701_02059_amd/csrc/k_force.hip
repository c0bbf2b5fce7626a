// Pair force / torque evaluation and the velocity-Verlet step on gfx950.
//
// Force Evaluation section: pairwise lipid-lipid, lipid-protein and
// protein-protein forces are found through the Voronoi cells (here: the
// per-particle neighbour lists built from the cell pairs at each cell update,
// valid while no particle has moved more than the skin), plus the bonds of
// physically linked proteins.  One wavefront owns a chunk of 64 consecutive
// cell-sorted particles; lane l accumulates the force and torque on particle
// base + l from every partner in column l of the chunk's ELL list, so the
// per-particle sums need no atomics and are bitwise reproducible.  Every
// candidate goes through the exact FP64 neighbour test; the pair law then runs
// in FP64 or, in mixed mode, in FP32 on the FP64-formed separation, while
// energy and virial sums stay FP64.
//
// Software Overview section (time-stepping loop): kick-drift advances positions
// and lipid orientations (free linear-rotor rotation about the angular
// velocity); the second half-kick is fused into the force kernel's epilogue.
#include "rbc_dev.h"

#include <mutex>

namespace rbc {

__device__ __forceinline__ int lane_id_f() { return threadIdx.x & (WAVE - 1); }

template <class T>
__device__ __forceinline__ T wave_sum(T v) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

template <class T>
__device__ __forceinline__ T ipow(T c, int e) {
    T r = (T)1;
    for (int q = 0; q < e; ++q) r *= c;
    return r;
}

// One of three FP64 cutoffs by partner type, as bit selects (no branches).
__device__ __forceinline__ double sel_cut(int t, double a, double b, double c) {
    long long r = (t == 1) ? __double_as_longlong(b) : __double_as_longlong(c);
    r = (t == 0) ? __double_as_longlong(a) : r;
    return __longlong_as_double(r);
}

__device__ __forceinline__ float sel_cutf(int t, float a, float b, float c) {
    int r = (t == 1) ? __float_as_int(b) : __float_as_int(c);
    r = (t == 0) ? __float_as_int(a) : r;
    return __int_as_float(r);
}

// ------------------------------------------------------------------ pair laws

// Lipid-lipid orientation-dependent law; d = x_i - x_j.  Adds the force and torque
// on i and returns U.  FAST: the default constants zeta = 4 and sin(theta0) = 0
// folded in at compile time (same arithmetic with the zero terms removed).
template <class T, bool FAST>
__device__ __forceinline__ T lipid_pair(const DevParams &P, T dx, T dy, T dz, T nix, T niy, T niz, T njx, T njy,
                                        T njz, T &fx, T &fy, T &fz, T &tx, T &ty, T &tz) {
    const T eps = (T)P.eps, mu = (T)P.mu, st0 = FAST ? (T)0 : (T)P.st0, rmin = (T)P.r_min;
    T r2 = dx * dx + dy * dy + dz * dz;
    T rinv, r;
    if constexpr (sizeof(T) == 4) {
        rinv = __builtin_amdgcn_rsqf(r2);
        r = r2 * rinv;
    } else {
        r = sqrt(r2);
        rinv = (T)1 / r;
    }
    const T ex = dx * rinv, ey = dy * rinv, ez = dz * rinv;
    const T s = nix * ex + niy * ey + niz * ez;
    const T t = njx * ex + njy * ey + njz * ez;
    const T c = nix * njx + niy * njy + niz * njz;
    T a = c - s * t;
    if (!FAST) a += st0 * (t - s) - st0 * st0;
    const T phi = (T)1 + mu * (a - (T)1);
    T U, dUdr, dUda;
    if (r < rmin) {
        const T q = (rmin * rinv) * (rmin * rinv);
        U = eps * (q * q - (T)2 * q) + ((T)1 - phi) * eps;
        dUdr = (T)4 * eps * (q - q * q) * rinv;
        dUda = -mu * eps;
    } else {
        T sx, cx;
        const T u = (r - rmin) * (T)P.inv_w;              // (r - r_min) / (r_c - r_min)
        if constexpr (sizeof(T) == 4) {
            // x = (pi/2) u; the hardware sine and cosine take revolutions: x / 2pi = u / 4
            sx = __builtin_amdgcn_sinf((T)0.25 * u);
            cx = __builtin_amdgcn_cosf((T)0.25 * u);
        } else {
            // x = (pi/2) u lies in [0, pi/2): Taylor series of the half angle (terms
            // through h^16; the first omitted one is below 1e-16 relative), then the
            // double-angle formulas
            const double h = 0.25 * M_PI * u, h2 = h * h;
            // nested factors 1 - h^2/(k(k+1)), multiplied by compile-time reciprocals
            const double sh = h * (1.0 - h2 * (1.0 / 6.0) * (1.0 - h2 * (1.0 / 20.0) * (1.0 - h2 * (1.0 / 42.0) *
                              (1.0 - h2 * (1.0 / 72.0) * (1.0 - h2 * (1.0 / 110.0) * (1.0 - h2 * (1.0 / 156.0) *
                              (1.0 - h2 * (1.0 / 210.0))))))));
            const double ch = 1.0 - h2 * 0.5 * (1.0 - h2 * (1.0 / 12.0) * (1.0 - h2 * (1.0 / 30.0) *
                              (1.0 - h2 * (1.0 / 56.0) * (1.0 - h2 * (1.0 / 90.0) * (1.0 - h2 * (1.0 / 132.0) *
                              (1.0 - h2 * (1.0 / 182.0) * (1.0 - h2 * (1.0 / 240.0))))))));
            sx = 2.0 * sh * ch;
            cx = (ch - sh) * (ch + sh);
        }
        const T c2 = cx * cx;
        T cz1;                                            // cos^(2 zeta - 2)
        if (FAST) cz1 = c2 * c2 * c2;
        else cz1 = ipow(c2, P.zeta - 1);
        const T uA = -eps * cz1 * c2;
        U = uA * phi;
        dUdr = phi * (T)P.dudr_k * sx * cz1 * cx;         // phi eps zeta pi / (r_c - r_min) sin x cos^(2 zeta - 1) x
        dUda = mu * uA;
    }
    T gx = -t * nix - s * njx, gy = -t * niy - s * njy, gz = -t * niz - s * njz;
    if (!FAST) {
        gx += st0 * (njx - nix);
        gy += st0 * (njy - niy);
        gz += st0 * (njz - niz);
    }
    const T proj = gx * ex + gy * ey + gz * ez;
    const T k = dUda * rinv;
    fx -= dUdr * ex + k * (gx - proj * ex);
    fy -= dUdr * ey + k * (gy - proj * ey);
    fz -= dUdr * ez + k * (gz - proj * ez);
    // torque on i: n_i x g_i with g_i = -dU/da (n_j - (t + sin th0) e)
    const T bb = t + st0;
    const T wx = -dUda * (njx - bb * ex), wy = -dUda * (njy - bb * ey), wz = -dUda * (njz - bb * ez);
    tx += niy * wz - niz * wy;
    ty += niz * wx - nix * wz;
    tz += nix * wy - niy * wx;
    return U;
}

// WCA for pairs with a protein bead; adds the force on i, returns U.
template <class T>
__device__ __forceinline__ T wca_pair(const DevParams &P, T dx, T dy, T dz, T &fx, T &fy, T &fz) {
    T r2 = dx * dx + dy * dy + dz * dz;
    T r2inv;
    if constexpr (sizeof(T) == 4) r2inv = __builtin_amdgcn_rcpf(r2);
    else r2inv = (T)1 / r2;
    T sr2 = (T)P.wca_sig2 * r2inv;
    T sr6 = sr2 * sr2 * sr2;
    T e = (T)P.wca_eps;
    T U = (T)4 * e * (sr6 * sr6 - sr6) + e;
    T f = (T)24 * e * ((T)2 * sr6 * sr6 - sr6) * r2inv;
    fx += f * dx;
    fy += f * dy;
    fz += f * dz;
    return U;
}

// sqrt(r2) and its reciprocal to within an ulp, from the hardware's approximate
// reciprocal square root by two Goldschmidt steps and a correction of each (10 fused
// multiply-adds; the library's square root and division take about 35 instructions
// with their scaling for subnormal and huge arguments, which squared separations are not).
__device__ __forceinline__ void sqrt_rsqrt(double r2, double &r, double &rinv) {
    const double y = __builtin_amdgcn_rsq(r2);
    double g = r2 * y, h = 0.5 * y;
    const double e = fma(-h, g, 0.5);
    g = fma(g, e, g);
    h = fma(h, e, h);
    r = fma(fma(-g, g, r2), h, g);
    rinv = 2.0 * h;
    rinv = fma(fma(-r, rinv, 1.0), rinv, rinv);
}

// ------------------------------------------------------------------ integrator pieces

// Free linear-rotor drift: n rotated about omega by the angle a = |omega| dt (Rodrigues), then
// renormalised:  n + S omega x n + C (omega (omega.n) - |omega|^2 n)  with S = sin a / |omega|
// and C = (1 - cos a) / |omega|^2, whose series need neither |omega| nor a division.
__device__ __forceinline__ D4 rotor_drift(D4 n, const D4 &w, double dt) {
#pragma clang fp contract(off)
    const double w2 = fma(w.z, w.z, fma(w.y, w.y, w.x * w.x));
    if (w2 > 0.0) {
        const double a2 = w2 * (dt * dt);
        double S, C;
        if (a2 < 0.0025) {
            // Taylor series; the first omitted terms are below 1e-18 relative here
            S = dt * fma(a2, fma(a2, fma(a2, fma(a2, 1.0 / 362880.0, -1.0 / 5040.0), 1.0 / 120.0), -1.0 / 6.0), 1.0);
            C = (dt * dt) * fma(a2, fma(a2, fma(a2, fma(a2, 1.0 / 3628800.0, -1.0 / 40320.0), 1.0 / 720.0), -1.0 / 24.0), 0.5);
        } else {
            const double wn = sqrt(w2);
            double sn, cs;
            sincos(wn * dt, &sn, &cs);
            S = sn / wn;
            C = (1.0 - cs) / w2;
        }
        const double kn = fma(w.z, n.z, fma(w.y, n.y, w.x * n.x));
        const double cx = fma(w.y, n.z, -(w.z * n.y)), cy = fma(w.z, n.x, -(w.x * n.z)), cz = fma(w.x, n.y, -(w.y * n.x));
        n = D4{fma(S, cx, fma(C, fma(w.x, kn, -(w2 * n.x)), n.x)), fma(S, cy, fma(C, fma(w.y, kn, -(w2 * n.y)), n.y)),
               fma(S, cz, fma(C, fma(w.z, kn, -(w2 * n.z)), n.z)), n.w};
    }
    const double nn2 = fma(n.z, n.z, fma(n.y, n.y, n.x * n.x));
    if (nn2 > 0.0) {
        double r, in;
        sqrt_rsqrt(nn2, r, in);
        n.x *= in; n.y *= in; n.z *= in;
    }
    return n;
}

// Half-kick v += h a, drift x += dt v, and the drift's statistics.  Every
// operation is rounded on its own (no contraction), so the drift fused into the
// force kernel and the standalone kick-drift give the same bits.
__device__ __forceinline__ void half_kick(D4 &v, double h, double ax, double ay, double az) {
#pragma clang fp contract(off)
    v.x += h * ax;
    v.y += h * ay;
    v.z += h * az;
}

__device__ __forceinline__ void drift_pos(D4 &x, const D4 &v, double dt) {
#pragma clang fp contract(off)
    x.x += dt * v.x;
    x.y += dt * v.y;
    x.z += dt * v.z;
}

// Displacements since the last list build and since the last prune, measured
// against FP32 copies of the reference positions (their rounding, below 6e-5 sigma for
// coordinates under 1000 sigma, is covered by the runtime's margins).
__device__ __forceinline__ void drift_measures(const D4 &x, const D4 &v, const F3 &b, const F3 &p, double &disp2,
                                               double &disp2p, double &v2, bool &bad) {
#pragma clang fp contract(off)
    const double ddx = x.x - (double)b.x, ddy = x.y - (double)b.y, ddz = x.z - (double)b.z;
    disp2 = ddx * ddx + ddy * ddy + ddz * ddz;
    const double dpx = x.x - (double)p.x, dpy = x.y - (double)p.y, dpz = x.z - (double)p.z;
    disp2p = dpx * dpx + dpy * dpy + dpz * dpz;
    v2 = v.x * v.x + v.y * v.y + v.z * v.z;
    bad = !isfinite(x.x + x.y + x.z + v.x + v.y + v.z);
}

// The volume's lipid sums of one particle (x.n, x, n, 1; zero for proteins) and
// their per-chunk totals, a fixed butterfly over the wavefront stored
// component-major at vpart[q * nchunk + chunk].  The drift computes them for the
// positions it writes, so the next force evaluation needs only the reduction.
__device__ __forceinline__ void volume_terms(const D4 &x, const D4 &n, double v[8]) {
#pragma clang fp contract(off)
    v[0] = x.x * n.x + x.y * n.y + x.z * n.z;
    v[1] = x.x; v[2] = x.y; v[3] = x.z;
    v[4] = n.x; v[5] = n.y; v[6] = n.z;
    v[7] = 1.0;
}

// Wavefront sum of a double by DPP lane moves in a fixed order (no LDS traffic):
// a Hillis-Steele scan within each 16-lane row (shifts 1, 2, 4, 8), then row 0's
// total into row 1 and row 2's into row 3 (row_bcast:15), then the first half's
// total into rows 2 and 3 (row_bcast:31).  Lane 63 ends with the total.
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_add(double v) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, ROWS, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, ROWS, 0xf, false);
    return v + __hiloint2double(hi, lo);
}

__device__ __forceinline__ double wave_total_lane63(double v) {
    v = dpp_add<0x111, 0xf>(v);     // row_shr:1
    v = dpp_add<0x112, 0xf>(v);     // row_shr:2
    v = dpp_add<0x114, 0xf>(v);     // row_shr:4
    v = dpp_add<0x118, 0xf>(v);     // row_shr:8
    v = dpp_add<0x142, 0xa>(v);     // row_bcast:15 into rows 1 and 3
    v = dpp_add<0x143, 0xc>(v);     // row_bcast:31 into rows 2 and 3
    return v;
}

// The same scan taking maxima, for non-negative values (lanes without a source
// contribute 0).  Lane 63 ends with the largest value.
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_max(double v) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, ROWS, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, ROWS, 0xf, false);
    return fmax(v, __hiloint2double(hi, lo));
}

__device__ __forceinline__ double wave_max_lane63(double v) {
    v = dpp_max<0x111, 0xf>(v);
    v = dpp_max<0x112, 0xf>(v);
    v = dpp_max<0x114, 0xf>(v);
    v = dpp_max<0x118, 0xf>(v);
    v = dpp_max<0x142, 0xa>(v);
    v = dpp_max<0x143, 0xc>(v);
    return v;
}

__device__ __forceinline__ void volume_chunk_store(const SysDev &S, int chunk, double v[8]) {
    for (int q = 0; q < 8; ++q) v[q] = wave_total_lane63(v[q]);
    if ((threadIdx.x & (WAVE - 1)) == WAVE - 1)
        for (int q = 0; q < 8; ++q) S.vpart[(size_t)q * S.nchunk + chunk] = v[q];
}

// Velocity quenching: keep the part of a along b when it points along b,
// a <- max(a.b, 0) b / |b|^2; and scale a so that |a| dt <= m.  No contraction,
// as for the kicks.
__device__ __forceinline__ void project_along(D4 &a, double bx, double by, double bz) {
#pragma clang fp contract(off)
    const double bb = bx * bx + by * by + bz * bz;
    const double ab = a.x * bx + a.y * by + a.z * bz;
    if (bb > 0.0 && ab > 0.0) {
        const double s = ab / bb;
        a.x = s * bx; a.y = s * by; a.z = s * bz;
    } else {
        a.x = 0.0; a.y = 0.0; a.z = 0.0;
    }
}

__device__ __forceinline__ void cap_move(D4 &a, double dt, double m) {
#pragma clang fp contract(off)
    const double s = sqrt(a.x * a.x + a.y * a.y + a.z * a.z) * dt;
    if (s > m) {
        const double f = m / s;
        a.x *= f; a.y *= f; a.z *= f;
    }
}

// Philox4x32-10 (Salmon, Moraes, Dror and Shaw, SC'11): ten rounds of two 32 x 32
// -> 64-bit products mixed with the other words and the key, which advances by
// the Weyl constants between rounds.
__device__ __forceinline__ void philox10(uint32_t &c0, uint32_t &c1, uint32_t &c2, uint32_t &c3, uint32_t k0,
                                         uint32_t k1) {
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const uint32_t hi0 = __umulhi(0xD2511F53u, c0), lo0 = 0xD2511F53u * c0;
        const uint32_t hi1 = __umulhi(0xCD9E8D57u, c2), lo1 = 0xCD9E8D57u * c2;
        c0 = hi1 ^ c1 ^ k0;
        c1 = lo1;
        c2 = hi0 ^ c3 ^ k1;
        c3 = lo0;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
}

// Thermostat update of one particle after its closing half-kick: the exact
// Ornstein-Uhlenbeck step v <- c v + sqrt((1 - c^2) kT / m) xi, xi uniform with unit
// variance from the Philox words of counter (caller id, step, 0); lipids also
// w <- c_r w + sqrt((1 - c_r^2) kT / I) (xi' - (xi'.n) n) from counter (.., 1).
// Every operation is rounded on its own (no contraction): the fused and the
// stored-then-reloaded step paths then agree bit for bit.
__device__ __forceinline__ void langevin_update(const DevParams &P, int gid, unsigned long long step, int t,
                                                const D4 &n, D4 &v, D4 &w) {
#pragma clang fp contract(off)
    const uint32_t s_lo = (uint32_t)step, s_hi = (uint32_t)(step >> 32);
    constexpr double half = 2147483647.5;   // (2^32 - 1) / 2: centres the words
    {
        uint32_t c0 = (uint32_t)gid, c1 = s_lo, c2 = s_hi, c3 = 0u;
        philox10(c0, c1, c2, c3, P.seed_lo, P.seed_hi);
        const double a = P.ou_a[t];
        v.x = P.ou_c * v.x + a * ((double)c0 - half);
        v.y = P.ou_c * v.y + a * ((double)c1 - half);
        v.z = P.ou_c * v.z + a * ((double)c2 - half);
    }
    if (t == 0) {
        uint32_t c0 = (uint32_t)gid, c1 = s_lo, c2 = s_hi, c3 = 1u;
        philox10(c0, c1, c2, c3, P.seed_lo, P.seed_hi);
        const double xx = (double)c0 - half, xy = (double)c1 - half, xz = (double)c2 - half;
        const double pn = xx * n.x + xy * n.y + xz * n.z;
        w.x = P.ou_cr * w.x + P.ou_ar * (xx - pn * n.x);
        w.y = P.ou_cr * w.y + P.ou_ar * (xy - pn * n.y);
        w.z = P.ou_cr * w.z + P.ou_ar * (xz - pn * n.z);
    }
}

// The volume's lipid sums of the whole system from their first-level reduction (VR1 partials
// of eight sums), one partial per thread of a 256-thread block: a fixed tree over the 32
// lanes of each sum.  The totals arrive in `tot` (LDS) with the next barrier.
constexpr int VR1 = 32;
__device__ __forceinline__ void volume_totals(double part, double *tot) {
    static_assert(VR1 == 32 && 8 * VR1 == BLOCK, "a partial per thread, 32 lanes per sum");
    part = dpp_add<0x111, 0xf>(part);
    part = dpp_add<0x112, 0xf>(part);
    part = dpp_add<0x114, 0xf>(part);
    part = dpp_add<0x118, 0xf>(part);
    part = dpp_add<0x142, 0xa>(part);
    if ((threadIdx.x & 31) == 31) tot[threadIdx.x >> 5] = part;
}
__device__ __forceinline__ double volume_partial(const SysDev &S) {
    return ldg(S.vred + (threadIdx.x & 31) * 8 + (threadIdx.x >> 5));
}

// V = a_L/3 (sum x.n - (sum x).(sum n) / N_L), U_V = k_V/2 (V - V0)^2 / V0 and the force
// constant dU_V/dV a_L/3.  V0 is the given target, else the first V (vol0, 0 before it).
struct Volume {
    double V, V0, kap, U, xbar[3], nbar[3];
};
__device__ __forceinline__ Volume volume_of(const DevParams &P, const double *t, double vol0) {
#pragma clang fp contract(off)
    Volume r{0.0, vol0, 0.0, 0.0, {0.0, 0.0, 0.0}, {0.0, 0.0, 0.0}};
    const double cnt = t[7];
    if (cnt == 0.0) return r;
    const double inv = 1.0 / cnt;
    r.V = P.vol_a3 * (t[0] - (t[1] * t[4] + t[2] * t[5] + t[3] * t[6]) * inv);
    for (int a = 0; a < 3; ++a) { r.xbar[a] = t[1 + a] * inv; r.nbar[a] = t[4 + a] * inv; }
    if (vol0 == 0.0) r.V0 = P.vol_target > 0.0 ? P.vol_target : r.V;
    if (P.vol_on && r.V0 > 0.0) {
        const double dv = (r.V - r.V0) / r.V0;
        r.kap = P.vol_k * dv * P.vol_a3;
        r.U = 0.5 * P.vol_k * (r.V - r.V0) * dv;
    }
    return r;
}

// Volume term on a lipid: F -= kap (n - nbar), tau += n x (-kap (x - xbar)), each
// operation rounded on its own (the same bits in every kernel variant).
__device__ __forceinline__ void volume_term(const Volume &c, const D4 &x, const D4 &n, double &Fx, double &Fy,
                                            double &Fz, D4 &Tq) {
#pragma clang fp contract(off)
    const double kap = c.kap;
    Fx -= kap * (n.x - c.nbar[0]);
    Fy -= kap * (n.y - c.nbar[1]);
    Fz -= kap * (n.z - c.nbar[2]);
    const double gx = -kap * (x.x - c.xbar[0]), gy = -kap * (x.y - c.xbar[1]), gz = -kap * (x.z - c.xbar[2]);
    Tq.x += n.y * gz - n.z * gy;
    Tq.y += n.z * gx - n.x * gz;
    Tq.z += n.x * gy - n.y * gx;
}

// Per-wavefront drift statistics: the largest |x - x_build|^2, |v|^2 and
// |x - x_prune|^2 of the wave's particles (chunk w of the particle block) go to the
// block's partial slots 3w, 3w+1 and 3w+2 in `out`; a non-finite state raises the
// system's error bit.
__device__ __forceinline__ void drift_stats(const SysDev &S, double *out, int blk, int w, double disp2, double v2,
                                            double disp2p, bool bad) {
    disp2 = wave_max_lane63(disp2);
    v2 = wave_max_lane63(v2);
    disp2p = wave_max_lane63(disp2p);
    const unsigned long long anybad = __ballot(bad);
    if (lane_id_f() == WAVE - 1) {
        out[(size_t)blk * BRED + 3 * w] = disp2;
        out[(size_t)blk * BRED + 3 * w + 1] = v2;
        out[(size_t)blk * BRED + 3 * w + 2] = disp2p;
        if (anybad) atomicOr(&S.sc->err, ERR_NONFINITE);
    }
}

// The statistics of one system's last drift, from the per-wavefront partials (three per
// 64-particle chunk), published to the host ring by one block: the largest displacements
// and speed, the error bits, and a tag of the drift's number and these words.  The step
// kernel runs one such block per system beside the blocks of the next step, so that no
// kernel of its own (6 us on any system, 8 us at 4M particles, and the gap before it) and
// no counting of finished blocks (about 4 us at the end of a small system's step) stands
// between two steps.
__device__ void stats_of(const double *part, int n, double *s_m) {       // into s_m[0..2], for thread 0
    constexpr int U = 8;                              // chunks per thread in flight
    const int nb = blockDim.x, lane = threadIdx.x & (WAVE - 1), w = threadIdx.x / WAVE;
    double d = 0.0, v = 0.0, dp = 0.0;
    for (int c0 = threadIdx.x; c0 < n; c0 += U * nb) {
        double a[U][3];
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const double *r = part + 3 * (size_t)min(c0 + k * nb, n - 1);    // (a chunk twice changes no maximum)
            a[k][0] = ldg(r);
            a[k][1] = ldg(r + 1);
            a[k][2] = ldg(r + 2);
        }
#pragma unroll
        for (int k = 0; k < U; ++k) {
            d = fmax(d, a[k][0]);
            v = fmax(v, a[k][1]);
            dp = fmax(dp, a[k][2]);
        }
    }
    d = wave_max_lane63(d);
    v = wave_max_lane63(v);
    dp = wave_max_lane63(dp);
    if (lane == WAVE - 1) {
        s_m[3 * w] = d;
        s_m[3 * w + 1] = v;
        s_m[3 * w + 2] = dp;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int q = 1; q < nb / WAVE; ++q) {
            s_m[0] = fmax(s_m[0], s_m[3 * q]);
            s_m[1] = fmax(s_m[1], s_m[3 * q + 1]);
            s_m[2] = fmax(s_m[2], s_m[3 * q + 2]);
        }
    }
}

__device__ void publish_stats(const SysDev &S, const double *part, int n, unsigned long long step, double *s_m,
                              unsigned long long with) {
    stats_of(part, n, s_m);
    if (threadIdx.x == 0) {
        StepStat *e = S.hstat + (step - 1) % STAT_RING;
        const unsigned long long err = (unsigned long long)(unsigned)S.sc->err | (unsigned long long)S.sc->level << STAT_LEVEL | with;
        const unsigned long long d2 = dbits(s_m[0]), v2 = dbits(s_m[1]), d2p = dbits(s_m[2]);
        auto put = [](void *p, unsigned long long v) {
            __hip_atomic_store((unsigned long long *)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        };
        put(&e->d2, d2);
        put(&e->v2, v2);
        put(&e->d2p, d2p);
        put(&e->err, err);
        put(&e->tag, stat_tag(step, d2, v2, d2p, err));
    }
}

// ------------------------------------------------------------------ force kernel

// Branch-free FP32 lipid-lipid law for the mixed-precision step kernel, on the
// separation (dx, dy, dz) = x_i - x_j with r2 = |d|^2 > 0.  Both radial branches are
// evaluated and selected (the repulsive core below r_min, the cos^(2 zeta) well above
// it); `on` masks the pair out (every coefficient and U zero) without a branch.
// With g = -t n_i - s n_j + sin(th0) (n_j - n_i) and k = dU/da / r, the force on i is
// -[(dU/dr - k g.e) e + k g], where g.e = -2 s t + sin(th0) (t - s), and the torque on i
// is n_i x g_i with g_i = -dU/da (n_j - (t + sin th0) e).  Both are returned as
// coefficients, so that the caller sums the terms along n_i, and forms the torque's
// cross product with n_i, once per particle instead of once per pair:
//   force on i  = -(A e + bi n_i + bj n_j),    g_i = cn n_j + ce e.
// Returns U; (ex, ey, ez) is the unit separation.
template <bool FAST>
__device__ __forceinline__ float lipid_coef(const DevParams &P, float dx, float dy, float dz, float r2, float nix,
                                            float niy, float niz, float njx, float njy, float njz, bool on,
                                            float &ex, float &ey, float &ez, float &A, float &bi, float &bj,
                                            float &cn, float &ce) {
    const float eps = (float)P.eps, mu = (float)P.mu, rmin = (float)P.r_min;
    const float st0 = FAST ? 0.0f : (float)P.st0;
    const float rinv = __builtin_amdgcn_rsqf(r2);
    const float r = r2 * rinv;
    ex = dx * rinv;
    ey = dy * rinv;
    ez = dz * rinv;
    const float s = nix * ex + niy * ey + niz * ez;
    const float t = njx * ex + njy * ey + njz * ez;
    const float c = nix * njx + niy * njy + niz * njz;
    float a = c - s * t;
    if (!FAST) a += st0 * (t - s) - st0 * st0;
    const float phi = mu * a + (1.0f - mu);
    // repulsive core, r < r_min: U = eps (q^2 - 2 q) + (1 - phi) eps with q = (r_min / r)^2
    const float q = (rmin * rmin) * (rinv * rinv);
    const float dUdrR = (4.0f * eps) * ((q - q * q) * rinv);
    const float dUdaR = -mu * eps;
    // attractive well, r_min <= r < r_c: x = (pi/2) u with u clamped to [0, 1]; the
    // hardware sine and cosine take revolutions, x / 2pi = u / 4
    const float w4 = 0.25f * (float)P.inv_w;
    const float arg = __builtin_amdgcn_fmed3f(r * w4 - rmin * w4, 0.0f, 0.25f);
    const float sx = __builtin_amdgcn_sinf(arg);
    const float cx = __builtin_amdgcn_cosf(arg);
    const float c2 = cx * cx;
    float cz1;                                           // cos^(2 zeta - 2)
    if (FAST) cz1 = (c2 * c2) * c2;
    else cz1 = ipow(c2, P.zeta - 1);
    const float c2z = cz1 * c2;                          // cos^(2 zeta)
    const float dUdrA = (phi * (float)P.dudr_k) * ((sx * cx) * cz1);
    const float dUdaA = (-mu * eps) * c2z;
    const bool rep = r < rmin;
    float dUdr = rep ? dUdrR : dUdrA;
    float dUda = rep ? dUdaR : dUdaA;
    float U = rep ? (eps * (q * q - 2.0f * q) + (1.0f - phi) * eps) : -eps * c2z * phi;
    dUdr = on ? dUdr : 0.0f;
    dUda = on ? dUda : 0.0f;
    U = on ? U : 0.0f;
    const float k = dUda * rinv;
    const float kt = k * t, ks = k * s;
    float ge2 = 2.0f * kt * s;                           // -k g.e
    if (!FAST) ge2 -= k * st0 * (t - s);
    A = dUdr + ge2;
    bi = -kt;                                            // k g = bi n_i + bj n_j
    bj = -ks;
    if (!FAST) {
        bi -= k * st0;
        bj += k * st0;
    }
    cn = -dUda;
    ce = dUda * (FAST ? t : t + st0);
    return U;
}

// The lipid-lipid law of the FP64 step kernel in the same coefficient form,
//   force on i  = -(A e + bi n_i + bj n_j),    g_i = cn n_j + ce e,
// for a pair in range.  Both radial branches are evaluated and selected: a wavefront
// nearly always holds lanes of both.
//  A Horner step a b + c with the coefficient c in scalar registers: the compiler's own form
// adds into a copy of it, which costs a move per step and registers to keep the coefficients
// (15 moves and 22 registers per row).
__device__ __forceinline__ double horner(double a, double b, double c) {
    double r;
    asm("v_fma_f64 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "s"(c));
    return r;
}

template <bool FAST, bool ENERGY>
__device__ __forceinline__ double lipid_coef64(const DevParams &P, double dx, double dy, double dz, double r2, double nix,
                                               double niy, double niz, double njx, double njy, double njz, double &ex,
                                               double &ey, double &ez, double &A, double &bi, double &bj, double &cn,
                                               double &ce) {
    const double eps = P.eps, mu = P.mu, rmin = P.r_min, st0 = FAST ? 0.0 : P.st0;
    double r, rinv;
    sqrt_rsqrt(r2, r, rinv);
    ex = dx * rinv;
    ey = dy * rinv;
    ez = dz * rinv;
    const double s = nix * ex + niy * ey + niz * ez;
    const double t = njx * ex + njy * ey + njz * ez;
    const double c = nix * njx + niy * njy + niz * njz;
    double a = c - s * t;
    if (!FAST) a += st0 * (t - s) - st0 * st0;
    const double phi = fma(mu, a, 1.0 - mu);
    // repulsive core
    const double q = (rmin * rinv) * (rmin * rinv);
    const double dUdrR = (4.0 * eps) * ((q - q * q) * rinv);
    // attractive well: x = (pi/2) u = 2 h with h in [0, pi/4], Taylor series of sin h / h and
    // cos h (terms through h^14 and h^16; the first omitted ones are below 1e-16), then the
    // double angle; a core lane's h is a small negative number and its result unused
    const double h = (0.25 * M_PI * P.inv_w) * (r - rmin), h2 = h * h;
    double sp = -1.0 / 1307674368000.0;
    sp = horner(sp, h2, 1.0 / 6227020800.0);
    sp = horner(sp, h2, -1.0 / 39916800.0);
    sp = horner(sp, h2, 1.0 / 362880.0);
    sp = horner(sp, h2, -1.0 / 5040.0);
    sp = horner(sp, h2, 1.0 / 120.0);
    sp = horner(sp, h2, -1.0 / 6.0);
    const double sh = fma(h * h2, sp, h);
    double cp = 1.0 / 20922789888000.0;
    cp = horner(cp, h2, -1.0 / 87178291200.0);
    cp = horner(cp, h2, 1.0 / 479001600.0);
    cp = horner(cp, h2, -1.0 / 3628800.0);
    cp = horner(cp, h2, 1.0 / 40320.0);
    cp = horner(cp, h2, -1.0 / 720.0);
    cp = horner(cp, h2, 1.0 / 24.0);
    cp = horner(cp, h2, -0.5);
    const double ch = fma(cp, h2, 1.0);
    const double sx = 2.0 * sh * ch, cx = (ch - sh) * (ch + sh);
    const double c2 = cx * cx;
    double cz1;                                          // cos^(2 zeta - 2)
    if (FAST) cz1 = (c2 * c2) * c2;
    else cz1 = ipow(c2, P.zeta - 1);
    const double c2z = cz1 * c2;
    const double dUdrA = (phi * P.dudr_k) * ((sx * cx) * cz1);
    const bool rep = r < rmin;
    const double dUdr = rep ? dUdrR : dUdrA;
    const double dUda = rep ? -mu * eps : (-mu * eps) * c2z;
    const double k = dUda * rinv;
    const double kt = k * t, ks = k * s;
    double ge2 = 2.0 * kt * s;                           // -k g.e
    if (!FAST) ge2 -= k * st0 * (t - s);
    A = dUdr + ge2;
    bi = -kt;
    bj = -ks;
    if (!FAST) {
        bi -= k * st0;
        bj += k * st0;
    }
    cn = -dUda;
    ce = dUda * (FAST ? t : t + st0);
    if (!ENERGY) return 0.0;
    return rep ? eps * (q * q - 2.0 * q) + (1.0 - phi) * eps : -eps * c2z * phi;
}

// LDS stage per 256-particle block, in 16-byte records at the offsets that the lists hold:
// FP64 positions, and either FP32 orientations with the type in w (mixed) or FP64
// orientations and a type byte.  The stage is the block's pruned partner set; entries
// beyond the LDS part (rare) are read from global memory (1600 entries in LDS instead of
// 800 made no difference to FP64 mode).  One more entry is a sentinel that list padding
// points to and that passes no test: its x is NaN (FP64), or it lies at finite far
// coordinates (mixed, whose branch-free rows would spread a NaN) with a NaN kind (FAST) or a
// padding type.  On periodic axes the wrap may bring it back into range, so those systems
// also test its type and give masked rows a separation that is not zero.
template <int MIXED>
struct Stage {
    static constexpr int lds = MIXED ? 640 : 800;
    static constexpr int ext = lds + 1;                  // LDS entries, with the sentinel
    static constexpr int bytes = MIXED ? ext * (3 * 8 + 16) : ext * (6 * 8 + 1);
};
static_assert(Stage<1>::lds < SMAX, "lists reach beyond the LDS part");
constexpr double SENTINEL = 1.0e8;    // sigma: the padding entry's coordinates (finite FP32 squares)
constexpr int PAD_TYPE = 3;           // the padding entry's type (a periodic wrap may bring it into range)
struct alignas(16) D2 {
    double x, y;
};

// One workgroup per 256 consecutive cell-sorted particles.  The block's pruned
// partners (its stage) are read once from HBM into LDS; lane i then walks column i of
// its chunk's pruned list of stage indices.
//  - Mixed mode: each row is evaluated without branches, two rows per trip.  The
//    FP64-formed separation is rounded to FP32 and its FP32 square decides the
//    neighbour test where it lies clear of the cutoff (beyond the FP32 rounding of the
//    square, a relative 4e-7 at most); in the band between, which a wavefront rarely
//    meets, the exact FP64 test of the neighbour-set definition decides.  The pair
//    law then runs in FP32.
//  - FP64 mode: every entry takes the exact FP64 test; the pair law runs in FP64.
// What bounds it on systems that fill the GPU: vector instructions (mixed: 151 per pair of
// rows and about 2,650 per wavefront, three quarters of the issue cycles of a 4M-particle
// launch; FP64: 209 per pair of rows) and, in mixed mode, memory traffic at three quarters of
// a plain copy's rate; on small systems one wavefront's latency: a chain of descriptor, entry
// and record loads, a quarter of the rows, the sums of the four wavefronts and the epilogue.
// At 4M particles 400 us mixed and 512 FP64 (439 and 677 with the bounds selected by type,
// checks per entry, spilled orientations, coefficients copied per row and FP32 copies of the
// orientations kept beside the FP64 ones: 32 bytes per particle and step); at 125k FP64 27.2
// us (31.8 before its rows were rewritten), at 2,704 13.0 mixed (15.6) and 13.4 FP64.  Six
// wavefronts per SIMD (80 registers, spills) ran 5 to 12% slower than five; loading the first
// rows and the epilogue's state before the barriers 2 to 4% slower.
// KICK: 0 stores F and tau; 1 also applies the closing half-kick of the step;
// 2 applies the closing half-kick and then, with the same force, the opening
// half-kick and drift of the next step (positions and orientations go to the
// second buffers, which the other descriptor table holds as the current ones),
// without storing F, tau.  With KICK, the grid's first blocks (one per system)
// publish the statistics of the drift that led to this step's positions.
template <int MIXED, int ENERGY, int KICK, int FAST>
__global__ __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(MIXED ? 5 : 4))) void k_force(const SysDev *Sd, Maps L_maps, DevParams P, double dt, int par) {
    using T = typename std::conditional<MIXED, float, double>::type;
    constexpr int SL = Stage<MIXED>::lds;
    constexpr int SX = Stage<MIXED>::ext;
    __shared__ __align__(16) unsigned char s_raw[Stage<MIXED>::bytes];
    __shared__ double s_vol[8];                                   // the volume's lipid sums
    // mixed: records of x, y; of orientation and type; z
    D2 *s_xy = reinterpret_cast<D2 *>(s_raw);
    F4 *s_n4 = reinterpret_cast<F4 *>(s_xy + SX);
    double *s_zm = reinterpret_cast<double *>(s_n4 + SX);
    // FP64: records of x, y; of z, n_x; of n_y, n_z; type
    D2 *s_zn = s_xy + SX, *s_nn = s_zn + SX;
    unsigned char *s_t = reinterpret_cast<unsigned char *>(s_nn + SX);
    const int nstat = KICK ? L_maps.nsys : 0;
    if (KICK && (int)blockIdx.x < nstat) {
        const SysDev &S = Sd[blockIdx.x];
        if (S.n <= 0) return;
        const unsigned long long step = S.sc->step[par];
        if (KICK == 2 && threadIdx.x == 0) S.sc->step[par ^ 1] = step + 1;       // the fused drift's number
        publish_stats(S, S.bred, S.nchunk, step, reinterpret_cast<double *>(s_raw), STAT_FORCE);
        return;
    }
    const int gb = xcd_group_block((int)blockIdx.x - nstat, (int)gridDim.x - nstat);
    const int s = find_sys(L_maps.f, L_maps.nsys, gb);
    const SysDev &S = Sd[s];
    const int fb = gb - L_maps.f[s];
    // a split system's particle block runs as four blocks, one per chunk, whose four
    // waves take every fourth row of that chunk (block-uniform)
    const bool split = S.split != 0;
    const int lb = split ? fb >> 2 : fb;
    const int tid = threadIdx.x;
    const int lane = tid & (WAVE - 1);
    const int csub = split ? (fb & 3) : (tid >> 6);   // the chunk within the particle block
    const int chunk = lb * (BLOCK / WAVE) + csub;
    const int i = lb * BLOCK + csub * WAVE + lane;
    const bool valid = i < S.n;
    const int scnt = __builtin_amdgcn_readfirstlane(S.iscount[lb]);
    const int nlds = min(scnt, SL);                 // stage entries held in LDS
    const double vpart = P.vol_on ? volume_partial(S) : 0.0;
    auto narrow = [](const V3 &n) { return F4{(float)n.x, (float)n.y, (float)n.z, 0.0f}; };
    // this lane's own particle, loaded while the stage is read
    const int traw = valid ? ldg(S.typ + i) : 0;
    const D4 pi = valid ? ld3(S.pos + i) : D4{0.0, 0.0, 0.0, 0.0};
    // (mixed mode's rows take the orientation in FP32; the FP64 one would be spilled over them
    // and is read again in the epilogue)
    D4 ni = {0.0, 0.0, 0.0, 0.0};
    F4 ni32 = {0.0f, 0.0f, 0.0f, 0.0f};
    if (valid) {
        if constexpr (MIXED) ni32 = narrow(ldg(S.ori + i));
        else ni = ld3(S.ori + i);
    }
    // mixed records carry the type's bits; FAST rows take 0 for a lipid and 1 for a protein (and
    // NaN, which passes no test, for the sentinel)
    auto with_kind = [](F4 n, int type) {
        n.w = FAST ? (type == 0 ? 0.0f : 1.0f) : __int_as_float(type);
        return n;
    };
    // the stage: every thread's (at most three) slots first, then their records
    constexpr int SPT = (SL + BLOCK - 1) / BLOCK;
    for (int q0 = tid; q0 < nlds; q0 += SPT * BLOCK) {
        int32_t ent[SPT];
#pragma unroll
        for (int k = 0; k < SPT; ++k) {
            const int q = q0 + k * BLOCK;
            ent[k] = q < nlds ? ldg(S.istage + (size_t)lb * SSTRIDE + q) : -1;
        }
#pragma unroll
        for (int k = 0; k < SPT; ++k) {
            const int q = q0 + k * BLOCK;
            if (ent[k] < 0) break;
            const V3 p = ldg(S.pos + stage_slot(ent[k]));
            const V3 o = ldg(S.ori + stage_slot(ent[k]));
            s_xy[q] = D2{p.x, p.y};
            if constexpr (MIXED) {
                s_zm[q] = p.z;
                s_n4[q] = with_kind(narrow(o), stage_type(ent[k]));
            } else {
                s_zn[q] = D2{p.z, o.x};
                s_nn[q] = D2{o.y, o.z};
                s_t[q] = (unsigned char)stage_type(ent[k]);
            }
        }
    }
    if (!MIXED && tid == 0) {                        // a separation that passes no test
        s_xy[SL] = D2{__builtin_nan(""), 0.0};
        s_zn[SL] = D2{0.0, 0.0};
        s_nn[SL] = D2{0.0, 0.0};
        s_t[SL] = 0;
    }
    if (MIXED && tid == 0) {
        s_xy[SL] = D2{SENTINEL, SENTINEL};
        s_zm[SL] = SENTINEL;
        s_n4[SL] = F4{0.0f, 0.0f, 1.0f, FAST ? __builtin_nanf("") : __int_as_float(PAD_TYPE)};
    }
    // (each block sums the 32 partials for itself: a launch between the steps took 6 us)
    if (P.vol_on) volume_totals(vpart, s_vol);
    __syncthreads();
    if (chunk >= S.nchunk) return;
    const int ti = traw & TYP_MASK;
    const T nix = MIXED ? (T)ni32.x : (T)ni.x, niy = MIXED ? (T)ni32.y : (T)ni.y, niz = MIXED ? (T)ni32.z : (T)ni.z;
    T fx = 0, fy = 0, fz = 0, tx = 0, ty = 0, tz = 0;
    double U = 0.0, W = 0.0;
    const int rows = __builtin_amdgcn_readfirstlane(min(S.ilk[chunk], MAXNB));   // wave-uniform
    // cutoff row of this particle's type, selected by the partner's type without
    // dynamic indexing; the periodic min-image only where the system has periodic axes
    const double rcA = ti == 0 ? P.rc2[0][0] : (ti == 1 ? P.rc2[1][0] : P.rc2[2][0]);
    const double rcB = ti == 0 ? P.rc2[0][1] : (ti == 1 ? P.rc2[1][1] : P.rc2[2][1]);
    const double rcC = ti == 0 ? P.rc2[0][2] : (ti == 1 ? P.rc2[1][2] : P.rc2[2][2]);
    const bool periodic = (S.per[0] | S.per[1] | S.per[2]) != 0;
    const double iLx = S.per[0] ? 1.0 / S.box[0] : 0.0, iLy = S.per[1] ? 1.0 / S.box[1] : 0.0,
                 iLz = S.per[2] ? 1.0 / S.box[2] : 0.0;

    // ---- mixed mode: branch-free rows, two per trip
    auto mixed_rows = [&](auto per_tag, auto part_tag, auto split_tag) {
        constexpr bool PER = decltype(per_tag)::value;
        constexpr bool PARTIAL = decltype(part_tag)::value;   // stage entries beyond the LDS part
        constexpr bool SPLIT = decltype(split_tag)::value;    // the four waves take every fourth pair of rows
        constexpr int UNR = 2;          // rows per trip (consecutive), evaluated side by side
        // The pruned lists are padded with 0xffff to an even row count in every lane, so
        // both rows of a trip are always valid entries or padding.
        const int npair = (rows + 1) >> 1;
        constexpr int tstride = SPLIT ? BLOCK / WAVE : 1;
        const int p0 = SPLIT ? tid >> 6 : 0;
        const unsigned *col = reinterpret_cast<const unsigned *>(S.il16 + (size_t)chunk * MAXNB * CHUNK) + p0 * CHUNK + lane;
        const int ntrip = npair > p0 ? (npair - p0 + tstride - 1) / tstride : 0;
        // this particle's row of the FP32 bounds, chosen by selects (no dynamic indexing
        // of the parameter block, which would go through scratch memory)
        auto row_of = [&](const float (&m)[3][3], int b) {
            return ti == 0 ? m[0][b] : (ti == 1 ? m[1][b] : m[2][b]);
        };
        const float loA = row_of(P.rc2lo, 0), loB = row_of(P.rc2lo, 1), loC = row_of(P.rc2lo, 2);
        const float hiA = row_of(P.rc2hi, 0), hiB = row_of(P.rc2hi, 1), hiC = row_of(P.rc2hi, 2);
        auto own = [&](const float (&m)[3]) { return ti == 0 ? m[0] : (ti == 1 ? m[1] : m[2]); };
        const float cutd = own(P.cutd), cutlo = own(P.cutlo), cuthi = own(P.cuthi);
        // wavefront masks: the lanes with a particle, and those with a lipid
        const unsigned long long lanes = __ballot(valid), lipids = __ballot(ti == 0);
        struct Rec {
            double x, y, z;
            float nx, ny, nz, w;
        };
        auto fetch = [&](unsigned e) {                  // e: a list entry (16 times the stage index)
            Rec c;
            if constexpr (PARTIAL) {
                const int k = (int)(e >> 4);
                if (k >= nlds && k < scnt) {            // stage entry beyond the LDS part
                    const int32_t ent = ldg(S.istage + (size_t)lb * SSTRIDE + k);
                    const V3 p = ldg(S.pos + stage_slot(ent));
                    const F4 o = with_kind(narrow(ldg(S.ori + stage_slot(ent))), stage_type(ent));
                    c.x = p.x; c.y = p.y; c.z = p.z;
                    c.nx = o.x; c.ny = o.y; c.nz = o.z; c.w = o.w;
                    return c;
                }
            }
            // padding -> the sentinel (every entry below the LDS part when not PARTIAL)
            const unsigned q = PARTIAL ? (e < 16u * (unsigned)nlds ? e : 16u * SL) : min(e, 16u * SL);
            const D2 xy = *reinterpret_cast<const D2 *>(s_raw + q);
            const F4 nj = *reinterpret_cast<const F4 *>(s_raw + 16 * SX + q);
            c.x = xy.x; c.y = xy.y;
            c.z = *reinterpret_cast<const double *>(s_raw + 32 * SX + (q >> 1));
            c.nx = nj.x; c.ny = nj.y; c.nz = nj.z; c.w = nj.w;
            return c;
        };
        // Software pipeline: the list entries of the next trip are loaded from global
        // memory while this trip's rows are evaluated (the lists carry padding rows past
        // the last chunk, so the load after the last trip stays in bounds).
        float sbi = 0.0f, gx = 0.0f, gy = 0.0f, gz = 0.0f;   // sum of bi; of g_i - cn n_i
        unsigned en = ntrip > 0 ? ldg(col) : 0xffffffffu;    // a pair of rows
        for (int it = 0; it < ntrip; ++it) {
            Rec c[UNR];
            c[0] = fetch(en & 0xffffu);
            c[1] = fetch(en >> 16);
            en = ldg(col + (size_t)(it + 1) * tstride * CHUNK);
            // separations and the neighbour test of every row of the trip
            double dx[UNR], dy[UNR], dz[UNR];
            float fdx[UNR], fdy[UNR], fdz[UNR], r2[UNR];
            // (wavefront masks: scalar registers and instructions beside the vector ones)
            unsigned long long in[UNR], band[UNR], lip[UNR];
            for (int q = 0; q < UNR; ++q) {
                dx[q] = pi.x - c[q].x;
                dy[q] = pi.y - c[q].y;
                dz[q] = pi.z - c[q].z;
                if constexpr (PER) {
                    if (S.per[0]) dx[q] = minimg_fast(dx[q], S.box[0], iLx);
                    if (S.per[1]) dy[q] = minimg_fast(dy[q], S.box[1], iLy);
                    if (S.per[2]) dz[q] = minimg_fast(dz[q], S.box[2], iLz);
                }
                fdx[q] = (float)dx[q];
                fdy[q] = (float)dy[q];
                fdz[q] = (float)dz[q];
                r2[q] = fdx[q] * fdx[q] + fdy[q] * fdy[q] + fdz[q] * fdz[q];
                if constexpr (FAST) {
                    const float r2s = fmaf(c[q].w, cutd, r2[q]);
                    in[q] = __ballot(r2s < cutlo);
                    band[q] = in[q] ^ __ballot(r2s < cuthi);
                    lip[q] = __ballot(c[q].w == 0.0f) & lipids;
                } else {
                    const int tj = __float_as_int(c[q].w);
                    in[q] = __ballot(r2[q] < sel_cutf(tj, loA, loB, loC));
                    band[q] = in[q] ^ __ballot(r2[q] < sel_cutf(tj, hiA, hiB, hiC));
                    lip[q] = __ballot(tj == 0) & lipids;
                    if constexpr (PER) {        // the wrapped sentinel may land anywhere
                        const unsigned long long real = __ballot(tj != PAD_TYPE);
                        in[q] &= real;
                        band[q] &= real;
                    }
                }
            }
            if (__builtin_expect((band[0] | band[1]) != 0ull, 0)) {
#pragma clang fp contract(off)
                // FP32 rounding cannot decide: the exact test of the neighbour-set definition
                for (int q = 0; q < UNR; ++q) {
                    const double d2 = (dx[q] * dx[q] + dy[q] * dy[q]) + dz[q] * dz[q];
                    const double cut = FAST ? (c[q].w == 0.0f ? rcA : rcB) : sel_cut(__float_as_int(c[q].w), rcA, rcB, rcC);
                    in[q] |= band[q] & __ballot(d2 < cut);
                }
            }
            for (int q = 0; q < UNR; ++q) in[q] &= lanes;
            // the pair law of every row, in one block of straight-line code, as coefficients
            float ex[UNR], ey[UNR], ez[UNR], A[UNR], bi[UNR], bj[UNR], cn[UNR], ce[UNR], u[UNR];
            unsigned long long anywca = 0ull;
            for (int q = 0; q < UNR; ++q) {
                const bool on = __builtin_amdgcn_inverse_ballot_w64(in[q] & lip[q]);
                // a masked row needs a root too: the wrapped sentinel may lie on the particle itself
                // (the origin of a box whose length divides the sentinel's coordinate)
                const float rr = PER && !on ? 1.0f : r2[q];
                u[q] = lipid_coef<FAST>(P, fdx[q], fdy[q], fdz[q], rr, nix, niy, niz, c[q].nx, c[q].ny, c[q].nz, on, ex[q],
                                        ey[q], ez[q], A[q], bi[q], bj[q], cn[q], ce[q]);
                anywca |= in[q] & ~lip[q];
            }
            for (int q = 0; q < UNR; ++q) {
                fx = fmaf(-A[q], ex[q], fx);
                fy = fmaf(-A[q], ey[q], fy);
                fz = fmaf(-A[q], ez[q], fz);
                fx = fmaf(-bj[q], c[q].nx, fx);
                fy = fmaf(-bj[q], c[q].ny, fy);
                fz = fmaf(-bj[q], c[q].nz, fz);
                sbi += bi[q];
                // the torque n_i x g_i with g_i = cn n_j + ce e: n_i x n_i = 0, so the sum
                // takes cn (n_j - n_i) + ce e instead, without g_i's large part along n_i
                // (which the FP32 sum would round before the cross product cancels it)
                gx = fmaf(cn[q], c[q].nx - nix, gx);
                gy = fmaf(cn[q], c[q].ny - niy, gy);
                gz = fmaf(cn[q], c[q].nz - niz, gz);
                gx = fmaf(ce[q], ex[q], gx);
                gy = fmaf(ce[q], ey[q], gy);
                gz = fmaf(ce[q], ez[q], gz);
                if (ENERGY) {
                    const float ax = A[q] * ex[q] + bi[q] * nix + bj[q] * c[q].nx;
                    const float ay = A[q] * ey[q] + bi[q] * niy + bj[q] * c[q].ny;
                    const float az = A[q] * ez[q] + bi[q] * niz + bj[q] * c[q].nz;
                    U += 0.5 * (double)u[q];
                    W -= 0.5 * (dx[q] * (double)ax + dy[q] * (double)ay + dz[q] * (double)az);
                }
            }
            if (__builtin_expect(anywca != 0ull, 0)) {
                for (int q = 0; q < UNR; ++q) {
                    const bool wca = __builtin_amdgcn_inverse_ballot_w64(in[q] & ~lip[q]);
                    float bx = 0.0f, by = 0.0f, bz = 0.0f;
                    const float uw = wca_pair<float>(P, wca ? fdx[q] : 2.0f, fdy[q], fdz[q], bx, by, bz);
                    if (wca) {
                        fx += bx;
                        fy += by;
                        fz += bz;
                        if (ENERGY) {
                            U += 0.5 * (double)uw;
                            W += 0.5 * (dx[q] * (double)bx + dy[q] * (double)by + dz[q] * (double)bz);
                        }
                    }
                }
            }
        }
        // the terms along n_i, and the torque n_i x (sum of the g_i - cn n_i)
        fx -= sbi * nix;
        fy -= sbi * niy;
        fz -= sbi * niz;
        tx += niy * gz - niz * gy;
        ty += niz * gx - nix * gz;
        tz += nix * gy - niy * gx;
    };

    // ---- FP64 mode: exact test on every entry, FP64 pair law
    auto fp64_rows = [&](auto per_tag, auto part_tag, auto split_tag) {
        constexpr bool PER = decltype(per_tag)::value;
        constexpr bool PARTIAL = decltype(part_tag)::value;
        constexpr bool SPLIT = decltype(split_tag)::value;
        constexpr int tstride = SPLIT ? BLOCK / WAVE : 1;    // pairs of rows, as in mixed mode
        const int p0 = SPLIT ? tid >> 6 : 0;
        // Software pipeline: the list entries two pairs of rows ahead are fetched from global
        // memory and the stage record of the next row from LDS while a row is evaluated (the
        // lists carry padding rows past the last chunk).
        const unsigned *col = reinterpret_cast<const unsigned *>(S.il16 + (size_t)chunk * MAXNB * CHUNK) + p0 * CHUNK + lane;
        constexpr int cstep = tstride * CHUNK;
        const int npair = (rows + 1) >> 1;
        const int ntrip = npair > p0 ? (npair - p0 + tstride - 1) / tstride : 0;
        unsigned w0 = ldg(col), w1 = ldg(col + cstep);
        const unsigned long long lipids = __ballot(ti == 0);
        struct Rec {
            double x, y, z;
            T nx, ny, nz;
            int t;
        };
        auto fetch = [&](unsigned e) {                  // e: a list entry (16 times the stage index)
            Rec c;
            if constexpr (PARTIAL) {
                const int k = (int)(e >> 4);
                if (k >= nlds && k < scnt) {
                    const int32_t ent = ldg(S.istage + (size_t)lb * SSTRIDE + k);
                    const V3 p = ldg(S.pos + stage_slot(ent));
                    const V3 o = ldg(S.ori + stage_slot(ent));
                    c.x = p.x; c.y = p.y; c.z = p.z;
                    c.nx = o.x; c.ny = o.y; c.nz = o.z;
                    c.t = stage_type(ent);
                    return c;
                }
            }
            // padding -> the sentinel
            const unsigned q = PARTIAL ? (e < 16u * (unsigned)nlds ? e : 16u * SL) : min(e, 16u * SL);
            const D2 xy = *reinterpret_cast<const D2 *>(s_raw + q);
            const D2 zn = *reinterpret_cast<const D2 *>(s_raw + 16 * SX + q);
            const D2 nn = *reinterpret_cast<const D2 *>(s_raw + 32 * SX + q);
            c.x = xy.x; c.y = xy.y; c.z = zn.x;
            c.nx = zn.y; c.ny = nn.x; c.nz = nn.y;
            c.t = s_raw[48 * SX + (q >> 4)];
            return c;
        };
        double sbi = 0.0, gx = 0.0, gy = 0.0, gz = 0.0;       // sum of bi; of g_i - cn n_i
        auto eval = [&](const Rec &c) {
            const int tj = c.t;
            double dx, dy, dz, d2;
            if constexpr (PER) {
                d2 = dist2_exact(S, pi.x, pi.y, pi.z, c.x, c.y, c.z, dx, dy, dz);
            } else {
                d2 = dist2_open(pi.x, pi.y, pi.z, c.x, c.y, c.z, dx, dy, dz);
            }
            // (wavefront masks, as in mixed mode; lanes without a particle hold only padding)
            const unsigned long long in = __ballot(d2 < (FAST ? (tj == 0 ? rcA : rcB) : sel_cut(tj, rcA, rcB, rcC)));
            const unsigned long long lip = __ballot(tj == 0) & lipids, wca = in & ~lip;
            if (__builtin_amdgcn_inverse_ballot_w64(in & lip)) {
                double ex, ey, ez, A, bi, bj, cn, ce;
                const double u = lipid_coef64<FAST, ENERGY>(P, dx, dy, dz, d2, nix, niy, niz, c.nx, c.ny, c.nz, ex, ey, ez,
                                                            A, bi, bj, cn, ce);
                fx = fma(-bj, c.nx, fma(-A, ex, fx));
                fy = fma(-bj, c.ny, fma(-A, ey, fy));
                fz = fma(-bj, c.nz, fma(-A, ez, fz));
                sbi += bi;
                gx = fma(ce, ex, fma(cn, c.nx - nix, gx));
                gy = fma(ce, ey, fma(cn, c.ny - niy, gy));
                gz = fma(ce, ez, fma(cn, c.nz - niz, gz));
                if (ENERGY) {
                    U += 0.5 * u;
                    W -= 0.5 * (dx * (A * ex + bi * nix + bj * c.nx) + dy * (A * ey + bi * niy + bj * c.ny) +
                                dz * (A * ez + bi * niz + bj * c.nz));
                }
            }
            if (__builtin_expect(wca != 0ull, 0)) {
                if (__builtin_amdgcn_inverse_ballot_w64(wca)) {
                    T ax = 0, ay = 0, az = 0;
                    const double u = wca_pair<T>(P, (T)dx, (T)dy, (T)dz, ax, ay, az);
                    fx += ax;
                    fy += ay;
                    fz += az;
                    if (ENERGY) {
                        U += 0.5 * u;
                        W += 0.5 * (dx * ax + dy * ay + dz * az);
                    }
                }
            }
        };
        Rec ra = fetch(w0 & 0xffffu);
        for (int it = 0; it < ntrip; ++it) {
            const Rec rb = fetch(w0 >> 16);
            w0 = w1;
            w1 = ldg(col + (it + 2) * cstep);
            eval(ra);
            ra = fetch(w0 & 0xffffu);
            eval(rb);
        }
        fx -= sbi * nix;
        fy -= sbi * niy;
        fz -= sbi * niz;
        tx += niy * gz - niz * gy;
        ty += niz * gx - nix * gz;
        tz += nix * gy - niy * gx;
    };

    if (scnt >= 0) {
        // block-uniform choices: periodic min-image, whether the stage overflows the LDS
        // part, and the row split, so ordinary blocks carry no per-entry test
        auto dispatch = [&](auto per_tag, auto part_tag) {
            if constexpr (MIXED) {
                if (split) mixed_rows(per_tag, part_tag, std::true_type{});
                else mixed_rows(per_tag, part_tag, std::false_type{});
            } else {
                if (split) fp64_rows(per_tag, part_tag, std::true_type{});
                else fp64_rows(per_tag, part_tag, std::false_type{});
            }
        };
        if (scnt > SL) {
            if (periodic) dispatch(std::true_type{}, std::true_type{});
            else dispatch(std::false_type{}, std::true_type{});
        } else {
            if (periodic) dispatch(std::true_type{}, std::false_type{});
            else dispatch(std::false_type{}, std::false_type{});
        }
    } else {
        // block whose partners did not fit a stage: its (unpruned) lists hold global slots.  A
        // row's records and the entry of the row after it are loaded while the row before is
        // evaluated (each row's entry, position and orientation in turn were three waits).
        const int32_t *col = S.nl + (size_t)chunk * MAXNB * CHUNK + lane;
        const int r0 = split ? (tid >> 6) : 0, rstep = split ? BLOCK / WAVE : 1;
        struct Row {
            D4 p;
            V3 n;
            bool real;
        };
        auto entry = [&](int r) { return valid && r < rows ? ldg(col + r * CHUNK) : -1; };
        auto record = [&](int j) {
            Row c;
            c.real = j >= 0 && j < S.n;
            const int js = c.real ? j : lb * BLOCK;
            c.p = ldpos(S, js);
            c.n = ldg(S.ori + js);
            return c;
        };
        Row nxt = record(entry(r0));
        int jn = entry(r0 + rstep);
        for (int r = r0; r < rows; r += rstep) {
            const Row cur = nxt;
            nxt = record(jn);
            jn = entry(r + 2 * rstep);
            if (!cur.real) continue;
            const D4 pj = cur.p;
            const int tj = (int)pj.w;
            double dx, dy, dz;
            const double d2 = dist2_exact(S, pi.x, pi.y, pi.z, pj.x, pj.y, pj.z, dx, dy, dz);
            if (!(d2 < P.rc2[ti][tj])) continue;
            T ax = 0, ay = 0, az = 0;
            T u;
            if ((ti | tj) == 0) {
                const V3 nj = cur.n;
                u = lipid_pair<T, FAST>(P, (T)dx, (T)dy, (T)dz, nix, niy, niz, (T)nj.x, (T)nj.y, (T)nj.z, ax, ay, az,
                                        tx, ty, tz);
            } else {
                u = wca_pair<T>(P, (T)dx, (T)dy, (T)dz, ax, ay, az);
            }
            fx += ax;
            fy += ay;
            fz += az;
            if (ENERGY) {
                U += 0.5 * (double)u;
                W += 0.5 * (dx * (double)ax + dy * (double)ay + dz * (double)az);
            }
        }
    }
    if (split) {
        // the four waves' partial sums, added in wave order by wave 0, which goes on
        // with the chunk's particles; the stage is free again
        __syncthreads();
        T *red = reinterpret_cast<T *>(s_raw);
        double *redd = reinterpret_cast<double *>(s_raw + 6 * BLOCK * sizeof(T));
        const int wv = tid >> 6;
        const T mine[6] = {fx, fy, fz, tx, ty, tz};
        for (int q = 0; q < 6; ++q) red[q * BLOCK + wv * WAVE + lane] = mine[q];
        if (ENERGY) {
            redd[wv * WAVE + lane] = U;
            redd[BLOCK + wv * WAVE + lane] = W;
        }
        __syncthreads();
        if (wv != 0) return;
        T sum[6];
        for (int q = 0; q < 6; ++q)
            sum[q] = ((red[q * BLOCK + lane] + red[q * BLOCK + WAVE + lane]) + red[q * BLOCK + 2 * WAVE + lane]) +
                     red[q * BLOCK + 3 * WAVE + lane];
        fx = sum[0]; fy = sum[1]; fz = sum[2];
        tx = sum[3]; ty = sum[4]; tz = sum[5];
        if (ENERGY) {
            U = ((redd[lane] + redd[WAVE + lane]) + redd[2 * WAVE + lane]) + redd[3 * WAVE + lane];
            W = ((redd[BLOCK + lane] + redd[BLOCK + WAVE + lane]) + redd[BLOCK + 2 * WAVE + lane]) +
                redd[BLOCK + 3 * WAVE + lane];
        }
    }
    double Fx = (double)fx, Fy = (double)fy, Fz = (double)fz;
    D4 v = {0.0, 0.0, 0.0, 0.0}, w = {0.0, 0.0, 0.0, 0.0};
    double disp2 = 0.0, disp2p = 0.0, vmax2 = 0.0;
    bool bad = false;
    D4 Tq = {(double)tx, (double)ty, (double)tz, 0.0};
    double vsum[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    if (valid) {
        // the own-state loads first, so that they are in flight during the bond lookups
        if constexpr (MIXED) ni = ld3(S.ori + i);
        if (KICK || ENERGY) {
            v = ld3(S.vel + i);
            if (ti == 0) w = ld3(S.angv + i);        // zero for protein beads
        }
        const F3 xb = KICK == 2 ? ldg(S.xb + i) : F3{0.f, 0.f, 0.f};
        const F3 xp = KICK == 2 ? ldg(S.xp + i) : F3{0.f, 0.f, 0.f};
        // bonds of this particle (CSR by caller id), FP64 in both modes; the table is
        // looked up only for particles flagged as bonded
        const bool bonded = (traw & TYP_BONDED) != 0;
        const int g = (bonded || P.thermo_on) ? S.gid[i] : 0;
        const int qb = bonded ? S.bstart[g] : 0, qe = bonded ? S.bstart[g + 1] : 0;
        for (int q = qb; q < qe; ++q) {
            const int j = S.slot[S.bpart[q]];
            const D4 pj = ld3(S.pos + j);
            double dx, dy, dz;
            const double d2 = dist2_exact(S, pi.x, pi.y, pi.z, pj.x, pj.y, pj.z, dx, dy, dz);
            const double r = sqrt(d2);
            const double ext = r - S.br0[q];
            const double f = (r > 0.0) ? -P.k_bond * ext / r : 0.0;
            Fx += f * dx;
            Fy += f * dy;
            Fz += f * dz;
            if (ENERGY) {
                U += 0.25 * P.k_bond * ext * ext;
                W += 0.5 * f * d2;
            }
        }
        if (P.vol_on && ti == 0) volume_term(volume_of(P, s_vol, S.sc->vol0), pi, ni, Fx, Fy, Fz, Tq);
        if (KICK != 2) {
            S.frc[i] = V3{Fx, Fy, Fz};
            st3(S.trq + i, Tq);
        }
        if (KICK) {
            const double h = 0.5 * dt * P.inv_mass[ti];
            const double hw = 0.5 * dt * P.inv_inertia;
            half_kick(v, h, Fx, Fy, Fz);
            if (ti == 0) half_kick(w, hw, Tq.x, Tq.y, Tq.z);
            if (P.thermo_on) langevin_update(P, g, S.sc->step[par], ti, ni, v, w);
            if (P.quench_on) {
                project_along(v, Fx, Fy, Fz);
                if (ti == 0) project_along(w, Tq.x, Tq.y, Tq.z);
            }
            if (KICK == 1) {
                st3(S.vel + i, v);
                if (ti == 0) st3(S.angv + i, w);
            } else {
                D4 vn = v, wn = w, xn = pi;
                half_kick(vn, h, Fx, Fy, Fz);
                if (P.quench_on) cap_move(vn, dt, P.quench_max);
                drift_pos(xn, vn, dt);
                st3(S.vel + i, vn);
                st3(S.pos2 + i, xn);
                D4 on = ni;
                if (ti == 0) {
                    half_kick(wn, hw, Tq.x, Tq.y, Tq.z);
                    if (P.quench_on) cap_move(wn, dt, P.quench_max);
                    st3(S.angv + i, wn);
                    on = rotor_drift(ni, wn, dt);
                }
                st3(S.ori2 + i, on);
                drift_measures(xn, vn, xb, xp, disp2, disp2p, vmax2, bad);
                if (P.vol_on && ti == 0) volume_terms(xn, on, vsum);
            }
        }
    }
    if (KICK == 2) {
        drift_stats(S, S.bred2, lb, csub, disp2, vmax2, disp2p, bad);
        if (P.vol_on) volume_chunk_store(S, chunk, vsum);
    }
    if (ENERGY) {
        // per-chunk partials of U, W, KE, sum F and sum (r x F + tau), reduced across
        // the wavefront in a fixed butterfly (deterministic)
        double vals[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
        if (valid) {
            const double m = 1.0 / P.inv_mass[ti];
            double ke = 0.5 * m * (v.x * v.x + v.y * v.y + v.z * v.z);
            if (ti == 0) ke += 0.5 / P.inv_inertia * (w.x * w.x + w.y * w.y + w.z * w.z);
            vals[0] = U;
            vals[1] = W;
            vals[2] = ke;
            vals[3] = Fx;
            vals[4] = Fy;
            vals[5] = Fz;
            vals[6] = pi.y * Fz - pi.z * Fy + Tq.x;
            vals[7] = pi.z * Fx - pi.x * Fz + Tq.y;
            vals[8] = pi.x * Fy - pi.y * Fx + Tq.z;
        }
        for (int q = 0; q < 9; ++q) vals[q] = wave_sum(vals[q]);
        if (lane == 0)
            for (int q = 0; q < 9; ++q) S.epart[chunk * 9 + q] = vals[q];
    }
}

template <int MIXED, int ENERGY, int KICK>
static void launch_force_t(const LaunchCtx &L, double dt) {
    // FAST: the default pair-law constants, and one cutoff for both protein types
    bool fast = L.prm.zeta == 4 && L.prm.st0 == 0.0;
    for (int t = 0; t < 3; ++t) fast = fast && L.prm.rc2[t][1] == L.prm.rc2[t][2];
    const int nblk = L.nblk_f + (KICK ? L.nsys : 0);
    if (fast)
        hipLaunchKernelGGL((k_force<MIXED, ENERGY, KICK, 1>), dim3(nblk), dim3(BLOCK), 0, L.st, L.S, L.maps, L.prm, dt,
                           L.par);
    else
        hipLaunchKernelGGL((k_force<MIXED, ENERGY, KICK, 0>), dim3(nblk), dim3(BLOCK), 0, L.st, L.S, L.maps, L.prm, dt,
                           L.par);
}

void launch_force(const LaunchCtx &L, int mixed, int energy, int kick, double dt) {
    if (L.prm.vol_on) launch_volume_reduce(L, kick == 0 || energy);   // V of the current state from its lipid sums
    if (kick == 2) {
        if (mixed) launch_force_t<1, 0, 2>(L, dt);
        else launch_force_t<0, 0, 2>(L, dt);
        return;
    }
    const int key = (mixed ? 4 : 0) | (energy ? 2 : 0) | (kick ? 1 : 0);
    switch (key) {
        case 0: launch_force_t<0, 0, 0>(L, dt); break;
        case 1: launch_force_t<0, 0, 1>(L, dt); break;
        case 2: launch_force_t<0, 1, 0>(L, dt); break;
        case 3: launch_force_t<0, 1, 1>(L, dt); break;
        case 4: launch_force_t<1, 0, 0>(L, dt); break;
        case 5: launch_force_t<1, 0, 1>(L, dt); break;
        case 6: launch_force_t<1, 1, 0>(L, dt); break;
        default: launch_force_t<1, 1, 1>(L, dt); break;
    }
}

// ------------------------------------------------------------------ kick + drift

// v += dt/2m F, omega += dt/2I tau (lipids); x += dt v; n rotated about omega by
// |omega| dt (Rodrigues) and renormalised, in place; with the drift's statistics and
// its number.
__global__ __launch_bounds__(BLOCK) void k_kick_drift(const SysDev *Sd, Maps L_maps, DevParams P, double dt, int par) {
    const int s = find_sys(L_maps.p, L_maps.nsys, blockIdx.x);
    const SysDev &S = Sd[s];
    const int lb = blockIdx.x - L_maps.p[s];
    const int i = lb * BLOCK + threadIdx.x;
    if (i == 0) S.sc->step[par] += 1;                 // no other block of this kernel reads it
    double disp2 = 0.0, disp2p = 0.0, v2 = 0.0;
    bool bad = false;
    double vsum[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    if (i < S.n) {
        D4 p = ldpos(S, i), v = ld3(S.vel + i);
        const D4 f = ld3(S.frc + i);
        const int t = (int)p.w;
        const double h = 0.5 * dt * P.inv_mass[t];
        half_kick(v, h, f.x, f.y, f.z);
        if (P.quench_on) cap_move(v, dt, P.quench_max);
        drift_pos(p, v, dt);
        st3(S.vel + i, v);
        st3(S.pos + i, p);
        if (t == 0) {
            D4 w = ld3(S.angv + i);
            const D4 tq = ld3(S.trq + i);
            const double hw = 0.5 * dt * P.inv_inertia;
            half_kick(w, hw, tq.x, tq.y, tq.z);
            if (P.quench_on) cap_move(w, dt, P.quench_max);
            const D4 n = rotor_drift(ld3(S.ori + i), w, dt);
            st3(S.angv + i, w);
            st3(S.ori + i, n);
            if (P.vol_on) volume_terms(p, n, vsum);
        }
        drift_measures(p, v, S.xb[i], S.xp[i], disp2, disp2p, v2, bad);
    }
    drift_stats(S, S.bred, lb, (threadIdx.x >> 6) & 3, disp2, v2, disp2p, bad);
    if (P.vol_on && i / CHUNK < S.nchunk) volume_chunk_store(S, i / CHUNK, vsum);
}

// The statistics by themselves, for the steps whose decisions wait for them.  Two levels: one
// block alone reads a 4M-particle system's 1.5 MB of partials in 30 us.
constexpr int SR1 = 32;

__global__ __launch_bounds__(BLOCK) void k_stats_part(const SysDev *Sd) {
    const SysDev &S = Sd[blockIdx.x / SR1];
    if (S.n <= 0) return;
    __shared__ double s_m[3 * BLOCK / WAVE];
    const int part = blockIdx.x % SR1, per = (S.nchunk + SR1 - 1) / SR1;
    const int c0 = part * per, n = min(S.nchunk - c0, per);
    stats_of(S.bred + 3 * (size_t)c0, n, s_m);       // (none: zeros)
    if (threadIdx.x == 0)
        for (int q = 0; q < 3; ++q) S.sred[3 * part + q] = s_m[q];
}

__global__ __launch_bounds__(WAVE) void k_stats(const SysDev *Sd, int par) {
    const SysDev &S = Sd[blockIdx.x];
    if (S.n <= 0) return;
    __shared__ double s_m[3];
    publish_stats(S, S.sred, SR1, S.sc->step[par], s_m, 0ull);
}

void launch_kick_drift(const LaunchCtx &L, double dt) {
    hipLaunchKernelGGL(k_kick_drift, dim3(L.nblk_p), dim3(BLOCK), 0, L.st, L.S, L.maps, L.prm, dt, L.par);
}

void launch_stats(const LaunchCtx &L) {
    hipLaunchKernelGGL(k_stats_part, dim3(L.nsys * SR1), dim3(BLOCK), 0, L.st, L.S);
    hipLaunchKernelGGL(k_stats, dim3(L.nsys), dim3(WAVE), 0, L.st, L.S, L.par);
}

// ------------------------------------------------------------------ energy reduction

// Fixed-order sum of the per-chunk partials of each system (one block per system).
__global__ __launch_bounds__(256) void k_reduce_energy(const SysDev *Sd, int nsys, int vol_on) {
    const SysDev &S = Sd[blockIdx.x];
    __shared__ double sh[9][4];
    double acc[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
    for (int c = threadIdx.x; c < S.nchunk; c += blockDim.x)
        for (int q = 0; q < 9; ++q) acc[q] += S.epart[c * 9 + q];
    for (int q = 0; q < 9; ++q) acc[q] = wave_sum(acc[q]);
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0)
        for (int q = 0; q < 9; ++q) sh[q][w] = acc[q];
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int q = 0; q < 9; ++q) S.sc->energy[q] = ((sh[q][0] + sh[q][1]) + (sh[q][2] + sh[q][3]));
        if (vol_on) S.sc->energy[0] += S.sc->volU;
    }
}

void launch_reduce_energy(const LaunchCtx &L) {
    hipLaunchKernelGGL(k_reduce_energy, dim3(L.nsys), dim3(256), 0, L.st, L.S, L.nsys, L.prm.vol_on);
}

// ------------------------------------------------------------------ volume

// The lipid sums per chunk of the current state, for force evaluations that no
// drift precedes (a freshly loaded system).
__global__ __launch_bounds__(BLOCK) void k_volume_partials(const SysDev *Sd, Maps L_maps) {
    const int s = find_sys(L_maps.p, L_maps.nsys, blockIdx.x);
    const SysDev &S = Sd[s];
    const int lb = blockIdx.x - L_maps.p[s];
    const int i = lb * BLOCK + threadIdx.x;
    if (i / CHUNK >= S.nchunk) return;           // whole wavefronts past the last chunk
    double v[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    if (i < S.n) {
        const D4 p = ldpos(S, i);
        if (p.w == 0.0) volume_terms(p, ld3(S.ori + i), v);
    }
    volume_chunk_store(S, i / CHUNK, v);
}

// First level of two: VR1 blocks per system each sum a contiguous range of chunk totals
// into vred[b * 8 + q].  The step kernel's blocks each take the second level themselves.
__global__ __launch_bounds__(256) void k_volume_reduce1(const SysDev *Sd, int nsys) {
    const SysDev &S = Sd[blockIdx.x / VR1];
    const int part = blockIdx.x % VR1;
    const int per = (S.nchunk + VR1 - 1) / VR1;
    const int c0 = part * per, c1 = min(S.nchunk, c0 + per);
    __shared__ double sh[8][4];
    double acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    for (int c = c0 + (int)threadIdx.x; c < c1; c += 256)
        for (int q = 0; q < 8; ++q) acc[q] += S.vpart[(size_t)q * S.nchunk + c];
    for (int q = 0; q < 8; ++q) acc[q] = wave_sum(acc[q]);
    const int w = threadIdx.x / WAVE;
    if ((threadIdx.x & (WAVE - 1)) == 0)
        for (int q = 0; q < 8; ++q) sh[q][w] = acc[q];
    __syncthreads();
    if (threadIdx.x < 8 && S.n > 0) {
        const int q = threadIdx.x;
        S.vred[part * 8 + q] = (sh[q][0] + sh[q][1]) + (sh[q][2] + sh[q][3]);
    }
}

// The second level into the system's record, for force evaluations outside the step loop
// (the first fixes V0, which the step kernel reads; the energy takes U_V).
__global__ __launch_bounds__(BLOCK) void k_volume_record(const SysDev *Sd, int nsys, DevParams P) {
    const SysDev &S = Sd[blockIdx.x];
    if (S.n == 0) return;
    __shared__ double s_vol[8];
    volume_totals(volume_partial(S), s_vol);
    __syncthreads();
    if (threadIdx.x != 0) return;
    const Volume r = volume_of(P, s_vol, S.sc->vol0);
    S.sc->vol0 = r.V0;
    S.sc->volV = r.V;
    S.sc->volU = r.U;
}

void launch_volume_partials(const LaunchCtx &L) {
    hipLaunchKernelGGL(k_volume_partials, dim3(L.nblk_p), dim3(BLOCK), 0, L.st, L.S, L.maps);
}

void launch_volume_reduce(const LaunchCtx &L, bool record) {
    hipLaunchKernelGGL(k_volume_reduce1, dim3(L.nsys * VR1), dim3(256), 0, L.st, L.S, L.nsys);
    if (record) hipLaunchKernelGGL(k_volume_record, dim3(L.nsys), dim3(BLOCK), 0, L.st, L.S, L.nsys, L.prm);
}

// ------------------------------------------------------------------ outputs in caller order

// The state and forces in the caller's order: a thread per slot (coalesced reads, scattered
// writes) or a thread per caller id (scattered reads, coalesced writes).  Scattered writes are
// complete lines by the time they leave the caches as long as the frame stays there: 35 us
// against 45 for the state of 500k particles, 67 against 90 at 1M, 81 against 109 at 1.2M, but
// 198 against 133 at 1.5M and 679 against 327 at 4M (forces: 19, 35, 44 against 23, 45, 55; 86
// against 78 at 1.8M).  Below 60 thousand particles the reads by id are the shorter chain (5.4
// and 6.8 us at 56 thousand).
constexpr int OUT_SCATTER_MIN = 1 << 16, OUT_SCATTER_MAX = 5 << 18;
static bool scatters(int count) { return count >= OUT_SCATTER_MIN && count <= OUT_SCATTER_MAX; }

// N arrays of 3-vectors from slot i to caller id g, the loads side by side
template <int N>
__device__ __forceinline__ void copy_out(const V3 *const (&src)[N], double *const (&dst)[N], int i, int g) {
    V3 r[N];
#pragma unroll
    for (int k = 0; k < N; ++k)
        if (dst[k]) r[k] = ldg(src[k] + i);
#pragma unroll
    for (int k = 0; k < N; ++k)
        if (dst[k]) st3(reinterpret_cast<V3 *>(dst[k]) + g, D4{r[k].x, r[k].y, r[k].z, 0.0});
}

template <int SCATTER>
__global__ void k_out_state(const SysDev *Sd, int s, double *x, double *n, double *v, double *w) {
    const SysDev &S = Sd[s];
    const int q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= S.n) return;
    const int p = ldg((SCATTER ? S.gid : S.slot) + q);
    const V3 *const src[4] = {S.pos, S.ori, S.vel, S.angv};
    double *const dst[4] = {x, n, v, w};
    copy_out(src, dst, SCATTER ? q : p, SCATTER ? p : q);
}

void launch_out_state(const LaunchCtx &L, int sys, double *x, double *n, double *v, double *w, int count) {
    if (count <= 0) return;
    const dim3 grid((count + BLOCK - 1) / BLOCK);
    if (scatters(count)) hipLaunchKernelGGL(k_out_state<1>, grid, dim3(BLOCK), 0, L.st, L.S, sys, x, n, v, w);
    else hipLaunchKernelGGL(k_out_state<0>, grid, dim3(BLOCK), 0, L.st, L.S, sys, x, n, v, w);
}

template <int SCATTER>
__global__ void k_out_forces(const SysDev *Sd, int s, double *F, double *T) {
    const SysDev &S = Sd[s];
    const int q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= S.n) return;
    const int p = ldg((SCATTER ? S.gid : S.slot) + q);
    const V3 *const src[2] = {S.frc, S.trq};
    double *const dst[2] = {F, T};
    copy_out(src, dst, SCATTER ? q : p, SCATTER ? p : q);
}

void launch_out_forces(const LaunchCtx &L, int sys, double *F, double *T, int count) {
    if (count <= 0) return;
    const dim3 grid((count + BLOCK - 1) / BLOCK);
    if (scatters(count)) hipLaunchKernelGGL(k_out_forces<1>, grid, dim3(BLOCK), 0, L.st, L.S, sys, F, T);
    else hipLaunchKernelGGL(k_out_forces<0>, grid, dim3(BLOCK), 0, L.st, L.S, sys, F, T);
}

// ------------------------------------------------------------------ neighbour-set export

// Pruned blocks keep indices into their pruned stage in the 16-bit lists (0xffff
// pads); the others keep global slots in the 32-bit lists (-1 pads).
__device__ __forceinline__ int entry_slot(const SysDev &S, int blk, int scnt, int chunk, int lane, int r) {
    const size_t base = (size_t)chunk * MAXNB * CHUNK;
    if (scnt >= 0) {
        const int e = S.il16[base + il_at(r, lane)] >> 4;
        return e < scnt ? stage_slot(S.istage[(size_t)blk * SSTRIDE + e]) : -1;
    }
    return S.nl[base + r * CHUNK + lane];
}

// Pairs (gid_i < gid_j) of the pruned lists the step kernel walks that pass the exact
// FP64 test, sorted by both ids: row g holds the partners of caller id g with larger
// ids.  A counting pass stores each row's length at its caller id, a scan places the
// rows, and the filling pass walks the lists again, keeps the lane's partners sorted by
// insertion in its own LDS column (a row has 9 entries on average, at most MAXNB) and
// writes the row where it belongs.  The walks are bound by the latency of dependent
// loads (list entry, stage slot, id and position); the export by the copy to the host.
// Before, one unsorted append per wavefront left the sort to the host: 47 ms for the
// 0.93M pairs of a 124,952-particle vesicle, 97% of it std::sort.
constexpr int PR_BLOCK = 128;         // MAXNB x 128 ids: 48 KB of LDS, three blocks per CU
constexpr int PR_TILE = 2048;         // rows per scan tile

template <int FILL>
__global__ __launch_bounds__(PR_BLOCK) void k_pair_rows(const SysDev *Sd, int s, DevParams P, int32_t *out, int64_t cap) {
    const SysDev &S = Sd[s];
    __shared__ int s_row[FILL ? MAXNB * PR_BLOCK : 1];
    const int i = blockIdx.x * PR_BLOCK + threadIdx.x;
    if (i >= S.n) return;
    const int chunk = i / CHUNK, lane = i % CHUNK, blk = i / BLOCK;
    const D4 pi = ldpos(S, i);
    const int ti = (int)pi.w, gi = S.gid[i];
    const int rows = min(S.ilk[chunk], MAXNB), scnt = S.iscount[blk];
    int32_t *len = reinterpret_cast<int32_t *>(S.key2);           // row lengths, then starts within a tile
    int k = 0;
    for (int r = 0; r < rows; ++r) {
        const int j = entry_slot(S, blk, scnt, chunk, lane, r);
        if (j < 0 || j >= S.n) continue;
        const int gj = S.gid[j];
        if (gj <= gi) continue;
        const D4 pj = ldpos(S, j);
        double dx, dy, dz;
        const double d2 = dist2_exact(S, pi.x, pi.y, pi.z, pj.x, pj.y, pj.z, dx, dy, dz);
        if (!(d2 < P.rc2[ti][(int)pj.w])) continue;
        if constexpr (FILL) {
            int q = k;
            while (q > 0) {
                const int v = s_row[(q - 1) * PR_BLOCK + threadIdx.x];
                if (v < gj) break;
                s_row[q * PR_BLOCK + threadIdx.x] = v;
                --q;
            }
            s_row[q * PR_BLOCK + threadIdx.x] = gj;
        }
        ++k;
    }
    if constexpr (FILL) {
        const int64_t at = reinterpret_cast<const int64_t *>(S.hist)[gi / PR_TILE] + len[gi];
        int2 *o = reinterpret_cast<int2 *>(out);
        for (int q = 0; q < k && at + q < cap; ++q) o[at + q] = make_int2(gi, s_row[q * PR_BLOCK + threadIdx.x]);
    } else {
        len[gi] = k;
    }
}

// Row starts from the row lengths: within a tile of PR_TILE rows (in place, with the
// tile's total in tile[]), then the tiles' starts by one block; tile[ntile] receives the
// number of pairs.  64-bit: the pairs of the largest system exceed 2^31.
__device__ __forceinline__ int64_t pair_block_scan(int64_t v, int64_t *s_w, int64_t &total) {
    const int lane = threadIdx.x & (WAVE - 1), w = threadIdx.x / WAVE;
    int64_t x = v;
    for (int o = 1; o < WAVE; o <<= 1) {
        const int64_t y = __shfl_up((long long)x, o);
        if (lane >= o) x += y;
    }
    __syncthreads();
    if (lane == WAVE - 1) s_w[w] = x;
    __syncthreads();
    int64_t base = 0;
    total = 0;
    for (int q = 0; q < BLOCK / WAVE; ++q) {
        if (q < w) base += s_w[q];
        total += s_w[q];
    }
    return base + x - v;
}

__global__ __launch_bounds__(BLOCK) void k_pair_tiles(const SysDev *Sd, int s) {
    const SysDev &S = Sd[s];
    __shared__ int64_t s_w[BLOCK / WAVE];
    constexpr int PER = PR_TILE / BLOCK;
    int32_t *len = reinterpret_cast<int32_t *>(S.key2);
    const int base = blockIdx.x * PR_TILE + threadIdx.x * PER;
    int v[PER], sum = 0;
    for (int q = 0; q < PER; ++q) {
        v[q] = base + q < S.n ? len[base + q] : 0;
        sum += v[q];
    }
    int64_t total;
    int run = (int)pair_block_scan(sum, s_w, total);
    for (int q = 0; q < PER; ++q) {
        if (base + q < S.n) len[base + q] = run;
        run += v[q];
    }
    if (threadIdx.x == 0) reinterpret_cast<int64_t *>(S.hist)[blockIdx.x] = total;
}

__global__ __launch_bounds__(BLOCK) void k_pair_tile_scan(const SysDev *Sd, int s, int ntile) {
    int64_t *tile = reinterpret_cast<int64_t *>(Sd[s].hist);
    __shared__ int64_t s_w[BLOCK / WAVE];
    int64_t carry = 0;
    for (int t0 = 0; t0 < ntile; t0 += BLOCK) {
        const int t = t0 + (int)threadIdx.x;
        int64_t total;
        const int64_t ex = pair_block_scan(t < ntile ? tile[t] : 0, s_w, total);
        if (t < ntile) tile[t] = carry + ex;
        carry += total;
    }
    if (threadIdx.x == 0) tile[ntile] = carry;
}

// Count and place the rows of system sys (count particles).  The scratch is the radix
// sort's, idle outside a cell update: row starts in key2 (4 of its 8 bytes per
// particle), tile starts in hist (8 bytes per 2,048 rows, of 1 KB per 4,096 particles).
// The number of pairs ends in hist, at the tile count.
int64_t launch_pair_count(const LaunchCtx &L, int sys, int count) {
    const int ntile = (count + PR_TILE - 1) / PR_TILE;
    hipLaunchKernelGGL(k_pair_rows<0>, dim3((count + PR_BLOCK - 1) / PR_BLOCK), dim3(PR_BLOCK), 0, L.st, L.S, sys, L.prm,
                       nullptr, (int64_t)0);
    hipLaunchKernelGGL(k_pair_tiles, dim3(ntile), dim3(BLOCK), 0, L.st, L.S, sys);
    hipLaunchKernelGGL(k_pair_tile_scan, dim3(1), dim3(BLOCK), 0, L.st, L.S, sys, ntile);
    return ntile;
}

void launch_pair_fill(const LaunchCtx &L, int sys, int count, int32_t *out, int64_t cap) {
    hipLaunchKernelGGL(k_pair_rows<1>, dim3((count + PR_BLOCK - 1) / PR_BLOCK), dim3(PR_BLOCK), 0, L.st, L.S, sys, L.prm,
                       out, cap);
}

// ------------------------------------------------------------------ allocation-free pair export

// Staging for the pair export of rbc_get_pairs_noalloc, for callers that cannot
// allocate device memory: up to PAIR_SCRATCH_PAIRS pairs from byte 256 on.  Each device holds its own copy until the process ends;
// host code reaches it only through the address hipGetSymbolAddress returns on that
// device (pair_scratch_address), never through the array's name.
constexpr int64_t PAIR_SCRATCH_BYTES = 32ll << 20;
static __device__ __align__(256) int32_t scratch[PAIR_SCRATCH_BYTES / 4];

hipError_t pair_scratch_address(int device, void **out) {
    static std::mutex mtx;
    static void *addr[64] = {};
    if (device < 0 || device >= 64) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(mtx);
    if (!addr[device]) {
        int cur = 0;
        hipError_t e = hipGetDevice(&cur);
        if (e != hipSuccess) return e;
        if (cur != device) return hipErrorInvalidDevice;      // the caller makes the device current
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        addr[device] = p;
    }
    *out = addr[device];
    return hipSuccess;
}

}  // namespace rbc
