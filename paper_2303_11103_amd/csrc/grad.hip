// Gradient of received power for gfx950 (paper Sec. I and II: channel
// responses are differentiable with respect to material properties,
// antenna orientations and positions; Sec. III-A learns (eps_r, sigma) and
// Sec. III-B optimises the transmitter orientation by gradient steps).
//
// Input: the paths of one transmitter as face sequences (the checkpoint kept
// by the forward pass).  A few lanes per (rx, path) recompute the path in
// fp64 and differentiate its power |a|^2:
//   * transmitter position (x, y, z) and orientation (yaw, pitch) with
//     forward-mode dual numbers, a tangent per lane, through the images,
//     reflection points, directions, length, Fresnel coefficients, field
//     bases and the transmit pattern;
//   * material (eps_r, sigma) of every face on the path by one reverse sweep:
//     a = g_K^T R_K ... R_1 E_0 is linear in each r_perp/r_par, so
//     da/dr_perp_k = (g_k . e_perp) (e_perp . E_{k-1}),
//     da/dr_par_k  = (g_k . e_par_r) (e_par_i . E_{k-1}), with
//     g_{k-1} = R_k^T g_k, dr_perp/deta = -cos / (s (cos + s)^2),
//     dr_par/deta = cos (eta - 2 sin^2) / (s (eta cos + s)^2),
//     deta/deps_r = 1, deta/dsigma = -j / (eps0 w).
// Power derivatives dP/dtheta = 2 Re(conj(a) da/dtheta) are contracted with
// the upstream adjoint dL/dP_r and summed per block in LDS, then with fp64
// atomics.
#include <algorithm>

#include "traverse.h"

namespace rt {
namespace {

constexpr int NT = 1;      // tangents a lane of the received-power gradient carries
constexpr int kTheta = 5;  // transmitter parameters: x, y, z, yaw, pitch
constexpr int kMaxK = 8;
constexpr double kEps0 = 8.8541878128e-12;

// Dual number with N tangents.
template <int N>
struct Dual {
    double v;
    double d[N];
};
using D = Dual<NT>;
template <int N>
__device__ __forceinline__ Dual<N> dconst(double v) {
    Dual<N> r;
    r.v = v;
    for (int i = 0; i < N; ++i) r.d[i] = 0.0;
    return r;
}
__device__ __forceinline__ D dc(double v) { return dconst<NT>(v); }
template <int N>
__device__ __forceinline__ Dual<N> operator+(Dual<N> a, Dual<N> b) {
    Dual<N> r;
    r.v = a.v + b.v;
    for (int i = 0; i < N; ++i) r.d[i] = a.d[i] + b.d[i];
    return r;
}
template <int N>
__device__ __forceinline__ Dual<N> operator-(Dual<N> a, Dual<N> b) {
    Dual<N> r;
    r.v = a.v - b.v;
    for (int i = 0; i < N; ++i) r.d[i] = a.d[i] - b.d[i];
    return r;
}
template <int N>
__device__ __forceinline__ Dual<N> operator-(Dual<N> a) {
    Dual<N> r;
    r.v = -a.v;
    for (int i = 0; i < N; ++i) r.d[i] = -a.d[i];
    return r;
}
template <int N>
__device__ __forceinline__ Dual<N> operator*(Dual<N> a, Dual<N> b) {
    Dual<N> r;
    r.v = a.v * b.v;
    for (int i = 0; i < N; ++i) r.d[i] = a.d[i] * b.v + a.v * b.d[i];
    return r;
}
template <int N>
__device__ __forceinline__ Dual<N> operator*(Dual<N> a, double s) {
    Dual<N> r;
    r.v = a.v * s;
    for (int i = 0; i < N; ++i) r.d[i] = a.d[i] * s;
    return r;
}
template <int N>
__device__ __forceinline__ Dual<N> operator/(Dual<N> a, Dual<N> b) {
    Dual<N> r;
    r.v = a.v / b.v;
    const double ib = 1.0 / b.v;
    for (int i = 0; i < N; ++i) r.d[i] = (a.d[i] - r.v * b.d[i]) * ib;
    return r;
}
template <int N>
__device__ __forceinline__ Dual<N> dsqrt(Dual<N> a) {
    Dual<N> r;
    r.v = sqrt(a.v);
    const double k = r.v > 0.0 ? 0.5 / r.v : 0.0;
    for (int i = 0; i < N; ++i) r.d[i] = a.d[i] * k;
    return r;
}
template <int N>
__device__ __forceinline__ Dual<N> dfun(Dual<N> a, double v, double dv) {
    Dual<N> r;
    r.v = v;
    for (int i = 0; i < N; ++i) r.d[i] = a.d[i] * dv;
    return r;
}
__device__ __forceinline__ D dcos(D a) { return dfun(a, cos(a.v), -sin(a.v)); }
__device__ __forceinline__ D dsin(D a) { return dfun(a, sin(a.v), cos(a.v)); }
template <int N>
__device__ __forceinline__ Dual<N> dacos(Dual<N> a) {
    const double x = fmin(fmax(a.v, -1.0), 1.0);
    const double den = sqrt(fmax(1.0 - x * x, 1e-300));
    return dfun(a, acos(x), -1.0 / den);
}
template <int N>
__device__ __forceinline__ Dual<N> datan2(Dual<N> y, Dual<N> x) {
    Dual<N> r;
    r.v = atan2(y.v, x.v);
    const double den = x.v * x.v + y.v * y.v;
    for (int i = 0; i < N; ++i) r.d[i] = den > 0.0 ? (x.v * y.d[i] - y.v * x.d[i]) / den : 0.0;
    return r;
}
template <int N>
__device__ __forceinline__ Dual<N> dexp10(Dual<N> a) {
    const double v = exp10(a.v);
    return dfun(a, v, v * 2.302585092994045684);
}
template <int N>
__device__ __forceinline__ Dual<N> dmin(Dual<N> a, Dual<N> b) { return a.v <= b.v ? a : b; }

template <int N>
struct Dual3 {
    Dual<N> x, y, z;
};
using D3 = Dual3<NT>;
__device__ __forceinline__ D3 operator+(D3 a, D3 b) { return D3{a.x + b.x, a.y + b.y, a.z + b.z}; }
__device__ __forceinline__ D3 operator-(D3 a, D3 b) { return D3{a.x - b.x, a.y - b.y, a.z - b.z}; }
__device__ __forceinline__ D3 operator*(D3 a, D s) { return D3{a.x * s, a.y * s, a.z * s}; }
__device__ __forceinline__ D3 operator*(D3 a, double s) { return D3{a.x * s, a.y * s, a.z * s}; }
__device__ __forceinline__ D ddot(D3 a, D3 b) { return a.x * b.x + a.y * b.y + a.z * b.z; }
__device__ __forceinline__ D ddot(D3 a, d3 b) { return a.x * b.x + a.y * b.y + a.z * b.z; }
__device__ __forceinline__ D3 dcross(D3 a, D3 b) {
    return D3{a.y * b.z - a.z * b.y, a.z * b.x - a.x * b.z, a.x * b.y - a.y * b.x};
}
__device__ __forceinline__ D3 dcross(D3 a, d3 b) {
    return D3{a.y * b.z - a.z * b.y, a.z * b.x - a.x * b.z, a.x * b.y - a.y * b.x};
}
__device__ __forceinline__ D3 dconst(d3 a) { return D3{dc(a.x), dc(a.y), dc(a.z)}; }
__device__ __forceinline__ d3 val(D3 a) { return d3{a.x.v, a.y.v, a.z.v}; }
__device__ __forceinline__ D dnorm(D3 a) { return dsqrt(ddot(a, a)); }

// complex dual
struct C {
    D re, im;
};
__device__ __forceinline__ C operator+(C a, C b) { return C{a.re + b.re, a.im + b.im}; }
__device__ __forceinline__ C operator-(C a, C b) { return C{a.re - b.re, a.im - b.im}; }
__device__ __forceinline__ C operator*(C a, C b) { return C{a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re}; }
__device__ __forceinline__ C operator*(C a, D s) { return C{a.re * s, a.im * s}; }
__device__ __forceinline__ C operator/(C a, C b) {
    D den = b.re * b.re + b.im * b.im;
    return C{(a.re * b.re + a.im * b.im) / den, (a.im * b.re - a.re * b.im) / den};
}
__device__ __forceinline__ C csqrt_d(C z) {
    D r = dsqrt(z.re * z.re + z.im * z.im);
    if (z.re.v >= 0.0) {
        D re = dsqrt((r + z.re) * 0.5);
        return C{re, z.im / (re * 2.0)};
    }
    D im = dsqrt((r - z.re) * 0.5);
    D absim = z.im.v >= 0.0 ? z.im : -z.im;
    return C{absim / (im * 2.0), z.im.v >= 0.0 ? im : -im};
}
struct C3 {
    C x, y, z;
};
__device__ __forceinline__ C cdot(C3 a, D3 b) { return C{ddot(D3{a.x.re, a.y.re, a.z.re}, b), ddot(D3{a.x.im, a.y.im, a.z.im}, b)}; }
__device__ __forceinline__ C3 cscale(D3 v, C s) {
    return C3{C{v.x * s.re, v.x * s.im}, C{v.y * s.re, v.y * s.im}, C{v.z * s.re, v.z * s.im}};
}
__device__ __forceinline__ C3 cadd3(C3 a, C3 b) { return C3{a.x + b.x, a.y + b.y, a.z + b.z}; }

struct DRot {
    D R[9];
};
__device__ DRot drot(D yaw, D pitch, D roll) {
    D cy = dcos(yaw), sy = dsin(yaw), cp = dcos(pitch), sp = dsin(pitch), cr = dcos(roll), sr = dsin(roll);
    DRot o;
    o.R[0] = cy * cp; o.R[1] = cy * sp * sr - sy * cr; o.R[2] = cy * sp * cr + sy * sr;
    o.R[3] = sy * cp; o.R[4] = sy * sp * sr + cy * cr; o.R[5] = sy * sp * cr - cy * sr;
    o.R[6] = -sp;     o.R[7] = cp * sr;                o.R[8] = cp * cr;
    return o;
}

// Field of an antenna with orientation R towards the local direction (lx, ly, lz).
template <int N>
__device__ Dual3<N> dantenna_local(const Dual<N>* R, int pattern, Dual<N> lx, Dual<N> ly, Dual<N> lz, int pol) {
    using T = Dual<N>;
    T rho = dsqrt(lx * lx + ly * ly);
    T cph = dconst<N>(1.0), sph = dconst<N>(0.0);
    if (rho.v > 0.0) {
        cph = lx / rho;
        sph = ly / rho;
    }
    T c = dconst<N>(1.0);
    if (pattern == kPatTR38901) {
        const double kDeg = 180.0 / kPi;
        T th = dacos(lz) * kDeg;
        T ph = datan2(ly, lx) * kDeg;
        T u = (th - dconst<N>(90.0)) * (1.0 / 65.0);
        T w = ph * (1.0 / 65.0);
        T av = -dmin(u * u * 12.0, dconst<N>(30.0));
        T ah = -dmin(w * w * 12.0, dconst<N>(30.0));
        T a = -dmin(-(av + ah), dconst<N>(30.0));
        c = dexp10((a + dconst<N>(8.0)) * (1.0 / 20.0));
    } else if (pattern == kPatDipole) {
        c = rho * 1.2247448713915890;  // sqrt(1.5) sin(theta)
    }
    double zc, zs;
    pol_angle(pol, zc, zs);
    const T ct = c * zc, cp = c * zs;
    T tx = ct * lz * cph - cp * sph, ty = ct * lz * sph + cp * cph, tz = -(ct * rho);
    return Dual3<N>{R[0] * tx + R[1] * ty + R[2] * tz, R[3] * tx + R[4] * ty + R[5] * tz,
                    R[6] * tx + R[7] * ty + R[8] * tz};
}

__device__ D3 dantenna(const DRot& Rr, int pattern, D3 d, int pol = 0) {
    const D* R = Rr.R;
    return dantenna_local(R, pattern, R[0] * d.x + R[3] * d.y + R[6] * d.z, R[1] * d.x + R[4] * d.y + R[7] * d.z,
                          R[2] * d.x + R[5] * d.y + R[8] * d.z, pol);
}

__device__ D3 dperp(D3 d, d3 n) {
    D3 e = dcross(d, n);
    D l = dnorm(e);
    if (l.v < 1e-12) {  // normal incidence: any unit vector orthogonal to d (result independent of it)
        d3 dv = val(d);
        double ax = fabs(dv.x), ay = fabs(dv.y), az = fabs(dv.z);
        d3 a = (ax <= ay && ax <= az) ? d3{1, 0, 0} : ((ay <= az) ? d3{0, 1, 0} : d3{0, 0, 1});
        e = dconst(a) - d * ddot(d, a);
        l = dnorm(e);
    }
    return e * (dc(1.0) / l);
}

__device__ __forceinline__ cd cdotv(const cd* g, d3 v) {
    return cd{g[0].re * v.x + g[1].re * v.y + g[2].re * v.z, g[0].im * v.x + g[1].im * v.y + g[2].im * v.z};
}

// kPathLanes lanes per path slot, one transmitter parameter each: most slots
// are empty and the launch lasts as long as one path, so a path is spread over
// lanes instead of carrying five tangents through one (6.6 KB of private arrays
// per lane).  The sums go to LDS first: with an atomic on a few addresses of
// memory per path and parameter, those bound full lists, the more so as lanes of
// different parameters cannot be summed within an instruction.  Depth 3, 256
// receivers x 128 slots, one in fifty full: five tangents a lane 93 us, one 36;
// 4096 receivers x 64 full slots: 7.6 and 10.3 ms, with the sums in LDS 0.86.
constexpr int kPathLanes = 8, kGradBlock = 128;
// Adds the derivatives of path slot `item` to out ([2 nm + 5], as g.grad): the
// transmitter parameter theta, and with theta 0 the materials.
__device__ __forceinline__ void power_grad_path(const GradArgs& g, const MatTable& mats, int64_t item, int theta,
                                                double* out) {
    const int r = (int)(item / g.P);
    const int K = g.depth[item];
    if (K < 0 || K > g.fd || K > kMaxK) return;  // empty slot (or not a path of this depth range)
    // adjoint of the path coefficient: the contribution of the path is
    // Re(gc * da/dtheta), gc given (coef_adj) or 2 w conj(a) for the power
    // |a|^2 weighted by the upstream w = dL/dP_r
    const double w_up = g.coef_adj ? 0.0 : g.dL_dP[r];
    if (g.coef_adj ? (g.coef_adj[2 * item] == 0.0 && g.coef_adj[2 * item + 1] == 0.0) : w_up == 0.0) return;
    int fc[kMaxK];
    for (int i = 0; i < K; ++i) {
        fc[i] = g.faces[item * g.fd + i];
        if (fc[i] < 0 || fc[i] >= g.sc.num_faces) return;
    }
    // seeds: theta 0..2 tx position, 3 yaw, 4 pitch
    D3 tx{dc(g.tx[0]), dc(g.tx[1]), dc(g.tx[2])};
    tx.x.d[0] = theta == 0 ? 1.0 : 0.0;
    tx.y.d[0] = theta == 1 ? 1.0 : 0.0;
    tx.z.d[0] = theta == 2 ? 1.0 : 0.0;
    D yaw = dc(g.yaw), pitch = dc(g.pitch);
    yaw.d[0] = theta == 3 ? 1.0 : 0.0;
    pitch.d[0] = theta == 4 ? 1.0 : 0.0;
    const DRot Rt = drot(yaw, pitch, dc(g.roll));
    const d3 rx{g.rx[3 * r], g.rx[3 * r + 1], g.rx[3 * r + 2]};
    D3 I[kMaxK + 1];
    I[0] = tx;
    for (int k = 1; k <= K; ++k) {
        const Face F = g.sc.faces[fc[k - 1]];
        const d3 n{F.n[0], F.n[1], F.n[2]}, q{F.q[0], F.q[1], F.q[2]};
        I[k] = I[k - 1] - dconst(n) * (ddot(I[k - 1] - dconst(q), n) * 2.0);
    }
    D3 X[kMaxK + 2];
    X[0] = tx;
    X[K + 1] = dconst(rx);
    for (int k = K; k >= 1; --k) {
        const Face F = g.sc.faces[fc[k - 1]];
        const d3 n{F.n[0], F.n[1], F.n[2]}, q{F.q[0], F.q[1], F.q[2]};
        const D3 A = X[k + 1];
        const D t = ddot(dconst(q) - A, n) / ddot(I[k] - A, n);
        X[k] = A + (I[k] - A) * t;
    }
    D3 dir[kMaxK + 1];
    D L = dc(0.0);
    for (int k = 0; k <= K; ++k) {
        const D3 s = X[k + 1] - X[k];
        const D l = dnorm(s);
        L = L + l;
        dir[k] = s * (dc(1.0) / l);
    }
    const D3 F0 = dantenna(Rt, g.tx_pattern, dir[0], g.tx_pol);
    C3 E{C{F0.x, dc(0.0)}, C{F0.y, dc(0.0)}, C{F0.z, dc(0.0)}};
    // values kept for the material sweep
    d3 ep_v[kMaxK], eli_v[kMaxK], elr_v[kMaxK];
    cd aperp[kMaxK], apar[kMaxK], rp_v[kMaxK], rl_v[kMaxK], drp[kMaxK], drl[kMaxK];
    int mat_k[kMaxK];
    for (int k = 1; k <= K; ++k) {
        const Face F = g.sc.faces[fc[k - 1]];
        d3 n{F.n[0], F.n[1], F.n[2]};
        const D3 din = dir[k - 1], dout = dir[k];
        if (ddot(din, n).v > 0.0) n = scale(n, -1.0);
        const D cos_i = -ddot(din, n);
        const Mat m = mats.m[F.mat];
        C rp, rl;
        cd drp_v{0, 0}, drl_v{0, 0};
        if (m.pec) {
            rp = C{dc(-1.0), dc(0.0)};
            rl = C{dc(1.0), dc(0.0)};
        } else {
            const C eta{dc(m.eta_re_d), dc(m.eta_im_d)};
            const D sin2 = dc(1.0) - cos_i * cos_i;
            const C s = csqrt_d(C{eta.re - sin2, eta.im});
            const C c{cos_i, dc(0.0)};
            rp = (c - s) / (c + s);
            const C ec = eta * cos_i;
            rl = (ec - s) / (ec + s);
            // d r / d eta (values)
            const cd sv{s.re.v, s.im.v}, cv{cos_i.v, 0.0}, ev{m.eta_re_d, m.eta_im_d};
            const cd cps = cadd(cv, sv), ecs = cadd(cmulr(ev, cos_i.v), sv);
            drp_v = cdiv(cd{-cos_i.v, 0.0}, cmul(sv, cmul(cps, cps)));
            const cd num = cmulr(csub(ev, cd{2.0 * sin2.v, 0.0}), cos_i.v);
            drl_v = cdiv(num, cmul(sv, cmul(ecs, ecs)));
        }
        {  // specular share of a scattering material (a constant factor)
            const double share = specular_share(m);
            rp = rp * dc(share);
            rl = rl * dc(share);
            drp_v = cmulr(drp_v, share);
            drl_v = cmulr(drl_v, share);
        }
        const D3 ep = dperp(din, n);
        const D3 eli = dcross(ep, din), elr = dcross(ep, dout);
        const C ap = cdot(E, ep), al = cdot(E, eli);
        ep_v[k - 1] = val(ep);
        eli_v[k - 1] = val(eli);
        elr_v[k - 1] = val(elr);
        aperp[k - 1] = cd{ap.re.v, ap.im.v};
        apar[k - 1] = cd{al.re.v, al.im.v};
        rp_v[k - 1] = cd{rp.re.v, rp.im.v};
        rl_v[k - 1] = cd{rl.re.v, rl.im.v};
        drp[k - 1] = drp_v;
        drl[k - 1] = drl_v;
        mat_k[k - 1] = F.mat;
        E = cadd3(cscale(ep, rp * ap), cscale(elr, rl * al));
    }
    const D3 mdK = dir[K] * -1.0;
    // receive pattern: receiver pose is not a differentiated parameter
    const Antenna ra = g.rx_ant[r];
    DRot Rr;
    for (int i = 0; i < 9; ++i) Rr.R[i] = dc(ra.Rd[i]);
    const D3 Fr = dantenna(Rr, ra.pattern, mdK, ra.pol);
    const D amp = dc(g.lambda / (4.0 * kPi)) / L;
    const C pr = cdot(E, Fr);
    const C a{pr.re * amp, pr.im * amp};
    const double gre = g.coef_adj ? g.coef_adj[2 * item] : 2.0 * w_up * a.re.v;
    const double gim = g.coef_adj ? g.coef_adj[2 * item + 1] : -2.0 * w_up * a.im.v;
    const int base = 2 * g.nm;
    atomicAdd(out + base + theta, gre * a.re.d[0] - gim * a.im.d[0]);
    if (theta != 0) return;
    // material sweep (values only, the same in every lane of the path)
    cd gv[3] = {cd{amp.v * Fr.x.v, 0.0}, cd{amp.v * Fr.y.v, 0.0}, cd{amp.v * Fr.z.v, 0.0}};
    const double w = 2.0 * kPi * g.freq;
    for (int k = K; k >= 1; --k) {
        const int i = k - 1;
        const cd gp = cdotv(gv, ep_v[i]);
        const cd gl = cdotv(gv, elr_v[i]);
        const cd da = cadd(cmul(cmul(gp, aperp[i]), drp[i]), cmul(cmul(gl, apar[i]), drl[i]));
        // d/deps_r: Re(gc da); d/dsigma: Re(gc da (-j / (eps0 w))) = Im(gc da) / (eps0 w)
        const double re_gd = gre * da.re - gim * da.im;
        const double im_gd = gre * da.im + gim * da.re;
        const double dsig = 1.0 / (kEps0 * w);
        if (drp[i].re != 0.0 || drp[i].im != 0.0 || drl[i].re != 0.0 || drl[i].im != 0.0) {
            atomicAdd(out + 2 * mat_k[i], re_gd);
            atomicAdd(out + 2 * mat_k[i] + 1, im_gd * dsig);
        }
        // g <- R_k^T g
        const cd p1 = cmul(rp_v[i], gp), p2 = cmul(rl_v[i], gl);
        const d3 e1 = ep_v[i], e2 = eli_v[i];
        gv[0] = cadd(cmulr(p1, e1.x), cmulr(p2, e2.x));
        gv[1] = cadd(cmulr(p1, e1.y), cmulr(p2, e2.y));
        gv[2] = cadd(cmulr(p1, e1.z), cmulr(p2, e2.z));
    }
}

__global__ __launch_bounds__(kGradBlock) void power_grad_kernel(GradArgs g, MatTable mats) {
    __shared__ double sum[2 * kMaxMaterials + kTheta];
    const int outs = 2 * g.nm + kTheta;
    for (int i = threadIdx.x; i < outs; i += kGradBlock) sum[i] = 0.0;
    __syncthreads();
    const int64_t item = ((int64_t)blockIdx.x * kGradBlock + threadIdx.x) / kPathLanes;
    const int theta = threadIdx.x % kPathLanes;
    if (item < (int64_t)g.nrx * g.P && theta < kTheta) power_grad_path(g, mats, item, theta, sum);
    __syncthreads();
    for (int i = threadIdx.x; i < outs; i += kGradBlock)
        if (sum[i] != 0.0) atomicAdd(g.grad + i, sum[i]);
}

// ------------------------------------------------------------------ coverage
// Gradient of the path gain summed over a region of coverage-map cells with
// respect to the radio materials and the transmitter orientation (the
// coverage analogue of the received-power gradient; Sec. III-B optimises a
// transmitter orientation by gradient steps).  Ray geometry does not depend
// on these parameters, so the recorded hits (triangle and distance per
// segment) fix every ray, replayed in fp64 with the formulas of the
// shoot-and-bounce kernel in two passes:
//   * a walk of the geometry alone, which marks the segments that cross the
//     grid plane inside the region;
//   * for the rays with a mark, the field E and its tangents dE/dtheta up to
//     the last marked segment.  At launch dE/d(yaw, pitch) comes from the
//     dual-number transmit pattern; at a reflection off material m, E' = R E
//     gives dE'/dtheta = R dE/dtheta + [theta of m] (dR/d eta) E (d eta/d theta),
//     with dR/d eta from d r_perp / d eta and d r_par / d eta as above.  As
//     d eta/d sigma = -j/(eps0 w) is a constant, so is the ratio of a
//     material's two tangents: only dE/d eps_r is carried.  Every mark adds
//     w = wscale |F_rx . E|^2 / |d_z| and dw = wscale 2 Re(conj(a) F_rx . dE) / |d_z|.
// Most rays never cross the region, and the second pass is fp64 arithmetic
// with antenna functions, so it runs over a queue, in a launch of its own: the
// walk needs a third of its registers and many waves to hide the records' and
// the normals' latency.  Rays without a reflection are kept apart from the
// others.  After a reflection a field is its two components on the segment's
// transverse basis.  Tangents are a template parameter: with ten for every
// scene one kernel for all took 220 registers.  Bound by fp64 arithmetic; 10^7
// rays of depth 3 over the street canyon's 770 triangles: 1380 us as one
// kernel of one thread per ray -> 170 (walk) + 151 us (replay).
constexpr int kCovWaves = 3;  // of the replay per SIMD: 168 registers; both grids are three blocks per CU
constexpr int kWalkTris = 1024;

// Marked rays (index, marks) in parts, one per wave: count[w] = (those from the
// back of part w, those from its front).
struct CovQueue {
    uint2* ray;
    uint2* count;
    int64_t part;
};

struct CovHit {
    d3 n;              // normal facing the ray
    double cos_i;
    d3 p, dout;        // reflection point, outgoing direction
    int32_t mat;
    bool diffuse;
};

// The reflection of recorded ray j at depth k: the specular direction, or the
// forward kernel's diffuse draw (it depends on no parameter).
__device__ __forceinline__ CovHit cov_reflect(const CovGradArgs& g, const MatTable& mats, int64_t j, int k,
                                              const Shade& sh, double t, d3 o, d3 d) {
    CovHit h;
    h.n = d3{sh.n[0], sh.n[1], sh.n[2]};
    if (dot(d, h.n) > 0.0) h.n = scale(h.n, -1.0);
    h.cos_i = -dot(d, h.n);
    h.dout = add(d, scale(h.n, 2.0 * h.cos_i));
    h.p = add(o, scale(d, t));
    h.mat = sh.mat;
    h.diffuse = false;
    if (g.scatters && mats.m[sh.mat].scat > 0.0f) {
        const uint64_t ri = (uint64_t)(g.begin + j * g.stride);
        const uint64_t c0 = (ri * (uint64_t)(g.max_depth + 1) + (uint64_t)k) * 3ull;
        const double S = (double)mats.m[sh.mat].scat;
        if (uniform01(g.scat_seed, c0) < S * S) {
            h.dout = lambert_dir(h.n, uniform01(g.scat_seed, c0 + 1), uniform01(g.scat_seed, c0 + 2));
            h.diffuse = true;
        }
    }
    return h;
}

// Bit k: segment k of recorded ray j crosses the grid plane inside the region.
// staged: the triangles' shades in input order (LDS), or null.
template <bool STAGED>
__device__ __forceinline__ uint32_t cov_walk(const CovGradArgs& g, const MatTable& mats, const Shade* staged,
                                             int64_t j) {
    uint32_t marks = 0;
    int32_t tri = g.hit_tri[j];
    double t = g.hit_t[j];
    d3 o{g.tx[0], g.tx[1], g.tx[2]};
    // A ray that neither hits nor crosses the plane (the sky: whole waves, as the
    // lattice is ordered by height) ends before its azimuth is computed.
    const double z = fib_height(g.begin + j * g.stride, g.num_rays);
    if (tri < 0 || g.max_depth == 0) {
        const double tc = (g.gz - o.z) / z;
        if (!(fabs(z) >= 1e-12 && tc > 0.0 && tc < t)) return 0;
    }
    d3 d = fib_dir(g.begin + j * g.stride, g.num_rays);
    for (int k = 0; k <= g.max_depth; ++k) {
        if (tri == -2) break;
        int32_t tri_next = -2;
        double t_next = 0.0;
        if (k < g.max_depth) {
            tri_next = g.hit_tri[(int64_t)(k + 1) * g.count + j];
            t_next = g.hit_t[(int64_t)(k + 1) * g.count + j];
        }
        if (fabs(d.z) >= 1e-12) {
            const double tc = (g.gz - o.z) / d.z;
            if (tc > 0.0 && tc < t) {
                const double x = o.x + tc * d.x, y = o.y + tc * d.y;
                const double fx = floor((x - g.gx0) / g.gcell), fy = floor((y - g.gy0) / g.gcell);
                if (fx >= 0.0 && fx < (double)g.gnx && fy >= 0.0 && fy < (double)g.gny) {
                    const int64_t cell = (int64_t)fy * g.gnx + (int64_t)fx;
                    if (!g.region || g.region[cell]) marks |= 1u << k;
                }
            }
        }
        if (tri < 0 || k == g.max_depth || tri >= g.sc.nt) break;
        const CovHit h = cov_reflect(g, mats, j, k, STAGED ? staged[tri] : g.sc.shades[g.sc.leaf_of_input[tri]], t, o,
                                     d);
        o = h.p;
        d = h.dout;
        tri = tri_next;
        t = t_next;
    }
    return marks;
}

// Sums of one thread: the gain, and its derivatives with respect to eps_r and
// eps0 w sigma per material, yaw and pitch.
template <int NM>
struct CovSums {
    double w, eps[NM], sig[NM], yaw, pitch;
};

// Complex field of one tangent on the transverse basis (u, v) of its segment.
struct Trans {
    cd u, v;
};

// Adds a marked segment: the amplitude and its tangents received along fr.
template <int NM>
__device__ __forceinline__ void cov_deposit(double w0, cd a, cd y, cd p, const cd* e, CovSums<NM>& acc) {
    acc.w += w0 * (a.re * a.re + a.im * a.im);
    const double w2 = 2.0 * w0;
    acc.yaw += w2 * (a.re * y.re + a.im * y.im);
    acc.pitch += w2 * (a.re * p.re + a.im * p.im);
#pragma unroll
    for (int m = 0; m < NM; ++m) {
        acc.eps[m] += w2 * (a.re * e[m].re + a.im * e[m].im);
        acc.sig[m] += w2 * (a.re * e[m].im - a.im * e[m].re);  // Re(conj(a) (-j) e)
    }
}

template <int NM>
__device__ __forceinline__ void cov_replay(const CovGradArgs& g, const MatTable& mats, int64_t j, uint32_t marks,
                                           CovSums<NM>& acc) {
    d3 d = fib_dir(g.begin + j * g.stride, g.num_rays);
    d3 o{g.tx[0], g.tx[1], g.tx[2]};
    // field and tangents of the segment: real vectors F from the transmitter,
    // then (after a reflection) transverse components on (u, v)
    d3 F, FY, FP, u, v;
    Trans E, Y, P, M[NM];
    {
        Dual<2> R[9];
#pragma unroll
        for (int i = 0; i < 9; ++i) R[i] = Dual<2>{g.R[i], {g.Ryaw[i], g.Rpitch[i]}};
        const Dual3<2> f = dantenna_local(R, g.tx_pattern, R[0] * d.x + R[3] * d.y + R[6] * d.z,
                                          R[1] * d.x + R[4] * d.y + R[7] * d.z, R[2] * d.x + R[5] * d.y + R[8] * d.z,
                                          g.tx_pol);
        F = d3{f.x.v, f.y.v, f.z.v};
        FY = d3{f.x.d[0], f.y.d[0], f.z.d[0]};
        FP = d3{f.x.d[1], f.y.d[1], f.z.d[1]};
    }
    for (int k = 0;; ++k) {
        if ((marks >> k) & 1u) {
            const d3 fr = antenna_field(g.rx_ant, d3{-d.x, -d.y, -d.z});
            const double w0 = g.wscale / fabs(d.z);
            if (k == 0) {
                const double a = dot(F, fr);
                acc.w += w0 * a * a;
                acc.yaw += 2.0 * w0 * a * dot(FY, fr);
                acc.pitch += 2.0 * w0 * a * dot(FP, fr);
            } else {
                const double fu = dot(u, fr), fv = dot(v, fr);
                auto at = [&](const Trans& x) { return cadd(cmulr(x.u, fu), cmulr(x.v, fv)); };
                cd e[NM];
#pragma unroll
                for (int m = 0; m < NM; ++m) e[m] = at(M[m]);
                cov_deposit<NM>(w0, at(E), at(Y), at(P), e, acc);
            }
        }
        if (!(marks >> (k + 1))) return;
        const int64_t at = (int64_t)k * g.count + j;
        const CovHit h = cov_reflect(g, mats, j, k, g.sc.shades[g.sc.leaf_of_input[g.hit_tri[at]]], g.hit_t[at], o, d);
        const d3 ep = perp_basis(d, h.n), eli = cross(ep, d);
        const d3 epo = h.diffuse ? perp_basis(h.dout, h.n) : ep;
        const Mat& mt = mats.m[h.mat];
        const double cos_i = h.cos_i;
        cd rp{-1.0, 0.0}, rl{1.0, 0.0}, drp{0.0, 0.0}, drl{0.0, 0.0};
        if (!mt.pec) {
            const cd eta{mt.eta_re_d, mt.eta_im_d}, c{cos_i, 0.0};
            const double sin2 = 1.0 - cos_i * cos_i;
            const cd s = csqrt(cd{eta.re - sin2, eta.im});
            const cd ec = cmulr(eta, cos_i);
            const cd ip = cdiv(cd{1.0, 0.0}, cadd(c, s)), il = cdiv(cd{1.0, 0.0}, cadd(ec, s));
            const cd is = cdiv(cd{cos_i, 0.0}, s);
            rp = cmul(csub(c, s), ip);
            rl = cmul(csub(ec, s), il);
            drp = cmul(cd{-is.re, -is.im}, cmul(ip, ip));
            drl = cmul(cmul(csub(eta, cd{2.0 * sin2, 0.0}), is), cmul(il, il));
        }
        if (k == 0) {
            const double fu = dot(F, ep), fv = dot(F, eli);
            E = Trans{cmulr(rp, fu), cmulr(rl, fv)};
            Y = Trans{cmulr(rp, dot(FY, ep)), cmulr(rl, dot(FY, eli))};
            P = Trans{cmulr(rp, dot(FP, ep)), cmulr(rl, dot(FP, eli))};
#pragma unroll
            for (int m = 0; m < NM; ++m)
                M[m] = m == h.mat ? Trans{cmulr(drp, fu), cmulr(drl, fv)} : Trans{cd{0.0, 0.0}, cd{0.0, 0.0}};
        } else {
            const double uu = dot(u, ep), vu = dot(v, ep), uv = dot(u, eli), vv = dot(v, eli);
            auto turn = [&](const Trans& x) {  // components on (ep, eli)
                return Trans{cadd(cmulr(x.u, uu), cmulr(x.v, vu)), cadd(cmulr(x.u, uv), cmulr(x.v, vv))};
            };
            auto through = [&](const Trans& x) { return Trans{cmul(rp, x.u), cmul(rl, x.v)}; };
            const Trans e = turn(E);
            E = through(e);
            Y = through(turn(Y));
            P = through(turn(P));
#pragma unroll
            for (int m = 0; m < NM; ++m) {
                M[m] = through(turn(M[m]));
                if (m == h.mat) M[m] = Trans{cadd(M[m].u, cmul(drp, e.u)), cadd(M[m].v, cmul(drl, e.v))};
            }
        }
        u = epo;
        v = cross(epo, h.dout);
        o = h.p;
        d = h.dout;
    }
}

// Rays [first, first + n).  Every wave writes the rays it marks to its own part
// of the queue, those marked on segment 0 alone from the back: appends to a
// shared queue took 140 us, atomics on two counters.
template <bool STAGED>
__global__ __launch_bounds__(256) void coverage_walk_kernel(CovGradArgs g, MatTable mats, int64_t first, int64_t n,
                                                            CovQueue q) {
    __shared__ Shade staged[STAGED ? kWalkTris : 1];
    if (STAGED) {
        for (int i = threadIdx.x; i < g.sc.nt; i += 256) staged[i] = g.sc.shades[g.sc.leaf_of_input[i]];
        __syncthreads();
    }
    const int lane = threadIdx.x & 63;
    const int64_t wave = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6), nwaves = (int64_t)gridDim.x * 4;
    uint2* out = q.ray + wave * q.part;
    uint32_t n0 = 0, n1 = 0;
    for (int64_t base = wave * 64; base < n; base += nwaves * 64) {
        const int64_t j = first + base + lane;
        const uint32_t marks = base + lane < n ? cov_walk<STAGED>(g, mats, staged, j) : 0u;
        const uint64_t below = (1ull << lane) - 1ull;
        const uint64_t b0 = __ballot(marks == 1u), b1 = __ballot(marks > 1u);
        if (marks == 1u) out[q.part - 1 - n0 - __popcll(b0 & below)] = uint2{(uint32_t)j, marks};
        if (marks > 1u) out[n1 + __popcll(b1 & below)] = uint2{(uint32_t)j, marks};
        n0 += (uint32_t)__popcll(b0);
        n1 += (uint32_t)__popcll(b1);
    }
    if (lane == 0) q.count[wave] = uint2{n0, n1};
}

// Adds a block's sums to the outputs: wave shuffles, then the four waves through
// LDS, one fp64 atomic per block and output.
template <int NM>
__device__ __forceinline__ void cov_reduce(const CovGradArgs& g, const CovSums<NM>& acc) {
    constexpr int kOut = 2 * NM + 3;  // the region sum, (eps_r, sigma) per material, yaw, pitch
    __shared__ double red[4][kOut];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    double v[kOut];
    const double dsig = 1.0 / (kEps0 * g.omega);
    v[0] = acc.w;
#pragma unroll
    for (int m = 0; m < NM; ++m) {
        v[1 + 2 * m] = acc.eps[m];
        v[2 + 2 * m] = acc.sig[m] * dsig;
    }
    v[kOut - 2] = acc.yaw;
    v[kOut - 1] = acc.pitch;
#pragma unroll
    for (int i = 0; i < kOut; ++i) {
        for (int off = 32; off >= 1; off >>= 1) v[i] += __shfl_xor(v[i], off);
        if (lane == 0) red[wave][i] = v[i];
    }
    __syncthreads();
    if (threadIdx.x < kOut) {
        const int i = threadIdx.x;
        const double s = red[0][i] + red[1][i] + red[2][i] + red[3][i];
        if (s != 0.0) atomicAdd(g.out + i, s);
    }
}

template <int NM>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(kCovWaves, kCovWaves)))
void coverage_grad_kernel(CovGradArgs g, MatTable mats, CovQueue q) {
    const int lane = threadIdx.x & 63;
    CovSums<NM> acc{};
    const int64_t part = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const uint2* in = q.ray + part * q.part;
    const uint32_t n0 = q.count[part].x, n1 = q.count[part].y;
    for (uint32_t i = (uint32_t)lane; i < n0 + n1; i += 64) {
        const uint2 e = in[i < n1 ? (int64_t)i : q.part - 1 - (int64_t)(i - n1)];
        cov_replay<NM>(g, mats, (int64_t)e.x, e.y, acc);
    }
    cov_reduce<NM>(g, acc);
}

// The same without memory outside the caller's, for calls recorded into a graph
// (which may be replayed at any time, beside any other call) and where the queue
// cannot be had: a wave walks 64 rays at a time, collects the marked ones of
// either kind in LDS and replays them 64 at a time.  The walk runs at the
// replay's three waves per SIMD: 10^7 rays of depth 3 over the street canyon take
// 323 us, with the queue 259; 10^6 rays 48 us either way.
template <int NM>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(kCovWaves, kCovWaves)))
void coverage_grad_direct_kernel(CovGradArgs g, MatTable mats) {
    __shared__ uint2 held[4][2][128];  // per wave: marked on segment 0 alone, marked later
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    CovSums<NM> acc{};
    int n0 = 0, n1 = 0;
    for (int64_t base = ((int64_t)blockIdx.x * 4 + wave) * 64;; base += (int64_t)gridDim.x * 256) {
        const bool more = base < g.count;
        if (more) {
            const int64_t j = base + lane;
            const uint32_t marks = j < g.count ? cov_walk<false>(g, mats, nullptr, j) : 0u;
            const uint64_t below = (1ull << lane) - 1ull;
            const uint64_t b0 = __ballot(marks == 1u), b1 = __ballot(marks > 1u);
            if (marks == 1u) held[wave][0][n0 + __popcll(b0 & below)] = uint2{(uint32_t)j, marks};
            if (marks > 1u) held[wave][1][n1 + __popcll(b1 & below)] = uint2{(uint32_t)j, marks};
            n0 += __popcll(b0);
            n1 += __popcll(b1);
        }
        // full batches of one kind while there are rays to walk, then what is left
        while (n0 >= 64 || n1 >= 64 || (!more && n0 + n1 > 0)) {
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            const int kind = n1 >= 64 || n0 < n1 ? 1 : 0, have = kind ? n1 : n0, take = min(have, 64);
            uint2 e{0u, 0u};
            if (lane < take) e = held[wave][kind][have - take + lane];
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            if (kind) n1 -= take;
            else n0 -= take;
            if (e.y) cov_replay<NM>(g, mats, (int64_t)e.x, e.y, acc);
        }
        if (!more) break;
    }
    cov_reduce<NM>(g, acc);
}

}  // namespace

hipError_t launch_power_grad(const GradArgs& a, const MatTable& mats, hipStream_t s) {
    const int64_t n = (int64_t)a.nrx * a.P * kPathLanes;
    const int64_t blocks = (n + kGradBlock - 1) / kGradBlock;
    if (blocks == 0) return hipSuccess;
    hipLaunchKernelGGL(power_grad_kernel, dim3((unsigned)blocks), dim3(kGradBlock), 0, s, a, mats);
    return hipGetLastError();
}

namespace {
int64_t cov_blocks(int64_t rays, int num_cu) {
    return std::min<int64_t>((rays + 255) / 256, (int64_t)num_cu * kCovWaves);
}
int64_t cov_part(int64_t rays, int num_cu) {
    const int64_t lanes = cov_blocks(rays, num_cu) * 256;
    return (rays + lanes - 1) / lanes * 64;
}
}  // namespace

size_t coverage_grad_scratch(int64_t rays, int num_cu) {
    return (size_t)cov_blocks(rays, num_cu) * 4 * (size_t)(cov_part(rays, num_cu) + 1) * sizeof(uint2);
}

namespace {
template <int NM>
hipError_t coverage_grad_launches(const CovGradArgs& a, const MatTable& mats, int num_cu, int64_t chunk, void* scratch,
                                  hipStream_t s) {
    const dim3 threads(256);
    if (!scratch) {
        hipLaunchKernelGGL(coverage_grad_direct_kernel<NM>, dim3((unsigned)cov_blocks(a.count, num_cu)), threads, 0, s,
                           a, mats);
        return hipGetLastError();
    }
    for (int64_t first = 0; first < a.count; first += chunk) {
        const int64_t n = std::min(chunk, a.count - first), nb = cov_blocks(n, num_cu);
        CovQueue q;
        q.part = cov_part(n, num_cu);
        q.count = (uint2*)scratch;
        q.ray = q.count + nb * 4;
        const dim3 blocks((unsigned)nb);
        if (a.sc.nt <= kWalkTris)
            hipLaunchKernelGGL(coverage_walk_kernel<true>, blocks, threads, 0, s, a, mats, first, n, q);
        else
            hipLaunchKernelGGL(coverage_walk_kernel<false>, blocks, threads, 0, s, a, mats, first, n, q);
        hipLaunchKernelGGL(coverage_grad_kernel<NM>, blocks, threads, 0, s, a, mats, q);
    }
    return hipGetLastError();
}
}  // namespace

hipError_t launch_coverage_grad(const CovGradArgs& a, const MatTable& mats, int num_cu, int64_t chunk, void* scratch,
                                hipStream_t s) {
    switch (a.nm) {
        case 1: return coverage_grad_launches<1>(a, mats, num_cu, chunk, scratch, s);
        case 2: return coverage_grad_launches<2>(a, mats, num_cu, chunk, scratch, s);
        case 3: return coverage_grad_launches<3>(a, mats, num_cu, chunk, scratch, s);
        case 4: return coverage_grad_launches<4>(a, mats, num_cu, chunk, scratch, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace rt
