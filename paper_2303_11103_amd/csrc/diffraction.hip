// First-order edge diffraction for gfx950 (paper Sec. II-B lists first-order
// diffraction among the interactions of the tracer).  Per (receiver, wedge)
// pair, in fp64:
//   * diffraction point Q on the edge by Keller's law (equal angles of the
//     incident and diffracted rays with the edge), inside the edge;
//   * angles phi' (transmitter) and phi (receiver) about the edge, measured
//     from the 0-face through the exterior (0 < phi', phi < n pi);
//   * both legs unoccluded (any-hit traversals with the wedge faces skipped);
//   * uniform-theory (UTD) coefficients of a wedge with exterior angle n pi:
//       D_{s,h} = -e^{-j pi/4} / (2 n sqrt(2 pi k) sin b0) [
//           cot((pi + (phi - phi'))/2n) F(kL a+(phi - phi'))
//         + cot((pi - (phi - phi'))/2n) F(kL a-(phi - phi'))
//         + R0 cot((pi - (phi + phi'))/2n) F(kL a-(phi + phi'))
//         + Rn cot((pi + (phi + phi'))/2n) F(kL a+(phi + phi')) ]
//     with the Fresnel coefficients R0, Rn (perpendicular for D_s, parallel
//     for D_h) of the two faces at the local incidence cosines sin(b0)|sin phi'|
//     and sin(b0)|sin(n pi - phi)|, L = s' s sin^2 b0 / (s' + s);
//   * the vector field through the dyadic -b'b D_s - p'p D_h in the edge-fixed
//     unit vectors, spherical spreading sqrt(s' / (s (s + s'))).
// The transition function F(x) = 2j sqrt(x) e^{jx} int_sqrt(x)^inf e^{-j t^2} dt
// is evaluated from erfc(sqrt(x) e^{j pi/4}): the Maclaurin series of erf for
// x < 6 and Laplace's continued fraction of erfc (60 levels, evaluated from the
// tail) above; both are accurate to about 1e-14 there.
#include "traverse.h"

namespace rt {
namespace {

constexpr double kC0d = 299792458.0;
constexpr double kOccEpsD = 1e-9;

__device__ __forceinline__ d3 ldw(const double* p) { return d3{p[0], p[1], p[2]}; }
__device__ __forceinline__ cd cexpj(double t) { return cd{cos(t), sin(t)}; }

// F(x) for x >= 0.
__device__ cd transition(double x) {
    const double sx = sqrt(x);
    const cd z{sx * 0.70710678118654752440, sx * 0.70710678118654752440};  // sqrt(x) e^{j pi/4}
    if (x < 6.0) {
        // erf(z) = (2 z / sqrt(pi)) sum_n (-j x)^n / (n! (2n + 1)),  since z^2 = j x
        cd term{1.0, 0.0}, sum{0.0, 0.0};
        for (int n = 0; n < 80; ++n) {
            sum = cadd(sum, cmulr(term, 1.0 / (2 * n + 1)));
            term = cmulr(cmul(term, cd{0.0, -x}), 1.0 / (n + 1));
            if (fabs(term.re) + fabs(term.im) < 1e-18 * (fabs(sum.re) + fabs(sum.im))) break;
        }
        const cd erf = cmul(cmulr(z, 1.1283791670955126), sum);  // 2 / sqrt(pi)
        const cd erfc{1.0 - erf.re, -erf.im};
        // F = j sqrt(pi x) e^{j (x - pi/4)} erfc
        const cd ph = cexpj(x - 0.25 * kPi);
        return cmul(cd{0.0, sqrt(kPi * x)}, cmul(ph, erfc));
    }
    // erfc(z) = e^{-z^2} / sqrt(pi) K, K = 1/(z + (1/2)/(z + 1/(z + (3/2)/(z + ...)))),
    // so F = j sqrt(x) e^{-j pi/4} K (the e^{jx} of F cancels e^{-z^2} = e^{-jx})
    cd t = z;
    for (int m = 60; m >= 1; --m) t = cadd(z, cdiv(cd{0.5 * m, 0.0}, t));
    const cd K = cdiv(cd{1.0, 0.0}, t);
    return cmul(cd{0.0, sx}, cmul(cd{0.70710678118654752440, -0.70710678118654752440}, K));
}

// cot((pi + sign b)/(2n)) F(kL a^sign(b)); on a shadow boundary (infinite
// cotangent, vanishing F) the limit n sqrt(2 pi kL) sgn(eps) e^{j pi/4}.
__device__ cd utd_term(double kL, double n, double b, double sign) {
    const double arg = (kPi + sign * b) / (2.0 * n);
    const double N = rint((b + sign * kPi) / (2.0 * kPi * n));
    const double c = cos((2.0 * kPi * n * N - b) / 2.0);
    const double a = 2.0 * c * c;
    const double sn = sin(arg);
    if (fabs(sn) < 1e-12) {
        const double Nb = rint((kPi + sign * b) / (2.0 * kPi * n));
        const double eps = (kPi + sign * b) - 2.0 * kPi * n * Nb;
        const double m = n * sqrt(2.0 * kPi * kL) * (eps >= 0.0 ? 1.0 : -1.0);
        return cd{m * 0.70710678118654752440, m * 0.70710678118654752440};
    }
    return cmulr(transition(kL * a), cos(arg) / sn);
}

__device__ __forceinline__ double angle_about(const Wedge& w, d3 X, d3 Q) {
    const d3 u = sub(X, Q);
    double ph = atan2(dot(u, ldw(w.n0)), dot(u, ldw(w.t0)));
    if (ph < 0.0) ph += 2.0 * kPi;
    return ph;
}

__device__ __forceinline__ void face_fresnel(const MatTable& mats, int m, double cos_i, cd& rs, cd& rh) {
    fresnel(mats.m[m], cos_i, rs, rh);
}

// The path over a wedge from S to P: diffraction point and the two angles
// about the edge.
struct EdgePoint {
    d3 Q;
    double phip, phi;
};

// False when the pair has no diffraction point inside the edge or either end
// lies outside the wedge's exterior.
__device__ __forceinline__ bool edge_point(const Wedge& w, d3 S, d3 P, EdgePoint& ep) {
    const d3 A = ldw(w.a), e = ldw(w.e);
    // Keller point: axial coordinates and distances from the edge line
    const double zs = dot(sub(S, A), e), zp = dot(sub(P, A), e);
    const double rs = norm(sub(sub(S, A), scale(e, zs))), rp = norm(sub(sub(P, A), scale(e, zp)));
    if (rs < 1e-9 || rp < 1e-9) return false;
    const double z = zs + (zp - zs) * rs / (rs + rp);
    if (!(z > 0.0 && z < w.len)) return false;
    ep.Q = add(A, scale(e, z));
    ep.phip = angle_about(w, S, ep.Q);
    ep.phi = angle_about(w, P, ep.Q);
    const double lim = w.n * kPi;
    return ep.phip > 0.0 && ep.phip < lim && ep.phi > 0.0 && ep.phi < lim;
}

// A leg of the path (open segment, the two wedge faces skipped) is blocked.
template <int BS, bool OVF>
__device__ __forceinline__ bool leg_blocked(const DevScene& sc, const Node* lds_nodes, int n_lds,
                                            int32_t (*stack)[BS], d3 from, d3 to, const Wedge& w) {
    double tb = 1.0;
    return traverse<true, false, BS, OVF>(sc, lds_nodes, n_lds, from, sub(to, from), w.face0, w.facen, kOccEpsD, tb,
                                          stack) >= 0;
}

// FULL also fills the transfer matrix and the directions; otherwise only the
// coefficient a.
struct DiffPath {
    cd a;
    cd T[4];
    double len;
    d3 s_in, s_out;
};

template <bool FULL>
__device__ void diffracted_path(const MatTable& mats, double lambda, d3 S, const Antenna& txa, d3 P,
                                const Antenna& rxa, const Wedge& w, const EdgePoint& pt, DiffPath& out) {
    const d3 e = ldw(w.e), Q = pt.Q;
    const double phip = pt.phip, phi = pt.phi, lim = w.n * kPi;
    // coefficients
    const double k = 2.0 * kPi / lambda;
    const d3 vin = sub(Q, S), vout = sub(P, Q);
    const double sp = norm(vin), s = norm(vout);
    const d3 sin_ = scale(vin, 1.0 / sp), sout = scale(vout, 1.0 / s);
    const double cb = fmin(fmax(dot(sin_, e), -1.0), 1.0);
    const double b0 = acos(cb);
    const double sb = sin(b0);
    const double L = sp * s * sb * sb / (sp + s);
    cd r0s, r0h, rns, rnh;
    face_fresnel(mats, w.mat0, sb * fabs(sin(phip)), r0s, r0h);
    face_fresnel(mats, w.matn, sb * fabs(sin(lim - phi)), rns, rnh);
    const double kL = k * L;
    const cd t1 = utd_term(kL, w.n, phi - phip, 1.0);
    const cd t2 = utd_term(kL, w.n, phi - phip, -1.0);
    const cd t3 = utd_term(kL, w.n, phi + phip, -1.0);
    const cd t4 = utd_term(kL, w.n, phi + phip, 1.0);
    // -e^{-j pi/4} / (2 n sqrt(2 pi k) sin b0)
    const double pm = -1.0 / (2.0 * w.n * sqrt(2.0 * kPi * k) * sb);
    const cd pre{pm * 0.70710678118654752440, -pm * 0.70710678118654752440};
    const cd t12 = cadd(t1, t2);
    const cd Ds = cmul(pre, cadd(t12, cadd(cmul(r0s, t3), cmul(rns, t4))));
    const cd Dh = cmul(pre, cadd(t12, cadd(cmul(r0h, t3), cmul(rnh, t4))));
    // edge-fixed unit vectors
    const d3 t0 = ldw(w.t0), n0 = ldw(w.n0);
    const d3 ph_in = add(scale(t0, -sin(phip)), scale(n0, cos(phip)));
    const d3 ph_out = add(scale(t0, -sin(phi)), scale(n0, cos(phi)));
    const d3 be_in = cross(ph_in, sin_), be_out = cross(ph_out, sout);
    // E_out = -Ds be_out (be_in . E) - Dh ph_out (ph_in . E); u . Dbar . v
    auto dyad = [&](d3 u, d3 v) {
        return csub(cmulr(Ds, -dot(u, be_out) * dot(be_in, v)), cmulr(Dh, dot(u, ph_out) * dot(ph_in, v)));
    };
    const double amp = 1.0 / sqrt(sp * s * (sp + s));
    const d3 Ft = antenna_field(txa, sin_);
    const d3 Fr = antenna_field(rxa, scale(sout, -1.0));
    out.a = cmulr(dyad(Fr, Ft), lambda / (4.0 * kPi) * amp);
    if (FULL) {
        // spherical unit vectors of s_in (departure) and s_out (direction of travel on arrival)
        auto basis = [](d3 d, d3& th, d3& ph) {
            const double rho = sqrt(d.x * d.x + d.y * d.y);
            double cp = 1.0, spn = 0.0;
            if (rho > 0.0) {
                cp = d.x / rho;
                spn = d.y / rho;
            }
            th = d3{d.z * cp, d.z * spn, -rho};
            ph = d3{-spn, cp, 0.0};
        };
        d3 thi, phi_i, tho, pho;
        basis(sin_, thi, phi_i);
        basis(sout, tho, pho);
        const double tsc = (sp + s) * amp;
        out.T[0] = cmulr(dyad(tho, thi), tsc);
        out.T[1] = cmulr(dyad(tho, phi_i), tsc);
        out.T[2] = cmulr(dyad(pho, thi), tsc);
        out.T[3] = cmulr(dyad(pho, phi_i), tsc);
        out.len = sp + s;
        out.s_in = sin_;
        out.s_out = sout;
    }
}

// Diffracted paths of a range of receivers in three passes, because a pair that
// has a path is rare (1 in 8,000 of a city's 133 million) and every step before
// it drops most pairs: one thread per pair through all steps kept a few lanes of
// each wave busy (30.4 ms for 1024 receivers and 129,768 wedges).

// Pass 1: 256 wedges per block against 64 receivers.  Keeps a pair unless it
// surely has no diffraction point inside the edge or its receiver surely lies
// inside the solid: axial and radial distances in fp32 of differences taken in
// fp64, against bounds 4e-6 (8 times the worst rounding) of their products.
// The transmitter's side is tested once per wedge.  Each thread gathers its
// wedge's receivers in a 64-bit mask, so the queue takes one atomic per block.
// `room` stands with the integers, which are loaded at the start: behind the
// pointers its load came into the serial step at the end (182 -> 190 us).
constexpr int kDiffRx = 64, kDiffSpill = kDiffRx * kBlock;  // entries behind the queue for a block without room
__global__ __launch_bounds__(kBlock) void diffraction_filter_kernel(PathArgs a, int32_t r0, int32_t r1,
                                                                    int32_t wedge_tiles, uint32_t room,
                                                                    uint32_t* __restrict__ queue,
                                                                    uint32_t* __restrict__ count) {
    __shared__ double rx[kDiffRx][3];
    __shared__ uint32_t wave_n[kBlock / 64];
    __shared__ uint32_t start;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int rb = r0 + (int)(blockIdx.x / wedge_tiles) * kDiffRx, nr = min(kDiffRx, r1 - rb);
    for (int i = tid; i < 3 * nr; i += kBlock) rx[i / 3][i % 3] = a.rx[3 * (int64_t)rb + i];
    __syncthreads();
    const int wi = (int)(blockIdx.x % wedge_tiles) * kBlock + tid;
    uint64_t keep = 0;
    if (wi < a.sc.num_wedges) {
        const Wedge w = a.sc.wedges[wi];
        const double lim = w.n * kPi;
        const float sl = (float)sin(lim), cl = (float)cos(lim), len = (float)w.len;
        const f3 e{(float)w.e[0], (float)w.e[1], (float)w.e[2]};
        const f3 t0{(float)w.t0[0], (float)w.t0[1], (float)w.t0[2]}, n0{(float)w.n0[0], (float)w.n0[1], (float)w.n0[2]};
        auto split = [&](double x, double y, double z, float& ax, float& rad, bool& outside) {
            const f3 d{(float)(x - w.a[0]), (float)(y - w.a[1]), (float)(z - w.a[2])};
            ax = dot(d, e);
            const f3 q{d.x - ax * e.x, d.y - ax * e.y, d.z - ax * e.z};
            rad = sqrtf(dot(q, q));
            // exterior: in front of the 0-face's plane or of the n-face's
            const float u0 = dot(d, t0), u1 = dot(d, n0), tol = -4e-6f * (fabsf(ax) + rad);
            outside = !(u1 < tol && u0 * sl - u1 * cl < tol);
        };
        float zs, rs;
        bool out_s;
        split(a.tx[0], a.tx[1], a.tx[2], zs, rs, out_s);
        if (out_s) {
            const float s0 = 4e-6f * (fabsf(zs) + rs + len);
            for (int r = 0; r < nr; ++r) {
                float zp, rp;
                bool out_p;
                split(rx[r][0], rx[r][1], rx[r][2], zp, rp, out_p);
                // 0 < z < len for z = (zs rp + zp rs) / (rs + rp)
                const float tol = s0 * (fabsf(zp) + rp + len);
                const bool no_point = zs * rp + zp * rs < -tol || (zs - len) * rp + (zp - len) * rs > tol;
                if (out_p && !no_point) keep |= 1ull << r;
            }
        }
    }
    const uint32_t n = (uint32_t)__popcll(keep);
    uint32_t incl = n;
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t v = __shfl_up(incl, off);
        if (lane >= off) incl += v;
    }
    if (lane == 63) wave_n[wv] = incl;
    __syncthreads();
    if (tid == 0) {
        uint32_t sum = 0;
        for (int i = 0; i < kBlock / 64; ++i) {
            const uint32_t c = wave_n[i];
            wave_n[i] = sum;
            sum += c;
        }
        start = sum ? atomicAdd(count, sum) : 0u;
        if (sum > room || start > room - sum) start = room;  // behind the queue: none of it is read then
    }
    __syncthreads();
    uint32_t at = start + wave_n[wv] + incl - n;
    while (keep) {
        const int r = __ffsll((long long)keep) - 1;
        keep &= keep - 1;
        queue[at++] = (uint32_t)(rb - r0 + r) * (uint32_t)a.sc.num_wedges + (uint32_t)wi;
    }
}

// Wedge and receiver position of queue entry `it` = (receiver - r0) * wedges + wedge.
__device__ __forceinline__ Wedge load_pair(const PathArgs& a, int32_t r0, uint32_t it, d3& P) {
    const double* rx = a.rx + 3 * ((int64_t)r0 + it / (uint32_t)a.sc.num_wedges);
    P = d3{rx[0], rx[1], rx[2]};
    return a.sc.wedges[it % (uint32_t)a.sc.num_wedges];
}

// Pass 2: the exact tests in fp64, then the leg to the receiver, then, for the
// survivors, the leg from the transmitter.  A wave collects survivors of the
// first leg in LDS until it has 64, so that the second leg runs with full waves
// too.  The first leg is traversed from the receiver: what blocks it mostly
// stands in the receiver's street, and boxes are visited by distance from the
// start.  Bound by the any-hit traversals: 0.51 ms for the pairs of 1024 street
// receivers and 129,768 wedges of a city (0.76 ms from the wedge, 0.94 ms with
// the transmitter's leg first, 1.40 ms that way with 12 instead of 16 waves per
// CU; blocks of 512 with 64 staged nodes leave room for two per CU).
constexpr int kLegBlock = 512, kLegNodes = 64;
template <bool OVF>
__global__ __launch_bounds__(kLegBlock) void diffraction_legs_kernel(PathArgs a, int32_t r0, uint32_t room,
                                                                     uint32_t out_room,
                                                                     const uint32_t* __restrict__ queue,
                                                                     const uint32_t* __restrict__ count,
                                                                     uint32_t* __restrict__ out,
                                                                     uint32_t* __restrict__ out_count) {
    __shared__ int32_t stack[kStack][kLegBlock];
    __shared__ Node lds_nodes[kLegNodes];
    __shared__ uint32_t held[kLegBlock / 64][128];
    const int n_lds = stage_nodes<kLegNodes>(a.sc, lds_nodes);
    const int lane = threadIdx.x & 63;
    uint32_t* mine = held[threadIdx.x >> 6];
    const d3 S{a.tx[0], a.tx[1], a.tx[2]};
    const int64_t n = *count > room ? 0 : (int64_t)*count;
    const int64_t nwaves = (int64_t)gridDim.x * (kLegBlock / 64);
    int have = 0;  // survivors of the first leg in `mine` (the same in every lane)
    auto second_leg = [&](int take) {
        bool ok = false;
        uint32_t it = 0u;
        if (lane < take) {
            it = mine[have - take + lane];
            d3 P;
            const Wedge w = load_pair(a, r0, it, P);
            EdgePoint pt;
            ok = edge_point(w, S, P, pt) && !leg_blocked<kLegBlock, OVF>(a.sc, lds_nodes, n_lds, stack, S, pt.Q, w);
        }
        have -= take;
        const uint64_t m = __ballot(ok);
        if (m) {
            uint32_t b = 0;
            if (lane == 0) b = atomicAdd(out_count, (uint32_t)__popcll(m));
            b = __builtin_amdgcn_readfirstlane(b);
            if (b + (uint32_t)__popcll(m) <= out_room && ok) out[b + __popcll(m & ((1ull << lane) - 1ull))] = it;
        }
    };
    for (int64_t base = ((int64_t)blockIdx.x * (kLegBlock / 64) + (threadIdx.x >> 6)) * 64; base < n; base += nwaves * 64) {
        bool ok = false;
        uint32_t it = 0u;
        if (base + lane < n) {
            it = queue[base + lane];
            d3 P;
            const Wedge w = load_pair(a, r0, it, P);
            EdgePoint pt;
            ok = edge_point(w, S, P, pt) && !leg_blocked<kLegBlock, OVF>(a.sc, lds_nodes, n_lds, stack, P, pt.Q, w);
        }
        const uint64_t m = __ballot(ok);
        if (ok) mine[have + __popcll(m & ((1ull << lane) - 1ull))] = it;
        have += __popcll(m);
        if (have >= 64) second_leg(64);
    }
    if (have) second_leg(have);
}

// Pass 3: coefficients of the pairs that have a path.  count: pairs that passed
// the filter and pairs that passed the legs; where more than fitted their queue,
// the first receiver's count says so and nothing of the queue is read.
__global__ __launch_bounds__(kBlock) void diffraction_paths_kernel(PathArgs a, MatTable mats, int32_t r0,
                                                                   const uint32_t* __restrict__ queue,
                                                                   uint32_t filter_room, uint32_t room,
                                                                   const uint32_t* __restrict__ count) {
    const d3 S{a.tx[0], a.tx[1], a.tx[2]};
    const bool over = count[0] > filter_room || count[1] > room;
    if (over && blockIdx.x == 0 && threadIdx.x == 0) a.counts[r0] = 0x80000000u;
    const uint32_t n = over ? 0u : count[1];
    for (uint32_t item = blockIdx.x * kBlock + threadIdx.x; item < n; item += gridDim.x * kBlock) {
        const int r = r0 + (int)(queue[item] / (uint32_t)a.sc.num_wedges);
        const int wi = (int)(queue[item] % (uint32_t)a.sc.num_wedges);
        d3 P;
        const Wedge w = load_pair(a, r0, queue[item], P);
        EdgePoint pt;
        if (!edge_point(w, S, P, pt)) continue;
        const uint32_t slot = atomicAdd(a.counts + r, 1u);
        if (slot >= (uint32_t)a.P) continue;
        DiffPath p;
        diffracted_path<true>(mats, a.lambda, S, a.tx_ant, P, a.rx_ant[r], w, pt, p);
        const int64_t at = (int64_t)r * a.P + slot;
        a.a[2 * at] = (float)p.a.re;
        a.a[2 * at + 1] = (float)p.a.im;
        float* T = a.T + 8 * at;
        for (int i = 0; i < 4; ++i) {
            T[2 * i] = (float)p.T[i].re;
            T[2 * i + 1] = (float)p.T[i].im;
        }
        a.tau[at] = (float)(p.len / kC0d);
        a.aod[2 * at] = (float)acos(fmin(fmax(p.s_in.z, -1.0), 1.0));
        a.aod[2 * at + 1] = (float)atan2(p.s_in.y, p.s_in.x);
        a.aoa[2 * at] = (float)acos(fmin(fmax(-p.s_out.z, -1.0), 1.0));
        a.aoa[2 * at + 1] = (float)atan2(-p.s_out.y, -p.s_out.x);
        a.depth[at] = 1;
        a.faces[at] = wi;
    }
}

// Diffraction part of a coverage map: one thread per cell adds the path gain
// |a|^2 of every wedge's diffracted path to the cell centre (fixed wedge
// order, so the sum is deterministic).
__global__ __launch_bounds__(kBlock) void coverage_diffraction_kernel(DevScene sc, MatTable mats, double lambda,
                                                                      d3 S, Antenna txa, Antenna rxa, double gx0,
                                                                      double gy0, double gcell, double gz,
                                                                      int32_t gnx, int64_t cells,
                                                                      float* __restrict__ gain) {
    __shared__ int32_t stack[kStack][kBlock];
    __shared__ Node lds_nodes[kLdsNodes];
    const int n_lds = stage_nodes(sc, lds_nodes);
    for (int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; c < cells;
         c += (int64_t)gridDim.x * blockDim.x) {
        const int64_t iy = c / gnx, ix = c - iy * gnx;
        const d3 P{gx0 + ((double)ix + 0.5) * gcell, gy0 + ((double)iy + 0.5) * gcell, gz};
        double acc = 0.0;
        for (int wi = 0; wi < sc.num_wedges; ++wi) {
            const Wedge w = sc.wedges[wi];
            EdgePoint pt;
            if (!edge_point(w, S, P, pt) || leg_blocked<kBlock, true>(sc, lds_nodes, n_lds, stack, S, pt.Q, w) ||
                leg_blocked<kBlock, true>(sc, lds_nodes, n_lds, stack, pt.Q, P, w))
                continue;
            DiffPath p;
            diffracted_path<false>(mats, lambda, S, txa, P, rxa, w, pt, p);
            acc += p.a.re * p.a.re + p.a.im * p.a.im;
        }
        gain[c] += (float)acc;
    }
}

}  // namespace

hipError_t launch_coverage_diffraction(const DevScene& sc, const MatTable& mats, double lambda, const double* tx,
                                      const Antenna& txa, const Antenna& rxa, double gx0, double gy0, double gcell,
                                      double gz, int32_t gnx, int32_t gny, float* gain, hipStream_t s) {
    const int64_t cells = (int64_t)gnx * gny;
    if (cells <= 0 || sc.num_wedges <= 0) return hipSuccess;
    const int64_t blocks = std::min<int64_t>((cells + kBlock - 1) / kBlock, 16384);
    hipLaunchKernelGGL(coverage_diffraction_kernel, dim3((unsigned)blocks), dim3(kBlock), 0, s, sc, mats, lambda,
                       d3{tx[0], tx[1], tx[2]}, txa, rxa, gx0, gy0, gcell, gz, gnx, cells, gain);
    return hipGetLastError();
}

DiffPlan diffraction_plan(int64_t nrx, int64_t num_wedges, int64_t most) {
    DiffPlan p{0, 0, 0};
    if (nrx <= 0 || num_wedges <= 0) return p;
    p.chunk = std::max<int64_t>(1, most / num_wedges);
    p.chunk = std::min<int64_t>(nrx, p.chunk > kDiffRx ? p.chunk / kDiffRx * kDiffRx : p.chunk);
    const int64_t pairs = p.chunk * num_wedges;
    const bool part = pairs > kDiffWholePairs && p.chunk >= 8;
    p.filtered = part ? pairs / 4 : pairs;
    p.clear = part ? pairs / 8 : pairs;
    return p;
}

DiffPlan diffraction_sure(const DiffPlan& p, int64_t num_wedges) {
    const int64_t chunk = std::min(p.chunk, (p.filtered + p.clear) / 2 / std::max<int64_t>(1, num_wedges));
    return DiffPlan{chunk, chunk * num_wedges, chunk * num_wedges};
}

size_t diffraction_scratch(const DiffPlan& p) {
    return p.chunk ? 256 + (size_t)(p.filtered + kDiffSpill + p.clear) * sizeof(uint32_t) : 0;
}

hipError_t launch_diffraction_paths(const PathArgs& a, const MatTable& mats, const DiffPlan& plan, void* scratch,
                                    hipStream_t s) {
    const int64_t nw = a.sc.num_wedges;
    if (a.nrx <= 0 || nw <= 0) return hipSuccess;
    const int64_t chunk = plan.chunk;
    const uint32_t room0 = (uint32_t)plan.filtered, room1 = (uint32_t)plan.clear;
    uint32_t* count = (uint32_t*)scratch;
    uint32_t* q0 = (uint32_t*)((char*)scratch + 256);
    uint32_t* q1 = q0 + plan.filtered + kDiffSpill;
    for (int64_t r0 = 0; r0 < a.nrx; r0 += chunk) {
        const int64_t r1 = std::min<int64_t>(a.nrx, r0 + chunk), pairs = (r1 - r0) * nw;
        hipError_t e = launch_fill_u32(count, 0u, 2, s);
        if (e != hipSuccess) return e;
        const int64_t wt = (nw + kBlock - 1) / kBlock, rt = (r1 - r0 + kDiffRx - 1) / kDiffRx;
        hipLaunchKernelGGL(diffraction_filter_kernel, dim3((unsigned)(wt * rt)), dim3(kBlock), 0, s, a, (int32_t)r0,
                           (int32_t)r1, (int32_t)wt, room0, q0, count);
        // two blocks of 76 KB per CU for the traversals
        const dim3 grid((unsigned)std::min<int64_t>((pairs + kLegBlock - 1) / kLegBlock, 256 * 2));
        if (a.sc.stack_need > kStack)
            hipLaunchKernelGGL(diffraction_legs_kernel<true>, grid, dim3(kLegBlock), 0, s, a, (int32_t)r0, room0, room1,
                               q0, count, q1, count + 1);
        else
            hipLaunchKernelGGL(diffraction_legs_kernel<false>, grid, dim3(kLegBlock), 0, s, a, (int32_t)r0, room0, room1,
                               q0, count, q1, count + 1);
        hipLaunchKernelGGL(diffraction_paths_kernel, dim3((unsigned)std::min<int64_t>((pairs + kBlock - 1) / kBlock, 512)),
                           dim3(kBlock), 0, s, a, mats, (int32_t)r0, q1, room0, room1, count);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace rt
