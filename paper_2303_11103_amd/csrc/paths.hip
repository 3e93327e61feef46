// Image-method kernels for gfx950 (paper Sec. II-B: for every candidate, an
// ordered list of scene primitives found by the shooting rays, the image
// method gives the specular path through the same primitives that ends
// exactly at the receiver; duplicates are removed, line of sight is added;
// Sec. II-A: paths are returned as coefficients and delays).
//
// Candidates are the distinct face sequences stored in the prefix table
// filled by the shoot-and-bounce kernels.  For every (receiver, candidate)
// pair, in fp64: images, back-traced reflection points, validity (segment
// parameter, front side, point inside the face); for the valid ones occlusion
// of every segment by an any-hit BVH traversal, then the field transfer
// through the Fresnel reflections and the receive pattern.
#include <algorithm>

#include "traverse.h"

namespace rt {
namespace {

constexpr int kMaxK = 8;
constexpr double kC0 = 299792458.0;
constexpr double kOccEps = 1e-9;     // open-segment parameter range (eps, 1 - eps)
constexpr double kInFaceTol = 1e-9;  // [m]

__global__ void extract_candidates_kernel(const uint64_t* __restrict__ table, uint64_t cap, int32_t max_depth,
                                          Cand* __restrict__ out, uint32_t* count, uint32_t max_out) {
    uint64_t s = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= cap) return;
    uint64_t key = table[s];
    if (key == kEmptyKey) return;
    Cand c;
    int faces_rev[kMaxK];
    int k = 0;
    while (true) {
        faces_rev[k++] = (int32_t)(uint32_t)(key & 0xffffffffull);
        int64_t parent = (int64_t)(key >> 32) - 1;
        if (parent < 0 || k >= kMaxK) break;
        key = table[parent];
    }
    c.depth = k;
    for (int i = 0; i < kMaxK; ++i) c.faces[i] = i < k ? faces_rev[k - 1 - i] : -1;
    uint32_t at = atomicAdd(count, 1u);
    if (at < max_out) out[at] = c;
}

// Reception-sphere pairs: every (receiver, prefix slot) of the pair set
// becomes a candidate (face sequence rebuilt from the prefix table) tied to
// its receiver.
__global__ void extract_pairs_kernel(const uint64_t* __restrict__ pairs, uint64_t pairs_cap,
                                     const uint64_t* __restrict__ table, Cand* __restrict__ out,
                                     int32_t* __restrict__ out_rx, uint32_t* count, uint32_t max_out) {
    const uint64_t s = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= pairs_cap) return;
    const uint64_t pk = pairs[s];
    if (pk == kEmptyKey) return;
    const int32_t r = (int32_t)(pk >> 32);
    const int32_t slot = (int32_t)(uint32_t)(pk & 0xffffffffull);
    int faces_rev[kMaxK];
    int k = 0;
    uint64_t key = table[slot];
    while (true) {
        faces_rev[k++] = (int32_t)(uint32_t)(key & 0xffffffffull);
        const int64_t parent = (int64_t)(key >> 32) - 1;
        if (parent < 0 || k >= kMaxK) break;
        key = table[parent];
    }
    Cand c;
    c.depth = k;
    for (int i = 0; i < kMaxK; ++i) c.faces[i] = i < k ? faces_rev[k - 1 - i] : -1;
    const uint32_t at = atomicAdd(count, 1u);
    if (at < max_out) {
        out[at] = c;
        out_rx[at] = r;
    }
}

__device__ __forceinline__ d3 ld3(const double* p) { return d3{p[0], p[1], p[2]}; }

__device__ __forceinline__ void sph_basis(d3 d, d3& th, d3& ph) {
    double rho = sqrt(d.x * d.x + d.y * d.y);
    double cp = 1.0, sp = 0.0;
    if (rho > 0.0) {
        cp = d.x / rho;
        sp = d.y / rho;
    }
    th = d3{d.z * cp, d.z * sp, -rho};
    ph = d3{-sp, cp, 0.0};
}

struct c3 {
    cd x, y, z;
};
__device__ __forceinline__ cd cdot(c3 a, d3 b) {
    return cd{a.x.re * b.x + a.y.re * b.y + a.z.re * b.z, a.x.im * b.x + a.y.im * b.y + a.z.im * b.z};
}
__device__ __forceinline__ c3 reflect_field(c3 E, d3 ep, d3 eli, d3 elr, cd rp, cd rl) {
    cd ap = cmul(rp, cdot(E, ep)), al = cmul(rl, cdot(E, eli));
    return c3{cadd(cmulr(ap, ep.x), cmulr(al, elr.x)), cadd(cmulr(ap, ep.y), cmulr(al, elr.y)),
              cadd(cmulr(ap, ep.z), cmulr(al, elr.z))};
}

// X lies in a triangle of face f, edges widened by kInFaceTol.  Coplanar walls
// of a street are one face, so the next triangle is fetched while one is
// tested, and the distance is compared as squares.
__device__ bool in_face(const DevScene& sc, int f, d3 X) {
    const int32_t* list = sc.face_tris + sc.faces[f].first;
    const int count = sc.faces[f].count;
    if (count <= 0) return false;
    d3 w0, w1, w2;
    auto fetch = [&](int i) {
        const Tri* t = sc.tris + list[i];
        w0 = ld3(t->v0);
        w1 = ld3(t->e1);
        w2 = ld3(t->e2);
    };
    fetch(0);
    for (int i = 0; i < count; ++i) {
        const d3 v0 = w0, e1 = w1, e2 = w2;
        if (i + 1 < count) fetch(i + 1);
        const d3 n = cross(e1, e2);
        const double nn = dot(n, n);
        const d3 v1 = add(v0, e1), v2 = add(v0, e2);
        auto inside = [&](d3 a, d3 b) {
            const d3 e = sub(b, a);
            const double c = dot(cross(e, sub(X, a)), n);  // distance times |n| |e|
            return c >= 0.0 || c * c <= (kInFaceTol * kInFaceTol) * nn * dot(e, e);
        };
        if (inside(v0, v1) && inside(v1, v2) && inside(v2, v0)) return true;
    }
    return false;
}

// The image method runs in three passes over queues: one (receiver, candidate)
// pair in a hundred has reflection points inside its faces, and one thread per
// pair through all steps ended with the longest chain of traversals in a wave
// that kept a few lanes busy.  D is the depth the arrays are sized for (a call's
// max_depth rounded up), so that unrolled loops keep them in registers; points
// beyond the last reflection hold the receiver.  All passes are chains of
// dependent loads and fp64 arithmetic on a chip that is far from full.  256
// receivers x 774 candidates of the street canyon: 228 -> 86 us (55 filter, 19
// legs, 12 coefficients); 4096 receivers of a city with their own candidates:
// 309 -> 126 us.

// Receiver and candidate of an item: every candidate for every receiver, each
// receiver's line of sight first, or (pair mode) the line of sight of every
// receiver followed by the receiver-tied candidates.
template <int D>
struct ImageItem {
    int r = 0, K = 0;
    int fc[D];
};

template <int D>
__device__ __forceinline__ bool image_item(const PathArgs& a, int64_t item, ImageItem<D>& it) {
    int64_t c;
    if (a.pair_rx) {
        it.r = item < a.nrx ? (int)item : a.pair_rx[item - a.nrx];
        c = item < a.nrx ? -1 : item - a.nrx;
    } else {
        const int64_t per_rx = (int64_t)(*a.ncand) + 1;
        it.r = item < (int64_t(1) << 32) ? (int)((uint32_t)item / (uint32_t)per_rx) : (int)(item / per_rx);
        c = item - (int64_t)it.r * per_rx - 1;
    }
    it.K = c >= 0 ? a.cands[c].depth : 0;
    if (it.K > a.max_depth) return false;
#pragma unroll
    for (int i = 0; i < D; ++i) it.fc[i] = i < it.K ? a.cands[c].faces[i] : -1;
    return true;
}

// Reflection points X[1..K] from the images of the transmitter (X[0]), traced
// back from the receiver.  CHECK: false when a point does not exist, lies
// outside its face, or its neighbours lie on different sides.
template <int D, bool CHECK>
__device__ __forceinline__ bool image_points(const PathArgs& a, const ImageItem<D>& it, d3 (&X)[D + 2]) {
    const d3 rx = ld3(a.rx + 3 * it.r);
    d3 I[D + 1];
    I[0] = d3{a.tx[0], a.tx[1], a.tx[2]};
    X[0] = I[0];
    X[D + 1] = rx;
#pragma unroll
    for (int k = 1; k <= D; ++k)
        if (k <= it.K) {
            const Face& F = a.sc.faces[it.fc[k - 1]];
            const d3 n = ld3(F.n), q = ld3(F.q);
            I[k] = sub(I[k - 1], scale(n, 2.0 * dot(sub(I[k - 1], q), n)));
        }
    bool valid = true;
#pragma unroll
    for (int k = D; k >= 1; --k) {
        X[k] = rx;
        if (k <= it.K && valid) {
            const Face& F = a.sc.faces[it.fc[k - 1]];
            const d3 n = ld3(F.n), q = ld3(F.q);
            const d3 A = X[k + 1];
            const double den = dot(sub(I[k], A), n);
            const double t = dot(sub(q, A), n) / den;
            if (CHECK && (den == 0.0 || !(t > 0.0 && t < 1.0))) valid = false;
            X[k] = add(A, scale(sub(I[k], A), t));
        }
    }
    if (!CHECK) return true;
#pragma unroll
    for (int k = 1; k <= D; ++k)
        if (k <= it.K && valid) {
            const Face& F = a.sc.faces[it.fc[k - 1]];
            const d3 n = ld3(F.n), q = ld3(F.q);
            const double sp = dot(sub(X[k - 1], q), n), sn = dot(sub(X[k + 1], q), n);
            if (!(sp * sn > 0.0)) valid = false;
            else if (!in_face(a.sc, it.fc[k - 1], X[k])) valid = false;
        }
    return valid;
}

// Pass 1: items [first, first + n) whose points exist, as offsets from first.
template <int D>
__global__ __launch_bounds__(kBlock) void image_filter_kernel(PathArgs a, int64_t first, int64_t n,
                                                              uint32_t* __restrict__ queue,
                                                              uint32_t* __restrict__ blocked,
                                                              uint32_t* __restrict__ count) {
    const int64_t at = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    bool ok = false;
    if (at < n) {
        ImageItem<D> it;
        d3 X[D + 2];
        ok = image_item<D>(a, first + at, it) && image_points<D, true>(a, it, X);
    }
    const int lane = threadIdx.x & 63;
    const uint64_t m = __ballot(ok);
    if (!m) return;
    uint32_t b = 0;
    if (lane == 0) b = atomicAdd(count, (uint32_t)__popcll(m));
    b = __shfl(b, 0) + __popcll(m & ((1ull << lane) - 1ull));
    if (ok) {
        queue[b] = (uint32_t)at;
        blocked[b] = 0u;
    }
}

// Pass 2: one thread per queued item and segment; a blocked segment marks the
// item.
template <int D>
__global__ __launch_bounds__(kBlock) void image_legs_kernel(PathArgs a, int64_t first,
                                                            const uint32_t* __restrict__ queue,
                                                            uint32_t* __restrict__ blocked,
                                                            const uint32_t* __restrict__ count) {
    __shared__ int32_t stack[kStack][kBlock];
    __shared__ Node lds_nodes[kLdsNodes];
    const int segs = a.max_depth + 1;
    const int64_t total = (int64_t)(*count) * segs;
    if ((int64_t)blockIdx.x * kBlock >= total) return;
    const int n_lds = stage_nodes(a.sc, lds_nodes);
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < total; i += (int64_t)gridDim.x * kBlock) {
        const uint32_t e = (uint32_t)(i / segs);
        const int k = (int)(i - (int64_t)e * segs);
        ImageItem<D> it;
        image_item<D>(a, first + queue[e], it);
        if (k > it.K) continue;
        d3 X[D + 2];
        image_points<D, false>(a, it, X);
        d3 from = X[0], to = X[1];
        int ea = -1, eb = it.K ? it.fc[0] : -1;
#pragma unroll
        for (int j = 1; j <= D; ++j)
            if (j == k) {
                from = X[j];
                to = X[j + 1];
                ea = it.fc[j - 1];
                eb = -1;
                if (j < D && j < it.K) eb = it.fc[j < D ? j : 0];
            }
        double tb = 1.0;
        if (traverse<true>(a.sc, lds_nodes, n_lds, from, sub(to, from), ea, eb, kOccEps, tb, stack) >= 0)
            blocked[e] = 1u;
    }
}

// Pass 3: coefficients of the items with no blocked segment.
constexpr int kImageBlock = 64;
template <int D>
__global__ __launch_bounds__(kImageBlock) void image_paths_kernel(PathArgs a, MatTable mats, int64_t first,
                                                                  const uint32_t* __restrict__ queue,
                                                                  const uint32_t* __restrict__ blocked,
                                                                  const uint32_t* __restrict__ count) {
    const uint32_t n = *count;
    for (uint32_t e = blockIdx.x * kImageBlock + threadIdx.x; e < n; e += gridDim.x * kImageBlock) {
        if (blocked[e]) continue;
        ImageItem<D> it;
        image_item<D>(a, first + queue[e], it);
        d3 X[D + 2];
        image_points<D, false>(a, it, X);
        d3 dir[D + 1];
        d3 dK{0.0, 0.0, 0.0};
        double L = 0.0;
#pragma unroll
        for (int k = 0; k <= D; ++k)
            if (k <= it.K) {
                const d3 s = sub(X[k + 1], X[k]);
                const double l = norm(s);
                L += l;
                dir[k] = scale(s, 1.0 / l);
                dK = dir[k];
            }
        const d3 F0 = antenna_field(a.tx_ant, dir[0]);
        c3 E{cd{F0.x, 0}, cd{F0.y, 0}, cd{F0.z, 0}};
        d3 th0, ph0;
        sph_basis(dir[0], th0, ph0);
        c3 B0{cd{th0.x, 0}, cd{th0.y, 0}, cd{th0.z, 0}};
        c3 B1{cd{ph0.x, 0}, cd{ph0.y, 0}, cd{ph0.z, 0}};
#pragma unroll
        for (int k = 1; k <= D; ++k)
            if (k <= it.K) {
                const Face& F = a.sc.faces[it.fc[k - 1]];
                d3 nf = ld3(F.n);
                const d3 din = dir[k - 1], dout = dir[k];
                if (dot(din, nf) > 0.0) nf = scale(nf, -1.0);
                const double cos_i = -dot(din, nf);
                cd rp, rl;
                fresnel(mats.m[F.mat], cos_i, rp, rl);
                const double share = specular_share(mats.m[F.mat]);
                rp = cmulr(rp, share);
                rl = cmulr(rl, share);
                const d3 ep = perp_basis(din, nf);
                const d3 eli = cross(ep, din), elr = cross(ep, dout);
                E = reflect_field(E, ep, eli, elr, rp, rl);
                B0 = reflect_field(B0, ep, eli, elr, rp, rl);
                B1 = reflect_field(B1, ep, eli, elr, rp, rl);
            }
        d3 thK, phK;
        sph_basis(dK, thK, phK);
        const d3 mdK = scale(dK, -1.0);
        const d3 Fr = antenna_field(a.rx_ant[it.r], mdK);
        const cd pr = cdot(E, Fr);
        const double amp = a.lambda / (4.0 * kPi * L);
        const uint32_t slot = atomicAdd(a.counts + it.r, 1u);
        if (slot >= (uint32_t)a.P) continue;
        const int64_t at = (int64_t)it.r * a.P + slot;
        a.a[2 * at] = (float)(amp * pr.re);
        a.a[2 * at + 1] = (float)(amp * pr.im);
        const cd t00 = cdot(B0, thK), t01 = cdot(B1, thK), t10 = cdot(B0, phK), t11 = cdot(B1, phK);
        float* T = a.T + 8 * at;
        T[0] = (float)t00.re; T[1] = (float)t00.im;
        T[2] = (float)t01.re; T[3] = (float)t01.im;
        T[4] = (float)t10.re; T[5] = (float)t10.im;
        T[6] = (float)t11.re; T[7] = (float)t11.im;
        a.tau[at] = (float)(L / kC0);
        a.aod[2 * at] = (float)acos(fmin(fmax(dir[0].z, -1.0), 1.0));
        a.aod[2 * at + 1] = (float)atan2(dir[0].y, dir[0].x);
        a.aoa[2 * at] = (float)acos(fmin(fmax(mdK.z, -1.0), 1.0));
        a.aoa[2 * at + 1] = (float)atan2(mdK.y, mdK.x);
        a.depth[at] = it.K;
#pragma unroll
        for (int i = 0; i < D; ++i)
            if (i < a.fd) a.faces[(int64_t)a.fd * at + i] = i < it.K ? it.fc[i] : -1;
    }
}

// Order the paths of one receiver by (depth, faces) and write them to the
// caller's arrays; unused slots get a = 0, tau = -1, depth = -1, faces = -1.
// One block per receiver: thread i counts the paths that come before path i
// (at most 256, keys in LDS), then all threads copy.  Bound by the writes (84
// bytes and more per slot); one thread per receiver, sorting by insertion and
// copying alone, took 806 us for 1024 receivers of 256 slots and 17,000 paths.
constexpr int kSortSlots = 256, kSortFaces = 8;
__global__ __launch_bounds__(kSortSlots) void sort_paths_kernel(PathArgs a, float* a_out, float* T_out,
                                                                float* tau_out, float* aod_out, float* aoa_out,
                                                                int32_t* depth_out, int32_t* faces_out,
                                                                int32_t nrx, int32_t* num_out) {
    __shared__ int32_t key[1 + kSortFaces][kSortSlots];
    __shared__ int32_t from[kSortSlots];
    const int tid = threadIdx.x;
    for (int r = blockIdx.x; r < nrx; r += gridDim.x) {
        const uint32_t cnt = a.counts[r];
        const int n = (int)(cnt < (uint32_t)a.P ? cnt : (uint32_t)a.P);
        const int64_t base = (int64_t)r * a.P;
        if (tid == 0) num_out[r] = (int32_t)cnt;
        if (tid < n) {
            key[0][tid] = a.depth[base + tid];
            for (int k = 0; k < a.fd; ++k) key[1 + k][tid] = a.faces[(base + tid) * a.fd + k];
        }
        __syncthreads();
        if (tid < n) {
            int rank = 0;
            for (int j = 0; j < n; ++j) {
                int before = j < tid;  // equal keys keep their order
                for (int k = 0; k <= a.fd; ++k) {
                    const int x = key[k][j], y = key[k][tid];
                    if (x != y) {
                        before = x < y;
                        break;
                    }
                }
                rank += before;
            }
            from[rank] = tid;
        }
        __syncthreads();
        auto copy = [&](float* dst, const float* src, int width, float none) {
            for (int e = tid; e < a.P * width; e += kSortSlots) {
                const int i = e / width;
                dst[base * width + e] = i < n ? src[(base + from[i]) * width + (e - i * width)] : none;
            }
        };
        copy(a_out, a.a, 2, 0.0f);
        copy(T_out, a.T, 8, 0.0f);
        copy(tau_out, a.tau, 1, -1.0f);
        copy(aod_out, a.aod, 2, 0.0f);
        copy(aoa_out, a.aoa, 2, 0.0f);
        for (int i = tid; i < a.P; i += kSortSlots) depth_out[base + i] = i < n ? key[0][from[i]] : -1;
        for (int e = tid; e < a.P * a.fd; e += kSortSlots) {
            const int i = e / a.fd;
            faces_out[base * a.fd + e] = i < n ? key[1 + e - i * a.fd][from[i]] : -1;
        }
        __syncthreads();
    }
}

// P[r] = sum over the valid slots of |a|^2 (fp64 accumulation of the fp32 a).
__global__ void paths_power_kernel(const float* __restrict__ a, const int32_t* __restrict__ depth, int64_t n, int P,
                                   double* __restrict__ power) {
    const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= n) return;
    double acc = 0.0;
    for (int j = 0; j < P; ++j) {
        const int64_t at = r * P + j;
        if (depth[at] < 0) continue;
        const double re = a[2 * at], im = a[2 * at + 1];
        acc += re * re + im * im;
    }
    power[r] = acc;
}

}  // namespace

hipError_t launch_paths_power(const float* a, const int32_t* depth, int64_t n, int P, double* power, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(paths_power_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, a, depth, n, P, power);
    return hipGetLastError();
}

hipError_t launch_extract_candidates(const uint64_t* table, uint64_t cap, int32_t max_depth, Cand* out,
                                     uint32_t* count, uint32_t max_out, hipStream_t s) {
    const uint64_t blocks = (cap + 255) / 256;
    hipLaunchKernelGGL(extract_candidates_kernel, dim3((unsigned)blocks), dim3(256), 0, s, table, cap, max_depth,
                       out, count, max_out);
    return hipGetLastError();
}

hipError_t launch_extract_pairs(const uint64_t* pairs, uint64_t pairs_cap, const uint64_t* table, Cand* out,
                                int32_t* out_rx, uint32_t* count, uint32_t max_out, hipStream_t s) {
    const uint64_t blocks = (pairs_cap + 255) / 256;
    hipLaunchKernelGGL(extract_pairs_kernel, dim3((unsigned)blocks), dim3(256), 0, s, pairs, pairs_cap, table, out,
                       out_rx, count, max_out);
    return hipGetLastError();
}

namespace {
template <int D>
hipError_t image_passes(const PathArgs& a, const MatTable& mats, int64_t items, int64_t chunk, uint32_t* scratch,
                        hipStream_t s) {
    uint32_t *count = scratch, *queue = scratch + 64, *blocked = queue + chunk;
    for (int64_t first = 0; first < items; first += chunk) {
        const int64_t n = std::min(chunk, items - first);
        hipError_t e = launch_fill_u32(count, 0u, 1, s);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(image_filter_kernel<D>, dim3((unsigned)((n + kBlock - 1) / kBlock)), dim3(kBlock), 0, s, a,
                           first, n, queue, blocked, count);
        // three blocks of 48 KB per CU for the traversals
        const int64_t legs = (n * (a.max_depth + 1) + kBlock - 1) / kBlock;
        hipLaunchKernelGGL(image_legs_kernel<D>, dim3((unsigned)std::min<int64_t>(legs, 256 * 3)), dim3(kBlock), 0, s,
                           a, first, queue, blocked, count);
        const int64_t paths = (n + kImageBlock - 1) / kImageBlock;
        hipLaunchKernelGGL(image_paths_kernel<D>, dim3((unsigned)std::min<int64_t>(paths, 1024)), dim3(kImageBlock), 0,
                           s, a, mats, first, queue, blocked, count);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    return hipSuccess;
}
}  // namespace

size_t image_scratch(int64_t chunk) { return (64 + 2 * (size_t)chunk) * sizeof(uint32_t); }

hipError_t launch_image_paths(const PathArgs& a, const MatTable& mats, int64_t items, int64_t chunk, void* scratch,
                              hipStream_t s) {
    if (items <= 0) return hipSuccess;
    uint32_t* q = (uint32_t*)scratch;
    if (a.max_depth <= 1) return image_passes<1>(a, mats, items, chunk, q, s);
    if (a.max_depth <= 3) return image_passes<3>(a, mats, items, chunk, q, s);
    if (a.max_depth <= 5) return image_passes<5>(a, mats, items, chunk, q, s);
    return image_passes<kMaxK>(a, mats, items, chunk, q, s);
}

hipError_t launch_sort_paths(const PathArgs& a, int32_t nrx, float* a_out, float* T_out, float* tau_out,
                             float* aod_out, float* aoa_out, int32_t* depth_out, int32_t* faces_out,
                             int32_t* num_paths_out, hipStream_t s) {
    if (a.P > kSortSlots || a.fd > kSortFaces) return hipErrorInvalidValue;
    hipLaunchKernelGGL(sort_paths_kernel, dim3(std::min(nrx, 1 << 20)), dim3(kSortSlots), 0, s, a, a_out, T_out,
                       tau_out, aod_out, aoa_out, depth_out, faces_out, nrx, num_paths_out);
    return hipGetLastError();
}

}  // namespace rt
