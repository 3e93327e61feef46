// Channel responses from paths for gfx950 (paper Sec. II-A: paths become
// channel impulse responses, with synthetic arrays and Doppler; Sec. III-A:
// channel frequency responses of an OFDM system with 128 subcarriers spaced
// 30 kHz apart).
//
// A path p has a coefficient a_p (without the delay phase), a delay tau_p and
// unit vectors k_t (departure, from the angles of departure) and k_r (from the
// receiver towards the arriving wave, from the angles of arrival).  With the
// e^{+j w t} convention, an array element at offset r from the array centre
// sees a plane wave earlier by (k . r) / c (synthetic array, plane-wave
// assumption at the carrier wavelength), and moving devices shift the path's
// frequency by f_D = (v_tx . k_t + v_rx . k_r) / lambda.  The response at time
// step n (t = n / fs), receive element j, transmit element i and subcarrier k
// (baseband frequency f_k = (k - floor(K/2)) spacing) is
//   H = sum_p a_p exp(j 2 pi phi_p),
//   phi_p = -(f_c + f_k) tau_p + (k_t . r_i + k_r . r_j) / lambda + f_D t,
// the phase in cycles evaluated in fp64 and reduced modulo 1 before the sine.
//
// The phase is a sum of a row part (n, j, i) and a subcarrier part k, so the
// responses of one link are a complex fp64 product H = L S with
//   L[row][p] = a_p exp(j 2 pi ((k_t . r_i + k_r . r_j) / lambda + f_D t)),
//   S[p][k]   = exp(-j 2 pi (f_c + f_k) tau_p),
// and the adjoint is S[p][k]-weighted sums of conj(G)^T L.  The tile kernels
// build the two factors in LDS (a sine per factor entry instead of one per
// output and path) and spend four fp64 FMAs per output and path; links with
// few outputs keep one sine per output and path.
#include <algorithm>

#include "kernels.h"

namespace rt {
namespace {

constexpr int kCfrBlock = 256;
constexpr int kTileMinRows = 8;        // rows below which the factors are not worth building
constexpr int64_t kTileMinOut = 1024;  // outputs per link below which a tile is mostly empty

__device__ __forceinline__ d3 unit_of(float th, float ph) {
    double st, ct, sp, cp;
    sincos((double)th, &st, &ct);
    sincos((double)ph, &sp, &cp);
    return d3{st * cp, st * sp, ct};
}

// The caller's complex arrays promise the alignment of one float or double only.
typedef float float2u __attribute__((ext_vector_type(2), aligned(4)));
typedef double double2u __attribute__((ext_vector_type(2), aligned(8)));

// What the phases of one path need.
struct PathTerm {
    d3 kt, kr;       // departure and arrival unit vectors
    double fd, tau;  // Doppler shift [Hz], delay [s]
    double ar, ai;   // coefficient
};

__device__ __forceinline__ PathTerm path_term(const CfrArgs& c, int64_t pair, int64_t slot) {
    PathTerm q;
    q.kt = unit_of(c.aod[2 * slot], c.aod[2 * slot + 1]);
    q.kr = unit_of(c.aoa[2 * slot], c.aoa[2 * slot + 1]);
    const double* vt = c.v_tx + 3 * (pair / c.nrx);
    const double* vr = c.v_rx + 3 * (pair % c.nrx);
    q.fd = (q.kt.x * vt[0] + q.kt.y * vt[1] + q.kt.z * vt[2] + q.kr.x * vr[0] + q.kr.y * vr[1] + q.kr.z * vr[2]) /
           c.lambda;
    q.tau = (double)c.tau[slot];
    q.ar = c.a[2 * slot];
    q.ai = c.a[2 * slot + 1];
    return q;
}

// Cycles of the row part (time step t, receive element j, transmit element i).
__device__ __forceinline__ double row_phase(const CfrArgs& c, const PathTerm& q, int t, int j, int i) {
    const double* ri = c.tx_el + 3 * i;
    const double* rj = c.rx_el + 3 * j;
    const double arr = (q.kt.x * ri[0] + q.kt.y * ri[1] + q.kt.z * ri[2] + q.kr.x * rj[0] + q.kr.y * rj[1] +
                        q.kr.z * rj[2]) /
                       c.lambda;
    return arr + q.fd * ((double)t / c.fs);
}

// Cycles of the subcarrier part.
__device__ __forceinline__ double sub_phase(const CfrArgs& c, const PathTerm& q, int k) {
    const double fk = (double)(k - c.K / 2) * c.spacing;
    return -(c.freq + fk) * q.tau;
}

__device__ __forceinline__ cd cycles(double ph) {
    double s, co;
    sincospi(2.0 * (ph - floor(ph)), &s, &co);
    return cd{co, s};
}

__device__ __forceinline__ void row_index(const CfrArgs& c, int64_t row, int& t, int& j, int& i) {
    if ((uint64_t)row >> 32) {
        i = (int)(row % c.nt_el);
        row /= c.nt_el;
        j = (int)(row % c.nr_el);
        t = (int)(row / c.nr_el);
    } else {
        uint32_t r = (uint32_t)row;
        i = (int)(r % (uint32_t)c.nt_el);
        r /= (uint32_t)c.nt_el;
        j = (int)(r % (uint32_t)c.nr_el);
        t = (int)(r / (uint32_t)c.nr_el);
    }
}

// Valid slots among [s0, s0 + N) of the pair, in slot order, by the first N
// threads of the block: their terms and slots; returns their number to every
// thread.  The caller synchronises before the arrays are refilled.
template <int N>
__device__ __forceinline__ int gather_terms(const CfrArgs& c, int64_t pair, int64_t s0, PathTerm* terms, int* slots,
                                            int* wave_n) {
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    bool valid = false;
    if (tid < N && s0 + tid < c.P) valid = c.depth[pair * c.P + s0 + tid] >= 0;
    const uint64_t m = __ballot(valid);
    if (tid < N && lane == 0) wave_n[w] = __popcll(m);
    __syncthreads();
    int before = 0, n = 0;
#pragma unroll
    for (int i = 0; i < N / 64; ++i) {
        if (i < w) before += wave_n[i];
        n += wave_n[i];
    }
    if (valid) {
        const int at = before + __popcll(m & ((1ull << lane) - 1ull));
        terms[at] = path_term(c, pair, pair * c.P + s0 + tid);
        slots[at] = (int)(s0 + tid);
    }
    __syncthreads();
    return n;
}

// Links with few outputs: 256 outputs of one link per block, one thread each,
// a sine per output and path.  The 256 threads look up 256 slots at once (most
// slots of a path list are empty) and build each valid path's terms once per
// block.  256 links x 128 slots x 128 outputs (300 paths): 25 us with a serial
// walk over the slots in every thread.
__global__ __launch_bounds__(kCfrBlock) void cfr_kernel(CfrArgs c, int64_t per, int64_t blocks_per) {
    __shared__ PathTerm terms[kCfrBlock];
    __shared__ int slots[kCfrBlock];
    __shared__ int wave_n[kCfrBlock / 64];
    for (int64_t b = blockIdx.x; b < c.npairs * blocks_per; b += gridDim.x) {
        const int64_t pair = b / blocks_per;
        const int64_t q = (b % blocks_per) * kCfrBlock + threadIdx.x;
        const int64_t row = q < per ? q / c.K : 0;
        const int k = (int)(q - row * c.K);
        int t, j, i;
        row_index(c, row, t, j, i);
        double re = 0.0, im = 0.0;
        for (int64_t s0 = 0; s0 < c.P; s0 += kCfrBlock) {
            const int n = gather_terms<kCfrBlock>(c, pair, s0, terms, slots, wave_n);
            for (int p = 0; p < n && q < per; ++p) {
                const PathTerm& x = terms[p];
                const cd e = cycles(sub_phase(c, x, k) + row_phase(c, x, t, j, i));
                re += x.ar * e.re - x.ai * e.im;
                im += x.ar * e.im + x.ai * e.re;
            }
            __syncthreads();
        }
        if (q < per) reinterpret_cast<float2u*>(c.H)[pair * per + q] = float2u{(float)re, (float)im};
    }
}

// Tile of 16 RM rows by 16 KM subcarriers of one link per block; each thread
// holds RM x KM complex fp64 sums (64 doubles).  Paths go through LDS in
// batches of PB: 16 RM PB row factors and 16 KM PB subcarrier factors.  Bound
// by fp64 FMAs (4 per output and path; 128 per thread and path against 12
// 16-byte LDS reads) and, for few paths, by the 8 bytes written per output.
// One sine per output and path took 1.62 ms for 16 links x 64 slots x 229,376
// outputs; with the adjoint below: 139 ms -> 0.17 ms for the pair of calls.
template <int KM, int RM, int PB>
__global__ __launch_bounds__(kCfrBlock) void cfr_tile_kernel(CfrArgs c, int64_t rows, int64_t row_tiles,
                                                             int64_t k_tiles) {
    constexpr int KT = 16 * KM, RT = 16 * RM;
    __shared__ PathTerm terms[kCfrBlock];
    __shared__ int slots[kCfrBlock];
    __shared__ int wave_n[kCfrBlock / 64];
    __shared__ cd Lf[PB][RT];
    __shared__ cd Sf[PB][KT];
    const int tid = threadIdx.x, tx = tid & 15, ty = tid >> 4;
    for (int64_t b = blockIdx.x; b < c.npairs * row_tiles * k_tiles; b += gridDim.x) {
        const int k0 = (int)(b % k_tiles) * KT;
        const int64_t r0 = (b / k_tiles) % row_tiles * RT;
        const int64_t pair = b / k_tiles / row_tiles;
        cd acc[RM][KM];
#pragma unroll
        for (int m = 0; m < RM; ++m)
#pragma unroll
            for (int u = 0; u < KM; ++u) acc[m][u] = cd{0.0, 0.0};
        for (int64_t s0 = 0; s0 < c.P; s0 += kCfrBlock) {
            const int n = gather_terms<kCfrBlock>(c, pair, s0, terms, slots, wave_n);
            for (int p0 = 0; p0 < n; p0 += PB) {
                const int nb = min(PB, n - p0);
                for (int e = tid; e < nb * RT; e += kCfrBlock) {
                    const int p = e / RT, r = e % RT;
                    cd v{0.0, 0.0};
                    if (r0 + r < rows) {
                        const PathTerm& x = terms[p0 + p];
                        int t, j, i;
                        row_index(c, r0 + r, t, j, i);
                        v = cmul(cd{x.ar, x.ai}, cycles(row_phase(c, x, t, j, i)));
                    }
                    Lf[p][r] = v;
                }
                // one sine for k and one for the step of 32 subcarriers; the entries
                // between follow by at most KM / 2 - 1 complex products (1e-15)
                for (int e = tid; e < nb * (KT < 32 ? KT : 32); e += kCfrBlock) {
                    constexpr int W = KT < 32 ? KT : 32;
                    const int p = e / W, k = e % W;
                    const PathTerm& x = terms[p0 + p];
                    cd v = cycles(sub_phase(c, x, k0 + k));
                    Sf[p][k] = v;
                    if (KT > 32) {
                        const cd w = cycles(-32.0 * c.spacing * x.tau);
#pragma unroll
                        for (int kk = 32; kk < KT; kk += 32) {
                            v = cmul(v, w);
                            Sf[p][k + kk] = v;
                        }
                    }
                }
                __syncthreads();
                for (int p = 0; p < nb; ++p) {
                    cd l[RM], s[KM];
#pragma unroll
                    for (int m = 0; m < RM; ++m) l[m] = Lf[p][ty + 16 * m];
#pragma unroll
                    for (int u = 0; u < KM; ++u) s[u] = Sf[p][tx + 16 * u];
#pragma unroll
                    for (int m = 0; m < RM; ++m)
#pragma unroll
                        for (int u = 0; u < KM; ++u) acc[m][u] = cadd(acc[m][u], cmul(l[m], s[u]));
                }
                __syncthreads();
            }
            __syncthreads();
        }
        float2u* H = reinterpret_cast<float2u*>(c.H) + pair * rows * c.K;
#pragma unroll
        for (int m = 0; m < RM; ++m) {
            const int64_t r = r0 + ty + 16 * m;
            if (r >= rows) continue;
#pragma unroll
            for (int u = 0; u < KM; ++u) {
                const int k = k0 + tx + 16 * u;
                if (k < c.K) H[r * c.K + k] = float2u{(float)acc[m][u].re, (float)acc[m][u].im};
            }
        }
    }
}

// Adjoint of the linear map a -> H: g_p = sum over the pair's outputs of
// conj(G) exp(j 2 pi phi_p).  Links with few outputs: one block per 256 slots
// of a link, one wave per valid path, lanes along the outputs.
__global__ __launch_bounds__(kCfrBlock) void cfr_adjoint_kernel(CfrArgs c, const float* __restrict__ G,
                                                                double* __restrict__ g, int64_t per,
                                                                int64_t blocks_per) {
    __shared__ PathTerm terms[kCfrBlock];
    __shared__ int slots[kCfrBlock];
    __shared__ int wave_n[kCfrBlock / 64];
    const int tid = threadIdx.x, lane = tid & 63;
    for (int64_t b = blockIdx.x; b < c.npairs * blocks_per; b += gridDim.x) {
        const int64_t pair = b / blocks_per;
        const int64_t s0 = (b % blocks_per) * kCfrBlock;
        const int n = gather_terms<kCfrBlock>(c, pair, s0, terms, slots, wave_n);
        double2u* gp = reinterpret_cast<double2u*>(g) + pair * c.P;
        if (s0 + tid < c.P && c.depth[pair * c.P + s0 + tid] < 0) gp[s0 + tid] = double2u{0.0, 0.0};
        const float2u* Gp = reinterpret_cast<const float2u*>(G) + pair * per;
        for (int p = tid >> 6; p < n; p += kCfrBlock / 64) {
            const PathTerm x = terms[p];
            double re = 0.0, im = 0.0;
            for (int64_t q = lane; q < per; q += 64) {
                const int64_t row = q / c.K;
                int t, j, i;
                row_index(c, row, t, j, i);
                const cd e = cycles(sub_phase(c, x, (int)(q - row * c.K)) + row_phase(c, x, t, j, i));
                const float2u v = Gp[q];
                const double gr = v.x, gi = -v.y;  // conj(G)
                re += gr * e.re - gi * e.im;
                im += gr * e.im + gi * e.re;
            }
            for (int off = 32; off >= 1; off >>= 1) {
                re += __shfl_xor(re, off);
                im += __shfl_xor(im, off);
            }
            if (lane == 0) gp[slots[p]] = double2u{re, im};
        }
        __syncthreads();
    }
}

// Adjoint tile: 64 slots of one link by 16 KM subcarriers over a range of
// rows per block: M[p][k] = sum_row conj(G[row][k]) exp(j 2 pi row phase), then
// sum_k S[p][k] M[p][k], one partial per block (part = row range and
// subcarrier tile), added in a fixed order by cfr_parts_kernel.  Valid slots
// are packed, and groups of 16 without a valid slot cost nothing.  One thread
// per path walking every output took 137 ms for 16 links x 64 paths x 229,376
// outputs: 16 waves on the whole chip, a sine and five more for the unit
// vectors per output.
constexpr int kAdjSlots = 64, kAdjRows = 8;
struct AdjPlan {
    int64_t rows, rows_per, row_parts, k_tiles, slot_tiles;
    int64_t parts;        // row_parts * k_tiles
    int64_t tile0, tiles;  // slot tiles (link * slot_tiles + tile of the link) of this launch
    int km;
};
template <int KM>
__global__ __launch_bounds__(kCfrBlock) void cfr_adjoint_tile_kernel(CfrArgs c, const float* __restrict__ G,
                                                                     double* __restrict__ g, double* __restrict__ part,
                                                                     AdjPlan a) {
    constexpr int KT = 16 * KM, PM = kAdjSlots / 16;
    __shared__ PathTerm terms[kAdjSlots];
    __shared__ int slots[kAdjSlots];
    __shared__ int wave_n[1];
    __shared__ cd Lf[kAdjRows][kAdjSlots];
    __shared__ cd Gf[kAdjRows][KT];
    const int tid = threadIdx.x, tx = tid & 15, ty = tid >> 4;
    const int64_t rows = a.rows;
    for (int64_t b = blockIdx.x; b < a.tiles * a.parts; b += gridDim.x) {
        const int64_t part_at = b % a.parts, rp = part_at / a.k_tiles, t = b / a.parts;
        const int64_t s0 = (a.tile0 + t) % a.slot_tiles * kAdjSlots, pair = (a.tile0 + t) / a.slot_tiles;
        const int k0 = (int)(part_at % a.k_tiles) * KT;
        double2u* out = a.parts == 1 ? reinterpret_cast<double2u*>(g) + pair * c.P + s0
                                     : reinterpret_cast<double2u*>(part) + (part_at * a.tiles + t) * kAdjSlots;
        if (tid < kAdjSlots && s0 + tid < c.P && c.depth[pair * c.P + s0 + tid] < 0) out[tid] = double2u{0.0, 0.0};
        const int n = gather_terms<kAdjSlots>(c, pair, s0, terms, slots, wave_n);
        if (n == 0) continue;
        cd acc[PM][KM];
#pragma unroll
        for (int m = 0; m < PM; ++m)
#pragma unroll
            for (int u = 0; u < KM; ++u) acc[m][u] = cd{0.0, 0.0};
        const float2u* Gp = reinterpret_cast<const float2u*>(G) + pair * rows * c.K;
        const int64_t r_end = min(rows, (rp + 1) * a.rows_per);
        for (int64_t r0 = rp * a.rows_per; r0 < r_end; r0 += kAdjRows) {
            const int nr = (int)min((int64_t)kAdjRows, r_end - r0);
            for (int e = tid; e < nr * KT; e += kCfrBlock) {
                const int r = e / KT, k = e % KT;
                cd v{0.0, 0.0};
                if (k0 + k < c.K) {
                    const float2u x = Gp[(r0 + r) * c.K + k0 + k];
                    v = cd{(double)x.x, -(double)x.y};
                }
                Gf[r][k] = v;
            }
            for (int e = tid; e < nr * kAdjSlots; e += kCfrBlock) {
                const int r = e / kAdjSlots, p = e % kAdjSlots;
                cd v{0.0, 0.0};
                if (p < n) {
                    int t, j, i;
                    row_index(c, r0 + r, t, j, i);
                    v = cycles(row_phase(c, terms[p], t, j, i));
                }
                Lf[r][p] = v;
            }
            __syncthreads();
            for (int r = 0; r < nr; ++r) {
                cd s[KM];
#pragma unroll
                for (int u = 0; u < KM; ++u) s[u] = Gf[r][tx + 16 * u];
#pragma unroll
                for (int m = 0; m < PM; ++m) {
                    if (16 * m >= n) break;
                    const cd l = Lf[r][ty + 16 * m];
#pragma unroll
                    for (int u = 0; u < KM; ++u) acc[m][u] = cadd(acc[m][u], cmul(l, s[u]));
                }
            }
            __syncthreads();
        }
#pragma unroll
        for (int m = 0; m < PM; ++m) {
            const int p = ty + 16 * m;
            if (16 * m >= n) break;
            cd sum{0.0, 0.0};
            if (p < n) {
                const PathTerm& x = terms[p];
                cd v = cycles(sub_phase(c, x, k0 + tx));
                const cd w = cycles(-16.0 * c.spacing * x.tau);
#pragma unroll
                for (int u = 0; u < KM; ++u) {
                    sum = cadd(sum, cmul(v, acc[m][u]));
                    v = cmul(v, w);
                }
            }
            for (int off = 8; off >= 1; off >>= 1) {
                sum.re += __shfl_xor(sum.re, off);
                sum.im += __shfl_xor(sum.im, off);
            }
            if (tx == 0 && p < n) out[slots[p] - s0] = double2u{sum.re, sum.im};
        }
        __syncthreads();
    }
}

__global__ void cfr_parts_kernel(const double2u* __restrict__ part, AdjPlan a, int64_t P, double2u* __restrict__ g) {
    const int64_t n = a.tiles * kAdjSlots;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const int64_t tile = a.tile0 + i / kAdjSlots, slot = tile % a.slot_tiles * kAdjSlots + i % kAdjSlots;
        if (slot >= P) continue;
        double2u s = part[i];
        for (int64_t p = 1; p < a.parts; ++p) s += part[p * n + i];
        g[tile / a.slot_tiles * P + slot] = s;
    }
}

int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// Whether a link's outputs fill tiles (see the file comment).  Measured per
// output and path: about 100 instructions with a sine each, 190 / 32 per
// thread-tile entry with the factors, of which a tile of 64 rows with 8 rows
// filled uses an eighth.
bool use_tiles(const CfrArgs& c, int64_t rows) {
    return rows >= kTileMinRows && rows * c.K >= kTileMinOut;
}

// Whether the responses of all links take tiles.  A tile is 2048 outputs or more
// and its block works through the paths alone: with 64 paths a link at least
// 115 us for up to 16 subcarriers, 65 for up to 32, 50 beyond, however few tiles
// there are, while a sine per output fills the chip and takes 23 us for up to
// 65,000 outputs, 54 for 230,000 and 180 for 10^6.  The lines lie where the two
// meet (one and 16 links, 64 paths, sines / tiles): 16 subcarriers 96 / 116 us at
// 460,000 outputs, 128 / 116 at 690,000; 32 subcarriers 47 / 58 at 260,000, 97 /
// 78 at 520,000; 64 and 128 subcarriers 29 / 47 and 29 / 42 at 130,000, 97 / 58
// and 99 / 51 at 520,000.  Below five subcarriers a tile's 16 columns are mostly
// empty (four, 10^6 outputs: 180 / 224 us).
bool responses_take_tiles(const CfrArgs& c, int64_t rows) {
    if (!use_tiles(c, rows) || c.K < 5) return false;
    return c.total >= (c.K > 32 ? int64_t(1) << 18 : c.K > 16 ? int64_t(3) << 17 : int64_t(5) << 17);
}

// Row ranges of the adjoint: enough blocks to fill the chip (2048), at least
// 32 rows each.  Where one part per tile does not do, as many tiles at a time as
// their partial sums fit kAdjScratch (one at least).
constexpr int64_t kAdjScratch = int64_t(64) << 20, kAdjTileBytes = kAdjSlots * (int64_t)sizeof(double2u);
AdjPlan adjoint_plan(const CfrArgs& c) {
    AdjPlan p{};
    p.rows = (int64_t)c.T * c.nr_el * c.nt_el;
    p.km = c.K > 64 ? 8 : c.K > 32 ? 4 : c.K > 16 ? 2 : 1;
    p.k_tiles = ceil_div(c.K, 16 * p.km);
    p.slot_tiles = ceil_div(c.P, kAdjSlots);
    const int64_t blocks = c.npairs * p.k_tiles * p.slot_tiles;
    const int64_t want = std::max<int64_t>(1, std::min<int64_t>(ceil_div(2048, blocks), p.rows / 32));
    p.rows_per = ceil_div(ceil_div(p.rows, want), kAdjRows) * kAdjRows;
    p.row_parts = ceil_div(p.rows, p.rows_per);
    p.parts = p.row_parts * p.k_tiles;
    p.tiles = c.npairs * p.slot_tiles;
    if (p.parts > 1) p.tiles = std::min(p.tiles, std::max<int64_t>(1, kAdjScratch / (p.parts * kAdjTileBytes)));
    return p;
}

dim3 grid_of(int64_t blocks) { return dim3((unsigned)std::min<int64_t>(blocks, 1 << 22)); }

}  // namespace

size_t cfr_adjoint_scratch(const CfrArgs& c) {
    const AdjPlan p = adjoint_plan(c);
    return use_tiles(c, p.rows) && p.parts > 1 ? (size_t)(p.tiles * p.parts * kAdjTileBytes) : 0;
}

hipError_t launch_cfr(const CfrArgs& c, hipStream_t s) {
    if (c.total <= 0) return hipSuccess;
    const int64_t rows = (int64_t)c.T * c.nr_el * c.nt_el;
    if (responses_take_tiles(c, rows)) {
        auto go = [&](auto kernel, int km, int rm) {
            const int64_t rt = ceil_div(rows, 16 * rm), kt = ceil_div(c.K, 16 * km);
            hipLaunchKernelGGL(kernel, grid_of(c.npairs * rt * kt), dim3(kCfrBlock), 0, s, c, rows, rt, kt);
        };
        if (c.K > 64) go(cfr_tile_kernel<8, 4, 8>, 8, 4);
        else if (c.K > 32) go(cfr_tile_kernel<4, 8, 8>, 4, 8);
        else if (c.K > 16) go(cfr_tile_kernel<2, 16, 4>, 2, 16);
        else go(cfr_tile_kernel<1, 32, 2>, 1, 32);
    } else {
        const int64_t per = rows * c.K, blocks = ceil_div(per, kCfrBlock);
        hipLaunchKernelGGL(cfr_kernel, grid_of(c.npairs * blocks), dim3(kCfrBlock), 0, s, c, per, blocks);
    }
    return hipGetLastError();
}

hipError_t launch_cfr_adjoint(const CfrArgs& c, const float* G, double* g, void* scratch, hipStream_t s) {
    const int64_t n = c.npairs * c.P;
    if (n <= 0) return hipSuccess;
    AdjPlan p = adjoint_plan(c);
    if (use_tiles(c, p.rows) && (p.parts == 1 || scratch)) {
        const int64_t all = c.npairs * p.slot_tiles, step = p.tiles;
        auto go = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, grid_of(p.tiles * p.parts), dim3(kCfrBlock), 0, s, c, G, g, (double*)scratch, p);
        };
        for (p.tile0 = 0; p.tile0 < all; p.tile0 += step) {
            p.tiles = std::min(step, all - p.tile0);
            if (p.km == 8) go(cfr_adjoint_tile_kernel<8>);
            else if (p.km == 4) go(cfr_adjoint_tile_kernel<4>);
            else if (p.km == 2) go(cfr_adjoint_tile_kernel<2>);
            else go(cfr_adjoint_tile_kernel<1>);
            if (p.parts > 1)
                hipLaunchKernelGGL(cfr_parts_kernel, grid_of(ceil_div(p.tiles * kAdjSlots, 256)), dim3(256), 0, s,
                                   (const double2u*)scratch, p, (int64_t)c.P, (double2u*)g);
        }
    } else {
        const int64_t blocks = ceil_div(c.P, kCfrBlock);
        hipLaunchKernelGGL(cfr_adjoint_kernel, grid_of(c.npairs * blocks), dim3(kCfrBlock), 0, s, c, G, g,
                           p.rows * c.K, blocks);
    }
    return hipGetLastError();
}

}  // namespace rt
