// One walk over M per iteration (ranks up to 4): two launches before the decompression instead of four or five.
//
// Algorithm 1 of arXiv 1905.13727 needs all of P = M Q before P_hat, and P_hat before Q = M^T P_hat.  But P_hat = P R^-1 with R the
// Cholesky factor of P^T P (the paper's remark "Orthogonalization is a linear operation"), hence Q = (M^T P) R^-1, and M^T P needs
// no more than the rows of P that belong to the rows of M at hand:
//
//   k_one_sweep   M_w = g_w + e_w over e_w; P = mean_w(M_w) Q row by row; S = M^T P and G = P^T P summed over the rows in the
//                 registers, one partial S and G per workgroup
//   k_solve       G and S added up, R, then P_hat = P R^-1 and Q = S R^-1
//
// M is then read by the decompression alone: 12 W bytes per element before it with fp32 gradients instead of 16 W (12 W + 8 with the
// products of the mean), and an iteration reads it once instead of twice.  G, S and the solutions are fp64, so that the division by R
// costs no digits of Q although P's columns are far from orthogonal: error against 64 bits, two walks / one: LSTM-shaped set,
// rank 4: Q 7.7e-8 / 3.7e-8, P 8.9e-8 / 8.8e-8; 24 matrices, 3 workers, rank 3: Q 8.1e-8 / 5.0e-8, P 7.9e-8 / 6.7e-8.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <string>

#include "psgd_device.h"
#include "psgd_internal.h"

namespace psgd {

// V consecutive gradient elements as they come (bf16: two to a register), widened when they are used
template <int V, bool BF>
struct graw {
    unsigned u[BF ? (V + 1) / 2 : V];
};
template <int V, bool BF>
__device__ __forceinline__ void ld_graw(buf_rsrc r, unsigned off, graw<V, BF>& g) {
    if constexpr (!BF) {
        float x[V];
        buf_ldv<V>(r, off, x, true);
#pragma unroll
        for (int i = 0; i < V; ++i) g.u[i] = __float_as_uint(x[i]);
    } else if constexpr (V == 4) {
        const v2u t = __builtin_amdgcn_raw_buffer_load_b64(r, (int)off, 0, 2);
        g.u[0] = t.x;
        g.u[1] = t.y;
    } else if constexpr (V == 2) {
        g.u[0] = __builtin_amdgcn_raw_buffer_load_b32(r, (int)off, 0, 2);
    } else {
        g.u[0] = (unsigned)(unsigned short)__builtin_amdgcn_raw_buffer_load_b16(r, (int)off, 0, 2);
    }
}
template <int V, bool BF>
__device__ __forceinline__ float graw_at(const graw<V, BF>& g, int x) {
    if constexpr (!BF) return __uint_as_float(g.u[x]);
    else return __uint_as_float(x % 2 ? g.u[x / 2] & 0xffff0000u : g.u[x / 2] << 16);
}

constexpr int pow2_at_least(int n) { return n <= 1 ? 1 : 2 * pow2_at_least((n + 1) / 2); }

// N <= 8 sums over the 64 lanes at once, in float or double: lane l < N returns the sum of x[l] (lane_sums is the one for more).  The values are handed
// over in halves between partners whose lane bit differs; the lane bits that chose nothing are added up afterwards.
template <int N, typename T>
__device__ __forceinline__ T few_lane_sums(const T (&x)[N]) {
    static_assert(N >= 1 && N <= 8, "one result per lane of eight");
    constexpr int NP = pow2_at_least(N);
    const int lane = threadIdx.x & (kWave - 1);
    const bool b2 = (lane & 4) != 0, b1 = (lane & 2) != 0, b0 = (lane & 1) != 0;
    T a[NP];
#pragma unroll
    for (int j = 0; j < NP; ++j) a[j] = j < N ? x[j] : T(0);
    if constexpr (NP >= 8) {
#pragma unroll
        for (int j = 0; j < 4; ++j) a[j] = (b2 ? a[j + 4] : a[j]) + dpp_mov<0x141>(b2 ? a[j] : a[j + 4]);   // row_half_mirror
    }
    if constexpr (NP >= 4) {
#pragma unroll
        for (int j = 0; j < 2; ++j) a[j] = (b1 ? a[j + 2] : a[j]) + dpp_mov<0x1B>(b1 ? a[j] : a[j + 2]);    // quad_perm [3,2,1,0]
    }
    T v = a[0];
    if constexpr (NP >= 2) v = (b0 ? a[1] : a[0]) + dpp_mov<0xB1>(b0 ? a[0] : a[1]);                        // quad_perm [1,0,3,2]
    if constexpr (NP < 2) v += dpp_mov<0xB1>(v);
    if constexpr (NP < 4) v += dpp_mov<0x4E>(v);    // quad_perm [2,3,0,1]
    v += dpp_mov<0x128>(v);                         // row_ror:8
    if constexpr (NP < 8) v += dpp_mov<0x124>(v);   // row_ror:4
    v += lane_read(v, lane ^ 16);
    return v + lane_read(v, lane ^ 32);
}

// LDS written by this wavefront is read by others after it; global loads stay in flight across it
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

extern __shared__ __attribute__((aligned(16))) char one_lds[];

// ---- k_one_sweep -------------------------------------------------------------------------------------------
//
// A workgroup owns a block of rows.  Its wavefronts form groups of 1, 2, 4 or 8 that hold a whole row between them (a lane 8 to 12
// columns of it) and walk a share of the block's rows, kOneRows at a time: M, the step's products (fp32, two chains a lane, reduced
// over the wavefront together and, where a row takes several wavefronts, through LDS), and with them the sums S += M^T P of the
// lane's columns in fp64 (on this chip an fp64 multiply-add costs what an fp32 one does).  A group's lanes keep S for the whole block;
// the groups' S are added in LDS at its end, in group order.  Bound by HBM: the loads of the next D steps (of one worker each) are
// in flight while a step is multiplied.  LSTM-shaped set, rank 4: 69 us, 5.5 TB/s, against 61 us and 22 us of the two walks; of it
// about 7 us are first loads and last sums, when little else moves.  What did not help there: fp64 products (70 us), more steps in
// flight with fewer columns a lane (78), a second generation of smaller blocks (76); non-temporal accesses to e on sets beyond the
// memory-side cache (LSTM-shaped set, 4 workers: the step 632 -> 675 us); leaving M unstored and forming g + e again in the
// decompression (159 -> 192).
// ADD = false: M is read from e (another iteration), nothing is added or stored.  MEAN: several workers, products of their mean.
// PT: the type the products are summed in (float; double where the rows are so long and the lanes' chains with them that rounding shows).
template <int R, int V, int NV, int RS, int D, typename PT, bool ADD, bool GBF, bool STORE, bool MEAN>
__device__ __forceinline__ void one_sweep_tile(const OneTile& t, const OneMat& d, const void* __restrict__ grad,
                                               float* __restrict__ err, const float* __restrict__ q, float* __restrict__ p,
                                               double* __restrict__ spart, double* __restrict__ gpart, int workers,
                                               int64_t gstride, int64_t estride, PT (*xsum)[kOneMaxWaves][kOneRows * kOneMaxRank],
                                               double (*xgram)[R * (R + 1) / 2]) {
    constexpr unsigned GS = GBF ? 2u : 4u;
    constexpr int NC = NV * V, N = RS * R;
    constexpr int NG = R * (R + 1) / 2;
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nwaves = blockDim.x >> 6;
    const int sh = d.waves_log2, per_row = 1 << sh;      // wavefronts that share a row
    const int group = wave >> sh, gw = wave & (per_row - 1), ngroups = nwaves >> sh;
    const int gl = gw * kWave + lane, glanes = per_row * kWave;   // lane within the row's wavefronts
    const int ri = d.r, m = d.m, nvec = m / V;

    // rows of this group; every group walks the same number of steps (they meet at barriers)
    const int base = t.nrows / ngroups, rem = t.nrows % ngroups;
    const int row0 = t.row0 + group * base + min(group, rem);
    const int rn = base + (group < rem ? 1 : 0);
    const int steps = (base + (rem ? 1 : 0) + RS - 1) / RS;

    // A descriptor per row, built with scalar instructions: columns past the row's end are out of range (zeros are read, stores
    // dropped), a row past the strip has an empty range; the lanes' offsets never change.
    unsigned coff[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        coff[v] = (unsigned)((gl + glanes * v) * V) * 4u;
    }
    const int64_t strip = d.off + (int64_t)row0 * m;
    const int nw = MEAN ? workers : 1;
    // item: a step's rows of one worker; the ring holds those of the next D items
    graw<V, GBF> gr[D][RS][NV];
    float ev[D][RS][NV][V];
    auto load = [&](int step, int w, graw<V, GBF> (&g)[RS][NV], float (&e)[RS][NV][V]) {   // past the last row: out of range, nothing is fetched
        if constexpr (ADD) {
#pragma unroll
            for (int i = 0; i < RS; ++i) {
                const int row = step * RS + i;
                const buf_rsrc gg = make_rsrc(static_cast<const char*>(grad) + ((int64_t)w * gstride + strip + (int64_t)row * m) * GS, row < rn ? (int64_t)m * GS : 0);
#pragma unroll
                for (int v = 0; v < NV; ++v) ld_graw<V, GBF>(gg, coff[v] * GS / 4u, g[i][v]);
            }
        }
#pragma unroll
        for (int i = 0; i < RS; ++i) {
            const int row = step * RS + i;
            const buf_rsrc er = make_rsrc(err + (int64_t)w * estride + strip + (int64_t)row * m, row < rn ? (int64_t)m * 4 : 0);
#pragma unroll
            for (int v = 0; v < NV; ++v) buf_ldv<V>(er, coff[v], e[i][v]);
        }
    };

    const buf_rsrc pres = make_rsrc(p + d.p_off + (int64_t)row0 * ri, gw == 0 ? (int64_t)rn * ri * 4 : 0);
    double S[NV][V][R];
#pragma unroll
    for (int v = 0; v < NV; ++v)
#pragma unroll
        for (int x = 0; x < V; ++x)
#pragma unroll
            for (int k = 0; k < R; ++k) S[v][x][k] = 0.0;
    double gsum = 0.0;
    int gab = 0;   // this lane's pair of columns a <= b of the Gram matrix: a + 16 b
    {
        int l = lane < NG ? lane : 0;
#pragma unroll
        for (int a = 0; a < R; ++a) {
            if (l >= 0 && l < R - a) gab = a + 16 * (a + l);
            l -= R - a;
        }
    }
    const float inv_w = 1.0f / (float)workers;

    int lstep = 0, lw = 0;   // the next item to request
    auto advance = [&]() {
        if (MEAN && ++lw < nw) return;
        lw = 0;
        ++lstep;
    };
#pragma unroll
    for (int u = 0; u < D; ++u) {
        load(lstep, lw, gr[u], ev[u]);
        advance();
    }
    // Q of the whole row, four floats of a lane's NC * R together, lane by lane (past NC * R: not read)
    float* qs = reinterpret_cast<float*>(one_lds);
    // (sizeof(PT) == 8: at a distance known when compiling, which an instruction's offset holds; else 16 addresses in registers)
    const int qdist = sizeof(PT) == 8 ? kOneMaxWaves * kWave : glanes;
    auto q_at = [&](int c) { return ((c >> 2) * qdist + gl) * 4 + (c & 3); };
    for (int v = group; v < NV; v += ngroups) {
        float f[V][R];
        const int jv = gl + glanes * v;
        load_factor_rows<R, V>(q + d.q_off + (int64_t)jv * V * ri, ri, jv < nvec, f);
#pragma unroll
        for (int x = 0; x < V; ++x)
#pragma unroll
            for (int k = 0; k < R; ++k) qs[q_at((v * V + x) * R + k)] = f[x][k];
    }
    __syncthreads();

    float M[RS][NV][V];
    if constexpr (MEAN) {
#pragma unroll
        for (int i = 0; i < RS; ++i)
#pragma unroll
            for (int v = 0; v < NV; ++v)
#pragma unroll
                for (int x = 0; x < V; ++x) M[i][v][x] = 0.f;
    }
    auto multiply = [&](int step) {
        int ln = lane;
        if constexpr (sizeof(PT) == 8) asm volatile("" : "+v"(ln));   // addresses are formed anew in every step, not held in registers
        // P of the step's rows, two chains per product and lane
        constexpr int CH = sizeof(PT) == 4 && V >= 2 ? 2 : 1;
        PT dot[RS][R][CH];
#pragma unroll
        for (int i = 0; i < RS; ++i)
#pragma unroll
            for (int k = 0; k < R; ++k)
#pragma unroll
                for (int x = 0; x < CH; ++x) dot[i][k][x] = PT(0);
#pragma unroll
        for (int c4 = 0; c4 < (NC * R + 3) / 4; ++c4) {
            if constexpr (sizeof(PT) == 8) {   // nor is M widened ahead of its products
                asm volatile("" : "+v"(M[0][4 * c4 / (R * V)][4 * c4 / R % V]));
            }
            if (c4 % (sizeof(PT) == 8 ? 2 : 3) == 0) asm volatile("" ::: "memory");   // Q is fetched from LDS a little at a time, in every step anew (registers)
            const f4 q4 = *reinterpret_cast<const f4*>(qs + (c4 * qdist + gl) * 4);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int c = 4 * c4 + u, k = c % R, x = c / R % V, v = c / (R * V);
                if (c >= NC * R) continue;
#pragma unroll
                for (int i = 0; i < RS; ++i) dot[i][k][x % CH] = fma((PT)M[i][v][x], (PT)q4[u], dot[i][k][x % CH]);
            }
        }
        PT part[N];
#pragma unroll
        for (int i = 0; i < RS; ++i)
#pragma unroll
            for (int k = 0; k < R; ++k) {
                if constexpr (CH == 2) part[i * R + k] = dot[i][k][0] + dot[i][k][1];
                else part[i * R + k] = dot[i][k][0];
            }
        PT sum = few_lane_sums<N>(part);
        if (per_row > 1) {
            if (ln < N) xsum[step & 1][wave][ln] = sum;
            lds_barrier();
            sum = PT(0);
            if (ln < N)
                for (int u = 0; u < per_row; ++u) sum += xsum[step & 1][(group << sh) + u][ln];
        }
        const float pf = (float)sum;   // lane i * R + k: row i, rank k
        {
            const int li = ln / R, lk = ln % R, row = step * RS + li;
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(pf), pres, ln < N && lk < ri ? (int)((row * ri + lk) * 4) : (int)kOutOfRange, 0, 0);
#pragma unroll
            for (int i = 0; i < RS; ++i) {
                const float pa = __int_as_float(__builtin_amdgcn_ds_bpermute((i * R + (gab & 15)) << 2, __float_as_int(pf)));
                const float pb = __int_as_float(__builtin_amdgcn_ds_bpermute((i * R + (gab >> 4)) << 2, __float_as_int(pf)));
                gsum = fma((double)pa, (double)pb, gsum);
            }
        }
        if constexpr (sizeof(PT) == 8) {   // M is widened again below, not kept in both widths
#pragma unroll
            for (int i = 0; i < RS; ++i)
#pragma unroll
                for (int v = 0; v < NV; ++v)
#pragma unroll
                    for (int x = 0; x < V; ++x) asm volatile("" : "+v"(M[i][v][x]));
        }
#pragma unroll
        for (int i = 0; i < RS; ++i) {
            double pd[R];
#pragma unroll
            for (int k = 0; k < R; ++k) pd[k] = (double)lane_bcast(pf, i * R + k);
#pragma unroll
            for (int v = 0; v < NV; ++v)
#pragma unroll
                for (int x = 0; x < V; ++x) {
                    const double md = (double)M[i][v][x];
#pragma unroll
                    for (int k = 0; k < R; ++k) S[v][x][k] = fma(md, pd[k], S[v][x][k]);
                    if constexpr (sizeof(PT) == 8) __builtin_amdgcn_sched_barrier(0);
                }
        }
    };
    int step = 0, w = 0;
    const int items = steps * nw;
    for (int it = 0; it < items; it += D) {   // items past the last one: zeros
#pragma unroll
        for (int u = 0; u < D; ++u) {
#pragma unroll
            for (int i = 0; i < RS; ++i) {
                const int row = step * RS + i;
                const buf_rsrc es = make_rsrc(err + (int64_t)w * estride + strip + (int64_t)row * m, row < rn ? (int64_t)m * 4 : 0);
#pragma unroll
                for (int v = 0; v < NV; ++v) {
                    float mw[V];
#pragma unroll
                    for (int x = 0; x < V; ++x) {
                        mw[x] = ev[u][i][v][x];
                        if constexpr (ADD) mw[x] += graw_at<V, GBF>(gr[u][i][v], x);
                    }
                    if constexpr (STORE) buf_stv<V>(es, coff[v], mw);
#pragma unroll
                    for (int x = 0; x < V; ++x) {
                        if constexpr (MEAN) M[i][v][x] = fmaf(mw[x], inv_w, M[i][v][x]);
                        else M[i][v][x] = mw[x];
                    }
                }
            }
            load(lstep, lw, gr[u], ev[u]);
            advance();
            __builtin_amdgcn_sched_barrier(0);   // the next step's work is not mixed into this one's (registers)
            if (!MEAN || w + 1 == nw) {
                multiply(step);
                if constexpr (MEAN) {
#pragma unroll
                    for (int i = 0; i < RS; ++i)
#pragma unroll
                        for (int v = 0; v < NV; ++v)
#pragma unroll
                            for (int x = 0; x < V; ++x) M[i][v][x] = 0.f;
                }
                ++step;
                w = 0;
            } else {
                ++w;
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    }

    // sums of the groups, in group order, VG column vectors of every lane at a time
    double* sdst = spart + d.s_off + (int64_t)t.block * m * ri;
    double* gdst = gpart + d.g_off + (int64_t)t.block * NG;
    constexpr int C = V * R;   // doubles of one column vector
    constexpr int VG = NV == one_nv(V, MEAN) ? one_deposit(R, V, MEAN) : 1;
    const int nthreads = blockDim.x;
    const int stride = nthreads + 1;
    double* gs = reinterpret_cast<double*>(one_lds);   // Q is no longer needed
    if (gw == 0 && lane < NG) xgram[group][lane] = gsum;
#pragma unroll
    for (int v0 = 0; v0 < NV; v0 += VG) {
        __syncthreads();
#pragma unroll
        for (int v = 0; v < VG; ++v)
#pragma unroll
            for (int c = 0; c < C; ++c) gs[(v * C + c) * stride + threadIdx.x] = S[v0 + v][c / R][c % R];
        __syncthreads();
        if (v0 == 0 && (int)threadIdx.x < NG) {
            double s = 0.0;
            for (int g = 0; g < ngroups; ++g) s += xgram[g][threadIdx.x];
            gdst[threadIdx.x] = s;
        }
        // column vector jv = glanes * v + l of the row, entry c
#pragma unroll
        for (int v = 0; v < VG; ++v) {
            const int total = min(glanes, nvec - glanes * (v0 + v)) * C;
            for (int idx = threadIdx.x; idx < total; idx += nthreads) {
                const int l = idx / C, c = idx % C, k = c % R;
                const double* src = gs + (v * C + c) * stride + l;
                double s = 0.0;
                for (int g = 0; g < ngroups; ++g) s += src[g * glanes];
                if (k < ri) sdst[(int64_t)((glanes * (v0 + v) + l) * V + c / R) * ri + k] = s;
            }
        }
    }
}

template <int R, bool ADD, bool GBF, bool STORE, bool MEAN>
__global__ __launch_bounds__(kOneMaxWaves * kWave, 2) void k_one_sweep(const OneMat* __restrict__ mats, const OneTile* __restrict__ tiles,
                                                                       const void* __restrict__ grad, float* __restrict__ err,
                                                                       const float* __restrict__ q, float* __restrict__ p,
                                                                       double* __restrict__ spart, double* __restrict__ gpart,
                                                                       int workers, int64_t gstride, int64_t estride) {
    __shared__ float xsum[2][kOneMaxWaves][kOneRows * kOneMaxRank];   // partial products of a step, by wavefront
    __shared__ double xgram[kOneMaxWaves][R * (R + 1) / 2];
    const OneTile t = tiles[blockIdx.x];
    const OneMat d = mats[t.mat];
#define PSGD_ONE_TILE(V)                                                                                                        \
    one_sweep_tile<R, V, one_nv(V, MEAN), kOneRows, one_depth(R, MEAN), float, ADD, GBF, STORE, MEAN>(                          \
        t, d, grad, err, q, p, spart, gpart, workers, gstride, estride, xsum, xgram)
    if (d.vec == 4) PSGD_ONE_TILE(4);
    else if (d.vec == 2) PSGD_ONE_TILE(2);
    else PSGD_ONE_TILE(1);
#undef PSGD_ONE_TILE
}

// ---- k_one_sweep_wide: rows of up to 8192 elements, bf16 gradients, one worker, M not stored ------------------------------
//
// What the sets beyond the memory-side cache take instead of the matrix cores' first two walks: they are bound by bytes, and 18 a step
// (6 here, 12 in a decompression that forms g + e again) are fewer than 24.  A row takes up to eight wavefronts with 16 columns a
// lane, whose fp64 sums are half of the registers, so a step is one row, two are in flight (98 KB a compute unit) and one workgroup fills
// a compute unit.  The products are summed in fp64 as on the matrix cores (error of P against 64 bits 3.7e-8 on either, of Q 1.7e-7 there,
// 2.6e-8 here).  24-layer transformer-shaped set: 1559 us, 5.0 TB/s.  Every register counts: with 33, 4 and 0 spilled ones, whose
// reloads wait for all loads before them, it took 3546, 1854 and 1559 us; hence Q at a fixed distance in shared memory, the
// addresses formed anew and M widened where it is used.
template <int R>
__global__ __launch_bounds__(kOneMaxWaves * kWave, 2) void k_one_sweep_wide(const OneMat* __restrict__ mats, const OneTile* __restrict__ tiles,
                                                                            const void* __restrict__ grad, float* __restrict__ err,
                                                                            const float* __restrict__ q, float* __restrict__ p,
                                                                            double* __restrict__ spart, double* __restrict__ gpart) {
    __shared__ double xsum[2][kOneMaxWaves][kOneRows * kOneMaxRank];
    __shared__ double xgram[kOneMaxWaves][R * (R + 1) / 2];
    const OneTile t = tiles[blockIdx.x];
    const OneMat d = mats[t.mat];
    one_sweep_tile<R, 4, kOneWideNV, 1, kOneWideDepth, double, true, true, false, false>(t, d, grad, err, q, p, spart, gpart, 1, 0, 0, xsum, xgram);
}

// ---- k_solve: R from the Gram matrix, P_hat = P R^-1, Q = S R^-1 -------------------------------------------
//
// A workgroup takes 256 rows of P (in place) or 16, 64 or 256 rows of Q, whose partial S its threads add up in slices of consecutive
// blocks; every workgroup adds the Gram matrices and factorises for itself (fp64; a pivot <= 1e-30 gives a zero column), so that
// none waits for another.  Bound by latency: LSTM-shaped set, rank 4: 8.4 us with 174 blocks, 12.3 with 350 (the two walks:
// k_gram_chol 10.7, k_q_reduce 6).
template <int R>
__global__ __launch_bounds__(kBlock) void k_solve(const OneMat* __restrict__ mats, const SolveTile* __restrict__ tiles,
                                                  const double* __restrict__ spart, const double* __restrict__ gpart,
                                                  float* __restrict__ p, float* __restrict__ q) {
    constexpr int NG = R * (R + 1) / 2;
    constexpr int GSL = kBlock / NG < 16 ? kBlock / NG : 16;   // slices of the row blocks' Gram matrices
    __shared__ double gred[GSL][NG];
    __shared__ double G[NG];
    __shared__ double Rm[R][R], rinv[R];
    __shared__ double sred[kBlock * R];
    const SolveTile t = tiles[blockIdx.x];
    const OneMat d = mats[t.mat];
    const int tid = threadIdx.x, r = d.r, nb = d.n_blocks;
    const int cpt = 1 << t.cols_log2, slices = kBlock >> t.cols_log2;
    const int c = tid & (cpt - 1), sl = tid >> t.cols_log2;
    // this thread's entry and slice of the row blocks' Gram matrices: the first eight are requested before anything is waited for
    constexpr int GU = 8;
    const int ent = tid % NG, gsl = tid / NG;
    const int gper = (nb + GSL - 1) / GSL;
    const int g0 = gsl < GSL ? min(nb, gsl * gper) : 0, g1 = gsl < GSL ? min(nb, g0 + gper) : 0;
    const double* gsrc = gpart + d.g_off + ent;
    double gx[GU];
#pragma unroll
    for (int u = 0; u < GU; ++u) gx[u] = g0 + u < g1 ? gsrc[(int64_t)(g0 + u) * NG] : 0.0;
    double row[R];
#pragma unroll
    for (int k = 0; k < R; ++k) row[k] = 0.0;
    if (t.rows) {
        if (tid < t.count) {
#pragma unroll
            for (int k = 0; k < R; ++k)
                if (k < r) row[k] = (double)p[d.p_off + (int64_t)(t.first + tid) * r + k];
        }
    } else if (c < t.count) {
        const int per = (nb + slices - 1) / slices;
        const int b0 = min(nb, sl * per), b1 = min(nb, b0 + per);
        const double* src = spart + d.s_off + (int64_t)(t.first + c) * r;
        const int64_t stride = (int64_t)d.m * r;
        int b = b0;
        constexpr int U = R <= 4 ? 8 : 4;
        for (; b + U <= b1; b += U) {
            double x[U][R];
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int k = 0; k < R; ++k) x[u][k] = k < r ? src[(int64_t)(b + u) * stride + k] : 0.0;
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int k = 0; k < R; ++k) row[k] += x[u][k];
        }
        for (; b < b1; ++b)
#pragma unroll
            for (int k = 0; k < R; ++k)
                if (k < r) row[k] += src[(int64_t)b * stride + k];
    }
    {
        double v = 0.0;
#pragma unroll
        for (int u = 0; u < GU; ++u) v += gx[u];
        for (int b = g0 + GU; b < g1; b += GU) {
#pragma unroll
            for (int u = 0; u < GU; ++u) gx[u] = b + u < g1 ? gsrc[(int64_t)(b + u) * NG] : 0.0;
#pragma unroll
            for (int u = 0; u < GU; ++u) v += gx[u];
        }
        if (gsl < GSL) gred[gsl][ent] = v;
    }
    if (!t.rows) {
#pragma unroll
        for (int k = 0; k < R; ++k) sred[(k * slices + sl) * cpt + c] = row[k];
    }
    __syncthreads();
    if (tid < NG) {
        double v = 0.0;
        for (int s = 0; s < GSL; ++s) v += gred[s][tid];
        G[tid] = v;
    }
    __syncthreads();
    if (tid == kBlock - 1) {   // the factor, by one thread (whose wavefront sums no columns below where several slices share one)
        double g[R][R], inv[R];
#pragma unroll
        for (int a = 0; a < R; ++a)
#pragma unroll
            for (int b = a; b < R; ++b) g[a][b] = G[a * R - a * (a - 1) / 2 + (b - a)];
        cholesky_rows<R>(g, inv, R);   // columns past the matrix's own rank: entries of zero
#pragma unroll
        for (int a = 0; a < R; ++a) {
            rinv[a] = inv[a];
#pragma unroll
            for (int b = a + 1; b < R; ++b) Rm[a][b] = g[a][b];
        }
    }
    if (!t.rows && sl == 0 && c < t.count) {
#pragma unroll
        for (int k = 0; k < R; ++k) {
            double v = 0.0;
            for (int s = 0; s < slices; ++s) v += sred[(k * slices + s) * cpt + c];
            row[k] = v;
        }
    }
    __syncthreads();
    const bool mine = t.rows ? tid < t.count : (sl == 0 && c < t.count);
    if (mine) {
        float* dst = t.rows ? p + d.p_off + (int64_t)(t.first + tid) * r : q + d.q_off + (int64_t)(t.first + c) * r;
#pragma unroll
        for (int j = 0; j < R; ++j) {
            double v = row[j];
#pragma unroll
            for (int k = 0; k < R; ++k)
                if (k < j) v -= row[k] * Rm[k][j];
            row[j] = v * rinv[j];
            if (j < r) dst[j] = (float)row[j];
        }
    }
}

// ---- host side ----------------------------------------------------------------------------------------------

// f<rank, ADD, GBF, STORE, MEAN>: what a plan runs when g is added (`add`), or on the M that err holds
template <int R, typename F>
static hipError_t one_sweep_variant(const psgd_plan* plan, bool add, F f) {
    const bool bf = plan->grad_dtype == PSGD_BF16;
    if (plan->workers > 1) {
        if (!add) return f(k_one_sweep<R, false, false, false, true>);
        return bf ? f(k_one_sweep<R, true, true, true, true>) : f(k_one_sweep<R, true, false, true, true>);
    }
    if (!add) return f(k_one_sweep<R, false, false, false, false>);
    return bf ? f(k_one_sweep<R, true, true, true, false>) : f(k_one_sweep<R, true, false, true, false>);
}
template <typename F>
static hipError_t one_sweep_dispatch(const psgd_plan* plan, bool add, F f) {
    switch (plan->rank) {
        case 1: return one_sweep_variant<1>(plan, add, f);
        case 2: return one_sweep_variant<2>(plan, add, f);
        case 3: return one_sweep_variant<3>(plan, add, f);
        case 4: return one_sweep_variant<4>(plan, add, f);
        default: return hipErrorInvalidValue;
    }
}

static psgd_status one_fail(psgd_plan* plan, hipError_t e, const char* what) {
    if (e == hipSuccess) return PSGD_OK;
    plan->last_error = std::string(what) + ": " + hipGetErrorString(e);
    return PSGD_EHIP;
}

psgd_status one_sweep_prepare(psgd_plan* plan) {   // more LDS than a workgroup has by default
    if (plan->one_wide)
        return one_fail(plan, hipFuncSetAttribute(reinterpret_cast<const void*>(k_one_sweep_wide<kOneMaxRank>),
                                                  hipFuncAttributeMaxDynamicSharedMemorySize, kOneWideLds),
                        "shared memory of k_one_sweep_wide");
    hipError_t e = hipSuccess;
    for (bool add : {true, false})
        if (e == hipSuccess)
            e = one_sweep_dispatch(plan, add, [&](auto kernel) {
                return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                           std::max(plan->one_lds_bytes, 128 << 10));
            });
    return one_fail(plan, e, "shared memory of k_one_sweep");
}

psgd_status launch_one_sweep(psgd_plan* plan, const void* grad, float* err, const float* q, float* p, void* stream, bool add) {
    double* spart = plan->one_part;
    double* gpart = spart + plan->one_s_doubles;
    hipError_t e = one_sweep_dispatch(plan, add, [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)plan->one_tiles.size()), dim3((unsigned)(plan->one_waves * kWave)),
                           (size_t)plan->one_lds_bytes, static_cast<hipStream_t>(stream), plan->dev.one_mats, plan->dev.one_tiles,
                           grad, err, q, p, spart, gpart, plan->workers, plan->sizes.grad_stride, plan->sizes.err_stride);
        return hipGetLastError();
    });
    return one_fail(plan, e, "launch k_one_sweep");
}

psgd_status launch_one_sweep_wide(psgd_plan* plan, const void* grad, float* err, const float* q, float* p, double* spart, double* gpart,
                                  void* stream) {
    hipLaunchKernelGGL(k_one_sweep_wide<kOneMaxRank>, dim3((unsigned)plan->one_tiles.size()), dim3(kOneMaxWaves * kWave),
                       (size_t)plan->one_lds_bytes, static_cast<hipStream_t>(stream), plan->dev.one_mats, plan->dev.one_tiles, grad, err, q,
                       p, spart, gpart);
    return one_fail(plan, hipGetLastError(), "launch k_one_sweep_wide");
}

psgd_status launch_solve(psgd_plan* plan, float* q, float* p, const double* spart, const double* gpart, void* stream) {
#define PSGD_SOLVE(RR)                                                                                                   \
    case RR:                                                                                                             \
        hipLaunchKernelGGL((k_solve<RR>), dim3((unsigned)plan->solve_tiles.size()), dim3(kBlock), 0,                     \
                           static_cast<hipStream_t>(stream), plan->dev.one_mats, plan->dev.solve_tiles, spart, gpart, p, q); \
        break
    switch (plan->rank) {
        PSGD_SOLVE(1);
        PSGD_SOLVE(2);
        PSGD_SOLVE(3);
        PSGD_SOLVE(4);
        default: return PSGD_EUNSUPPORTED;
    }
#undef PSGD_SOLVE
    return one_fail(plan, hipGetLastError(), "launch k_solve");
}

}  // namespace psgd
