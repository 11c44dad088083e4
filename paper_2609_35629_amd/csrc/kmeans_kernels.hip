// Minibatch k-means parents (Alg. "Global minibatch k-means parent partition"
// and the settings stated after it: greedy k-means++ seeding on a sample,
// minibatches drawn with replacement, cumulative-count center updates,
// reassignment of starved centers, a no-improvement rule on the smoothed
// minibatch inertia), and the parent member lists that feed the team build.
//
// Every (sequence, KV head) runs its own k-means on its prompt keys; all
// heads share the random draws (one seed serves every head's fit).  Draws:
// Philox4x64-10, key (seed, 1), counter (a / 4, tag, s, 0), word a mod 4; an
// index in [0, n) is floor(w n / 2^64), a uniform in [0, 1) is (w >> 11) 2^-53.
//   tag 0  seeding sample position a        tag 1  first center (a = 0)
//   tag 2  trial a of seeding round s        tag 3  batch position a of step s
//   tag 4  the a-th reassigned center of step s
//
// A distance between a key and a center is an fp64 sum over dimensions in
// index order with no fused multiply-add, so it equals the plain definition's
// value bit for bit when the center does.  Sums over many points (center
// updates, seeding potentials, the batch inertia) are blocked: per workgroup
// in point order, then over workgroups in order.  For bf16 keys these sums
// are exact in fp64 unless the keys span more than about 40 binary orders of
// magnitude, so they equal a sequential sum; otherwise they differ from it in
// the last bits.
//
// Kernels (one launch serves every (sequence, KV head); y = the pair)
//   k_kpp_sample   the seeding sample (token indices) and the first candidate
//   k_kpp_dist     seeding round c: min(D^2_j, |x_j - cand_t|^2) per sample
//                  point and candidate, and per-workgroup potential sums
//   k_kpp_pick     round c: the candidate with the smallest potential becomes
//                  center c, D^2 follows it, the next round's candidates are
//                  drawn from the running sums of D^2
//   k_km_assign    nearest center of each batch point (FINAL: of every
//                  token, written as its label); per-workgroup center sums
//   k_km_update    cumulative-count update of one center
//   k_km_control   reassignment, smoothed inertia and the stopping rule
//   k_parent_lists members of each parent in token order, parent and team
//                  offsets (Alg. "Build actual-key teams from a parent
//                  partition" numbers teams parent by parent)
#include <math.h>

#include <algorithm>

#include "common.h"
#include "internal.h"

namespace santapp {

namespace {

constexpr int kKppThreads = 256;
constexpr int kPickThreads = 1024;
constexpr int kPickCache = 16;  // sample values per thread k_kpp_pick keeps in registers
constexpr int kAsgThreads = 256;
constexpr int kAsgPts = 64;   // batch points per assignment workgroup
constexpr int kAsgCen = 32;   // centers per LDS tile
constexpr int kFullTile = 12; // points of a workgroup past which all are compared with every center together
constexpr int kUpdBatch = 32; // workgroup partials the center update loads at once
constexpr int kListThreads = 1024;
constexpr int kListWaves = kListThreads / kWave;
constexpr int kListAhead = 8;  // 64-token groups whose labels a wave reads at once

__device__ __forceinline__ uint64_t km_word(uint64_t seed, uint64_t a, uint64_t tag, uint64_t s) {
    const u64x4 r = philox4x64_10(a >> 2, tag, s, 0, seed, 1);
    const int e = static_cast<int>(a & 3);
    return e == 0 ? r.v[0] : e == 1 ? r.v[1] : e == 2 ? r.v[2] : r.v[3];
}

__device__ __forceinline__ int draw_index(uint64_t w, int n) {
    return static_cast<int>(__umul64hi(w, static_cast<uint64_t>(n)));
}

__device__ __forceinline__ double draw_unit(uint64_t w) {
    return static_cast<double>(w >> 11) * 0x1.0p-53;
}

// 16 bytes of a key row as floats (8 bf16 or 4 fp32 values, in order).
__device__ __forceinline__ void load_row16(const bf16_t* p, float (&v)[8]) {
    const uint4 w = *reinterpret_cast<const uint4*>(p);
    const uint32_t ws[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        v[2 * q] = bf16lo(ws[q]);
        v[2 * q + 1] = bf16hi(ws[q]);
    }
}

__device__ __forceinline__ void load_row16(const float* p, float (&v)[4]) {
    const uint4 w = *reinterpret_cast<const uint4*>(p);
    v[0] = __uint_as_float(w.x);
    v[1] = __uint_as_float(w.y);
    v[2] = __uint_as_float(w.z);
    v[3] = __uint_as_float(w.w);
}

// Sum of one value per lane over the wave, halves first (lane i + lane i ^ 32,
// then ^ 16, 8, 4, 2, 1); within 16 lanes a rotation reads what the xor would.
__device__ __forceinline__ double wave_sum_halves(double v) {
#pragma clang fp contract(off)
    v = v + __shfl_xor(v, 32);
    v = v + __shfl_xor(v, 16);
    v = v + dpp_f64<0x128>(v);
    v = v + dpp_f64<0x124>(v);
    v = v + dpp_f64<0x122>(v);
    v = v + dpp_f64<0x121>(v);
    return v;
}

__global__ __launch_bounds__(kKppThreads) void k_kpp_sample(int* __restrict__ samp, int s0, int N,
                                                            int* __restrict__ cand, int L, int BH,
                                                            uint64_t seed) {
    const int j = blockIdx.x * kKppThreads + threadIdx.x;
    if (j < s0) samp[j] = draw_index(km_word(seed, static_cast<uint64_t>(j), 0, 0), N);
    if (j == 0) {
        const int pos0 = draw_index(km_word(seed, 0, 1, 0), s0);
        for (int bh = 0; bh < BH; ++bh) cand[bh * L] = pos0;
    }
}

// A point per thread, the candidates' rows in LDS, 32 dimensions at a time: the
// point's next 32 are requested ahead, and a candidate's 32 are one run of LDS
// reads without a branch (a branch per candidate and dimension made every read
// a round trip).  At 12288 points, five candidates, four pairs, d = 128, bf16:
// 23.5 us a round before, now 11.1, of which the 128 x 5 fp64 terms take 3.
template <typename T, int D>
__global__ __launch_bounds__(kKppThreads) void k_kpp_dist(
    const T* __restrict__ K, int N, const int* __restrict__ samp, int s0, const int* __restrict__ cand,
    int L, int c, double* __restrict__ D2, double* __restrict__ Dt, double* __restrict__ part) {
#pragma clang fp contract(off)
    __shared__ __align__(16) double s_cand[kKmMaxTrials][D];
    __shared__ double s_w[kKmMaxTrials][kKppThreads / kWave];
    __shared__ int s_ctok[kKmMaxTrials];
    const int bh = blockIdx.y, tid = threadIdx.x, lane = lane_id(), wv = wave_id();
    const int nc = c == 0 ? 1 : L;
    const T* X = K + static_cast<size_t>(bh) * N * D;
    const int j = blockIdx.x * kKppThreads + tid;
    const bool valid = j < s0;
    constexpr int kPer = 16 / static_cast<int>(sizeof(T));
    if (tid < nc) s_ctok[tid] = samp[cand[bh * L + tid]];
    const T* x = X + static_cast<size_t>(samp[valid ? j : 0]) * D;
    const double dcur = (valid && c > 0) ? D2[static_cast<size_t>(bh) * s0 + j] : 0.0;
    constexpr int kDims = 32, kRaw = kDims / kPer;
    uint4 raw[kRaw];
#pragma unroll
    for (int q = 0; q < kRaw; ++q) raw[q] = reinterpret_cast<const uint4*>(x)[q];
    __syncthreads();
    for (int e = tid; e < nc * (D / kPer); e += kKppThreads) {
        const int t = e / (D / kPer), k0 = (e % (D / kPer)) * kPer;
        float v[kPer];
        load_row16(X + static_cast<size_t>(s_ctok[t]) * D + k0, v);
#pragma unroll
        for (int r = 0; r < kPer; ++r) s_cand[t][k0 + r] = static_cast<double>(v[r]);
    }
    __syncthreads();
    double acc[kKmMaxTrials];
#pragma unroll
    for (int t = 0; t < kKmMaxTrials; ++t) acc[t] = 0.0;
#pragma unroll 1
    for (int k0 = 0; k0 < D; k0 += kDims) {
        float xv[kDims];
#pragma unroll
        for (int q = 0; q < kRaw; ++q) load_row16(reinterpret_cast<const T*>(&raw[q]), *reinterpret_cast<float(*)[kPer]>(&xv[q * kPer]));
        const int kn = min(k0 + kDims, D - kDims);
#pragma unroll
        for (int q = 0; q < kRaw; ++q) raw[q] = reinterpret_cast<const uint4*>(x + kn)[q];
        // candidate t's sum runs in dimension order
#pragma unroll
        for (int t = 0; t < kKmMaxTrials; ++t) {
            if (t < nc) {  // uniform
                double2 y[kDims / 2];
#pragma unroll
                for (int q = 0; q < kDims / 2; ++q) y[q] = *reinterpret_cast<const double2*>(&s_cand[t][k0 + 2 * q]);
#pragma unroll
                for (int q = 0; q < kDims / 2; ++q) {
                    const double e0 = static_cast<double>(xv[2 * q]) - y[q].x;
                    acc[t] = acc[t] + e0 * e0;
                    const double e1 = static_cast<double>(xv[2 * q + 1]) - y[q].y;
                    acc[t] = acc[t] + e1 * e1;
                }
            }
        }
    }
#pragma unroll
    for (int t = 0; t < kKmMaxTrials; ++t) {
        if (t < nc) {  // uniform
            double m = 0.0;
            if (valid) {
                m = (c == 0) ? acc[t] : (acc[t] < dcur ? acc[t] : dcur);
                Dt[(static_cast<size_t>(bh) * L + t) * s0 + j] = m;
            }
            const double tot = wave_sum_halves(m);
            if (lane == 0) s_w[t][wv] = tot;
        }
    }
    __syncthreads();
    if (tid < nc) {  // the waves in order
        double r = 0.0;
        for (int w = 0; w < kKppThreads / kWave; ++w) r = r + s_w[tid][w];
        part[(static_cast<size_t>(bh) * gridDim.x + blockIdx.x) * L + tid] = r;
    }
}

// One workgroup per pair: a chain of round trips.  The sample's distances come
// in with neighbouring threads on neighbouring values and reach their owners
// (contiguous ranges) through LDS, and only the thread in whose range a trial's
// draw falls looks for the position.  Reading the ranges in place and
// comparing every value with every trial's draw took 18 us (12288 values, five
// trials, four pairs); now 11.7.
template <typename T, int D>
__global__ __launch_bounds__(kPickThreads) void k_kpp_pick(
    const T* __restrict__ K, int N, const int* __restrict__ samp, int s0, int* __restrict__ cand,
    int L, int c, int M, int nblk, double* __restrict__ D2, const double* __restrict__ Dt,
    const double* __restrict__ part, double* __restrict__ cent, uint64_t seed) {
#pragma clang fp contract(off)
    __shared__ double s_pot[kKmMaxTrials];
    __shared__ double s_tot[kPickThreads / kWave];
    __shared__ int s_first[kKmMaxTrials], s_ctok[kKmMaxTrials];
    __shared__ double s_u[kKmMaxTrials];
    __shared__ double s_val[kPickThreads * (kPickCache + 1)];  // a range's values, one place of padding per range
    const int bh = blockIdx.x, tid = threadIdx.x;
    const int nc = c == 0 ? 1 : L;
    const T* X = K + static_cast<size_t>(bh) * N * D;
    if (tid < nc) s_ctok[tid] = samp[cand[bh * L + tid]];
    if (tid >= kPickThreads - L)
        s_u[kPickThreads - 1 - tid] =
            draw_unit(km_word(seed, static_cast<uint64_t>(kPickThreads - 1 - tid), 2, static_cast<uint64_t>(c + 1)));
    if (wave_id() < nc) {  // wave t sums trial t's workgroup partials
        const int t = wave_id();
        double p = 0.0;
        for (int b = lane_id(); b < nblk; b += kWave) p = p + part[(static_cast<size_t>(bh) * nblk + b) * L + t];
        for (int off = kWave / 2; off > 0; off >>= 1) p = p + __shfl_xor(p, off);
        if (lane_id() == 0) s_pot[t] = p;
    }
    if (tid < kKmMaxTrials) s_first[tid] = kPickThreads;
    __syncthreads();
    int best = 0;
    for (int t = 1; t < nc; ++t)
        if (s_pot[t] < s_pot[best]) best = t;
    const int tok = s_ctok[best];
    for (int k = tid; k < D; k += kPickThreads)
        cent[(static_cast<size_t>(bh) * M + c) * D + k] = static_cast<double>(load_elem(X + static_cast<size_t>(tok) * D, k));
    const double* src = Dt + (static_cast<size_t>(bh) * L + best) * s0;
    double* dst = D2 + static_cast<size_t>(bh) * s0;
    if (c + 1 >= M) {
        for (int j = tid; j < s0; j += kPickThreads) dst[j] = src[j];
        return;
    }
    // running sums of D^2 over the sample in index order: thread tid owns
    // the contiguous range [tid per, (tid + 1) per)
    const int per = (s0 + kPickThreads - 1) / kPickThreads;
    const int j0 = min(s0, tid * per), j1 = min(s0, j0 + per);
    double vals[kPickCache];
    double loc = 0.0;
    if (per <= kPickCache) {  // uniform
#pragma unroll
        for (int q = 0; q < kPickCache; ++q) vals[q] = src[min(q * kPickThreads + tid, s0 - 1)];
#pragma unroll
        for (int q = 0; q < kPickCache; ++q) {
            const int j = q * kPickThreads + tid;
            if (j < s0) {
                dst[j] = vals[q];
                s_val[j + j / per] = vals[q];
            }
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < kPickCache; ++q) {
            vals[q] = s_val[tid * (per + 1) + q];
            if (j0 + q < j1) loc = loc + vals[q];
        }
    } else {
        for (int j = j0; j < j1; ++j) {
            const double v = src[j];
            dst[j] = v;
            loc = loc + v;
        }
    }
    // scan of the thread sums in thread order
    double inc = loc;
    for (int off = 1; off < kWave; off <<= 1) {
        const double y = __shfl_up(inc, off);
        if (lane_id() >= off) inc = y + inc;
    }
    double exc = __shfl_up(inc, 1);
    if (lane_id() == 0) exc = 0.0;
    if (lane_id() == kWave - 1) s_tot[wave_id()] = inc;
    __syncthreads();
    double wpre = 0.0, total = 0.0;
    for (int w = 0; w < kPickThreads / kWave; ++w) {
        if (w < wave_id()) wpre = wpre + s_tot[w];
        total = total + s_tot[w];
    }
    const double pre = wpre + exc;
    // trial t takes the first position whose running sum exceeds its draw.  The
    // values are not negative, so a range holds such a position exactly when the
    // running sum at its end exceeds the draw; the first such range's thread
    // looks for it (a draw that is not finite is exceeded nowhere).
    double run = pre;
    if (per <= kPickCache) {
#pragma unroll
        for (int q = 0; q < kPickCache; ++q)
            if (j0 + q < j1) run = run + vals[q];
    } else {
        for (int j = j0; j < j1; ++j) run = run + src[j];
    }
    for (int t = 0; t < L; ++t) {  // uniform
        const uint64_t over = __ballot(j0 < j1 && run > s_u[t] * total);
        if (lane_id() == 0 && over != 0)
            atomicMin(&s_first[t], wave_id() * kWave + __ffsll(static_cast<unsigned long long>(over)) - 1);
    }
    __syncthreads();
    for (int t = 0; t < L; ++t) {
        const int owner = s_first[t];
        if (owner == kPickThreads) {  // the draw is the total: the last position
            if (tid == 0) cand[bh * L + t] = s0 - 1;
        } else if (owner == tid) {
            const double target = s_u[t] * total;
            double at = pre;
            int found = -1;
            if (per <= kPickCache) {
#pragma unroll
                for (int q = 0; q < kPickCache; ++q) {
                    if (j0 + q < j1) at = at + vals[q];
                    if (found < 0 && at > target) found = j0 + q;
                }
            } else {
                for (int j = j0; found < 0; ++j) {
                    at = at + src[j];
                    if (at > target || j + 1 >= j1) found = j;
                }
            }
            cand[bh * L + t] = found;
        }
    }
}

// |x - c|^2 of a staged point (fp32, exact values) and a center, the
// definition's way: fp64 in dimension order, no fused multiply-add.
template <int D>
__device__ __forceinline__ double point_dist(const float* x, const double* __restrict__ c) {
#pragma clang fp contract(off)
    double acc = 0.0;
#pragma unroll 1
    for (int k = 0; k < D; k += 32) {  // 32 dimensions in flight
        double2 v[16];
        float xs[32];
#pragma unroll
        for (int q = 0; q < 16; ++q) v[q] = reinterpret_cast<const double2*>(c + k)[q];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const float4 y = reinterpret_cast<const float4*>(x + k)[q];
            xs[4 * q] = y.x;
            xs[4 * q + 1] = y.y;
            xs[4 * q + 2] = y.z;
            xs[4 * q + 3] = y.w;
        }
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            const double t0 = static_cast<double>(xs[2 * q]) - v[q].x;
            acc = acc + t0 * t0;
            const double t1 = static_cast<double>(xs[2 * q + 1]) - v[q].y;
            acc = acc + t1 * t1;
        }
    }
    return acc;
}

// A point's three smallest estimated distances and the centers of the first
// two.
struct Near3 {
    float d1, d2, d3;
    int u1, u2;
    __device__ __forceinline__ void add(float d, int u) {
        const bool first = d < d1, second = d < d2;
        d3 = fminf(d3, fmaxf(d2, d));
        d2 = fminf(d2, fmaxf(d1, d));
        d1 = fminf(d1, d);
        u2 = first ? u1 : second ? u : u2;
        u1 = first ? u : u1;
    }
    // with the lane CTRL (a DPP row rotation) away
    template <int CTRL>
    __device__ __forceinline__ void merge() {
        const float o1 = dpp_f32<CTRL>(d1), o2 = dpp_f32<CTRL>(d2), o3 = dpp_f32<CTRL>(d3);
        const int w1 = __builtin_amdgcn_update_dpp(0, u1, CTRL, 0xF, 0xF, false);
        const int w2 = __builtin_amdgcn_update_dpp(0, u2, CTRL, 0xF, 0xF, false);
        add(o1, w1);
        add(o2, w2);
        d3 = fminf(d3, o3);
    }
};

// Nearest center of 64 points per workgroup.  The centers are compared on fp32
// estimates |c|^2 - 2 x.c, center tiles of 32 in LDS: a wave's 16 points
// against 16 centers as one tile of v_mfma_f32_16x16x4_f32 (A point i on lanes
// 16 c + i, B center j on lanes 16 c + j, lane group c holding dims [c D / 4,
// (c + 1) D / 4); register r of lane 16 c + j is point 4 c + r, center j).  The
// definition's fp64 distance is then formed for the nearest center (the batch
// inertia sums it) and, where the estimates of the two nearest lie within the
// error bound, for the second; a point with a third that close, or whose
// estimates left fp32's range, is compared with every center that way.
//
// Error bound: an inner product rounds at most five times per product step and
// D / 4 <= 32 steps, each by at most 2^-23 of |x| |c|; with the norms' own
// sums and the centers' rounding an estimate is off by less than 700 x 2^-24
// (|x| |c| + |c|^2).
//
// With fp64 distances to all centers a step took 23.2 us (32 centers, 4096
// points, four pairs, d = 128, bf16) and the labels of 32K tokens 82 us; now
// 15.2 and 41 us, one workgroup per CU and a chain of latencies: the draw, the
// rows, the estimates, one fp64 distance, the sort by center and the sums.
template <typename T, int D, bool FINAL>
__global__ __launch_bounds__(kAsgThreads) void k_km_assign(
    const T* __restrict__ K, int N, int M, int batch, int step, uint64_t seed,
    const double* __restrict__ cent, const KmState* __restrict__ state, int* __restrict__ labels,
    double* __restrict__ bpart, int* __restrict__ bcnt, double* __restrict__ binert) {
#pragma clang fp contract(off)
    constexpr int S = D + 4;  // row stride: whole 16-byte reads, rows spread over the banks
    __shared__ __align__(16) float s_x[kAsgPts][S];  // exact key values
    __shared__ __align__(16) float s_c[kAsgCen][S];  // centers rounded to fp32
    __shared__ __align__(16) double s_cd[FINAL ? 1 : kAsgCen][D + 2];  // the first tile's centers as they are
    __shared__ int s_tok[kAsgPts];
    __shared__ int s_lab[kAsgPts];
    __shared__ double s_e[kAsgPts];
    __shared__ int s_ord[kAsgPts];
    __shared__ Near3 s_near[kAsgPts];
    __shared__ double s_second[kAsgPts];
    __shared__ float s_err[kAsgThreads / kWave];  // twice a wave's error bound; negative: all zero
    __shared__ int s_full, s_list[kAsgPts];
    const int bh = blockIdx.y, tid = threadIdx.x;
    if (!FINAL && state[bh].stop) return;
    const T* X = K + static_cast<size_t>(bh) * N * D;
    const int npts = FINAL ? N : batch;
    const int p0 = blockIdx.x * kAsgPts;
    const double* cb = cent + static_cast<size_t>(bh) * M * D;
    // a tile's centers (rows past the last center read center 0 and are not
    // compared), the first tile's requested before the points are drawn
    static_assert(kAsgCen * D % (4 * kAsgThreads) == 0, "whole tile quads per thread");
    constexpr int kQuads = kAsgCen * D / (4 * kAsgThreads);
    double2 cv0[kQuads], cv1[kQuads];
    auto load_tile = [&](int ct) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < kQuads; ++q) {
            const int e = q * kAsgThreads + tid, u = e / (D / 4), k = 4 * (e % (D / 4));
            const double2* src = reinterpret_cast<const double2*>(cb + static_cast<size_t>(ct + u < M ? ct + u : 0) * D + k);
            cv0[q] = src[0];
            cv1[q] = src[1];
        }
    };
    load_tile(0);
    if (tid < kAsgPts) {
        const int j = p0 + tid;
        int tok = -1;
        if (j < npts) tok = FINAL ? j : draw_index(km_word(seed, static_cast<uint64_t>(j), 3, static_cast<uint64_t>(step)), N);
        s_tok[tid] = tok;
    }
    if (tid == 0) s_full = 0;
    __syncthreads();
    // point rows, 16 bytes per load: every load of a thread is independent
    {
        constexpr int kPer = 16 / static_cast<int>(sizeof(T));
        constexpr int kChunks = kAsgPts * D / kPer;
        static_assert(kChunks % kAsgThreads == 0, "whole 16-byte chunks per thread");
        float v[kChunks / kAsgThreads][kPer];
#pragma unroll
        for (int q = 0; q < kChunks / kAsgThreads; ++q) {
            const int e = q * kAsgThreads + tid;
            const int p = e / (D / kPer), k0 = (e % (D / kPer)) * kPer;
            const int tok = s_tok[p];
            load_row16(X + static_cast<size_t>(tok >= 0 ? tok : 0) * D + k0, v[q]);
        }
#pragma unroll
        for (int q = 0; q < kChunks / kAsgThreads; ++q) {
            const int e = q * kAsgThreads + tid;
            const int p = e / (D / kPer), k0 = (e % (D / kPer)) * kPer;
            const bool ok = s_tok[p] >= 0;
#pragma unroll
            for (int r = 0; r < kPer; r += 4) {
                const float4 y = ok ? make_float4(v[q][r], v[q][r + 1], v[q][r + 2], v[q][r + 3]) : make_float4(0.f, 0.f, 0.f, 0.f);
                *reinterpret_cast<float4*>(&s_x[p][k0 + r]) = y;
            }
        }
    }
    constexpr int kVec = D / 16;  // 16-byte pieces of a lane's quarter row
    const int lane = lane_id(), wv = wave_id(), cgrp = lane >> 4, j16 = lane & 15;
    float4 xf[kVec];
    float xn2 = 0.f, xabs = 0.f, cn2 = 0.f, cabs = 0.f;  // largest squared norms and magnitudes
    Near3 nr[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) nr[i] = Near3{INFINITY, INFINITY, INFINITY, 0x7fffffff, 0x7fffffff};
    auto quarter = [&](const float* row, float4 (&v)[kVec], float& n2, float& mx) __attribute__((always_inline)) {
        n2 = 0.f;
        mx = 0.f;
#pragma unroll
        for (int q = 0; q < kVec; ++q) {
            v[q] = reinterpret_cast<const float4*>(row + cgrp * (D / 4))[q];
            n2 = fmaf(v[q].x, v[q].x, fmaf(v[q].y, v[q].y, fmaf(v[q].z, v[q].z, fmaf(v[q].w, v[q].w, n2))));
            mx = fmaxf(mx, fmaxf(fmaxf(fabsf(v[q].x), fabsf(v[q].y)), fmaxf(fabsf(v[q].z), fabsf(v[q].w))));
        }
        n2 += __shfl_xor(n2, 16);
        n2 += __shfl_xor(n2, 32);
    };
    for (int ct = 0; ct < M; ct += kAsgCen) {
        if (ct > 0) {
            load_tile(ct);
            __syncthreads();  // the previous tile is no longer read
        }
        const int nct = min(kAsgCen, M - ct);
#pragma unroll
        for (int q = 0; q < kQuads; ++q) {
            const int e = q * kAsgThreads + tid, u = e / (D / 4), k = 4 * (e % (D / 4));
            *reinterpret_cast<float4*>(&s_c[u][k]) = make_float4(static_cast<float>(cv0[q].x), static_cast<float>(cv0[q].y),
                                                                 static_cast<float>(cv1[q].x), static_cast<float>(cv1[q].y));
            if (!FINAL && ct == 0) {
                *reinterpret_cast<double2*>(&s_cd[FINAL ? 0 : u][k]) = cv0[q];
                *reinterpret_cast<double2*>(&s_cd[FINAL ? 0 : u][k + 2]) = cv1[q];
            }
        }
        __syncthreads();
        if (ct == 0) quarter(s_x[16 * wv + j16], xf, xn2, xabs);
#pragma unroll
        for (int t = 0; t < kAsgCen / 16; ++t) {
            float4 cf[kVec];
            float n2, mx;
            quarter(s_c[16 * t + j16], cf, n2, mx);
            f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int q = 0; q < kVec; ++q) {
                acc = __builtin_amdgcn_mfma_f32_16x16x4f32(xf[q].x, cf[q].x, acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_16x16x4f32(xf[q].y, cf[q].y, acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_16x16x4f32(xf[q].z, cf[q].z, acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_16x16x4f32(xf[q].w, cf[q].w, acc, 0, 0, 0);
            }
            if (16 * t + j16 < nct) {
                cn2 = fmaxf(cn2, n2);
                cabs = fmaxf(cabs, mx);
                if (!(n2 < INFINITY)) cn2 = INFINITY;  // NaN too
#pragma unroll
                for (int r = 0; r < 4; ++r) nr[r].add(fmaf(-2.f, acc[r], n2), ct + 16 * t + j16);
            }
        }
    }
    // the 16 lanes that share a point's centers
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        nr[r].merge<0x128>();
        nr[r].merge<0x124>();
        nr[r].merge<0x122>();
        nr[r].merge<0x121>();
        if (j16 == r) s_near[16 * wv + 4 * cgrp + r] = nr[r];
    }
    {
        const bool odd = __ballot(!(xn2 < INFINITY)) != 0;
        const float x2 = odd ? INFINITY : wave_max_f32(xn2), c2 = wave_max_f32(cn2);
        const bool zero = !odd && c2 < INFINITY && wave_max_f32(fmaxf(xabs, cabs)) == 0.f;  // every distance is 0
        const float size = __fsqrt_rn(x2) * __fsqrt_rn(c2) + c2;
        if (lane == 0) s_err[wv] = zero ? -1.f : c2 > 1e-30f && size < 1e30f && x2 < 1e30f ? 1400.f * 0x1.0p-24f * size : INFINITY;
    }
    __syncthreads();
    // threads 0 .. 63: a point and its nearest center, 64 .. 127: its second
    // nearest where the estimates leave the choice open
    if (tid < 2 * kAsgPts) {
        const int p = tid & (kAsgPts - 1);
        Near3 x = s_near[p];
        const float err2 = s_err[p >> 4];
        if (err2 < 0.f) {
            x.u1 = 0;
            s_near[p].u1 = 0;
        }
        const bool two = err2 >= 0.f && M > 1 && !(x.d2 - x.d1 > err2);
        const bool full = err2 == INFINITY || (two && M > 2 && !(x.d3 - x.d1 > err2));
        if (s_tok[p] >= 0) {
            if (full) {
                if (tid < kAsgPts) s_list[atomicAdd(&s_full, 1)] = p;
            } else if (tid < kAsgPts) {
                if (!FINAL && x.u1 < kAsgCen)
                    s_e[p] = point_dist<D>(s_x[p], s_cd[FINAL ? 0 : x.u1]);
                else if (!FINAL || two)
                    s_e[p] = point_dist<D>(s_x[p], cb + static_cast<size_t>(x.u1) * D);
                s_lab[p] = x.u1;
            } else {
                s_second[p] = two ? point_dist<D>(s_x[p], cb + static_cast<size_t>(x.u2) * D) : INFINITY;
            }
        }
    }
    __syncthreads();
    if (tid < kAsgPts && s_tok[tid] >= 0) {
        const Near3 x = s_near[tid];
        bool listed = false;
        for (int i = 0; i < s_full; ++i) listed = listed || s_list[i] == tid;
        const double second = listed ? INFINITY : s_second[tid];
        if (!listed && second < INFINITY && (second < s_e[tid] || (second == s_e[tid] && x.u2 < x.u1))) {
            s_e[tid] = second;
            s_lab[tid] = x.u2;
        }
    }
    // every center: half a wave per point, or, for many points, all points
    // against 16 centers at a time in LDS (a lane per point, a wave per four
    // centers).  Where every point comes here (keys whose common offset is 100
    // times their spread), k-means parents of 32K tokens (32 centers, four pairs,
    // d = 128, bf16) took 2600 us with half a wave per point alone, 2210 with fp64
    // distances throughout; now 1590.  The line: eight points take half a wave
    // each 2 us, all points together 2.7.
    if (s_full > kFullTile) {  // uniform
        typedef double f64x2 __attribute__((ext_vector_type(2)));
        constexpr int kCen = 16, kRow = D + 2;
        static_assert(kCen * kRow * sizeof(double) <= sizeof(s_c), "the fp64 tile lies where the fp32 one was");
        double* const s_t = reinterpret_cast<double*>(&s_c[0][0]);
        double bd = INFINITY;
        int bu = 0x7fffffff;
        for (int ct = 0; ct < M; ct += kCen) {
            constexpr int kPieces = kCen * D / (2 * kAsgThreads);
            f64x2 v[kPieces];
#pragma unroll
            for (int q = 0; q < kPieces; ++q) {
                const int e = q * kAsgThreads + tid, u = e / (D / 2), k = 2 * (e % (D / 2));
                v[q] = *reinterpret_cast<const f64x2*>(cb + static_cast<size_t>(min(ct + u, M - 1)) * D + k);
            }
            __syncthreads();
#pragma unroll
            for (int q = 0; q < kPieces; ++q) {
                const int e = q * kAsgThreads + tid, u = e / (D / 2), k = 2 * (e % (D / 2));
                *reinterpret_cast<f64x2*>(s_t + u * kRow + k) = v[q];
            }
            __syncthreads();
            double acc[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 2
            for (int k = 0; k < D; k += 4) {
                const float4 x = *reinterpret_cast<const float4*>(&s_x[lane][k]);
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const double2 y0 = *reinterpret_cast<const double2*>(s_t + (4 * wv + c) * kRow + k);
                    const double2 y1 = *reinterpret_cast<const double2*>(s_t + (4 * wv + c) * kRow + k + 2);
                    const double t0 = static_cast<double>(x.x) - y0.x;
                    acc[c] = acc[c] + t0 * t0;
                    const double t1 = static_cast<double>(x.y) - y0.y;
                    acc[c] = acc[c] + t1 * t1;
                    const double t2 = static_cast<double>(x.z) - y1.x;
                    acc[c] = acc[c] + t2 * t2;
                    const double t3 = static_cast<double>(x.w) - y1.y;
                    acc[c] = acc[c] + t3 * t3;
                }
            }
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const int u = ct + 4 * wv + c;
                if (u < M && acc[c] < bd) {
                    bd = acc[c];
                    bu = u;
                }
            }
        }
        // the four waves' best of each point
        static_assert(kAsgPts == kWave && kAsgThreads == 4 * kWave, "a lane per point, four centers a wave");
        int* const s_u = reinterpret_cast<int*>(s_t + kAsgThreads);
        __syncthreads();
        s_t[tid] = bd;
        s_u[tid] = bu;
        __syncthreads();
        if (tid < s_full) {
            const int p = s_list[tid];
            for (int w = 0; w < kAsgThreads / kWave; ++w) {
                const double od = s_t[w * kWave + p];
                const int ou = s_u[w * kWave + p];
                if (w == 0 || od < bd || (od == bd && ou < bu)) {
                    bd = od;
                    bu = ou;
                }
            }
            s_lab[p] = bu < M ? bu : 0;  // as below
            s_e[p] = bd;
        }
    } else {
        for (int i = tid >> 5; i < s_full; i += kAsgThreads / 32) {
            const int p = s_list[i];
            double bd = INFINITY;
            int bu = 0x7fffffff;
            for (int u = tid & 31; u < M; u += 32) {
                const double d2 = point_dist<D>(s_x[p], cb + static_cast<size_t>(u) * D);
                if (d2 < bd) {
                    bd = d2;
                    bu = u;
                }
            }
            for (int off = 16; off > 0; off >>= 1) {
                const double od = __shfl_xor(bd, off);
                const int ou = __shfl_xor(bu, off);
                if (od < bd || (od == bd && ou < bu)) {
                    bd = od;
                    bu = ou;
                }
            }
            if ((tid & 31) == 0) {
                // no winner (NaN keys): center 0, so every label stays in range
                s_lab[p] = bu < M ? bu : 0;
                s_e[p] = bd;
            }
        }
    }
    __syncthreads();
    if (FINAL) {
        if (tid < kAsgPts && s_tok[tid] >= 0) labels[static_cast<size_t>(bh) * N + s_tok[tid]] = s_lab[tid];
        return;
    }
    const int nv = min(kAsgPts, npts - p0);  // valid points: 0 .. nv - 1
    const size_t blk = static_cast<size_t>(bh) * gridDim.x + blockIdx.x;
    if (tid == 2 * kAsgPts) {
        double s = 0.0;
        for (int q0 = 0; q0 < nv; q0 += 16) {
            double v[16];
#pragma unroll
            for (int q = 0; q < 16; ++q) v[q] = s_e[min(q0 + q, nv - 1)];
#pragma unroll
            for (int q = 0; q < 16; ++q)
                if (q0 + q < nv) s = s + v[q];
        }
        binert[blk] = s;
    }
    // points ordered by (center, position), a stable counting sort, by wave 0;
    // the centers' counts by the waves after it (lane p holds point p's label)
    static_assert(kAsgPts == kWave, "a lane per point");
    {
        const int lab = lane < nv ? s_lab[lane] : 0x7fffffff;
        if (wv == 0) {
            int r = 0;
#pragma unroll 8
            for (int q = 0; q < kAsgPts; ++q) {
                const int v = readlane(lab, q);
                r += (v < lab || (v == lab && q < lane)) ? 1 : 0;
            }
            if (lane < nv) s_ord[r] = lane;
        } else {
            for (int u0 = (wv - 1) * kWave; u0 < M; u0 += kAsgThreads - kWave) {  // uniform
                const int u = u0 + lane;
                int n = 0;
#pragma unroll 8
                for (int q = 0; q < kAsgPts; ++q) n += readlane(lab, q) == u ? 1 : 0;
                if (u < M) bcnt[blk * M + u] = n;
            }
        }
    }
    __syncthreads();
    // each present center's sum, in point order: a wave takes the centers whose
    // first sorted point lies in its quarter of the order, a lane D / 64
    // dimensions; eight points' values are read ahead of their additions
    {
        constexpr int kDims = D / kWave;
        const int ord = lane < nv ? s_ord[lane] : 0, lab = lane < nv ? s_lab[ord] : -1;
        const int before = __shfl_up(lab, 1);
        const uint64_t starts = __ballot(lane < nv && (lane == 0 || lab != before));
        constexpr int kPart = kAsgPts / (kAsgThreads / kWave);
        auto first = [&](int from) {  // the first center start at or after `from`
            const uint64_t x = from < kWave ? starts >> from : 0;
            return x != 0 ? from + __ffsll(static_cast<unsigned long long>(x)) - 1 : nv;
        };
        const int r1 = first((wv + 1) * kPart);
        double acc[kDims];
        for (int r0 = first(wv * kPart); r0 < r1; r0 += 8) {
            float xx[8][kDims];
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const int p = readlane(ord, min(r0 + q, r1 - 1));
#pragma unroll
                for (int e = 0; e < kDims; ++e) xx[q][e] = s_x[p][kDims * lane + e];
            }
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const int r = r0 + q;
                if (r < r1) {  // uniform
                    const bool start = (starts >> r) & 1ull;
#pragma unroll
                    for (int e = 0; e < kDims; ++e)
                        acc[e] = (start ? 0.0 : acc[e]) + static_cast<double>(xx[q][e]);
                    if (r + 1 == r1 || ((starts >> (r + 1)) & 1ull)) {  // the center's last point
#pragma unroll
                        for (int e = 0; e < kDims; ++e)
                            bpart[(blk * M + readlane(lab, r)) * D + kDims * lane + e] = acc[e];
                    }
                }
            }
        }
    }
}

template <int D>
__global__ __launch_bounds__(D) void k_km_update(int M, int nblk, const double* __restrict__ bpart,
                                                 const int* __restrict__ bcnt, double* __restrict__ cent,
                                                 double* __restrict__ w, const KmState* __restrict__ state) {
#pragma clang fp contract(off)
    const int u = blockIdx.x, bh = blockIdx.y, k = threadIdx.x;
    if (state[bh].stop) return;
    // kUpdBatch workgroups' counts and partial sums loaded together (a
    // partial of a center the workgroup did not see is stale and not added),
    // then added in workgroup order
    double S = 0.0;
    int n = 0;
    for (int b0 = 0; b0 < nblk; b0 += kUpdBatch) {
        int c[kUpdBatch];
        double v[kUpdBatch];
#pragma unroll
        for (int q = 0; q < kUpdBatch; ++q) {
            const size_t blk = static_cast<size_t>(bh) * nblk + min(b0 + q, nblk - 1);
            c[q] = b0 + q < nblk ? bcnt[blk * M + u] : 0;
            v[q] = bpart[(blk * M + u) * D + k];
        }
#pragma unroll
        for (int q = 0; q < kUpdBatch; ++q) {
            if (c[q]) {
                S = S + v[q];
                n += c[q];
            }
        }
    }
    if (n == 0) return;  // uniform over the workgroup
    const double wu = w[static_cast<size_t>(bh) * M + u];
    double* m = cent + (static_cast<size_t>(bh) * M + u) * D + k;
    *m = (*m * wu + S) / (wu + static_cast<double>(n));
    __syncthreads();  // every thread has read w before it changes
    if (k == 0) w[static_cast<size_t>(bh) * M + u] = wu + static_cast<double>(n);
}

// One workgroup per pair: wave 0 adds the batch inertia, wave 1 marks the
// starved centers, each 64 at a time from one load (scanned by one thread, in
// batches of eight loads, the two took 6.7 us together at 32 centers and 64
// partials; now 4.0).
template <typename T, int D>
__global__ __launch_bounds__(256) void k_km_control(
    const T* __restrict__ K, int N, int M, int batch, int step, uint64_t seed, int nblk, double alpha,
    double ratio, int max_no_improvement, const double* __restrict__ binert, double* __restrict__ cent,
    double* __restrict__ w, KmState* __restrict__ state) {
#pragma clang fp contract(off)
    __shared__ int s_mark[kKmMaxCenters];
    __shared__ int s_count;
    __shared__ double s_wkeep;
    const int bh = blockIdx.x, tid = threadIdx.x, lane = lane_id();
    KmState* st = state + bh;
    KmState next = *st;
    double* wb = w + static_cast<size_t>(bh) * M;
    const double* bi = binert + static_cast<size_t>(bh) * nblk;
    const double first = wave_id() == 0 ? bi[min(lane, nblk - 1)] : wave_id() == 1 ? wb[min(lane, M - 1)] : 0.0;
    if (next.stop) return;
    if (wave_id() == 0) {
        // the workgroups' sums in order
        double I = 0.0;
        for (int b0 = 0; b0 < nblk; b0 += kWave) {
            const double v = b0 == 0 ? first : bi[min(b0 + lane, nblk - 1)];
            const int n = min(kWave, nblk - b0);
#pragma unroll 8
            for (int q = 0; q < n; ++q)
                I = I + __longlong_as_double(static_cast<long long>(readlane(static_cast<uint64_t>(__double_as_longlong(v)), q)));
        }
        I = I / static_cast<double>(batch);
        next.ewa = step == 0 ? I : next.ewa * (1.0 - alpha) + I * alpha;
        if (next.ewa < next.ewa_min) {
            next.ewa_min = next.ewa;
            next.no_imp = 0;
        } else {
            next.no_imp += 1;
        }
        next.steps = step + 1;
        if (max_no_improvement > 0 && next.no_imp >= max_no_improvement) next.stop = 1;
    } else if (wave_id() == 1) {
        // centers under ratio x the largest weight, in index order, up to half
        // a batch of them; the smallest weight among the others
        int count = 0;
        double wkeep = INFINITY;
        if (ratio > 0.0) {
            double wmax = first;
            for (int u0 = kWave; u0 < M; u0 += kWave) wmax = fmax(wmax, wb[min(u0 + lane, M - 1)]);
            for (int off = kWave / 2; off > 0; off >>= 1) wmax = fmax(wmax, __shfl_xor(wmax, off));
            const double thr = ratio * wmax;
            for (int u0 = 0; u0 < M; u0 += kWave) {
                const int u = u0 + lane;
                const double v = u0 == 0 ? first : wb[min(u, M - 1)];
                const uint64_t low = __ballot(u < M && v < thr);
                const int at = count + static_cast<int>(__popcll(low & lanemask_lt()));
                const bool marked = u < M && v < thr && at < batch / 2;
                if (marked) s_mark[at] = u;
                if (u < M && !marked && v < wkeep) wkeep = v;
                count = min(count + static_cast<int>(__popcll(low)), batch / 2);
            }
            for (int off = kWave / 2; off > 0; off >>= 1) wkeep = fmin(wkeep, __shfl_xor(wkeep, off));
        }
        if (lane == 0) {
            s_count = count;
            s_wkeep = wkeep;
        }
    }
    __syncthreads();
    if (tid == 0) *st = next;  // every wave has read the old one
    const int count = s_count;
    const T* X = K + static_cast<size_t>(bh) * N * D;
    for (int r = 0; r < count; ++r) {
        const int u = s_mark[r];
        const int j = draw_index(km_word(seed, static_cast<uint64_t>(r), 4, static_cast<uint64_t>(step)), batch);
        const int tok = draw_index(km_word(seed, static_cast<uint64_t>(j), 3, static_cast<uint64_t>(step)), N);
        for (int k = tid; k < D; k += 256)
            cent[(static_cast<size_t>(bh) * M + u) * D + k] = static_cast<double>(load_elem(X + static_cast<size_t>(tok) * D, k));
        if (tid == 0) wb[u] = s_wkeep;
    }
}

__global__ __launch_bounds__(256) void k_km_init_state(KmState* __restrict__ state, double* __restrict__ w,
                                                       int BH, int M) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < BH) {
        KmState s;
        s.ewa = 0.0;
        s.ewa_min = INFINITY;
        s.no_imp = 0;
        s.stop = 0;
        s.steps = 0;
        s.pad = 0;
        state[i] = s;
    }
    if (i < BH * M) w[i] = 0.0;
}

// Parents of one (sequence, KV head) from its labels: wave w counts and then
// places the tokens of its own contiguous segment, so members of a parent
// land in token order.  Outputs: members [N] (parent by parent), pbeg
// [Mp + 1] (first member position of each parent), toff [Mp + 1] (first team
// of each parent: sum of min(R, |C|) over the parents before it), and the
// pair's team count.  A label outside [0, Mp) sets *bad and is skipped.
// Labels are read eight groups of 64 ahead, and a group's tokens find those of
// their own label by one ballot per label bit (a ballot and an LDS round trip
// per distinct label of a group took 167 us at 32K tokens and 32 parents; now
// 27).
__global__ __launch_bounds__(kListThreads) void k_parent_lists(
    const int* __restrict__ labels, int N, int Mp, int R, int* __restrict__ members,
    int* __restrict__ pbeg, int* __restrict__ toff, int* __restrict__ team_count, int* __restrict__ bad) {
    __shared__ int s_off[kListWaves][kMaxLabels];
    __shared__ int s_wt[2][kListWaves];
    __shared__ int s_carry[2];
    const int bh = blockIdx.x, tid = threadIdx.x, w = wave_id(), lane = lane_id();
    const int* lab = labels + static_cast<size_t>(bh) * N;
    int* mem = members + static_cast<size_t>(bh) * N;
    for (int e = tid; e < kListWaves * Mp; e += kListThreads) s_off[e / Mp][e % Mp] = 0;
    if (tid < 2) s_carry[tid] = 0;
    __syncthreads();
    const int seg = (N + kListWaves - 1) / kListWaves;
    const int i0 = min(N, w * seg), i1 = min(N, i0 + seg);
    for (int g0 = i0; g0 < i1; g0 += kListAhead * kWave) {
        int Ls[kListAhead];
#pragma unroll
        for (int q = 0; q < kListAhead; ++q) Ls[q] = lab[min(g0 + q * kWave + lane, i1 - 1)];
#pragma unroll
        for (int q = 0; q < kListAhead; ++q) {
            if (g0 + q * kWave + lane < i1) {
                if (Ls[q] < 0 || Ls[q] >= Mp)
                    atomicOr(bad, 1);
                else
                    atomicAdd(&s_off[w][Ls[q]], 1);
            }
        }
    }
    __syncthreads();
    // parent sizes and team counts, scanned over labels in chunks
    for (int base = 0; base < Mp; base += kListThreads) {
        const int u = base + tid;
        int cnt[kListWaves];
        int tot = 0;
#pragma unroll
        for (int v = 0; v < kListWaves; ++v) {
            cnt[v] = u < Mp ? s_off[v][u] : 0;
            tot += cnt[v];
        }
        const int x[2] = {tot, min(R, tot)};
        int ex[2];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int inc = wave_incl_scan(x[q]);
            if (lane == kWave - 1) s_wt[q][w] = inc;
            ex[q] = inc - x[q];
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            int pre = s_carry[q];
            for (int v = 0; v < w; ++v) pre += s_wt[q][v];
            ex[q] += pre;
        }
        if (u < Mp) {
            pbeg[static_cast<size_t>(bh) * (Mp + 1) + u] = ex[0];
            toff[static_cast<size_t>(bh) * (Mp + 1) + u] = ex[1];
            int run = ex[0];
#pragma unroll
            for (int v = 0; v < kListWaves; ++v) {
                s_off[v][u] = run;
                run += cnt[v];
            }
        }
        __syncthreads();
        if (tid < 2) {
            int add = 0;
            for (int v = 0; v < kListWaves; ++v) add += s_wt[tid][v];
            s_carry[tid] += add;
        }
        __syncthreads();
    }
    if (tid == 0) {
        pbeg[static_cast<size_t>(bh) * (Mp + 1) + Mp] = s_carry[0];
        toff[static_cast<size_t>(bh) * (Mp + 1) + Mp] = s_carry[1];
        team_count[bh] = s_carry[1];
    }
    // placement, a 64-token group at a time
    const uint64_t lt = lanemask_lt();
    const int bits = 32 - __clz(Mp);
    for (int g0 = i0; g0 < i1; g0 += kListAhead * kWave) {
        int Ls[kListAhead];
#pragma unroll
        for (int q = 0; q < kListAhead; ++q) Ls[q] = lab[min(g0 + q * kWave + lane, i1 - 1)];
#pragma unroll
        for (int q = 0; q < kListAhead; ++q) {
            const int i = g0 + q * kWave + lane, L = Ls[q];
            const bool ok = i < i1 && L >= 0 && L < Mp;
            uint64_t same = __ballot(ok);
            for (int b = 0; b < bits; ++b) {  // uniform
                const uint64_t set = __ballot((L >> b) & 1);
                same &= (L >> b) & 1 ? set : ~set;
            }
            const int base = ok ? s_off[w][L] : 0;
            wave_lds_sync();
            if (ok) {
                mem[base + __popcll(same & lt)] = i;
                if ((same & lt) == 0) s_off[w][L] = base + static_cast<int>(__popcll(same));
            }
            wave_lds_sync();
        }
    }
}

// Absent teams past each pair's team count: no rows, log n = kAbsentLogN.
__global__ __launch_bounds__(256) void k_pad_teams(const int* __restrict__ team_count, int M, int N,
                                                   int BH, int* __restrict__ team_begin,
                                                   int* __restrict__ team_size, double* __restrict__ log_n,
                                                   int* __restrict__ rep_token) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= BH * M) return;
    const int bh = i / M, g = i % M;
    if (g < team_count[bh]) return;
    team_begin[i] = N;
    team_size[i] = 0;
    log_n[i] = kAbsentLogN;
    rep_token[i] = 0;
}

}  // namespace

KmLayout kmeans_layout(int BH, int N, int d, int M, int batch, int s0) {
    KmLayout L{};
    L.M = M;
    L.s0 = s0;
    L.L = 2 + static_cast<int>(floor(log(static_cast<double>(M))));
    L.nkpp = (s0 + kKppThreads - 1) / kKppThreads;
    L.nasg = (batch + kAsgPts - 1) / kAsgPts;
    size_t off = 0;
    auto take = [&](size_t bytes) {
        const size_t o = off;
        off += (bytes + 255) / 256 * 256;
        return o;
    };
    L.samp = take(sizeof(int) * static_cast<size_t>(s0));
    L.cand = take(sizeof(int) * static_cast<size_t>(BH) * L.L);
    L.D2 = take(sizeof(double) * static_cast<size_t>(BH) * s0);
    L.Dt = take(sizeof(double) * static_cast<size_t>(BH) * L.L * s0);
    L.part = take(sizeof(double) * static_cast<size_t>(BH) * L.nkpp * L.L);
    L.cent = take(sizeof(double) * static_cast<size_t>(BH) * M * d);
    L.w = take(sizeof(double) * static_cast<size_t>(BH) * M);
    L.state = take(sizeof(KmState) * static_cast<size_t>(BH));
    L.bpart = take(sizeof(double) * static_cast<size_t>(BH) * L.nasg * M * d);
    L.bcnt = take(sizeof(int) * static_cast<size_t>(BH) * L.nasg * M);
    L.binert = take(sizeof(double) * static_cast<size_t>(BH) * L.nasg);
    L.total = off;
    return L;
}

hipError_t launch_kmeans_seed(const void* K, santapp_dtype dtype, int BH, int N, int d,
                              const KmLayout& L, char* ws, uint64_t seed, hipStream_t s) {
    int* samp = reinterpret_cast<int*>(ws + L.samp);
    int* cand = reinterpret_cast<int*>(ws + L.cand);
    double* D2 = reinterpret_cast<double*>(ws + L.D2);
    double* Dt = reinterpret_cast<double*>(ws + L.Dt);
    double* part = reinterpret_cast<double*>(ws + L.part);
    double* cent = reinterpret_cast<double*>(ws + L.cent);
    k_kpp_sample<<<L.nkpp, kKppThreads, 0, s>>>(samp, L.s0, N, cand, L.L, BH, seed);
    for (int c = 0; c < L.M; ++c) {
#define SANTAPP_KPP(TT, DD)                                                                       \
    do {                                                                                         \
        k_kpp_dist<TT, DD><<<dim3(L.nkpp, BH), kKppThreads, 0, s>>>(                             \
            static_cast<const TT*>(K), N, samp, L.s0, cand, L.L, c, D2, Dt, part);              \
        k_kpp_pick<TT, DD><<<BH, kPickThreads, 0, s>>>(static_cast<const TT*>(K), N, samp, L.s0, \
                                                       cand, L.L, c, L.M, L.nkpp, D2, Dt, part,  \
                                                       cent, seed);                              \
    } while (0)
        if (dtype == SANTAPP_BF16 && d == 128) SANTAPP_KPP(bf16_t, 128);
        else if (dtype == SANTAPP_BF16) SANTAPP_KPP(bf16_t, 64);
        else if (d == 128) SANTAPP_KPP(float, 128);
        else SANTAPP_KPP(float, 64);
#undef SANTAPP_KPP
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    k_km_init_state<<<(BH * L.M + 255) / 256, 256, 0, s>>>(reinterpret_cast<KmState*>(ws + L.state),
                                                           reinterpret_cast<double*>(ws + L.w), BH, L.M);
    return hipGetLastError();
}

hipError_t launch_kmeans_steps(const void* K, santapp_dtype dtype, int BH, int N, int d,
                               const KmLayout& L, char* ws, int batch, int first, int count,
                               double alpha, double ratio, int max_no_improvement, uint64_t seed,
                               hipStream_t s) {
    double* cent = reinterpret_cast<double*>(ws + L.cent);
    double* w = reinterpret_cast<double*>(ws + L.w);
    KmState* st = reinterpret_cast<KmState*>(ws + L.state);
    double* bpart = reinterpret_cast<double*>(ws + L.bpart);
    int* bcnt = reinterpret_cast<int*>(ws + L.bcnt);
    double* binert = reinterpret_cast<double*>(ws + L.binert);
    for (int step = first; step < first + count; ++step) {
#define SANTAPP_STEP(TT, DD)                                                                          \
    do {                                                                                             \
        k_km_assign<TT, DD, false><<<dim3(L.nasg, BH), kAsgThreads, 0, s>>>(                        \
            static_cast<const TT*>(K), N, L.M, batch, step, seed, cent, st, nullptr, bpart, bcnt,  \
            binert);                                                                                 \
        k_km_update<DD><<<dim3(L.M, BH), DD, 0, s>>>(L.M, L.nasg, bpart, bcnt, cent, w, st);        \
        k_km_control<TT, DD><<<BH, 256, 0, s>>>(static_cast<const TT*>(K), N, L.M, batch, step,     \
                                                seed, L.nasg, alpha, ratio, max_no_improvement,     \
                                                binert, cent, w, st);                               \
    } while (0)
        if (dtype == SANTAPP_BF16 && d == 128) SANTAPP_STEP(bf16_t, 128);
        else if (dtype == SANTAPP_BF16) SANTAPP_STEP(bf16_t, 64);
        else if (d == 128) SANTAPP_STEP(float, 128);
        else SANTAPP_STEP(float, 64);
#undef SANTAPP_STEP
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_kmeans_labels(const void* K, santapp_dtype dtype, int BH, int N, int d,
                                const KmLayout& L, char* ws, int* labels, hipStream_t s) {
    const double* cent = reinterpret_cast<const double*>(ws + L.cent);
    const dim3 grid((N + kAsgPts - 1) / kAsgPts, BH);
#define SANTAPP_LAB(TT, DD)                                                                            \
    k_km_assign<TT, DD, true><<<grid, kAsgThreads, 0, s>>>(static_cast<const TT*>(K), N, L.M, 0, 0, 0, \
                                                           cent, nullptr, labels, nullptr, nullptr,   \
                                                           nullptr)
    if (dtype == SANTAPP_BF16 && d == 128) SANTAPP_LAB(bf16_t, 128);
    else if (dtype == SANTAPP_BF16) SANTAPP_LAB(bf16_t, 64);
    else if (d == 128) SANTAPP_LAB(float, 128);
    else SANTAPP_LAB(float, 64);
#undef SANTAPP_LAB
    return hipGetLastError();
}

hipError_t launch_parent_lists(const int* labels, int BH, int N, int Mp, int R, int* members, int* pbeg,
                               int* toff, int* team_count, int* bad, hipStream_t s) {
    k_parent_lists<<<BH, kListThreads, 0, s>>>(labels, N, Mp, R, members, pbeg, toff, team_count, bad);
    return hipGetLastError();
}

hipError_t launch_pad_teams(const int* team_count, int BH, int M, int N, int* team_begin, int* team_size,
                            double* log_n, int* rep_token, hipStream_t s) {
    const int total = BH * M;
    k_pad_teams<<<(total + 255) / 256, 256, 0, s>>>(team_count, M, N, BH, team_begin, team_size, log_n,
                                                    rep_token);
    return hipGetLastError();
}

}  // namespace santapp
