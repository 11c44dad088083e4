// Routing-key variants and the KL routing diagnostic (section
// "Attention-distribution diagnostic"; appendix "Dense-trajectory KL and
// task-variant evaluation", eq. diagnostic-kl).
//
// k_team_centroid   the team mean as routing key (centroid-guided sampling)
// k_team_repkey     the representative's key again (the table's default)
// k_kl_rows         per (query head, 256 packed rows): max, sum of e^(s - max),
//                   of e^(s - max) s and of e^(s - max) r, fp64 (s the row's
//                   score, r its team's routing score)
// k_kl_merge        per query head: KL(p || q) from those sums and the
//                   routing logits phi
#include "common.h"
#include "internal.h"

namespace santapp {

namespace {

// fp64 -> bf16, round to nearest with ties to even: round to fp32 with
// round-to-odd (toward zero, then the last bit set when inexact), then to
// bf16 to nearest even.  fp32 keeps 16 more significand bits than bf16, so
// the two steps round correctly (no double-rounding error).
__device__ __forceinline__ uint16_t f64_to_bf16(double x) {
    if (x != x) return 0x7fc0;
    const float f = static_cast<float>(x);
    uint32_t u = __float_as_uint(f);
    if (static_cast<double>(f) != x) {
        if (fabs(static_cast<double>(f)) > fabs(x)) u -= 1u;  // one step toward zero
        u |= 1u;
    }
    u += 0x7fffu + ((u >> 16) & 1u);
    return static_cast<uint16_t>(u >> 16);
}

__device__ __forceinline__ void store_mean(bf16_t* p, double v) { p->bits = f64_to_bf16(v); }
__device__ __forceinline__ void store_mean(float* p, double v) { *p = static_cast<float>(v); }

// U rows' values of dimension j of a team's rows from row i on, all in flight,
// then added in order (cnt of them; a sum from 0.0 is never -0.0, so adding 0.0
// changes nothing).
template <int U, bool FULL, typename T, int D>
__device__ __forceinline__ double add_rows(double s, const T* __restrict__ col, int i, int cnt) {
    float v[U];
#pragma unroll
    for (int k = 0; k < U; ++k) v[k] = load_elem(col, static_cast<size_t>(i + (FULL ? k : min(k, cnt - 1))) * D);
#pragma unroll
    for (int k = 0; k < U; ++k) s = s + (FULL || k < cnt ? static_cast<double>(v[k]) : 0.0);
    return s;
}

// Team means: thread j sums dimension j over the team's rows in packed
// order (ascending token index), then divides by n_g.  The order of the sum
// is the definition's, so a team is one serial chain, and the largest team
// bounds the launch: its rows are requested 32 at a time, the last ones in the
// smallest block that holds them.  One call at 32K tokens, d = 128: P = 1024, R =
// 16 (largest team 700 rows) bf16 33 us, fp32 48; bf16 P = 16, R = 4 18.5; 30000
// tokens of fp32 d = 64 in teams of two 15.8.  Eight rows at a time took 48, 51,
// 21.4 and 16.1; 64 at a time through LDS was slower the smaller the teams (36.5
// and 61 for the last two).
template <typename T, int D>
__global__ __launch_bounds__(D) void k_team_centroid(const T* __restrict__ packed_K,
                                                      const int* __restrict__ team_begin,
                                                      const int* __restrict__ team_size, int N, int M,
                                                      T* __restrict__ reps) {
#pragma clang fp contract(off)
    const int g = blockIdx.x, bh = blockIdx.y, j = threadIdx.x;
    const size_t t = static_cast<size_t>(bh) * M + g;
    const int begin = team_begin[t], n = team_size[t];
    if (n <= 0) {  // an absent team keeps a zero key; its log n excludes it
        store_mean(reps + t * D + j, 0.0);
        return;
    }
    const T* const col = packed_K + (static_cast<size_t>(bh) * N + begin) * D + j;
    double s = 0.0;
    int i = 0;
    for (; n - i >= 32; i += 32) s = add_rows<32, true, T, D>(s, col, i, 32);
    if (n - i > 16)
        s = add_rows<32, false, T, D>(s, col, i, n - i);
    else if (n - i > 8)
        s = add_rows<16, false, T, D>(s, col, i, n - i);
    else if (n - i > 4)
        s = add_rows<8, false, T, D>(s, col, i, n - i);
    else if (n - i > 2)
        s = add_rows<4, false, T, D>(s, col, i, n - i);
    else if (n - i > 0)
        s = add_rows<2, false, T, D>(s, col, i, n - i);
    store_mean(reps + t * D + j, s / static_cast<double>(n));
}

// The representative's key: its packed row is found among the team's rows
// (perm maps packed rows to tokens) and copied.
template <typename T, int D>
__global__ __launch_bounds__(kWave) void k_team_repkey(const T* __restrict__ packed_K,
                                                       const int* __restrict__ team_begin,
                                                       const int* __restrict__ team_size,
                                                       const int* __restrict__ rep_token,
                                                       const int* __restrict__ perm, int N, int M,
                                                       T* __restrict__ reps) {
    const int g = blockIdx.x, bh = blockIdx.y, lane = lane_id();
    const size_t t = static_cast<size_t>(bh) * M + g;
    const int begin = team_begin[t], n = team_size[t], tok = rep_token[t];
    const int* pm = perm + static_cast<size_t>(bh) * N + begin;
    int found = -1;
    for (int base = 0; base < n && found < 0; base += kWave) {  // uniform
        const int i = base + lane;
        const uint64_t hit = __ballot(i < n && pm[i] == tok);
        if (hit) found = base + __ffsll(static_cast<unsigned long long>(hit)) - 1;
    }
    if (found < 0) return;  // a table's representative is always a member of its team
    constexpr int kChunks = D * static_cast<int>(sizeof(T)) / 16;
    const uint4* src = reinterpret_cast<const uint4*>(packed_K + (static_cast<size_t>(bh) * N + begin + found) * D);
    uint4* dst = reinterpret_cast<uint4*>(reps + t * D);
    for (int c = lane; c < kChunks; c += kWave) dst[c] = src[c];
}

struct KlPart {
    double m;  // max score of the rows
    double z;  // sum of e^(s - m)
    double s;  // sum of e^(s - m) s
    double r;  // sum of e^(s - m) r
};

constexpr int kKlThreads = 256;
constexpr int kKlWaves = kKlThreads / kWave;

// The last team whose first row is at or before `row` (team_begin ascends and
// starts at 0): the wave samples 64 teams of the range left at a time.
__device__ __forceinline__ int team_of_row(const int* __restrict__ begin, int M, int row) {
    int lo = 0, hi = M;
    while (hi - lo > 1) {  // uniform
        const int step = (hi - lo + kWave - 1) / kWave;
        const int i = lo + lane_id() * step;
        const uint64_t at = __ballot(i < hi && begin[min(i, M - 1)] <= row);
        lo += (static_cast<int>(__popcll(at)) - 1) * step;
        hi = min(hi, lo + step);
        if (step == 1) break;
    }
    return lo;
}

// A wave takes 64 packed rows, whatever teams they belong to (a wave per team
// waited for the largest team: 160 us at the 32K prompt, whose largest has
// 700 rows; 21 us now).  The scores of 16 rows and the G <= 8 heads
// are one 16 x 16 tile of v_mfma_f64_16x16x4_f64 (A: head i on lanes 16 c + i,
// B: row j on lanes 16 c + j, each lane group c holding dims [c D / 4,
// (c + 1) D / 4)); register q of the result is head 4 q + c of row j, so
// registers 0 and 1 hold every head.  All rows are requested before the teams
// are looked up.
template <typename T, int D, int G>
__global__ __launch_bounds__(kKlThreads) void k_kl_rows(const T* __restrict__ packed_K,
                                                        const int* __restrict__ team_begin,
                                                        const double* __restrict__ log_n,
                                                        const float* __restrict__ q,
                                                        const double* __restrict__ phi, int N, int M, int Hkv,
                                                        int Hq, double scale, KlPart* __restrict__ part) {
    using Q = Quarter<T, D>;
    typedef double f64x4 __attribute__((ext_vector_type(4)));
    __shared__ int s_team[kKlWaves][kWave];
    __shared__ KlPart s_part[kKlWaves][8];
    const int bh = blockIdx.y, lane = lane_id(), w = wave_id();
    const int b = bh / Hkv, kv = bh - b * Hkv;
    const int c = lane >> 4, j = lane & 15;
    const int row0 = blockIdx.x * kKlThreads + w * kWave;
    const T* const Kp = packed_K + static_cast<size_t>(bh) * N * D + c * Q::E;
    Q rows[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) rows[t].load(Kp + static_cast<size_t>(min(row0 + 16 * t + j, N - 1)) * D);
    float qv[Q::E];
    {
        const float* const qh = q + (static_cast<size_t>(b) * Hq + kv * G + min(j, G - 1)) * D + c * Q::E;
#pragma unroll
        for (int e = 0; e < Q::E; e += 4) {
            const float4 x = *reinterpret_cast<const float4*>(qh + e);
            qv[e] = x.x;
            qv[e + 1] = x.y;
            qv[e + 2] = x.z;
            qv[e + 3] = x.w;
        }
    }

    // the team of each of the wave's rows: marked at the teams' first rows,
    // then a running maximum
    const int* const begin = team_begin + static_cast<size_t>(bh) * M;
    const int last = min(row0 + kWave, N) - 1;
    int team = 0;
    if (row0 < N) {  // uniform
        const int g0 = team_of_row(begin, M, row0);
        s_team[w][lane] = g0;
        wave_lds_sync();
        for (int g = g0 + 1 + lane;; g += kWave) {
            const int first = g < M ? begin[g] : N;
            if (first <= last) atomicMax(&s_team[w][first - row0], g);
            if (__ballot(first <= last) != ~0ull) break;
        }
        wave_lds_sync();
        team = s_team[w][lane];
#pragma unroll
        for (int off = 1; off < kWave; off <<= 1) {
            const int o = __shfl_up(team, off);
            if (lane >= off) team = max(team, o);
        }
    }
    const double* const ln = log_n + static_cast<size_t>(bh) * M;
    const size_t hq0 = static_cast<size_t>(b) * Hq + kv * G;
    double rr[4][2];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const int g = __shfl(team, 16 * t + j);
        const double l = ln[g];
#pragma unroll
        for (int k = 0; k < 2; ++k) rr[t][k] = phi[(hq0 + min(4 * k + c, G - 1)) * M + g] - l;
    }

    double sc[4][2];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        f64x4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int e = 0; e < Q::E; ++e)
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(static_cast<double>(qv[e]), static_cast<double>(rows[t].elem(e)),
                                                       acc, 0, 0, 0);
        sc[t][0] = scale * acc[0];
        sc[t][1] = scale * acc[1];
    }
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        double m = -INFINITY;
#pragma unroll
        for (int t = 0; t < 4; ++t)
            if (row0 + 16 * t + j < N) m = fmax(m, sc[t][k]);
        m = fmax(m, dpp_f64<0x128>(m));
        m = fmax(m, dpp_f64<0x124>(m));
        m = fmax(m, dpp_f64<0x122>(m));
        m = fmax(m, dpp_f64<0x121>(m));
        double z = 0.0, s = 0.0, r = 0.0;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            if (row0 + 16 * t + j < N) {
                const double e = exp(sc[t][k] - m);
                z += e;
                s = fma(e, sc[t][k], s);
                r = fma(e, rr[t][k], r);
            }
        }
        z = row16_sum(z);
        s = row16_sum(s);
        r = row16_sum(r);
        if (j == 0) s_part[w][4 * k + c] = KlPart{m, z, s, r};
    }
    __syncthreads();
    const int h = threadIdx.x;
    if (h < G) {
        KlPart p{-INFINITY, 0.0, 0.0, 0.0};
        for (int v = 0; v < kKlWaves; ++v) p.m = fmax(p.m, s_part[v][h].m);
        for (int v = 0; v < kKlWaves; ++v) {
            const KlPart x = s_part[v][h];
            if (x.z == 0.0) continue;  // a wave past the last row
            const double f = exp(x.m - p.m);
            p.z += x.z * f;
            p.s += x.s * f;
            p.r += x.r * f;
        }
        part[(hq0 + h) * gridDim.x + blockIdx.x] = p;
    }
}

template <bool kMax>
__device__ double kl_block_reduce(double v, double* s_red) {
    for (int off = kWave / 2; off > 0; off >>= 1) {
        const double o = __shfl_xor(v, off);
        v = kMax ? fmax(v, o) : v + o;
    }
    if (lane_id() == 0) s_red[wave_id()] = v;
    __syncthreads();
    double r = s_red[0];
    for (int w = 1; w < kKlThreads / kWave; ++w) r = kMax ? fmax(r, s_red[w]) : r + s_red[w];
    __syncthreads();
    return r;
}

// KL(p || q) = E_p[s] - E_p[r] - LSE(s) + LSE(phi), with r_g = phi_g - log n_g
// the routing score of team g (log q_i = r_g(i) - LSE(phi)).
__global__ __launch_bounds__(kKlThreads) void k_kl_merge(const double* __restrict__ phi,
                                                         const KlPart* __restrict__ part, int M,
                                                         int chunks, double* __restrict__ kl) {
    __shared__ double s_red[kKlThreads / kWave];
    const int bhq = blockIdx.x, tid = threadIdx.x;
    const double* ph = phi + static_cast<size_t>(bhq) * M;
    const KlPart* pt = part + static_cast<size_t>(bhq) * chunks;
    double pmax = -INFINITY, mmax = -INFINITY;
    for (int g = tid; g < M; g += kKlThreads) pmax = fmax(pmax, ph[g]);
    for (int i = tid; i < chunks; i += kKlThreads) mmax = fmax(mmax, pt[i].m);
    pmax = kl_block_reduce<true>(pmax, s_red);
    mmax = kl_block_reduce<true>(mmax, s_red);
    double ep = 0.0, Z = 0.0, S = 0.0, Rr = 0.0;
    for (int g = tid; g < M; g += kKlThreads) ep += exp(ph[g] - pmax);
    for (int i = tid; i < chunks; i += kKlThreads) {
        const KlPart x = pt[i];
        const double c = exp(x.m - mmax);
        Z += x.z * c;
        S += x.s * c;
        Rr += x.r * c;
    }
    ep = kl_block_reduce<false>(ep, s_red);
    Z = kl_block_reduce<false>(Z, s_red);
    S = kl_block_reduce<false>(S, s_red);
    Rr = kl_block_reduce<false>(Rr, s_red);
    if (tid == 0) kl[bhq] = (S - Rr) / Z - (mmax + log(Z)) + (pmax + log(ep));
}

template <typename T, int D>
hipError_t route_keys_d(const void* packed_K, const int* team_begin, const int* team_size,
                        const int* rep_token, const int* perm, int BH, int N, int M, bool centroid,
                        void* reps, hipStream_t s) {
    const dim3 grid(M, BH);
    if (centroid)
        k_team_centroid<T, D><<<grid, D, 0, s>>>(static_cast<const T*>(packed_K), team_begin, team_size, N, M,
                                                 static_cast<T*>(reps));
    else
        k_team_repkey<T, D><<<grid, kWave, 0, s>>>(static_cast<const T*>(packed_K), team_begin, team_size,
                                                   rep_token, perm, N, M, static_cast<T*>(reps));
    return hipGetLastError();
}

template <typename T, int D>
hipError_t kl_d(const KlArgs& a, hipStream_t s) {
    KlPart* part = static_cast<KlPart*>(a.part);
    const dim3 grid(kl_chunks(a.N), a.B * a.Hkv);
#define SANTAPP_KL(GG)                                                                                  \
    case GG:                                                                                            \
        k_kl_rows<T, D, GG><<<grid, kKlThreads, 0, s>>>(static_cast<const T*>(a.packed_K), a.team_begin, \
                                                        a.log_n, a.q, a.phi, a.N, a.M, a.Hkv, a.Hq,     \
                                                        a.scale, part);                                 \
        break
    switch (a.Hq / a.Hkv) {
        SANTAPP_KL(1); SANTAPP_KL(2); SANTAPP_KL(3); SANTAPP_KL(4);
        SANTAPP_KL(5); SANTAPP_KL(6); SANTAPP_KL(7); SANTAPP_KL(8);
        default: return hipErrorInvalidValue;
    }
#undef SANTAPP_KL
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    k_kl_merge<<<a.B * a.Hq, kKlThreads, 0, s>>>(a.phi, part, a.M, kl_chunks(a.N), a.kl);
    return hipGetLastError();
}

}  // namespace

size_t kl_part_bytes() { return sizeof(KlPart); }

int kl_chunks(int N) { return (N + kKlThreads - 1) / kKlThreads; }

hipError_t launch_route_keys(const void* packed_K, const int* team_begin, const int* team_size,
                             const int* rep_token, const int* perm, int BH, int N, int M, int d,
                             santapp_dtype dtype, bool centroid, void* reps, hipStream_t s) {
    if (dtype == SANTAPP_BF16) {
        if (d == 128) return route_keys_d<bf16_t, 128>(packed_K, team_begin, team_size, rep_token, perm, BH, N, M, centroid, reps, s);
        if (d == 64) return route_keys_d<bf16_t, 64>(packed_K, team_begin, team_size, rep_token, perm, BH, N, M, centroid, reps, s);
    } else {
        if (d == 128) return route_keys_d<float, 128>(packed_K, team_begin, team_size, rep_token, perm, BH, N, M, centroid, reps, s);
        if (d == 64) return route_keys_d<float, 64>(packed_K, team_begin, team_size, rep_token, perm, BH, N, M, centroid, reps, s);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_routing_kl(const KlArgs& a, hipStream_t s) {
    if (a.dtype == SANTAPP_BF16) {
        if (a.d == 128) return kl_d<bf16_t, 128>(a, s);
        if (a.d == 64) return kl_d<bf16_t, 64>(a, s);
    } else {
        if (a.d == 128) return kl_d<float, 128>(a, s);
        if (a.d == 64) return kl_d<float, 64>(a, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace santapp
