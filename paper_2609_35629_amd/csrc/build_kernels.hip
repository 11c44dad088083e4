// Team construction and packing (section "Preparing parent groups and teams";
// Alg. "Contiguous parent partition", Alg. "Build actual-key teams from a
// parent partition"; packed team-contiguous copy of the prompt K/V as in the
// appendix "Triton decode kernels").
//
// One workgroup builds one parent of one (sequence, KV head).  The
// farthest-first rounds and the nearest-representative assignment share one
// running minimum per member: after round u, m[i] = min_{v<=u} |k_i-k_{j_v}|^2
// and the owner of i is the first v attaining it, which is exactly the
// assignment rule (ties to the earliest-chosen representative) once all r
// rounds ran.
//
// The definition's distance is an fp64 sum over dimensions in index order
// with no fused multiply-add, and every choice (nearest the mean, farthest,
// owner) is the definition's bit for bit.  Few choices need that arithmetic:
// the rounds run on an fp32 estimate |k|^2 + |c|^2 - 2 k.c whose error is
// bounded, and only members whose estimates lie within twice the bound of the
// best one are compared by the definition's distance.
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "internal.h"

namespace santapp {

namespace {

constexpr int kBuildThreads = 1024;  // most threads of a build workgroup
constexpr int kBuildWaves = kBuildThreads / kWave;
constexpr int kTie = 64;             // members one exact comparison takes
constexpr int kRankBlock = kWave;    // representatives ranked per ballot block
constexpr float kInf = __builtin_inff();

// Bound on |estimate - the definition's distance| over a parent whose largest
// squared norm is nmax.  An inner product rounds at most twelve times on any
// path (a lane's chain: eight fused multiply-adds, or four dot products of two
// exact bf16 products with two roundings each; then four additions over the
// lanes), each time by at most 2^-23 of sum |x_i c_i| <= nmax.  |x|^2, |c|^2 and
// twice x.c are off by 48 x 2^-23 nmax, their combination rounds by 6 x 2^-23
// nmax more, and the rounding of the mean to fp32 adds 3: below 64 x 2^-23 nmax
// with what products below fp32's normal range can lose (kNormMin).
constexpr float kEstimate = 64.f * 0x1.0p-23f;
// Parents whose largest squared norm lies outside this range (fp32 products
// could overflow or vanish, or a key is not finite) are built by the
// definition's arithmetic throughout.
constexpr float kNormMin = 1e-28f, kNormMax = 1e30f;

// A tie within estimates wider than this share of the farthest distance takes
// the parent to the definition's arithmetic: at 32K tokens (bf16, d = 128, P =
// 1024, R = 16) keys with four channels at 300 times the others' spread (share
// 0.014) take 179 us compared member by member, 276 by the definition; all
// channels at 100 times it (0.05) take 404 us so, 228 by the definition.
constexpr float kWide = 1.f / 32.f;

// (value, index) reductions with ties broken toward the lower index.
struct ArgVal {
    double v;
    int i;
};

__device__ __forceinline__ ArgVal pick_min(ArgVal a, ArgVal b) {
    return (b.v < a.v || (b.v == a.v && b.i < a.i)) ? b : a;
}

__device__ __forceinline__ ArgVal pick_max(ArgVal a, ArgVal b) {
    return (b.v > a.v || (b.v == a.v && b.i < a.i)) ? b : a;
}

// The best of the wave's lanes (no lane's value is NaN).
template <bool kMax>
__device__ __forceinline__ ArgVal wave_arg(ArgVal x) {
    const double v = kMax ? x.v : -x.v;
    double m = v;
    m = fmax(m, dpp_f64<0x128>(m));
    m = fmax(m, dpp_f64<0x124>(m));
    m = fmax(m, dpp_f64<0x122>(m));
    m = fmax(m, dpp_f64<0x121>(m));
    m = fmax(m, __shfl_xor(m, 16));
    m = fmax(m, __shfl_xor(m, 32));
    const uint64_t at = __ballot(v == m);
    int i;
    if (__popcll(at) == 1) {  // uniform
        i = readlane(x.i, __ffsll(static_cast<unsigned long long>(at)) - 1);
    } else {
        i = v == m ? x.i : 0x7fffffff;
        for (int off = kWave / 2; off > 0; off >>= 1) i = min(i, __shfl_xor(i, off));
    }
    return ArgVal{kMax ? m : -m, i};
}

template <bool kMax>
__device__ ArgVal block_arg(ArgVal x, ArgVal* s_red, int nw) {
    const int lane = lane_id();
    x = wave_arg<kMax>(x);
    if (lane == 0) s_red[wave_id()] = x;
    __syncthreads();
    ArgVal r{kMax ? -INFINITY : INFINITY, 0x7fffffff};
    if (lane < nw) r = s_red[lane];
    r = wave_arg<kMax>(r);
    __syncthreads();
    return r;
}

// |k_i - c|^2 with c held in LDS as fp64, summed in dimension order; the row
// is read 16 bytes at a time (rows are 16-byte aligned, d a multiple of 8).
template <typename T>
__device__ double sqdist_to(const T* __restrict__ row, const double* __restrict__ c, int d) {
#pragma clang fp contract(off)
    double acc = 0.0;
    constexpr int kPer = 16 / static_cast<int>(sizeof(T));
#pragma unroll 4
    for (int j = 0; j < d; j += kPer) {
        const uint4 w = *reinterpret_cast<const uint4*>(row + j);
        float v[kPer];
        if constexpr (sizeof(T) == 2) {
            const uint32_t ws[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                v[2 * q] = bf16lo(ws[q]);
                v[2 * q + 1] = bf16hi(ws[q]);
            }
        } else {
            v[0] = __uint_as_float(w.x);
            v[1] = __uint_as_float(w.y);
            v[2] = __uint_as_float(w.z);
            v[3] = __uint_as_float(w.w);
        }
#pragma unroll
        for (int q = 0; q < kPer; ++q) {
            const double t = static_cast<double>(v[q]) - c[j + q];
            acc = acc + t * t;
        }
    }
    return acc;
}

// s plus `n` values in order, at(i) apart from p, sixteen read ahead of their
// additions.
template <typename T, typename At>
__device__ __forceinline__ double sum_rows(double s, const T* p, int n, At at) {
    int i = 0;
    for (; i + 16 <= n; i += 16) {
        float x[16];
#pragma unroll
        for (int q = 0; q < 16; ++q) x[q] = load_elem(p, at(i + q));
#pragma unroll
        for (int q = 0; q < 16; ++q) s = s + static_cast<double>(x[q]);
    }
    for (; i < n; ++i) s = s + static_cast<double>(load_elem(p, at(i)));
    return s;
}

// |a - c|^2 of two rows in memory.
template <typename T, int D>
__device__ double sqdist_rows(const T* __restrict__ a, const T* __restrict__ c) {
#pragma clang fp contract(off)
    constexpr int kPer = 16 / static_cast<int>(sizeof(T));
    double acc = 0.0;
#pragma unroll 4
    for (int j = 0; j < D; j += kPer) {
        const uint4 x = *reinterpret_cast<const uint4*>(a + j), y = *reinterpret_cast<const uint4*>(c + j);
        const uint32_t xs[4] = {x.x, x.y, x.z, x.w}, ys[4] = {y.x, y.y, y.z, y.w};
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if constexpr (sizeof(T) == 2) {
                const double t0 = static_cast<double>(bf16lo(xs[q])) - static_cast<double>(bf16lo(ys[q]));
                acc = acc + t0 * t0;
                const double t1 = static_cast<double>(bf16hi(xs[q])) - static_cast<double>(bf16hi(ys[q]));
                acc = acc + t1 * t1;
            } else {
                const double t = static_cast<double>(__uint_as_float(xs[q])) - static_cast<double>(__uint_as_float(ys[q]));
                acc = acc + t * t;
            }
        }
    }
    return acc;
}

// A row in registers, and its squared distance to c in LDS the same way.
template <typename T, int D>
struct Row {
    static constexpr int V = D * static_cast<int>(sizeof(T)) / 16;
    uint4 v[V];
    __device__ __forceinline__ void load(const T* p) {
#pragma unroll
        for (int q = 0; q < V; ++q) v[q] = reinterpret_cast<const uint4*>(p)[q];
    }
    __device__ __forceinline__ void store(T* p) const {
#pragma unroll
        for (int q = 0; q < V; ++q) reinterpret_cast<uint4*>(p)[q] = v[q];
    }
    __device__ __forceinline__ double sqdist(const double* __restrict__ c) {
#pragma clang fp contract(off)
        constexpr int kPer = 16 / static_cast<int>(sizeof(T));
        double acc = 0.0;
#pragma unroll
        for (int q = 0; q < V; ++q) {
            // 16 bytes of the row are widened at a time (widened as a whole it
            // would not fit the registers)
            asm volatile("" : "+v"(acc), "+v"(v[q].x), "+v"(v[q].y), "+v"(v[q].z), "+v"(v[q].w) : : "memory");
            const uint32_t w[4] = {v[q].x, v[q].y, v[q].z, v[q].w};
#pragma unroll
            for (int k = 0; k < kPer; k += 2) {
                const double2 y = *reinterpret_cast<const double2*>(c + q * kPer + k);
                const float x0 = kPer == 8 ? bf16lo(w[k / 2]) : __uint_as_float(w[k & 3]);
                const float x1 = kPer == 8 ? bf16hi(w[k / 2]) : __uint_as_float(w[(k + 1) & 3]);
                const double t0 = static_cast<double>(x0) - y.x;
                acc = acc + t0 * t0;
                const double t1 = static_cast<double>(x1) - y.y;
                acc = acc + t1 * t1;
            }
        }
        return acc;
    }
};

// Completes x here: work on rows streamed through registers is not put off
// (which would keep the rows alive).
__device__ __forceinline__ void done(float& x) { asm volatile("" : "+v"(x)); }
__device__ __forceinline__ void done(double& x) { asm volatile("" : "+v"(x)); }

// One of sixteen lanes' share of a row: d / 16 consecutive elements.
template <typename T, int D>
struct Chunk {
    static constexpr int E = D / 16;
    static constexpr int W = E * static_cast<int>(sizeof(T)) / 4;  // 32-bit words
    static_assert(W == 2 || W == 4 || W == 8, "8, 16 or 32 bytes per lane");
    uint32_t w[W];

    __device__ __forceinline__ void clear() {
#pragma unroll
        for (int i = 0; i < W; ++i) w[i] = 0;
    }
    // hides the words from code motion (rows kept in registers would
    // otherwise be kept a second time, widened)
    __device__ __forceinline__ void opaque() {
#pragma unroll
        for (int i = 0; i < W; ++i) asm volatile("" : "+v"(w[i]));
    }
    __device__ __forceinline__ void load(const T* p) {
        if constexpr (W == 2) {
            const uint2 x = *reinterpret_cast<const uint2*>(p);
            w[0] = x.x;
            w[1] = x.y;
        } else {
#pragma unroll
            for (int i = 0; i < W; i += 4) {
                const uint4 x = *reinterpret_cast<const uint4*>(reinterpret_cast<const uint32_t*>(p) + i);
                w[i] = x.x;
                w[i + 1] = x.y;
                w[i + 2] = x.z;
                w[i + 3] = x.w;
            }
        }
    }
    __device__ __forceinline__ void store(T* p) const {
        if constexpr (W == 2) {
            *reinterpret_cast<uint2*>(p) = make_uint2(w[0], w[1]);
        } else {
#pragma unroll
            for (int i = 0; i < W; i += 4)
                *reinterpret_cast<uint4*>(reinterpret_cast<uint32_t*>(p) + i) = make_uint4(w[i], w[i + 1], w[i + 2], w[i + 3]);
        }
    }
    __device__ __forceinline__ float elem(int e) const {
        if constexpr (sizeof(T) == 2)
            return (e & 1) ? bf16hi(w[e >> 1]) : bf16lo(w[e >> 1]);
        else
            return __uint_as_float(w[e]);
    }
    // this lane's part of the inner product of two rows
    __device__ __forceinline__ float dot(const Chunk& o) const {
        float acc = 0.f;
        if constexpr (sizeof(T) == 2) {
            typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
#pragma unroll
            for (int i = 0; i < W; ++i)
                acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, w[i]),
                                                      __builtin_bit_cast(bf16x2, o.w[i]), acc, false);
        } else {
#pragma unroll
            for (int i = 0; i < W; ++i) acc = fmaf(__uint_as_float(w[i]), __uint_as_float(o.w[i]), acc);
        }
        return acc;
    }
    __device__ __forceinline__ float dot(const float (&c)[E]) const {
        float acc = 0.f;
#pragma unroll
        for (int e = 0; e < E; ++e) acc = fmaf(elem(e), c[e], acc);
        return acc;
    }
};

// Sixteen rows' partial sums per lane -> lane j of the sixteen holds row j's
// total: four halving exchanges (partners l ^ 15, l ^ 7, l ^ 3, l ^ 1).
__device__ __forceinline__ float transpose_sum16(const float (&v)[16]) {
    const int l = lane_id();
    float a[8], b[4], c[2];
    const bool h3 = l & 8, h2 = l & 4, h1 = l & 2, h0 = l & 1;
#pragma unroll
    for (int k = 0; k < 8; ++k) a[k] = (h3 ? v[k + 8] : v[k]) + dpp_f32<0x140>(h3 ? v[k] : v[k + 8]);  // row_mirror
#pragma unroll
    for (int k = 0; k < 4; ++k) b[k] = (h2 ? a[k + 4] : a[k]) + dpp_f32<0x141>(h2 ? a[k] : a[k + 4]);  // row_half_mirror
#pragma unroll
    for (int k = 0; k < 2; ++k) c[k] = (h1 ? b[k + 2] : b[k]) + dpp_f32<0x1B>(h1 ? b[k] : b[k + 2]);   // quad [3,2,1,0]
    return (h0 ? c[1] : c[0]) + dpp_f32<0xB1>(h0 ? c[0] : c[1]);                                      // quad [1,0,3,2]
}

// A member's running minimum over the representatives so far: the three
// smallest estimates and the representatives of the first two (own = first |
// second << 16).  A chosen representative has m1 = -inf and owns itself.
// While a parent is built by the definition's distances (m1, m2) hold the
// bits of its fp64 minimum and own its owner.
struct MemberState {
    float m1, m2, m3;
    uint32_t own;
    float nx;  // the member's squared norm (kept here in memory only)
    __device__ __forceinline__ void reset() {
        m1 = m2 = m3 = kInf;
        own = 0;
    }
    __device__ __forceinline__ void add(float a, uint32_t u) {
        const bool first = a < m1, second = a < m2;
        m3 = fminf(m3, fmaxf(m2, a));
        m2 = fminf(m2, fmaxf(m1, a));
        m1 = fminf(m1, a);
        own = first ? (own << 16) | u : second ? (own & 0xffffu) | (u << 16) : own;
    }
    __device__ __forceinline__ void choose(uint32_t u) {
        m1 = -kInf;
        own = (own & 0xffff0000u) | u;
    }
    __device__ __forceinline__ double exact() const {
        return __hiloint2double(__float_as_int(m2), __float_as_int(m1));
    }
    __device__ __forceinline__ void set_exact(double m, int o) {
        m1 = __int_as_float(__double2loint(m));
        m2 = __int_as_float(__double2hiint(m));
        own = static_cast<uint32_t>(o);
    }
};

// LDS of a build workgroup of nw waves and up to r representatives (bytes).
struct BuildLds {
    int part, vec, row, best, red, tie_i, tie_v, reps, cnt, off, wcnt, misc, total;
};
__host__ __device__ inline BuildLds build_lds(int nw, int r, int d, int esz) {
    BuildLds L{};
    int o = 0;
    auto take = [&](int bytes) {
        const int at = o;
        o += (bytes + 15) / 16 * 16;
        return at;
    };
    L.part = take(nw * d * 8);  // the waves' mean sums; then the waves' farthest rows (2 nw rows)
    L.row = L.part;
    static_assert(2 * 4 <= 8, "two fp32 rows fit a row of doubles");
    L.vec = take(d * 8);
    L.best = take(2 * nw * 16);
    L.red = take(nw * static_cast<int>(sizeof(ArgVal)));
    L.tie_i = take(kTie * 4);
    L.tie_v = take(kTie * 8);
    L.reps = take(r * 4);
    L.cnt = take(r * 4);
    L.off = take(r * 4);
    L.wcnt = take(nw * (r < kRankBlock ? r : kRankBlock) * 4);
    L.misc = take((nw + 4) * 4);
    L.total = o;
    return L;
}

// The thread index as a value of its own: what is derived from it here is not
// kept in registers from (or for) another phase of the kernel.
__device__ __forceinline__ int fresh_tid() {
    int t = threadIdx.x;
    asm volatile("" : "+v"(t));
    return t;
}

// Arrays of a table, written by the build kernels.
template <typename T>
struct TeamArrays {
    int* team_begin;
    int* team_size;
    double* log_n;
    int* rep_token;
    int* perm;
    T* packed_K;
    T* packed_V;
    T* reps;
};

// The end of a parent's build: its teams (of the representatives in LDS and
// owner(i) of each member), its part of perm and, with PACK, its packed rows and
// routing keys.  store_row(k, to) writes row k of a lane group's sixteen, for
// the HELD rows that registers hold.
template <typename T, int D, bool ONE, bool PACK, int HELD, typename Tok, typename Owner, typename Store>
__device__ __forceinline__ void write_teams(const TeamArrays<T>& out, const T* __restrict__ K, const T* __restrict__ V,
                                            int N, int R, int M, int bh, int start, int n, int team0, int nt, char* lds,
                                            Tok tok, Owner owner, Store store_row) {
    using C = Chunk<T, D>;
    constexpr int E = C::E;
    const int tid = fresh_tid(), nw = nt / kWave;
    const int lane = tid & (kWave - 1), w = tid / kWave, sub = tid & 15, g16 = tid & ~15, lbase = lane & 48;
    const int r = min(R, n), nblk = ONE ? 1 : (n + nt - 1) / nt, wstride = min(R, kRankBlock);
    const BuildLds L = build_lds(nw, R, D, sizeof(T));
    const int* const s_reps = reinterpret_cast<const int*>(lds + L.reps);
    int* const s_cnt = reinterpret_cast<int*>(lds + L.cnt);
    int* const s_off = reinterpret_cast<int*>(lds + L.off);
    int* const s_wcnt = reinterpret_cast<int*>(lds + L.wcnt);
    int* const s_misc = reinterpret_cast<int*>(lds + L.misc);

            // team sizes and offsets inside the parent
            __syncthreads();
            for (int u = tid; u < r; u += nt) s_cnt[u] = 0;
            __syncthreads();
            for (int i = tid; i < n; i += nt) atomicAdd(&s_cnt[owner(i)], 1);
            __syncthreads();
            for (int base = 0; base < r; base += nt) {
                const int u = base + tid;
                const int c = u < r ? s_cnt[u] : 0;
                const int inc = wave_incl_scan(c);
                if (lane == kWave - 1) s_misc[4 + w] = inc;
                __syncthreads();
                int pre = base > 0 ? s_off[base - 1] + s_cnt[base - 1] : 0;
                for (int v = 0; v < w; ++v) pre += s_misc[4 + v];
                if (u < r) s_off[u] = pre + inc - c;
                __syncthreads();
            }
            const size_t tbase = static_cast<size_t>(bh) * M + team0;
            for (int u = tid; u < r; u += nt) {
                out.team_begin[tbase + u] = start + s_off[u];
                out.team_size[tbase + u] = s_cnt[u];
                out.log_n[tbase + u] = log(static_cast<double>(s_cnt[u]));
                out.rep_token[tbase + u] = tok(s_reps[u]);
            }
            __syncthreads();

            // packed position of each member: its team's offset plus its rank among
            // the team's members in token order, per block of nt members and of 64
            // representatives, one ballot per representative and wave
            int* const pperm = out.perm + static_cast<size_t>(bh) * N + start;
            const uint64_t lt = lanemask_lt();
            int pos = 0;
            for (int b = 0; b < nblk; ++b) {
                const int i = b * nt + tid;
                const int o = i < n ? owner(i) : -1;
                for (int ub = 0; ub < r; ub += kRankBlock) {
                    const int nb = min(kRankBlock, r - ub);
                    int rank = 0;
                    for (int q = 0; q < nb; ++q) {
                        const uint64_t bm = __ballot(o == ub + q);
                        if (o == ub + q) rank = __popcll(bm & lt);
                        if (lane == 0) s_wcnt[w * wstride + q] = __popcll(bm);
                    }
                    __syncthreads();
                    if (o >= ub && o < ub + nb) {
                        int ps = s_off[o] + rank;
                        for (int v = 0; v < w; ++v) ps += s_wcnt[v * wstride + o - ub];
                        pperm[ps] = tok(i);
                        pos = ps;
                    }
                    __syncthreads();
                    if (!ONE) {  // the next block's members follow
                        for (int q = tid; q < nb; q += nt) {
                            int add = 0;
                            for (int v = 0; v < nw; ++v) add += s_wcnt[v * wstride + q];
                            s_off[ub + q] += add;
                        }
                        __syncthreads();
                    }
                }
            }

            // packed copies of a contiguous parent of one block: whole rows, sixteen
            // lanes each, keys from the registers that hold them
            if constexpr (PACK) {
                const size_t prow0 = static_cast<size_t>(bh) * N + start;
                auto dst = [&](T* base, int k) { return base + (prow0 + __shfl(pos, lbase + k)) * D + sub * E; };
    #pragma unroll
                for (int k = 0; k < HELD; ++k) {
                    T* const to = dst(out.packed_K, k);
                    if (g16 + k < n) store_row(k, to);
                }
                // rows k0 .. 15 of src
                auto copy = [&](const T* src, T* to, int k0) {
    #pragma unroll 1
                    for (; k0 < 16; k0 += 4) {
                        C x[4];
    #pragma unroll
                        for (int k = 0; k < 4; ++k)
                            if (g16 + k0 + k < n) x[k].load(src + (prow0 + g16 + k0 + k) * D + sub * E);
    #pragma unroll
                        for (int k = 0; k < 4; ++k) {
                            T* const p = dst(to, k0 + k);
                            if (g16 + k0 + k < n) x[k].store(p);
                        }
                    }
                };
                copy(K, out.packed_K, HELD);
                copy(V, out.packed_V, 0);
                for (int e = tid; e < r * 16; e += nt) {
                    const int u = e >> 4, c = e & 15;
                    C x;
                    x.load(K + (static_cast<size_t>(bh) * N + tok(s_reps[u])) * D + c * E);
                    x.store(out.reps + (tbase + u) * D + c * E);
                }
            }
}

// Thread t owns members t, t + nt, ... of its parent (nt threads run; ONE:
// at most nt members, so one each, its state in registers, else in `state`).
// Each sixteen lanes hold the rows of their sixteen members of a block of nt
// together, one sixteenth of every row per lane, so that rows are read and
// written whole and a round needs one sixteenth of the representative per
// lane; the first block's first CACHE rows stay in registers for the whole
// build, the rest are read again each round (from the L2).
//
// What bounds it: instruction issue in the rounds (per sixteen members of a
// lane group 64 dot products of bf16 pairs, the exchange that hands each lane
// its member's sum, about 100 instructions of state and maximum; one barrier),
// and the rows' traffic before and after them.  32K tokens of bf16 d = 128 for
// four KV heads, P = 1024, R = 16: 74 us, of which 38 us with R = 1, so 2.2 us
// a round (fp64 distances of rows in registers took 6.7 us a round, 178 us in
// all).  9001 tokens of fp32 d = 128: 117 us, most rows read again from the L2
// every round (4.1 us a round; 620 us in fp64 with 256 threads).  P = 16, R = 4
// at 32K: 64 us, one wave per parent (518 us).  K-means parents at 32K: 140 us
// (782 us).
template <typename T, int D, bool LIST, bool ONE>
__device__ void build_parent(const T* __restrict__ K, const T* __restrict__ V, int N, int R, int M, int bh, int start,
                             int n, int team0, int nt, const int* __restrict__ mem,
                             MemberState* __restrict__ state_all, const TeamArrays<T>& out, char* lds) {
    using C = Chunk<T, D>;
    constexpr int E = C::E;
    // rows kept in registers, and rows of the others in flight at once: what
    // 128 registers a thread hold beside the sixteen sums
    constexpr int CACHE = C::W == 2 ? 16 : C::W == 4 && ONE ? 16 : 4;
    constexpr int BATCH = C::W == 2 ? 8 : C::W == 4 ? 4 : 2;
    // whole rows fit the registers: parents that the estimates leave open are
    // built by k_build_open
    constexpr bool DEFER = ONE && !LIST && CACHE == 16;
    const int tid = threadIdx.x, nw = nt / kWave;
    const int w = wave_id(), lane = lane_id(), sub = lane & 15, g16 = tid & ~15, lbase = lane & 48;
    const int r = min(R, n);
    const int nblk = ONE ? 1 : (n + nt - 1) / nt;
    const BuildLds L = build_lds(nw, R, D, sizeof(T));
    double* const s_part = reinterpret_cast<double*>(lds + L.part);
    char* const s_row = lds + L.row;
    double* const s_vec = reinterpret_cast<double*>(lds + L.vec);
    float4* const s_best = reinterpret_cast<float4*>(lds + L.best);
    ArgVal* const s_red = reinterpret_cast<ArgVal*>(lds + L.red);
    int* const s_ti = reinterpret_cast<int*>(lds + L.tie_i);
    unsigned long long* const s_tv = reinterpret_cast<unsigned long long*>(lds + L.tie_v);
    int* const s_reps = reinterpret_cast<int*>(lds + L.reps);
    int* const s_misc = reinterpret_cast<int*>(lds + L.misc);

    const T* const Kb = K + static_cast<size_t>(bh) * N * D;
    auto tok = [&](int i) { return LIST ? mem[i] : start + i; };
    auto row = [&](int i) { return Kb + static_cast<size_t>(tok(i)) * D; };
    MemberState* const state = ONE ? nullptr : state_all + static_cast<size_t>(bh) * N + start;

    // the rows of this lane's sixteen members of block b
    const int mytok = tid < n ? tok(tid) : start;
    C cache[CACHE];
#pragma unroll
    for (int k = 0; k < CACHE; ++k) {
        const int t = LIST ? __shfl(mytok, lbase + k) : start + g16 + k;
        cache[k].clear();
        if (g16 + k < n) cache[k].load(Kb + static_cast<size_t>(t) * D + sub * E);
    }
    // f(k, chunk) for the sixteen rows of block b (k a compile-time index;
    // rows past the last member are zero)
    auto rows_of = [&](int b, auto&& f) {
        auto stream = [&](int i0, int tk, auto first) {
            constexpr int kFirst = decltype(first)::value;
#pragma unroll
            for (int k0 = kFirst; k0 < 16; k0 += BATCH) {
                // addresses are formed anew for each batch (kept over the
                // rounds they would take two registers per row), and a batch
                // is used before the next is requested
                asm volatile("" : "+v"(i0), "+v"(tk));
                C x[BATCH];
#pragma unroll
                for (int k = 0; k < BATCH; ++k) {
                    const int t = LIST ? __shfl(tk, lbase + k0 + k) : start + i0 + k0 + k;
                    x[k].clear();
                    if (i0 + k0 + k < n) x[k].load(Kb + static_cast<size_t>(t) * D + sub * E);
                }
#pragma unroll
                for (int k = 0; k < BATCH; ++k) {
                    x[k].opaque();
                    f(k0 + k, x[k]);
                }
            }
        };
        if (ONE || b == 0) {
#pragma unroll
            for (int k = 0; k < CACHE; ++k) {
                cache[k].opaque();
                f(k, cache[k]);
            }
            if constexpr (CACHE < 16) stream(g16, mytok, std::integral_constant<int, CACHE>{});
        } else {
            stream(b * nt + g16, b * nt + tid < n ? tok(b * nt + tid) : start, std::integral_constant<int, 0>{});
        }
    };

    // squared norms (one per member; of the first block kept), the largest,
    // and the sums of each dimension over the lane's rows
    float nx0 = 0.f, nmax = 0.f;
    bool odd = false;  // a norm that is not finite
    {
        double sums[E];
#pragma unroll
        for (int e = 0; e < E; ++e) sums[e] = 0.0;
        for (int b = 0; b < nblk; ++b) {
            float pp[16];
            rows_of(b, [&](int k, const C& x) {
                pp[k] = x.dot(x);
                done(pp[k]);
#pragma unroll
                for (int e = 0; e < E; ++e) {
                    sums[e] += static_cast<double>(x.elem(e));
                    done(sums[e]);
                }
            });
            const float nx = transpose_sum16(pp);
            if (ONE)
                nx0 = nx;
            else if (b * nt + tid < n)
                state[b * nt + tid].nx = nx;
            odd = odd || !(nx <= kNormMax);
            nmax = fmaxf(nmax, nx);
        }
#pragma unroll
        for (int e = 0; e < E; ++e) {
            double s = sums[e];
            s += __shfl_xor(s, 16);
            s += __shfl_xor(s, 32);
            if (lane < 16) s_part[w * D + sub * E + e] = s;
        }
    }
    nmax = wave_max_f32(__ballot(odd) ? kInf : nmax);
    if (lane == 0) s_best[w].x = nmax;
    __syncthreads();
    for (int v = 0; v < nw; ++v) nmax = fmaxf(nmax, s_best[v].x);
    for (int j = tid; j < D; j += nt) {
        double s = 0.0;
        for (int v = 0; v < nw; ++v) s += s_part[v * D + j];
        s_vec[j] = s / static_cast<double>(n);
    }
    if (tid == 0) s_misc[0] = 0;
    __syncthreads();
    bool exact = !(nmax >= kNormMin && nmax <= kNormMax);  // uniform
    bool zero = false;
    if (nmax == 0.f) {  // uniform: padding, as a rule; every distance is 0 then
        const int tid = fresh_tid();
        uint32_t bits = 0;
        for (int i = tid; i < n; i += nt) {
#pragma unroll 4
            for (int q = 0; q < D * static_cast<int>(sizeof(T)) / 16; ++q) {
                const uint4 x = reinterpret_cast<const uint4*>(row(i))[q];
                bits |= x.x | x.y | x.z | x.w;
            }
        }
        bits &= sizeof(T) == 2 ? 0x7fff7fffu : 0x7fffffffu;  // (zeros of either sign)
        if (__ballot(bits != 0) != 0 && (tid & (kWave - 1)) == 0) s_misc[0] = 1;
        __syncthreads();
        zero = s_misc[0] == 0;
        __syncthreads();
        if (tid == 0) s_misc[0] = 0;
    }
    const float err2 = 2.f * kEstimate * nmax;

    MemberState st;
    st.reset();
    st.nx = nx0;
    int rep = 0;

    // s_vec = the members' mean, each dimension summed in token order.
    auto definition_mean = [&]() {
        const int tid = fresh_tid(), sub = tid & 15, g16 = tid & ~15;
        __syncthreads();
        // rows held in registers reach the summing threads through LDS
        const int stage = DEFER ? nw * 8 / static_cast<int>(sizeof(T)) : 0;
        if (stage >= 16 && D <= nt) {  // uniform
            T* const s_rows = reinterpret_cast<T*>(s_row);
            const int step = stage & ~15;
            double s = 0.0;
            for (int i0 = 0; i0 < n; i0 += step) {
                if (g16 >= i0 && g16 < i0 + step) {
#pragma unroll
                    for (int k = 0; k < CACHE; ++k) cache[k].store(s_rows + (g16 - i0 + k) * D + sub * E);
                }
                __syncthreads();
                if (tid < D) s = sum_rows(s, s_rows + tid, min(step, n - i0), [](int i) { return static_cast<size_t>(i) * D; });
                __syncthreads();
            }
            if (tid < D) s_vec[tid] = s / static_cast<double>(n);
        } else {
            for (int j = tid; j < D; j += nt) {
                const double s = sum_rows(0.0, Kb + j, n, [&](int i) { return static_cast<size_t>(tok(i)) * D; });
                s_vec[j] = s / static_cast<double>(n);
            }
        }
        __syncthreads();
    };

    // The member nearest that mean.  A reduction without a winner (NaN keys)
    // falls back to member 0, so that every index stays inside the parent.
    auto first_by_definition = [&]() {
        definition_mean();
        const int tid = fresh_tid();
        ArgVal best{INFINITY, 0x7fffffff};
        for (int i = tid; i < n; i += nt) best = pick_min(best, ArgVal{sqdist_to(row(i), s_vec, D), i});
        best = block_arg<false>(best, s_red, nw);
        return best.i < n ? best.i : 0;
    };

    // The members listed in s_ti (cnt <= kTie of them, s_tv preset to ~0):
    // their running minima over the first nv representatives by the
    // definition's distances, into s_tv; a (member, representative) pair per
    // thread.
    auto tie_minima = [&](int cnt, int nv) {
        for (int e = tid; e < cnt * nv; e += nt) {
            const int c = e / nv, v = e - c * nv;
            const double d2 = sqdist_rows<T, D>(row(s_ti[c]), row(s_reps[v]));
            atomicMin(&s_tv[c], static_cast<unsigned long long>(__double_as_longlong(d2)));
        }
    };

    int known = 0;  // representatives the estimates found
    if (!exact) {
        // first representative: the member nearest the mean
        const int tid = fresh_tid(), lane = tid & (kWave - 1), w = tid / kWave;
        float mean[E];
        float mm = 0.f;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            mean[e] = static_cast<float>(s_vec[sub * E + e]);
            mm = fmaf(mean[e], mean[e], mm);
        }
        mm = row16_sum(mm);
        float near = kInf, near2 = kInf;  // this thread's two smallest
        int ni = 0;
        for (int b = 0; b < nblk; ++b) {
            float pp[16];
            rows_of(b, [&](int k, const C& x) {
                pp[k] = x.dot(mean);
                if (k >= CACHE || !ONE) done(pp[k]);
            });
            const float dt = transpose_sum16(pp);
            const int i = b * nt + tid;
            if (i < n) {
                const float nx = ONE ? nx0 : state[i].nx;
                const float a = nx + mm - 2.f * dt;
                near2 = fminf(near2, fmaxf(near, a));
                if (a < near) {
                    near = a;
                    ni = i;
                }
            }
        }
        {
            const float wm = -wave_max_f32(-near);
            const uint64_t in = __ballot(near <= wm + err2 && near < kInf);
            const uint64_t in2 = __ballot(near2 <= wm + err2 && near2 < kInf);
            const uint64_t at = __ballot(near == wm);
            const int idx = readlane(ni, at ? __ffsll(static_cast<unsigned long long>(at)) - 1 : 0);
            if (lane == 0)
                s_best[w] = make_float4(wm, __int_as_float(idx), __int_as_float(__popcll(in) > 1 || in2 != 0 ? 1 : 0), 0.f);
        }
        __syncthreads();
        const float4 eb = s_best[min(lane, nw - 1)];
        const float T0 = -wave_max_f32(lane < nw ? -eb.x : -kInf);
        const uint64_t nearw = __ballot(lane < nw && eb.x <= T0 + err2);
        const int wsel = __ffsll(static_cast<unsigned long long>(nearw)) - 1;
        const bool alone = __popcll(nearw) == 1 && readlane(__float_as_int(eb.z), wsel) == 0;
        rep = readlane(__float_as_int(eb.y), wsel);
        if (!alone) {
            // several members: their distances to the fp64 mean.  That mean's
            // sums run in another order than the definition's, so the winner
            // has to be clear of the others by the difference this can make;
            // otherwise (equal rows, as a rule) the definition's own mean
            // decides.
            for (int b = 0; b < nblk; ++b) {
                // (the estimates again: only a thread's smallest was kept)
                float pp[16];
                rows_of(b, [&](int k, const C& x) {
                pp[k] = x.dot(mean);
                if (k >= CACHE || !ONE) done(pp[k]);
            });
                const float dt = transpose_sum16(pp);
                const int i = b * nt + tid;
                if (i < n && (ONE ? nx0 : state[i].nx) + mm - 2.f * dt <= T0 + err2) {
                    const int at = atomicAdd(&s_misc[0], 1);
                    if (at < kTie) s_ti[at] = i;
                }
            }
            __syncthreads();
            const int cnt = s_misc[0];
            if (cnt == n && n > kTie) {
                exact = true;  // uniform
            } else if (cnt > kTie) {
                rep = first_by_definition();
            } else {
                if (tid < cnt) s_tv[tid] = static_cast<unsigned long long>(__double_as_longlong(sqdist_to(row(s_ti[tid]), s_vec, D)));
                __syncthreads();
                ArgVal win{INFINITY, 0x7fffffff};
                for (int c = 0; c < cnt; ++c)
                    win = pick_min(win, ArgVal{__longlong_as_double(static_cast<long long>(s_tv[c])), s_ti[c]});
                const double slack = static_cast<double>(n + 256) * 0x1.0p-49 * static_cast<double>(nmax);
                bool clear = true;
                for (int c = 0; c < cnt; ++c)
                    clear = clear && (s_ti[c] == win.i || __longlong_as_double(static_cast<long long>(s_tv[c])) > win.v + slack);
                rep = win.i;
                if (!clear) {  // uniform
                    definition_mean();
                    if (tid < cnt) s_tv[tid] = static_cast<unsigned long long>(__double_as_longlong(sqdist_to(row(s_ti[tid]), s_vec, D)));
                    __syncthreads();
                    win = ArgVal{INFINITY, 0x7fffffff};
                    for (int c = 0; c < cnt; ++c)
                        win = pick_min(win, ArgVal{__longlong_as_double(static_cast<long long>(s_tv[c])), s_ti[c]});
                    rep = win.i;
                }
            }
            __syncthreads();
            if (tid == 0) s_misc[0] = 0;
        }
        known = exact ? 0 : 1;
        if (tid == 0) s_reps[0] = rep;
    }

    if (!exact) {
        // farthest-first rounds.  Every wave publishes its farthest member
        // (and, with one member per thread, that member's row), and after the
        // round's one barrier each wave finds the workgroup's.  s_best and
        // s_row alternate between two sets: a set is rewritten two rounds
        // after it was read, past the barrier of the round between.
        const int tid = fresh_tid(), lane = tid & (kWave - 1), w = tid / kWave;
        C rc;
        rc.load(row(rep) + sub * E);
        float nr = row16_sum(rc.dot(rc));
        for (int u = 0; u < r; ++u) {
            if (tid == 0) s_reps[u] = rep;
            float far = -kInf, far2 = -kInf;
            int fi = 0;
            for (int b = 0; b < nblk; ++b) {
                float pp[16];
                rows_of(b, [&](int k, const C& x) {
                    pp[k] = x.dot(rc);
                    if (k >= CACHE || !ONE) done(pp[k]);
                });
                const float dt = transpose_sum16(pp);
                const int i = b * nt + tid;
                if (i < n) {
                    MemberState s = ONE ? st : state[i];
                    if (u == 0) s.reset();
                    s.add((ONE ? nx0 : s.nx) + nr - 2.f * dt, static_cast<uint32_t>(u));
                    if (i == rep) s.choose(static_cast<uint32_t>(u));
                    if (ONE)
                        st = s;
                    else
                        state[i] = s;
                    far2 = fmaxf(far2, fminf(far, s.m1));
                    if (s.m1 > far) {
                        far = s.m1;
                        fi = i;
                    }
                }
            }
            if (u + 1 == r) break;
            const int set = ((u + 1) & 1) * nw;  // (the first representative used set 0)
            const float wm = wave_max_f32(far);
            const uint64_t in = __ballot(far >= wm - err2 && far > -kInf);
            const uint64_t in2 = ONE ? 0 : __ballot(far2 >= wm - err2 && far2 > -kInf);
            const uint64_t at = __ballot(far == wm);
            const int lsel = __ffsll(static_cast<unsigned long long>(at)) - 1;
            const int idx = readlane(fi, lsel);
            const float nidx = __int_as_float(readlane(__float_as_int(nx0), lsel));
            if (lane == 0)
                s_best[set + w] = make_float4(wm, __int_as_float(idx), __int_as_float(__popcll(in) > 1 || in2 != 0 ? 1 : 0), nidx);
            if constexpr (ONE) {
                if ((lane >> 4) == (lsel >> 4)) {
                    const int kk = lsel & 15;  // wave-uniform
                    T* const dst = reinterpret_cast<T*>(s_row + (set + w) * D * static_cast<int>(sizeof(T))) + sub * E;
                    if (kk < CACHE) {
#pragma unroll
                        for (int hi = 0; hi < CACHE; hi += 4) {
                            if ((kk & ~3) != hi) continue;
#pragma unroll
                            for (int k = hi; k < hi + 4; ++k)
                                if (k == kk) cache[k].store(dst);
                        }
                    } else if (idx < n) {
                        C x;
                        x.load(row(idx) + sub * E);
                        x.store(dst);
                    }
                }
            }
            __syncthreads();
            const float4 eb = s_best[set + min(lane, nw - 1)];
            const float T0 = wave_max_f32(lane < nw ? eb.x : -kInf);
            const uint64_t farw = __ballot(lane < nw && eb.x >= T0 - err2);
            const int wsel = __ffsll(static_cast<unsigned long long>(farw)) - 1;
            const bool alone = __popcll(farw) == 1 && readlane(__float_as_int(eb.z), wsel) == 0;
            rep = readlane(__float_as_int(eb.y), wsel);
            if (alone) {
                if constexpr (ONE) {
                    rc.load(reinterpret_cast<const T*>(s_row + (set + wsel) * D * static_cast<int>(sizeof(T))) + sub * E);
                    nr = __int_as_float(readlane(__float_as_int(eb.w), wsel));
                } else {
                    rc.load(row(rep) + sub * E);
                    nr = row16_sum(rc.dot(rc));
                }
                continue;
            }
            // several members within the bound: the definition's minima
            for (int b = 0; b < nblk; ++b) {
                const int i = b * nt + tid;
                if (i < n) {
                    const float m1 = ONE ? st.m1 : state[i].m1;
                    if (m1 >= T0 - err2 && m1 > -kInf) {
                        const int at = atomicAdd(&s_misc[0], 1);
                        if (at < kTie) {
                            s_ti[at] = i;
                            s_tv[at] = ~0ull;
                        }
                    }
                }
            }
            __syncthreads();
            const int cnt = s_misc[0];
            if (cnt > kTie || err2 > kWide * T0) {
                exact = true;  // uniform
                known = u + 1;
                break;
            }
            tie_minima(cnt, u + 1);
            __syncthreads();
            ArgVal win{-INFINITY, 0x7fffffff};
            for (int c = 0; c < cnt; ++c)
                win = pick_max(win, ArgVal{__longlong_as_double(static_cast<long long>(s_tv[c])), s_ti[c]});
            rep = win.i < n ? win.i : 0;
            rc.load(row(rep) + sub * E);
            nr = row16_sum(rc.dot(rc));
            __syncthreads();  // s_ti and s_tv are rewritten by a later round
            if (tid == 0) s_misc[0] = 0;
        }
    }
    if (zero) {
        // the lowest members become the representatives, the rest join the first
        const int tid = fresh_tid();
        for (int u = tid; u < r; u += nt) s_reps[u] = u;
        for (int i = tid; i < n; i += nt) {
            const uint32_t o = i < r ? static_cast<uint32_t>(i) : 0u;
            if (ONE)
                st.own = o;
            else
                state[i].own = o;
        }
    } else if (!exact) {
        // owners the estimates leave open: the definition's distances to the
        // two nearest representatives, or to all where a third is as near (by
        // sixteen lanes each, where members have a thread of their own)
        const int tid = fresh_tid();
        __syncthreads();
        int* const s_list = reinterpret_cast<int*>(s_row);
        int listed = -1;
        for (int b = 0; b < nblk; ++b) {
            const int i = b * nt + tid;
            if (i >= n) continue;
            MemberState s = ONE ? st : state[i];
            if (s.m1 > -kInf && s.m2 - s.m1 <= err2) {
                int o = static_cast<int>(s.own & 0xffffu);
                if (s.m3 - s.m1 <= err2) {
                    if (ONE) {
                        listed = atomicAdd(&s_misc[0], 1);
                        s_list[listed] = i;
                        continue;
                    }
                    double m = INFINITY;
                    for (int v = 0; v < r; ++v) {
                        const double d2 = sqdist_rows<T, D>(row(i), row(s_reps[v]));
                        if (d2 < m) {
                            m = d2;
                            o = v;
                        }
                    }
                } else {
                    const int o1 = min(o, static_cast<int>(s.own >> 16)), o2 = max(o, static_cast<int>(s.own >> 16));
                    const double d1 = sqdist_rows<T, D>(row(i), row(s_reps[o1]));
                    const double d2 = sqdist_rows<T, D>(row(i), row(s_reps[o2]));
                    o = d2 < d1 ? o2 : o1;
                }
                if (ONE)
                    st.own = static_cast<uint32_t>(o);
                else
                    state[i].own = static_cast<uint32_t>(o);
            }
        }
        if (ONE) {
            __syncthreads();
            const int cnt = s_misc[0];
            for (int c = tid >> 4; c < cnt; c += nt / 16) {
                const T* const x = row(s_list[c]);
                double m = INFINITY;
                int o = 0x7fffffff;
                for (int v = tid & 15; v < r; v += 16) {
                    const double d2 = sqdist_rows<T, D>(x, row(s_reps[v]));
                    if (d2 < m) {
                        m = d2;
                        o = v;
                    }
                }
                for (int off = 8; off > 0; off >>= 1) {
                    const double om = __shfl_xor(m, off);
                    const int oo = __shfl_xor(o, off);
                    if (om < m || (om == m && oo < o)) {
                        m = om;
                        o = oo;
                    }
                }
                if ((tid & 15) == 0) s_list[c] = o;
            }
            __syncthreads();
            if (listed >= 0) st.own = static_cast<uint32_t>(s_list[listed]);
        }
    } else if constexpr (DEFER) {
        // left to k_build_open, with the representatives found so far
        const int tid = fresh_tid();
        const size_t tbase = static_cast<size_t>(bh) * M + team0;
        __syncthreads();
        for (int u = tid; u < known; u += nt) out.rep_token[tbase + u] = start + s_reps[u];
        if (tid == 0) out.team_size[tbase] = -1 - known;
        return;
    } else {
        // the definition's arithmetic throughout (the representatives that the
        // estimates found are the definition's)
        const int tid = fresh_tid();
        if (known == 0) {
            rep = first_by_definition();
            known = 1;
            if (tid == 0) s_reps[0] = rep;
        }
        for (int u = 0; u < r; ++u) {
            __syncthreads();
            if (u < known)
                rep = s_reps[u];
            else if (tid == 0)
                s_reps[u] = rep;
            for (int j = tid; j < D; j += nt) s_vec[j] = static_cast<double>(load_elem(row(rep), j));
            __syncthreads();
            // fold the new representative into the running minimum; a chosen
            // representative gets -1 so that it is never chosen again
            ArgVal far{-INFINITY, 0x7fffffff};
            for (int b = 0; b < nblk; ++b) {
                const int i = b * nt + tid;
                if (i >= n) continue;
                const double dd = sqdist_to(row(i), s_vec, D);
                double m = dd;
                int o = u;
                if (u > 0) {
                    const MemberState s = ONE ? st : state[i];
                    m = s.exact();
                    o = static_cast<int>(s.own);
                    if (dd < m) {
                        m = dd;
                        o = u;
                    }
                }
                if (i == rep) {
                    m = -1.0;
                    o = u;
                }
                if (ONE)
                    st.set_exact(m, o);
                else
                    state[i].set_exact(m, o);
                far = pick_max(far, ArgVal{m, i});
            }
            if (u + 1 < r && u + 1 >= known) {
                far = block_arg<true>(far, s_red, nw);
                rep = far.i < n ? far.i : 0;
            }
        }
    }
    write_teams<T, D, ONE, ONE && !LIST, CACHE>(
        out, K, V, N, R, M, bh, start, n, team0, nt, lds, tok,
        [&](int i) { return static_cast<int>((ONE ? st.own : state[i].own) & 0xffffu); },
        [&](int k, T* to) { cache[k].store(to); });
}

// Contiguous parents [pP, min(pP + P, N)); every pair has M teams.
template <typename T, int D, bool ONE>
__global__ __launch_bounds__(kBuildThreads) void k_build_contiguous(
    const T* __restrict__ K, const T* __restrict__ V, int N, int P, int R, int M, MemberState* __restrict__ state,
    TeamArrays<T> out, int* __restrict__ team_count) {
    extern __shared__ __align__(16) char s_build[];
    const int p = blockIdx.x, bh = blockIdx.y, start = p * P;
    if (p == 0 && threadIdx.x == 0) team_count[bh] = M;
    build_parent<T, D, false, ONE>(K, V, N, R, M, bh, start, min(P, N - start), p * min(R, P), blockDim.x, nullptr, state, out,
                                   s_build);
}

// LDS of k_build_open: build_lds, then the rows that nt threads load at once, one
// 16-byte piece each (16 bytes of padding a row spread them over the banks).
template <typename T, int D>
__host__ __device__ constexpr int open_rows(int nt) { return nt * 16 / (D * static_cast<int>(sizeof(T))); }
template <typename T, int D>
__host__ __device__ constexpr int open_stage_bytes(int nt) { return open_rows<T, D>(nt) * (D * static_cast<int>(sizeof(T)) + 16); }

// The contiguous parents that k_build_contiguous left open (first team's size
// negative: -1 - the representatives it found, which stand in rep_token): the
// definition's arithmetic throughout, each thread's member in its registers.
// What bounds it is fp64 issue, 128 dimensions x 5 operations a member and
// representative.  A 32K table of equal rows (bf16, d = 128, P = 1024, R = 16;
// host time, an allocation included) takes 231 us, with rows past fp32's range
// 214; with every row read from memory each round they took 341 and 331, with all
// tables built by the definition 263 and 257.
template <typename T, int D>
__global__ __launch_bounds__(kBuildThreads) void k_build_open(const T* __restrict__ K, const T* __restrict__ V, int N,
                                                              int P, int R, int M, TeamArrays<T> out) {
    extern __shared__ __align__(16) char s_build[];
    const int p = blockIdx.x, bh = blockIdx.y, start = p * P, n = min(P, N - start), team0 = p * min(R, P);
    const size_t tbase = static_cast<size_t>(bh) * M + team0;
    const int left = out.team_size[tbase];
    if (left >= 0) return;  // uniform
    const int known = -1 - left, r = min(R, n);
    const int tid = threadIdx.x, nt = blockDim.x, nw = nt / kWave;
    const BuildLds L = build_lds(nw, R, D, sizeof(T));
    double* const s_vec = reinterpret_cast<double*>(s_build + L.vec);
    ArgVal* const s_red = reinterpret_cast<ArgVal*>(s_build + L.red);
    int* const s_reps = reinterpret_cast<int*>(s_build + L.reps);
    T* const s_rows = reinterpret_cast<T*>(s_build + L.total);
    constexpr int kPieces = D * static_cast<int>(sizeof(T)) / 16, kStride = D + 16 / static_cast<int>(sizeof(T));
    for (int u = tid; u < known; u += nt) s_reps[u] = out.rep_token[tbase + u] - start;

    // the members' rows, whole lines from memory, through LDS to their threads;
    // and their mean on the way, each dimension summed in token order
    const int step = open_rows<T, D>(nt);
    const T* const Kp = K + (static_cast<size_t>(bh) * N + start) * D;
    const int lr = tid / kPieces, lc = tid % kPieces;
    auto piece = [&](int i) { return reinterpret_cast<const uint4*>(Kp + static_cast<size_t>(min(i, n - 1)) * D)[lc]; };
    Row<T, D> own;
#pragma unroll
    for (int q = 0; q < Row<T, D>::V; ++q) own.v[q] = make_uint4(0, 0, 0, 0);
    double sum[D / kWave];
#pragma unroll
    for (int q = 0; q < D / kWave; ++q) sum[q] = 0.0;
    uint4 next = piece(lr);
    for (int i0 = 0; i0 < n; i0 += step) {
        reinterpret_cast<uint4*>(s_rows + lr * kStride)[lc] = next;
        next = piece(i0 + step + lr);
        __syncthreads();
        if (known == 0) {
#pragma unroll
            for (int q = 0; q < D / kWave; ++q)
                if (q * nt + tid < D)
                    sum[q] = sum_rows(sum[q], s_rows + q * nt + tid, min(step, n - i0),
                                      [](int i) { return static_cast<size_t>(i) * kStride; });
        }
        if (tid >= i0 && tid < i0 + step) own.load(s_rows + (tid - i0) * kStride);
        __syncthreads();
    }
    int rep = 0;
    if (known == 0) {
#pragma unroll
        for (int q = 0; q < D / kWave; ++q)
            if (q * nt + tid < D) s_vec[q * nt + tid] = sum[q] / static_cast<double>(n);
        __syncthreads();
        const double dd = own.sqdist(s_vec);
        ArgVal best{INFINITY, 0x7fffffff};
        if (tid < n) best = pick_min(best, ArgVal{dd, tid});
        best = block_arg<false>(best, s_red, nw);
        rep = best.i < n ? best.i : 0;  // no winner among NaN keys: member 0
    }
    double m = 0.0;
    int owner = 0;
    for (int u = 0; u < r; ++u) {
        if (u < known)
            rep = s_reps[u];
        else if (tid == 0)
            s_reps[u] = rep;
        if (tid == rep) own.store(s_rows);
        __syncthreads();
        for (int j = tid; j < D; j += nt) s_vec[j] = static_cast<double>(load_elem(s_rows, j));
        __syncthreads();
        // fold the new representative into the running minimum; a chosen
        // representative gets -1 so that it is never chosen again
        const double dd = own.sqdist(s_vec);
        if (u == 0 || dd < m) {
            m = dd;
            owner = u;
        }
        if (tid == rep) {
            m = -1.0;
            owner = u;
        }
        if (u + 1 < r && u + 1 >= known) {
            ArgVal far{-INFINITY, 0x7fffffff};
            if (tid < n) far = pick_max(far, ArgVal{m, tid});
            far = block_arg<true>(far, s_red, nw);
            rep = far.i < n ? far.i : 0;
        }
    }
    write_teams<T, D, true, true, 0>(out, K, V, N, R, M, bh, start, n, team0, nt, s_build, [=](int i) { return start + i; },
                                     [=](int) { return owner; }, [](int, T*) {});
}

// Label-defined parents: the members are the token indices mem[0 .. n)
// (ascending) of the pair's member lists.
template <typename T, int D>
__global__ __launch_bounds__(kBuildThreads) void k_build_lists(
    const T* __restrict__ K, int N, int R, int M, MemberState* __restrict__ state, TeamArrays<T> out,
    const int* __restrict__ members, const int* __restrict__ pbeg, const int* __restrict__ toff, int Mp) {
    extern __shared__ __align__(16) char s_build[];
    const int p = blockIdx.x, bh = blockIdx.y;
    const size_t at = static_cast<size_t>(bh) * (Mp + 1) + p;
    const int start = pbeg[at], n = pbeg[at + 1] - start;
    if (n <= 0) return;  // empty parents are omitted (uniform over the workgroup)
    const int* const mem = members + static_cast<size_t>(bh) * N + start;
    // waves without members end here (a barrier counts the waves that have not
    // ended), so that small parents leave room for others: a table of 2600 parents
    // of one or a few members takes 223 us, 310 with all waves kept
    const int nt = min(kBuildThreads, (n + kWave - 1) / kWave * kWave);
    if (static_cast<int>(threadIdx.x) >= nt) return;
    if (n <= nt)  // uniform
        build_parent<T, D, true, true>(K, nullptr, N, R, M, bh, start, n, toff[at], nt, mem, state, out, s_build);
    else
        build_parent<T, D, true, false>(K, nullptr, N, R, M, bh, start, n, toff[at], nt, mem, state, out, s_build);
}

// Row gather into team order: packed[bh][pos] = src[bh][perm[bh][pos]], and the
// representative keys reps[bh][g] = K[bh][rep_token[bh][g]].  One thread per
// 16-byte chunk of a row.
__global__ __launch_bounds__(256) void k_gather_rows(const uint4* __restrict__ src,
                                                     uint4* __restrict__ dst,
                                                     const int* __restrict__ index, int rows_out,
                                                     int rows_in, int chunks_per_row, int BH) {
    const size_t total = static_cast<size_t>(BH) * rows_out * chunks_per_row;
    for (size_t t = blockIdx.x * static_cast<size_t>(blockDim.x) + threadIdx.x; t < total;
         t += static_cast<size_t>(gridDim.x) * blockDim.x) {
        const size_t row = t / chunks_per_row;
        const int c = static_cast<int>(t - row * chunks_per_row);
        const size_t bh = row / rows_out;
        const int srow = index[row];
        dst[t] = src[(bh * rows_in + srow) * chunks_per_row + c];
    }
}

}  // namespace

size_t build_state_bytes() { return sizeof(MemberState); }

// A parent of at most kBuildThreads members is one member per thread: its
// state stays in registers and the workgroup writes the packed rows itself.
bool build_packs_in_place(int N, int P) { return std::min(P, N) <= kBuildThreads; }

namespace {

// f(element type, dims) of a build
template <typename F>
hipError_t build_forms(santapp_dtype dtype, int d, F&& f) {
    if (dtype == SANTAPP_BF16 && d == 128) return f(bf16_t{}, std::integral_constant<int, 128>{});
    if (dtype == SANTAPP_BF16 && d == 64) return f(bf16_t{}, std::integral_constant<int, 64>{});
    if (dtype == SANTAPP_FP32 && d == 128) return f(float{}, std::integral_constant<int, 128>{});
    if (dtype == SANTAPP_FP32 && d == 64) return f(float{}, std::integral_constant<int, 64>{});
    return hipErrorInvalidValue;
}

template <typename T>
TeamArrays<T> team_arrays(const TeamTable& t) {
    return TeamArrays<T>{t.team_begin, t.team_size, t.log_n, t.rep_token, t.perm,
                         static_cast<T*>(t.packed_K), static_cast<T*>(t.packed_V), static_cast<T*>(t.reps)};
}

int build_threads(int N, int P) { return std::min(kBuildThreads, (std::min(P, N) + kWave - 1) / kWave * kWave); }

}  // namespace

hipError_t launch_build_parents(const void* K, const void* V, santapp_dtype dtype, int BH, int N, int d, int P, int R,
                                int M, void* state, const TeamTable& t, int* team_count, hipStream_t s) {
    const dim3 grid((N + P - 1) / P, BH);
    const int threads = build_threads(N, P);
    const int lds = build_lds(threads / kWave, R, d, dtype == SANTAPP_BF16 ? 2 : 4).total;
    return build_forms(dtype, d, [&](auto elem, auto dims) {
        using T = decltype(elem);
        constexpr int D = decltype(dims)::value;
        auto kern = build_packs_in_place(N, P) ? k_build_contiguous<T, D, true> : k_build_contiguous<T, D, false>;
        kern<<<grid, threads, lds, s>>>(static_cast<const T*>(K), static_cast<const T*>(V), N, P, R, M,
                                        static_cast<MemberState*>(state), team_arrays<T>(t), team_count);
        return hipGetLastError();
    });
}

hipError_t launch_build_open(const void* K, const void* V, santapp_dtype dtype, int BH, int N, int d, int P, int R, int M,
                             const TeamTable& t, hipStream_t s) {
    const dim3 grid((N + P - 1) / P, BH);
    const int threads = build_threads(N, P);
    const int lds = build_lds(threads / kWave, R, d, dtype == SANTAPP_BF16 ? 2 : 4).total;
    return build_forms(dtype, d, [&](auto elem, auto dims) -> hipError_t {
        using T = decltype(elem);
        constexpr int D = decltype(dims)::value;
        if constexpr (D * sizeof(T) > 256) {
            return hipErrorInvalidValue;  // such parents are never left open
        } else {
            k_build_open<T, D><<<grid, threads, lds + open_stage_bytes<T, D>(threads), s>>>(
                static_cast<const T*>(K), static_cast<const T*>(V), N, P, R, M, team_arrays<T>(t));
            return hipGetLastError();
        }
    });
}

hipError_t launch_build_parent_lists(const void* K, santapp_dtype dtype, int BH, int N, int d, int Mp, int R, int M,
                                     const int* members, const int* pbeg, const int* toff, void* state,
                                     const TeamTable& t, hipStream_t s) {
    const dim3 grid(Mp, BH);
    const int lds = build_lds(kBuildWaves, R, d, dtype == SANTAPP_BF16 ? 2 : 4).total;
    return build_forms(dtype, d, [&](auto elem, auto dims) {
        using T = decltype(elem);
        k_build_lists<T, decltype(dims)::value><<<grid, kBuildThreads, lds, s>>>(
            static_cast<const T*>(K), N, R, M, static_cast<MemberState*>(state), team_arrays<T>(t), members, pbeg, toff, Mp);
        return hipGetLastError();
    });
}

hipError_t launch_gather_rows(const void* src, void* dst, const int* index, int BH, int rows_out,
                              int rows_in, size_t row_bytes, hipStream_t s) {
    const int chunks = static_cast<int>(row_bytes / 16);
    const size_t total = static_cast<size_t>(BH) * rows_out * chunks;
    const size_t want = (total + 255) / 256;
    const unsigned blocks = static_cast<unsigned>(want < 65536 ? want : 65536);
    k_gather_rows<<<blocks, 256, 0, s>>>(static_cast<const uint4*>(src), static_cast<uint4*>(dst),
                                         index, rows_out, rows_in, chunks, BH);
    return hipGetLastError();
}

}  // namespace santapp
