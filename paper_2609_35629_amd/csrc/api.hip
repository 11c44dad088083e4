// C ABI of libsantapp: argument checks, buffer ownership, workspace layout and
// launch sequencing.  All arithmetic runs in the kernels.
#include <math.h>
#include <stdarg.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <atomic>
#include <functional>
#include <mutex>
#include <string>
#include <vector>

#include "internal.h"

struct santapp_teams {
    int B, Hkv, N, d;
    santapp_dtype dtype;
    int P, R, M;
    void* packed_K;
    void* packed_V;
    void* reps;
    int* team_begin;
    int* team_size;
    double* log_n;
    int* rep_token;
    int* perm;
    int* team_count;  // [B*Hkv] teams of each pair (M for contiguous parents)
    void* block;      // the one device allocation every array above is carved from
    size_t block_bytes;
    // cap[x]: the most attention chunks any x distinct teams of one (b, kv)
    // need (sum of their x largest chunk counts, maximum over (b, kv))
    std::vector<int> cap;
    int cus;  // compute units of the device the handle was built on
};

namespace {

thread_local std::string g_err;

santapp_status fail(santapp_status st, const char* fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof(buf), fmt, ap);
    va_end(ap);
    g_err = buf;
    return st;
}

santapp_status ok() {
    g_err.clear();
    return SANTAPP_OK;
}

santapp_status hip_fail(hipError_t e, const char* what) {
    return fail(SANTAPP_EHIP, "%s: %s", what, hipGetErrorString(e));
}

size_t elem_size(santapp_dtype dt) { return dt == SANTAPP_BF16 ? 2 : 4; }

bool dtype_ok(santapp_dtype dt) { return dt == SANTAPP_BF16 || dt == SANTAPP_FP32; }

size_t align_up(size_t x) { return (x + 255) & ~static_cast<size_t>(255); }

constexpr int kWaves8 = santapp::kDecodeThreads / 64;  // waves of a decode workgroup

// Device buffers are read and written with 16-byte vector accesses.
bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

// Compute units of the current device (0 if the query fails), looked up once
// per device.
int device_cus() {
    constexpr int kDevs = 64;
    static std::atomic<int> cache[kDevs];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) {
        (void)hipGetLastError();
        return 0;
    }
    if (dev < 0 || dev >= kDevs) return 0;
    int n = cache[dev].load(std::memory_order_relaxed);
    if (n > 0) return n;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n < 0) {
        (void)hipGetLastError();
        return 0;
    }
    cache[dev].store(n, std::memory_order_relaxed);
    return n;
}

// Teams per (b, kv) for contiguous parents: every parent but the last has P
// members and min(R, P) teams.
long long team_count(int N, int P, int R) {
    const long long np = (static_cast<long long>(N) + P - 1) / P;
    const long long last = N - (np - 1) * static_cast<long long>(P);
    return (np - 1) * std::min<long long>(R, P) + std::min<long long>(R, last);
}

// Device blocks kept for the next table or preparation scratch of a similar
// size.  A hipMalloc and a hipFree of a 68 MiB table take 40 and 260 us (and
// at times a millisecond), more than the 75 us kernel that builds it.
//   - A block is only given out again once nothing can still use it: release()
//     waits for the whole device first, as hipFree does, so that a table may be
//     destroyed under the same conditions as before; release_idle() is for
//     scratch whose only stream the caller has waited for.
//   - Bounded: at most kBlocks blocks and kBytes bytes over all devices; what
//     does not fit is freed, the oldest first, and all of it is freed when an
//     allocation fails or the caller asks for it (santapp_trim).
//   - Any thread may call; a block goes back to the device it came from.
class BlockPool {
   public:
    // A block of at least `bytes` on the current device; its size in *got.
    hipError_t acquire(void** p, size_t bytes, size_t* got) {
        bytes = (bytes + kGrain - 1) / kGrain * kGrain;
        int dev = 0;
        hipError_t e = hipGetDevice(&dev);
        if (e != hipSuccess) return e;
        {
            std::lock_guard<std::mutex> lock(mu_);
            int best = -1;
            for (int i = 0; i < n_; ++i)
                if (b_[i].dev == dev && b_[i].bytes >= bytes && b_[i].bytes <= bytes + bytes / 4 &&
                    (best < 0 || b_[i].bytes < b_[best].bytes))
                    best = i;
            if (best >= 0) {
                const Block x = take(best);
                *p = x.p;
                *got = x.bytes;
                return hipSuccess;
            }
        }
        e = hipMalloc(p, bytes);
        if (e != hipSuccess) {
            (void)hipGetLastError();
            (void)drop_all();
            e = hipMalloc(p, bytes);
        }
        *got = bytes;
        return e;
    }

    // Back to the pool once the device that holds p is idle.
    void release(void* p, size_t bytes) {
        if (!p) return;
        int dev = 0, cur = 0;
        hipPointerAttribute_t at;
        bool idle = hipPointerGetAttributes(&at, p) == hipSuccess && hipGetDevice(&cur) == hipSuccess;
        if (idle) {
            dev = at.device;
            if (dev != cur) idle = hipSetDevice(dev) == hipSuccess;
            // hipFree's own wait for the device, on a block of no size to
            // speak of (hipDeviceSynchronize would end a graph capture that
            // another stream has in progress in relaxed mode; hipFree does not)
            void* small = nullptr;
            idle = idle && hipMalloc(&small, 256) == hipSuccess && hipFree(small) == hipSuccess;
            if (dev != cur) (void)hipSetDevice(cur);
        }
        if (idle) {
            keep(p, bytes, dev);
        } else {
            (void)hipGetLastError();
            (void)hipFree(p);
        }
    }

    // The same for a block of the current device that nothing uses any more.
    void release_idle(void* p, size_t bytes) {
        int dev = 0;
        if (!p) return;
        if (hipGetDevice(&dev) == hipSuccess)
            keep(p, bytes, dev);
        else
            (void)hipFree(p);
    }

    // Frees every block kept.
    hipError_t drop_all() {
        Block out[kBlocks];
        int nout = 0;
        {
            std::lock_guard<std::mutex> lock(mu_);
            while (n_ > 0) out[nout++] = take(0);
        }
        hipError_t first = hipSuccess;
        for (int i = 0; i < nout; ++i) {
            const hipError_t e = hipFree(out[i].p);
            if (first == hipSuccess) first = e;
        }
        return first;
    }

   private:
    static constexpr int kBlocks = 16;
    static constexpr size_t kBytes = size_t(1) << 30, kGrain = size_t(1) << 16;
    struct Block {
        void* p;
        size_t bytes;
        int dev;
    };
    std::mutex mu_;
    Block b_[kBlocks];  // oldest first
    int n_ = 0;
    size_t held_ = 0;

    Block take(int i) {
        const Block x = b_[i];
        for (int j = i + 1; j < n_; ++j) b_[j - 1] = b_[j];
        --n_;
        held_ -= x.bytes;
        return x;
    }
    void keep(void* p, size_t bytes, int dev) {
        Block out[kBlocks + 1];
        int nout = 0;
        {
            std::lock_guard<std::mutex> lock(mu_);
            while (n_ > 0 && (n_ == kBlocks || held_ + bytes > kBytes)) out[nout++] = take(0);
            if (bytes <= kBytes) {
                b_[n_++] = Block{p, bytes, dev};
                held_ += bytes;
            } else {
                out[nout++] = Block{p, bytes, dev};
            }
        }
        for (int i = 0; i < nout; ++i) (void)hipFree(out[i].p);
    }
};

// Never destroyed: tables may outlive this library's static objects.
BlockPool& pool() {
    static BlockPool* const p = new BlockPool;
    return *p;
}

void free_teams(santapp_teams* t) {
    if (!t) return;
    pool().release(t->block, t->block_bytes);
    delete t;
}

santapp::TeamTable table_arrays(const santapp_teams* t) {
    return santapp::TeamTable{t->packed_K, t->packed_V, t->reps, t->team_begin, t->team_size,
                              t->log_n, t->rep_token, t->perm};
}

// Waits for the build queued on s (and for build_open's launches, where parents
// were left open), then sets the chunk capacities and the
// device's compute units of the table; frees it on failure.
template <typename Open>
santapp_status finish_table(santapp_teams* t, hipStream_t s, santapp_teams** out, Open&& build_open) {
    const size_t BH = static_cast<size_t>(t->B) * t->Hkv;
    std::vector<int> sizes(BH * t->M);
    auto fetch = [&]() {
        const hipError_t e = hipMemcpyAsync(sizes.data(), t->team_size, sizes.size() * sizeof(int), hipMemcpyDeviceToHost, s);
        return e == hipSuccess ? hipStreamSynchronize(s) : e;
    };
    hipError_t e = fetch();
    int sign = 0;
    if (e == hipSuccess)
        for (int x : sizes) sign |= x;
    if (sign < 0) {  // parents left open
        e = build_open();
        if (e == hipSuccess) e = fetch();
    }
    if (e != hipSuccess) {
        free_teams(t);
        return hip_fail(e, "team build");
    }
    int dev = 0;
    t->cus = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&t->cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
        t->cus = 0;
    (void)hipGetLastError();
    t->cap.assign(t->M + 1, 0);
    std::vector<int> cnt(t->M);
    for (size_t bh = 0; bh < BH; ++bh) {
        for (int g = 0; g < t->M; ++g) cnt[g] = santapp::chunk_count(sizes[bh * t->M + g]);
        std::sort(cnt.begin(), cnt.end(), std::greater<int>());
        int run = 0;
        for (int x = 1; x <= t->M; ++x) {
            run += cnt[x - 1];
            t->cap[x] = std::max(t->cap[x], run);
        }
    }
    *out = t;
    return ok();
}

}  // namespace

namespace santapp {

int decode_wgs(int cus, long long BH, long long units_per_pair) {
    if (cus < 1) cus = 8;
    long long want = (BH * units_per_pair + kWaves8 - 1) / kWaves8;  // a unit per wave
    want = std::max<long long>(want, std::min<long long>(BH, cus));   // every pair a workgroup
    want = std::min<long long>(want, cus);
    if (cus % 8 == 0) want = std::min<long long>(cus, (want + 7) / 8 * 8);
    return static_cast<int>(std::max<long long>(want, 1));
}

namespace {

struct Carver {
    size_t off = 0;
    size_t take(size_t bytes) {
        const size_t at = off;
        off = align_up(off + bytes);
        return at;
    }
};

// Every device array of a table (t->B, Hkv, N, M, d and dtype set) from one
// allocation, each 256-byte aligned.
hipError_t alloc_table(santapp_teams* t) {
    const size_t BH = static_cast<size_t>(t->B) * t->Hkv;
    const size_t N = static_cast<size_t>(t->N), M = static_cast<size_t>(t->M);
    const size_t row = static_cast<size_t>(t->d) * elem_size(t->dtype);
    Carver c;
    const size_t oK = c.take(BH * N * row), oV = c.take(BH * N * row), oR = c.take(BH * M * row);
    const size_t ob = c.take(BH * M * sizeof(int)), os = c.take(BH * M * sizeof(int));
    const size_t ol = c.take(BH * M * sizeof(double)), ot = c.take(BH * M * sizeof(int));
    const size_t op = c.take(BH * N * sizeof(int)), oc = c.take(BH * sizeof(int));
    void* p = nullptr;
    const hipError_t e = pool().acquire(&p, c.off, &t->block_bytes);
    if (e != hipSuccess) return e;
    char* const b = static_cast<char*>(p);
    t->block = b;
    t->packed_K = b + oK;
    t->packed_V = b + oV;
    t->reps = b + oR;
    t->team_begin = reinterpret_cast<int*>(b + ob);
    t->team_size = reinterpret_cast<int*>(b + os);
    t->log_n = reinterpret_cast<double*>(b + ol);
    t->rep_token = reinterpret_cast<int*>(b + ot);
    t->perm = reinterpret_cast<int*>(b + op);
    t->team_count = reinterpret_cast<int*>(b + oc);
    return hipSuccess;
}

}  // namespace

namespace {

// Launch mode asked for by SANTAPP_DECODE_LAUNCH (read once per process):
// "split" or "fused" take the three-launch kernels (fused: in one launch);
// anything else takes the single-launch step wherever it applies.
enum class LaunchMode { kStep, kSplit, kFused };

LaunchMode launch_mode() {
    static const LaunchMode m = [] {
        const char* e = getenv("SANTAPP_DECODE_LAUNCH");
        if (e != nullptr && strcmp(e, "fused") == 0) return LaunchMode::kFused;
        if (e != nullptr && strcmp(e, "split") == 0) return LaunchMode::kSplit;
        return LaunchMode::kStep;
    }();
    return m;
}

// The single-launch step's own workspace: epochs, the tagged exchange words
// (sampled steps) and the tagged partial states.
void step_regions(DecodeLayout& L, size_t BH, int G, int M, int d, bool dense, size_t& off) {
    auto take = [&](size_t bytes) {
        const size_t at = off;
        off = (off + bytes + 255) & ~static_cast<size_t>(255);
        return at;
    };
    L.epoch = take(BH * sizeof(uint32_t));
    if (!dense) {
        L.xk = take(BH * G * 3 * static_cast<size_t>(M) * 8);
    }
    L.part = take(BH * L.maxwp * G * static_cast<size_t>(step_state_bytes(d)));
}

// A 64-bit value that no earlier call had and that memory holds only by a
// chance of 2^-64: a counter through an invertible mixing of its bits
// (Steele, Lea, Flood: SplitMix64).
uint64_t call_token() {
    static std::atomic<uint64_t> calls{0x5bf03635u};
    uint64_t z = (calls.fetch_add(1, std::memory_order_relaxed) + 1) * 0x9e3779b97f4a7c15ull;
    z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
    z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
    z ^= z >> 31;
    return z != 0 ? z : 1;
}

bool fused_wanted() { return launch_mode() == LaunchMode::kFused; }

}  // namespace

bool step_mode(santapp_dtype dt, int d, long long BH, int M, int Kp, bool dense, int cus) {
    if (launch_mode() != LaunchMode::kStep) return false;
    if (dt != SANTAPP_BF16 || (d != 64 && d != 128) || cus < 8 || BH < 1 || BH > cus) return false;
    return dense || (M <= kStepMaxTeams && Kp <= kStepMaxKp);
}

int step_wgs(int cus, long long BH) {
    if (cus % 8 == 0 && BH * 8 <= cus) {
        const long long per = std::min<long long>(kStepMaxWgs, 8 * (cus / (8 * BH)));
        return static_cast<int>(BH * per);
    }
    return static_cast<int>(BH * std::min<long long>(kStepMaxWgs, cus / BH));
}

bool fused_step(santapp_dtype dt, const DecodeLayout& L) {
    return !L.step && dt == SANTAPP_BF16 && fused_wanted() && L.nwg % 8 == 0;
}

StepLayout decode_layout(int B, int Hq, int Hkv, int T, int d, int M, int Kp, const int* cap, int cus,
                         santapp_dtype dt, size_t ws_bytes) {
    StepLayout L;
    const size_t BH = static_cast<size_t>(B) * Hkv, BQ = static_cast<size_t>(B) * Hq;
    const int G = Hq / Hkv;
    if (step_mode(dt, d, static_cast<long long>(BH), M, Kp, false, cus)) {
        L.step = true;
        L.nwg = step_wgs(cus, static_cast<long long>(BH));
        L.maxwp = pair_wgs(0, L.nwg, static_cast<int>(BH));
        L.swords = (M + 63) / 64;
        size_t off = 0;
        step_regions(L, BH, G, M, d, false, off);
        L.total = off;
        return L;
    }
    const long long xs = std::min<long long>(M, static_cast<long long>(G) * Kp);
    L.nwg = decode_wgs(cus, static_cast<long long>(BH), chunk_count(T) + static_cast<long long>(std::max(1, cap[xs])));
    L.maxwp = BH <= static_cast<size_t>(L.nwg) ? pair_wgs(0, L.nwg, static_cast<int>(BH)) : 1;
    L.swords = (M + 63) / 64;
    Carver c;
    L.ctr = c.take((BH + BH * G) * sizeof(int));
    L.sbits = c.take(BQ * L.swords * sizeof(uint64_t));
    L.lc = c.take(BQ * M * sizeof(float));
    L.part = c.take(BH * L.maxwp * G * state_stride(d) * sizeof(float));
    L.total = c.off;
    // The launch over all teams pays from about 1200 teams on, while the heads
    // leave half the compute units to it (one step, this against a workgroup per
    // head): 28 heads 656 teams 32.3 / 28.0 us, 1024 33.9 / 32.4, 1280 35.0 /
    // 35.6, 2048 37.1 / 43.1; 112 heads 1024 teams 48.4 / 46.9, 1100 35.3 / 34.4,
    // 1280 51.3 / 51.4, 2048 62.7 / 68.4; 256 heads 1024 teams 51.4 / 50.2, 2048
    // 68.9 / 64.5.  And for budgets whose teams, with those that the bound lets in
    // beside them (about 210 at K = 144, 250 at 160, whatever the table), fit its
    // list of 256; past that it ranks all teams (28 heads, K = 300: 2048 teams 59 /
    // 46.6 us, 8192 teams 130 / 117).  The regions are part of the size from 1024
    // teams on and for every budget, so that a workspace for one budget of a table
    // serves its others.
    if (M > kKeyMinTeams && BQ <= static_cast<size_t>(cus) / 2 && !fused_step(dt, L)) {
        StepLayout X = L;
        X.keys = M > kKeyUseTeams && Kp <= kKeyMaxK;
        X.key.stride = (M + 3) / 4 * 4;
        const size_t n = BQ * X.key.stride;
        X.key.yu = c.take(n * sizeof(uint32_t));
        X.key.yk = c.take(n * sizeof(uint64_t));
        X.key.phi = c.take(n * sizeof(double));
        X.key.tokens = c.take(BH * key_blocks(M) * sizeof(uint64_t));
        X.total = c.off;
        if (X.total <= ws_bytes) return X;
    }
    return L;
}

StepLayout dense_layout(int B, int Hq, int Hkv, int N, int T, int d, int cus, santapp_dtype dt) {
    StepLayout L;
    const size_t BH = static_cast<size_t>(B) * Hkv;
    const int G = Hq / Hkv;
    if (step_mode(dt, d, static_cast<long long>(BH), 0, 0, true, cus)) {
        L.step = true;
        L.nwg = step_wgs(cus, static_cast<long long>(BH));
        L.maxwp = pair_wgs(0, L.nwg, static_cast<int>(BH));
        size_t off = 0;
        step_regions(L, BH, G, 0, d, true, off);
        L.total = off;
        return L;
    }
    L.nwg = decode_wgs(cus, static_cast<long long>(BH), chunk_count(N) + static_cast<long long>(chunk_count(T)));
    L.maxwp = BH <= static_cast<size_t>(L.nwg) ? pair_wgs(0, L.nwg, static_cast<int>(BH)) : 1;
    Carver c;
    L.ctr = c.take((BH + BH * G) * sizeof(int));
    L.part = c.take(BH * L.maxwp * G * state_stride(d) * sizeof(float));
    L.total = c.off;
    return L;
}

}  // namespace santapp

using namespace santapp;

extern "C" {

const char* santapp_last_error(void) { return g_err.c_str(); }

santapp_status santapp_budget_to_K(int S, int P, int R, int M, int* K) {
    if (!K) return fail(SANTAPP_EINVAL, "K is NULL");
    if (S < 1 || P < 1 || R < 1 || M < 1)
        return fail(SANTAPP_EINVAL, "S, P, R and M must be positive (got %d, %d, %d, %d)", S, P, R, M);
    if (P % R != 0) return fail(SANTAPP_EINVAL, "P (%d) must be divisible by R (%d)", P, R);
    const int per = P / R;
    if (S % per != 0) return fail(SANTAPP_EINVAL, "S (%d) must be divisible by P/R (%d)", S, per);
    *K = std::min(M, S / per);
    return ok();
}

santapp_status santapp_build_teams(const void* K, const void* V, int B, int Hkv, int N, int d,
                                   santapp_dtype dtype, int parent_size, int reps_per_parent,
                                   void* stream, santapp_teams** out) {
    if (!out) return fail(SANTAPP_EINVAL, "out is NULL");
    *out = nullptr;
    if (!K || !V) return fail(SANTAPP_EINVAL, "K and V must be device pointers");
    if (!aligned16(K) || !aligned16(V)) return fail(SANTAPP_EINVAL, "K and V must be 16-byte aligned");
    if (B < 1 || Hkv < 1 || N < 1) return fail(SANTAPP_EINVAL, "B, Hkv, N must be >= 1");
    if (parent_size < 1) return fail(SANTAPP_EINVAL, "parent_size must be >= 1");
    if (reps_per_parent < 1) return fail(SANTAPP_EINVAL, "reps_per_parent must be >= 1");
    if (!dtype_ok(dtype)) return fail(SANTAPP_EDTYPE, "unsupported dtype %d", static_cast<int>(dtype));
    if (d != 64 && d != 128) return fail(SANTAPP_ELIMIT, "head dim %d not supported (64 or 128)", d);
    if (reps_per_parent > kMaxReps)
        return fail(SANTAPP_ELIMIT, "reps_per_parent %d exceeds %d", reps_per_parent, kMaxReps);
    const long long M = team_count(N, parent_size, reps_per_parent);
    const size_t BH = static_cast<size_t>(B) * Hkv;
    if (BH * static_cast<size_t>(N) > static_cast<size_t>(0x7fffffff))
        return fail(SANTAPP_ELIMIT, "B*Hkv*N exceeds 2^31");
    hipStream_t s = static_cast<hipStream_t>(stream);
    const size_t esz = elem_size(dtype);
    const size_t row = static_cast<size_t>(d) * esz;

    santapp_teams* t = new santapp_teams();
    t->B = B;
    t->Hkv = Hkv;
    t->N = N;
    t->d = d;
    t->dtype = dtype;
    t->P = parent_size;
    t->R = reps_per_parent;
    t->M = static_cast<int>(M);
    void* state = nullptr;
    size_t state_bytes = 0;
    hipError_t e = alloc_table(t);
    const bool packed = build_packs_in_place(N, parent_size);
    if (e == hipSuccess && !packed) e = pool().acquire(&state, BH * N * build_state_bytes(), &state_bytes);
    if (e != hipSuccess) {
        free_teams(t);
        (void)hipGetLastError();
        return fail(SANTAPP_ENOMEM, "device allocation failed: %s", hipGetErrorString(e));
    }
    const char* what = "team build";
    e = launch_build_parents(K, V, dtype, static_cast<int>(BH), N, d, parent_size, reps_per_parent,
                             t->M, state, table_arrays(t), t->team_count, s);
    if (e == hipSuccess && !packed) {
        what = "packing K";
        e = launch_gather_rows(K, t->packed_K, t->perm, static_cast<int>(BH), N, N, row, s);
    }
    if (e == hipSuccess && !packed) {
        what = "packing V";
        e = launch_gather_rows(V, t->packed_V, t->perm, static_cast<int>(BH), N, N, row, s);
    }
    if (e == hipSuccess && !packed) {
        what = "gathering representatives";
        e = launch_gather_rows(K, t->reps, t->rep_token, static_cast<int>(BH), t->M, N, row, s);
    }
    if (e != hipSuccess) {
        // a launch failed: an earlier one of this call may still run, so the
        // buffers go back through a wait for the device
        pool().release(state, state_bytes);
        free_teams(t);
        return hip_fail(e, what);
    }
    const santapp_status st = finish_table(t, s, out, [&]() {  // waits for the build
        return launch_build_open(K, V, dtype, static_cast<int>(BH), N, d, parent_size, reps_per_parent, t->M,
                                 table_arrays(t), s);
    });
    if (st == SANTAPP_OK)
        pool().release_idle(state, state_bytes);
    else
        pool().release(state, state_bytes);
    return st;
}

santapp_status santapp_kmeans_parents(const void* K, int B, int Hkv, int N, int d, santapp_dtype dtype,
                                      int parent_size, const santapp_kmeans_settings* theta, int* labels,
                                      int* num_parents, int* steps, void* stream) {
    if (!K || !labels || !theta) return fail(SANTAPP_EINVAL, "K, labels and theta must not be NULL");
    if (!aligned16(K) || !aligned16(labels)) return fail(SANTAPP_EINVAL, "K and labels must be 16-byte aligned");
    if (B < 1 || Hkv < 1 || N < 2) return fail(SANTAPP_EINVAL, "B, Hkv must be >= 1 and N >= 2");
    if (parent_size < 1) return fail(SANTAPP_EINVAL, "parent_size must be >= 1");
    if (theta->batch_size < 1 || theta->max_iter < 0 || theta->max_no_improvement < 0 ||
        theta->init_size < 0 || !(theta->reassignment_ratio >= 0.0 && theta->reassignment_ratio < 1.0))
        return fail(SANTAPP_EINVAL, "invalid k-means settings");
    if (!dtype_ok(dtype)) return fail(SANTAPP_EDTYPE, "unsupported dtype %d", static_cast<int>(dtype));
    if (d != 64 && d != 128) return fail(SANTAPP_ELIMIT, "head dim %d not supported (64 or 128)", d);
    const int M = std::min(N, std::max(2, N / parent_size));
    if (M > kKmMaxCenters) return fail(SANTAPP_ELIMIT, "%d k-means parents exceed %d", M, kKmMaxCenters);
    const size_t BH = static_cast<size_t>(B) * Hkv;
    if (BH * static_cast<size_t>(N) > static_cast<size_t>(0x7fffffff))
        return fail(SANTAPP_ELIMIT, "B*Hkv*N exceeds 2^31");
    const long long steps_total = static_cast<long long>(theta->max_iter) * N / theta->batch_size;
    if (steps_total > 0x7fffffff) return fail(SANTAPP_ELIMIT, "too many minibatch steps");
    int s0 = theta->init_size > 0 ? theta->init_size : 3 * theta->batch_size;
    if (s0 < M) s0 = 3 * M;
    if (s0 > N) s0 = N;
    const KmLayout L = kmeans_layout(static_cast<int>(BH), N, d, M, theta->batch_size, s0);
    hipStream_t s = static_cast<hipStream_t>(stream);
    void* block = nullptr;
    size_t block_bytes = 0;
    hipError_t e = pool().acquire(&block, L.total, &block_bytes);
    char* const ws = static_cast<char*>(block);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        return fail(SANTAPP_ENOMEM, "k-means scratch (%zu bytes): %s", L.total, hipGetErrorString(e));
    }
    const char* what = "k-means seeding";
    e = launch_kmeans_seed(K, dtype, static_cast<int>(BH), N, d, L, ws, theta->seed, s);
    const double alpha = std::min(1.0, 2.0 * theta->batch_size / (static_cast<double>(N) + 1.0));
    std::vector<KmState> st(BH);
    // minibatch steps in groups; stopped pairs skip the rest, and the loop
    // ends once every pair has stopped
    constexpr int kGroup = 16;
    for (long long first = 0; e == hipSuccess && first < steps_total; first += kGroup) {
        const int count = static_cast<int>(std::min<long long>(kGroup, steps_total - first));
        what = "k-means steps";
        e = launch_kmeans_steps(K, dtype, static_cast<int>(BH), N, d, L, ws, theta->batch_size,
                                static_cast<int>(first), count, alpha, theta->reassignment_ratio,
                                theta->max_no_improvement, theta->seed, s);
        if (e == hipSuccess && theta->max_no_improvement > 0) {
            what = "k-means state";
            e = hipMemcpyAsync(st.data(), ws + L.state, BH * sizeof(KmState), hipMemcpyDeviceToHost, s);
            if (e == hipSuccess) e = hipStreamSynchronize(s);
            if (e == hipSuccess &&
                std::all_of(st.begin(), st.end(), [](const KmState& x) { return x.stop != 0; }))
                break;
        }
    }
    if (e == hipSuccess) {
        what = "k-means labels";
        e = launch_kmeans_labels(K, dtype, static_cast<int>(BH), N, d, L, ws, labels, s);
    }
    if (e == hipSuccess) {
        what = "k-means state";
        e = hipMemcpyAsync(st.data(), ws + L.state, BH * sizeof(KmState), hipMemcpyDeviceToHost, s);
        if (e == hipSuccess) e = hipStreamSynchronize(s);
    }
    if (e != hipSuccess) {
        pool().release(block, block_bytes);
        return hip_fail(e, what);
    }
    pool().release_idle(block, block_bytes);  // the stream has been waited for
    if (num_parents) *num_parents = M;
    if (steps)
        for (size_t i = 0; i < BH; ++i) steps[i] = st[i].steps;
    return ok();
}

santapp_status santapp_build_teams_from_labels(const void* K, const void* V, int B, int Hkv, int N, int d,
                                               santapp_dtype dtype, const int* labels, int num_labels,
                                               int reps_per_parent, void* stream, santapp_teams** out) {
    if (!out) return fail(SANTAPP_EINVAL, "out is NULL");
    *out = nullptr;
    if (!K || !V || !labels) return fail(SANTAPP_EINVAL, "K, V and labels must be device pointers");
    if (!aligned16(K) || !aligned16(V) || !aligned16(labels))
        return fail(SANTAPP_EINVAL, "K, V and labels must be 16-byte aligned");
    if (B < 1 || Hkv < 1 || N < 1) return fail(SANTAPP_EINVAL, "B, Hkv, N must be >= 1");
    if (num_labels < 1) return fail(SANTAPP_EINVAL, "num_labels must be >= 1");
    if (reps_per_parent < 1) return fail(SANTAPP_EINVAL, "reps_per_parent must be >= 1");
    if (!dtype_ok(dtype)) return fail(SANTAPP_EDTYPE, "unsupported dtype %d", static_cast<int>(dtype));
    if (d != 64 && d != 128) return fail(SANTAPP_ELIMIT, "head dim %d not supported (64 or 128)", d);
    if (num_labels > kMaxLabels) return fail(SANTAPP_ELIMIT, "num_labels %d exceeds %d", num_labels, kMaxLabels);
    if (reps_per_parent > kMaxReps)
        return fail(SANTAPP_ELIMIT, "reps_per_parent %d exceeds %d", reps_per_parent, kMaxReps);
    const size_t BH = static_cast<size_t>(B) * Hkv;
    if (BH * static_cast<size_t>(N) > static_cast<size_t>(0x7fffffff))
        return fail(SANTAPP_ELIMIT, "B*Hkv*N exceeds 2^31");
    hipStream_t s = static_cast<hipStream_t>(stream);
    const size_t esz = elem_size(dtype);
    const size_t row = static_cast<size_t>(d) * esz;
    const int Mp = num_labels;

    // parent lists, then the team counts that size the table; the build's
    // scratch arrays are carved from one allocation
    Carver sc;
    const size_t o_mem = sc.take(BH * N * sizeof(int)), o_pbeg = sc.take(BH * (Mp + 1) * sizeof(int));
    const size_t o_toff = sc.take(BH * (Mp + 1) * sizeof(int)), o_tcount = sc.take(BH * sizeof(int));
    const size_t o_bad = sc.take(sizeof(int)), o_state = sc.take(BH * N * build_state_bytes());
    void* block = nullptr;
    size_t block_bytes = 0;
    hipError_t e = pool().acquire(&block, sc.off, &block_bytes);
    char* const scratch = static_cast<char*>(block);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        return fail(SANTAPP_ENOMEM, "device allocation failed: %s", hipGetErrorString(e));
    }
    auto cleanup = [&]() { pool().release(block, block_bytes); };
    int* members = reinterpret_cast<int*>(scratch + o_mem);
    int* pbeg = reinterpret_cast<int*>(scratch + o_pbeg);
    int* toff = reinterpret_cast<int*>(scratch + o_toff);
    int* tcount = reinterpret_cast<int*>(scratch + o_tcount);
    int* bad = reinterpret_cast<int*>(scratch + o_bad);
    const char* what = "parent lists";
    e = hipMemsetAsync(bad, 0, sizeof(int), s);
    if (e == hipSuccess)
        e = launch_parent_lists(labels, static_cast<int>(BH), N, Mp, reps_per_parent, members, pbeg, toff,
                                tcount, bad, s);
    std::vector<int> counts(BH);
    int flag = 0;
    if (e == hipSuccess) e = hipMemcpyAsync(counts.data(), tcount, BH * sizeof(int), hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipMemcpyAsync(&flag, bad, sizeof(int), hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) {
        cleanup();
        return hip_fail(e, what);
    }
    if (flag) {
        cleanup();
        return fail(SANTAPP_EINVAL, "a label lies outside [0, %d)", Mp);
    }
    const int M = *std::max_element(counts.begin(), counts.end());

    santapp_teams* t = new santapp_teams();
    t->B = B;
    t->Hkv = Hkv;
    t->N = N;
    t->d = d;
    t->dtype = dtype;
    t->P = 0;
    t->R = reps_per_parent;
    t->M = M;
    e = alloc_table(t);
    if (e != hipSuccess) {
        cleanup();
        free_teams(t);
        (void)hipGetLastError();
        return fail(SANTAPP_ENOMEM, "device allocation failed: %s", hipGetErrorString(e));
    }
    what = "team counts";
    e = hipMemcpyAsync(t->team_count, tcount, BH * sizeof(int), hipMemcpyDeviceToDevice, s);
    if (e == hipSuccess) {
        what = "absent teams";
        e = launch_pad_teams(tcount, static_cast<int>(BH), M, N, t->team_begin, t->team_size, t->log_n,
                             t->rep_token, s);
    }
    if (e == hipSuccess) {
        what = "team build";
        e = launch_build_parent_lists(K, dtype, static_cast<int>(BH), N, d, Mp, reps_per_parent, M, members,
                                      pbeg, toff, scratch + o_state, table_arrays(t), s);
    }
    if (e == hipSuccess) {
        what = "packing K";
        e = launch_gather_rows(K, t->packed_K, t->perm, static_cast<int>(BH), N, N, row, s);
    }
    if (e == hipSuccess) {
        what = "packing V";
        e = launch_gather_rows(V, t->packed_V, t->perm, static_cast<int>(BH), N, N, row, s);
    }
    if (e == hipSuccess) {
        what = "gathering representatives";
        e = launch_gather_rows(K, t->reps, t->rep_token, static_cast<int>(BH), M, N, row, s);
    }
    if (e != hipSuccess) {
        cleanup();
        free_teams(t);
        return hip_fail(e, what);
    }
    const santapp_status st = finish_table(t, s, out, []() { return hipErrorUnknown; });  // waits for the build
    if (st == SANTAPP_OK)
        pool().release_idle(block, block_bytes);
    else
        cleanup();
    return st;
}

santapp_status santapp_teams_info(const santapp_teams* t, santapp_teams_desc* d) {
    if (!t || !d) return fail(SANTAPP_EINVAL, "NULL argument");
    d->B = t->B;
    d->Hkv = t->Hkv;
    d->N = t->N;
    d->d = t->d;
    d->dtype = t->dtype;
    d->parent_size = t->P;
    d->reps_per_parent = t->R;
    d->M = t->M;
    d->packed_K = t->packed_K;
    d->packed_V = t->packed_V;
    d->reps = t->reps;
    d->team_begin = t->team_begin;
    d->team_size = t->team_size;
    d->log_n = t->log_n;
    d->rep_token = t->rep_token;
    d->perm = t->perm;
    d->team_count = t->team_count;
    return ok();
}

void santapp_teams_destroy(santapp_teams* t) { free_teams(t); }

santapp_status santapp_trim(void) {
    const hipError_t e = pool().drop_all();
    return e == hipSuccess ? ok() : hip_fail(e, "freeing kept blocks");
}

santapp_status santapp_teams_set_route_keys(santapp_teams* t, santapp_route_key kind, void* stream) {
    if (!t) return fail(SANTAPP_EINVAL, "teams is NULL");
    if (kind != SANTAPP_ROUTE_REPRESENTATIVE && kind != SANTAPP_ROUTE_CENTROID)
        return fail(SANTAPP_EINVAL, "unknown routing key kind %d", static_cast<int>(kind));
    const hipError_t e = launch_route_keys(t->packed_K, t->team_begin, t->team_size, t->rep_token, t->perm,
                                           t->B * t->Hkv, t->N, t->M, t->d, t->dtype,
                                           kind == SANTAPP_ROUTE_CENTROID, t->reps, static_cast<hipStream_t>(stream));
    return e == hipSuccess ? ok() : hip_fail(e, "routing keys");
}

namespace {

// KL workspace: phi [B, Hq, M] and the sums of each stretch of packed rows
// [B, Hq, kl_chunks(N)].
struct KlLayout {
    size_t phi, part, total;
};

KlLayout kl_layout(int B, int Hq, int N, int M) {
    const size_t n = static_cast<size_t>(B) * Hq;
    KlLayout L;
    L.phi = 0;
    L.part = align_up(L.phi + n * M * sizeof(double));
    L.total = align_up(L.part + n * kl_chunks(N) * kl_part_bytes());
    return L;
}

}  // namespace

santapp_status santapp_routing_kl_workspace_bytes(const santapp_teams* t, int Hq, size_t* bytes) {
    if (!t || !bytes) return fail(SANTAPP_EINVAL, "NULL argument");
    if (Hq < 1 || Hq % t->Hkv != 0) return fail(SANTAPP_EINVAL, "Hq must be a positive multiple of Hkv");
    *bytes = kl_layout(t->B, Hq, t->N, t->M).total;
    return ok();
}

santapp_status santapp_routing_kl(const santapp_teams* t, const float* q, int Hq, double scale, double* kl,
                                  void* workspace, size_t ws_bytes, void* stream) {
    if (!t) return fail(SANTAPP_EINVAL, "teams is NULL");
    if (!q || !kl) return fail(SANTAPP_EINVAL, "q and kl must be device pointers");
    if (Hq < 1 || Hq % t->Hkv != 0) return fail(SANTAPP_EINVAL, "Hq (%d) must be a positive multiple of Hkv (%d)", Hq, t->Hkv);
    if (Hq / t->Hkv > kMaxGroup) return fail(SANTAPP_ELIMIT, "%d query heads per KV head exceed %d", Hq / t->Hkv, kMaxGroup);
    if (!(scale >= 0.0) || !isfinite(scale)) return fail(SANTAPP_EINVAL, "scale must be finite and >= 0");
    if (scale == 0.0) scale = 1.0 / sqrt(static_cast<double>(t->d));
    const KlLayout L = kl_layout(t->B, Hq, t->N, t->M);
    if (!workspace || ws_bytes < L.total)
        return fail(SANTAPP_EWORKSPACE, "workspace of %zu bytes needed (got %zu)", L.total, ws_bytes);
    if (!aligned16(q) || !aligned16(kl) || !aligned16(workspace))
        return fail(SANTAPP_EINVAL, "q, kl and workspace must be 16-byte aligned");
    hipStream_t s = static_cast<hipStream_t>(stream);
    char* ws = static_cast<char*>(workspace);
    double* phi = reinterpret_cast<double*>(ws + L.phi);
    RouteArgs R{};
    R.reps = t->reps;
    R.log_n = t->log_n;
    R.q = q;
    R.B = t->B;
    R.Hkv = t->Hkv;
    R.Hq = Hq;
    R.G = Hq / t->Hkv;
    R.d = t->d;
    R.M = t->M;
    R.dtype = t->dtype;
    R.scale = scale;
    hipError_t e = launch_route_phi(R, phi, s);
    if (e != hipSuccess) return hip_fail(e, "routing kernel");
    KlArgs A{};
    A.packed_K = t->packed_K;
    A.team_begin = t->team_begin;
    A.log_n = t->log_n;
    A.q = q;
    A.phi = phi;
    A.part = ws + L.part;
    A.kl = kl;
    A.B = t->B;
    A.Hkv = t->Hkv;
    A.Hq = Hq;
    A.N = t->N;
    A.M = t->M;
    A.d = t->d;
    A.dtype = t->dtype;
    A.scale = scale;
    e = launch_routing_kl(A, s);
    return e == hipSuccess ? ok() : hip_fail(e, "KL kernels");
}

santapp_status santapp_workspace_zero(void* ws, size_t bytes, void* stream) {
    if (bytes == 0) return ok();
    if (!ws) return fail(SANTAPP_EINVAL, "workspace is NULL");
    const hipError_t e = launch_zero(ws, bytes, static_cast<hipStream_t>(stream));
    return e == hipSuccess ? ok() : hip_fail(e, "workspace zero");
}

santapp_status santapp_decode_workspace_bytes(const santapp_teams* t, int Hq, int T, int K,
                                              size_t* bytes) {
    if (!t || !bytes) return fail(SANTAPP_EINVAL, "NULL argument");
    if (Hq < 1 || Hq % t->Hkv != 0) return fail(SANTAPP_EINVAL, "Hq must be a positive multiple of Hkv");
    if (T < 0 || K < 1) return fail(SANTAPP_EINVAL, "T must be >= 0 and K >= 1");
    const int Kp = std::min(K, t->M);
    *bytes = Kp == t->M ? dense_layout(t->B, Hq, t->Hkv, t->N, T, t->d, t->cus, t->dtype).total
                        : decode_layout(t->B, Hq, t->Hkv, T, t->d, t->M, Kp, t->cap.data(), t->cus, t->dtype).total;
    return ok();
}

santapp_status santapp_decode_launch_info(const santapp_teams* t, int Hq, int T, int K, int* kernels,
                                         int* workgroups) {
    if (!t || !kernels || !workgroups) return fail(SANTAPP_EINVAL, "NULL argument");
    if (Hq < 1 || Hq % t->Hkv != 0) return fail(SANTAPP_EINVAL, "Hq must be a positive multiple of Hkv");
    if (T < 0 || K < 1) return fail(SANTAPP_EINVAL, "T must be >= 0 and K >= 1");
    const int Kp = std::min(K, t->M);
    const bool dense = Kp == t->M;
    const StepLayout L = dense ? dense_layout(t->B, Hq, t->Hkv, t->N, T, t->d, t->cus, t->dtype)
                               : decode_layout(t->B, Hq, t->Hkv, T, t->d, t->M, Kp, t->cap.data(), t->cus,
                                               t->dtype);
    const bool fused = fused_step(t->dtype, L);
    *kernels = L.step || fused ? 1 : (dense ? 2 : 3);
    *workgroups = L.nwg;
    return ok();
}

santapp_status santapp_dense_workspace_bytes(int B, int Hq, int Hkv, int N, int T, int d,
                                             size_t* bytes) {
    if (!bytes) return fail(SANTAPP_EINVAL, "NULL argument");
    if (B < 1 || Hkv < 1 || Hq < 1 || Hq % Hkv != 0 || N < 0 || T < 0 || N + T < 1 || d < 1)
        return fail(SANTAPP_EINVAL, "invalid sizes");
    // the larger of the two element types' layouts (the call's type is not an argument)
    const int cus = device_cus();
    *bytes = std::max(dense_layout(B, Hq, Hkv, N, T, d, cus, SANTAPP_BF16).total,
                      dense_layout(B, Hq, Hkv, N, T, d, cus, SANTAPP_FP32).total);
    return ok();
}

namespace {

santapp_status check_suffix(const void* sK, const void* sV, int T, int& stride) {
    if (T < 0) return fail(SANTAPP_EINVAL, "T must be >= 0");
    if (stride == 0) stride = T;
    if (stride < T) return fail(SANTAPP_EINVAL, "suffix_stride (%d) is smaller than T (%d)", stride, T);
    if (T > 0 && (!sK || !sV)) return fail(SANTAPP_EINVAL, "suffix K/V are NULL with T > 0");
    if (T > 0 && (!aligned16(sK) || !aligned16(sV))) return fail(SANTAPP_EINVAL, "suffix K/V must be 16-byte aligned");
    return SANTAPP_OK;
}

}  // namespace

santapp_status santapp_decode(const santapp_teams* t, const float* q, const void* suffix_K,
                              const void* suffix_V, int T, int suffix_stride, int Hq, int K, uint64_t seed,
                              uint64_t step, double scale, float* out, void* workspace,
                              size_t ws_bytes, const santapp_decode_debug* dbg, void* stream) {
    if (!t) return fail(SANTAPP_EINVAL, "teams is NULL");
    if (!q || !out) return fail(SANTAPP_EINVAL, "q and out must be device pointers");
    if (Hq < 1 || Hq % t->Hkv != 0) return fail(SANTAPP_EINVAL, "Hq (%d) must be a positive multiple of Hkv (%d)", Hq, t->Hkv);
    const int G = Hq / t->Hkv;
    if (G > kMaxGroup) return fail(SANTAPP_ELIMIT, "%d query heads per KV head exceed %d", G, kMaxGroup);
    if (santapp_status st = check_suffix(suffix_K, suffix_V, T, suffix_stride)) return st;
    if (!aligned16(q) || !aligned16(out) || !aligned16(workspace))
        return fail(SANTAPP_EINVAL, "q, out and workspace must be 16-byte aligned");
    if (K < 1) return fail(SANTAPP_EINVAL, "K must be >= 1 (got %d)", K);
    if (!(scale >= 0.0) || !isfinite(scale)) return fail(SANTAPP_EINVAL, "scale must be finite and >= 0");
    if (scale == 0.0) scale = 1.0 / sqrt(static_cast<double>(t->d));
    const int Kp = std::min(K, t->M);
    const bool dense = Kp == t->M;
    if (!dense && t->M > kMaxTeams) return fail(SANTAPP_ELIMIT, "%d teams per KV head exceed %d", t->M, kMaxTeams);
    const StepLayout L = dense ? dense_layout(t->B, Hq, t->Hkv, t->N, T, t->d, t->cus, t->dtype)
                               : decode_layout(t->B, Hq, t->Hkv, T, t->d, t->M, Kp, t->cap.data(), t->cus,
                                               t->dtype, ws_bytes);
    if (!workspace || ws_bytes < L.total)
        return fail(SANTAPP_EWORKSPACE, "workspace of %zu bytes needed (got %zu)", L.total, ws_bytes);
    hipStream_t s = static_cast<hipStream_t>(stream);

    DecodeArgs A{};
    A.reps = t->reps;
    A.log_n = t->log_n;
    A.team_begin = t->team_begin;
    A.team_size = t->team_size;
    A.K = t->packed_K;
    A.V = t->packed_V;
    A.sK = suffix_K;
    A.sV = suffix_V;
    A.q = q;
    A.out = out;
    A.B = t->B;
    A.Hkv = t->Hkv;
    A.Hq = Hq;
    A.G = G;
    A.d = t->d;
    A.N = t->N;
    A.T = T;
    A.sstride = suffix_stride;
    A.M = t->M;
    A.Kp = Kp;
    A.dtype = t->dtype;
    A.dense = dense;
    A.scale = scale;
    A.scale_log2 = static_cast<float>(scale * 1.4426950408889634);
    A.seed = seed;
    A.step = step;
    if (L.keys) A.token = call_token();
    A.lay = L;
    A.key = L.key;
    A.ws = static_cast<char*>(workspace);
    if (dbg) {
        A.dbg_phi = dbg->phi;
        A.dbg_Y = dbg->Y;
        A.dbg_sel = dbg->sel;
        A.dbg_logc = dbg->logc;
        A.dbg_tau = dbg->tau;
        A.dbg_uteams = dbg->union_teams;
        A.dbg_urows = dbg->union_rows;
        // events 1 and 2 are stamped by the attention launch itself, at the
        // kernel's start and end
        A.ev_start = static_cast<hipEvent_t>(dbg->events[1]);
        A.ev_stop = static_cast<hipEvent_t>(dbg->events[2]);
    }
    A.fused = fused_step(t->dtype, L);

    hipError_t e;
    auto mark = [&](int i) -> hipError_t {
        if (dbg && dbg->events[i]) return hipEventRecord(static_cast<hipEvent_t>(dbg->events[i]), s);
        return hipSuccess;
    };
    if ((e = mark(0)) != hipSuccess) return hip_fail(e, "event record");
    if ((e = launch_decode(A, s)) != hipSuccess) return hip_fail(e, "decode kernels");
    if ((e = mark(3)) != hipSuccess) return hip_fail(e, "event record");
    return ok();
}

// ---------------------------------------------------------------------------
// santapp_decode_static: santapp_decode over a scratch buffer the library
// owns, a file-scope device array of kStaticScratchBytes that every GPU the
// library runs on holds until the process ends.  Its device address is taken
// once per device (with that device current) and used for every launch; its
// first use on a device clears it with the fill kernel (the counters must
// start at zero; every completed call leaves them at zero).
// ---------------------------------------------------------------------------
namespace {

constexpr size_t kStaticScratchBytes = size_t(4) << 20;
constexpr int kMaxDevices = 64;

static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

struct ScratchSlot {
    void* ptr = nullptr;  // device address of `scratch` on this device
    bool cleared = false;
};
static ScratchSlot g_scratch[kMaxDevices];
static std::mutex g_scratch_mu;

static santapp_status static_scratch(hipStream_t s, void** out) {
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
    if (dev < 0 || dev >= kMaxDevices) return fail(SANTAPP_ELIMIT, "device %d beyond the %d devices supported", dev, kMaxDevices);
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    ScratchSlot& sl = g_scratch[dev];
    if (!sl.ptr) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p) return hip_fail(e != hipSuccess ? e : hipErrorInvalidSymbol, "hipGetSymbolAddress(scratch)");
        sl.ptr = p;
    }
    if (!sl.cleared) {
        e = launch_zero(sl.ptr, kStaticScratchBytes, s);
        if (e != hipSuccess) return hip_fail(e, "static scratch clear");
        sl.cleared = true;
    }
    *out = sl.ptr;
    return SANTAPP_OK;
}

}  // namespace

santapp_status santapp_decode_static(const santapp_teams* t, const float* q, const void* suffix_K,
                                     const void* suffix_V, int T, int suffix_stride, int Hq, int K,
                                     uint64_t seed, uint64_t step, double scale, float* out,
                                     const santapp_decode_debug* dbg, void* stream) {
    if (!t) return fail(SANTAPP_EINVAL, "teams is NULL");
    size_t need = 0;
    if (santapp_status st = santapp_decode_workspace_bytes(t, Hq, T, K, &need)) return st;
    if (need > kStaticScratchBytes && K < t->M)  // the least that a sampled step takes
        need = decode_layout(t->B, Hq, t->Hkv, T, t->d, t->M, K, t->cap.data(), t->cus, t->dtype, kStaticScratchBytes).total;
    if (need > kStaticScratchBytes)
        return fail(SANTAPP_ELIMIT, "this step needs %zu bytes of scratch; the static scratch holds %zu "
                    "(use santapp_decode with a workspace)", need, kStaticScratchBytes);
    void* ws = nullptr;
    if (santapp_status st = static_scratch(static_cast<hipStream_t>(stream), &ws)) return st;
    return santapp_decode(t, q, suffix_K, suffix_V, T, suffix_stride, Hq, K, seed, step, scale, out, ws,
                          kStaticScratchBytes, dbg, stream);
}

santapp_status santapp_dense_decode(const float* q, const void* K, const void* V, int B, int Hkv,
                                    int N, int d, santapp_dtype dtype, const void* suffix_K,
                                    const void* suffix_V, int T, int suffix_stride, int Hq, double scale,
                                    float* out, void* workspace, size_t ws_bytes,
                                    const santapp_decode_debug* dbg, void* stream) {
    if (!q || !out) return fail(SANTAPP_EINVAL, "q and out must be device pointers");
    if (B < 1 || Hkv < 1 || N < 0 || T < 0 || N + T < 1)
        return fail(SANTAPP_EINVAL, "invalid sizes");
    if (N > 0 && (!K || !V)) return fail(SANTAPP_EINVAL, "K and V are NULL with N > 0");
    if (santapp_status st = check_suffix(suffix_K, suffix_V, T, suffix_stride)) return st;
    if (!aligned16(q) || !aligned16(out) || !aligned16(workspace) || (N > 0 && (!aligned16(K) || !aligned16(V))))
        return fail(SANTAPP_EINVAL, "q, out, K/V and workspace must be 16-byte aligned");
    if (Hq < 1 || Hq % Hkv != 0) return fail(SANTAPP_EINVAL, "Hq must be a positive multiple of Hkv");
    if (Hq / Hkv > kMaxGroup) return fail(SANTAPP_ELIMIT, "more than %d query heads per KV head", kMaxGroup);
    if (!dtype_ok(dtype)) return fail(SANTAPP_EDTYPE, "unsupported dtype %d", static_cast<int>(dtype));
    if (d != 64 && d != 128) return fail(SANTAPP_ELIMIT, "head dim %d not supported (64 or 128)", d);
    if (!(scale >= 0.0) || !isfinite(scale)) return fail(SANTAPP_EINVAL, "scale must be finite and >= 0");
    if (scale == 0.0) scale = 1.0 / sqrt(static_cast<double>(d));
    const StepLayout L = dense_layout(B, Hq, Hkv, N, T, d, device_cus(), dtype);
    if (!workspace || ws_bytes < L.total)
        return fail(SANTAPP_EWORKSPACE, "workspace of %zu bytes needed (got %zu)", L.total, ws_bytes);
    DecodeArgs A{};
    A.K = K;
    A.V = V;
    A.sK = suffix_K;
    A.sV = suffix_V;
    A.q = q;
    A.out = out;
    A.B = B;
    A.Hkv = Hkv;
    A.Hq = Hq;
    A.G = Hq / Hkv;
    A.d = d;
    A.N = N;
    A.T = T;
    A.sstride = suffix_stride;
    A.M = 0;
    A.Kp = 0;
    A.dtype = dtype;
    A.dense = true;
    A.scale = scale;
    A.scale_log2 = static_cast<float>(scale * 1.4426950408889634);
    A.lay = L;
    A.key = L.key;
    A.ws = static_cast<char*>(workspace);
    A.fused = fused_step(dtype, L);
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (dbg) {  // the stage events only
        A.ev_start = static_cast<hipEvent_t>(dbg->events[1]);
        A.ev_stop = static_cast<hipEvent_t>(dbg->events[2]);
    }
    auto mark = [&](int i) -> hipError_t {
        if (dbg && dbg->events[i]) return hipEventRecord(static_cast<hipEvent_t>(dbg->events[i]), s);
        return hipSuccess;
    };
    hipError_t e;
    if ((e = mark(0)) != hipSuccess) return hip_fail(e, "event record");
    if ((e = launch_decode(A, s)) != hipSuccess) return hip_fail(e, "dense decode kernels");
    if ((e = mark(3)) != hipSuccess) return hip_fail(e, "event record");
    return ok();
}

}  // extern "C"
