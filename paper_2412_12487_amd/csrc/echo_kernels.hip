// echo_kernels.hip -- gfx950 kernels of the timeline composer.
//
//   k_init     clear barrier state and outputs, check scenario ranges
//   k_clear    clear barrier state between passes
//   k_cc_cost  CC estimator (Sec. 5.3, Eq. 2-5): one lane per (collective or cost class, scenario)
//   k_sum      what-if durations: per segment and scenario, the sum of its ops' jittered
//              base durations (first pass)
//   k_walk     timeline composer (Sec. 4.2) with the collective synchronisation
//              rule (Sec. 5.2): one wavefront per (walker, 64-scenario tile) walks
//              the segments and comm ops of its ranks in level order, max-plus
//              relaxation in registers
//   k_overlap  validator input (Sec. 6): per compute op and scenario, the mask of
//              collective types among the comm ops of its rank that overlap it, and the
//              segments' new durations
//   k_expand   the ops' starts and finishes (and their digest) from the segments' starts
//
// Everything is int64 nanoseconds and Q16 factors, bit-exact by construction:
// max, add, 64-bit multiply and shifts only (no floating point on the path).
#include <algorithm>
#include <mutex>
#include <type_traits>

#include "echo_internal.h"

namespace echo {
namespace {

constexpr uint64_t kGolden = 0x9E3779B97F4A7C15ull;  // SplitMix64 increment
constexpr uint64_t kMixA = 0xBF58476D1CE4E5B9ull;    // SplitMix64 output function
constexpr uint64_t kMixB = 0x94D049BB133111EBull;
constexpr int64_t kKnobLimit = int64_t(1) << 40;
constexpr int64_t kInf = INT64_MAX;
// s_waitcnt immediate for "vmcnt(0)" on gfx9-family targets (expcnt and lgkmcnt left at their maxima)
constexpr int kWaitVm0 = 0x0F70;
// polls between reads of the abort bit and the clock: of a barrier in device memory (a
// poll is a memory round trip) and of one in LDS
constexpr unsigned kCheckPollsGlobal = 16;
constexpr unsigned kCheckPollsLocal = 256;

__device__ __forceinline__ uint64_t mix64(uint64_t z) {
    z = (z ^ (z >> 30)) * kMixA;
    z = (z ^ (z >> 27)) * kMixB;
    return z ^ (z >> 31);
}

// (d * f + 2^15) >> 16 in unsigned 64-bit: d < 2^44 and f < 2^20 never wrap.
__device__ __forceinline__ int64_t q16(int64_t d, uint32_t f) {
    return int64_t(((uint64_t)d * (uint64_t)f + 32768ull) >> 16);
}

// Base duration with uniform jitter of amplitude amp (Q16) from the k-th
// SplitMix64 output of the scenario's seed, k = jstream * 2^36 + v + 1.  The
// SplitMix64 state seed + k * golden is split into a per-scenario part
// (base = seed + jstream * 2^36 * golden) and a per-op part ((v + 1) * golden,
// the same for every lane).  The factor is f = 65536 - amp + J with J the high word
// of the output scaled to [0, 2 amp]; the lane's constants 65536 - amp and 2 amp + 1
// are taken once.
struct Jitter {
    uint64_t base;
    uint32_t f0;      // 65536 - amp
    uint32_t span;    // 2 amp + 1
};
__device__ __forceinline__ Jitter make_jitter(uint64_t seed, uint32_t jstream, int32_t amp) {
    return Jitter{seed + ((uint64_t)jstream << 36) * kGolden, (uint32_t)(65536 - amp), (uint32_t)(2 * amp + 1)};
}
__device__ __forceinline__ uint32_t jitter_factor(int32_t v, const Jitter &jt) {
    // (v + 1) * golden is the same for every lane: two scalar multiplies (kept opaque so the
    // compiler does not fold them into a vector multiply-add with the lane's base)
    const uint32_t k = (uint32_t)v + 1u;
    uint32_t lo, hi;
    asm("s_mul_i32 %0, %1, %2" : "=s"(lo) : "s"(k), "s"((uint32_t)kGolden));
    asm("s_mul_hi_u32 %0, %1, %2" : "=s"(hi) : "s"(k), "s"((uint32_t)kGolden));
    hi += k * (uint32_t)(kGolden >> 32);
    const uint64_t u = mix64(jt.base + (((uint64_t)hi << 32) | lo));
    return jt.f0 + __umulhi((uint32_t)(u >> 32), jt.span);
}
// q16(d0, f) for a wave-uniform d0: below 2^32 (durations under 4.3 s) one 32 x 32-bit
// multiply-add gives the whole product.  The branch is explicit: left to itself the
// compiler evaluates the general two-multiply form for every d0.
__device__ __forceinline__ int64_t q16u(int64_t d0, uint32_t f) {
    const uint32_t dh = (uint32_t)((uint64_t)d0 >> 32);
    uint64_t p = (uint64_t)(uint32_t)d0 * f + 32768ull;
    if (__builtin_expect(__builtin_amdgcn_readfirstlane(dh) != 0, 0)) {
        uint32_t hp;
        asm volatile("v_mul_lo_u32 %0, %1, %2" : "=v"(hp) : "s"(dh), "v"(f));
        p += (uint64_t)hp << 32;
    }
    return (int64_t)(p >> 16);
}
__device__ __forceinline__ int64_t jittered(int64_t d0, int32_t v, const Jitter &jt) {
    return q16u(d0, jitter_factor(v, jt));
}
// the same for a base duration known to be below 2^32 ns
__device__ __forceinline__ int64_t jittered32(uint32_t d0, int32_t v, const Jitter &jt) {
    return (int64_t)(((uint64_t)d0 * jitter_factor(v, jt) + 32768ull) >> 16);
}

__device__ __forceinline__ int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }

__device__ __forceinline__ int64_t clog2(int64_t x) {
    int64_t k = 0;
    while ((int64_t(1) << k) < x) ++k;
    return k;
}

__device__ __forceinline__ unsigned ld_relaxed(const unsigned *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// ------------------------------------------------------------------ set-up
__global__ void k_init(const echo_scenario *scen, int32_t n_scen, unsigned long long *arrive,
                       int64_t n_arrive, unsigned *count, int64_t n_count, int64_t *slots, int64_t n_slots,
                       int64_t *step, uint64_t *digest, int32_t n_tables, unsigned *status) {
    const int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t nth = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = tid; i < n_arrive; i += nth) arrive[i] = 0;
    for (int64_t i = tid; i < n_count; i += nth) count[i] = 0;
    for (int64_t i = tid; i < n_slots; i += nth) slots[i] = -1;
    for (int64_t i = tid; i < n_scen; i += nth) {
        if (step) step[i] = 0;
        if (digest) digest[i] = 0;
        const echo_scenario &s = scen[i];
        bool ok = s.alpha_ns >= 0 && s.alpha_ns < kKnobLimit && s.bw_intra_MBps >= 1 &&
                  s.bw_intra_MBps < kKnobLimit && s.bw_inter_MBps >= 1 &&
                  s.bw_inter_MBps < kKnobLimit && s.reduce_MBps >= 1 &&
                  s.reduce_MBps < kKnobLimit && s.jitter_amp_q16 >= 0 &&
                  s.jitter_amp_q16 <= 65535 && s.ar_algo <= ECHO_TREE && s.cc_model <= ECHO_CC_ALPHA_BETA &&
                  s.cc_table >= 0 && s.cc_table <= n_tables;
        for (int k = 0; k < kClasses; ++k)
            for (int t = 0; t < kTypes; ++t) {
                const uint32_t f = s.slowdown_q16[k][t];
                ok = ok && f >= 65536u && f < (1u << 20);
            }
        if (!ok) __hip_atomic_fetch_or(status, kStatusRange, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

__global__ void k_clear(unsigned long long *arrive, int64_t n_arrive, unsigned *count, int64_t n_count,
                        int64_t *slots, int64_t n_slots) {
    const int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t nth = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = tid; i < n_arrive; i += nth) arrive[i] = 0;
    for (int64_t i = tid; i < n_count; i += nth) count[i] = 0;
    for (int64_t i = tid; i < n_slots; i += nth) slots[i] = -1;
}

// ------------------------------------------------------------------ CC estimator
// One block per collective or cost class; lanes stride over scenarios.  Row of c: t.row[c], or c.
__global__ __launch_bounds__(64) void k_cc_cost(CollTable t, const echo_cc_table *tables, const echo_scenario *scen,
                                                int32_t n_scen, int64_t *cost, unsigned *status) {
    const int64_t c = blockIdx.x;
    const int64_t row = t.row ? t.row[c] : c;
    const int type = t.type[c];
    const int64_t S = t.bytes[c];
    const int64_t N = t.N[c], M = t.M[c], K = t.K[c];
    const unsigned __int128 n1 = (unsigned __int128)(N - 1);
    for (int64_t s = (int64_t)blockIdx.y * blockDim.x + threadIdx.x; s < n_scen; s += (int64_t)gridDim.y * blockDim.x) {
        const echo_scenario &sc = scen[s];
        // invalid knobs are reported by k_init; keep the divisions defined
        const int64_t bwa = sc.bw_intra_MBps >= 1 ? sc.bw_intra_MBps : 1;
        const int64_t bwe = sc.bw_inter_MBps >= 1 ? sc.bw_inter_MBps : 1;
        const int64_t red = sc.reduce_MBps >= 1 ? sc.reduce_MBps : 1;
        unsigned __int128 alpha = (unsigned __int128)(sc.alpha_ns >= 0 ? sc.alpha_ns : 0);
        unsigned __int128 T;
        if (sc.cc_model == ECHO_CC_ALPHA_BETA) {
            // latency-bandwidth baseline: ring steps move ceil(S / N) bytes, tree steps all of S
            const int64_t B = M > 1 ? bwe : bwa;
            const int64_t part = cdiv(S, N);
            const unsigned __int128 tbp = (unsigned __int128)cdiv(part * 1000, B);
            const unsigned __int128 trp = (unsigned __int128)cdiv(part * 1000, red);
            if (type == ECHO_AG) {
                T = n1 * (alpha + tbp);
            } else if (type == ECHO_RS) {
                T = n1 * (alpha + tbp + trp);
            } else if (type == ECHO_AR) {
                if (sc.ar_algo == ECHO_TREE)
                    T = (unsigned __int128)clog2(N) * (2 * alpha + 2 * (unsigned __int128)cdiv(S * 1000, B) +
                                                       (unsigned __int128)cdiv(S * 1000, red));
                else
                    T = n1 * (2 * alpha + 2 * tbp + trp);
            } else {
                T = alpha + (unsigned __int128)cdiv(S * 1000, B);
            }
        } else {
            int64_t chunk, eta_r, eta_t, b, g, r;
            if (sc.cc_table > 0 && tables) {
                // profiled parameters: the first row whose size bound covers S
                const echo_cc_table &tb = tables[sc.cc_table - 1];
                int i = 0;
                while (i < ECHO_CC_ROWS - 1 && S > tb.max_bytes[i]) ++i;
                chunk = tb.chunk[i] >= 1 ? tb.chunk[i] : 1;
                eta_r = cdiv(S, N * chunk);
                eta_t = cdiv(S, chunk);
                alpha = (unsigned __int128)tb.alpha_ns[i];
                b = tb.beta_ns[i];
                g = tb.gamma_ns[i];
                r = tb.reduce_MBps[i] >= 1 ? tb.reduce_MBps[i] : 1;
            } else {
                chunk = t.chunk[c];
                eta_r = t.eta_ring[c];
                eta_t = t.eta_chunks[c];
                b = cdiv(chunk * 1000, bwa);
                g = cdiv(chunk * 1000, bwe);
                r = red;
            }
            const unsigned __int128 eta_ring = (unsigned __int128)eta_r, eta_chunks = (unsigned __int128)eta_t;
            const unsigned __int128 beta = (unsigned __int128)b;
            const unsigned __int128 hop = M > 1 ? (unsigned __int128)g : beta;
            const unsigned __int128 reduce = (unsigned __int128)cdiv(S * 1000, r);
            if (type == ECHO_AG) {
                T = alpha + hop * eta_ring * n1;                                    // Eq. 2
            } else if (type == ECHO_RS) {
                T = alpha + eta_ring * (n1 * beta + n1 * hop) + reduce;             // Eq. 3
            } else if (type == ECHO_AR) {
                if (sc.ar_algo == ECHO_TREE)                                        // Eq. 5
                    T = alpha + hop * (eta_chunks > 0 ? eta_chunks - 1 : 0) +
                        2 * beta * (unsigned __int128)(K - 1) +
                        2 * hop * (unsigned __int128)clog2(M) + reduce;
                else                                                                // Eq. 4
                    T = alpha + eta_ring * (n1 * beta + 2 * n1 * hop) + reduce;
            } else {                                                                // P2P
                T = alpha + eta_chunks * hop;
            }
        }
        if (T >= (unsigned __int128)kTimeLimit) {
            __hip_atomic_fetch_or(status, kStatusOverflow, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            T = (unsigned __int128)(kTimeLimit - 1);
        }
        cost[row * n_scen + s] = (int64_t)T;
    }
}

// Cost of every collective: its class's, from the row of the class's first collective.  The
// 64-bit divisions and 128-bit products of the model (about a thousand instructions per
// class and scenario) then run once per class; what is left is bound by the stores (23,808
// collectives of 19 classes x 4000 scenarios, 762 MB: 1.88 ms per call when every collective
// was costed by itself, 0.16 now).  T: two scenarios per store where rows are 16-byte aligned.
template <class T>
__global__ __launch_bounds__(256) void k_cc_spread(const int32_t *class_of, const int32_t *row, int64_t n,
                                                   int32_t per_row, T *cost) {
    const int lane = threadIdx.x & 63;
    const int64_t step = (int64_t)gridDim.x * 4;
    for (int64_t c = (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); c < n; c += step) {
        const int64_t from = __builtin_amdgcn_readfirstlane(row[class_of[c]]);
        if (from == c) continue;
        const T *const src = cost + from * per_row;
        T *const dst = cost + c * per_row;
#pragma unroll 4
        for (int32_t i = lane; i < per_row; i += 64) dst[i] = src[i];
    }
}

// ------------------------------------------------------------------ composer
// Bounded waits.  A wait polls; every kCheckPollsGlobal-th poll of device memory (every
// kCheckPollsLocal-th of LDS) it also reads the abort bit and the 100 MHz wall clock, which
// it first reads at that poll (a clock read on the way into a wait would delay the first
// polls, and a wait is usually over within a few).  It gives up -- and tells every other
// waiter to give up -- once spin_limit ticks have passed since then.
struct WaitClock {
    uint64_t t0 = 0;
    bool started = false;
    // false: give up (abort seen, or the limit passed: then the abort bit is set)
    __device__ bool check(unsigned *status, int64_t limit) {
        if (__builtin_amdgcn_readfirstlane(ld_relaxed(status)) & kStatusAbort) return false;
        const uint64_t now = wall_clock64();
        if (!started) {
            started = true;
            t0 = now;
        } else if ((int64_t)(now - t0) > limit) {
            __hip_atomic_fetch_or(status, kStatusTimeout | kStatusAbort, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            return false;
        }
        return true;
    }
};

// Wait until `need` member wavefronts of one scenario tile have published
// their launch times.
__device__ bool wait_arrivals(const unsigned *cnt, unsigned need, unsigned *status, int64_t limit) {
    // Issue priority on the SIMD follows lateness: the last member to arrive is what the
    // others wait for, so it runs at raised priority until it next arrives early.
    if (__builtin_amdgcn_readfirstlane(ld_relaxed(cnt)) >= need) {
        __builtin_amdgcn_s_setprio(3);
        return true;
    }
    __builtin_amdgcn_s_setprio(0);
    WaitClock clk;
    for (unsigned it = 1;; ++it) {
        __builtin_amdgcn_s_sleep(2);
        if (__builtin_amdgcn_readfirstlane(ld_relaxed(cnt)) >= need) return true;
        if ((it & (kCheckPollsGlobal - 1)) == 0 && !clk.check(status, limit)) return false;
    }
}

// Barrier of a collective met through member slots: the latest launch time over
// its n members' slots p[m * ns] (m < n <= MOST), once every member of every
// lane's scenario has stored its launch (a slot reads -1 until then).  All slots are
// read in one memory round trip per poll.  Bounded like wait_arrivals; on giving up
// it returns 0 and clears *ok.
template <int MOST>
__device__ int64_t wait_slots(const int64_t *p, unsigned n, int64_t ns, unsigned *status, int64_t limit, bool *ok) {
    WaitClock clk;
    for (unsigned poll = 0;; ++poll) {
        int64_t v[MOST];
#pragma unroll
        for (int m = 0; m < MOST; ++m)
            v[m] = m < (int)n ? __hip_atomic_load(p + m * ns, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
        int64_t mx = 0;
        bool all = true;
#pragma unroll
        for (int m = 0; m < MOST; ++m) {
            all = all && v[m] >= 0;
            mx = v[m] > mx ? v[m] : mx;
        }
        if (!__builtin_amdgcn_readfirstlane(__ballot(!all) != 0)) {
            // every member had launched at the first look (poll 0): this wave was the last to
            // arrive and the others wait for it (issue priority as in wait_arrivals)
            if (poll == 0) __builtin_amdgcn_s_setprio(3);
            return mx;
        }
        if (poll == 0) __builtin_amdgcn_s_setprio(0);
        __builtin_amdgcn_s_sleep(2);
        if (((poll + 1) & (kCheckPollsGlobal - 1)) == 0 && !clk.check(status, limit)) break;
    }
    *ok = false;
    return 0;
}

typedef __attribute__((address_space(1))) int64_t GlobalI64;     // global, not flat, when made from an integer
// The sweep's stores go through the cache: overlap detection and k_expand read the rows again,
// and a later poll of the same wavefront waits for them.
__device__ __forceinline__ void put(GlobalI64 *p, int64_t v) { *p = v; }
// The other timeline stores are read by nothing here, or only by far predecessors.
__device__ __forceinline__ void put_stream(GlobalI64 *p, int64_t v) {
    __builtin_nontemporal_store(v, p);
}

// Duration d inflated by the slowdown factor of overlap mask m (Sec. 6): the largest entry
// of the op's class row x over the collective types in m; an empty mask keeps factor 65536,
// which q16 maps to d itself.  Entry t takes part through an AND with bit t of m widened to
// a whole word (all ones or zero), and the largest is taken three at a time.
__device__ __forceinline__ int64_t inflate_row(int64_t d, uint32_t m, uint4 x) {
    static_assert(kTypes == 4, "two three-way maxima cover 65536 and four entries");
    const uint32_t a0 = x.x & (uint32_t)__builtin_amdgcn_sbfe((int)m, 0, 1);
    const uint32_t a1 = x.y & (uint32_t)__builtin_amdgcn_sbfe((int)m, 1, 1);
    const uint32_t a2 = x.z & (uint32_t)__builtin_amdgcn_sbfe((int)m, 2, 1);
    const uint32_t a3 = x.w & (uint32_t)__builtin_amdgcn_sbfe((int)m, 3, 1);
    const uint32_t F0 = a0 > 65536u ? a0 : 65536u;
    const uint32_t F1 = F0 > a1 ? F0 : a1;
    const uint32_t F2 = a2 > a3 ? a2 : a3;
    return q16(d, F1 > F2 ? F1 : F2);
}
// Arrive at an LDS barrier with launch time v: raises the lanes' latest launch, then counts.
// A wavefront's LDS operations are performed in order, so whoever sees the count sees the
// launch; nothing is waited for.
__device__ __forceinline__ void arrive_local(unsigned long long *bar, unsigned *cnt, int64_t v, int lane) {
    __hip_atomic_fetch_max(&bar[lane], (unsigned long long)v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    asm volatile("" ::: "memory");                 // keep the compiler's order as well
    if (lane == 0) __hip_atomic_fetch_add(cnt, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Wait until `need` members have arrived at an LDS barrier; *b gets the lane's latest launch,
// read behind the count in each poll (in order, so it is whole when the count is).
__device__ bool wait_local(const unsigned *cnt, unsigned need, const unsigned long long *bar, int lane, uint64_t *b,
                           unsigned *status, int64_t limit) {
    auto look = [&]() -> unsigned {
        const unsigned c = __hip_atomic_load(cnt, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        asm volatile("" ::: "memory");             // keep the compiler's order as well
        *b = __hip_atomic_load(&bar[lane], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        return __builtin_amdgcn_readfirstlane(c);
    };
    if (look() >= need) {
        __builtin_amdgcn_s_setprio(3);             // last to arrive: see wait_arrivals
        return true;
    }
    __builtin_amdgcn_s_setprio(0);
    WaitClock clk;
    for (unsigned it = 1;; ++it) {
        __builtin_amdgcn_s_sleep(1);
        if (look() >= need) return true;
        if ((it & (kCheckPollsLocal - 1)) == 0 && !clk.check(status, limit)) return false;
    }
}

// The scenario knobs a lane needs to draw durations, and what it reads and writes: lane l of a
// tile's wavefront is scenario tile * 64 + l.  Idle lanes of the last tile mirror its last
// scenario: they compute the same values and store them to the same places; only active
// lanes issue global atomics.
struct Lane {
    int32_t col, sigma;      // column within the tile, scenario
    bool active;
    bool any_jitter;         // some lane draws jitter (a lane without draws the identity factor:
                             // amplitude 0 gives f = 65536 and q16(d, 65536) = d)
    Jitter jt;
};
// half: lanes 32..63 repeat lanes 0..31 (a tile of at most 32 scenarios)
__device__ __forceinline__ Lane make_lane(const echo_scenario *scen, int32_t n_scen, int32_t tile, int lane,
                                          bool half = false) {
    Lane x;
    if (half) lane &= kLanes / 2 - 1;
    x.active = tile * kLanes + lane < n_scen;
    x.col = x.active ? lane : n_scen - 1 - tile * kLanes;
    x.sigma = tile * kLanes + x.col;
    const echo_scenario *sc = scen + x.sigma;
    const int32_t amp = sc->jitter_amp_q16;
    x.jt = make_jitter(sc->jitter_seed, sc->jitter_stream, amp);
    x.any_jitter = __builtin_amdgcn_readfirstlane(__ballot(amp != 0) != 0);
    return x;
}

// A workgroup of kBlockWalkers wavefronts walks the walkers of one block for
// one 64-scenario tile; wavefront w walks walker block * kBlockWalkers + w.  IN (kIn*):
// what the pass is refined by, or kInOps.  FINAL: the pass produces the step time (and DIGEST:
// the comm ops' share of the digest).
//
// What bounds it: latency.  The sweep is one chain of segments and barriers per
// scenario tile (on the 1024-rank workload the longest passes 1135 barriers in LDS and 265 in
// device memory), and a wavefront runs its items one after the other.  So an item costs its
// instructions, and everything an item could wait for is fetched a round (32 items, kDurs
// segments) ahead and settled by one wait.
//
// kInOps is bound by its stores once enough wavefronts share the chip: with draws, barriers and
// stores of different wavefronts side by side 1024 ranks x 256 scenarios take 11.5 to 14.0 ms, by how
// the two arrays lie in memory (65 GB at 4.7 to 5.7 TB/s), where k_sum, this sweep and k_expand one
// after another take 15.0 to 17.0; 640 x 768 4.7 and 6.2.  All its stores are non-temporal (with
// the last finish of a segment and the comm ops' times through the cache 32 ranks x 5000 take
// 0.90 instead of 0.83 ms, 1024 x 256 11.9 instead of 11.5).
template <int IN, bool FINAL, bool DIGEST>
__global__ __launch_bounds__(kBlockWalkers * 64) __attribute__((amdgpu_waves_per_eu(4))) void k_walk(WalkArgs a) {
    constexpr bool OPS = IN == kInOps, REFINED = IN != kInNone && !OPS;
    static_assert(!OPS || (FINAL && !DIGEST), "the sweep of the ops is the only pass, without digests");
    __shared__ unsigned long long lbar[kChannels * 2][kLanes];   // per channel and slot: latest launch per lane
    __shared__ unsigned lcnt[kChannels * 2];                      // per channel and slot: members arrived
    __shared__ int64_t ccost[kClassSlots][kLanes];                // staged class costs of this tile
    __shared__ int64_t slotmem[kBlockWalkers * kStreams * kLanes];   // slots 1..7 of every wave (slot 0 stays in a register)
    // durations of every wave's round; OPS: the records of its segments, kSegOps each
    __shared__ __align__(16) int64_t durmem[kBlockWalkers * kDurs * kLanes];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // uniform within a wavefront
    const int32_t blk = blockIdx.x / a.tiles;
    const int32_t tile = a.tile0 + blockIdx.x % a.tiles;
    const int32_t w = blk * kBlockWalkers + wave;
    const Lane ln = make_lane(a.scen, a.n_scen, tile, lane);
    const int32_t col = ln.col, sigma = ln.sigma;
    const bool active = ln.active;
    const bool mirror = (tile + 1) * kLanes > a.n_scen;
    const int64_t ns = a.n_scen;

    // block set-up: clear the barrier channels, stage the block's class costs
    for (int i = threadIdx.x; i < kChannels * 2 * kLanes; i += blockDim.x) (&lbar[0][0])[i] = 0;
    if (threadIdx.x < kChannels * 2) lcnt[threadIdx.x] = 0;
    if (wave < kClassSlots) {
        const int32_t cls = a.block_class[(int64_t)blk * kClassSlots + wave];
        ccost[wave][lane] = cls >= 0 ? a.class_cost[(int64_t)cls * ns + sigma] : 0;
    }
    __syncthreads();
    if (w >= a.n_walkers) return;
    // every scenario reached its fixed point in an earlier pass: nothing left to refine
    if (a.stable && __builtin_amdgcn_readfirstlane(__hip_atomic_load(a.stable, __ATOMIC_RELAXED,
                                                                      __HIP_MEMORY_SCOPE_AGENT)))
        return;

    int64_t *const sbase = a.start + (int64_t)tile * kLanes;    // row v of tile: sbase + v * ns
    int64_t *const fbase = a.finish + (int64_t)tile * kLanes;
    const unsigned *tile_count = a.count + tile;
    // every pass but a last one without timelines or digest stores the segments' and comm
    // ops' times: overlap detection, the next pass's durations and k_expand read them
    const bool keep = !FINAL || DIGEST || a.timelines;

    // Per slot: finish of the latest op (of a comm op: once its resolve item ran;
    // no item reads the slot in between).
    int64_t lf0 = 0;
    int64_t *const smem = slotmem + wave * kStreams * kLanes + lane;
#pragma unroll
    for (int j = 1; j < kStreams; ++j) smem[j * kLanes] = 0;
    // A wait that gave up (timeout or abort) marks the wave dead: it finishes its
    // list without waiting again; the times it writes are meaningless and the
    // status word already reports the failure.
    bool dead = false;
    int64_t xmax = 0;            // latest finish among ops kept out of the register slots
    uint64_t dig = 0;
    uint32_t hi_or = 0;          // OR of the high words of every time: bit 30 set <=> some time >= 2^62
    unsigned err = 0;
    const int64_t beg = a.round_off[w], end = a.round_off[w + 1];
    // lane j < 32 holds the first half of item j of the round, lane 32 + j its second half
    const int4 *items4 = reinterpret_cast<const int4 *>(a.items) + 2 * (lane & 31) + (lane >> 5);
    auto load_items = [&](int64_t r) -> int4 {
        return r < end ? items4[2 * kBlock * r] : make_int4(0, (int)kEmpty, 0, 0);
    };
    // Rows are addressed by the lanes: lane j computes the addresses of item j's rows once per
    // round, and a row is then two lane reads and a store with the lane's column as offset
    // (five instructions when computed per store; an item costs its instructions here).
    const uint32_t coff = (uint32_t)col * 8u;
    const uint64_t sadr = reinterpret_cast<uint64_t>(sbase), fadr = reinterpret_cast<uint64_t>(fbase);
    const uint64_t row_bytes = (uint64_t)a.n_scen * 8u;
    auto row_at = [&](uint64_t base, int32_t row) -> uint64_t { return base + (uint64_t)(uint32_t)row * row_bytes; };
    auto row_of = [&](uint64_t rows, int j) -> GlobalI64 * {
        const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)rows, j);
        const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(rows >> 32), j);
        return reinterpret_cast<GlobalI64 *>((((uint64_t)hi << 32) | lo) + coff);
    };
    // OPS: nothing but a far predecessor reads the times again
    auto put_time = [&](GlobalI64 *p, int64_t v) {
        if (OPS) put_stream(p, v);
        else put(p, v);
    };
    // Segment durations (see WalkArgs): lane q < kDurs holds the last op of the round's segment
    // q (unused ones name op 0), fetched a round before the durations.
    const bool load_d = REFINED || (!OPS && ln.any_jitter);
    auto load_rows = [&](int64_t r) -> int32_t {
        return (OPS || load_d) && r < end ? (OPS ? a.rec_rows : a.rows)[r * kDurs + (lane & (kDurs - 1))] : 0;
    };
    int64_t *const dmem = durmem + wave * kDurs * kLanes + lane;
    int64_t in_d[kDurs] = {};
    // OPS: the records instead, lanes 32 * (q & 1) onwards of in_rec[q / 2] holding segment q's
    // (records behind a shorter segment's are fetched too, and not looked at)
    constexpr int kRecLoads = kDurs * kSegOps / kLanes;
    static_assert(kSegOps == kLanes / 2 && kRecLoads * sizeof(SegRec) == kDurs * sizeof(int64_t), "records fill the durations' place");
    typedef int Rec __attribute__((ext_vector_type(4)));
    Rec *const rmem = reinterpret_cast<Rec *>(durmem + wave * kDurs * kLanes);
    Rec in_rec[kRecLoads] = {};
    auto load_durs = [&](int32_t rows) {
        if (OPS) {
#pragma unroll
            for (int p = 0; p < kRecLoads; ++p) {
                const int64_t at = (int64_t)__shfl(rows, 2 * p + (lane >> 5)) + (lane & (kSegOps - 1));
                in_rec[p] = reinterpret_cast<const Rec *>(a.recs)[at < a.n_recs ? at : 0];
            }
            return;
        }
        if (!load_d) return;
        const uint64_t fr = row_at(fadr, rows);
#pragma unroll
        for (int q = 0; q < kDurs; ++q) in_d[q] = *row_of(fr, q);
    };
    int4 nxt = load_items(beg);
    int32_t rows = load_rows(beg);
    __builtin_amdgcn_s_waitcnt(kWaitVm0);
    load_durs(rows);
    rows = load_rows(beg + 1);

    for (int64_t r = beg; r < end; ++r) {
        // Everything fetched for this round is settled here, once; then the next round's items
        // and durations are fetched, and the rows of the one after.
        const int4 cur = nxt;
        __builtin_amdgcn_s_waitcnt(kWaitVm0);
        if (load_d) {
#pragma unroll
            for (int q = 0; q < kDurs; ++q) dmem[q * kLanes] = in_d[q];
        }
        if (OPS) {
#pragma unroll
            for (int p = 0; p < kRecLoads; ++p) rmem[p * kLanes + lane] = in_rec[p];
        }
        nxt = load_items(r + 1);
        load_durs(rows);
        rows = load_rows(r + 2);
        const int nb = __builtin_popcountll(__builtin_amdgcn_read_exec() &
                                            __ballot(lane < kBlock && !((uint32_t)cur.y & kEmpty)));
        // the round's segments (a duration's index is a count of bits)
        const uint32_t seg_bits = (uint32_t)(__builtin_amdgcn_read_exec() &
                                             __ballot(lane < kBlock && ((uint32_t)cur.y & (kEmpty | 1u)) == 0));
        const uint64_t srow = row_at(sadr, cur.x);                                  // start: the (first) op
        const uint64_t frow = row_at(fadr, ((uint32_t)cur.y & 1u) ? cur.x : cur.w);  // finish: the (last) op
        for (int j = 0; j < nb; ++j) {
            const uint32_t meta = (uint32_t)__builtin_amdgcn_readlane(cur.y, j);
            const int kind = item_kind(meta);
            const int sq = (meta & kNoReg) ? kStreams : item_stream(meta);  // kStreams: no slot
            const bool storef = keep || (meta & kNeedF);
            if (kind == kResolve) {
                // a comm op's barrier, due right before its first successor: its finish is the
                // latest member launch plus the collective's cost
                const uint32_t aux = (uint32_t)__builtin_amdgcn_readlane(cur.w, j + 32);
                // The cost: from the workgroup's LDS slot, read first on every path; a class without
                // a slot reads device memory and waits for that load inside its own branch, so
                // the common path carries no wait on vector memory (which on this target would also
                // wait for every timeline store still in flight).  Distinct load kinds keep the two
                // reads from merging into one flat load.
                const int sl = aux_slot(aux);
                int64_t t = ccost[sl & (kClassSlots - 1)][lane];
                int64_t own = 0;                             // linked: this member's published launch
                uint64_t b = 0;
                if (aux & kAuxLocal) {
                    const int ch = aux_barrier(aux);
                    if (meta & kLaunch) {
                        if (keep) put(row_of(srow, j), lf0);
                        arrive_local(lbar[ch], &lcnt[ch], lf0, lane);
                    }
                    if (!dead && !__builtin_amdgcn_readfirstlane(wait_local(&lcnt[ch], aux_expected(aux), lbar[ch], lane,
                                                                            &b, a.status, a.spin_limit)))
                        dead = true;
                } else if (aux & kAuxSlots) {
                    // the own launch is fetched with the members' (one round trip)
                    if (keep && (meta & kLinked)) own = *row_of(srow, j);
                    bool ok = true;
                    if (!dead) {
                        const int64_t *p = a.slots + (int64_t)__builtin_amdgcn_readlane(cur.z, j) * ns + sigma;
                        const unsigned n = aux_expected(aux);
                        b = n <= 2 ? (uint64_t)wait_slots<2>(p, n, ns, a.status, a.spin_limit, &ok)
                                   : (uint64_t)wait_slots<kSlotMembers>(p, n, ns, a.status, a.spin_limit, &ok);
                    }
                    __builtin_amdgcn_s_waitcnt(kWaitVm0);    // settled on this path, not at the join
                    if (!__builtin_amdgcn_readfirstlane(ok)) dead = true;
                } else {
                    const int32_t coll = __builtin_amdgcn_readlane(cur.w, j);
                    if (keep && (meta & kLinked)) own = *row_of(srow, j);
                    if (!dead && !__builtin_amdgcn_readfirstlane(wait_arrivals(tile_count + (int64_t)coll * a.n_tiles,
                                                                               (unsigned)a.c_N[coll], a.status,
                                                                               a.spin_limit)))
                        dead = true;
                    if (active)
                        b = __hip_atomic_fetch_max(a.arrive + (int64_t)coll * ns + sigma, 0ull, __ATOMIC_RELAXED,
                                                   __HIP_MEMORY_SCOPE_AGENT);
                    __builtin_amdgcn_s_waitcnt(kWaitVm0);    // settled on this path, not at the join
                    b = mirror ? (uint64_t)__shfl((long long)b, col) : b;
                }
                if (sl >= kClassSlots) {
                    const int64_t cls = __builtin_amdgcn_readlane(cur.x, j + 32);
                    t = __hip_atomic_load(a.class_cost + cls * ns + sigma, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    __builtin_amdgcn_s_waitcnt(kWaitVm0);
                }
                if (meta & kLinked) {
                    // the op it is linked to finished at p: the barrier, and this member's own
                    // launch, are no earlier
                    int64_t p;
                    if (sq == 0) {
                        p = lf0;
                    } else if (sq < kStreams) {
                        p = smem[sq * kLanes];
                    } else {
                        p = (fbase + (int64_t)__builtin_amdgcn_readlane(cur.z, j + 32) * ns)[col];
                        __builtin_amdgcn_s_waitcnt(kWaitVm0);    // settled on this path, not at the join
                    }
                    b = (uint64_t)p > b ? (uint64_t)p : b;
                    own = p > own ? p : own;
                    if (keep) put(row_of(srow, j), own);
                }
                const int64_t f = (int64_t)b + t;
                hi_or |= (uint32_t)((uint64_t)f >> 32);
                if (storef) put_time(row_of(frow, j), f);
                if (DIGEST) {
                    const int32_t op = __builtin_amdgcn_readlane(cur.x, j);
                    const int64_t s = *row_of(srow, j);
                    dig += mix64(mix64((uint64_t)op ^ (uint64_t)s) ^ (uint64_t)f);
                }
                if (sq == 0) lf0 = f;
                else if (sq < kStreams) smem[sq * kLanes] = f;
                else xmax = f > xmax ? f : xmax;
                if (meta & kFold) lf0 = f > lf0 ? f : lf0;
                continue;
            }
            const unsigned mask = item_regmask(meta);
            int64_t ready = 0;
            if (mask & 1u) ready = lf0;
            for (unsigned m = mask & ~1u; m; m &= m - 1) {
                const int64_t x = smem[__builtin_ctz(m) * kLanes];
                ready = x > ready ? x : ready;
            }
            if (meta & kHasFar) {
                const int32_t far_off = __builtin_amdgcn_readlane(cur.z, j);
                const int32_t nfar = __builtin_amdgcn_readlane(cur.z, j + 32);
                for (int32_t q = 0; q < nfar; ++q) {
                    const RowPair u = a.far[far_off + q];
                    int64_t fu = (fbase + (int64_t)u.last * ns)[col];
                    // before the last pass a segment's row holds its duration
                    if (!FINAL && u.first >= 0) fu += (sbase + (int64_t)u.first * ns)[col];
                    ready = fu > ready ? fu : ready;
                }
                __builtin_amdgcn_s_waitcnt(kWaitVm0);        // settled on this path, not at the join
            }
            if (keep) put_time(row_of(srow, j), ready);
            if (kind == ECHO_COMM) {
                // launch: publish this member's launch time, then count the arrival
                const uint32_t aux = (uint32_t)__builtin_amdgcn_readlane(cur.w, j + 32);
                if (aux & kAuxLocal) {
                    const int ch = aux_barrier(aux);
                    arrive_local(lbar[ch], &lcnt[ch], ready, lane);
                } else if (aux & kAuxSlots) {
                    // this member's slot (its index is in the item's duration field): one store,
                    // no wait -- the value is its own arrival flag
                    const int64_t slot = (int64_t)(((uint64_t)(uint32_t)__builtin_amdgcn_readlane(cur.y, j + 32) << 32) |
                                                   (uint32_t)__builtin_amdgcn_readlane(cur.x, j + 32));
                    if (active)
                        __hip_atomic_store(a.slots + slot * ns + sigma, ready, __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_AGENT);
                } else {
                    const int32_t coll = __builtin_amdgcn_readlane(cur.w, j);
                    if (active)
                        __hip_atomic_fetch_max(a.arrive + (int64_t)coll * ns + sigma, (unsigned long long)ready,
                                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                    if (lane == 0)
                        __hip_atomic_fetch_add(a.count + (int64_t)coll * a.n_tiles + tile, 1u, __ATOMIC_RELAXED,
                                               __HIP_MEMORY_SCOPE_AGENT);
                }
            } else {
                int64_t f;
                if (OPS) {
                    // the segment's ops one after the other: each finish but the last is the next op's start
                    const Rec rec = rmem[__builtin_popcount(seg_bits & ((1u << j) - 1)) * kSegOps + (lane & (kSegOps - 1))];
                    const int n = __builtin_amdgcn_readlane(cur.w, j + 32);
                    const uint64_t prow = row_at(fadr, rec.x), qrow = row_at(sadr, rec.x);
                    f = ready;
                    auto steps = [&](auto jit, auto is_small) {
                        for (int i = 0; i < n; ++i) {
                            const int32_t op = decltype(jit)::value ? __builtin_amdgcn_readlane(rec.x, i) : 0;
                            const uint32_t dlo = (uint32_t)__builtin_amdgcn_readlane(rec.z, i);
                            if (decltype(is_small)::value) {
                                f += decltype(jit)::value ? jittered32(dlo, op, ln.jt) : (int64_t)dlo;
                            } else {
                                const uint32_t dhi = (uint32_t)__builtin_amdgcn_readlane(rec.w, i);
                                const int64_t d0 = (int64_t)(((uint64_t)dhi << 32) | dlo);
                                f += decltype(jit)::value ? jittered(d0, op, ln.jt) : d0;
                            }
                            put_time(row_of(prow, i), f);
                            if (i + 1 < n) put_time(row_of(qrow, i + 1), f);
                        }
                    };
                    // (of the records behind the segment too: the general form is right for all)
                    const bool small = __builtin_amdgcn_readfirstlane(__ballot(rec.w != 0) == 0);
                    if (!ln.any_jitter) steps(std::false_type{}, std::false_type{});
                    else if (small) steps(std::true_type{}, std::true_type{});
                    else steps(std::true_type{}, std::false_type{});
                    hi_or |= (uint32_t)((uint64_t)f >> 32);
                    if (sq == 0) lf0 = f;
                    else if (sq < kStreams) smem[sq * kLanes] = f;
                    else xmax = f > xmax ? f : xmax;
                    continue;
                }
                int64_t d;
                if (load_d) {
                    d = dmem[__builtin_popcount(seg_bits & ((1u << j) - 1)) * kLanes];
                } else {
                    d = (int64_t)(((uint64_t)(uint32_t)__builtin_amdgcn_readlane(cur.y, j + 32) << 32) |
                                  (uint32_t)__builtin_amdgcn_readlane(cur.x, j + 32));
                }
                f = ready + d;
                hi_or |= (uint32_t)((uint64_t)f >> 32);
                if (FINAL) {
                    if (storef) put(row_of(frow, j), f);
                } else if (!load_d) {
                    put(row_of(frow, j), d);
                }
                if (sq == 0) lf0 = f;
                else if (sq < kStreams) smem[sq * kLanes] = f;
                else xmax = f > xmax ? f : xmax;
            }
        }
    }
    if (hi_or >> 30) err |= kStatusOverflow;
    if (active && err) __hip_atomic_fetch_or(a.status, err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (FINAL && active && !dead) {
        // finishes along a FIFO stream never decrease: the last op of each slot holds its
        // maximum; ops without a slot went into xmax
        int64_t smax = lf0 > xmax ? lf0 : xmax;
#pragma unroll
        for (int q = 1; q < kStreams; ++q) smax = smem[q * kLanes] > smax ? smem[q * kLanes] : smax;
        __hip_atomic_fetch_max(reinterpret_cast<unsigned long long *>(a.step) + sigma, (unsigned long long)smax,
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (DIGEST)
            __hip_atomic_fetch_add(reinterpret_cast<unsigned long long *>(a.digest) + sigma,
                                   (unsigned long long)dig, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

using WalkKernel = void (*)(WalkArgs);
WalkKernel walk_kernel(int in, bool final_pass, bool digest) {
    // a digest only in a final pass, kInMaskFlags too; kInOps is a final pass without one
    if (!final_pass) {
        if (in == kInNone) return k_walk<kInNone, false, false>;
        return in == kInExtFlags ? k_walk<kInExtFlags, false, false> : k_walk<kInMasks, false, false>;
    }
    switch (in) {
    case kInOps: return k_walk<kInOps, true, false>;
    case kInNone: return digest ? k_walk<kInNone, true, true> : k_walk<kInNone, true, false>;
    case kInMasks: return digest ? k_walk<kInMasks, true, true> : k_walk<kInMasks, true, false>;
    case kInMaskFlags: return digest ? k_walk<kInMaskFlags, true, true> : k_walk<kInMaskFlags, true, false>;
    default: return digest ? k_walk<kInExtFlags, true, true> : k_walk<kInExtFlags, true, false>;
    }
}

// ------------------------------------------------------------------ the ops of segments
// One wavefront per (part, tile): the chunks part, part + parts, ... of segment records for
// one tile.  Consecutive wavefronts take the tiles of one chunk, so that a row is written
// whole by one workgroup at about one time, and each keeps its tile's scenario knobs.
constexpr int kRecWaves = 4;             // wavefronts per workgroup
// Wavefronts of a launch, unless there are more tiles: eight rounds of what the chip holds, so
// that the last round is short against the rest (on the 1024-rank workload k_expand takes
// 12.1 ms with one round, 11.8 with eight, 11.7 with a wavefront per chunk, which makes a
// k_sum that has nothing to do eight times longer).
constexpr int64_t kRecParts = 65536;

__device__ __forceinline__ int4 load_chunk(const WalkArgs &a, int64_t chunk, int lane, int *n) {
    *n = 0;
    if (chunk >= a.n_chunks) return make_int4(0, 0, 0, 0);
    const int32_t r0 = __builtin_amdgcn_readfirstlane(a.chunks[chunk].rec0);
    *n = __builtin_amdgcn_readfirstlane(a.chunks[chunk + 1].rec0) - r0;
    return lane < *n ? reinterpret_cast<const int4 *>(a.recs)[r0 + lane] : make_int4(0, 0, 0, 0);
}

// First pass, tiles with jitter: the sum of each segment's jittered durations, into the
// finish row of its last op.  Bound by the draws (25 vector instructions per op and
// wavefront); the records of the next chunk are fetched while the current one is summed.
__global__ __launch_bounds__(kRecWaves * 64) void k_sum(WalkArgs a, int64_t parts) {
    const int lane = threadIdx.x & 63;
    const int64_t unit = (int64_t)blockIdx.x * kRecWaves + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int32_t tile = a.tile0 + (int32_t)(unit % a.tiles);
    const int64_t part = unit / a.tiles;
    if (part >= parts) return;
    const Lane ln = make_lane(a.scen, a.n_scen, tile, lane);
    if (!ln.any_jitter) return;
    const int64_t ns = a.n_scen;
    int64_t *const fbase = a.finish + (int64_t)tile * kLanes + ln.col;
    int nn;
    int4 nxt = load_chunk(a, part, lane, &nn);
    for (int64_t chunk = part; chunk < a.n_chunks; chunk += parts) {
        const int4 cur = nxt;
        const int n = nn;
        __builtin_amdgcn_s_waitcnt(kWaitVm0);
        nxt = load_chunk(a, chunk + parts, lane, &nn);
        const uint64_t last_bits = __builtin_amdgcn_read_exec() & __ballot((uint32_t)cur.y & kRecLast);
        const bool small = __builtin_amdgcn_readfirstlane((__builtin_amdgcn_read_exec() & __ballot(cur.w != 0)) == 0);
        int64_t sum = 0;
        auto body = [&](auto is_small) {
            for (int j = 0; j < n; ++j) {
                const int32_t op = __builtin_amdgcn_readlane(cur.x, j);
                const uint32_t dlo = (uint32_t)__builtin_amdgcn_readlane(cur.z, j);
                if (decltype(is_small)::value) {
                    sum += jittered32(dlo, op, ln.jt);
                } else {
                    const uint32_t dhi = (uint32_t)__builtin_amdgcn_readlane(cur.w, j);
                    sum += jittered((int64_t)(((uint64_t)dhi << 32) | dlo), op, ln.jt);
                }
                if ((last_bits >> j) & 1u) {
                    fbase[(int64_t)op * ns] = sum;
                    sum = 0;
                }
            }
        };
        if (small) body(std::true_type{});
        else body(std::false_type{});
    }
}

// After the last pass: the start and finish of every op that the sweep has not written (all
// but each segment's first start and last finish), and with DIGEST the segments' share of
// the digest.  IN: what flagged segments carry per op -- nothing (no refinement), overlap
// masks, or extra times.  Bound by the timeline stores (57 GB in 11.9 ms on the
// 1024-rank workload, its wavefronts 68 % of their cycles waiting to issue; a store-only probe
// of the pattern takes 10.2 at 5.6 TB/s).  An op's finish is the
// next op's start, so a step of the loop is one draw and two stores, the last op of a segment
// takes neither, and the lanes compute the chunk's row addresses once.
template <int IN, bool DIGEST>
__global__ __launch_bounds__(kRecWaves * 64) void k_expand(WalkArgs a, int64_t parts) {
    const int lane = threadIdx.x & 63;
    const int64_t unit = (int64_t)blockIdx.x * kRecWaves + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int32_t tile = a.tile0 + (int32_t)(unit % a.tiles);
    const int64_t part = unit / a.tiles;
    if (part >= parts) return;
    // A tile of at most 32 scenarios fills half the lanes: the other half repeats it, and a
    // finish and the next op's start, the same value, go out in one store (the store path takes
    // a wavefront's store in about 32 cycles however many lanes it has).
    const bool half = a.n_scen - tile * kLanes <= kLanes / 2;
    const Lane ln = make_lane(a.scen, a.n_scen, tile, lane, half);
    const int64_t ns = a.n_scen;
    const uint64_t sadr = reinterpret_cast<uint64_t>(a.start + (int64_t)tile * kLanes);
    const uint64_t fadr = reinterpret_cast<uint64_t>(a.finish + (int64_t)tile * kLanes);
    const uint32_t coff = (uint32_t)ln.col * 8u;
    const uint64_t row_bytes = (uint64_t)ns * 8u;
    auto row_of = [&](uint64_t rows, int j) -> GlobalI64 * {
        const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)rows, j);
        const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(rows >> 32), j);
        return reinterpret_cast<GlobalI64 *>((((uint64_t)hi << 32) | lo) + coff);
    };
    const uint4 *const slow = reinterpret_cast<const uint4 *>(&a.scen[ln.sigma].slowdown_q16[0][0]);
    uint64_t dig = 0;
    typedef int64_t Starts __attribute__((ext_vector_type(8)));
    typedef uint32_t Ins __attribute__((ext_vector_type(8)));
    int nn;
    int4 nxt = load_chunk(a, part, lane, &nn);
    for (int64_t chunk = part; chunk < a.n_chunks; chunk += parts) {
        const int4 cur = nxt;
        const int n = nn;
        const uint64_t frow = fadr + (uint64_t)(uint32_t)cur.x * row_bytes, srow = sadr + (uint64_t)(uint32_t)cur.x * row_bytes;
        const uint64_t first_bits = __builtin_amdgcn_read_exec() & __ballot((uint32_t)cur.y & kRecFirst);
        const uint64_t last_bits = __builtin_amdgcn_read_exec() & __ballot((uint32_t)cur.y & kRecLast);
        const bool small = __builtin_amdgcn_readfirstlane((__builtin_amdgcn_read_exec() & __ballot(cur.w != 0)) == 0);
        const uint64_t cand_bits = IN == kInNone ? 0 : __builtin_amdgcn_read_exec() & __ballot((uint32_t)cur.y & kRecCand);
        const int64_t rec0 = __builtin_amdgcn_readfirstlane(a.chunks[chunk].rec0);
        uint64_t flag_bits = 0;                   // flags of the chunk's overlap segments, in order
        if (cand_bits) {
            const int64_t c0 = __builtin_amdgcn_readfirstlane(a.chunks[chunk].cand0);
            const int nc = __builtin_popcountll(cand_bits);
            const uint8_t fl = lane < nc ? a.xflag[(c0 + lane) * a.n_tiles + tile] : 0;
            flag_bits = __ballot(fl != 0);
        }
        // starts of the chunk's next eight segments, fetched together
        uint64_t todo = first_bits;
        Starts s8 = 0;
        int is = 8, ic = 0;
        auto steps = [&](auto jit, auto is_small, bool flagged, int64_t s, int j0, int end) {
            Ins x8 = 0;
            for (int j = j0; j < end; ++j) {
                const int32_t op = decltype(jit)::value || DIGEST ? __builtin_amdgcn_readlane(cur.x, j) : 0;
                const uint32_t dlo = (uint32_t)__builtin_amdgcn_readlane(cur.z, j);
                int64_t d;
                if (decltype(is_small)::value) {
                    d = decltype(jit)::value ? jittered32(dlo, op, ln.jt) : (int64_t)dlo;
                } else {
                    const uint32_t dhi = (uint32_t)__builtin_amdgcn_readlane(cur.w, j);
                    const int64_t d0 = (int64_t)(((uint64_t)dhi << 32) | dlo);
                    d = decltype(jit)::value ? jittered(d0, op, ln.jt) : d0;
                }
                if (IN != kInNone && flagged) {
                    const int q0 = (j - j0) & 7;
                    if (q0 == 0) {
                        // the segment's next eight masks (extra times), in one round trip
#pragma unroll
                        for (int q = 0; q < 8; ++q) {
                            if (j + q >= end) continue;
                            const int64_t at = (rec0 + j + q) * a.mstride + (int64_t)tile * kLanes + ln.col;
                            x8[q] = IN == kInExtFlags ? a.ext[at] : (uint32_t)a.tmask[at];
                        }
                    }
                    const uint32_t meta = (uint32_t)__builtin_amdgcn_readlane(cur.y, j);
                    if (meta & kRecCompute) {
                        const uint32_t x = x8[q0];
                        if (IN == kInExtFlags) {
                            d += x;
                        } else if (__ballot(x != 0)) {
                            const uint4 row = slow[meta & 7u];
                            d = inflate_row(d, x, row);
                        }
                    }
                }
                const int64_t f = s + d;
                if (DIGEST) dig += mix64(mix64((uint64_t)op ^ (uint64_t)s) ^ (uint64_t)f);
                if (!DIGEST || a.timelines) {
                    if ((!DIGEST || j + 1 < end) && ln.active) {
                        GlobalI64 *const pf = row_of(frow, j), *const ps = row_of(srow, j + 1);
                        if (half) {
                            put_stream(lane < kLanes / 2 ? pf : ps, f);
                        } else {
                            put_stream(pf, f);
                            put_stream(ps, f);
                        }
                    }
                }
                s = f;
            }
        };
        nxt = load_chunk(a, chunk + parts, lane, &nn);
        for (int j = 0; j < n;) {
            // a segment: its ops but the last (with DIGEST the last too, without stores)
            const int end = j + __builtin_ctzll(last_bits >> j);
            if (is == 8) {
#pragma unroll
                for (int q = 0; q < 8; ++q)
                    if (todo) {
                        s8[q] = *row_of(srow, __builtin_ctzll(todo));
                        todo &= todo - 1;
                    }
                is = 0;
            }
            const int64_t s = s8[is];
            ++is;
            bool flagged = false;
            if (IN != kInNone && ((cand_bits >> j) & 1u)) {
                flagged = (flag_bits >> ic) & 1u;
                ++ic;
            }
            const int stop = DIGEST ? end + 1 : end;
            if (ln.any_jitter) {
                if (small) steps(std::true_type{}, std::true_type{}, flagged, s, j, stop);
                else steps(std::true_type{}, std::false_type{}, flagged, s, j, stop);
            } else {
                steps(std::false_type{}, std::false_type{}, flagged, s, j, stop);
            }
            j = end + 1;
        }
    }
    if (DIGEST && ln.active && !(half && lane >= kLanes / 2))
        __hip_atomic_fetch_add(reinterpret_cast<unsigned long long *>(a.digest) + ln.sigma, (unsigned long long)dig,
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// ------------------------------------------------------------------ overlap detection
// A wavefront takes groups of kOverlapGroup segments for one tile.  Comm ops of a stream
// finish in order, so a segment overlaps none of a range's comm ops when the range's last
// one finishes by the segment's start: one load per range settles most segments, which
// then cost nothing more.  For the others the range's first comm op that ends after the
// segment's start is searched (backwards from the last, in doubling steps), and from
// there a cursor that only moves forward meets every comm op overlapping the segment's
// ops in turn.  The ops' intervals are rebuilt, not read: the first starts with the segment,
// each later one where the one before finished, and a finish is start + base duration (the
// same jitter draw as the composer pass, inflated by the factor that pass used).  With
// the new factors the segment's new duration is known at once and goes where the next pass
// takes it from.
// Factor of a class-cls compute op overlapping the collective types in mask m:
// the largest entry of the scenario's table row over them, 65536 for none.
__device__ __forceinline__ uint32_t factor_of(uint32_t m, const uint32_t *slow, int cls) {
    uint32_t F = 65536u;
    for (int t = 0; t < kTypes; ++t)
        if ((m >> t) & 1u) {
            const uint32_t x = slow[cls * kTypes + t];
            F = x > F ? x : F;
        }
    return F;
}

// Factor predicted by the tree ensemble for a compute op (class cls, base
// duration d0) overlapped by the collective types in mask m (Sec. 6): for each
// type, the base score plus one leaf per tree, kept inside [65536, 2^20); the
// largest over the types.  Trees are walked from device memory (the walk stops at
// a leaf; paths are at most ECHO_TREE_DEPTH splits long): when every lane that
// needs a type shares one feature vector, once for the wavefront with one tree
// per lane, else per lane.  Called with every lane active (m 0: 65536): a lane that
// needs no type still walks its trees for the others.
constexpr int kForestLanes = 16;
// In the compact form the node reads are LDS reads and bound by its throughput (random banks):
// a batch stops once its walks have reached their leaves, and a small one does so earlier
// (64 trees, 64 ranks x 200 scenarios: 9.1 ms with 16 trees and 12 steps, 8.8 with 8, 9.2 and
// 7.9 with the stop).
constexpr int kFxLanes = 8;

// feat: this wavefront's LDS feature rows, feature k of lane l at feat[k * 64 + l].
__device__ uint32_t forest_factor(const OverlapArgs &a, uint32_t m, const int64_t *smax, const int32_t *nmax,
                                  int cls, int64_t d0, const echo_scenario *sc, int64_t *feat, bool knobs_uniform,
                                  int lane) {
    const int64_t *met = a.class_metrics + cls * kClassMetrics;
    feat[0 * kLanes + lane] = cls;
    feat[1 * kLanes + lane] = d0;
    feat[5 * kLanes + lane] = sc->ar_algo;
    feat[6 * kLanes + lane] = sc->bw_intra_MBps;
    feat[7 * kLanes + lane] = sc->bw_inter_MBps;
#pragma unroll
    for (int k = 0; k < kClassMetrics; ++k) feat[(8 + k) * kLanes + lane] = met[k];
    uint32_t best = 65536u;
#pragma unroll
    for (int t = 0; t < kTypes; ++t) {
        const bool has = (m >> t) & 1u;
        const uint64_t lanes_t = __ballot(has);
        if (!lanes_t) continue;
        feat[2 * kLanes + lane] = t;
        feat[3 * kLanes + lane] = smax[t];
        feat[4 * kLanes + lane] = nmax[t];
        const int first = __builtin_ctzll(lanes_t);
        const int64_t s0 = __shfl(smax[t], first);
        const int32_t n0 = __shfl(nmax[t], first);
        const bool uniform = knobs_uniform && __ballot(has && (smax[t] != s0 || nmax[t] != n0)) == 0;
        int64_t sum = a.forest_base;
        if (uniform) {
            // every lane that needs type t has lane `first`'s feature vector: the trees are
            // walked side by side, one per lane, and their leaves summed across the wavefront
            for (int32_t tr0 = 0; tr0 < a.n_trees; tr0 += kLanes) {
                const bool live = tr0 + lane < a.n_trees;
                int32_t idx = a.forest_roots[live ? tr0 + lane : 0];
                for (int step = 0; step < ECHO_TREE_DEPTH; ++step) {
                    const int4 nd = reinterpret_cast<const int4 *>(a.forest_nodes)[idx];
                    const int64_t x = feat[nd.z * kLanes + first];
                    const int64_t thr = (int64_t)(((uint64_t)(uint32_t)nd.y << 32) | (uint32_t)nd.x);
                    idx = nd.w + (x < thr ? 0 : 1);
                }
                int64_t leaf = live ? (int64_t)a.forest_leaf[idx] : 0;
#pragma unroll
                for (int o = kLanes / 2; o > 0; o >>= 1) leaf += __shfl_xor(leaf, o);
                sum += leaf;
            }
        } else if (has) {
            // kForestLanes trees walked side by side: their node loads are independent
            for (int32_t tr0 = 0; tr0 < a.n_trees; tr0 += kForestLanes) {
                int32_t idx[kForestLanes];
                bool live[kForestLanes];
#pragma unroll
                for (int q = 0; q < kForestLanes; ++q) {
                    live[q] = tr0 + q < a.n_trees;
                    idx[q] = live[q] ? a.forest_roots[tr0 + q] : 0;
                }
                // every path has at most ECHO_TREE_DEPTH splits and a leaf loops to itself, so
                // after that many steps each walk rests on its leaf: no per-lane exit
                for (int step = 0; step < ECHO_TREE_DEPTH; ++step) {
                    int4 nd[kForestLanes];          // threshold low, threshold high, feature, left
#pragma unroll
                    for (int q = 0; q < kForestLanes; ++q)
                        nd[q] = reinterpret_cast<const int4 *>(a.forest_nodes)[idx[q]];
#pragma unroll
                    for (int q = 0; q < kForestLanes; ++q) {
                        const int64_t x = feat[nd[q].z * kLanes + lane];
                        const int64_t thr = (int64_t)(((uint64_t)(uint32_t)nd[q].y << 32) | (uint32_t)nd[q].x);
                        idx[q] = nd[q].w + (x < thr ? 0 : 1);
                    }
                }
#pragma unroll
                for (int q = 0; q < kForestLanes; ++q)
                    if (live[q]) sum += a.forest_leaf[idx[q]];
            }
        }
        sum = sum < 65536 ? 65536 : sum;
        sum = sum >= (int64_t(1) << 20) ? (int64_t(1) << 20) - 1 : sum;
        if (has) best = (uint32_t)sum > best ? (uint32_t)sum : best;
    }
    return best;
}

// ---- compact ensemble (LDS): features compared by bin (see CompactForest)
// Bin of x for a feature with sorted thresholds T[0..n): how many are <= x.
__device__ __forceinline__ int32_t fx_bin(const int64_t *T, int32_t n, int64_t x) {
    int32_t lo = 0, hi = n;
    while (lo < hi) {
        const int32_t mid = (lo + hi) >> 1;
        if (T[mid] <= x) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

// Bins of every collective's S and cost N (features 3 and 4) and of every segment
// record's base duration (feature 1).
__global__ void k_forest_bins(CollTable colls, const SegRec *recs, int64_t n_recs, CompactForest fx) {
    const int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t nth = (int64_t)gridDim.x * blockDim.x;
    const int64_t *T1 = fx.thr + fx.thr_off[1], *T3 = fx.thr + fx.thr_off[3], *T4 = fx.thr + fx.thr_off[4];
    const int32_t n1 = fx.thr_off[2] - fx.thr_off[1], n3 = fx.thr_off[4] - fx.thr_off[3],
                  n4 = fx.thr_off[5] - fx.thr_off[4];
    for (int64_t c = tid; c < colls.n; c += nth) {
        fx.coll_bin[2 * c] = fx_bin(T3, n3, colls.bytes[c]);
        fx.coll_bin[2 * c + 1] = fx_bin(T4, n4, colls.N[c]);
    }
    for (int64_t i = tid; i < n_recs; i += nth) fx.cp_bin[i] = fx_bin(T1, n1, recs[i].dur);
}

// Ensemble prediction from the compact LDS form, for the collective types in mask m
// (per lane), as forest_factor computes it.  fb: this wavefront's bin rows in LDS,
// feature f of lane l at fb[f * 64 + l] (rows 5-7: the scenario's knobs, set once;
// rows 12-15: 0).  bS/bN: per type, the largest bins of S and N among the overlapping
// type-t comm ops.  When every lane that has type t in its mask shares its feature
// vector (knobs_uniform and equal S and N bins), the trees are walked once for the
// wavefront, one tree per lane (every lane must be active); otherwise each lane that has
// the type walks every tree on its own path.
__device__ uint32_t forest_factor_compact(const OverlapArgs &a, uint32_t m, const int32_t *bS, const int32_t *bN,
                                          int cls, int32_t bd0, const uint32_t *fw, const int32_t *froots, uint16_t *fb,
                                          bool knobs_uniform, int lane) {
    const int32_t *cb = a.fx.cbin + cls * kFxFeatures;
    fb[0 * kLanes + lane] = (uint16_t)cb[0];
    fb[1 * kLanes + lane] = (uint16_t)bd0;
#pragma unroll
    for (int k = 8; k < kFxFeatures; ++k) fb[k * kLanes + lane] = (uint16_t)cb[k];
    uint32_t best = 65536u;
#pragma unroll
    for (int t = 0; t < kTypes; ++t) {
        const bool has = (m >> t) & 1u;
        const uint64_t lanes_t = __ballot(has);
        if (!lanes_t) continue;
        fb[2 * kLanes + lane] = (uint16_t)a.fx.tbin[t];
        fb[3 * kLanes + lane] = (uint16_t)bS[t];
        fb[4 * kLanes + lane] = (uint16_t)bN[t];
        const int first = __builtin_ctzll(lanes_t);
        const int32_t s0 = __builtin_amdgcn_readlane(bS[t], first), n0 = __builtin_amdgcn_readlane(bN[t], first);
        const bool uniform = knobs_uniform && __ballot(has && (bS[t] != s0 || bN[t] != n0)) == 0;
        int64_t sum = a.forest_base;
        if (uniform) {
            // One feature vector (lane `first`'s) for every lane that needs type t: the
            // trees are walked side by side, one per lane, and their leaves summed across
            // the wavefront.
            for (int32_t tr0 = 0; tr0 < a.n_trees; tr0 += kLanes) {
                const bool live = tr0 + lane < a.n_trees;
                int32_t idx = froots[live ? tr0 + lane : 0];
                for (int step = 0; step < ECHO_TREE_DEPTH; ++step) {
                    const uint32_t w = fw[idx];
                    const uint32_t f = w & 15u;
                    const uint32_t r = (w >> 4) & ((1u << kFxRankBits) - 1);
                    const int32_t off = f == kFxLeaf ? 0 : (int32_t)(w >> (4 + kFxRankBits));
                    const uint32_t x = fb[f * kLanes + first];
                    idx += off + (x > r ? 1 : 0);
                }
                int64_t leaf = live ? (int64_t)((int32_t)fw[idx] >> 4) : 0;
#pragma unroll
                for (int o = kLanes / 2; o > 0; o >>= 1) leaf += __shfl_xor(leaf, o);
                sum += leaf;
            }
        } else if (has) {
            for (int32_t tr0 = 0; tr0 < a.n_trees; tr0 += kFxLanes) {
                int32_t idx[kFxLanes];
                bool live[kFxLanes];
#pragma unroll
                for (int q = 0; q < kFxLanes; ++q) {
                    live[q] = tr0 + q < a.n_trees;
                    idx[q] = froots[live[q] ? tr0 + q : 0];
                }
                for (int step = 0; step < ECHO_TREE_DEPTH; ++step) {
                    int32_t moved = 0;
                    uint32_t w[kFxLanes];
#pragma unroll
                    for (int q = 0; q < kFxLanes; ++q) w[q] = fw[idx[q]];
#pragma unroll
                    for (int q = 0; q < kFxLanes; ++q) {
                        const uint32_t f = w[q] & 15u;
                        const uint32_t r = (w[q] >> 4) & ((1u << kFxRankBits) - 1);
                        const int32_t off = f == kFxLeaf ? 0 : (int32_t)(w[q] >> (4 + kFxRankBits));
                        const uint32_t x = fb[f * kLanes + lane];
                        idx[q] += off + (x > r ? 1 : 0);
                        moved |= off;
                    }
                    // every walk of the lanes that need type t rests on its leaf
                    if (!__builtin_amdgcn_readfirstlane(__ballot(moved != 0) != 0)) break;
                }
#pragma unroll
                for (int q = 0; q < kFxLanes; ++q)
                    if (live[q]) sum += (int32_t)fw[idx[q]] >> 4;
            }
        }
        sum = sum < 65536 ? 65536 : sum;
        sum = sum >= (int64_t(1) << 20) ? (int64_t(1) << 20) - 1 : sum;
        if (has) best = (uint32_t)sum > best ? (uint32_t)sum : best;
    }
    return best;
}

// PRORATE: also measure o, the part of [s_v, f_v) covered by the union of the
// overlapping comm intervals (a merge of the per-stream interval lists in start
// order), and record the extra time q16(min(o, D), F) - min(o, D) instead of a mask.
// DETECT: flag the scenarios whose durations change (fixed-point iteration).
// FOREST: the factor is the tree ensemble's prediction (recorded as an extra time):
// 1 walks the ensemble from device memory, 2 from its compact form in LDS (the
// workgroup's wavefronts share one copy of the nodes).
// NC: room for this many comm ranges per segment (the cursor and merge state scale with it).
constexpr int kOverlapWaves = 4;         // wavefronts per workgroup
constexpr int kXcds = 8;
template <bool PRORATE, bool DETECT, int FOREST, int NC>
__global__ __launch_bounds__(64 * kOverlapWaves) void k_overlap(OverlapArgs a, int64_t parts) {
    constexpr bool EXT = PRORATE || FOREST != 0;  // output: extra time per op instead of a mask
    constexpr int W = kOverlapWaves;
    __shared__ int64_t feat_all[FOREST == 1 ? W * 12 * kLanes : 1];   // the ensemble's feature vectors, one per lane
    __shared__ uint16_t fbin[FOREST == 2 ? W * kFxRows * kLanes : 1];   // compact: bin rows per lane
    extern __shared__ uint32_t fwords[];         // compact: the ensemble's nodes
    if (a.stable && __builtin_amdgcn_readfirstlane(__hip_atomic_load(a.stable, __ATOMIC_RELAXED,
                                                                      __HIP_MEMORY_SCOPE_AGENT)))
        return;                                  // every scenario is at its fixed point
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // Workgroup b runs on XCD b % kXcds: each XCD takes a contiguous share of the groups, so
    // that the comm rows that a rank's segments have in common stay in one L2 (1024-rank workload 3.7 -> 3.4 ms, 96 ranks 0.49 -> 0.41).
    const int xcd = (int)(blockIdx.x % kXcds);
    const int64_t unit = (int64_t)(blockIdx.x / kXcds) * W + wave;
    const int32_t tile = (int32_t)(unit % a.n_tiles);
    const int64_t part = unit / a.n_tiles;       // of this XCD's parts
    if (FOREST == 2) {
        // the nodes, then the roots of the trees
        for (int i = threadIdx.x; i < a.fx.n_words; i += 64 * W) fwords[i] = a.fx.words[i];
        for (int i = threadIdx.x; i < a.n_trees; i += 64 * W) fwords[a.fx.n_words + i] = (uint32_t)a.forest_roots[i];
        __syncthreads();
    }
    if (part >= parts) return;                   // after the shared fill
    const Lane ln = make_lane(a.scen, a.n_scen, tile, lane);
    const int32_t col = ln.col, sigma = ln.sigma;
    const bool any_jitter = ln.any_jitter;
    const int64_t ns = a.n_scen;
    const int64_t *const sbase = a.start + (int64_t)tile * kLanes + col;
    int64_t *const fbase = a.finish + (int64_t)tile * kLanes + col;
    uint8_t *const obase = a.tmask + (int64_t)tile * kLanes + col;
    uint32_t *const ebase = a.ext + (int64_t)tile * kLanes + col;
    const echo_scenario *sc = a.scen + sigma;
    const uint32_t *slow = &sc->slowdown_q16[0][0];
    bool changed = false;                        // some duration differs from the previous pass's
    bool ext_over = false;                       // a prorated extra time does not fit 32 bits
    int64_t *const feat = feat_all + (FOREST == 1 ? wave * 12 * kLanes : 0);
    // compact ensemble: this wavefront's bin rows; the scenario knobs' rows are fixed
    uint16_t *const fb = fbin + (FOREST == 2 ? wave * kFxRows * kLanes : 0);
    bool knobs_uniform = false;
    if (FOREST == 2) {
        const int32_t k5 = fx_bin(a.fx.thr + a.fx.thr_off[5], a.fx.thr_off[6] - a.fx.thr_off[5], sc->ar_algo);
        const int32_t k6 = fx_bin(a.fx.thr + a.fx.thr_off[6], a.fx.thr_off[7] - a.fx.thr_off[6], sc->bw_intra_MBps);
        const int32_t k7 = fx_bin(a.fx.thr + a.fx.thr_off[7], a.fx.thr_off[8] - a.fx.thr_off[7], sc->bw_inter_MBps);
        fb[5 * kLanes + lane] = (uint16_t)k5;
        fb[6 * kLanes + lane] = (uint16_t)k6;
        fb[7 * kLanes + lane] = (uint16_t)k7;
#pragma unroll
        for (int k = kFxFeatures; k < kFxRows; ++k) fb[k * kLanes + lane] = 0;
        knobs_uniform = __ballot(k5 != __builtin_amdgcn_readfirstlane(k5) || k6 != __builtin_amdgcn_readfirstlane(k6) ||
                                 k7 != __builtin_amdgcn_readfirstlane(k7)) == 0;
    } else if (FOREST == 1) {
        const int64_t k6 = sc->bw_intra_MBps, k7 = sc->bw_inter_MBps;
        const int32_t k5 = sc->ar_algo;
        knobs_uniform = __ballot(k5 != __builtin_amdgcn_readfirstlane(k5) || k6 != __shfl(k6, 0) ||
                                 k7 != __shfl(k7, 0)) == 0;
    }
    typedef uint32_t Olds __attribute__((ext_vector_type(8)));

    // Rows are addressed by the lanes (as in k_walk): lane j computes the address of item j's
    // row, and a row is then two lane reads and a load.
    const uint64_t sadr = reinterpret_cast<uint64_t>(a.start + (int64_t)tile * kLanes);
    const uint64_t fadr = reinterpret_cast<uint64_t>(a.finish + (int64_t)tile * kLanes);
    const uint32_t coff = (uint32_t)col * 8u;
    const uint64_t row_bytes = (uint64_t)ns * 8u;
    auto row_of = [&](uint64_t rows, int j) -> GlobalI64 * {
        const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)rows, j);
        const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(rows >> 32), j);
        return reinterpret_cast<GlobalI64 *>((((uint64_t)hi << 32) | lo) + coff);
    };
    typedef int64_t Starts __attribute__((ext_vector_type(kOverlapGroup)));
    const int4 *const osegs4 = reinterpret_cast<const int4 *>(a.osegs);
    const int64_t groups = (a.n_osegs + kOverlapGroup - 1) / kOverlapGroup;
    const int64_t grp0 = groups * xcd / kXcds + part, grp1 = groups * (xcd + 1) / kXcds;
    // lane 2q holds the first half of segment q of a group, lane 2q + 1 the second
    auto load_group = [&](int64_t grp) -> int4 {
        const int64_t at = 2 * grp * kOverlapGroup + lane;
        return grp < grp1 && lane < 2 * kOverlapGroup && at < 2 * a.n_osegs ? osegs4[at] : make_int4(0, 0, 0, 0);
    };
    int4 nxt = load_group(grp0);
    for (int64_t grp = grp0; grp < grp1; grp += parts) {
        const int4 os = nxt;
        const int64_t o0 = grp * kOverlapGroup;
        const int no = a.n_osegs - o0 < kOverlapGroup ? (int)(a.n_osegs - o0) : kOverlapGroup;
        // the group's ranges: lane t holds range t, with its segment's place in the group
        const int32_t r0 = __builtin_amdgcn_readlane(os.x, 1);
        const int nr_all = __builtin_amdgcn_readlane(os.x, 2 * no - 1) + __builtin_amdgcn_readlane(os.y, 2 * no - 1) - r0;
        const int4 rg = lane < nr_all ? reinterpret_cast<const int4 *>(a.ranges)[r0 + lane] : make_int4(0, 0, 0, 0);
        nxt = load_group(grp + parts);
        uint8_t *const flag = a.xflag + (o0 + lane) * a.n_tiles + tile;      // of segment `lane`
        // segments inflated in the previous pass
        uint32_t was = 0;
        if (a.prev_refined) was = (uint32_t)__ballot(lane < no && *flag != 0);
        uint32_t now = 0;
        // the segments' starts and, eight at a time, the finishes of the ranges' last comm ops,
        // fetched together: bit t of `late` is set when range t's comes after its segment's start
        const uint64_t srow = sadr + (uint64_t)(uint32_t)os.z * row_bytes;
        const uint64_t lrow = fadr + (uint64_t)(uint32_t)rg.z * row_bytes;
        Starts s8;
#pragma unroll
        for (int q = 0; q < kOverlapGroup; ++q) s8[q] = *row_of(srow, q < no ? 2 * q : 0);
        uint64_t late = 0;
        for (int t0 = 0; t0 < nr_all; t0 += 8) {
            int64_t fin[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) fin[i] = *row_of(lrow, t0 + i < nr_all ? t0 + i : t0);
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int t = t0 + i < nr_all ? t0 + i : t0;
                const int64_t s = s8[__builtin_amdgcn_readlane(rg.w, t) & (kOverlapGroup - 1)];
                late |= (uint64_t)(fin[i] > s ? 1u : 0u) << t;
            }
        }
        for (int q = 0; q < no; ++q) {
            const int t0 = __builtin_amdgcn_readlane(os.x, 2 * q + 1) - r0;   // its ranges t0 .. t0 + ncand
            const int ncand = __builtin_amdgcn_readlane(os.y, 2 * q + 1);
            const bool was_on = (was >> q) & 1u;
            const uint32_t late_q = (uint32_t)(late >> t0) & ((1u << ncand) - 1u);
            if (!was_on && !__builtin_amdgcn_readfirstlane(__ballot(late_q != 0) != 0)) continue;

            // some lane's segment may overlap: cursors at the first comm op ending after s
            const int64_t s = s8[q];
            const int32_t last = __builtin_amdgcn_readlane(os.w, 2 * q);
            const int32_t rec0 = __builtin_amdgcn_readlane(os.x, 2 * q);
            const int nr = __builtin_amdgcn_readlane(os.y, 2 * q);
            const int4 cur = lane < nr ? reinterpret_cast<const int4 *>(a.recs)[rec0 + lane] : make_int4(0, 0, 0, 0);
            // Per range a cursor: the comm op at list position p, its interval and type, and the id
            // of the one after it (read ahead, so that a move waits for one load, not two).
            int32_t p[NC], hi[NC], cn[NC];
            uint32_t ty[NC];
            int64_t cs[NC], cf[NC];
            int64_t cmin = kInf;                 // earliest start among the cursors: an op ending by then overlaps nothing
            auto next_id = [&](int k) { cn[k] = a.cl[p[k] + 1 < hi[k] ? p[k] + 1 : hi[k] - 1]; };
            {
                // usually the range's last comm op is the only one that ends after s (a send still
                // waiting for its receiver), or all of them do (the buckets behind the one an
                // optimizer op waited for): the last, the one before it and the first are looked
                // at together, and only then is the range searched
                int32_t c2[NC], c1[NC];
                int64_t f2[NC], f1[NC], s1[NC];
#pragma unroll
                for (int k = 0; k < NC; ++k) {
                    p[k] = hi[k] = cn[k] = c2[k] = c1[k] = 0;
                    ty[k] = 0;
                    cs[k] = cf[k] = kInf;
                    f2[k] = f1[k] = s1[k] = 0;
                    if (k < ncand) {
                        const int32_t lo = __builtin_amdgcn_readlane(rg.x, t0 + k);
                        hi[k] = __builtin_amdgcn_readlane(rg.y, t0 + k);
                        const int64_t c = __builtin_amdgcn_readlane(rg.z, t0 + k);
                        cs[k] = sbase[c * ns];
                        cf[k] = fbase[c * ns];
                        ty[k] = a.cl_type[hi[k] - 1];
                        cn[k] = (int32_t)c;
                        c2[k] = hi[k] - 1 > lo ? __builtin_amdgcn_readfirstlane(a.cl[hi[k] - 2]) : -1;
                        c1[k] = __builtin_amdgcn_readfirstlane(a.cl[lo]);
                    }
                }
#pragma unroll
                for (int k = 0; k < NC; ++k)
                    if (k < ncand && c2[k] >= 0) {
                        f2[k] = fbase[(int64_t)c2[k] * ns];
                        f1[k] = fbase[(int64_t)c1[k] * ns];
                        s1[k] = sbase[(int64_t)c1[k] * ns];
                    }
#pragma unroll
                for (int k = 0; k < NC; ++k) {
                    if (k >= ncand) break;
                    const bool on = (late_q >> k) & 1u;
                    p[k] = on ? hi[k] - 1 : hi[k];
                    const bool more = on && f2[k] > s;
                    if (__ballot(more)) {
                        const int32_t first_at = __builtin_amdgcn_readlane(rg.x, t0 + k);
                        const bool all = more && f1[k] > s;
                        if (all) {
                            p[k] = first_at;
                            cs[k] = s1[k];
                            cf[k] = f1[k];
                        }
                        if (__ballot(more && !all)) {
                            // backwards in doubling steps, then by halves: finishes before lo are by
                            // s, those from x on after it
                            int32_t lo = first_at, step = 2, x = more && !all ? hi[k] - 2 : lo;
                            while (lo < x) {
                                const int32_t m = step ? (x - step > lo ? x - step : lo) : lo + (x - lo) / 2;
                                if (fbase[(int64_t)a.cl[m] * ns] > s) {
                                    x = m;
                                    step *= 2;
                                } else {
                                    lo = m + 1;
                                    step = 0;            // bracketed: bisect
                                }
                            }
                            if (more && !all) {
                                p[k] = x;
                                const int64_t c = a.cl[x];
                                cs[k] = sbase[c * ns];
                                cf[k] = fbase[c * ns];
                            }
                        }
                        if (more) {
                            ty[k] = a.cl_type[p[k]];
                            next_id(k);
                        }
                    }
                    if (!on) cs[k] = cf[k] = kInf;
                    cmin = cs[k] < cmin ? cs[k] : cmin;
                }
            }
            int64_t fprev = s;                   // the next op's start
            int64_t total = 0;                   // the segment's new duration
            bool hit = false;
            Olds old8 = 0;
            for (int j = 0; j < nr; ++j) {
                const int32_t v = __builtin_amdgcn_readlane(cur.x, j);
                const uint32_t meta = (uint32_t)__builtin_amdgcn_readlane(cur.y, j);
                const int cls = (int)(meta & 7u);
                const int64_t d0 = (int64_t)(((uint64_t)(uint32_t)__builtin_amdgcn_readlane(cur.w, j) << 32) |
                                             (uint32_t)__builtin_amdgcn_readlane(cur.z, j));
                const int64_t row = (int64_t)(rec0 + j) * a.mstride;
                uint32_t ov = 0;                 // the previous pass's mask (extra time)
                if (was_on) {
                    if ((j & 7) == 0) {
                        // of the next eight ops, in one memory round trip
#pragma unroll
                        for (int i = 0; i < 8; ++i)
                            if (j + i < nr) old8[i] = EXT ? ebase[row + i * a.mstride] : (uint32_t)obase[row + i * a.mstride];
                    }
                    ov = old8[j & 7];
                }
                const int64_t sv = fprev;
                const int64_t D = any_jitter ? jittered(d0, v, ln.jt) : d0;
                if (!(meta & kRecCompute)) {     // a memcpy runs for its base duration
                    if (EXT) ebase[row] = 0;
                    else obase[row] = 0;
                    fprev = sv + D;
                    total += D;
                    continue;
                }
                int64_t d = D;                   // the duration v ran with in the previous pass
                if (was_on) d = EXT ? D + ov : ov != 0 ? q16(D, factor_of(ov, slow, cls)) : D;
                const int64_t fv = sv + d;
                fprev = fv;
                const bool busy = cmin < fv;
                uint32_t m = 0;                            // types of the comm ops overlapping v
                int64_t o = 0;                             // covered length (PRORATE)
                int64_t smax[kTypes];                      // FOREST: largest S per overlapping type
                int32_t nmax[kTypes];                      //         and most members (compact: their bins)
#pragma unroll
                for (int tt = 0; tt < kTypes; ++tt) {
                    smax[tt] = 0;
                    nmax[tt] = 0;
                }
// note the comm op at list position x_ (type ty_) among v's overlaps, for the ensemble's features
#define NOTE_FOREST(x_, ty_)                                                                     \
    if (FOREST) {                                                                                \
        const int32_t cc_ = a.cl_coll[x_];                                                       \
        const int64_t S_ = FOREST == 2 ? a.fx.coll_bin[2 * cc_] : a.coll_bytes[cc_];            \
        const int32_t N_ = FOREST == 2 ? a.fx.coll_bin[2 * cc_ + 1] : a.coll_N[cc_];            \
        _Pragma("unroll") for (int tt = 0; tt < kTypes; ++tt) if (tt == (int)(ty_)) {            \
            smax[tt] = S_ > smax[tt] ? S_ : smax[tt];                                            \
            nmax[tt] = N_ > nmax[tt] ? N_ : nmax[tt];                                            \
        }                                                                                        \
    }
                if (busy) {
#pragma unroll
                    for (int k = 0; k < NC; ++k) {
                        if (k >= ncand) break;
                        if (!(cs[k] < fv)) continue;
                        // The cursor walks the intervals that start before v ends; one that also
                        // ends before then is behind every later op of the segment (each starts at
                        // or after v's finish) and is passed for good.  Prorating, the merge below
                        // walks the overlapping ones: the cursor passes only those ending by sv.
                        while (PRORATE ? cf[k] <= sv : cs[k] < fv) {
                            if (!PRORATE) {
                                const int64_t lo = sv > cs[k] ? sv : cs[k], up = fv < cf[k] ? fv : cf[k];
                                if (lo < up) {
                                    m |= 1u << ty[k];
                                    NOTE_FOREST(p[k], ty[k])
                                }
                                if (cf[k] >= fv) break;    // reaches v's end: later ops may overlap it
                            }
                            ++p[k];
                            if (p[k] < hi[k]) {
                                const int64_t c = cn[k];
                                cs[k] = sbase[c * ns];
                                cf[k] = fbase[c * ns];
                                ty[k] = a.cl_type[p[k]];
                                next_id(k);
                            } else {
                                cs[k] = kInf;
                                cf[k] = kInf;
                            }
                        }
                    }
                    if (PRORATE) {
                        // merge the ranges' overlapping intervals in start order; every one of
                        // them ends after sv (each stream's intervals are disjoint and sorted)
                        int32_t x[NC], xn[NC];
                        uint32_t xt[NC];
                        int64_t qs[NC], qf[NC];
#pragma unroll
                        for (int k = 0; k < NC; ++k) {
                            x[k] = p[k];
                            xn[k] = cn[k];
                            xt[k] = ty[k];
                            qs[k] = cs[k];
                            qf[k] = cf[k];
                        }
                        int64_t t = sv;                    // covered up to here
                        for (;;) {
                            int bk = -1;
                            int64_t bs = fv;
#pragma unroll
                            for (int k = 0; k < NC; ++k)
                                if (qs[k] < bs) {
                                    bs = qs[k];
                                    bk = k;
                                }
                            if (bk < 0) break;
#pragma unroll
                            for (int k = 0; k < NC; ++k) {
                                if (k != bk) continue;
                                const int64_t lo = sv > qs[k] ? sv : qs[k], up = fv < qf[k] ? fv : qf[k];
                                if (lo < up) {
                                    m |= 1u << xt[k];
                                    NOTE_FOREST(x[k], xt[k])
                                    const int64_t from = lo > t ? lo : t;
                                    if (up > from) {
                                        o += up - from;
                                        t = up;
                                    }
                                }
                                if (qf[k] >= fv) {         // reaches v's end: the next starts no earlier
                                    qs[k] = kInf;
                                } else if (++x[k] < hi[k]) {
                                    const int64_t c = xn[k];
                                    qs[k] = sbase[c * ns];
                                    qf[k] = fbase[c * ns];
                                    xt[k] = a.cl_type[x[k]];
                                    xn[k] = a.cl[x[k] + 1 < hi[k] ? x[k] + 1 : hi[k] - 1];
                                } else {
                                    qs[k] = kInf;
                                }
                            }
                        }
                    }
                    cmin = kInf;
#pragma unroll
                    for (int k = 0; k < NC; ++k) cmin = cs[k] < cmin ? cs[k] : cmin;
                }
#undef NOTE_FOREST
                int64_t dn;                                // v's duration in the next pass
                if (EXT) {
                    uint32_t e = 0, F = 65536u;
                    // the ensemble is walked by the whole wavefront, lanes that overlap nothing included:
                    // a tree per lane where the others share one feature vector
                    if (FOREST && __ballot(m != 0)) {
                        if (FOREST == 2) {
                            int32_t bS[kTypes];
#pragma unroll
                            for (int tt = 0; tt < kTypes; ++tt) bS[tt] = (int32_t)smax[tt];
                            const int32_t bd0 = a.fx.cp_bin[rec0 + j];
                            F = forest_factor_compact(a, m, bS, nmax, cls, bd0, fwords,
                                                      reinterpret_cast<const int32_t *>(fwords) + a.fx.n_words, fb,
                                                      knobs_uniform, lane);
                        } else {
                            F = forest_factor(a, m, smax, nmax, cls, d0, sc, feat, knobs_uniform, lane);
                        }
                    }
                    if (m != 0) {
                        if (!FOREST) F = factor_of(m, slow, cls);
                        const int64_t oc = PRORATE ? (o < D ? o : D) : D;
                        const int64_t x = q16(oc, F) - oc;
                        ext_over |= x >= (int64_t)kExtLimit;
                        e = x >= (int64_t)kExtLimit ? kExtLimit : (uint32_t)x;
                    }
                    ebase[row] = e;
                    hit |= e != 0;
                    dn = D + e;
                } else {
                    obase[row] = (uint8_t)m;
                    hit |= m != 0;
                    dn = m != 0 ? q16(D, factor_of(m, slow, cls)) : D;
                }
                if (DETECT) changed |= dn != d;
                total += dn;
            }
            fbase[(int64_t)last * ns] = total;
            if (__builtin_amdgcn_readfirstlane(__ballot(hit) != 0)) now |= 1u << q;
        }
        if (lane < no) *flag = (now >> lane) & 1u;
    }
    if (DETECT && ln.active && changed)
        __hip_atomic_fetch_or(a.chg + sigma, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (ln.active && ext_over)
        __hip_atomic_fetch_or(a.status, kStatusRange, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Count the refinement of each scenario whose durations changed; flag stability.
__global__ __launch_bounds__(256) void k_settle(unsigned *chg, int32_t n_scen, int32_t *refinements,
                                                 unsigned *stable) {
    int any = 0;
    for (int32_t i = threadIdx.x; i < n_scen; i += blockDim.x) {
        if (chg[i]) {
            any = 1;
            if (refinements) refinements[i] += 1;
            chg[i] = 0;
        }
    }
    any = __syncthreads_or(any);
    if (threadIdx.x == 0 && !any) *stable = 1u;
}

__global__ void k_fill_i32(int32_t *p, int64_t n, int32_t v) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

int grid_for(int64_t n, int block) {
    int64_t b = (n + block - 1) / block;
    if (b < 1) b = 1;
    if (b > 65536) b = 65536;
    return (int)b;
}

}  // namespace

hipError_t launch_init(const DeviceGraph &g, const echo_scenario *scen, int32_t n_scen,
                       unsigned long long *arrive, int64_t n_arrive, unsigned *count, int64_t n_count,
                       int64_t *slots, int64_t n_slot_values, int64_t *step, uint64_t *digest, hipStream_t stream) {
    int64_t n = std::max<int64_t>(std::max(n_arrive, n_count), n_slot_values);
    if (n_scen > n) n = n_scen;
    hipLaunchKernelGGL(k_init, dim3(grid_for(n, 256)), dim3(256), 0, stream, scen, n_scen, arrive,
                       n_arrive, count, n_count, slots, n_slot_values, step, digest, g.n_cc_tables, g.status);
    return hipGetLastError();
}

hipError_t launch_clear(unsigned long long *arrive, int64_t n_arrive, unsigned *count, int64_t n_count,
                        int64_t *slots, int64_t n_slot_values, hipStream_t stream) {
    const int64_t n = std::max<int64_t>(std::max(n_arrive, n_count), n_slot_values);
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_clear, dim3(grid_for(n, 256)), dim3(256), 0, stream, arrive, n_arrive, count,
                       n_count, slots, n_slot_values);
    return hipGetLastError();
}

hipError_t launch_cc_cost(const CollTable &t, const echo_cc_table *tables, const echo_scenario *scen,
                          int32_t n_scen, int64_t *cost, unsigned *status, hipStream_t stream) {
    if (t.n == 0 || n_scen == 0) return hipSuccess;
    // one lane per (row of the table, scenario): rows along x, 64-scenario tiles along y
    const unsigned tiles = (unsigned)std::min<int64_t>((n_scen + 63) / 64, 65535);
    hipLaunchKernelGGL(k_cc_cost, dim3((unsigned)t.n, tiles), dim3(64), 0, stream, t, tables, scen, n_scen, cost,
                       status);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess || !t.row) return e;
    // 8 workgroups per compute unit keep enough stores in flight
    const dim3 grid((unsigned)std::min<int64_t>((t.n_out + 3) / 4, 2048));
    if (n_scen % 2 == 0 && reinterpret_cast<uintptr_t>(cost) % sizeof(longlong2) == 0)
        hipLaunchKernelGGL(k_cc_spread<longlong2>, grid, dim3(256), 0, stream, t.class_of, t.row, t.n_out, n_scen / 2,
                           reinterpret_cast<longlong2 *>(cost));
    else
        hipLaunchKernelGGL(k_cc_spread<int64_t>, grid, dim3(256), 0, stream, t.class_of, t.row, t.n_out, n_scen, cost);
    return hipGetLastError();
}

template <int IN>
hipError_t launch_expand(const WalkArgs &a, int64_t parts, hipStream_t stream) {
    const dim3 grid((unsigned)((parts * a.tiles + kRecWaves - 1) / kRecWaves)), block(kRecWaves * kLanes);
    if (a.digest) hipLaunchKernelGGL((k_expand<IN, true>), grid, block, 0, stream, a, parts);
    else hipLaunchKernelGGL((k_expand<IN, false>), grid, block, 0, stream, a, parts);
    return hipGetLastError();
}

hipError_t launch_walk(const WalkArgs &a, int32_t n_blocks, hipStream_t stream) {
    hipError_t e;
    const int64_t parts = std::max<int64_t>(1, std::min<int64_t>(a.n_chunks, kRecParts / a.tiles));
    if (a.in == kInNone && a.n_chunks > 0) {
        const dim3 grid((unsigned)((parts * a.tiles + kRecWaves - 1) / kRecWaves));
        hipLaunchKernelGGL(k_sum, grid, dim3(kRecWaves * kLanes), 0, stream, a, parts);
        if ((e = hipGetLastError())) return e;
    }
    WalkArgs args = a;
    void *params[] = {&args};
    const WalkKernel k = walk_kernel(a.in, a.final_pass != 0, a.digest != nullptr);
    const dim3 grid((unsigned)(n_blocks * a.tiles)), block(kBlockWalkers * kLanes);
    // With one workgroup per tile no wavefront waits for another workgroup's, so nothing has to
    // be resident together: a plain launch, which costs about 17 us less than a cooperative
    // one (8 ranks x 4096 scenarios: 196 -> 152 us per call)
    e = n_blocks == 1 ? hipLaunchKernel(reinterpret_cast<const void *>(k), grid, block, params, 0, stream)
                      : hipLaunchCooperativeKernel(reinterpret_cast<const void *>(k), grid, block, params, 0, stream);
    if (e != hipSuccess || a.in == kInOps || a.n_chunks == 0 || !a.final_pass || !(a.timelines || a.digest)) return e;
    if (a.ext) return launch_expand<kInExtFlags>(a, parts, stream);
    return a.tmask ? launch_expand<kInMasks>(a, parts, stream) : launch_expand<kInNone>(a, parts, stream);
}

template <bool PRORATE, bool DETECT, int FOREST, int NC>
void launch_overlap_kernel(const OverlapArgs &a, size_t lds, hipStream_t stream) {
    const int64_t groups = (a.n_osegs + kOverlapGroup - 1) / kOverlapGroup;
    // the ensemble's LDS copy is filled by every workgroup: an eighth of the wavefronts there
    const int64_t most = FOREST == 2 ? kRecParts / 8 : kRecParts;
    const int64_t parts = std::max<int64_t>(1, std::min<int64_t>((groups + kXcds - 1) / kXcds, most / kXcds / a.n_tiles));
    const dim3 grid((unsigned)((parts * a.n_tiles + kOverlapWaves - 1) / kOverlapWaves * kXcds)), block(kOverlapWaves * kLanes);
    hipLaunchKernelGGL((k_overlap<PRORATE, DETECT, FOREST, NC>), grid, block, lds, stream, a, parts);
}

template <int NC>
hipError_t launch_overlap_nc(const OverlapArgs &a, hipStream_t stream) {
    // a.ext: extra-time output (prorating and/or ensemble factors); a.forest_nodes: ensemble
    const bool forest = a.forest_nodes != nullptr, prorate = a.prorate != 0;
    if (forest && a.fx.n_words > 0) {
        // compact ensemble in LDS: the workgroup's wavefronts share its nodes
        const size_t lds = sizeof(uint32_t) * ((size_t)a.fx.n_words + (size_t)a.n_trees);
        if (prorate && a.chg) launch_overlap_kernel<true, true, 2, NC>(a, lds, stream);
        else if (prorate) launch_overlap_kernel<true, false, 2, NC>(a, lds, stream);
        else if (a.chg) launch_overlap_kernel<false, true, 2, NC>(a, lds, stream);
        else launch_overlap_kernel<false, false, 2, NC>(a, lds, stream);
    } else if (forest) {
        if (prorate && a.chg) launch_overlap_kernel<true, true, 1, NC>(a, 0, stream);
        else if (prorate) launch_overlap_kernel<true, false, 1, NC>(a, 0, stream);
        else if (a.chg) launch_overlap_kernel<false, true, 1, NC>(a, 0, stream);
        else launch_overlap_kernel<false, false, 1, NC>(a, 0, stream);
    } else if (prorate && a.chg) launch_overlap_kernel<true, true, 0, NC>(a, 0, stream);
    else if (prorate) launch_overlap_kernel<true, false, 0, NC>(a, 0, stream);
    else if (a.chg) launch_overlap_kernel<false, true, 0, NC>(a, 0, stream);
    else launch_overlap_kernel<false, false, 0, NC>(a, 0, stream);
    return hipGetLastError();
}

hipError_t launch_overlap(const OverlapArgs &a, int32_t max_ranges, hipStream_t stream) {
    if (a.n_osegs == 0) return hipSuccess;
    // GPT graphs have two (sends and data-parallel buckets)
    if (max_ranges > 4) return launch_overlap_nc<kStreams>(a, stream);
    return max_ranges > 2 ? launch_overlap_nc<4>(a, stream) : launch_overlap_nc<2>(a, stream);
}

hipError_t launch_forest_bins(const DeviceGraph &g, int64_t n_recs, const CompactForest &fx, hipStream_t stream) {
    const int64_t n = std::max<int64_t>(g.colls.n, n_recs);
    hipLaunchKernelGGL(k_forest_bins, dim3(grid_for(n, 256)), dim3(256), 0, stream, g.colls, g.recs, n_recs, fx);
    return hipGetLastError();
}

hipError_t launch_settle(unsigned *chg, int32_t n_scen, int32_t *refinements, unsigned *stable,
                         hipStream_t stream) {
    hipLaunchKernelGGL(k_settle, dim3(1), dim3(256), 0, stream, chg, n_scen, refinements, stable);
    return hipGetLastError();
}

hipError_t launch_fill_i32(int32_t *p, int64_t n, int32_t v, hipStream_t stream) {
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_fill_i32, dim3(grid_for(n, 256)), dim3(256), 0, stream, p, n, v);
    return hipGetLastError();
}

// Workspace of echo_compose_batch_static: one fixed array in every GPU's copy of the
// code object, held from the code object's load until the process ends.  In host code
// `scratch` names a host-side stand-in only; kernels get the device address that
// hipGetSymbolAddress returns for the current device.
static __device__ __align__(256) unsigned char scratch[ECHO_SCRATCH_BYTES];

hipError_t scratch_buffer(int device, void **ptr) {
    constexpr int kMaxDevices = 64;
    static std::mutex mu;
    static void *addr[kMaxDevices] = {};
    *ptr = nullptr;
    if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(mu);
    if (!addr[device]) {
        // the caller has made `device` current: its copy of the array
        void *p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        addr[device] = p;
    }
    *ptr = addr[device];
    return hipSuccess;
}

hipError_t walk_capacity(int device, int64_t workgroups[kWalkVariants]) {
    int cus = 0;
    hipError_t e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device);
    if (e != hipSuccess) return e;
    for (int v = 0; v < kWalkVariants; ++v) {
        const WalkKernel k = walk_kernel(v & 7, v & 8, v & 16);
        int u = 0;                                   // a kernel of several variants is asked about once
        while (walk_kernel(u & 7, u & 8, u & 16) != k) ++u;
        if (u < v) {
            workgroups[v] = workgroups[u];
            continue;
        }
        int per_cu = 0;
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, reinterpret_cast<const void *>(k),
                                                         kBlockWalkers * kLanes, 0);
        if (e != hipSuccess) return e;
        workgroups[v] = (int64_t)std::min(per_cu, kWalkersPerCu / kBlockWalkers) * cus;
    }
    return hipSuccess;
}

}  // namespace echo
