// Bounded-delay SGD (gfx950, wave64), the relaxation of Sec. 7: an
// iteration may read a partition once the write of iteration alpha - 1 -
// delay to it is done (Asynchronous Read Constraint), instead of waiting for
// every earlier writer.  The execution computed here reads as early as that
// allows: example alpha reads, for each of its features, the value written
// by the latest earlier example before alpha - delay (the initial weight if
// there is none), and every example's update is applied in example order to
// each of its features, w = fma(-s, x, w), so no update is lost.  delay = 0
// is the sequential computation.
//
// A first pass finds each stored entry's read source -- the previous entry
// on its feature, followed back past the entries of the last `delay`
// examples -- and its next writer.  Two executions follow.
//
// Windowed (one block): examples in windows of W = delay + 1.  Every read
// of window k has its source in window k - 1 or earlier, so the block holds
// the values written by the last windows in LDS and older ones in w: it takes
// window k's reads, forms the W steps (a wave per example), then runs each
// feature's writes through the window in example order.  Chosen when a
// window's entries fit the block's LDS.  Passes over all windows before it lay
// every window's entries out by feature, in example order (an entry's place),
// so that a feature's chain is a stretch of consecutive places.  (Wide
// windows are staged and run by all waves together, without those passes.)
//
// Sync-free (otherwise): every stored entry owns a 64-bit word (the value it
// wrote, its own index as the tag); waves take examples in index order; an
// example waits for its read sources' words, computes its step, then waits
// for each entry's previous writer and publishes its own words.  The
// earliest unfinished example never waits on a later one.  A last pass
// copies each feature's final value (the entry nothing overwrites) into w.
#include <climits>

#include "pdb_math.h"
#include "pdb_words.h"

namespace pdbk {

namespace {

constexpr int kSWaves = kBlock / kWave;
constexpr int kWinCap = 2048;          // entries (and examples) of a window held in LDS
constexpr int kWinWide = kWinCap * 3 / 4;  // wider windows: k_stale_wide
constexpr int kWinThreads = 1024;
constexpr int kWinWaves = kWinThreads / kWave;

struct StaleWs {
    Ctrl *ctrl;
    unsigned long long *words;  // [nnz] sync-free: (value, entry); windowed: chain
    int32_t *rd;                // [nnz] read source, -1 = the initial weight
    int32_t *overwritten;       // [nnz] sync-free: 1 when a later entry writes the same
                                // feature; windowed: the entry's place in its window
    int32_t *next;              // [nnz] windowed: where the entry's read is taken from, or in
                                // wide windows the next entry on the feature, -1 = none
    size_t total;
};

__device__ __forceinline__ int64_t cdiv_dev(int64_t a, int64_t b) { return (a + b - 1) / b; }

StaleWs stale_layout(void *base, int64_t nnz) {
    StaleWs w{};
    char *p = static_cast<char *>(base);
    size_t off = 0;
    auto take = [&](int64_t bytes) {
        char *r = p ? p + off : nullptr;
        off += (size_t)align_up(bytes);
        return r;
    };
    const int64_t z = std::max<int64_t>(nnz, 1);
    w.ctrl = reinterpret_cast<Ctrl *>(take(sizeof(Ctrl)));
    w.words = reinterpret_cast<unsigned long long *>(take(8 * z));
    w.rd = reinterpret_cast<int32_t *>(take(4 * z));
    w.overwritten = reinterpret_cast<int32_t *>(take(4 * z));
    w.next = reinterpret_cast<int32_t *>(take(4 * z));
    w.total = off;
    return w;
}

__global__ void k_stale_clear(unsigned long long *__restrict__ words,
                              int32_t *__restrict__ overwritten, int64_t nnz) {
    for (int64_t q = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; q < nnz;
         q += (int64_t)gridDim.x * blockDim.x) {
        words[q] = word_pack(0.0f, -1);
        overwritten[q] = 0;
    }
}

// What the choice of an execution looks at: examples (after the first of m)
// that share no feature with the example before them, few on chain-like inputs,
// where the windowed execution pays; and the largest number of entries in a
// window of W of the n examples.  One launch for both, since the host waits for
// them: 1,000 examples of 10 of 100,000 features, delay 8, 86 us with a launch each, 83 with one.
constexpr int kShapeBlocks = 4096;  // that look at windows
__global__ __launch_bounds__(kBlock) void k_stale_shape(const int64_t *__restrict__ row_ptr,
                                                        int64_t n, int64_t W, int64_t m,
                                                        const int32_t *__restrict__ prev,
                                                        Ctrl *ctrl) {
    const int lane = lane_id();
    const int64_t nw = (int64_t)gridDim.x * kSWaves;
    int breaks = 0;
    for (int64_t i = 1 + blockIdx.x * (int64_t)kSWaves + wave_in_block(); i < m; i += nw) {
        const int64_t lo = row_ptr[i - 1], b = row_ptr[i], e = row_ptr[i + 1];
        bool found = false;
        for (int64_t p = b + lane; p < e && !found; p += kWave) found = prev[p] >= lo;
        if (__ballot(found) == 0ull) ++breaks;
    }
    if (lane == 0 && breaks) atomicAdd(&ctrl->chain_breaks, breaks);
    if (blockIdx.x >= kShapeBlocks) return;
    const int64_t nwin = cdiv_dev(n, W);
    long long best = 0;
    for (int64_t k = blockIdx.x * (int64_t)kBlock + threadIdx.x; k < nwin;
         k += (int64_t)min((int)gridDim.x, kShapeBlocks) * kBlock)
        best = max(best, (long long)(row_ptr[min(n, (k + 1) * W)] - row_ptr[k * W]));
    if (best > 0) atomicMax(&ctrl->max_width, best);
}

__global__ void k_stale_ctrl_zero(Ctrl *c) {
    int *w = reinterpret_cast<int *>(c);
    for (int i = threadIdx.x; i < (int)(sizeof(Ctrl) / sizeof(int)); i += blockDim.x) w[i] = 0;
}

// Read sources, one wave per example a: the previous entry on the feature,
// then back while it belongs to one of the examples a - delay .. a - 1 (their
// entries are the CSR positions from row_ptr[a - delay] on).  Also marks
// every previous entry as overwritten.
__global__ __launch_bounds__(kBlock) void k_stale_sources(const int64_t *__restrict__ row_ptr,
                                                          int64_t n,
                                                          const int32_t *__restrict__ prev,
                                                          int64_t delay, int32_t *__restrict__ rd,
                                                          int32_t *__restrict__ overwritten) {
    const int lane = lane_id();
    const int64_t nw = (int64_t)gridDim.x * kSWaves;
    for (int64_t a = blockIdx.x * (int64_t)kSWaves + wave_in_block(); a < n; a += nw) {
        const int64_t b = row_ptr[a], e = row_ptr[a + 1];
        const bool all_in_window = a - delay <= 0;
        const int64_t lim = all_in_window ? 0 : row_ptr[a - delay];
        for (int64_t q = b + lane; q < e; q += kWave) {
            const int32_t pq = prev[q];
            if (pq >= 0) overwritten[pq] = 1;
            int32_t k = all_in_window ? -1 : pq;
            while (k >= 0 && (int64_t)k >= lim) k = prev[k];
            rd[q] = k;
        }
    }
}

// Examples are dealt to the waves in turn (wave k of W runs examples k,
// k + W, ...); the grid is launched cooperatively, so the earliest
// unfinished example is always being worked on.  A shared ticket counter
// would serve one request about every 200 ns.  An example of up to 2 x 64
// entries issues the loads and polls of both chunks together.
template <int LOSS, bool VAL>
__global__ __launch_bounds__(kBlock) void k_stale_epoch(
    const int64_t *__restrict__ row_ptr, const int32_t *__restrict__ col,
    const float *__restrict__ val, const float *__restrict__ y, const float *__restrict__ w0,
    const int32_t *__restrict__ prev, const int32_t *__restrict__ rd, unsigned long long *words,
    int64_t n, float lr, Ctrl *ctrl, int64_t timeout) {
    const int lane = lane_id();
    const int64_t nw = (int64_t)gridDim.x * kSWaves;
    for (int64_t a = (int64_t)blockIdx.x * kSWaves + wave_in_block(); a < n; a += nw) {
        const int64_t b = row_ptr[a];
        const int64_t m = row_ptr[a + 1] - b;
        if (m <= 2 * kWave) {
            const bool l0 = lane < m, l1 = kWave + lane < m;
            const int64_t q0 = b + lane, q1 = b + kWave + lane;
            const int32_t s0 = l0 ? rd[q0] : -1, s1 = l1 ? rd[q1] : -1;
            const int32_t p0 = l0 ? prev[q0] : -1, p1 = l1 ? prev[q1] : -1;
            const int32_t c0 = l0 ? col[q0] : 0, c1 = l1 ? col[q1] : 0;
            const float x0 = (VAL && l0) ? val[q0] : 1.0f, x1 = (VAL && l1) ? val[q1] : 1.0f;
            const float i0 = l0 ? w0[c0] : 0.0f, i1 = l1 ? w0[c1] : 0.0f;
            // reads: the value of each entry's read source (waits for it)
            unsigned long long v0 = 0, v1 = 0;
            if (!word_wait_wave2(words, s0 >= 0, s0, s0, &v0, s1 >= 0, s1, s1, &v1, ctrl, timeout))
                return;
            float acc = 0.0f;
            if (l0) acc = __builtin_fmaf(s0 >= 0 ? word_value(v0) : i0, x0, acc);
            if (l1) acc = __builtin_fmaf(s1 >= 0 ? word_value(v1) : i1, x1, acc);
            const float st = sgd_scale<LOSS>(wave_sum64(acc), y[a], lr);
            // writes: onto the value of each entry's previous writer
            if (!word_wait_wave2(words, p0 >= 0, p0, p0, &v0, p1 >= 0, p1, p1, &v1, ctrl, timeout))
                return;
            if (l0)
                word_put(words, q0,
                         word_pack(__builtin_fmaf(-st, x0, p0 >= 0 ? word_value(v0) : i0), (int)q0));
            if (l1)
                word_put(words, q1,
                         word_pack(__builtin_fmaf(-st, x1, p1 >= 0 ? word_value(v1) : i1), (int)q1));
            continue;
        }
        // reads: the value of each entry's read source (waits for it)
        float acc = 0.0f;
        for (int64_t k0 = 0; k0 < m; k0 += kWave) {
            const int64_t k = k0 + lane;
            const bool live = k < m;
            const int32_t src = live ? rd[b + k] : -1;
            unsigned long long v = 0;
            if (!word_wait_wave(words, src >= 0, src, src, &v, ctrl, timeout)) return;
            if (live) {
                const float r = src >= 0 ? word_value(v) : w0[col[b + k]];
                acc = __builtin_fmaf(r, VAL ? val[b + k] : 1.0f, acc);
            }
        }
        const float st = sgd_scale<LOSS>(wave_sum64(acc), y[a], lr);
        // writes: onto the value of each entry's previous writer
        for (int64_t k0 = 0; k0 < m; k0 += kWave) {
            const int64_t k = k0 + lane;
            const bool live = k < m;
            const int32_t pq = live ? prev[b + k] : -1;
            unsigned long long v = 0;
            if (!word_wait_wave(words, pq >= 0, pq, pq, &v, ctrl, timeout)) return;
            if (live) {
                const float cur = pq >= 0 ? word_value(v) : w0[col[b + k]];
                const float nv = __builtin_fmaf(-st, VAL ? val[b + k] : 1.0f, cur);
                word_put(words, b + k, word_pack(nv, (int)(b + k)));
            }
        }
    }
}

// Windowed, pass 1: read sources as k_stale_sources finds them, and each
// entry's chain in its window: the first entry on its feature (the head) and
// how many lie before it.  One wave per example; at most `delay` steps back.
__global__ __launch_bounds__(kBlock) void k_win_chains(const int64_t *__restrict__ row_ptr,
                                                       int64_t n,
                                                       const int32_t *__restrict__ prev,
                                                       int64_t delay, int64_t W,
                                                       int32_t *__restrict__ rd,
                                                       unsigned long long *__restrict__ chain) {
    const int lane = lane_id();
    const int64_t nw = (int64_t)gridDim.x * kSWaves;
    for (int64_t a = blockIdx.x * (int64_t)kSWaves + wave_in_block(); a < n; a += nw) {
        const int64_t b = row_ptr[a], e = row_ptr[a + 1], qw = row_ptr[a / W * W];
        const bool all_in_window = a - delay <= 0;
        const int64_t lim = all_in_window ? 0 : row_ptr[a - delay];
        for (int64_t q = b + lane; q < e; q += kWave) {
            int32_t k = prev[q], head = (int32_t)q;
            int rank = 0;
            while (k >= 0 && (int64_t)k >= lim) {  // lim <= qw
                if ((int64_t)k >= qw) {
                    head = k;
                    ++rank;
                }
                k = prev[k];
            }
            rd[q] = all_in_window ? -1 : k;
            chain[q] = (unsigned long long)(unsigned)rank << 32 | (unsigned)head;
        }
    }
}

// Pass 2, one block per window: places 0 .. E - 1, each chain's consecutive;
// place[q] = the entry's place | its chain's length << kPlaceShift at a head.
// chain[q] becomes the window's first entry, and above it the slot of the
// entry's value in the LDS ring of k_stale_window.
constexpr int kPlaceShift = 11;
static_assert(kWinCap <= 1 << kPlaceShift, "a place fits below kPlaceShift");
constexpr int kWinV = 8192;  // values in the LDS ring: the last four windows at least
static_assert(kWinV >= 4 * kWinCap, "see k_stale_window");

__global__ __launch_bounds__(kBlock) void k_win_places(const int64_t *__restrict__ row_ptr,
                                                       int64_t n, int64_t W,
                                                       unsigned long long *__restrict__ chain,
                                                       int32_t *__restrict__ place) {
    __shared__ int32_t s_len[kWinWide], s_base[kWinWide];
    __shared__ int32_t s_next;
    for (int64_t k = blockIdx.x; k < cdiv_dev(n, W); k += gridDim.x) {
        const int64_t q0 = row_ptr[k * W];
        const int E = (int)(row_ptr[min(n, (k + 1) * W)] - q0);
        for (int e = threadIdx.x; e < E; e += kBlock) s_len[e] = 0;
        if (threadIdx.x == 0) s_next = 0;
        __syncthreads();
        for (int e = threadIdx.x; e < E; e += kBlock) {
            const unsigned long long c = chain[q0 + e];
            atomicMax(&s_len[(int)((int64_t)(unsigned)c - q0)], (int)(c >> 32) + 1);
        }
        __syncthreads();
        for (int e = threadIdx.x; e < E; e += kBlock)
            if (s_len[e] > 0) s_base[e] = atomicAdd(&s_next, s_len[e]);
        __syncthreads();
        for (int e = threadIdx.x; e < E; e += kBlock) {
            const unsigned long long c = chain[q0 + e];
            const int at = s_base[(int)((int64_t)(unsigned)c - q0)] + (int)(c >> 32);
            place[q0 + e] = at | s_len[e] << kPlaceShift;
            chain[q0 + e] = (unsigned long long)((q0 + at) & (kWinV - 1)) << 32 | (unsigned)q0;
        }
        __syncthreads();
    }
}

// Pass 3: where the weight the entry reads comes from, in the low half, and
// at a chain's head where the value before the chain does, in the high half:
// kInRing | the slot in the LDS ring of values, or 0: from w (the head: from
// where the read does).  A slot holds its value as long as no more than kWinV
// entries lie from its window's first to the last of this one.
constexpr int kInRing = kWinV;
static_assert(2 * kInRing <= 1 << 15, "two halves");

__global__ __launch_bounds__(kBlock) void k_win_from(const int64_t *__restrict__ row_ptr, int64_t n,
                                                     int64_t W, const int32_t *__restrict__ prev,
                                                     const int32_t *__restrict__ rd,
                                                     const unsigned long long *__restrict__ chain,
                                                     int32_t *__restrict__ from) {
    const int lane = lane_id();
    const int64_t nw = (int64_t)gridDim.x * kSWaves;
    for (int64_t a = blockIdx.x * (int64_t)kSWaves + wave_in_block(); a < n; a += nw) {
        const int64_t b = row_ptr[a], e = row_ptr[a + 1], k = a / W;
        const int64_t qk = row_ptr[k * W], q1 = row_ptr[max(k - 1, (int64_t)0) * W];
        const int64_t qe = row_ptr[min(n, (k + 1) * W)];
        for (int64_t q = b + lane; q < e; q += kWave) {
            const int64_t r = rd[q], pv = prev[q];
            int f = 0;
            if (r >= 0) {
                const unsigned long long c = chain[r];
                if (qe - (int64_t)(unsigned)c <= kWinV) f = kInRing | (int)(c >> 32);
            }
            if (pv >= q1 && pv < qk) f |= (kInRing | (int)(chain[pv] >> 32)) << 16;
            from[q] = f;
        }
    }
}

// The windowed execution, one block.  The chain of windows is what it costs,
// so the waves that run it touch no memory but LDS and their stores to w:
//  * kWinProd producer waves stage the windows in turn, as far ahead as the
//    staging ring has room: entries by CSR index, values by place, the
//    weights that come from w.
//  * A consumer wave takes an example: it reads the weights (from the ring of
//    values that the last windows wrote, or as staged), sums them, and puts the
//    step at each entry's place.  After a barrier the consumers take an entry
//    each; those that head a chain run it over its places, eight reads at a
//    time, into the ring of values.  After another barrier the next window
//    goes.
//  * The last write of each feature of window k goes to w when window k + 1 is
//    staged (the weights it reads from w are then in LDS).  It is complete
//    when the wave stores the next window's.  A producer reads w for window
//    k once every window that is not wholly in the ring of values is complete.
// A weight comes from w only if its source is not in the ring, which holds the
// last windows of kWinV entries together, at least three before this one; so
// no window from k - 3 on wrote it.
// 200,000 examples of 20-40 entries over 100,000 Zipf-1.1 features, delay 8:
// 54.0 -> 28.5 ms (2.4 -> 1.3 us a window of 9); delay 1 42 -> 21.8 ms for
// 50,000, delay 31 7.6 -> 5.1 ms. Before, every wave loaded, staged and waited
// for memory in every window, and a chain followed its entries' links, two
// dependent LDS reads each.  With the same data flow but the staging done by
// all the waves, loads two windows ahead, a window took 2.1 us.  What is left
// is one wave's issue and LDS latency per window, not memory: the barrier that
// waits for the stores of a window before, or for several, took the same.
constexpr int kWinProd = 4;
constexpr int kWinCons = kWinWaves - kWinProd;
// a consumer thread's entries of the widest window that the launcher sends here
constexpr int kWinPer = (kWinWide + kWinCons * kWave - 1) / (kWinCons * kWave);
constexpr int kWinS = 2 * kWinCap;  // staged entries, and examples
constexpr int kWinAhead = 16;       // staged windows
constexpr int kWinU = 6;            // chunks of 64 entries whose loads a producer holds ahead

typedef __attribute__((address_space(3))) float lds_f32;

struct WinShared {
    float v[kWinV];       // the values the entries wrote, by slot
    float xp[kWinS + 8];  // by place from the window's first entry on: value (the first 8 again)
    int32_t place[kWinS], from[kWinS], col[kWinS];  // by entry
    float wv[kWinS];      // by entry: its feature's weight in w
    int32_t rb[kWinS];    // by example: first entry
    float y[kWinS];
    float st[kWinCap + 8];  // by place (below 2^kPlaceShift): step
    float sink;
    int2 win[kWinAhead];  // first entry, last + 1
    int staged[kWinProd];  // producer: its windows before this one are staged
    alignas(16) int done;  // windows the consumers are through with
    int freeq;             // their entries end here
    int ackq;              // entries of the windows whose writes are in w
    int stop;              // a producer gave up: every wave leaves
    unsigned arrived;      // consumer waves at the barriers so far
    int tripped;           // one producer marks them
};

struct WinArgs {
    const int64_t *row_ptr;
    const int32_t *col;
    const float *val, *y;
    float *w;
    const int32_t *place, *from;
    int64_t n, nnz, W;
    float lr;
    Ctrl *ctrl;
    int64_t timeout;
};

__device__ __forceinline__ int win_get(const int *p) {
    return __builtin_amdgcn_readfirstlane(
        __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP));
}
__device__ __forceinline__ void win_set(int *p, int v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// the words that a producer's wait for room looks at, by one LDS read
struct WinRoom {
    int done, freeq, ackq, stop;
};
__device__ __forceinline__ WinRoom win_room(const WinShared &S) {
    __asm__ __volatile__("" ::: "memory");  // read again at every poll
    const int4 r = *reinterpret_cast<const int4 *>(&S.done);
    __asm__ __volatile__("" ::: "memory");
    return WinRoom{__builtin_amdgcn_readfirstlane(r.x), __builtin_amdgcn_readfirstlane(r.y),
                   __builtin_amdgcn_readfirstlane(r.z), __builtin_amdgcn_readfirstlane(r.w)};
}

// The watchdog.  Every wait of the block is for a producer, or for consumers
// that wait for one, and a producer waits only for room, which the consumers
// make.  So the producers watch for all: in their waits for room, and producer 0
// until the consumers are through.  The first to give up makes the barriers'
// count jump far ahead and sets the stop word, which ends the other producers'
// waits; each marks its `staged` as it leaves.  The consumers' polls are on the
// chain and look at nothing else: a marked word ends the wait, and the
// window's last barrier tells by its count whether there is a next window.
// (A clock and a stop word in the consumers' own polls: 50,000 examples of
// 20-40 entries, delay 1, 32.5 ms; a test after each of their waits 27.6; this
// 22.5, where window numbers of 64 bits took 25.5 and no watchdog at all, with
// 64 bits, 24.2.)
constexpr unsigned kWinGone = 1u << 30;  // beyond what a barrier's count runs ahead
struct WinWatch {
    int polls = 0;
    int64_t t0 = 0;
    // after every failed poll of a producer
    __device__ __forceinline__ void check(const WinArgs &p, WinShared &S) {
        if (++polls % 16) return;
        const int64_t now = now_ticks();
        if (polls == 16) t0 = now;
        if (now - t0 <= p.timeout) return;
        record_error(p.ctrl, DERR_WAIT_TIMEOUT);
        if (lane_id() == 0 && atomicExch(&S.tripped, 1) == 0) {
            atomicAdd(&S.arrived, kWinGone);
            win_set(&S.stop, 1);  // LDS runs one wave's operations in order
        }
    }
};

// A barrier of the consumer waves (the producers do not take part), for LDS
// only, in two halves: the LDS runs each wave's operations in order, so a
// wave's writes are there once its arrival is counted.
struct WinBarrier {
    unsigned passed = 0;  // arrivals of the barriers so far
    __device__ __forceinline__ void arrive(WinShared &S) {
        passed += kWinCons;
        __asm__ __volatile__("" ::: "memory");
        if (lane_id() == 0) atomicAdd(&S.arrived, 1u);
        __asm__ __volatile__("" ::: "memory");
    }
    // returns how far the count is past this barrier
    __device__ __forceinline__ int wait(WinShared &S) {
        int ahead;
        __asm__ __volatile__("" ::: "memory");
        do {
            ahead = (int)((unsigned)win_get(reinterpret_cast<const int *>(&S.arrived)) - passed);
        } while (ahead < 0);
        __asm__ __volatile__("" ::: "memory");
        return ahead;
    }
};

// The ring slot of the window's entry (or place) e.  An entry's index reaches
// 2^31 - 2, and a chunk or a chain's reads run past the window's end, so the
// sum is unsigned.
__host__ __device__ constexpr int win_slot(unsigned qs, int e) {
    return (int)((qs + (unsigned)e) & (unsigned)(kWinS - 1));
}
static_assert(win_slot(INT_MAX - 2u, kWinU * kWave) == ((INT_MAX - 2ll + kWinU * kWave) & (kWinS - 1)),
              "past the last entry of the largest CSR");

// loads of kWinU chunks of entries from q on (clamped into the arrays)
template <bool VAL>
struct WinChunk {
    int32_t col[kWinU], place[kWinU], from[kWinU];
    float x[kWinU];
    __device__ __forceinline__ void load(const WinArgs &p, int64_t q0) {
#pragma unroll
        for (int u = 0; u < kWinU; ++u) {
            const int64_t q = min(q0 + u * kWave + lane_id(), p.nnz - 1);
            col[u] = p.col[q];
            place[u] = p.place[q];
            from[u] = p.from[q];
            x[u] = VAL ? p.val[q] : 1.0f;
        }
    }
    // entries off .. of the window [qs, qs + E) into LDS
    __device__ __forceinline__ void put(WinShared &S, const float *wv, int off, unsigned qs, int E) {
#pragma unroll
        for (int u = 0; u < kWinU; ++u) {
            const int e = off + u * kWave + lane_id();
            if (off + u * kWave >= E) break;
            if (e < E) {
                const int i = win_slot(qs, e);
                S.col[i] = col[u];
                S.place[i] = place[u];
                S.from[i] = from[u];
                S.wv[i] = wv[u];
                const int at = win_slot(qs, place[u] & ((1 << kPlaceShift) - 1));
                S.xp[at] = x[u];
                if (at < 8) S.xp[kWinS + at] = x[u];
            }
        }
    }
};

template <bool VAL>
__device__ void win_produce(const WinArgs &p, WinShared &S, int id, int64_t nwin) {
    const int lane = lane_id();
    auto astart = [&](int64_t k) { return min(p.n, k * p.W); };
    // first entry of window k, by a vector load: it is waited for when it is
    // used, not with the next LDS operation
    auto qstart = [&](int64_t k) {
        int zero = 0;
        __asm__ volatile("" : "+v"(zero));
        return (int32_t)p.row_ptr[astart(k) + zero];  // nnz < 2^31
    };
    if (id >= nwin || p.nnz == 0) {
        // no entries: bounds alone
        for (int64_t k = id; k < nwin; k += kWinProd) {
            WinWatch watch;
            for (;;) {
                const WinRoom r = win_room(S);
                if (r.stop) {
                    win_set(&S.staged[id], INT_MAX);
                    return;
                }
                if (k < r.done + kWinAhead && astart(k + 1) - astart(r.done) <= kWinS) break;
                watch.check(p, S);
                __builtin_amdgcn_s_sleep(1);
            }
            if (lane == 0) S.win[k & (kWinAhead - 1)] = make_int2(0, 0);
            for (int64_t a = astart(k) + lane; a < astart(k + 1); a += kWave) {
                S.rb[a & (kWinS - 1)] = 0;
                S.y[a & (kWinS - 1)] = p.y[a];
            }
            __asm__ __volatile__("" ::: "memory");
            if (lane == 0) win_set(&S.staged[id], (int)k + 1);
        }
        return;
    }
    // A window's first loads are issued while the producer's window before it
    // is staged, and its bounds a window before that.  Loads complete in
    // order: a window's weights are asked for before the next one's first
    // loads, so that they are not waited for with them.
    struct Ahead {
        WinChunk<VAL> c;
        int32_t rb;
        float y;
    } A, B;
    auto load = [&](Ahead &x, int64_t k, int64_t qs) {
        x.c.load(p, qs);
        const int64_t a = min(astart(k) + lane, p.n - 1);
        x.rb = (int32_t)p.row_ptr[a];
        x.y = p.y[a];
    };
    int64_t qs = __builtin_amdgcn_readfirstlane(qstart(id));
    int64_t qe = __builtin_amdgcn_readfirstlane(qstart(id + 1));
    int32_t ns = qstart(id + kWinProd), ne = qstart(id + kWinProd + 1);
    load(A, id, qs);
    auto stage = [&](int64_t k, Ahead &cur, Ahead &nxt) {
        const int64_t a0 = astart(k), a1 = astart(k + 1);
        // room for its entries, examples and bounds, and nothing to read from
        // w that is not there yet
        WinWatch watch;
        for (;;) {
            const WinRoom r = win_room(S);
            if (r.stop) {
                win_set(&S.staged[id], INT_MAX);
                return false;
            }
            if (k < r.done + kWinAhead && a1 - astart(r.done) <= kWinS && qe - r.freeq <= kWinS &&
                qe - r.ackq <= kWinV)
                break;
            watch.check(p, S);
            __builtin_amdgcn_s_sleep(1);
        }
        __asm__ __volatile__("" ::: "memory");
        float wv[kWinU];
#pragma unroll
        for (int u = 0; u < kWinU; ++u)
            wv[u] = __hip_atomic_load(&p.w[cur.c.col[u]], __ATOMIC_RELAXED,
                                      __HIP_MEMORY_SCOPE_WORKGROUP);
        const int64_t s1 = __builtin_amdgcn_readfirstlane(ns), e1 = __builtin_amdgcn_readfirstlane(ne);
        load(nxt, k + kWinProd, s1);
        ns = qstart(k + 2 * kWinProd);
        ne = qstart(k + 2 * kWinProd + 1);
        if (a0 + lane < a1) {
            S.rb[(a0 + lane) & (kWinS - 1)] = cur.rb;
            S.y[(a0 + lane) & (kWinS - 1)] = cur.y;
        }
        cur.c.put(S, wv, 0, (unsigned)qs, (int)(qe - qs));
        // what is more than a wave's first loads
        for (int64_t a = a0 + kWave + lane; a < a1; a += kWave) {
            S.rb[a & (kWinS - 1)] = (int32_t)p.row_ptr[a];
            S.y[a & (kWinS - 1)] = p.y[a];
        }
        for (int64_t q = qs + kWinU * kWave; q < qe; q += kWinU * kWave) {
            cur.c.load(p, q);
#pragma unroll
            for (int u = 0; u < kWinU; ++u)
                wv[u] = __hip_atomic_load(&p.w[cur.c.col[u]], __ATOMIC_RELAXED,
                                          __HIP_MEMORY_SCOPE_WORKGROUP);
            cur.c.put(S, wv, (int)(q - qs), (unsigned)qs, (int)(qe - qs));
        }
        if (lane == 0) S.win[k & (kWinAhead - 1)] = make_int2((int)qs, (int)qe);
        __asm__ __volatile__("" ::: "memory");  // LDS runs one wave's operations in order
        if (lane == 0) win_set(&S.staged[id], (int)k + 1);
        qs = s1;
        qe = e1;
        return true;
    };
    for (int64_t k = id; k < nwin; k += 2 * kWinProd) {
        if (!stage(k, A, B)) return;
        if (k + kWinProd >= nwin) break;
        if (!stage(k + kWinProd, B, A)) return;
    }
}

// What a consumer wave holds of a window before its turn: the bounds, and of
// its first kWinTurn examples the bounds, the labels (example i's in lane i)
// and each lane's entry.
constexpr int kWinTurn = 1;  // three took as long, also where windows hold 16 to 61 examples
struct WinTurn {
    unsigned qs;
    int E;
    float y;
    int b[kWinTurn], m[kWinTurn];
    int f[kWinTurn], pl[kWinTurn];  // as S.from (the read) and S.place
    float wq[kWinTurn], x[kWinTurn];
};

__device__ __forceinline__ WinTurn win_turn(const WinArgs &p, WinShared &S, int wave, unsigned k) {
    constexpr int mask = (1 << kPlaceShift) - 1;
    const int lane = lane_id();
    WinTurn t;
    while (win_get(&S.staged[k & (kWinProd - 1)]) <= (int)k) {
    }
    __asm__ __volatile__("" ::: "memory");
    const int2 win = S.win[k & (kWinAhead - 1)];
    t.qs = __builtin_amdgcn_readfirstlane(win.x);
    const int qe = __builtin_amdgcn_readfirstlane(win.y);
    t.E = qe - (int)t.qs;
    const unsigned W = (unsigned)p.W, a0 = k * W;  // below 2^31 + W
    const int nex = (int)(min((unsigned)p.n, a0 + W) - a0), j = kWinCons - 1 - wave;
    if (j < nex) {
        const int jl = min(j + min(lane, kWinTurn - 1) * kWinCons, nex - 1);
        const int bl = S.rb[(a0 + jl) & (kWinS - 1)];
        const int el = jl + 1 < nex ? S.rb[(a0 + jl + 1) & (kWinS - 1)] : qe;
        t.y = S.y[(a0 + jl) & (kWinS - 1)];
#pragma unroll
        for (int i = 0; i < kWinTurn; ++i) {
            if (j + i * kWinCons >= nex) break;
            t.b[i] = __builtin_amdgcn_readlane(bl, i);
            t.m[i] = __builtin_amdgcn_readlane(el, i) - t.b[i];
            const int q = (t.b[i] + min(lane, max(t.m[i] - 1, 0))) & (kWinS - 1);
            t.f[i] = S.from[q];
            t.pl[i] = S.place[q] & mask;
            t.wq[i] = S.wv[q];
            t.x[i] = S.xp[win_slot(t.qs, t.pl[i])];
        }
    }
    return t;
}

template <int LOSS, bool VAL>
__device__ void win_consume(const WinArgs &p, WinShared &S, int wave, unsigned nwin) {
    constexpr int mask = (1 << kPlaceShift) - 1;
    const int lane = lane_id(), tid = wave * kWave + lane, w0 = wave * kWave;
    const unsigned v_a = (unsigned)(uintptr_t)(const lds_f32 *)S.v;
    const unsigned sink_a = (unsigned)(uintptr_t)(const lds_f32 *)&S.sink;
    float last_v[kWinPer];
    int32_t last_c[kWinPer];  // the last writes of the window before
#pragma unroll
    for (int u = 0; u < kWinPer; ++u) {
        last_c[u] = -1;
        last_v[u] = 0.0f;
    }
    int qb = 0;  // first entry of the window before
    WinBarrier bar;
    WinTurn T = win_turn(p, S, wave, 0);
    if (win_get(&S.stop)) return;  // window 0 was not staged
    const unsigned W = (unsigned)p.W;
    for (unsigned k = 0;;) {
        const unsigned qs = T.qs;
        const int E = T.E;
        const unsigned a0 = k * W;
        const int nex = (int)(min((unsigned)p.n, a0 + W) - a0);
        // steps, a wave per example (the last waves first: the first ones head
        // the chains); dot products in the matched order
        const int j = kWinCons - 1 - wave;
        if (j < nex) {
            float acc[kWinTurn], z = 0.0f;
#pragma unroll
            for (int i = 0; i < kWinTurn; ++i) {
                if (j + i * kWinCons >= nex) break;
                const float v = S.v[T.f[i] & (kWinV - 1)];
                acc[i] = lane < T.m[i]
                             ? __builtin_fmaf(T.f[i] & kInRing ? v : T.wq[i], T.x[i], 0.0f)
                             : 0.0f;
                for (int t = kWave + lane; t < T.m[i]; t += kWave) {
                    const int q = (T.b[i] + t) & (kWinS - 1);
                    const int f = S.from[q], pl = S.place[q] & mask;
                    const float wq = S.wv[q], vr = S.v[f & (kWinV - 1)];
                    acc[i] = __builtin_fmaf(f & kInRing ? vr : wq, S.xp[win_slot(qs, pl)],
                                            acc[i]);
                }
            }
#pragma unroll
            for (int i = 0; i < kWinTurn; ++i) {
                if (j + i * kWinCons >= nex) break;
                const float zi = wave_sum64(acc[i]);
                z = lane == i ? zi : z;
            }
            const float st = sgd_scale<LOSS>(z, T.y, p.lr);
#pragma unroll
            for (int i = 0; i < kWinTurn; ++i) {
                if (j + i * kWinCons >= nex) break;
                const float si = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(st), i));
                if (lane < T.m[i]) S.st[T.pl[i]] = si;
                for (int t = kWave + lane; t < T.m[i]; t += kWave)
                    S.st[S.place[(T.b[i] + t) & (kWinS - 1)] & mask] = si;
            }
        }
        // the others of a window of many examples, four of a wave side by side
        for (int j0 = j + kWinTurn * kWinCons; j0 < nex; j0 += 4 * kWinCons) {
            float z = 0.0f;
            const int jl = j0 + lane * kWinCons;  // lane i < 4: example j0 + kWinCons i
            const bool has = lane < 4 && jl < nex;
            const int bl = has ? S.rb[(a0 + jl) & (kWinS - 1)] : 0;
            const int el = has && jl + 1 < nex ? S.rb[(a0 + jl + 1) & (kWinS - 1)] : (int)qs + E;
            const float yl = has ? S.y[(a0 + jl) & (kWinS - 1)] : 0.0f;
            int at[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (j0 + i * kWinCons >= nex) break;
                const int b = __builtin_amdgcn_readlane(bl, i);
                const int m = __builtin_amdgcn_readlane(el, i) - b;
                float acc = 0.0f;
                for (int t0 = 0; t0 < m; t0 += kWave) {
                    const int t = t0 + lane;
                    if (t < m) {
                        const int q = (b + t) & (kWinS - 1);
                        const int f = S.from[q], pl = S.place[q] & mask;
                        const float wq = S.wv[q];
                        const float v = S.v[f & (kWinV - 1)], x = S.xp[win_slot(qs, pl)];
                        acc = __builtin_fmaf(f & kInRing ? v : wq, x, acc);
                        if (t0 == 0) at[i] = pl;
                    }
                }
                const float zi = wave_sum64(acc);
                z = lane == i ? zi : z;
            }
            const float st = sgd_scale<LOSS>(z, yl, p.lr);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (j0 + i * kWinCons >= nex) break;
                const int b = __builtin_amdgcn_readlane(bl, i);
                const int m = __builtin_amdgcn_readlane(el, i) - b;
                const float si =
                    __int_as_float(__builtin_amdgcn_readlane(__float_as_int(st), i));
                if (lane < m) S.st[at[i]] = si;
                for (int t = kWave + lane; t < m; t += kWave)
                    S.st[S.place[(b + t) & (kWinS - 1)] & mask] = si;
            }
        }
        // the writes of window k - 2 are in w; those of window k - 1 go
        __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
        bar.arrive(S);
#pragma unroll
        for (int u = 0; u < kWinPer; ++u)
            if (last_c[u] >= 0)
                __hip_atomic_store(&p.w[last_c[u]], last_v[u], __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_WORKGROUP);
        // the chains' heads, and the value before each
        int head[kWinPer];
        float base[kWinPer];
#pragma unroll
        for (int u = 0; u < kWinPer; ++u) {
            head[u] = 0;
            last_c[u] = -1;
            base[u] = 0.0f;
            const int e = tid + u * kWinCons * kWave;
            if (w0 + u * kWinCons * kWave >= E) continue;
            const int q = win_slot(qs, e);
            const int pl = S.place[q], f = S.from[q], c = S.col[q];
            const float wq = S.wv[q];
            const float vr = S.v[f & (kWinV - 1)], vh = S.v[f >> 16 & (kWinV - 1)];
            if (e < E && pl >> kPlaceShift) {
                head[u] = pl;
                last_c[u] = c;
                base[u] = f >> 16 & kInRing ? vh : f & kInRing ? vr : wq;
            }
        }
        bar.wait(S);
        if (tid == 0) win_set(&S.ackq, qb);
        // writes: each chain's entries in example order, from the value before
        // it, eight at a time (reads past its end and past the window's are
        // not used, writes there go to the sink)
#pragma unroll
        for (int u = 0; u < kWinPer; ++u) {
            if (w0 + u * kWinCons * kWave >= E) continue;
            const int len = head[u] >> kPlaceShift, a = head[u] & mask;
            float v = base[u];
            for (int i = 0; __ballot(i < len) != 0ull; i += 8) {
                const int ai = min(a + i, kWinCap);
                const float *const st = &S.st[ai], *const xp = &S.xp[win_slot(qs, ai)];
                float sv[8], xv[8];
#pragma unroll
                for (int t = 0; t < 8; ++t) {
                    sv[t] = st[t];
                    xv[t] = xp[t];
                }
#pragma unroll
                for (int t = 0; t < 8; ++t) {
                    const bool on = i + t < len;
                    if (t > 0 && __ballot(on) == 0ull) break;
                    const float nv = __builtin_fmaf(-sv[t], xv[t], v);
                    v = on ? nv : v;
                    const unsigned to = on ? v_a + ((qs + (unsigned)(a + i + t)) & (kWinV - 1)) * 4u : sink_a;
                    *(lds_f32 *)(uintptr_t)to = v;
                }
            }
            last_v[u] = v;
        }
        bar.arrive(S);
        qb = (int)qs;
        if (k + 1 < nwin) T = win_turn(p, S, wave, k + 1);
        const unsigned last = bar.wait(S) < kWinCons ? nwin : k + 1;
        if (tid == 0) {
            win_set(&S.freeq, (int)qs + E);
            win_set(&S.done, (int)k + 1);
        }
        if (++k == last) break;
    }
    // the last window's writes, after those of the one before it
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
    bar.arrive(S);
    bar.wait(S);
#pragma unroll
    for (int u = 0; u < kWinPer; ++u)
        if (last_c[u] >= 0) p.w[last_c[u]] = last_v[u];
}

template <int LOSS, bool VAL>
__global__ __launch_bounds__(kWinThreads) void k_stale_window(WinArgs p) {
    __shared__ WinShared S;
    if (threadIdx.x < kWinProd) S.staged[threadIdx.x] = 0;
    if (threadIdx.x == 0) {
        S.done = S.freeq = S.ackq = S.stop = S.tripped = 0;
        S.arrived = 0;
    }
    __syncthreads();
    const int wave = __builtin_amdgcn_readfirstlane(wave_in_block());
    const int64_t nwin = cdiv_dev(p.n, p.W);
    if (wave < kWinCons)
        win_consume<LOSS, VAL>(p, S, wave, (unsigned)nwin);
    else
        win_produce<VAL>(p, S, wave - kWinCons, nwin);
    if (wave == kWinCons) {
        // no window left to stage: until the consumers are through
        for (int done = -1;;) {
            WinWatch watch;
            WinRoom r;
            while ((r = win_room(S)).done == done && !r.stop) {
                watch.check(p, S);
                __builtin_amdgcn_s_sleep(8);
            }
            if (r.stop || r.done >= nwin) return;
            done = r.done;
        }
    }
}

constexpr int kWidePer = kWinCap / kWinThreads;  // entries per thread

__global__ void k_stale_no_next(int32_t *__restrict__ next, int64_t nnz) {
    for (int64_t q = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; q < nnz;
         q += (int64_t)gridDim.x * blockDim.x)
        next[q] = -1;
}

// next writer: the entry whose previous entry on the feature is q
__global__ void k_stale_next(const int32_t *__restrict__ prev, int64_t nnz,
                             int32_t *__restrict__ next) {
    for (int64_t q = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; q < nnz;
         q += (int64_t)gridDim.x * blockDim.x) {
        const int32_t p = prev[q];
        if (p >= 0) next[p] = (int32_t)q;
    }
}

// The windowed execution where windows are large, one block of kWinThreads
// threads that all load, stage and compute.  Thread t handles entries t and
// t + kWinThreads of every window, and examples t and t + kWinThreads.  What
// a window reads from memory that earlier windows do
// not change (columns, values, read sources, previous and next writers, row
// bounds, labels) is loaded two windows ahead into registers; the weights it
// reads from w are loaded one window ahead, right after the commit that
// makes w the state they need.
struct WideBuf {
    int32_t col[kWinCap];
    float x[kWinCap];
    float rv[kWinCap];     // the value the entry reads
    float v[kWinCap];      // the value the entry writes
    int32_t nxt[kWinCap];  // next entry on the feature (CSR index), -1 = none
    int16_t ex[kWinCap];   // the entry's example within the window
    int32_t rp[kWinCap + 1];  // example bounds, relative to the window's first entry
    float y[kWinCap];
};

// a window's loads, per thread
struct WideMeta {
    int32_t col[kWidePer], rd[kWidePer], pv[kWidePer], nx[kWidePer];
    float x[kWidePer];
    int64_t rp[kWidePer + 1];  // row_ptr of examples t, t + kWinThreads (and the end)
    float y[kWidePer];
};

template <bool VAL>
__device__ __forceinline__ void wide_load(WideMeta &m, int64_t k, int64_t nwin, int64_t W,
                                         int64_t n, int64_t nnz, int64_t q0,
                                         const int64_t *__restrict__ row_ptr,
                                         const int32_t *__restrict__ col,
                                         const float *__restrict__ val,
                                         const float *__restrict__ y,
                                         const int32_t *__restrict__ prev,
                                         const int32_t *__restrict__ rd,
                                         const int32_t *__restrict__ next) {
    if (k >= nwin) return;
    const int tid = threadIdx.x;
    const int64_t a0 = k * W, a1 = min(n, a0 + W);
#pragma unroll
    for (int u = 0; u < kWidePer; ++u) {
        // entries past the window's end are loaded (clamped) and ignored
        const int64_t q = min(q0 + tid + u * kWinThreads, nnz - 1);
        if (nnz > 0) {
            m.col[u] = col[q];
            m.rd[u] = rd[q];
            m.pv[u] = prev[q];
            m.nx[u] = next[q];
            m.x[u] = VAL ? val[q] : 1.0f;
        }
        const int64_t a = min(a0 + tid + u * kWinThreads, a1);
        m.rp[u] = row_ptr[a];
        m.y[u] = y[min(a, n - 1)];
    }
    m.rp[kWidePer] = row_ptr[min(a0 + tid + kWidePer * kWinThreads, a1)];
}

template <int LOSS, bool VAL>
__global__ __launch_bounds__(kWinThreads) void k_stale_wide(
    const int64_t *__restrict__ row_ptr, const int32_t *__restrict__ col,
    const float *__restrict__ val, const float *__restrict__ y, float *w,
    const int32_t *__restrict__ prev, const int32_t *__restrict__ rd,
    const int32_t *__restrict__ next, int64_t n, int64_t nnz, int64_t W, float lr) {
    __shared__ WideBuf buf[2];
    __shared__ float S[kWinCap];
    const int tid = threadIdx.x, lane = lane_id(), wave = wave_in_block();
    const int64_t nwin = cdiv_dev(n, W);
    auto qstart = [&](int64_t k) { return row_ptr[min(n, k * W)]; };
    WideMeta m0, m1, m2;
    int64_t q0 = qstart(0), q1 = qstart(1), q2 = qstart(2);
    wide_load<VAL>(m0, 0, nwin, W, n, nnz, q0, row_ptr, col, val, y, prev, rd, next);
    wide_load<VAL>(m1, 1, nwin, W, n, nnz, q1, row_ptr, col, val, y, prev, rd, next);
    float wv[kWidePer];
#pragma unroll
    for (int u = 0; u < kWidePer; ++u) wv[u] = (nnz > 0) ? w[m0.col[u]] : 0.0f;
    int cur = 0;
    int64_t pq0 = 0;  // first entry of the previous window (its end is the current start)
    int pE = 0;       // entries of the previous window
    // One window.  mc, mn, mnn: the loads of windows k, k + 1, k + 2 (mnn is
    // issued here); qa, qb, qc: the first entries of windows k, k + 1, k + 2
    // (qa receives that of window k + 3).  The three calls per loop
    // iteration rotate the roles, so no register copy waits on a load still
    // in flight.
    auto window = [&](int64_t k, WideMeta &mc, WideMeta &mn, WideMeta &mnn, int64_t &qa,
                      int64_t qb, int64_t qc) {
        const int64_t a0 = k * W, a1 = min(n, a0 + W);
        const int64_t qs = qa;
        const int E = (int)(qb - qs), nex = (int)(a1 - a0);
        WideBuf &C = buf[cur];
        const WideBuf &P = buf[cur ^ 1];
        // window k into LDS; reads from window k - 1's writes, else from w
        // as it was before window k - 1
#pragma unroll
        for (int u = 0; u < kWidePer; ++u) {
            const int e = tid + u * kWinThreads;
            if (e < E) {
                const int32_t r = mc.rd[u];
                C.col[e] = mc.col[u];
                C.x[e] = mc.x[u];
                C.nxt[e] = mc.nx[u];
                C.rv[e] = (r >= pq0) ? P.v[r - pq0] : wv[u];
            }
            if (e <= nex) C.rp[e] = (int32_t)(mc.rp[u] - qs);
            if (e < nex) C.y[e] = mc.y[u];
        }
        if (tid + kWidePer * kWinThreads <= nex)
            C.rp[tid + kWidePer * kWinThreads] = (int32_t)(mc.rp[kWidePer] - qs);
        __syncthreads();
        // commit window k - 1: the last write of each feature it touched
        for (int e = tid; e < pE; e += kWinThreads) {
            const int32_t nx = P.nxt[e];
            if (nx < 0 || nx >= qs) w[P.col[e]] = P.v[e];
        }
        // window k + 2's loads, in flight while this window computes
        wide_load<VAL>(mnn, k + 2, nwin, W, n, nnz, qc, row_ptr, col, val, y, prev, rd, next);
        qa = qstart(k + 3);
        // steps, a wave per example, dot products in the matched order
        for (int j = wave; j < nex; j += kWinWaves) {
            const int b = C.rp[j], mm = C.rp[j + 1] - b;
            float acc = 0.0f;
            for (int t = lane; t < mm; t += kWave) {
                acc = __builtin_fmaf(C.rv[b + t], C.x[b + t], acc);
                C.ex[b + t] = (int16_t)j;
            }
            const float z = wave_sum64(acc);
            if (lane == 0) S[j] = sgd_scale<LOSS>(z, C.y[j], lr);
        }
        __syncthreads();
        // window k + 1's reads of w: w is now the state before window k
        if (k + 1 < nwin && nnz > 0) {
#pragma unroll
            for (int u = 0; u < kWidePer; ++u) wv[u] = w[mn.col[u]];
        }
        // writes: each feature's entries of the window in example order,
        // from the value its previous writer left
#pragma unroll
        for (int u = 0; u < kWidePer; ++u) {
            const int e = tid + u * kWinThreads;
            const int32_t pv = mc.pv[u];
            if (e < E && pv < qs) {
                float v = (pv >= pq0) ? P.v[pv - pq0] : C.rv[e];
                int ee = e;
                for (;;) {
                    v = __builtin_fmaf(-S[C.ex[ee]], C.x[ee], v);
                    C.v[ee] = v;
                    const int32_t nx = C.nxt[ee];
                    if (nx < 0 || nx >= qb) break;
                    ee = (int)(nx - qs);
                }
            }
        }
        __syncthreads();
        pq0 = qs;
        pE = E;
        cur ^= 1;
    };
    for (int64_t k = 0; k < nwin; k += 3) {
        window(k, m0, m1, m2, q0, q1, q2);
        if (k + 1 >= nwin) break;
        window(k + 1, m1, m2, m0, q1, q2, q0);
        if (k + 2 >= nwin) break;
        window(k + 2, m2, m0, m1, q2, q0, q1);
    }
    const WideBuf &P = buf[cur ^ 1];
    for (int e = tid; e < pE; e += kWinThreads)
        if (P.nxt[e] < 0) w[P.col[e]] = P.v[e];
}

// each feature's final value: the entry no later entry overwrites
__global__ __launch_bounds__(kBlock) void k_stale_final(const int32_t *__restrict__ col,
                                                        const unsigned long long *__restrict__ words,
                                                        const int32_t *__restrict__ overwritten,
                                                        int64_t nnz, float *__restrict__ w) {
    for (int64_t q = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; q < nnz;
         q += (int64_t)gridDim.x * blockDim.x)
        if (!overwritten[q]) w[col[q]] = word_value(words[q]);
}

template <int LOSS, bool VAL>
int launch_stale(const pdb_csr *csr, const float *labels, int64_t n, float *w, float lr,
                 int64_t delay, const int32_t *prev, StaleWs &ws, const Opts &opt, hipStream_t s) {
    const int64_t nnz = csr->nnz;
    const int64_t timeout = opt.timeout;
    k_stale_ctrl_zero<<<1, 64, 0, s>>>(ws.ctrl);
    PDB_LAUNCHED();
    // windows of delay + 1 examples.  The windowed execution needs the
    // largest window to fit the block, and pays on chain-like inputs (most
    // examples share a feature with the one before: one block then beats a
    // device-scope hop per example); elsewhere the sync-free one runs many
    // examples at once.  Read back: this call synchronises the stream.
    const int mode = opt.stale_mode;
    const int64_t W = delay >= n ? std::max<int64_t>(n, 1) : delay + 1;  // no overflow at huge delays
    bool windowed = false;
    int64_t widest = 0;
    if (mode != PDB_STALE_SYNCFREE && W <= kWinCap) {
        k_stale_shape<<<grid_for(n, kSWaves, 65536), kBlock, 0, s>>>(csr->row_ptr, n, W,
                                                                     nnz > 0 ? n : 0, prev, ws.ctrl);
        PDB_LAUNCHED();
        Ctrl host{};
        PDB_HIP(hipMemcpyAsync(&host, ws.ctrl, sizeof(Ctrl), hipMemcpyDeviceToHost, s));
        PDB_HIP(hipStreamSynchronize(s));
        const bool chain_like = 4 * (int64_t)host.chain_breaks <= n;
        widest = host.max_width;
        windowed = host.max_width <= kWinCap && (mode == PDB_STALE_WINDOWED || chain_like);
    }
    // Windows of more than kWinWide entries: the producers' buffers hold fewer
    // than three, so at most two producers load at a time and the chain waits
    // for them (valued Zipf-1.2 features: 5 x 200-400 58.9 ms that way, 32.9
    // here; 31 x 50 9.7 and 8.8; below the line 9 x 100-180, the widest 1.5K
    // entries, 15.2 and 17.1).
    if (windowed && widest > kWinWide) {
        k_stale_no_next<<<grid_for(nnz, kBlock, 8192), kBlock, 0, s>>>(ws.next, nnz);
        k_stale_sources<<<grid_for(n, kSWaves, 65536), kBlock, 0, s>>>(csr->row_ptr, n, prev,
                                                                       delay, ws.rd,
                                                                       ws.overwritten);
        k_stale_next<<<grid_for(nnz, kBlock, 8192), kBlock, 0, s>>>(prev, nnz, ws.next);
        PDB_LAUNCHED();
        k_stale_wide<LOSS, VAL><<<1, kWinThreads, 0, s>>>(csr->row_ptr, csr->col, csr->val, labels,
                                                          w, prev, ws.rd, ws.next, n, nnz, W, lr);
        PDB_LAUNCHED();
        return PDB_OK;
    }
    if (windowed) {
        // the words hold the entries' chains, the other arrays their places
        // and where their values come from
        int32_t *place = ws.overwritten, *from = ws.next;
        if (nnz > 0) {
            k_win_chains<<<grid_for(n, kSWaves, 65536), kBlock, 0, s>>>(csr->row_ptr, n, prev,
                                                                        delay, W, ws.rd, ws.words);
            k_win_places<<<grid_for(cdiv(n, W), 1, 65536), kBlock, 0, s>>>(csr->row_ptr, n, W,
                                                                           ws.words, place);
            k_win_from<<<grid_for(n, kSWaves, 65536), kBlock, 0, s>>>(csr->row_ptr, n, W, prev,
                                                                      ws.rd, ws.words, from);
            PDB_LAUNCHED();
        }
        const WinArgs p{csr->row_ptr, csr->col, csr->val, labels, w, place, from, n, nnz, W, lr,
                        ws.ctrl, timeout};
        k_stale_window<LOSS, VAL><<<1, kWinThreads, 0, s>>>(p);
        PDB_LAUNCHED();
        return PDB_OK;
    }
    if (nnz > 0) {
        k_stale_clear<<<grid_for(nnz, kBlock, 8192), kBlock, 0, s>>>(ws.words, ws.overwritten, nnz);
        PDB_LAUNCHED();
        k_stale_sources<<<grid_for(n, kSWaves, 65536), kBlock, 0, s>>>(csr->row_ptr, n, prev,
                                                                       delay, ws.rd,
                                                                       ws.overwritten);
        PDB_LAUNCHED();
    }
    // every block resident (a cooperative launch: the waves wait on each
    // other), at most one wave per example
    const void *fn = reinterpret_cast<const void *>(&k_stale_epoch<LOSS, VAL>);
    int dev = 0, cus = 0, per_cu = 0;
    PDB_HIP(hipGetDevice(&dev));
    PDB_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
    PDB_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, kBlock, 0));
    const int64_t grid = std::max<int64_t>(
        1, std::min<int64_t>((int64_t)cus * std::max(per_cu, 1), cdiv(n, (int64_t)kSWaves)));
    {
        const int64_t *a_rp = csr->row_ptr;
        const int32_t *a_col = csr->col, *a_rd = ws.rd;
        const float *a_val = csr->val, *a_y = labels, *a_w0 = w;
        const int32_t *a_prev = prev;
        unsigned long long *a_words = ws.words;
        Ctrl *a_ctrl = ws.ctrl;
        int64_t a_n = n, a_timeout = timeout;
        float a_lr = lr;
        void *args[] = {&a_rp, &a_col, &a_val, &a_y, &a_w0, &a_prev, &a_rd, &a_words,
                        &a_n, &a_lr, &a_ctrl, &a_timeout};
        PDB_HIP(hipLaunchCooperativeKernel(fn, dim3((unsigned)grid), dim3(kBlock), args, 0, s));
    }
    if (nnz > 0) {
        k_stale_final<<<grid_for(nnz, kBlock, 8192), kBlock, 0, s>>>(csr->col, ws.words,
                                                                    ws.overwritten, nnz, w);
        PDB_LAUNCHED();
    }
    return PDB_OK;
}

}  // namespace
}  // namespace pdbk

using namespace pdbk;

extern "C" int pdb_stale_workspace_bytes(int64_t nnz, size_t *bytes) {
    if (!bytes || nnz < 0) return PDB_ERR_INVALID_ARG;
    if (nnz >= INT32_MAX) return PDB_ERR_UNSUPPORTED;
    *bytes = stale_layout(nullptr, nnz).total;
    return PDB_OK;
}

extern "C" int pdb_stale_epoch(const pdb_csr *csr, const float *labels, int64_t n, int64_t d,
                               float *w, float lr, int loss, int64_t delay,
                               const int32_t *prev_nz, void *ws, size_t ws_bytes,
                               const pdb_options *opt, hipStream_t s) {
    if (!csr || !ws || n < 0 || d < 0 || delay < 0) return PDB_ERR_INVALID_ARG;
    Opts o;
    const int orc = resolve_opts(opt, &o);
    if (orc != PDB_OK) return orc;
    if (n >= INT32_MAX || d >= INT32_MAX || csr->nnz >= INT32_MAX || csr->nnz < 0)
        return PDB_ERR_UNSUPPORTED;
    if (loss != PDB_LOGISTIC && loss != PDB_SQUARED) return PDB_ERR_INVALID_ARG;
    if (n > 0 && (!csr->row_ptr || !labels || !w)) return PDB_ERR_INVALID_ARG;
    if (csr->nnz > 0 && (!csr->col || !prev_nz)) return PDB_ERR_INVALID_ARG;
    StaleWs lay = stale_layout(ws, csr->nnz);
    if (ws_bytes < lay.total) return PDB_ERR_WORKSPACE;
    if (n == 0) return PDB_OK;
    const bool has_val = csr->val != nullptr;
    if (loss == PDB_LOGISTIC)
        return has_val ? launch_stale<PDB_LOGISTIC, true>(csr, labels, n, w, lr, delay, prev_nz, lay, o, s)
                       : launch_stale<PDB_LOGISTIC, false>(csr, labels, n, w, lr, delay, prev_nz, lay, o, s);
    return has_val ? launch_stale<PDB_SQUARED, true>(csr, labels, n, w, lr, delay, prev_nz, lay, o, s)
                   : launch_stale<PDB_SQUARED, false>(csr, labels, n, w, lr, delay, prev_nz, lay, o, s);
}
