// Mini-batch gradient descent (gfx950, wave64): a batch of B consecutive
// examples is one iteration (Sec. 6.3 runs gradient descent with a fixed
// batch of examples per iteration).  Its parameter set is the union of its
// examples' features; within the iteration every read precedes every write
// (Definition 3), so all examples of a batch see the batch-start weights.
// Batches conflict when their unions share a feature; the read and write
// constraints of Sec. 4.4 at feature grain then order them, and Theorem 2
// lets batches of one conflict level run concurrently.
//
// Schedule: the union of each batch (features ascending) with, per union
// feature, the batch's entries on it in example order -- a stable sort of
// the entries by feature, then by batch -- is itself a CSR whose rows are the
// batches.  pdb_schedule on that CSR gives the batch levels.
//
// Epoch: one block per batch.  Phase 1: one wave per example, the dot
// product in the matched order (lane k holds entries k, k+64, ...), the step
// s_i = lr * g_i into LDS.  Phase 2: one thread per union feature applies the
// batch's contributions in example order, w = fma(-s_i, x, w), and writes the
// weight once.  Levels run one after another: a level wider than `thin` is
// spread over the grid followed by a device-wide barrier, runs of narrow
// levels go to block 0 with block barriers between batches.
//
// Sync-free epoch (no levels): blocks take batches in index order, and each
// weight and the union entry that last wrote it share a 64-bit word.  A batch
// waits for the words of its union, then runs the two phases
// (k_batch_syncfree); or, where few entries share their feature with another
// of the batch, its examples wait each for its own words (k_batch_flow).
#include <climits>

#include "pdb_math.h"
#include "pdb_words.h"

namespace pdbk {

namespace {

constexpr int kBB = 1024;                 // threads per batch block
constexpr int kBWaves = kBB / kWave;
constexpr int64_t kMaxBatch = 4096;       // examples per batch (LDS steps)
constexpr int kG = 8;                     // examples a wave loads together in phase 1
constexpr int kH = 8;                     // union features a thread takes in phase 2
constexpr int64_t kCap = kBB * kH;        // entries of a batch staged in LDS (8192)

// the sync-free epoch example by example (k_batch_flow): entries and examples of
// a batch, entries on features with several
constexpr int kFlowCap = 16384;
constexpr int kFlowB = 256;
constexpr int kFlowOcc = 4096;
constexpr int kFlowMany = kFlowCap;  // codes from here on: features with several entries
// the block's waves: workers, which run up to kFlowG examples each, and
// pollers, which wait for up to kFlowSlots words per lane
constexpr int kFlowWorkers = 13;
constexpr int kFlowPollers = kBWaves - kFlowWorkers;
constexpr int kFlowG = 8;
constexpr int kFlowSlots = 16;
constexpr int kFlowList = kFlowPollers * kWave * kFlowSlots;

// LDS of a batch block: steps by example; for staged batches the weights read
// in phase 1 by entry, and per occurrence its example (relative to the
// batch) and value
struct BatchShared {
    float s[kMaxBatch];
    float w[kCap];
    int32_t oi[kCap];
    float ox[kCap];
};

__device__ __forceinline__ int64_t readlane64(int64_t v, int lane) {
    const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)v, lane);
    const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)((uint64_t)v >> 32), lane);
    return (int64_t)(((uint64_t)hi << 32) | lo);
}

// row of every stored entry, one wave per row
__global__ __launch_bounds__(kBlock) void k_entry_row(const int64_t *__restrict__ row_ptr,
                                                      int64_t n, int32_t *__restrict__ row_idx) {
    const int lane = lane_id();
    const int64_t nw = (int64_t)gridDim.x * (kBlock / kWave);
    for (int64_t i = blockIdx.x * (int64_t)(kBlock / kWave) + wave_in_block(); i < n; i += nw) {
        const int64_t b = row_ptr[i], e = row_ptr[i + 1];
        for (int64_t p = b + lane; p < e; p += kWave) row_idx[p] = (int32_t)i;
    }
}

// keys of the second sort: the batch of each entry, in feature order
__global__ __launch_bounds__(kBlock) void k_batch_keys(const uint32_t *__restrict__ sv1,
                                                       int64_t nnz,
                                                       const int32_t *__restrict__ row_idx,
                                                       int64_t B, uint32_t *__restrict__ key2,
                                                       uint32_t *__restrict__ val2) {
    for (int64_t q = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; q < nnz;
         q += (int64_t)gridDim.x * blockDim.x) {
        const uint32_t p = sv1[q];
        key2[q] = (uint32_t)((int64_t)row_idx[p] / B);
        val2[q] = p;
    }
}

// entries in (batch, feature, index) order: occurrence lists, and a 1 at the
// first entry of every (batch, feature) group
__global__ __launch_bounds__(kBlock) void k_union_flags(const uint32_t *__restrict__ sk2,
                                                        const uint32_t *__restrict__ sv2,
                                                        int64_t nnz, const int32_t *__restrict__ col,
                                                        const int32_t *__restrict__ row_idx,
                                                        uint32_t *__restrict__ flag,
                                                        int32_t *__restrict__ occ,
                                                        int32_t *__restrict__ occ_row) {
    for (int64_t q = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; q < nnz;
         q += (int64_t)gridDim.x * blockDim.x) {
        const uint32_t p = sv2[q];
        occ[q] = (int32_t)p;
        occ_row[q] = row_idx[p];
        flag[q] = (q == 0 || sk2[q] != sk2[q - 1] || col[p] != col[sv2[q - 1]]) ? 1u : 0u;
    }
}

// union entries: feature, first occurrence, batch; the union size into
// *u_total (and uptr[U] = nnz)
__global__ __launch_bounds__(kBlock) void k_union_write(
    const uint32_t *__restrict__ sk2, const uint32_t *__restrict__ sv2, int64_t nnz,
    const int32_t *__restrict__ col, const uint32_t *__restrict__ uidx,
    int32_t *__restrict__ ucol, int64_t *__restrict__ uptr, uint32_t *__restrict__ ubatch,
    int32_t *__restrict__ occ_u, int64_t *__restrict__ u_total) {
    for (int64_t q = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; q < nnz;
         q += (int64_t)gridDim.x * blockDim.x) {
        const uint32_t p = sv2[q];
        const bool head = q == 0 || sk2[q] != sk2[q - 1] || col[p] != col[sv2[q - 1]];
        const int64_t u = uidx[q];
        // uidx counts the heads before q: q's own union entry is uidx[q] at a
        // head, uidx[q] - 1 elsewhere
        occ_u[q] = (int32_t)(head ? u : u - 1);
        if (head) {
            ucol[u] = col[p];
            uptr[u] = q;
            ubatch[u] = sk2[q];
        }
        if (q == nnz - 1) {
            const int64_t U = u + (head ? 1 : 0);
            uptr[U] = nnz;
            *u_total = U;
        }
    }
}

// bptr[b] = first union entry of batch b (union entries are in batch order);
// bptr[nb] already holds U
__global__ __launch_bounds__(kBlock) void k_bptr(const uint32_t *__restrict__ ubatch, int64_t nb,
                                                 int64_t *__restrict__ bptr) {
    const int64_t U = bptr[nb];
    for (int64_t b = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; b < nb;
         b += (int64_t)gridDim.x * blockDim.x) {
        int64_t lo = 0, hi = U;
        while (lo < hi) {
            const int64_t mid = (lo + hi) >> 1;
            if ((int64_t)ubatch[mid] < b) lo = mid + 1; else hi = mid;
        }
        bptr[b] = lo;
    }
}

// next union entry on the same feature (the inverse of the previous-writer
// relation over union entries), -1 if none
__global__ __launch_bounds__(kBlock) void k_union_next(const int32_t *__restrict__ uprev,
                                                       int64_t U, int32_t *__restrict__ unext) {
    for (int64_t u = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; u < U;
         u += (int64_t)gridDim.x * blockDim.x)
        if (uprev[u] >= 0) unext[uprev[u]] = (int32_t)u;
}

__global__ void k_fill32(int32_t *p, int64_t count, int32_t v) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < count;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

__global__ void k_fill64(int64_t *p, int64_t count, int64_t v) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < count;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

// ---------------------------------------------------------------------------
// epoch

// oi[q] (an example relative to the batch) becomes that example's step,
// stored in place as the float's bits; count occurrences, the whole block
__device__ __forceinline__ void resolve_steps(int32_t *oi, const float *s, int64_t count) {
    for (int64_t q = threadIdx.x; q < count; q += kBB) oi[q] = __float_as_int(s[oi[q]]);
}

// w after the contributions of occurrences [q0, q1): w = fma(-step, x, w)
// in order; the loads of a group of 8 are issued before its fmas
template <bool VAL>
__device__ __forceinline__ float chain_apply(float w, const float *step, const float *x,
                                             int32_t q0, int32_t q1) {
    int32_t q = q0;
    for (; q + 8 <= q1; q += 8) {
        float sv[8], xv[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            sv[k] = step[q + k];
            xv[k] = VAL ? x[q + k] : 1.0f;
        }
#pragma unroll
        for (int k = 0; k < 8; ++k) w = __builtin_fmaf(-sv[k], xv[k], w);
    }
    for (; q < q1; ++q) w = __builtin_fmaf(-step[q], VAL ? x[q] : 1.0f, w);
    return w;
}

template <int LOSS, bool VAL>
struct BatchOp {
    const int64_t *row_ptr;
    const int32_t *col;
    const float *val;
    const float *y;
    float *w;
    const int64_t *bptr;
    const int32_t *ucol;
    const int64_t *uptr;
    const int32_t *occ;
    const int32_t *occ_row;
    const int32_t *occ_u;
    const int32_t *unext;  // may be null
    int64_t n, B;
    float lr;

    // Batch b with the whole block.  Sh holds the batch's steps and, when the
    // batch has at most kCap entries, the weights phase 1 read (by entry) and
    // each occurrence's example and value, so that phase 2 reads LDS only.
    __device__ __forceinline__ void run(int64_t b, BatchShared &Sh) const {
        const int lane = lane_id();
        const int wave = (int)(threadIdx.x >> 6);
        const int64_t i0 = b * B, i1 = min(i0 + B, n);
        const int64_t pb = row_ptr[i0], pe = row_ptr[i1];   // the batch's entries
        const int64_t ub = bptr[b], ue = bptr[b + 1];       // its union features
        const bool staged = pe - pb <= kCap;
        // union features this thread updates, and (staged) the entry of each
        // one's first occurrence, whose weight phase 1 reads
        // (positions fit in 32 bits: nnz < 2^31)
        int32_t f[kH], q0[kH], q1[kH], pf[kH];
        const int64_t u0 = ub + threadIdx.x;
#pragma unroll
        for (int h = 0; h < kH; ++h) {
            const int64_t u = u0 + (int64_t)kBB * h;
            const bool live = u < ue;
            f[h] = live ? ucol[u] : 0;
            q0[h] = live ? (int32_t)uptr[u] : 0;
            q1[h] = live ? (int32_t)uptr[u + 1] : 0;
        }
        if (staged) {
#pragma unroll
            for (int h = 0; h < kH; ++h)
                pf[h] = (u0 + (int64_t)kBB * h < ue) ? occ[q0[h]] - (int32_t)pb : 0;
            // occurrences of the batch are its entries' positions [pb, pe)
            for (int64_t q = pb + threadIdx.x; q < pe; q += kBB) {
                Sh.oi[q - pb] = occ_row[q] - (int32_t)i0;
                if (VAL) Sh.ox[q - pb] = val[occ[q]];
            }
        }
        // phase 1: every example against the batch-start weights.  A wave
        // takes kG examples at a time; every load is unconditional (indices
        // clamped into the batch's entries), so all of them are in flight
        // before the first use: row bounds (lane j for example j), two chunks
        // of 64 columns per example, then the weights.
        if (pe > pb) {
            for (int64_t base = i0 + wave; base < i1; base += (int64_t)kBWaves * kG) {
                const int64_t my_i = base + (int64_t)kBWaves * lane;
                const bool has = lane < kG && my_i < i1;
                const int64_t rb = row_ptr[has ? my_i : i0];
                const int64_t re = has ? row_ptr[my_i + 1] : rb;
                const float yv = y[has ? my_i : i0];
                int64_t p[kG], m[kG];
#pragma unroll
                for (int j = 0; j < kG; ++j) {
                    p[j] = readlane64(rb, j);
                    m[j] = readlane64(re, j) - p[j];
                }
                int c[2 * kG];
                float x[2 * kG], wv[2 * kG], acc[kG];
#pragma unroll
                for (int t = 0; t < 2 * kG; ++t) {
                    const int64_t e = min(max(p[t >> 1] + (t & 1) * kWave + lane, pb), pe - 1);
                    c[t] = col[e];
                    x[t] = VAL ? val[e] : 1.0f;
                }
#pragma unroll
                for (int t = 0; t < 2 * kG; ++t) wv[t] = w[c[t]];
#pragma unroll
                for (int j = 0; j < kG; ++j) {
                    const int k0 = lane, k1 = kWave + lane;
                    // lanes without an entry hold +0, as in the summation order
                    acc[j] = k0 < m[j] ? __builtin_fmaf(wv[2 * j], x[2 * j], 0.0f) : 0.0f;
                    if (k1 < m[j]) acc[j] = __builtin_fmaf(wv[2 * j + 1], x[2 * j + 1], acc[j]);
                    if (staged) {
                        if (k0 < m[j]) Sh.w[p[j] + k0 - pb] = wv[2 * j];
                        if (k1 < m[j]) Sh.w[p[j] + k1 - pb] = wv[2 * j + 1];
                    }
                }
#pragma unroll
                for (int j = 0; j < kG; ++j) {
                    if (base + (int64_t)kBWaves * j >= i1) break;  // wave-uniform
                    for (int64_t k = 2 * kWave + lane; k < m[j]; k += kWave) {
                        const float wk = w[col[p[j] + k]];
                        acc[j] = __builtin_fmaf(wk, VAL ? val[p[j] + k] : 1.0f, acc[j]);
                        if (staged) Sh.w[p[j] + k - pb] = wk;
                    }
                    const float yj =
                        __int_as_float(__builtin_amdgcn_readlane(__float_as_int(yv), j));
                    const float sj = sgd_scale<LOSS>(wave_sum64(acc[j]), yj, lr);
                    if (lane == 0) Sh.s[base + (int64_t)kBWaves * j - i0] = sj;
                }
            }
        } else {
            // no entries: z = 0 for every example
            for (int64_t i = i0 + threadIdx.x; i < i1; i += kBB)
                Sh.s[i - i0] = sgd_scale<LOSS>(0.0f, y[i], lr);
        }
        __syncthreads();
        // phase 2: each union feature takes the batch's contributions in
        // example order; no other batch of the level touches it
        if (staged) {
            resolve_steps(Sh.oi, Sh.s, pe - pb);
            __syncthreads();
#pragma unroll
            for (int h = 0; h < kH; ++h) {
                if (u0 + (int64_t)kBB * h >= ue) break;
                w[f[h]] = chain_apply<VAL>(Sh.w[pf[h]], reinterpret_cast<const float *>(Sh.oi),
                                           Sh.ox, q0[h] - (int32_t)pb, q1[h] - (int32_t)pb);
            }
        } else {
            for (int64_t u = u0; u < ue; u += kBB) {
                const int32_t fu = ucol[u];
                const int64_t qe = uptr[u + 1];
                float v = w[fu];
                for (int64_t q = uptr[u]; q < qe; ++q)
                    v = __builtin_fmaf(-Sh.s[occ_row[q] - i0], VAL ? val[occ[q]] : 1.0f, v);
                w[fu] = v;
            }
        }
        __syncthreads();
    }
};

// first level >= l whose width exceeds thin (L if none); block-uniform
__device__ int64_t batch_run_end(int64_t l, int64_t L, const int64_t *level_ptr, int64_t thin) {
    __shared__ int64_t s_w[kBWaves];
    for (int64_t start = l; start < L; start += kBB) {
        const int64_t c = start + threadIdx.x;
        const bool wide = c < L && level_ptr[c + 1] - level_ptr[c] > thin;
        const unsigned long long bal = __ballot(wide);
        if (lane_id() == 0)
            s_w[threadIdx.x >> 6] = bal ? start + (threadIdx.x & ~63) + (__ffsll(bal) - 1)
                                        : INT64_MAX;
        __syncthreads();
        int64_t m = INT64_MAX;
#pragma unroll
        for (int v = 0; v < kBWaves; ++v) m = min(m, s_w[v]);
        __syncthreads();
        if (m != INT64_MAX) return m;
    }
    return L;
}

template <int LOSS, bool VAL>
__global__ __launch_bounds__(kBB) void k_batch_levels(BatchOp<LOSS, VAL> op,
                                                     const int32_t *__restrict__ perm,
                                                     const int64_t *__restrict__ level_ptr,
                                                     const int32_t *__restrict__ n_levels,
                                                     int64_t thin, Ctrl *ctrl, int64_t timeout) {
    __shared__ BatchShared Sh;
    const int64_t L = *n_levels;
    if (gridDim.x == 1) {
        // one block: every batch in level order, one after another
        const int64_t nb = level_ptr[L];
        for (int64_t e = 0; e < nb; ++e) op.run(perm[e], Sh);
        return;
    }
    int64_t l = 0;
    while (l < L) {
        const int64_t beg = level_ptr[l], end = level_ptr[l + 1];
        if (end - beg <= thin) {
            const int64_t l2 = batch_run_end(l, L, level_ptr, thin);
            if (blockIdx.x == 0)
                for (int64_t e = beg; e < level_ptr[l2]; ++e) op.run(perm[e], Sh);
            l = l2;
        } else {
            for (int64_t e = beg + blockIdx.x; e < end; e += gridDim.x) op.run(perm[e], Sh);
            ++l;
        }
        if (l < L && !grid_barrier(ctrl, timeout)) return;
    }
}

// ---------------------------------------------------------------------------
// Sync-free mini-batch epoch (the Read Protocol of Sec. 5 at feature grain,
// with a batch as the iteration): no batch levels, no barriers.  Each
// feature's weight and the union entry that last wrote it share one 64-bit
// word.  Blocks take batches in index order; a batch waits until each of its
// union features' words carries that feature's previous union entry (the
// schedule's prev_nz over the union CSR, -1 for none), runs both phases on
// those values and publishes (new weight, its union entry).  The earliest
// unfinished batch never waits for a later one, so the grid always makes
// progress; batches that share no feature run concurrently on different CUs.

__global__ void k_bw_in(const float *__restrict__ w, unsigned long long *__restrict__ bw,
                        int64_t d) {
    for (int64_t f = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; f < d;
         f += (int64_t)gridDim.x * blockDim.x)
        bw[f] = word_pack(w[f], -1);
}

__global__ void k_bw_out(const unsigned long long *__restrict__ bw, float *__restrict__ w,
                         int64_t d) {
    for (int64_t f = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; f < d;
         f += (int64_t)gridDim.x * blockDim.x)
        w[f] = word_value(bw[f]);
}

// A value every thread of the block reads from the same LDS word after a
// barrier, made wave-uniform for the compiler: the ticket loop's exits and
// the block barriers inside it then compile to scalar branches, so every
// wave runs the same sequence of barriers by construction.
__device__ __forceinline__ int block_uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ int64_t block_uniform64(int64_t v) {
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)((uint64_t)v >> 32));
    return (int64_t)(((uint64_t)hi << 32) | lo);
}

// LDS of a sync-free batch block: steps; for staged batches the weights of
// the union features, each entry's union feature, and per occurrence its
// example and value
struct SfShared {
    float s[kMaxBatch];
    float uw[kCap];
    int32_t eu[kCap];   // fast_batch: union feature | occurrence position << 16
    int32_t oi[kCap];   // fast_batch: the occurrences' steps
    float ox[kCap];
    int64_t ticket;
    int ok;
};

// A batch of any size: wait for every union feature's previous writer, then
// both phases on the words themselves (staged in LDS when they fit).  False
// when a wait gave up; every thread of the block returns the same.
template <int LOSS, bool VAL>
__device__ bool general_batch(const BatchOp<LOSS, VAL> &op, const int32_t *uprev,
                              unsigned long long *bw, SfShared &Sh, int64_t i0, int64_t i1,
                              int64_t pb, int64_t pe, int64_t ub, int64_t ue, Ctrl *ctrl,
                              int64_t timeout) {
    const int lane = lane_id();
    const int wave = (int)(threadIdx.x >> 6);
    const bool staged = pe - pb <= kCap;  // (ue - ub <= pe - pb)
    bool ok = true;
    for (int64_t u0 = ub + wave * kWave; u0 < ue; u0 += kBB) {
        const int64_t u = u0 + lane;
        const bool live = u < ue;
        const int32_t f = live ? op.ucol[u] : 0;
        const int tag = live ? uprev[u] : -1;
        unsigned long long v = 0;
        if (!word_wait_wave(bw, live, f, tag, &v, ctrl, timeout)) {
            ok = false;
            break;
        }
        if (staged && live) {
            Sh.uw[u - ub] = word_value(v);
            const int64_t q1 = op.uptr[u + 1];
            for (int64_t q = op.uptr[u]; q < q1; ++q) {
                const int32_t p = op.occ[q];
                Sh.eu[p - pb] = (int32_t)(u - ub);
                Sh.oi[q - pb] = op.occ_row[q] - (int32_t)i0;
                if (VAL) Sh.ox[q - pb] = op.val[p];
            }
        }
    }
    if (!ok && lane == 0) Sh.ok = 0;
    __syncthreads();
    if (block_uniform(Sh.ok) == 0) return false;
    // phase 1: every example against the weights the batch read
    for (int64_t i = i0 + wave; i < i1; i += kBWaves) {
        const int64_t p0 = op.row_ptr[i], m = op.row_ptr[i + 1] - p0;
        float acc = 0.0f;
        for (int64_t k = lane; k < m; k += kWave) {
            const int64_t p = p0 + k;
            const float wk = staged ? Sh.uw[Sh.eu[p - pb]] : word_value(word_get(bw, op.col[p]));
            acc = __builtin_fmaf(wk, VAL ? op.val[p] : 1.0f, acc);
        }
        const float s = sgd_scale<LOSS>(wave_sum64(acc), op.y[i], op.lr);
        if (lane == 0) Sh.s[i - i0] = s;
    }
    __syncthreads();
    if (staged) {
        resolve_steps(Sh.oi, Sh.s, pe - pb);
        __syncthreads();
    }
    // phase 2: contributions in example order, then publish
    for (int64_t u = ub + threadIdx.x; u < ue; u += kBB) {
        const int32_t f = op.ucol[u];
        const int64_t qa = op.uptr[u], qe = op.uptr[u + 1];
        float v = staged ? Sh.uw[u - ub] : word_value(word_get(bw, f));
        if (staged) {
            v = chain_apply<VAL>(v, reinterpret_cast<const float *>(Sh.oi), Sh.ox,
                                 (int32_t)(qa - pb), (int32_t)(qe - pb));
        } else {
            for (int64_t q = qa; q < qe; ++q)
                v = __builtin_fmaf(-Sh.s[op.occ_row[q] - i0], VAL ? op.val[op.occ[q]] : 1.0f, v);
        }
        word_put(bw, f, word_pack(v, (int)u));
    }
    __syncthreads();
    return true;
}

// A batch of at most kBWaves * kG examples and kCap entries.  Everything
// that does not depend on other batches comes first -- each wave's example
// bounds, labels and values in registers, every entry's union feature and
// occurrence position and every occurrence's value in LDS, each thread's union
// features in registers -- then the words are read once and only those not
// yet written by their previous writer are polled; after that both phases
// run from LDS.  Sixteen waves share the unit's issue slots, and what lies
// between the last word's arrival and the publish is bound by them: every
// loop over a wave's examples or union features ends, by a scalar branch,
// with the ones the batch has (issuing all kG and kH of them, masked, took
// 35.1 ms where this takes 25.5: 5,000 batches of 100 examples of 50 Zipf-1.2
// features, 7.0 -> 5.1 us a batch).
template <int LOSS, bool VAL>
__device__ bool fast_batch(const BatchOp<LOSS, VAL> &op, const int32_t *uprev,
                           unsigned long long *bw, SfShared &Sh, int64_t b, int64_t nb,
                           int64_t i0, int64_t i1, int64_t pb, int64_t pe, int64_t ub,
                           int64_t ue, Ctrl *ctrl, int64_t timeout) {
    const int lane = lane_id();
    const int wave = block_uniform((int)(threadIdx.x >> 6));
    const int nE = (int)(pe - pb), nU = (int)(ue - ub);
    // this wave's examples i0 + wave + kBWaves * j, j < jn; this lane's union
    // features u0 + kBB * h, h < hn (the last may lie past nU)
    const int jn = block_uniform(max((int)(i1 - i0) - wave + kBWaves - 1, 0) / kBWaves);
    const int hn = block_uniform(max(nU - wave * kWave + kBB - 1, 0) / kBB);
    const int u0 = wave * kWave + lane;
    const int64_t my_i = i0 + wave + (int64_t)kBWaves * lane;
    const bool has = lane < kG && my_i < i1;
    const int64_t rb = op.row_ptr[has ? my_i : i0];
    const int num = has ? (int)(op.row_ptr[my_i + 1] - rb) : 0;
    const int rel = (int)(rb - pb);
    const float yv = op.y[has ? my_i : i0];
    // example j's first entry relative to pb, and its entry count
    auto first = [&](int j) { return __builtin_amdgcn_readlane(rel, j); };
    auto count = [&](int j) { return __builtin_amdgcn_readlane(num, j); };
    for (int q = threadIdx.x; q < nE; q += kBB) {
        const int32_t pq = op.occ[pb + q];
        if (VAL) Sh.ox[q] = op.val[pq];
        Sh.eu[pq - pb] = (op.occ_u[pb + q] - (int32_t)ub) | q << 16;
    }
    // union features: feature, previous union entry, occurrences q0 | q1 << 16,
    // and whether the next batch writes the feature too (publish those first;
    // union entries of the batches up to the next one end at soon_end)
    int32_t f[kH], tag[kH], qq[kH];
    float w[kH];
    unsigned urgent = 0, pend = 0;
    const int64_t soon_end = op.unext ? op.bptr[min(b + 2, nb)] : 0;
#pragma unroll
    for (int h = 0; h < kH; ++h) {
        f[h] = tag[h] = qq[h] = 0;
        w[h] = 0.0f;
        if (h >= hn) continue;
        const int u = u0 + kBB * h;
        if (u < nU) {
            f[h] = op.ucol[ub + u];
            tag[h] = uprev[ub + u];
            qq[h] = (int)(op.uptr[ub + u] - pb) | (int)(op.uptr[ub + u + 1] - pb) << 16;
            const int32_t nx = op.unext ? op.unext[ub + u] : -1;
            urgent |= nx >= 0 && nx < soon_end ? 1u << h : 0u;
            pend |= 1u << h;
        }
    }
    float x[VAL ? 2 * kG : 1];
    if constexpr (VAL) {
#pragma unroll
        for (int t = 0; t < 2 * kG; ++t) {
            const int k = (t & 1) * kWave + lane;
            x[t] = k < count(t >> 1) ? op.val[pb + first(t >> 1) + k] : 0.0f;
        }
    }
    __syncthreads();
    int32_t at[2 * kG];  // each entry's union feature | occurrence position << 16
#pragma unroll
    for (int t = 0; t < 2 * kG; ++t) {
        const int k = (t & 1) * kWave + lane;
        at[t] = k < count(t >> 1) ? Sh.eu[first(t >> 1) + k] : 0;
    }
    // reads: every word once, then those not yet written until they are
    int64_t t0 = 0;
    bool ok = true;
    for (int round = 0;; ++round) {
        unsigned long long v[kH];
#pragma unroll
        for (int h = 0; h < kH; ++h) {
            if (h >= hn) break;
            if (pend >> h & 1) v[h] = word_get(bw, f[h]);
        }
#pragma unroll
        for (int h = 0; h < kH; ++h) {
            if (h >= hn) break;
            if ((pend >> h & 1) && word_tag(v[h]) == tag[h]) {
                w[h] = word_value(v[h]);
                pend &= ~(1u << h);
            }
        }
        if (__ballot(pend != 0) == 0ull) break;
        // the abort flag is a device-scope load: not on the path of every poll
        if (round == 0) {
            t0 = now_ticks();
        } else if ((round & 31) == 0) {
            ok = !aborted(ctrl);
            if (ok && now_ticks() - t0 > timeout) {
                record_error(ctrl, DERR_WAIT_TIMEOUT);
                ok = false;
            }
            if (!ok) break;
        }
        word_backoff_short(round);
        __asm__ __volatile__("" ::: "memory");  // the next round loads again
    }
#pragma unroll
    for (int h = 0; h < kH; ++h) {
        if (h >= hn) break;
        Sh.uw[u0 + kBB * h] = w[h];
    }
    if (!ok && lane == 0) Sh.ok = 0;
    __syncthreads();
    if (block_uniform(Sh.ok) == 0) return false;
    // phase 1 from LDS: the wave's examples' sums, the step of example j in
    // lane j, all of them at once, then each entry's step to its occurrence
    float acc[kG], z = 0.0f;
#pragma unroll
    for (int j = 0; j < kG; ++j) {
        acc[j] = 0.0f;
        if (j >= jn) continue;
        const int m = count(j);
        const float a0 = Sh.uw[at[2 * j] & 0xFFFF];
        acc[j] = lane < m ? __builtin_fmaf(a0, VAL ? x[2 * j] : 1.0f, 0.0f) : 0.0f;
        if (m > kWave) {
            const float a1 = Sh.uw[at[2 * j + 1] & 0xFFFF];
            if (kWave + lane < m) acc[j] = __builtin_fmaf(a1, VAL ? x[2 * j + 1] : 1.0f, acc[j]);
            for (int k = 2 * kWave + lane; k < m; k += kWave) {
                const int e = Sh.eu[first(j) + k];
                acc[j] = __builtin_fmaf(Sh.uw[e & 0xFFFF], VAL ? Sh.ox[(unsigned)e >> 16] : 1.0f,
                                        acc[j]);
            }
        }
    }
#pragma unroll
    for (int j = 0; j < kG; ++j) {
        if (j >= jn) break;
        const float zj = wave_sum64(acc[j]);
        z = lane == j ? zj : z;
    }
    const float s = sgd_scale<LOSS>(z, yv, op.lr);
    float *const step = reinterpret_cast<float *>(Sh.oi);
#pragma unroll
    for (int j = 0; j < kG; ++j) {
        if (j >= jn) break;
        const int m = count(j);
        const float sj = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(s), j));
        if (lane < m) step[at[2 * j] >> 16] = sj;
        if (m > kWave) {
            if (kWave + lane < m) step[at[2 * j + 1] >> 16] = sj;
            for (int k = 2 * kWave + lane; k < m; k += kWave) step[Sh.eu[first(j) + k] >> 16] = sj;
        }
    }
    __syncthreads();
    // phase 2 from LDS; the features the next batch waits for are published
    // before the others (one CU issues a batch's thousands of scattered
    // stores, and the waiting batch needs only a few of them), before those of
    // any wave: a wave that is through with its chains would put its others ahead
    // of what a longer chain still owes.  With the barrier in between, batches of
    // 100 examples of 80 uniform features over 280,000 take 9.5 us for 15.1, of 30
    // over 200,000 4.5 for 7.3 (5.2 with every chain before any store), of 30-50
    // Zipf-1.2 features 3.4 for 4.1.
#pragma unroll
    for (int h = 0; h < kH; ++h) {
        if (h >= hn) break;
        w[h] = chain_apply<VAL>(w[h], step, Sh.ox, qq[h] & 0xFFFF, qq[h] >> 16);
        if (urgent >> h & 1) word_put(bw, f[h], word_pack(w[h], (int)ub + u0 + kBB * h));
    }
    __syncthreads();
#pragma unroll
    for (int h = 0; h < kH; ++h) {
        if (h >= hn) break;
        if (u0 + kBB * h < nU && !(urgent >> h & 1))
            word_put(bw, f[h], word_pack(w[h], (int)ub + u0 + kBB * h));
    }
    __syncthreads();
    return true;
}

// Which of the two executions takes an epoch's batches (by_example), from what
// the batches hold: nb of them of B examples, `samples` of them looked at for
// the counts of Ctrl (flow_*); fast: on average they fit fast_batch.
struct FlowRule {
    int64_t nb, samples, B;
    bool fast;
};
constexpr int64_t kFlowSamples = 128;
constexpr int kFlowNear = 8;

// Batches that cannot run example by example (k_batch_flow), counted over all
// batches, a wave per batch; and the sampled batches' counts, a block per
// batch, one batch from each of r.samples equal stretches of them (not every
// k-th: inputs repeat).  Batches beyond kFlowCap are not looked at.
__global__ __launch_bounds__(kBB) void k_batch_fit(const int64_t *__restrict__ row_ptr, int64_t n,
                                                   int64_t B, const int64_t *__restrict__ bptr,
                                                   const int64_t *__restrict__ uptr,
                                                   const int32_t *__restrict__ uprev, FlowRule r,
                                                   Ctrl *ctrl) {
    __shared__ int s_count;
    __shared__ unsigned s_awaited, s_crowded;
    if (threadIdx.x == 0) s_count = 0;
    __syncthreads();
    const int64_t nw = (int64_t)gridDim.x * kBWaves;
    int count = 0;
    for (int64_t b = (blockIdx.x * (int64_t)kBB + threadIdx.x) / kWave; b < r.nb; b += nw) {
        const int64_t i0 = b * B, i1 = min(i0 + B, n);
        bool over = row_ptr[i1] - row_ptr[i0] > kFlowCap;
        for (int64_t i = i0 + lane_id(); i < i1; i += kWave)
            over |= row_ptr[i + 1] - row_ptr[i] > 2 * kWave;
        count += __ballot(over) != 0;
    }
    if (lane_id() == 0 && count) atomicAdd(&s_count, count);
    for (int64_t s = blockIdx.x; s < r.samples; s += gridDim.x) {
        if (threadIdx.x == 0) s_awaited = s_crowded = 0;
        __syncthreads();
        const int64_t lo = s * r.nb / r.samples, hi = (s + 1) * r.nb / r.samples;
        const int64_t b = lo + (int64_t)((unsigned)s * 2654435761u >> 8) % (hi - lo);
        const int64_t ub = bptr[b], ue = bptr[b + 1], near = bptr[max(b - kFlowNear, (int64_t)0)];
        unsigned awaited = 0, crowded = 0;  // sums below kFlowCap and B kFlowCap
        if (uptr[ue] - uptr[ub] <= kFlowCap) {
            for (int64_t u = ub + threadIdx.x; u < ue; u += kBB) {
                const int64_t pv = uprev[u];
                const unsigned c = (unsigned)(uptr[u + 1] - uptr[u]);
                awaited += pv >= near;  // -1: none
                crowded += c >= 4 ? c * c : 0;
            }
            awaited = wave_sum_u32(awaited);
            crowded = wave_sum_u32(crowded);
            if (lane_id() == 0) {
                atomicAdd(&s_awaited, awaited);
                atomicAdd(&s_crowded, crowded);
            }
        }
        __syncthreads();
        if (threadIdx.x == 0 && uptr[ue] - uptr[ub] <= kFlowCap) {
            atomicAdd(&ctrl->flow_unions, (unsigned long long)(ue - ub));
            atomicAdd(&ctrl->flow_awaited, (unsigned long long)s_awaited);
            atomicAdd(&ctrl->flow_crowded, (unsigned long long)s_crowded);
        }
    }
    __syncthreads();
    if (threadIdx.x == 0 && s_count) atomicAdd(&ctrl->whole_batches, s_count);
}

// Example by example (k_batch_flow), where all of this holds; measured on both
// executions over some 500 inputs: uniform features, permuted ones, Zipf 0.3-1.0
// and features that a share of the examples has, 3 to 80 entries, batches of 8
// to 256 (us a batch, as a whole | by example):
//  * At most one batch in four does not fit.  k_batch_flow runs such a batch as a
//    whole too, but without fast_batch, whose registers would cost every batch
//    (8.9 -> 11.0 ms for 5,000 batches of 100).  100-180 uniform features,
//    batches of 50, none of which fits: 11.4 | 24; about 100 features, batches of
//    64, 19% of them too long: 11.5 | 5.6.
//  * Few words are awaited (union entries that one of the kFlowNear batches before
//    wrote): as a whole, a batch waits once for all of them, by example each is
//    polled by itself.  What it costs goes with the words per example, what
//    it gains with the share of the entries that need no wait.  Batches of 100 x 80
//    uniform features: 12.5 words, 0.16 of the entries, 10.1 | 7.3; 20 and 0.25 9.1 |
//    10.3; the same 8,000 features in every batch 5.0 | 33.  50 x 80: 12.6 and 0.16
//    5.3 | 4.7, 20 and 0.25 4.9 | 6.5.  32 x 80: 12.6 and 0.16 3.6 | 3.4; 32 x 30:
//    9 and 0.30 1.6 | 2.1.  16 x 80: 6.8 and 0.08 2.1 | 1.7, 12.5 and 0.16 2.1 | 2.5.
//    100 x 3: 1.1 and 0.38 2.5 | 0.67.  Batches beyond fast_batch take longer
//    as a whole: 200 x 30 11 and 0.38 20 | 7.1, 128 x 80 30 and 0.38 46 | 16, 200 x
//    40 36 and 0.90 29 | 17 (consecutive features 20 | 21.6), all 27.6 | 28.8.
//    Beyond 208 examples a batch takes two turns: 256 x 3 0.3 and 0.08 11.7 | 10.5,
//    0.8 and 0.25 12.1 | 13.2.
//  * At least two a batch are awaited, else little waits and what counts is the
//    staging: 32 x 10 of 40 million features 0.31 | 0.48, 8 x 3 0.6 words 0.17 |
//    0.30, 2 words 0.39 | 0.32; 100 x 10 2.5 words 1.2 | 0.54.
//  * No crowded features (of fast_batch's batches), which four or more of a
//    batch's examples share: those all wait for one word and the last of them
//    applies its list alone.  Squares of their counts per union entry: one
//    feature in every example beside 80 rare ones, batches of 50 0.6 5.4 | 12.0,
//    of 100 1.2 11.1 | 24.8, of 16 0.2 1.7 | 4.0; in half of them, batches of 32
//    0.1 3.3 | 4.1; 80 Zipf-0.7 features of 20 million, batches of 32 0.017
//    2.4 | 3.9, of 16 0.004 1.65 | 2.2; one in a tenth of the examples, batches of
//    100 0.014 10.7 | 3.6, of 32 0.004 3.2 | 1.8, of 16 0.0009 1.6 | 1.25.
__device__ __forceinline__ bool by_example(const Ctrl *ctrl, FlowRule r) {
    const unsigned long long unions = ctrl->flow_unions, awaited = ctrl->flow_awaited;
    const unsigned long long samples = r.samples, examples = samples * r.B;
    if (4 * (int64_t)ctrl->whole_batches > r.nb || awaited < 2 * samples) return false;
    if (!r.fast)
        return r.B > 2 * kFlowWorkers * kFlowG ? 8 * awaited <= unions
                                               : awaited <= 30 * examples &&
                                                     10 * awaited <= 9 * unions;
    const bool few = r.B < 32;  // at most two or three examples a worker
    if ((few ? 512 : r.B < 64 ? 128 : 64) * ctrl->flow_crowded > unions) return false;
    return (awaited <= 4 * examples && 2 * awaited <= unions) ||
           (few ? awaited <= 7 * examples && 10 * awaited <= unions
                : awaited <= 13 * examples && 5 * awaited <= unions);
}

template <int LOSS, bool VAL>
__global__ __launch_bounds__(kBB) void k_batch_syncfree(BatchOp<LOSS, VAL> op,
                                                       const int32_t *__restrict__ uprev,
                                                       unsigned long long *bw, int64_t nb,
                                                       bool flow, FlowRule rule, Ctrl *ctrl,
                                                       int64_t timeout) {
    __shared__ SfShared Sh;
    if (flow && by_example(ctrl, rule)) return;
    for (;;) {
        if (threadIdx.x == 0) {
            Sh.ticket = (int64_t)atomicAdd(&ctrl->ticket, 1ull);
            Sh.ok = 1;
        }
        __syncthreads();
        const int64_t b = block_uniform64(Sh.ticket);
        if (b >= nb) return;
        const int64_t i0 = b * op.B, i1 = min(i0 + op.B, op.n);
        const int64_t pb = op.row_ptr[i0], pe = op.row_ptr[i1];
        const int64_t ub = op.bptr[b], ue = op.bptr[b + 1];
        if (pe - pb <= kCap && i1 - i0 <= (int64_t)kBWaves * kG) {
            if (!fast_batch(op, uprev, bw, Sh, b, nb, i0, i1, pb, pe, ub, ue, ctrl, timeout))
                return;
        } else {
            if (!general_batch(op, uprev, bw, Sh, i0, i1, pb, pe, ub, ue, ctrl, timeout)) return;
        }
    }
}

// LDS of a batch run example by example (flow_batch).  Per entry, the weight
// its example reads (until that word is read: the tag it waits for) and a
// code: its union feature relative to the batch, or, where the feature has
// several entries in the batch, kFlowMany + a number into the m arrays.  Those hold
// the feature, its entries' examples and values in example order, and how
// many of its examples have not run yet.
struct FlowShared {
    float w[kFlowCap];
    uint16_t code[kFlowCap];
    float s[kFlowB];           // steps by example
    float mx[kFlowOcc];
    uint16_t mi[kFlowOcc];
    uint16_t mfeat[kFlowOcc / 2], mbase[kFlowOcc / 2], mcount[kFlowOcc / 2];
    int32_t mleft[kFlowOcc / 2];
    // awaited entries: e | (worker << 4 | its example) << 16
    int32_t list[kFlowList];
    int32_t cnt[kFlowWorkers * 16];  // words an example still waits for
    int32_t ready[kFlowWorkers];     // a worker's examples that wait for none
    int nm, nocc, np, stop;
};
static_assert(2 * kFlowG <= 16 && kFlowWorkers <= 16 && kFlowCap <= 1 << 16, "packing of list");

// The batch's structure into LDS, none of it dependent on earlier batches.
// False when too many entries share their feature.
template <int LOSS, bool VAL>
__device__ bool flow_stage(const BatchOp<LOSS, VAL> &op, const int32_t *uprev, FlowShared &S,
                           int64_t i0, int64_t pb, int64_t ub, int64_t ue) {
    if (threadIdx.x == 0) S.nm = S.nocc = 0;
    __syncthreads();
    // kH union features per thread at a time, each of their loads in flight
    // together
    for (int64_t u0 = ub + threadIdx.x; u0 < ue; u0 += kCap) {
        int32_t a[kH], z[kH], e[kH], tag[kH];
#pragma unroll
        for (int h = 0; h < kH; ++h) {
            const int64_t u = min(u0 + (int64_t)kBB * h, ue - 1);
            a[h] = (int32_t)op.uptr[u];  // nnz < 2^31
            z[h] = (int32_t)op.uptr[u + 1];
            tag[h] = uprev[u];
        }
#pragma unroll
        for (int h = 0; h < kH; ++h) e[h] = op.occ[a[h]] - (int32_t)pb;
#pragma unroll
        for (int h = 0; h < kH; ++h) {
            const int64_t u = u0 + (int64_t)kBB * h;
            if (u >= ue) break;
            const int n = z[h] - a[h];
            if (n == 1) {
                S.code[e[h]] = (uint16_t)(u - ub);
                S.w[e[h]] = __int_as_float(tag[h]);
                continue;
            }
            const int base = atomicAdd(&S.nocc, n);
            if (base + n > kFlowOcc) continue;  // seen below
            const int mid = atomicAdd(&S.nm, 1);
            S.mfeat[mid] = (uint16_t)(u - ub);
            S.mbase[mid] = (uint16_t)base;
            S.mcount[mid] = (uint16_t)n;
            S.mleft[mid] = n;
            for (int k = 0; k < n; ++k) {
                const int32_t q = op.occ[a[h] + k];
                S.code[q - (int32_t)pb] = (uint16_t)(kFlowMany + mid);
                S.w[q - (int32_t)pb] = __int_as_float(tag[h]);
                S.mi[base + k] = (uint16_t)(op.occ_row[a[h] + k] - (int32_t)i0);
                S.mx[base + k] = VAL ? op.val[q] : 1.0f;
            }
        }
    }
    __syncthreads();
    return block_uniform(S.nocc) <= kFlowOcc;
}

// the wave's number in the block, wave-uniform for the compiler too: the waves'
// roles then are scalar branches, and neither role keeps the other's registers
__device__ __forceinline__ int flow_wave() {
    return __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
}

// v, opaque to the compiler: what is computed from it is computed where it is
// used and not kept in registers from the start
__device__ __forceinline__ int here(int v) {
    __asm__ volatile("" : "+v"(v));
    return v;
}

// words by 32-bit byte offset (one scalar base for every access)
__device__ __forceinline__ unsigned long long flow_get(const unsigned long long *bw, unsigned off) {
    return __hip_atomic_load(reinterpret_cast<const unsigned long long *>(
                                 reinterpret_cast<const char *>(bw) + (size_t)(unsigned)here((int)off)),
                             __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void flow_put(unsigned long long *bw, unsigned off,
                                         unsigned long long w) {
    __hip_atomic_store(
        reinterpret_cast<unsigned long long *>(reinterpret_cast<char *>(bw) +
                                               (size_t)(unsigned)here((int)off)),
        w,
        __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// A worker: examples g + wave + kFlowWorkers j, j < G.
template <int LOSS, bool VAL, int G>
struct FlowWorker {
    int rel, num;  // lane j: first entry (relative to the batch's) and entry count of example j
    float y;       // lane j: its label
    unsigned c[2 * G];  // entry 64 h + lane of example j at t = 2 j + h: its word's offset, value
    // stored values: kept where they fit the registers, else read again by run()
    static constexpr bool kKeep = VAL && G <= kFlowG;
    float x[kKeep ? 2 * G : 1];
    unsigned todo;  // examples still to run (wave-uniform)

    __device__ __forceinline__ int first(int j) const { return __builtin_amdgcn_readlane(rel, j); }
    __device__ __forceinline__ int count(int j) const { return __builtin_amdgcn_readlane(num, j); }

    // this lane's value of example j's entry 64 h + lane (which exists)
    __device__ __forceinline__ float value(const BatchOp<LOSS, VAL> &op, int64_t pb, int j,
                                           int h) const {
        if constexpr (kKeep) return x[2 * j + h];
        if constexpr (VAL) return op.val[pb + first(j) + h * kWave + lane_id()];
        return 1.0f;
    }

    // returns the lane's live entries as a bit mask
    __device__ __forceinline__ unsigned load(const BatchOp<LOSS, VAL> &op, int64_t g, int64_t i1,
                                             int64_t pb) {
        const int lane = lane_id();
        const int64_t i = g + flow_wave() + (int64_t)kFlowWorkers * lane;
        const bool has = lane < G && i < i1;
        const int64_t rb = op.row_ptr[has ? i : g];
        num = has ? (int)(op.row_ptr[i + 1] - rb) : 0;
        rel = (int)(rb - pb);
        y = op.y[has ? i : g];
        todo = (unsigned)__ballot(has);
        unsigned live = 0;
#pragma unroll
        for (int t = 0; t < 2 * G; ++t) {
            const int k = (t & 1) * kWave + lane;
            const bool lv = k < count(t >> 1);
            const int64_t e = pb + first(t >> 1) + k;
            live |= lv ? 1u << t : 0u;
            c[t] = lv ? 8u * (unsigned)op.col[e] : 0u;
            if constexpr (kKeep) x[t] = lv ? op.val[e] : 1.0f;
        }
        return live;
    }

    // reads the words of the lane's entries in `pend`; those that carry their
    // tag go to LDS, the others are returned
    __device__ __forceinline__ unsigned read(unsigned long long *bw, FlowShared &S, unsigned pend) {
        const int lane = lane_id();
        constexpr int kC = 8;  // words in flight per lane
#pragma unroll
        for (int t0 = 0; t0 < 2 * G; t0 += kC) {
            if (__ballot(pend >> t0 & ((1u << kC) - 1)) == 0ull) continue;
            unsigned long long v[kC];
#pragma unroll
            for (int k = 0; k < kC; ++k)
                if (pend >> (t0 + k) & 1) v[k] = flow_get(bw, c[t0 + k]);
#pragma unroll
            for (int k = 0; k < kC; ++k) {
                const int t = t0 + k;
                if (pend >> t & 1) {
                    float &w = S.w[first(t >> 1) + here((t & 1) * kWave + lane)];
                    if (word_tag(v[k]) == __float_as_int(w)) {
                        w = word_value(v[k]);
                        pend &= ~(1u << t);
                    }
                }
            }
        }
        return pend;
    }

    // lists the awaited entries from list position `at` on, counts them per
    // example and marks the examples that wait for none
    __device__ __forceinline__ void list(FlowShared &S, unsigned pend, int at) {
        const int lane = lane_id(), wave = flow_wave();
        int mine = 0;
#pragma unroll
        for (int t = 0; t < 2 * G; ++t) {
            const unsigned long long bal = __ballot(pend >> t & 1);
            if (pend >> t & 1)
                S.list[at + (int)lanes_below(bal)] =
                    (first(t >> 1) + (t & 1) * kWave + lane) | (wave << 4 | t >> 1) << 16;
            at += __popcll(bal);
            mine += lane == t >> 1 ? __popcll(bal) : 0;
        }
        if (lane < G) S.cnt[wave * 16 + lane] = mine;
        const unsigned none = (unsigned)__ballot(mine == 0) & todo;
        if (lane == 0) S.ready[wave] = (int)none;
    }

    // Runs the examples in `ready`: their sums, then lane j takes example j's step
    // (all lanes at once), then their entries' new weights.
    __device__ __forceinline__ void run(const BatchOp<LOSS, VAL> &op, unsigned long long *bw,
                                        FlowShared &S, unsigned ready, int ex0, int64_t pb, int ub) {
        const int lane = lane_id();
        float z = 0.0f;
#pragma unroll
        for (int j = 0; j < G; ++j) {
            if (!(ready >> j & 1)) continue;
            const int p = here(first(j)), m = count(j);
            float acc = 0.0f;
            if (lane < m) acc = __builtin_fmaf(S.w[p + lane], value(op, pb, j, 0), 0.0f);
            if (kWave + lane < m)
                acc = __builtin_fmaf(S.w[p + kWave + lane], value(op, pb, j, 1), acc);
            const float zj = wave_sum64(acc);
            z = lane == j ? zj : z;
        }
        const float s = sgd_scale<LOSS>(z, y, op.lr);
        if (lane < G && (ready >> lane & 1)) S.s[ex0 + kFlowWorkers * lane] = s;
        __asm__ __volatile__("" ::: "memory");
#pragma unroll
        for (int j = 0; j < G; ++j) {
            if (!(ready >> j & 1)) continue;
            const float sj = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(s), j));
            const int p = here(first(j)), m = count(j);
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int k = h * kWave + lane;
                if (k >= m) continue;
                const float w = S.w[p + k];
                int f = S.code[p + k];
                float nv = __builtin_fmaf(-sj, value(op, pb, j, h), w);
                if (f >= kFlowMany) {
                    // LDS runs one wave's operations in order: the step is
                    // there before the count says so
                    const int mid = f - kFlowMany;
                    if (atomicSub(&S.mleft[mid], 1) != 1) continue;
                    __asm__ __volatile__("" ::: "memory");
                    const int q0 = S.mbase[mid], n = S.mcount[mid];
                    nv = w;
                    for (int q = q0; q < q0 + n; ++q)
                        nv = __builtin_fmaf(-S.s[S.mi[q]], S.mx[q], nv);
                    f = S.mfeat[mid];
                }
                flow_put(bw, c[2 * j + h], word_pack(nv, ub + f));
            }
        }
    }
};

// A poller: waits for its share of the listed words, puts each into LDS as it
// comes and hands an example to its worker with its last one.
template <int LOSS, bool VAL>
__device__ void flow_poll(const BatchOp<LOSS, VAL> &op, unsigned long long *bw, FlowShared &S,
                          int64_t pb, int np, Ctrl *ctrl, int64_t timeout) {
    const int lane = lane_id();
    const int first = (flow_wave() - kFlowWorkers) * kWave + lane;
    int le[kFlowSlots], lt[kFlowSlots];
    unsigned lc[kFlowSlots];
    unsigned lp = 0;  // bit k: the lane awaits its k-th word
#pragma unroll
    for (int k = 0; k < kFlowSlots; ++k) {
        const int r = first + k * kFlowPollers * kWave;
        const bool in = r < np;
        le[k] = in ? S.list[r] : 0;
        lc[k] = in ? 8u * (unsigned)op.col[pb + (le[k] & 0xFFFF)] : 0u;
        lt[k] = in ? __float_as_int(S.w[le[k] & 0xFFFF]) : 0;
        lp |= in ? 1u << k : 0u;
    }
    int64_t t0 = now_ticks();  // last time the watchdog saw a word come
    unsigned seen = lp;
    for (int round = 0; __ballot(lp != 0) != 0ull; ++round) {
        if ((round & 31) == 31) {
            const int64_t t = now_ticks();
            if (__ballot(seen != lp) != 0ull) t0 = t;
            seen = lp;
            const bool late = t - t0 > timeout;
            if (late) record_error(ctrl, DERR_WAIT_TIMEOUT);
            if (late || aborted(ctrl)) {
                S.stop = 1;
                return;
            }
        }
        constexpr int kC = 8;
#pragma unroll
        for (int k0 = 0; k0 < kFlowSlots; k0 += kC) {
            if (__ballot(lp >> k0 & ((1u << kC) - 1)) == 0ull) continue;
            __asm__ __volatile__("" ::: "memory");  // the loads below are issued again
            unsigned long long v[kC];
#pragma unroll
            for (int k = 0; k < kC; ++k)
                if (lp >> (k0 + k) & 1) v[k] = flow_get(bw, lc[k0 + k]);
#pragma unroll
            for (int i = 0; i < kC; ++i) {
                const int k = k0 + i;
                if ((lp >> k & 1) && word_tag(v[i]) == lt[k]) {
                    lp &= ~(1u << k);
                    S.w[here(le[k]) & 0xFFFF] = word_value(v[i]);
                    __asm__ __volatile__("" ::: "memory");  // LDS runs one wave's operations in order
                    const int ex = here(le[k]) >> 16;
                    if (atomicSub(&S.cnt[ex], 1) == 1) atomicOr(&S.ready[ex >> 4], 1 << (ex & 15));
                }
            }
        }
    }
}

// Examples g .. (up to kFlowWorkers * G of them) of a staged batch.
// False when a wait gave up; every thread of the block returns the same.
template <int LOSS, bool VAL, int G>
__device__ bool flow_group(const BatchOp<LOSS, VAL> &op, unsigned long long *bw, FlowShared &S,
                           int64_t i0, int64_t g, int64_t i1, int64_t pb, int64_t ub, Ctrl *ctrl,
                           int64_t timeout) {
    const int wave = flow_wave();
    const bool worker = wave < kFlowWorkers;
    FlowWorker<LOSS, VAL, G> W;
    unsigned pend = 0;
    if (worker) pend = W.load(op, g, i1, pb);
    if (threadIdx.x == 0) S.np = S.stop = 0;
    __syncthreads();
    // every word once (again while more of them are awaited than the list holds)
    const int64_t t0 = now_ticks();
    int at = 0, np = 0;
    for (;;) {
        if (worker) {
            pend = W.read(bw, S, pend);
            int n = 0;
#pragma unroll
            for (int t = 0; t < 2 * G; ++t) n += __popcll(__ballot(pend >> t & 1));
            if (lane_id() == 0) at = atomicAdd(&S.np, n);
            at = __builtin_amdgcn_readfirstlane(at);
        }
        __syncthreads();
        np = block_uniform(S.np);
        if (np <= kFlowList) break;
        __syncthreads();
        if (threadIdx.x == 0) {
            S.np = 0;
            const bool late = now_ticks() - t0 > timeout;
            if (late) record_error(ctrl, DERR_WAIT_TIMEOUT);
            if (late || aborted(ctrl)) S.stop = 1;
        }
        __syncthreads();
        if (block_uniform(S.stop)) return false;
    }
    if (worker) W.list(S, pend, at);
    __syncthreads();
    if (worker) {
        const int ex0 = (int)(g - i0) + wave;
        for (int spin = 0; W.todo;) {
            const unsigned r = (unsigned)__builtin_amdgcn_readfirstlane(
                __hip_atomic_load(&S.ready[wave], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP));
            const unsigned ready = r & W.todo;
            if (ready) {
                __builtin_amdgcn_s_setprio(2);
                __asm__ __volatile__("" ::: "memory");
                W.run(op, bw, S, ready, ex0, pb, (int)ub);
                W.todo &= ~ready;
                __builtin_amdgcn_s_setprio(0);
                spin = 0;
                continue;
            }
            if ((++spin & 15) == 0 &&
                __builtin_amdgcn_readfirstlane(__hip_atomic_load(
                    &S.stop, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)))
                break;
            __builtin_amdgcn_s_sleep(1);
        }
    } else {
        __builtin_amdgcn_s_setprio(1);
        flow_poll<LOSS, VAL>(op, bw, S, pb, np, ctrl, timeout);
        __builtin_amdgcn_s_setprio(0);
    }
    __syncthreads();
    return block_uniform(S.stop) == 0;
}

// Sync-free epoch where a batch's features mostly have one entry each: batches
// run example by example.  An example runs as soon as its own words carry
// their previous union entries, not when the whole batch's do, so a hand-over
// between batches costs one device-scope hop and one example's arithmetic, and
// only examples that share a feature wait for each other: the chain is 2,738
// hops long where 5,000 batches of 100 examples of 80 uniform features over
// 2 million form a chain of 5,000 whole batches (94 -> 8.8 ms; batches of
// 200: 285 -> 20.8 ms).  An entry that is its feature's only one in the batch
// publishes the new weight at once (no other example of the batch reads it);
// of several, the example that gets there last applies all of them in example
// order and publishes.  Nothing in a batch waits for the same batch, so the
// earliest unfinished batch always makes progress.
//
// The block's waves split into workers and pollers: vector memory operations
// complete in order, so a wave that both published and polled would see its
// next words only after its stores were acknowledged (10.3 ms with sixteen
// waves that each did both).  A worker reads its examples' words once, then
// touches only LDS and its registers until it publishes.  Sixteen waves leave a
// lane 128 registers; of what the roles hold 35 to 47 go to scratch with G = 8,
// 83 to 119 with 16 (fast_batch: 0 to 2, with stored values 17 to 21).
template <int LOSS, bool VAL, int G>
__global__ __launch_bounds__(kBB) void k_batch_flow(BatchOp<LOSS, VAL> op,
                                                   const int32_t *__restrict__ uprev,
                                                   unsigned long long *bw, int64_t nb,
                                                   FlowRule rule, Ctrl *ctrl, int64_t timeout) {
    __shared__ union {
        SfShared g;
        FlowShared f;
    } Sh;
    __shared__ int64_t s_ticket;
    __shared__ int s_long;
    if (!by_example(ctrl, rule)) return;
    for (;;) {
        if (threadIdx.x == 0) {
            s_ticket = (int64_t)atomicAdd(&ctrl->ticket, 1ull);
            s_long = 0;
        }
        __syncthreads();
        const int64_t b = block_uniform64(s_ticket);
        if (b >= nb) return;
        const int64_t i0 = b * op.B, i1 = min(i0 + op.B, op.n);
        const int64_t pb = op.row_ptr[i0], pe = op.row_ptr[i1];
        const int64_t ub = op.bptr[b], ue = op.bptr[b + 1];
        bool fits = pe - pb <= kFlowCap && i1 - i0 <= kFlowB;
        if (fits) {
            const int64_t i = i0 + threadIdx.x;
            if (i < i1 && op.row_ptr[i + 1] - op.row_ptr[i] > 2 * kWave) s_long = 1;
            fits = flow_stage<LOSS, VAL>(op, uprev, Sh.f, i0, pb, ub, ue);
            fits = fits && block_uniform(s_long) == 0;
            __syncthreads();
        }
        if (fits) {
            for (int64_t g = i0; g < i1; g += kFlowWorkers * G)
                if (!flow_group<LOSS, VAL, G>(op, bw, Sh.f, i0, g, i1, pb, ub, ctrl, timeout)) return;
        } else {
            if (threadIdx.x == 0) Sh.g.ok = 1;
            __syncthreads();
            if (!general_batch(op, uprev, bw, Sh.g, i0, i1, pb, pe, ub, ue, ctrl, timeout)) return;
        }
    }
}

__global__ void k_batch_ctrl_zero(Ctrl *c) {
    int *w = reinterpret_cast<int *>(c);
    for (int i = threadIdx.x; i < (int)(sizeof(Ctrl) / sizeof(int)); i += blockDim.x) w[i] = 0;
}

template <int LOSS, bool VAL>
int launch_batch(const BatchOp<LOSS, VAL> &op, const pdb_levels *lv, Ctrl *ctrl, const Opts &opt,
                 hipStream_t s) {
    const int64_t thin = opt.batch_thin_max;
    const int64_t timeout = opt.timeout;
    k_batch_ctrl_zero<<<1, 64, 0, s>>>(ctrl);
    PDB_LAUNCHED();
    const void *fn = reinterpret_cast<const void *>(&k_batch_levels<LOSS, VAL>);
    int grid = 1;
    if (lv->max_width_host > thin) {
        // the level barrier needs every block of the grid resident at once:
        // one block per CU at most (a 1024-thread block always fits one CU)
        int dev = 0, cus = 0, per_cu = 0;
        PDB_HIP(hipGetDevice(&dev));
        PDB_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
        PDB_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, kBB, 0));
        if (per_cu < 1) return PDB_ERR_HIP;
        grid = (int)std::max<int64_t>(1, std::min<int64_t>(cus, lv->max_width_host));
    }
    BatchOp<LOSS, VAL> o = op;
    const int32_t *perm = lv->perm;
    const int64_t *level_ptr = lv->level_ptr;
    const int32_t *n_levels = lv->n_levels;
    if (grid == 1) {
        k_batch_levels<LOSS, VAL><<<1, kBB, 0, s>>>(o, perm, level_ptr, n_levels, thin, ctrl,
                                                    timeout);
        PDB_LAUNCHED();
    } else {
        int64_t thin_arg = thin, to = timeout;
        void *args[] = {&o, &perm, &level_ptr, &n_levels, &thin_arg, &ctrl, &to};
        PDB_HIP(hipLaunchCooperativeKernel(fn, dim3(grid), dim3(kBB), args, 0, s));
    }
    return PDB_OK;
}

int64_t batch_sf_ws_bytes(int64_t d) { return (int64_t)sizeof(Ctrl) + align_up(8 * d); }

template <int LOSS, bool VAL>
int launch_batch_syncfree(const BatchOp<LOSS, VAL> &op, const pdb_levels *lv, int64_t d,
                          int64_t nb, int64_t nnz, int64_t U, void *ws, const Opts &opt,
                          hipStream_t s) {
    Ctrl *ctrl = static_cast<Ctrl *>(ws);
    unsigned long long *bw =
        reinterpret_cast<unsigned long long *>(static_cast<char *>(ws) + sizeof(Ctrl));
    const int64_t timeout = opt.timeout;
    k_batch_ctrl_zero<<<1, 64, 0, s>>>(ctrl);
    PDB_LAUNCHED();
    if (d > 0) {
        k_bw_in<<<grid_for(d, kBlock, 8192), kBlock, 0, s>>>(op.w, bw, d);
        PDB_LAUNCHED();
    }
    // one block per CU (the LDS of a block fills most of a CU); blocks need
    // not be co-resident: the earliest unfinished batch is always running
    int dev = 0, cus = 0;
    PDB_HIP(hipGetDevice(&dev));
    PDB_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
    // at most 32 blocks by default: more batches in flight only add polls
    // that slow the frontier's memory accesses
    const int64_t cap = opt.batch_sf_blocks;
    const int grid = (int)std::max<int64_t>(1, std::min<int64_t>(std::min<int64_t>(cus, cap), nb));
    // Example by example where by_example says so, else a batch at a time.  Asked
    // only where few entries share their feature with another of the batch (at
    // 3.6% of them 200,000 examples of 30 uniform features over 20,000, batches of
    // 50, took 16.7 ms a batch at a time and 15.7 by example, at 5.8% 20.9 and
    // 26.9, at 58%, Zipf 1.2, 25 and 87).  A block takes one batch, so batches of
    // fewer examples than about half a block's waves leave it idle (50,000
    // examples of 80 features over 2 million: batches of 4 3.1 and 3.8 ms, of 8
    // 4.4 and 2.3 ms).  It addresses words with 32-bit byte offsets.
    const bool flow = U > 0 && 32 * (nnz - U) <= nnz && op.B >= 8 && op.B <= kFlowB &&
                      d <= int64_t(1) << 28;
    const bool fast = op.B <= (int64_t)kBWaves * kG && nnz <= kCap * nb;  // fast_batch, on average
    const FlowRule rule{nb, std::min(nb, kFlowSamples), op.B, fast};
    if (flow) {
        // what a batch holds is on the device: both kernels are launched, and
        // one of them returns at once (5 us)
        k_batch_fit<<<grid_for(std::max(rule.samples, cdiv(nb, kBWaves)), 1, 512), kBB, 0, s>>>(
            op.row_ptr, op.n, op.B, op.bptr, op.uptr, lv->prev_nz, rule, ctrl);
        PDB_LAUNCHED();
        // the most examples per worker that a batch needs, so that they are all in
        // flight together: with half as many, batches of 128 took 50 ms, not 15.7
        if (op.B <= kFlowWorkers * kFlowG)
            k_batch_flow<LOSS, VAL, kFlowG><<<grid, kBB, 0, s>>>(op, lv->prev_nz, bw, nb, rule,
                                                                 ctrl, timeout);
        else
            k_batch_flow<LOSS, VAL, 2 * kFlowG><<<grid, kBB, 0, s>>>(op, lv->prev_nz, bw, nb,
                                                                     rule, ctrl, timeout);
        PDB_LAUNCHED();
    }
    k_batch_syncfree<LOSS, VAL><<<grid, kBB, 0, s>>>(op, lv->prev_nz, bw, nb, flow, rule, ctrl,
                                                       timeout);
    PDB_LAUNCHED();
    if (d > 0) {
        k_bw_out<<<grid_for(d, kBlock, 8192), kBlock, 0, s>>>(bw, op.w, d);
        PDB_LAUNCHED();
    }
    return PDB_OK;
}

int check_batch_sizes(int64_t n, int64_t d, int64_t nnz, int64_t B) {
    if (n < 0 || d < 0 || nnz < 0 || B < 1) return PDB_ERR_INVALID_ARG;
    if (B > kMaxBatch) return PDB_ERR_INVALID_ARG;
    if (n >= INT32_MAX || d >= INT32_MAX || nnz >= INT32_MAX) return PDB_ERR_UNSUPPORTED;
    return PDB_OK;
}

int bits_for(uint64_t maxval) {
    int b = 0;
    while (maxval) {
        ++b;
        maxval >>= 1;
    }
    return b > 0 ? b : 1;
}

}  // namespace
}  // namespace pdbk

using namespace pdbk;

extern "C" int pdb_batch_schedule(const pdb_csr *csr, int64_t n, int64_t d, int64_t batch,
                                  pdb_batches *bt, pdb_levels *lv, int method,
                                  pdb_schedule_info *info, void *ws, size_t ws_bytes,
                                  const pdb_options *opt, hipStream_t s) {
    if (!csr || !bt || !lv || !ws || (n > 0 && !csr->row_ptr) || (csr->nnz > 0 && !csr->col))
        return PDB_ERR_INVALID_ARG;
    const int64_t nnz = csr->nnz;
    int rc = check_batch_sizes(n, d, nnz, batch);
    if (rc != PDB_OK) return rc;
    {
        Opts o;
        rc = resolve_opts(opt, &o);  // checked here, applied by pdb_schedule
        if (rc != PDB_OK) return rc;
    }
    if (d == 0 && nnz > 0) return PDB_ERR_BAD_CSR;
    if (!bt->bptr || !bt->uptr ||
        (nnz > 0 && (!bt->ucol || !bt->occ || !bt->occ_row || !bt->occ_u)))
        return PDB_ERR_INVALID_ARG;
    SchedWs w = sched_ws_layout(ws, n, d, nnz);
    if (ws_bytes < w.total) return PDB_ERR_WORKSPACE;
    const int64_t nb = cdiv(n, batch);
    if (nnz == 0) {
        k_fill64<<<grid_for(nb + 1, kBlock, 4096), kBlock, 0, s>>>(bt->bptr, nb + 1, 0);
        k_fill64<<<1, 64, 0, s>>>(bt->uptr, 1, 0);
        PDB_LAUNCHED();
        bt->U_host = 0;
    } else {
        k_entry_row<<<grid_for(n, kBlock / kWave, 65536), kBlock, 0, s>>>(csr->row_ptr, n,
                                                                          w.row_idx);
        PDB_LAUNCHED();
        // entries by feature (stable), then by batch (stable): (batch, feature, index)
        uint32_t *sk1, *sv1, *sk2, *sv2;
        PDB_HIP(radix_sort_pairs(reinterpret_cast<const uint32_t *>(csr->col), nullptr, nnz,
                                 bits_for((uint64_t)(d > 1 ? d - 1 : 1)), w.kA, w.vA, w.kB, w.vB,
                                 w.hist, w.scan_tmp, &sk1, &sv1, s));
        // the second sort reads its input from the occurrence arrays, which
        // are rewritten below
        uint32_t *key2 = reinterpret_cast<uint32_t *>(bt->occ);
        uint32_t *val2 = reinterpret_cast<uint32_t *>(bt->occ_row);
        k_batch_keys<<<grid_for(nnz, kBlock, 1 << 16), kBlock, 0, s>>>(sv1, nnz, w.row_idx, batch,
                                                                      key2, val2);
        PDB_LAUNCHED();
        PDB_HIP(radix_sort_pairs(key2, val2, nnz, bits_for((uint64_t)(nb > 1 ? nb - 1 : 1)), w.kA,
                                 w.vA, w.kB, w.vB, w.hist, w.scan_tmp, &sk2, &sv2, s));
        uint32_t *flag = (sk2 == w.kA) ? w.kB : w.kA;   // the pair not holding the result
        uint32_t *ubatch = (sk2 == w.kA) ? w.vB : w.vA;
        k_union_flags<<<grid_for(nnz, kBlock, 1 << 16), kBlock, 0, s>>>(
            sk2, sv2, nnz, csr->col, w.row_idx, flag, bt->occ, bt->occ_row);
        PDB_LAUNCHED();
        PDB_HIP(exclusive_scan_u32(flag, flag, nnz, w.scan_tmp, s));
        k_union_write<<<grid_for(nnz, kBlock, 1 << 16), kBlock, 0, s>>>(
            sk2, sv2, nnz, csr->col, flag, bt->ucol, bt->uptr, ubatch, bt->occ_u, bt->bptr + nb);
        PDB_LAUNCHED();
        if (nb > 0) {
            k_bptr<<<grid_for(nb, kBlock, 65536), kBlock, 0, s>>>(ubatch, nb, bt->bptr);
            PDB_LAUNCHED();
        }
        int64_t U = 0;
        PDB_HIP(hipMemcpyAsync(&U, bt->bptr + nb, sizeof(U), hipMemcpyDeviceToHost, s));
        PDB_HIP(hipStreamSynchronize(s));
        bt->U_host = U;
    }
    // the batch levels: conflict levels of the union CSR, whose rows are the batches
    const pdb_csr ucsr{bt->bptr, bt->ucol, nullptr, bt->U_host};
    rc = pdb_schedule(&ucsr, nullptr, nb, d, lv, method, info, ws, ws_bytes, opt, s);
    if (rc != PDB_OK) return rc;
    // each union entry's next writer, when asked for and known
    if (bt->unext && bt->U_host > 0) {
        k_fill32<<<grid_for(bt->U_host, kBlock, 65536), kBlock, 0, s>>>(bt->unext, bt->U_host, -1);
        PDB_LAUNCHED();
        if (lv->prev_nz) {
            k_union_next<<<grid_for(bt->U_host, kBlock, 65536), kBlock, 0, s>>>(
                lv->prev_nz, bt->U_host, bt->unext);
            PDB_LAUNCHED();
        }
        PDB_HIP(hipStreamSynchronize(s));
    }
    return PDB_OK;
}

extern "C" int pdb_batch_epoch(const pdb_csr *csr, const float *labels, int64_t n, int64_t d,
                               int64_t batch, float *w, float lr, int loss,
                               const pdb_batches *bt, const pdb_levels *lv, void *ws,
                               size_t ws_bytes, const pdb_options *opt, hipStream_t s) {
    if (!csr || !labels || !w || !bt || !lv || !ws || !lv->perm || !lv->level_ptr ||
        !lv->n_levels)
        return PDB_ERR_INVALID_ARG;
    const int64_t nnz = csr->nnz;
    int rc = check_batch_sizes(n, d, nnz, batch);
    if (rc != PDB_OK) return rc;
    if (loss != PDB_LOGISTIC && loss != PDB_SQUARED) return PDB_ERR_INVALID_ARG;
    if (ws_bytes < sizeof(Ctrl)) return PDB_ERR_WORKSPACE;
    if (n == 0) return PDB_OK;
    if (!bt->bptr || !bt->uptr ||
        (nnz > 0 && (!bt->ucol || !bt->occ || !bt->occ_row || !bt->occ_u)))
        return PDB_ERR_INVALID_ARG;
    Ctrl *ctrl = static_cast<Ctrl *>(ws);
    Opts o;
    rc = resolve_opts(opt, &o);
    if (rc != PDB_OK) return rc;
    // sync-free when the previous writers over the union CSR are known and the
    // workspace holds a word per feature, unless the epoch mode option asks
    // for batch levels
    const bool sf_ok = lv->prev_nz != nullptr && (int64_t)ws_bytes >= batch_sf_ws_bytes(d);
    const bool syncfree = sf_ok && o.epoch_mode != PDB_EPOCH_LEVELS;
    const int64_t nb = cdiv(n, batch);
#define PDB_BATCH(LOSS, VAL)                                                                     \
    (syncfree ? launch_batch_syncfree<LOSS, VAL>(                                              \
                    BatchOp<LOSS, VAL>{csr->row_ptr, csr->col, csr->val, labels, w, bt->bptr,   \
                                       bt->ucol, bt->uptr, bt->occ, bt->occ_row, bt->occ_u,         \
                                       bt->unext, n, batch, lr}, \
                    lv, d, nb, nnz, bt->U_host, ws, o, s)                                                        \
              : launch_batch<LOSS, VAL>(                                                       \
                    BatchOp<LOSS, VAL>{csr->row_ptr, csr->col, csr->val, labels, w, bt->bptr,   \
                                       bt->ucol, bt->uptr, bt->occ, bt->occ_row, bt->occ_u,         \
                                       bt->unext, n, batch, lr}, \
                    lv, ctrl, o, s))
    if (loss == PDB_LOGISTIC) return csr->val ? PDB_BATCH(PDB_LOGISTIC, true) : PDB_BATCH(PDB_LOGISTIC, false);
    return csr->val ? PDB_BATCH(PDB_SQUARED, true) : PDB_BATCH(PDB_SQUARED, false);
#undef PDB_BATCH
}
