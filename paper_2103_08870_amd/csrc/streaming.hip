// The streaming kernels of liblgc for gfx950 (wave64): the passes that touch every element of g, u, v.
//
// What is computed (paper: Alg. 1 / Alg. 2, first line of the layer loop, with the momentum correction of
// Sec. V-A):   u <- m*u + g ; v <- v + u   -- three separately rounded fp32 operations per element --
// and, in the candidate pass, the flags "key(v) >= t_est" (key = bits(v) & 0x7fffffff) that the selection
// kernels (topk.hip, segmented.hip) work from: one bit per element in a dense bitmap, one count per row of
// 1024 elements.  One wavefront per row, twelve 16-byte loads in flight before anything depends on them,
// non-temporal loads and stores, no barrier, no atomics, nothing shared between wavefronts.

#include "device_helpers.h"

namespace lgc {

// ------------------------------------------------------------------ one row of a wavefront

// One full row of a wavefront: 4 x 256 consecutive elements, lane l holds elements 4l..4l+3 of
// each 256.  All twelve 16-byte loads are issued before anything depends on them.  Every stream
// is touched once per call, so all loads and stores are non-temporal: on this part that alone
// lifts the fused kernel from about 60 % to 72-77 % of the HBM peak (and the plain read of v in
// the selection-only form likewise; the few candidates' values are read again by the gather).
// ZERO: elements with key >= t_zero are stored as zeros; bits, ubits: what v and u would have been.
template <bool FUSED, bool ZERO>
__device__ __forceinline__ void full_row(const float *__restrict__ g, float *__restrict__ u, float *__restrict__ v,
                                         const float m, uint32_t (&bits)[4][4], const uint32_t t_zero, uint32_t (&ubits)[4][4]) {
    static_assert(FUSED || !ZERO, "a pass that writes");
    f4 gg[4], uu[4], vv[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        if (FUSED) {
            gg[s] = __builtin_nontemporal_load((const f4u *)(g + s * 256));
            uu[s] = __builtin_nontemporal_load((const f4u *)(u + s * 256));
        }
        vv[s] = __builtin_nontemporal_load((const f4u *)(v + s * 256));
    }
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        if (FUSED) {
#pragma unroll
            for (int j = 0; j < 4; ++j) { float x = uu[s][j], y = vv[s][j]; accum1(gg[s][j], x, y, m); uu[s][j] = x; vv[s][j] = y; }
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            bits[s][j] = __float_as_uint(vv[s][j]);
            if (ZERO) {
                ubits[s][j] = __float_as_uint(uu[s][j]);
                const bool zero = (bits[s][j] & 0x7fffffffu) >= t_zero;
                vv[s][j] = zero ? 0.f : vv[s][j];
                uu[s][j] = zero ? 0.f : uu[s][j];
            }
        }
        if (FUSED) {
            __builtin_nontemporal_store(uu[s], (f4u *)(u + s * 256));
            __builtin_nontemporal_store(vv[s], (f4u *)(v + s * 256));
        }
    }
}

// ------------------------------------------------------------------ plain accumulation

// Same traversal as the candidate pass below: one wavefront per row of 1024 elements,
// all twelve 16-byte loads of a row in flight before anything depends on them, non-temporal.
__global__ __launch_bounds__(kBlock) void k_accumulate(const float *__restrict__ g, float *__restrict__ u,
                                                       float *__restrict__ v, uint32_t n, uint64_t stride,
                                                       float m) {
    const size_t off = (size_t)blockIdx.y * stride;
    g += off; u += off; v += off;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint32_t nrows = (n + kRow - 1) / kRow;
    for (uint32_t r = blockIdx.x * kWaves + wave; r < nrows; r += gridDim.x * kWaves) {
        const uint32_t row = r * (uint32_t)kRow;
        const uint32_t end = (n - row > (uint32_t)kRow) ? row + kRow : n;
        if (row + 1024 <= end) {
            uint32_t bits[4][4], ubits[4][4];
            full_row<true, false>(g + row + lane * 4, u + row + lane * 4, v + row + lane * 4, m, bits, 0u, ubits);
        } else {
            for (uint32_t e = row + lane; e < end; e += 64) {
                float uu = u[e], vv = v[e];
                accum1(g[e], uu, vv, m);
                u[e] = uu; v[e] = vv;
            }
        }
    }
}

// Calls launch(node0, nodes, row_begin, row_end, events) for equal shares of at most kRowsPerLaunch rows:
// several whole nodes per launch while they fit, else one node in row ranges.  `events` carries the bracket's
// start event for the first share and its stop event for the last one.
template <typename F>
static void for_each_share(uint32_t nrows, int batch, Bracket br, F launch) {
    if ((uint64_t)nrows * batch <= kRowsPerLaunch) { launch(0u, batch, 0u, nrows, br); return; }
    if (nrows <= kRowsPerLaunch) {
        const int fit = (int)(kRowsPerLaunch / nrows);              // nodes that fit one launch
        const int launches = (batch + fit - 1) / fit;
        const int per = (batch + launches - 1) / launches;          // evened out
        for (int b = 0; b < batch; b += per) {
            Bracket e;
            if (b == 0) e.start = br.start;
            if (b + per >= batch) e.stop = br.stop;
            launch((uint32_t)b, batch - b < per ? batch - b : per, 0u, nrows, e);
        }
        return;
    }
    const uint32_t ranges = (nrows + kRowsPerLaunch - 1) / kRowsPerLaunch;
    const uint32_t per = ((nrows + ranges - 1) / ranges + (uint32_t)kWaves - 1) / kWaves * kWaves;   // whole blocks
    for (int b = 0; b < batch; ++b)
        for (uint32_t r = 0; r < nrows; r += per) {
            Bracket e;
            if (b == 0 && r == 0) e.start = br.start;
            if (b == batch - 1 && nrows - r <= per) e.stop = br.stop;
            launch((uint32_t)b, 1, r, nrows - r < per ? nrows : r + per, e);
        }
}

void launch_accumulate(const float *g, float *u, float *v, uint32_t n, int batch, uint64_t stride,
                       float momentum, hipStream_t st, Bracket br) {
    const uint32_t nrows = (n + kRow - 1) / kRow;
    for_each_share(nrows, batch, br, [&](uint32_t node0, int nodes, uint32_t r0, uint32_t r1, Bracket e) {
        // a share is passed as shifted pointers and its own length 
        const size_t off = (size_t)node0 * stride + (size_t)r0 * kRow;
        const uint32_t len = (r1 == nrows ? n : r1 * (uint32_t)kRow) - r0 * (uint32_t)kRow;
        dim3 grid((r1 - r0 + kWaves - 1) / kWaves, nodes);
        launch_timed(k_accumulate, grid, dim3(kBlock), st, e, g + off, u + off, v + off, len, stride, momentum);
    });
}

// ------------------------------------------------------------------ candidate pass (the streaming kernel)

// x with lane `lane` replaced by the wave-uniform value.  (A choice by lane number takes three instructions and, hoisted,
// 32 scalar registers: 72 -> 68 vector registers without records, 92 -> 70 with; 8 x 44.5 M elements, whole step: 1333 -> 1322 us.)  It is the compiler's own instruction and not inline assembly because it reads scalar registers that a compare
// has just written: the compiler puts the wait states in between that the hardware does not supply.
__device__ uint32_t write_lane(uint32_t value, uint32_t lane, uint32_t x) __asm("llvm.amdgcn.writelane.i32");

// ------------------------------------------------------------------ sampled candidate threshold

// A node without a carried threshold: the pass samples kSample of the keys that it WILL produce (the fused source recomputes
// v + (m*u + g) without storing it) and takes t_est = (roughly) the rank-th largest of them, to 2^-13 relative resolution: a
// first level from a histogram of key >> 20, a second from the keys.  The sample is cut into shares that are handed out
// through a ticket counter; the block that finishes the last one works out the estimate, and no block goes on to its rows, and
// so writes u or v, before it stands.  The first kShares blocks of the node take shares at once, the others (whose tickets would only
// queue up: atomics on one word take turns) after they have waited for some tens of microseconds.  So every share is with a running
// block or free for any block that waits, and the waits end whatever number of the kernel's blocks the device holds and
// whatever runs beside it.  They are bounded all the same.  A block that has waited too long settles on "no candidates", for the whole node:
// ctr->ready holds the one threshold that all of its blocks go by, whoever sets it first.  Rows cut at different thresholds would
// make a list that lacks elements above T*; a node without candidates takes the exact path.
// A launch of its own costs 4.6 us in a full queue where thresholds are carried and it has nothing to do, and 14 us where it samples; here sampling takes
// 25 to 300 us, as all blocks wait.  So this is for the odd selection in a run of carried ones (offers_hold, kOfferRun in api.hip).
constexpr uint32_t kShares = kSample / (4 * kBlock);
constexpr uint32_t kNoCandidates = 0x80000000u;   // a threshold above every key

template <bool FUSED>
__device__ __forceinline__ uint32_t sample_threshold(const SelArgs &a, const int node, uint32_t *hist /*[kSampleBins]*/) {
    __shared__ uint32_t wave_tmp[kWaves], res[2], word, stands;
    const int tid = threadIdx.x;
    Ctr *ctr = a.ctr + node;
    const size_t off = (size_t)node * a.stride;
    uint32_t *smp = a.samples + (size_t)node * kSample, *all = a.sample_hist + node * kSampleBins;
    bool helps = blockIdx.x < kShares;
    uint32_t spins = 0;
    for (;;) {
        __syncthreads();
        if (tid == 0) {
            uint32_t next = kShares, set = ld_agent32(&ctr->ready);   // a share's number (kShares: none left, or not asked yet); 1 + the threshold
            if (set == 0 && spins >= a.sample_spins) {
                set = atomicCAS(&ctr->ready, 0u, kNoCandidates + 1);
                if (set == 0) set = kNoCandidates + 1;
            }
            if (set == 0 && (helps || spins == 64)) { next = atomicAdd(&ctr->share, 1u); next = next < kShares ? next : kShares; }
            if (set == 0 && next == kShares) __builtin_amdgcn_s_sleep(16);
            word = next; stands = set;
        }
        __syncthreads();
        const uint32_t share = __builtin_amdgcn_readfirstlane(word), set = __builtin_amdgcn_readfirstlane(stands);
        if (set != 0) return set - 1;
        if (share == kShares) { helps = false; ++spins; continue; }      // (block-uniform)
        helps = true;
        const uint32_t j = share * kBlock + tid, e = sample_place(j, node, a.n);
        for (int i = tid; i < kSampleBins; i += kBlock) hist[i] = 0;
        __syncthreads();
        u4 keys;
        f4 vv, uu = {0.f, 0.f, 0.f, 0.f}, gg = {0.f, 0.f, 0.f, 0.f};
        vv = *(const f4u *)(a.v + off + e);
        if (FUSED) { uu = *(const f4u *)(a.u + off + e); gg = *(const f4u *)(a.g + off + e); }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float x = uu[i], y = vv[i];
            if (FUSED) accum1(gg[i], x, y, a.momentum);
            keys[i] = key_of(y);
            atomicAdd(&hist[keys[i] >> 20], 1u);
        }
        *(u4 *)(smp + j * 4) = keys;
        __syncthreads();
        for (int i = tid; i < kSampleBins; i += kBlock) { const uint32_t h = hist[i]; if (h) atomicAdd(&all[i], h); }
        // Every wavefront waits until its stores and atomics have been acknowledged, one thread releases them to the device and
        // counts the share.
        __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0)
        __syncthreads();
        if (tid == 0) {
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
            word = atomicAdd(&ctr->sampled, 1u) == kShares - 1 ? 1u : 0u;
        }
        __syncthreads();
        if (__builtin_amdgcn_readfirstlane(word) == 0) continue;
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");   // the other blocks' keys, through this XCD's caches
        // the key of the rank-th largest: first level, second level
        for (int i = tid; i < kSampleBins; i += kBlock) hist[i] = ld_agent32(&all[i]);
        __syncthreads();
        find_rank_bin<kSampleBins, kBlock>(hist, a.rank, wave_tmp, res);
        const uint32_t bin = res[0], rank = a.rank - res[1];
        __syncthreads();
        for (int i = tid; i < 1024; i += kBlock) hist[i] = 0;
        __syncthreads();
        constexpr int kAhead = 2;   // (four: 76 registers, room for six wavefronts per SIMD instead of seven; 3 x 3.33 M, whole step: 62.1 us for 61.7)
        static_assert(kSample / 4 % (kAhead * kBlock) == 0, "whole rounds");
#pragma unroll 1
        for (uint32_t i0 = tid; i0 < kSample / 4; i0 += kAhead * kBlock) {
            u4 x[kAhead];
#pragma unroll
            for (int r = 0; r < kAhead; ++r) x[r] = *(const u4 *)(smp + (i0 + r * kBlock) * 4);
#pragma unroll
            for (int r = 0; r < kAhead; ++r)
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    if ((x[r][c] >> 20) == bin) atomicAdd(&hist[(x[r][c] >> 10) & 1023u], 1u);
        }
        __syncthreads();
        find_rank_bin<1024, kBlock>(hist, rank, wave_tmp, res);
        if (tid == 0) atomicCAS(&ctr->ready, 0u, 1u + ((bin << 20) | ((res[0] == 0xffffffffu ? 0u : res[0]) << 10)));
    }
}

// FUSED: reads g,u,v, writes u,v (the accumulation) and classifies the new v; otherwise reads v.
// One wavefront per row of 1024 elements.  The flags "key >= t_est" of the row go out as one
// full 128-byte line of the candidate bitmap (dense, coalesced: no partial-line writes), the
// row's candidate count as one word.  REC: and the candidates of a row that holds a few (up to kRecord) as one
// record: their values and positions, so that the kernels after this one neither search the bitmap nor read v again at
// scattered places.  No barrier, no atomics, nothing shared (a wavefront puts its record together in its own part of the LDS).
// SEG: per-layer selection; the threshold of an element is that of its segment (a.seg_t, one per
// node and segment; 0xffffffff flags nothing).  a.row_seg names the segment of a row's first
// element, with bit 31 set when the row runs into further segments.
// ZERO (with REC; a.zero_early): elements with key >= t_zero, which are taken for selected, go out as zeros in u and v, and the
// record keeps their u as well; a row with more candidates than that record holds is written as it is after all.
// SAMPLE: takes the carried threshold, or samples one, itself, and clears the next call's state set (otherwise the launch before did).
template <bool FUSED, bool SEG, bool SAMPLE, bool ZERO, bool REC>
__global__ __launch_bounds__(kBlock) void k_candidates(SelArgs a) {
    __shared__ uint32_t record_lds[REC ? kWaves : 1][kRecordWords];
    const int node = a.node0 + blockIdx.y, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const size_t off = (size_t)node * a.stride;
    const float *__restrict__ g = a.g + off;
    float *__restrict__ u = a.u + off;
    float *__restrict__ v = a.v + off;
    static_assert(!ZERO || (FUSED && REC && !SEG), "zeros need records");
    constexpr uint32_t kMost = ZERO ? kZeroRecord : kRecord;   // candidates that a record holds
    static_assert(!SAMPLE || (!SEG && !ZERO), "one threshold");
    uint32_t t_est = SEG || SAMPLE ? 0u : a.sel[node].t_est;
    const uint32_t t_zero = ZERO ? a.sel[node].t_zero : 0u;
    if (SAMPLE) {
        __shared__ __align__(16) uint32_t hist[kSampleBins];
        // scalar loads, as nothing has been stored yet: vector loads here hold up the row's (4 x 25.6 M: 386 us for 382.6)
        const Carry *c = a.carry + node;
        const uint32_t c_n = c->n, c_k = c->k, c_est = c->next_t_est;
        // A node whose record of carried thresholds offers one for this very selection (same shape, the selection right after
        // the one that wrote it) takes that one and samples nothing.
        const bool offered = c_n == a.n && c_k == a.k && c_est != 0;
        t_est = offered ? c_est : sample_threshold<FUSED>(a, node, hist);
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            a.sel[node].t_est = t_est;
            if (offered) { a.sel[node].carried = 1; atomicAdd(&a.stats->carried, 1u); }
        }
    }
    const uint32_t *seg_t = SEG ? a.seg_t + (size_t)node * a.n_seg : nullptr;
    const float m = a.momentum;
    unsigned long long *bitmap = a.bitmap + (size_t)node * a.rows * kRowWords;
    uint32_t *row_count = a.row_count + (size_t)node * a.rows;
    const uint32_t r = a.row_begin + blockIdx.x * kWaves + wave;   // one row per wavefront (the launcher's grid)
    if (r < a.row_end) {
        const uint32_t row = r * (uint32_t)kRow;
        const uint32_t end = (a.n - row > (uint32_t)kRow) ? row + kRow : a.n;
        uint32_t bits[4][4], ubits[4][4];
        uint32_t thr[4][4];
        if (SEG) {
            const uint32_t rs = a.row_seg[r];
            uint32_t l = rs & 0x7fffffffu;
            const uint32_t t0 = seg_t[l];
#pragma unroll
            for (int s = 0; s < 4; ++s)
#pragma unroll
                for (int j = 0; j < 4; ++j) thr[s][j] = t0;
            if (rs >> 31) {   // wave-uniform: the row crosses into the next segment(s)
                for (++l; l < a.n_seg && a.seg_off[l] < end; ++l) {
                    const uint32_t ol = a.seg_off[l], tl = seg_t[l];
#pragma unroll
                    for (int s = 0; s < 4; ++s)
#pragma unroll
                        for (int j = 0; j < 4; ++j)
                            if (row + s * 256 + lane * 4 + j >= ol) thr[s][j] = tl;
                }
            }
        }
        if (row + 1024 <= end) {
            full_row<FUSED, ZERO>(g + row + lane * 4, u + row + lane * 4, v + row + lane * 4, m, bits, t_zero, ubits);
        } else {
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const uint32_t e0 = row + s * 256 + lane * 4;
                f4 vv = {0.f, 0.f, 0.f, 0.f}, uu = {0.f, 0.f, 0.f, 0.f};
                if (e0 + 3 < end) {
                    vv = *(const f4u *)(v + e0);
                    if (FUSED) {
                        const f4 gg = *(const f4u *)(g + e0);
                        uu = *(const f4u *)(u + e0);
#pragma unroll
                        for (int j = 0; j < 4; ++j) { float x = uu[j], y = vv[j]; accum1(gg[j], x, y, m); uu[j] = x; vv[j] = y; }
                        *(f4u *)(u + e0) = uu;
                        *(f4u *)(v + e0) = vv;
                    }
                } else {
                    for (int j = 0; j < 4; ++j) if (e0 + j < end) {
                        float y = v[e0 + j];
                        if (FUSED) {
                            float x = u[e0 + j];
                            accum1(g[e0 + j], x, y, m);
                            u[e0 + j] = x; v[e0 + j] = y;
                            uu[j] = x;
                        }
                        vv[j] = y;
                    }
                }
#pragma unroll
                for (int j = 0; j < 4; ++j) { bits[s][j] = __float_as_uint(vv[j]); if (ZERO) ubits[s][j] = __float_as_uint(uu[j]); }
            }
        }
        // 16 flag words of the row; lane i < 16 ends up holding word i
        uint32_t lo = 0, hi = 0, count = 0;
        unsigned long long flags[4][4];
#pragma unroll
        for (int s = 0; s < 4; ++s) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t e = row + s * 256 + lane * 4 + j;
                const unsigned long long mk = __ballot(e < end && (bits[s][j] & 0x7fffffffu) >= (SEG ? thr[s][j] : t_est));
                flags[s][j] = mk;
                count += (uint32_t)__popcll(mk);
                lo = write_lane((uint32_t)mk, s * 4 + j, lo);
                hi = write_lane((uint32_t)(mk >> 32), s * 4 + j, hi);
            }
        }
        if (lane < kRowWords && (count != 0 || !a.sparse_bitmap)) bitmap[(size_t)r * kRowWords + lane] = ((unsigned long long)hi << 32) | lo;
        if (lane == 0) row_count[r] = count;
        // the row's record, put together in the LDS and stored as whole lines (wave-uniform condition)
        if (ZERO) {   // (wave-uniform conditions)
            const bool whole = row + 1024 <= end;
            if (whole && count > kMost && t_zero != ~0u) {   // no record: what has gone out as zeros is written after all
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    const uint32_t e0 = row + s * 256 + lane * 4;
                    *(u4u *)(u + e0) = (u4){ubits[s][0], ubits[s][1], ubits[s][2], ubits[s][3]};
                    *(u4u *)(v + e0) = (u4){bits[s][0], bits[s][1], bits[s][2], bits[s][3]};
                }
            } else if (!whole && count <= kMost) { // the vector's last, shorter row has gone out as it is
#pragma unroll
                for (int s = 0; s < 4; ++s)
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        if (((flags[s][j] >> lane) & 1u) && (bits[s][j] & 0x7fffffffu) >= t_zero) {
                            u[row + s * 256 + lane * 4 + j] = 0.f;
                            v[row + s * 256 + lane * 4 + j] = 0.f;
                        }
            }
        }
        if (REC && count != 0 && count <= kMost) {
            uint32_t *rec = record_lds[wave];
            uint32_t at = 0;
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                if ((flags[s][0] | flags[s][1] | flags[s][2] | flags[s][3]) != 0) {
                    uint32_t mine = at;
#pragma unroll
                    for (int j = 0; j < 4; ++j) { mine += lanes_below(flags[s][j]); at += (uint32_t)__popcll(flags[s][j]); }
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        if ((flags[s][j] >> lane) & 1u) {
                            rec[mine] = bits[s][j];
                            ((uint16_t *)(rec + kMost))[mine] = (uint16_t)(s * 256 + lane * 4 + j);
                            if (ZERO) rec[kMost + kMost / 2 + mine] = ubits[s][j];
                            ++mine;
                        }
                    }
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            if (lane < (int)(ZERO ? 2 * kMost + kMost / 2 : kMost + kMost / 2)) a.row_rec[((size_t)node * a.rec_stride + r) * kRecordWords + lane] = rec[lane];
        }
    }
    if (SAMPLE) {
        const uint32_t gt = (blockIdx.y * gridDim.x + blockIdx.x) * kBlock + threadIdx.x, nt = gridDim.x * gridDim.y * kBlock;
        for (uint32_t i = gt; i < a.next_words; i += nt) a.next_state[i] = 0;
    }
}

void launch_candidates(const SelArgs &args, int batch, bool fused, hipStream_t st, Bracket br) {
    const uint32_t nrows = (args.n + kRow - 1) / kRow;
    const bool seg = args.seg_t != nullptr;
    for_each_share(nrows, batch, br, [&](uint32_t node0, int nodes, uint32_t r0, uint32_t r1, Bracket e) {
        SelArgs a = args;
        // Passes of several launches leave out the bitmap lines of rows without candidates (whole step without / with: 8 x 44.5 M 1316 / 1306 us,
        // 4 x 40 M 595 / 593); a pass of one launch writes them all, which then lie in the caches (4 x 25.6 M 382.6 when left out, 378.5 when not;
        // 60 M 240.7 / 242.3).  By layers it gains nothing (7 x 33.6 M 932 / 932), and the selection, which looks for a layer's ends in them, would have
        // to read the row's count first (4 x 3.1 M, 14 layers: 0.3 us).
        a.sparse_bitmap = !seg && (uint64_t)nrows * batch > kRowsPerLaunch;
        a.node0 = node0; a.row_begin = r0; a.row_end = r1;
        dim3 grid((r1 - r0 + kWaves - 1) / kWaves, nodes);
#define LGC_CAND(F, S, M, Z, R) launch_timed(k_candidates<F, S, M, Z, R>, grid, dim3(kBlock), st, e, a)
#define LGC_CAND_M(F, R) do { if (a.sample_in_pass) LGC_CAND(F, false, true, false, R); else LGC_CAND(F, false, false, false, R); } while (0)
        if (seg) { if (fused) LGC_CAND(true, true, false, false, false); else LGC_CAND(false, true, false, false, false); }
        else if (a.zero_early) LGC_CAND(true, false, false, true, true);
        else if (a.row_rec) { if (fused) LGC_CAND_M(true, true); else LGC_CAND_M(false, true); }
        else { if (fused) LGC_CAND_M(true, false); else LGC_CAND_M(false, false); }
#undef LGC_CAND_M
#undef LGC_CAND
    });
}

}  // namespace lgc
