// Exact top-k of short vectors (n < kMinFastN) without a sample: their first two launches (the third is
// k_finish_or_exact, topk.hip).
//
// A short vector's selection is a chain of latencies, not of bytes: the radix select over several blocks
// (k_exact, topk.hip) exchanges its histograms through the device five times, at 5-8 us each.  Here the pass that
// touches every element (the accumulation, or the read of v) leaves a histogram of its 4096 keys per block; the
// second launch adds those up, which finds T*'s bin, and flags the keys from there on; the third
// lists them in one block's LDS and selects there.  Nothing crosses blocks but by the launches' ends.
// Measured, accumulate + top-k of one node of 100 003 elements, k = 1 000, without a context: 44.5 us before (a
// clearing launch, the accumulation, k_exact 38 us), 20.4 us now.  A single block that scans v for itself in
// place of the last two launches took 31 us alone: reading and testing 400 KB is too much for one compute unit.
#include "device_helpers.h"

namespace lgc {

constexpr uint32_t kSmallChunk = 4096;   // elements per block of the first launch
constexpr int kSmallBins = 2048;

// The bins: octaves cut into 32 parts from 2^-27 to 2^8, into 8 from 2^-60 and up to 2^73, whole beyond.  What shares T*'s bin
// is listed and finished by one block: in a run in progress the residuals lie close below T*, and with 8 parts throughout (key >> 20)
// up to 21 000 of 262 143 elements did (k = 2 621; the list overflows at 12 288), with 32 parts 7 000.  Accumulate + top-k in such a
// run without a context, us, radix path / 8 parts / 32 parts: 262 143, k = 2 621: 46.9 / 55.8 / 30.9; k = 262: 45.0 / 31.1 / 20.2; 100 003, k = 4 000:
// 45.8 / 52.8 / 36.9; k = 1 000: 44.9 / 31.6 / 21.2; 20 000, k = 200: 35.6 / 15.6 / 15.7.
struct SmallZone { uint32_t octave, shift, bin; };
constexpr SmallZone kSmallZones[] = {{0, 23, 0}, {67, 20, 67}, {100, 18, 67 + 33 * 8}, {135, 20, 331 + 35 * 32}, {200, 23, 1451 + 65 * 8}};
static_assert(kSmallZones[4].bin + 56 <= kSmallBins, "bins");

__device__ __forceinline__ uint32_t small_bin(const uint32_t key) {
    uint32_t bin = key >> 23;
#pragma unroll
    for (int z = 1; z < 5; ++z) {
        const uint32_t first = kSmallZones[z].octave << 23;
        bin = key >= first ? kSmallZones[z].bin + ((key - first) >> kSmallZones[z].shift) : bin;
    }
    return bin;
}

// the least key of a bin
__device__ __forceinline__ uint32_t small_bin_key(const uint32_t bin) {
    uint32_t key = bin << 23;
#pragma unroll
    for (int z = 1; z < 5; ++z)
        key = bin >= kSmallZones[z].bin ? (kSmallZones[z].octave << 23) + ((bin - kSmallZones[z].bin) << kSmallZones[z].shift) : key;
    return key;
}

// the chunks' histograms lie where a sampled selection keeps its keys: two 16-bit counts per word
static_assert((size_t)((kMinFastN + kSmallChunk - 1) / kSmallChunk) * (kSmallBins / 2) <= kSample, "room for the chunks' histograms");

// u <- m u + g, v <- v + u (FUSED), the chunk's histogram, and the next call's state set cleared.  Four
// elements per thread: the shortest chain.
template <bool FUSED>
__global__ __launch_bounds__(1024) void k_small_pass(SelArgs a) {
    __shared__ __align__(16) uint32_t hist[kSmallBins];
    const int node = blockIdx.y, tid = threadIdx.x;
    {
        const uint32_t gt = (blockIdx.y * gridDim.x + blockIdx.x) * 1024u + tid, nt = gridDim.x * gridDim.y * 1024u;
        for (uint32_t i = gt; i < a.next_words; i += nt) a.next_state[i] = 0;
    }
    hist[tid] = 0; hist[tid + 1024] = 0;
    const size_t off = (size_t)node * a.stride;
    const uint32_t e = blockIdx.x * kSmallChunk + tid * 4;
    float *v = a.v + off, *u = a.u + off;
    const float *g = a.g + off;
    f4 vv = {0.f, 0.f, 0.f, 0.f};
    const uint32_t count = e >= a.n ? 0u : a.n - e < 4 ? a.n - e : 4u;
    if (count == 4) {
        vv = *(const f4u *)(v + e);
        if (FUSED) {
            f4 uu = *(const f4u *)(u + e);
            const f4 gg = *(const f4u *)(g + e);
#pragma unroll
            for (int j = 0; j < 4; ++j) { float x = uu[j], y = vv[j]; accum1(gg[j], x, y, a.momentum); uu[j] = x; vv[j] = y; }
            *(f4u *)(u + e) = uu;
            *(f4u *)(v + e) = vv;
        }
    } else {
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if ((uint32_t)j < count) {
                float y = v[e + j];
                if (FUSED) {
                    float x = u[e + j];
                    accum1(g[e + j], x, y, a.momentum);
                    u[e + j] = x; v[e + j] = y;
                }
                vv[j] = y;
            }
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 4; ++j)
        if ((uint32_t)j < count) atomicAdd(&hist[small_bin(key_of(vv[j]))], 1u);
    __syncthreads();
    a.samples[(size_t)node * kSample + blockIdx.x * (kSmallBins / 2) + tid] = hist[2 * tid] | (hist[2 * tid + 1] << 16);
}

// The candidate bitmap, row counts and records (as k_candidates writes them) of the keys in T*'s bin or above:
// every block adds up the chunks' histograms for itself.  Wavefront w of a block takes 256 elements: part w % 4 of row w / 4.
__global__ __launch_bounds__(1024) void k_small_flags(SelArgs a) {
    __shared__ __align__(16) uint32_t hist[kSmallBins];
    __shared__ uint32_t wave_tmp[16], res[2];
    constexpr int kRowsHere = kSmallChunk / kRow;
    __shared__ uint32_t part_sum[kRowsHere][4], rec[kRowsHere][kRecordWords];
    const int node = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint32_t chunks = gridDim.x, e = blockIdx.x * kSmallChunk + tid * 4;
    const float *v = a.v + (size_t)node * a.stride;
    f4 x = {0.f, 0.f, 0.f, 0.f};
    if (e < a.n && a.n - e >= 4) x = *(const f4u *)(v + e);
    else {
#pragma unroll
        for (int j = 0; j < 4; ++j) if (e + j < a.n) x[j] = v[e + j];
    }
    const uint32_t *h = a.samples + (size_t)node * kSample + tid;
    uint32_t lo = 0, hi = 0;
    for (uint32_t c0 = 0; c0 < chunks; c0 += 16) {
        uint32_t y[16];
#pragma unroll
        for (int c = 0; c < 16; ++c) y[c] = c0 + c < chunks ? h[(c0 + c) * (kSmallBins / 2)] : 0u;
#pragma unroll
        for (int c = 0; c < 16; ++c) { lo += y[c] & 0xffffu; hi += y[c] >> 16; }
    }
    hist[2 * tid] = lo; hist[2 * tid + 1] = hi;
    __syncthreads();
    find_rank_bin<kSmallBins, 1024>(hist, a.k, wave_tmp, res);
    const uint32_t least = small_bin_key(res[0]);   // (n >= k keys were counted: the bin exists)
    const int local = wave >> 2, part = wave & 3;
    const uint32_t row = blockIdx.x * kRowsHere + local, nrows = (a.n + kRow - 1) / kRow;
    unsigned long long word = 0;
    bool f[4];
    uint32_t count = 0, mine = 0;      // flags of the wavefront, of its lower lanes
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        f[j] = e + j < a.n && key_of(x[j]) >= least;
        const unsigned long long m = __ballot(f[j]);
        count += (uint32_t)__popcll(m);
        mine += lanes_below(m);
        if (lane == j) word = m;
    }
    if (row < nrows && lane < 4) a.bitmap[((size_t)node * a.rows + row) * kRowWords + part * 4 + lane] = word;
    if (lane == 0) part_sum[local][part] = count;
    __syncthreads();
    uint32_t total = 0;
#pragma unroll
    for (int p = 0; p < 4; ++p) { mine += p < part ? part_sum[local][p] : 0u; total += part_sum[local][p]; }
    if (total <= (uint32_t)kRecord) {
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (f[j]) {
                rec[local][mine] = __float_as_uint(x[j]);
                ((uint16_t *)(rec[local] + kRecord))[mine] = (uint16_t)(part * 256 + lane * 4 + j);
                ++mine;
            }
    }
    if (row < nrows && part == 0 && lane == 0) a.row_count[(size_t)node * a.rows + row] = total;
    __syncthreads();
    if (a.row_rec && row < nrows && part == 0 && lane < kRecord + kRecord / 2)   // (rows with more hold nothing of use)
        a.row_rec[((size_t)node * a.rec_stride + row) * kRecordWords + lane] = rec[local][lane];
}

// the finishing launch's list has to hold the selection and the keys that share T*'s bin
bool small_select_covers(uint64_t n, uint64_t k) { return n < kMinFastN && k <= kFinishList / 3; }

void launch_small_select(const SelArgs &a, int batch, bool fused, int cus, hipStream_t st, Bracket br) {
    const dim3 grid((a.n + kSmallChunk - 1) / kSmallChunk, batch);
    if (fused) launch_timed(k_small_pass<true>, grid, dim3(1024), st, br, a);
    else hipLaunchKernelGGL(k_small_pass<false>, grid, dim3(1024), 0, st, a);
    hipLaunchKernelGGL(k_small_flags, grid, dim3(1024), 0, st, a);
    launch_finish_from_bitmap(a, batch, false, cus, st);
}

}  // namespace lgc
