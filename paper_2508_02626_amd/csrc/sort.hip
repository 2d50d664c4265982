// Device-wide exclusive scan and stable LSD radix sort of (u64 key, i32 value)
// pairs, written for 64-wide wavefronts.
//
// Sort: 8-bit digits.  Ranks among equal digits come from wavefront ballots (8
// ballots give each lane the mask of lanes sharing its digit) and per-digit
// prefixes over the wavefronts, so equal keys keep their input order
// (stability).  Ties of the Morton keys are thereby broken by the original
// index, which the values start out as.
//
// Plans of small and middling trees are bound by the number of launches (about
// 4.5 us each, back to back), so a sort or scan takes as few as its size allows:
//   sort   up to kSmallSort elements: one block holds them in LDS and runs every
//          pass (one launch); up to kDirectBlocks tiles: per pass a histogram and a
//          scatter whose blocks add up the histograms before them (two); beyond
//          that a scan of the histograms between the two (as many as it takes)
//   scan   up to kDirectTiles tiles: every block adds up what is before it (one);
//          up to kSumTiles of them: the tiles' sums, then the scan with
//          each block adding up the sums before it (two); else three
// Launches of a plan, its evaluation and its end, before -> with these: 1,000
// uniform points, order 4 82 -> 43 (458 -> 345 us), 17,389 Plummer points, order
// 8 105 -> 80 (1091 -> 984 us), 100,000 Gaussian points, order 6 1306 -> 1157 us.
// A scatter of 1024-element tiles over kDirectBlocks of them takes 10.8 us, 6 us
// over 34 tiles of 512: the sum over the blocks, which then outweighs the launch
// it saves if there are more.
#include "sort.h"

#include <algorithm>

namespace fmm {

constexpr int kThreads = 256;
constexpr int kItems = 8;
constexpr int kTile = kThreads * kItems;
constexpr int kWaves = kThreads / 64;

// ---------------- scan ----------------
template <typename T>
__global__ __launch_bounds__(kThreads) void k_scan_block_sums(const T *in, int64_t n, T *sums)
{
    __shared__ T sh[kWaves];
    int64_t base = (int64_t)blockIdx.x * kTile;
    T s = 0;
    for (int r = 0; r < kItems; ++r) {
        int64_t i = base + r * kThreads + threadIdx.x;
        if (i < n) s += in[i];
    }
    for (int o = 32; o > 0; o >>= 1) s += __shfl_down(s, o);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        T t = 0;
        for (int w = 0; w < kWaves; ++w) t += sh[w];
        sums[blockIdx.x] = t;
    }
}

// one block scans the block sums in place (exclusive), total at sums[nb]
template <typename T>
__device__ inline void k_scan_sums_body(T *sums, int nb)
{
    __shared__ T sh[1024];
    __shared__ T carry;
    if (threadIdx.x == 0) carry = 0;
    __syncthreads();
    for (int base = 0; base < nb; base += 1024) {
        int i = base + threadIdx.x;
        T v = i < nb ? sums[i] : 0;
        sh[threadIdx.x] = v;
        __syncthreads();
        for (int o = 1; o < 1024; o <<= 1) {
            T t = threadIdx.x >= o ? sh[threadIdx.x - o] : 0;
            __syncthreads();
            sh[threadIdx.x] += t;
            __syncthreads();
        }
        if (i < nb) sums[i] = carry + sh[threadIdx.x] - v;
        __syncthreads();
        if (threadIdx.x == 1023) carry += sh[1023];
        __syncthreads();
    }
    if (threadIdx.x == 0) sums[nb] = carry;
}

// the block's tile of the exclusive scan, `before` the sum of what precedes it;
// the last block writes the total to out[n] if asked
template <typename T>
__device__ inline void k_scan_apply_body(const T *in, int64_t n, T before, T *out, bool write_total)
{
    __shared__ T sh[kThreads];
    int64_t base = (int64_t)blockIdx.x * kTile;
    T v[kItems];
    T tot = 0;
    for (int r = 0; r < kItems; ++r) {
        int64_t i = base + threadIdx.x * kItems + r;
        v[r] = i < n ? in[i] : 0;
        tot += v[r];
    }
    sh[threadIdx.x] = tot;
    __syncthreads();
    for (int o = 1; o < kThreads; o <<= 1) {
        T t = threadIdx.x >= o ? sh[threadIdx.x - o] : 0;
        __syncthreads();
        sh[threadIdx.x] += t;
        __syncthreads();
    }
    T run = before + sh[threadIdx.x] - tot;
    for (int r = 0; r < kItems; ++r) {
        int64_t i = base + threadIdx.x * kItems + r;
        if (i < n) out[i] = run;
        run += v[r];
    }
    if (write_total && blockIdx.x == gridDim.x - 1 && threadIdx.x == kThreads - 1) out[n] = run;
}

template <typename T>
__global__ __launch_bounds__(1024) void k_scan_sums(T *sums, int nb)
{
    k_scan_sums_body(sums, nb);
}

template <typename T>
__global__ __launch_bounds__(kThreads) void k_scan_apply(const T *in, int64_t n, const T *sums,
                                                         T *out)
{
    k_scan_apply_body(in, n, sums[blockIdx.x], out, false);
}

// sum of v over the block's threads (kThreads of them), on every thread
template <typename T> __device__ inline T block_sum(T v)
{
    __shared__ T sh[kWaves];
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    T t = 0;
    for (int w = 0; w < kWaves; ++w) t += sh[w];
    __syncthreads();
    return t;
}

// the tiles' sums not scanned: each block adds up those before it
constexpr unsigned kSumTiles = kThreads * kItems;
template <typename T> __device__ inline T sum_before(const T *sums)
{
    T t = 0;
    for (unsigned i = threadIdx.x; i < blockIdx.x; i += kThreads) t += sums[i];
    return block_sum(t);
}

template <typename T>
__global__ __launch_bounds__(kThreads) void k_scan_apply_sums(const T *in, int64_t n, const T *sums, T *out)
{
    k_scan_apply_body(in, n, sum_before(sums), out, false);
}

// Several scans of equal length in one set of launches (blockIdx.y = scan).
struct ScanBatch {
    const int64_t *in[kMaxScanBatch];
    int64_t *out[kMaxScanBatch];
};

__global__ __launch_bounds__(kThreads) void k_scan_block_sums_m(ScanBatch sb, int64_t n, int64_t *sums,
                                                                 int64_t stride)
{
    __shared__ int64_t sh[kWaves];
    const int64_t *in = sb.in[blockIdx.y];
    int64_t base = (int64_t)blockIdx.x * kTile;
    int64_t s = 0;
    for (int r = 0; r < kItems; ++r) {
        int64_t i = base + r * kThreads + threadIdx.x;
        if (i < n) s += in[i];
    }
    for (int o = 32; o > 0; o >>= 1) s += __shfl_down(s, o);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        int64_t t = 0;
        for (int w = 0; w < kWaves; ++w) t += sh[w];
        sums[blockIdx.y * stride + blockIdx.x] = t;
    }
}

__global__ __launch_bounds__(1024) void k_scan_sums_m(int64_t *sums, int nb, int64_t stride)
{
    k_scan_sums_body(sums + blockIdx.x * stride, nb);
}

__global__ __launch_bounds__(kThreads) void k_scan_apply_m(ScanBatch sb, int64_t n, const int64_t *sums,
                                                           int64_t stride)
{
    const int64_t *sm = sums + blockIdx.y * stride;
    k_scan_apply_body(sb.in[blockIdx.y], n, sm[blockIdx.x], sb.out[blockIdx.y], true);
}

__global__ __launch_bounds__(kThreads) void k_scan_apply_sums_m(ScanBatch sb, int64_t n, const int64_t *sums,
                                                                int64_t stride)
{
    const int64_t before = sum_before(sums + blockIdx.y * stride);
    k_scan_apply_body(sb.in[blockIdx.y], n, before, sb.out[blockIdx.y], true);
}

// in one launch: each block adds up the elements before its tile
constexpr int kDirectTiles = 8;
__global__ __launch_bounds__(kThreads) void k_scan_direct_m(ScanBatch sb, int64_t n)
{
    const int64_t *in = sb.in[blockIdx.y];
    int64_t t = 0;
#pragma unroll 8
    for (int i = threadIdx.x; i < (int)blockIdx.x * kTile; i += kThreads) t += in[i];
    k_scan_apply_body(in, n, block_sum(t), sb.out[blockIdx.y], true);
}

size_t scan_multi_scratch_bytes(int64_t n, int count)
{
    return sizeof(int64_t) * (ceil_div(n > 0 ? n : 1, kTile) + 2) * (size_t)count;
}

void scan_exclusive_multi(const int64_t *const *in, int64_t *const *out, int count, int64_t n,
                          int64_t *scratch, hipStream_t s)
{
    ScanBatch sb{};
    for (int i = 0; i < count; ++i) { sb.in[i] = in[i]; sb.out[i] = out[i]; }
    unsigned nb = ceil_div(n > 0 ? n : 1, kTile);
    int64_t stride = nb + 2;
    if (nb <= kDirectTiles) {
        k_scan_direct_m<<<dim3(nb, count), kThreads, 0, s>>>(sb, n);
        return;
    }
    k_scan_block_sums_m<<<dim3(nb, count), kThreads, 0, s>>>(sb, n, scratch, stride);
    if (nb <= kSumTiles) {
        k_scan_apply_sums_m<<<dim3(nb, count), kThreads, 0, s>>>(sb, n, scratch, stride);
        return;
    }
    k_scan_sums_m<<<count, 1024, 0, s>>>(scratch, (int)nb, stride);
    k_scan_apply_m<<<dim3(nb, count), kThreads, 0, s>>>(sb, n, scratch, stride);
}

size_t scan_scratch_bytes(int64_t n) { return scan_multi_scratch_bytes(n, 1); }

void scan_exclusive(const int64_t *in, int64_t *out, int64_t n, int64_t *scratch, hipStream_t s)
{
    scan_exclusive_multi(&in, &out, 1, n, scratch, s);
}

// in place; scratch: a sum per tile and the total
static void scan_exclusive_i32(int32_t *data, int64_t n, int32_t *scratch, hipStream_t s)
{
    unsigned nb = ceil_div(n > 0 ? n : 1, kTile);
    k_scan_block_sums<int32_t><<<nb, kThreads, 0, s>>>(data, n, scratch);
    if (nb <= kSumTiles) {
        k_scan_apply_sums<int32_t><<<nb, kThreads, 0, s>>>(data, n, scratch, data);
        return;
    }
    k_scan_sums<int32_t><<<1, 1024, 0, s>>>(scratch, (int)nb);
    k_scan_apply<int32_t><<<nb, kThreads, 0, s>>>(data, n, scratch, data);
}

// ---------------- radix sort ----------------
// A block owns a tile of ITEMS * 256 consecutive elements: smaller tiles for
// fewer elements, so that the passes of a middling sort fill some of the chip.
// hist: per (block, digit) with BLOCK_MAJOR, else per (digit, block).
template <int ITEMS, bool BLOCK_MAJOR>
__global__ __launch_bounds__(kThreads) void k_digit_hist(const uint64_t *keys, int n, int shift, int mask,
                                                         int nblocks, int32_t *hist)
{
    __shared__ int32_t h[256];
    h[threadIdx.x] = 0;
    __syncthreads();
    int base = blockIdx.x * (ITEMS * kThreads);
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        int i = base + r * kThreads + threadIdx.x;
        if (i < n) atomicAdd(&h[(int)(keys[i] >> shift) & mask], 1);
    }
    __syncthreads();
    hist[BLOCK_MAJOR ? blockIdx.x * 256 + threadIdx.x : threadIdx.x * nblocks + blockIdx.x] = h[threadIdx.x];
}

// lanes of the wavefront with the same 8-bit digit (valid lanes only)
__device__ inline uint64_t digit_peers(int d, bool valid)
{
    uint64_t peers = __ballot(valid);
#pragma unroll
    for (int b = 0; b < 8; ++b) {
        const uint64_t m = __ballot((d >> b) & 1);
        peers &= ((d >> b) & 1) ? m : ~m;
    }
    return peers;
}

// DIRECT: offs holds the blocks' histograms (block-major); the block adds up
// those before it and the totals of the lower digits.  Else: their scan.
template <int ITEMS, bool DIRECT>
__global__ __launch_bounds__(kThreads) void k_digit_scatter(const uint64_t *keys, const int32_t *vals,
                                                            int n, int shift, int mask, int nblocks,
                                                            const int32_t *offs, uint64_t *okeys,
                                                            int32_t *ovals)
{
    __shared__ int32_t run[256];        // running count per digit over earlier rounds
    __shared__ int32_t wcnt[kWaves][256];
    __shared__ int32_t wbase[kWaves][256];
    __shared__ int32_t wsum[kWaves];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if constexpr (DIRECT) {
        int pre = 0, tot = 0;
#pragma unroll 8
        for (int b = 0; b < nblocks; ++b) {
            const int c = offs[b * 256 + tid];
            tot += c;
            pre += b < (int)blockIdx.x ? c : 0;
        }
        int incl = tot;
        for (int o = 1; o < 64; o <<= 1) {
            const int t = __shfl_up(incl, o);
            if (lane >= o) incl += t;
        }
        if (lane == 63) wsum[wave] = incl;
        __syncthreads();
        for (int w = 0; w < wave; ++w) incl += wsum[w];
        run[tid] = incl - tot + pre;
    } else {
        run[tid] = offs[tid * nblocks + blockIdx.x];
    }
    int base = blockIdx.x * (ITEMS * kThreads);
    for (int r = 0; r < ITEMS; ++r) {
        for (int w = 0; w < kWaves; ++w) wcnt[w][tid] = 0;
        __syncthreads();
        int i = base + r * kThreads + tid;
        bool valid = i < n;
        uint64_t key = valid ? keys[i] : 0;
        int32_t val = valid ? vals[i] : 0;
        int d = valid ? (int)(key >> shift) & mask : 0;
        const uint64_t peers = digit_peers(d, valid), below = peers & lanes_below(lane);
        const int rank = __popcll(below);
        if (valid && below == 0) wcnt[wave][d] = __popcll(peers);
        __syncthreads();
        { // per digit: offsets of each wave, then advance the running count
            int s = run[tid];
            for (int w = 0; w < kWaves; ++w) {
                wbase[w][tid] = s;
                s += wcnt[w][tid];
            }
            run[tid] = s;
        }
        __syncthreads();
        if (valid) {
            int pos = wbase[wave][d] + rank;
            okeys[pos] = key;
            ovals[pos] = val;
        }
        __syncthreads();
    }
}

// One block of 16 wavefronts, the pairs in LDS, every pass in it; wavefront w
// owns elements [64 ITEMS w, 64 ITEMS (w + 1)) of the current order.
constexpr int kSmallSort = 8192;
template <int ITEMS>
__global__ __launch_bounds__(1024) void k_sort_small(uint64_t *keys, int32_t *vals, int n, int lo, int hi)
{
    constexpr int W = 16;
    __shared__ uint64_t sk[1024 * ITEMS];
    __shared__ int32_t sv[1024 * ITEMS];
    __shared__ int32_t cnt[W][256]; // digits of each wavefront, then where its first of each digit goes
    __shared__ int32_t wsum[W];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, base = wave * 64 * ITEMS + lane;
    uint64_t key[ITEMS];
    int32_t val[ITEMS], rank[ITEMS];
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        const int e = base + 64 * r;
        key[r] = e < n ? keys[e] : 0;
        val[r] = e < n ? vals[e] : 0;
    }
    for (int shift = lo; shift < hi; shift += 8) {
        const int mask = hi - shift < 8 ? (1 << (hi - shift)) - 1 : 255;
        for (int i = tid; i < W * 256; i += 1024) (&cnt[0][0])[i] = 0;
        __syncthreads();
#pragma unroll
        for (int r = 0; r < ITEMS; ++r) {
            const bool valid = base + 64 * r < n;
            const int d = (int)(key[r] >> shift) & mask;
            const uint64_t peers = digit_peers(d, valid), below = peers & lanes_below(lane);
            const int before = cnt[wave][d];
            rank[r] = before + __popcll(below);
            wave_sync();
            if (valid && below == 0) cnt[wave][d] = before + __popcll(peers);
            wave_sync();
        }
        __syncthreads();
        { // exclusive scan over (digit, wavefront), four entries per thread
            const int d = tid >> 2, w0 = (tid & 3) * 4;
            int c[4], t = 0;
            for (int i = 0; i < 4; ++i) { c[i] = cnt[w0 + i][d]; t += c[i]; }
            int incl = t;
            for (int o = 1; o < 64; o <<= 1) {
                const int u = __shfl_up(incl, o);
                if (lane >= o) incl += u;
            }
            if (lane == 63) wsum[wave] = incl;
            __syncthreads();
            int run = incl - t;
            for (int w = 0; w < wave; ++w) run += wsum[w];
            for (int i = 0; i < 4; ++i) { cnt[w0 + i][d] = run; run += c[i]; }
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < ITEMS; ++r)
            if (base + 64 * r < n) {
                const int pos = cnt[wave][(int)(key[r] >> shift) & mask] + rank[r];
                sk[pos] = key[r];
                sv[pos] = val[r];
            }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < ITEMS; ++r) {
            const int e = base + 64 * r;
            key[r] = e < n ? sk[e] : 0;
            val[r] = e < n ? sv[e] : 0;
        }
    }
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        const int e = base + 64 * r;
        if (e < n) { keys[e] = key[r]; vals[e] = val[r]; }
    }
}

constexpr int kDirectBlocks = 128;
// elements per tile / 256: 512-element tiles up to 32k elements, then 1024 up to
// kDirectBlocks of them
static int sort_items(int n) { return n <= 32768 ? 2 : n <= kDirectBlocks * 1024 ? 4 : kItems; }

size_t sort_scratch_bytes(int n)
{
    // grows with n: a scratch serves every shorter sort too
    const size_t m = n > 0 ? n : 1, small = ceil_div(m, 2 * kThreads), large = ceil_div(m, kTile);
    const size_t h = 256 * std::max(large, std::min<size_t>(small, kDirectBlocks));
    return sizeof(int32_t) * (h + ceil_div((long long)h, kTile) + 2);
}

bool sort_lands_in_tmp(int n, int lo, int hi) { return n > kSmallSort && ((hi - lo + 7) / 8) % 2 == 1; }

template <int ITEMS, bool DIRECT>
static void sort_pass(const uint64_t *ik, const int32_t *iv, uint64_t *ok, int32_t *ov, int n, int shift, int mask,
                      int32_t *hist, hipStream_t s)
{
    const int nb = (int)ceil_div(n, ITEMS * kThreads);
    k_digit_hist<ITEMS, DIRECT><<<nb, kThreads, 0, s>>>(ik, n, shift, mask, nb, hist);
    if (!DIRECT) scan_exclusive_i32(hist, 256LL * nb, hist + 256 * (size_t)nb, s);
    k_digit_scatter<ITEMS, DIRECT><<<nb, kThreads, 0, s>>>(ik, iv, n, shift, mask, nb, hist, ok, ov);
}

// Stable sort by bits [lo, hi) of the keys.  The result is in (tk, tv) if
// sort_lands_in_tmp(n, lo, hi), else in (keys, vals).
void radix_sort_pairs(uint64_t *keys, int32_t *vals, uint64_t *tk, int32_t *tv, int n, int lo, int hi,
                      int32_t *hist, hipStream_t s)
{
    if (n <= kSmallSort) {
        if (n <= 1 || hi <= lo) return;
        if (n <= 1024) k_sort_small<1><<<1, 1024, 0, s>>>(keys, vals, n, lo, hi);
        else if (n <= 2048) k_sort_small<2><<<1, 1024, 0, s>>>(keys, vals, n, lo, hi);
        else if (n <= 4096) k_sort_small<4><<<1, 1024, 0, s>>>(keys, vals, n, lo, hi);
        else k_sort_small<8><<<1, 1024, 0, s>>>(keys, vals, n, lo, hi);
        return;
    }
    const int items = sort_items(n);
    for (int shift = lo; shift < hi; shift += 8) {
        const int mask = hi - shift < 8 ? (1 << (hi - shift)) - 1 : 255;
        if (items == 2) sort_pass<2, true>(keys, vals, tk, tv, n, shift, mask, hist, s);
        else if (items == 4) sort_pass<4, true>(keys, vals, tk, tv, n, shift, mask, hist, s);
        else sort_pass<kItems, false>(keys, vals, tk, tv, n, shift, mask, hist, s);
        uint64_t *t = keys; keys = tk; tk = t;
        int32_t *u = vals; vals = tv; tv = u;
    }
}

} // namespace fmm
