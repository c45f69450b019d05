// Compressed columns of R from its compressed rows: the CSC that "Update Theta" (eq. (3)) walks.
// A stable sort of the stored entries by column id keeps the rows of every column ascending, so the result is the
// canonical CSC and is reproducible bit for bit.  The sort is a least-significant-digit radix sort, one to four passes
// of up to 10 bits, of the entries themselves: (column id, row, rating) travel together, so nothing has to be looked
// up at the end.  Per pass a digit histogram of every tile, one prefix sum over (digit, tile), and a scatter in which a
// workgroup first sorts its tile of 8192 entries in LDS and then writes it digit by digit, in runs of consecutive
// addresses (32 entries a run at 8 bits).  No atomics whose order could matter.  Off the per-sweep path: once per matrix.
#include <cstring>

#include "als_internal.h"

namespace als {

template <typename PtrT>
__device__ __forceinline__ int64_t row_of_entry(const PtrT *__restrict__ ptr, int64_t nrows, int64_t q) {
    // largest row with ptr[row] <= q
    int64_t lo = 0, hi = nrows;  // ptr[lo] <= q < ptr[hi]
    while (hi - lo > 1) {
        const int64_t mid = (lo + hi) >> 1;
        if ((int64_t)ptr[mid] <= q) lo = mid; else hi = mid;
    }
    return lo;
}

constexpr int kMaxDigitBits = 10;   // the counters of a tile (16 bits per wavefront and digit) stay below 20 KB of LDS
constexpr int kSortThreads = 512, kSortItems = 16, kSortWaves = kSortThreads / 64;
constexpr int64_t kTile = kSortThreads * kSortItems;   // entries per tile: positions in a tile fit 16 bits
constexpr int kTileRows = 1024;                        // row offsets of a tile kept in LDS (first pass)

// counts[d * ntiles + t] = number of keys of tile t whose digit (bits shift .. shift+bits-1) is d
__global__ __launch_bounds__(256) void k_digit_hist(const uint32_t *__restrict__ keys, int64_t n, int64_t tile, int shift,
                                                    int bits, int64_t ntiles, uint32_t *__restrict__ counts) {
    __shared__ uint32_t cnt[1 << kMaxDigitBits];
    const int nd = 1 << bits;
    for (int d = threadIdx.x; d < nd; d += 256) cnt[d] = 0u;
    __syncthreads();
    const int64_t t = blockIdx.x, lo = t * tile, hi = lo + tile < n ? lo + tile : n;
    for (int64_t q = lo + threadIdx.x; q < hi; q += 256) atomicAdd(&cnt[(keys[q] >> shift) & (uint32_t)(nd - 1)], 1u);
    __syncthreads();
    for (int d = threadIdx.x; d < nd; d += 256) counts[(int64_t)d * ntiles + t] = cnt[d];
}

// One tile per workgroup.  offsets[d * ntiles + t]: where the entries of tile t with digit d start in the output (the
// prefix sums of the counts).  Each wavefront ranks 1024 consecutive entries, 64 at a time, in order:
// lanes with the same digit find each other with one ballot per digit bit, the lower lanes of such a group come first, and
// a counter per wavefront and digit carries on from group to group.  The counters are then summed digit by digit over the
// wavefronts in order, which gives every entry its place in the sorted tile: the pass is stable.  Entries go to their
// places through LDS, one of the three arrays after the other, and from there to memory, neighbours to neighbours.
// FIRST: the row of an entry follows from its position (ptr), the rating from val; otherwise both come from the pass before.
// Bound: the memory traffic, 8 + 12 bytes an entry in the first pass and 24 in the others.  99M entries,
// 17,770 columns (two passes of 8 bits): 1.14 + 0.91 ms = 1.7 + 2.6 TB/s; the whole call 9.9 -> 2.4 ms (before, one wavefront per tile wrote
// its entries where they fell, 3.7 + 2.2 ms, and rows and ratings were looked up afterwards, 2.9 ms).
template <typename PtrT, bool FIRST>
__global__ __launch_bounds__(kSortThreads) void k_sort_tile(const uint32_t *__restrict__ keys, const int32_t *__restrict__ rows,
                                                            const float *__restrict__ vals, const PtrT *__restrict__ ptr,
                                                            int64_t nrows, int64_t n, int shift, int bits, int64_t ntiles,
                                                            const uint32_t *__restrict__ offsets, uint32_t *__restrict__ keys_out,
                                                            int32_t *__restrict__ rows_out, float *__restrict__ vals_out) {
    __shared__ uint32_t stage[kTile];                    // one array of the tile, sorted
    __shared__ uint32_t wsum[kSortWaves];
    __shared__ int64_t row_span[2];
    extern __shared__ __attribute__((aligned(16))) uint32_t dyn[];                    // [nd] output position of place 0 of a digit, then the counters
    const int nd = 1 << bits;
    uint32_t *const goff = dyn;
    uint16_t *const cnt = reinterpret_cast<uint16_t *>(dyn + nd);   // [wavefront][digit]
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t t = blockIdx.x, lo = t * kTile;
    const int len = (int)(lo + kTile < n ? kTile : n - lo);
    for (int k = tid; k < nd * kSortWaves / 2; k += kSortThreads) reinterpret_cast<uint32_t *>(cnt)[k] = 0u;
    if (FIRST && tid < 2) row_span[tid] = row_of_entry(ptr, nrows, tid == 0 ? lo : lo + len - 1);
    const int e0 = wave * (64 * kSortItems) + lane;      // this lane's entries: e0 + 64 j
    uint32_t key[kSortItems];
#pragma unroll
    for (int j = 0; j < kSortItems; ++j) key[j] = e0 + 64 * j < len ? keys[lo + e0 + 64 * j] : 0u;
    __syncthreads();
    const unsigned long long below = (1ull << lane) - 1ull;
    uint16_t *const mine = cnt + wave * nd;
    int place[kSortItems];                               // rank inside the wavefront's entries of the digit, then place in the tile
#pragma unroll
    for (int j = 0; j < kSortItems; ++j) {
        const bool ok = e0 + 64 * j < len;
        const uint32_t d = (key[j] >> shift) & (uint32_t)(nd - 1);
        unsigned long long same = __ballot(ok);
        for (int k = 0; k < bits; ++k) {
            const bool bit = ((d >> k) & 1u) != 0u;
            const unsigned long long m = __ballot(bit);
            same &= bit ? m : ~m;
        }
        // (a wavefront's LDS reads and writes are performed in program order: every lane of a group has read the
        // counter before the first lane of the group moves it on)
        const int before = ok ? mine[d] : 0, rank = __popcll(same & below);
        if (ok && rank == 0) mine[d] = (uint16_t)(before + __popcll(same));
        place[j] = before + rank;
        __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
    // exclusive prefix sums over (digit, wavefront): thread t owns the digits [t per, (t + 1) per)
    const int per = nd > kSortThreads ? nd / kSortThreads : 1;
    uint32_t sum = 0u;
    for (int k = 0; k < per; ++k) {
        const int d = tid * per + k;
        if (d < nd)
            for (int w = 0; w < kSortWaves; ++w) sum += cnt[w * nd + d];
    }
    uint32_t run = sum;                                  // inclusive over the wavefront, then over the workgroup
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t v = (uint32_t)__shfl_up((int)run, o);
        if (lane >= o) run += v;
    }
    if (lane == 63) wsum[wave] = run;
    __syncthreads();
    uint32_t base = run - sum;
    for (int w = 0; w < wave; ++w) base += wsum[w];
    for (int k = 0; k < per; ++k) {
        const int d = tid * per + k;
        if (d < nd) {
            goff[d] = offsets[(int64_t)d * ntiles + t] - base;   // (modulo 2^32: a place of the digit is added to it)
            for (int w = 0; w < kSortWaves; ++w) {
                const uint32_t c = cnt[w * nd + d];
                cnt[w * nd + d] = (uint16_t)base;
                base += c;
            }
        }
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kSortItems; ++j)
        if (e0 + 64 * j < len) {
            place[j] += mine[(key[j] >> shift) & (uint32_t)(nd - 1)];
            stage[place[j]] = key[j];
        }
    __syncthreads();
    uint32_t to[kSortItems];                             // output positions of the places tid + 512 j
#pragma unroll
    for (int j = 0; j < kSortItems; ++j) {
        const int k = tid + kSortThreads * j;
        if (k < len) {
            const uint32_t v = stage[k];
            to[j] = goff[(v >> shift) & (uint32_t)(nd - 1)] + (uint32_t)k;
            keys_out[to[j]] = v;
        }
    }
    __syncthreads();
    // the rows
    if constexpr (FIRST) {
        const int64_t r0 = row_span[0], nr = row_span[1] - r0 + 1;   // the rows that have entries in the tile lie in these
        PtrT *const pl = reinterpret_cast<PtrT *>(dyn);               // (goff and the counters are done with)
        const bool in_lds = nr <= kTileRows;
        if (in_lds)
            for (int k = tid; k < (int)nr; k += kSortThreads) pl[k] = ptr[r0 + k];
        __syncthreads();
#pragma unroll
        for (int j = 0; j < kSortItems; ++j)
            if (e0 + 64 * j < len) {
                const int64_t q = lo + e0 + 64 * j;
                int64_t a = 0, b = nr;                   // ptr[r0 + a] <= q < ptr[r0 + b]
                while (b - a > 1) {
                    const int64_t mid = (a + b) >> 1;
                    if ((int64_t)(in_lds ? pl[mid] : ptr[r0 + mid]) <= q) a = mid; else b = mid;
                }
                stage[place[j]] = (uint32_t)(r0 + a);
            }
    } else {
#pragma unroll
        for (int j = 0; j < kSortItems; ++j)
            if (e0 + 64 * j < len) stage[place[j]] = (uint32_t)rows[lo + e0 + 64 * j];
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kSortItems; ++j)
        if (tid + kSortThreads * j < len) rows_out[to[j]] = (int32_t)stage[tid + kSortThreads * j];
    __syncthreads();
    // the ratings
#pragma unroll
    for (int j = 0; j < kSortItems; ++j)
        if (e0 + 64 * j < len) stage[place[j]] = __builtin_bit_cast(uint32_t, vals[lo + e0 + 64 * j]);
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kSortItems; ++j)
        if (tid + kSortThreads * j < len) vals_out[to[j]] = __builtin_bit_cast(float, stage[tid + kSortThreads * j]);
}

template <typename PtrT>
__global__ __launch_bounds__(256) void k_column_starts(const uint32_t *__restrict__ sorted_cols, int64_t nnz,
                                                       int64_t ncols, PtrT *__restrict__ cptr) {
    const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v > ncols) return;
    int64_t lo = 0, hi = nnz;  // first position whose column id is >= v
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if ((int64_t)sorted_cols[mid] < v) lo = mid + 1; else hi = mid;
    }
    cptr[v] = (PtrT)lo;
}

template <typename PtrT>
static hipError_t transpose_t(hipStream_t st, int64_t nrows, int64_t ncols, int64_t nnz, const PtrT *ptr,
                              const int32_t *idx, const float *val, PtrT *cptr, int32_t *cidx, float *cval, void **scratch,
                              size_t *scratch_bytes) {
    hipError_t e = hipSuccess;
    // the last pass writes the caller's arrays (and the sorted column ids); the passes before it alternate
    uint32_t *keys[2] = {nullptr, nullptr}, *counts = nullptr;
    int32_t *rows[2] = {cidx, nullptr};
    float *vals[2] = {cval, nullptr};
    int key_bits = 1;   // bits of the largest column id
    while (key_bits < 32 && (1ll << key_bits) < ncols) ++key_bits;
    const int npass = (key_bits + kMaxDigitBits - 1) / kMaxDigitBits, bits = (key_bits + npass - 1) / npass;
    const uint32_t *sorted_cols = nullptr;
    if (nnz > 0) {
        const int64_t ntiles = (nnz + kTile - 1) / kTile, ncount = ntiles << bits;
        // one buffer: the counters and their prefix sums' scratch, the sorted column ids, and with several passes a second
        // set of the three arrays
        const size_t array = (4 * (size_t)nnz + 255) / 256 * 256, cbytes = (4 * (size_t)(ncount + scan_scratch_ints(ncount)) + 255) / 256 * 256;
        if ((e = ensure_scratch(scratch, scratch_bytes, cbytes + (npass > 1 ? 4 : 1) * array, false)) != hipSuccess) return e;
        char *p0 = static_cast<char *>(*scratch);
        counts = reinterpret_cast<uint32_t *>(p0);
        keys[0] = reinterpret_cast<uint32_t *>(p0 + cbytes);
        if (npass > 1) {
            keys[1] = reinterpret_cast<uint32_t *>(p0 + cbytes + array);
            rows[1] = reinterpret_cast<int32_t *>(p0 + cbytes + 2 * array);
            vals[1] = reinterpret_cast<float *>(p0 + cbytes + 3 * array);
        }
        const uint32_t *kin = reinterpret_cast<const uint32_t *>(idx);
        const int32_t *rin = nullptr;
        const float *vin = val;
        const size_t dyn_words = ((size_t)1 << bits) + ((size_t)kSortWaves << bits) / 2, row_words = kTileRows * sizeof(PtrT) / 4;
        const unsigned lds = 4 * (unsigned)(dyn_words > row_words ? dyn_words : row_words);
        for (int p = 0; p < npass; ++p) {
            const int out = (npass - 1 - p) & 1;
            hipLaunchKernelGGL(k_digit_hist, dim3((unsigned)ntiles), dim3(256), 0, st, kin, nnz, kTile, p * bits, bits, ntiles, counts);
            if ((e = hipGetLastError()) != hipSuccess) return e;
            if ((e = exclusive_scan_u32(st, counts, ncount, counts + ncount)) != hipSuccess) return e;
            if (p == 0)
                hipLaunchKernelGGL((k_sort_tile<PtrT, true>), dim3((unsigned)ntiles), dim3(kSortThreads), lds, st, kin, rin, vin, ptr,
                                   nrows, nnz, p * bits, bits, ntiles, counts, keys[out], rows[out], vals[out]);
            else
                hipLaunchKernelGGL((k_sort_tile<PtrT, false>), dim3((unsigned)ntiles), dim3(kSortThreads), lds, st, kin, rin, vin, ptr,
                                   nrows, nnz, p * bits, bits, ntiles, counts, keys[out], rows[out], vals[out]);
            if ((e = hipGetLastError()) != hipSuccess) return e;
            kin = keys[out];
            rin = rows[out];
            vin = vals[out];
        }
        sorted_cols = kin;
    }
    hipLaunchKernelGGL((k_column_starts<PtrT>), dim3((unsigned)((ncols + 1 + 255) / 256)), dim3(256), 0, st,
                       sorted_cols, nnz, ncols, cptr);
    e = hipGetLastError();
    hipError_t e2 = hipStreamSynchronize(st);   // the caller may free the scratch buffer
    return e != hipSuccess ? e : e2;
}

hipError_t transpose_csr(bool ptr64, hipStream_t st, int64_t nrows, int64_t ncols, int64_t nnz, const void *ptr,
                         const int32_t *idx, const float *val, void *cptr, int32_t *cidx, float *cval, void **scratch,
                         size_t *scratch_bytes) {
    if (ptr64)
        return transpose_t<int64_t>(st, nrows, ncols, nnz, (const int64_t *)ptr, idx, val, (int64_t *)cptr, cidx,
                                    cval, scratch, scratch_bytes);
    return transpose_t<int32_t>(st, nrows, ncols, nnz, (const int32_t *)ptr, idx, val, (int32_t *)cptr, cidx, cval, scratch,
                                scratch_bytes);
}

}  // namespace als
