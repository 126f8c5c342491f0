// Device-wide exclusive prefix sums.  A launch costs a call about 5 us, so
// arrays of up to kBlockItems values take one workgroup and one launch,
// longer ones two: the tiles' sums, then every tile's scan, its workgroup
// adding up the sums before it by itself (at most kOwnSums, 16 KB from L2).
// Past that many tiles a third launch scans the sums in one workgroup.
#include "common.h"
#include "internal.h"

namespace spsyrk {
namespace {

constexpr int kItems = 16;
constexpr int kTile = kBlock * kItems;

template <typename T>
__global__ __launch_bounds__(kBlock) void tile_reduce(const T* __restrict__ in, int64_t n, T* __restrict__ sums) {
    __shared__ T wt[kWavesPerBlock];
    const int64_t base = int64_t(blockIdx.x) * kTile;
    T s = 0;
#pragma unroll
    for (int k = 0; k < kItems; ++k) {
        int64_t i = base + int64_t(k) * kBlock + threadIdx.x;
        if (i < n) s += in[i];
    }
    s = wave_reduce_sum(s);
    if (lane_id() == 0) wt[threadIdx.x / kWave] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        T t = 0;
        for (int w = 0; w < kWavesPerBlock; ++w) t += wt[w];
        sums[blockIdx.x] = t;
    }
}

// exclusive scan of nb tile sums in place by one workgroup; total -> *total
template <typename T>
__global__ __launch_bounds__(kBlock) void scan_sums(T* __restrict__ sums, int64_t nb, T* __restrict__ total) {
    __shared__ T wt[kWavesPerBlock];
    T carry = 0;
    for (int64_t base = 0; base < nb; base += kTile) {
        // each thread takes kItems consecutive sums
        T v[kItems];
        T s = 0;
#pragma unroll
        for (int k = 0; k < kItems; ++k) {
            int64_t i = base + int64_t(threadIdx.x) * kItems + k;
            v[k] = i < nb ? sums[i] : T(0);
            s += v[k];
        }
        T tot;
        T off = block_exclusive_scan(s, wt, &tot);
        off += carry;
#pragma unroll
        for (int k = 0; k < kItems; ++k) {
            int64_t i = base + int64_t(threadIdx.x) * kItems + k;
            if (i < nb) sums[i] = off;
            off += v[k];
        }
        carry += tot;
        __syncthreads();
    }
    if (threadIdx.x == 0 && total) *total = carry;
}

// Exclusive scan of the tile at base (kTile values of in, zero past n) into
// out, starting from carry.  The tile is read whole into LDS before any of it
// is written, so in may equal out.  The LDS rows of kItems values are padded
// by one, so that the threads' runs of kItems do not start in one bank.
template <typename T>
__device__ inline T scan_tile(const T* __restrict__ in, T* __restrict__ out, int64_t n, int64_t base, T carry,
                              T* buf, T* wt) {
    // coalesced loads into LDS, then a blocked arrangement: thread t holds
    // kItems consecutive elements
    auto at = [](int x) { return x + x / kItems; };
#pragma unroll
    for (int k = 0; k < kItems; ++k) {
        const int64_t i = base + int64_t(k) * kBlock + threadIdx.x;
        buf[at(k * kBlock + int(threadIdx.x))] = i < n ? in[i] : T(0);
    }
    __syncthreads();
    T v[kItems];
    T s = 0;
#pragma unroll
    for (int k = 0; k < kItems; ++k) {
        v[k] = buf[at(threadIdx.x * kItems + k)];
        s += v[k];
    }
    T tot;
    T off = block_exclusive_scan(s, wt, &tot) + carry;
#pragma unroll
    for (int k = 0; k < kItems; ++k) {
        buf[at(threadIdx.x * kItems + k)] = off;
        off += v[k];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kItems; ++k) {
        const int64_t i = base + int64_t(k) * kBlock + threadIdx.x;
        if (i < n) out[i] = buf[at(k * kBlock + int(threadIdx.x))];
    }
    return tot;
}

// SUMS: sums holds the tiles' sums (not scanned); the last tile writes
// *total.  Otherwise sums is their exclusive scan.
template <typename T, bool SUMS>
__global__ __launch_bounds__(kBlock) void tile_scan(const T* __restrict__ in, T* __restrict__ out, int64_t n,
                                                    const T* __restrict__ sums, T* __restrict__ total) {
    __shared__ T wt[kWavesPerBlock];
    __shared__ T wb[kWavesPerBlock];
    __shared__ T buf[kTile + kTile / kItems];
    T before = 0;
    if constexpr (SUMS) {
        for (int64_t q = threadIdx.x; q < int64_t(blockIdx.x); q += kBlock) before += sums[q];
        before = wave_reduce_sum(before);
        if (lane_id() == 0) wb[threadIdx.x / kWave] = before;
        __syncthreads();
        before = 0;
        for (int w = 0; w < kWavesPerBlock; ++w) before += wb[w];
    } else {
        before = sums[blockIdx.x];
    }
    const T tot = scan_tile(in, out, n, int64_t(blockIdx.x) * kTile, before, buf, wt);
    if (SUMS && total && blockIdx.x + 1 == gridDim.x && threadIdx.x == 0) *total = before + tot;
}

// short arrays: one workgroup of 1024 threads, kShort values each in
// registers, all loaded at once (one launch; total -> *total)
constexpr int kOneBlock = 1024;
constexpr int kShort = 8;
constexpr int64_t kBlockItems = 2 * kOneBlock * kShort;
template <typename T>
__global__ __launch_bounds__(kOneBlock) void scan_one_block(const T* __restrict__ in, T* __restrict__ out, int64_t n,
                                                            T* __restrict__ total) {
    __shared__ T wt[kOneBlock / kWave];
    T carry = 0;
    for (int64_t base = 0; base < n; base += kOneBlock * kShort) {
        const int64_t i0 = base + int64_t(threadIdx.x) * kShort;
        T v[kShort];
        T s = 0;
#pragma unroll
        for (int k = 0; k < kShort; ++k) v[k] = i0 + k < n ? in[i0 + k] : T(0);
#pragma unroll
        for (int k = 0; k < kShort; ++k) s += v[k];
        T tot;
        // (its barriers also order these loads before the stores: in may be out)
        T off = block_exclusive_scan<T, kOneBlock>(s, wt, &tot) + carry;
#pragma unroll
        for (int k = 0; k < kShort; ++k) {
            if (i0 + k < n) out[i0 + k] = off;
            off += v[k];
        }
        carry += tot;
    }
    if (total && threadIdx.x == 0) *total = carry;
}

constexpr int64_t kOwnSums = 2048;

template <typename T>
void scan_impl(const T* in, T* out, int64_t n, T* total, void* tmp, hipStream_t s) {
    const int64_t nb = (n + kTile - 1) / kTile;
    T* sums = static_cast<T*>(tmp);
    if (nb == 0) {
        if (total) (void)hipMemsetAsync(total, 0, sizeof(T), s);
        return;
    }
    if (n <= kBlockItems) {
        scan_one_block<T><<<1, kOneBlock, 0, s>>>(in, out, n, total);
        return;
    }
    tile_reduce<T><<<dim3(unsigned(nb)), dim3(kBlock), 0, s>>>(in, n, sums);
    if (nb <= kOwnSums) {
        tile_scan<T, true><<<dim3(unsigned(nb)), dim3(kBlock), 0, s>>>(in, out, n, sums, total);
        return;
    }
    scan_sums<T><<<1, kBlock, 0, s>>>(sums, nb, total);
    tile_scan<T, false><<<dim3(unsigned(nb)), dim3(kBlock), 0, s>>>(in, out, n, sums, nullptr);
}

}  // namespace

size_t scan_tmp_bytes(int64_t n) { return size_t((n + kTile - 1) / kTile + 1) * sizeof(int64_t); }

void scan_u32(const uint32_t* in, uint32_t* out, int64_t n, uint32_t* total, void* tmp, hipStream_t s) {
    scan_impl<uint32_t>(in, out, n, total, tmp, s);
}

void scan_i64(const int64_t* in, int64_t* out, int64_t n, int64_t* total, void* tmp, hipStream_t s) {
    scan_impl<int64_t>(in, out, n, total, tmp, s);
}

}  // namespace spsyrk
