// GPU-side TCA-TBE packer (Algorithm 1 and Section 4.2 of the ZipServ paper): the same blob,
// byte for byte, as the host packer zs_encode, from a matrix that already lies in device memory.
//
//   1. sample_kernel  predicts the exponent window from 16 K of the weights
//   2. hist_kernel    exponent histogram of all weights, and the in-window elements of every
//                     BlockTile under the predicted window (parked where the bit-planes will be)
//   3. recount_kernel repeats the counts when the window of the full histogram is another one
//                     (near ties only); otherwise it ends at once
//   4. scan_kernel    segment offsets = prefix sums of the padded segment sizes, totals
//   5. pack_kernel    one wave per BlockTile: bit-planes, H bytes, L halfwords, assembled in LDS;
//                     one more workgroup zeroes the gaps between the sections
// The matrix is read twice.  Window, offsets and the start of the L section stay on the device;
// the host waits once, at the end, for the totals that fill the descriptor.
// Every store is checked against the caller's capacity, whatever the counts say.
#include <hip/hip_runtime.h>

#include <atomic>
#include <cstring>
#include <mutex>

#include "zipserv.h"
#include "zs_device.h"
#include "zs_format.h"

using namespace zs;

namespace {

typedef uint16_t __attribute__((ext_vector_type(2))) u16x2;

constexpr int kHistWords = 256;                         // uint64 bins at the start of the workspace
constexpr size_t kTotalsAt = kHistWords * 8;            // then: struct Totals
struct Totals {
    uint64_t h_units, l_units, n_high;
    uint32_t max_h, max_l;
    uint32_t win_lo;       // first exponent of the window (Algorithm 1, phase I)
    uint32_t predicted_lo; // the window the parked counts were taken with
};
static_assert(kTotalsAt + sizeof(Totals) <= ZS_ENCODE_WORKSPACE_BYTES, "workspace layout");

__host__ __device__ inline uint64_t align_up(uint64_t x, uint64_t a) { return (x + a - 1) / a * a; }

// The eight weights of FragTile row `lane` of TensorCoreTile tt of a BlockTile (the lane order of
// Section 4.2: lane l <-> FragTile l / 8, row l % 8), as 16 bytes.
__device__ __forceinline__ u32x4 load_row(const uint16_t *tile, int64_t ldw, int tt, uint32_t lane)
{
    const uint32_t ft = lane >> 3, r = lane & 7u;
    const uint32_t row = 16 * (tt & 3) + 8 * (ft & 1u) + r, col = 32 * (tt >> 2) + 8 * (ft >> 1);
    return *reinterpret_cast<const u32x4 *>(tile + (int64_t)row * ldw + col);
}
__device__ __forceinline__ const uint16_t *tile_at(const uint16_t *W, int64_t ldw, uint32_t k_blocks, uint32_t bt)
{
    return W + (int64_t)(bt / k_blocks) * 64 * ldw + (int64_t)(bt % k_blocks) * 64;
}

// Codewords of two weights, one per halfword: exponent - (lo - 1) = 1..7 inside the window, 8
// outside it (low three bits zero, as the format wants them, and bit 3 marks the fallback).
__device__ __forceinline__ uint32_t codes_of(uint32_t pair, uint32_t lo2)
{
    const u16x2 e = __builtin_bit_cast(u16x2, (pair >> 7) & 0x00FF00FFu);
    const u16x2 d = e - __builtin_bit_cast(u16x2, lo2);
    const u16x2 c = __builtin_elementwise_min(d, u16x2{7, 7}) + u16x2{1, 1};
    return __builtin_bit_cast(uint32_t, c);
}

// Bits 0, 4, ..., 28 of x (one per weight: even ones in the low half, odd ones in the high half) as
// a byte in element order.
__device__ __forceinline__ uint32_t gather_bits(uint32_t x)
{
    x &= 0x11111111u;
    x |= x >> 15;                   // e1 -> 1, e3 -> 5, e5 -> 9, e7 -> 13
    x = (x | (x >> 2)) & 0x0F0Fu;   // e0..e3 -> 0..3, e4..e7 -> 8..11
    return (x | (x >> 4)) & 0xFFu;
}

// The window of maximal coverage, smallest start on ties; every thread of a workgroup of at least
// 256 takes part and gets the result.  sums: 256 words of LDS for the reduction.
struct Window {
    uint32_t lo;
    uint64_t covered;
};
__device__ inline Window pick_window(const unsigned long long *bins, unsigned long long *sums)
{
    const uint32_t t = threadIdx.x;
    if (t < 256) {
        unsigned long long s = 0;
        if (t + ZS_WINDOW <= 256)
            for (int j = 0; j < ZS_WINDOW; ++j) s += bins[t + j];
        // one key: coverage first (below 2^56: N K < 2^35), then the smaller start
        sums[t] = t + ZS_WINDOW <= 256 ? (s << 8) | (255u - t) : 0ull;
    }
    __syncthreads();
    // the largest key: every wave takes it of all 256 by itself (four each, then between lanes), behind one barrier
    // instead of nine
    const uint32_t lane = t & 63u;
    unsigned long long best = 0;
#pragma unroll
    for (uint32_t i = 0; i < 4; ++i) best = sums[lane + 64 * i] > best ? sums[lane + 64 * i] : best;
#pragma unroll
    for (uint32_t d = 32; d > 0; d >>= 1) {
        const unsigned long long other = __shfl_xor(best, (int)d);
        best = other > best ? other : best;
    }
    return Window{255u - (uint32_t)(best & 255u), best >> 8};
}

// Exponent histogram in LDS, 32 copies of each bin side by side: a lane adds to copy lane % 32, so
// that the few exponents that hold most of the weights are spread over the banks (with one copy
// the 64 lanes of a wave pile up on a handful of addresses).  A bin's copies take 128 bytes, so
// that bits 14..7 of a weight are the byte offset of its bin as they stand.
constexpr uint32_t kCopies = 32;
__device__ __forceinline__ void count_pair(uint8_t *bins, uint32_t pair, uint32_t copy4)
{
    __hip_atomic_fetch_add(reinterpret_cast<uint32_t *>(bins + ((pair & 0x7F80u) | copy4)), 1u, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_WORKGROUP);
    __hip_atomic_fetch_add(reinterpret_cast<uint32_t *>(bins + (((pair >> 16) & 0x7F80u) | copy4)), 1u, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ uint32_t bin_total(const uint8_t *bins, uint32_t bin)
{
    uint32_t s = 0;
    for (uint32_t j = 0; j < kCopies; ++j) s += reinterpret_cast<const uint32_t *>(bins)[bin * kCopies + ((bin + j) & (kCopies - 1))];
    return s;
}

// One workgroup: clears the workspace and predicts the window from kSampleUnits 16-byte units of
// the matrix, spread over it by a multiplicative sequence (no row or column stride is favoured).
// The prediction is only that: the counts taken with it are used if the full histogram agrees.
// Bound by the latency of scattered reads from one compute unit: 8192 units took 21.9 us, 2048 take
// 7.7 us, and 16 K weights still place the window of most laws: the best two windows of N(0, 0.02) weights
// differ by 1.8 % of coverage, some fifteen standard deviations of the sample.  How far they differ depends on where
// the scale lies between powers of two (nothing to 2.6 %); near a tie the prediction may fail, and the call then
// reads the matrix once more (28672 x 4096: some 40 us).
constexpr uint32_t kSampleUnits = 2048;
__global__ __launch_bounds__(1024) void sample_kernel(const uint16_t *W, int64_t N, int64_t K, int64_t ldw, unsigned long long *hist,
                                                      Totals *totals)
{
    __shared__ __attribute__((aligned(16))) uint8_t bins[256 * kCopies * 4];
    __shared__ unsigned long long sums[256], all[256];
    const uint32_t t = threadIdx.x;
    for (uint32_t i = t; i < 256 * kCopies; i += 1024) reinterpret_cast<uint32_t *>(bins)[i] = 0;
    if (t < 256) hist[t] = 0;
    __syncthreads();
    const uint32_t row_units = (uint32_t)(K / 8);
    const uint64_t units = (uint64_t)N * row_units;
    u32x4 v[kSampleUnits / 1024];
#pragma unroll
    for (uint32_t i = 0; i < kSampleUnits / 1024; ++i) {
        const uint32_t h = (i * 1024 + t) * 0x9E3779B1u; // a permutation of 32-bit numbers
        const uint32_t u = (uint32_t)((uint64_t)h * units >> 32); // units < 2^32 (checked by the host)
        v[i] = *reinterpret_cast<const u32x4 *>(W + (int64_t)(u / row_units) * ldw + (int64_t)(u % row_units) * 8);
    }
#pragma unroll
    for (uint32_t i = 0; i < kSampleUnits / 1024; ++i)
        for (int c = 0; c < 4; ++c) count_pair(bins, v[i][c], (t & (kCopies - 1)) * 4);
    __syncthreads();
    if (t < 256) all[t] = bin_total(bins, t);
    __syncthreads();
    const Window w = pick_window(all, sums);
    if (t == 0) totals->predicted_lo = w.lo;
}

// In-window elements of a BlockTile, per wave (all lanes get the sum of the fallbacks).
__device__ __forceinline__ uint32_t fallbacks_of(const u32x4 (&v)[ZS_TT_PER_BT], uint32_t lo2)
{
    uint32_t f = 0; // two counters, one per halfword (a lane has 64 weights)
#pragma unroll
    for (int tt = 0; tt < ZS_TT_PER_BT; ++tt)
#pragma unroll
        for (int c = 0; c < 4; ++c) f += (codes_of(v[tt][c], lo2) >> 3) & 0x00010001u;
    f = (f & 0xFFFFu) + (f >> 16);
    return __builtin_amdgcn_readlane(wave_inclusive_scan(f), 63);
}

// Bound by the read of the matrix (235 MB of the 28672 x 4096 layer in 45.5 us, 5.2 TB/s; with one copy of
// the bins, one BlockTile per workgroup and a separate counting pass it was 482 + 36 us).  A wave takes whole
// BlockTiles, so their counts need no exchange between waves; two workgroups of 16 waves on a
// compute unit keep 256 KB of loads in flight, and the global histogram gets one addition per
// workgroup and bin in use.
constexpr uint32_t kHistWaves = 16;
__global__ __launch_bounds__(64 * kHistWaves) void hist_kernel(const uint16_t *W, int64_t ldw, uint32_t k_blocks, uint32_t n_bt,
                                                               unsigned long long *hist, const Totals *totals, uint32_t *counts)
{
    __shared__ __attribute__((aligned(16))) uint8_t bins[256 * kCopies * 4];
    for (uint32_t i = threadIdx.x; i < 256 * kCopies; i += blockDim.x) reinterpret_cast<uint32_t *>(bins)[i] = 0;
    __syncthreads();
    const uint32_t lane = threadIdx.x & 63u, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t lo2 = totals->predicted_lo * 0x00010001u, copy4 = (lane & (kCopies - 1)) * 4;
    for (uint64_t bt = (uint64_t)blockIdx.x * kHistWaves + wave; bt < n_bt; bt += (uint64_t)gridDim.x * kHistWaves) {
        const uint16_t *tile = tile_at(W, ldw, k_blocks, (uint32_t)bt);
        u32x4 v[ZS_TT_PER_BT];
#pragma unroll
        for (int tt = 0; tt < ZS_TT_PER_BT; ++tt) v[tt] = load_row(tile, ldw, tt, lane);
#pragma unroll
        for (int tt = 0; tt < ZS_TT_PER_BT; ++tt)
#pragma unroll
            for (int c = 0; c < 4; ++c) count_pair(bins, v[tt][c], copy4);
        const uint32_t f = fallbacks_of(v, lo2);
        if (lane == 0) counts[bt] = ZS_BT_ELEMS - f;
    }
    __syncthreads();
    if (threadIdx.x < 256) {
        const uint32_t s = bin_total(bins, threadIdx.x);
        if (s) atomicAdd(&hist[threadIdx.x], (unsigned long long)s);
    }
}

// The counts again, under the window of the full histogram, when it is not the predicted one.
__global__ __launch_bounds__(64 * kHistWaves) void recount_kernel(const uint16_t *W, int64_t ldw, uint32_t k_blocks, uint32_t n_bt,
                                                      const unsigned long long *hist, const Totals *totals, uint32_t *counts)
{
    __shared__ unsigned long long sums[256];
    const Window w = pick_window(hist, sums);
    if (w.lo == totals->predicted_lo) return;
    const uint32_t lane = threadIdx.x & 63u, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    for (uint64_t bt = (uint64_t)blockIdx.x * kHistWaves + wave; bt < n_bt; bt += (uint64_t)gridDim.x * kHistWaves) {
        const uint16_t *tile = tile_at(W, ldw, k_blocks, (uint32_t)bt);
        u32x4 v[ZS_TT_PER_BT];
#pragma unroll
        for (int tt = 0; tt < ZS_TT_PER_BT; ++tt) v[tt] = load_row(tile, ldw, tt, lane);
        const uint32_t f = fallbacks_of(v, w.lo * 0x00010001u);
        if (lane == 0) counts[bt] = ZS_BT_ELEMS - f;
    }
}

// offsets[bt] = {sum of H units before bt, sum of L units before bt}; offsets[n_bt], the window and the
// totals at the end.  A workgroup takes per_wg BlockTiles (a multiple of kScanRound) and adds up the
// counts of all BlockTiles before them itself: reading them again (4 bytes a BlockTile, from L2) costs less
// than passing sums from one workgroup to the next.  Bound by latency: one workgroup that took the BlockTiles in
// turn needed 16 us for the 28672 of a 28672 x 4096 layer; with seven the whole call went from 178 to 171 us.
// (Unit sums stay below 2^32: the host refuses larger matrices.)
constexpr uint32_t kScanRound = 4096, kScanWgs = 64;
__global__ __launch_bounds__(1024) void scan_kernel(const uint32_t *counts, uint32_t *offsets, uint32_t n_bt, uint32_t per_wg,
                                                    const unsigned long long *hist, Totals *totals, Totals *host)
{
    __shared__ unsigned long long sums[256];
    __shared__ uint32_t wave_h[2][16], wave_l[2][16], max_h, max_l;
    const uint32_t t = threadIdx.x, lane = t & 63u, wave = t >> 6;
    const uint32_t first = blockIdx.x * per_wg, end = n_bt - first < per_wg ? n_bt : first + per_wg;
    uint32_t mh = 0, ml = 0;
    auto units = [&](uint32_t nh, uint32_t &hu, uint32_t &lu) {
        hu = (nh + 15u) / 16u, lu = (2u * (ZS_BT_ELEMS - nh) + 15u) / 16u;
        mh = max(mh, hu), ml = max(ml, lu);
    };
    // ---- what lies before this workgroup's BlockTiles (first is a multiple of kScanRound)
    uint32_t before_h = 0, before_l = 0;
#pragma unroll 4
    for (uint32_t bt = 4 * t; bt < first; bt += kScanRound) {
        const u32x4 q = *reinterpret_cast<const u32x4 *>(counts + bt);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            uint32_t hu, lu;
            units(q[i], hu, lu);
            before_h += hu, before_l += lu;
        }
    }
    uint32_t run_h = 0, run_l = 0;
    // Sums of h and l over the threads before this one, on top of run_h and run_l, which move on by the
    // sums over all.  (Two sets of wave sums by turns, so one barrier is enough.)
    auto exclusive = [&](uint32_t par, uint32_t h, uint32_t l, uint32_t &at_h, uint32_t &at_l) {
        const uint32_t inc_h = wave_inclusive_scan(h), inc_l = wave_inclusive_scan(l);
        if (lane == 63) wave_h[par][wave] = inc_h, wave_l[par][wave] = inc_l;
        __syncthreads();
        at_h = run_h + inc_h - h, at_l = run_l + inc_l - l;
        for (uint32_t i = 0; i < 16; ++i) {
            const uint32_t sh = wave_h[par][i], sl = wave_l[par][i];
            at_h += i < wave ? sh : 0u, at_l += i < wave ? sl : 0u;
            run_h += sh, run_l += sl;
        }
    };
    uint32_t at_h, at_l, par = 1;
    exclusive(0, before_h, before_l, at_h, at_l);
    for (uint32_t base = first; base < end; base += kScanRound, par ^= 1) {
        const uint32_t bt0 = base + 4 * t, live = bt0 >= end ? 0u : min(end - bt0, 4u);
        u32x4 q = {0u, 0u, 0u, 0u};
        if (live == 4) q = *reinterpret_cast<const u32x4 *>(counts + bt0);
        else
            for (uint32_t i = 0; i < live; ++i) q[i] = counts[bt0 + i];
        uint32_t hu[4] = {0u, 0u, 0u, 0u}, lu[4] = {0u, 0u, 0u, 0u}, h = 0, l = 0;
#pragma unroll
        for (uint32_t i = 0; i < 4; ++i) {
            if (i < live) units(q[i], hu[i], lu[i]);
            h += hu[i], l += lu[i];
        }
        exclusive(par, h, l, at_h, at_l);
#pragma unroll
        for (uint32_t i = 0; i < 4; ++i) {
            if (i < live) *reinterpret_cast<u32x2 *>(offsets + 2 * ((size_t)bt0 + i)) = u32x2{at_h, at_l};
            at_h += hu[i], at_l += lu[i];
        }
    }
    if (end != n_bt) return;
    if (t == 0) max_h = 0, max_l = 0;
    const Window w = pick_window(hist, sums); // (its barrier is also that of the maxima)
    atomicMax(&max_h, mh);
    atomicMax(&max_l, ml);
    __syncthreads();
    if (t == 0) {
        offsets[2 * (size_t)n_bt] = run_h;
        offsets[2 * (size_t)n_bt + 1] = run_l;
        totals->h_units = run_h, totals->l_units = run_l, totals->n_high = w.covered;
        totals->max_h = max_h, totals->max_l = max_l, totals->win_lo = w.lo;
        if (host) *host = Totals{run_h, run_l, w.covered, max_h, max_l, w.lo, 0u};
    }
}

// Where scan_kernel leaves the totals for the host: pinned memory that the GPU writes itself.  A copy to the
// caller's stack is a launch of its own behind pack_kernel and goes through a staging buffer of the runtime:
// with it (and nine barriers to a window instead of one) 28672 x 4096 took 156.5 us instead of 148.4, 6144 x 4096 76.9
// instead of 68.8, 1024 x 4096 53.6 instead of 44.9.  One page for the process, allocated at the first call, in slots that a call takes
// and gives back before it returns; a call that finds none free (more than kSlots at a time, or no pinned memory)
// copies instead.
class HostTotals {
public:
    explicit HostTotals(hipStream_t s)
    {
        // Under capture the wait is refused, and a slot would be kept for good by each such call.
        hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
        if (hipStreamIsCapturing(s, &capture) != hipSuccess) {
            (void)hipGetLastError(); // (the wait will say)
            return;
        }
        if (capture != hipStreamCaptureStatusNone) return;
        static std::once_flag once;
        std::call_once(once, [] {
            void *p = nullptr;
            if (hipHostMalloc(&p, kSlots * kSlotBytes, hipHostMallocPortable | hipHostMallocMapped | hipHostMallocCoherent) == hipSuccess)
                page_ = static_cast<uint8_t *>(p);
            else
                (void)hipGetLastError(); // (the calls copy)
        });
        for (int i = 0; page_ && i < kSlots && slot_ < 0; ++i)
            if (!taken_[i].exchange(true, std::memory_order_acquire)) slot_ = i;
        void *p = nullptr;
        if (host() && hipHostGetDevicePointer(&p, host(), 0) != hipSuccess) {
            (void)hipGetLastError(); // (the call copies)
            give_back();
            p = nullptr;
        }
        device_ = static_cast<Totals *>(p);
    }
    ~HostTotals() { give_back(); }
    HostTotals(const HostTotals &) = delete;
    HostTotals &operator=(const HostTotals &) = delete;
    Totals *host() const { return slot_ < 0 ? nullptr : reinterpret_cast<Totals *>(page_ + slot_ * kSlotBytes); }
    Totals *device() const { return device_; } // the same for the device that was current
    void keep() { slot_ = -1; }                // not given back: the GPU may still write it

private:
    void give_back()
    {
        if (slot_ >= 0) taken_[slot_].store(false, std::memory_order_release);
        slot_ = -1;
    }

    static constexpr int kSlots = 16, kSlotBytes = 64;
    static_assert(sizeof(Totals) <= kSlotBytes, "a slot holds the totals");
    static inline uint8_t *page_ = nullptr;
    static inline std::atomic<bool> taken_[kSlots] = {};
    int slot_ = -1;
    Totals *device_ = nullptr;
};

// One wave per BlockTile.  A lane owns one FragTile row per TensorCoreTile: its byte of each
// bit-plane, its in-window bytes and its fallback halfwords, placed by prefix sums over the lanes.
// Bound by memory (the matrix once, the blob once; 28672 x 4096: 75 us, 5.3 TB/s, a plain copy's rate;
// with byte stores to global memory it was 148 us): everything is assembled in LDS and leaves in
// 16-byte pieces.  The wave's buffer holds the bit-planes first and, once they are stored, the H
// segment with the L segment behind it (together at most 8208 bytes whatever the mix), so four
// workgroups fit on a compute unit.  A row's in-window bytes are compacted with two v_perm (selectors
// from a table over the indicator byte), shifted to their byte position and combined with their
// neighbours' by LDS OR; the buffer starts from zero, which also makes the segments' padding.
// The stores are non-temporal: with ordinary ones the kernel takes as long, but leaves its last lines dirty in the
// caches, and whoever reads memory next waits for their way out (hist_kernel of the next 28672 x 4096 call 55.8 us instead of
// 45.9, the call 170.3 instead of 156.5; 6144 x 4096 80.2 / 76.9; 1024 x 4096 no difference).
constexpr uint32_t kPackBuf = 2 * ZS_BT_ELEMS + 32;
__global__ __launch_bounds__(256) void pack_kernel(const uint16_t *W, int64_t ldw, uint32_t k_blocks, uint32_t n_bt,
                                                   const Totals *totals, uint8_t *blob, uint64_t cap, const uint32_t *offsets,
                                                   uint64_t off_offsets, uint64_t off_H)
{
    __shared__ __attribute__((aligned(16))) uint8_t bufs[4][kPackBuf];
    __shared__ __attribute__((aligned(8))) u32x2 compact[256];
    const uint64_t off_L = align_up(off_H + totals->h_units * 16, ZS_SECTION_ALIGN);
    if (blockIdx.x == gridDim.x - 1) { // the gaps behind the four sections (each below 256 bytes)
        const uint64_t end_L = off_L + totals->l_units * 16;
        const uint64_t from[4] = {(uint64_t)n_bt * ZS_BT_BITMAP_BYTES, off_offsets + ((uint64_t)n_bt + 1) * 8,
                                  off_H + totals->h_units * 16, end_L};
        const uint64_t to[4] = {off_offsets, off_H, off_L, align_up(end_L, ZS_SECTION_ALIGN)};
        for (int g = 0; g < 4; ++g)
            if (from[g] + threadIdx.x < min(to[g], cap)) blob[from[g] + threadIdx.x] = 0;
        return;
    }
    { // selectors that move the bytes of in-window elements to the front, zeros (0x0C) behind them
        const uint32_t m = threadIdx.x;
        uint64_t sel = 0x0C0C0C0C0C0C0C0Cull;
        for (int e = 7; e >= 0; --e)
            if ((m >> e) & 1u) sel = (sel << 8) | (uint32_t)e;
        compact[m] = u32x2{(uint32_t)sel, (uint32_t)(sel >> 32)};
    }
    __syncthreads();
    const uint32_t lane = threadIdx.x & 63u, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t bt = blockIdx.x * 4 + wave;
    if (bt >= n_bt) return;
    const uint16_t *tile = tile_at(W, ldw, k_blocks, bt);
    uint8_t *buf = bufs[wave];
    u32x4 v[ZS_TT_PER_BT];
#pragma unroll
    for (int tt = 0; tt < ZS_TT_PER_BT; ++tt) v[tt] = load_row(tile, ldw, tt, lane);
    const uint32_t lo2 = totals->win_lo * 0x00010001u;

    // ---- bit-planes: byte r of a FragTile's 64-bit plane holds elements 8 r .. 8 r + 7, this lane's row
    uint32_t ind[ZS_TT_PER_BT]; // indicator bytes (1 = in-window element)
#pragma unroll
    for (int tt = 0; tt < ZS_TT_PER_BT; ++tt) {
        const uint32_t nib = codes_of(v[tt].x, lo2) | (codes_of(v[tt].y, lo2) << 4) | (codes_of(v[tt].z, lo2) << 8) |
                             (codes_of(v[tt].w, lo2) << 12);
        uint8_t *p = buf + (tt * ZS_FT_PER_TT + (lane >> 3)) * ZS_FT_BITMAP_BYTES + (lane & 7u);
        p[0] = (uint8_t)gather_bits(nib), p[8] = (uint8_t)gather_bits(nib >> 1), p[16] = (uint8_t)gather_bits(nib >> 2);
        ind[tt] = gather_bits(nib >> 3) ^ 0xFFu;
    }
    auto lds_done = []() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }; // lanes exchange through LDS
    auto send = [&](uint64_t at, const uint8_t *from, uint32_t units, uint32_t max_units) {
        for (uint32_t c = 0; c < max_units; c += 64) {
            if (c >= units) break;
            const uint32_t u = c + lane;
            if (u < units && at + 16ull * u + 16 <= cap) // (non-temporal: see above the kernel)
                __builtin_nontemporal_store(*reinterpret_cast<const u32x4 *>(from + 16 * u),
                                            reinterpret_cast<u32x4 *>(blob + at + 16ull * u));
        }
    };
    lds_done();
    send((uint64_t)bt * ZS_BT_BITMAP_BYTES, buf, ZS_BT_BITMAP_BYTES / 16, 96);

    // ---- positions: in-window elements before the lane's row, three TensorCoreTiles to a prefix sum
    uint32_t before[ZS_TT_PER_BT], nh = 0;
#pragma unroll
    for (int g = 0; g < ZS_TT_PER_BT; g += 3) {
        uint32_t pk = 0;
#pragma unroll
        for (int i = 0; i < 3; ++i)
            if (g + i < ZS_TT_PER_BT) pk |= (uint32_t)__builtin_popcount(ind[g + i]) << (10 * i);
        const uint32_t inc = wave_inclusive_scan(pk), exc = inc - pk, tot = __builtin_amdgcn_readlane(inc, 63);
#pragma unroll
        for (int i = 0; i < 3; ++i)
            if (g + i < ZS_TT_PER_BT) {
                before[g + i] = nh + ((exc >> (10 * i)) & 0x3FFu);
                nh += (tot >> (10 * i)) & 0x3FFu;
            }
    }
    const uint32_t h_units = (nh + 15u) / 16u, l_units = (2u * (ZS_BT_ELEMS - nh) + 15u) / 16u;
    lds_done(); // the bit-planes have left the buffer
    for (uint32_t u = lane; u < h_units + l_units; u += 64) *reinterpret_cast<u32x4 *>(buf + 16 * u) = u32x4{0u, 0u, 0u, 0u};
    lds_done();

    // ---- H bytes (sign and mantissa) and L halfwords
    uint8_t *l_buf = buf + 16 * h_units;
#pragma unroll
    for (int tt = 0; tt < ZS_TT_PER_BT; ++tt) {
        const uint32_t m = ind[tt];
        const u32x2 sel = compact[m];
        uint32_t b[4]; // bytes 0 and 2: sign << 7 | mantissa of the pair
#pragma unroll
        for (int c = 0; c < 4; ++c) b[c] = (v[tt][c] & 0x007F007Fu) | ((v[tt][c] >> 8) & 0x00800080u);
        const uint32_t lo = __builtin_amdgcn_perm(b[1], b[0], 0x06040200u), hi = __builtin_amdgcn_perm(b[3], b[2], 0x06040200u);
        const uint64_t row = __builtin_amdgcn_perm(hi, lo, sel.x) | (uint64_t)__builtin_amdgcn_perm(hi, lo, sel.y) << 32;
        const uint32_t sh = 8 * (before[tt] & 3u);
        const uint64_t low = row << sh;
        const uint32_t top = (uint32_t)(row >> 32 >> 8) >> (24 - sh);
        uint32_t *at = reinterpret_cast<uint32_t *>(buf + (before[tt] & ~3u));
        // (a row that ends at an exact dword leaves zeros for the words behind it: not touched, they
        // may lie in the L segment)
        if ((uint32_t)low) __hip_atomic_fetch_or(at, (uint32_t)low, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        if ((uint32_t)(low >> 32)) __hip_atomic_fetch_or(at + 1, (uint32_t)(low >> 32), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        if (top) __hip_atomic_fetch_or(at + 2, top, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        uint32_t l_at = 2u * (512u * tt + 8u * lane - before[tt]);
#pragma unroll
        for (int e = 0; e < 8; ++e)
            if (!((m >> e) & 1u)) {
                *reinterpret_cast<uint16_t *>(l_buf + l_at) = (uint16_t)(v[tt][e >> 1] >> (16 * (e & 1)));
                l_at += 2;
            }
    }
    lds_done();
    // the segments as the offsets bound them (the same sizes, unless W changed during the call)
    const uint32_t h0 = offsets[2 * (size_t)bt], l0 = offsets[2 * (size_t)bt + 1];
    const uint32_t h_room = offsets[2 * (size_t)bt + 2] - h0, l_room = offsets[2 * (size_t)bt + 3] - l0;
    send(off_H + (uint64_t)h0 * 16, buf, min(h_units, h_room), ZS_BT_ELEMS / 16);
    send(off_L + (uint64_t)l0 * 16, l_buf, min(l_units, l_room), ZS_BT_ELEMS / 8);
}

} // namespace

extern "C" int zs_encode_device(const uint16_t *W_dev, int64_t N, int64_t K, int64_t ldw, void *blob_dev, size_t blob_cap,
                                zs_desc *out, void *workspace_dev, size_t workspace_bytes, void *hip_stream)
{
    if (!W_dev || !blob_dev || !out || !workspace_dev) return ZS_ERR_ARG;
    if (reinterpret_cast<uintptr_t>(W_dev) % 16 || reinterpret_cast<uintptr_t>(blob_dev) % ZS_SECTION_ALIGN ||
        reinterpret_cast<uintptr_t>(workspace_dev) % 16)
        return ZS_ERR_ARG;
    if (N <= 0 || K <= 0 || N % ZS_BT_DIM || K % ZS_BT_DIM || ldw < K || ldw % 8) return ZS_ERR_SHAPE;
    if (workspace_bytes < ZS_ENCODE_WORKSPACE_BYTES || blob_cap < zs_encode_bound(N, K)) return ZS_ERR_SIZE;
    const uint64_t n_bt64 = (uint64_t)(N / ZS_BT_DIM) * (uint64_t)(K / ZS_BT_DIM);
    if (n_bt64 >= (1ull << 31) || (uint64_t)N * (uint64_t)K / 8 >= (1ull << 32)) return ZS_ERR_SHAPE; // 32-bit unit offsets
    const uint32_t n_bt = (uint32_t)n_bt64, k_blocks = (uint32_t)(K / ZS_BT_DIM);
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    uint8_t *blob = static_cast<uint8_t *>(blob_dev), *ws = static_cast<uint8_t *>(workspace_dev);
    unsigned long long *hist_dev = reinterpret_cast<unsigned long long *>(ws);
    Totals *totals_dev = reinterpret_cast<Totals *>(ws + kTotalsAt);
    auto ok = [](hipError_t e) { return e == hipSuccess; };

    const uint64_t off_bitmaps = 0;
    const uint64_t off_offsets = align_up((uint64_t)n_bt * ZS_BT_BITMAP_BYTES, ZS_SECTION_ALIGN);
    const uint64_t off_H = align_up(off_offsets + ((uint64_t)n_bt + 1) * 8, ZS_SECTION_ALIGN);
    uint32_t *offsets_dev = reinterpret_cast<uint32_t *>(blob + off_offsets);
    // the counts of the BlockTiles lie where the bit-planes will be: pack_kernel writes those last
    uint32_t *counts_dev = reinterpret_cast<uint32_t *>(blob + off_bitmaps);

    // ---- window and counts (Algorithm 1, phase I), segment offsets, then the tiles (phase II)
    const uint32_t wgs = (uint32_t)(2 * zs_compute_units());
    auto at_most = [](uint64_t want, uint32_t limit) { return dim3((unsigned)(want < limit ? want : limit)); };
    hipLaunchKernelGGL(sample_kernel, dim3(1), dim3(1024), 0, s, W_dev, N, K, ldw, hist_dev, totals_dev);
    hipLaunchKernelGGL(hist_kernel, at_most((n_bt + kHistWaves - 1) / kHistWaves, wgs), dim3(64 * kHistWaves), 0, s, W_dev, ldw, k_blocks,
                       n_bt, hist_dev, totals_dev, counts_dev);
    hipLaunchKernelGGL(recount_kernel, at_most((n_bt + kHistWaves - 1) / kHistWaves, wgs), dim3(64 * kHistWaves), 0, s, W_dev, ldw, k_blocks,
                       n_bt, hist_dev, totals_dev, counts_dev);
    if (!ok(hipGetLastError())) return ZS_ERR_HIP; // (the pinned slot clears errors of its own, and these with them)
    HostTotals pinned(s);
    Totals *const mapped = pinned.device();
    const uint32_t per_wg = kScanRound * ((n_bt + kScanRound * kScanWgs - 1) / (kScanRound * kScanWgs));
    hipLaunchKernelGGL(scan_kernel, dim3((n_bt + per_wg - 1) / per_wg), dim3(1024), 0, s, counts_dev, offsets_dev, n_bt, per_wg, hist_dev,
                       totals_dev, mapped);
    hipLaunchKernelGGL(pack_kernel, dim3((n_bt + 3) / 4 + 1), dim3(256), 0, s, W_dev, ldw, k_blocks, n_bt, totals_dev, blob,
                       (uint64_t)blob_cap, offsets_dev, off_offsets, off_H);
    Totals tot;
    if (!ok(hipGetLastError()) || (!mapped && !ok(hipMemcpyAsync(&tot, totals_dev, sizeof tot, hipMemcpyDeviceToHost, s))) ||
        !ok(hipStreamSynchronize(s))) {
        pinned.keep();
        return ZS_ERR_HIP;
    }
    if (mapped) tot = *pinned.host();
    const uint64_t off_L = align_up(off_H + tot.h_units * 16, ZS_SECTION_ALIGN);
    const uint64_t total = align_up(off_L + tot.l_units * 16, ZS_SECTION_ALIGN);
    if (total > blob_cap) return ZS_ERR_SIZE;

    std::memset(out, 0, sizeof *out);
    out->magic = ZS_MAGIC;
    out->version = ZS_FORMAT_VERSION;
    out->N = N;
    out->K = K;
    out->base_exp = (int32_t)tot.win_lo - 1;
    out->tile_cfg = ZS_TILE_CFG_FT8_TT16x32_BT64;
    out->n_high = tot.n_high;
    out->n_fallback = (uint64_t)N * (uint64_t)K - tot.n_high;
    out->off_bitmaps = off_bitmaps;
    out->off_offsets = off_offsets;
    out->off_H = off_H;
    out->off_L = off_L;
    out->h_bytes = tot.h_units * 16;
    out->l_bytes = tot.l_units * 16;
    out->total_bytes = total;
    out->max_h_units = tot.max_h;
    out->max_l_units = tot.max_l;
    return ZS_OK;
}
