// HIP kernels and device entry points of libzipserv_hip.so (gfx950 only).
//   zs_decompress : TCA-TBE blob -> row-major BF16 (standalone kernel, Section 4.4)
//   zs_gemm       : C = A * decode(W)^T, decode fused into the MFMA loop (ZipGEMM, Section 4.3)
//
// Both kernels are built from independent waves.  A wave streams BlockTiles: the compressed
// bytes of the next DEPTH - 1 tiles are in flight from HBM straight into LDS
// (global_load_lds_dwordx4, the "tile loading" stage of Section 4.3.1) while the current tile
// is decoded from LDS into registers (Algorithm 2) and, in ZipGEMM, multiplied on the matrix
// cores.  No barrier is needed inside the stream: a wave only reads what it staged itself.
#include <hip/hip_runtime.h>

#include <atomic>
#include <cstring>
#include <type_traits>

#include "zipserv.h"
#include "zs_device.h"

using namespace zs;


namespace {

constexpr uint32_t kMaxLds = 160 * 1024;
constexpr int kMaxDevices = 64;

// ---- slot = LDS image of one BlockTile -------------------------------------------------
//   [0, 1536)            bit-planes
//   [1536, 5632)         H segment (at most 4096 bytes)
//   [5632, +LW)          first LW bytes of the L segment (LW = 512, 1024 or 4096)
//   64 bytes of slack    for the aligned over-read of the byte gathers
template <int LW>
struct Slot {
    static constexpr uint32_t kPlanes = 0, kH = ZS_BT_BITMAP_BYTES, kL = kH + 4096;
    static constexpr uint32_t kBytes = kL + LW + 64;
    static constexpr int kLChunks = (LW + 1023) / 1024;
    static constexpr int kLoads = 2 + 4 + kLChunks; // LDS-direct instructions per BlockTile
    // what the LDS-direct loads of a tile can write: 1536 bytes of bit-planes, four 1 KB pieces of
    // H, kLChunks pieces of L (one 512-byte piece for LW = 512); all of it lies inside the slot
    static_assert(kPlanes + ZS_BT_BITMAP_BYTES <= kH && kH + 4 * 1024 <= kL, "sections of a slot overlap");
    static_assert(kL + (LW == 512 ? 512 : kLChunks * 1024) <= kBytes, "the staged L window leaves the slot");
};

// LDS image of a gemm_stream_kernel workgroup, shared by the kernel (addresses) and the host
// (bytes to request): tables | accumulation tiles | control words | WAVES rings of kDepth slots.
// Where they fit (eight waves at 16 tokens, seven at 32), every streaming wave has an accumulation tile of its own;
// else there are two, used by turns under a lock.  Measured against two tiles there as well (cleared only where a
// range has more than one task), the line is not clear-cut, us, own / two: 28672 x 1024, 32 tokens 18.3 / 18.7; 32768 x
// 2048, 16 tokens 23.8 / 24.5; but 3072 x 4096, 16 tokens 13.4 / 12.2; 6144 x 4096, 16 tokens 15.1 / 14.6; 10240 x 4096,
// 32 tokens 23.1 / 22.0; 14336 x 1024, one token 12.4 / 11.7; of 45 sizes and token counts half differ by less than 1 %.
template <int MT, int LW, int WAVES>
struct StreamLds {
    static constexpr uint32_t kDepth = 2; // ring positions per wave: one tile decoded, one in flight
    static constexpr uint32_t kUnits = 16 * MT * 16, kTileBytes = 16 * kUnits; // float4 units of an accumulation tile
    // a wave's ring; at the end of the launch it holds the wave's sums of the last task
    static constexpr uint32_t kRingBytes = kDepth * Slot<LW>::kBytes > kTileBytes ? kDepth * Slot<LW>::kBytes : kTileBytes;
    static constexpr bool kOwnTiles = kTableBytes + 64 + WAVES * (kTileBytes + kRingBytes) <= kMaxLds;
    static constexpr uint32_t kTiles = kOwnTiles ? WAVES : 2;
    static constexpr uint32_t kRed = kTableBytes, kCtl = kRed + kTiles * kTileBytes, kRings = kCtl + 64;
    static constexpr uint32_t kTotal = kRings + WAVES * kRingBytes;
    static_assert(kTotal <= kMaxLds, "variant does not fit the 160 KB of LDS");
};

struct Segments {
    const uint8_t *h, *l;
    uint32_t h_bytes, l_bytes;
    uint32_t h_room, l_room; // 16-byte units from the segment's start to the end of its section
};

// The two offset pairs that bracket BlockTile bt.  The offset array is read-only for the whole
// launch: reading it through the constant address space lets a wave-uniform index use scalar
// loads, which do not share the vector-memory counter with the LDS-direct loads.
struct OffsetPairs {
    u32x2 o0, o1;
};
__device__ __forceinline__ OffsetPairs offset_pairs(const BlobView &bv, uint32_t bt)
{
    typedef const u32x2 __attribute__((address_space(4))) *ConstPairs;
    const ConstPairs off = (ConstPairs)(uintptr_t)bv.offsets;
    return OffsetPairs{off[bt], off[bt + 1]};
}

// Start and size of a BlockTile's H and L segments, clamped so that no read can leave the
// blob sections or a slot whatever the offset array holds.
__device__ __forceinline__ Segments segments_from(const BlobView &bv, const OffsetPairs &o)
{
    const uint32_t h0 = min(o.o0.x, bv.h_units), l0 = min(o.o0.y, bv.l_units);
    const uint32_t h1 = min(max(o.o1.x, h0), bv.h_units), l1 = min(max(o.o1.y, l0), bv.l_units);
    Segments s;
    s.h = bv.H + (size_t)h0 * 16;
    s.l = bv.L + (size_t)l0 * 16;
    s.h_bytes = min(h1 - h0, (uint32_t)(ZS_BT_ELEMS / 16)) * 16;
    s.l_bytes = min(l1 - l0, (uint32_t)(2 * ZS_BT_ELEMS / 16)) * 16;
    s.h_room = bv.h_units - h0;
    s.l_room = bv.l_units - l0;
    return s;
}
__device__ __forceinline__ Segments segments_of(const BlobView &bv, uint32_t bt)
{
    return segments_from(bv, offset_pairs(bv, bt));
}

__device__ __forceinline__ uint32_t uniform(uint32_t x) { return __builtin_amdgcn_readfirstlane(x); }

// LDS address of the dynamic shared array: it follows the kernel's static LDS (a link-time
// constant; these kernels have none).  Taking the address through a pointer cast instead
// leaves a null-pointer select at every use.
__device__ __forceinline__ uint32_t dynamic_lds_base() { return __builtin_amdgcn_groupstaticsize(); }

// All LDS-direct loads of a BlockTile whose segments start far enough from the ends of their
// sections (BlobView::h_fast, l_fast): 1536 bytes of bit-planes, 4096 bytes from the start of
// the H segment and LW bytes from the start of the L segment, whatever the segments' lengths
// (what lies beyond them belongs to the next BlockTiles and is ignored).  No address or lane
// mask is computed: three base registers, instruction offsets, and the lower half of the wave
// for the two 512-byte pieces.  Exactly Slot<LW>::kLoads instructions; nothing is waited for.
// All operands except lane16 (= 16 * lane) are wave-uniform; all 64 lanes must be active.
template <int LW>
__device__ __forceinline__ void stage_fast(uint32_t lane16, uint32_t slot_at, const uint8_t *planes, const uint8_t *h,
                                           const uint8_t *l)
{
    using S = Slot<LW>;
    static_assert(S::kPlanes == 0 && S::kH == 1536 && S::kL == 5632, "the LDS offsets below assume this slot layout");
    static_assert(LW == 512 || LW == 1024 || LW == 4096, "L windows staged below");
#define ZS_LOAD "global_load_lds_dwordx4 %[l16], "
    if constexpr (LW == 512) {
        asm volatile("s_mov_b32 m0, %[slot]\n\ts_nop 0\n\t" ZS_LOAD "%[bp]\n\t"
                     "s_add_u32 m0, %[slot], 1536\n\ts_nop 0\n\t" ZS_LOAD "%[bh]\n\t" ZS_LOAD "%[bh] offset:1024\n\t"
                     ZS_LOAD "%[bh] offset:2048\n\t" ZS_LOAD "%[bh] offset:3072\n\t"
                     "s_mov_b32 m0, %[slot]\n\ts_mov_b64 exec, %[half]\n\t" ZS_LOAD "%[bp] offset:1024\n\t"
                     "s_add_u32 m0, %[slot], 5632\n\ts_nop 0\n\t" ZS_LOAD "%[bl]\n\t"
                     "s_mov_b64 exec, -1"
                     :
                     : [l16] "v"(lane16), [slot] "s"(slot_at), [bp] "s"(planes), [bh] "s"(h), [bl] "s"(l),
                       [half] "s"(0xFFFFFFFFull)
                     : "memory", "scc", "m0");
    } else if constexpr (LW == 1024) {
        asm volatile("s_mov_b32 m0, %[slot]\n\ts_nop 0\n\t" ZS_LOAD "%[bp]\n\t"
                     "s_add_u32 m0, %[slot], 1536\n\ts_nop 0\n\t" ZS_LOAD "%[bh]\n\t" ZS_LOAD "%[bh] offset:1024\n\t"
                     ZS_LOAD "%[bh] offset:2048\n\t" ZS_LOAD "%[bh] offset:3072\n\t"
                     "s_add_u32 m0, %[slot], 5632\n\ts_nop 0\n\t" ZS_LOAD "%[bl]\n\t"
                     "s_mov_b32 m0, %[slot]\n\ts_mov_b64 exec, %[half]\n\t" ZS_LOAD "%[bp] offset:1024\n\t"
                     "s_mov_b64 exec, -1"
                     :
                     : [l16] "v"(lane16), [slot] "s"(slot_at), [bp] "s"(planes), [bh] "s"(h), [bl] "s"(l),
                       [half] "s"(0xFFFFFFFFull)
                     : "memory", "scc", "m0");
    } else {
        asm volatile("s_mov_b32 m0, %[slot]\n\ts_nop 0\n\t" ZS_LOAD "%[bp]\n\t"
                     "s_add_u32 m0, %[slot], 1536\n\ts_nop 0\n\t" ZS_LOAD "%[bh]\n\t" ZS_LOAD "%[bh] offset:1024\n\t"
                     ZS_LOAD "%[bh] offset:2048\n\t" ZS_LOAD "%[bh] offset:3072\n\t"
                     "s_add_u32 m0, %[slot], 5632\n\ts_nop 0\n\t" ZS_LOAD "%[bl]\n\t" ZS_LOAD "%[bl] offset:1024\n\t"
                     ZS_LOAD "%[bl] offset:2048\n\t" ZS_LOAD "%[bl] offset:3072\n\t"
                     "s_mov_b32 m0, %[slot]\n\ts_mov_b64 exec, %[half]\n\t" ZS_LOAD "%[bp] offset:1024\n\t"
                     "s_mov_b64 exec, -1"
                     :
                     : [l16] "v"(lane16), [slot] "s"(slot_at), [bp] "s"(planes), [bh] "s"(h), [bl] "s"(l),
                       [half] "s"(0xFFFFFFFFull)
                     : "memory", "scc", "m0");
    }
#undef ZS_LOAD
}

// A BlockTile as the issuing side of a wave knows it (everything wave-uniform): its number and
// the two offset pairs {H start, L start} that bracket it.  "No tile" is g = kNoTileG with
// offsets of all ones (BlockTile numbers are below 2^31; the offsets then fail the bounds test
// of the common staging path).
struct TileRef {
    uint32_t g;
    u32x4 off; // {H start, L start, next H start, next L start}, 16-byte units
};
constexpr uint32_t kNoTileG = ~0u;
#define kNoTileOff (u32x4{~0u, ~0u, ~0u, ~0u})

// What the decoding side needs to know about the L segment of a staged tile.
struct StagedL {
    const uint8_t *l; // the segment in global memory
    uint32_t big;     // nonzero: it is longer than the staged window, fallbacks are read from `l`
};

// Both offset pairs of BlockTile bt with one scalar load (the offset array is read-only for the
// launch: through the constant address space a wave-uniform index becomes a scalar load, which
// does not share the vector-memory counter with the LDS-direct loads).
__device__ __forceinline__ u32x4 offset_quad(const BlobView &bv, uint32_t bt)
{
    typedef uint32_t __attribute__((ext_vector_type(4), aligned(8))) Quad;
    typedef const Quad __attribute__((address_space(4))) *ConstQuad;
    const Quad q = *(ConstQuad)(uintptr_t)(bv.offsets + bt);
    return u32x4{q.x, q.y, q.z, q.w};
}

// Stages tile t into the slot at slot_at with exactly Slot<LW>::kLoads LDS-direct instructions
// (also for "no tile": then only lane 0 runs, on a dummy address).  No read can leave the blob
// sections or the slot whatever the offset array holds: the common path checks the segment
// starts against the precomputed bounds, the other one clamps every start and length.
template <int LW>
__device__ __forceinline__ StagedL stage_tile(const BlobView &bv, const TileRef &t, uint32_t slot_at, uint32_t lane)
{
    using S = Slot<LW>;
    const uint32_t h0 = t.off.x, l0 = t.off.y;
    if (h0 < bv.h_fast && l0 < bv.l_fast) {
        const uint8_t *l = bv.L + (size_t)l0 * 16;
        stage_fast<LW>(lane * 16, slot_at, bv.bitmaps + (size_t)t.g * ZS_BT_BITMAP_BYTES, bv.H + (size_t)h0 * 16, l);
        // a wrong length can only choose the wrong source of fallbacks: both are readable
        return StagedL{l, t.off.w - l0 > (uint32_t)(LW / 16) ? 1u : 0u};
    }
    const bool valid = t.g != kNoTileG;
    Segments sg = {bv.H, bv.L, 0u, 0u, 0u, 0u};
    if (valid) sg = segments_from(bv, OffsetPairs{u32x2{t.off.x, t.off.y}, u32x2{t.off.z, t.off.w}});
    const uint8_t *planes = bv.bitmaps + (size_t)(valid ? t.g : 0u) * ZS_BT_BITMAP_BYTES;
    dma_segment<2>(planes, valid ? ZS_BT_BITMAP_BYTES : 0u, slot_at + S::kPlanes, lane * 16, bv.bitmaps);
    dma_segment<4>(sg.h, sg.h_bytes, slot_at + S::kH, lane * 16, bv.bitmaps);
    dma_segment<S::kLChunks>(sg.l, min(sg.l_bytes, (uint32_t)LW), slot_at + S::kL, lane * 16, bv.bitmaps);
    return StagedL{sg.l, sg.l_bytes > (uint32_t)LW ? 1u : 0u};
}

// --------------------------------------------------------------------------------------
// Standalone decompression: waves take BlockTiles round-robin; 16 bytes (8 weights) per lane
// and TensorCoreTile are stored row-major, in whole cache lines.  Bound by memory: 28672 x 4096 reads
// and writes 403 MB in 76.5 us, 5.3 TB/s, the rate of a device copy; with half lines it wrote 265 MB
// for 235 and took 98.8 us.  4096 x 14336: 37.7 -> 33.8 us.  Without the non-temporal hint 83 and 44 us.
// LINES = false stores each TensorCoreTile as it is decoded, in half lines (zs_decompress says when).
// --------------------------------------------------------------------------------------
template <int LW, int DEPTH, int WAVES, bool BASE_M1, Fallbacks CAREFUL, bool LINES>
__global__ __launch_bounds__(64 * WAVES) void decompress_kernel(BlobView bv, uint16_t *out, int64_t ldw)
{
    using S = Slot<LW>;
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    const uint32_t lane = threadIdx.x & 63u, wave = uniform(threadIdx.x >> 6);
    const uint32_t tab = dynamic_lds_base();
    const uint32_t ring = tab + kTableBytes + wave * (DEPTH * S::kBytes);
    const uint32_t n_bt = (uint32_t)bv.strips * (uint32_t)bv.k_blocks;
    const uint32_t first = blockIdx.x * WAVES + wave, stride = gridDim.x * WAVES;
    // what the lane stores, see below: row lane % 8 of eight, 16 bytes of its 128; without LINES the row it
    // decodes (FragTiles run N-fastest), 16 bytes of its 64
    const bool upper = (lane & 8u) != 0;
    const uint32_t row = LINES ? lane & 7u : lane & 15u, col = (lane >> 4) * 8u + (LINES ? (lane & 8u) * 4u : 0u);

#pragma unroll
    for (int j = 0; j < DEPTH - 1; ++j) {
        const uint32_t bt = first + j * stride;
        const bool valid = bt < n_bt;
        stage_tile<LW>(bv, valid ? TileRef{bt, offset_quad(bv, bt)} : TileRef{kNoTileG, kNoTileOff}, ring + j * S::kBytes, lane);
    }
    // Built behind the first loads, which hide it: 1024 x 4096 7.25 -> 7.0 us, 6144 x 4096 17.4 -> 16.3, 4096 x 14336 40.4 -> 39.7
    // (one matrix after the other, cold); nothing beyond the noise at 28672 x 4096.
    build_tables(smem, bv.base_exp);
    __syncthreads();
    uint32_t cur = 0, nxt = DEPTH - 1; // ring positions of the tile being decoded / being issued
    for (uint32_t bt = first; bt < n_bt; bt += stride) {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); // every LDS read of the slot about to be refilled is done
        const uint32_t ahead = bt + (DEPTH - 1) * stride;
        const bool valid = ahead < n_bt;
        stage_tile<LW>(bv, valid ? TileRef{ahead, offset_quad(bv, ahead)} : TileRef{kNoTileG, kNoTileOff},
                       ring + nxt * S::kBytes, lane);
        wait_dma<(DEPTH - 1) * S::kLoads>();

        const uint32_t slot = ring + cur * S::kBytes;
        const Segments sg = segments_of(bv, bt);
        HalfIndex h0;
        const uint32_t pa = plane_address(slot + S::kPlanes, lane);
        read_planes<0, 0, false>(pa, h0);
        uint32_t h_base = slot + S::kH;
        index_half<true>(h_base, h0);
        const FallbackSource fs = {slot + S::kL, reinterpret_cast<const uint16_t *>(sg.l), sg.l_bytes > (uint32_t)LW};
        const uint32_t strip = bt / (uint32_t)bv.k_blocks, kb = bt % (uint32_t)bv.k_blocks;
        // A decoded TensorCoreTile is 16 rows of 64 bytes: stored as it is, every store instruction writes
        // halves of cache lines.  Two that are neighbours along K make whole lines of 128 bytes: lanes of
        // rows 0 .. 7 and of rows 8 .. 15 (lane ^ 8) swap, so that one store writes rows 0 .. 7 of both, the
        // other rows 8 .. 15.
        uint16_t *dst = out + ((int64_t)strip * 64 + row) * ldw + (int64_t)kb * 64 + col;
        u32x4 left[4]; // the TensorCoreTiles of the first k half, until their neighbours are decoded
        decode_block_tile<BASE_M1, 0, 0, CAREFUL>(tab, pa, h0, h_base, l_lane_of(slot + S::kH, slot + S::kL, lane), fs,
                                         [&](int tt, const u32x4 &w) {
                                             if (!LINES) {
                                                 __builtin_nontemporal_store(
                                                     w, reinterpret_cast<u32x4 *>(dst + (int64_t)((tt & 3) * 16) * ldw + (tt >> 2) * 32));
                                                 return;
                                             }
                                             if (tt < 4) {
                                                 left[tt] = w;
                                                 return;
                                             }
                                             u32x4 lo, hi;
#pragma unroll
                                             for (int c = 0; c < 4; ++c) {
                                                 const uint32_t a = left[tt & 3][c], b = w[c];
                                                 const uint32_t got = __builtin_amdgcn_update_dpp(
                                                     0u, upper ? a : b, 0x128, 0xf, 0xf, false); // row_ror:8 = lane ^ 8
                                                 lo[c] = upper ? got : a, hi[c] = upper ? b : got;
                                             }
                                             uint16_t *at = dst + (int64_t)((tt & 3) * 16) * ldw;
                                             __builtin_nontemporal_store(lo, reinterpret_cast<u32x4 *>(at));
                                             __builtin_nontemporal_store(hi, reinterpret_cast<u32x4 *>(at + 8 * ldw));
                                         });
        cur = cur + 1 == DEPTH ? 0 : cur + 1;
        nxt = nxt + 1 == DEPTH ? 0 : nxt + 1;
    }
    wait_dma<0>();
}

// --------------------------------------------------------------------------------------
// ZipGEMM, skinny-M regime.  W is the MFMA A operand (rows = output features), the
// activations are the B operand (columns = tokens, 16 per MFMA, MT MFMAs per weight tile).
//
// Work split (a refinement of the split-K tiling of Section 4.3.1): the BlockTiles of the
// matrix, in storage order (K-fastest inside 64-row strips), form one sequence that is cut
// into gridDim.x equal contiguous ranges, one per workgroup, wherever the cuts fall.  The
// part of a strip inside a range is a task (tasks are numbered locally, j = 0, 1, ..., in the
// order they are processed: the range's last strip first, then from its beginning).
//
// Inside a workgroup WAVES streaming waves take BlockTiles from the range one at a time off
// a shared counter (so a wave that shares its SIMD with fewer others simply takes more), each
// staging its next tile with LDS-direct loads while it decodes and multiplies the current one.
// A wave keeps the 64 x (16 MT) FP32 partial sums of one task in registers; when its next
// tile belongs to another task it leaves them in an LDS tile of its own, or adds them, under a
// lock, into that task's tile (two tiles, by parity of j) where LDS has no room, and reports how
// many BlockTiles they covered.  One more wave, the writer, waits until a task's count is complete,
// takes the sums out of LDS, hands the tile back and stores it to C when the task is a whole strip.
// The last task is finished by the streaming waves themselves, a few rows each.  The tile of a
// strip shared with other workgroups goes to global scratch instead, and the last workgroup
// to contribute adds the tiles up and stores the strip (without scratch memory: FP32 atomics
// onto a C cleared beforehand).  Streaming waves never meet at a barrier.
//
// The activations of a 64-wide K slab (L2-resident) are loaded straight from A into registers,
// in B-operand lane order, at the top of the step that uses them: before the LDS-direct loads
// of the next tile, so that the staging and the indexing cover their L2 round trip.
// --------------------------------------------------------------------------------------
typedef __attribute__((address_space(3))) uint32_t *LdsU32;
typedef __attribute__((address_space(3))) f32x4 *LdsF32x4;

__device__ __forceinline__ uint32_t lds_poll(uint32_t at)
{
    return __hip_atomic_load((LdsU32)at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
// Waits for every LDS and scalar-memory operation of the wave.  The builtin (not inline
// assembly) lets the compiler's own wait-count bookkeeping see the wait, so it does not wait
// again, later and for more, for a scalar load that this one already covered.
__device__ __forceinline__ void lds_fence()
{
    __builtin_amdgcn_s_waitcnt(0xC07F); // lgkmcnt(0), the other counters untouched
    asm volatile("" ::: "memory");
}

// Control words in LDS (byte offsets from the control block).
enum : uint32_t { kCtlNext = 0, kCtlWritten = 4, kCtlLock = 8, kCtlFrom = 8, kCtlDone = 16, kCtlArrived = 24, kCtlCounted = 28, kCtlBytes = 64 };

// How the partial sums of a strip that several workgroups contribute to become C.
//   kSumCleared  the host cleared the strip's columns with a kernel of its own before this
//                launch; contributors add with FP32 atomics (no scratch memory needed)
//   kSumParked   contributors park their partial tiles in scratch memory and count themselves
//                in; the last one adds the tiles up and stores the strip
// count[b] belongs to the shared strip whose first contributor is workgroup b (unique: a range
// that holds the starts of two strips holds the first of them whole); it is zero between
// launches (whoever counts last takes it down).  tiles holds two slots per workgroup (for its
// first and its last task), each 64 rows x 16 MT tokens of FP32, all zero bits between
// launches as well (the last contributor clears what it has read).
// Measured and dropped: the first contributor zeroing the columns and raising a flag, everybody
// adding with atomics once the flag is up (no round trip at the end of the kernel, but the
// atomics themselves take longer than the exchange through kSumParked at 32 tokens).
enum : uint32_t { kSumCleared = 0, kSumParked = 1 };
struct SharedSums {
    uint32_t *count;
    float *tiles;
    uint32_t mode;
    uint32_t out_bf16;    // nonzero: C holds BF16 bit patterns (ldc in those elements); needs kSumParked
    uint32_t tiles_bytes; // size of the slot area at `tiles` (two slots per workgroup)
};

// FP32 -> BF16 bit pattern, round to nearest even; NaN stays NaN (quiet bit set, sign and the
// upper payload bits kept).
__device__ __forceinline__ uint32_t bf16_rne(float x)
{
    const uint32_t u = __builtin_bit_cast(uint32_t, x);
    const uint32_t rounded = (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
    return (u & 0x7FFFFFFFu) > 0x7F800000u ? ((u >> 16) | 0x40u) : rounded;
}

// Division of a number below 2^31 by d >= 1 with one multiplication: with 2^(l-1) < d <= 2^l and
// magic = ceil(2^(31+l) / d) (below 2^32) the quotient is floor(n magic / 2^(31+l)), because magic d exceeds
// 2^(31+l) by less than d <= 2^l.  A division by a run-time value is some thirty dependent vector
// instructions; the kernels do it before their first load and between their last BlockTile and the end.
struct Divider {
    uint32_t d, magic;
    static constexpr __host__ __device__ uint32_t log2_up(uint32_t d) { return d > 1 ? 32u - (uint32_t)__builtin_clz(d - 1) : 0u; }
    static constexpr Divider by(uint32_t d) { return Divider{d, (uint32_t)(((1ull << (31 + log2_up(d))) + d - 1) / d)}; }
    constexpr __host__ __device__ uint32_t operator()(uint32_t n) const
    {
        return (uint32_t)((uint64_t)(2 * n) * magic >> 32) >> log2_up(d);
    }
};
constexpr bool divides(uint32_t d) // at both ends of the range and around the multiples of d there
{
    constexpr uint32_t top = (1u << 31) - 1;
    const uint32_t last = top / d * d, at[] = {0u, d - 1, d, last - 1, last, top, top - 1};
    for (uint32_t n : at)
        if (n <= top && Divider::by(d)(n) != n / d) return false;
    return true;
}
static_assert(divides(1) && divides(2) && divides(3) && divides(7) && divides(16) && divides(63) && divides(64) && divides(65) &&
                  divides(224) && divides(448) && divides(65535) && divides(65537) && divides((1u << 30) - 1) &&
                  divides((1u << 30) + 1) && divides((1u << 31) - 1), "division by multiplication");

// The BlockTile sequence [0, total) is cut into `parts` contiguous ranges of q or q + 1
// BlockTiles (the first r ranges have q + 1), total = parts * q + r.  The host fills the
// struct, so that no kernel divides by a run-time value on its main path.
struct RangeSplit {
    uint32_t total, parts, q, r;
    uint32_t magic_q, magic_q1; // of the Dividers by q and q + 1
    __host__ __device__ uint32_t begin(uint32_t b) const { return b * q + (b < r ? b : r); }
    // the range that BlockTile g lies in
    __host__ __device__ uint32_t of(uint32_t g) const
    {
        const uint32_t wide = r * (q + 1);
        return g < wide ? Divider{q + 1, magic_q1}(g) : r + Divider{q, magic_q}(g - wide);
    }
};

// Arguments of gemm_stream_kernel beyond the scalar ones in front.
struct StreamArgs {
    const uint16_t *A;
    int64_t lda;
    float *C;
    int64_t ldc;
    SharedSums ws;
    int M;
    int32_t base_exp;
    uint32_t h_units, l_units, h_fast, l_fast, magic_q, magic_q1;
};

// Where the StreamArgs lie in the memory of the arguments: behind the scalar ones, each at the next multiple of its
// alignment.  The launch checks that the kernel's arguments are those of StreamKernel.
using StreamKernel = void (*)(const u32x2 *, const uint8_t *, const uint8_t *, const uint8_t *, uint32_t, uint32_t, uint32_t, uint32_t,
                              uint32_t, StreamArgs);
template <class... Args>
constexpr size_t last_argument_at(void (*)(Args...))
{
    size_t end = 0, at = 0;
    ((at = (end + alignof(Args) - 1) / alignof(Args) * alignof(Args), end = at + sizeof(Args)), ...);
    return at;
}
constexpr size_t kStreamArgsAt = last_argument_at(StreamKernel{});

// The scalar arguments in front, 13 words, arrive in registers with the launch (the build asks for kernel
// argument preloading): what the offsets of the first BlockTile depend on is there at the first instruction, and
// the others are loaded behind those offsets, so that they are no link of the chain arguments -> offsets -> BlockTile.
// The first BlockTile's loads are issued 430 to 1580 cycles earlier (the same stamped copies before and after); with the
// divisions and the tables' halves on different waves, us: 1024 x 4096, one token 8.4 -> 8.2; 6144 x 4096, 7 tokens 14.55 -> 14.2;
// 28672 x 4096, 16 tokens 38.6 -> 38.0, 50 tokens 52.9 -> 52.1; 4096 x 14336, 16 tokens, row-scaled 31.75 -> 31.1.
template <int MT, int LW, int WAVES, bool BASE_M1, Fallbacks CAREFUL>
__global__ __launch_bounds__(64 * (WAVES + 1)) void gemm_stream_kernel(const u32x2 *offsets, const uint8_t *bitmaps,
                                                                  const uint8_t *H, const uint8_t *L, uint32_t q,
                                                                  uint32_t r, uint32_t parts, uint32_t k_blocks,
                                                                  uint32_t magic_k, StreamArgs)
{
    BlobView bv = {bitmaps, offsets, H, L, 0u, 0u, 0u, 0u, 0, (int32_t)k_blocks, 0}; // (the rest below)
    const Divider by_k = {k_blocks, magic_k};
    using S = Slot<LW>;
    using Lds = StreamLds<MT, LW, WAVES>;
    constexpr int DEPTH = Lds::kDepth;
    // LDS after the tables: accumulation tiles (16 MT tokens x 64 rows, FP32, in units of
    // float4 = 4 consecutive rows; unit (m, c) lives at m * 16 + (c ^ (m & 15)) so that the 16
    // tokens of one MFMA result hit 16 different bank groups), the control words, the rings.
    constexpr uint32_t kUnits = Lds::kUnits, kTileBytes = Lds::kTileBytes;
    static_assert(Lds::kRings == Lds::kCtl + kCtlBytes, "control block size");
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    const uint32_t lane = threadIdx.x & 63u, wave = uniform(threadIdx.x >> 6);
    const uint32_t tab = dynamic_lds_base();
    const uint32_t red = tab + Lds::kRed, ctl = tab + Lds::kCtl;
    // the last byte any wave's ring can reach is Lds::kTotal, which is what the host requests
    const uint32_t rings = tab + Lds::kRings, ring = rings + wave * Lds::kRingBytes;
    const uint32_t m_lane = lane & 15u, kgrp = lane >> 4;
    // this workgroup's range [g0, g1) of the BlockTile sequence and its tasks
    // Workgroups are dealt out to the chip's eight dies round-robin (workgroup b runs on die
    // b % 8).  Neighbouring ranges share a strip and exchange partial tiles, so a die takes a
    // run of consecutive ranges; a bijection on [0, parts) whenever 8 divides the grid.
    const uint32_t range_id = (parts & 7u) == 0 ? (blockIdx.x & 7u) * (parts >> 3) + (blockIdx.x >> 3) : blockIdx.x;
    RangeSplit rs = {0u, parts, q, r, 0u, 0u}; // (the total is not needed here, the magic numbers are loaded at the end)
    const uint32_t g0 = rs.begin(range_id), g1 = rs.begin(range_id + 1);
    const uint32_t strip0 = by_k(g0);
    if (g0 >= g1) return;
    // Processing order: a range that touches several strips starts with its last one and then
    // runs from its beginning.  The (possibly shared) strips at both ends of the range are
    // then finished early, and what shared strips cost on top (parking the partial tile in
    // global memory, counting in, summing up) overlaps with the remaining work instead of
    // standing at the end of the kernel.  Tasks are numbered in processing order; the counter
    // that hands out BlockTiles counts positions c = 0 .. g1 - g0 - 1 in that order.
    const uint32_t strip_last = by_k(g1 - 1), n_tasks = strip_last - strip0 + 1;
    const uint32_t rot = n_tasks > 1 ? g1 - strip_last * k_blocks : 0u; // BlockTiles taken before g0
    auto task_strip = [&](uint32_t j) { return rot ? (j ? strip0 + j - 1 : strip_last) : strip0 + j; };

    // ---- issuing side: takes the next BlockTile off the shared counter and looks up its offsets.
    // The counter hands out positions c = 0 .. g1 - g0 - 1 in processing order; positions below
    // rot lie in the range's last strip (task 0), the others count from g0.
    const uint32_t n_pos = g1 - g0, first_a = strip_last * k_blocks, first_b = g0 - rot;
    uint32_t it_j = rot ? 1u : 0u, it_base = strip0 * k_blocks; // task and first BlockTile of the strip the counter is in
    uint32_t p_valid = 0;                                       // the next BlockTile to issue ... (0 / 1: plain scalars)
    uint32_t p_j = 0, p_kb = 0;
    TileRef p_t = {kNoTileG, kNoTileOff};
    // Taking the next BlockTile is spread over two points of a step so that neither the LDS
    // atomic nor the scalar load is waited for where it is issued.
    uint32_t g_taken = 0; // (per lane) what the counter returned
    auto take_begin = [&]() {
        g_taken = 0;
        if (lane == 0)
            g_taken = __hip_atomic_fetch_add((LdsU32)(ctl + kCtlNext), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    };
    auto take_lookup = [&]() {
        const uint32_t c = uniform(g_taken);
        p_valid = (c - n_pos) >> 31; // c < n_pos (both below 2^31), kept a number in a scalar register
        p_t = TileRef{kNoTileG, kNoTileOff};
        if (p_valid) {
            if (c < rot) { // the range's last strip, task 0
                p_t.g = first_a + c, p_j = 0, p_kb = c;
            } else {
                const uint32_t g = first_b + c;
                while (g - it_base >= k_blocks) it_base += k_blocks, ++it_j;
                p_t.g = g, p_j = it_j, p_kb = g - it_base;
            }
            p_t.off = offset_quad(bv, p_t.g);
        }
    };
    // what the decoding side needs to know about a staged tile, per ring position (wave-uniform)
    uint32_t s_valid[DEPTH], s_j[DEPTH], s_kb[DEPTH];
    StagedL s_l[DEPTH];
#pragma unroll
    for (int d = 0; d < DEPTH; ++d) s_valid[d] = 0, s_j[d] = 0, s_kb[d] = 0, s_l[d] = StagedL{bv.L, 0u};
    // Issues the LDS-direct loads of the pending tile into ring position d.
    auto stage = [&](int d) {
        s_l[d] = stage_tile<LW>(bv, p_t, ring + d * S::kBytes, lane);
        s_valid[d] = p_valid, s_j[d] = p_j, s_kb[d] = p_valid ? p_kb : 0u;
    };

    // The first BlockTile of every streaming wave is assigned statically (position = wave) and
    // staged before anything else: its loads are in flight while the tables are built.
    if (wave < WAVES) {
        g_taken = wave;
        take_lookup();
    }
    typedef const StreamArgs __attribute__((address_space(4))) *ConstArgs;
    ConstArgs in_memory = (ConstArgs)((uintptr_t)__builtin_amdgcn_kernarg_segment_ptr() + kStreamArgsAt);
    asm volatile("" : "+s"(in_memory)); // (not loaded before the offsets are asked for)
    const uint16_t *const A = in_memory->A;
    const int64_t lda = in_memory->lda;
    bv.h_units = in_memory->h_units, bv.l_units = in_memory->l_units;
    bv.h_fast = in_memory->h_fast, bv.l_fast = in_memory->l_fast, bv.base_exp = in_memory->base_exp;
    if (wave < WAVES) stage(0);
    // B operand of the 16x16x32 MFMA: lane l holds token l % 16 and the 8 consecutive k that
    // start at 8 * (l / 16).  Tokens >= M read token 0 instead (their columns are never stored).
    uint32_t rowoff[MT];
#pragma unroll
    for (int j = 0; j < MT; ++j) {
        const uint32_t m = j * 16 + m_lane;
        rowoff[j] = ((int)m < in_memory->M ? m : 0u) * (uint32_t)lda * 2u + kgrp * 16u;
    }

    build_tables(smem, bv.base_exp);
    constexpr uint32_t kClear = Lds::kOwnTiles ? 0 : 2 * kTileBytes; // (tiles of their own are written before they are read)
    for (uint32_t i = threadIdx.x; i < (kClear + kCtlBytes) / 4; i += blockDim.x)
        *((LdsU32)(ctl - kClear + 4 * i)) = i == (kClear + kCtlNext) / 4 ? (uint32_t)WAVES : 0u;
    __syncthreads();

    // ---- results
    constexpr uint32_t kRows = kUnits / 64;                // rows of 64 float4 units (four tokens each) of a tile
    // What only results need: loaded where they start (results_begin), so that the streaming loop does not hold it.
    float *C;
    int64_t ldc;
    int M;
    SharedSums ws;
    uint32_t rows; // rows that hold tokens
    __amdgpu_buffer_rsrc_t slots;
    auto results_begin = [&]() {
        ConstArgs again = in_memory;
        asm volatile("" : "+s"(again));
        C = again->C, ldc = again->ldc, M = again->M;
        ws = SharedSums{again->ws.count, again->ws.tiles, again->ws.mode, again->ws.out_bf16, again->ws.tiles_bytes};
        rows = min(((uint32_t)M + 3u) / 4u, kRows);
        slots = __builtin_amdgcn_make_buffer_rsrc(ws.tiles, 0, (int)ws.tiles_bytes, 0x00020000);
    };
    auto task_tiles = [&](uint32_t strip) -> uint32_t { return min(g1, (strip + 1) * k_blocks) - max(g0, strip * k_blocks); };
    // [first, last] contributing workgroup of a strip that this range holds only a part of
    auto contributors = [&](uint32_t strip, uint32_t &b_lo, uint32_t &b_hi) {
        if (task_tiles(strip) == k_blocks) return false;
        ConstArgs again = in_memory;
        asm volatile("" : "+s"(again)); // (not held in registers through the launch)
        rs.magic_q = again->magic_q, rs.magic_q1 = again->magic_q1;
        b_lo = rs.of(strip * k_blocks), b_hi = rs.of((strip + 1) * k_blocks - 1);
        return true;
    };
    // Per-lane addresses are formed where they are used, from a copy of the lane number the
    // compiler cannot see through: hoisted out of the task loop they would all stay in
    // registers for the whole loop.
    auto opaque_lane = [&]() {
        uint32_t l = lane;
        asm volatile("" : "+v"(l));
        return l;
    };
    // LDS address of float4 unit 64 q + l of a tile: token 4 q + l / 16, rows 4 (l % 16) .. + 3 of the strip
    auto unit_at = [&](uint32_t tile, uint32_t q, uint32_t l) {
        const uint32_t m = 4 * q + (l >> 4);
        return tile + 16 * (m * 16 + ((l & 15u) ^ (m & 15u)));
    };
    auto store_row = [&](uint32_t strip, uint32_t q, uint32_t l, const f32x4 &v) {
        const uint32_t m = 4 * q + (l >> 4);
        const int64_t at = (int64_t)m * ldc + (int64_t)strip * 64 + 4 * (l & 15u);
        if ((int)m >= M) return;
        if (ws.out_bf16) // the same unit as four BF16: 8 bytes at the same element offset
            *reinterpret_cast<u32x2 *>(reinterpret_cast<uint16_t *>(C) + at) =
                u32x2{bf16_rne(v.x) | (bf16_rne(v.y) << 16), bf16_rne(v.z) | (bf16_rne(v.w) << 16)};
        else
            *reinterpret_cast<f32x4 *>(C + at) = v;
    };
    auto add_row = [&](uint32_t strip, uint32_t q, uint32_t l, const f32x4 &v) { // kSumCleared
        const uint32_t m = 4 * q + (l >> 4);
        if ((int)m < M)
#pragma unroll
            for (int i = 0; i < 4; ++i) unsafeAtomicAdd(C + (int64_t)m * ldc + (int64_t)strip * 64 + 4 * (l & 15u) + i, v[i]);
    };
    // kSumParked.  Every contributor parks its partial tile in its slot of the scratch buffer and
    // counts itself in; whoever counted last adds the tiles up, in the order of the workgroups, and
    // stores the strip.  A slot word is its own "arrived" flag: slots are all zero bits between launches, a
    // parked +0.0 is written as -0.0 (which adds the same), and the last contributor reads a slot
    // until none of its words is zero, then zeroes it again.  So nothing orders the tile stores
    // against the counter.  The slots are accessed through a buffer descriptor over the slot area: 16-byte
    // loads and stores that the compiler issues and waits for itself, that carry the
    // sc1 bit like the agent-scope atomics on the counter (coherent between the L2s of
    // the chip's dies without cache-wide write-backs or invalidations), and that the
    // hardware checks against the size of the area (an out-of-range read returns zero,
    // an out-of-range write is dropped).  "Volatile": the polling reads must be repeated.
    // Stores have the whole offset in the lanes' registers (store_unit): a store of more than eight bytes a lane still
    // reads its data while the next instructions issue, and the compiler keeps the two wait states before a
    // vector instruction overwrites them, except behind a buffer store with a scalar register as offset, where it
    // keeps none.  A word parked by such a store was seen lost; how many that form needs is not known, so it is not used.
    constexpr int kCoherent = 16 | (int)0x80000000u; // sc1 | volatile (compiler-level)
    auto store_unit = [&](const u32x4 &w, uint32_t at) { __builtin_amdgcn_raw_buffer_store_b128(w, slots, at, 0, kCoherent); };
    // byte offset of the slot of workgroup b for this strip: slot 0 of a workgroup holds
    // the strip its range starts in, slot 1 the one it ends in
    auto slot_of = [&](uint32_t strip, uint32_t b) {
        const uint32_t first = rs.begin(b) >= strip * k_blocks ? 0u : 1u;
        return uniform((2 * b + first) * kTileBytes);
    };
    // the same for a contributor b of [b_lo, b_hi] (all but the first start inside the strip)
    auto contributor_slot = [&](uint32_t slot_lo, uint32_t b_lo, uint32_t b) { return b == b_lo ? slot_lo : uniform(2 * b * kTileBytes); };
    auto park_row = [&](uint32_t strip, uint32_t q, uint32_t l, const f32x4 &v) {
        u32x4 w = __builtin_bit_cast(u32x4, v);
        w.x = w.x ? w.x : 0x80000000u, w.y = w.y ? w.y : 0x80000000u;
        w.z = w.z ? w.z : 0x80000000u, w.w = w.w ? w.w : 0x80000000u;
        store_unit(w, l * 16 + (slot_of(strip, range_id) + q * 1024));
    };
    // Partial rows in flight: ROWS rows from row q on, of CNT contributors from workgroup b on (the last one
    // again where there are fewer: a load that is made or not would be waited for by itself).
    auto request_rows = [&](auto &t, uint32_t slot_lo, uint32_t b_lo, uint32_t q, uint32_t l, uint32_t b, uint32_t b_hi) {
        constexpr uint32_t ROWS = sizeof(t) / sizeof(t[0]), CNT = sizeof(t[0]) / 16;
#pragma unroll
        for (uint32_t i = 0; i < CNT; ++i) {
            const uint32_t slot = contributor_slot(slot_lo, b_lo, min(b + i, b_hi)) + q * 1024;
#pragma unroll
            for (uint32_t r = 0; r < ROWS; ++r) t[r][i] = __builtin_amdgcn_raw_buffer_load_b128(slots, l * 16, slot + r * 1024, kCoherent);
        }
    };
    // Waits for the requested rows, adds them up and clears their slots.  A parked row arrives within a round
    // trip of its owner's count.  The bound only matters when the scratch contract was broken (a buffer
    // that was not zero-filled once, or calls overlapping on it): then this gives up and the strip is wrong.
    // (Rows beyond the last one with tokens are not parked: they are neither waited for nor cleared.)
    auto take_rows = [&](auto &t, auto &sum, uint32_t slot_lo, uint32_t b_lo, uint32_t q, uint32_t l, uint32_t b, uint32_t b_hi) {
        constexpr uint32_t ROWS = sizeof(t) / sizeof(t[0]), CNT = sizeof(t[0]) / 16;
        for (uint32_t polls = 0;; ++polls) {
            bool missing = false;
#pragma unroll
            for (uint32_t i = 0; i < CNT; ++i)
#pragma unroll
                for (uint32_t r = 0; r < ROWS; ++r)
                    missing |= (r == 0 || q + r < rows) && (t[r][i].x == 0u || t[r][i].y == 0u || t[r][i].z == 0u || t[r][i].w == 0u);
            if (__builtin_amdgcn_ballot_w64(missing) == 0 || polls == (1u << 15)) break;
            __builtin_amdgcn_s_sleep(1);
            request_rows(t, slot_lo, b_lo, q, l, b, b_hi);
        }
        u32x4 zero4 = {0u, 0u, 0u, 0u};
        asm volatile("" : "+v"(zero4)); // (formed here: held through the writer's loop it does not fit the registers)
#pragma unroll
        for (uint32_t i = 0; i < CNT; ++i)
            if (b + i <= b_hi) {
                const uint32_t slot = contributor_slot(slot_lo, b_lo, b + i) + q * 1024;
#pragma unroll
                for (uint32_t r = 0; r < ROWS; ++r) {
                    sum[r] += __builtin_bit_cast(f32x4, t[r][i]);
                    // (same address as the load above, same wave: stays behind it)
                    if (r == 0 || q + r < rows) store_unit(zero4, l * 16 + (slot + r * 1024));
                }
            }
    };
    // Adds up and stores rows q .. of a strip; the first batch of them is in t.
    auto finish_rows = [&](auto &t, uint32_t strip, uint32_t slot_lo, uint32_t q, uint32_t l, uint32_t b_lo, uint32_t b_hi) {
        constexpr uint32_t ROWS = sizeof(t) / sizeof(t[0]), CNT = sizeof(t[0]) / 16;
        f32x4 sum[ROWS] = {};
        for (uint32_t b = b_lo;;) {
            take_rows(t, sum, slot_lo, b_lo, q, l, b, b_hi);
            b += CNT;
            if (b > b_hi) break;
            request_rows(t, slot_lo, b_lo, q, l, b, b_hi);
        }
#pragma unroll
        for (uint32_t r = 0; r < ROWS; ++r) store_row(strip, q + r, l, sum[r]); // (stores tokens below M only)
    };
    auto count_in = [&](uint32_t b_lo) {
        uint32_t old = 0;
        if (lane == 0) old = __hip_atomic_fetch_add(ws.count + b_lo, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return old;
    };
    auto reset_count = [&](uint32_t b_lo) {
        if (lane == 0) __hip_atomic_store(ws.count + b_lo, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };

    // The last task of the range.  Every streaming wave has left its sums in its own ring and counted itself
    // in; then they add up rows of them, so that what stands between the last BlockTile and the
    // end of the launch is the count, one round trip to the other contributors' rows, all at a time, and the
    // stores.  With the sums under a lock in one tile and one wave for the exchange that took 6 us of 15.8 at 32
    // tokens on 4096 x 4096 (now 3.3 of 12.9), 8.2 of 30.3 on 4096 x 14336 (now 5.4 of 27.3), 5.1 of 9.7 at one
    // token on 1024 x 4096 (3.4 of 8.0): medians of the last BlockTile's end to the launch's.  Reading the
    // rows before the count is known saves no round trip (the rows are not there yet) and costs traffic: 14.0 -> 12.7 us
    // at 16 tokens on 4096 x 4096 without.
    auto finish_last_task = [&]() {
        constexpr uint32_t kAtATime = MT; // rows to a wave, so that one round serves up to 16 MT tokens with four waves
        const uint32_t strip = task_strip(n_tasks - 1), q0 = wave * kAtATime;
        if (q0 >= rows) return; // (one wave at least stays: wave 0)
        uint32_t b_lo = 0, b_hi = 0; // (before the wait, which hides it)
        const bool shared = contributors(strip, b_lo, b_hi), parked = shared && ws.mode == kSumParked;
        while (uniform(lds_poll(ctl + kCtlArrived)) != (uint32_t)WAVES) __builtin_amdgcn_s_sleep(1);
        asm volatile("" ::: "memory");
        const uint32_t l = opaque_lane();
#pragma unroll
        for (uint32_t r = 0; r < kAtATime; ++r) {
            const uint32_t q = q0 + r;
            if (r && q >= rows) break;
            f32x4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (uint32_t w = 0; w < (uint32_t)WAVES; ++w) v += *((LdsF32x4)(unit_at(rings, q, l) + w * Lds::kRingBytes));
            if (parked) park_row(strip, q, l, v);
            else if (shared) add_row(strip, q, l, v);
            else store_row(strip, q, l, v);
        }
        if (!parked) return;
        uint32_t old = 0;
        if (wave == 0) old = count_in(b_lo);
        if (wave == 0) {
            old = uniform(old);
            if (lane == 0) __hip_atomic_store((LdsU32)(ctl + kCtlCounted), old + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        } else {
            while ((old = uniform(lds_poll(ctl + kCtlCounted))) == 0) __builtin_amdgcn_s_sleep(1);
            --old;
        }
        if (old != b_hi - b_lo) return; // somebody else finishes the strip
        auto collect = [&](auto count) {
            u32x4 t[kAtATime][decltype(count)::value];
            const uint32_t slot_lo = slot_of(strip, b_lo);
            request_rows(t, slot_lo, b_lo, q0, l, b_lo, b_hi);
            finish_rows(t, strip, slot_lo, q0, l, b_lo, b_hi);
        };
        // From five contributors on 16 / MT at a time, us, four always / so: 1024 x 4096, one token 9.0 / 8.2, 32 tokens 11.7 /
        // 11.3; 1024 x 14336, 16 tokens 13.3 / 12.4, 32 tokens 15.7 / 15.3 (sixteen contributors and more; with two to four no difference).
        if (16 / MT == 4 || b_hi - b_lo < 4) collect(std::integral_constant<int, 4>{});
        else collect(std::integral_constant<int, 16 / MT>{});
        if (wave == 0) reset_count(b_lo);
    };

    // ---- the last wave of the workgroup only writes results.  Stores count in the same
    //      vector-memory counter as the LDS-direct loads, and a store is acknowledged late while
    //      HBM is saturated with reads; a streaming wave that stored would stall its own pipeline.
    if (wave == WAVES) {
        results_begin();
        for (uint32_t j = 0; j + 1 < n_tasks; ++j) {
            const uint32_t strip = task_strip(j), par = j & 1u, n = task_tiles(strip);
            while (uniform(lds_poll(ctl + kCtlDone + 4 * par)) != n) __builtin_amdgcn_s_sleep(2);
            lds_fence();
            f32x4 v[kRows];
            const uint32_t l = opaque_lane();
            if constexpr (Lds::kOwnTiles) {
                const uint32_t from = uniform(lds_poll(ctl + kCtlFrom + 4 * par)); // waves that have sums of this task
#pragma unroll
                for (uint32_t q = 0; q < kRows; ++q) v[q] = f32x4{0.f, 0.f, 0.f, 0.f};
                for (uint32_t w = 0; w < (uint32_t)WAVES; ++w)
                    if ((from >> w) & 1u)
#pragma unroll
                        for (uint32_t q = 0; q < kRows; ++q) v[q] += *((LdsF32x4)(unit_at(red, q, l) + w * kTileBytes));
                if (lane == 0)
                    __hip_atomic_store((LdsU32)(ctl + kCtlFrom + 4 * par), 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            } else {
#pragma unroll
                for (uint32_t q = 0; q < kRows; ++q) {
                    const LdsF32x4 at = (LdsF32x4)unit_at(red + par * kTileBytes, q, l);
                    v[q] = *at;
                    *at = f32x4{0.f, 0.f, 0.f, 0.f};
                }
            }
            lds_fence(); // the sums are read, and the tile cleared: hand it back
            if (lane == 0) {
                __hip_atomic_store((LdsU32)(ctl + kCtlDone + 4 * par), 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                lds_fence();
                __hip_atomic_store((LdsU32)(ctl + kCtlWritten), j + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            }
            uint32_t b_lo = 0, b_hi = 0;
            const bool shared = contributors(strip, b_lo, b_hi), parked = shared && ws.mode == kSumParked;
#pragma unroll
            for (uint32_t q = 0; q < kRows; ++q)
                if (q < rows) {
                    if (parked) park_row(strip, q, l, v[q]);
                    else if (shared) add_row(strip, q, l, v[q]); // (the host's clear kernel zeroed the columns before)
                    else store_row(strip, q, l, v[q]);
                }
            if (!parked) continue;
            const uint32_t old = count_in(b_lo);
            u32x4 t[4][4];
            if (uniform(old) != b_hi - b_lo) continue; // somebody else finishes the strip
            const uint32_t slot_lo = slot_of(strip, b_lo);
            request_rows(t, slot_lo, b_lo, 0, l, b_lo, b_hi);
            for (uint32_t q = 0;;) {
                finish_rows(t, strip, slot_lo, q, l, b_lo, b_hi);
                q += 4;
                if (q >= rows) break;
                request_rows(t, slot_lo, b_lo, q, l, b_lo, b_hi);
            }
            reset_count(b_lo);
        }
    } else {

    f32x4 acc[4][MT];
    auto clear_acc = [&]() {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < MT; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    };
    // LDS address of the lane's float4 unit of a tile for 16-row block i and token block jj.  D layout of
    // the 16x16 MFMA: a lane holds token lane % 16 and rows 4 * (lane / 16) .. + 3 of the 16-row block.
    // Formed where it is used, from a copy of the lane number the compiler cannot see through: hoisted
    // out of the tile loop the addresses would hold 4 MT + 1 registers for good.
    auto result_at = [&](uint32_t tile, uint32_t l, int i, int jj) {
        const uint32_t m = jj * 16 + (l & 15u), c = i * 4 + (l >> 4);
        return (LdsF32x4)(tile + 16 * (m * 16 + (c ^ (m & 15u))));
    };
    // Hands the partial sums of n BlockTiles of task j, not the range's last one, to the writer: in the wave's own
    // tile, or added to the task's tile under a lock.
    uint32_t handed = 0; // 1 + the task whose sums were last left in the wave's own tile
    auto flush = [&](uint32_t j, uint32_t n) {
        const uint32_t par = j & 1u;
        // the tile may still hold sums that the writer has not taken: wait until it has handed it back
        // (and be not more than two tasks ahead of it, whose counts go by turns)
        while ((int32_t)uniform(lds_poll(ctl + kCtlWritten)) < max((int32_t)j - 1, (int32_t)handed)) __builtin_amdgcn_s_sleep(2);
        if constexpr (!Lds::kOwnTiles)
            for (;;) {
                uint32_t old = 1;
                if (lane == 0) {
                    uint32_t expect = 0;
                    __hip_atomic_compare_exchange_strong((LdsU32)(ctl + kCtlLock + 4 * par), &expect, 1u, __ATOMIC_RELAXED,
                                                         __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                    old = expect;
                }
                if (uniform(old) == 0) break;
                __builtin_amdgcn_s_sleep(1);
            }
        lds_fence();
        const uint32_t l = opaque_lane();
#pragma unroll
        for (int jj = 0; jj < MT; ++jj) {
            const uint32_t tile = red + (Lds::kOwnTiles ? wave : par) * kTileBytes;
            f32x4 sum[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) sum[i] = acc[i][jj];
            if constexpr (!Lds::kOwnTiles) {
                // Four units read before the first is written: a quarter of the LDS round trips under the lock, for which
                // the other waves queue.  6144 x 4096, 50 tokens 26.5 -> 24.4 us, row-scaled, 64 tokens 29.9 -> 26.4; 28672 x
                // 4096, 50 tokens 53.1 -> 51.8.  LDS float additions without a lock are no way: 57.8 and 115.6 us.
                f32x4 old[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) old[i] = *result_at(tile, l, i, jj);
#pragma unroll
                for (int i = 0; i < 4; ++i) sum[i] += old[i];
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) *result_at(tile, l, i, jj) = sum[i];
        }
        lds_fence(); // sums written before the lock opens and the count rises
        if (lane == 0) {
            if constexpr (Lds::kOwnTiles) {
                __hip_atomic_fetch_or((LdsU32)(ctl + kCtlFrom + 4 * par), 1u << wave, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                lds_fence();
            } else {
                __hip_atomic_store((LdsU32)(ctl + kCtlLock + 4 * par), 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            }
            __hip_atomic_fetch_add((LdsU32)(ctl + kCtlDone + 4 * par), n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
        if (Lds::kOwnTiles) handed = j + 1;
    };

    take_begin();
    take_lookup();
    clear_acc();
    uint32_t acc_j = s_j[0], acc_n = 0;

    // Activation fragments (B operands) of the tile about to be decoded: requested at the top
    // of its step, before the LDS-direct loads of the next tile, and awaited right before the
    // first MFMA, so the L2 round trip is covered by the staging and indexing in between.  The
    // compiler cannot count the LDS-direct loads, so it cannot place that wait: the loads are
    // issued by hand and awaited with vmcnt(S::kLoads), the number of vector-memory
    // instructions every step issues after them.  The fragment registers are operands of the
    // wait, so nothing that uses them can move above it.
    auto request_fragments = [&](uint32_t kb, u32x4 (&f)[2][MT]) {
        const uint16_t *src = A + (size_t)kb * 64;
#pragma unroll
        for (int kh = 0; kh < 2; ++kh)
#pragma unroll
            for (int j = 0; j < MT; ++j)
                asm volatile("global_load_dwordx4 %0, %1, %2 offset:%3" : "=v"(f[kh][j]) : "v"(rowoff[j]), "s"(src), "n"(64 * kh));
    };
    auto fragments_arrived = [&](u32x4 (&f)[2][MT]) {
        static_assert(MT == 1 || MT == 2 || MT == 4, "the wait below names every fragment register");
        if constexpr (MT == 1)
            asm volatile("s_waitcnt vmcnt(%2)" : "+v"(f[0][0]), "+v"(f[1][0]) : "n"(S::kLoads));
        else if constexpr (MT == 2)
            asm volatile("s_waitcnt vmcnt(%4)" : "+v"(f[0][0]), "+v"(f[0][1]), "+v"(f[1][0]), "+v"(f[1][1]) : "n"(S::kLoads));
        else
            asm volatile("s_waitcnt vmcnt(%8)"
                         : "+v"(f[0][0]), "+v"(f[0][1]), "+v"(f[0][2]), "+v"(f[0][3]), "+v"(f[1][0]), "+v"(f[1][1]),
                           "+v"(f[1][2]), "+v"(f[1][3])
                         : "n"(S::kLoads));
    };

    // per-lane addresses shared by both ring positions (the distance between the positions goes
    // into the offset fields of the reads)
    const uint32_t pa0 = plane_address(ring + S::kPlanes, lane);
    const uint32_t l_lane0 = l_lane_of(ring + S::kH, ring + S::kL, lane);

    // One iteration decodes the tile in ring position CUR while position CUR ^ 1 is refilled.
    auto step = [&](auto cur_c) {
        constexpr int CUR = decltype(cur_c)::value, NXT = CUR ^ 1;
        wait_dma<0>(); // tile CUR and its L window have landed
        lds_fence();   // all LDS reads of the slot to refill are done; the offsets of the next tile are here
        // the bit-plane bytes of tile CUR's first half are read while the next tile is staged
        HalfIndex h0;
        read_planes<CUR * S::kBytes, 0, false>(pa0, h0);
        u32x4 bfrag[2][MT];
        request_fragments(s_kb[CUR], bfrag);
        take_begin();
        stage(NXT); // (waits for the scalar load of the offsets, issued a tile ago)
        take_lookup();
        if (s_j[CUR] != acc_j) {
            flush(acc_j, acc_n);
            clear_acc();
            acc_j = s_j[CUR], acc_n = 0;
        }
        // L addresses are formed relative to ring position 0 (the distance, three times over,
        // is the constant kLX of the decode), so both positions share their per-lane registers
        const uint32_t slot = ring + CUR * S::kBytes;
        constexpr uint32_t kLX = 3 * CUR * S::kBytes;
        uint32_t h_base = slot + S::kH;
        index_half<true>(h_base, h0);
        const FallbackSource fs = {slot + S::kL, reinterpret_cast<const uint16_t *>(s_l[CUR].l), s_l[CUR].big != 0};
        fragments_arrived(bfrag);
        bf16x8 bop[2][MT];
#pragma unroll
        for (int kh = 0; kh < 2; ++kh)
#pragma unroll
            for (int j = 0; j < MT; ++j) {
                bop[kh][j] = __builtin_bit_cast(bf16x8, bfrag[kh][j]);
            }
        decode_block_tile<BASE_M1, CUR * S::kBytes, kLX, CAREFUL>(tab, pa0, h0, h_base, l_lane0, fs, [&](int tt, const u32x4 &w) {
            const bf16x8 wop = __builtin_bit_cast(bf16x8, w);
#pragma unroll
            for (int j = 0; j < MT; ++j)
                acc[tt & 3][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wop, bop[tt >> 2][j], acc[tt & 3][j], 0, 0, 0);
        });
        ++acc_n;
    };
    for (;;) {
        if (!s_valid[0]) break;
        step(std::integral_constant<int, 0>{});
        if (!s_valid[1]) break;
        step(std::integral_constant<int, 1>{});
    }
    if (acc_n && acc_j != n_tasks - 1) {
        flush(acc_j, acc_n);
        clear_acc();
    }
    // The last task's sums go to the wave's own ring (nothing is read there any more, and the loads
    // of "no tile" have landed), not under a lock: there the waves queued, 1.2 us at 16 tokens and 2.4 at 32.
    results_begin(); // (arrives while the sums are written)
    wait_dma<0>();
    const uint32_t l = opaque_lane();
#pragma unroll
    for (int jj = 0; jj < MT; ++jj)
#pragma unroll
        for (int i = 0; i < 4; ++i) *result_at(ring, l, i, jj) = acc[i][jj];
    lds_fence(); // sums written before the count rises
    if (lane == 0) __hip_atomic_fetch_add((LdsU32)(ctl + kCtlArrived), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    if (wave < (uint32_t)WAVES) finish_last_task();
}

// --------------------------------------------------------------------------------------
// ZipGEMM, wider M (up to 16 MT Q tokens per launch): producer and consumer waves.
//
// The decode cost of a BlockTile does not depend on M, so for more than a few tokens it is
// paid once per workgroup and shared: P producer waves stream and decode BlockTiles exactly
// as above but hand the decoded weights on, already in MFMA operand lane order, through a ring
// of R dense tiles in LDS (8 KB each); up to Q consumer waves, each owning 16 MT tokens,
// read every dense tile and run the MFMAs against their own activation fragments.  A token
// belongs to one consumer, so nothing is reduced across waves: a consumer stores (whole
// strip) or atomically adds (strip shared between workgroups) its registers when the strip
// changes.  Consumers issue no LDS-direct loads, so their global loads and stores are ordinary
// compiler-tracked ones.
//
// Work split and tile hand-out are those of gemm_stream_kernel.  Tile i of the workgroup's
// range lives in dense slot i % R.  ready[slot] = i + 1 once tile i is complete in LDS;
// consumed[slot] counts consumer passes over the slot.  A producer may write tile i when
// consumed[slot] has reached q_active * (i / R); a consumer reads tile i when ready[slot] is
// i + 1, and still holds slot (i - 1) % R while it waits for that, so R is at least 2.  Tiles
// are handed out in order and a producer waits for the consumption of an earlier tile than its
// own, so the smallest unfinished tile can always complete.
//
// A producer decodes into registers and claims its dense slot only to write the finished tile:
// were the slot held for the whole decode, R slots would allow R tiles in all the stages from
// decode to consumption, fewer than there are producers plus consumers' backlog.
// --------------------------------------------------------------------------------------

// acc[j] += frag[j] * w for the MT token blocks of a consumer, in place.  Written out because the
// compiler's own MFMAs write to other registers than they add to: 153 registers with 32 tokens to a
// consumer where sixteen waves have 128 each.  The leading s_nop covers an operand that a vector
// instruction has just written (two wait states); an accumulator is next touched by the MFMAs of the
// next half tile, or after accumulators_done().
template <int MT>
__device__ __forceinline__ void mfma_rows(f32x4 (&acc)[MT], const u32x4 (&frag)[MT], const u32x4 &w)
{
    static_assert(MT == 1 || MT == 2, "operands below");
#define ZS_MFMA(I, A, W) "v_mfma_f32_16x16x32_bf16 %" #I ", %" #A ", %" #W ", %" #I "\n\t"
    if constexpr (MT == 1)
        asm volatile("s_nop 1\n\t" ZS_MFMA(0, 1, 2) : "+v"(acc[0]) : "v"(frag[0]), "v"(w));
    else
        asm volatile("s_nop 1\n\t" ZS_MFMA(0, 2, 4) ZS_MFMA(1, 3, 4) : "+v"(acc[0]), "+v"(acc[1]) : "v"(frag[0]), "v"(frag[1]), "v"(w));
#undef ZS_MFMA
}
// Before anything but an MFMA reads or writes accumulators: the last MFMA's four passes plus the write
// are over (sixteen wait states, seven are needed).
template <int MT>
__device__ __forceinline__ void accumulators_done(f32x4 (&acc)[4][MT])
{
#pragma unroll
    for (int j = 0; j < MT; ++j)
        asm volatile("s_nop 15" : "+v"(acc[0][j]), "+v"(acc[1][j]), "+v"(acc[2][j]), "+v"(acc[3][j]));
}
enum : uint32_t { kPcNext = 0, kPcReady = 64, kPcConsumed = 128, kPcCtlBytes = 192, kDenseBytes = 8192 };

template <int MT, int LW, int P, int R, int Q, int F, bool BASE_M1, Fallbacks CAREFUL>
__global__ __launch_bounds__(64 * (P + Q)) void gemm_pc_kernel(BlobView bv, const uint16_t *A, int64_t lda,
                                                                          float *C, int64_t ldc, int M, int q_active,
                                                                          RangeSplit rs)
{
    static_assert(R >= 2 && R <= 16, "two slots at least (above); ready / consumed words are laid out for at most 16");
    using S = Slot<LW>;
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    build_tables(smem, bv.base_exp);

    const uint32_t lane = threadIdx.x & 63u, wave = uniform(threadIdx.x >> 6);
    const uint32_t tab = dynamic_lds_base();
    const uint32_t ctl = tab + kTableBytes, dense0 = ctl + kPcCtlBytes;

    const uint32_t k_blocks = (uint32_t)bv.k_blocks;
    // neighbouring ranges (which share strips, and slabs of A) on one die, as in gemm_stream_kernel
    const uint32_t range_id = (rs.parts & 7u) == 0 ? (blockIdx.x & 7u) * (rs.parts >> 3) + (blockIdx.x >> 3) : blockIdx.x;
    const uint32_t g0 = rs.begin(range_id), g1 = rs.begin(range_id + 1);

    for (uint32_t i = threadIdx.x; i < kPcCtlBytes / 4; i += blockDim.x) *((LdsU32)(ctl + 4 * i)) = i == kPcNext / 4 ? g0 : 0u;
    __syncthreads();
    if (g0 >= g1) return;
    const uint32_t n_tiles = g1 - g0;

    if (wave >= (uint32_t)P) {
        // ------------------------------------------------------------------ consumer
        // What bounds it: the L2 -> CU transfer of the activations (128 M bytes per BlockTile) from about
        // 200 tokens on, the decode below.  Nothing of a tile may be waited for when it is used, since a
        // chain of four LDS round trips per tile (poll, operands, fence, hand back) is longer than the
        // decode: operands are read a tile ahead, "ready" is polled a tile before it is looked at, a
        // slot is handed back without a fence, and the consumers' waves go first on their SIMD.
        // 4096 x 14336, 128 / 200 tokens: 61.5 / 88.1 -> 42.6 / 60 us; 28672 x 4096, 128 / 256: 93.7 / 161 -> 75 / 126 us.
        __builtin_amdgcn_s_setprio(2);
        const uint32_t c = wave - P;
        if ((int)c >= q_active) return;
        const uint32_t m_lane = lane & 15u, kgrp = lane >> 4;
        const uint32_t tok0 = c * 16u * MT;
        // A operand of the 16x16x32 MFMA: lane l holds token l % 16 and the 8 consecutive k that
        // start at 8 * (l / 16).  Tokens >= M read token 0 instead (their rows are never stored).
        uint32_t rowoff[MT];
#pragma unroll
        for (int j = 0; j < MT; ++j) {
            const uint32_t m = tok0 + j * 16 + m_lane;
            rowoff[j] = ((int)m < M ? m : 0u) * (uint32_t)lda * 2u + kgrp * 16u;
        }
        // Through a buffer descriptor: per-lane row offset + uniform position in k, no address
        // arithmetic, and nothing is read beyond the last token's row.
        const __amdgpu_buffer_rsrc_t rows = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<uint16_t *>(A), 0, (int)(((uint32_t)M - 1u) * (uint32_t)lda * 2u + k_blocks * 128u), 0x00020000);
        // F = fragment buffers, one half tile (32 of the 64 k) each, requested F / 2 tiles before they are
        // used; both halves of a tile together, since they share the cache lines.  (Q = 8: 128 registers
        // per wave, room for two tiles' worth.)
        static_assert(F % 2 == 0 && F <= 6, "the loop below");
        u32x4 frag[F][MT];
        const uint32_t strip0 = g0 / k_blocks;
        uint32_t strip = strip0, kb = g0 - strip0 * k_blocks; // of the tile being consumed
        // k block of the half whose fragments are requested next.  At the start nothing is asked for beyond
        // the range's end: a range of one or two tiles would wait behind it (always F halves / what there is:
        // 64 x 64, 256 tokens 7.9 / 6.5 us; 1024 x 1024, 128 tokens 14.9 / 14.1).  In the loop eight consumers keep to
        // that; four ask on (valid addresses: it wraps around with the strips), since the branch costs them more
        // than the loads (28672 x 4096, 96 tokens, with / without it 67.3 / 66.4 us; eight, 256 tokens, 126.8 / 127.5).
        uint32_t req_kb = kb;
        auto request = [&](int f, int kh) {
#pragma unroll
            for (int j = 0; j < MT; ++j) frag[f][j] = __builtin_amdgcn_raw_buffer_load_b128(rows, rowoff[j], req_kb * 128 + 64 * kh, 0);
            if (kh == 1) req_kb = req_kb + 1 == k_blocks ? 0u : req_kb + 1;
        };
        f32x4 acc[4][MT];
        auto clear_acc = [&]() {
#pragma unroll
            for (int j = 0; j < MT; ++j)
#pragma unroll
                for (int i = 0; i < 4; ++i) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
        };
        clear_acc();
#pragma unroll
        for (int f = 0; f < F; ++f)
            if (f < 2 || (uint32_t)(f / 2) < n_tiles) request(f, f & 1);

        uint32_t slot = 0, i = 0, in_strip = 0; // tile being consumed, tiles of its strip consumed so far
        // Decoded weights: each operand of the next tile is read as soon as the MFMAs of this tile's are issued.
        u32x4 w[8];
        auto poll_ready = [&](uint32_t sl) { return lds_poll(ctl + kPcReady + 4 * sl); };
        auto wait_ready = [&](uint32_t seen, uint32_t tile, uint32_t sl) {
            while (uniform(seen) != tile + 1) {
                __builtin_amdgcn_s_sleep(1);
                seen = poll_ready(sl);
            }
            asm volatile("" ::: "memory");
        };
        auto read_weight = [&](int t, uint32_t at) { w[t % 8] = *((const __attribute__((address_space(3))) u32x4 *)(at + t * 1024)); };
        auto address = [&](uint32_t sl) { return dense0 + sl * kDenseBytes + lane * 16; };
        wait_ready(poll_ready(0), 0, 0);
#pragma unroll
        for (int t = 0; t < 8; ++t) read_weight(t, address(0));
        uint32_t seen = poll_ready(1 % R);
        auto consume = [&](auto f_c) { // buffer of the tile's first half
            constexpr int f0 = decltype(f_c)::value, f1 = f0 + 1;
            const uint32_t slot_next = slot + 1 == (uint32_t)R ? 0u : slot + 1;
            const uint32_t at_next = address(slot_next);
            if (i + 1 < n_tiles) wait_ready(seen, i + 1, slot_next);
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                __builtin_amdgcn_sched_barrier(0);
                mfma_rows<MT>(acc[t & 3], frag[t < 4 ? f0 : f1], w[t]);
                __builtin_amdgcn_sched_barrier(0);
                read_weight(t, at_next); // (after the last tile: bytes that nobody uses)
            }
            // every operand of the tile has been in an MFMA, so the slot has been read: hand it back, and ask
            // for the state of the tile after the next one (looked at a tile later)
            asm volatile("" ::: "memory");
            if (lane == 0)
                __hip_atomic_fetch_add((LdsU32)(ctl + kPcConsumed + 4 * slot), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            seen = poll_ready(slot_next + 1 == (uint32_t)R ? 0u : slot_next + 1);
            if (Q <= 4 || i + F / 2 < n_tiles) { // (see req_kb)
                request(f0, 0); // the halves F further on; both at once: they share the cache lines
                request(f1, 1);
            }
            ++in_strip;
            const bool last_of_strip = kb + 1 == k_blocks;
            if (last_of_strip || i + 1 == n_tiles) {
                // D layout of the 16x16 MFMA with the activations as A operand: a lane holds feature
                // lane % 16 and tokens 4 * (lane / 16) .. + 3, so that the 64 lanes of a store or an
                // atomic cover four runs of 64 bytes (with the operands the other way round an
                // atomic touches 16 rows, four words each)
                // (one per-lane offset, formed here from a copy of the lane number the compiler cannot
                // see through, and uniform rows: as per-lane row addresses they do not fit the registers)
                const bool whole = in_strip == k_blocks;
                accumulators_done<MT>(acc);
                uint32_t l = lane;
                asm volatile("" : "+v"(l));
                const int64_t lane_at = (int64_t)(4 * (l >> 4)) * ldc + (l & 15u);
                float *row0 = C + (int64_t)tok0 * ldc + (int64_t)strip * 64;
#pragma unroll
                for (int j = 0; j < MT; ++j)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        __builtin_amdgcn_sched_barrier(0);
                        float *dst = row0 + (int64_t)(j * 16 + e) * ldc + lane_at;
                        if ((int)(tok0 + j * 16 + e + 4 * (l >> 4)) < M) {
#pragma unroll
                            for (int rb = 0; rb < 4; ++rb) {
                                if (whole) dst[16 * rb] = acc[rb][j][e];
                                else unsafeAtomicAdd(dst + 16 * rb, acc[rb][j][e]);
                            }
                        }
                    }
                clear_acc();
                in_strip = 0;
                ++strip;
            }
            kb = last_of_strip ? 0u : kb + 1;
            slot = slot_next;
            ++i;
        };
        for (;;) { // F is even: the buffers' roles repeat every F / 2 tiles
            if (i >= n_tiles) break;
            consume(std::integral_constant<int, 0>{});
            if constexpr (F > 2) {
                if (i >= n_tiles) break;
                consume(std::integral_constant<int, 2>{});
            }
            if constexpr (F > 4) {
                if (i >= n_tiles) break;
                consume(std::integral_constant<int, 4>{});
            }
        }
        return;
    }

    // ---------------------------------------------------------------------- producer
    const uint32_t ring = dense0 + R * kDenseBytes + wave * (2 * S::kBytes);
    bool p_valid = false;
    TileRef p_t = {kNoTileG, kNoTileOff};
    uint32_t g_taken = 0;
    auto take_begin = [&]() {
        g_taken = 0;
        if (lane == 0)
            g_taken = __hip_atomic_fetch_add((LdsU32)(ctl + kPcNext), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    };
    auto take_lookup = [&]() {
        const uint32_t g = uniform(g_taken);
        p_valid = g < g1;
        p_t = TileRef{kNoTileG, kNoTileOff};
        if (p_valid) {
            p_t.g = g;
            p_t.off = offset_quad(bv, g);
        }
    };
    bool s_valid[2] = {false, false};
    uint32_t s_i[2] = {0u, 0u};
    StagedL s_l[2] = {StagedL{bv.L, 0u}, StagedL{bv.L, 0u}};
    // Issues the Slot::kLoads LDS-direct loads of the pending tile into ring position d.
    auto stage = [&](int d) {
        s_l[d] = stage_tile<LW>(bv, p_t, ring + d * S::kBytes, lane);
        s_valid[d] = p_valid, s_i[d] = p_t.g - g0;
    };

    take_begin();
    take_lookup();
    stage(0);
    take_begin();
    take_lookup();

    auto step = [&](auto cur_c) {
        constexpr int CUR = decltype(cur_c)::value, NXT = CUR ^ 1;
        lds_fence(); // all LDS reads of the slot to refill are done
        stage(NXT);
        take_begin();
        wait_dma<S::kLoads>(); // everything older than the tile just staged has landed
        take_lookup();

        const uint32_t slot = ring + CUR * S::kBytes;
        HalfIndex h0;
        const uint32_t pa = plane_address(slot + S::kPlanes, lane);
        read_planes<0, 0, false>(pa, h0);
        uint32_t h_base = slot + S::kH;
        index_half<true>(h_base, h0);
        const FallbackSource fs = {slot + S::kL, reinterpret_cast<const uint16_t *>(s_l[CUR].l), s_l[CUR].big != 0};
        u32x4 dec[8];
        decode_block_tile<BASE_M1, 0, 0, CAREFUL>(tab, pa, h0, h_base, l_lane_of(slot + S::kH, slot + S::kL, lane), fs,
                                         [&](int tt, const u32x4 &w) { dec[tt] = w; });

        // the dense slot must have been read by every consumer before it is overwritten
        const uint32_t i = s_i[CUR], dslot = i % (uint32_t)R, need = (uint32_t)q_active * (i / (uint32_t)R);
        while ((int32_t)(uniform(lds_poll(ctl + kPcConsumed + 4 * dslot)) - need) < 0) __builtin_amdgcn_s_sleep(1);
        asm volatile("" ::: "memory"); // no write of the tile moves above the poll
        const uint32_t out = dense0 + dslot * kDenseBytes + lane * 16;
#pragma unroll
        for (int tt = 0; tt < 8; ++tt) *((__attribute__((address_space(3))) u32x4 *)(out + tt * 1024)) = dec[tt];
        lds_fence(); // the tile is complete in LDS before it is announced
        if (lane == 0)
            __hip_atomic_store((LdsU32)(ctl + kPcReady + 4 * dslot), i + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    };
    for (;;) {
        if (!s_valid[0]) break;
        step(std::integral_constant<int, 0>{});
        if (!s_valid[1]) break;
        step(std::integral_constant<int, 1>{});
    }
    wait_dma<0>();
}

// Clears the columns of C that belong to strips shared by several workgroups of the ZipGEMM
// launch that follows (they are summed with atomics).  The host lists those strips (a range
// boundary that is not a multiple of k_blocks cuts exactly one strip, so there are fewer than
// the number of workgroups); the list travels in the kernel arguments.  A thread stores 16 bytes, a
// workgroup 16 tokens of a strip: with one workgroup to a strip a thread stored up to sixteen times, one behind
// the other (1024 x 4096, 128 tokens 16.3 -> 15.7 us, 1024 x 1024 14.05 -> 13.55, 4096 x 14336, 200 tokens 60.7 -> 60.4).
constexpr int kMaxSharedStrips = 512;
struct SharedStrips {
    uint32_t n;
    uint32_t strip[kMaxSharedStrips];
};

__global__ void clear_shared_strips_kernel(float *C, int64_t ldc, int M, SharedStrips list)
{
    const uint32_t strip = list.strip[blockIdx.x], m = blockIdx.y * 16 + (threadIdx.x >> 4), c = threadIdx.x & 15u;
    if (m < (uint32_t)M) *reinterpret_cast<f32x4 *>(C + (int64_t)m * ldc + (int64_t)strip * 64 + 4 * c) = f32x4{0.f, 0.f, 0.f, 0.f};
}

// --------------------------------------------------------------------------------------
// Host side
// --------------------------------------------------------------------------------------
int make_view(const zs_desc *d, const void *blob, BlobView *bv)
{
    if (!d || !blob) return ZS_ERR_ARG;
    int rc = zs_desc_validate(d);
    if (rc != ZS_OK) return rc;
    if (reinterpret_cast<uintptr_t>(blob) % ZS_SECTION_ALIGN) return ZS_ERR_ARG;
    if ((uint64_t)(d->N / 64) * (uint64_t)(d->K / 64) >= (1ull << 31)) return ZS_ERR_SHAPE;
    const uint8_t *b = static_cast<const uint8_t *>(blob);
    bv->bitmaps = b + d->off_bitmaps;
    bv->offsets = reinterpret_cast<const u32x2 *>(b + d->off_offsets);
    bv->H = b + d->off_H;
    bv->L = b + d->off_L;
    bv->h_units = (uint32_t)(d->h_bytes / 16);
    bv->l_units = (uint32_t)(d->l_bytes / 16);
    bv->h_fast = bv->h_units >= 256u ? bv->h_units - 255u : 0u;
    bv->l_fast = bv->l_units >= 512u ? bv->l_units - 511u : 0u;
    bv->base_exp = d->base_exp;
    bv->k_blocks = (int32_t)(d->K / 64);
    bv->strips = (int32_t)(d->N / 64);
    return ZS_OK;
}

// The current device and its number of compute units (queried once per device).
struct DeviceInfo {
    int id, cus;
};
int device_info(DeviceInfo *di)
{
    static std::atomic<int> cus[kMaxDevices];
    if (hipGetDevice(&di->id) != hipSuccess) return ZS_ERR_HIP;
    if (di->id < 0 || di->id >= kMaxDevices) return ZS_ERR_HIP;
    di->cus = cus[di->id].load(std::memory_order_relaxed);
    if (di->cus == 0) {
        if (hipDeviceGetAttribute(&di->cus, hipDeviceAttributeMultiprocessorCount, di->id) != hipSuccess || di->cus < 1)
            return ZS_ERR_HIP;
        cus[di->id].store(di->cus, std::memory_order_relaxed);
    }
    return ZS_OK;
}

// Lets kernel k use `bytes` of dynamic LDS.  The attribute sticks to (kernel, device), so it
// is set once per pair: `done` is the call site's bit set of devices already served.
template <class Kernel>
int allow_big_lds(Kernel k, uint32_t bytes, int device, std::atomic<uint64_t> &done)
{
    if (bytes > kMaxLds) return ZS_ERR_CONFIG;
    if (bytes <= 48 * 1024 || (done.load(std::memory_order_acquire) >> device & 1u)) return ZS_OK;
    if (hipFuncSetAttribute(reinterpret_cast<const void *>(k), hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes) !=
        hipSuccess)
        return ZS_ERR_HIP;
    done.fetch_or(1ull << device, std::memory_order_release);
    return ZS_OK;
}

// Compute units assumed by the sizing queries when no device can be asked (they are plain
// host arithmetic and also run on machines without a GPU): those of one MI355X.
constexpr int kDefaultCus = 256;
int cus_or_default()
{
    DeviceInfo di;
    return device_info(&di) == ZS_OK ? di.cus : kDefaultCus;
}

RangeSplit split_ranges(uint32_t total, uint32_t parts) // parts <= total
{
    const uint32_t q = total / parts;
    return RangeSplit{total, parts, q, total % parts, Divider::by(q).magic, Divider::by(q + 1).magic};
}

// Window of the L segment staged in LDS, in bytes: twice the average BlockTile's segment
// (BlockTiles with more take their fallbacks from global memory).
int pick_l_window(const zs_desc *d)
{
    const uint64_t n_bt = (uint64_t)(d->N / 64) * (uint64_t)(d->K / 64);
    const uint64_t avg = 2 * d->n_fallback / n_bt; // bytes per BlockTile
    const uint64_t want = d->max_l_units * 16ull < 2 * avg ? d->max_l_units * 16ull : 2 * avg;
    return want <= 512 ? 512 : 4096;
}

// How a matrix's rows with more than two fallbacks are decoded (enum Fallbacks).  With the short L
// window they are rare: one at a time.  With the long one they are the rule, unless the fallbacks are
// few and lie evenly, so that three in a row of eight stay the exception: at most one weight in 18,
// and no BlockTile with more than one and a half times the average (L segments in bytes).  Measured
// with a share of the weights outside the window, 4096 x 14336, 16 tokens, kLoop / kMany: anywhere in the
// matrix 4.2 % 25.9 / 25.9 us, 5 % 28.9 / 29.9, 5.5 % 30.1 / 30.6, 6 % 31.3 / 31.0, 8 % 34.5 / 31.7; 5 % of
// them in a tenth of the rows (2.8 times the average in the fullest BlockTile) 59.3 / 31.3.  (Where base_exp
// is -1 the long window has kMany alone: no such matrix is worth another kernel.)
bool careful_loop(const zs_desc *d)
{
    const uint64_t n_bt = (uint64_t)(d->N / 64) * (uint64_t)(d->K / 64);
    return pick_l_window(d) == 512 ||
           (18 * d->n_fallback <= n_bt * ZS_BT_ELEMS && d->max_l_units * 16ull * n_bt <= 3 * d->n_fallback);
}

struct GemmVariant {
    const char *name;
    int mt, lw, waves;
    int consumers; // 0: gemm_stream_kernel (16 mt tokens); else gemm_pc_kernel with that many consumer waves
    bool shared_decode() const { return consumers > 0; }
    int tokens() const { return 16 * mt * (consumers ? consumers : 1); }
};

// id = index + 1.  The first entry of each (tokens, lw, kernel) triple is the default for it.
// Names: m<tokens per launch>_l<0: 512-byte, 4: 4 KB L window>_w<streaming waves> for
// gemm_stream_kernel, p<tokens per launch>_l<..>_w<producer waves> for gemm_pc_kernel.  Callers look
// configurations up by name, so a name stays when its kernel changes: 8 and 9 run eight producers now.
const GemmVariant kVariants[] = {
    {"m16_l0_w11", 1, 512, 11, 0}, {"m16_l0_w8", 1, 512, 8, 0},   {"m32_l0_w10", 2, 512, 10, 0},
    {"m32_l0_w7", 2, 512, 7, 0},   {"m16_l4_w7", 1, 4096, 7, 0},  {"m32_l4_w6", 2, 4096, 6, 0},
    {"p64_l0_w7", 1, 512, 7, 4},   {"p128_l0_w7", 2, 512, 8, 4},  {"p256_l0_w7", 2, 512, 8, 8},
    {"p64_l4_w5", 1, 4096, 5, 4},  {"p128_l4_w5", 2, 4096, 5, 4}, {"p256_l4_w5", 2, 4096, 5, 8},
    {"m64_l0_w7", 4, 512, 7, 0},   {"m64_l4_w5", 4, 4096, 5, 0},
};
constexpr int kNumVariants = (int)(sizeof(kVariants) / sizeof(kVariants[0]));

// Workgroups of a ZipGEMM launch: one per CU, fewer when there are fewer BlockTiles.
uint32_t auto_workgroups(uint64_t total, int cus) { return (uint32_t)(total < (uint64_t)cus ? total : (uint64_t)cus); }

// C must start from zero where some workgroup's range begins or ends inside a strip: those
// strips are summed from several workgroups with atomics.
void clear_shared_strips(const BlobView &bv, float *C, int64_t ldc, int M, const RangeSplit &rs, hipStream_t s)
{
    SharedStrips list;
    list.n = 0;
    for (uint32_t b = 1; b < rs.parts; ++b) {
        const uint32_t g = rs.begin(b);
        if (g % (uint32_t)bv.k_blocks == 0) continue;
        const uint32_t strip = g / (uint32_t)bv.k_blocks;
        if (list.n && list.strip[list.n - 1] == strip) continue; // boundaries ascend: duplicates are adjacent
        list.strip[list.n++] = strip;
        if (list.n == (uint32_t)kMaxSharedStrips) { // flush a full list
            hipLaunchKernelGGL(clear_shared_strips_kernel, dim3(list.n, ((unsigned)M + 15) / 16), dim3(256), 0, s, C, ldc, M, list);
            list.n = 0;
        }
    }
    if (list.n) hipLaunchKernelGGL(clear_shared_strips_kernel, dim3(list.n, ((unsigned)M + 15) / 16), dim3(256), 0, s, C, ldc, M, list);
}

// Layout of the scratch buffer of gemm_stream_kernel: kMaxSharedCounters counter words (zero
// between launches), then two partial tiles of 4096 MT bytes per workgroup.  The header has
// one size for every matrix and configuration, so that a buffer which served one call has
// zero counters for any other.
constexpr uint32_t kMaxSharedCounters = 1024;
constexpr uint32_t kScratchHeaderBytes = kMaxSharedCounters * 4;
size_t shared_sums_bytes(uint32_t wgs, int mt) { return kScratchHeaderBytes + (size_t)2 * wgs * 4096 * (size_t)mt; }

template <int MT, int LW, int WAVES>
int launch_gemm(const BlobView &bv, const uint16_t *A, int64_t lda, float *C, int64_t ldc, int M, uint32_t wgs,
                int device, bool loop, void *scratch, bool out_bf16, hipStream_t s)
{
    using S = Slot<LW>;
    constexpr uint32_t lds = StreamLds<MT, LW, WAVES>::kTotal;
    static_assert(lds <= kMaxLds, "variant does not fit the 160 KB of LDS");
    static_assert(S::kLoads < 64, "vmcnt cannot count that many loads");
    static std::atomic<uint64_t> lds_allowed[3];
    constexpr Fallbacks kRows = LW == 512 ? kLoop : kMany; // careful_loop is about the long window
    const int site = bv.base_exp < 0 ? 0 : loop ? 1 : 2;
    auto kern = site == 0   ? gemm_stream_kernel<MT, LW, WAVES, true, kRows>
                : site == 1 ? gemm_stream_kernel<MT, LW, WAVES, false, kLoop>
                            : gemm_stream_kernel<MT, LW, WAVES, false, kRows>;
    static_assert(std::is_same_v<decltype(kern), StreamKernel>, "the kernel finds its StreamArgs by the arguments before them");
    int rc = allow_big_lds(kern, lds, device, lds_allowed[site]);
    if (rc != ZS_OK) return rc;
    const RangeSplit rs = split_ranges((uint32_t)bv.strips * (uint32_t)bv.k_blocks, wgs);
    SharedSums ws = {nullptr, nullptr, kSumCleared, out_bf16 ? 1u : 0u, 0u};
    if (out_bf16 && !scratch) return ZS_ERR_SIZE; // partial sums of BF16 output cannot be added on C
    if (scratch) {
        ws.count = static_cast<uint32_t *>(scratch);
        ws.tiles = reinterpret_cast<float *>(static_cast<uint8_t *>(scratch) + kScratchHeaderBytes);
        ws.tiles_bytes = (uint32_t)(shared_sums_bytes(wgs, MT) - kScratchHeaderBytes);
        ws.mode = kSumParked;
    } else {
        clear_shared_strips(bv, C, ldc, M, rs, s);
    }
    const StreamArgs args = {A, lda, C, ldc, ws, M, bv.base_exp, bv.h_units, bv.l_units, bv.h_fast, bv.l_fast, rs.magic_q, rs.magic_q1};
    hipLaunchKernelGGL(kern, dim3(wgs), dim3(64 * (WAVES + 1)), lds, s, bv.offsets, bv.bitmaps, bv.H, bv.L, rs.q, rs.r, rs.parts,
                       (uint32_t)bv.k_blocks, Divider::by((uint32_t)bv.k_blocks).magic, args);
    return hipGetLastError() == hipSuccess ? ZS_OK : ZS_ERR_HIP;
}

template <int MT, int LW, int P, int R, int Q, int F>
int launch_pc(const BlobView &bv, const uint16_t *A, int64_t lda, float *C, int64_t ldc, int M, uint32_t wgs,
              int device, bool loop, hipStream_t s)
{
    using S = Slot<LW>;
    constexpr uint32_t lds = kTableBytes + kPcCtlBytes + R * kDenseBytes + P * 2 * S::kBytes;
    static_assert(lds <= kMaxLds, "variant does not fit the 160 KB of LDS");
    static_assert(S::kLoads < 64, "vmcnt cannot count that many loads");
    static std::atomic<uint64_t> lds_allowed[3];
    constexpr Fallbacks kRows = LW == 512 ? kLoop : kMany;
    const int site = bv.base_exp < 0 ? 0 : loop ? 1 : 2;
    auto kern = site == 0   ? gemm_pc_kernel<MT, LW, P, R, Q, F, true, kRows>
                : site == 1 ? gemm_pc_kernel<MT, LW, P, R, Q, F, false, kLoop>
                            : gemm_pc_kernel<MT, LW, P, R, Q, F, false, kRows>;
    int rc = allow_big_lds(kern, lds, device, lds_allowed[site]);
    if (rc != ZS_OK) return rc;
    const RangeSplit rs = split_ranges((uint32_t)bv.strips * (uint32_t)bv.k_blocks, wgs);
    clear_shared_strips(bv, C, ldc, M, rs, s);
    const int q_active = ((M + 15) / 16 + MT - 1) / MT; // consumers with at least one token
    hipLaunchKernelGGL(kern, dim3(wgs), dim3(64 * (P + Q)), lds, s, bv, A, lda, C, ldc, M, q_active, rs);
    return hipGetLastError() == hipSuccess ? ZS_OK : ZS_ERR_HIP;
}

int variant_for(const zs_desc *d, int64_t M, int cus)
{
    // Up to 64 tokens every wave decodes and multiplies for itself; beyond, the decode is shared.  (From 33
    // tokens, FP32 output, p64 / m64: 50 tokens, 6144 x 4096 20.2 / 24.4 us, 1024 x 4096 11.8 / 16.7; but 4096 x 4096, 48 tokens, 16.1 / 15.5;
    // 64 tokens, 8192 x 4096 23.7 / 21.5, 28672 x 4096 57.3 / 53.3, 4096 x 14336 33.2 / 30.7.  Which is faster goes with the
    // contributors to a strip and the tasks of a range; no line over them has been drawn.)
    const int lw = pick_l_window(d);
    const int tokens = M <= 16 ? 16 : M <= 32 ? 32 : M <= 64 ? 64 : M <= 128 ? 128 : 256;
    const bool shared_decode = tokens > 64;
    // Waves take BlockTiles one at a time, so a workgroup's last round is rarely full.  With few
    // tiles per workgroup fewer waves (faster each, fuller rounds) win: measured on the 8B
    // shapes, 16 tokens: eight beat eleven up to 64 tiles per workgroup; 32 tokens: seven beat
    // ten below 56.
    const int64_t tiles_per_wg = (d->N / 64) * (d->K / 64) / cus;
    int waves = 0;
    if (lw == 512 && tokens == 16 && tiles_per_wg <= 64) waves = 8;
    if (lw == 512 && tokens == 32 && tiles_per_wg < 56) waves = 7;
    for (int i = 0; waves && i < kNumVariants; ++i)
        if (kVariants[i].tokens() == tokens && kVariants[i].lw == lw && !kVariants[i].shared_decode() &&
            kVariants[i].waves == waves)
            return i + 1;
    for (int i = 0; i < kNumVariants; ++i)
        if (kVariants[i].tokens() == tokens && kVariants[i].lw == lw && kVariants[i].shared_decode() == shared_decode)
            return i + 1;
    return 1;
}

} // namespace

extern "C" int zs_decompress(const zs_desc *d, const void *blob_dev, uint16_t *W_out_dev, int64_t ldw,
                             void *hip_stream)
{
    BlobView bv;
    int rc = make_view(d, blob_dev, &bv);
    if (rc != ZS_OK) return rc;
    if (!W_out_dev || reinterpret_cast<uintptr_t>(W_out_dev) % 16) return ZS_ERR_ARG;
    if (ldw < d->K || ldw % 8) return ZS_ERR_SHAPE;
    const int64_t n_bt = (int64_t)bv.strips * bv.k_blocks;
    DeviceInfo di;
    if ((rc = device_info(&di)) != ZS_OK) return rc;
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    static std::atomic<uint64_t> lds_allowed[8];
    auto launch = [&](auto kern, uint32_t lds, int waves, int site) {
        int r = allow_big_lds(kern, lds, di.id, lds_allowed[site]);
        if (r != ZS_OK) return r;
        int64_t wgs = (n_bt + waves - 1) / waves;
        if (wgs > di.cus) wgs = di.cus;
        hipLaunchKernelGGL(kern, dim3((unsigned)wgs), dim3(64 * waves), lds, s, bv, W_out_dev, ldw);
        return hipGetLastError() == hipSuccess ? (int)ZS_OK : (int)ZS_ERR_HIP;
    };
    // Whole cache lines hold back the first half of a BlockTile's stores, which a wave with one or two
    // BlockTiles does not catch up with, and the later the more it decodes.  Half / whole lines, 2 % fallbacks:
    // 1024 x 1024 6.14 / 6.47 us, 3072 x 4096 9.92 / 10.5, 3840 x 4096 (15 BlockTiles per CU) 10.8 / 11.3, 4096 x 4096 11.8 /
    // 11.5, 6144 x 4096 17.8 / 15.8; 4.4 %: 4096 x 4096 11.9 / 12.5, 4608 x 4096 (18) 15.1 / 15.9, 5120 x 4096 15.9 / 16.1, 6144 x
    // 4096 18.0 / 16.8; 32 %: 4096 x 4096 15.9 / 16.3, 4608 x 4096 16.0 / 16.1, 5120 x 4096 17.0 / 16.7.
    const bool lines = n_bt > (int64_t)(32 * d->n_fallback <= (uint64_t)n_bt * ZS_BT_ELEMS ? 15 : 18) * di.cus;
    const bool m1 = d->base_exp < 0;
    if (pick_l_window(d) == 512) {
        // eight waves with three tiles in flight each (measured against 7 x 3 with a 1 KB window,
        // 11 x 2, 10 x 2, 6 x 4 and 5 x 4: 2 to 10 % faster on the 8B shapes)
        constexpr uint32_t lds = kTableBytes + 8 * 3 * Slot<512>::kBytes;
        static_assert(lds <= kMaxLds, "variant does not fit the 160 KB of LDS");
        return m1      ? launch(decompress_kernel<512, 3, 8, true, kLoop, true>, lds, 8, 0)
               : lines ? launch(decompress_kernel<512, 3, 8, false, kLoop, true>, lds, 8, 1)
                       : launch(decompress_kernel<512, 3, 8, false, kLoop, false>, lds, 8, 2);
    }
    constexpr uint32_t lds = kTableBytes + 7 * 2 * Slot<4096>::kBytes;
    if (m1) return launch(decompress_kernel<4096, 2, 7, true, kMany, true>, lds, 7, 3);
    if (careful_loop(d))
        return lines ? launch(decompress_kernel<4096, 2, 7, false, kLoop, true>, lds, 7, 4)
                     : launch(decompress_kernel<4096, 2, 7, false, kLoop, false>, lds, 7, 5);
    return lines ? launch(decompress_kernel<4096, 2, 7, false, kMany, true>, lds, 7, 6)
                 : launch(decompress_kernel<4096, 2, 7, false, kMany, false>, lds, 7, 7);
}

extern "C" int zs_compute_units(void) { return cus_or_default(); }

extern "C" int zs_gemm_num_configs(void) { return kNumVariants; }

extern "C" const char *zs_gemm_config_name(int config)
{
    return (config >= 1 && config <= kNumVariants) ? kVariants[config - 1].name : nullptr;
}

extern "C" int zs_gemm_pick_config(const zs_desc *d, int64_t M)
{
    if (!d || M < 1 || zs_desc_validate(d) != ZS_OK) return 0;
    return variant_for(d, M, cus_or_default());
}

namespace {

// What a ZipGEMM call will launch for (d, M, config): the variant, the number of workgroups
// and the scratch bytes its kernel can use (0 for the producer / consumer kernel).
struct GemmPlan {
    int variant;
    uint32_t wgs;
    size_t scratch_bytes;
};
int plan_gemm(const zs_desc *d, int64_t M, int config, int cus, GemmPlan *p)
{
    if (config < 0) return ZS_ERR_CONFIG;
    p->variant = config & 0xFF;
    if (p->variant == 0) p->variant = variant_for(d, M, cus);
    if (p->variant < 1 || p->variant > kNumVariants) return ZS_ERR_CONFIG;
    const GemmVariant &v = kVariants[p->variant - 1];
    const uint64_t total = (uint64_t)(d->N / 64) * (uint64_t)(d->K / 64);
    p->wgs = (uint32_t)(config >> 8); // bits 8 and up of config: number of workgroups (0 = one per CU)
    if (p->wgs == 0) p->wgs = auto_workgroups(total, cus);
    if (p->wgs > total) p->wgs = (uint32_t)total;
    // the producer / consumer kernel sums shared strips with atomics on C and uses no scratch
    p->scratch_bytes = !v.shared_decode() && p->wgs <= kMaxSharedCounters ? shared_sums_bytes(p->wgs, v.mt) : 0;
    return ZS_OK;
}

int gemm_impl(const zs_desc *d, const void *blob_dev, const uint16_t *A_dev, int64_t lda, float *C_dev, int64_t ldc,
              int64_t M, void *workspace_dev, size_t workspace_bytes, hipStream_t s, int config, const DeviceInfo &di,
              bool out_bf16 = false)
{
    BlobView bv;
    int rc = make_view(d, blob_dev, &bv);
    if (rc != ZS_OK) return rc;
    if (!A_dev || !C_dev) return ZS_ERR_ARG;
    if (reinterpret_cast<uintptr_t>(A_dev) % 16 || reinterpret_cast<uintptr_t>(C_dev) % 16) return ZS_ERR_ARG;
    if (M < 1 || M > (1 << 20) || lda < d->K || lda % 8 || ldc < d->N || ldc % 4) return ZS_ERR_SHAPE;
    GemmPlan plan;
    // BF16 output exists in the streaming kernel only (at most 64 tokens per launch; more tokens
    // run as 64-token panels) and always goes through the scratch buffer
    if ((rc = plan_gemm(d, out_bf16 && M > 64 ? 64 : M, config, di.cus, &plan)) != ZS_OK) return rc;
    const GemmVariant &v = kVariants[plan.variant - 1];
    if (out_bf16 && v.shared_decode()) return ZS_ERR_CONFIG;
    const uint32_t wgs = plan.wgs;
    // row offsets (token * lda * 2 bytes, token < the launch's width) are 32-bit inside the kernels
    if ((uint64_t)lda * 2u * (uint64_t)v.tokens() >= (1ull << 32)) return ZS_ERR_SHAPE;
    // scratch is optional: without it (or with too little) shared strips go through atomics on C
    void *scratch = nullptr;
    if (workspace_dev && plan.scratch_bytes && reinterpret_cast<uintptr_t>(workspace_dev) % 256 == 0 &&
        workspace_bytes >= plan.scratch_bytes)
        scratch = workspace_dev;
    if (out_bf16 && !scratch) return ZS_ERR_SIZE;
    // tokens beyond the variant's width are handled in successive column panels
    const int width = v.tokens();
    const bool loop = careful_loop(d);
    for (int64_t m0 = 0; m0 < M; m0 += width) {
        const int m = (int)((M - m0) < width ? (M - m0) : width);
        const uint16_t *Ap = A_dev + m0 * lda;
        float *Cp = out_bf16 ? reinterpret_cast<float *>(reinterpret_cast<uint16_t *>(C_dev) + m0 * ldc) : C_dev + m0 * ldc;
#define ZS_PC_CASE(ID, MT, LW, P, R, Q, F) \
    case ID: rc = launch_pc<MT, LW, P, R, Q, F>(bv, Ap, lda, Cp, ldc, m, wgs, di.id, loop, s); break;
#define ZS_CASE(ID, MT, LW, WAVES) \
    case ID: rc = launch_gemm<MT, LW, WAVES>(bv, Ap, lda, Cp, ldc, m, wgs, di.id, loop, scratch, out_bf16, s); break;
        switch (plan.variant) {
            ZS_CASE(1, 1, 512, 11)
            ZS_CASE(2, 1, 512, 8)
            ZS_CASE(3, 2, 512, 10)
            ZS_CASE(4, 2, 512, 7)
            ZS_CASE(5, 1, 4096, 7)
            ZS_CASE(6, 2, 4096, 6)
            ZS_PC_CASE(7, 1, 512, 7, 7, 4, 6)
            ZS_PC_CASE(8, 2, 512, 8, 6, 4, 6)
            ZS_PC_CASE(9, 2, 512, 8, 6, 8, 4)
            ZS_PC_CASE(10, 1, 4096, 5, 6, 4, 6)
            ZS_PC_CASE(11, 2, 4096, 5, 6, 4, 6)
            ZS_PC_CASE(12, 2, 4096, 5, 6, 8, 4)
            ZS_CASE(13, 4, 512, 7)
            ZS_CASE(14, 4, 4096, 5)
        default: rc = ZS_ERR_CONFIG;
        }
#undef ZS_CASE
#undef ZS_PC_CASE
        if (rc != ZS_OK) return rc;
    }
    return ZS_OK;
}

} // namespace

extern "C" size_t zs_gemm_workspace_ex(const zs_desc *d, int64_t M, int config)
{
    if (!d || M < 1 || zs_desc_validate(d) != ZS_OK) return 0;
    GemmPlan plan;
    return plan_gemm(d, M, config, cus_or_default(), &plan) == ZS_OK ? plan.scratch_bytes : 0;
}
extern "C" size_t zs_gemm_workspace(const zs_desc *d, int64_t M) { return zs_gemm_workspace_ex(d, M, 0); }

extern "C" int zs_gemm_ex(const zs_desc *d, const void *blob_dev, const uint16_t *A_dev, int64_t lda, float *C_dev,
                          int64_t ldc, int64_t M, void *workspace_dev, size_t workspace_bytes, void *hip_stream,
                          int config)
{
    DeviceInfo di;
    int rc = device_info(&di);
    if (rc != ZS_OK) return rc;
    return gemm_impl(d, blob_dev, A_dev, lda, C_dev, ldc, M, workspace_dev, workspace_bytes,
                     static_cast<hipStream_t>(hip_stream), config, di);
}

extern "C" int zs_gemm_bf16(const zs_desc *d, const void *blob_dev, const uint16_t *A_dev, int64_t lda, uint16_t *C_dev,
                            int64_t ldc, int64_t M, void *workspace_dev, size_t workspace_bytes, void *hip_stream)
{
    DeviceInfo di;
    int rc = device_info(&di);
    if (rc != ZS_OK) return rc;
    return gemm_impl(d, blob_dev, A_dev, lda, reinterpret_cast<float *>(C_dev), ldc, M, workspace_dev, workspace_bytes,
                     static_cast<hipStream_t>(hip_stream), 0, di, true);
}

extern "C" int zs_gemm(const zs_desc *d, const void *blob_dev, const uint16_t *A_dev, int64_t lda, float *C_dev,
                       int64_t ldc, int64_t M, void *workspace_dev, size_t workspace_bytes, void *hip_stream)
{
    return zs_gemm_ex(d, blob_dev, A_dev, lda, C_dev, ldc, M, workspace_dev, workspace_bytes, hip_stream, 0);
}

// ---- ZipGEMM for callers that cannot allocate ----------------------------------------------
// The scratch buffer of gemm_stream_kernel (strip counters + two partial tiles per workgroup)
// lives in a file-scope device array instead of caller memory.  Sized for the widest variant
// (64 tokens) at kStaticWorkgroups workgroups; every GPU the library runs on holds its own copy
// until the process ends.
namespace {
constexpr uint32_t kStaticWorkgroups = 256;
constexpr size_t kStaticScratchBytes = kScratchHeaderBytes + (size_t)2 * kStaticWorkgroups * 4096 * 4;
}
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];
namespace {

__global__ void zero_units_kernel(u32x4 *p, uint32_t n) // n 16-byte units
{
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = u32x4{0u, 0u, 0u, 0u};
}

// Device address of `scratch` on the current device (the array's name is only a host-side
// handle): looked up once per device and kept.
int static_scratch(int device, void **out)
{
    static std::atomic<void *> ptr[kMaxDevices];
    void *p = ptr[device].load(std::memory_order_acquire);
    if (!p) {
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return ZS_ERR_HIP;
        ptr[device].store(p, std::memory_order_release);
    }
    *out = p;
    return ZS_OK;
}
} // namespace

extern "C" int zs_gemm_noalloc(const zs_desc *d, const void *blob_dev, const uint16_t *A_dev, int64_t lda,
                               float *C_dev, int64_t ldc, int64_t M, void *hip_stream)
{
    if (!d || M < 1) return d ? ZS_ERR_SHAPE : ZS_ERR_ARG;
    int rc = zs_desc_validate(d);
    if (rc != ZS_OK) return rc;
    DeviceInfo di;
    if ((rc = device_info(&di)) != ZS_OK) return rc;
    GemmPlan plan;
    if ((rc = plan_gemm(d, M, 0, di.cus, &plan)) != ZS_OK) return rc;
    if (plan.scratch_bytes > kStaticScratchBytes) return ZS_ERR_SIZE; // more workgroups than the array was sized for
    void *ptr = nullptr;
    if ((rc = static_scratch(di.id, &ptr)) != ZS_OK) return rc;
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    if (plan.scratch_bytes) {
        // The array keeps whatever the last call left.  Counters and slots must start at zero;
        // a completed call leaves them so, one that overlapped with another may not, so the
        // part this call uses is cleared every time.  A fill kernel, not a memset: callers may
        // be capturing.
        const uint32_t units = (uint32_t)(plan.scratch_bytes / 16);
        hipLaunchKernelGGL(zero_units_kernel, dim3((units + 255) / 256), dim3(256), 0, s, static_cast<u32x4 *>(ptr), units);
        if (hipGetLastError() != hipSuccess) return ZS_ERR_HIP;
    }
    return gemm_impl(d, blob_dev, A_dev, lda, C_dev, ldc, M, ptr, kStaticScratchBytes, s, 0, di);
}

extern "C" const char *zs_strerror(int status)
{
    switch (status) {
    case ZS_OK: return "ok";
    case ZS_ERR_ARG: return "bad argument (null or misaligned pointer)";
    case ZS_ERR_SHAPE: return "unsupported shape (N, K must be positive multiples of 64; check M, ld*)";
    case ZS_ERR_SIZE: return "buffer too small";
    case ZS_ERR_FORMAT: return "descriptor does not describe a valid TCA-TBE blob";
    case ZS_ERR_HIP: return "HIP runtime error";
    case ZS_ERR_CONFIG: return "unknown kernel configuration";
    default: return "unknown status";
    }
}

extern "C" int zs_version(void) { return 1; }
