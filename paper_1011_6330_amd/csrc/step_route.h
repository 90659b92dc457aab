// step_route.h -- rules of the step's launches: plain C++, so that they can be tested
// without a GPU (constexpr functions are device functions too).
#pragma once

#include <stdint.h>

namespace pcpic {

// Slots up to which a tube, or all tubes of a batch together, take fused steps; past
// them, forming the kicks per wave costs more than a kernel.  Per step, push and field
// kernels against fused, ordered beams: FP64 of 16,384 cells 7e5 particles 11.9 / 9.5 us,
// 1.2e6 14.8 / 13.3, 1.8e6 18.5 / 18.7, 2.5e6 22.0 / 24.2, of 65,536 cells 7e5 11.1 /
// 10.0, 1.2e6 14.4 / 14.6, 1.8e6 17.4 / 18.4; FP32-bulk of 65,536 cells 1.2e6 14.2 / 12.7,
// 1.5e6 14.6 / 13.9, 2.1e6 17.6 / 18.3; batches of eight (three kernels when not fused) FP64 of
// 10,000 cells 2.4e6 30.2 / 27.4, 4e6 39.2 / 38.7, 6e6 50.8 / 54.2, FP32-bulk 4e6 36.0 /
// 33.8.  An adjoint run always takes fused steps, as it also saves a kernel per step
// there that notes the slot count.
constexpr int64_t fuse_slots(bool batch, bool f32)
{
    return batch ? (int64_t)1 << 22 : (f32 ? (int64_t)1 << 21 : (int64_t)3 << 19);
}

// Slots that a tube is expected to hold: twice its particles at the corotation density,
// as far as its capacity goes, or those it held when the host last saw their count
// (loading, read-outs, pic_sync), if these are more.  (By the density alone, a tube of
// 20,000 cells and ppc 20 took fused steps whatever it was loaded with: 1.2e7 particles
// 116.9 us a step against 108.6 in separate kernels, 3e7 302.7 against 268.0; a batch
// of eight with 3e6 each 195.0 against 180.4.)
inline int64_t expected_slots(double ppc, int64_t n_cells, int64_t capacity, int64_t seen)
{
    const double e = 2.0 * ppc * (double)n_cells;
    const int64_t slots = e < (double)capacity ? (int64_t)e : capacity;
    return seen > slots ? seen : slots;
}

// Order of a single tube's push over its slots: ascending and descending in turn.  What
// one step touched last the next touches first, while it is still in the 256 MiB
// last-level cache.  Blocks go to the 8 XCDs in turn, each with an L2 of 4 MiB: the
// descending order reverses groups of 8 tiles and keeps a tile on the XCD that had it
// the step before.  (Reversed tile by tile, every tile changed its XCD: 1e6 FP64
// particles took 16.3 us a step where ascending ones take 13.0, and 9e6 took 53.1 where
// this order takes 50.4.)
// The streams are read and written with plain accesses where they take more than the
// L2s and up to CACHED_BYTES (nontemporal ones pass the last-level cache by).  Per step
// in this order, nontemporal / plain, and ascending and nontemporal: FP64 particles
// 1e6 (16 MB) 12.8 / 13.5, 12.9; 2e6 19.7 / 18.4, 19.7; 4.6e6 33.2 / 30.5, 34.4; 9e6
// 56.9 / 50.4, 58.6; 4e7 (0.64 GB) 223.5 / 212.1, 231.1; FP32-bulk 1.4e6 (17 MB) 14.4 /
// 15.1, 14.5; 2.8e6 20.6 / 20.1, 21.3; 4e7 172.1 / 159.4, 177.6.  Past 1 GiB they are
// within 1% (FP64 8.5e7, 1.36 GB: 473 / 468; FP32-bulk 1.3e8, 1.56 GB: 531 / 535).
constexpr int64_t CACHED_BYTES = (int64_t)1 << 30, L2_BYTES = (int64_t)32 << 20;
constexpr bool push_nontemporal(int64_t bytes) { return bytes <= L2_BYTES || bytes > CACHED_BYTES; }

// A fused step's push keeps the kicks at 64 faces per wave and forms those past them from
// the fields, about ten words from four arrays where a separate push reads two.  A slot
// more than 62 cells above the lowest of its wave's and not in the 8 cells of the slot
// before it is a jump: a load of cache lines of its own.  Slots in order have them
// where they are sparse (a wave takes 128 of them, 256 in FP32-bulk): `slots` spread
// evenly over n_cells.
inline int64_t ordered_jumps(int64_t slots, int64_t n_cells, bool f32)
{
    if (slots <= 0) return 0;
    const double gap = (double)n_cells / (double)slots, span = (f32 ? 256.0 : 128.0) * gap;
    return span > 63.0 ? (int64_t)((double)slots * (1.0 - 63.0 / span) * (gap < 8.0 ? gap / 8.0 : 1.0)) : 0;
}

// Jumps from which on a tube's steps are faster in separate kernels.  Per step, push and
// field kernels against fused, shuffled slots: FP64 of 2,048 cells 1e5 18.9 / 17.1 us,
// 4e5 54.1 / 55.8; of 10,000 cells 1e5 15.0 / 13.8, 4e5 39.3 / 43.3; of 65,536 cells 2e4
// 8.3 / 9.1, 4e5 35.3 / 41.8; of 2^20 cells 2e5 30.4 / 45.7, 3e6 216 / 403; FP32-bulk of
// 10,000 cells 2e4 10.6 / 10.5, 4e5 39.2 / 46.5; of 65,536 cells 2e4 9.9 / 12.4.  A tenth of the
// slots shuffled, 65,536 cells: FP64 1e5 9.2 / 9.0, 1e6 19.9 / 22.4.  Sparse and in order:
// FP64 of 65,536 cells 2e4 8.1 / 6.9, of 200,000 1e5 11.6 / 12.1, of 2^20 4e5 34.1 / 36.3,
// FP32-bulk 42.6 / 50.5.
inline int64_t most_jumps(int64_t jumps, int64_t slots, int64_t n_cells, bool f32)
{
    const bool most = 2 * jumps > slots;
    if (n_cells < 4096) return 1 << 17;
    if (n_cells < 32768) return f32 ? (most ? 1 << 10 : 1 << 16) : 1 << 17;
    if (most) return f32 ? 1 << 10 : 1 << 12;
    return n_cells < 131072 ? 1 << 13 : 1 << 12;
}
// The same for one tube of a batch, whose tubes hide each other's latencies and which
// takes three kernels when not fused (eight shuffled tubes of 10,000 cells, FP64: 5,000
// particles each 17.4 / 13.2, 50,000 43.3 / 43.9, 2e5 135.5 / 141.3; of 65,536 cells 5,000
// 20.7 / 19.8, 50,000 48.7 / 57.2).
constexpr int64_t most_jumps_batch(int64_t n_cells)
{
    return n_cells < 4096 ? 1 << 19 : (n_cells < 32768 ? 1 << 17 : 1 << 16);
}

// Sampling of the loaded slots in which jumps are counted: every jump_stride-th group of
// 256, so that about 1024 groups add to the count.
constexpr int64_t jump_stride(int64_t n) { return (n + 256 * 1024 - 1) / (256 * 1024); }

// Blocks of a sort's scatter over `tiles` tiles of slots: they also clear the key counts,
// so a tube of many keys and few slots gets blocks for these, 2048 keys each.  (Clearing
// by 1 block instead of 512, 2^20 keys of a tube of 1,024 slots took 48.5 us a step with a
// sort every 4, where these take 21.6.)
constexpr int64_t scatter_blocks(int64_t tiles, int64_t n_keys)
{
    const int64_t clear = (n_keys + 2047) / 2048;
    return tiles > clear ? tiles : clear;
}

constexpr int XCDS = 8;
// The tile of block k of `tiles` (past the ends, < 0 or >= tiles: the block is idle), and
// the blocks to launch for them.
constexpr int64_t push_tile(int64_t k, int64_t tiles, int rev)
{
    return rev ? ((tiles + XCDS - 1) / XCDS - 1 - k / XCDS) * XCDS + k % XCDS : k;
}
constexpr unsigned push_blocks(int64_t tiles) { return (unsigned)((tiles + XCDS - 1) / XCDS * XCDS); }

}  // namespace pcpic
