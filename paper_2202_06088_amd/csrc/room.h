// Arithmetic of a room of items (trace entries, adjoint records, merge-list
// entries) that wavefronts fill in blocks taken from one counter. Plain
// integers, without the device headers, so that the host can check it up to
// the largest room.
#pragma once

#include <stdint.h>

namespace neuvv {

// Items a wavefront takes from the room's counter at a time: a 16,384th of the
// room, between 128 (the most that one iteration of a wavefront asks for) and
// 2048. The rest of a wavefront's last block stays unused, so the block is kept
// small against the room's share per wavefront; the floor of 16,384 blocks also
// bounds the atomics on the one counter (12 thousand on the 16.6 M-ray ring).
// Blocks of 2048 from one counter per XCD left 38 % of the ring's trace room
// unused and, in rooms below 2 M items, let 8 wavefronts per XCD exhaust it: the
// rays left over were walked again (65,536 training rays with room for two
// samples each: 222 us of 717 us; 4 layers at 1920 x 1080: 1462 us of 4247 us).
__host__ __device__ __forceinline__ int item_block(int64_t cap) {
    const int b = (int)(cap >> 14);
    return b < 128 ? 128 : (b > 2048 ? 2048 : b);
}

// Whether n >= 0 more items fit in what is left of a block, [cur, end) (end =
// -1: the room is exhausted). Rooms reach 2^31 - 1 items, so cur + n may not fit
// int32, but end - cur does.
__host__ __device__ __forceinline__ bool items_fit(int cur, int end, int n) { return n <= end - cur; }

// The block that starts at `first` of a room of cap items, clamped to the room
// (which is below 2^31 items, so the bounds fit int32).
__host__ __device__ __forceinline__ void open_block(int64_t first, int64_t cap, int& cur, int& end) {
    const int block = item_block(cap);
    cur = (int)(first < cap ? first : cap);
    end = (int)(first + block <= cap ? first + block : cap);
}

}  // namespace neuvv
