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
// Records are taken in blocks twice that size: a wavefront waits for the one
// counter at every block (with an item_block, 2 x 1920 x 1080 per-point rays
// replayed 148 us against 136 us, 1024 x 1024 rays walked and reduced 492 against
// 484 us), and their rooms are wide enough.
__host__ __device__ __forceinline__ int record_block(int64_t cap) {
    const int b = (int)(cap >> 13);
    return b < 128 ? 128 : (b > 2048 ? 2048 : b);
}

// Whether n >= 0 more items fit in what is left of a block, [cur, end) (end =
// -1: the room is exhausted). Rooms reach 2^31 - 1 items, so cur + n may not fit
// int32, but end - cur does.
__host__ __device__ __forceinline__ bool items_fit(int cur, int end, int n) { return n <= end - cur; }

// The block that starts at `first` of a room of cap items, clamped to the room
// (which is below 2^31 items, so the bounds fit int32).
__host__ __device__ __forceinline__ void open_block(int64_t first, int64_t cap, int block, int& cur, int& end) {
    cur = (int)(first < cap ? first : cap);
    end = (int)(first + block <= cap ? first + block : cap);
}

// Records of an adjoint: as many as the device has memory for, between `least`
// and `most`. Samples beyond the room take per-sample atomics.
struct RecordRoom {
    int64_t most, least;
};

// Two samples per ray or, after a traced forward, as many as the trace has room
// for if that is more (so that every replayed sample has a record), at least
// 2^20, are what a call asks for at least. Rays of a close view may all hit,
// six or more samples each on average (scattering 2.7 M samples of 427,000 rays
// one by one cost 1.7 ms), so up to 2^23 records, 256 MiB, it asks for sixteen
// per ray (up to 2^24, 512 MiB, 2.1 M rays with half of their samples traced took
// 1042 us instead of 1059, and no other call less). Below 2^31.
__host__ __device__ inline RecordRoom record_room(int64_t n_rays, int64_t trace_cap) {
    const int64_t most = 1ll << 23, last = INT32_MAX;
    int64_t least = 2 * n_rays > trace_cap ? 2 * n_rays : trace_cap;
    if (least < 1ll << 20) least = 1ll << 20;
    if (least > last) least = last;
    const int64_t many = n_rays < most / 16 ? 16 * n_rays : most;
    return {least > many ? least : many, least};
}

// Takes the room that alloc(records), returning a status, finds memory for: the
// most, then half of that and so on, at last the least. Sets cap to it.
template <class Alloc, class NoMemory>
auto take_room(const RecordRoom& room, int64_t& cap, Alloc&& alloc, NoMemory&& no_memory) {
    for (cap = room.most;; cap = cap / 2 > room.least ? cap / 2 : room.least) {
        const auto e = alloc(cap);
        if (cap <= room.least || !no_memory(e)) return e;
    }
}

}  // namespace neuvv
