// Launchers of the gfx950 kernels (internal to the library; the public ABI is hmar_attn.h).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

namespace hmar {

// Device copy of the tile schedule of one (device, scale schedule) pair.
struct DeviceSchedule {
    const void* items[2];      // Item[n_items[dir]]
    int32_t n_items[2];
    int32_t max_tiles[2];      // streamed 64-row tiles of a list's longest item
    int64_t total_tiles[2];    // and of all its items
    int32_t long_items;        // of the forward's list: items_to_last_long
    const int32_t* row_lo[2];  // L entries
    const int32_t* row_hi[2];
    int32_t L;                 // rows of Q, O, LSE per head
    int32_t Lk;                // rows of K, V per head
    int32_t num_cus;           // compute units of the device the tables live on
    bool causal;               // the block-causal mask
};

// Number of head groups (8 heads each) in the batch that ends a launch item by item (see
// map_workgroup): about twice as many (head, item) units as one XCD keeps resident at four
// workgroups per CU.  Measured on the 256px and 512px training shapes (forward+backward step):
// without the batch +1.5 % and +3.8 %; half the size 0 and +1.7 %; twice the size +1.7 % and +1 %;
// batching the whole launch this way instead of its end only loses more in L2 locality than it
// gains.
#ifndef HMAR_TUNE_TAIL_PERCENT
#define HMAR_TUNE_TAIL_PERCENT 100     // measurement builds: size of the batch relative to the shipped one
#endif
inline int tail_groups_for(int num_cus, int n_items) {
    const int g = ((num_cus / 8) * 8) * HMAR_TUNE_TAIL_PERCENT / 100 / (n_items > 0 ? n_items : 1);
    return g < 1 ? 1 : g;
}

// The inverse by which divide() (csrc/device_common.h) divides by d: the quotient from the high half of a product is
// at most one too small for every n below 2^31.
inline uint32_t inverse_of(int d) { return d > 1 ? (uint32_t)((1ull << 32) / (unsigned)d) : 0xffffffffu; }

// The order in which the workgroups of a launch take its (head, item) units (see map_unit).
struct UnitMap {
    int n_items;
    int head_major;            // workgroups before the batch that ends the launch
    int batch_head;            // first head of the batch
    int batch, batch_grouped;  // its heads, and those of them that fill groups of eight
    int last_group_head;       // first head of the last group
    uint32_t inv_items, inv_batch;
    int turned;                // 0, or: an XCD's workgroups turned .. 2 * turned - 1 are taken backwards
    int units;                 // workgroups of the launch
};
inline UnitMap unit_map_for(int n_items, int n_heads, int batch_groups, int turned = 0) {
    const int n_groups = n_heads / 8, tail = std::min(batch_groups, n_groups);
    const int batch = 8 * tail + n_heads % 8;
    return {n_items, 8 * (n_groups - tail) * n_items, 8 * (n_groups - tail), batch, 8 * tail, 8 * (n_groups - 1),
            inverse_of(n_items), inverse_of(batch), turned, n_items * n_heads};
}
// measurement builds: 0 takes the order, or the form, out of every launch
#ifndef HMAR_TUNE_TURN
#define HMAR_TUNE_TURN 1
#endif
#ifndef HMAR_TUNE_HALF_BATCH
#define HMAR_TUNE_HALF_BATCH 1
#endif
#ifndef HMAR_TUNE_WHOLE_ROWS
#define HMAR_TUNE_WHOLE_ROWS 1
#endif
#ifndef HMAR_TUNE_KEYS_AHEAD
#define HMAR_TUNE_KEYS_AHEAD 1
#endif

// How a kind of launch orders its units (launch_map).
struct Order {
    int turn_rounds;           // the second unit of every compute unit is dealt backwards up to so many units per compute unit
    int half_below;            // the batch is halved for lists of fewer items than this,
    int half_whole_below;      // and, where it would be the whole launch, for lists of fewer items than this
};
constexpr Order kOrderFwd = {6, 8, 8}, kOrderFwdCausal = {6, 0, 0}, kOrderDq = {6, 8, 16};
constexpr Order kOrderDkDv = {2, 8, 16};       // and both lists in one launch
// The map of a launch.
//  1. Head by head, with a batch of tail_groups_for() groups at the end that is walked item by item.
//  2. The same with half that batch, for short lists.  A launch that is one batch starts with its heaviest items alone, in
//     step, all waiting for memory and then all computing, and leaves the L2 no locality.
//  3. Item by item altogether, where less than one unit per compute unit would be left ahead of the batch.
//  4. Item by item with the second unit of every compute unit dealt backwards, in launches of at most `turn_rounds`
//     units per compute unit: the heaviest first unit meets the lightest second one.
// What they measured (profiles/launch_rules.txt; us, forward / backward, one card, unless it says otherwise; a compute unit
// holds four workgroups of the forward and dQ, two of dK/dV):
//   1 -> 2   7 items (680 tokens): 200 heads 20.6 / 61.0 -> 20.2 / 56.9, 256 heads 25.9 / 77.1 -> 25.8 / 73.5, 320 heads
//            33.8 / 94.4 -> 30.9 / 88.8
//            8 to 15 items, launches that are one batch, 150 schedules: forward +2 % (-8..+21 %), dK,dV -0.3 %, dQ -0.1 %
//            20 items (2240 tokens), 64 heads, another card: forward / dK,dV / dQ 52.8 / 91.5 / 69.4 -> 55.2 / 93.4 / 70.5
//            block-causal, 2 to 7 items, 4 to 24 units per compute unit, 126 schedules: backward -1.1 % (-10..+4 %), but
//            forward +0.1 % (-11..+6 %), whose items share a head's first keys: it keeps the full batch
//   2 -> 3   160 heads of 680 tokens, dK,dV, another card: two groups ahead of the batch 34.2, none 32.2
//   3 -> 4   680 tokens: 32 heads, both lists in one launch, 16.3 -> 14.4; 64 heads, backward, 25.6 -> 24.5; 160 heads 18.3 / 49.8
//            -> 17.8 / 49.0; 21 heads of 2240 tokens, backward, 69.8 -> 65.7.  140 schedules, 2 to 3.5 units per compute unit:
//            forward -1.4 % (-17..+9 %); 196 of 3.5 to 6: -0.2 % (-8..+2 %).  Beyond that many for each kernel (dK,dV of 83
//            heads of 680 tokens, another card, 18.6 -> 19.0) it does not pay
inline UnitMap launch_map(int num_cus, int n_items, int n_heads, const Order& order) {
    const int cus = num_cus / 8, n_groups = n_heads / 8;                    // of an XCD; heads of an XCD
    int tail = tail_groups_for(num_cus, n_items);
    if (HMAR_TUNE_HALF_BATCH && (n_items < order.half_below || (n_items < order.half_whole_below && tail >= n_groups))) tail = std::max(1, tail / 2);
    if ((long long)(n_groups - tail) * n_items >= cus) return unit_map_for(n_items, n_heads, tail);
    const long long units = (long long)n_items * n_heads;
    const bool turned = HMAR_TUNE_TURN && units > num_cus && units <= 8LL * order.turn_rounds * cus;
    return unit_map_for(n_items, n_heads, std::max(1, n_groups), turned ? cus : 0);
}

// Workgroups of a launch over n_items items of each head, or 0 if they would be too many for a grid.
inline unsigned launch_groups(int n_items, int n_heads) {
    if (n_items < 1 || n_heads < 1 || 8LL * ((n_heads + 7LL) / 8) * n_items > 0x7fffffffLL) return 0;
    return (unsigned)n_items * (unsigned)n_heads;
}

// Whether a forward launch leaves the maxima of most tiles out (csrc/fwd.hip; no bits depend on it): streams of 16 tiles
// and more, and work for 7/4 of its longest items on every compute unit.  Time against taking every maximum, at
// `fill` = tiles of the launch / (tiles of the longest item * compute units), 256 compute units:
//   19 to 100 tiles: fill 0.2 to 1.0 +9..12 %, 1.1 to 1.4 -2..+11 %, 1.5 to 1.7 -4..+5 %, 1.8 to 2.6 -5..+1.5 %, beyond
//     -1..-8 % (25 tiles, fill 9.3: 141 -> 139 us; 100 tiles, fill 8.3: 480 -> 464; equal items of 25 tiles, 2.25: 49.5 ->
//     48.3): on few wavefronts the second contraction waits for the sum, on many the vector instructions count;
//   7 to 13 tiles: up to +11 % below 1.5, then -2..+2 %, on full chips -2 %: they keep the plain form.
#ifndef HMAR_TUNE_LONG_STREAM
#define HMAR_TUNE_LONG_STREAM 16           // measurement builds: where long streams begin
#endif
inline bool leaves_maxima_out(int max_tiles, long long total_tiles, int n_heads, int num_cus) {
    return max_tiles >= HMAR_TUNE_LONG_STREAM && 4 * total_tiles * n_heads >= 7LL * num_cus * max_tiles;
}

// Whether a forward of the training shapes that takes every maximum requests all key operands of a tile ahead of its first
// contraction (csrc/fwd.hip; no bits depend on it).  That shortens the chain of a workgroup that has its compute unit to
// itself; where two long chains share one (their wavefronts the same SIMDs), each covers the other's waits and the earlier
// reads only get in the way.  `long units` = heads * items up to the last long one.  Time with the compiler's order / ahead,
// geometric mean (least .. most), 256 compute units, by long units per compute unit:
//   up to 1:   1.05 (0.99..1.06) for 16 to 64 tiles, 1.04 (0.98..1.06) for 3 to 15, 1.00 for fewer; 4 heads of 2240 tokens
//              25.6 -> 24.1 us, 32 of 680 tokens 11.6 -> 11.2
//   1 .. 2:    0.95 (0.92..0.98) and 0.99 (0.94..1.02); 14 heads of 64, 256, 784, 1296 tokens a scale 37.3 -> 40.1 us, 10 of 4089
//              tokens 72.4 -> 75.9
//   beyond 2:  0.96 and 1.00 (0.91..1.04): no difference on short streams
inline bool keys_ahead(int max_tiles, int long_items, int n_heads, int num_cus) {
    const long long units = (long long)long_items * n_heads;
    return HMAR_TUNE_KEYS_AHEAD && (units <= num_cus || (max_tiles < HMAR_TUNE_LONG_STREAM && units > 2LL * num_cus));
}

// Whether the wavefronts of a launch ask for their own rows as whole rows and turn them round (request_rows in
// csrc/device_common.h; no bits depend on it).  So they cost less address work (a dQ workgroup asks for 48 loads ahead of
// its first tile), which is what a workgroup's start waits for while the launch leaves the chip room; on a fuller chip it
// waits for memory, and the detour through LDS comes on top.  The backward of short streams, mostly starts with two
// or three operands each, still gains there.  (A switch inside the kernels costs launches of either kind 1 to 2 %: they are
// built twice.)  In operand layout -> as whole rows, us, by workgroups per compute unit:
//   forward: 1.8 12.4 -> 12.0 (64 heads of 680 tokens), 3.6 19.5 -> 20.1, 21 72.1 -> 72.4; where maxima are left out 142.2 ->
//     145.6 (192 heads of 2240 tokens); steps: 0.4 8.85 -> 8.60 (48 heads, 256 queries, 425 keys), 6 23.9 -> 25.5 (1536 heads,
//     100 queries, 164 keys)
//   dQ, 7 tiles: 1.8 14.7 -> 13.7, 21 90.6 -> 88.4; dK/dV, 7 tiles: 1.8 16.0 -> 15.4, 3.6 26.9 -> 25.5, 21 127.1 -> 126.5
// and the whole backward, geometric mean (least .. most) of 540 schedules, both masks:
//   workgroups     2 .. 3             3 .. 4             4 .. 5.5           5.5 .. 7           7 .. 9
//    1 to 7 tiles  0.98 (0.96..1.00)  0.96 (0.92..1.01)  0.99 (0.95..1.05)  0.98 (0.94..1.02)  0.98 (0.95..1.03)
//    8 to 15       0.99 (0.96..1.00)  0.99 (0.96..1.04)  1.00 (0.98..1.02)  1.00 (0.97..1.02)  0.99 (0.96..1.01)
//   16 to 35       0.99 (0.98..1.01)  1.00 (0.99..1.01)  1.01 (0.99..1.02)  1.01 (0.99..1.03)  1.00 (0.99..1.02)
//   36 to 64       1.00 (0.99..1.01)  1.01 (1.00..1.01)  1.01 (1.00..1.02)  1.02 (1.00..1.03)  1.01 (1.00..1.02)
constexpr int kShortStream = 16;
inline bool whole_rows_fwd(long long units, int num_cus) { return HMAR_TUNE_WHOLE_ROWS && units <= 3LL * num_cus; }
inline bool whole_rows_dq(long long units, int max_tiles, int num_cus) {
    return HMAR_TUNE_WHOLE_ROWS && (units <= 3LL * num_cus || max_tiles < kShortStream);
}
inline bool whole_rows_dkdv(long long units, int max_tiles, int num_cus) {
    return HMAR_TUNE_WHOLE_ROWS && (units <= 2LL * num_cus || max_tiles < kShortStream);
}

// Whether a backward is one launch of both kernels' items (hmar_bwd_both_kernel; no bits depend on it): work for at
// most two of the longest items on every compute unit, 9/5 of them where streams are long, and windows whose statistics
// fit the LDS of two workgroups per compute unit.  What it saves is a launch and the wait for the first kernel's last item;
// what it costs is that dQ items run two to a compute unit, not four, and that a window is read twice, which weighs
// more the longer the streams.  Time of two launches / of one, geometric mean (least .. most) over
// schedules of both masks, by `fill` = tiles of both lists / (tiles of the longest item * compute units), 256 compute units:
//   fill             up to 1.1          1.1 .. 1.5         1.5 .. 1.8         1.8 .. 2
//    1 to 7 tiles    1.64 (1.39..1.76)  1.38 (1.24..1.59)  1.30 (1.20..1.53)  1.22 (1.03..1.53)
//    8 to 15         1.53 (1.18..1.68)  1.21 (1.12..1.40)  1.19 (0.99..1.39)  1.09 (0.95..1.26)
//   16 to 25         1.51 (1.21..1.60)  1.17 (1.08..1.36)  1.14 (0.95..1.39)  1.03 (0.91..1.26)
//   26 to 32         1.47 (1.16..1.55)  1.12 (1.05..1.28)  1.10 (1.02..1.22)  1.01 (0.90..1.19)
//   33 to 64         1.45 (1.11..1.59)  1.10 (1.00..1.25)  1.07 (0.91..1.22)  0.97 (0.86..1.06)
constexpr int kBothMaxTiles = 64;          // tiles a dK/dV item may visit
constexpr int kBothLongTiles = 33;         // from where on streams are long
#ifndef HMAR_TUNE_BOTH_FILL
#define HMAR_TUNE_BOTH_FILL 2              // measurement builds: the line for short streams (0: always two launches)
#endif
inline bool one_backward_launch(const DeviceSchedule& s, int n_heads) {
    const long long total = (s.total_tiles[0] + s.total_tiles[1]) * n_heads, longest = std::max(s.max_tiles[0], s.max_tiles[1]);
    const int tenths = 10 * HMAR_TUNE_BOTH_FILL - (longest >= kBothLongTiles ? 2 : 0);
    return s.n_items[0] == s.n_items[1] && s.max_tiles[1] <= kBothMaxTiles && 10 * total <= tenths * longest * s.num_cus;
}

// Per-kernel event bracketing for hmar_profile_begin/end (no-ops unless profiling is on).
enum KernelId { kKernelFwd = 0, kKernelDkDv = 1, kKernelDq = 2, kNumKernels = 3 };
void profile_before(int kernel_id, hipStream_t stream);
void profile_after(int kernel_id, hipStream_t stream);

// Up to kMaxSteps independent inference steps in one launch (host view; the launcher turns it
// into kernel arguments).  Steps must be ordered by decreasing work.
constexpr int kMaxSteps = 16;
struct StepLaunch {
    struct Step {
        const void* Q; const void* K; const void* V; void* O; float* LSE;
        const int32_t* rows;    // device, optional: the n_q rows of Q/O/LSE the step covers
        int32_t n_q, q_stride, Lk;
    } step[kMaxSteps];
    int32_t n_steps;
};
hipError_t launch_fwd_steps(const StepLaunch& L, int n_heads, float sm_scale, int num_cus, hipStream_t stream);

hipError_t launch_fwd(const void* Q, const void* K, const void* V, void* O, float* LSE,
                      const DeviceSchedule& s, int n_heads, float sm_scale, hipStream_t stream);

hipError_t launch_bwd(const void* Q, const void* K, const void* V, const void* O, const void* dO,
                      const float* LSE, void* dQ, void* dK, void* dV, float* workspace,
                      const DeviceSchedule& s, int n_heads, float sm_scale, hipStream_t stream);

hipError_t launch_copy(void* dst, const void* src, size_t bytes, hipStream_t stream);

}  // namespace hmar
