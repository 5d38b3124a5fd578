// Launchers of the gfx950 kernels (internal to the library; the public ABI is hmar_attn.h).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace hmar {

// Device copy of the tile schedule of one (device, scale schedule) pair.
struct DeviceSchedule {
    const void* items[2];      // Item[n_items[dir]]
    int32_t n_items[2];
    int32_t max_tiles[2];      // streamed 64-row tiles of the longest item
    const int32_t* row_lo[2];  // L entries
    const int32_t* row_hi[2];
    int32_t L;                 // rows of Q, O, LSE per head
    int32_t Lk;                // rows of K, V per head
    int32_t num_cus;           // compute units of the device the tables live on
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

// Workgroups of a launch over n_items items of each head (see map_unit), or 0 if they would be too many
// for a grid.
inline unsigned launch_groups(int n_items, int n_heads) {
    if (n_items < 1 || n_heads < 1 || 8LL * ((n_heads + 7LL) / 8) * n_items > 0x7fffffffLL) return 0;
    return 8u * ((unsigned)(n_heads / 8) * (unsigned)n_items + ((unsigned)(n_heads % 8) * (unsigned)n_items + 7) / 8);
}

// How a workgroup's wavefronts divide the work: rw of them own 32 rows each, ks such sets take every
// ks-th streamed tile and their results are added up at the end.  {4, 1} is the form for launches that
// fill the chip.  A launch of few (head, item) units leaves compute units empty or with one wavefront
// per SIMD, and then lasts as long as one workgroup needs for its tiles one after the other (1.3 us
// each); dividing the tiles shortens that chain, at one workgroup of 128 KB LDS (ks = 4) or two (ks = 2)
// per compute unit.
struct Split { int rw, ks; };
// The rules below: us measured as {4, 1} -> chosen, on 256 compute units; `units` counts 128-row items.
// A measurement build may name one form for all launches (-DHMAR_FORCE_SPLIT=Split{4,2}).
//
// Forward, steps and dQ (at most 128 VGPRs).  A short stream has too few tiles to divide.
//   up to half a unit per compute unit: 64-row halves, tiles by four.  7 tiles (256px), 70 units: 10.5 ->
//     8.3 forward, 11.9 -> 10.9 dQ; 25 tiles (512px), 120 units: 27.7 -> 15.4, 30.1 -> 17.8; 100 tiles
//     (8640 tokens), 68 units: 97.9 -> 42.9, 106.6 -> 49.0.  At 140 units of 7 tiles {4, 2} is ahead.
//   up to 5/4 and a long stream: tiles by four.  25 tiles, 240 units: 27.6 -> 19.8 ({4, 2}: 20.7); dQ has
//     more to do per tile and gains from it only on the longest, 100 tiles, 272 units: 111 -> 73 ({4, 2}: 78;
//     at 25 tiles 24.9 against 23.4).
//   tiles by two: long streams up to 2 (25 tiles, 480 units: 28.5 -> 25.7, dQ even; 100 tiles, 476 units: 102 ->
//     81, 120 -> 103; a refinement pass of 576 equal units is 4 % slower), shorter ones up to 5/4 and not for dQ
//     (7 tiles, 308 units: forward 11.6 -> 10.4, dQ 13.2 -> 13.0; 6 tiles, 384 units: 10.9 -> 11.3, dQ 9 % slower).
#ifndef HMAR_TUNE_LONG_STREAM
#define HMAR_TUNE_LONG_STREAM 16           // measurement builds: where long streams begin
#endif
constexpr int kLongStream = HMAR_TUNE_LONG_STREAM;      // tiles
inline Split choose_split(long long units, int max_tiles, int num_cus, bool dq) {
#ifdef HMAR_FORCE_SPLIT
    return HMAR_FORCE_SPLIT;
#endif
    if (max_tiles < 4) return {4, 1};          // 3 tiles: 6.4 -> 6.7
    if (2 * units <= num_cus) return {2, 4};
    const bool at_most_5_4 = 4 * units <= 5LL * num_cus;
    if (max_tiles < kLongStream) return at_most_5_4 && !dq ? Split{4, 2} : Split{4, 1};
    if (at_most_5_4 && (!dq || max_tiles >= 48)) return {4, 4};
    return units <= 2LL * num_cus ? Split{4, 2} : Split{4, 1};
}
// dK/dV (252 VGPRs: eight wavefronts fill a compute unit): 64-row halves.
//   long streams, up to half a unit per compute unit: tiles by four (25 tiles, 120 units: 30.9 -> 20.1; 100 tiles,
//     68 units: 107 -> 57);
//   tiles by two: long streams up to 5/4 (25 tiles, 300 units: 32.8 -> 29.2; 100 tiles, 272 units: 113 -> 86; 340 units
//     even), shorter ones up to 5/8 (7 tiles, 28 to 140 units: 11.8 -> 10.2; 168 units 11.7 -> 10.8; 196 even).
inline Split choose_split_dkdv(long long units, int max_tiles, int num_cus) {
#ifdef HMAR_FORCE_SPLIT_DKDV
    return HMAR_FORCE_SPLIT_DKDV;
#endif
    if (max_tiles < 4) return {4, 1};
    if (max_tiles < kLongStream) return 8 * units <= 5LL * num_cus ? Split{2, 2} : Split{4, 1};
    if (2 * units <= num_cus) return {2, 4};
    return 4 * units <= 5LL * num_cus ? Split{2, 2} : Split{4, 1};
}
// Call f with the split as two compile-time constants.
template <int RW, int KS, typename F>
void as_split(F&& f) { f(std::integral_constant<int, RW>{}, std::integral_constant<int, KS>{}); }
template <typename F>
void with_split(const Split& s, F&& f) {
    if (s.rw == 2) as_split<2, 4>(f);
    else if (s.ks == 4) as_split<4, 4>(f);
    else if (s.ks == 2) as_split<4, 2>(f);
    else as_split<4, 1>(f);
}
template <typename F>
void with_split_dkdv(const Split& s, F&& f) {
    if (s.rw == 4) as_split<4, 1>(f);
    else if (s.ks == 4) as_split<2, 4>(f);
    else as_split<2, 2>(f);
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
