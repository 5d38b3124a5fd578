// Backward kernels of the Markovian next-scale attention (paper Sec. "Efficient Markovian Next-Scale Prediction", appendix "Efficient Attention Performance") for gfx950.
//
//   hmar_dq_kernel    : query-stationary, same walk as the forward but over the heads in reverse
//                       order (the forward before it and the dK/dV kernel after it both walk
//                       forwards, so each kernel begins where its predecessor ended).  First
//                       forms, for its own rows, -Delta_i = -sum_d dO_id O_id and
//                       -LSE_i * log2(e) and leaves them in the workspace for the dK/dV kernel
//                       (launched after it).  Recomputes P^T = exp(S^T - LSE), dP^T = V dO^T,
//                       dS^T = P^T o (dP^T - Delta) and accumulates dQ^T += K^T dS^T.
//   hmar_dkdv_kernel  : key-stationary, walks the transposed schedule (a key of scale k is
//                       seen by the queries of scales k and k+1).  Recomputes P and dS with
//                       the keys in the lane dimension and accumulates dV^T += dO^T P,
//                       dK^T += Q^T dS.
//   hmar_bwd_both_kernel: both kernels' items in one launch, for backwards that leave the chip room.
// Both main kernels recompute the probabilities, so no gradient is accumulated across
// workgroups: results are deterministic and nothing needs zero-initialising.  Streamed
// tiles are row-major in LDS and serve both as row-wise operands (S, dP) and, through the
// LDS transpose load, as transposed operands (dQ, dK, dV).
#include <algorithm>
#include <type_traits>

#include "device_common.h"
#include "kernels.h"

namespace hmar {

struct BwdParams {
    const __bf16* Q; const __bf16* K; const __bf16* V; const __bf16* dO;
    const __bf16* O; const float* LSE;
    float* neg_lse2;         // -LSE * log2(e): written by the dQ kernel, read by the dK/dV kernel
    float* neg_delta;        // -Delta: likewise
    __bf16* dQ; __bf16* dK; __bf16* dV;
    const Item* items; const int32_t* row_lo; const int32_t* row_hi;
    UnitMap map;
    int L;
    float c;          // sm_scale * log2(e)
    float sm_scale;
};

// ------------------------------------------------------------------------------------- dQ
#ifndef HMAR_DQ_MIN_WAVES
#define HMAR_DQ_MIN_WAVES 4
#endif
// acc + the dot product of eight elements of an O row with those of the dO row: two products per instruction
// (v_dot2c_f32_bf16), fp32 accumulation
__device__ __forceinline__ float delta_of_chunk(bf16x8 o, bf16x8 g, float acc) {
    acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(o, o, 0, 1), __builtin_shufflevector(g, g, 0, 1), acc, false);
    acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(o, o, 2, 3), __builtin_shufflevector(g, g, 2, 3), acc, false);
    acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(o, o, 4, 5), __builtin_shufflevector(g, g, 4, 5), acc, false);
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(o, o, 6, 7), __builtin_shufflevector(g, g, 6, 7), acc, false);
}
// -Delta of a row from the lane's half of it: chunks h, 2 + h, 4 + h, 6 + h of the row's eight
__device__ __forceinline__ float neg_delta_of_row(const OwnRows& o, const OwnRows& dob) {
    float acc = 0.f;
#pragma unroll
    for (int t = 0; t < 4; ++t) acc = delta_of_chunk(o.chunk[t], dob.chunk[t], acc);
    return -half_sum(acc);
}

// The statistics of a tile of 64 rows, formed by the four wavefronts of a workgroup, 16 rows each, 8 rows per load with a
// chunk of a row per lane: whole cache lines (two lanes per row, as above, make a load touch 32 of them: 3.0 us for the
// 425 rows that an item of the 680-token schedule visits, against 1.5).  The sum of a row is handed from lane to lane in
// the order of neg_delta_of_row, so that the bits are the same.
struct TileStats {
    bf16x8 o[2], g[2];
    float lse[2];
    __device__ __forceinline__ void request(const __bf16* O, const __bf16* dO, const float* LSE, int row0, int row_max, int lane, int wave) {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const size_t row = min(row0 + 16 * wave + 8 * j + (lane >> 3), row_max);
            o[j] = *reinterpret_cast<const bf16x8*>(O + row * kD + 8 * (lane & 7));
            g[j] = *reinterpret_cast<const bf16x8*>(dO + row * kD + 8 * (lane & 7));
            lse[j] = LSE[row];
        }
    }
    __device__ __forceinline__ void form(float* nl2, float* delta, int lane, int wave) const {
        float acc[2] = {0.f, 0.f};
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                // from the lane two to the left (row_shr:2); after step t the lanes of chunks 2t, 2t + 1 hold theirs
                if (t > 0) acc[j] = __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, acc[j]), 0x112, 0xf, 0xf, true));
                acc[j] = delta_of_chunk(o[j], g[j], acc[j]);
            }
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const float other = __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, acc[j]), 0xB1, 0xf, 0xf, true));
            if ((lane & 7) == 7) {
                const int r = 16 * wave + 8 * j + (lane >> 3);
                delta[r] = -(acc[j] + other);
                nl2[r] = -lse[j] * kLog2e;
            }
        }
    }
};

// The work of one dQ item.  smem: ring of 2 stages, each a K tile followed by a V tile.
// Where the row statistics come from: formed here and left in the workspace for the dK/dV kernel, formed here
// for this item alone, or read from the workspace.
enum class Stats { kFormAndLeave, kForm, kRead };
template <Stats STATS, bool WHOLE>
__device__ __forceinline__ void dq_body(const BwdParams& p, const Item it, const int32_t* row_lo, const int32_t* row_hi,
                                        int head, int item_id, char* smem) {
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lr = lane & 31, h = lane >> 5;
    const size_t head_off = (size_t)head * p.L * kD;
    const size_t head_in = (size_t)HMAR_INPUT_HEAD(head) * p.L * kD;     // == head_off outside measurements
    const __bf16* Kh = p.K + head_in;
    const __bf16* Vh = p.V + head_in;
    const LaneOffsets lo_ = make_lane_offsets(lane, wave);
    const uint32_t smem_base = lds_address(smem);

    const int k_begin = it.other_begin, k_end = it.other_end, kmax = k_end - 1;
    const int ntiles = (k_end - k_begin + kTile - 1) / kTile;

    auto issue = [&](int ti, int st) {       // 4 DMA loads per lane and tile
        const uint32_t stage = smem_base + st * (2 * kTileBytes);
        dma_tile(Kh, k_begin + ti * kTile, kmax, stage, lo_, lane, wave);
        dma_tile(Vh, k_begin + ti * kTile, kmax, stage + kTileBytes, lo_, lane, wave);
    };
    issue(0, 0);

    const int wq0 = it.own_begin + wave * kRowsPerWave;
    const bool wave_active = wq0 < it.own_end;
    const int qrow = min(wq0 + lr, it.own_end - 1);
    const int lo = row_lo[qrow], hi = row_hi[qrow];
    // pair ranges never decrease along the rows: the wavefront's extremes are at its first and last row
    const int rfirst = min(wq0, it.own_end - 1), rlast = min(wq0 + kRowsPerWave - 1, it.own_end - 1);
    const int wlo = row_lo[rfirst], whi = row_hi[rlast];        // union of the wavefront's ranges
    const int full_lo = row_lo[rlast], full_hi = row_hi[rfirst];  // what every one of its rows pairs with

    const uint32_t patch = smem_base + 2 * kTileBytes + wave * 4096;      // in the stage that no load runs into before the barrier
    auto own = [&](int r) { return min(wq0 + r, it.own_end - 1); };
    OwnRows q = request_rows<WHOLE>(p.Q + head_in, qrow, own, lane), dob = request_rows<WHOLE>(p.dO + head_in, qrow, own, lane);
    float nl2, ndelta;
    if constexpr (STATS != Stats::kRead) {
        OwnRows o = request_rows<WHOLE>(p.O + head_in, qrow, own, lane);
        nl2 = -p.LSE[(size_t)HMAR_INPUT_HEAD(head) * p.L + qrow] * kLog2e;
        turn_rows<WHOLE>(patch, q, lo_, lane);
        turn_rows<WHOLE>(patch, dob, lo_, lane);
        turn_rows<WHOLE>(patch, o, lo_, lane);
        ndelta = neg_delta_of_row(o, dob);
        if (STATS == Stats::kFormAndLeave && wq0 + lr < it.own_end && h == 0) {
            p.neg_lse2[(size_t)head * p.L + qrow] = nl2;
            p.neg_delta[(size_t)head * p.L + qrow] = ndelta;
        }
    } else {
        nl2 = p.neg_lse2[(size_t)head * p.L + qrow];
        ndelta = p.neg_delta[(size_t)head * p.L + qrow];
        turn_rows<WHOLE>(patch, q, lo_, lane);
        turn_rows<WHOLE>(patch, dob, lo_, lane);
    }

    f32x16 dq[2];
#pragma unroll
    for (int mb = 0; mb < 2; ++mb)
#pragma unroll
        for (int i = 0; i < 16; ++i) dq[mb][i] = 0.f;

    // make the compiler wait for these registers here, not inside the loop (see the forward);
    // loads complete in order, so tile 0 has landed as well
    asm volatile("" :: "v"(q.chunk[0]), "v"(q.chunk[1]), "v"(q.chunk[2]), "v"(q.chunk[3]), "v"(dob.chunk[0]), "v"(dob.chunk[1]),
                 "v"(dob.chunk[2]), "v"(dob.chunk[3]), "v"(nl2), "v"(ndelta));
    HMAR_WAIT_DMA_AND_BARRIER(0);

    // one tile: request the next one, compute, wait for the request; the stage is a template
    // constant so that every LDS address of the step is a per-lane register plus an immediate
    auto tile_step = [&](const int ti, auto stage_c) {
        constexpr int ST = decltype(stage_c)::value;
        const int kt = k_begin + ti * kTile;
        if (ti + 1 < ntiles) issue(ti + 1, ST ^ 1);
#ifdef HMAR_TUNE_NO_COMPUTE_DQ
        if (false) {
#else
        if (wave_active && kt < whi && kt + kTile > wlo) {
#endif
            const uint32_t Kt = smem_base + ST * (2 * kTileBytes);
            const uint32_t Vt = Kt + kTileBytes;
            const bool need_lo = kt < full_lo, need_hi = kt + kTile > full_hi;
            const int lim_lo = lo - kt - 4 * h, lim_hi = hi - kt - 4 * h;
#pragma unroll
            for (int kb = 0; kb < 2; ++kb) {
                // (no explicit operand staging here: at 4 wavefronts per SIMD the extra
                // registers cost more in occupancy than the batched LDS reads gain)
                f32x16 s, dp;
#pragma unroll
                for (int i = 0; i < 16; ++i) { s[i] = 0.f; dp[i] = 0.f; }
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    s = mfma32(lds_a_row(Kt, lo_, kb, t), q.chunk[t], s);
                    dp = mfma32(lds_a_row(Vt, lo_, kb, t), dob.chunk[t], dp);
                }
                mask_block(s, 32 * kb, lim_lo, lim_hi, need_lo, need_hi);     // exp2(-inf) = 0
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const float pv = __builtin_amdgcn_exp2f(__builtin_fmaf(s[i], p.c, nl2));
                    s[i] = pv * (dp[i] + ndelta);
                }
#pragma unroll
                for (int sub = 0; sub < 2; ++sub) {
                    const int e0 = 8 * sub, tp = 2 * kb + sub;
                    const bf16x8 dsb = pack8(s[e0 + 0], s[e0 + 1], s[e0 + 2], s[e0 + 3],
                                             s[e0 + 4], s[e0 + 5], s[e0 + 6], s[e0 + 7]);
#pragma unroll
                    for (int mb = 0; mb < 2; ++mb)
                        dq[mb] = mfma32(lds_a_tr(Kt, lo_, mb, tp), dsb, dq[mb]);
                }
            }
        }
        HMAR_WAIT_DMA_AND_BARRIER(0);     // the tile requested above has landed and this one is free
    };
    for (int ti = 0; ti < ntiles; ti += 2) {
        tile_step(ti, std::integral_constant<int, 0>{});
        if (ti + 1 >= ntiles) break;
        tile_step(ti + 1, std::integral_constant<int, 1>{});
    }

    if (wave_active)
        store_block_rows(smem_base + wave * kPatchBytes, dq, p.sm_scale, p.dQ + head_off, wq0, it.own_end - wq0, lane, nullptr, HMAR_NT_GRADS != 0);
}

template <bool WHOLE>
__global__ __launch_bounds__(kThreads, HMAR_DQ_MIN_WAVES) void hmar_dq_kernel(BwdParams p) {
    __shared__ __attribute__((aligned(1024))) char smem[2 * 2 * kTileBytes];
#ifdef HMAR_TUNE_LDS_PAD_DQ
    HMAR_TUNE_LDS_PAD(HMAR_TUNE_LDS_PAD_DQ)
#endif
    int head, item_id;
    map_workgroup(p.map, &head, &item_id, true);
    dq_body<Stats::kFormAndLeave, WHOLE>(p, p.items[item_id], p.row_lo, p.row_hi, head, item_id, smem);
}

// ---------------------------------------------------------------------------------- dK, dV
// Register budget: the two result accumulators, the own K and V rows, both blocks' scores and
// the batched LDS operands need about 250 VGPRs, which means two wavefronts per SIMD (two
// workgroups per CU); the leanest form of the kernel would still need about 190, more than
// the 168 that three wavefronts allow.
#ifndef HMAR_DKDV_MIN_WAVES
#define HMAR_DKDV_MIN_WAVES 2
#endif
// One tile of the dK/dV computation: the wavefront's 32 keys (rows kreg, vreg) against the 64
// query rows of the tile at LDS addresses Qt (Q) and Gt (dO), whose statistics are at nl2_t and
// delta_t.  lim_lo, lim_hi: the lane's key pairs with tile rows [lim_lo + 4h, lim_hi + 4h).
__device__ __forceinline__ void dkdv_tile(uint32_t Qt, uint32_t Gt, uint32_t nl2_t, uint32_t delta_t,
                                          const bf16x8 (&kreg)[4], const bf16x8 (&vreg)[4], f32x16 (&dk)[2], f32x16 (&dv)[2],
                                          int lim_lo, int lim_hi, bool need_lo, bool need_hi, float c,
                                          const LaneOffsets& lo_) {
    // Operands are fetched from LDS in batches ahead of the contractions that use them
    // (the scheduling barriers keep the compiler from sinking each read next to its use,
    // which would expose the LDS latency once per matrix instruction).  The score and dP
    // contractions of both 32-query blocks are issued first, so that the matrix pipe works
    // on the second block while the vector units form the first block's probabilities.
    f32x16 s[2], dp[2];
#pragma unroll
    for (int qb = 0; qb < 2; ++qb) {
        bf16x8 aq[4], ag[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            aq[t] = lds_a_row(Qt, lo_, qb, t);
            ag[t] = lds_a_row(Gt, lo_, qb, t);
        }
        // statistics of the block's query rows 32qb + 8j + 4h + r (register 4j + r):
        // -Delta seeds the dP accumulator, so dP - Delta costs no vector instruction
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const f32x4 d4 = *(lds_f32x4*)(delta_t + (32 * qb + 8 * j) * 4);
#pragma unroll
            for (int r = 0; r < 4; ++r) { s[qb][4 * j + r] = 0.f; dp[qb][4 * j + r] = d4[r]; }
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            s[qb] = mfma32(aq[t], kreg[t], s[qb]);
            dp[qb] = mfma32(ag[t], vreg[t], dp[qb]);
        }
    }
#pragma unroll
    for (int qb = 0; qb < 2; ++qb) {
        // transposed operands of the second pair of contractions and the row statistics,
        // requested before the exponentials so that their latency hides behind them
        bf16x8 tg[2][2], tq[2][2];
        f32x4 l4[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) l4[j] = *(lds_f32x4*)(nl2_t + (32 * qb + 8 * j) * 4);
#pragma unroll
        for (int sub = 0; sub < 2; ++sub)
#pragma unroll
            for (int mb = 0; mb < 2; ++mb) {
                tg[sub][mb] = lds_a_tr(Gt, lo_, mb, 2 * qb + sub);
                tq[sub][mb] = lds_a_tr(Qt, lo_, mb, 2 * qb + sub);
            }
        __builtin_amdgcn_sched_barrier(0);
        mask_block(s[qb], 32 * qb, lim_lo, lim_hi, need_lo, need_hi);
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int i = 4 * j + r;
                const float pv = __builtin_amdgcn_exp2f(__builtin_fmaf(s[qb][i], c, l4[j][r]));
                s[qb][i] = pv;
                dp[qb][i] = pv * dp[qb][i];
            }
#pragma unroll
        for (int sub = 0; sub < 2; ++sub) {
            const int e0 = 8 * sub;
            const bf16x8 pb = pack8(s[qb][e0 + 0], s[qb][e0 + 1], s[qb][e0 + 2], s[qb][e0 + 3],
                                    s[qb][e0 + 4], s[qb][e0 + 5], s[qb][e0 + 6], s[qb][e0 + 7]);
            const bf16x8 dsb = pack8(dp[qb][e0 + 0], dp[qb][e0 + 1], dp[qb][e0 + 2], dp[qb][e0 + 3],
                                     dp[qb][e0 + 4], dp[qb][e0 + 5], dp[qb][e0 + 6], dp[qb][e0 + 7]);
#pragma unroll
            for (int mb = 0; mb < 2; ++mb) {
                dv[mb] = mfma32(tg[sub][mb], pb, dv[mb]);
                dk[mb] = mfma32(tq[sub][mb], dsb, dk[mb]);
            }
        }
    }
}

// The work of one dK/dV item.  smem: ring of 2 stages, each a Q tile followed by a dO tile;
// nl2_s, delta_s: the statistics of the tiles' rows: of the two stages, streamed with them from the workspace, or
// (STATS == kForm) of all tiles, formed here before the first step.
template <Stats STATS, bool WHOLE>
__device__ __forceinline__ void dkdv_body(const BwdParams& p, const Item it, const int32_t* row_lo, const int32_t* row_hi,
                                          int head, int item_id, char* smem, float (*nl2_s)[kTile], float (*delta_s)[kTile]) {
    static_assert(STATS != Stats::kFormAndLeave, "the dQ kernel leaves them");
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lr = lane & 31, h = lane >> 5;
    const size_t head_off = (size_t)head * p.L * kD;
    const size_t head_in = (size_t)HMAR_INPUT_HEAD(head) * p.L * kD;     // == head_off outside measurements
    const __bf16* Qh = p.Q + head_in;
    const __bf16* Gh = p.dO + head_in;
    const float* NLh = p.neg_lse2 + (size_t)head * p.L;
    const float* Dh = p.neg_delta + (size_t)head * p.L;
    const LaneOffsets lo_ = make_lane_offsets(lane, wave);
    const uint32_t smem_base = lds_address(smem);
    const uint32_t nl2_base = lds_address(nl2_s), delta_base = lds_address(delta_s);

    const int q_begin = it.other_begin, q_end = it.other_end, qmax = q_end - 1;
    const int ntiles = (q_end - q_begin + kTile - 1) / kTile;

    // per lane and tile: 4 DMA loads, plus one for wavefronts 0 (-LSE*log2e) and 1 (Delta)
    auto issue = [&](int ti, int st) {
        const uint32_t stage = smem_base + st * (2 * kTileBytes);
        const int qt = q_begin + ti * kTile;
        dma_tile(Qh, qt, qmax, stage, lo_, lane, wave);
        dma_tile(Gh, qt, qmax, stage + kTileBytes, lo_, lane, wave);
        if constexpr (STATS == Stats::kRead) {
            if (wave == 0) dma_floats(NLh, qt, qmax, nl2_base + st * (kTile * 4), lane);
            else if (wave == 1) dma_floats(Dh, qt, qmax, delta_base + st * (kTile * 4), lane);
        }
    };
    issue(0, 0);

    const int wk0 = it.own_begin + wave * kRowsPerWave;
    const bool wave_active = wk0 < it.own_end;
    const int krow = min(wk0 + lr, it.own_end - 1);
    const int lo = row_lo[krow], hi = row_hi[krow];       // queries that see this key
    // pair ranges never decrease along the rows: the wavefront's extremes are at its first and last row
    const int rfirst = min(wk0, it.own_end - 1), rlast = min(wk0 + kRowsPerWave - 1, it.own_end - 1);
    const int wlo = row_lo[rfirst], whi = row_hi[rlast];        // union of the wavefront's ranges
    const int full_lo = row_lo[rlast], full_hi = row_hi[rfirst];  // what every one of its rows pairs with

    auto own = [&](int r) { return min(wk0 + r, it.own_end - 1); };
    OwnRows krows = request_rows<WHOLE>(p.K + head_in, krow, own, lane), vrows = request_rows<WHOLE>(p.V + head_in, krow, own, lane);

    if constexpr (STATS == Stats::kForm) {
        constexpr int kStatsAhead = 4;      // tiles whose rows are requested together; 2: +0.2 us, 7: the same
        // rows past the last one get the last one's statistics, as they get its row (finite: their probabilities are 0)
        for (int t0 = 0; t0 < ntiles; t0 += kStatsAhead) {
            TileStats stats[kStatsAhead];
#pragma unroll
            for (int j = 0; j < kStatsAhead; ++j)
                stats[j].request(p.O + head_in, Gh, p.LSE + (size_t)HMAR_INPUT_HEAD(head) * p.L, q_begin + (t0 + j) * kTile, qmax, lane, wave);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int j = 0; j < kStatsAhead; ++j)
                if (t0 + j < ntiles) stats[j].form(nl2_s[t0 + j], delta_s[t0 + j], lane, wave);
        }
    }

    f32x16 dk[2], dv[2];
#pragma unroll
    for (int mb = 0; mb < 2; ++mb)
#pragma unroll
        for (int i = 0; i < 16; ++i) { dk[mb][i] = 0.f; dv[mb][i] = 0.f; }

    const uint32_t patch = smem_base + 2 * kTileBytes + wave * 4096;      // in the stage that no load runs into before the barrier
    turn_rows<WHOLE>(patch, krows, lo_, lane);
    turn_rows<WHOLE>(patch, vrows, lo_, lane);
    const bf16x8 (&kreg)[4] = krows.chunk, (&vreg)[4] = vrows.chunk;
    asm volatile("" :: "v"(kreg[0]), "v"(kreg[1]), "v"(kreg[2]), "v"(kreg[3]), "v"(vreg[0]), "v"(vreg[1]),
                 "v"(vreg[2]), "v"(vreg[3]));
    HMAR_WAIT_DMA_AND_BARRIER(0);

    auto tile_step = [&](const int ti, auto stage_c) {     // see the dQ kernel
        constexpr int ST = decltype(stage_c)::value;
        const int qt = q_begin + ti * kTile;
        if (ti + 1 < ntiles) issue(ti + 1, ST ^ 1);
#ifdef HMAR_TUNE_NO_COMPUTE_DKDV
        if (false) {
#else
        if (wave_active && qt < whi && qt + kTile > wlo) {
#endif
            const uint32_t Qt = smem_base + ST * (2 * kTileBytes);
            const uint32_t stats = (STATS == Stats::kForm ? ti : ST) * (kTile * 4) + 16 * h;
            const uint32_t nl2_t = nl2_base + stats, delta_t = delta_base + stats;
            dkdv_tile(Qt, Qt + kTileBytes, nl2_t, delta_t, kreg, vreg, dk, dv, lo - qt - 4 * h, hi - qt - 4 * h,
                      qt < full_lo, qt + kTile > full_hi, p.c, lo_);
        }
        HMAR_WAIT_DMA_AND_BARRIER(0);
    };
    for (int ti = 0; ti < ntiles; ti += 2) {
        tile_step(ti, std::integral_constant<int, 0>{});
        if (ti + 1 >= ntiles) break;
        tile_step(ti + 1, std::integral_constant<int, 1>{});
    }

    if (wave_active) {
        const uint32_t out = smem_base + wave * kPatchBytes;
        store_block_rows(out, dk, p.sm_scale, p.dK + head_off, wk0, it.own_end - wk0, lane, nullptr, HMAR_NT_GRADS != 0);
        store_block_rows(out, dv, 1.0f, p.dV + head_off, wk0, it.own_end - wk0, lane, nullptr, HMAR_NT_GRADS != 0);
    }
}

template <bool WHOLE>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(HMAR_DKDV_MIN_WAVES, HMAR_DKDV_MIN_WAVES))) void hmar_dkdv_kernel(BwdParams p) {
    __shared__ __attribute__((aligned(1024))) char smem[2 * 2 * kTileBytes];
    __shared__ __attribute__((aligned(256))) float nl2_s[2][kTile];
    __shared__ __attribute__((aligned(256))) float delta_s[2][kTile];
#ifdef HMAR_TUNE_LDS_PAD_DKDV
    HMAR_TUNE_LDS_PAD(HMAR_TUNE_LDS_PAD_DKDV)
#endif
    int head, item_id;
    map_workgroup(p.map, &head, &item_id);
    dkdv_body<Stats::kRead, WHOLE>(p, p.items[item_id], p.row_lo, p.row_hi, head, item_id, smem, nl2_s, delta_s);
}

// Both kernels' items in one launch, for launches too small to fill the chip, which are bound by the latency of one
// item's chain of tiles (about 1 us a tile) and of the launch itself.  What puts the dK/dV kernel behind the dQ
// kernel are the two row statistics; here every dK/dV item forms those of the rows it visits by itself, before its first
// step (in the step ahead of their use they cost registers: spills, 0.7 us a tile).  Both work lists hold the same number of
// items, heaviest first: the units of a head alternate between them.  32 heads of 680 tokens: 22.0 us in two
// launches, 14.4 in one; 4 heads 20.9 -> 12.5.  Where the line lies: one_backward_launch (csrc/kernels.h).
struct BwdBothParams {
    BwdParams p;                                    // items, row_lo, row_hi: of the dQ list; map: of both lists
    const Item* k_items; const int32_t* k_row_lo; const int32_t* k_row_hi;
};
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(HMAR_DKDV_MIN_WAVES, HMAR_DKDV_MIN_WAVES))) void hmar_bwd_both_kernel(BwdBothParams b) {
    __shared__ __attribute__((aligned(1024))) char smem[2 * 2 * kTileBytes];
    __shared__ __attribute__((aligned(256))) float nl2_s[kBothMaxTiles][kTile];
    __shared__ __attribute__((aligned(256))) float delta_s[kBothMaxTiles][kTile];
    int head, unit;
    map_workgroup(b.p.map, &head, &unit);
    const int item_id = unit >> 1;
    if (unit & 1) dq_body<Stats::kForm, true>(b.p, b.p.items[item_id], b.p.row_lo, b.p.row_hi, head, item_id, smem);
    else          dkdv_body<Stats::kForm, true>(b.p, b.k_items[item_id], b.k_row_lo, b.k_row_hi, head, item_id, smem, nl2_s, delta_s);
}

#if defined(HMAR_BWD_MERGED)
#include "../tuning/bwd_merged.inc"
#endif
#if defined(HMAR_DKDV_PERSIST)
#include "../tuning/dkdv_persist.inc"
#endif

#if defined(HMAR_DKDV_PIPE) || (defined(HMAR_DKDV_KEYS_PER_WAVE) && HMAR_DKDV_KEYS_PER_WAVE == 16)
#include "../tuning/dkdv_variants.inc"
#endif

// Plain copy, 16 bytes per lane, grid-stride: calibration of the HBM traffic counters.
__global__ __launch_bounds__(256) void hmar_copy_kernel(u32x4* __restrict__ dst, const u32x4* __restrict__ src,
                                                        size_t n16) {
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n16; i += stride) dst[i] = src[i];
}

hipError_t launch_copy(void* dst, const void* src, size_t bytes, hipStream_t stream) {
    const size_t n16 = bytes / 16;
    if (n16 == 0) return hipSuccess;
    const size_t want = (n16 + 255) / 256;
    const unsigned groups = (unsigned)(want < 256 * 64 ? want : 256 * 64);
    hipLaunchKernelGGL(hmar_copy_kernel, dim3(groups), dim3(256), 0, stream, static_cast<u32x4*>(dst),
                       static_cast<const u32x4*>(src), n16);
    return hipGetLastError();
}

#ifndef HMAR_DKDV_KEYS_PER_WAVE
#define HMAR_DKDV_KEYS_PER_WAVE 32
#endif

hipError_t launch_bwd(const void* Q, const void* K, const void* V, const void* O, const void* dO,
                      const float* LSE, void* dQ, void* dK, void* dV, float* workspace,
                      const DeviceSchedule& s, int n_heads, float sm_scale, hipStream_t stream) {
    const long long n_rows = (long long)n_heads * s.L;
    BwdParams p;
    p.Q = static_cast<const __bf16*>(Q);
    p.K = static_cast<const __bf16*>(K);
    p.V = static_cast<const __bf16*>(V);
    p.dO = static_cast<const __bf16*>(dO);
    p.O = static_cast<const __bf16*>(O);
    p.LSE = LSE;
    p.neg_delta = workspace;
    p.neg_lse2 = workspace + n_rows;
    p.dQ = static_cast<__bf16*>(dQ);
    p.dK = static_cast<__bf16*>(dK);
    p.dV = static_cast<__bf16*>(dV);
    p.L = s.L;
    p.c = sm_scale * kLog2e;
    p.sm_scale = sm_scale;

#if defined(HMAR_BWD_MERGED)
    return launch_bwd_merged(p, s, n_heads, stream);
#endif
    if (one_backward_launch(s, n_heads)) {
        BwdBothParams b;
        b.k_items = static_cast<const Item*>(s.items[1]);
        b.k_row_lo = s.row_lo[1];
        b.k_row_hi = s.row_hi[1];
        p.items = static_cast<const Item*>(s.items[0]);
        p.row_lo = s.row_lo[0];
        p.row_hi = s.row_hi[0];
        const int units = s.n_items[0] + s.n_items[1];
        p.map = launch_map(s.num_cus, units, n_heads, kOrderDkDv);
        b.p = p;
        profile_before(kKernelDkDv, stream);
        hipLaunchKernelGGL(hmar_bwd_both_kernel, dim3(launch_groups(units, n_heads)), dim3(kThreads), 0, stream, b);
        const hipError_t e = hipGetLastError();
        profile_after(kKernelDkDv, stream);
        return e;
    }
    // dQ first: it also produces the per-row statistics the dK/dV kernel streams
    for (int dir = 0; dir < 2; ++dir) {
        p.items = static_cast<const Item*>(s.items[dir]);
        p.row_lo = s.row_lo[dir];
        p.row_hi = s.row_hi[dir];
        const unsigned groups = launch_groups(s.n_items[dir], n_heads);
        if (groups == 0) return hipErrorInvalidValue;
        p.map = launch_map(s.num_cus, s.n_items[dir], n_heads, dir == 1 ? kOrderDkDv : kOrderDq);
        const bool whole = dir == 1 ? whole_rows_dkdv(groups, s.max_tiles[dir], s.num_cus) : whole_rows_dq(groups, s.max_tiles[dir], s.num_cus);
        const int kid = dir == 1 ? kKernelDkDv : kKernelDq;
        profile_before(kid, stream);
#if HMAR_DKDV_KEYS_PER_WAVE == 16
        if (dir == 1) hipLaunchKernelGGL(hmar_dkdv16_kernel, dim3(groups), dim3(kThreads16), 0, stream, p);
#elif defined(HMAR_DKDV_PIPE)
        if (dir == 1) hipLaunchKernelGGL(hmar_dkdv_pipe_kernel, dim3(groups), dim3(kThreads), 0, stream, p);
#elif defined(HMAR_DKDV_PERSIST)
        if (dir == 1) {
            const long long resident = 2LL * s.num_cus / 8 * 8;       // two workgroups per CU, a multiple of 8
            hipLaunchKernelGGL(hmar_dkdv_persist_kernel, dim3((unsigned)std::min((long long)groups, resident)), dim3(kThreads), 0, stream,
                               p, (int)groups);
        }
#else
        if (dir == 1) hipLaunchKernelGGL(whole ? hmar_dkdv_kernel<true> : hmar_dkdv_kernel<false>, dim3(groups), dim3(kThreads), 0, stream, p);
#endif
        else          hipLaunchKernelGGL(whole ? hmar_dq_kernel<true> : hmar_dq_kernel<false>, dim3(groups), dim3(kThreads), 0, stream, p);
        const hipError_t e = hipGetLastError();
        profile_after(kid, stream);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace hmar
