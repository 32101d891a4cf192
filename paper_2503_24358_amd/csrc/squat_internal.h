// Internal helpers shared by the HIP sources of libsquat (not installed).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>

#include "squat.h"

namespace squat {

constexpr int kD = 128;            // head size supported by this version
constexpr int kWave = 64;          // CDNA wavefront
constexpr int kTileTokens = 32;    // tokens per wavefront tile (MFMA N dimension)
constexpr float kQuantFastOffset = 32.0f;   // per-token quantizers: largest |zero| / scale for which the one-multiply-add path is used

inline int elem_size(squat_dtype dt) {
    switch (dt) {
        case SQUAT_F32: return 4;
        case SQUAT_F16: return 2;
        case SQUAT_BF16: return 2;
    }
    return 0;
}

inline bool aligned(const void* p, size_t a) { return (reinterpret_cast<uintptr_t>(p) % a) == 0; }

inline int check_launch() {
    return hipGetLastError() == hipSuccess ? SQUAT_OK : SQUAT_E_HIP;
}

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half2v __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
// 16 bytes in global memory at a multiple of 4: a 16-byte load needs no more.  The logits kernels read stores with an odd
// number of tokens per head so; word by word against this, 2-bit, groups of 32, GQA 4, us: 64 x 8 x 2081 tokens 33.9 ->
// 19.5, 32 x 32 x 4097 130.6 -> 83.3, 1 x 8 x 32767 10.2 -> 8.3; rotary keys 62.1 -> 28.4, 223 -> 99, 18.0 -> 12.1.
typedef uint32_t u32x4_dwords __attribute__((ext_vector_type(4), aligned(4)));
// At a multiple of 2 (compute on gfx950 runs with unaligned access on): groups of 128, whose scales are 2 bytes a token.  Word by word against
// this, us: 2 bits, 252 x 10541 tokens, 2 query heads 52.2 -> 34.6, rotary keys 91.8 -> 59.0, 4 bits 91.5 -> 55.2 and 94.8 -> 69.1; 64 x 8 x
// 2081, 4 query heads 28.7 -> 20.6, rotary keys 61.1 -> 30.9; 1 x 8 x 32767, 8 query heads, rotary keys 20.2 -> 14.5.
typedef uint32_t u32x4_halves __attribute__((ext_vector_type(4), aligned(2)));
template <int NG>                                         // groups per key
struct StorePiece {
    typedef u32x4_dwords type;
};
template <>
struct StorePiece<1> {
    typedef u32x4_halves type;
};
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ float as_f32(uint32_t u) { return __builtin_bit_cast(float, u); }
__device__ __forceinline__ uint32_t as_u32(float f) { return __builtin_bit_cast(uint32_t, f); }

// Round an fp32 value to fp16 (nearest even) and return it widened again.
__device__ __forceinline__ float round_f16(float v, uint16_t& bits) {
    _Float16 h = static_cast<_Float16>(v);
    bits = __builtin_bit_cast(uint16_t, h);
    return static_cast<float>(h);
}

// MFMA 32x32 accumulator layout on a 64-lane wavefront: lane (hh = lane >> 5,
// n = lane & 31) owns column n and rows 8*q + 4*hh + i for q, i in 0..3, in
// accumulator register 4*q + i.  The kernels that keep a 32-channel tile of a
// key in such an accumulator name the rows so that each lane owns 16
// CONSECUTIVE channels: row m  <->  channel 16*((m>>2)&1) + 4*(m>>3) + (m&3),
// i.e. lane half hh, register e  <->  channel 16*hh + e of the tile.
__host__ __device__ __forceinline__ int row_to_channel(int m) {
    return 16 * ((m >> 2) & 1) + 4 * (m >> 3) + (m & 3);
}

// Tile pairs (jt, s) of 32-channel tiles with a non-zero update panel: block(jt) > block(s), BT tiles
// per block, kD / 32 tiles per key.  Enumerated in the order the panels are laid out in LDS.
__host__ __device__ constexpr int n_pairs(int BT) {
    int c = 0;
    for (int s = 0; s < kD / 32; ++s)
        for (int jt = (s / BT + 1) * BT; jt < kD / 32; ++jt) ++c;
    return c;
}
__host__ __device__ constexpr int pair_index(int BT, int jt, int s) {
    int c = 0;
    for (int ss = 0; ss < kD / 32; ++ss)
        for (int j = (ss / BT + 1) * BT; j < kD / 32; ++j) {
            if (ss == s && j == jt) return c;
            ++c;
        }
    return -1;
}

// min / max as the single machine instruction (the C library functions add one instruction per
// operand that only matters for signalling NaNs when the operands come out of a lane exchange).
__device__ __forceinline__ float raw_min(float a, float b) {
    float r;
    asm("v_min_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
__device__ __forceinline__ float raw_max(float a, float b) {
    float r;
    asm("v_max_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

// min (or max) of a value with the same value in lane ^ 32.
__device__ __forceinline__ float pair_min(float v) {
    auto r = __builtin_amdgcn_permlane32_swap(as_u32(v), as_u32(v), false, false);
    return raw_min(as_f32(r[0]), as_f32(r[1]));
}
__device__ __forceinline__ float pair_max(float v) {
    auto r = __builtin_amdgcn_permlane32_swap(as_u32(v), as_u32(v), false, false);
    return raw_max(as_f32(r[0]), as_f32(r[1]));
}

// Entry points with an explicit output / input placement inside a larger store (used by the cache).
int quantize_keys_into(const void* k, squat_dtype k_dt, int64_t n_batch, int n_heads, int64_t n_tokens, int d,
                       int64_t k_stride_batch, int64_t k_stride_head, int64_t k_stride_token, const float* update,
                       int64_t update_stride_batch, int bits, int group, int g, uint32_t* codes, uint16_t* scale,
                       uint16_t* zero, int64_t out_stride, int64_t out_offset, squat_stream stream);
int quantize_keys_pc_into(const void* k, squat_dtype k_dt, int64_t n_batch, int n_heads, int64_t n_tokens, int d,
                          int64_t k_stride_batch, int64_t k_stride_head, int64_t k_stride_token, const float* update,
                          int64_t update_stride_batch, int bits, int group, int g, uint32_t* codes, uint16_t* scale,
                          uint16_t* zero, int64_t out_stride, int64_t out_offset, squat_stream stream);
struct ResidualKeys;               // squat_residual.h; a cache's full-precision keys, or NULL
int key_scores_from(const uint32_t* codes, const uint16_t* scale, const uint16_t* zero, int64_t n_batch,
                    int n_kv_heads, int64_t n_tokens, int64_t store_stride, int d, int bits, int group,
                    const void* q, squat_dtype q_dt, int q_per_kv, int64_t q_stride_batch, int64_t q_stride_head,
                    float out_scale, float* scores, int64_t s_stride_batch, int64_t s_stride_head,
                    const ResidualKeys* residual, squat_stream stream);
int key_scores_pc_from(const uint32_t* codes, const uint16_t* scale, const uint16_t* zero, int64_t n_batch,
                       int n_kv_heads, int64_t n_tokens, int64_t store_tokens, int d, int bits, int group,
                       const void* q, squat_dtype q_dt, int q_per_kv, int64_t q_stride_batch, int64_t q_stride_head,
                       float out_scale, float* scores, int64_t s_stride_batch, int64_t s_stride_head,
                       const ResidualKeys* residual, squat_stream stream);

int key_scores_rope_from(const uint32_t* codes, const uint16_t* scale, const uint16_t* zero, int64_t n_batch,
                         int n_kv_heads, int64_t n_tokens, int64_t store_stride, int d, int bits, int group,
                         const float* inv_freq, int64_t pos0, const void* q, squat_dtype q_dt, int q_per_kv,
                         int64_t q_stride_batch, int64_t q_stride_head, float out_scale, float* scores,
                         int64_t s_stride_batch, int64_t s_stride_head, squat_stream stream);

int key_scores_pc_rope_from(const uint32_t* codes, const uint16_t* scale, const uint16_t* zero, int64_t n_batch,
                            int n_kv_heads, int64_t n_tokens, int64_t store_tokens, int d, int bits, int group,
                            const float* inv_freq, int64_t pos0, const void* q, squat_dtype q_dt, int q_per_kv,
                            int64_t q_stride_batch, int64_t q_stride_head, float out_scale, float* scores,
                            int64_t s_stride_batch, int64_t s_stride_head, squat_stream stream);

#if defined(__HIPCC__)
// Logits: 4 consecutive channels of a query head, thread by thread over the KV head's queries (256 threads, 8 x 128 values).  Asked for in
// front of the first keys: loads come back in order, so that what is needed first is not behind the keys, which come from
// memory.
template <int QDT>
struct QueryPiece {
    u32x4 raw;
    int row, ch;
    bool live;                                            // a row of this KV head
    template <class Params>
    __device__ __forceinline__ QueryPiece(const Params& p, int64_t b, int kvh) {
        const int e0 = 4 * static_cast<int>(threadIdx.x);
        row = e0 / kD;
        ch = e0 % kD;
        live = row < p.qpk;
        // (a row of another head's place reads the last one; a load under a condition would be waited for there)
        const int64_t off = b * p.qsb + (static_cast<int64_t>(kvh) * p.qpk + (live ? row : p.qpk - 1)) * p.qsh + ch;
        if constexpr (QDT == SQUAT_F32) {
            raw = *reinterpret_cast<const u32x4*>(p.q + off * 4);
        } else {
            const u32x2 t = *reinterpret_cast<const u32x2*>(p.q + off * 2);
            raw = u32x4{t[0], t[1], 0u, 0u};
        }
    }
    __device__ __forceinline__ float value(int i) const {
        if constexpr (QDT == SQUAT_F32) return as_f32(raw[i]);
        const uint32_t h = (i & 1) ? (raw[i >> 1] >> 16) : (raw[i >> 1] & 0xFFFFu);
        return QDT == SQUAT_BF16 ? as_f32(h << 16) : static_cast<float>(__builtin_bit_cast(_Float16, static_cast<uint16_t>(h)));
    }
};

// cos and sin of position * freq: the product is reduced to a fraction of a turn in fp64 first
__device__ __forceinline__ void turn_sincos(double position, float freq, float& c, float& s) {
    const double turns = position * static_cast<double>(freq) * 0.15915494309189535;   // / (2 pi)
    const double frac = turns - rint(turns);                                           // [-0.5, 0.5]
    sincospif(static_cast<float>(2.0 * frac), &s, &c);
}
#endif

// Raises a kernel's dynamic-LDS limit once per device and process.  `done` holds one bit per device
// ordinal; threads that race only repeat the (idempotent) runtime call.
inline int set_max_lds_once(std::atomic<uint64_t>& done, const void* kernel, int bytes) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return SQUAT_E_HIP;
    const uint64_t bit = uint64_t(1) << (dev & 63);
    if (done.load(std::memory_order_acquire) & bit) return SQUAT_OK;
    if (hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes) != hipSuccess) {
        (void)hipGetLastError();
        return SQUAT_E_HIP;
    }
    done.fetch_or(bit, std::memory_order_release);
    return SQUAT_OK;
}

// How a quantize launch spreads its 32-token tiles: `problems` update matrices, each served by
// `wgs_per_prob` persistent workgroups of `waves` wavefronts that stride over `units_per_prob` tiles.
struct QuantPlan {
    int64_t n_prob;
    int64_t n_inner;         // batch entries that share one update matrix
    int64_t tiles_per_seq;
    int64_t units_per_prob;
    int wgs_per_prob;
    int waves;
};
// Logits: result rows that begin on 64-byte lines are written by non-temporal stores (whole lines leave the chip once; 64 x 256 x 2080
// tokens 373 us, 381 with ordinary ones); others (an odd number of tokens) by ordinary ones, whose partial lines the L2 puts together
// where non-temporal stores send each part (per-channel store, 4 query heads per KV head, 8 MB of logits: 1.24 times the write
// requests, 47 MB 1.21; 8 query heads, 17 MB 1.47, 94 MB 1.31).  An ordinary store's line waits in the L2 until the kernel
// ends, which costs the kernels that leave the memory time to spare more than the requests do: the per-channel and the rotary
// kernel have a range of sizes of their own beside this rule.  Per-token store, rows off the lines, us with non-temporal | ordinary stores, 2 bits, heads of about 2050 tokens (medians of 15 graphs of 20 calls on
// four sets of buffers in turn; their spread is 1 %): 1 query head, 1 MB 6.6 | 6.4, 2 MB 9.4 | 9.5, 4 MB 14.3 | 13.9, 8 MB 26.3 | 25.0, 30
// MB 90 | 89; 4, 1 MB 4.6 | 4.2, 2.8 MB 6.6 | 6.7, 4 MB 7.0 | 7.0, 8 MB 11.0 | 10.7, 16 MB 20.9 | 18.8, 45 MB 59 | 45; 8, 1 MB 4.3 | 3.9, 4
// MB 6.3 | 6.1, 5.6 MB 7.3 | 7.6, 8 MB 8.0 | 8.3, 11 MB 11.8 | 10.5, 45 MB 50 | 32.
inline bool rows_on_lines(const float* scores, int64_t stride_batch, int64_t stride_head) {
    return aligned(scores, 64) && stride_batch % 16 == 0 && stride_head % 16 == 0;
}
// One logit; LINES: see rows_on_lines.
template <bool LINES>
__device__ __forceinline__ void put_score(float* p, float v) {
    if constexpr (LINES) __builtin_nontemporal_store(v, p);
    else *p = v;
}

int plan_quantize(squat_dtype k_dt, int64_t n_batch, int n_heads, int64_t n_tokens, bool has_update,
                  int64_t update_stride_batch, int group, int g, QuantPlan& out);
int plan_quantize_pc(squat_dtype k_dt, int64_t n_batch, int n_heads, int64_t n_tokens, bool has_update,
                     int64_t update_stride_batch, int g, QuantPlan& out);

// Units of 16 tokens per wavefront that a per-token logits launch aims at.  `most` amortises a wavefront's
// set-up and is taken while `sequences` of `units` units fill the chip with it; a launch with less work (few sequences)
// spreads it over about `workgroups` workgroups instead, down to `least` units a wavefront.
inline int64_t units_per_wave(int64_t units, int64_t sequences, int waves, int64_t workgroups, int64_t least, int64_t most) {
    const int64_t spread = (units * sequences + waves * workgroups - 1) / (waves * workgroups);
    return spread > most ? most : (spread < least ? least : spread);
}

// How the other logits launches deal out a sequence: its steps (epochs, pairs of token groups) go to `waves` x gx wavefronts, the i-th
// of which takes the steps from deal.start(i) to deal.start(i + 1), the same number within one; the larger number ends with the
// last wavefront (whose last step may be a part of one) or, `late` being false, the smaller.  With a multiple of a step
// for every wavefront, rounded up, 8 sequences of 32800 tokens ran half as long again as of 32768.  us, so | dealt out (2 bits, 4 query
// heads; rotary per channel, rotary, per channel): 8 x 32800 13.8 | 11.5, 12.7 | 10.9, 8.8 | 8.4; 8 x 4128 8.2 | 6.3, 8.0 | 6.3, 5.6 | 4.8; 58 x
// 17472 39 | 33.5, 33 | 28.4, 20.4 | 20.1; 8 x 32768 and 90 x 4992 the same.  (The per-token kernel gains nothing and loses up to 6 % by more,
// shorter workgroups: 256 x 1056 6.9 | 7.4.)
struct Deal {
    uint64_t mul;            // steps per wavefront, times 2^32, rounded up (late) or down
    uint32_t add;            // 0, or 2^32 - 1
#if defined(__HIPCC__)
    __device__ __forceinline__ int start(uint32_t wavefront) const { return static_cast<int>((wavefront * mul + add) >> 32); }
#endif
};
// `wanted` workgroups per sequence, but at least `least` steps a wavefront, and where there is more work than `most` steps a wavefront, which
// amortise its set-up, as many as that makes.
inline Deal deal_steps(int64_t steps, int64_t wanted, int waves, int64_t least, int64_t most, bool late, int64_t& gx) {
    gx = wanted;
    const int64_t full = (2 * steps + waves * most) / (2 * waves * most), room = (steps + waves * least - 1) / (waves * least);
    gx = gx < full ? full : gx;
    gx = gx > room ? room : gx;
    gx = gx < 1 ? 1 : gx;
    const uint64_t all = static_cast<uint64_t>(waves * gx);
    return Deal{((static_cast<uint64_t>(steps) << 32) + (late ? all - 1 : 0)) / all, late ? 0u : 0xFFFFFFFFu};
}

// Number of compute units of the current device (256 if the query fails); a device is asked once per process.
inline int device_cu_count() {
    static std::atomic<int> known[64];
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 256;
    std::atomic<int>& slot = known[dev & 63];
    if (dev < 64) cus = slot.load(std::memory_order_relaxed);
    if (cus > 0) return cus;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0)
        return 256;
    if (dev < 64) slot.store(cus, std::memory_order_relaxed);
    return cus;
}

// Workgroups per problem of a quantize launch: as many as the device holds at once (a workgroup's LDS fills a compute unit), at
// least one and at most one per tile.  Rounded down: where rounding up makes a launch of 257 to 381 workgroups, those beyond 256
// start when the others have ended and read their share alone.  Up | down, us, 2 bits, bf16, groups of 32, 16384 tiles in all: 3 heads
// 59.8 | 42.7, 7 58.7 | 42.1, 40 57.3 | 41.8, 56 59.0 | 44.9, 98 54.3 | 44.2, 200 48.5 | 46.8; 4096 tiles: 7 heads 22.0 | 14.5,
// 40 22.8 | 14.9, 130 22.5 | 17.8; 16 tiles a head, 24 heads 9.6 | 6.1, 56 11.4 | 7.1; per channel, 4 bits, g = 64, 40 heads 56.8 | 42.9; fp32, 7 heads 45.2 | 31.9.  Up to half of
// the compute units stay idle so, and a launch's few more rounds still cost more than they give: 129 heads x 1, 128 tiles each 57.8 | 50.6, 16 15.5 | 11.5,
// fp32, 48 40.2 | 33.8; 86 x 2, 128 41.1 | 30.0; 170 x 1, 128 66.5 | 52.0.
inline int spread_problems(QuantPlan& plan) {
    const int64_t cus = device_cu_count(), tiles = plan.units_per_prob;
    int64_t held = cus / plan.n_prob;
    held = held > tiles ? tiles : (held < 1 ? 1 : held);
    if (plan.n_prob * held > 0x7FFFFFFF) return SQUAT_E_BADSHAPE;
    plan.wgs_per_prob = static_cast<int>(held);
    return SQUAT_OK;
}

}  // namespace squat
