// Device pieces the cache shares with the kernels it appends to and reads with: the logits of the full-precision tail of
// a cache (computed by extra workgroups of the logits kernels, so that a decode step's logits are one launch) and the
// per-token round-to-nearest of one token held by a team of lanes.
#pragma once

#include "squat_internal.h"

namespace squat {

// The full-precision keys of a cache: [batch, KV head, slots, 128], the first `count` slots in use; logit t of a row goes
// behind the ones of the packed keys.  rows == nullptr: none.
struct ResidualKeys {
    const unsigned char* rows;
    int dt;                          // squat_dtype
    int slots;
    int count;
    unsigned first_row;              // grid rows (y) from this one on belong to these keys, a wavefront per eight of them
};

constexpr int kResTokens = 8;            // keys per wavefront
constexpr int kResWaves = 4;             // wavefronts per workgroup: that of the logits kernels

// Whether the logits of `count` full-precision keys, of `row_bytes` each, of every (batch, KV head) pair go into the packed
// keys' launch: a launch of their own costs 2 to 3 us, but has twice the wavefronts per SIMD and so reads them at
// 6 TB/s against 4.  The line lies where the two weigh the same, at 24 MB of keys, counted in the wavefronts' whole eights.
// Measured (2-bit, bf16; us in one launch | in two, for 1, 4 and 8 query heads per KV head), at 4 MB, 1024 pairs of 1024
// packed keys and 16: 13 | 15, 16 | 18, 22 | 24; 17 MB, 4096 of 1024 and 16: 46 | 48, 55 | 56, 76 | 78; 33 MB, 2048 of 256
// and 64: 19 | 18, 23 | 22, 30 | 28; 134 MB, 4096 of 256 and 127: 50 | 42, 61 | 54, 89 | 77; 266 MB, 8192 of 1024 and
// 127: 148 | 127, 233 | 213, 394 | 356; 33 MB as 16384 pairs of 1024 and 1: 171 | 168, 284 | 279, 518 | 505.
inline bool residual_beside(int64_t pairs, int count, int row_bytes) {
    constexpr int64_t kMost = int64_t(24) << 20;
    return pairs * ((count + kResTokens - 1) / kResTokens * kResTokens) * row_bytes <= kMost;
}

// The grid rows behind the gy rows of gx workgroups each that they take there.  They come behind the others and not as one
// more column: with one workgroup per pair before it, a column puts all short workgroups on every other XCD and all
// long ones on the rest (seen at 16384 pairs of 2048 packed keys and 16: 530 us against 394).
inline unsigned residual_rows(const ResidualKeys& r, int64_t gx, int64_t gy) {
    const int64_t workgroups = (gy * ((r.count + kResTokens - 1) / kResTokens) + kResWaves - 1) / kResWaves;
    return static_cast<unsigned>((workgroups + gx - 1) / gx);
}

// 8 consecutive elements (16-byte aligned) as floats
template <int DT>
__device__ __forceinline__ void load8(const unsigned char* p, float* out) {
    if constexpr (DT == SQUAT_F32) {
        const f32x4 a = *reinterpret_cast<const f32x4*>(p);
        const f32x4 b = *reinterpret_cast<const f32x4*>(p + 16);
        out[0] = a[0]; out[1] = a[1]; out[2] = a[2]; out[3] = a[3];
        out[4] = b[0]; out[5] = b[1]; out[6] = b[2]; out[7] = b[3];
    } else {
        const u32x4 v = *reinterpret_cast<const u32x4*>(p);
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            if constexpr (DT == SQUAT_BF16) {
                out[2 * w] = as_f32(v[w] << 16);
                out[2 * w + 1] = as_f32(v[w] & 0xFFFF0000u);
            } else {
                out[2 * w] = static_cast<float>(__builtin_bit_cast(_Float16, static_cast<uint16_t>(v[w] & 0xFFFFu)));
                out[2 * w + 1] = static_cast<float>(__builtin_bit_cast(_Float16, static_cast<uint16_t>(v[w] >> 16)));
            }
        }
    }
}

// scores[b, hq, t0 + t] = out_scale * q[b, hq, :] . rows[b, kvh, t, :] for t < count and the query heads hq of KV head kvh:
// called by every workgroup from row p.res.first_row on, each wavefront takes eight keys of one (batch, KV head).  Eight
// lanes per key: each loads its 16 channels of the key once and meets the same channels of the query heads one after
// the other (the buffer is read once, not once per query head); a dot product is summed by three lane exchanges
// inside the group.  (As a launch of its own behind the logits kernel: 3.8 us more per decoded token for 64
// heads; by the workgroups of the same launch it hides behind the others, 5.2 us for both.)
template <int QDT, typename Params>
__device__ __forceinline__ void residual_scores(const Params& p, int64_t t0) {
    constexpr int QES = QDT == SQUAT_F32 ? 4 : 2;
    const ResidualKeys& r = p.res;
    const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
    const unsigned i = ((blockIdx.y - r.first_row) * gridDim.x + blockIdx.x) * kResWaves + wave;
    const unsigned chunks = static_cast<unsigned>(r.count + kResTokens - 1) / kResTokens;
    const unsigned head = i / chunks;
    if (head >= r.first_row) return;                      // uniform per wavefront
    const int64_t bh = head;
    const int64_t b = bh / p.n_kv_heads;
    const int kvh = static_cast<int>(bh - b * p.n_kv_heads);
    const int part = static_cast<int>(threadIdx.x) & 7;
    const int kes = r.dt == SQUAT_F32 ? 4 : 2;
    const int slot = static_cast<int>(i - head * chunks) * kResTokens + ((static_cast<int>(threadIdx.x) & 63) >> 3);
    const int t = slot < r.count ? slot : r.count - 1;                               // keep the whole wavefront in the exchanges
    const unsigned char* krow = r.rows + ((bh * r.slots + t) * kD + part * 16) * kes;
    float ka[16];
    if (r.dt == SQUAT_F32) {
        load8<SQUAT_F32>(krow, ka);
        load8<SQUAT_F32>(krow + 32, ka + 8);
    } else if (r.dt == SQUAT_BF16) {
        load8<SQUAT_BF16>(krow, ka);
        load8<SQUAT_BF16>(krow + 16, ka + 8);
    } else {
        load8<SQUAT_F16>(krow, ka);
        load8<SQUAT_F16>(krow + 16, ka + 8);
    }
    for (int h0 = 0; h0 < p.qpk; h0 += 4) {               // four query heads' loads in flight
        float qa[4][16];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int hq = kvh * p.qpk + (h0 + j < p.qpk ? h0 + j : p.qpk - 1);
            const unsigned char* qrow = p.q + (b * p.qsb + hq * p.qsh) * QES + part * 16 * QES;
            load8<QDT>(qrow, qa[j]);
            load8<QDT>(qrow + 8 * QES, qa[j] + 8);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (h0 + j >= p.qpk) break;                   // uniform
            float acc = 0.0f;
#pragma unroll
            for (int e = 0; e < 16; ++e) acc = fmaf(qa[j][e], ka[e], acc);
            acc += __shfl_xor(acc, 1, 64);
            acc += __shfl_xor(acc, 2, 64);
            acc += __shfl_xor(acc, 4, 64);
            const int hq = kvh * p.qpk + h0 + j;
            if (part == 0 && slot < r.count) p.scores[b * p.ssb + hq * p.ssh + t0 + slot] = p.out_scale * acc;
        }
    }
}

// Round-to-nearest (Section 2's quantizer, no update matrix) of one token held by a team of eight lanes (an aligned run of
// the wavefront), 16 consecutive channels x per lane; groups of LG lanes.  The same arithmetic, instruction by instruction,
// as the tile kernel of squat_quantize_keys runs with update = NULL on a tile of this one token.  (A tile of more tokens
// takes the form with the clamp for all of them if one needs it, so its words can differ from these by a code where a
// value falls on a rounding boundary.)  words: BITS / 2 packed words of the lane's channels; sbits, zbits: its
// group's scale and zero-point.
template <int BITS>
__device__ __forceinline__ void quantize_token(const float (&x)[16], int lg, uint32_t (&words)[BITS / 2], uint16_t& sbits,
                                               uint16_t& zbits) {
    constexpr float LV = static_cast<float>((1 << BITS) - 1);
    constexpr int CPH = 16 / BITS;                        // codes per 16-bit half-word
    float mn = x[0], mx = x[0];
#pragma unroll
    for (int e = 0; e < 16; ++e) {
        mn = fminf(mn, x[e]);
        mx = fmaxf(mx, x[e]);
    }
    for (int o = 1; o < lg; o <<= 1) {                    // uniform
        mn = raw_min(mn, __shfl_xor(mn, o, 64));
        mx = raw_max(mx, __shfl_xor(mx, o, 64));
    }
    const float rng = mx - mn;
    constexpr float RL = 1.0f / LV;
    const float q0 = rng * RL;
    const float dl = fmaf(fmaf(-q0, LV, rng), RL, q0);    // correctly rounded (max - min) / (2^b - 1)
    const float sh = round_f16(dl, sbits);
    const float mh = round_f16(mn, zbits);
    const bool live = sh > 0.0f;
    const float sp = live ? sh : 1.0f;
    float inv = __builtin_amdgcn_rcpf(sp);
    inv = fmaf(fmaf(-sp, inv, 1.0f), inv, inv);
    const float top = live ? LV : 0.0f;
    // the written-out form with the clamp if any group of the token needs it, else one multiply-add per code
    const bool risky = !(sh >= 6.2e-5f) || fabsf(mh) * inv > kQuantFastOffset;
    const uint64_t team = 0xFFull << (threadIdx.x & 56);
    const bool clamp = (__ballot(risky) & team) != 0ull;
    const float nmi = -mh * inv;
    uint32_t hw[16 / CPH];
#pragma unroll
    for (int q = 16 / CPH - 1; q >= 0; --q) {
        float accf = 0.0f;
#pragma unroll
        for (int e = CPH - 1; e >= 0; --e) {
            const int c = q * CPH + e;
            const float u = __builtin_amdgcn_fmed3f((x[c] - mh) * inv, 0.0f, top);
            const float v = fmaf(x[c], inv, nmi);
            accf = fmaf(accf, static_cast<float>(1 << BITS), __builtin_rintf(clamp ? u : v));
        }
        hw[q] = static_cast<uint32_t>(accf);
    }
#pragma unroll
    for (int w = 0; w < BITS / 2; ++w) words[w] = hw[2 * w] | (hw[2 * w + 1] << 16);
}

}  // namespace squat
