// squat_dequantize_keys: deq(c) = c * Delta + m (Section 2 of the paper) over the
// packed store written by squat_quantize_keys.  Pure streaming: one thread turns
// 16 channels of one key (a word or two, or the parts of four that it needs) into
// two or four 16-byte pieces of output, 128 bytes apart: in each store the eight
// threads of a key write one whole line, which a non-temporal store sends as it
// is.  A wavefront covers 8 consecutive keys.
//
// squat_dequantize_keys_per_channel reads the token-major store of the
// per-channel mode: one wavefront rebuilds one tile of 32 tokens; a lane owns 8
// channels (one 16-byte piece of an output row, or two of fp32) of 8 tokens, so it
// needs 8 packed words, 8 scales and 8 zero-points, and writes whole lines.
#include "squat_internal.h"

using namespace squat;

namespace {

struct DeqParams {
    const uint32_t* codes;
    const uint16_t* scale;
    const uint16_t* zero;
    unsigned char* out;
    int64_t ob, oh, ot;      // output strides in BYTES
    int64_t n_tokens;
    int n_heads;
    uint32_t div_mul, div_shift;    // bh / n_heads == (bh * div_mul) >> div_shift for bh < 2^31
};

// Two floats -> two bf16 (round to nearest even, NaN stays NaN) in one word: the hardware conversion.
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{lo, hi}, bf16x2));
}

// 16 bytes of output.
template <int DT, bool NT>
__device__ __forceinline__ void store_piece(unsigned char* dst, const float* v) {
    if constexpr (DT == SQUAT_F32) {
        const f32x4 w = {v[0], v[1], v[2], v[3]};
        if constexpr (NT) __builtin_nontemporal_store(w, reinterpret_cast<f32x4*>(dst));
        else *reinterpret_cast<f32x4*>(dst) = w;
    } else {
        u32x4 w;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if constexpr (DT == SQUAT_F16) {
                half2v h;
                h[0] = static_cast<_Float16>(v[2 * i]);
                h[1] = static_cast<_Float16>(v[2 * i + 1]);
                w[i] = __builtin_bit_cast(uint32_t, h);
            } else {
                w[i] = pack_bf16(v[2 * i], v[2 * i + 1]);
            }
        }
        if constexpr (NT) __builtin_nontemporal_store(w, reinterpret_cast<u32x4*>(dst));
        else *reinterpret_cast<u32x4*>(dst) = w;
    }
}

// Bound by HBM.  With 16 consecutive channels a thread, its pieces beside each other, a store wrote 16 of every 32 (fp32: 64) bytes, which the
// L2 had to put together, and ordinary stores were the only ones fit for that.  us, before | now: 2 bits, groups of 32, bf16, 256 x 32768
// tokens 514 | 441 (5.8 TB/s), 648 x 1296 54.2 | 38.5; 4 bits, groups of 128, bf16, 32 x 8191 tokens 16.9 | 14.6, fp32, 324 x 1296 71.1 | 37.4,
// 16 x 2049 9.3 | 4.4.
// grid: x over (token, thread of a key), y/z over (batch, head)
template <int BITS, int GROUP, int DT, bool NT>
__global__ void __launch_bounds__(256) dequantize_kernel(const DeqParams p) {
    constexpr int ES = (DT == SQUAT_F32) ? 4 : 2;
    constexpr int WPK = kD * BITS / 32;       // words per key
    constexpr int NG = kD / GROUP;            // groups per key
    const int64_t bh = static_cast<int64_t>(blockIdx.z) * gridDim.y + blockIdx.y;
    const int64_t flat = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    const int64_t tok = flat >> 3;
    const int chunk = static_cast<int>(flat & 7);
    if (tok >= p.n_tokens) return;
    // exact multiply-shift division (a 64-bit division is ~60 scalar instructions in front of every
    // wavefront's first load, and the wavefronts of this kernel are short)
    const int64_t b = static_cast<int64_t>((static_cast<uint64_t>(bh) * p.div_mul) >> p.div_shift);
    const int64_t h = bh - b * p.n_heads;
    const int64_t row = bh * p.n_tokens + tok;

    // 16 bytes of output of every 128: the eight threads of a key write whole lines
    constexpr int CH = 16 / ES;                           // channels per piece
    constexpr int NP = 16 / CH;                           // pieces per thread
    constexpr int IPW = 32 / BITS;
    constexpr uint32_t MASK = (1u << BITS) - 1u;
    uint32_t w[NP];
    float sc[NP], zp[NP];
#pragma unroll
    for (int i = 0; i < NP; ++i) w[i] = p.codes[row * WPK + (8 * CH * i + CH * chunk) / IPW];
#pragma unroll
    for (int i = 0; i < NP; ++i) {
        const int gi = (8 * CH * i + CH * chunk) / GROUP;
        sc[i] = static_cast<float>(__builtin_bit_cast(_Float16, p.scale[row * NG + gi]));
        zp[i] = static_cast<float>(__builtin_bit_cast(_Float16, p.zero[row * NG + gi]));
    }
    unsigned char* dst = p.out + b * p.ob + h * p.oh + tok * p.ot + chunk * 16;
#pragma unroll
    for (int i = 0; i < NP; ++i) {
        // converted once: folded into the multiply-adds as mixed-precision operands they would issue at half rate
        asm volatile("" : "+v"(sc[i]), "+v"(zp[i]));
        const uint32_t c = w[i] >> (CH * chunk % IPW * BITS);
        float v[CH];
#pragma unroll
        for (int e = 0; e < CH; ++e) v[e] = fmaf(static_cast<float>((c >> (BITS * e)) & MASK), sc[i], zp[i]);
        store_piece<DT, NT>(dst + 128 * i, v);
    }
}

// One wavefront per tile of 32 tokens.  Lane (s = lane >> 4, pc = lane & 15): channels 8 pc .. 8 pc + 7 (fp32: 4 pc .. 4 pc + 3 of
// each half, 324 x 1312 tokens, 4 bits: 55.5 -> 48.3 us), tokens 8 s .. 8 s + 7 of the tile.  Token j of the tile sits in word j / (32 / BITS) of its channel
// at bit BITS * (j mod 32 / BITS), so the lane's 8 tokens are BITS consecutive bytes of one word.
template <int BITS, int DT, bool NT>
__global__ void __launch_bounds__(256) dequantize_pc_kernel(const DeqParams p, const int64_t tiles_per_seq) {
    constexpr int ES = (DT == SQUAT_F32) ? 4 : 2;
    const int lane = threadIdx.x & 63;
    const int64_t bh = static_cast<int64_t>(blockIdx.z) * gridDim.y + blockIdx.y;
    const int64_t tile = static_cast<int64_t>(blockIdx.x) * 4 + (threadIdx.x >> 6);
    if (tile >= tiles_per_seq) return;
    // exact multiply-shift division (a 64-bit division is ~60 scalar instructions in front of every
    // wavefront's first load, and the wavefronts of this kernel are short)
    const int64_t b = static_cast<int64_t>((static_cast<uint64_t>(bh) * p.div_mul) >> p.div_shift);
    const int64_t h = bh - b * p.n_heads;
    const int64_t gt = bh * tiles_per_seq + tile;
    const int s = lane >> 4, pc = lane & 15;

    const int widx = 8 * s * BITS / 32;               // word of the channel that holds tokens 8 s .. 8 s + 7
    const int shift0 = (8 * s * BITS) % 32;
    // The tile's packed words come in with one (two for 4 bits) 16-byte load per lane, contiguous over the
    // wavefront, and go through a wavefront-private LDS tile to the lanes that unpack them (a lane's own 8
    // words are 4 BITS bytes apart in memory: fetched directly, every load instruction touched 16 to 32
    // sectors for 256 bytes).  Every 16 words of the tile are followed by 4 words of padding, which spreads
    // the 16 lanes of a token group over the banks.
    constexpr int TW = kD * BITS;                     // words per tile
    __shared__ __attribute__((aligned(16))) uint32_t tile_lds[4][TW + TW / 4];
    uint32_t* tl = tile_lds[threadIdx.x >> 6];
    const uint32_t* ct = p.codes + gt * TW;
#pragma unroll
    for (int i = 0; i < TW / 256; ++i) {
        const int idx = (i * 64 + lane) * 4;
        *reinterpret_cast<u32x4*>(tl + idx + (idx >> 4) * 4) =
            __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(ct + idx));
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    // The lane's channels: CH of every 16 CH, so that 16 lanes write whole lines.
    constexpr int CH = 16 / ES, NP = 8 / CH;
    uint32_t w[8];
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        const int idx = (16 * CH * (c / CH) + CH * pc + c % CH) * BITS + widx;
        w[c] = tl[idx + (idx >> 4) * 4] >> shift0;
    }
    uint32_t sraw[4], zraw[4];
#pragma unroll
    for (int i = 0; i < NP; ++i) {
        typedef uint32_t piece __attribute__((ext_vector_type(CH / 2)));
        const piece sv = *reinterpret_cast<const piece*>(p.scale + gt * kD + 16 * CH * i + CH * pc);
        const piece zv = *reinterpret_cast<const piece*>(p.zero + gt * kD + 16 * CH * i + CH * pc);
#pragma unroll
        for (int k = 0; k < CH / 2; ++k) {
            sraw[i * CH / 2 + k] = sv[k];
            zraw[i * CH / 2 + k] = zv[k];
        }
    }
    float sc[8], zp[8];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        sc[2 * c] = static_cast<float>(__builtin_bit_cast(_Float16, static_cast<uint16_t>(sraw[c] & 0xFFFFu)));
        sc[2 * c + 1] = static_cast<float>(__builtin_bit_cast(_Float16, static_cast<uint16_t>(sraw[c] >> 16)));
        zp[2 * c] = static_cast<float>(__builtin_bit_cast(_Float16, static_cast<uint16_t>(zraw[c] & 0xFFFFu)));
        zp[2 * c + 1] = static_cast<float>(__builtin_bit_cast(_Float16, static_cast<uint16_t>(zraw[c] >> 16)));
    }
    constexpr uint32_t MASK = (1u << BITS) - 1u;
    unsigned char* dst = p.out + b * p.ob + h * p.oh + (tile * kTileTokens + 8 * s) * p.ot + pc * 16;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        float v[8];
#pragma unroll
        for (int c = 0; c < 8; ++c)
            v[c] = fmaf(static_cast<float>((w[c] >> (BITS * i)) & MASK), sc[c], zp[c]);
#pragma unroll
        for (int k = 0; k < NP; ++k) store_piece<DT, NT>(dst + i * p.ot + 256 * k, v + CH * k);
    }
}

template <int BITS, bool NT>
int launch_pc(squat_dtype dt, const DeqParams& p, int64_t tiles, dim3 grid, hipStream_t s) {
    switch (dt) {
        case SQUAT_F32: hipLaunchKernelGGL((dequantize_pc_kernel<BITS, SQUAT_F32, NT>), grid, dim3(256), 0, s, p, tiles); break;
        case SQUAT_F16: hipLaunchKernelGGL((dequantize_pc_kernel<BITS, SQUAT_F16, NT>), grid, dim3(256), 0, s, p, tiles); break;
        case SQUAT_BF16: hipLaunchKernelGGL((dequantize_pc_kernel<BITS, SQUAT_BF16, NT>), grid, dim3(256), 0, s, p, tiles); break;
        default: return SQUAT_E_BADDTYPE;
    }
    return check_launch();
}

// Non-temporal stores for outputs of 4 MB and more.  The last of them is on its way to memory when the kernel ends, which a short
// launch waits for.  us, ordinary | non-temporal stores (graphs of such calls): fp16, 4 bits, groups of 128, 0.7 MB 2.8 | 3.0, 8.4 MB
// 4.1 | 3.5; bf16, 215 MB 47.8 | 41.2; fp32, 215 MB 47.3 | 37.1; per channel, bf16, 0.7 MB 3.0 | 3.2, 3 MB 3.3 | 3.5, 8.4 MB 4.2 | 3.9, 109
// MB 29.6 | 25.9, fp32, 217 MB 50.1 | 48.3.
//
// Only where the rows are whole lines, or begin on half lines with room between them: of a line that two rows share a non-temporal
// store sends each part, which the L2 puts together for ordinary ones.  2 bits, bf16, rows of 272 bytes, 25 MB 7.6 | 10.8, 272 MB 112 | 154; of
// 256 bytes 16 bytes off a line, 24 MB 7.5 | 9.7, 256 MB 70 | 120, 64 bytes off, 24 MB 6.8 | 7.5, 512 MB 154 | 175; of 320 bytes, 30 MB
// 6.8 | 6.2, 320 MB 89 | 63; per channel, rows of 272 bytes, 272 MB 117 | 136, 256 bytes 16 off, 256 MB 67 | 95, 320 bytes, 320 MB 91 | 64.
//
// Per channel, whole lines: up to 512 MB, fp32 256 MB (us, ordinary | non-temporal, dense rows, 2 bits: bf16, 256 MB 59.0 | 57.5, 384 MB 86.8 | 87.2, 512 MB
// 115 | 117, 768 MB 170 | 178, 2 GB 465 | 479; fp32, 192 MB 42.5 | 41.3, 256 MB 55.9 | 55.5, 384 MB 81.9 | 84.9, 1 GB 217 | 226; 4 bits: bf16, 512 MB
// 124 | 122, 768 MB 186 | 189, 1 GB 249 | 254; fp32, 256 MB 59.3 | 59.0, 384 MB 86.7 | 89.3, 1 GB 226 | 240).  Half lines (rows of 320 bytes)
// 1280 MB 351 | 261.
bool streamed(const DeqParams& p, int64_t n_batch, int es, bool per_channel) {
    const int64_t row = kD * es, oh = p.n_heads > 1 ? p.oh : p.ot, ob = n_batch > 1 ? p.ob : p.ot;
    const uint64_t starts = reinterpret_cast<uintptr_t>(p.out) | static_cast<uint64_t>(p.ot | oh | ob);
    const bool apart = p.ot > row && oh > row && ob > row;
    if (starts % (apart ? 64 : 128)) return false;
    const double megabytes = static_cast<double>(n_batch) * p.n_heads * p.n_tokens * row / (1 << 20);
    return megabytes >= 4 && !(per_channel && starts % 128 == 0 && megabytes > (es == 4 ? 256 : 512));
}

// (batch, head) pairs over grid y / z: an exact factorisation so that every (y, z) is a real pair.
bool split_bh(int64_t bh, int64_t& gy, int64_t& gz) {
    gy = bh;
    gz = 1;
    if (gy > 65535) {
        gy = 0;
        for (int64_t cand = 65535; cand >= 1; --cand)
            if (bh % cand == 0) { gy = cand; break; }
        gz = bh / gy;
    }
    return gz <= 65535;
}

template <int BITS, int GROUP, bool NT>
int launch_dt(squat_dtype dt, const DeqParams& p, dim3 grid, hipStream_t s) {
    switch (dt) {
        case SQUAT_F32: hipLaunchKernelGGL((dequantize_kernel<BITS, GROUP, SQUAT_F32, NT>), grid, dim3(256), 0, s, p); break;
        case SQUAT_F16: hipLaunchKernelGGL((dequantize_kernel<BITS, GROUP, SQUAT_F16, NT>), grid, dim3(256), 0, s, p); break;
        case SQUAT_BF16: hipLaunchKernelGGL((dequantize_kernel<BITS, GROUP, SQUAT_BF16, NT>), grid, dim3(256), 0, s, p); break;
        default: return SQUAT_E_BADDTYPE;
    }
    return check_launch();
}

template <int BITS, bool NT>
int launch_group(int group, squat_dtype dt, const DeqParams& p, dim3 grid, hipStream_t s) {
    switch (group) {
        case 32: return launch_dt<BITS, 32, NT>(dt, p, grid, s);
        case 64: return launch_dt<BITS, 64, NT>(dt, p, grid, s);
        case 128: return launch_dt<BITS, 128, NT>(dt, p, grid, s);
    }
    return SQUAT_E_BADSHAPE;
}

}  // namespace

extern "C" int squat_dequantize_keys(const uint32_t* codes, const uint16_t* scale, const uint16_t* zero,
                                     int64_t n_batch, int n_heads, int64_t n_tokens, int d, int bits,
                                     int group, void* k_out, squat_dtype out_dt, int64_t o_stride_batch,
                                     int64_t o_stride_head, int64_t o_stride_token, squat_stream stream) {
    if (d != kD) return SQUAT_E_BADSHAPE;
    if (bits != 2 && bits != 4) return SQUAT_E_BADSHAPE;
    if (group != 32 && group != 64 && group != 128) return SQUAT_E_BADSHAPE;
    if (n_batch < 0 || n_heads < 0 || n_tokens < 0) return SQUAT_E_BADSHAPE;
    if (out_dt != SQUAT_F32 && out_dt != SQUAT_F16 && out_dt != SQUAT_BF16) return SQUAT_E_BADDTYPE;
    if (n_batch == 0 || n_heads == 0 || n_tokens == 0) return SQUAT_OK;
    if (!codes || !scale || !zero || !k_out) return SQUAT_E_NULLPTR;
    if (o_stride_token < d || o_stride_batch < 0 || o_stride_head < 0) return SQUAT_E_BADSHAPE;
    if ((o_stride_token % 8) || (o_stride_head % 8) || (o_stride_batch % 8)) return SQUAT_E_ALIGN;
    if (!aligned(k_out, 16) || !aligned(codes, 16) || !aligned(scale, 2) || !aligned(zero, 2)) return SQUAT_E_ALIGN;

    const int es = elem_size(out_dt);
    DeqParams p;
    p.codes = codes;
    p.scale = scale;
    p.zero = zero;
    p.out = static_cast<unsigned char*>(k_out);
    p.ob = o_stride_batch * es;
    p.oh = o_stride_head * es;
    p.ot = o_stride_token * es;
    p.n_tokens = n_tokens;
    p.n_heads = n_heads;
    if (n_batch * n_heads >= (int64_t(1) << 31)) return SQUAT_E_BADSHAPE;
    {
        // floor(u / d) for u < 2^31: shift = 31 + ceil(log2 d), mul = floor(2^shift / d) + 1
        const uint64_t dv = static_cast<uint64_t>(n_heads);
        uint32_t l = 0;
        while ((uint64_t(1) << l) < dv) ++l;
        p.div_shift = 31 + l;
        p.div_mul = static_cast<uint32_t>(((uint64_t(1) << p.div_shift) / dv) + 1);
    }

    const int64_t gx = (n_tokens * 8 + 255) / 256;
    int64_t gy, gz;
    if (!split_bh(n_batch * n_heads, gy, gz) || gx > 0x7FFFFFFF) return SQUAT_E_BADSHAPE;
    const dim3 grid(static_cast<unsigned>(gx), static_cast<unsigned>(gy), static_cast<unsigned>(gz));
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (streamed(p, n_batch, es, false))
        return bits == 2 ? launch_group<2, true>(group, out_dt, p, grid, s) : launch_group<4, true>(group, out_dt, p, grid, s);
    return bits == 2 ? launch_group<2, false>(group, out_dt, p, grid, s) : launch_group<4, false>(group, out_dt, p, grid, s);
}

extern "C" int squat_dequantize_keys_per_channel(const uint32_t* codes, const uint16_t* scale,
                                                 const uint16_t* zero, int64_t n_batch, int n_heads,
                                                 int64_t n_tokens, int d, int bits, int group, void* k_out,
                                                 squat_dtype out_dt, int64_t o_stride_batch,
                                                 int64_t o_stride_head, int64_t o_stride_token,
                                                 squat_stream stream) {
    if (d != kD) return SQUAT_E_BADSHAPE;
    if (bits != 2 && bits != 4) return SQUAT_E_BADSHAPE;
    if (group != kTileTokens) return SQUAT_E_BADSHAPE;
    if (n_batch < 0 || n_heads < 0 || n_tokens < 0 || n_tokens % group) return SQUAT_E_BADSHAPE;
    if (out_dt != SQUAT_F32 && out_dt != SQUAT_F16 && out_dt != SQUAT_BF16) return SQUAT_E_BADDTYPE;
    if (n_batch == 0 || n_heads == 0 || n_tokens == 0) return SQUAT_OK;
    if (!codes || !scale || !zero || !k_out) return SQUAT_E_NULLPTR;
    if (o_stride_token < d || o_stride_batch < 0 || o_stride_head < 0) return SQUAT_E_BADSHAPE;
    if ((o_stride_token % 8) || (o_stride_head % 8) || (o_stride_batch % 8)) return SQUAT_E_ALIGN;
    if (!aligned(k_out, 16) || !aligned(codes, 16) || !aligned(scale, 16) || !aligned(zero, 16)) return SQUAT_E_ALIGN;

    const int es = elem_size(out_dt);
    DeqParams p;
    p.codes = codes;
    p.scale = scale;
    p.zero = zero;
    p.out = static_cast<unsigned char*>(k_out);
    p.ob = o_stride_batch * es;
    p.oh = o_stride_head * es;
    p.ot = o_stride_token * es;
    p.n_tokens = n_tokens;
    p.n_heads = n_heads;
    if (n_batch * n_heads >= (int64_t(1) << 31)) return SQUAT_E_BADSHAPE;
    {
        // floor(u / d) for u < 2^31: shift = 31 + ceil(log2 d), mul = floor(2^shift / d) + 1
        const uint64_t dv = static_cast<uint64_t>(n_heads);
        uint32_t l = 0;
        while ((uint64_t(1) << l) < dv) ++l;
        p.div_shift = 31 + l;
        p.div_mul = static_cast<uint32_t>(((uint64_t(1) << p.div_shift) / dv) + 1);
    }

    const int64_t tiles = n_tokens / kTileTokens;
    const int64_t gx = (tiles + 3) / 4;
    int64_t gy, gz;
    if (!split_bh(n_batch * n_heads, gy, gz) || gx > 0x7FFFFFFF) return SQUAT_E_BADSHAPE;
    const dim3 grid(static_cast<unsigned>(gx), static_cast<unsigned>(gy), static_cast<unsigned>(gz));
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (streamed(p, n_batch, es, true))
        return bits == 2 ? launch_pc<2, true>(out_dt, p, tiles, grid, s) : launch_pc<4, true>(out_dt, p, tiles, grid, s);
    return bits == 2 ? launch_pc<2, false>(out_dt, p, tiles, grid, s) : launch_pc<4, false>(out_dt, p, tiles, grid, s);
}
