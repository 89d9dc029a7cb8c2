// Gradient Vectorized Quantization on gfx950: channel statistics, discriminator + clip solve,
// and the int8 packing kernels (Algorithm 1, per-channel loop and the two quantizations), plus
// the per-tensor quantization of X and W used by the forward pass.
//
// All kernels here are meant to be bandwidth bound, which on this chip takes care with the instruction count too
// (buffer loads instead of selects, 24-bit multiplies, one-instruction rounding).  Float reductions use fixed
// trees and a fixed-order second stage (no float atomics), so results do not depend on scheduling.  Compile with
// -ffp-contract=off: the rounding of every fp32/fp64 expression below is part of the contract.
#include <algorithm>
#include <cmath>
#include <mutex>

#include "daq_internal.h"

namespace daq {

namespace {

typedef uint32_t v4u __attribute__((ext_vector_type(4)));
typedef uint32_t v2u __attribute__((ext_vector_type(2)));

constexpr int kBlock = 256;
constexpr int kStatsElems = 4096;  // elements one statistics workgroup sweeps per iteration (16 per thread, all in flight)
constexpr int kMaxSlabs = 16;      // statistics partials per channel (every consumer re-folds them)
// What the memory-side cache holds.  A tensor that does not fit is read with the streaming hint, and what else there is stays in the caches
// until whole lines of it are written back (128 x 96 x 112 x 112, 617 MB, both copies 243 -> 224 us; tensors of 50 to 230 MB, that the
// statistics sweep has just read, 2 to 10 % slower with the hint).
constexpr int64_t kCacheBytes = (int64_t)256 << 20;

int64_t channel_units(int N, int HW);

// ---------------------------------------------------------------------------------------------
// workspace carving
// ---------------------------------------------------------------------------------------------
struct QuantWs {
    float* gmax;          // [C]  |g|max, mean, sigma: written by the counting pass for the packing pass
    float* mean;          // [C]
    float* sigma;         // [C]
    float* s_prev;        // [C]  copy of the clip state taken before anything overwrites it
    uint32_t* pred;       // [C]  class the counting pass assumed when it wrote the per-channel copy early (see k_count_qg)
    float* layer;         // [8]  whole-tensor values for the ablation schemes: |g|max (not zeroed when tiny), mean, sigma,
                          //      tail mass P, clip value, class
    uint32_t* layer_cnt;  // [counting waves]  #{|g| > sigma} over all 16 channels of a counting wave (layer-wise clipping)
    float* part_max;      // [C][slabs]
    double* part_s1;      // [C][slabs]
    double* part_s2;      // [C][slabs]
    uint32_t* part_cnt;   // [C][cgroups]  #{|g| > sigma} seen by counting workgroup p of the channel's block
    int chunks;           // 4096-element chunks of one channel
    int slabs;            // statistics workgroups (partials) per channel
    int part_n;           // entries of part_max whose maximum is the scale of the per-tensor copy (C * slabs)
    CountPlan cp;         // how the counting pass is dealt out
    int scheme;           // daq_scheme the launches of this call follow
    int64_t total_bytes;
};

}  // namespace

// A block is the channels whose shares of an NHWC record a workgroup writes as one run, a wave to 16 of them.  Its width goes by the size of
// the tensor, in steps of 64 pixels x 64 channels, of which the chip holds 1024 at once.  Quantizing calls (both copies in one sweep) of 16 G channels, 6 to
// 100 M elements, both roundings, planes of whole units and not: the speed with blocks of 128 and of 192 channels (G up to 12: whole records) over that of 64
//   1 to 2 Ki steps    G 8 0.97, 0.97    G 9 to 12 0.97, 0.97    G from 13 on 0.98, 0.98    more and smaller workgroups are the faster
//   2 to 4 Ki               1.01, 1.01              1.01, 0.99                1.03, 1.00    a CU holds 16 waves in blocks of 128, but 12 in blocks of 192
//   4 to 10 Ki              1.00, 1.00              1.01, 0.99                1.01, 1.00
//   10 to 18 Ki             1.08, 1.08              1.04, 1.06                1.05, 1.05    the pieces of a record no longer meet in the caches: the fewer
//   from 18 Ki on           1.06, 1.06              1.05, 1.10                1.05, 1.05    the better, and whole records best
// Workgroups of five waves are the slowest at any size (80 channels whole over 64 + 16: 0.84 and 0.87 up to 10 Ki steps, beyond 0.96, in bfloat16 1.15;
// 240 channels as 3 x 80 over 128 + 112: 0.84 to 0.87): only whole records of a large tensor take them.  Six are no faster than 64 + 32 up to 10 Ki steps (0.97
// to 0.99), seven are faster than 64 + 48 from 1 Ki on (1.02 to 1.04).
static int block_width(int G, int64_t steps) {
    if (steps > 10 * 1024) {   // the width up to 12, from six on, that leaves the fewest waves of the last block idle, the largest of equals
        int width = std::min(G, 12);
        for (int w = std::min(G, 11); w >= 6; --w)
            if (ceil_div(G, w) * w < ceil_div(G, width) * width) width = w;
        return width;
    }
    if (G == 7 ? steps > 1024 : G > 7 && steps > 2 * 1024) return std::min(G, 8);
    return std::min(G, 4);
}

// `given`: the waves of a launch that has other roles too; `held_given`: how many workgroups of it the chip is to hold.
CountPlan plan_count(int C, int N, int HW, int given, int held_given) {
    CountPlan p{};
    const int G = (int)ceil_div(C, 16);
    p.tiles = (int)ceil_div(channel_units(N, HW), 16);
    p.width = given ? std::min(G, given) : block_width(G, (int64_t)p.tiles * ceil_div(G, 4));
    p.waves = given ? given : p.width == 1 ? 4 : p.width <= 3 ? 2 * p.width : p.width;
    p.blocks = (int)ceil_div(G, p.width);
    const int side = p.waves / p.groups(C, p.blocks - 1);   // tiles at a time of a workgroup of the last block
    const int64_t last = ceil_div(p.tiles, side), most = p.blocks > 1 ? p.tiles : last;
    // the last block gets as many workgroups fewer as they are quicker
    const int64_t held = held_given ? held_given : 256 * (kCountWaves / p.waves);   // workgroups at once
    int64_t want = std::max<int64_t>(1, std::min<int64_t>(kCountGroups, p.blocks > 1 ? held * side / ((int64_t)(p.blocks - 1) * side + 1) : held));
    if (want >= 2 * kXcd) want -= want % kXcd;
    const int64_t turns = ceil_div(most, want);
    auto groups = [&](int64_t n) {
        const int64_t q = ceil_div(n, turns);
        return (int)(q >= 2 * kXcd ? round_up(q, kXcd) : q);   // whole rounds over the XCDs (see k_count_qg)
    };
    p.cgroups = groups(most);
    if (C > 1024) {   // many channels: no more partial counts than the scratch of daq_quantize_grad_noalloc was laid out for
        const int64_t tiles = ceil_div((int64_t)N * HW, kWave), n = std::max<int64_t>(1, 1024 / ceil_div(C, 64)), q = ceil_div(tiles, ceil_div(tiles, n));
        p.cgroups = std::min(p.cgroups, (int)(q >= 2 * kXcd ? round_up(q, kXcd) : q));
    }
    p.cgroups_last = std::min(p.cgroups, groups(last));
    p.div_cgroups = make_fastdiv((uint32_t)p.cgroups);
    for (int b = 0; b < 2; ++b) {
        const int gb = p.groups(C, b ? p.blocks - 1 : 0);
        p.by_groups[b] = (uint32_t)((65536 + gb - 1) / gb);
    }
    return p;
}

// Workgroups of the forward sweep over X that writes both copies: eight waves, so that a block is 128 channels and 128 bytes of a record leave as one run,
// or four.  Speed of its launch with eight over four waves, 80 to 1024 channels, planes of 27 x 31 to 71 x 70, by millions of elements
//                                    12 to 13         28 to 30         57 to 60         100 to 115
//   up to 64 channels                never: four waves hold the whole record
//   80, 112 channels                 0.97 to 1.05     1.10 to 1.14     1.13 to 1.33     1.12 to 1.28
//   96 channels                      0.96 to 1.03     1.04 to 1.09     1.17 to 1.20     1.05 to 1.19
//   a last block of one group        0.97 to 1.10     0.98 to 1.05     0.98 to 1.02     0.98 to 1.03
//   others                           0.93 to 1.08     0.94 to 1.08     1.02 to 1.21     1.01 to 1.22
// In four waves a record of several times 64 bytes leaves from as many workgroups, which do not keep step; up to some 20 M elements the caches
// bring the pieces together all the same.  Whole pass, 384 channels: 55 of 71 x 70, 1 x 1,
// 336 us with four waves, 319 with eight; 60 of 58 x 58, 3 x 3, 282 and 272; 96 channels, 128 of 105 x 105, 1 x 1, 431 and 365.
// The filter's workgroups come first in the launch, and where they are many a CU that holds one is short of a workgroup of twice the size: over 400
// drawn tensors of 24 to 112 Mi elements 1.04 to 1.12 times the speed up to a workgroup a CU, 0.98 up to 400, 0.95 beyond (768 channels and more, 5 x 5: 0.83 to
// 0.95).  Beyond 2048 channels, where they are 130 and more for any filter, level or down to 0.90.
int forward_waves(int C, int N, int HW, int w_blocks) {
    return C > 64 && HW >= 4 && (int64_t)C * N * HW > (int64_t)24 << 20 && C <= 2048 && w_blocks <= 256 ? 8 : kBlock / kWave;
}

namespace {

QuantWs carve_quant_ws(void* base, int C, int N, int HW, int given_waves = 0, int given_held = 0) {
    QuantWs w{};
    const int64_t M = (int64_t)N * HW;
    // statistics sweep groups of four elements per plane (k_stats): the axis is padded to whole groups
    const int64_t Mstats = HW >= 4 ? (int64_t)N * ((HW + 3) / 4) * 4 : M;
    w.chunks = (int)ceil_div(Mstats, kStatsElems);
    const int iters = (int)ceil_div(w.chunks, kMaxSlabs);
    w.slabs = (int)ceil_div(w.chunks, iters);
    w.part_n = C * w.slabs;
    w.cp = plan_count(C, N, HW, given_waves, given_held);
    // byte offsets first; pointers only when there is a buffer (a size query passes none)
    int64_t off = 0;
    const int64_t o_head = off;
    off += round_up(((int64_t)5 * C + 8) * 4, 256);
    const int64_t o_s1 = off;
    off += round_up((int64_t)2 * C * w.slabs * 8, 256);
    const int64_t o_max = off;
    off += round_up((int64_t)C * w.slabs * 4, 256);
    const int64_t o_cnt = off;
    off += round_up((int64_t)C * w.cp.cgroups * 4, 256);
    const int64_t o_lcnt = off;
    off += round_up((int64_t)w.cp.workgroups() * w.cp.waves * 4, 256);
    w.total_bytes = off;
    if (base) {
        char* p = (char*)base;
        w.gmax = (float*)(p + o_head);
        w.mean = w.gmax + C;
        w.sigma = w.mean + C;
        w.s_prev = w.sigma + C;
        w.pred = (uint32_t*)(w.s_prev + C);
        w.layer = (float*)(w.pred + C);
        w.part_s1 = (double*)(p + o_s1);
        w.part_s2 = w.part_s1 + (int64_t)C * w.slabs;
        w.part_max = (float*)(p + o_max);
        w.part_cnt = (uint32_t*)(p + o_cnt);
        w.layer_cnt = (uint32_t*)(p + o_lcnt);
    }
    return w;
}

// ---------------------------------------------------------------------------------------------
// device helpers
// ---------------------------------------------------------------------------------------------
// Stochastic rounding: a counter-based generator on 32-bit arithmetic.  fmix32 is the finalizer of MurmurHash3
// (Appleby, public domain), a bijection of 32-bit words with full avalanche.  A launch derives one key from the
// caller's 64-bit seed (round_key, on the host); element i (its NCHW index, below 2^31) hashes once,
//     h = fmix32(i ^ key),
// and the two int8 copies take disjoint halves of the word as 16-bit uniforms: the per-channel copy (t = 0) U = h >> 16,
// the per-tensor copy (t = 1) U = h & 0xFFFF, u = U * 2^-16.  A kernel that writes both copies of an element pays for
// one hash (the calls below are pure, the compiler merges them); nothing is carried from one element to the next.
__host__ __device__ __forceinline__ uint32_t fmix32_rest(uint32_t h) {   // fmix32 behind its first step
    h *= 0x85EBCA6Bu;
    h ^= h >> 13;
    h *= 0xC2B2AE35u;
    h ^= h >> 16;
    return h;
}
__host__ __device__ __forceinline__ uint32_t fmix32(uint32_t h) { return fmix32_rest(h ^ (h >> 16)); }
// key = fmix32(seed_lo ^ fmix32(seed_hi ^ 0x9E3779B9)); it travels in the kernels' 64-bit seed argument
inline uint64_t round_keys(uint64_t seed) {
    const uint32_t lo = (uint32_t)seed, hi = (uint32_t)(seed >> 32);
    return (uint64_t)fmix32(lo ^ fmix32(hi ^ 0x9E3779B9u));
}
// What the kernels carry is the complement of the word: each half of it is then 65535 - U, the form the rounding below adds.
__device__ __forceinline__ uint32_t draw_word(uint64_t keys, uint32_t idx) { return ~fmix32(idx ^ (uint32_t)keys); }
// The words of elements idx .. idx + 3, idx a multiple of four: (idx + e) ^ key is (idx ^ key) ^ e, and as e < 4 touches no bit that
// the mixer's first shift brings down, its first step is shared too (6.5 instead of 9 instructions an element).
__device__ __forceinline__ void draw_words4(uint64_t keys, uint32_t idx, uint32_t (&w)[4]) {
    uint32_t h = idx ^ (uint32_t)keys;
    h ^= h >> 16;
#pragma unroll
    for (int e = 0; e < 4; ++e) w[e] = ~fmix32_rest(h ^ (uint32_t)e);
}
__device__ __forceinline__ uint32_t draw_half(uint32_t w, uint32_t tensor) { return tensor == 0u ? w >> 16 : w & 0xFFFFu; }

// 127/s, or 0 when the scale is treated as zero (then every code is 0).
__device__ __forceinline__ float inv_scale(float s) { return (s >= kTinyScale) ? 127.0f / s : 0.0f; }

// Eq. "suq" in code space: round(clamp(x*inv, -127, 127)).  Stochastic rounding: floor(t) + [frac(t) > U * 2^-16] with
// the element's 16-bit draw U, evaluated in integers: with c = ceil(t * 2^16) (exact: |t| <= 127) the bracket is
// [c mod 2^16 > U] - a fraction of exactly 0 never rounds up, one above U * 2^-16 always - so the code is
// (c + V) >> 16, V = 65535 - U, with an arithmetic shift.
// The code is left in byte kCodeByte of a 32-bit word, the other bytes are don't-care: the shift is the packing's choice of byte.
// Nearest: adding 1.5 * 2^23 to a value of magnitude <= 127 rounds it to an integer, ties to even, and leaves that integer
// in two's complement in the low mantissa bits - one instruction instead of round + convert + mask.
template <bool STOCH> constexpr int kCodeByte = STOCH ? 2 : 0;
template <bool STOCH>
__device__ __forceinline__ uint32_t quant_bits(float x, float inv, uint32_t V) {
    const float t = __builtin_amdgcn_fmed3f(x * inv, -127.0f, 127.0f);   // (a NaN gives -127)
    if constexpr (STOCH) {
        // -ceil(t * 2^16) = floor(-t * 2^16), floor and conversion in one instruction (|t * 2^16| < 2^23: exact)
        int nc;
        asm("v_cvt_flr_i32_f32 %0, %1" : "=v"(nc) : "v"(t * -65536.0f));
        return V - (uint32_t)nc;
    }
    return __float_as_uint(t + 12582912.0f);
}
template <bool STOCH>
__device__ __forceinline__ int8_t code_byte(uint32_t w) { return (int8_t)(w >> (8 * kCodeByte<STOCH>)); }
// Byte B of four words -> one dword (a in byte 0).
template <int B>
__device__ __forceinline__ uint32_t pack4(uint32_t a, uint32_t b, uint32_t c, uint32_t d) {
    constexpr uint32_t sel = 0x0c0c0400u + 0x0101u * B;
    return __builtin_amdgcn_perm(__builtin_amdgcn_perm(d, c, sel), __builtin_amdgcn_perm(b, a, sel), 0x05040100u);
}

// fp32 tensors are read through a buffer descriptor with 32-bit byte offsets: an offset of kOobOff (or
// anything past the extent) returns 0.0f, which is how ragged tiles and padding positions are read
// without branches or selects on the loaded value.  Tensors must be smaller than 2 GiB.
constexpr uint32_t kOobOff = 0x80000000u;
__device__ __forceinline__ __amdgpu_buffer_rsrc_t f32_rsrc(const void* p, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc((void*)p, 0, (int)bytes, 0x00020000);
}
// The tensor to quantize is fp32 (T = float) or bfloat16 (T = uint16_t, the upper half of the fp32 pattern: widening
// is exact, so everything downstream is the fp32 arithmetic on the widened values).  Offsets are in bytes of T.
__device__ __forceinline__ float widen_bf16(uint32_t b) { return __uint_as_float(b << 16); }
template <typename T>
__device__ __forceinline__ float buf_ld(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff) {
    if constexpr (sizeof(T) == 4) return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, (int)voff, (int)soff, 0));
    else return widen_bf16((uint32_t)(uint16_t)__builtin_amdgcn_raw_buffer_load_b16(r, (int)voff, (int)soff, 0));
}
// four consecutive elements as fp32 bit patterns / one element, or zeros (see ld16_or_zero)
template <typename T>
__device__ __forceinline__ uint4 ld4_or_zero(const T* p, bool ok) {
    if constexpr (sizeof(T) == 4) {
        return ld16_or_zero(p, ok);
    } else {
        typedef uint32_t u2_a2 __attribute__((ext_vector_type(2), aligned(2)));
        const u2_a2 v = *reinterpret_cast<const u2_a2*>(ok ? (const void*)p : (const void*)g_zero64);
        return make_uint4(v[0] << 16, v[0] & 0xffff0000u, v[1] << 16, v[1] & 0xffff0000u);
    }
}
template <typename T>
__device__ __forceinline__ float ld1_or_zero(const T* p, bool ok) {
    if constexpr (sizeof(T) == 4) return ldf_or_zero(p, ok);
    else return widen_bf16(*(ok ? p : reinterpret_cast<const uint16_t*>(g_zero64)));
}
__device__ __forceinline__ float buf_ldf(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff) {
    return __uint_as_float((uint32_t)__builtin_amdgcn_raw_buffer_load_b32(r, (int)voff, (int)soff, 0));
}

__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_down(v, o));
    return v;
}
__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o);
    return v;
}
__device__ __forceinline__ uint32_t wave_sum_u32(uint32_t v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o);
    return v;
}

// Fixed-shape workgroup reduction of (max, sum, sum); the result is valid in thread 0.
__device__ __forceinline__ void block_reduce(float& mx, double& s1, double& s2) {
    __shared__ float l_mx[kBlock / kWave];
    __shared__ double l_s1[kBlock / kWave], l_s2[kBlock / kWave];
    mx = wave_max(mx);
    s1 = wave_sum(s1);
    s2 = wave_sum(s2);
    const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
    if (lane == 0) { l_mx[wave] = mx; l_s1[wave] = s1; l_s2[wave] = s2; }
    __syncthreads();
    if (threadIdx.x == 0)
        for (int w = 1; w < kBlock / kWave; ++w) { mx = fmaxf(mx, l_mx[w]); s1 += l_s1[w]; s2 += l_s2[w]; }
}

// ---------------------------------------------------------------------------------------------
// S1: per-channel |g|max, sum, sum of squares.  Workgroup (c, j) sweeps the 4096-element chunks
// j, j + slabs, ... of channel c's flattened (n, h*w) axis, the loads of the next chunk in flight
// while the current one is reduced, and stores one partial.  A channel has at most 16 partials, so
// the kernels that need mean and sigma fold them again themselves (fold_stats) in a fixed order
// instead of waiting for a reduction launch.  Channel c runs on XCD c % 8 in every pass over dY.
// ---------------------------------------------------------------------------------------------
// TAIL: the plane size is not a multiple of four (the last group of a plane needs the move-back and the mask).
template <typename T, bool VEC4, bool TAIL>
__global__ __launch_bounds__(kBlock) void k_stats(const T* __restrict__ g, int N, int C, int HW, FastDiv div_hw,
                                                  QuantWs ws) {
    constexpr int NV = VEC4 ? 4 : 16;
    const int b = blockIdx.x;
    const int xcd = b % kXcd, q = b / kXcd;
    const int c = (q / ws.slabs) * kXcd + xcd;
    const int j = q % ws.slabs;
    if (c >= C) return;
    const int M = N * HW;
    const int tid = threadIdx.x;

    // VEC4: a thread takes groups of four consecutive elements of one (image, channel) plane, any plane size >= 4:
    // planes are cut into ceil(HW/4) groups and the last group of a plane is moved back to end with the plane (its
    // leading elements, already covered by the group before, are zeroed), so every load is a dword-aligned 16-byte
    // load inside the plane.  The flattened axis of a channel is then N * ceil(HW/4) * 4 element slots long.
    const int G4 = (HW + 3) >> 2;
    uint4 v[NV];   // VEC4: four floats each; otherwise only .x is used
    auto fetch = [&](int chunk, uint4 (&dst)[NV]) {
        const bool live = chunk < ws.chunks;
        const int m0 = chunk * kStatsElems;
#pragma unroll
        for (int u = 0; u < NV; ++u) {
            if (VEC4) {
                const int q4 = (m0 >> 2) + tid + u * kBlock;            // group index inside the channel
                const bool ok = live && q4 < N * G4;
                const int qc = ok ? q4 : 0;
                const int n = (int)fdiv((uint32_t)qc, div_hw), gi = qc - n * G4;   // div_hw divides by G4 here
                const int i = TAIL ? min(4 * gi, HW - 4) : 4 * gi;
                uint4 r = ld4_or_zero<T>(g + ((int64_t)n * C + c) * HW + i, ok);
                if (TAIL) {
                    const int skip = 4 * gi - i;   // > 0 only in a plane's last group
                    r.x = skip > 0 ? 0u : r.x;
                    r.y = skip > 1 ? 0u : r.y;
                    r.z = skip > 2 ? 0u : r.z;
                }
                dst[u] = r;
            } else {
                const int m = m0 + tid + u * kBlock;
                const bool ok = live && m < M;
                const int mc = ok ? m : 0;
                const int n = (int)fdiv((uint32_t)mc, div_hw), i = mc - n * HW;
                dst[u].x = __float_as_uint(ld1_or_zero<T>(g + ((int64_t)n * C + c) * HW + i, ok));
            }
        }
    };
    float mx = 0.0f;
    double s1 = 0.0, s2 = 0.0;
    fetch(j, v);
    for (int chunk = j; chunk < ws.chunks; chunk += ws.slabs) {
        uint4 nv[NV];
        fetch(chunk + ws.slabs, nv);
#pragma unroll
        for (int u = 0; u < NV; ++u) {
            const float f0 = __uint_as_float(v[u].x);
            mx = fmaxf(mx, fabsf(f0));
            const double a = f0;
            s1 += a;
            s2 += a * a;
            if (VEC4) {
                const float f1 = __uint_as_float(v[u].y), f2 = __uint_as_float(v[u].z), f3 = __uint_as_float(v[u].w);
                mx = fmaxf(mx, fmaxf(fabsf(f1), fmaxf(fabsf(f2), fabsf(f3))));
                const double bq = f1, cq = f2, d = f3;
                s1 += bq; s1 += cq; s1 += d;
                s2 += bq * bq; s2 += cq * cq; s2 += d * d;
            }
        }
#pragma unroll
        for (int u = 0; u < NV; ++u) v[u] = nv[u];
    }
    block_reduce(mx, s1, s2);
    if (tid == 0) {
        const int64_t slot = (int64_t)c * ws.slabs + j;
        ws.part_max[slot] = mx;
        ws.part_s1[slot] = s1;
        ws.part_s2[slot] = s2;
    }
}

// The value of the lane before, within rows of 16 lanes (of the first of a row: its own).
__device__ __forceinline__ float lane_before(float v) {
    const int b = __builtin_bit_cast(int, v);
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(b, b, 0x111, 0xF, 0xF, false));
}
__device__ __forceinline__ double lane_before(double v) {
    v2u b = __builtin_bit_cast(v2u, v);
#pragma unroll
    for (int i = 0; i < 2; ++i) b[i] = (uint32_t)__builtin_amdgcn_update_dpp((int)b[i], (int)b[i], 0x111, 0xF, 0xF, false);
    return __builtin_bit_cast(double, b);
}

// Partials of channel c (of C) -> |g|max, mean, sigma (population std about the mean, fp64, rounded once), by four adjacent lanes, a
// quarter of the slots each; valid in the last of the four.  The sum runs through the slots in their order, from lane to lane, so
// every workgroup that calls it gets the same bits.  All partials are requested before the first one is used; slots past
// `slabs` read zeros, which change nothing.
__device__ __forceinline__ void fold_stats(const QuantWs& ws, int c, int C, double Md, float& gmax, float& mean, float& sigma) {
    constexpr int kEach = kMaxSlabs / 4;
    const int part = (int)threadIdx.x % 4;
    float pm[kEach];
    double p1[kEach], p2[kEach];
#pragma unroll
    for (int j = 0; j < kEach; ++j) {
        const int at = kEach * part + j;
        const bool ok = at < ws.slabs && c < C;
        const int64_t slot = (int64_t)c * ws.slabs + at;
        pm[j] = ldf_or_zero(ws.part_max + slot, ok);
        p1[j] = *(ok ? ws.part_s1 + slot : reinterpret_cast<const double*>(g_zero64));
        p2[j] = *(ok ? ws.part_s2 + slot : reinterpret_cast<const double*>(g_zero64));
    }
    float mx = 0.0f;
    double s1 = 0.0, s2 = 0.0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        if (k) {   // what the lane before has: after step k lane k of the four is complete
            mx = lane_before(mx);
            s1 = lane_before(s1);
            s2 = lane_before(s2);
        }
#pragma unroll
        for (int j = 0; j < kEach; ++j) {
            mx = fmaxf(mx, pm[j]);
            s1 += p1[j];
            s2 += p2[j];
        }
    }
    const double mu = s1 / Md;
    double var = s2 / Md - mu * mu;
    if (var < 0.0) var = 0.0;
    gmax = mx;
    mean = (float)mu;
    sigma = (float)sqrt(var);
}

// S4: clip value of a channel of the given class (Eq. "gaus": |g|max; Eq. "fats": (1-kA) s_prev + A |g|max, with a
// non-positive state meaning "no history" and a non-positive result replaced by |g|max).
__device__ __forceinline__ float clip_rule(int klass, float gm, float prev, float k, float A) {
    float s = gm;
    if (klass == DAQ_CLASS_INVT) {
        if (!(prev > 0.0f)) prev = gm;
        s = (float)((1.0 - (double)k * (double)A) * (double)prev + (double)A * (double)gm);
        if (!(s > 0.0f)) s = gm;
    }
    return s;
}

// What the counting pass needs to write the per-channel copy of channels whose class it can guess.
struct EarlyVq {
    int8_t* vq;            // nullptr: the counting pass does not write the per-channel copy
    int8_t* qg;            // a global copy in the same layout (depthwise layers), or nullptr
    int64_t chan_pitch;
    int32_t lead, img_rows, row_pitch, W;
    FastDiv div_w;
    float k, A;
    float ratio;           // a channel with |g|max > ratio * sigma is taken for long-tailed
    int flat;              // no padding between rows and images: element m of a channel is byte lead + m
    int once;              // larger than the caches hold to the end: read past them
    int whole;             // four pixels of a unit are four consecutive bytes (flat, or rows of whole units)
};

// How the counting pass reads a channel plane: in units of four consecutive pixels (kWhole: planes are whole units; kTail: the
// last unit of a plane is moved back to end with it, what it shares with the unit before is written twice, the same both
// times, and counted once), or, planes of less than four pixels, four consecutive pixels of the flattened axis one by one.
enum : int { kWhole, kTail, kElems };
inline int unit_kind(int HW) { return HW < 4 ? kElems : HW % 4 ? kTail : kWhole; }
__host__ __device__ inline int plane_units(int HW) { return (HW + 3) / 4; }
int64_t channel_units(int N, int HW) { return HW < 4 ? ceil_div((int64_t)N * HW, 4) : (int64_t)N * plane_units(HW); }
inline uint32_t unit_divisor(int HW) { return (uint32_t)(HW < 4 ? HW : plane_units(HW)); }   // what div_u of the pass divides by

// Four registers of four rows of 16 lanes, transposed: register k of row r receives register r of row k.
__device__ __forceinline__ void transpose_rows(uint32_t (&w)[4]) {
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const auto t = __builtin_amdgcn_permlane32_swap(w[k], w[k + 2], false, false);
        w[k] = t[0];
        w[k + 2] = t[1];
    }
#pragma unroll
    for (int k = 0; k < 4; k += 2) {
        const auto t = __builtin_amdgcn_permlane16_swap(w[k], w[k + 1], false, false);
        w[k] = t[0];
        w[k + 1] = t[1];
    }
}

// ---------------------------------------------------------------------------------------------
// S2 (+ the global copy of S5): tail-mass count per channel, fused with the globally quantized
// NHWC copy.  A workgroup owns a block of up to 192 channels (block_width) and walks tiles of 16 units (64 pixels) of the
// flattened (n, h*w) axis; a wave handles 16 of the channels.  Where the block leaves waves over (thin tensors, the smaller
// last block), the waves form several sides, each with a tile of its own.  Lane 16 r + q holds unit q of channels 4r .. 4r+3 of
// the wave's: four 16-byte loads, each 256 consecutive bytes of four channels a wave, the random words of a unit from one
// first step, a per-channel unit is one dword, and four instructions between the lanes (transpose_rows) turn the codes of
// four channels x one unit into 16 channels x one pixel for the NHWC copy.
// A wave first folds the statistics partials of its own 16 channels (sigma), the workgroup those of all channels
// (the global scale max_c |g|max); then the pass counts into registers and stores one
// count partial per channel: no atomics, no reduction launch.
// Registers: 128, four waves a SIMD.  The copy alone needs 54 to 64 of them, the count with it 80 to 90, all of it with stochastic codes 127 on
// planes of whole units, with 22 scalars kept in vector lanes; with a shorter last unit 3 vector registers are spilled, on planes of
// less than a unit (kElems, which loads and places each element by itself) 32.
// ---------------------------------------------------------------------------------------------
//
// EARLY: the pass also writes the per-channel copy vq.  The class of a channel is only known once the counts of all
// its workgroups are in, but |g|max / sigma, known here, separates bell-shaped from long-tailed channels almost
// always: every workgroup derives the same guess and the clip value that follows from it (same arithmetic as the
// final decision), quantizes with it and stores the bytes of the real elements; the packing pass, which takes the
// decision, then only rewrites the channels whose guess was wrong (and writes the padding).  A correct guess saves
// the third sweep over dY for that channel; a wrong one costs nothing but the bytes written here.
// `bid`: the workgroup's number among those of this role (the forward pass launches it with other roles, k_fwd_quant).
template <typename T, bool STOCH, bool WRITE_QG, bool COUNT, bool EARLY, int UNIT>
__device__ __forceinline__ void count_qg_role(const int bid, const T* __restrict__ g, int N, int C, int HW, int c_pitch, FastDiv div_u,
                                              const QuantWs& ws, int8_t* __restrict__ qg, uint64_t seed, const float* __restrict__ s_state,
                                              float* __restrict__ s_global, const EarlyVq& ev, int qg_tail, uint32_t* l_tile, int tile_dw) {
    __shared__ __align__(16) float l_max[kCountMaxWaves];
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid / kWave), lane = tid % kWave;
    const int uq = lane % 16, row = lane / 16;
    const CountPlan& cp = ws.cp;
    const int cb = min((int)fdiv((uint32_t)bid, cp.div_cgroups), cp.blocks - 1);
    const int p = bid - cb * cp.cgroups;
    const int cgroups = cb + 1 == cp.blocks ? cp.cgroups_last : cp.cgroups;
    // A wave to 16 channels of the block; where that leaves waves over (thin tensors, a last block), the workgroup has several
    // sides, each with a tile of its own.
    const int gb = cp.groups(C, cb);   // uniform, as are the next two
    const uint32_t by_gb = cp.by_groups[cb + 1 == cp.blocks ? 1 : 0];
    const int sides = (int)(((uint32_t)cp.waves * by_gb) >> 16);
    const int side = (int)(((uint32_t)wave * by_gb) >> 16), kg = wave - side * gb;
    const int c0 = 16 * (cb * cp.width + kg);
    const int cl = c0 + 4 * row;                              // the lane's first channel
    const int wg_tiles = (cp.tiles + sides - 1) / sides;
    const int pitch = CountPlan::pitch_dwords(gb), step = CountPlan::step_dwords(gb);
    const uint32_t M = (uint32_t)N * (uint32_t)HW;
    constexpr uint32_t EB = sizeof(T);   // bytes of a source element
    const __amdgpu_buffer_rsrc_t rs = f32_rsrc(g, (uint32_t)M * (uint32_t)C * EB);
    const uint32_t upp = (uint32_t)plane_units(HW), units = UNIT == kElems ? (M + 3) / 4 : (uint32_t)N * upp;

    // Which tiles the workgroup walks.  A tile's 256-byte pieces of its channel planes start wherever the plane starts, so
    // neighbouring tiles share cache lines; with the workgroups of a channel block dealt round-robin over the tiles,
    // neighbours ran on different XCDs and both L2s fetched the shared lines (1.4 x the tensor on 14 x 14 planes).  With
    // a multiple of eight workgroups per block, workgroup p runs on XCD p % 8: each XCD takes one contiguous eighth of
    // the tiles, and its workgroups p / 8 walk that range side by side.
    int t_first = p, t_step = cgroups, t_end = wg_tiles;
    if (((cp.cgroups | cgroups) & (kXcd - 1)) == 0) {   // uniform
        const int per_xcd = (wg_tiles + kXcd - 1) / kXcd, xcd = p % kXcd;
        t_first = xcd * per_xcd + p / kXcd;
        t_step = cgroups / kXcd;
        t_end = min(wg_tiles, (xcd + 1) * per_xcd);
    }

    // image and first pixel of unit u of the channel, and how many of its pixels belong to the unit before (kWhole, kTail)
    auto place = [&](uint32_t u, uint32_t& n, uint32_t& px, uint32_t& dup) {
        n = fdiv(u, div_u);
        const uint32_t at = (u - n * upp) * 4u;
        px = UNIT == kTail ? min(at, (uint32_t)HW - 4u) : at;
        dup = at - px;
    };
    // pixel e of a unit of kElems
    auto pixel = [&](uint32_t u, uint32_t e, uint32_t& n, uint32_t& px) {
        const uint32_t P = min(4u * u + e, M - 1u);
        n = fdiv(P, div_u);
        px = P - n * (uint32_t)HW;
    };
    struct Unit {
        float x[4][4];     // channel, pixel
        uint32_t u;
        bool ok;
    };
    auto fetch = [&](int tile, Unit& t) {
        const uint32_t u = (uint32_t)(sides * tile + side) * 16u + (uint32_t)uq;
        t.ok = tile < t_end && side < sides && u < units;
        t.u = t.ok ? u : 0u;
        if constexpr (UNIT == kElems) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                uint32_t n, px;
                pixel(t.u, e, n, px);
                const uint32_t off = ((n * (uint32_t)C + (uint32_t)cl) * (uint32_t)HW + px) * EB;
#pragma unroll
                for (int j = 0; j < 4; ++j) t.x[j][e] = buf_ld<T>(rs, t.ok && 4u * t.u + e < M && cl + j < C ? off : kOobOff, (uint32_t)(j * HW) * EB);
            }
        } else {
            uint32_t n, px, dup;
            place(t.u, n, px, dup);
            const uint32_t at = (n * (uint32_t)C + (uint32_t)cl) * (uint32_t)HW + px;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const bool ok = t.ok && cl + j < C;
                if constexpr (EB == 4) {
                    const int voff = (int)(ok ? at * EB : kOobOff), soff = (int)((uint32_t)(j * HW) * EB);
                    v4u raw;
                    if (EARLY && ev.once) raw = __builtin_amdgcn_raw_buffer_load_b128(rs, voff, soff, 2);   // uniform; nt
                    else raw = __builtin_amdgcn_raw_buffer_load_b128(rs, voff, soff, 0);
#pragma unroll
                    for (int e = 0; e < 4; ++e) t.x[j][e] = __uint_as_float(raw[e]);
                } else {
                    const uint4 raw = ld4_or_zero<T>(g + at + (uint32_t)(j * HW), ok);
                    t.x[j][0] = __uint_as_float(raw.x);
                    t.x[j][1] = __uint_as_float(raw.y);
                    t.x[j][2] = __uint_as_float(raw.z);
                    t.x[j][3] = __uint_as_float(raw.w);
                }
            }
        }
    };
    Unit a, b;
    fetch(t_first, a);

    // scale of the global copy: the maximum over the partials of the launch before
    const int threads = cp.waves * kWave;
    {
        float m = 0.0f;
        const int total = ws.part_n;
        for (int base = 0; base < total; base += 8 * threads) {
            float v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = ldf_or_zero(ws.part_max + base + u * threads + tid, base + u * threads + tid < total);
#pragma unroll
            for (int u = 0; u < 8; ++u) m = fmaxf(m, v[u]);
        }
        m = wave_max(m);
        if (lane == 0) l_max[wave] = m;
        if (tid < kCountMaxWaves && tid >= cp.waves) l_max[tid] = 0.0f;
    }
    // sigma and 127/s of the lane's four channels, from the wave's own fold.  Lanes without a unit and channels past C hold x = 0, and
    // 0 > sigma is false for every sigma >= 0, so the comparison needs no validity mask.
    float sig[4] = {}, inv_c[4] = {};
    if constexpr (COUNT) {
        const int c = c0 + lane / 4;   // four lanes to a channel; the last of them ends up with the fold
        float gm, mu, sg_c, inv_e = 0.0f;
        fold_stats(ws, c, C, (double)N * (double)HW, gm, mu, sg_c);
        const bool mine = lane % 4 == 3 && c < C;
        if (mine && side == 0 && p == 0) { ws.gmax[c] = gm; ws.mean[c] = mu; ws.sigma[c] = sg_c; }
        if constexpr (EARLY) {
            const int guess = gm > ev.ratio * sg_c ? DAQ_CLASS_INVT : DAQ_CLASS_GAUSS;
            inv_e = inv_scale(clip_rule(guess, gm, c < C ? s_state[c] : 0.0f, ev.k, ev.A));
            if (mine && side == 0 && p == 0) ws.pred[c] = (uint32_t)guess;
        }
        // layer-wise clipping compares every element with the standard deviation of the whole tensor
        if (ws.scheme == DAQ_SCHEME_MCS) sg_c = ws.layer[2];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            sig[j] = __shfl(sg_c, 16 * row + 4 * j + 3);
            if (EARLY) inv_c[j] = __shfl(inv_e, 16 * row + 4 * j + 3);
        }
    }
    __syncthreads();
    float sg = 0.0f;
#pragma unroll
    for (int w = 0; w < kCountMaxWaves; ++w) sg = fmaxf(sg, l_max[w]);
    const float sg_raw = sg;
    if (!(sg >= kTinyScale)) sg = 0.0f;
    if (COUNT && bid == 0) {
        // the clip state is overwritten by the packing pass: keep what this iteration started from
        for (int i = tid; i < C; i += threads) ws.s_prev[i] = s_state[i];
    }
    if (bid == 0 && tid == 0) {
        *s_global = sg;
        ws.layer[0] = sg_raw;
    }
    // the NHWC buffer is a multiple of 256 bytes long: the bytes behind the last pixel hold no element and are zero
    if (WRITE_QG && bid == 0)
        for (int i = tid; i < qg_tail; i += threads) qg[(int64_t)M * c_pitch + i] = 0;
    const float inv = inv_scale(sg);
    if constexpr (EARLY && !COUNT) {   // forward: one scale
#pragma unroll
        for (int j = 0; j < 4; ++j) inv_c[j] = inv;
    }
    // what the lane stores of a tile: a 16-byte unit of one of its side's pixels
    const int at_px = (int)(((uint32_t)(kg * kWave + lane) * by_gb) >> 16), at_ch = (kg * kWave + lane) - at_px * gb;
    int8_t* const qg_lane = WRITE_QG ? qg + 16 * (cb * cp.width + (gb == 1 ? 0 : at_ch)) : nullptr;
    int8_t* const vq_lane = EARLY ? ev.vq + (int64_t)cl * ev.chan_pitch + (uint32_t)ev.lead : nullptr;
    constexpr bool BOTH = EARLY && COUNT && !WRITE_QG;   // both copies channel-major
    const int64_t to_qg = BOTH ? ev.qg - ev.vq : 0;

    uint32_t cnt[4] = {0u, 0u, 0u, 0u};
    auto work = [&](int tile, const Unit& t, uint32_t* tile_buf) {
        uint32_t n = 0, px = 0, dup = 0;
        if constexpr (UNIT != kElems) place(t.u, n, px, dup);
        const uint32_t idx0 = (n * (uint32_t)C + (uint32_t)cl) * (uint32_t)HW + px;   // NCHW index; the lane's channels are one plane apart
        // channel-major copy: the unit sits at the same offset of each of the lane's four channel planes
        uint32_t at_vq = 0;
        uint32_t in_row = 4u, gap = 0u;   // pixels of the unit in its first row, bytes between the rows
        bool whole = true;   // the unit does not run on into the next row
        if constexpr (EARLY && UNIT != kElems) {
            const uint32_t h = ev.flat ? 0u : fdiv(px, ev.div_w);
            const uint32_t col = px - h * (uint32_t)ev.W;
            in_row = (uint32_t)ev.W - col;
            gap = (uint32_t)ev.row_pitch - (uint32_t)ev.W;
            whole = ev.whole || col + 4u <= (uint32_t)ev.W;
            at_vq = ev.flat ? n * (uint32_t)HW + px : (n * (uint32_t)ev.img_rows + h) * (uint32_t)ev.row_pitch + col;
        }
        uint32_t d[4];   // global codes: pixel k of the unit, the lane's four channels
        uint32_t half[4];
        constexpr uint32_t kB = 0x0101u * kCodeByte<STOCH>;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            uint32_t draw[4] = {0u, 0u, 0u, 0u};
            if constexpr (STOCH && (WRITE_QG || EARLY)) {
                const uint32_t idx = idx0 + (uint32_t)(j * HW);
                if constexpr (UNIT == kWhole) {
                    draw_words4(seed, idx, draw);
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        uint32_t at = idx + (uint32_t)e;
                        if constexpr (UNIT == kElems) {
                            uint32_t ne, pe;
                            pixel(t.u, e, ne, pe);
                            at = (ne * (uint32_t)C + (uint32_t)(cl + j)) * (uint32_t)HW + pe;
                        }
                        draw[e] = draw_word(seed, at);
                    }
                }
            }
            uint32_t vb[4], gb4[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float v = t.x[j][e];
                if (COUNT) cnt[j] += (fabsf(v) > sig[j] && (UNIT != kTail || e == 3 || (uint32_t)e >= dup)) ? 1u : 0u;
                if (WRITE_QG) {
                    const uint32_t w = quant_bits<STOCH>(v, inv, draw_half(draw[e], 1u));
                    if (j % 2 == 0) half[e] = w;
                    else half[e] = __builtin_amdgcn_perm(w, half[e], 0x0c0c0400u + kB);
                    if (j == 1) d[e] = half[e];
                    if (j == 3) d[e] = __builtin_amdgcn_perm(half[e], d[e], 0x05040100u);
                }
                if (EARLY) vb[e] = quant_bits<STOCH>(v, inv_c[j], draw_half(draw[e], 0u));
                if (BOTH) gb4[e] = quant_bits<STOCH>(v, inv, draw_half(draw[e], 1u));
            }
            if (EARLY && t.ok && cl + j < C) {
                const uint32_t wv = pack4<kCodeByte<STOCH>>(vb[0], vb[1], vb[2], vb[3]);
                const uint32_t wg = BOTH ? pack4<kCodeByte<STOCH>>(gb4[0], gb4[1], gb4[2], gb4[3]) : 0u;
                int8_t* plane = vq_lane + (int64_t)j * ev.chan_pitch;
                if (UNIT != kElems && whole) {
                    __builtin_memcpy(plane + at_vq, &wv, 4);   // byte aligned only
                    if (BOTH) __builtin_memcpy(plane + to_qg + at_vq, &wg, 4);
                } else if (UNIT != kElems && !COUNT && ev.W >= 4 && ev.W % 2 == 0) {
                    // Rows of an even length: units begin at even columns, and two pixels are here, two in the next row, in half the stores (a forward call of 109 x 743 x 26 x 26, padded, 203 -> 197 us, 49 layers of such rows
                    // 0.98 -> 1.00 of a byte at a time for all of them; the counting forms lose 1 % on other rows to one more spilled scalar)
                    const uint16_t two[2] = {(uint16_t)wv, (uint16_t)(wv >> 16)};
#pragma unroll
                    for (int e = 0; e < 2; ++e) __builtin_memcpy(plane + at_vq + (uint32_t)e * (2u + gap), &two[e], 2);
                } else if (UNIT != kElems && ev.W >= 4) {   // into the next row at most
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const uint32_t at = at_vq + (uint32_t)e + ((uint32_t)e >= in_row ? gap : 0u);
                        plane[at] = (int8_t)(wv >> (8 * e));
                        if (BOTH) plane[to_qg + at] = (int8_t)(wg >> (8 * e));
                    }
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        uint32_t ne = n, pe = px + (uint32_t)e;
                        if constexpr (UNIT == kElems) pixel(t.u, e, ne, pe);
                        const uint32_t he = fdiv(pe, ev.div_w);
                        const uint32_t at = (ne * (uint32_t)ev.img_rows + he) * (uint32_t)ev.row_pitch + (pe - he * (uint32_t)ev.W);
                        if (UNIT != kElems || 4u * t.u + e < M) {
                            plane[at] = (int8_t)(wv >> (8 * e));
                            if (BOTH) plane[to_qg + at] = (int8_t)(wg >> (8 * e));
                        }
                    }
                }
            }
            if (EARLY && j < 3) __builtin_amdgcn_sched_barrier(0);   // a channel at a time: four at once do not fit the registers
        }
        if (WRITE_QG) {
            // then pixel `row` of the unit, channels 4k .. 4k+3 of the wave's
            transpose_rows(d);
            const uint4 rec = make_uint4(d[0], d[1], d[2], d[3]);
            if (gb == 1) {   // uniform
                const uint32_t P = (UNIT == kElems ? 4u * t.u : n * (uint32_t)HW + px) + (uint32_t)row;
                if (t.ok && (UNIT != kElems || P < M)) *reinterpret_cast<uint4*>(qg_lane + (int64_t)P * c_pitch) = rec;   // bytes of channels past C are codes of 0.0f: zeros
            } else {
                // A lane holds 16 channel bytes of ONE pixel, so a direct store would put 16 bytes into each of 64 different
                // places.  The tile goes through LDS instead and leaves as whole runs: gb adjacent lanes write what the block
                // has of a pixel's record.
                uint32_t* l = tile_buf + side * 4 * step;
                if (side < sides) *reinterpret_cast<uint4*>(l + row * step + uq * pitch + 4 * kg) = rec;
                __syncthreads();   // (a wave that is here again for the next tile but one has seen all others read this one)
                const uint32_t u = (uint32_t)(sides * tile + side) * 16u + (uint32_t)(at_px >> 2);
                uint32_t P = 4u * u;
                if constexpr (UNIT == kTail) {
                    uint32_t on, opix, odup;
                    place(u, on, opix, odup);
                    P = on * (uint32_t)HW + opix;
                }
                P += (uint32_t)(at_px & 3);
                if (side < sides && u < units && (UNIT != kElems || P < M))
                    *reinterpret_cast<uint4*>(qg_lane + (int64_t)P * c_pitch) =
                        *reinterpret_cast<const uint4*>(l + (at_px & 3) * step + (at_px >> 2) * pitch + 4 * at_ch);
            }
        }
    };
    // the next tile's loads are in flight while a tile is worked on; two buffers that take turns
    for (int tile = t_first; tile < t_end; tile += 2 * t_step) {
        fetch(tile + t_step, b);
        work(tile, a, l_tile);
        if (tile + t_step >= t_end) break;
        fetch(tile + 2 * t_step, a);
        work(tile + t_step, b, l_tile + tile_dw);
    }
    if (COUNT) {
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int o = 8; o > 0; o >>= 1) cnt[j] += __shfl_xor(cnt[j], o);   // over the row's 16 units
        uint32_t mine = 0;   // lane 16 r + j, j < 4: channel 4 r + j of the wave's
#pragma unroll
        for (int j = 0; j < 4; ++j) mine = uq == j ? cnt[j] : mine;
        const bool mine_ok = uq < 4 && cl + uq < C && side < sides;
        if (sides > 1) {   // uniform: waves counted the same channels on different tiles
            __shared__ uint32_t l_cnt[kCountMaxWaves * 16];
            if (uq < 4) l_cnt[16 * wave + 4 * row + uq] = mine;
            __syncthreads();
            if (side == 0 && mine_ok) {
                uint32_t all = 0;
                for (int w = kg; w < sides * gb; w += gb) all += l_cnt[16 * w + 4 * row + uq];
                ws.part_cnt[(int64_t)(cl + uq) * cp.cgroups + p] = all;
            }
        } else if (mine_ok) {
            ws.part_cnt[(int64_t)(cl + uq) * cp.cgroups + p] = mine;
        }
        if (ws.scheme == DAQ_SCHEME_MCS) {   // uniform: one population; its count is the sum over all counting waves
            const uint32_t all = wave_sum_u32(mine_ok ? mine : 0u);
            if (lane == 0) ws.layer_cnt[bid * cp.waves + wave] = all;
        }
    }
}

template <typename T, bool STOCH, bool WRITE_QG, bool COUNT, bool EARLY, int UNIT>
__global__ __launch_bounds__(kCountMaxWaves * kWave, 4) void k_count_qg(const T* __restrict__ g, int N, int C, int HW, int c_pitch, FastDiv div_u,
                                                        QuantWs ws, int8_t* __restrict__ qg, uint64_t seed,
                                                        const float* __restrict__ s_state, float* __restrict__ s_global, EarlyVq ev,
                                                        int qg_tail, int tile_dw) {
    extern __shared__ __align__(16) uint32_t l_records[];   // two tiles (CountPlan::tile_dwords)
    count_qg_role<T, STOCH, WRITE_QG, COUNT, EARLY, UNIT>((int)blockIdx.x, g, N, C, HW, c_pitch, div_u, ws, qg, seed, s_state, s_global, ev, qg_tail, l_records, tile_dw);
}

// ---------------------------------------------------------------------------------------------
// Layer-wise Magnitude-aware Clipping (ablation study, the variant without vectorized quantization): the
// tensor is one population.  Two single-workgroup launches around the counting pass: before it, the statistics
// partials of all channels are folded into the tensor's mean and sigma (fixed summation order, so the result does
// not depend on the launch); after it, the counts of the counting waves into the tail mass, the class (Eq.
// "judge") and the clip value (Eq. "gaus" / Eq. "fats", with s_state[0] as the history).
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(kBlock) void k_layer_stats(QuantWs ws, int C, double Mtot) {
    __shared__ double l_1[kBlock], l_2[kBlock];
    const int tid = threadIdx.x;
    double s1 = 0.0, s2 = 0.0;
    const int total = C * ws.slabs;
    for (int i = tid; i < total; i += kBlock) {
        s1 += ws.part_s1[i];
        s2 += ws.part_s2[i];
    }
    l_1[tid] = s1;
    l_2[tid] = s2;
    __syncthreads();
    for (int h = kBlock / 2; h > 0; h >>= 1) {
        if (tid < h) {
            l_1[tid] += l_1[tid + h];
            l_2[tid] += l_2[tid + h];
        }
        __syncthreads();
    }
    if (tid == 0) {
        const double mu = l_1[0] / Mtot;
        double var = l_2[0] / Mtot - mu * mu;
        if (var < 0.0) var = 0.0;
        ws.layer[1] = (float)mu;
        ws.layer[2] = (float)sqrt(var);
    }
}

__global__ __launch_bounds__(kBlock) void k_layer_decide(QuantWs ws, int waves, double Mtot, float k, float A, float lambda) {
    __shared__ uint32_t l_c[kBlock];
    const int tid = threadIdx.x;
    uint32_t cnt = 0;
    for (int base = 0; base < waves; base += 8 * kBlock) {   // eight loads in flight per thread
        uint32_t v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int i = base + u * kBlock + tid;
            v[u] = i < waves ? ws.layer_cnt[i] : 0u;
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) cnt += v[u];
    }
    l_c[tid] = cnt;
    __syncthreads();
    for (int h = kBlock / 2; h > 0; h >>= 1) {
        if (tid < h) l_c[tid] += l_c[tid + h];
        __syncthreads();
    }
    if (tid == 0) {
        const double n = (double)l_c[0];
        const int klass = (n > (double)lambda * Mtot) ? DAQ_CLASS_GAUSS : DAQ_CLASS_INVT;
        ws.layer[3] = (float)(n / Mtot);
        ws.layer[4] = clip_rule(klass, ws.layer[0], ws.s_prev[0], k, A);
        ws.layer[5] = (float)klass;
    }
}

struct ClipArgs {
    float k, A, lambda;
    float* s_state;
    float* s_chan;
    uint8_t* cls;
    float* stats;
};

// ---------------------------------------------------------------------------------------------
// S5, channel-major copy: fp32 NCHW -> int8 CNHW (the dimension transformation G -> G', X -> X'),
// with S3 + S4 folded in for the per-channel copy of dY.
//
// Output driven: a workgroup produces 4096 consecutive bytes of one channel's plane, a thread four
// aligned dwords (256 dwords apart), including the zero bytes that serve as convolution padding, so
// every byte of the buffer is written exactly once, stores are 256-byte runs per wave and the loads
// of neighbouring lanes fall into the same cache lines.  All 16 loads of a thread are in flight
// before the scale is needed.
//
// CLIP: the scale is the channel's Magnitude-aware Clipping value.  Every workgroup of the channel
// sums the count partials of the counting pass, applies the discriminator (Eq. "judge") and the clip
// rule (Eq. "gaus" / Eq. "fats") to identical inputs in identical order, and the channel's first
// workgroup publishes s_chan, the class, the new state and the optional statistics.
// ---------------------------------------------------------------------------------------------
// S2 (sum of the count partials) + S3 discriminator + S4 clip rule for channel c, evaluated by a whole
// workgroup; every workgroup of the channel gets the same value, `publish` marks the one that writes it out.
__device__ __forceinline__ float clip_value(const QuantWs& ws, const ClipArgs& ca, int c, double Md, bool publish,
                                            uint32_t* l_cnt, int* klass_out = nullptr) {
    const int tid = threadIdx.x;
    if (ws.scheme == DAQ_SCHEME_MCS) {   // uniform: the layer's clip value, decided by k_layer_decide, for every channel
        const float s = ws.layer[4];
        if (klass_out) *klass_out = (int)ws.layer[5];
        if (publish && tid == 0) {
            ca.s_state[c] = s;
            ca.s_chan[c] = (s >= kTinyScale) ? s : 0.0f;
            ca.cls[c] = (uint8_t)ws.layer[5];
            if (ca.stats) {
                ca.stats[4 * c + 0] = ws.layer[0];
                ca.stats[4 * c + 1] = ws.layer[1];
                ca.stats[4 * c + 2] = ws.layer[2];
                ca.stats[4 * c + 3] = ws.layer[3];
            }
        }
        return s;
    }
    uint32_t cnt = 0;
    static_assert(kCountGroups <= 4 * kBlock, "a thread sums at most four count partials");
    {
        const int have = c / (16 * ws.cp.width) + 1 == ws.cp.blocks ? ws.cp.cgroups_last : ws.cp.cgroups;
        uint32_t v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int i = tid + u * kBlock;
            v[u] = __float_as_uint(ldf_or_zero(reinterpret_cast<const float*>(ws.part_cnt + (int64_t)c * ws.cp.cgroups + i), i < have));
        }
        cnt = v[0] + v[1] + v[2] + v[3];
    }
    cnt = wave_sum_u32(cnt);
    if (tid % kWave == 0) l_cnt[tid / kWave] = cnt;
    __syncthreads();
    cnt = l_cnt[0] + l_cnt[1] + l_cnt[2] + l_cnt[3];
    const int klass = ((double)cnt > (double)ca.lambda * Md) ? DAQ_CLASS_GAUSS : DAQ_CLASS_INVT;
    if (klass_out) *klass_out = klass;   // every thread holds the same sum, hence the same class
    const float gm = ws.gmax[c];
    // ablation baselines: the tensor's |g|max for every channel (GQ) or the channel's own without clipping (GVQ);
    // class and statistics are reported as Algorithm 1 computes them
    const float s = ws.scheme == DAQ_SCHEME_GQ    ? ws.layer[0]
                    : ws.scheme == DAQ_SCHEME_GVQ ? gm
                                                  : clip_rule(klass, gm, ws.s_prev[c], ca.k, ca.A);
    if (publish && tid == 0) {
        ca.s_state[c] = s;
        ca.s_chan[c] = (s >= kTinyScale) ? s : 0.0f;
        ca.cls[c] = (uint8_t)klass;
        if (ca.stats) {
            ca.stats[4 * c + 0] = gm;
            ca.stats[4 * c + 1] = ws.mean[c];
            ca.stats[4 * c + 2] = ws.sigma[c];
            ca.stats[4 * c + 3] = (float)((double)cnt / Md);
        }
    }
    return s;
}

// Scale of a per-tensor copy from the partial maxima of the launch before (fixed tree; every thread gets it).  Called by
// all kBlock threads; `l` is kBlock / kWave floats of LDS.
__device__ __forceinline__ float fold_scale(const float* __restrict__ part, int n, float* l) {
    float m = 0.0f;
    for (int i = threadIdx.x; i < n; i += kBlock) m = fmaxf(m, part[i]);
    m = wave_max(m);
    if (threadIdx.x % kWave == 0) l[threadIdx.x / kWave] = m;
    __syncthreads();
    return fmaxf(fmaxf(l[0], l[1]), fmaxf(l[2], l[3]));
}

// The scale of a per-tensor copy: a value, or the maximum of part_n partials, which `first` (one workgroup) publishes.
__device__ __forceinline__ float given_scale(const float* __restrict__ scale, int part_n, float* publish, float* publish_raw, bool first, float* l) {
    if (!part_n) return scale[0];
    const float s = fold_scale(scale, part_n, l);
    if (publish && first && threadIdx.x == 0) {
        *publish = s >= kTinyScale ? s : 0.0f;
        *publish_raw = s;
    }
    return s;
}

// The same by one workgroup, for packing launches whose own many would spend longer on it (fold_in_packing).
__global__ __launch_bounds__(kBlock) void k_fold_scale(const float* __restrict__ part, int n, float* publish, float* publish_raw) {
    __shared__ float l_m[kBlock / kWave];
    given_scale(part, n, publish, publish_raw, true, l_m);
}

struct PackArgs {
    FastDiv div_slot, div_pitch;
    int per_chan;          // workgroups per (channel, phase) plane
    int lead_imgs;         // whole images that cover the leading zeros
    int part_n;            // > 0: the scale is the maximum of that many partials behind the scale pointer (ignored with CLIP)
    float* publish;        // where the first workgroup leaves that scale (two floats: as reported, as found), or null
    float* publish_raw;
    uint32_t tensor;       // random stream id
    uint64_t seed;
};

template <typename T, bool STOCH, bool CLIP>
__device__ __forceinline__ void pack_cnhw_role(const int b, const int phase, const T* __restrict__ src, const CnhwView& L,
                                               const float* __restrict__ scale, int8_t* __restrict__ dst, const PackArgs& pa,
                                               const QuantWs& ws, const ClipArgs& ca) {
    __shared__ uint32_t l_cnt[kBlock / kWave];
    const int xcd = b % kXcd, q = b / kXcd;
    const int c = (q / pa.per_chan) * kXcd + xcd;  // channel c runs on XCD c % 8
    const int jb = q % pa.per_chan;                // block of 1024 dwords along the flattened axis
    if (c >= L.C) return;
    const int tid = threadIdx.x;
    const int ph = phase / L.phases_w, pw = phase % L.phases_w;
    const int plane_dw = (int)(L.plane_pitch >> 2);
    const uint32_t slot = (uint32_t)(L.img_rows * L.row_pitch);
    const uint32_t HW = (uint32_t)(L.H * L.W);
    constexpr uint32_t EB = sizeof(T);   // bytes of a source element
    const __amdgpu_buffer_rsrc_t rs = f32_rsrc(src, (uint32_t)L.N * (uint32_t)L.C * HW * EB);

    // All index products below have factors under 2^24 and results under 2^31 (checked by the host), so the
    // full-rate 24-bit multiplier serves.  A destination row (n, r) reads source row h = r*phases_h + ph - org_h
    // of image n; stepping to the next destination row moves the source offset by one of two launch constants.
    const uint32_t W4 = (uint32_t)L.W * EB;
    const uint32_t step_row = (uint32_t)L.phases_h * W4;                                  // next row, same image
    const uint32_t step_img = (uint32_t)L.C * HW * EB - (uint32_t)(L.img_rows - 1) * step_row;  // row 0 of the next image
    const int h_first = ph - L.org_h, w_first = pw - L.org_w;

    float x[4][4];
    uint32_t eoff[4][4];   // byte offset of the element in the source (its index times the element size), or >= kOobOff
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int d = jb * 1024 + tid + 256 * u;   // dword inside the plane
        // first byte of the dword as (image, row, column); shifted by whole images so that the bytes in
        // front of the first image (the leading zeros) decompose to negative image numbers
        const uint32_t o = (uint32_t)(4 * d - (int)L.lead) + (uint32_t)pa.lead_imgs * slot;
        const uint32_t nq = fdiv(o, pa.div_slot);
        const uint32_t rem = o - __umul24(nq, slot);
        const uint32_t r = fdiv(rem, pa.div_pitch);
        const int col = (int)(rem - __umul24(r, (uint32_t)L.row_pitch));
        const int n = (int)nq - pa.lead_imgs;
        int h = (int)__umul24(r, (uint32_t)L.phases_h) + h_first;
        // n and h may be negative here (leading padding): signed multiplies keep the offset linear modulo 2^32,
        // so the row steps below land on the right value once the walk reaches a real row
        uint32_t raw = (uint32_t)(__mul24(__mul24(n, L.C) + c, (int)HW) + __mul24(h, L.W)) * EB;
        int w = (int)__umul24((uint32_t)col, (uint32_t)L.phases_w) + w_first;
        int nn = n, rr = (int)r, cc = col;
        const bool live = d < plane_dw;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const bool ok = live & ((unsigned)nn < (unsigned)L.N) & ((unsigned)h < (unsigned)L.H) & ((unsigned)w < (unsigned)L.W);
            eoff[u][i] = ok ? raw + EB * (uint32_t)w : kOobOff;
            x[u][i] = buf_ld<T>(rs, eoff[u][i], 0u);
            // step to the next byte of the plane: next column, possibly next row, possibly next image
            const bool wrap = cc + 1 == L.row_pitch;
            const bool last = wrap & (rr + 1 == L.img_rows);
            cc = wrap ? 0 : cc + 1;
            w = wrap ? w_first : w + L.phases_w;
            raw += wrap ? (last ? step_img : step_row) : 0u;
            h = wrap ? (last ? h_first : h + L.phases_h) : h;
            rr = wrap ? (last ? 0 : rr + 1) : rr;
            nn += last ? 1 : 0;
        }
    }

    float s;
    if (CLIP) s = clip_value(ws, ca, c, (double)L.N * (double)L.H * (double)L.W, jb == 0 && phase == 0, l_cnt);
    else s = given_scale(scale, pa.part_n, pa.publish, pa.publish_raw, c == 0 && jb == 0 && phase == 0, reinterpret_cast<float*>(l_cnt));
    const float inv = inv_scale(s);

    // Padding positions were read as 0.0f and quantize to code 0 in either rounding mode
    // (stochastic: floor(0) + (0 > u) = 0), so no select is needed here.
    int8_t* plane = dst + (int64_t)c * L.chan_pitch + (int64_t)phase * L.plane_pitch;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int d = jb * 1024 + tid + 256 * u;
        uint32_t bits[4];
#pragma unroll
        for (int i = 0; i < 4; ++i)
            bits[i] = quant_bits<STOCH>(x[u][i], inv, STOCH ? draw_half(draw_word(pa.seed, eoff[u][i] / EB), pa.tensor) : 0u);
        if (d < plane_dw) *reinterpret_cast<uint32_t*>(plane + 4 * (int64_t)d) = pack4<kCodeByte<STOCH>>(bits[0], bits[1], bits[2], bits[3]);
    }
}

template <typename T, bool STOCH, bool CLIP>
__global__ __launch_bounds__(kBlock) void k_pack_cnhw(const T* __restrict__ src, CnhwView L, const float* __restrict__ scale,
                                                      int8_t* __restrict__ dst, PackArgs pa, QuantWs ws, ClipArgs ca) {
    pack_cnhw_role<T, STOCH, CLIP>((int)blockIdx.x, (int)blockIdx.z, src, L, scale, dst, pa, ws, ca);
}

// ---------------------------------------------------------------------------------------------
// S5, channel-major copy, fast path for unsplit layouts (one stride phase) whose row length is a
// multiple of V = 4 or 2.  Source driven: a thread loads V consecutive floats of one row with one
// aligned vector load (neighbouring lanes are contiguous: 1 KiB per wave instruction for V = 4),
// quantizes them and stores V consecutive bytes; no element needs a validity test and the index
// arithmetic is shared by V elements.  The zero bytes between the rows are written by the thread
// that owns the end of the row; the padding rows between images, the bytes in front of the first
// row and behind the last one by one extra workgroup per channel.  Every byte of the buffer is
// still written exactly once per call.
// ---------------------------------------------------------------------------------------------
struct RowsArgs {
    FastDiv div_hwv, div_wv, div_prb;
    int per_chan;          // blocks of 1024 element groups per channel
    int grid_per_chan;     // data workgroups per channel (one more zeroes the padding); fewer than per_chan (early): they loop
    int part_n;            // this and the next two as in PackArgs
    float* publish;
    float* publish_raw;
    int early;             // the counting pass has written the real elements of channels whose class it guessed
    uint32_t tensor;
    uint64_t seed;
    // optional second copy of the same tensor in the same layout, quantized with its own per-tensor scale
    // (the globally quantized gradient of a depthwise layer): one read of the source serves both
    int8_t* dst2;
    const float* scale2;
    uint32_t tensor2;
};

template <int V>
__device__ __forceinline__ void store_codes(int8_t* p, uint32_t w) {
    // the destination has no alignment beyond one byte; the compiler picks the widest legal store
    if (V == 4) {
        __builtin_memcpy(p, &w, 4);
    } else if (V == 1) {
        *p = (int8_t)w;
    } else {
        const uint16_t h = (uint16_t)w;
        __builtin_memcpy(p, &h, 2);
    }
}

template <typename T, bool STOCH, bool CLIP, int V>
__device__ __forceinline__ void pack_rows_role(const int b, const T* __restrict__ src, const CnhwView& L, const float* __restrict__ scale,
                                               int8_t* __restrict__ dst, const RowsArgs& pa, const QuantWs& ws, const ClipArgs& ca) {
    __shared__ uint32_t l_cnt[kBlock / kWave];
    const int xcd = b % kXcd, q = b / kXcd;
    const int c = (q / (pa.grid_per_chan + 1)) * kXcd + xcd;  // channel c runs on XCD c % 8
    const int jb0 = q % (pa.grid_per_chan + 1);
    if (c >= L.C) return;
    const int tid = threadIdx.x;
    int8_t* plane = dst + (int64_t)c * L.chan_pitch;
    int8_t* plane2 = pa.dst2 ? pa.dst2 + (int64_t)c * L.chan_pitch : nullptr;   // uniform
    const uint32_t slot = (uint32_t)(L.img_rows * L.row_pitch);

    if (jb0 == pa.grid_per_chan) {
        // padding rows behind every image, then the bytes in front of the first row and behind the last image
        const uint32_t prb = (uint32_t)(L.img_rows - L.H) * (uint32_t)L.row_pitch;
        const uint32_t total = (uint32_t)L.N * prb;
        for (int copy = 0; copy < (plane2 ? 2 : 1); ++copy) {
            int8_t* pl = copy ? plane2 : plane;
            for (uint32_t t = tid; t < total; t += kBlock) {
                const uint32_t n = fdiv(t, pa.div_prb);
                pl[(uint32_t)L.lead + n * slot + (uint32_t)L.H * (uint32_t)L.row_pitch + (t - n * prb)] = 0;
            }
            for (uint32_t t = tid; t < (uint32_t)L.lead; t += kBlock) pl[t] = 0;
            for (uint32_t t = (uint32_t)L.lead + (uint32_t)L.N * slot + tid; t < (uint32_t)L.plane_pitch; t += kBlock) pl[t] = 0;
        }
        return;
    }

    // The counting pass guessed this channel's class: its bytes are in place if the guess was right (same clip rule
    // on the same inputs, hence the same scale and the same codes), and then nothing of dY is read here.
    float s = 0.0f;
    if (pa.early) {
        // the data workgroups of a correctly guessed channel return below: the zero bytes between the rows, which they
        // would have written along with the codes, are shared out among them first
        const uint32_t pw = (uint32_t)(L.row_pitch - L.W), rows = (uint32_t)L.N * (uint32_t)L.H;
        for (uint32_t t = (uint32_t)jb0 * kBlock + tid; t < rows * pw; t += (uint32_t)pa.grid_per_chan * kBlock) {
            const uint32_t r = t / pw, n = r / (uint32_t)L.H;
            const uint32_t at = (uint32_t)L.lead + (n * (uint32_t)L.img_rows + (r - n * (uint32_t)L.H)) * (uint32_t)L.row_pitch + (uint32_t)L.W + (t - r * pw);
            plane[at] = 0;
            if (plane2) plane2[at] = 0;
        }
        if constexpr (!CLIP) {
            return;   // a copy under a given scale (forward pass) is complete once its padding is written
        } else {
            int klass;
            s = clip_value(ws, ca, c, (double)L.N * (double)L.H * (double)L.W, jb0 == 0, l_cnt, &klass);
            if ((uint32_t)klass == ws.pred[c]) return;   // uniform
        }
    }
    if (CLIP && !pa.early) s = clip_value(ws, ca, c, (double)L.N * (double)L.H * (double)L.W, jb0 == 0, l_cnt);
    float inv = CLIP ? inv_scale(s) : 0.0f;

    const uint32_t HW = (uint32_t)(L.H * L.W), HWV = HW / V, WV = (uint32_t)L.W / V;
    const uint32_t groups = (uint32_t)L.N * HWV;
    const int padw = L.row_pitch - L.W;
    constexpr uint32_t EB = sizeof(T);   // bytes of a source element
    const __amdgpu_buffer_rsrc_t rs = f32_rsrc(src, (uint32_t)L.N * (uint32_t)L.C * HW * EB);

  // one pass unless the grid was cut down (early mode: the few channels left to do are walked by a few workgroups)
  for (int jb = jb0; jb < pa.per_chan; jb += pa.grid_per_chan) {
    float x[4][V];
    uint32_t eoff[4], doff[4];
    bool live[4], row_end[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const uint32_t gi = (uint32_t)jb * 1024u + tid + 256u * u;   // group of V elements inside the channel
        live[u] = gi < groups;
        const uint32_t gc = live[u] ? gi : 0u;
        const uint32_t n = fdiv(gc, pa.div_hwv);
        const uint32_t rem = gc - __umul24(n, HWV);
        const uint32_t h = fdiv(rem, pa.div_wv);
        const uint32_t wv = rem - __umul24(h, WV);
        row_end[u] = live[u] & (wv + 1 == WV);
        eoff[u] = live[u] ? __umul24(__umul24(n, (uint32_t)L.C) + (uint32_t)c, HW) * EB + rem * (EB * V) : kOobOff;
        doff[u] = (uint32_t)L.lead + __umul24(__umul24(n, (uint32_t)L.img_rows) + h, (uint32_t)L.row_pitch) + wv * V;
        if constexpr (EB == 4 && V == 4) {
            const v4u raw = __builtin_amdgcn_raw_buffer_load_b128(rs, (int)eoff[u], 0, 0);
#pragma unroll
            for (int i = 0; i < V; ++i) x[u][i] = __uint_as_float(raw[i]);
        } else if constexpr (V == 1) {
            x[u][0] = buf_ld<T>(rs, eoff[u], 0u);
        } else if constexpr (EB == 4) {
            const v2u raw = __builtin_amdgcn_raw_buffer_load_b64(rs, (int)eoff[u], 0, 0);
#pragma unroll
            for (int i = 0; i < V; ++i) x[u][i] = __uint_as_float(raw[i]);
        } else if constexpr (V == 4) {   // four bfloat16 in two dwords
            const v2u raw = __builtin_amdgcn_raw_buffer_load_b64(rs, (int)eoff[u], 0, 0);
            x[u][0] = __uint_as_float(raw[0] << 16);
            x[u][1] = __uint_as_float(raw[0] & 0xffff0000u);
            x[u][2] = __uint_as_float(raw[1] << 16);
            x[u][3] = __uint_as_float(raw[1] & 0xffff0000u);
        } else {                          // two bfloat16 in one dword
            const uint32_t raw = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(rs, (int)eoff[u], 0, 0);
            x[u][0] = __uint_as_float(raw << 16);
            x[u][1] = __uint_as_float(raw & 0xffff0000u);
        }
    }

    uint32_t draw[4][V];   // of the elements: the two copies draw from the two halves
    if constexpr (STOCH) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if constexpr (V == 4) draw_words4(pa.seed, eoff[u] / EB, draw[u]);   // rows and planes are whole groups
#pragma unroll
            for (int i = 0; i < V; ++i) {
                if constexpr (V != 4) draw[u][i] = draw_word(pa.seed, eoff[u] / EB + i);
                asm volatile("" : "+v"(draw[u][i]));   // computed once, not once a copy
            }
        }
    }
    // a given scale is folded while the loads are in flight (without `early` there is one pass)
    if constexpr (!CLIP)
        inv = inv_scale(given_scale(scale, pa.part_n, pa.publish, pa.publish_raw, c == 0 && jb == 0, reinterpret_cast<float*>(l_cnt)));
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        uint32_t bits[4] = {0u, 0u, 0u, 0u};
#pragma unroll
        for (int i = 0; i < V; ++i) bits[i] = quant_bits<STOCH>(x[u][i], inv, STOCH ? draw_half(draw[u][i], pa.tensor) : 0u);
        if (live[u]) store_codes<V>(plane + doff[u], pack4<kCodeByte<STOCH>>(bits[0], bits[1], bits[2], bits[3]));
        if (row_end[u])
            for (int k = 0; k < padw; ++k) plane[doff[u] + V + k] = 0;
    }
    if (plane2) {
        const float inv2 = inv_scale(pa.scale2[0]);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            uint32_t bits[4] = {0u, 0u, 0u, 0u};
#pragma unroll
            for (int i = 0; i < V; ++i) bits[i] = quant_bits<STOCH>(x[u][i], inv2, STOCH ? draw_half(draw[u][i], pa.tensor2) : 0u);
            if (live[u]) store_codes<V>(plane2 + doff[u], pack4<kCodeByte<STOCH>>(bits[0], bits[1], bits[2], bits[3]));
            if (row_end[u])
                for (int k = 0; k < padw; ++k) plane2[doff[u] + V + k] = 0;
        }
    }
  }
}

template <typename T, bool STOCH, bool CLIP, int V>
__global__ __launch_bounds__(kBlock) void k_pack_rows(const T* __restrict__ src, CnhwView L, const float* __restrict__ scale,
                                                      int8_t* __restrict__ dst, RowsArgs pa, QuantWs ws, ClipArgs ca) {
    pack_rows_role<T, STOCH, CLIP, V>((int)blockIdx.x, src, L, scale, dst, pa, ws, ca);
}

// ---------------------------------------------------------------------------------------------
// Channel-resident schedule: S1 - S5 for the per-channel copy with ONE read of dY.
//
// From the middle of a network on, a channel of the gradient is small (ResNet-50 at batch 64: 50176 elements at
// 28 x 28, 12544 at 14 x 14, 3136 at 7 x 7): the REGISTERS of one workgroup hold it.  One workgroup per channel
// loads its channel once and keeps it: statistics, tail mass, the discriminator's decision, the clip value and the
// per-channel quantization all run on registers.  The codes are assembled in an LDS image of the channel's plane
// (zero-filled first: the padding) and leave as whole 16-byte stores, so that every byte of the plane is written once.
// Only the globally quantized copy, whose scale is the maximum over ALL channels, needs a second launch (the counting
// kernel in its copy-only form), which finds a small tensor in the caches.
// ---------------------------------------------------------------------------------------------
constexpr int64_t kResidentMaxLds = 96 * 1024;   // bytes of a channel's int8 plane (the LDS image)

struct ResArgs {
    FastDiv div_u, div_w;  // div_u: load units of a plane
    int N, C, HW;
    float k, A, lambda;
    uint64_t seed;         // the keys of stochastic rounding (round_keys)
    // the form that writes the NHWC global copy too
    int8_t* qg;
    float* s_global;
    int c_pitch, qg_tail;
};

// A load unit is four consecutive elements of one plane (VEC4, planes of at least four elements) or one element; a thread
// holds NU units, a workgroup has TH threads.  TAIL: the plane is not a multiple of four long, and its last unit is moved
// back to end with it: the elements it shares with the unit before are zeroed for the statistics and not written again.
// Every load is then 16 (bfloat16: 8) consecutive bytes at the alignment of an element, and a plane of 49 takes 13 of them
// instead of 49.  (512 -> 2048 1 x 1 at 7 x 7, batch 128, bfloat16: 27 us with a load an element, 22.5 here.)
// FLAT (without TAIL): the plane has no padding between rows or images (1 x 1 layers), so element m of the channel sits at
// byte lead + m and a unit's four codes are one aligned dword of the plane: they go straight to memory, no LDS image.
// ALL: the global copy as well, in the same launch.  Its scale is the maximum over all channels, so every workgroup reads the whole tensor
// for it, 16 bytes a thread and eight loads at a time, and its codes leave as single bytes of the NHWC records: a few microseconds
// where tensors are small, less than the launch they replace (resident_all_pays).
template <typename T, bool STOCH, bool VEC4, int NU, bool FLAT, bool TAIL, bool ALL>
__global__ __launch_bounds__(1024, NU <= 2 ? 8 : NU <= 8 ? 6 : 4) void k_chan_resident(const T* __restrict__ g, CnhwView L, int8_t* __restrict__ vq,
                                                      ResArgs ra, QuantWs ws, ClipArgs ca) {
    extern __shared__ __align__(16) int8_t l_img[];   // the channel's plane as it will sit in memory
    constexpr int kMaxWaves = 1024 / kWave;
    __shared__ float l_mx[kMaxWaves];
    __shared__ double l_s1[kMaxWaves], l_s2[kMaxWaves];
    __shared__ uint32_t l_cnt[kMaxWaves];
    __shared__ float l_all[ALL ? kMaxWaves : 1];
    const int TH = (int)blockDim.x;
    __shared__ float l_bc[5];   // |g|max, mean, sigma, clip value, the tensor's |g|max
    // workgroup b runs on XCD b % 8: an XCD takes a contiguous eighth of the channels, whose planes are neighbours in
    // every image and share cache lines where a plane is not a whole number of them
    const int per_xcd = (ra.C + kXcd - 1) / kXcd;
    const int c = ((int)blockIdx.x % kXcd) * per_xcd + (int)blockIdx.x / kXcd;
    if ((int)blockIdx.x / kXcd >= per_xcd || c >= ra.C) return;   // uniform: padding of the grid
    const int tid = threadIdx.x, wave = tid / kWave, lane = tid % kWave;
    const int HW = ra.HW, M = ra.N * HW;
    constexpr uint32_t EB = sizeof(T);
    constexpr int PER = VEC4 ? 4 : 1;
    const __amdgpu_buffer_rsrc_t rs = f32_rsrc(g, (uint32_t)M * (uint32_t)ra.C * EB);
    const uint32_t upp = (uint32_t)(HW + PER - 1) / PER, units = (uint32_t)ra.N * upp;   // load units of a plane, of the channel
    // unit q -> image, first element in its plane (TAIL: after the move back), leading elements that belong to the unit before
    auto place = [&](uint32_t q, uint32_t& n, uint32_t& i, uint32_t& dup) {
        n = fdiv(q, ra.div_u);
        const uint32_t at = (q - n * upp) * PER;
        i = TAIL ? min(at, (uint32_t)HW - 4u) : at;
        dup = at - i;
    };
    // a thread's number again, where kept places would spill a new one for the compiler: they are worked out afresh in every phase
    auto again = [&]() {
        uint32_t t = (uint32_t)tid;
        if constexpr (TAIL || (FLAT && NU == 16)) asm volatile("" : "+v"(t));
        return t;
    };
    // NCHW index of a unit's first element; planes of whole units need no place for it (two instructions in 30 an element fewer)
    const uint32_t image = (uint32_t)ra.C * (uint32_t)HW, first = (uint32_t)c * (uint32_t)HW, skip = image - upp * PER;
    auto index = [&](uint32_t q) {
        if constexpr (!TAIL) return q * PER + fdiv(q, ra.div_u) * skip + first;
        uint32_t n, i, dup;
        place(q, n, i, dup);
        return n * image + first + i;
    };

    const float s_prev = ca.s_state[c];   // needed by one thread, late: requested with the channel, its latency does not show
    // ---- S1: the channel comes in, all loads of the thread in flight at once ----
    float x[NU][PER];
#pragma unroll
    for (int u = 0; u < NU; ++u) {
        const uint32_t q = (uint32_t)(u * TH + tid);
        const bool ok = q < units;
        const uint32_t at = index(ok ? q : 0u);
        if constexpr (VEC4 && EB == 4) {
            const v4u raw = __builtin_amdgcn_raw_buffer_load_b128(rs, (int)(ok ? at * EB : kOobOff), 0, 0);
#pragma unroll
            for (int e = 0; e < 4; ++e) x[u][e] = __uint_as_float(raw[e]);
        } else if constexpr (VEC4) {
            const uint4 raw = ld4_or_zero<T>(g + at, ok);
            x[u][0] = __uint_as_float(raw.x);
            x[u][1] = __uint_as_float(raw.y);
            x[u][2] = __uint_as_float(raw.z);
            x[u][3] = __uint_as_float(raw.w);
        } else {
            x[u][0] = buf_ld<T>(rs, ok ? at * EB : kOobOff, 0u);
        }
    }
    if constexpr (STOCH) __builtin_amdgcn_sched_barrier(0);   // every load of the channel is requested before the hashes below start
    // Stochastic rounding: an element's draw depends on its index alone, so the hashes are computed here, while the
    // loads are on their way and the vector ALU has nothing else to do, and kept as 16-bit halves (element k of the
    // thread in half k % 2 of word k / 2).
    uint32_t draw[STOCH ? (NU * PER + 1) / 2 : 1];
    if constexpr (STOCH) {
        const uint32_t tid2 = again();
        uint32_t h[PER == 4 ? 4 : 2] = {};   // (units past the channel hash a number nobody uses)
#pragma unroll
        for (int k = 0; k < NU * PER; ++k) {
            const int u = k / PER, e = k % PER;
            if constexpr (PER == 4 && !TAIL) {
                if (e == 0) draw_words4(ra.seed, index((uint32_t)(u * TH) + tid2), h);
            } else {
                h[k % (PER == 4 ? 4 : 2)] = draw_word(ra.seed, index((uint32_t)(u * TH) + tid2) + (uint32_t)e);
            }
            // the per-channel copy draws from the upper half of the word
            if (k % 2 == 1) draw[k / 2] = (h[k % (PER == 4 ? 4 : 2) - 1] >> 16) | (h[k % (PER == 4 ? 4 : 2)] & 0xffff0000u);
            else if (k + 1 == NU * PER) draw[k / 2] = h[0] >> 16;
        }
        // (without this the compiler moves the hashes down to where they are used, behind the barriers; as many of
        // them as the registers of the form allow)
        constexpr int W = (NU * PER + 1) / 2;
        constexpr int PIN = NU <= 8 ? (FLAT || !VEC4 ? W : W / 2) : FLAT ? 3 * W / 4 : W / 2;
#pragma unroll
        for (int k = 0; k < PIN; ++k) asm volatile("" : "+v"(draw[k]));
        __builtin_amdgcn_sched_barrier(0);
    }
    auto draw_of = [&](int u, int e) -> uint32_t {
        if constexpr (!STOCH) return 0u;
        const int k = u * PER + e;
        return (k & 1) ? draw[k / 2] >> 16 : draw[k / 2] & 0xffffu;
    };
    uint32_t dups = 0;   // TAIL: leading elements of unit u that belong to the unit before, two bits each
    if constexpr (TAIL) {
        const uint32_t tid2 = again();
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            uint32_t n, i, dup;
            place((uint32_t)(u * TH) + tid2, n, i, dup);
            dups |= dup << (2 * u);
        }
    }
    // element e of unit u as the statistics see it
    auto own = [&](int u, int e) -> float {
        if (!TAIL || e == 3) return x[u][e];
        return (dups >> (2 * u) & 3u) > (uint32_t)e ? 0.0f : x[u][e];
    };
    float all = 0.0f;   // |g|max of the tensor
    if constexpr (ALL) {
        const uint32_t total = (uint32_t)M * (uint32_t)ra.C, quads = (total + 3u) / 4u;
        if (total >= 4u) {   // uniform
            for (uint32_t q0 = (uint32_t)tid; q0 < quads; q0 += 8u * (uint32_t)TH) {
                uint4 v[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) {   // (what lies past the end is the last one again; the last one ends with the tensor)
                    const uint32_t at = min(4u * min(q0 + (uint32_t)(u * TH), quads - 1u), total - 4u);
                    v[u] = ld4_or_zero<T>(g + at, true);
                }
#pragma unroll
                for (int u = 0; u < 8; ++u)
                    all = fmaxf(fmaxf(all, fmaxf(fabsf(__uint_as_float(v[u].x)), fabsf(__uint_as_float(v[u].y)))),
                                fmaxf(fabsf(__uint_as_float(v[u].z)), fabsf(__uint_as_float(v[u].w))));
            }
        } else if ((uint32_t)tid < total) {
            all = fabsf(ld1_or_zero<T>(g + tid, true));
        }
        all = wave_max(all);
    }
    float mx = 0.0f;
    double s1 = 0.0, s2 = 0.0;
#pragma unroll
    for (int u = 0; u < NU; ++u)
#pragma unroll
        for (int e = 0; e < PER; ++e) {   // units past the channel were read as zeros and change nothing
            const float v = own(u, e);
            mx = fmaxf(mx, fabsf(v));
            const double a = v;
            s1 += a;
            s2 = __builtin_fma(a, a, s2);   // the square of a widened fp32 is exact in fp64: the same sum as s2 + a * a, one instruction
        }
    mx = wave_max(mx);
    s1 = wave_sum(s1);
    s2 = wave_sum(s2);
    if (lane == 0) { l_mx[wave] = mx; l_s1[wave] = s1; l_s2[wave] = s2; }
    if (ALL && lane == 0) l_all[wave] = all;
    // the padding of the plane image, while the partials settle
    if constexpr (!FLAT)
        for (int i = tid; i < (int)(L.plane_pitch >> 4); i += TH) reinterpret_cast<uint4*>(l_img)[i] = make_uint4(0u, 0u, 0u, 0u);
    __syncthreads();
    if (tid == 0) {
        for (int w = 1; w < TH / kWave; ++w) { mx = fmaxf(mx, l_mx[w]); s1 += l_s1[w]; s2 += l_s2[w]; }
        const double Md = (double)ra.N * (double)HW;
        const double mu = s1 / Md;
        double var = s2 / Md - mu * mu;
        if (var < 0.0) var = 0.0;
        l_bc[0] = mx;
        l_bc[1] = (float)mu;
        l_bc[2] = (float)sqrt(var);
        if constexpr (ALL) {
            for (int w = 1; w < TH / kWave; ++w) all = fmaxf(all, l_all[w]);
            l_bc[4] = all >= kTinyScale ? all : 0.0f;
            if (c == 0) *ra.s_global = l_bc[4];
        }
    }
    __syncthreads();
    const float gm = l_bc[0], sigma = l_bc[2];

    // ---- S2: tail mass (a zero never exceeds sigma, so the units past the channel need no mask) ----
    uint32_t cnt = 0;   // of the whole wave: a scalar counter
#pragma unroll
    for (int u = 0; u < NU; ++u)
#pragma unroll
        for (int e = 0; e < PER; ++e) cnt += (uint32_t)__popcll(__ballot(fabsf(own(u, e)) > sigma));
    if (lane == 0) l_cnt[wave] = cnt;
    __syncthreads();
    if (tid == 0) {
        // S3 + S4: discriminator (Eq. "judge") and clip value (Eq. "gaus" / Eq. "fats"), then what the channel publishes
        for (int w = 1; w < TH / kWave; ++w) cnt += l_cnt[w];
        const double Md = (double)ra.N * (double)HW;
        const int klass = ((double)cnt > (double)ra.lambda * Md) ? DAQ_CLASS_GAUSS : DAQ_CLASS_INVT;
        const float sc = clip_rule(klass, gm, s_prev, ra.k, ra.A);
        l_bc[3] = sc;
        ca.s_state[c] = sc;
        ca.s_chan[c] = (sc >= kTinyScale) ? sc : 0.0f;
        ca.cls[c] = (uint8_t)klass;
        if (ca.stats) {
            ca.stats[4 * c + 0] = gm;
            ca.stats[4 * c + 1] = l_bc[1];
            ca.stats[4 * c + 2] = sigma;
            ca.stats[4 * c + 3] = (float)((double)cnt / Md);
        }
        if constexpr (!ALL) ws.part_max[c] = gm;   // one partial per channel: the copy-only launch folds them into the global scale
    }
    if constexpr (ALL) {
        // ---- S5, the global copy: the channel's byte of every record (the upper halves of the words above are the per-channel copy's) ----
        const float inv_g = inv_scale(l_bc[4]);
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            const uint32_t q = (uint32_t)(u * TH + tid);
            if (q < units) {
                uint32_t n, i, dup, w[4] = {0u, 0u, 0u, 0u};
                place(q, n, i, dup);
                const uint32_t at = n * image + first + i;
                if constexpr (STOCH && PER == 4 && !TAIL) draw_words4(ra.seed, at, w);
                int8_t* rec = ra.qg + (int64_t)(n * (uint32_t)HW + i) * ra.c_pitch + c;
#pragma unroll
                for (int e = 0; e < PER; ++e) {   // (what a unit shares with the one before it, both write the same)
                    if constexpr (STOCH && (PER != 4 || TAIL)) w[e] = draw_word(ra.seed, at + (uint32_t)e);
                    rec[(int64_t)e * ra.c_pitch] = code_byte<STOCH>(quant_bits<STOCH>(x[u][e], inv_g, draw_half(w[e], 1u)));
                }
            }
        }
        if (c == ra.C - 1) {   // the bytes of channels past the last one, and those behind the last record
            const uint32_t pad = (uint32_t)(ra.c_pitch - ra.C), bytes = (uint32_t)M * pad;
            for (uint32_t t = (uint32_t)tid; t < bytes; t += (uint32_t)TH) {
                const uint32_t P = t / pad;
                ra.qg[(int64_t)P * ra.c_pitch + ra.C + (t - P * pad)] = 0;
            }
            for (int t = tid; t < ra.qg_tail; t += TH) ra.qg[(int64_t)M * ra.c_pitch + t] = 0;
        }
    }
    __syncthreads();
    const float inv = inv_scale(l_bc[3]);

    if constexpr (FLAT) {
        // ---- S5, plane without padding: a unit's four codes are four consecutive bytes of the plane's payload ----
        // (TAIL: at any byte; what a unit shares with the one before it, both write the same)
        int8_t* plane = vq + (int64_t)c * L.chan_pitch;
        const uint32_t tid2 = again(), payload = (uint32_t)M;
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            const uint32_t q = (uint32_t)(u * TH) + tid2;
            if (q < units) {
                uint32_t b[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) b[e] = quant_bits<STOCH>(x[u][e], inv, draw_of(u, e));
                const uint32_t w = pack4<kCodeByte<STOCH>>(b[0], b[1], b[2], b[3]);
                if constexpr (TAIL) {
                    uint32_t n, i, dup;
                    place(q, n, i, dup);
                    __builtin_memcpy(plane + (uint32_t)L.lead + n * (uint32_t)HW + i, &w, 4);
                } else {
                    reinterpret_cast<uint32_t*>(plane + L.lead)[q] = w;
                }
            }
        }
        // the zeros in front of and behind the payload (the plane and its lead are whole dwords, the payload need not be)
        const uint32_t head = (uint32_t)L.lead, tail = head + payload, total = (uint32_t)L.plane_pitch;
        for (uint32_t t = 4u * tid; t < head; t += 4u * TH) *reinterpret_cast<uint32_t*>(plane + t) = 0u;
        const uint32_t tail4 = (tail + 3u) & ~3u;
        if (TAIL && tid < (int)(tail4 - tail)) plane[tail + tid] = 0;
        for (uint32_t t = tail4 + 4u * tid; t < total; t += 4u * TH) *reinterpret_cast<uint32_t*>(plane + t) = 0u;
        return;
    }
    // ---- S5: the per-channel codes go to their places in the plane image ----
    const uint32_t slot = (uint32_t)(L.img_rows * L.row_pitch), tid2 = again();
#pragma unroll
    for (int u = 0; u < NU; ++u) {
        const uint32_t q = (uint32_t)(u * TH) + tid2;
        if (q < units) {
            uint32_t n, px, dup;
            place(q, n, px, dup);
            uint32_t r = fdiv(px, ra.div_w);
            uint32_t col = px - r * (uint32_t)L.W;
            uint32_t pos = (uint32_t)L.lead + n * slot + r * (uint32_t)L.row_pitch + col;
#pragma unroll
            for (int e = 0; e < PER; ++e) {
                if (!TAIL || e == 3 || (uint32_t)e >= dup) l_img[pos] = code_byte<STOCH>(quant_bits<STOCH>(x[u][e], inv, draw_of(u, e)));
                const bool wrap = ++col == (uint32_t)L.W;   // a unit stays inside its image, but may run on into the next row
                col = wrap ? 0u : col;
                pos += wrap ? (uint32_t)(L.row_pitch - L.W) + 1u : 1u;
            }
        }
    }
    __syncthreads();
    uint4* plane = reinterpret_cast<uint4*>(vq + (int64_t)c * L.chan_pitch);   // chan_pitch is a multiple of 256
    for (int i = tid; i < (int)(L.plane_pitch >> 4); i += TH) plane[i] = reinterpret_cast<const uint4*>(l_img)[i];
}

// ---------------------------------------------------------------------------------------------
// per-tensor helpers for the forward pass
// ---------------------------------------------------------------------------------------------
// max |x| of X and of W in one launch: the first bx workgroups sweep X, the next bw sweep W, each stores its maximum as one
// partial, and whoever needs the scale folds the partials (an atomic per workgroup on one address is served one after the
// other, about 10 ns each, and needs a cleared word first).  Eight 16-byte loads in flight per thread; a load past the end
// reads the last quad again, which changes no maximum.  (64 x 64 x 56 x 56: 19 us with atomics, 10 us here, 5.1 TB/s.)
constexpr int kAbsmaxBlocksX = 512, kAbsmaxBlocksW = 256;   // a plain read loop is fastest with 512 workgroups on this chip
struct AbsmaxArgs {
    const float* x[2];
    int64_t n[2];
    int blocks[2];
    float* part[2];
};
__global__ __launch_bounds__(kBlock) void k_absmax(AbsmaxArgs a) {
    __shared__ float l_m[kBlock / kWave];
    const bool second = (int)blockIdx.x >= a.blocks[0];
    const int b = (int)blockIdx.x - (second ? a.blocks[0] : 0);
    const float* __restrict__ x = second ? a.x[1] : a.x[0];
    const int64_t n = second ? a.n[1] : a.n[0];
    const int64_t stride = (int64_t)(second ? a.blocks[1] : a.blocks[0]) * kBlock;
    float m = 0.0f;
    const int64_t n4 = ((uintptr_t)x & 15u) ? 0 : n / 4;   // whole aligned quads; the rest goes element by element
    const float4* x4 = reinterpret_cast<const float4*>(x);
    for (int64_t i = (int64_t)b * kBlock + threadIdx.x; i < n4; i += 8 * stride) {
        float4 v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = x4[std::min(i + u * stride, n4 - 1)];
#pragma unroll
        for (int u = 0; u < 8; ++u) m = fmaxf(m, fmaxf(fmaxf(fabsf(v[u].x), fabsf(v[u].y)), fmaxf(fabsf(v[u].z), fabsf(v[u].w))));
    }
    for (int64_t j = 4 * n4 + (int64_t)b * kBlock + threadIdx.x; j < n; j += 8 * stride) {
        float v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = x[std::min(j + u * stride, n - 1)];
#pragma unroll
        for (int u = 0; u < 8; ++u) m = fmaxf(m, fabsf(v[u]));
    }
    m = wave_max(m);
    if (threadIdx.x % kWave == 0) l_m[threadIdx.x / kWave] = m;
    __syncthreads();
    if (threadIdx.x == 0) (second ? a.part[1] : a.part[0])[b] = fmaxf(fmaxf(l_m[0], l_m[1]), fmaxf(l_m[2], l_m[3]));
}

// q(W) in its arrangements (see daq_wpack_layout), every byte of the buffer written once, zeros included.
struct PackWArgs {
    const float* w;
    int8_t* out;
    float* s_w;
    const float* part;     // partial maxima of |W|
    int part_n;
    int Cout, Cin, groups, taps, cig, cog;
    int chunks, ci_tiles;  // groups == 1: tap chunks and 32-channel tiles of the grid
    int blocks;            // workgroups of this role; 0: no filter
    FastDiv div_run, div_tap, div_runl, div_tapl;   // (32 * taps of a chunk, taps of a chunk), the last chunk's own
    daq_wpack_layout L;
};
constexpr int kWTaps = 3;                   // taps a workgroup takes at once: twelve weights a thread
constexpr int kWPlane = 32 * 32 + 16;       // bytes of a tap's 32 x 32 codes in LDS; the 16 spread the taps over the banks

// One group: a workgroup takes 32 x 32 channels (the tile of the fragment order) x up to three taps, twelve weights a thread,
// all loads in flight at once (nine taps, whose weights are contiguous, made each thread's work a chain of 36: 3 x 3, 128 ->
// 128 at 28 x 28, batch 8, forward 26.7 us against 17.7); the codes go to LDS in both orders, [co][ci] and
// [ci][co], and leave as 16-byte units: whole KiB of the two fragment copies, 32-byte runs of the other two.  (Scattering
// each code to five places in byte stores behind a fill of the buffer: 3 x 3, 272 -> 912, fill 12.6 and packing 24.7 us.)
template <int NT>
__device__ __forceinline__ void pack_w_tile(const int b, const PackWArgs& a, float* l_red, int8_t* l_f, int8_t* l_b) {
    const int tid = threadIdx.x;
    const int tc = b % a.chunks, tile = b / a.chunks;
    const int ct = tile / a.ci_tiles, it = tile - ct * a.ci_tiles;
    const int co0 = 32 * ct, ci0 = 32 * it, t0 = tc * kWTaps;
    const bool last = tc + 1 == a.chunks;
    const int nt = NT == 1 ? 1 : min(kWTaps, a.taps - t0);
    const FastDiv div_run = last ? a.div_runl : a.div_run, div_tap = last ? a.div_tapl : a.div_tap;
    // element e of the tile: weight index (~0: none there) and place in LDS, tap << 10 | co << 5 | ci (~0: past the tile)
    auto place = [&](uint32_t e, uint32_t& at, uint32_t& pl) {
        const uint32_t co = fdiv(e, div_run), r = e - co * (uint32_t)(32 * nt), ci = fdiv(r, div_tap), t = r - ci * (uint32_t)nt;
        const bool ok = co < 32u && co0 + (int)co < a.Cout && ci0 + (int)ci < a.Cin;
        at = ok ? (uint32_t)((co0 + (int)co) * a.cig + ci0 + (int)ci) * (uint32_t)a.taps + (uint32_t)t0 + t : ~0u;
        pl = co < 32u ? t << 10 | co << 5 | ci : ~0u;
    };
    float x[4 * NT];
    uint32_t at, pl;
#pragma unroll
    for (int k = 0; k < 4 * NT; ++k) {
        place((uint32_t)tid + kBlock * k, at, pl);
        x[k] = ldf_or_zero(a.w + at, at != ~0u);
    }
    const float s = fold_scale(a.part, a.part_n, l_red);
    if (b == 0 && tid == 0) *a.s_w = s >= kTinyScale ? s : 0.0f;
    const float inv = inv_scale(s);
    uint32_t e0 = (uint32_t)tid;
    asm volatile("" : "+v"(e0));   // the places are worked out again: kept since the loads, they would spill
#pragma unroll
    for (int k = 0; k < 4 * NT; ++k) {
        place(e0 + kBlock * k, at, pl);
        const int8_t code = at != ~0u ? code_byte<false>(quant_bits<false>(x[k], inv, 0u)) : (int8_t)0;
        if (at != ~0u) a.out[a.L.off_plain + at] = code;
        if (pl != ~0u) {
            const uint32_t t = pl >> 10, co = pl >> 5 & 31u, ci = pl & 31u;
            l_f[t * kWPlane + co * 32 + ci] = code;
            l_b[t * kWPlane + ci * 32 + co] = code;
        }
    }
    __syncthreads();
    const int rbf = (a.Cout + 31) / 32, rbb = (a.Cin + 31) / 32;
    for (int u = tid; u < nt * 64; u += kBlock) {
        const int t = u >> 6, h = (u >> 5) & 1, row = u & 31;
        const int64_t tap = t0 + t;
        const uint4 f = *reinterpret_cast<const uint4*>(l_f + t * kWPlane + row * 32 + 16 * h);
        const uint4 g = *reinterpret_cast<const uint4*>(l_b + t * kWPlane + row * 32 + 16 * h);
        if (co0 + row < a.Cout && ci0 + 16 * h < a.L.cig_pitch)
            *reinterpret_cast<uint4*>(a.out + a.L.off_fwd + (tap * a.Cout + co0 + row) * a.L.cig_pitch + ci0 + 16 * h) = f;
        if (ci0 + row < a.Cin && co0 + 16 * h < a.L.cog_pitch)
            *reinterpret_cast<uint4*>(a.out + a.L.off_bwd + (tap * a.Cin + ci0 + row) * a.L.cog_pitch + co0 + 16 * h) = g;
        const int in_tile = h * 512 + row * 16;
        if (ct < rbf)
            *reinterpret_cast<uint4*>(a.out + a.L.off_fwd_frag + (((((int64_t)(ci0 >> 6) * a.taps + tap) * rbf + ct) * 2 + (it & 1)) << 10) + in_tile) = f;
        if (it < rbb)
            *reinterpret_cast<uint4*>(a.out + a.L.off_bwd_frag + (((((int64_t)(co0 >> 6) * a.taps + tap) * rbb + it) * 2 + (ct & 1)) << 10) + in_tile) = g;
    }
    if (b == 0) {   // the bytes between the copies
        const int64_t z0 = (int64_t)a.Cout * a.cig * a.taps, z1 = a.L.off_fwd + (int64_t)a.taps * a.Cout * a.L.cig_pitch,
                      z2 = a.L.off_bwd + (int64_t)a.taps * a.Cin * a.L.cog_pitch;
        if (z0 + tid < a.L.off_fwd) a.out[z0 + tid] = 0;
        if (z1 + tid < a.L.off_bwd) a.out[z1 + tid] = 0;
        if (z2 + tid < a.L.off_fwd_frag) a.out[z2 + tid] = 0;
    }
}

// Grouped layers: a thread writes 16 bytes of one of the three copies.  Their weights are few.
__device__ __forceinline__ void pack_w_units(const int b, const PackWArgs& a, float* l_red) {
    const int64_t o = 16 * ((int64_t)b * kBlock + threadIdx.x);
    const int64_t n = (int64_t)a.Cout * a.cig * a.taps;
    int64_t first = -1, step = 0;   // weight of the unit's first byte, distance to the next one's, how many bytes hold a weight
    int count = 0;
    if (o < a.L.off_fwd) {
        first = o;
        step = 1;
        count = (int)std::max<int64_t>(0, std::min<int64_t>(16, n - o));
    } else if (o < a.L.off_bwd) {
        const int64_t q = (o - a.L.off_fwd) / 16, upr = a.L.cig_pitch / 16, row = q / upr, k0 = 16 * (q - row * upr);
        const int64_t tap = row / a.Cout, co = row - tap * a.Cout;
        first = (co * a.cig + k0) * a.taps + tap;
        step = a.taps;
        count = tap < a.taps ? (int)std::min<int64_t>(16, a.cig - k0) : 0;
    } else if (o < a.L.bytes) {
        const int64_t q = (o - a.L.off_bwd) / 16, upr = a.L.cog_pitch / 16, row = q / upr, k0 = 16 * (q - row * upr);
        const int64_t tap = row / a.Cin, ci = row - tap * a.Cin, grp = ci / a.cig;
        first = ((grp * a.cog + k0) * a.cig + (ci - grp * a.cig)) * a.taps + tap;
        step = (int64_t)a.cig * a.taps;
        count = tap < a.taps ? (int)std::min<int64_t>(16, a.cog - k0) : 0;
    }
    float x[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) x[i] = ldf_or_zero(a.w + first + i * step, i < count);
    const float s = fold_scale(a.part, a.part_n, l_red);
    if (b == 0 && threadIdx.x == 0) *a.s_w = s >= kTinyScale ? s : 0.0f;
    const float inv = inv_scale(s);
    uint32_t c[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) c[i] = i < count ? quant_bits<false>(x[i], inv, 0u) : 0u;
    if (o < a.L.bytes)
        *reinterpret_cast<uint4*>(a.out + o) = make_uint4(pack4<0>(c[0], c[1], c[2], c[3]), pack4<0>(c[4], c[5], c[6], c[7]),
                                                          pack4<0>(c[8], c[9], c[10], c[11]), pack4<0>(c[12], c[13], c[14], c[15]));
}

// Everything the forward pass quantizes, in one launch behind k_absmax: q(W), the two copies of q(X).  The three are
// independent of each other, and most layers are small: the launches and the gaps between them cost more than the bytes
// (eleven launches a forward pass with a launch for each step; three with the product now.  3 x 3, 128 -> 128 at 28 x 28,
// batch 8, whole pass: 39.8 -> 26.7 us; 1 x 1, 64 -> 256 at 56 x 56, batch 64: 91 -> 66; 416 -> 320 3 x 3 at 21 x 21: 59 -> 36).
// Each role starts at a multiple of eight workgroups, so that its own mapping to the XCDs holds.
// EARLY: the NHWC role writes both copies from one read of X, the channel-major role only the zeros round about the rows.
// V: elements per thread of the source-driven channel-major role, 0: the output-driven one; 1 only with EARLY.  UNIT: see the NHWC role.
struct FwdQuantArgs {
    const float* x;
    int8_t *nhwc, *cnhw;
    float* s_x;
    int N, C, HW, c_pitch, tail;
    int w_blocks, x_blocks;   // of the first two roles, rounded up to a multiple of eight
    int phase_blocks;         // output-driven channel-major role: workgroups per stride phase
    FastDiv div_u;
    CnhwView Lc;
    PackArgs pa;
    RowsArgs ra;
    EarlyVq ev;
    QuantWs ws;
    PackWArgs w;
};
// WAVES: of a workgroup, four or (EARLY) eight, see forward_waves; the other roles are written for four.
template <bool EARLY, int V, int UNIT, int WAVES>
__global__ __launch_bounds__(WAVES * kWave, 4) void k_fwd_quant(FwdQuantArgs a) {
    constexpr int kTileDw = CountPlan::most_tile_dwords(WAVES);
    __shared__ float l_red[kBlock / kWave];
    __shared__ __align__(16) int8_t l_w[2 * kWTaps * kWPlane];
    __shared__ __align__(16) uint32_t l_records[2 * kTileDw];
    int b = (int)blockIdx.x;
    if (b < a.w_blocks) {   // uniform, as all branches on b
        if (b >= a.w.blocks) return;
        if (WAVES * kWave > kBlock && threadIdx.x >= kBlock) return;   // (a barrier waits for the waves that are still there)
        if (a.w.groups > 1) pack_w_units(b, a.w, l_red);
        else if (a.w.taps == 1) pack_w_tile<1>(b, a.w, l_red, l_w, l_w + kWTaps * kWPlane);
        else pack_w_tile<kWTaps>(b, a.w, l_red, l_w, l_w + kWTaps * kWPlane);
        return;
    }
    b -= a.w_blocks;
    if (b < a.x_blocks) {
        if (b >= a.ws.cp.workgroups()) return;
        count_qg_role<float, false, true, false, EARLY, UNIT>(b, a.x, a.N, a.C, a.HW, a.c_pitch, a.div_u, a.ws, a.nhwc, 0, nullptr, a.s_x, a.ev, a.tail, l_records, kTileDw);
        return;
    }
    if (WAVES * kWave > kBlock && threadIdx.x >= kBlock) return;
    b -= a.x_blocks;
    if constexpr (V > 0) pack_rows_role<float, false, false, V>(b, a.x, a.Lc, a.ws.part_max, a.cnhw, a.ra, a.ws, ClipArgs{});
    else pack_cnhw_role<float, false, false>(b % a.phase_blocks, b / a.phase_blocks, a.x, a.Lc, a.ws.part_max, a.cnhw, a.pa, a.ws, ClipArgs{});
}

// grid of k_pack_cnhw: x enumerates (channel, block of 1024 dwords) with the channel's XCD in the low bits,
// z the stride phase
int pack_per_chan(const daq_layout& L) { return (int)ceil_div(L.plane_pitch / 4, 4 * kBlock); }
dim3 pack_grid(const daq_layout& L) {
    return dim3((unsigned)(round_up(L.C, kXcd) * pack_per_chan(L)), 1u, (unsigned)(L.phases_h * L.phases_w));
}
PackArgs pack_args(const daq_layout& L, int part_n, uint32_t tensor, uint64_t seed) {
    PackArgs pa{};
    pa.div_slot = make_fastdiv((uint32_t)(L.img_rows * L.row_pitch));
    pa.div_pitch = make_fastdiv((uint32_t)L.row_pitch);
    pa.per_chan = pack_per_chan(L);
    pa.lead_imgs = (int)ceil_div(L.lead, (int64_t)L.img_rows * L.row_pitch);
    pa.part_n = part_n;
    pa.tensor = tensor;
    pa.seed = seed;
    return pa;
}
// The packing kernel indexes a plane with 32-bit integers.
bool pack_supported(const daq_layout& L) {
    const int64_t lim24 = (int64_t)1 << 24;
    return L.plane_pitch + L.lead + (int64_t)L.img_rows * L.row_pitch < ((int64_t)1 << 31) && (L.plane_pitch & 3) == 0 &&
           (int64_t)L.img_rows * L.row_pitch < lim24 &&
           (int64_t)(L.N + 1 + ceil_div(L.lead, (int64_t)L.img_rows * L.row_pitch)) * L.C < lim24 / 2 && (int64_t)L.H * L.W < lim24 / 2 &&
           (int64_t)L.img_rows * L.phases_h < lim24 && (int64_t)L.row_pitch * L.phases_w < lim24;
}
// The quantization kernels read an fp32 tensor through a buffer descriptor with 32-bit offsets.
bool f32_tensor_supported(int64_t elems) { return elems * 4 < ((int64_t)1 << 31); }


// Bytes of an NHWC buffer behind its last pixel (the buffer is rounded up to 256 bytes).
int nhwc_tail(const daq_layout& L) { return (int)(L.bytes - (int64_t)L.N * L.H * L.W * L.c_pitch); }

// Elements per thread of the source-driven row kernel (4 or 2), or 0 when the layout needs the output-driven one.
// `any`: a row length or an alignment that fits neither is served element by element (1), which pays where the kernel only writes
// the padding and the channels whose class was guessed wrong.
int rows_vector(const daq_layout& Ld, const void* src, int elem_bytes = 4, bool any = false) {
    const int64_t lim24 = (int64_t)1 << 24;
    const bool unsplit = Ld.phases_h == 1 && Ld.phases_w == 1 && Ld.org_h == 0 && Ld.org_w == 0 &&
                         (int64_t)Ld.N * Ld.img_rows < lim24 && (int64_t)Ld.H * Ld.W < lim24 &&
                         (int64_t)(Ld.N + 1) * Ld.C < lim24 && Ld.plane_pitch < ((int64_t)1 << 31);
    // the vector of 4 or 2 source elements a thread loads must be aligned as a whole
    if (unsplit && Ld.W % 4 == 0 && ((uintptr_t)src & (uintptr_t)(4 * elem_bytes - 1)) == 0) return 4;
    if (unsplit && Ld.W % 2 == 0 && ((uintptr_t)src & (uintptr_t)(2 * elem_bytes - 1)) == 0) return 2;
    return unsplit && any ? 1 : 0;
}

// Whether the NHWC pass over a tensor can write the channel-major copy of this layout too, and what it needs for that.
bool early_copy_supported(const daq_layout& Ld, const void* src, int elem_bytes) {
    return rows_vector(Ld, src, elem_bytes, true) != 0 && Ld.lead + (int64_t)Ld.N * Ld.img_rows * Ld.row_pitch < ((int64_t)1 << 31);
}
// A tensor larger than the caches hold to the end is read with the streaming hint, on planes of whole units only: elsewhere units are not
// aligned, neighbouring tiles share lines that the hint gives up between the two (quantizing launch, us, with and without: 128 x 96 x 112 x 112
// 167 and 230; call of 128 x 144 x 70 x 70 172 and 189; 55 x 384 x 71 x 70 153 and 133, call of 64 x 128 x 101 x 101 305 and 294).
bool read_once(int64_t bytes, int HW) { return bytes > kCacheBytes && unit_kind(HW) == kWhole; }

}  // namespace

// Where the guess was right each workgroup of the packing launch behind an early copy folds the channel's counts and returns, so there are no more
// of them where rows are read an element at a time: its time is their number, not what they read (a workgroup to 1024 and to 4096 elements, packing
// launch and whole call with statistics given, us: 209 x 880 x 7 x 7 15.9 and 9.1, 32.9 and 26.0; 218 x 1500 x 7 x 7, padded, 27.1 and 15.7, 62.8 and 51.3).
int early_pack_blocks(int64_t channel_elems) { return (int)std::min<int64_t>(ceil_div(channel_elems, 16 * kBlock), 16); }

namespace {

EarlyVq early_vq(const daq_layout& Ld, int8_t* dst) {
    EarlyVq ev{};
    ev.vq = dst;
    ev.chan_pitch = Ld.chan_pitch;
    ev.lead = (int32_t)Ld.lead;
    ev.img_rows = Ld.img_rows;
    ev.row_pitch = Ld.row_pitch;
    ev.W = Ld.W;
    ev.div_w = make_fastdiv((uint32_t)Ld.W);
    ev.flat = Ld.row_pitch == Ld.W && Ld.img_rows == Ld.H;
    ev.whole = ev.flat || Ld.W % 4 == 0;
    return ev;
}

RowsArgs rows_args(const daq_layout& Ld, int v, bool early, int part_n, uint32_t tensor, uint64_t seed) {
    RowsArgs ra{};
    const uint32_t hwv = (uint32_t)(Ld.H * Ld.W / v);
    ra.div_hwv = make_fastdiv(hwv);
    ra.div_wv = make_fastdiv((uint32_t)(Ld.W / v));
    ra.div_prb = make_fastdiv((uint32_t)std::max(1, (Ld.img_rows - Ld.H) * Ld.row_pitch));
    ra.per_chan = (int)ceil_div((int64_t)Ld.N * hwv, 4 * kBlock);
    ra.grid_per_chan = early ? early_pack_blocks((int64_t)Ld.N * Ld.H * Ld.W) : ra.per_chan;
    ra.part_n = part_n;
    ra.early = early ? 1 : 0;
    ra.tensor = tensor;
    ra.seed = seed;
    return ra;
}
int64_t rows_blocks(const daq_layout& Ld, const RowsArgs& ra) { return round_up(Ld.C, kXcd) * (ra.grid_per_chan + 1); }

// Workgroups of the launch below for one copy.
int64_t pack_blocks(const daq_layout& Ld, const void* src, int elem_bytes) {
    const int v = rows_vector(Ld, src, elem_bytes);
    if (v) return rows_blocks(Ld, rows_args(Ld, v, false, 0, 0u, 0));
    const dim3 g = pack_grid(Ld);
    return (int64_t)g.x * g.z;
}

// Launches the channel-major packing of one fp32 NCHW tensor: the source-driven row kernel when the
// layout allows it, the output-driven kernel otherwise.
// With dst2 the same pass also writes a second copy quantized with the per-tensor scale scale2 (random stream
// tensor2); *fused tells whether that happened - the output-driven kernel writes one copy per launch.
template <typename T>
daq_status launch_pack(const char* name, bool stoch, bool clip, const T* src, const daq_layout& Ld,
                       const float* scale, int8_t* dst, uint32_t tensor, uint64_t seed,
                       const QuantWs& ws, const ClipArgs& ca, hipStream_t st, int8_t* dst2 = nullptr,
                       const float* scale2 = nullptr, uint32_t tensor2 = 0, bool* fused = nullptr, bool early = false, int part_n = 0,
                       float* publish = nullptr) {
    if (fused) *fused = false;
    const CnhwView V = cnhw_view(Ld);
    const int v = rows_vector(Ld, src, (int)sizeof(T), early);
    if (early && !v) return DAQ_ERR_INVALID_ARG;   // the caller checks rows_vector before it asks for the early copy
    if (v) {
        RowsArgs ra = rows_args(Ld, v, early, part_n, tensor, seed);
        ra.publish = publish;
        ra.publish_raw = ws.layer;
        ra.dst2 = dst2;
        ra.scale2 = scale2;
        ra.tensor2 = tensor2;
        if (fused) *fused = dst2 != nullptr;
        const dim3 grid((unsigned)rows_blocks(Ld, ra));
#define DAQ_ROWS(S, CL, VV) \
    DAQ_LAUNCH(name, st, hipLaunchKernelGGL((k_pack_rows<T, S, CL, VV>), grid, dim3(kBlock), 0, st, src, V, scale, dst, ra, ws, ca))
        if (v == 4) {
            if (stoch) { if (clip) DAQ_ROWS(true, true, 4); else DAQ_ROWS(true, false, 4); }
            else { if (clip) DAQ_ROWS(false, true, 4); else DAQ_ROWS(false, false, 4); }
        } else if (v == 1) {
            if (!clip) return DAQ_ERR_INVALID_ARG;
            if (stoch) DAQ_ROWS(true, true, 1); else DAQ_ROWS(false, true, 1);
        } else {
            if (stoch) { if (clip) DAQ_ROWS(true, true, 2); else DAQ_ROWS(true, false, 2); }
            else { if (clip) DAQ_ROWS(false, true, 2); else DAQ_ROWS(false, false, 2); }
        }
#undef DAQ_ROWS
        return DAQ_OK;
    }
    if (!pack_supported(Ld)) return DAQ_ERR_UNSUPPORTED;
    PackArgs pa = pack_args(Ld, part_n, tensor, seed);
    pa.publish = publish;
    pa.publish_raw = ws.layer;
    const dim3 grid = pack_grid(Ld);
#define DAQ_PACK(S, CL) \
    DAQ_LAUNCH(name, st, hipLaunchKernelGGL((k_pack_cnhw<T, S, CL>), grid, dim3(kBlock), 0, st, src, V, scale, dst, pa, ws, ca))
    if (stoch) { if (clip) DAQ_PACK(true, true); else DAQ_PACK(true, false); }
    else { if (clip) DAQ_PACK(false, true); else DAQ_PACK(false, false); }
#undef DAQ_PACK
    return DAQ_OK;
}

}  // namespace

size_t quantize_grad_ws_bytes(const daq_conv_desc& d) {
    return (size_t)carve_quant_ws(nullptr, d.Cout, d.N, daq_out_h(&d) * daq_out_w(&d)).total_bytes;
}

// Forward workspace, in floats: the partial maxima of X, those of W, what the shared quantizer code writes beside its
// results, and room for the callers of 3-D layers (kFwdWsFree).
size_t fwd_quant_ws_bytes(const daq_conv_desc&) { return 4096; }
static_assert(kAbsmaxBlocksX + kAbsmaxBlocksW + 8 <= kFwdWsFree && kFwdWsFree + 8 <= 4096 / 4, "forward workspace");

// A wave's work is serial, some 100 instructions a unit.  While the chip holds a wave of every workgroup at once, fewer units to a
// thread are faster (16 channels of 832 units: 7.2, 7.4, 8.2, 11.0 us with 2, 4, 8, 16); from there on the form that keeps the most
// waves on a CU, which takes 24 of 2 to 8 units and 16 of 16 (1024 channels of 5289 units, whole call: 54.9 us as 12 waves of 8
// units, two workgroups a CU; 60.8 as 8 of 16, 75.3 as 6 of 16), of equals the one whose waves have less to do, then the one with fewer
// slots (1240 channels of 2401 units: 8 waves of 8, five of them in use, 33 us; 12 of 4 35).  From five waves on they
// come in fours, one to a SIMD: a SIMD with a wave more than the others sets the time (546 channels of 14256 units: 67.5 us with 14
// waves, 59.3 with 16).  Over 528 sizes the choice is 0.7 % from the fastest form, at most 10 %.
ResidentForm resident_form(int C, int64_t units) {
    constexpr int kUnits[4] = {2, 4, 8, 16}, kHeld[4] = {24, 24, 24, 16};
    ResidentForm best{16, 16};
    int64_t best_held = 0, best_work = 0;
    for (int i = 0; i < 4; ++i) {
        int64_t w = ceil_div(units, kUnits[i] * kWave);
        if (w > 16) continue;
        if (w > 4) w = round_up(w, 4);
        const int64_t per_cu = kHeld[i] / w, held = per_cu * w, work = w * ceil_div(units, w * kWave);
        if (i < 3 && C <= 256 * per_cu) return ResidentForm{kUnits[i], (int)w};
        if (held > best_held || (held == best_held && (work < best_work || (work == best_work && kUnits[i] * w <= best.nu * best.waves)))) {
            best = ResidentForm{kUnits[i], (int)w};
            best_held = held;
            best_work = work;
        }
    }
    return best;
}

// The fold is a load, a reduction and a barrier in front of each workgroup's codes, a launch of its own some 3.5 us: level at two to
// three rounds of eight workgroups a CU (depthwise, packing alone: 492 channels of 24 x 24, batch 92, 6888 workgroups, 27.5 us without the
// fold and 30.8 with it; 672 of 38 x 38, batch 34, 16800: 38 and 48).
bool fold_in_packing(int64_t workgroups) { return workgroups <= 4096; }

// A workgroup per channel leaves CUs idle where channels are few, and a large one takes 10 to 30 us; three sweeps of a tensor of a few
// channels take 13 to 15.  What a unit costs the workgroup: finding its row where planes are padded, elements one by one where they are
// not whole units, and twice that the random word of a stochastic code.  Level with the sweeps, by these and by thousands of units, at
// (resident and sweeps in us)
//   units         6.5 Ki                    9.5 Ki                    14 Ki
//   plain         4: 10.8 and 12.7          4: 12.0 and 13.2          16 (1.04 of the sweeps)
//   padded        4: 0.97 of them           32: 14.9 and 15.0         64 (1.00)
//   both          32: 14.7 and 14.9         64 (1.04)                 96 (1.02)
//   stochastic    16: 13.9 and 14.1         64: 17.6 and 18.6         80 (1.02)
//   and padded    48: 15.5 and 16.2         80 (0.98)                 96 (1.01)
//   and both      80 (0.95)                 96 (1.04)                 128 (1.01)
// channels.  Channels of more than 8 Ki units run one to a CU, and a second round for a few of them does not pay either (268 of 11952
// units in bfloat16: 46 and 43 us).  (512 channels of 12544 units in two rounds are level with the sweeps, 59 + 27 us against 31 + 50 + 8,
// but save a launch.)
bool resident_pays(int C, int64_t units, bool padded, bool tails, bool stochastic) {
    if (units > 8 * 1024 && C > 256 && C < 288) return false;
    constexpr int kChannels[] = {1, 1, 32, 64, 88, 112, 128};
    const int size = units <= 8 * 1024 ? 0 : units <= 12 * 1024 ? 1 : 2;
    return units <= 6 * 1024 || C >= kChannels[size + padded + tails + 2 * stochastic];
}

// Both copies in the counting sweep save a read of dY and cost it instructions and stores of four bytes; the packing launch behind it is left with
// the padding between the rows, its own line where an image has any.  Speed of the early copy over three sweeps, by millions of elements (16 to 200
// channels, fp32; bfloat16 the same but where it is given):
//                                         4      5      6      8      10
//   stochastic, rows of whole vectors     1.02   1.04   1.04   1.07   1.11       odd rows 1.06 to 1.18
//   nearest, no padding, 4 to a vector    0.95   0.99   1.02   1.06   1.08       2 to a vector and odd 1.06 and more
//   nearest, padded                       0.95   0.96   0.97   0.99   1.02       bfloat16, 2 to a vector and odd 0.99, 0.99, 1.02, 1.03, 1.05
// With the producer's statistics the sweep is the only read of dY left and writes both copies at any size, but for odd rows, where the
// packing launch is slow: without padding 1.06 at 3 to 4 M, 1.15 from 4 on, padded and nearest 0.93 to 1.0 up to 16 M (48 to 3000 channels), stochastic 1.03.
// Depthwise gradients of odd rows, whose two copies are both channel-major: 1.08 to 1.4, but nearest on rows of 7 0.95 (of 29: 1.10; with the producer's
// statistics 1.00).
int64_t early_copy_from(const EarlyCase& e) {
    constexpr int64_t kMi = (int64_t)1 << 20;
    if (e.channel_major) return e.given ? 3 * kMi : e.nearest && e.W < 16 ? INT64_MAX : 4 * kMi;
    if (e.given) return e.vector ? 0 : (e.nearest && e.padded ? 16 : 3) * kMi;
    if (!e.nearest) return 4 * kMi;
    if (e.padded) return (e.bf16 && e.vector != 4 ? 6 : 8) * kMi;
    return (e.vector == 4 ? 6 : 4) * kMi;
}

// Whether the resident launch writes the NHWC copy as well: every workgroup of eight waves then reads the whole tensor and stores its
// codes byte by byte.  What a CU reads is C * M elements for each of its workgroups, one to 256 channels, and that sets the time: two launches
// are 9.9 to 10.2 us a call at any of these sizes, one launch 7.0 to 7.3 up to 32 Ki elements a CU and (channels of elements; elements a CU)
//   one workgroup a CU     64 of 1024 (64 Ki) 7.5, 256 of 256 (64 Ki) 8.0, 96 of 784 (74 Ki) 8.3; 160 of 784 (123 Ki) 10.5, 256 of 512 (128 Ki) 10.7
//   two                    512 of 64 (64 Ki) 8.3, 264 of 160 (83 Ki) 8.4, 384 of 160 (120 Ki) 9.4; 512 of 128 (128 Ki) 10.4, 448 of 160 10.9
//   three                  768 of 16 (36 Ki) 8.2, 576 of 49 (83 Ki) 10.0, 520 of 64 (98 Ki) 9.3; 576 of 64 (108 Ki) 10.4, 640 of 64 (120 Ki) 10.9
//   four                   1024 of 16 (64 Ki) 9.3; 1024 of 49 (196 Ki) 14.2
//   six and more           1536 of 1 11.0, 2048 of 16 17, 5120 of 16 57, 8192 of 8 72
bool resident_all_pays(int C, int64_t M, int64_t units) {
    constexpr int kMost[4] = {80, 120, 98, 80};   // Ki elements a CU, by its workgroups
    const int64_t each = ceil_div(C, 256);
    return units <= 2 * 8 * kWave && M <= 1024 && each <= 4 && each * C * M <= kMost[each - 1] * 1024;
}

// ---------------------------------------------------------------------------------------------
// forward-side quantization of X (two layouts) and W (packed)
// ---------------------------------------------------------------------------------------------
// Whether the forward pass can quantize this activation: everything that could fail is decided here, before the
// first launch, so that an unsupported problem leaves every output untouched.
daq_status quantize_activation_check(const daq_conv_desc& d, const float* X) {
    daq_layout Ln, Lc;
    if (daq_layout_qx_nhwc(&d, &Ln) != DAQ_OK || daq_layout_qx_cnhw(&d, &Lc) != DAQ_OK) return DAQ_ERR_INVALID_ARG;
    if (!f32_tensor_supported((int64_t)d.N * d.Cin * d.Hin * d.Win)) return DAQ_ERR_UNSUPPORTED;
    if (rows_vector(Lc, X) == 0 && !pack_supported(Lc)) return DAQ_ERR_UNSUPPORTED;
    return DAQ_OK;
}

daq_status quantize_forward(const daq_conv_desc& d, const float* X, int8_t* qx_nhwc, int8_t* qx_cnhw, float* s_x, const float* W,
                            int8_t* qw, float* s_w, void* wsp, hipStream_t st, daq_schedule schedule) {
    const daq_status ok = quantize_activation_check(d, X);
    if (ok != DAQ_OK) return ok;
    daq_layout Ln, Lc;
    if (daq_layout_qx_nhwc(&d, &Ln) != DAQ_OK || daq_layout_qx_cnhw(&d, &Lc) != DAQ_OK) return DAQ_ERR_INVALID_ARG;
    float* part = (float*)wsp;
    const int taps = d.kH * d.kW;
    const int64_t n = (int64_t)d.N * d.Cin * d.Hin * d.Win, nw = W ? (int64_t)d.Cout * (d.Cin / d.groups) * taps : 0;
    AbsmaxArgs m{};
    m.x[0] = X; m.n[0] = n; m.part[0] = part;
    m.x[1] = W; m.n[1] = nw; m.part[1] = part + kAbsmaxBlocksX;
    m.blocks[0] = (int)std::min<int64_t>(ceil_div(n, kBlock * 32), kAbsmaxBlocksX);
    m.blocks[1] = (int)std::min<int64_t>(ceil_div(nw, kBlock * 32), kAbsmaxBlocksW);

    const int HW = d.Hin * d.Win;
    FwdQuantArgs a{};
    a.x = X; a.nhwc = qx_nhwc; a.cnhw = qx_cnhw; a.s_x = s_x;
    a.N = d.N; a.C = d.Cin; a.HW = HW; a.c_pitch = Ln.c_pitch; a.tail = nhwc_tail(Ln);
    a.div_u = make_fastdiv(unit_divisor(HW));
    a.Lc = cnhw_view(Lc);
    // Unit-stride layers whose channel-major layout the row kernel serves: one sweep over X writes both copies (the
    // mechanism of the early per-channel copy of dY, with the per-tensor scale), and only the padding bytes are left.
    // (by default from 8 Mi elements on: below that the two lean passes are as fast or faster; 28 x 176 x 27 x 31, 4.1 Mi: 49.6 and 50.5 us a call)
    const bool early = (schedule == DAQ_SCHEDULE_EARLY_COPY || (schedule == DAQ_SCHEDULE_AUTO && n >= ((int64_t)8 << 20))) &&
                       early_copy_supported(Lc, X, 4);
    if (W) {
        PackWArgs& w = a.w;
        if (daq_layout_qw(&d, &w.L) != DAQ_OK) return DAQ_ERR_INVALID_ARG;
        w.w = W; w.out = qw; w.s_w = s_w; w.part = m.part[1]; w.part_n = m.blocks[1];
        w.Cout = d.Cout; w.Cin = d.Cin; w.groups = d.groups; w.taps = taps;
        w.cig = d.Cin / d.groups; w.cog = d.Cout / d.groups;
        if (d.groups == 1) {
            w.chunks = (int)ceil_div(taps, kWTaps);
            w.ci_tiles = 2 * (int)ceil_div(d.Cin, 64);
            const int first = std::min(taps, kWTaps), last = taps - (w.chunks - 1) * kWTaps;
            w.div_run = make_fastdiv((uint32_t)(32 * first)); w.div_tap = make_fastdiv((uint32_t)first);
            w.div_runl = make_fastdiv((uint32_t)(32 * last)); w.div_tapl = make_fastdiv((uint32_t)last);
            w.blocks = 2 * (int)ceil_div(d.Cout, 64) * w.ci_tiles * w.chunks;
        } else {
            w.blocks = (int)ceil_div(w.L.bytes, 16 * kBlock);
        }
        a.w_blocks = (int)round_up(w.blocks, kXcd);
    }
    // Where the channel-major copy has workgroups of its own, both kinds read X side by side, and the sweep over NHWC records is
    // one workgroup a CU: more of them take from the other kind more than they gain (quantizing launch, us, 4, 1 a CU: 12 x 224 x 37 x 37
    // 14.9 and 12.0, 9 x 640 x 25 x 25 17.8 and 14.4, 7 x 464 x 83 x 83 at stride 2 67.6 and 64.8).  Alone it takes all the chip
    // holds (29 x 224 x 48 x 47 18.7, one a CU 21.2; 72 x 49 x 99 x 99 47.6 and 57.0).
    const int waves = early ? forward_waves(d.Cin, d.N, HW, a.w_blocks) : kBlock / kWave;
    a.ws = carve_quant_ws(nullptr, d.Cin, d.N, HW, waves, early ? 0 : 256);   // only the tile geometry is used: nothing is counted here
    a.ws.part_max = part;
    a.ws.part_n = m.blocks[0];
    a.ws.layer = part + kAbsmaxBlocksX + kAbsmaxBlocksW;
    a.x_blocks = (int)round_up(a.ws.cp.workgroups(), kXcd);
    const int v = rows_vector(Lc, X, 4, early);
    int64_t c_blocks;
    if (v) {
        a.ra = rows_args(Lc, v, early, a.ws.part_n, 0u, 0);
        c_blocks = rows_blocks(Lc, a.ra);
    } else {
        a.pa = pack_args(Lc, a.ws.part_n, 0u, 0);
        const dim3 g = pack_grid(Lc);
        a.phase_blocks = (int)g.x;
        c_blocks = (int64_t)g.x * g.z;
    }
    if (early) {
        a.ev = early_vq(Lc, qx_cnhw);
        a.ev.once = read_once(n * 4, HW);
    }
    const int64_t blocks = a.w_blocks + a.x_blocks + c_blocks;
    if (blocks >= ((int64_t)1 << 31)) return DAQ_ERR_UNSUPPORTED;
    DAQ_LAUNCH("absmax", st, hipLaunchKernelGGL(k_absmax, dim3((unsigned)(m.blocks[0] + m.blocks[1])), dim3(kBlock), 0, st, m));   // the first launch: nothing behind it fails
#define DAQ_FWD_QUANT(E, VV, UN, WV) \
    DAQ_LAUNCH("quant_fwd", st, hipLaunchKernelGGL((k_fwd_quant<E, VV, UN, WV>), dim3((unsigned)blocks), dim3(WV * kWave), 0, st, a))
#define DAQ_FWD_EARLY(VV, UN) do { if (waves == 8) DAQ_FWD_QUANT(true, VV, UN, 8); else DAQ_FWD_QUANT(true, VV, UN, 4); } while (0)
    const int unit = unit_kind(HW);
    if (v == 4) { if (early) DAQ_FWD_EARLY(4, kWhole); else DAQ_FWD_QUANT(false, 4, kWhole, 4); }   // rows of whole units
    else if (unit == kWhole) {
        if (v == 2) { if (early) DAQ_FWD_EARLY(2, kWhole); else DAQ_FWD_QUANT(false, 2, kWhole, 4); }
        else if (early) DAQ_FWD_EARLY(1, kWhole);
        else DAQ_FWD_QUANT(false, 0, kWhole, 4);
    } else if (unit == kTail) {
        if (v == 2) { if (early) DAQ_FWD_EARLY(2, kTail); else DAQ_FWD_QUANT(false, 2, kTail, 4); }
        else if (early) DAQ_FWD_EARLY(1, kTail);
        else DAQ_FWD_QUANT(false, 0, kTail, 4);
    } else {
        if (v == 2) { if (early) DAQ_FWD_QUANT(true, 2, kElems, 4); else DAQ_FWD_QUANT(false, 2, kElems, 4); }
        else if (early) DAQ_FWD_QUANT(true, 1, kElems, 4);
        else DAQ_FWD_QUANT(false, 0, kElems, 4);
    }
#undef DAQ_FWD_EARLY
#undef DAQ_FWD_QUANT
    return DAQ_OK;
}

}  // namespace daq

using namespace daq;

// ---------------------------------------------------------------------------------------------
// Algorithm 1, per-channel loop + vectorized and global quantization
// ---------------------------------------------------------------------------------------------
namespace {

// Orders everything launched on `later` from now on behind everything launched on `first` so far.  One event per
// device, created on first use and kept: a wait refers to the state of the event at the time of the call, so the
// next record does not disturb it.
daq_status stream_follows(hipStream_t later, hipStream_t first) {
    static std::mutex mu;
    static hipEvent_t ev[64] = {};
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return DAQ_ERR_HIP;
    std::lock_guard<std::mutex> lock(mu);
    if (!ev[dev] && hipEventCreateWithFlags(&ev[dev], hipEventDisableTiming) != hipSuccess) return DAQ_ERR_HIP;
    if (hipEventRecord(ev[dev], first) != hipSuccess || hipStreamWaitEvent(later, ev[dev], 0) != hipSuccess) return DAQ_ERR_HIP;
    return DAQ_OK;
}

// Per-channel statistics that the producer of dY already has (S1 of Algorithm 1): |g|max, sum and sum of squares.
struct ProducerStats {
    const float* absmax;
    const double* sum;
    const double* sumsq;
};

// T = float or uint16_t (bfloat16): the element type of dY
template <typename T>
daq_status quantize_grad_impl(const daq_conv_desc* desc, const T* dY, float* s_state, float k, float A, float lambda,
                              daq_round mode, uint64_t seed, daq_scheme scheme, daq_schedule schedule, int8_t* vq,
                              int8_t* qg, float* s_chan, float* s_global, uint8_t* cls, float* stats, void* workspace,
                              size_t workspace_bytes, void* stream, void* side_stream = nullptr,
                              const ProducerStats* given = nullptr) {
    if (!desc_valid(desc) || !dY || !s_state || !vq || !qg || !s_chan || !s_global || !cls)
        return DAQ_ERR_INVALID_ARG;
    if (given && (!given->absmax || !given->sum || !given->sumsq || ((uintptr_t)given->absmax & 3u) ||
                  ((uintptr_t)given->sum & 7u) || ((uintptr_t)given->sumsq & 7u)))
        return DAQ_ERR_INVALID_ARG;
    if (mode != DAQ_ROUND_NEAREST && mode != DAQ_ROUND_STOCHASTIC) return DAQ_ERR_INVALID_ARG;
    if (scheme != DAQ_SCHEME_DAQ && scheme != DAQ_SCHEME_GQ && scheme != DAQ_SCHEME_GVQ && scheme != DAQ_SCHEME_MCS)
        return DAQ_ERR_INVALID_ARG;
    if (schedule != DAQ_SCHEDULE_AUTO && schedule != DAQ_SCHEDULE_THREE_SWEEPS && schedule != DAQ_SCHEDULE_EARLY_COPY &&
        schedule != DAQ_SCHEDULE_CHANNEL_RESIDENT)
        return DAQ_ERR_INVALID_ARG;
    if (((uintptr_t)dY & (sizeof(T) - 1)) || ((uintptr_t)vq & 15u) || ((uintptr_t)qg & 15u)) return DAQ_ERR_INVALID_ARG;
    daq_layout Lv, Lg;
    daq_status rc = daq_layout_vq(desc, &Lv);
    if (rc != DAQ_OK) return rc;
    rc = daq_layout_qg(desc, &Lg);
    if (rc != DAQ_OK) return rc;
    const size_t need = daq_workspace_bytes(DAQ_OP_QUANTIZE_GRAD, desc);
    if (!workspace || workspace_bytes < need || ((uintptr_t)workspace & 255u)) return DAQ_ERR_WORKSPACE;

    // the kernels address dY with 32-bit byte offsets
    if (!((int64_t)desc->N * desc->Cout * daq_out_h(desc) * daq_out_w(desc) * (int64_t)sizeof(T) < ((int64_t)1 << 31)))
        return DAQ_ERR_UNSUPPORTED;
    // the packing pass is the last launch: what it cannot serve is refused here, before the first one
    if (rows_vector(Lv, dY, (int)sizeof(T)) == 0 && !pack_supported(Lv)) return DAQ_ERR_UNSUPPORTED;

    hipStream_t st = (hipStream_t)stream;
    // With a side stream, what only the filter gradient consumes leaves the stream of the data gradient: from the
    // point where qg and s_global need nothing more, the side stream waits for `st` and takes the remaining launches.
    hipStream_t side = (side_stream && side_stream != stream) ? (hipStream_t)side_stream : nullptr;
    const int N = desc->N, C = desc->Cout, Ho = daq_out_h(desc), Wo = daq_out_w(desc);
    const int HW = Ho * Wo;
    const bool stoch = (mode == DAQ_ROUND_STOCHASTIC);
    const uint64_t keys = round_keys(seed);   // what the kernels receive in the place of the seed
    const bool qg_nhwc = (Lg.kind == DAQ_LAYOUT_NHWC);
    QuantWs ws = carve_quant_ws(workspace, C, N, HW);
    ws.scheme = (int)scheme;
    const double Mtot = (double)N * (double)C * (double)HW;

    const int unit = unit_kind(HW);
    const FastDiv div_hw = make_fastdiv((uint32_t)HW), div_u = make_fastdiv(unit_divisor(HW));

    // Channels that fit in LDS: one read of dY serves statistics, count, decision and the per-channel copy
    // (k_chan_resident); the global copy follows in the counting kernel's copy-only form.
    const bool res_v4 = HW >= 4;   // dword-aligned 16-byte loads run at full rate, as in the statistics sweep
    const int res_upp = res_v4 ? (HW + 3) / 4 : HW;
    const int64_t res_units = (int64_t)N * res_upp;
    const ResidentForm res = resident_form(C, res_units);
    // planes without padding between rows and images hold element m at byte lead + m
    const bool res_flat = res_v4 && Lv.row_pitch == Lv.W && Lv.img_rows == Lv.H && (Lv.lead & 3) == 0 && (Lv.plane_pitch & 3) == 0 &&
                          Lv.lead + (int64_t)N * HW <= Lv.plane_pitch;
    const bool resident_ok = scheme == DAQ_SCHEME_DAQ && res_units <= 16 * 1024 && Lv.plane_pitch <= kResidentMaxLds &&
                             (Lv.plane_pitch & 15) == 0 && (Lv.chan_pitch & 15) == 0;
    if (!given && resident_ok && (schedule == DAQ_SCHEDULE_CHANNEL_RESIDENT || (schedule == DAQ_SCHEDULE_AUTO && resident_pays(C, res_units, !res_flat, HW % 4 != 0, stoch)))) {
        ws.slabs = 1;   // one |g|max partial per channel
        ws.part_n = C;
        const bool all = qg_nhwc && resident_all_pays(C, (int64_t)N * HW, res_units);
        const ResArgs ra{make_fastdiv((uint32_t)res_upp), make_fastdiv((uint32_t)Wo), N, C, HW, k, A, lambda, keys, qg, s_global, all ? Lg.c_pitch : 0, all ? nhwc_tail(Lg) : 0};
        const int res_waves = all ? 8 : res.waves;
        const ClipArgs ca{k, A, lambda, s_state, s_chan, cls, stats};
        const size_t lds = res_flat ? 0 : (size_t)Lv.plane_pitch;
        const dim3 rgrid((unsigned)round_up(C, kXcd));
#define DAQ_RES_LAUNCH(S, V, NUV, FL, TL, AL)                                                                           \
    {                                                                                                                \
        auto kern = k_chan_resident<T, S, V, NUV, FL, TL, AL>;                                                           \
        if (!FL && !allow_lds((const void*)kern, lds)) \
            return DAQ_ERR_HIP;                                                                                      \
        DAQ_LAUNCH("chan_resident", st, hipLaunchKernelGGL(kern, rgrid, dim3((unsigned)(res_waves * kWave)), lds, st, dY, cnhw_view(Lv), vq, ra, ws, ca)); \
    }
#define DAQ_RES_FORM(S, NUV, AL)                                                                                         \
    {                                                                                                                \
        if (!res_v4) DAQ_RES_LAUNCH(S, false, NUV, false, false, AL)                                                     \
        else if (res_flat && HW % 4 == 0) DAQ_RES_LAUNCH(S, true, NUV, true, false, AL)                                  \
        else if (res_flat) DAQ_RES_LAUNCH(S, true, NUV, true, true, AL)                                                  \
        else if (HW % 4 == 0) DAQ_RES_LAUNCH(S, true, NUV, false, false, AL)                                             \
        else DAQ_RES_LAUNCH(S, true, NUV, false, true, AL)                                                               \
    }
#define DAQ_RES_SIZE(S)                                                                                              \
    {                                                                                                                \
        if (all) DAQ_RES_FORM(S, 2, true)                                                                            \
        else if (res.nu == 2) DAQ_RES_FORM(S, 2, false)                                                                          \
        else if (res.nu == 4) DAQ_RES_FORM(S, 4, false)                                                                     \
        else if (res.nu == 8) DAQ_RES_FORM(S, 8, false)                                                                     \
        else DAQ_RES_FORM(S, 16, false)                                                                                     \
    }
        if (stoch) DAQ_RES_SIZE(true) else DAQ_RES_SIZE(false)
#undef DAQ_RES_FORM
#undef DAQ_RES_SIZE
#undef DAQ_RES_LAUNCH
        // the per-channel copy, its scales, classes and clip state are complete here; the global copy follows on `st`
        if (side && stream_follows(side, st) != DAQ_OK) return DAQ_ERR_HIP;
        if (all) return DAQ_OK;
        if (!qg_nhwc) {
            // depthwise layers: the per-tensor copy is channel-major too
            if (!fold_in_packing(pack_blocks(Lv, dY, (int)sizeof(T)))) {
                DAQ_LAUNCH("fold_scale", st, hipLaunchKernelGGL(k_fold_scale, dim3(1), dim3(kBlock), 0, st, ws.part_max, ws.part_n, s_global, ws.layer));
                return launch_pack("pack_qg", stoch, false, dY, Lv, s_global, qg, 1u, keys, ws, ClipArgs{}, st);
            }
            return launch_pack("pack_qg", stoch, false, dY, Lv, ws.part_max, qg, 1u, keys, ws, ClipArgs{}, st, nullptr, nullptr, 0, nullptr, false,
                               ws.part_n, s_global);
        }
        // The copy-only form has half the registers and is held to as many waves a CU as the counting one, which is the faster up to some 2000 channels;
        // beyond, blocks are many, workgroups of each few, and what is lost by whole rounds over the XCDs is more than that (sixteen and
        // twenty-four waves a CU, nearest, us: 27 x 2051 x 43 x 9 27 and 23, 3 x 3655 x 54 x 54 38 and 30, 47 x 3819 x 12 x 11 in bfloat16 24 and 16).
        if (C > 2000) ws.cp = plan_count(C, N, HW, 0, 256 * (24 / ws.cp.waves));
        const dim3 cgrid((unsigned)ws.cp.workgroups()), cblock((unsigned)(ws.cp.waves * kWave));
        const int tile_dw = ws.cp.tile_dwords(C);
        const size_t clds = (size_t)tile_dw * 8;
#define DAQ_COPY_LAUNCH(S, UN)                                                                                        \
    DAQ_LAUNCH("global_copy", st,                                                                                    \
               hipLaunchKernelGGL((k_count_qg<T, S, true, false, false, UN>), cgrid, cblock, clds, st, dY, N, C, HW, Lg.c_pitch, \
                                  div_u, ws, qg, keys, (const float*)s_state, s_global, EarlyVq{}, nhwc_tail(Lg), tile_dw))
        if (unit == kWhole) { if (stoch) DAQ_COPY_LAUNCH(true, kWhole); else DAQ_COPY_LAUNCH(false, kWhole); }
        else if (unit == kTail) { if (stoch) DAQ_COPY_LAUNCH(true, kTail); else DAQ_COPY_LAUNCH(false, kTail); }
        else if (stoch) DAQ_COPY_LAUNCH(true, kElems);
        else DAQ_COPY_LAUNCH(false, kElems);
#undef DAQ_COPY_LAUNCH
        return DAQ_OK;
    }

    // S1: statistics partials, at most 16 per channel - or the producer's: one partial per channel, read in place
    const bool vec4 = HW >= 4;   // dword-aligned 16-byte loads run at full rate; only tiny planes take the scalar path
    const unsigned sblocks = (unsigned)(round_up(C, kXcd) * ws.slabs);
    const FastDiv div_g4 = make_fastdiv((uint32_t)((HW + 3) / 4));
    if (given) {
        ws.slabs = 1;
        ws.part_n = C;
        ws.part_max = const_cast<float*>(given->absmax);   // the consumers only read the partials
        ws.part_s1 = const_cast<double*>(given->sum);
        ws.part_s2 = const_cast<double*>(given->sumsq);
    } else if (vec4 && HW % 4 == 0)
        DAQ_LAUNCH("stats", st, hipLaunchKernelGGL((k_stats<T, true, false>), dim3(sblocks), dim3(kBlock), 0, st, dY, N, C, HW, div_g4, ws));
    else if (vec4)
        DAQ_LAUNCH("stats", st, hipLaunchKernelGGL((k_stats<T, true, true>), dim3(sblocks), dim3(kBlock), 0, st, dY, N, C, HW, div_g4, ws));
    else
        DAQ_LAUNCH("stats", st, hipLaunchKernelGGL((k_stats<T, false, false>), dim3(sblocks), dim3(kBlock), 0, st, dY, N, C, HW, div_hw, ws));

    if (scheme == DAQ_SCHEME_MCS)
        DAQ_LAUNCH("layer_stats", st, hipLaunchKernelGGL(k_layer_stats, dim3(1), dim3(kBlock), 0, st, ws, C, Mtot));

    // S2 (+ the NHWC global copy); folds the statistics itself
    const dim3 cgrid((unsigned)ws.cp.workgroups()), cblock((unsigned)(ws.cp.waves * kWave));
    const int tile_dw = qg_nhwc ? ws.cp.tile_dwords(C) : 0;
    const size_t clds = (size_t)tile_dw * 8;
    // Large gradients: the counting pass also writes the per-channel copy under a guessed class (see k_count_qg), so
    // that the third sweep over dY only touches the channels whose guess was wrong.  Small ones are bound by launch
    // latency, not by bytes, and keep the leaner counting kernel.
    const int rows_v = rows_vector(Lv, dY, (int)sizeof(T));
    const bool padded = Lv.row_pitch != Lv.W || Lv.img_rows != Lv.H;
    const bool want_early = schedule == DAQ_SCHEDULE_EARLY_COPY ||
                            ((schedule == DAQ_SCHEDULE_AUTO || (given && schedule != DAQ_SCHEDULE_THREE_SWEEPS)) &&
                             (int64_t)N * C * HW >= early_copy_from({given != nullptr, !stoch, padded, sizeof(T) == 2, !qg_nhwc, rows_v, Wo}));
    // Two channel-major copies: where the packing kernel takes rows in whole vectors, one read of dY for both copies behind the counting
    // sweep is as fast (128 x 144 x 56 x 56, depthwise: 138 and 157 us); where rows are odd it would take two launches, an element at a time
    // (40 x 200 x 59 x 63: 116 and 90; 20 x 100 x 61 x 63: 44 and 37).
    const bool early = want_early && scheme == DAQ_SCHEME_DAQ && early_copy_supported(Lv, dY, (int)sizeof(T)) &&
                       (qg_nhwc || rows_v == 0);
    EarlyVq ev{};
    if (early) {
        // |g|max / sigma of M Gaussian samples is about sqrt(2 ln M), of M Laplace samples ln M / sqrt 2: halfway
        const double lnM = std::log((double)N * HW);
        ev = early_vq(Lv, vq);
        ev.once = read_once((int64_t)N * C * HW * (int64_t)sizeof(T), HW);
        ev.qg = qg_nhwc ? nullptr : qg;
        ev.k = k;
        ev.A = A;
        ev.ratio = (float)(0.5 * (std::sqrt(2.0 * lnM) + lnM / std::sqrt(2.0)));
    }
#define DAQ_COUNT_LAUNCH(S, Q, E, UN)                                                                                \
    DAQ_LAUNCH("count_qg", st,                                                                                       \
               hipLaunchKernelGGL((k_count_qg<T, S, Q, true, E, UN>), cgrid, cblock, clds, st, dY, N, C, HW,         \
                                  qg_nhwc ? Lg.c_pitch : 0, div_u, ws, qg, keys, (const float*)s_state,    \
                                  s_global, ev, qg_nhwc ? nhwc_tail(Lg) : 0, tile_dw))
#define DAQ_COUNT_UNIT(S, Q, E)                                                                                      \
    {                                                                                                                \
        if (unit == kWhole) DAQ_COUNT_LAUNCH(S, Q, E, kWhole);                                                       \
        else if (unit == kTail) DAQ_COUNT_LAUNCH(S, Q, E, kTail);                                                    \
        else DAQ_COUNT_LAUNCH(S, Q, E, kElems);                                                                      \
    }
    if (early) {
        if (qg_nhwc) { if (stoch) DAQ_COUNT_UNIT(true, true, true) else DAQ_COUNT_UNIT(false, true, true) }
        else { if (stoch) DAQ_COUNT_UNIT(true, false, true) else DAQ_COUNT_UNIT(false, false, true) }
    } else if (qg_nhwc) {
        if (stoch) DAQ_COUNT_UNIT(true, true, false) else DAQ_COUNT_UNIT(false, true, false)
    } else {
        DAQ_COUNT_UNIT(false, false, false)
    }
#undef DAQ_COUNT_UNIT
#undef DAQ_COUNT_LAUNCH
    if (scheme == DAQ_SCHEME_MCS)
        DAQ_LAUNCH("layer_decide", st,
                   hipLaunchKernelGGL(k_layer_decide, dim3(1), dim3(kBlock), 0, st, ws, (int)cgrid.x * ws.cp.waves, Mtot, k, A,
                                      lambda));

    // S3 + S4 + S5: discriminator, clip rule and the per-channel copy in CNHW (and the global copy for
    // depthwise layers, whose data gradient also runs channel-major)
    ClipArgs ca{k, A, lambda, s_state, s_chan, cls, stats};
    bool fused = false;
    // an NHWC global copy is complete here: the packing launch can move to the side stream.  (A channel-major global
    // copy is written by the packing launches themselves: they stay, and the side stream follows at the end.)
    hipStream_t sp = st;
    if (side && qg_nhwc) {
        if (stream_follows(side, st) != DAQ_OK) return DAQ_ERR_HIP;
        sp = side;
    }
    rc = launch_pack("pack_vq", stoch, true, dY, Lv, nullptr, vq, 0u, keys, ws, ca, sp, qg_nhwc ? nullptr : qg, s_global,
                     1u, &fused, early);
    if (rc != DAQ_OK) return rc;
    if (!qg_nhwc && !fused)
        rc = launch_pack("pack_qg", stoch, false, dY, Lv, s_global, qg, 1u, keys, ws, ClipArgs{}, st);
    if (rc == DAQ_OK && side && !qg_nhwc && stream_follows(side, st) != DAQ_OK) return DAQ_ERR_HIP;
    return rc;
}

}  // namespace

extern "C" daq_status daq_quantize_grad_ex(const daq_conv_desc* desc, const void* dY, float* s_state, float k, float A,
                                           float lambda, daq_round mode, uint64_t seed, const daq_quantize_opts* opts,
                                           int8_t* vq, int8_t* qg, float* s_chan, float* s_global, uint8_t* cls,
                                           float* stats, void* workspace, size_t workspace_bytes, void* stream) {
    const daq_quantize_opts def{DAQ_SCHEME_DAQ, DAQ_SCHEDULE_AUTO, 0, 0};
    const daq_quantize_opts& o = opts ? *opts : def;
    // the options arrive as plain integers: they are checked as integers, before anything treats them as enumerators
    if (o.dy_bf16 != 0 && o.dy_bf16 != 1) return DAQ_ERR_INVALID_ARG;
    if (o.scheme < DAQ_SCHEME_DAQ || o.scheme > DAQ_SCHEME_MCS || o.schedule < DAQ_SCHEDULE_AUTO || o.schedule > DAQ_SCHEDULE_CHANNEL_RESIDENT ||
        o.reserved != 0)
        return DAQ_ERR_INVALID_ARG;
    if (o.dy_bf16)
        return quantize_grad_impl<uint16_t>(desc, static_cast<const uint16_t*>(dY), s_state, k, A, lambda, mode, seed,
                                            (daq_scheme)o.scheme, (daq_schedule)o.schedule, vq, qg, s_chan, s_global, cls,
                                            stats, workspace, workspace_bytes, stream);
    return quantize_grad_impl<float>(desc, static_cast<const float*>(dY), s_state, k, A, lambda, mode, seed,
                                     (daq_scheme)o.scheme, (daq_schedule)o.schedule, vq, qg, s_chan, s_global, cls, stats,
                                     workspace, workspace_bytes, stream);
}

extern "C" daq_status daq_quantize_grad_split(const daq_conv_desc* desc, const void* dY, float* s_state, float k, float A,
                                              float lambda, daq_round mode, uint64_t seed, const daq_quantize_opts* opts,
                                              int8_t* vq, int8_t* qg, float* s_chan, float* s_global, uint8_t* cls,
                                              float* stats, void* workspace, size_t workspace_bytes, void* stream,
                                              void* side_stream) {
    const daq_quantize_opts def{DAQ_SCHEME_DAQ, DAQ_SCHEDULE_AUTO, 0, 0};
    const daq_quantize_opts& o = opts ? *opts : def;
    if (o.dy_bf16 != 0 && o.dy_bf16 != 1) return DAQ_ERR_INVALID_ARG;
    if (o.scheme < DAQ_SCHEME_DAQ || o.scheme > DAQ_SCHEME_MCS || o.schedule < DAQ_SCHEDULE_AUTO || o.schedule > DAQ_SCHEDULE_CHANNEL_RESIDENT ||
        o.reserved != 0)
        return DAQ_ERR_INVALID_ARG;
    if (o.dy_bf16)
        return quantize_grad_impl<uint16_t>(desc, static_cast<const uint16_t*>(dY), s_state, k, A, lambda, mode, seed,
                                            (daq_scheme)o.scheme, (daq_schedule)o.schedule, vq, qg, s_chan, s_global, cls,
                                            stats, workspace, workspace_bytes, stream, side_stream);
    return quantize_grad_impl<float>(desc, static_cast<const float*>(dY), s_state, k, A, lambda, mode, seed,
                                     (daq_scheme)o.scheme, (daq_schedule)o.schedule, vq, qg, s_chan, s_global, cls, stats,
                                     workspace, workspace_bytes, stream, side_stream);
}

extern "C" daq_status daq_quantize_grad_from_stats(const daq_conv_desc* desc, const void* dY, const float* ch_absmax,
                                                   const double* ch_sum, const double* ch_sumsq, float* s_state, float k,
                                                   float A, float lambda, daq_round mode, uint64_t seed,
                                                   const daq_quantize_opts* opts, int8_t* vq, int8_t* qg, float* s_chan,
                                                   float* s_global, uint8_t* cls, float* stats, void* workspace,
                                                   size_t workspace_bytes, void* stream, void* side_stream) {
    const daq_quantize_opts def{DAQ_SCHEME_DAQ, DAQ_SCHEDULE_AUTO, 0, 0};
    const daq_quantize_opts& o = opts ? *opts : def;
    if (o.dy_bf16 != 0 && o.dy_bf16 != 1) return DAQ_ERR_INVALID_ARG;
    if (o.scheme < DAQ_SCHEME_DAQ || o.scheme > DAQ_SCHEME_MCS || o.schedule < DAQ_SCHEDULE_AUTO || o.schedule > DAQ_SCHEDULE_CHANNEL_RESIDENT ||
        o.reserved != 0)
        return DAQ_ERR_INVALID_ARG;
    const ProducerStats ps{ch_absmax, ch_sum, ch_sumsq};
    if (o.dy_bf16)
        return quantize_grad_impl<uint16_t>(desc, static_cast<const uint16_t*>(dY), s_state, k, A, lambda, mode, seed,
                                            (daq_scheme)o.scheme, (daq_schedule)o.schedule, vq, qg, s_chan, s_global, cls,
                                            stats, workspace, workspace_bytes, stream, side_stream, &ps);
    return quantize_grad_impl<float>(desc, static_cast<const float*>(dY), s_state, k, A, lambda, mode, seed,
                                     (daq_scheme)o.scheme, (daq_schedule)o.schedule, vq, qg, s_chan, s_global, cls, stats,
                                     workspace, workspace_bytes, stream, side_stream, &ps);
}

extern "C" daq_status daq_quantize_grad_scheme(const daq_conv_desc* desc, const float* dY, float* s_state, float k,
                                               float A, float lambda, daq_round mode, uint64_t seed, daq_scheme scheme,
                                               int8_t* vq, int8_t* qg, float* s_chan, float* s_global, uint8_t* cls,
                                               float* stats, void* workspace, size_t workspace_bytes, void* stream) {
    const daq_quantize_opts o{(int32_t)scheme, DAQ_SCHEDULE_AUTO, 0, 0};
    return daq_quantize_grad_ex(desc, dY, s_state, k, A, lambda, mode, seed, &o, vq, qg, s_chan, s_global, cls, stats,
                                workspace, workspace_bytes, stream);
}

extern "C" daq_status daq_quantize_grad_bf16(const daq_conv_desc* desc, const uint16_t* dY_bf16, float* s_state, float k,
                                             float A, float lambda, daq_round mode, uint64_t seed, daq_scheme scheme,
                                             int8_t* vq, int8_t* qg, float* s_chan, float* s_global, uint8_t* cls,
                                             float* stats, void* workspace, size_t workspace_bytes, void* stream) {
    const daq_quantize_opts o{(int32_t)scheme, DAQ_SCHEDULE_AUTO, 1, 0};
    return daq_quantize_grad_ex(desc, dY_bf16, s_state, k, A, lambda, mode, seed, &o, vq, qg, s_chan, s_global, cls, stats,
                                workspace, workspace_bytes, stream);
}

extern "C" daq_status daq_quantize_grad(const daq_conv_desc* desc, const float* dY, float* s_state, float k, float A,
                                        float lambda, daq_round mode, uint64_t seed, int8_t* vq, int8_t* qg,
                                        float* s_chan, float* s_global, uint8_t* cls, float* stats, void* workspace,
                                        size_t workspace_bytes, void* stream) {
    return daq_quantize_grad_ex(desc, dY, s_state, k, A, lambda, mode, seed, nullptr, vq, qg, s_chan, s_global, cls, stats,
                                workspace, workspace_bytes, stream);
}

// ---------------------------------------------------------------------------------------------
// The quantizer for callers that cannot allocate: its scratch is a fixed array in device memory.
// ---------------------------------------------------------------------------------------------
// Every GPU the library runs on holds its own copy of this array, at its own address, until the process ends.
static __device__ __align__(256) unsigned char scratch[DAQ_STATIC_SCRATCH_BYTES];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};   // device address of `scratch` on each device, looked up on first use

// Address of the current device's copy of the array.  In host code the array's name is only a handle for this
// lookup, never a device address: kernels, fills and copies get the pointer returned here.
daq_status static_scratch(void** out) {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return DAQ_ERR_HIP;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return DAQ_ERR_HIP;
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return DAQ_OK;
}
}  // namespace

extern "C" daq_status daq_quantize_grad_noalloc(const daq_conv_desc* desc, const float* dY, float* s_state, float k, float A,
                                                float lambda, daq_round mode, uint64_t seed, int8_t* vq, int8_t* qg,
                                                float* s_chan, float* s_global, uint8_t* cls, float* stats, void* stream) {
    if (!desc_valid(desc)) return DAQ_ERR_INVALID_ARG;
    const size_t need = daq_workspace_bytes(DAQ_OP_QUANTIZE_GRAD, desc);
    if (need == 0) return DAQ_ERR_UNSUPPORTED;
    if (need > (size_t)DAQ_STATIC_SCRATCH_BYTES) return DAQ_ERR_SCRATCH_LIMIT;
    void* ws = nullptr;
    const daq_status rc = static_scratch(&ws);
    if (rc != DAQ_OK) return rc;
    // The kernels take the array through the same workspace argument as in daq_quantize_grad.  Nothing in it has to
    // start at zero: every partial result is written before it is read (no counters, no atomics).
    return daq_quantize_grad_ex(desc, dY, s_state, k, A, lambda, mode, seed, nullptr, vq, qg, s_chan, s_global, cls, stats, ws,
                                (size_t)DAQ_STATIC_SCRATCH_BYTES, stream);
}
