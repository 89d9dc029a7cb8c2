// Internal declarations shared by the translation units of libdaq.so (gfx950 only).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <algorithm>

#include "daq.h"

namespace daq {

constexpr int kWave = 64;            // CDNA wavefront width
constexpr int kXcd = 8;              // accelerator complex dies; workgroup i is dispatched to XCD i % 8
constexpr float kTinyScale = 7.888609052210118e-31f;  // 2^-100: below this a scale is reported as 0
// fp32 results of at least this many bytes leave through streaming (nontemporal) stores: written back as they are
// produced instead of at the end of the kernel, and without evicting the int8 operands the next kernels read.
// Smaller results stay in the write-back caches, which is faster for them (measured: 12.8 MB slower, 25.7 MB faster).
constexpr int64_t kStreamBytes = (int64_t)24 << 20;
// And only where a result plane is a whole number of 64-byte half-lines: the pieces of a line that two tiles share otherwise
// reach memory one by one (1 x 1, 1024 -> 256 at 14 x 14, batch 64, planes of 784 bytes, data gradient: 17 against 24 us).
// The tile kernel's 3-D forms and the depthwise kernels go by the size alone, as the shape of their planes made no difference:
// 3 x 3 x 3, 256 -> 256, 16 x 14 x 14, batch 8, 72 us either way (512 -> 512 at 16 x 7 x 7, batch 16, 127 us), the product being
// the longer part; depthwise 3 x 3, 384 channels at 18 x 18, batch 96, 21 us: neighbouring threads write neighbouring planes.
inline bool stream_result(int64_t bytes, int64_t plane_bytes) { return bytes >= kStreamBytes && plane_bytes % 64 == 0; }
constexpr int kKAlign = 256;         // the flattened (n,h,w) axis of a CNHW buffer is padded to this many bytes

inline int64_t round_up(int64_t v, int64_t m) { return (v + m - 1) / m * m; }
inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// Into how many parts to split the n steps of each of a launch's tiles, when a CU holds one workgroup at a time:
//     rounds over the CUs * max(steps of the longest part * t_step + t_fixed, t_floor) + (several parts: t_reduce + parts * t_part) .
// The count with the least of it, the smallest of equals, at most `limit`.
struct SplitModel {
    int64_t n, tiles, limit;
    double t_step, t_fixed, t_floor, t_reduce, t_part;
    double cost(int64_t s) const;
};
int cheapest_split(const SplitModel& m, int* tried = nullptr);

bool desc_valid(const daq_conv_desc* d);
bool plannable(const daq_conv_desc* d);   // valid, and of a size the kernels' indices hold
inline bool is_depthwise(const daq_conv_desc& d) { return d.groups > 1 && d.groups == d.Cin && d.groups == d.Cout; }

// ---- profiling hooks (prof.hip) ------------------------------------------------------------
bool prof_active();
void prof_push(const char* name, hipStream_t s);  // records the start event
void prof_pop(hipStream_t s);                     // records the stop event

// Launch helper: brackets the launch with profiling events when enabled and maps launch errors.
#define DAQ_LAUNCH(name, stream, ...)                          \
    do {                                                       \
        if (::daq::prof_active()) ::daq::prof_push(name, stream); \
        __VA_ARGS__;                                           \
        if (::daq::prof_active()) ::daq::prof_pop(stream);     \
        if (hipGetLastError() != hipSuccess) return DAQ_ERR_HIP; \
    } while (0)

// Dynamic LDS beyond 64 KiB has to be asked for, kernel by kernel and on every device; below that (48 KiB here: some kernels
// have a static part as well) the call would only cost host time, in launches that are often shorter than it takes to make them.
inline bool allow_lds(const void* kernel, size_t bytes) {
    return bytes <= 48 * 1024 || hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes) == hipSuccess;
}

// ---- predicated loads without control flow ------------------------------------------------
// A load guarded by an `if` becomes an exec-masked branch with a full memory wait at its join, and a
// select applied to the loaded value makes the compiler wait right behind the load; either way a
// software pipeline is serialised.  These helpers always issue the load and redirect a false
// predicate to 64 bytes of zeros in device memory, so nothing depends on the value until it is used.
static __device__ uint4 g_zero64[4];  // zero-initialised, never written (kept non-const so it shares the global address space)
__device__ __forceinline__ uint4 ld16_or_zero(const void* p, bool ok) {
    return *reinterpret_cast<const uint4*>(ok ? p : (const void*)g_zero64);
}
__device__ __forceinline__ float ldf_or_zero(const float* p, bool ok) {
    return *(ok ? p : reinterpret_cast<const float*>(g_zero64));
}

// ---- results that are fp32 or, on request, bfloat16 -------------------------------------------
// fp32 -> bfloat16 bits, round to nearest even (finite inputs)
__device__ __forceinline__ uint32_t bf16_bits(float f) {
    const uint32_t u = __float_as_uint(f);
    return (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
}
// Element `off` of a result tensor whose storage is fp32, or bfloat16 when `bf16` is set (uniform).
__device__ __forceinline__ void store_result(float* base, int64_t off, float v, int bf16) {
    if (bf16) reinterpret_cast<uint16_t*>(base)[off] = (uint16_t)bf16_bits(v);
    else base[off] = v;
}
// Four consecutive results starting at element `off`, a multiple of four: one 16-byte store, or one 8-byte store of
// four bfloat16; `nt` asks for a streaming store.
typedef float daq_v4f __attribute__((ext_vector_type(4)));
typedef uint32_t daq_v2u __attribute__((ext_vector_type(2)));
__device__ __forceinline__ void store_result4(float* base, int64_t off, float a, float b, float c, float d, int bf16, int nt) {
    if (bf16) {
        const daq_v2u w = {bf16_bits(a) | (bf16_bits(b) << 16), bf16_bits(c) | (bf16_bits(d) << 16)};
        daq_v2u* z = reinterpret_cast<daq_v2u*>(reinterpret_cast<uint16_t*>(base) + off);
        if (nt) __builtin_nontemporal_store(w, z);
        else *z = w;
    } else {
        const daq_v4f w = {a, b, c, d};
        daq_v4f* z = reinterpret_cast<daq_v4f*>(base + off);
        if (nt) __builtin_nontemporal_store(w, z);
        else *z = w;
    }
}

// ---- division by a launch-invariant divisor ---------------------------------------------------
// Exact unsigned division by an invariant divisor (Granlund-Montgomery round-up multiplier).
struct FastDiv {
    uint32_t mul;
    int32_t shift;
    int32_t one;
};
inline FastDiv make_fastdiv(uint32_t d) {
    FastDiv f{};
    f.one = (d == 1);
    int L = 0;
    while (((uint64_t)1 << L) < d) ++L;
    f.shift = L > 0 ? L - 1 : 0;
    f.mul = (uint32_t)((((uint64_t)1 << 32) * (((uint64_t)1 << L) - d)) / d + 1);
    return f;
}
__device__ __forceinline__ uint32_t fdiv(uint32_t x, const FastDiv& f) {
    const uint32_t t = __umulhi(x, f.mul);
    const uint32_t q = (t + ((x - t) >> 1)) >> f.shift;
    return f.one ? x : q;   // a select, not a branch: branches here split the prologues that call this many times
}

// ---- device-side view of an int8 layout ----------------------------------------------------
struct CnhwView {
    int64_t chan_pitch, plane_pitch, lead;
    int32_t img_rows, row_pitch;
    int32_t phases_h, phases_w, org_h, org_w;
    int32_t C, N, H, W;
    __host__ __device__ int64_t offset(int n, int c, int h, int w) const {
        const int hh = h + org_h, ww = w + org_w;
        const int ph = hh % phases_h, pw = ww % phases_w;
        return (int64_t)c * chan_pitch + (int64_t)(ph * phases_w + pw) * plane_pitch + lead +
               ((int64_t)n * img_rows + hh / phases_h) * row_pitch + ww / phases_w;
    }
};

struct NhwcView {
    int32_t c_pitch, C, N, H, W;
    __host__ __device__ int64_t offset(int n, int c, int h, int w) const {
        return (((int64_t)n * H + h) * W + w) * c_pitch + c;
    }
};

inline CnhwView cnhw_view(const daq_layout& L) {
    return CnhwView{L.chan_pitch, L.plane_pitch, L.lead, L.img_rows, L.row_pitch, L.phases_h, L.phases_w,
                    L.org_h, L.org_w, L.C, L.N, L.H, L.W};
}
inline NhwcView nhwc_view(const daq_layout& L) { return NhwcView{L.c_pitch, L.C, L.N, L.H, L.W}; }

// ---- kernels behind the entry points (one translation unit each) -----------------------------
// quantize.hip
size_t quantize_grad_ws_bytes(const daq_conv_desc& d);
size_t fwd_quant_ws_bytes(const daq_conv_desc& d);
daq_status quantize_activation_check(const daq_conv_desc& d, const float* X);   // host only: can this X be quantized?
// q(X) in both layouts and, with W, q(W): two launches.  From float kFwdWsFree on the workspace is the caller's.
constexpr int kFwdWsFree = 1000;
daq_status quantize_forward(const daq_conv_desc& d, const float* X, int8_t* qx_nhwc, int8_t* qx_cnhw, float* s_x, const float* W,
                            int8_t* qw_packed, float* s_w, void* ws, hipStream_t st, daq_schedule schedule);

// How the counting pass is dealt out.
constexpr int kCountWaves = 16;      // waves of the counting pass that a CU holds
constexpr int kCountMaxWaves = 12;   // of one workgroup
constexpr int kCountGroups = 1024;   // count partials of a channel, at most
struct CountPlan {
    int tiles;         // tiles of 16 units (64 pixels) of the flattened (n, h*w) axis
    int waves;         // of a workgroup
    int width;         // groups of 16 channels of a block, a wave each
    int blocks;        // blocks of channels
    int cgroups;       // workgroups of a block, and entries of part_cnt a channel has room for
    int cgroups_last;  // of the last block
    FastDiv div_cgroups;
    uint32_t by_groups[2];   // 2^16 over the groups of a full block, of the last one, rounded up: exact quotients below 768
    __host__ __device__ int workgroups() const { return (blocks - 1) * cgroups + cgroups_last; }
    // groups of 16 channels in block b of C channels; a workgroup with more waves than that takes several tiles at a time
    __host__ __device__ int groups(int C, int b) const { return b + 1 < blocks ? width : (C + 15) / 16 - (blocks - 1) * width; }
    // LDS of one of the two tiles a workgroup keeps: by pixel of a unit, unit and 16-byte share of the record, units an odd number of
    // 16 bytes apart and pixels 64 bytes more than 16 units: no bank conflicts either way
    __host__ __device__ static constexpr int pitch_dwords(int gb) { return 4 * (gb | 1); }
    __host__ __device__ static constexpr int step_dwords(int gb) { return 16 * pitch_dwords(gb) + 16; }
    static constexpr int block_dwords(int waves, int gb) { return gb == 1 ? 0 : waves / gb * 4 * step_dwords(gb); }
    static constexpr int most_tile_dwords(int waves) {
        int most = 0;
        for (int gb = 1; gb <= waves; ++gb) most = std::max(most, block_dwords(waves, gb));
        return most;
    }
    int tile_dwords(int C) const { return std::max(block_dwords(waves, groups(C, 0)), block_dwords(waves, groups(C, blocks - 1))); }
};
CountPlan plan_count(int C, int N, int HW, int given = 0, int held_given = 0);
// Waves of a workgroup of the forward quantizing launch, where its sweep writes both copies of X; w_blocks: its workgroups for the filter.
int forward_waves(int C, int N, int HW, int w_blocks);

// Channel-resident quantizer: `units` load units of a channel (four elements of a plane each, fewer at its end) on a workgroup of
// `waves` waves, `nu` units to a thread.
struct ResidentForm { int nu, waves; };
ResidentForm resident_form(int C, int64_t units);
bool resident_pays(int C, int64_t units, bool padded, bool tails, bool stochastic);   // tails: planes that are not whole units
bool resident_all_pays(int C, int64_t M, int64_t units);   // whether the launch also writes the global copy of C channels of M elements
// From how many elements on the counting sweep writes the per-channel copy too.  vector: elements of a row a thread of the packing launch
// loads at once, 0: rows of no whole vectors; channel_major: the global copy is (depthwise layers).
struct EarlyCase { bool given, nearest, padded, bf16, channel_major; int vector, W; };
int64_t early_copy_from(const EarlyCase& e);
int early_pack_blocks(int64_t channel_elems);   // workgroups a channel of the packing launch behind an early copy
bool fold_in_packing(int64_t workgroups);   // whether those of a channel-major packing launch fold its scale themselves

// clip_search.hip
size_t clip_search_ws_bytes(const daq_conv_desc& d);

// conv_generic.hip: direct kernels, any descriptor
daq_status conv_fwd_generic(const daq_conv_desc& d, const int8_t* qx_nhwc, const int8_t* qw, const float* s_x,
                            const float* s_w, float* Y, int32_t* acc, hipStream_t st);
// With `bf16` the result pointer of a gradient routine (dX, dW) is bfloat16 storage: same product, rounded to nearest even.
daq_status conv_bwd_data_generic(const daq_conv_desc& d, const int8_t* qg, const float* s_g, const int8_t* qw,
                                 const float* s_w, float* dX, int32_t* acc, hipStream_t st, bool bf16 = false);
daq_status conv_bwd_filter_generic(const daq_conv_desc& d, const int8_t* qx, const float* s_x, const int8_t* vq,
                                   const float* s_chan, float* dW, int32_t* acc, hipStream_t st, bool bf16 = false);

// conv_mfma_*.hip: int8 MFMA kernels; *_supported() says whether a descriptor is covered
bool bwd_filter_mfma_supported(const daq_conv_desc& d);
size_t bwd_filter_mfma_ws_bytes(const daq_conv_desc& d);
daq_status conv_bwd_filter_mfma(const daq_conv_desc& d, const int8_t* qx, const float* s_x, const int8_t* vq,
                                const float* s_chan, float* dW, int32_t* acc, void* ws, hipStream_t st, bool bf16 = false);
bool bwd_data_mfma_supported(const daq_conv_desc& d);
daq_status conv_bwd_data_mfma(const daq_conv_desc& d, const int8_t* qg, const float* s_g, const int8_t* qw,
                              const float* s_w, float* dX, int32_t* acc, hipStream_t st, bool bf16 = false);
bool fwd_mfma_supported(const daq_conv_desc& d);
daq_status conv_fwd_mfma(const daq_conv_desc& d, const int8_t* qx_nhwc, const int8_t* qw, const float* s_x,
                         const float* s_w, float* Y, int32_t* acc, hipStream_t st);


// conv_mfma_dw32.hip: 3 x 3 unit-stride filter gradient on the 32x32x32 MFMA, operands staged through LDS
// A 3-D layer is the 2-D problem of its frames, `depth` times over: depth tap kd pairs the gradient's frames with the
// activation's frames (kd * dD) / sD further on in depth-stride phase (kd * dD) % sD of the buffer.
struct DwDepth {
    int kD, dD, sD;
    int64_t x_chan_pitch, x_plane_pitch, x_depth_phase;
};
struct Plan32 {
    bool ok;              // these kernels serve the layer; an entry point makes its plan once and hands it on
    bool k11;             // 1 x 1 filter: the plain GEMM kernel
    bool s2;              // 3 x 3 filter at stride 2: four stride-phase planes per input channel
    int wm, wn, wk;       // tiles of a workgroup along co and ci; waves that share them: 1, or 8 (1 x 1: a K step each; 3 x 3: four multiply and four ask)
    int splits, tiles_m, tiles_n, nchunks, pb, b_units, ch;
    int splits_tail;      // K splits where the reduction can ride along in the next kernel (with `defer`)
    int bands_m, bands_n, band_m, band_n;   // rectangles of the tile grid per K split when there are 1, 2 or 4 splits (else 0)
    int64_t blocks;       // workgroups of the launch
    size_t lds_bytes;
    int64_t part_slots;   // int32 entries of one split's partial tiles
};
// depth: depth taps of a 3-D layer (its frames are the images of `d`); the launch has that many times the tiles
Plan32 make_plan32(const daq_conv_desc& d, int depth = 1);
bool dw11_long(int64_t chunks);   // 1 x 1: whether a workgroup of so many chunks addresses its requests by vector instructions
size_t bwd_filter_lds_ws_bytes(const Plan32& pl, int depth = 1);
int64_t bwd_filter_lds_row_bytes(const Plan32& pl);   // read of an activation row, from its start on
// With `defer`, a K-split launch leaves its last stage (sum of the partial tiles, de-quantization) undone and
// describes it in *defer (blocks == 0: nothing is left) for a later kernel's extra workgroups, see dw_tail.h.
struct DwTail;
daq_status conv_bwd_filter_lds(const daq_conv_desc& d, const Plan32& plan, const int8_t* qx, const float* s_x, const int8_t* vq,
                               const float* s_chan, float* dW, int32_t* acc, void* ws, hipStream_t st,
                               DwTail* defer = nullptr, bool bf16 = false, const DwDepth* dp = nullptr);

// conv_mfma_halo.hip: halo-tile form of the channel-contracting kernel (unit stride; stride 2 for the data gradient)
bool bwd_data_halo_supported(const daq_conv_desc& d);
// With `tail` (blocks > 0), extra workgroups of the launch finish a deferred filter gradient.
// With `bf16`, dX points to bfloat16 storage (2 bytes per element) and receives the result rounded to nearest even.
daq_status conv_bwd_data_halo(const daq_conv_desc& d, const int8_t* qg, const float* s_g, const int8_t* qw,
                              const float* s_w, float* dX, int32_t* acc, hipStream_t st, const DwTail* tail = nullptr,
                              bool bf16 = false);
// Both gradients of a small layer in one launch (and a reduction, if the filter gradient is split); false: the layer has no
// such form, and nothing was launched.
bool conv_bwd_both_small(const daq_conv_desc& d, const Plan32& plan_w, const int8_t* qx, const float* s_x, const int8_t* vq, const float* s_chan, float* dW,
                         int32_t* dW_acc, const int8_t* qg, const float* s_g, const int8_t* qw, const float* s_w, float* dX, int32_t* dX_acc,
                         void* ws, hipStream_t st, daq_status& rc);
bool fwd_halo_supported(const daq_conv_desc& d);
daq_status conv_fwd_halo(const daq_conv_desc& d, const int8_t* qx_nhwc, const int8_t* qw, const float* s_x,
                         const float* s_w, float* Y, int32_t* acc, hipStream_t st);
// 3-D layers on the same kernel.  The workspace holds the filter in fragment order; 0 bytes: the layer stays on the kernels of conv3d.hip.
size_t conv3d_halo_ws_bytes(bool backward, const daq_conv3d_desc& d);
daq_status conv3d_bwd_data_halo(const daq_conv3d_desc& d, const int8_t* qg, const float* s_g, const int8_t* w_bwd, const float* s_w, float* dX,
                                int32_t* acc, void* frag, hipStream_t st);
daq_status conv3d_fwd_halo(const daq_conv3d_desc& d, const int8_t* qx, const int8_t* w_fwd, const float* s_x, const float* s_w, float* Y,
                           int32_t* acc, void* frag, hipStream_t st);

// conv_mfma_halo.hip, 1 x 1 products on 128-pixel tiles: whether their workgroups go row tile after row tile
bool tiles_by_rows(int TH, int TW, int tiles_h, int tiles_w, int stride, int Hd, int Wd, int bytes, int64_t tiles, int row_tiles);
// of 256-pixel tiles at unit stride: whether an XCD has every eighth tile instead of an eighth of them
bool tiles_spread(int TH, int TW, int tiles_h, int tiles_w, int Hd, int Wd, int bytes, int64_t tiles, int row_tiles);
bool wide_waves(int64_t blocks, int chunks, int taps);   // a run-time tap list: waves of 32 rows x 128 pixels instead of 64 x 64
bool wide_waves1(int64_t blocks, int stride, int Wd);           // the same of 1 x 1 filters
// streaming 1 x 1 products: blocks that an XCD takes in a row, 0: one by one
int64_t stream_deal(int64_t out_bytes, int64_t plane_bytes, int cp, int pairs, int64_t blocks);

// conv_mfma_direct.hip: the same products for layers of few tiles, operands straight from global memory.  `other` is what would serve
// the layer otherwise, with its workgroups and the steps (tap x 64 channels) of each; false: that is the faster one by the two's cost
// models, or these kernels do not serve the layer, and nothing was launched.
struct DwTail;
enum class TileForm { kTaps9, kNarrow, kTaps, kRing1, kNhwc };
struct OtherKernel {
    TileForm form;
    bool classes;      // a strided data gradient, by parity class
    int64_t blocks;
    int steps;
};
OtherKernel fwd_nhwc_as_other(const daq_conv_desc& d);   // conv_mfma_nhwc.hip
int direct_waves(bool backward, const daq_conv_desc& d, const OtherKernel& other, bool bf16);   // waves to a tile, 0: `other` is the faster
int product_direct_waves(bool backward, const daq_conv_desc& d, bool bf16);   // conv_mfma_halo.hip: the same with what would serve the product
bool conv_direct(bool backward, const daq_conv_desc& d, const OtherKernel& other, const int8_t* src, const int8_t* qw, const float* s_a,
                 const float* s_b, float* out, int32_t* acc, hipStream_t st, const DwTail* tail, bool bf16, daq_status& rc);

// conv_depthwise.hip: groups == channels, both operands channel-major
bool depthwise_dx_supported(const daq_conv_desc& d);
daq_status conv_bwd_data_depthwise(const daq_conv_desc& d, const int8_t* qg, const float* s_g, const int8_t* qw,
                                   const float* s_w, float* dX, int32_t* acc, hipStream_t st, bool per_channel = false,
                                   bool bf16 = false);
bool depthwise_fwd_supported(const daq_conv_desc& d);
daq_status conv_fwd_depthwise(const daq_conv_desc& d, const int8_t* qx_cnhw, const int8_t* qw, const float* s_x,
                              const float* s_w, float* Y, int32_t* acc, hipStream_t st);
bool depthwise_dw_supported(const daq_conv_desc& d);
size_t depthwise_dw_ws_bytes(const daq_conv_desc& d);

// layout.hip: workspace of a filter gradient (a multiple of 256), `pl` being its make_plan32
size_t bwd_filter_ws_bytes(const daq_conv_desc& d, const Plan32& pl);
daq_status conv_bwd_filter_depthwise(const daq_conv_desc& d, const int8_t* qx, const float* s_x, const int8_t* vq,
                                     const float* s_chan, float* dW, int32_t* acc, void* ws, hipStream_t st, bool bf16 = false);

}  // namespace daq
