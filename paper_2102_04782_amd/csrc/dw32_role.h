// Device code of the filter gradient for 3 x 3 (dw32_role) and 1 x 1 (dw11_role) filters, see conv_mfma_dw32.hip: what a
// workgroup of the launch does, as functions, so that a launch can hold other work beside it.
#pragma once

#include <type_traits>

#include "daq_internal.h"
#include "dw_tail.h"

namespace daq {

struct Dw32Args {
    const int8_t* g;      // vq, [Cout][klen]
    const int8_t* x;      // q(X'), [Cin][x_chan_pitch]
    int64_t klen;
    int64_t x_chan_pitch;
    int64_t x_plane_pitch;   // stride 2: bytes of one stride-phase plane of an activation channel
    int Cout, Cin;
    int row_pitch;
    int pb;               // LDS pitch of an activation row in bytes (a multiple of 4 with pb/4 odd; dw32_role)
    int b_units;          // 16-byte units of an activation row that are staged per chunk
    int nchunks, splits;
    int bands_m, bands_n;  // > 0: fewer than eight K splits, the tile grid is cut into bands_m x bands_n rectangles (dw_block_map)
    int band_m, band_n;    // tiles per rectangle along co and ci
    int tiles_n, tiles_m;
    int32_t* part;        // splits > 1: [tile][split][wave tile][slot = tap*16 + reg][lane]
    const float* s_x;
    const float* s_chan;
    float* dW;
    int32_t* acc_out;
    int bf16;             // dW is bfloat16 storage
    // 3-D layers: depth tap kd = blockIdx.y is the same product against the activation's frames kd * dD further on (all
    // 0 / taps / 0 for a 2-D layer, whose grid has one row)
    int dD, sD, taps_all;
    int64_t x_frame, x_depth_phase;   // bytes from a frame to the next, and from a depth-stride phase to the next
    int64_t part_kd;                  // int32 entries of the partial tiles of one depth tap
};

// A filter gradient of at most max_blocks workgroups to run beside other work of about other_us in one launch: false where
// the layer has no such form or is faster in launches of its own (false also leaves everything untouched).  tail.blocks > 0: launch_dw_reduce has to follow.
struct DwBeside {
    Dw32Args a;
    bool k11;            // dw11_role<1, 1, 8, 3, 1, true>; otherwise dw32_ring_role<false>
    int blocks;
    size_t lds_bytes;
    DwTail tail;
};
bool bwd_filter_beside(const daq_conv_desc& d, Plan32 pl, const int8_t* qx, const float* s_x, const int8_t* vq, const float* s_chan, float* dW,
                       int32_t* acc, void* ws, int max_blocks, double other_us, bool other_streams, DwBeside& out);
double beside_data_us(bool nine_taps, int chunks);   // conv_mfma_halo.hip: time of the data gradient's part of that launch

namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef int v2i __attribute__((ext_vector_type(2)));
typedef int v4i_a4 __attribute__((ext_vector_type(4), aligned(4)));
typedef int v2i_a4 __attribute__((ext_vector_type(2), aligned(4)));

constexpr int kKC = 256;        // K bytes staged per chunk (8 MFMA K-steps of 32)
constexpr int kPA = kKC + 16;   // LDS pitch of a gradient row: 16-byte aligned, rotates banks between rows
constexpr int kT = 9;

// 16 bytes of every lane to 64 consecutive slots of LDS from `dst` on (lane l: slot l), without registers in between, the address being a
// descriptor's base, a constant of the lane and a scalar.  A request so takes no vector instruction, which
// matters beside matrix instructions (a CU whose other waves multiply, 960 requests of 1 KiB: 12.9 us of the 19.2 that the multiplies take;
// with an addition for each address none before the multiplies were through).  kNoByte: no address, the lane's slot is cleared.
constexpr uint32_t kNoByte = 0xFFFFFFF0u;
__device__ __forceinline__ __amdgpu_buffer_rsrc_t tile_rsrc(const int8_t* base) {
    return __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, (int)0xFFFFFF00u, 0x00020000);
}
__device__ __forceinline__ void load_to_lds(__amdgpu_buffer_rsrc_t src, uint32_t lane_off, uint32_t off, int8_t* dst) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(src, (__attribute__((address_space(3))) void*)dst, 16, (int)lane_off, (int)off, 0, 0);
}

// The launch's share for depth tap blockIdx.y: where it reads the activation and where it leaves its results.
__device__ __forceinline__ void dw_depth(Dw32Args& p, int taps) {
    const int kd = blockIdx.y;
    if (kd == 0) return;
    p.x += (int64_t)((kd * p.dD) % p.sD) * p.x_depth_phase + (int64_t)((kd * p.dD) / p.sD) * p.x_frame;
    p.part += kd * p.part_kd;
    p.dW += kd * taps;   // (3-D results are fp32)
    if (p.acc_out) p.acc_out += kd * taps;
}

// f(0), f(1), ... f(N - 1) with constant arguments.
template <int N, int I = 0, typename F>
__device__ __forceinline__ void ring_round(F f) {
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        ring_round<N, I + 1>(f);
    }
}

__device__ __forceinline__ int alignbyte(int hi, int lo, int sh) {
    return (int)__builtin_amdgcn_alignbyte((unsigned)hi, (unsigned)lo, (unsigned)sh);
}

// The 16 bytes from byte S of a row of dwords on.
template <int S, int N>
__device__ __forceinline__ v4i window_at(const int (&d)[N]) {
    constexpr int j = S >> 2, sh = S & 3;
    if constexpr (sh == 0) return v4i{d[j], d[j + 1], d[j + 2], d[j + 3]};
    else
        return v4i{alignbyte(d[j + 1], d[j], sh), alignbyte(d[j + 2], d[j + 1], sh), alignbyte(d[j + 3], d[j + 2], sh),
                   alignbyte(d[j + 4], d[j + 3], sh)};
}

// Workgroup b of the product -> (K split, output tile).  It runs on XCD b % 8, and what an XCD's workgroups read together is what
// its L2 has to fetch.  With eight or more splits an XCD takes whole splits: every tile of the split, i.e. one K slice
// of every operand row - each byte of the operands enters exactly one L2.  With 1, 2 or 4 splits the eight XCDs share a
// split among 8, 4 or 2 of them, and each takes a rectangle of the tile grid (bands_m x bands_n rectangles per split,
// chosen on the host to minimise rows of G plus rows of X per rectangle) instead of tiles dealt round-robin, which
// made every XCD read nearly all rows of one operand.  Returns false for the padding of the grid.
__device__ __forceinline__ bool dw_block_map(const Dw32Args& p, const int b, int& split, int& tile) {
    const int tiles = p.tiles_n * p.tiles_m;
    const int x = b % kXcd, q = b / kXcd;
    if (p.bands_m > 0) {
        split = x % p.splits;
        const int rect = x / p.splits;
        const int rm = rect / p.bands_n, rn = rect % p.bands_n;
        const int lm = q / p.band_n, ln = q % p.band_n;
        const int tm = rm * p.band_m + lm, tn = rn * p.band_n + ln;
        if (lm >= p.band_m || tm >= p.tiles_m || tn >= p.tiles_n) return false;
        tile = tm * p.tiles_n + tn;
        return true;
    }
    const int full = (p.splits / kXcd) * kXcd;
    if (q < (full / kXcd) * tiles) {
        split = (q / tiles) * kXcd + x;
        tile = q % tiles;
    } else {
        const int rb = b - full * tiles;
        split = full + rb % (p.splits - full);
        tile = rb / (p.splits - full);
    }
    return true;
}

// WQ4 = row_pitch mod 4.  Four waves, a tile each: 64 x 64 results per workgroup, for layers with enough of them to fill the chip.
// The loads of the next chunk but one are in flight while a chunk is multiplied (register ring of one set).
template <int WQ4>
__device__ __forceinline__ void dw32_role(Dw32Args& p, const int bid) {
    constexpr int WN = 2, NT = 256;
    constexpr int BM = 64, BN = 64;
    constexpr int A_PER_T = BM * (kKC / 16) / NT;    // 16-byte units of the gradient tile per thread
    constexpr int A_BYTES = BM * kPA;
    constexpr int B_MAX = 4 * WN * 256 / NT;  // 16-byte units of the activation tile per thread, at most
    extern __shared__ __align__(16) int8_t lds[];

    dw_depth(p, kT);
    const int tid = threadIdx.x, lane = tid % kWave;
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int wn = wave % WN, wm = wave / WN;
    const int l32 = lane & 31, lh = lane >> 5;
    const int STAGE = A_BYTES + BN * p.pb;

    int split, tile;
    if (!dw_block_map(p, bid, split, tile)) return;   // uniform
    const int tn = tile % p.tiles_n, tm = tile / p.tiles_n;
    const int co0 = tm * BM, ci0 = tn * BN;
    const int per = p.nchunks / p.splits, rem = p.nchunks % p.splits;
    const int c_begin = split * per + min(split, rem);
    const int c_end = c_begin + per + (split < rem ? 1 : 0);
    const float sx = *p.s_x / 127.0f;

    // ---- staging assignment ----
    // gradient: unit u = tid + 256*i -> row u / 16, 16-byte column u % 16
    uint32_t a_src[A_PER_T];
    int a_dst[A_PER_T];
#pragma unroll
    for (int i = 0; i < A_PER_T; ++i) {
        const int u = tid + NT * i;
        const int row = u >> 4, c16 = u & 15;
        const int co = co0 + row;
        a_src[i] = (uint32_t)((int64_t)(co < p.Cout ? co : 0) * p.klen + 16 * c16);   // rows past Cout recompute row 0, never stored
        a_dst[i] = row * kPA + 16 * c16;
    }
    // activation: unit u = tid + 256*i of the BN x b_units tile (row-major): consecutive lanes, consecutive 16 bytes
    uint32_t b_src[B_MAX];
    int b_dst[B_MAX];
    const int b_total = BN * p.b_units;
#pragma unroll
    for (int i = 0; i < B_MAX; ++i) {
        const int u = tid + NT * i;
        const int uc = u < b_total ? u : 0;
        const int row = uc / p.b_units, col = uc - row * p.b_units;
        const int ci = ci0 + row;
        b_src[i] = (uint32_t)((int64_t)(ci < p.Cin ? ci : 0) * p.x_chan_pitch + 16 * col);
        b_dst[i] = u < b_total ? A_BYTES + row * p.pb + 16 * col : -1;
    }
    // Every call issues the same loads (past the end the last chunk is fetched again, which the caches absorb):
    // only then can the compiler count the loads in flight and wait for exactly the oldest set.
    v4i ra[A_PER_T], rb[B_MAX];
    const int c_last = max(c_end - 1, 0);
    auto load_chunk = [&](int chunk) {
        const int64_t k0 = (int64_t)min(chunk, c_last) * kKC;
        const int8_t* gk = p.g + k0;
        const int8_t* xk = p.x + k0;
#pragma unroll
        for (int i = 0; i < A_PER_T; ++i) ra[i] = *reinterpret_cast<const v4i*>(gk + a_src[i]);
#pragma unroll
        for (int i = 0; i < B_MAX; ++i) rb[i] = *reinterpret_cast<const v4i*>(xk + b_src[i]);
        __builtin_amdgcn_sched_barrier(0);   // keep the sets in program order
    };
    auto store_chunk = [&](int buf) {
        int8_t* base = lds + buf * STAGE;
#pragma unroll
        for (int i = 0; i < A_PER_T; ++i) *reinterpret_cast<v4i*>(base + a_dst[i]) = ra[i];
#pragma unroll
        for (int i = 0; i < B_MAX; ++i)
            if (b_dst[i] >= 0) *reinterpret_cast<v4i_a4*>(base + b_dst[i]) = rb[i];   // rows are only dword aligned
    };

    v16i acc[kT];
#pragma unroll
    for (int t = 0; t < kT; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[t][r] = 0;

    load_chunk(c_begin);
    store_chunk(0);
    load_chunk(c_begin + 1);
    __syncthreads();

    const int arow = (wm * 32 + l32) * kPA + 16 * lh;
    const int brow = A_BYTES + (wn * 32 + l32) * p.pb + 16 * lh;
    for (int chunk = c_begin; chunk < c_end; ++chunk) {
        const int buf = (chunk - c_begin) & 1;
        const int8_t* A = lds + buf * STAGE + arow;
        const int8_t* B = lds + buf * STAGE + brow;
        // All LDS reads of this wave's K steps are issued before the first multiply: with one wave per SIMD nothing
        // else hides their latency.
        constexpr int KS = kKC / 32;
        v4i fa[KS];
        int fd[KS][3][6];
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            fa[ks] = *reinterpret_cast<const v4i*>(A + 32 * ks);
#pragma unroll
            for (int kh = 0; kh < 3; ++kh) {
                // 24 bytes from the dword at or below this filter row's first window
                const int8_t* src = B + 32 * ks + ((kh * p.row_pitch) & ~3);
                const v4i_a4 lo = *reinterpret_cast<const v4i_a4*>(src);
                const v2i_a4 hi = *reinterpret_cast<const v2i_a4*>(src + 16);
                fd[ks][kh][0] = lo[0]; fd[ks][kh][1] = lo[1]; fd[ks][kh][2] = lo[2]; fd[ks][kh][3] = lo[3];
                fd[ks][kh][4] = hi[0]; fd[ks][kh][5] = hi[1];
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        ring_round<KS>([&](auto ks) {
            ring_round<3>([&](auto kh) {
                ring_round<3>([&](auto kw) {
                    constexpr int s = ((decltype(kh)::value * WQ4) & 3) + decltype(kw)::value;
                    acc[kh * 3 + kw] =
                        __builtin_amdgcn_mfma_i32_32x32x32_i8(fa[ks], window_at<s>(fd[ks][kh]), acc[kh * 3 + kw], 0, 0, 0);
                });
            });
        });
        // chunk+1 goes to the other LDS buffer, chunk+2 on its way
        store_chunk(buf ^ 1);
        load_chunk(chunk + 2);
        __syncthreads();
    }

    // register r of a 32 x 32 tile: row (co) 8*(r/4) + 4*lh + r%4, column (ci) l32
    const int ci = ci0 + wn * 32 + l32;
    if (ci >= p.Cin) return;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int co = co0 + wm * 32 + 8 * (r >> 2) + 4 * lh + (r & 3);
        if (co < p.Cout) {
            const int64_t off = ((int64_t)co * p.Cin + ci) * p.taps_all;
            const float sc = sx * (p.s_chan[co] / 127.0f);
#pragma unroll
            for (int t = 0; t < kT; ++t) {
                store_result(p.dW, off + t, (float)acc[t][r] * sc, p.bf16);
                if (p.acc_out) p.acc_out[off + t] = acc[t][r];
            }
        }
    }
}

// One 32 x 32 x 9 tile to a workgroup.  Waves 0 to 3, one to a SIMD, take two of the eight K steps of every chunk each (combined through LDS
// at the end); waves 4 to 7 ask for the operands, which go from global memory straight into LDS: D stage buffers, one barrier per chunk.
//
// S2: the same product for a 3 x 3 filter at stride 2.  The activation is stored as its four stride-phase planes
// (row parity, column parity), each with the gradient's slot geometry, so tap (kh, kw) pairs gradient byte f with byte
// f + (kh/2)*row_pitch + kw/2 of plane (kh%2, kw%2): still shifted correlations over the flat axis, now against four
// staged rows per input channel.  Six windows per K step - one per (plane, row shift) - serve the nine taps.
//
// What bounds it: 18 multiplies a wave and chunk, 576 cycles, of which a chunk takes about 790, the rest being what reads of LDS
// (fourteen a wave) cost a wave that multiplies, the barrier and the loop.  128 x 512 -> 512 at 7 x 7, 33 chunks on 256 workgroups: 1.6 us to the first
// operands, 15 for the chunks at the 1.75 GHz that the chip holds under this load, 2 to combine and 1 to store, 19.6 us in the kernel (1.13 times the
// speed over 109 drawn layers, 1.11 at stride 2) where eight waves with a K step each took 1 us more, 17.6, 3 and 2.4.
//   Vector instructions of a wave wait behind the matrix instructions of another on its SIMD, and a request behind the
//   addition for its address: asked for by multiplying waves, or with vector addresses, requests and multiplies took turns (910 to 1020 cycles a chunk; the requests
//   alone 380).  Hence waves that only ask, with scalar addresses and the higher priority, and one multiplying wave to a SIMD.
//   The columns of a filter row differ by a byte in f, and it is the gradient that is shifted by it (G[f - kw] X[f + kh row_pitch] instead of
//   G[f] X[f + kh row_pitch + kw]): two shifted fragments serve all rows, 47 instead of 71 vector instructions a chunk.
//
// Only aligned 16-byte reads are fast (the reads of a chunk by eight waves: 145 ns in dwords, 110 to 130 in aligned pieces, 300 to 1300
// in unaligned ones), so a window is the one or two pieces it lies in, and its place in them, Q = row shift mod 16, is a constant of the
// loop: sixteen of them, chosen once.  Slot column c of row r holds the row's piece c ^ (r % 16) (the four last columns of the strided
// form's rows of twenty c ^ (r % 4)), so that the lanes of a read fall into different banks.
template <bool S2>
struct Ring32 {
    static constexpr int PL = S2 ? 4 : 1;              // staged rows per input channel
    static constexpr int UP = S2 ? 20 : 32;            // 16-byte slots of a staged activation row
    static constexpr int D = S2 ? 3 : 6;               // stage buffers
    static constexpr int NEXT = S2 ? D : D - 1;        // chunks asked for ahead of the present one
    // requests of an asking wave for a chunk: of the gradient's pieces, of the activation's, and one (eight lanes) of the gradient's before
    static constexpr int AREQ = 2, XREQ = PL * 32 * UP / 256, REQ = AREQ + XREQ + 1;
    static constexpr int BEFORE = 32 * kKC, A_BYTES = BEFORE + 32 * 16, ROW = 16 * UP, STAGE = A_BYTES + PL * 32 * ROW;
    static constexpr int LDS = D * STAGE;
    __host__ __device__ static constexpr int slot_of(int col, int row) {
        return S2 && col >= 16 ? 16 + ((col - 16) ^ (row & 3)) : (col & 16) | ((col & 15) ^ (row & 15));
    }
    // Windows of a K step: shift in rows, staged plane; first tap, the step to the next one, which takes the gradient a byte later, and how many.
    //   unit stride: a filter row each; stride 2: planes (even, even), both shifts, (even, odd), both, (odd, even), (odd, odd)
    static constexpr int WINDOWS = S2 ? 6 : 3;
    struct Window { int shift, plane, tap, step, taps; };
    __host__ __device__ static constexpr Window window(int w) {
        constexpr Window unit[3] = {{0, 0, 0, 1, 3}, {1, 0, 3, 1, 3}, {2, 0, 6, 1, 3}};
        constexpr Window strided[6] = {{0, 0, 0, 2, 2}, {1, 0, 6, 2, 2}, {0, 1, 1, 2, 1}, {1, 1, 7, 2, 1}, {0, 2, 3, 2, 2}, {0, 3, 4, 2, 1}};
        return S2 ? strided[w] : unit[w % 3];
    }
    __host__ __device__ static constexpr int window_of(int m) { int w = 0; while (m >= window(w).taps) m -= window(w++).taps; return w; }   // of multiply m
    __host__ __device__ static constexpr int column_of(int m) { int w = 0; while (m >= window(w).taps) m -= window(w++).taps; return m; }
};
// Row pitches it serves (slot column UP - 1, with which the last window of a chunk may end, is reached at 63 and 127 only; longer rows than these
// have always gone to the tap-table kernel, and were not timed here), and the slots of a row that are filled.
template <bool S2>
constexpr int ring32_max_pitch() { return S2 ? 54 : 123; }
inline int ring32_units(bool s2, int row_pitch) { return 16 + (s2 ? row_pitch : 2 * row_pitch) / 16 + 1; }

// Dwords FROM .. FROM + COUNT - 1 of the piece at `at` into the same places of d (three of them with the fourth).
template <int FROM, int COUNT>
__device__ __forceinline__ void read_piece(const int8_t* at, int* d) {
    static_assert(FROM + COUNT == 4 || FROM == 0, "the end or the beginning of a piece");
    if constexpr (COUNT == 1) {
        d[FROM] = *reinterpret_cast<const int*>(at + 4 * FROM);
    } else if constexpr (COUNT == 2) {
        const v2i v = *reinterpret_cast<const v2i*>(at + 4 * FROM);
        d[FROM] = v[0]; d[FROM + 1] = v[1];
    } else {
        const v4i v = *reinterpret_cast<const v4i*>(at);
#pragma unroll
        for (int i = 0; i < 4; ++i) d[i] = v[i];
    }
}
// Piece K of the one or two that bytes Q .. Q + 15 lie in, dword by dword.
template <int Q, int K>
__device__ __forceinline__ void read_window(const int8_t* at, int (&d)[8]) {
    constexpr int first = Q / 4, last = (Q + 15) / 4;
    if constexpr (K == 0) read_piece<first, 4 - first>(at, d);
    else if constexpr (last >= 4) read_piece<0, last - 3>(at, d + 4);
}
// The window itself.  The fourth dword of a piece of which three are used counts as used here as well (otherwise its register is given to
// a later read of the same batch, which then waits for the whole batch before it), and whole dwords of two pieces are put together here, by a
// shift of no bytes (plain copies the compiler makes where they are read, and waits there; moves in inline assembly it does not see: a matrix
// instruction may read a register no sooner than two wait states after a vector instruction wrote it, and the compiler counts those only
// from instructions that it knows).
template <int Q>
__device__ __forceinline__ v4i window(const int (&d)[8]) {
    if constexpr (Q / 4 == 1) asm volatile("" ::"v"(d[0]));
    if constexpr ((Q + 15) / 4 == 6) asm volatile("" ::"v"(d[7]));
    if constexpr (Q % 4 == 0 && Q != 0) {
        constexpr int j = Q / 4;
        return v4i{alignbyte(d[j], d[j], 0), alignbyte(d[j + 1], d[j + 1], 0), alignbyte(d[j + 2], d[j + 2], 0), alignbyte(d[j + 3], d[j + 3], 0)};
    } else {
        return window_at<Q>(d);
    }
}

// The K loop of a multiplying wave over n chunks.
template <bool S2, int Q>
__device__ __forceinline__ void ring32_loop(const int n, const int kq, const int l32, const int lh, const int row_pitch, v16i (&acc)[kT]) {
    using R = Ring32<S2>;
    extern __shared__ __align__(16) int8_t lds[];
    int at_g[2], at_before[2], at_x[2][3][2];   // by K step; by row shift and piece
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int u = 2 * (kq + 4 * i) + lh;
        at_g[i] = l32 * kKC + 16 * (u ^ (l32 & 15));
        at_before[i] = (u == 0 ? R::BEFORE + 16 * l32 : l32 * kKC + 16 * ((u - 1) ^ (l32 & 15))) + 12;
#pragma unroll
        for (int s = 0; s < 3; ++s)
#pragma unroll
            for (int k = 0; k < 2; ++k) at_x[i][s][k] = R::A_BYTES + l32 * R::ROW + 16 * R::slot_of(u + k + s * row_pitch / 16, l32);
    }
    struct Raw {
        int before;   // the four bytes before g
        v4i g;
        int x[R::WINDOWS][8];
    };
    // read k of K step I: the gradient, then the windows, two pieces each at most
    constexpr int READS = 2 + 2 * R::WINDOWS;
    auto read = [&](Raw& r, const int8_t* S, auto I, auto k) {
        if constexpr (k == 0) r.g = *reinterpret_cast<const v4i*>(S + at_g[I]);
        else if constexpr (k == 1) r.before = *reinterpret_cast<const int*>(S + at_before[I]);
        else {
            constexpr int w = (k - 2) / 2;
            constexpr auto win = R::window(w);
            read_window<win.shift * Q % 16, k % 2>(S + win.plane * 32 * R::ROW + at_x[I][win.shift][k % 2], r.x[w]);
        }
    };
    v4i g[3], x;   // the gradient's bytes, and those one and two before; the window
    auto mul = [&](const Raw& r, auto m) {
        constexpr int w = R::window_of(m), c = R::column_of(m);
        constexpr auto win = R::window(w);
        if constexpr (m == 0) g[0] = r.g;
        if constexpr (w == 0 && c > 0) {
            const int d[5] = {r.before, r.g[0], r.g[1], r.g[2], r.g[3]};
            g[c] = window_at<4 - c>(d);
        }
        if constexpr (c == 0) x = window<win.shift * Q % 16>(r.x[w]);
        acc[win.tap + c * win.step] = __builtin_amdgcn_mfma_i32_32x32x32_i8(g[c], x, acc[win.tap + c * win.step], 0, 0, 0);
    };
    // Multiplies the K step in `now` and reads step I of the chunk at S into `next`, the reads one by one between the multiplies: in a
    // row they wait for one another, and the multiplies behind them with them.
    auto half = [&](const Raw& now, Raw& next, const int8_t* S, auto I) {
        ring_round<kT>([&](auto m) {
            __builtin_amdgcn_sched_barrier(0);
            mul(now, m);
            ring_round<READS>([&](auto k) {
                if constexpr (k * (kT - 1) / READS == m) read(next, S, I, k);
            });
        });
        __builtin_amdgcn_sched_barrier(0);
    };
    constexpr std::integral_constant<int, 0> first;
    constexpr std::integral_constant<int, 1> second;

    Raw r0, r1;
    __builtin_amdgcn_s_barrier();           // chunk 0 has landed
    ring_round<READS>([&](auto k) { read(r0, lds, first, k); });
    for (int i = 0, buf = 0; i < n; ++i) {
        half(r0, r1, lds + buf * R::STAGE, second);
        if constexpr (S2) asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // chunk i is read out, its place is the next to be taken
        __builtin_amdgcn_s_barrier();       // chunk i + 1 has landed
        buf = buf + 1 == R::D ? 0 : buf + 1;
        half(r1, r0, lds + buf * R::STAGE, first);
    }
}

template <bool S2>
__device__ __forceinline__ void dw32_ring_role(Dw32Args& p, const int bid) {
    using R = Ring32<S2>;
    extern __shared__ __align__(16) int8_t lds[];
    __shared__ float l_scale[32];

    dw_depth(p, kT);
    const int tid = threadIdx.x, lane = tid % kWave;
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int l32 = lane & 31, lh = lane >> 5;

    int split, tile;
    if (!dw_block_map(p, bid, split, tile)) return;   // uniform
    const int tn = tile % p.tiles_n, tm = tile / p.tiles_n;
    const int co0 = tm * 32, ci0 = tn * 32;
    const int per = p.nchunks / p.splits, rem = p.nchunks % p.splits;
    const int c_begin = split * per + min(split, rem);
    const int n = per + (split < rem ? 1 : 0);

    v16i acc[kT];
    if (wave >= 4) {   // uniform: asks
        __builtin_amdgcn_s_setprio(3);
        // piece by piece of the stacked slots, the gradient's [32][16] and the activation's [32 * PL][UP], 64 at a time
        const __amdgpu_buffer_rsrc_t rs_g = tile_rsrc(p.g + (int64_t)co0 * p.klen), rs_x = tile_rsrc(p.x + (int64_t)ci0 * p.x_chan_pitch);
        uint32_t from[R::REQ];
#pragma unroll
        for (int j = 0; j < R::REQ; ++j) {
            const int u = (j * 4 + wave - 4) * 64 + lane;
            if (j == R::REQ - 1) {   // the pieces before the chunk
                const int row = 8 * (wave - 4) + lane;
                from[j] = (uint32_t)((int64_t)(co0 + row < p.Cout ? row : 0) * p.klen);   // (of the first eight lanes)
            } else if (j < R::AREQ) {   // rows past Cout / Cin recompute the first one and are never stored
                const int row = u >> 4;
                from[j] = (uint32_t)((int64_t)(co0 + row < p.Cout ? row : 0) * p.klen + 16 * ((u & 15) ^ (row & 15)));
            } else {
                const int row = (u - 512) / R::UP, slot = (u - 512) - row * R::UP;   // staged row = plane * 32 + channel of the tile
                const int col = R::slot_of(slot, row), ci = row % 32;                // (its own inverse)
                from[j] = (uint32_t)((int64_t)(ci0 + ci < p.Cin ? ci : 0) * p.x_chan_pitch + (int64_t)(row / 32) * p.x_plane_pitch + 16 * col);
                if (col >= p.b_units) from[j] = kNoByte;
            }
        }
        // a chunk is REQ requests a wave (past the end the last chunk again, into a buffer nobody reads), so that the
        // count of outstanding requests in the waits is a constant
        auto ask = [&](int i, int buf) {
            const uint32_t k0 = (uint32_t)(c_begin + min(i, n - 1)) * (uint32_t)kKC;
            int8_t* const stage = lds + buf * R::STAGE;
            ring_round<R::AREQ>([&](auto j) { load_to_lds(rs_g, from[j], k0, stage + 1024 * (j * 4 + wave - 4)); });
            // (a plane begins with zeros: they stand for what is before its first byte)
            if (lane < 8) load_to_lds(rs_g, from[R::REQ - 1], k0 == 0 ? 0u : k0 - 16u, stage + R::BEFORE + 128 * (wave - 4));
            ring_round<R::XREQ>([&](auto j) {
                load_to_lds(rs_x, from[R::AREQ + j], k0, stage + R::A_BYTES + 1024 * (j * 4 + wave - 4));
            });
        };
        ask(0, 0);
        ask(1, 1);
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(R::REQ) : "memory");   // chunk 0 has landed
        __builtin_amdgcn_s_barrier();   // (the plain barrier: __syncthreads would wait for all requests)
        for (int s = 2; s < R::NEXT; ++s) ask(s, s);
        for (int i = 0, buf = 0; i < n; ++i) {
            asm volatile("s_waitcnt vmcnt(%0)" ::"n"((R::NEXT - 2) * R::REQ) : "memory");   // chunk i + 1 has landed
            __builtin_amdgcn_s_barrier();
            ask(i + R::NEXT, S2 ? buf : buf == 0 ? R::D - 1 : buf - 1);   // where chunk i was (S2), or the one before it, which is multiplied
            buf = buf + 1 == R::D ? 0 : buf + 1;
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the requests past the end have landed before LDS is put to other use
        __builtin_amdgcn_s_setprio(0);
    } else {
#pragma unroll
        for (int t = 0; t < kT; ++t)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[t][r] = 0;
        switch (p.row_pitch & 15) {   // uniform
#define DAQ_RING32(Q) case Q: ring32_loop<S2, Q>(n, wave, l32, lh, p.row_pitch, acc); break;
            DAQ_RING32(0) DAQ_RING32(1) DAQ_RING32(2) DAQ_RING32(3) DAQ_RING32(4) DAQ_RING32(5) DAQ_RING32(6) DAQ_RING32(7)
            DAQ_RING32(8) DAQ_RING32(9) DAQ_RING32(10) DAQ_RING32(11) DAQ_RING32(12) DAQ_RING32(13) DAQ_RING32(14) DAQ_RING32(15)
#undef DAQ_RING32
        }
    }

    // ---- combine the four multiplying waves.  Of the 36 quads of slots (four consecutive registers of a tap: one 16-byte LDS access a
    // lane) a pair of waves w, w + 4 owns nine: wave w sums five, three hand-overs and its own part, wave w + 4 four, all handed over;
    // area [owner][quad][source][lane] ----
    // register r of a 32 x 32 tile: row (co) 8*(r/4) + 4*lh + r%4, column (ci) l32; slot = tap*16 + r
    // A complete tile: dW[co][ci][t] has the 32 ci x 9 taps of one co contiguous (1152 bytes), but a lane holds one
    // ci and a register one (co, t).  The tile is transposed through LDS so that the global stores are row runs.
    constexpr int SLOTS = kT * 16, OWN = kT, FIRST = 5, PAIR = 3 * FIRST + 4 * (OWN - FIRST);   // quads of a pair, of its first wave; entries
    constexpr int COLS = 32 * kT, ROWW = COLS + 4;   // ints per co row in LDS
    static_assert(4 * PAIR * 1024 <= R::LDS && 32 * ROWW * 4 <= R::LDS, "fits");
    v4i* area = reinterpret_cast<v4i*>(lds);
    int* red = reinterpret_cast<int*>(lds);
    int32_t* dst = p.part + ((int64_t)tile * p.splits + split) * SLOTS * kWave + lane;
    auto quad = [&](int q) { return v4i{acc[q / 4][4 * (q % 4)], acc[q / 4][4 * (q % 4) + 1], acc[q / 4][4 * (q % 4) + 2], acc[q / 4][4 * (q % 4) + 3]}; };
    __syncthreads();   // the staging buffers are dead from here on
    if (wave < 4) {
#pragma unroll
        for (int q = 0; q < 4 * OWN; ++q) {
            const int w = q / OWN, j = q % OWN;
            if (j >= FIRST) area[(w * PAIR + 3 * FIRST + 4 * (j - FIRST) + wave) * kWave + lane] = quad(q);
            else if (w != wave) area[(w * PAIR + 3 * j + (wave < w ? wave : wave - 1)) * kWave + lane] = quad(q);   // uniform
        }
    } else if (tid < 256 + 32) {
        l_scale[tid - 256] = (*p.s_x / 127.0f) * (p.s_chan[min(co0 + tid - 256, p.Cout - 1)] / 127.0f);
    }
    __syncthreads();
    v4i sum[4][OWN];   // (of one of the four pairs, the wave's part of the nine)
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        const v4i* from = area + w * PAIR * kWave + lane;
        if (wave == w) {   // uniform
#pragma unroll
            for (int j = 0; j < FIRST; ++j) sum[w][j] = quad(w * OWN + j) + from[3 * j * kWave] + from[(3 * j + 1) * kWave] + from[(3 * j + 2) * kWave];
        } else if (wave == w + 4) {   // uniform
#pragma unroll
            for (int j = 0; j < OWN - FIRST; ++j) {
                const v4i* f = from + (3 * FIRST + 4 * j) * kWave;
                sum[w][FIRST + j] = f[0] + f[kWave] + f[2 * kWave] + f[3 * kWave];
            }
        }
    }
    if (p.splits == 1) __syncthreads();   // everyone is done reading the hand-over area
#pragma unroll
    for (int w = 0; w < 4; ++w)
#pragma unroll
        for (int j = 0; j < OWN; ++j) {
            if (wave != w + (j < FIRST ? 0 : 4)) continue;   // uniform
            const int q = w * OWN + j;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int r = 4 * (q % 4) + e;
                if (p.splits > 1) __builtin_nontemporal_store(sum[w][j][e], &dst[(4 * q + e) * kWave]);   // uniform; read next by other CUs, not by this one
                else red[(8 * (r >> 2) + 4 * lh + (r & 3)) * ROWW + l32 * kT + q / 4] = sum[w][j][e];
            }
        }
    if (p.splits > 1) return;
    __syncthreads();
    const int ncol = min(32, p.Cin - ci0) * kT, nrow = min(32, p.Cout - co0);   // valid ints of a row, valid rows
    const int64_t first = ((int64_t)co0 * p.Cin + ci0) * p.taps_all;
    const int row_step = p.Cin * p.taps_all;   // (below 2^31 over the rows of dW)
    if (ncol == COLS && p.taps_all == kT && p.Cin % 4 == 0 && ((uintptr_t)p.dW & (p.bf16 ? 7 : 15)) == 0 && !p.acc_out) {   // uniform
        // four results a thread at a time (one at a time, with an address for each, this took 2.3 us)
        constexpr int V = COLS / 4;
        int row = tid / V, col = tid - row * V;
#pragma unroll
        for (int k = 0; k < (32 * V + 511) / 512; ++k) {
            if (row < nrow) {
                const v4i v = *reinterpret_cast<const v4i*>(red + row * ROWW + 4 * col);
                const float sc = l_scale[row];
                store_result4(p.dW, first + row * row_step + 4 * col, (float)v[0] * sc, (float)v[1] * sc, (float)v[2] * sc, (float)v[3] * sc, p.bf16, 0);
            }
            const int c = col + 512 % V;
            row += 512 / V + (c >= V);
            col = c >= V ? c - V : c;
        }
        return;
    }
    int row = tid / COLS, col = tid - row * COLS;
    for (int k = 0; k < 32 * COLS / 512; ++k) {
        if (row < nrow && col < ncol) {
            // (3-D: a depth tap's nine results, then the next input channel's)
            const int64_t at = first + row * row_step + (p.taps_all == kT ? col : (col / kT) * p.taps_all + col % kT);
            const int v = red[row * ROWW + col];
            store_result(p.dW, at, (float)v * l_scale[row], p.bf16);
            if (p.acc_out) p.acc_out[at] = v;
        }
        const int c = col + 512 % COLS;
        row += 512 / COLS + (c >= COLS);
        col = c >= COLS ? c - COLS : c;
    }
}

// ---------------------------------------------------------------------------------------------
// 1 x 1 filters at unit stride: no tap shifts, so the product is a plain int8 GEMM over the flat axis,
//     acc[co][ci] = sum_f  G[co][f] * X[ci][f] ,
// with both operands staged the same way (rows of 256 + 16 bytes, aligned 16-byte fragment reads).
// A wave owns 64 (co) x 64 (ci): four 32 x 32 tiles, so every fragment it reads feeds two multiplies.
// K splits, and waves that share a tile combined through LDS, as above.
// ---------------------------------------------------------------------------------------------
// DMA (the eight-wave form): the operands go from global memory straight into LDS (the 64 lanes' 16-byte pieces land in 64
// consecutive slots), four stage buffers of unpadded 256-byte rows, three stages on
// their way; no staging registers, no LDS stores, one barrier per chunk.  Slot column c of row r holds the row's
// 16-byte column c ^ (r % 16), so that the 16 lanes of a fragment read still fall into different banks.
// LONG: the requests' addresses are made by vector instructions (64 bits a lane) instead of scalar ones, which lets them go out behind the
// multiplies of the chunk before.  A workgroup of many chunks is the faster for it, a short one the slower (dw11_long).
template <int WM, int WN, int WK, int PF, int CH, bool DMA, bool LONG = false>
__device__ __forceinline__ void dw11_role(Dw32Args& p, const int bid) {
    constexpr int WAVES = WM * WN * WK, NT = 64 * WAVES;
    static_assert(WAVES == 4 || WAVES == 8, "four or eight waves");
    constexpr int BM = 64 * WM, BN = 64 * WN;
    constexpr int KCS = CH * kKC;                           // K bytes of a stage: CH chunks between two barriers
    constexpr int PAS = KCS + 16;                           // LDS row pitch of a stage
    constexpr int UPR = KCS / 16;                           // 16-byte units per staged row
    constexpr int UNITS = (BM + BN) * UPR / NT;             // 16-byte units of the two tiles per thread
    constexpr int STAGE = (BM + BN) * PAS;
    static_assert(NT % UPR == 0, "a thread's units all sit in the same 16-byte column of their rows");
    extern __shared__ __align__(16) int8_t lds[];

    dw_depth(p, 1);
    const int tid = threadIdx.x, lane = tid % kWave;
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int wk = wave % WK, wn = (wave / WK) % WN, wm = wave / (WK * WN);
    const int l32 = lane & 31, lh = lane >> 5;

    int split, tile;
    if (!dw_block_map(p, bid, split, tile)) return;   // uniform
    const int tn = tile % p.tiles_n, tm = tile / p.tiles_n;
    const int co0 = tm * BM, ci0 = tn * BN;
    const int per = p.nchunks / p.splits, rem = p.nchunks % p.splits;
    const int c_begin = split * per + min(split, rem);
    const int c_end = c_begin + per + (split < rem ? 1 : 0);
    const int c_last = max(c_end - 1, 0);

    // a complete tile is de-quantized here: its scales are requested now, long before they are needed
    float sx = 0.0f, sc_own[WK > 1 ? 8 : 1];
    if (WK > 1 && p.splits == 1) {   // uniform
        sx = *p.s_x;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int q = wk * 8 + e, r = q % 16;
            const int co = co0 + wm * 64 + 32 * (q / 32) + 8 * (r >> 2) + 4 * lh + (r & 3);
            sc_own[e] = p.s_chan[co < p.Cout ? co : 0];
        }
    }

    v16i acc[2][2];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[a][b][r] = 0;

    if constexpr (DMA) {
        static_assert(WM == 1 && WN == 1 && WK == 8 && CH == 1, "the direct-to-LDS form is the eight-wave one");
        constexpr int D = 4;                     // stage buffers
        constexpr int SB = (BM + BN) * kKC;      // bytes of a stage
        // request i of wave w fills rows 16w + 4i .. + 3 of the stage: lane l -> row + l / 16, slot column l % 16; the first four waves the
        // gradient's rows, the others the activation's
        const bool grad = wave < 4;   // uniform
        const __amdgpu_buffer_rsrc_t rs = tile_rsrc(grad ? p.g + (int64_t)co0 * p.klen : p.x + (int64_t)ci0 * p.x_chan_pitch);
        uint32_t from[4];
        const int8_t* src[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {   // rows past Cout / Cin recompute the first one and are never stored
            const int row = 16 * (wave % 4) + 4 * i + lane / 16;
            const int col = (lane % 16) ^ (row & 15);
            const bool live = row < (grad ? p.Cout - co0 : p.Cin - ci0);
            from[i] = (uint32_t)((int64_t)(live ? row : 0) * (grad ? p.klen : p.x_chan_pitch) + 16 * col);
            if constexpr (LONG) {   // (one base a lane: with a base for the wave the compiler keeps the addresses scalar)
                const int g_row = 16 * wave + 4 * i + lane / 16;
                src[i] = g_row < BM ? p.g + (int64_t)(live ? co0 + row : 0) * p.klen + 16 * col : p.x + (int64_t)(live ? ci0 + row : 0) * p.x_chan_pitch + 16 * col;
            }
        }
        // every call issues four requests (past the end the last chunk again, into a buffer nobody reads), so that the
        // count of outstanding requests below is a constant
        auto issue = [&](int chunk, int buf) {
            const uint32_t k0 = (uint32_t)min(chunk, c_last) * (uint32_t)kKC;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                int8_t* const dst = lds + buf * SB + (16 * wave + 4 * i) * kKC;
                if constexpr (LONG) __builtin_amdgcn_global_load_lds(src[i] + k0, (__attribute__((address_space(3))) void*)dst, 16, 0, 0);
                else load_to_lds(rs, from[i], k0, dst);
            }
        };
#pragma unroll
        for (int st = 0; st < D - 1; ++st) issue(c_begin + st, st);
        // fragment of K step wk: row l32 (+ 32 t), the row's column 2 wk + lh
        const int fcol = 16 * ((2 * wk + lh) ^ (l32 & 15));
        const int arow = l32 * kKC + fcol, brow = (BM + l32) * kKC + fcol;
        int buf = 0;
        for (int chunk = c_begin; chunk < c_end; ++chunk) {
            asm volatile("s_waitcnt vmcnt(8)" ::: "memory");   // this wave's share of the chunk has landed; two more stages may be on their way
            __builtin_amdgcn_s_barrier();                       // everybody's share has, and the buffer refilled next has been read out
                                                                // (the plain barrier: __syncthreads would wait for the stages on their way too)
            issue(chunk + D - 1, (buf + D - 1) % D);
            const int8_t* A = lds + buf * SB + arow;
            const int8_t* B = lds + buf * SB + brow;
            v4i fa[2], fb[2];
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                fa[t] = *reinterpret_cast<const v4i*>(A + t * 32 * kKC);
                fb[t] = *reinterpret_cast<const v4i*>(B + t * 32 * kKC);
            }
#pragma unroll
            for (int a = 0; a < 2; ++a)
#pragma unroll
                for (int b = 0; b < 2; ++b) acc[a][b] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fa[a], fb[b], acc[a][b], 0, 0, 0);
            buf = (buf + 1) % D;
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the requests past the end have landed before LDS is put to other use
    } else {
    // unit u = tid + NT*i -> row u / UPR of the stacked (gradient, activation) tile, 16-byte column u % UPR of the stage;
    // the column - and with it the chunk of the stage the unit belongs to - is the same for all units of a thread
    const int c16 = tid % UPR, sub = c16 / (kKC / 16);
    const int8_t* u_src[UNITS];
    int u_dst[UNITS];
#pragma unroll
    for (int i = 0; i < UNITS; ++i) {
        const int row = (tid + NT * i) / UPR;
        if (row < BM) {   // rows past Cout / Cin recompute row 0 and are never stored
            const int co = co0 + row;
            u_src[i] = p.g + (int64_t)(co < p.Cout ? co : 0) * p.klen + 16 * (c16 % (kKC / 16));
        } else {
            const int ci = ci0 + row - BM;
            u_src[i] = p.x + (int64_t)(ci < p.Cin ? ci : 0) * p.x_chan_pitch + 16 * (c16 % (kKC / 16));
        }
        u_dst[i] = row * PAS + 16 * c16;
    }
    // Every call issues the same loads (past the end the last chunk is fetched again, which the caches absorb, and
    // never multiplied): only then can the compiler count the loads in flight and wait for exactly the oldest set.
    v4i ring[PF][UNITS];
    auto load_stage = [&](int chunk, int set) {   // chunk: the first of the stage
        const int64_t k0 = (int64_t)min(chunk + sub, c_last) * kKC;
#pragma unroll
        for (int i = 0; i < UNITS; ++i) ring[set][i] = *reinterpret_cast<const v4i*>(u_src[i] + k0);
        __builtin_amdgcn_sched_barrier(0);   // keep the sets in program order
    };
    auto store_stage = [&](int buf, int set) {
#pragma unroll
        for (int i = 0; i < UNITS; ++i) *reinterpret_cast<v4i*>(lds + buf * STAGE + u_dst[i]) = ring[set][i];
    };

    load_stage(c_begin, 0);
    store_stage(0, 0);
#pragma unroll
    for (int i = 1; i <= PF; ++i) load_stage(c_begin + i * CH, i % PF);
    __syncthreads();

    const int arow = (wm * 64 + l32) * PAS + 16 * lh;
    const int brow = (BM + wn * 64 + l32) * PAS + 16 * lh;
    int buf = 0;
    for (int base = c_begin; base < c_end; base += PF * CH) {
#pragma unroll
      for (int u = 0; u < PF; ++u) {
        const int chunk = base + u * CH;
        if (chunk >= c_end) break;   // uniform
        const int8_t* A = lds + buf * STAGE + arow;
        const int8_t* B = lds + buf * STAGE + brow;
        constexpr int KS = (kKC / 32) / WK;
        v4i fa[CH][KS][2], fb[CH][KS][2];
#pragma unroll
        for (int j = 0; j < CH; ++j)
#pragma unroll
            for (int i = 0; i < KS; ++i) {
                const int ks = wk + i * WK;
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    fa[j][i][t] = *reinterpret_cast<const v4i*>(A + t * 32 * PAS + j * kKC + 32 * ks);
                    fb[j][i][t] = *reinterpret_cast<const v4i*>(B + t * 32 * PAS + j * kKC + 32 * ks);
                }
            }
#pragma unroll
        for (int j = 0; j < CH; ++j) {
            if (j > 0 && chunk + j >= c_end) break;   // uniform: the stage's later chunks lie past this split's share
#pragma unroll
            for (int i = 0; i < KS; ++i)
#pragma unroll
                for (int a = 0; a < 2; ++a)
#pragma unroll
                    for (int b = 0; b < 2; ++b)
                        acc[a][b] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fa[j][i][a], fb[j][i][b], acc[a][b], 0, 0, 0);
        }
        store_stage(buf ^ 1, (u + 1) % PF);
        load_stage(chunk + (1 + PF) * CH, (u + 1) % PF);
        buf ^= 1;
        __syncthreads();
      }
    }
    }

    // slot q = (a*2 + b)*16 + r: tile (a, b) of the wave, register r -> row (co) 32a + 8*(r/4) + 4*lh + r%4, column (ci) 32b + l32
    constexpr int SLOTS = 64;
    v4i own[2];   // WK = 8: the two quads of slots (four consecutive registers of one tile) this wave owns
    if constexpr (WK > 1) {
        // parallel combine of the eight waves, each of which has a part of the whole tile, in one round: 16 quads, two per wave,
        // hand-over area [quad][source wave][lane] of 16-byte entries
        static_assert(WK == 8, "the combine below is laid out for eight waves");
        v4i* red4 = reinterpret_cast<v4i*>(lds);
        __syncthreads();   // the staging buffers are dead from here on
#pragma unroll
        for (int Q = 0; Q < SLOTS / 4; ++Q) {
            const int owner = Q / 2;
            if (owner != wk) {   // uniform
                const int srcw = wk < owner ? wk : wk - 1;
                const int g4 = 4 * (Q % 4);
                const v16i& tl = acc[Q / 8][(Q / 4) % 2];
                red4[(Q * (WK - 1) + srcw) * kWave + lane] = v4i{tl[g4], tl[g4 + 1], tl[g4 + 2], tl[g4 + 3]};
            }
        }
        __syncthreads();
#pragma unroll
        for (int Q = 0; Q < SLOTS / 4; ++Q) {
            if (Q / 2 != wk) continue;   // uniform
            const int g4 = 4 * (Q % 4);
            const v16i& tl = acc[Q / 8][(Q / 4) % 2];
            v4i v = {tl[g4], tl[g4 + 1], tl[g4 + 2], tl[g4 + 3]};
#pragma unroll
            for (int w = 0; w < WK - 1; ++w) v += red4[(Q * (WK - 1) + w) * kWave + lane];
            own[Q % 2] = v;
        }
    }
    int32_t* dst = p.part + (((int64_t)tile * p.splits + split) * (WM * WN) + wm * WN + wn) * SLOTS * kWave + lane;
    if (WK == 1 && p.splits == 1) sx = *p.s_x;
    sx = sx / 127.0f;
#pragma unroll
    for (int q = 0; q < SLOTS; ++q) {
        if (WK > 1 && q / 8 != wk) continue;   // uniform: not this wave's slot
        const int v = WK > 1 ? own[(q / 4) % 2][q % 4] : acc[q / 32][(q / 16) % 2][q % 16];
        if (p.splits > 1) {
            __builtin_nontemporal_store(v, &dst[q * kWave]);   // read next by other CUs, not by this one
        } else {
            const int r = q % 16;
            const int co = co0 + wm * 64 + 32 * (q / 32) + 8 * (r >> 2) + 4 * lh + (r & 3);
            const int ci = ci0 + wn * 64 + 32 * ((q / 16) % 2) + l32;
            if (co < p.Cout && ci < p.Cin) {
                const int64_t off = ((int64_t)co * p.Cin + ci) * p.taps_all;   // 32 lanes = 32 consecutive ci: 128-byte runs (2-D)
                const float sc = WK > 1 ? sc_own[q % 8] : p.s_chan[co];
                store_result(p.dW, off, (float)v * (sx * (sc / 127.0f)), p.bf16);
                if (p.acc_out) p.acc_out[off] = v;
            }
        }
    }
}

}  // namespace

}  // namespace daq
