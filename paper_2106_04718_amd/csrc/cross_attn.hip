// Encoder-decoder cross-attention over a de-duplicated K/V cache, for gfx950.
//
// The operation is Eq. 4 of the paper (Appendix B): the k beam queries of
// source b read the one copy K[b], V[b] of that source's encoder keys and
// values, and each computes softmax(q K^T / sqrt(D)) V over the valid keys
// j < src_len[b].  Per head it is a GEMV-like contraction with k query rows
// (about k flop per byte of K/V), so it is bound by HBM bandwidth.  The
// kernel reads every valid K/V byte exactly once with coalesced,
// non-temporal 16-byte loads and keeps all k beams' work on that data in
// registers.
//
// Tiles.  A wave attends one tile of 4096 / D keys for all k beams; kWaves
// tiles make a chunk.  A group of kLpr lanes shares a row (16 bytes per lane),
// so a wave instruction reads kRpi whole rows.
//   bf16, D >= 32 (MfmaTile): the K rows go through LDS to the A operand of
//     v_mfma_f32_16x16x32_bf16, the beams' queries are its columns; a lane then
//     holds 16 scores of one beam.  V is read back transposed for PV.
//   fp32, and D = 16 (ValuTile): each lane dots its 16 bytes of the row with
//     the same 16 bytes of the beams' queries, a reduce-scatter in the lane
//     group completes the scores, and PV accumulates in fp32 in the row layout.
//     Many beams go a group at a time, so that their sums stay in registers.
//   Both keep a tile's state as (maximum, sum, unnormalised output) per beam.
// Decompositions, one launch each, chosen by choose_attn_path:
//   attn_whole_kernel: one workgroup of 4, 8 or 16 waves per (b, h), which
//     walks the row's tile tasks one per wave and round (walk_row) and folds
//     each round's states into the row's.  No workspace.
//   cross_attn_kernel (split-KV, few long rows): one workgroup per chunk.  Rows
//     of more than one chunk store one record per chunk in the workspace, and a
//     merger workgroup per (b, h), after all chunk workgroups in the grid (so
//     dispatched after them), folds them in chunk order.  Each record word
//     carries a tag of the call, so the merger knows when a record is
//     complete; no fence or clearing of the workspace is needed.  The tag is
//     the host's call epoch, or, for a call captured into a graph, a per-row
//     counter in the workspace that the row's merger advances.
// Generated tokens of a split cache are the same tiles: tasks of the walk, or,
// where beam_waves says so, a beam per wave before it (generated_beams).
// Every form folds the same states in the same order (the chunks of the prefix,
// then each beam's generated tiles), so all give the same bits.
// Rows j >= src_len[b] are never read.  The chunk size depends only on the
// row size, and each beam's arithmetic is the same whatever k is, so the
// output bits do not depend on k, B or the beam's position.
#include <math.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <atomic>
#include <type_traits>

#include "div.h"
#include "launch.h"
#include "ngram_row.h"
#include "trace.h"

namespace fs {
namespace {

constexpr int kWave = 64;
constexpr int kWaves = 4;
constexpr int kBlock = kWave * kWaves;
constexpr int kIt = 8;   // row loads of K (and of V) per lane per tile
constexpr int kXcds = 8; // MI355X: workgroups go round-robin to 8 XCDs
constexpr int kCus = 256;                // MI355X compute units
constexpr int kSplitMaxRows = 128;       // rows of many tiles are split across workgroups below this

typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));

template <bool BF16>
struct Elem {
    static constexpr int size = BF16 ? 2 : 4;
    static constexpr int per16 = 16 / size;  // elements in 16 bytes
};

template <int D, bool BF16>
struct Geo {
    static constexpr int kEpl = Elem<BF16>::per16;   // elements per lane slice
    static constexpr int kLpr = D / kEpl;            // lanes sharing one row
    static constexpr int kRpi = kWave / kLpr;        // rows per wave instruction
    static constexpr int kTile = kIt * kRpi;         // keys per wave tile
    static constexpr int kChunk = kWaves * kTile;    // keys per workgroup
    static constexpr int kDup = kLpr > kIt ? kLpr / kIt : 1;   // lanes sharing a score row
    static constexpr int kRows = kLpr < kIt ? kIt / kLpr : 1;  // score rows per lane
    static constexpr int kPStride = kTile + kTile / 8;     // LDS rows per wave (padded)
    static_assert(kLpr >= 2 && kLpr <= 32, "row must be 32..512 bytes");
    static_assert(kIt == 8 || kIt == 16, "the row-load count must be a power of two >= 8");
};

__device__ __forceinline__ uint4 load_nt(const uint4 *p) {
    const u32x4_t t = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t *>(p));
    return make_uint4(t.x, t.y, t.z, t.w);
}

// Buffer resource over the first `bytes` bytes at p (raw addressing, no
// stride): loads past the end return zero without touching memory.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t row_rsrc(const void *p, int bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, bytes, 0x00020000);
}
// 16-byte non-temporal buffer load at byte offset voff + soff.
__device__ __forceinline__ uint4 load_rows(__amdgpu_buffer_rsrc_t r, int voff, int soff) {
    const u32x4_t t = __builtin_bit_cast(u32x4_t, __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, 2));
    return make_uint4(t.x, t.y, t.z, t.w);
}

__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

__device__ __forceinline__ float dot2_bf16(uint32_t a, uint32_t b, float c) {
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, a),
                                           __builtin_bit_cast(bf16x2_t, b), c, false);
}

// Dot product of two 16-byte slices, accumulated into c in element order.
template <bool BF16>
__device__ __forceinline__ float dot16(uint4 a, uint4 b, float c) {
    if constexpr (BF16) {
        c = dot2_bf16(a.x, b.x, c);
        c = dot2_bf16(a.y, b.y, c);
        c = dot2_bf16(a.z, b.z, c);
        c = dot2_bf16(a.w, b.w, c);
    } else {
        c = fmaf(__uint_as_float(a.x), __uint_as_float(b.x), c);
        c = fmaf(__uint_as_float(a.y), __uint_as_float(b.y), c);
        c = fmaf(__uint_as_float(a.z), __uint_as_float(b.z), c);
        c = fmaf(__uint_as_float(a.w), __uint_as_float(b.w), c);
    }
    return c;
}

// Unpack a 16-byte slice to fp32 values (exact).
template <bool BF16>
__device__ __forceinline__ void unpack16(uint4 a, float *f) {
    if constexpr (BF16) {
        f[0] = bf16_lo(a.x); f[1] = bf16_hi(a.x);
        f[2] = bf16_lo(a.y); f[3] = bf16_hi(a.y);
        f[4] = bf16_lo(a.z); f[5] = bf16_hi(a.z);
        f[6] = bf16_lo(a.w); f[7] = bf16_hi(a.w);
    } else {
        f[0] = __uint_as_float(a.x); f[1] = __uint_as_float(a.y);
        f[2] = __uint_as_float(a.z); f[3] = __uint_as_float(a.w);
    }
}

// ---- cross-lane exchange ---------------------------------------------------
// DPP stays inside a row of 16 lanes, ds_swizzle inside 32 lanes, and
// ds_bpermute covers the whole wave.
template <int CTRL>
__device__ __forceinline__ float dpp(float x) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(
        0, __builtin_bit_cast(int, x), CTRL, 0xF, 0xF, true));
}
template <int PATTERN>
__device__ __forceinline__ float swizzle(float x) {
    return __builtin_bit_cast(float, __builtin_amdgcn_ds_swizzle(__builtin_bit_cast(int, x), PATTERN));
}
__device__ __forceinline__ float lane_xor(float x, int mask) {
    return __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute((__lane_id() ^ mask) << 2,
                                                                  __builtin_bit_cast(int, x)));
}

// Value of lane (lane ^ MASK), for MASK a power of two below 64.
template <int MASK>
__device__ __forceinline__ float xor_lane(float x) {
    if constexpr (MASK == 1) return dpp<0xB1>(x);              // quad_perm [1,0,3,2]
    else if constexpr (MASK == 2) return dpp<0x4E>(x);         // quad_perm [2,3,0,1]
    else if constexpr (MASK == 8) return dpp<0x128>(x);        // row_ror:8 == xor 8 in a row
    else if constexpr (MASK < 32) return swizzle<0x1F | (MASK << 10)>(x);  // bit mode, xor MASK
    else return lane_xor(x, MASK);
}

// Sum over the kLpr lanes of a row group (every lane of the group gets the
// bit-identical result: each step pairs lanes and adds commutatively).
template <int G>
__device__ __forceinline__ float group_sum(float x) {
    if constexpr (G >= 2) x += dpp<0xB1>(x);
    if constexpr (G >= 4) x += dpp<0x4E>(x);
    if constexpr (G >= 8) x += dpp<0x141>(x);   // row_half_mirror: other quad of the 8
    if constexpr (G >= 16) x += dpp<0x140>(x);  // row_mirror: other 8 of the 16
    if constexpr (G >= 32) x += swizzle<0x401F>(x);
    return x;
}

// Reduction over the row groups of a wave (lanes sharing lane % G).
template <int G, int MASK = G>
__device__ __forceinline__ float groups_max(float x) {
    if constexpr (MASK < kWave) {
        x = fmaxf(x, xor_lane<MASK>(x));
        return groups_max<G, MASK * 2>(x);
    } else {
        return x;
    }
}
template <int G, int MASK = G>
__device__ __forceinline__ float groups_sum(float x) {
    if constexpr (MASK < kWave) {
        x += xor_lane<MASK>(x);
        return groups_sum<G, MASK * 2>(x);
    } else {
        return x;
    }
}

// All-reduce over the 64 lanes (every lane gets the bit-identical result).
__device__ __forceinline__ float wave_max(float x) {
    x = fmaxf(x, dpp<0xB1>(x));
    x = fmaxf(x, dpp<0x4E>(x));
    x = fmaxf(x, dpp<0x141>(x));
    x = fmaxf(x, dpp<0x140>(x));
    x = fmaxf(x, swizzle<0x401F>(x));
    x = fmaxf(x, lane_xor(x, 32));
    return x;
}
__device__ __forceinline__ float wave_sum(float x) {
    x += dpp<0xB1>(x);
    x += dpp<0x4E>(x);
    x += dpp<0x141>(x);
    x += dpp<0x140>(x);
    x += swizzle<0x401F>(x);
    x += lane_xor(x, 32);
    return x;
}

// Partner value for step MASK of a butterfly inside a row group of G lanes.
// The first step (MASK == G/2) may pair lane s with G-1-s (a mirror, which
// DPP does cheaply); later steps must pair s with s ^ MASK exactly.
template <int G, int MASK>
__device__ __forceinline__ float group_partner(float x) {
    if constexpr (MASK == G / 2 && MASK == 4) return dpp<0x141>(x);   // row_half_mirror
    else if constexpr (MASK == G / 2 && MASK == 8) return dpp<0x140>(x);  // row_mirror
    else return xor_lane<MASK>(x);
}

// Reduce-scatter of the QK^T partial sums inside a row group of G lanes.
// On entry every lane holds, for the tile's NI row loads u and each beam i,
// its own 16-byte slice of the dot product d[u][i].  On exit d[j][i],
// j < max(1, NI/G), holds the complete dot product of row
// u = (sub / max(1, G/NI)) * max(1, NI/G) + j: the NI*KB sums are spread
// over the group instead of being repeated in every lane, so each score is
// turned into a probability once (G/NI times when G > NI).
template <int G, int KB, int NI, int MASK = G / 2, int NR = NI>
__device__ __forceinline__ void group_reduce_scatter(float (&d)[NI][KB], int sub) {
    if constexpr (MASK >= 1) {
        if constexpr (NR > 1) {
            constexpr int HALF = NR / 2;
            const bool up = (sub & MASK) != 0;
#pragma unroll
            for (int j = 0; j < HALF; ++j) {
#pragma unroll
                for (int i = 0; i < KB; ++i) {
                    const float send = up ? d[j][i] : d[j + HALF][i];
                    const float keep = up ? d[j + HALF][i] : d[j][i];
                    d[j][i] = keep + group_partner<G, MASK>(send);
                }
            }
            group_reduce_scatter<G, KB, NI, MASK / 2, HALF>(d, sub);
        } else {
#pragma unroll
            for (int i = 0; i < KB; ++i) d[0][i] += group_partner<G, MASK>(d[0][i]);
            group_reduce_scatter<G, KB, NI, MASK / 2, 1>(d, sub);
        }
    }
}

// Index of this wave in its workgroup, as a wave-uniform (scalar) value, so
// that branches on it are uniform and each side keeps its own registers.
#if FS_TRACE
__device__ trace::Target g_trace{nullptr, 0};
#endif
// this workgroup's timeline words in a trace build, else null
__device__ __forceinline__ unsigned long long *trace_slot() {
#if FS_TRACE
    return trace::slot(g_trace);
#else
    return nullptr;
#endif
}

__device__ __forceinline__ int wave_id() {
    return __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
}

// Merge softmax state (mb, lb, ab) into (m, l, a); m in the base-2 domain.
// The fused multiply-adds are written out, so that every decomposition rounds
// the same product.
__device__ __forceinline__ void merge_state(float &m, float &l, float &a, float mb, float lb, float ab) {
    const float mx = fmaxf(m, mb);
    const float ms = (mx == -INFINITY) ? 0.f : mx;
    const float fa = __builtin_amdgcn_exp2f(m - ms);
    const float fb = __builtin_amdgcn_exp2f(mb - ms);
    l = fmaf(lb, fb, l * fa);
    a = fmaf(ab, fb, a * fa);
    m = mx;
}

__device__ __forceinline__ uint16_t f32_to_bf16_rne(float f) {
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40u);  // quiet NaN
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

template <bool BF16>
__device__ __forceinline__ void store_out(void *out, size_t idx, float v) {
    if constexpr (BF16)
        static_cast<uint16_t *>(out)[idx] = f32_to_bf16_rne(v);
    else
        static_cast<float *>(out)[idx] = v;
}

// Bound on re-reads of a partial-record word that does not yet carry the
// current call's tag (about 10 ms at most; not reached in practice).
constexpr int kMaxSpins = 1 << 14;

// One wave tile's K and V rows, in the coalesced layout: instruction u reads
// rows t0 + u*kRpi + grp whole, kLpr lanes per row (loads of 16 half rows
// each are markedly slower).
struct Rows {
    uint4 k[kIt], v[kIt];
};

// Issues the loads of keys [t0, t0 + kTile) of a stream of j1 rows at Kb/Vb.
// Buffer loads whose range ends at row j1: rows past it read as zero without
// a memory access and are masked by the tile, and K and V share one offset
// register.  All K first, so that the tile can start while V is in flight
// (ORDER holds the compiler to it, where the loads and the tile are apart).
template <int D, bool BF16, bool ORDER>
__device__ __forceinline__ void load_tile(Rows &r, const uint4 *__restrict__ Kb, const uint4 *__restrict__ Vb, int t0,
                                          int j1, int lane)
{
    using G = Geo<D, BF16>;
    constexpr int kRow = D * Elem<BF16>::size;
    const auto kres = row_rsrc(Kb, j1 * kRow), vres = row_rsrc(Vb, j1 * kRow);
    const int off = (t0 + lane / G::kLpr) * kRow + lane % G::kLpr * 16;
    if constexpr (ORDER) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < kIt; ++u) r.k[u] = load_rows(kres, off, u * G::kRpi * kRow);
    if constexpr (ORDER) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < kIt; ++u) r.v[u] = load_rows(vres, off, u * G::kRpi * kRow);
    if constexpr (ORDER) __builtin_amdgcn_sched_barrier(0);
}

// The same with an offset per row load and a range of `bytes`: the tiles of a
// row read through an ancestry table.
__device__ __forceinline__ void load_tile_at(Rows &r, const uint4 *__restrict__ Kb, const uint4 *__restrict__ Vb,
                                             int bytes, const int (&off)[kIt])
{
    const auto kres = row_rsrc(Kb, bytes), vres = row_rsrc(Vb, bytes);
#pragma unroll
    for (int u = 0; u < kIt; ++u) r.k[u] = load_rows(kres, off[u], 0);
#pragma unroll
    for (int u = 0; u < kIt; ++u) r.v[u] = load_rows(vres, off[u], 0);
}

// Barrier of a workgroup for LDS only: this wave's global loads in flight are
// not waited for (unlike __syncthreads).
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Orders this wave's LDS accesses before and after it.
__device__ __forceinline__ void wave_lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// State of one wave tile: keys [t0, min(t0 + kTile, j1)), rows kr/vr (t0 <
// j1), attended by the KB queries qr.  On return m[i], l[i] (base-2 max and
// sum of exp2) are wave-uniform and acc[i][e] holds, in every lane, the
// unnormalised output for dims sub*kEpl + e.  prow is this wave's LDS area.
template <int D, bool BF16, int KB>
__device__ __forceinline__ void tile_attend(const uint4 (&qr)[KB], const uint4 (&kr)[kIt], const uint4 (&vr)[kIt],
                                            int t0, int j1, int sub,
                                            int grp, float *prow, float scale_log2, float (&m)[KB],
                                            float (&l)[KB], float (&acc)[KB][Geo<D, BF16>::kEpl])
{
    using G = Geo<D, BF16>;
    constexpr int kEpl = G::kEpl, kLpr = G::kLpr, kRpi = G::kRpi;
    // QK^T: partial dots of this lane's slice, then a reduce-scatter in the
    // row group, after which the lane owns whole score rows.
    float d[kIt][KB];
#pragma unroll
    for (int u = 0; u < kIt; ++u) {
#pragma unroll
        for (int i = 0; i < KB; ++i) d[u][i] = dot16<BF16>(qr[i], kr[u], 0.f);
    }
    group_reduce_scatter<kLpr, KB, kIt>(d, sub);
    constexpr int kRows = G::kRows, kDup = G::kDup;
    const int u0 = (sub / kDup) * kRows;  // first score row of this lane
    float mt[KB];
#pragma unroll
    for (int i = 0; i < KB; ++i) {
        float mx = -INFINITY;
#pragma unroll
        for (int j = 0; j < kRows; ++j) {
            const bool ok = t0 + (u0 + j) * kRpi + grp < j1;
            d[j][i] = ok ? d[j][i] * scale_log2 : -INFINITY;
            mx = fmaxf(mx, d[j][i]);
        }
        mt[i] = wave_max(mx);  // tile maximum (finite: key t0 is valid)
    }
#pragma unroll
    for (int i = 0; i < KB; ++i) {
        float lsum = 0.f;
#pragma unroll
        for (int j = 0; j < kRows; ++j) {
            d[j][i] = __builtin_amdgcn_exp2f(d[j][i] - mt[i]);
            lsum += d[j][i];
        }
        l[i] = wave_sum(sub % kDup == 0 ? lsum : 0.f);
        m[i] = mt[i];
    }
#pragma unroll
    for (int j = 0; j < kRows; ++j) {
        const int r = (u0 + j) * kRpi + grp;
#pragma unroll
        for (int i = 0; i < KB; ++i) prow[(r + (r >> 3)) * KB + i] = d[j][i];
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    // PV: the coalesced V rows with their weights read back from LDS
#pragma unroll
    for (int i = 0; i < KB; ++i) {
#pragma unroll
        for (int e = 0; e < kEpl; ++e) acc[i][e] = 0.f;
    }
#pragma unroll
    for (int u = 0; u < kIt; ++u) {
        const int r = u * kRpi + grp;
        float pw[KB];
#pragma unroll
        for (int i = 0; i < KB; ++i) pw[i] = prow[(r + (r >> 3)) * KB + i];
        float vf[kEpl];
        unpack16<BF16>(vr[u], vf);
#pragma unroll
        for (int i = 0; i < KB; ++i) {
#pragma unroll
            for (int e = 0; e < kEpl; ++e) acc[i][e] = fmaf(pw[i], vf[e], acc[i][e]);
        }
    }
    // the row groups hold partial sums of the same dims for different rows
#pragma unroll
    for (int i = 0; i < KB; ++i) {
#pragma unroll
        for (int e = 0; e < kEpl; ++e) acc[i][e] = groups_sum<kLpr>(acc[i][e]);
    }
    // keep the next tile's LDS writes behind this tile's reads
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Tag of the record words of a call, in their high 32 bits.  Outside graph
// capture the host passes an epoch in [1, 2^31).  A call captured into a
// graph passes 0 and takes, for each (b, h) row, that row's counter in the
// workspace with bit 31 set (so no host epoch equals it); the row's merger
// advances the counter once it has every record, so each replay of the
// graph tags its records anew.  c0 receives the counter value.
__device__ __forceinline__ unsigned long long call_tag(unsigned long long epoch, const unsigned long long *ctr,
                                                       unsigned long long &c0) {
    if (epoch != 0) return (epoch & 0xffffffffull) << 32;
    c0 = __hip_atomic_load(ctr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return (0x80000000ull | ((c0 % 0x7fffffffull) + 1)) << 32;
}

// Store one record word (call tag << 32 | fp32 bits) with a device-scope atomic.
__device__ __forceinline__ void store_word(unsigned long long *p, unsigned long long tag, float v) {
    __hip_atomic_store(p, tag | __float_as_uint(v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}


// ---- tile policies -----------------------------------------------------------
// A policy attends one wave tile of keys and keeps one wave's softmax state
// per beam.  The kernels below only move these states through LDS and the
// workspace, so every decomposition of a call folds the same tile states in
// the same order.
//   ValuTile  fp32, and bf16 with D = 16: the VALU routine above.
//   MfmaTile  bf16 with D >= 32: both contractions on the matrix cores.

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef float f32x8_t __attribute__((ext_vector_type(8)));
typedef short i16x4_t __attribute__((ext_vector_type(4)));

template <int D, bool BF16, int KB, int NG>
struct ValuTile {
    using G = Geo<D, BF16>;
    static constexpr int kEpl = G::kEpl, kLpr = G::kLpr;
    // NG < KB: NG beams are attended at a time, over the tile's rows in
    // registers, with the queries in LDS (a beam's arithmetic is the same).
    static constexpr bool kGroups = NG < KB;
    static constexpr int kAStride = D;  // floats between the beams of a wave's state in LDS
    // a wave's LDS: the accumulators of its state, a tile's weights from
    // kScratch on (groups: behind the accumulators of the groups before), its queries
    static constexpr int kScratch = kGroups ? KB * kAStride * 4 : 0;
    static constexpr int kTileBytes = G::kPStride * NG * 4;
    static constexpr int kQBytes = kGroups ? KB * D * Elem<BF16>::size : 0;
    struct Q {
        uint4 r[kGroups ? 1 : KB];
        const uint4 *lds;
    };
    // m, l wave-uniform; acc[i][e] holds dims sub*kEpl + e in every lane
    struct St { float m[NG], l[NG], acc[NG][kEpl]; };

    // queries of hypotheses hyp0 .. hyp0 + KB - 1, head h; q_lds: kQBytes of this wave's LDS
    static __device__ __forceinline__ void load_q(Q &q, const uint4 *__restrict__ qp, size_t hyp0, int h, int H,
                                                  int lane, void *q_lds = nullptr) {
        const int sub = lane % kLpr;
        if constexpr (kGroups) {
            uint4 *to = static_cast<uint4 *>(q_lds);
            uint4 r[KB];
#pragma unroll
            for (int i = 0; i < KB; ++i) r[i] = qp[((hyp0 + i) * H + h) * kLpr + sub];
            if (lane < kLpr) {
#pragma unroll
                for (int i = 0; i < KB; ++i) to[i * kLpr + lane] = r[i];
            }
            wave_lds_fence();
            q.lds = to;
        } else {
#pragma unroll
            for (int i = 0; i < KB; ++i) q.r[i] = qp[((hyp0 + i) * H + h) * kLpr + sub];
        }
    }
    static __device__ __forceinline__ void attend(const Q &q, const Rows &r, int t0, int j1, int lane, void *lds,
                                                  float scale_log2, St &s) {
        static_assert(!kGroups, "the state is that of one group");
        tile_attend<D, BF16, KB>(q.r, r.k, r.v, t0, j1, lane % kLpr, lane / kLpr, static_cast<float *>(lds),
                                 scale_log2, s.m, s.l, s.acc);
    }
    // this wave's state into LDS: m_w and l_w (beam i at i * ms), a_w[KB][kAStride]
    static __device__ __forceinline__ void to_lds(const St &s, int lane, float *m_w, float *l_w, int ms, float *a_w) {
        put<NG>(s, lane, m_w, l_w, ms, a_w);
    }
    // attend and to_lds group by group
    template <int I0 = 0>
    static __device__ __forceinline__ void attend_groups(const Q &q, const Rows &r, int t0, int j1, int lane,
                                                         void *lds, float scale_log2, float *m_w, float *l_w, int ms,
                                                         float *a_w) {
        constexpr int N = KB - I0 < NG ? KB - I0 : NG;
        uint4 qr[N];
#pragma unroll
        for (int i = 0; i < N; ++i) qr[i] = q.lds[(I0 + i) * kLpr + lane % kLpr];
        typename ValuTile<D, BF16, N, N>::St s;
        tile_attend<D, BF16, N>(qr, r.k, r.v, t0, j1, lane % kLpr, lane / kLpr, static_cast<float *>(lds), scale_log2,
                                s.m, s.l, s.acc);
        put<N>(s, lane, m_w + I0 * ms, l_w + I0 * ms, ms, a_w + I0 * kAStride);
        if constexpr (I0 + N < KB) {
            __builtin_amdgcn_sched_barrier(0);   // the next group takes this one's registers
            attend_groups<I0 + N>(q, r, t0, j1, lane, lds, scale_log2, m_w, l_w, ms, a_w);
        }
    }

private:
    template <int N, class S>
    static __device__ __forceinline__ void put(const S &s, int lane, float *m_w, float *l_w, int ms, float *a_w) {
        if (lane < kLpr) {
#pragma unroll
            for (int i = 0; i < N; ++i) {
#pragma unroll
                for (int e = 0; e < kEpl; ++e) a_w[i * kAStride + lane * kEpl + e] = s.acc[i][e];
            }
        }
        if (lane == 0) {
#pragma unroll
            for (int i = 0; i < N; ++i) {
                m_w[i * ms] = s.m[i];
                l_w[i * ms] = s.l[i];
            }
        }
    }
};

// Value of x in lanes l & ~MASK and l | MASK (MASK = 16 or 32), in that
// order, in both lanes: combining the pair commutes nothing, so both lanes
// get bit-identical results.
template <int MASK>
__device__ __forceinline__ void lane_pair(float x, float &lo, float &hi) {
    const unsigned u = __float_as_uint(x);
    if constexpr (MASK == 16) {
        const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
        lo = __uint_as_float(r[0]);
        hi = __uint_as_float(r[1]);
    } else {
        const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
        lo = __uint_as_float(r[0]);
        hi = __uint_as_float(r[1]);
    }
}
// max / sum over the four lanes n, n + 16, n + 32, n + 48 of a column
__device__ __forceinline__ float col_max(float x) {
    float a, b;
    lane_pair<16>(x, a, b);
    x = fmaxf(a, b);
    lane_pair<32>(x, a, b);
    return fmaxf(a, b);
}
__device__ __forceinline__ float col_sum(float x) {
    float a, b;
    lane_pair<16>(x, a, b);
    x = a + b;
    lane_pair<32>(x, a, b);
    return a + b;
}

// bf16 tile on the matrix cores (v_mfma_f32_16x16x32_bf16; D = 32, 64, 128).
// The tile has T = 4096 / D keys (the row-load geometry of the VALU
// routine, so chunks are the same size).  K and V rows are loaded whole
// and coalesced, then pass through one swizzled LDS tile per wave (K first,
// then V in its place) to reach the operand layouts.  Lane l = 16 g + n:
//   QK^T  S^T[key][beam] = K[key][:] . q[beam][:]: the A operand is K
//         (lane: key 16 kb + n, 16 bytes at dim 32 s + 8 g), the B operand
//         the queries (column n = beam n < KB, the other columns zero).
//         Lane l gets the scores of beam n for keys 16 kb + 4 g + i.
//   softmax  per lane over its 4 NKB scores, then over the four lanes of
//         its column: every beam at once, no LDS.
//   PV    O^T[dim][beam] = V^T[dim][key] . P^T[key][beam].  P^T is the B
//         operand straight from the score registers (rounded to bf16; the
//         sum uses the rounded weights, so they add up to one).  V^T comes
//         from the tile's V rows staged in LDS and read back with
//         ds_read_b64_tr_b16, which transposes 16-bit elements within each
//         group of 16 lanes.  Lane l gets dims 16 mb + 4 g + i of beam n.
template <int D, int KB>
struct MfmaTile {
    static constexpr int T = 4096 / D;    // keys per tile
    static constexpr int NKB = T / 16;    // 16-key blocks
    static constexpr int NS = D / 32;     // 32-dim steps of QK^T
    static constexpr int NU = D / 16;     // 32-byte units per row = 16-dim output blocks
    static constexpr int kLpr = D / 8;    // 16-byte slices per row
    // a wave's LDS: one tile of rows (8 KB), K, then V, then the accumulators in its place
    static constexpr bool kGroups = false;
    static constexpr int kScratch = 0, kTileBytes = T * D * 2, kQBytes = 0;
    static_assert(D == 32 || D == 64 || D == 128, "MFMA tile needs D in {32, 64, 128}");
    static_assert(KB <= 16, "beams are the 16 columns of the MFMA");
    static_assert(NKB % 2 == 0, "PV takes 32 keys per instruction");
    struct Q { bf16x8_t b[NS]; };
    // floats between the beams of a wave's state in LDS: the 16 lanes of one
    // store (one beam each) land on distinct banks (a stride of D puts them
    // all on the same four banks)
    static constexpr int kAStride = D + 4;
    // column state of beam n = lane & 15: m, l identical in the column's
    // four lanes; acc[mb][i] holds dim 16 mb + 4 (lane >> 4) + i
    struct St { float m, l; f32x4_t acc[NU]; };

    // 32-byte unit of row r holding unit c: a XOR swizzle that spreads the
    // 16 rows of one transposed read over all LDS banks
    static __device__ __forceinline__ int unit(int r, int c) {
        constexpr int sh = NU == 2 ? 2 : NU == 4 ? 1 : 0;
        return c ^ ((r >> sh) & (NU - 1));
    }
    static __device__ __forceinline__ void load_q(Q &q, const uint4 *__restrict__ qp, size_t hyp0, int h, int H,
                                                  int lane, void * = nullptr) {
        const int n = lane & 15, g = lane >> 4;
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            uint4 v = make_uint4(0u, 0u, 0u, 0u);
            if (n < KB) v = qp[((hyp0 + n) * H + h) * kLpr + 4 * s + g];
            q.b[s] = __builtin_bit_cast(bf16x8_t, v);
        }
    }
    // row r of the tile (2 D bytes), 16-byte slice sl, in the swizzled LDS tile
    static __device__ __forceinline__ int lds_off(int r, int sl) {
        return r * (2 * D) + (unit(r, sl >> 1) << 5) + ((sl & 1) << 4);
    }
    static __device__ __forceinline__ void lds_fence() {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
    static __device__ __forceinline__ void attend(const Q &q, const Rows &rw, int t0, int j1, int lane, void *lds,
                                                  float scale_log2, St &st) {
        const int n = lane & 15, g = lane >> 4;
        constexpr int kRpi = kWave / kLpr;
        const int sub = lane % kLpr, grp = lane / kLpr;
        // K through LDS into the MFMA A layout: lane l takes row 16 kb + n,
        // dims 32 s + 8 g .. + 8
        char *vt = static_cast<char *>(lds);
#pragma unroll
        for (int u = 0; u < kIt; ++u) *reinterpret_cast<uint4 *>(vt + lds_off(u * kRpi + grp, sub)) = rw.k[u];
        lds_fence();
        uint4 ka[NKB][NS];
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb) {
#pragma unroll
            for (int s = 0; s < NS; ++s) ka[kb][s] = *reinterpret_cast<const uint4 *>(vt + lds_off(16 * kb + n, 4 * s + g));
        }
        lds_fence();
        // the V rows take the K rows' place (this wave's reads of K are done:
        // LDS instructions of one wave complete in order)
#pragma unroll
        for (int u = 0; u < kIt; ++u) *reinterpret_cast<uint4 *>(vt + lds_off(u * kRpi + grp, sub)) = rw.v[u];
        f32x4_t sc[NKB];
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb) {
            sc[kb] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int s = 0; s < NS; ++s)
                sc[kb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, ka[kb][s]), q.b[s],
                                                                 sc[kb], 0, 0, 0);
        }
        // scores in the base-2 domain; keys past j1 get weight zero
        float mx = -INFINITY;
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const bool ok = t0 + 16 * kb + 4 * g + i < j1;
                sc[kb][i] = ok ? sc[kb][i] * scale_log2 : -INFINITY;
                mx = fmaxf(mx, sc[kb][i]);
            }
        }
        mx = col_max(mx);  // finite: key t0 is valid
        bf16x8_t pb[NKB / 2];
        float ls = 0.f;
#pragma unroll
        for (int pp = 0; pp < NKB / 2; ++pp) {
            f32x8_t e;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                e[i] = __builtin_amdgcn_exp2f(sc[2 * pp][i] - mx);
                e[4 + i] = __builtin_amdgcn_exp2f(sc[2 * pp + 1][i] - mx);
            }
            pb[pp] = __builtin_convertvector(e, bf16x8_t);
#pragma unroll
            for (int i = 0; i < 8; ++i) ls += (float)pb[pp][i];
        }
        ls = col_sum(ls);
        lds_fence();
        // PV: MFMA pp contracts over keys [32 pp, 32 pp + 32) in the order
        // the score registers hold them: k = 8 g + j stands for key
        // 16 (2 pp + j / 4) + 4 g + j % 4.
        f32x4_t o[NU];
#pragma unroll
        for (int mb = 0; mb < NU; ++mb) o[mb] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int pp = 0; pp < NKB / 2; ++pp) {
#pragma unroll
            for (int mb = 0; mb < NU; ++mb) {
                i16x4_t t[2];
#pragma unroll
                for (int r = 0; r < 2; ++r) {
                    const int row = 32 * pp + 16 * r + 4 * g + (n >> 2);
                    const int off = row * (2 * D) + (unit(row, mb) << 5) + ((n & 3) << 3);
                    t[r] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                        (__attribute__((address_space(3))) i16x4_t *)(vt + off));
                }
                const auto a = __builtin_shufflevector(t[0], t[1], 0, 1, 2, 3, 4, 5, 6, 7);
                o[mb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a), pb[pp], o[mb],
                                                                0, 0, 0);
            }
        }
        // keep the next tile's LDS writes behind this tile's reads
        lds_fence();
        st.m = mx;
        st.l = ls;
#pragma unroll
        for (int mb = 0; mb < NU; ++mb) st.acc[mb] = o[mb];
    }
    static __device__ __forceinline__ void to_lds(const St &s, int lane, float *m_w, float *l_w, int ms, float *a_w) {
        const int n = lane & 15, g = lane >> 4;
        if (n < KB) {
#pragma unroll
            for (int mb = 0; mb < NU; ++mb)
                *reinterpret_cast<f32x4_t *>(a_w + n * kAStride + 16 * mb + 4 * g) = s.acc[mb];
            if (g == 0) {
                m_w[n * ms] = s.m;
                l_w[n * ms] = s.l;
            }
        }
    }
};

// Beams the VALU tile attends at a time in a workgroup of KW waves (0: the
// kernel of one chunk per workgroup, whose waves attend one tile each: all at
// once).  Its registers grow with the beams (eight: 146 without generated
// tokens, 185 with, and scratch in sixteen waves' 128), so from seven on, with
// generated tokens from six, they go in groups (104 and 143).  fp32, 8 beams,
// 192 rows of 700 keys: D = 64 24.2 us with all at once, 18.6 in groups of 4;
// 640 rows of 300 + 20: 46.0 and 33.5.  Pairs cost time where few rows leave
// each wave's chain of groups exposed (64 rows of 200 + 30: 8.6 us against 7.3).
constexpr int valu_group(bool bf16, int KB, bool gen, int KW) {
    if (KW == 0) return KB;
    if (gen) return KB < 6 ? KB : 2;
    return KB < 7 || bf16 ? KB : KB == 8 ? 4 : KW == 8 ? 2 : KB;
}
template <int D, bool BF16, int KB, bool GEN, int KW>
using Tile = typename std::conditional<(BF16 && D >= 32), MfmaTile<D, KB>,
                                       ValuTile<D, BF16, KB, valu_group(BF16, KB, GEN, KW)>>::type;

// Tile policy of a generated-token tile that belongs to one beam.  The matrix
// cores take the beam as one of the KB columns at no extra cost (only its
// column is used); the VALU tile attends it alone.
template <int D, bool BF16, int KB>
using OwnTile = typename std::conditional<(BF16 && D >= 32), MfmaTile<D, KB>, ValuTile<D, BF16, 1, 1>>::type;

// LDS area of one wave: its state's accumulators (KB rows of kAStride floats),
// the scratch of a tile of KB beams or of one beam from kScratch on, and its
// queries; 16-byte multiples.
template <int D, bool BF16, int KB, bool GEN, int KW>
struct WaveLds {
    using TL = Tile<D, BF16, KB, GEN, KW>;
    using TC = Tile<D, BF16, KB, GEN, 0>;   // of the kernel of one chunk (KW = kWaves)
    static constexpr int a = TL::kTileBytes, b = OwnTile<D, BF16, KB>::kTileBytes;
    static constexpr int c0 = KB * TL::kAStride * 4, c1 = KW == kWaves ? TC::kTileBytes : 0;
    static constexpr int c = c0 > c1 ? c0 : c1, d = TL::kScratch + (a > b ? a : b);
    static constexpr int kQ = ((c > d ? c : d) + 15) / 16 * 16;   // offset of the queries
    static constexpr int kBytes = kQ + TL::kQBytes;
};

// What the kWaves waves from w0 on left in LDS for output (beam i, dim d):
// their tiles' maxima and sums (beam-major, so one 16-byte read each) and
// accumulators.
struct TileStates {
    float m[kWaves], l[kWaves], a[kWaves];
};
template <int AS, class L>
__device__ __forceinline__ void load_states(L &lds, int w0, int i, int d, TileStates &s)
{
    static_assert(kWaves == 4, "four waves' maxima and sums in one read");
    const f32x4_t m = *reinterpret_cast<const f32x4_t *>(&lds.m[i][w0]);
    const f32x4_t l = *reinterpret_cast<const f32x4_t *>(&lds.l[i][w0]);
#pragma unroll
    for (int ww = 0; ww < kWaves; ++ww) {
        s.m[ww] = m[ww];
        s.l[ww] = l[ww];
        s.a[ww] = lds.acc(w0 + ww)[i * AS + d];
    }
}

// State of one chunk: its n tile states (the first n of s; the others, stale
// or of other tiles, are masked) scaled to their common maximum and added in
// key order.  Independent exponentials, where folding the tiles one by one
// into the row's state is a chain of them.
__device__ __forceinline__ void chunk_state(const TileStates &s, int n, float &m, float &l, float &a)
{
    m = -INFINITY;
#pragma unroll
    for (int ww = 0; ww < kWaves; ++ww) m = fmaxf(m, ww < n ? s.m[ww] : -INFINITY);
    const float ms = (m == -INFINITY) ? 0.f : m;
    l = 0.f;
    a = 0.f;
#pragma unroll
    for (int ww = 0; ww < kWaves; ++ww) {
        const float f = __builtin_amdgcn_exp2f((ww < n ? s.m[ww] : -INFINITY) - ms);
        l = fmaf(ww < n ? s.l[ww] : 0.f, f, l);
        a = fmaf(ww < n ? s.a[ww] : 0.f, f, a);
    }
}

// Merger for (b, h) = bh: merges the chunk records of a source with more
// than one chunk, in chunk order, and writes the normalised output.
//
// Each record word is (call tag << 32 | fp32 bits), written and read with
// device-scope atomics: every word is coherent across XCDs by itself, and
// the tag tells whether it was written by this call, so no fence or counter
// is needed.  The chunk workgroups have lower ids and were dispatched
// earlier, and they wait on nothing, so their records arrive; a word that
// does not carry this call's tag yet is re-read a bounded number of times,
// and the output becomes NaN if it never does (a loud failure instead of a
// silent wrong merge or an endless wait).
//
// The records are the row's chunk states, in key order (record slot c holds
// chunk c), folded one by one from the empty state.  With a generated-token
// segment (SPLIT), record slot NT of (b, h) holds the per-beam state of that
// segment; it is merged after the prefix chunks, and the merger also writes
// the rows whose prefix has at most one chunk.
template <int D, bool BF16, int KB, bool SPLIT>
__device__ __forceinline__ void merge_chunks(const unsigned long long *__restrict__ part,
                                             const int32_t *__restrict__ src_len, void *__restrict__ out,
                                             int bh, int n_bh, int H, Div by_H, int S, int NT, int t,
                                             unsigned long long epoch, unsigned long long *__restrict__ ctr)
{
    using G = Geo<D, BF16>;
    if (bh >= n_bh) return;
    const int b = by_H(bh);
    const int h = bh - b * H;
    const int L = min(max(src_len[b], 0), S);
    const int nc = (L + G::kChunk - 1) / G::kChunk;           // chunk records of the prefix, in key order
    if (!SPLIT && nc <= 1) return;                            // written by the chunk workgroup itself
    const int nrec = nc + (SPLIT && t > 0 ? 1 : 0);          // records to merge, in order
    constexpr int kRec = KB * (D + 2);
    unsigned long long c0 = 0;
    const unsigned long long tag = call_tag(epoch, ctr + bh, c0);
    const unsigned long long *recs = part + (size_t)bh * (NT + (SPLIT ? 1 : 0)) * kRec;
    bool stale_any = false;
    const size_t obase = ((size_t)b * KB * H + h) * D;
    constexpr int kBatch = 4;  // records whose words are loaded together
    for (int x = threadIdx.x; x < KB * D; x += kBlock) {
        const int i = x / D, d = x - i * D;
        const int at[3] = {KB * D + i, KB * D + KB + i, x};  // m, l, acc
        float mm = -INFINITY, ll = 0.f, aa = 0.f;
        bool stale = false;
        for (int c0 = 0; c0 < nrec; c0 += kBatch) {
            unsigned long long wv[kBatch][3];
#pragma unroll
            for (int q2 = 0; q2 < kBatch; ++q2) {
                // the generated-token record sits in slot NT
                const int slot = (SPLIT && c0 + q2 == nc) ? NT : c0 + q2;
#pragma unroll
                for (int f = 0; f < 3; ++f) {
                    wv[q2][f] = tag;
                    if (c0 + q2 < nrec)
                        wv[q2][f] = __hip_atomic_load(recs + (size_t)slot * kRec + at[f],
                                                      __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
            }
#pragma unroll
            for (int q2 = 0; q2 < kBatch; ++q2) {
                if (c0 + q2 >= nrec) break;
                const int slot = (SPLIT && c0 + q2 == nc) ? NT : c0 + q2;
#pragma unroll
                for (int f = 0; f < 3; ++f) {
                    const unsigned long long *a = recs + (size_t)slot * kRec + at[f];
                    for (int spin = 0; (wv[q2][f] & 0xffffffff00000000ull) != tag && spin < kMaxSpins; ++spin) {
                        __builtin_amdgcn_s_sleep(2);
                        wv[q2][f] = __hip_atomic_load(a, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    }
                    stale |= (wv[q2][f] & 0xffffffff00000000ull) != tag;
                }
                merge_state(mm, ll, aa, __uint_as_float((uint32_t)wv[q2][0]),
                            __uint_as_float((uint32_t)wv[q2][1]), __uint_as_float((uint32_t)wv[q2][2]));
            }
        }
        const float o = nrec == 0 ? 0.f : aa / ll;  // no key at all: zero row
        store_out<BF16>(out, obase + (size_t)i * H * D + d, stale ? NAN : o);
        stale_any |= stale;
    }
    // a captured call: every record of the row is in (or the wait ran out),
    // so every workgroup of the row has read the counter; the next call takes
    // the next value (skipping one after a wait that ran out, so that a late
    // record of this call can never pass for the next call's)
    const int any = __syncthreads_or(stale_any);
    if (epoch == 0 && threadIdx.x == 0)
        __hip_atomic_store(ctr + bh, c0 + (any ? 2 : 1), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Generated rows of one (source, head) row: Kt/Vt [B*k, H, T, D], rows < t,
// read directly or (anc != null) through the ancestry table.
struct GenRows {
    const uint4 *Kt, *Vt;
    int T, t;
    const int32_t *anc;
    int ld;
};

// LDS of a workgroup of KW waves that walks a row: each wave's tile area
// (which then holds its acc for the fold), its (max, sum) per beam, and for
// generated tiles the beam its task belongs to (-1: every beam) and, with an
// ancestry table (ANC), per tile of a batch whether the beams share it and the
// owners of its rows if so.
template <int D, bool BF16, int KB, int KW, bool GEN, bool ANC, bool BM>
struct RowLds {
    __attribute__((aligned(16))) float m[KB][KW], l[KB][KW];
    __attribute__((aligned(16))) char t[KW][WaveLds<D, BF16, KB, GEN, KW>::kBytes];
    int task[KW];
    // (tiles of more rows, D = 16 and 32 in bf16, would not fit beside 16 waves)
    static constexpr bool kOwners = ANC && !BM && Geo<D, BF16>::kTile <= kWave;
    unsigned char shared[kWave], owner[kOwners ? kWave : 1][Geo<D, BF16>::kTile];
    // generated tokens' states, where a wave walks a beam's (BM)
    float gm[BM ? KB : 1], gl[BM ? KB : 1], ga[BM ? KB : 1][D];
    __device__ __forceinline__ float *acc(int w) { return reinterpret_cast<float *>(&t[w][0]); }
    __device__ __forceinline__ void *scratch(int w) { return &t[w][Tile<D, BF16, KB, GEN, KW>::kScratch]; }
    __device__ __forceinline__ void *queries(int w) { return &t[w][WaveLds<D, BF16, KB, GEN, KW>::kQ]; }
};

// Running softmax state of a thread's outputs x = tid + p * threads (beam
// x / D, dim x % D).
template <int N>
struct OutState {
    float m[N], l[N], a[N];
    __device__ __forceinline__ void init() {
#pragma unroll
        for (int p = 0; p < N; ++p) {
            m[p] = -INFINITY;
            l[p] = 0.f;
            a[p] = 0.f;
        }
    }
};

// Generated tokens of the row's beams w, w + gw, ... (this wave's), each over
// its tiles in order, into lds.gm, gl and ga.  Through a table the owners of the
// next tile's rows are read while a tile's rows are on their way.
template <int D, bool BF16, int KB, int KW, bool ANC>
__device__ __forceinline__ void generated_beams(RowLds<D, BF16, KB, KW, true, ANC, true> &lds,
                                                const uint4 *__restrict__ q, int w, int gw, int b, int h, int H,
                                                const GenRows &gr, float scale_log2)
{
    using TO = OwnTile<D, BF16, 1>;   // of one query
    using G = Geo<D, BF16>;
    constexpr int kTile = G::kTile, kLpr = G::kLpr, kRpi = G::kRpi, kRow = kLpr * 16;
    const int lane = threadIdx.x & (kWave - 1);
    const size_t hyp0 = (size_t)b * KB;
    for (int i = w; i < KB; i += gw) {
        typename TO::Q qo;
        TO::load_q(qo, q, hyp0 + i, h, H, lane);
        // read through the table: from the source's beam-0 block on
        const size_t base = ((ANC ? hyp0 : hyp0 + i) * H + h) * (size_t)gr.T * kLpr;
        constexpr int kE = (D + kWave - 1) / kWave;
        float gm = -INFINITY, gl = 0.f, ga[kE];   // ga[e]: of dim (e * kWave + lane) % D
#pragma unroll
        for (int e = 0; e < kE; ++e) ga[e] = 0.f;
        int own[kIt] = {};   // owners of the next tile's rows, on their way during this one
        auto look = [&](int t0) {
            if constexpr (ANC) {
                const int32_t *row = gr.anc + (hyp0 + i) * gr.ld;
#pragma unroll
                for (int u = 0; u < kIt; ++u) own[u] = row[min(t0 + u * kRpi + lane / kLpr, gr.t - 1)];
            }
        };
        look(0);
        for (int t0 = 0; t0 < gr.t; t0 += kTile) {
            Rows rows;
            if constexpr (ANC) {
                const int stride = H * gr.T * kRow;   // bytes between two beams' blocks
                int off[kIt];
#pragma unroll
                for (int u = 0; u < kIt; ++u) {
                    const int j = t0 + u * kRpi + lane / kLpr;
                    const int o = (own[u] >= 0 && own[u] < KB) ? own[u] : i;
                    const int at = o * stride + j * kRow + lane % kLpr * 16;
                    off[u] = j < gr.t ? at : 0x7ffffff0;   // past the range: zero, no access
                }
                load_tile_at(rows, gr.Kt + base, gr.Vt + base, KB * stride, off);
                look(min(t0 + kTile, gr.t - 1));
            } else {
                load_tile<D, BF16, false>(rows, gr.Kt + base, gr.Vt + base, t0, gr.t, lane);
            }
            typename TO::St st;
            TO::attend(qo, rows, t0, gr.t, lane, lds.scratch(w), scale_log2, st);
            TO::to_lds(st, lane, &lds.m[0][w], &lds.l[0][w], KW, lds.acc(w));
            wave_lds_fence();
            const float tm = lds.m[0][w], tl = lds.l[0][w];
#pragma unroll
            for (int e = 0; e < kE; ++e) {
                float m = gm, l = gl;   // the same for every dim
                merge_state(m, l, ga[e], tm, tl, lds.acc(w)[(e * kWave + lane) % D]);
                if (e == kE - 1) {
                    gm = m;
                    gl = l;
                }
            }
            wave_lds_fence();
        }
#pragma unroll
        for (int e = 0; e < kE; ++e)
            if (e * kWave + lane < D) lds.ga[i][e * kWave + lane] = ga[e];
        if (lane == 0) {
            lds.gm[i] = gm;
            lds.gl[i] = gl;
        }
    }
}

// One (source, head) row walked by the KW waves of a workgroup in rounds of
// KW tile tasks, one task per wave: the npt tiles of the prefix (Kbh/Vbh, L
// keys), then with GEN the tiles of the generated tokens.  R receives the
// prefix state (its chunks of kWaves tiles folded in key order), Gs the
// generated tokens' state (tiles folded in key order), so the bits depend on
// neither KW nor the rounds.
//
// A generated tile is one task per beam, over that beam's rows.  Through an
// ancestry table (ANC), a tile whose rows have the same owner for every beam
// -- beam search soon leaves one ancestor for all but the latest tokens -- is
// one task for all of them, read once like a prefix tile.  The split cache
// with 512 generated rows and 5 beams (512 rows of 75 to 300 prefix keys)
// took 72 us when the first four waves walked each beam's tiles in turn; the
// tasks spread over all waves take 23 us.  With BM (beam_waves) the first waves
// do walk each beam's tiles, in the place of the round's first tasks: the VALU
// tile of a beam and that of all beams do not share a loop then, which in one
// cost up to 80 registers more.
//
// The latest generated tile is one task per beam in any case (each beam's
// last token is its own).  Its tasks go first, beside the first prefix tiles:
// its rows lie in k separate blocks of memory, which a last round of a few
// waves reads slowly (192 rows of up to 1024 prefix keys, 64 generated, k = 4:
// 12.0 us, against 12.2 us with every generated tile after the prefix).
template <int D, bool BF16, int KB, int KW, bool GEN, bool ANC, bool BM>
__device__ __forceinline__ void walk_row(RowLds<D, BF16, KB, KW, GEN, ANC, BM> &lds,
                                         const typename Tile<D, BF16, KB, GEN, KW>::Q &qv,
                                         const uint4 *__restrict__ q, const uint4 *__restrict__ Kbh,
                                         const uint4 *__restrict__ Vbh, int L, int b, int h, int H, const GenRows &gr,
                                         float scale_log2, OutState<(KB * D + KW * kWave - 1) / (KW * kWave)> &R,
                                         OutState<(KB * D + KW * kWave - 1) / (KW * kWave)> &Gs,
                                         unsigned long long *trs)
{
    using G = Geo<D, BF16>;
    using TL = Tile<D, BF16, KB, GEN, KW>;
    using TO = OwnTile<D, BF16, KB>;
    using Lds = RowLds<D, BF16, KB, KW, GEN, ANC, BM>;
    constexpr bool kOwnIsTile = std::is_same<TL, TO>::value;
    constexpr int kTile = G::kTile, kLpr = G::kLpr, kRpi = G::kRpi;
    // Rows of the next round on their way during this round's fold.  Where
    // there is a next round (the size rule gives four waves one round of prefix
    // tiles) and the registers for it (D = 64: 124, four waves per SIMD) are
    // there: with D = 128, the VALU tile or generated tokens it costs a wave
    // per SIMD, with D = 32 and 16 waves it spills.
    constexpr bool kAhead = BF16 && (D == 64 || (D == 32 && KW < 16)) && !GEN && KW > kWaves;
    constexpr int kThreads = KW * kWave, kPer = (KB * D + kThreads - 1) / kThreads;
    constexpr int kBatch = kWave;   // generated tiles whose sharing one ballot holds
    const int tid = threadIdx.x, lane = tid & (kWave - 1), w = wave_id();
    const int npt = (L + kTile - 1) / kTile;
    const int ngt = GEN && !BM ? (gr.t + kTile - 1) / kTile : 0;
    const size_t hyp0 = (size_t)b * KB;
    float *const m_w = &lds.m[0][w], *const l_w = &lds.l[0][w];   // beam i at i * KW

    // Early tasks (below) keep their states in registers, which the VALU tile
    // has for D = 16 and for five beams without a table only.
    constexpr bool kEarly = GEN && KB >= kWaves && !BM && ((BF16 && D >= 32) || D == 16 || (KB == 5 && !ANC));
    // waves that walk beams in the place of the first tasks (a multiple of
    // kWaves): one per beam, but half as many of eight where the others take
    // the whole prefix meanwhile
    int beams = 0;
    if constexpr (BM) {
        if (gr.t > 0) beams = kWaves;
        if (KB > kWaves && KW > kWaves &&
            (KW > 2 * kWaves || npt == 0 || npt > KW - kWaves || gr.t > 2 * kTile)) beams *= 2;
        if (w < beams) generated_beams<D, BF16, KB, KW, ANC>(lds, q, w, beams, b, h, H, gr, scale_log2);
    }
    R.init();
    OutState<kPer> last;   // the early tasks' states, folded at the end
    if constexpr (GEN) {
        Gs.init();
        if constexpr (kEarly) last.init();
    }

    // owner of generated row j of beam i, in [0, KB)
    auto owner = [&](int a, int i) { return (a >= 0 && a < KB) ? a : i; };

    for (int gb = 0; gb == 0 || gb < ngt; gb += kBatch) {
        const int npre = gb == 0 ? npt : 0;
        const int ng = min(kBatch, ngt - gb);
        // the tasks before the prefix: beams 0 .. early - 1 of the last tile
        // (a multiple of kWaves, so that the prefix's chunks stay aligned)
        const int early = BM ? beams : kEarly && ng > 0 && ngt <= kBatch ? KB / kWaves * kWaves : 0;
        const int pre1 = early + npre;   // end of the prefix tasks
        unsigned long long sh = 0;      // tiles of the batch with one owner per row for every beam
        int ntask = BM ? pre1 : npre + ng * KB;
        // Does tile jt of the batch have one owner per row?  (one wave per
        // tile, which leaves the owners in LDS)
        auto mark_shared = [&]() {
            for (int jt = w; jt < ng; jt += KW) {
                bool same = KB == 1 || gb + jt < ngt - 1;
                for (int p = lane; same && p < kTile; p += kWave) {
                    const int j = min((gb + jt) * kTile + p, gr.t - 1);   // past t with one beam only
                    const int32_t *col = gr.anc + hyp0 * gr.ld + j;
                    int a[KB];
#pragma unroll
                    for (int i = 0; i < KB; ++i) a[i] = col[(size_t)i * gr.ld];
#pragma unroll
                    for (int i = 1; i < KB; ++i) same &= owner(a[i], i) == owner(a[0], 0);
                    if (Lds::kOwners) lds.owner[jt][p] = (unsigned char)owner(a[0], 0);
                }
                const bool all = __builtin_amdgcn_ballot_w64(!same) == 0ull;
                if (lane == 0) lds.shared[jt] = all;
            }
        };
        auto read_shared = [&]() {
            sh = __builtin_amdgcn_ballot_w64(lane < ng && lds.shared[lane] != 0);
            ntask = npre + ng * KB - (int)__popcll(sh) * (KB - 1);
        };
        // This wave's position in the batch's generated tasks (tile by tile,
        // in each the shared task or one per beam); advances with the rounds.
        int cur_tile = 0, cur_first = pre1;
        int g_tile = 0, g_beam = 0;
        auto locate = [&](int task) {
            if (task < early) {
                g_tile = ng - 1;
                g_beam = task;
            } else if constexpr (ANC) {
                for (;;) {
                    const int c = (sh >> cur_tile) & 1ull ? 1 : KB;
                    if (task < cur_first + c) break;
                    cur_first += c;
                    ++cur_tile;
                }
                g_tile = cur_tile;
                g_beam = (sh >> cur_tile) & 1ull ? -1 : task - cur_first;
            } else {
                g_tile = (task - pre1) / KB;
                g_beam = (task - pre1) - g_tile * KB;
            }
            if (task >= early && g_tile == ng - 1) g_beam += early;   // never shared (or KB == 1: early == 0)
        };
        // This wave's task of a round: where its keys are, and its loads.  A
        // task read through the table first needs the table entries of its
        // rows (find), then its rows' loads go out (fetch).
        Rows rows;
        typename TO::Q qo;
        int own[kIt] = {};   // (fetch reads it for prefix tasks too, times a stride of 0)
        int t0 = 0, j1 = 0;
        bool gen = false;
        auto find = [&](int task) {
            gen = GEN && !BM && (task < early || task >= pre1);
            t0 = (task - early) * kTile;
            j1 = task < ntask ? L : 0;   // no task: loads of an empty range
            if (!gen || task >= ntask) return;
            locate(task);
            t0 = (gb + g_tile) * kTile;
            j1 = gr.t;
            if constexpr (ANC) {
                if (Lds::kOwners && g_beam < 0) {
#pragma unroll
                    for (int u = 0; u < kIt; ++u) own[u] = lds.owner[g_tile][u * kRpi + lane / kLpr];
                } else {
                    const int32_t *row = gr.anc + (hyp0 + max(g_beam, 0)) * gr.ld;
#pragma unroll
                    for (int u = 0; u < kIt; ++u) own[u] = row[min(t0 + u * kRpi + lane / kLpr, gr.t - 1)];
                }
            }
            if constexpr (!kOwnIsTile) {
                if (g_beam >= 0) TO::load_q(qo, q, hyp0 + g_beam, h, H, lane);
            }
        };
        auto fetch = [&]() {
            constexpr int kRow = kLpr * 16;
            const uint4 *Kw = Kbh, *Vw = Vbh;
            if constexpr (GEN) {
                if (gen) {
                    // read through the table: from the source's beam-0 block on
                    const size_t base = ((ANC ? hyp0 : hyp0 + g_beam) * H + h) * (size_t)gr.T * kLpr;
                    Kw = gr.Kt + base;
                    Vw = gr.Vt + base;
                }
            }
            if constexpr (ANC) {
                const int stride = gen ? H * gr.T * kRow : 0;   // bytes between two beams' blocks
                int off[kIt];
#pragma unroll
                for (int u = 0; u < kIt; ++u) {
                    const int j = t0 + u * kRpi + lane / kLpr;
                    const int at = owner(own[u], max(g_beam, 0)) * stride + j * kRow + lane % kLpr * 16;
                    off[u] = j < j1 ? at : 0x7ffffff0;   // past the range: zero, no access
                }
                load_tile_at(rows, Kw, Vw, gen ? KB * stride : j1 * kRow, off);
            } else {
                load_tile<D, BF16, kAhead>(rows, Kw, Vw, t0, j1, lane);
            }
        };
        bool marked = !(ANC && ng > 0);
        if constexpr (ANC) {
            // when the first round needs no more than the early tasks and
            // prefix tiles, the table is looked at after its loads have gone out
            if (!marked && pre1 < KW) {
                mark_shared();
                lds_barrier();
                read_shared();
                marked = true;
            }
        }
        find(w);
        if constexpr (kAhead) fetch();
        for (int q0 = 0; q0 < ntask; q0 += KW) {
            const int task = q0 + w;
            if (task < ntask && !(BM && task < early)) {
                if constexpr (GEN && !BM) {
                    if (gen && lane == 0) lds.task[w] = g_beam;
                }
                // the loads beside their use: the VALU tile takes its V rows late
                if (kOwnIsTile || BM || !gen || g_beam < 0) {
                    if constexpr (!kAhead) fetch();
                    if constexpr (TL::kGroups) {
                        TL::attend_groups(qv, rows, t0, j1, lane, lds.scratch(w), scale_log2, m_w, l_w, KW, lds.acc(w));
                    } else {
                        typename TL::St st;
                        TL::attend(qv, rows, t0, j1, lane, &lds.t[w][0], scale_log2, st);
                        TL::to_lds(st, lane, m_w, l_w, KW, lds.acc(w));
                    }
                } else if constexpr (!kOwnIsTile) {
                    typename TO::St st;
                    fetch();
                    TO::attend(qo, rows, t0, j1, lane, lds.scratch(w), scale_log2, st);
                    TO::to_lds(st, lane, m_w + g_beam * KW, l_w + g_beam * KW, KW, lds.acc(w) + g_beam * TL::kAStride);
                }
            }
            bool fresh = false;
            if constexpr (ANC) {
                if (!marked) {
                    mark_shared();
                    marked = fresh = true;
                }
            }
            lds_barrier();
            if constexpr (ANC) {
                if (fresh) read_shared();
            }
            // the next round's rows, or the table entries they are found by,
            // are on their way during the fold
            if (q0 + KW < ntask) {   // of the workgroup: no branch parts a wave from its loads
                find(task + KW);
                if constexpr (kAhead) fetch();
            }
#pragma unroll
            for (int p = 0; p < kPer; ++p) {
                const int x = tid + p * kThreads;
                if (x < KB * D) {
                    const int i = x / D, d = x - i * D;
                    if constexpr (BM) {
                        if (q0 == 0 && beams) {
                            Gs.m[p] = lds.gm[i];
                            Gs.l[p] = lds.gl[i];
                            Gs.a[p] = lds.ga[i][d];
                        }
                    }
                    if constexpr (kEarly) {
                        const int we = i - q0;   // the wave of beam i's early task
                        if (q0 < early && i < early && we >= 0 && we < KW) {
                            last.m[p] = lds.m[i][we];
                            last.l[p] = lds.l[i][we];
                            last.a[p] = lds.acc(we)[i * TL::kAStride + d];
                        }
                    }
#pragma unroll
                    for (int g = 0; g < KW / kWaves; ++g) {
                        const int n = pre1 - (q0 + g * kWaves);   // prefix tiles of this chunk, if any
                        if (n > 0 && q0 + g * kWaves >= early) {
                            TileStates ts;
                            float cm, cl, ca;
                            load_states<TL::kAStride>(lds, g * kWaves, i, d, ts);
                            chunk_state(ts, n, cm, cl, ca);
                            merge_state(R.m[p], R.l[p], R.a[p], cm, cl, ca);
                        }
                    }
                    if constexpr (GEN && !BM) {
                        // generated tiles, those of this beam, in order
                        for (int ww = max(pre1 - q0, 0); ww < min(KW, ntask - q0); ++ww) {
                            const int tb = __builtin_amdgcn_readfirstlane(lds.task[ww]);
                            if (tb < 0 || tb == i)
                                merge_state(Gs.m[p], Gs.l[p], Gs.a[p], lds.m[i][ww], lds.l[i][ww],
                                            lds.acc(ww)[i * TL::kAStride + d]);
                        }
                    }
                }
            }
            if (q0 + KW < ntask || gb + kBatch < ngt) lds_barrier();
            if (gb == 0 && q0 == 0) trace::stamp(trs, 5);
        }
    }
    if constexpr (kEarly) {
#pragma unroll
        for (int p = 0; p < kPer; ++p) merge_state(Gs.m[p], Gs.l[p], Gs.a[p], last.m[p], last.l[p], last.a[p]);
    }
}

// Generated-token segment of (b, h) = bh (SPLIT only): its state goes to
// record slot NT of (b, h).
template <int D, bool BF16, int KB, bool ANC, bool BM>
__device__ __forceinline__ void attend_generated(RowLds<D, BF16, KB, kWaves, true, ANC, BM> &lds,
                                                 const uint4 *__restrict__ q,
                                                 unsigned long long *__restrict__ part, int bh, int n_bh, int H,
                                                 Div by_H, int NT, const GenRows &gr, float scale_log2,
                                                 unsigned long long epoch,
                                                 const unsigned long long *__restrict__ ctr)
{
    using TL = Tile<D, BF16, KB, true, kWaves>;
    constexpr int kPer = (KB * D + kBlock - 1) / kBlock;
    if (bh >= n_bh || gr.t <= 0) return;
    const int b = by_H(bh);
    const int h = bh - b * H;
    constexpr int kRec = KB * (D + 2);
    unsigned long long c0;
    const unsigned long long tag = call_tag(epoch, ctr + bh, c0);
    typename TL::Q qv;
    TL::load_q(qv, q, (size_t)b * KB, h, H, threadIdx.x & (kWave - 1), lds.queries(wave_id()));
    OutState<kPer> R, Gs;
    walk_row<D, BF16, KB, kWaves, true, ANC, BM>(lds, qv, q, nullptr, nullptr, 0, b, h, H, gr, scale_log2, R, Gs,
                                                 nullptr);
    unsigned long long *rec = part + ((size_t)bh * (NT + 1) + NT) * kRec;
#pragma unroll
    for (int p = 0; p < kPer; ++p) {
        const int x = threadIdx.x + p * kBlock;
        if (x < KB * D) {
            store_word(rec + x, tag, Gs.a[p]);
            if (x % D == 0) {
                store_word(rec + KB * D + x / D, tag, Gs.m[p]);
                store_word(rec + KB * D + KB + x / D, tag, Gs.l[p]);
            }
        }
    }
}

template <int D, bool BF16, int KB, bool SPLIT, bool ANC, bool BM>
__global__ __launch_bounds__(kBlock) void cross_attn_kernel(
    const uint4 *__restrict__ q, const uint4 *__restrict__ K, const uint4 *__restrict__ V,
    const int32_t *__restrict__ src_len, int ng_blocks, int n_bh, int H, unsigned h_mul, int h_shift, int NC, int S,
    float scale_log2, void *__restrict__ out,
    unsigned long long *__restrict__ part, unsigned long long epoch,
    unsigned long long *__restrict__ ctr,
    const uint4 *__restrict__ Kt, const uint4 *__restrict__ Vt, int T, int t, const int32_t *__restrict__ anc,
    int ld_anc, NgramJob ngj)
{
    using G = Geo<D, BF16>;
    using TL = Tile<D, BF16, KB, SPLIT, 0>;
    constexpr int kLpr = G::kLpr;
    constexpr int kTile = G::kTile, kChunk = G::kChunk;

    const Div by_H{h_mul, h_shift};
    // A fused decode step's n-gram rows take the first workgroups (a
    // multiple of 8, so the XCD residues of the ids below are kept).
    if ((int)blockIdx.x < ng_blocks) {
        ngram_job_block(ngj, blockIdx.x, kWaves);
        return;
    }

    __shared__ RowLds<D, BF16, KB, kWaves, SPLIT, ANC, BM> lds;

    // Workgroup g runs on XCD g % 8 (round-robin dispatch).  All chunks of
    // one (b, h), its generated-token workgroup and its merger get ids with
    // the same residue, so they share an L2.  Order of the id ranges: the
    // generated-token workgroups (SPLIT only; each walks its tiles in
    // sequence, so they start first), the chunk workgroups, the mergers.
    const int n_bh8 = ((n_bh + kXcds - 1) / kXcds) * kXcds;
    int g = blockIdx.x - ng_blocks;
    if constexpr (SPLIT) {
        if (g < n_bh8) {
            attend_generated<D, BF16, KB, ANC, BM>(lds, q, part, g, n_bh, H, by_H, NC * kWaves,
                                               GenRows{Kt, Vt, T, t, anc, ld_anc}, scale_log2, epoch, ctr);
            return;
        }
        g -= n_bh8;
    }
    const int n_chunk_blocks = n_bh8 * NC;
    if (g >= n_chunk_blocks) {
        merge_chunks<D, BF16, KB, SPLIT>(part, src_len, out, g - n_chunk_blocks, n_bh, H, by_H, S, NC * kWaves, t, epoch,
                                         ctr);
        return;
    }
    const int xcd = g % kXcds;
    const int slot = g / kXcds;
    const int bh = (slot / NC) * kXcds + xcd;
    const int c = slot - (slot / NC) * NC;
    if (bh >= n_bh) return;
    const int b = by_H(bh);
    const int h = bh - b * H;
    const int L = min(max(src_len[b], 0), S);
    const int j0 = c * kChunk;
    const int nc = (L + kChunk - 1) / kChunk;
    const int tid = threadIdx.x;
    const size_t obase = ((size_t)b * KB * H + h) * D;  // out[b, 0, h, 0]
    if (!SPLIT && L == 0) {  // no valid key: the output row is zero
        if (c == 0)
            for (int x = tid; x < KB * D; x += kBlock)
                store_out<BF16>(out, obase + (size_t)(x / D) * H * D + x % D, 0.f);
        return;
    }
    if (c >= nc) return;  // chunk lies in the padding: never read
    const int j1 = min(j0 + kChunk, L);
    // the call's tag (for a captured call a load, issued before the row's)
    unsigned long long c0;
    const unsigned long long tag = call_tag(epoch, ctr + bh, c0);

    const int lane = tid & (kWave - 1);
    const int w = wave_id();

    const int t0 = j0 + w * kTile;
    Rows rows;
    if (t0 < j1) load_tile<D, BF16, false>(rows, K + (size_t)bh * S * kLpr, V + (size_t)bh * S * kLpr, t0, j1, lane);
    typename TL::Q qv;
    TL::load_q(qv, q, (size_t)b * KB, h, H, lane);
    if (t0 < j1) {
        typename TL::St st;
        TL::attend(qv, rows, t0, j1, lane, &lds.t[w][0], scale_log2, st);
        TL::to_lds(st, lane, &lds.m[0][w], &lds.l[0][w], kWaves, lds.acc(w));
    }
    __syncthreads();

    // The chunk's state.  A whole row (one chunk) is folded from the empty
    // state and finished here; otherwise it goes to record slot c of the row:
    // acc[KB][D], then m[KB], then l[KB].
    const int ntile = min(kWaves, (j1 - j0 + kTile - 1) / kTile);   // tiles of this chunk that hold keys
    unsigned long long *rec = part + ((size_t)bh * (NC * kWaves + (SPLIT ? 1 : 0)) + c) * (KB * (D + 2));
    for (int x = tid; x < KB * D; x += kBlock) {
        const int i = x / D, d = x - i * D;
        float cm, cl, ca;
        TileStates ts;
        load_states<TL::kAStride>(lds, 0, i, d, ts);
        chunk_state(ts, ntile, cm, cl, ca);
        if (!SPLIT && nc == 1) {
            float mm = -INFINITY, ll = 0.f, aa = 0.f;
            merge_state(mm, ll, aa, cm, cl, ca);
            store_out<BF16>(out, obase + (size_t)i * H * D + d, aa / ll);
        } else {
            store_word(rec + x, tag, ca);
            if (d == 0) {
                store_word(rec + KB * D + i, tag, cm);
                store_word(rec + KB * D + KB + i, tag, cl);
            }
        }
    }
}

// One workgroup per (b, h) that walks all of its tiles itself (walk_row): no
// partial records, no merger, no cross-workgroup wait.  The arithmetic and
// its order are those of cross_attn_kernel -- each chunk's tile states
// combined, the chunk states folded in chunk order from the empty state, the
// generated-token state last -- so both kernels give the same bits.  It pays
// when there are enough (b, h) rows to fill the chip without splitting them.
template <int D, bool BF16, int KB, bool SPLIT, int P, bool ANC, bool BM>
__global__ __launch_bounds__(kBlock * P) void attn_whole_kernel(
    const uint4 *__restrict__ q, const uint4 *__restrict__ K, const uint4 *__restrict__ V,
    const int32_t *__restrict__ src_len, int ng_blocks, int H, unsigned h_mul, int h_shift, int S, float scale_log2,
    void *__restrict__ out, const uint4 *__restrict__ Kt, const uint4 *__restrict__ Vt, int T, int t,
    const int32_t *__restrict__ anc, int ld_anc, NgramJob ngj)
{
    using G = Geo<D, BF16>;
    constexpr int kLpr = G::kLpr;
    constexpr int kW = kWaves * P;                        // waves per workgroup
    using TL = Tile<D, BF16, KB, SPLIT, kW>;
    constexpr int kThreads = kBlock * P;
    constexpr int kPer = (KB * D + kThreads - 1) / kThreads;  // outputs per thread

    __shared__ RowLds<D, BF16, KB, kW, SPLIT, ANC, BM> lds;

    const Div by_H{h_mul, h_shift};
    // A fused decode step's n-gram rows take the first workgroups.
    if ((int)blockIdx.x < ng_blocks) {
        ngram_job_block(ngj, blockIdx.x, kW);
        return;
    }
    const int bh = blockIdx.x - ng_blocks;   // the grid holds no workgroup past the rows
    // trace words: 0 start, 1 end, 2 hardware ids, 3 row, 4 jobs, 5 first round folded
    unsigned long long *trs = trace_slot();
    trace::stamp(trs, 0);
    const int b = by_H(bh);
    const int h = bh - b * H;
    int L = 0;
    if (!SPLIT || S > 0) L = min(max(src_len[b], 0), S);   // without a prefix, no trip to memory for its length
    const int tid = threadIdx.x;
    const size_t obase = ((size_t)b * KB * H + h) * D;  // out[b, 0, h, 0]
    typename TL::Q qv;
    TL::load_q(qv, q, (size_t)b * KB, h, H, tid & (kWave - 1), lds.queries(wave_id()));
    OutState<kPer> R, Gs;
    walk_row<D, BF16, KB, kW, SPLIT, ANC, BM>(lds, qv, q, K + (size_t)bh * S * kLpr, V + (size_t)bh * S * kLpr, L, b, h,
                                              H, GenRows{Kt, Vt, T, t, anc, ld_anc}, scale_log2, R, Gs, trs);
    if constexpr (SPLIT) {
        if (t > 0) {
#pragma unroll
            for (int p = 0; p < kPer; ++p) merge_state(R.m[p], R.l[p], R.a[p], Gs.m[p], Gs.l[p], Gs.a[p]);
        }
    }
    const int njobs = (L + G::kChunk - 1) / G::kChunk + (SPLIT && t > 0 ? 1 : 0);   // chunks, generated tokens
    const bool any = njobs > 0;
#pragma unroll
    for (int p = 0; p < kPer; ++p) {
        const int x = tid + p * kThreads;
        if (x < KB * D) {
            const int i = x / D, d = x - i * D;
            store_out<BF16>(out, obase + (size_t)i * H * D + d, any ? R.a[p] / R.l[p] : 0.f);  // no key: zero row
        }
    }
    trace::stamp(trs, 1);
    trace::put(trs, 2, trace::where());
    trace::put(trs, 3, (unsigned long long)bh);
    trace::put(trs, 4, (unsigned long long)njobs);
}

}  // namespace

// Whether a wave walks a beam's generated tokens by itself.  Without a table
// every beam's rows are read in any case.  On the vector tile the loop of tasks
// costs the registers of two tiles then; on the matrix cores a wave per beam
// saves the barrier and the fold that tasks take every KW tiles, which pays
// from a few tiles on (us, bf16, D = 64, 8 beams, 144 rows of 0 + 300: beams
// 18.3, tasks 22.6; D = 128, 4 beams: 18.9 and 23.4).  Through a table,
// tasks read what the beams share once, which pays from the second tile on; on
// the vector tile a beam's wave saves the look at the table (us, fp32, D = 64,
// k = 8, 300 keys, n rows, t tokens, beams' waves / tasks: n = 256, t = 20 19 /
// 23; n = 640, t = 500 128 / 91).
inline bool beam_waves(int n_bh, int D, int esize, int k, int nt, int t, bool table) {
    const int tile = kIt * kWave * 16 / (D * esize);
    if (esize == 2 && D >= 32) return !table && k >= 4 && t > tile * (k >= 6 ? 1 : 3);
    if (!table) return D == 16 ? k >= 3 : k == 4 || k >= 6;
    if (k < (D == 16 ? 3 : 4)) return false;
    const bool few = n_bh <= kCus || (nt == 0 && D > 16 && k >= 6);
    return t <= tile * (!few ? 1 : k >= 6 ? 3 : D == 16 && esize == 2 ? 2 : 1);
}

// Launch arguments shared by both entry points.  For the encoder-decoder
// form Kt/Vt are null and T = t = 0.
struct AttnArgs {
    const void *q, *K, *V;
    const int32_t *src_len;
    void *out;
    int B, k, H, S, D;
    const void *Kt, *Vt;
    int T, t;
    const int32_t *anc;   // ancestry table of the generated rows, or null
    int ld_anc;
    float *ws;
    unsigned long long epoch;
    hipStream_t stream;
    NgramJob ng;          // n-gram rows of a fused decode step (ng.rows == 0: none)
    AttnPath path;        // decomposition chosen for the call
    bool beams;           // generated tokens by beam_waves, where there are both kernels
};

namespace {

template <int D, bool BF16, int KB, bool SPLIT, bool ANC, bool BM>
hipError_t launch_split(const AttnArgs &a, int NC)
{
    const int n_bh = a.B * a.H;
    const long long n_bh8 = ((long long)n_bh + kXcds - 1) / kXcds * kXcds;
    const double scale_log2 = 1.4426950408889634074 / sqrt((double)D);
    unsigned long long *part = reinterpret_cast<unsigned long long *>(a.ws);
    // the rows' counters for captured calls follow the records
    unsigned long long *ctr = part + (size_t)n_bh * (NC * kWaves + (SPLIT ? 1 : 0)) * (KB * (D + 2));
    // [generated-token workgroups] [chunk workgroups] [mergers]
    const long long mergers = (SPLIT || NC > 1) ? n_bh : 0;
    // n-gram workgroups first, rounded to a multiple of 8 so that the XCD
    // residues of the ids after them are kept
    NgramJob ng = a.ng;
    ng.blocks = ng.rows > 0 ? (ng.rows + kWaves - 1) / kWaves : 0;
    ng.blocks = (ng.blocks + kXcds - 1) / kXcds * kXcds;
    const long long nblk = ng.blocks + (SPLIT ? n_bh8 : 0) + n_bh8 * NC + mergers;
    const Div dv = make_div(a.H);
    hipLaunchKernelGGL((cross_attn_kernel<D, BF16, KB, SPLIT, ANC, BM>), dim3((unsigned)nblk), dim3(kBlock), 0,
                       a.stream, static_cast<const uint4 *>(a.q), static_cast<const uint4 *>(a.K),
                       static_cast<const uint4 *>(a.V), a.src_len, ng.blocks, n_bh, a.H, dv.mul, dv.shift, NC, a.S,
                       (float)scale_log2, a.out, part, a.epoch, ctr, static_cast<const uint4 *>(a.Kt),
                       static_cast<const uint4 *>(a.Vt), a.T, a.t, a.anc, a.ld_anc, ng);
    return hipGetLastError();
}

template <int D, bool BF16, int KB, bool SPLIT, int P, bool ANC, bool BM>
hipError_t launch_whole(const AttnArgs &a)
{
    const int n_bh = a.B * a.H;
    const double scale_log2 = 1.4426950408889634074 / sqrt((double)D);
    NgramJob ng = a.ng;
    ng.blocks = ng.rows > 0 ? (ng.rows + kWaves * P - 1) / (kWaves * P) : 0;
    const Div dv = make_div(a.H);
    hipLaunchKernelGGL((attn_whole_kernel<D, BF16, KB, SPLIT, P, ANC, BM>), dim3((unsigned)(ng.blocks + n_bh)),
                       dim3(kBlock * P), 0,
                       a.stream, static_cast<const uint4 *>(a.q), static_cast<const uint4 *>(a.K),
                       static_cast<const uint4 *>(a.V), a.src_len, ng.blocks, a.H, dv.mul, dv.shift, a.S,
                       (float)scale_log2, a.out,
                       static_cast<const uint4 *>(a.Kt), static_cast<const uint4 *>(a.Vt), a.T, a.t, a.anc,
                       a.ld_anc, ng);
    return hipGetLastError();
}

template <int D, bool BF16, int KB, bool SPLIT, bool ANC, bool BM>
hipError_t launch_path(const AttnArgs &a)
{
    // at least one chunk column, so that a source with no valid key (or
    // S == 0) still has a workgroup to write its zero output
    constexpr int kChunk = Geo<D, BF16>::kChunk;
    switch (a.path) {
    case AttnPath::kWhole1: return launch_whole<D, BF16, KB, SPLIT, 1, ANC, BM>(a);
    case AttnPath::kWhole2: return launch_whole<D, BF16, KB, SPLIT, 2, ANC, BM>(a);
    case AttnPath::kWhole4: return launch_whole<D, BF16, KB, SPLIT, 4, ANC, BM>(a);
    default: return launch_split<D, BF16, KB, SPLIT, ANC, BM>(a, max(1, (a.S + kChunk - 1) / kChunk));
    }
}

template <int D, bool BF16, int KB, bool SPLIT>
hipError_t launch_typed(const AttnArgs &a)
{
    if constexpr (SPLIT) {
        // Generated rows through the ancestry table: their own kernels, so that
        // the table-free ones keep their registers.
        constexpr bool kValu = !(BF16 && D >= 32);
        if (a.anc) {
            if constexpr (kValu && KB >= (D == 16 ? 3 : 4)) {
                if (a.beams) return launch_path<D, BF16, KB, true, true, true>(a);
            }
            return launch_path<D, BF16, KB, true, true, false>(a);
        }
        if constexpr (!kValu && KB >= 4) {
            if (!a.beams) return launch_path<D, BF16, KB, true, false, false>(a);
            return launch_path<D, BF16, KB, true, false, true>(a);
        } else {
            return launch_path<D, BF16, KB, true, false, kValu && (D == 16 ? KB >= 3 : KB == 4 || KB >= 6)>(a);
        }
    } else {
        return launch_path<D, BF16, KB, false, false, false>(a);
    }
}

template <int D, bool BF16, bool SPLIT>
hipError_t launch_k(const AttnArgs &a)
{
    switch (a.k) {
    case 1: return launch_typed<D, BF16, 1, SPLIT>(a);
    case 2: return launch_typed<D, BF16, 2, SPLIT>(a);
    case 3: return launch_typed<D, BF16, 3, SPLIT>(a);
    case 4: return launch_typed<D, BF16, 4, SPLIT>(a);
    case 5: return launch_typed<D, BF16, 5, SPLIT>(a);
    case 6: return launch_typed<D, BF16, 6, SPLIT>(a);
    case 7: return launch_typed<D, BF16, 7, SPLIT>(a);
    case 8: return launch_typed<D, BF16, 8, SPLIT>(a);
    default: return hipErrorInvalidValue;
    }
}

template <bool BF16, bool SPLIT>
hipError_t launch_d(const AttnArgs &a)
{
    switch (a.D) {
    case 16: return launch_k<16, BF16, SPLIT>(a);
    case 32: return launch_k<32, BF16, SPLIT>(a);
    case 64: return launch_k<64, BF16, SPLIT>(a);
    case 128: return launch_k<128, BF16, SPLIT>(a);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace

// This file is compiled once per part -- 0: bf16 encoder-decoder and the host
// functions, 1: f32 encoder-decoder, 2: bf16 split cache, 3: f32 split cache --
// so that the kernels' instances build side by side.
#ifndef FS_ATTN_PART
#define FS_ATTN_PART 0
#endif
template <int PART>
hipError_t launch_part(const AttnArgs &a);
template <int PART>
hipError_t trace_part(unsigned long long *buf, unsigned int cap);
template <>
hipError_t launch_part<FS_ATTN_PART>(const AttnArgs &a) {
    return launch_d<FS_ATTN_PART % 2 == 0, (FS_ATTN_PART >= 2)>(a);
}
template <>
hipError_t trace_part<FS_ATTN_PART>(unsigned long long *buf, unsigned int cap) {
#if FS_TRACE
    const trace::Target t{buf, cap};
    return hipMemcpyToSymbol(HIP_SYMBOL(g_trace), &t, sizeof(t));
#else
    (void)buf;
    (void)cap;
    return hipErrorNotSupported;
#endif
}

#if FS_ATTN_PART == 0
template <>
hipError_t launch_part<1>(const AttnArgs &a);
template <>
hipError_t launch_part<2>(const AttnArgs &a);
template <>
hipError_t launch_part<3>(const AttnArgs &a);
template <>
hipError_t trace_part<1>(unsigned long long *buf, unsigned int cap);
template <>
hipError_t trace_part<2>(unsigned long long *buf, unsigned int cap);
template <>
hipError_t trace_part<3>(unsigned long long *buf, unsigned int cap);

namespace {
std::atomic<int> g_path_override{0};
}  // namespace

hipError_t set_attn_trace(unsigned long long *buf, unsigned int cap) {
    hipError_t e = trace_part<0>(buf, cap);
    if (e == hipSuccess) e = trace_part<1>(buf, cap);
    if (e == hipSuccess) e = trace_part<2>(buf, cap);
    if (e == hipSuccess) e = trace_part<3>(buf, cap);
    return e;
}

AttnPath set_attn_path_override(AttnPath p) {
    return static_cast<AttnPath>(g_path_override.exchange(static_cast<int>(p), std::memory_order_relaxed));
}

AttnPath choose_attn_path(int n_bh, int S, int D, int esize, int k, int t, bool table) {
    const AttnPath forced = static_cast<AttnPath>(g_path_override.load(std::memory_order_relaxed));
    if (forced != AttnPath::kAuto) return forced;
    // Wave tasks of a row at most: its prefix tiles, and its generated tiles
    // once per beam (through a table, all but the last are mostly shared).
    const int tile = cross_attn_chunk_keys(D, esize) / kWaves;
    const long long nt = (S + tile - 1) / tile, ngt = (t + tile - 1) / tile;
    const long long gen = ngt == 0 ? 0 : table ? ngt - 1 + k : ngt * k;
    const long long tasks = nt + gen;
    // In bf16 the kernels that read through a table with D = 128 have more than
    // 128 registers (130 to 208): three or two waves per SIMD.
    const bool heavy = table && t > 0 && D >= 128 && esize == 2;
    // The lines below were measured on MI355X over 16 to 1024 rows, 128 to 2048
    // keys, 0 to 500 generated tokens, D = 64 and 128, bf16 and f32 (graph
    // replays of three rotated inputs).
    const bool bm = t > 0 && beam_waves(n_bh, D, esize, k, (int)nt, t, table);
    // Beams' waves on the matrix cores spill in sixteen waves with D = 128 (us,
    // bf16, 144 rows of 0 + 300, k = 4: 18.9 with eight, 26.2 with sixteen; D =
    // 64, 48 rows of 200 + 300, k = 6: 14.9 and 13.6).
    const bool split_gen = n_bh < kSplitMaxRows && nt >= 8 * kWaves && 2 * gen <= nt;   // as below
    if (esize == 2 && D == 128 && bm && n_bh <= kCus && !split_gen) return AttnPath::kWhole2;
    if ((esize == 4 || D == 16) && t > 0) {
        // Generated tokens on the VALU tile (fp32, and D = 16).  More rows than
        // CUs: four waves where eight have more than 128 registers (one
        // workgroup per CU then), eight where the prefix is long beside what is
        // generated (us, fp32, D = 64, 4 beams through a table, 640 rows of 200 +
        // 30: 18 with four, 24 with eight; 5 beams, no table, 320 rows of 900 +
        // 10: 39 / 30).
        if (n_bh > kCus) {
            if (D == 16 && (esize == 2 || bm || table)) return AttnPath::kWhole1;
            if (table)
                return k <= 3 && nt >= gen && tasks > kWaves && n_bh <= 2 * kCus ? AttnPath::kWhole2
                                                                               : AttnPath::kWhole1;
            if (k == 5 && nt <= 4 * kWaves) return AttnPath::kWhole1;
        } else if (D == 16 && esize == 2 && k >= 3) {
            return AttnPath::kWhole2;   // sixteen spill (192 rows of 300 + 300, 8 beams: 27 us against 16)
        } else if (table && !bm && tasks > 2 * kWaves) {
            // six beams' tasks and more spill in sixteen waves
            if (D == 16) return AttnPath::kWhole2;
            if (k >= 6 && n_bh < kSplitMaxRows && nt >= 4 * kWaves && gen <= nt) return AttnPath::kSplit;
            if (k >= 6 && (n_bh >= kSplitMaxRows || tasks <= 4 * kWaves)) return AttnPath::kWhole2;
        } else if (bm) {
            // the generated tokens go to one workgroup of the split form, a
            // beam or two per wave, beside the prefix's
            if (n_bh < kSplitMaxRows && nt >= (k >= 6 ? 3 : 4) * kWaves &&
                2 * nt >= 3 * ngt * ((k + kWaves - 1) / kWaves))
                return AttnPath::kSplit;
            if (k >= 6 && nt <= kWaves) return AttnPath::kWhole2;
        }
    }
    if (n_bh > kCus) {
        // More rows than CUs. Four waves where one round of four takes the row
        // (1024 rows of 16 generated tokens: 8.5 us against 10.0 with eight),
        // eight otherwise (768 rows of 512 keys: 12.6 against 13.5). Of three
        // waves per SIMD, workgroups of eight leave a third unused.
        return tasks <= kWaves || heavy ? AttnPath::kWhole1 : AttnPath::kWhole2;
    }
    // A CU for every row: as many waves as the row has tasks, so that all of
    // its loads are in flight at once.
    if (tasks <= kWaves && table && t > 0) return AttnPath::kWhole1;
    if (tasks <= 2 * kWaves) return AttnPath::kWhole2;
    // Few rows of many tiles go to several workgroups each, whose records cost
    // a round trip through memory (about 4 us): 64 rows of 2048 keys 12.2
    // against 12.9 us, but 16 rows of 1024 keys 7.5 against 4.5, and, with the
    // larger records of D = 128, 64 rows of 1024 keys 14.7 against 13.2.  The
    // generated tokens all go to one of those workgroups: 64 more with f32,
    // 2048 keys and 64 rows 18.4 against 30.4 us, but 300 more with 1024 keys
    // in bf16 19.3 against 16.9.
    if (n_bh < kSplitMaxRows) {
        if (t > 0 ? split_gen
                  : nt > 8 * kWaves || (nt > 4 * kWaves && n_bh > 16 && D < 128))
            return AttnPath::kSplit;
    }
    // Sixteen waves with D = 128 and a table spill: 256 rows of 256 + 64 rows
    // 14.8 us against 10.9 with eight.
    return heavy ? AttnPath::kWhole2 : AttnPath::kWhole4;
}

bool may_split(int n_bh, int S, int D, int esize) {
    return g_path_override.load(std::memory_order_relaxed) == static_cast<int>(AttnPath::kAuto) &&
           n_bh < kSplitMaxRows && S > 2 * cross_attn_chunk_keys(D, esize);
}

int cross_attn_chunk_keys(int D, int esize) {
    // kWaves * kIt rows of 64/(lanes per row) = 4 * 8 * 64 * 16 / (D * esize)
    return kWaves * kIt * kWave * 16 / (D * esize);
}

size_t cross_attn_workspace_floats(int B, int k, int H, int S, int D, int esize, bool split) {
    const int C = cross_attn_chunk_keys(D, esize);
    // Records are one per chunk, and one for the generated tokens of the split
    // cache; kWaves slots per chunk are asked for, so that what callers have
    // sized, and what fs_beam_decode_step_noalloc refuses, stays as it was.
    const size_t NT = (size_t)std::max(1, (S + C - 1) / C) * kWaves + (split ? 1 : 0);
    const size_t n_bh = (size_t)B * H;
    const size_t part = n_bh * NT * (size_t)k * (size_t)(D + 2);
    return 2 * (part + n_bh);  // 64-bit words: the partial records, then one counter per row
}

hipError_t launch_cross_attn(const void *q, const void *K, const void *V, const int32_t *src_len,
                             void *out, int B, int k, int H, int S, int D, bool bf16,
                             float *workspace, unsigned long long epoch, hipStream_t stream,
                             AttnPath path, const NgramRows *ngram)
{
    AttnArgs a{q, K, V, src_len, out, B, k, H, S, D, nullptr, nullptr, 0, 0, nullptr, 0, workspace, epoch, stream,
               NgramJob{nullptr, nullptr, 0, 0, 0, 0, 0, 0}, path, false};
    if (ngram)
        a.ng = NgramJob{ngram->tokens, ngram->logits, ngram->ld, ngram->t, ngram->n - 1, ngram->V, ngram->rows, 0};
    return bf16 ? launch_part<0>(a) : launch_part<1>(a);
}

hipError_t launch_prefix_attn(const void *q, const void *Kp, const void *Vp, const int32_t *prefix_len,
                              const void *Kt, const void *Vt, int T, int t, const int32_t *anc, int ld_anc,
                              void *out, int B, int k, int H, int N, int D, bool bf16, float *workspace,
                              unsigned long long epoch, hipStream_t stream, AttnPath path)
{
    const int esize = bf16 ? 2 : 4, tile = cross_attn_chunk_keys(D, esize) / kWaves;
    const AttnArgs a{q, Kp, Vp, prefix_len, out, B, k, H, N, D, Kt, Vt, T, t, anc, ld_anc, workspace, epoch, stream,
                     NgramJob{nullptr, nullptr, 0, 0, 0, 0, 0, 0}, path,
                     beam_waves(B * H, D, esize, k, (N + tile - 1) / tile, t, anc != nullptr)};
    return bf16 ? launch_part<2>(a) : launch_part<3>(a);
}
#endif  // FS_ATTN_PART == 0

}  // namespace fs
