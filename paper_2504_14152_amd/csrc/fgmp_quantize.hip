// FGMP block scoring, precision decision, encoding and packing (Sec. 3.1,
// Sec. 3.3 "dynamic max", Sec. 4, Sec. 4.2), one 16-element block per lane.
//
// Arithmetic per block (every FP32 step is one separately rounded IEEE
// operation -- this file is compiled with -ffp-contract=off):
//   amax = max|x_i|; u = amax / (6 S); sc = E4M3(u); d = value(sc) * S
//   inv_d = 1 / d (0 when sc == 0); q_i = E2M1(x_i * inv_d); xh_i = value(q_i) * d
//   t_i = ((x_i - xh_i) * (x_i - xh_i)) * F_i                        (Eq. 2, Eq. 6)
//   score = balanced pairwise tree over t_0..t_15 (adjacent pairs first)
//   FP8 iff score > T (Sec. 4.2); FP8 codes c_i = E4M3(x_i * (1 / S))  (Sec. 5.1)
#include <algorithm>
#include <type_traits>

#include "fgmp_elementwise.hpp"
#include "fgmp_internal.hpp"
#include "fgmp_quant_block.hpp"

namespace fgmp {

typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));

struct QuantParams {
    const void *X;
    int64_t ldx, rows, nb;
    const float *fisher;
    int64_t ld_fisher;
    float T, S;
    PackedView out;
    int64_t n_rt, n_kt;
    float *scores;
    int mode;          // kModeStrided / kModeCompact / kModeF16
    int rt_per_wave;
    PackedLayout layout;   // for the header, written by the first launch of a call
    uint32_t compact;
    _Float16 *x16;         // kModeF16: dequantized values (without the tensor scale), [8 n_rt][ld16]
    int64_t ld16;
    uint32_t *zero;        // words cleared by the first workgroup (counters of the kernel that follows)
    int zero_n;
    bool delta;            // Eq. 8 scoring (see quantize_kernel)
    bool no_fp8;           // the threshold is +inf: no block is kept in FP8, and the first pass of packing weights is the only one
};

// kModeCompact leaves planes T and H to pack_upper_halves_kernel.
// kModeF16 writes, instead of the packed planes, the FP16 value of every stored
// code (exact: an E2M1 value times an E4M3 scale, or an E4M3 value), which is
// what the prefill GEMM consumes; only the header goes to the packed buffer.
enum { kModeStrided = 0, kModeCompact = 2, kModeF16 = 3 };


// Raw (unconverted) 16 input elements of one block: 2 x 16 B of bf16 or 4 x 16 B of fp32.
// Gated: a staged FP32 product whose columns come in groups of 32 gate and 32 up values; a block is SiLU(gate) * up of 16 of
// them.  (With the gated values written by a launch of their own and read by this kernel as FP32, us for the two products of an
// MLP, before / now: 1 x 2544 x 1600 20.0 / 16.8, 5 x 528 x 12032 20.2 / 18.4, 64 x 592 x 21952 36.6 / 34.7, 300 x 2080 x 7936 48.2 / 46.1.)
struct Gated { float v; };
template <typename Tin> struct RawBlock;
template <> struct RawBlock<uint16_t> { uint4 v[2]; };
template <> struct RawBlock<float> { uint4 v[4]; };
template <> struct RawBlock<Gated> { uint4 v[8]; };

// where block kb of a row starts
template <typename Tin> __device__ __forceinline__ int64_t block_at(int64_t kb)
{
    if constexpr (std::is_same_v<Tin, Gated>) return (kb >> 1) * kGateGroup + (kb & 1) * kBlock;
    else return kb * kBlock;
}

template <typename Tin> __device__ __forceinline__ void load_raw(const Tin *src, RawBlock<Tin> &r)
{
    const uint4 *p = reinterpret_cast<const uint4 *>(src);
#pragma unroll
    for (int i = 0; i < (int)(sizeof(r.v) / sizeof(uint4)); ++i) r.v[i] = p[i];
}

template <> __device__ __forceinline__ void load_raw(const Gated *src, RawBlock<Gated> &r)
{
    const uint4 *gate = reinterpret_cast<const uint4 *>(src), *up = reinterpret_cast<const uint4 *>(src + kGateGroup / 2);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        r.v[i] = gate[i];
        r.v[4 + i] = up[i];
    }
}

__device__ __forceinline__ void widen(const RawBlock<Gated> &r, float (&x)[16])
{
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        x[4 * i + 0] = silu_mul(u2f(r.v[i].x), u2f(r.v[4 + i].x));
        x[4 * i + 1] = silu_mul(u2f(r.v[i].y), u2f(r.v[4 + i].y));
        x[4 * i + 2] = silu_mul(u2f(r.v[i].z), u2f(r.v[4 + i].z));
        x[4 * i + 3] = silu_mul(u2f(r.v[i].w), u2f(r.v[4 + i].w));
    }
}

__device__ __forceinline__ void widen(const RawBlock<uint16_t> &r, float (&x)[16])
{
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const uint32_t w[4] = {r.v[i].x, r.v[i].y, r.v[i].z, r.v[i].w};
#pragma unroll
        for (int j = 0; j < 4; ++j) {   // bf16 -> fp32 is a 16-bit shift
            x[8 * i + 2 * j + 0] = u2f(w[j] << 16);
            x[8 * i + 2 * j + 1] = u2f(w[j] & 0xFFFF0000u);
        }
    }
}

__device__ __forceinline__ void widen(const RawBlock<float> &r, float (&x)[16])
{
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        x[4 * i + 0] = u2f(r.v[i].x); x[4 * i + 1] = u2f(r.v[i].y);
        x[4 * i + 2] = u2f(r.v[i].z); x[4 * i + 3] = u2f(r.v[i].w);
    }
}

// bytes_used of a compact tensor: at least one entry stays readable, kernels that load plane H unconditionally read entry 0
__device__ __forceinline__ uint64_t compact_bytes(const PackedLayout &l, uint64_t entries) { return l.off_H + (entries > 0 ? entries : 1) * 8; }

__device__ __forceinline__ void write_packed_header(const QuantParams &p)
{
    write_header(p.out.hdr, p.layout, p.S, p.compact);
    if (p.no_fp8) {
        p.out.hdr->h_entries = 0;
        p.out.hdr->bytes_used = compact_bytes(p.layout, 0);
    }
}

// The planes of one tile, a slot per lane: plane M and the slots' plane-L words and plane-S bytes; in strided mode also planes
// T and H.  hi: the block is kept in FP8 (ballot: of all lanes).
template <bool kHW, int kMode, bool kDelta>
__device__ __forceinline__ void store_tile(const QuantParams &p, int64_t tile, int lane, bool hi, uint64_t ballot, const BlockCodes &bc,
                                           const float (&x)[16], float amax, float inv_S)
{
    const uint32_t prefix = (uint32_t)__popcll(ballot & ((1ull << lane) - 1ull));
    const uint32_t hbase = (uint32_t)(tile * kTileSlots);
    if constexpr (kMode == kModeStrided) {
        if (lane == 0) p.out.T[tile] = hbase;
    }
    if (lane == 0) p.out.M[tile] = ballot;
    if constexpr (kMode == kModeCompact) {
        if (p.no_fp8 && lane == 0) p.out.T[tile] = 0u;
    }

    uint2 lword = make_uint2(bc.q[0], bc.q[1]);
    uint32_t sbyte = bc.sc;
    if (ballot != 0ull) {
        // values beyond the FP8 range only occur when the caller's S is below amax / 448
        const bool any_big = __ballot(hi && amax * inv_S > 448.0f) != 0ull;
        if (hi) {
            uint32_t c[4];
            if constexpr (kDelta) {
#pragma unroll
                for (int j = 0; j < 4; ++j) c[j] = bc.c8[j];
            } else {
                float r[16];
#pragma unroll
                for (int i = 0; i < 16; ++i) r[i] = x[i] * inv_S;
                if (any_big) encode_fp8_block<kHW, true>(r, c);
                else encode_fp8_block<kHW, false>(r, c);
            }
            lword = make_uint2(c[0], c[1]);
            if constexpr (kMode == kModeStrided) p.out.H[(uint64_t)hbase + prefix] = make_uint2(c[2], c[3]);
            sbyte = prefix;
        }
    }
    p.out.L[tile * kTileSlots + lane] = lword;
    p.out.S[tile * kTileSlots + lane] = (uint8_t)sbyte;
}

// grid.x = K-tiles, grid.y = groups of 4 * rt_per_wave row-tiles; 4 waves per
// workgroup work on 4 adjacent row-tiles of the same K-tile at a time, so the
// per-channel sensitivities stay in registers across the loop.  The input of
// the next row-tile is fetched while the current one is processed.
// kDelta: the score is Eq. 8's (weighted square of Q_NVFP4(x) - Q_FP8(x)) instead of Eq. 6's NVFP4 error;
// the FP8 codes are then computed for every block and reused when the block is kept in FP8.
template <typename Tin, bool kPerElem, bool kHW, int kMode, bool kDelta>
__global__ __launch_bounds__(256) void quantize_kernel(QuantParams p)
{
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int64_t kt = blockIdx.x;
    const int64_t kb = kt * kTileBlocks + (lane & 7);
    const bool kvalid = kb < p.nb;
    const int rloc = lane >> 3;
    const Tin *X = static_cast<const Tin *>(p.X);

    float f[16];
    if constexpr (!kPerElem) {
        if (kvalid) load16(p.fisher + kb * kBlock, f);
        else {
#pragma unroll
            for (int i = 0; i < 16; ++i) f[i] = 0.0f;
        }
    }
    const float inv_S = 1.0f / p.S;
    const float S6 = 6.0f * p.S;
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0 && p.out.hdr != nullptr)
        write_packed_header(p);
    if (blockIdx.x == 0 && blockIdx.y == 0)
        for (int i = threadIdx.x; i < p.zero_n; i += 256) p.zero[i] = 0u;

    const int64_t rt0 = (int64_t)blockIdx.y * p.rt_per_wave * 4 + wave;
    // out-of-range lanes read a valid address (their own K-tile's first block of row 0) and are masked
    auto src_of = [&](int64_t rt) -> const Tin * {
        const int64_t row = rt * kTileRows + rloc;
        const bool ok = kvalid && row < p.rows;
        return X + (ok ? row * p.ldx + block_at<Tin>(kb) : 0);
    };
    if (rt0 >= p.n_rt) return;
    const int64_t left = (p.n_rt - rt0 + 3) / 4;
    const int n_it = (int)(left < p.rt_per_wave ? left : p.rt_per_wave);

    auto process = [&](int64_t rt, const RawBlock<Tin> &raw_in) {
        const int64_t row = rt * kTileRows + rloc;
        const bool valid = kvalid && row < p.rows;

        float x[16];
        widen(raw_in, x);
        if (!valid) {
#pragma unroll
            for (int i = 0; i < 16; ++i) x[i] = 0.0f;
        }
        if constexpr (kPerElem) {
            if (valid) load16(p.fisher + row * p.ld_fisher + kb * kBlock, f);
            else {
#pragma unroll
                for (int i = 0; i < 16; ++i) f[i] = 0.0f;
            }
        }

        // block scale (dynamic max), NVFP4 codes, score; in the Eq. 8 mode also the
        // FP8 codes of every block (values beyond the FP8 range only occur when the caller's S is below
        // amax / 448: then the wave clamps before converting)
        const float amax = block_amax(x);
        bool clamp8 = false;
        if constexpr (kDelta) clamp8 = __ballot(amax * inv_S > 448.0f) != 0ull;
        BlockCodes bc;
        quantize_block_math<kHW, kDelta>(x, f, amax, p.S, inv_S, S6, -1, clamp8, bc);
        const uint32_t sc = bc.sc;
        const uint32_t (&q)[2] = bc.q;
        const uint32_t (&c8)[4] = bc.c8;
        const float score = bc.score;

        const bool hi = valid && (score > p.T);
        const uint64_t ballot = __ballot(hi);
        const int64_t tile = rt * p.n_kt + kt;
        if (p.scores != nullptr && valid) p.scores[row * p.nb + kb] = score;

        if constexpr (kMode == kModeF16) {
            static_assert(kHW, "the FP16 output mode uses the conversion instructions");
            half2_t o[8];
            if (hi) {
                uint32_t c[4];
                if constexpr (kDelta) {
#pragma unroll
                    for (int j = 0; j < 4; ++j) c[j] = c8[j];
                } else {
                    float r[16];
#pragma unroll
                    for (int i = 0; i < 16; ++i) r[i] = x[i] * inv_S;
                    if (amax * inv_S > 448.0f) encode_fp8_block<kHW, true>(r, c);
                    else encode_fp8_block<kHW, false>(r, c);
                }
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    o[2 * j] = __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(c[j], 1.0f, false);
                    o[2 * j + 1] = __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(c[j], 1.0f, true);
                }
            } else {
                const half2_t s = __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(sc | (sc << 8), 1.0f, false);
                o[0] = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(q[0], 1.0f, 0) * s;
                o[1] = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(q[0], 1.0f, 1) * s;
                o[2] = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(q[0], 1.0f, 2) * s;
                o[3] = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(q[0], 1.0f, 3) * s;
                o[4] = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(q[1], 1.0f, 0) * s;
                o[5] = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(q[1], 1.0f, 1) * s;
                o[6] = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(q[1], 1.0f, 2) * s;
                o[7] = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(q[1], 1.0f, 3) * s;
            }
            // every slot of the tile is written (zeros where the tensor ends), so the GEMM can read whole tiles
            union { half2_t h[8]; uint4 v[2]; } pack;
#pragma unroll
            for (int j = 0; j < 8; ++j) pack.h[j] = o[j];
            uint4 *dst = reinterpret_cast<uint4 *>(p.x16 + (rt * kTileRows + rloc) * p.ld16 +
                                                   (kt * kTileBlocks + (lane & 7)) * kBlock);
            dst[0] = pack.v[0];
            dst[1] = pack.v[1];
        } else {
            store_tile<kHW, kMode, kDelta>(p, tile, lane, hi, ballot, bc, x, amax, inv_S);
        }
    };

    // software pipeline: the next row-tile's input is in flight while this one is processed
    RawBlock<Tin> cur, nxt;
    load_raw(src_of(rt0), cur);
    for (int it = 0; it + 1 < n_it; ++it) {
        load_raw(src_of(rt0 + 4 * (int64_t)(it + 1)), nxt);
        process(rt0 + 4 * (int64_t)it, cur);
        cur = nxt;
    }
    process(rt0 + 4 * (int64_t)(n_it - 1), cur);
}

// ---------------------------------------------------------------------------
// The activation hot path (Sec. 4.2) once more, trimmed: same arithmetic, result for result, as
// quantize_kernel (NVFP4-error score, one sensitivity per channel, dynamic-max scale).
//   * d = value(sc) * S and 1 / d depend only on the scale code: a table of 127 {d, 1/d} pairs per
//     workgroup (LDS) replaces the decode, the multiply and the division of every block;
//   * u = amax / (6 S) is one multiply by the correctly rounded reciprocal r and one correction step,
//     q1 = fma(fma(-q0, 6S, amax), r, q0): the correctly rounded quotient (q0 is within one unit of it and
//     the residual is exact; magnitudes near the ends of the FP32 range, where that fails, take the plain
//     division instead);
//   * input through range-checked buffer loads: rows beyond the tensor read zeros without a select;
//   * a workgroup's eight waves take eight consecutive K-tiles of one row-tile at a time (2 KB of every
//     row, 4 KB of plane L, 512 B of plane S: contiguous), and workgroups that run at the same time cover
//     whole rows; the launch is one resident set of workgroups that stride over the row-tiles, so a wave
//     keeps its K-tile and the sensitivities stay in registers;
//   * the 12 bytes of per-tile words are not stored tile by tile (those small stores alone cost 6% of the
//     run time): the plane-M and plane-T words of eight row-tiles are gathered in LDS and leave as 64- and
//     32-byte pieces;
//   * the FP8 upper halves of the tiles a wave visits are appended to a region of plane H that belongs to
//     the wave (see h_cnt below).
// Tensors up to 4 GB (32-bit offsets).
// ---------------------------------------------------------------------------
constexpr int kQWaves = 8;    // waves per workgroup = consecutive K-tiles
constexpr int kQBatch = 8;    // row-tiles between two writes of the gathered plane-M words
constexpr int64_t kQMinTiles = 65536;   // smaller tensors do not fill the resident set for long enough: general kernel

// kTraffic (measurement builds only): the kernel's loads and stores with next to no arithmetic between them
// -- the plane-L words are input words, a fixed tenth of the slots counts as FP8 -- i.e. what the memory
// system alone takes for this access pattern; the benchmark times it beside the real kernel.
// kDelta: the score of Eq. 8 (the FP8 codes of every block are computed first and reused for the blocks kept in FP8).
template <typename Tin, int kMode, bool kTraffic = false, bool kDelta = false>
__global__ __launch_bounds__(64 * kQWaves) void quantize_act_kernel(QuantParams p, uint32_t x_bytes, uint32_t out_bytes, int n_kg)
{
    static_assert(kMode == kModeStrided || kMode == kModeF16, "one-pass modes only");
    static_assert(!kTraffic || kMode == kModeStrided, "the traffic model writes packed planes");
    constexpr int kVec = (int)(sizeof(RawBlock<Tin>) / sizeof(uint4));   // 16-byte loads per block
    __shared__ float2 tbl[128];                                            // {d, 1/d} by scale code
    __shared__ uint4 m_lds[kQBatch][kQWaves];                              // plane-M word and plane-T entry, [row-tile of the batch][K-tile]
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kg = (int)blockIdx.x % n_kg;                 // the grid is a multiple of n_kg: the K group never changes
    const int rt_first = (int)blockIdx.x / n_kg, rt_step = (int)gridDim.x / n_kg;
    const uint32_t kt = (uint32_t)(kg * kQWaves + wave);
    const uint32_t kb = kt * kTileBlocks + (lane & 7);
    const bool kvalid = kb < (uint32_t)p.nb;               // (a whole wave may lie beyond K: it idles but keeps the barriers)
    const int rloc = lane >> 3;
    const float S = p.S, inv_S = 1.0f / S, S6 = 6.0f * S, r_S6 = 1.0f / S6;
    if (tid < 128) {
        const float d = e4m3_decode_int((uint32_t)tid) * S;
        tbl[tid] = make_float2(d, tid != 0 ? 1.0f / d : 0.0f);
    }
    const __amdgpu_buffer_rsrc_t obuf =
        __builtin_amdgcn_make_buffer_rsrc(p.out.hdr, 0, (int)out_bytes, 0x00020000);
    const uint32_t off_L = (uint32_t)p.layout.off_L, off_S = (uint32_t)p.layout.off_S, off_M = (uint32_t)p.layout.off_M,
                   off_T = (uint32_t)p.layout.off_T, off_H = (uint32_t)p.layout.off_H;
    if (blockIdx.x == 0) {
        if (tid == 0 && p.out.hdr != nullptr) write_header(p.out.hdr, p.layout, S, 0u);
        for (int i = tid; i < p.zero_n; i += 64 * kQWaves) p.zero[i] = 0u;
    }
    float f[16];
    if (kvalid) load16(p.fisher + kb * kBlock, f);
    else {
#pragma unroll
        for (int i = 0; i < 16; ++i) f[i] = 0.0f;
    }
    __syncthreads();
    if (rt_first >= (int)p.n_rt) return;
    const int n_it = ((int)p.n_rt - rt_first + rt_step - 1) / rt_step;
    // Plane H: the FP8 upper halves of all the tiles a wave visits go, in visiting order, into one region
    // of the plane that belongs to the wave (64 entries per tile it owns: the worst case), so that the few
    // entries of a tile continue where the previous tile's stopped instead of starting a 512-byte
    // region of their own (those partial-line writes cost 7% of the run time at 10% FP8).  The regions
    // of the waves with the same K-tile follow each other in the order of their first row-tile.
    uint32_t h_cnt;
    {
        const uint32_t q = (uint32_t)p.n_rt / (uint32_t)rt_step, r = (uint32_t)p.n_rt % (uint32_t)rt_step, y = (uint32_t)rt_first;
        h_cnt = (kt * (uint32_t)p.n_rt + y * q + (y < r ? y : r)) * kTileSlots;
    }

    // input: per-lane byte offset of the lane's block in the workgroup's first row-tile, advanced by rt_step
    // row-tiles per iteration; rows beyond the tensor fall outside the buffer and read zeros; lanes
    // beyond K stay parked outside it
    const __amdgpu_buffer_rsrc_t xbuf = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p.X), 0, (int)x_bytes, 0x00020000);
    const uint32_t row_bytes = (uint32_t)p.ldx * (uint32_t)sizeof(Tin);
    uint32_t xoff = kvalid ? (uint32_t)(rt_first * kTileRows + rloc) * row_bytes + kb * (uint32_t)(kBlock * sizeof(Tin)) : 0xFFFFFF00u;
    const uint32_t xstep = kvalid ? (uint32_t)rt_step * kTileRows * row_bytes : 0u;
    auto load_block = [&](RawBlock<Tin> &r) {

        // (a load past the last row-tile lies beyond the buffer -- zeros -- or is unused; offsets stay below 2^32
        // for the tensors this kernel accepts plus one step, which the host checks)
#pragma unroll
        for (int i = 0; i < kVec; ++i) {
            const u32x4_t v = __builtin_amdgcn_raw_buffer_load_b128(xbuf, (int)xoff + 16 * i, 0, 0);
            r.v[i] = make_uint4(v[0], v[1], v[2], v[3]);
        }
        xoff += xstep;
    };

    auto process = [&](int it, const RawBlock<Tin> &raw_in) {
        const int rt = rt_first + it * rt_step;
        if constexpr (kTraffic) {
            uint32_t w[4] = {raw_in.v[0].x ^ raw_in.v[1].z, raw_in.v[0].y ^ raw_in.v[1].w, raw_in.v[0].z ^ raw_in.v[1].x, raw_in.v[0].w ^ raw_in.v[1].y};
            if constexpr (kVec == 4) {
                w[0] ^= raw_in.v[2].x ^ raw_in.v[3].z; w[1] ^= raw_in.v[2].y ^ raw_in.v[3].w;
                w[2] ^= raw_in.v[2].z ^ raw_in.v[3].x; w[3] ^= raw_in.v[2].w ^ raw_in.v[3].y;
            }
            const uint32_t row = (uint32_t)(rt * kTileRows + rloc);
            const bool valid = kvalid && row < (uint32_t)p.rows;
            const uint32_t tile = (uint32_t)rt * (uint32_t)p.n_kt + kt, slot = tile * kTileSlots + lane;
            const bool hi = valid && ((slot * 2654435761u) >> 24) < 26u;
            const uint64_t ballot = __ballot(hi);
            const uint32_t prefix = __builtin_amdgcn_mbcnt_hi((uint32_t)(ballot >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)ballot, 0u));
            if (lane == 0) m_lds[it % kQBatch][wave] = make_uint4((uint32_t)ballot, (uint32_t)(ballot >> 32), h_cnt, 0u);
            if (hi) __builtin_amdgcn_raw_buffer_store_b64(u32x2_t{w[2], w[3]}, obuf, (int)(off_H + (h_cnt + prefix) * 8u), 0, 0);
            if (kt < (uint32_t)p.n_kt) {
                __builtin_amdgcn_raw_buffer_store_b64(u32x2_t{w[0], w[1]}, obuf, (int)(off_L + slot * 8u), 0, 0);
                __builtin_amdgcn_raw_buffer_store_b8((uint8_t)(hi ? prefix : (w[2] & 0x7Fu)), obuf, (int)(off_S + slot), 0, 0);
            }
            h_cnt += (uint32_t)__popcll(ballot);
            return;
        }
        float x[16];
        widen(raw_in, x);
        const float amax = block_amax(x);
        // block scale: correctly rounded amax / (6 S)
        float u = amax * r_S6;
        // (outside [1e-30, 1e30) -- where a residual could lose bits or the product overflow -- the wave
        // divides; zero is exact either way)
        const bool odd_range = (amax < 1e-30f && amax != 0.0f) || !(u < 1e30f);
        if (__builtin_expect(__ballot(odd_range) != 0ull, 0)) u = amax / S6;
        else u = __builtin_fmaf(__builtin_fmaf(-u, S6, amax), r_S6, u);
        const uint32_t sc = e4m3_encode_pair_hw(u, 0.0f) & 0xFFu;
        const float2 dd = tbl[sc];
        const float d = dd.x, inv_d = dd.y;
        // (Eq. 8: the FP8 codes of every block; values beyond the FP8 range only occur when the caller's S is
        // below amax / 448, then the wave clamps before converting -- clamping changes no value in range)
        uint32_t c8[4] = {0u, 0u, 0u, 0u};
        if constexpr (kDelta) {
            float r8[16];
#pragma unroll
            for (int i = 0; i < 16; ++i) r8[i] = x[i] * inv_S;
            if (__ballot(amax * inv_S > 448.0f) != 0ull) encode_fp8_block<true, true>(r8, c8);
            else encode_fp8_block<true, false>(r8, c8);
        }
        uint32_t q[2] = {0u, 0u};
        float t[16];
#define FGMP_ENC(W, B, I) q[W] = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(q[W], x[I] * inv_d, x[I + 1] * inv_d, 1.0f, B)
        FGMP_ENC(0, 0, 0); FGMP_ENC(0, 1, 2); FGMP_ENC(0, 2, 4); FGMP_ENC(0, 3, 6);
        FGMP_ENC(1, 0, 8); FGMP_ENC(1, 1, 10); FGMP_ENC(1, 2, 12); FGMP_ENC(1, 3, 14);
#undef FGMP_ENC
#define FGMP_ERR(W, B, I)                                                                \
    {                                                                                    \
        const float2_t v = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(q[W], 1.0f, B);      \
        float e0, e1;                                                                    \
        if constexpr (kDelta) {                                                          \
            const float2_t v8 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp8(c8[(I) / 4], 1.0f, ((I) % 4) >= 2); \
            e0 = v[0] * d - v8[0] * S;                                                   \
            e1 = v[1] * d - v8[1] * S;                                                   \
        } else {                                                                         \
            e0 = x[I] - v[0] * d;                                                        \
            e1 = x[I + 1] - v[1] * d;                                                    \
        }                                                                                \
        t[I] = (e0 * e0) * f[I];                                                         \
        t[I + 1] = (e1 * e1) * f[I + 1];                                                 \
    }
        FGMP_ERR(0, 0, 0) FGMP_ERR(0, 1, 2) FGMP_ERR(0, 2, 4) FGMP_ERR(0, 3, 6)
        FGMP_ERR(1, 0, 8) FGMP_ERR(1, 1, 10) FGMP_ERR(1, 2, 12) FGMP_ERR(1, 3, 14)
#undef FGMP_ERR
#pragma unroll
        for (int w = 16; w > 1; w >>= 1)
#pragma unroll
            for (int i = 0; i < w / 2; ++i) t[i] = t[2 * i] + t[2 * i + 1];
        const float score = t[0];
        // (lanes outside the tensor hold zeros: score 0; a negative or -inf threshold must not select them)
        const uint32_t row = (uint32_t)(rt * kTileRows + rloc);
        const bool valid = kvalid && row < (uint32_t)p.rows;
        const bool hi = valid && (score > p.T);
        const uint64_t ballot = __ballot(hi);
        const uint32_t tile = (uint32_t)rt * (uint32_t)p.n_kt + kt;
        if (p.scores != nullptr && valid) p.scores[(int64_t)row * p.nb + kb] = score;

        if constexpr (kMode == kModeF16) {
            half2_t o[8];
            if (hi) {
                uint32_t c[4];
                if constexpr (kDelta) {
#pragma unroll
                    for (int j = 0; j < 4; ++j) c[j] = c8[j];
                } else {
                    float r[16];
#pragma unroll
                    for (int i = 0; i < 16; ++i) r[i] = x[i] * inv_S;
                    if (amax * inv_S > 448.0f) encode_fp8_block<true, true>(r, c);
                    else encode_fp8_block<true, false>(r, c);
                }
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    o[2 * j] = __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(c[j], 1.0f, false);
                    o[2 * j + 1] = __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(c[j], 1.0f, true);
                }
            } else {
                const half2_t s = __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(sc | (sc << 8), 1.0f, false);
                o[0] = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(q[0], 1.0f, 0) * s;
                o[1] = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(q[0], 1.0f, 1) * s;
                o[2] = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(q[0], 1.0f, 2) * s;
                o[3] = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(q[0], 1.0f, 3) * s;
                o[4] = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(q[1], 1.0f, 0) * s;
                o[5] = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(q[1], 1.0f, 1) * s;
                o[6] = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(q[1], 1.0f, 2) * s;
                o[7] = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(q[1], 1.0f, 3) * s;
            }
            union { half2_t h[8]; uint4 v[2]; } pack;
#pragma unroll
            for (int j = 0; j < 8; ++j) pack.h[j] = o[j];
            // every slot of the tile is written (zeros where the tensor ends), so the GEMM can read whole tiles
            if (kt < (uint32_t)p.n_kt) {
                uint4 *dst = reinterpret_cast<uint4 *>(p.x16 + (int64_t)row * p.ld16 + (int64_t)kb * kBlock);
                dst[0] = pack.v[0];
                dst[1] = pack.v[1];
            }
        } else {
            const uint32_t prefix = __builtin_amdgcn_mbcnt_hi((uint32_t)(ballot >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)ballot, 0u));
            const uint32_t slot = tile * kTileSlots + lane;
            if (lane == 0) m_lds[it % kQBatch][wave] = make_uint4((uint32_t)ballot, (uint32_t)(ballot >> 32), h_cnt, 0u);
            uint32_t lw0 = q[0], lw1 = q[1], sbyte = sc;
            if (ballot != 0ull) {
                // values beyond the FP8 range only occur when the caller's S is below amax / 448
                const bool any_big = __ballot(hi && amax * inv_S > 448.0f) != 0ull;
                if (hi) {
                    uint32_t c[4];
                    if constexpr (kDelta) {
#pragma unroll
                        for (int j = 0; j < 4; ++j) c[j] = c8[j];
                    } else {
                        float r[16];
#pragma unroll
                        for (int i = 0; i < 16; ++i) r[i] = x[i] * inv_S;
                        if (any_big) encode_fp8_block<true, true>(r, c);
                        else encode_fp8_block<true, false>(r, c);
                    }
                    lw0 = c[0];
                    lw1 = c[1];
                    sbyte = prefix;
                    __builtin_amdgcn_raw_buffer_store_b64(u32x2_t{c[2], c[3]}, obuf, (int)(off_H + (h_cnt + prefix) * 8u), 0, 0);
                }
            }
            if (kt < (uint32_t)p.n_kt) {
                __builtin_amdgcn_raw_buffer_store_b64(u32x2_t{lw0, lw1}, obuf, (int)(off_L + slot * 8u), 0, 0);
                __builtin_amdgcn_raw_buffer_store_b8((uint8_t)sbyte, obuf, (int)(off_S + slot), 0, 0);
            }
            h_cnt += (uint32_t)__popcll(ballot);
        }
    };
    // the gathered plane-M and plane-T words of the last `n` iterations (a batch): 64 and 32 contiguous bytes per row-tile
    auto write_masks = [&](int it_first, int n) {
        if constexpr (kMode == kModeStrided) {
            __syncthreads();
            const int i = tid / kQWaves, w = tid % kQWaves;
            const uint32_t kt_w = (uint32_t)(kg * kQWaves + w);
            if (i < n && kt_w < (uint32_t)p.n_kt) {
                const uint4 m = m_lds[(it_first + i) % kQBatch][w];
                const uint32_t tile = (uint32_t)(rt_first + (it_first + i) * rt_step) * (uint32_t)p.n_kt + kt_w;
                __builtin_amdgcn_raw_buffer_store_b64(u32x2_t{m.x, m.y}, obuf, (int)(off_M + tile * 8u), 0, 0);
                __builtin_amdgcn_raw_buffer_store_b32(m.z, obuf, (int)(off_T + tile * 4u), 0, 0);
            }
            __syncthreads();
        }
    };

    // two row-tiles per turn, each one's input in flight while the other is processed (two register sets
    // that swap roles: no copies)
    RawBlock<Tin> a, b;
    load_block(a);
    int it = 0;
    for (; it + 2 <= n_it; it += 2) {
        load_block(b);
        process(it, a);
        load_block(a);
        process(it + 1, b);
        if ((it + 2) % kQBatch == 0) write_masks(it + 2 - kQBatch, kQBatch);
    }
    if (it < n_it) {
        process(it, a);
        ++it;
    }
    if (it % kQBatch != 0) write_masks(it - it % kQBatch, it % kQBatch);
}

// The NVFP4 error of a block under the scale value d (inv_d = 1 / d, 0 for d = 0): operation for operation the score
// that quantize_block_math computes.
__device__ __forceinline__ float nvfp4_error(const float (&x)[16], const float (&f)[16], float d, float inv_d)
{
    uint32_t q[2] = {any_value(), any_value()};
    float t[16];
#define FGMP_ENC(W, B, I) q[W] = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(q[W], x[I] * inv_d, x[I + 1] * inv_d, 1.0f, B)
    FGMP_ENC(0, 0, 0); FGMP_ENC(0, 1, 2); FGMP_ENC(0, 2, 4); FGMP_ENC(0, 3, 6);
    FGMP_ENC(1, 0, 8); FGMP_ENC(1, 1, 10); FGMP_ENC(1, 2, 12); FGMP_ENC(1, 3, 14);
#undef FGMP_ENC
#define FGMP_ERR(W, B, I)                                                                \
    {                                                                                    \
        const float2_t v = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(q[W], 1.0f, B);      \
        const float e0 = x[I] - v[0] * d, e1 = x[I + 1] - v[1] * d;                      \
        t[I] = (e0 * e0) * f[I];                                                         \
        t[I + 1] = (e1 * e1) * f[I + 1];                                                 \
    }
    FGMP_ERR(0, 0, 0) FGMP_ERR(0, 1, 2) FGMP_ERR(0, 2, 4) FGMP_ERR(0, 3, 6)
    FGMP_ERR(1, 0, 8) FGMP_ERR(1, 1, 10) FGMP_ERR(1, 2, 12) FGMP_ERR(1, 3, 14)
#undef FGMP_ERR
#pragma unroll
    for (int w = 16; w > 1; w >>= 1)
#pragma unroll
        for (int i = 0; i < w / 2; ++i) t[i] = t[2 * i] + t[2 * i + 1];
    return t[0];
}

// Nearly the same error for less than two thirds of the instructions: sum of (g_i x_i - v_i (g_i d))^2 with g_i the root of the
// sensitivity.  t = x / d and gd = g d belong to a scale whose mantissa is the candidate's; the candidate's scale is `up` (a power
// of two) times that one, which the conversions apply exactly.
__device__ __forceinline__ float nvfp4_error_estimate(const float (&t)[16], const float (&gd)[16], const float (&y)[16], float up)
{
    uint32_t q[2] = {any_value(), any_value()};
    float sum[2] = {0.0f, 0.0f};
#define FGMP_ENC(W, B, I) q[W] = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(q[W], t[I], t[I + 1], up, B)
    FGMP_ENC(0, 0, 0); FGMP_ENC(0, 1, 2); FGMP_ENC(0, 2, 4); FGMP_ENC(0, 3, 6);
    FGMP_ENC(1, 0, 8); FGMP_ENC(1, 1, 10); FGMP_ENC(1, 2, 12); FGMP_ENC(1, 3, 14);
#undef FGMP_ENC
#define FGMP_ERR(W, B, I)                                                                \
    {                                                                                    \
        const float2_t v = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(q[W], up, B);        \
        const float e0 = __builtin_fmaf(-v[0], gd[I], y[I]), e1 = __builtin_fmaf(-v[1], gd[I + 1], y[I + 1]); \
        sum[0] = __builtin_fmaf(e0, e0, sum[0]);                                         \
        sum[1] = __builtin_fmaf(e1, e1, sum[1]);                                         \
    }
    FGMP_ERR(0, 0, 0) FGMP_ERR(0, 1, 2) FGMP_ERR(0, 2, 4) FGMP_ERR(0, 3, 6)
    FGMP_ERR(1, 0, 8) FGMP_ERR(1, 1, 10) FGMP_ERR(1, 2, 12) FGMP_ERR(1, 3, 14)
#undef FGMP_ERR
    return sum[0] + sum[1];
}

// Sensitivity-weighted clipping (Sec. 3.3, Eq. 11): for every block, the E4M3 scale code (0 .. 0x7E)
// whose NVFP4 quantization has the smallest weighted error, the smallest code among equal errors, and the first pass of
// packing (compact) under the scales found.  One wave per tile, one block per lane; the error of a candidate is computed
// exactly as quantize_kernel computes a block's score.  Offline (weights); bound: vector ALU (a candidate costs 112 vector
// instructions, 16 of them conversions at half rate), so what counts is how few candidates are tried.
//
// A candidate whose error is certain to exceed B, the smaller one of the errors under code 0 and under the dynamic-max
// code, cannot be the answer.  An error is a sum of non-negative terms added in FP32, so it is at least each of them:
//   too small a scale clips element i to 6 d: its term is at least F_i (|x_i| - 6 d)^2 > B where
//     6 d < |x_i| - sqrt(B / F_i);
//   too large a scale rounds element i to zero (|x_i| < d / 4): its term is F_i x_i^2, exactly as computed here; the sum of
//     these terms only grows with d, so four steps of bisection move the end of the range by up to 15 codes.
// The bounds are taken 1e-5 wide of these (the sum 1e-4), the rounding errors of a term being below 1e-6, and one code wide
// on top.  Where the argument needs more than that (negative or non-finite sensitivities, errors or scales near the ends of
// the FP32 range) every code is tried.
//
// The ranges of a wave's 64 blocks differ: on N(0, 0.02^2) weights with lognormal sensitivities 20 codes are left on
// average, 33 for the longest.  Lanes therefore try the mean number each, and what is left of the longer ranges is dealt out
// in equal pieces, the blocks going through LDS: 25 rounds instead of 33.
// 12288 x 4096 bf16, per-element sensitivities, the whole call: 1427 us with all 127 codes tried (and one division and one decode
// of the scale per candidate), 454 with the single-element bounds, 401 with the ranges dealt out, 328 with the packing
// pass done here (it read W and the sensitivities again, 65 us), 304 with the bisection, 250 with the candidates ranked by an
// estimate (74 instructions a candidate, its share of the preparation included, instead of 127) and one root per element for bounds and
// estimates.  6144 x 4096, FP32, without / with estimates: 153 / 118, pruned to a half 163 / 131, three values only 144 / 118, one
// sensitivity for all 143 / 112.  Where more than three codes tie in a block -- often in 4-bit integers with one sensitivity, and in
// weights with heavy tails, whose blocks are one or two elements and nothing -- its whole range is dealt out with what is left of
// the longer ones: 154 / 126 and 133 / 115 (tried by the block's own lane while the other 63 wait: 152 and 140).
template <typename Tin, bool kPerElem, bool kHW>
__global__ __launch_bounds__(256, 4) void clip_kernel(QuantParams p)
{
    constexpr uint32_t kOwnMore = 2;   // (codes beyond the mean number by estimate, the cheaper ones: 0 and 4 measure 1.5% more)
    constexpr int kStride = 36;   // floats per block in LDS: 16-byte pieces of neighbouring blocks in different banks
    __shared__ float2 tbl[128];   // {d, 1 / d} by scale code
    __shared__ __attribute__((aligned(16))) float blocks[4][64 * kStride];
    __shared__ uint64_t answer[4][64];
    __shared__ uint32_t pieces[4][64];
    if (threadIdx.x < 128) {
        const float d = e4m3_decode_int(threadIdx.x) * p.S;
        tbl[threadIdx.x] = make_float2(d, threadIdx.x != 0 ? 1.0f / d : 0.0f);
    }
    __syncthreads();
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t kt = blockIdx.x;
    const int64_t kb = kt * kTileBlocks + (lane & 7);
    const int64_t rt = (int64_t)blockIdx.y * 4 + wave;
    const int64_t row = rt * kTileRows + (lane >> 3);
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) write_packed_header(p);
    if (rt >= p.n_rt) return;
    const bool inside = kb < p.nb && row < p.rows;
    float x[16], f[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) x[i] = f[i] = 0.0f;
    if (inside) {
        RawBlock<Tin> raw;
        load_raw(static_cast<const Tin *>(p.X) + row * p.ldx + kb * kBlock, raw);
        widen(raw, x);
        load16(p.fisher + (kPerElem ? row * p.ld_fisher : 0) + kb * kBlock, f);
    }

    const float amax = block_amax(x);
    const float inv_S = 1.0f / p.S, S6 = 6.0f * p.S;
    auto error_with = [&](uint32_t sc) {
        if constexpr (kHW) {
            const float2 s = tbl[sc];
            return nvfp4_error(x, f, s.x, s.y);
        } else {
            BlockCodes bc;
            quantize_block_math<kHW, false>(x, f, amax, p.S, inv_S, S6, (int)sc, false, bc);
            return bc.score;
        }
    };
    uint32_t best = 0u;
    float lost[16], sum[16];   // the error under code 0: every element is lost
#pragma unroll
    for (int i = 0; i < 16; ++i) sum[i] = lost[i] = (x[i] * x[i]) * f[i];
#pragma unroll
    for (int w = 16; w > 1; w >>= 1)
#pragma unroll
        for (int i = 0; i < w / 2; ++i) sum[i] = sum[2 * i] + sum[2 * i + 1];
    float best_err = sum[0];
    uint32_t first = 1u, last = 0x7Eu;
    const float bound = fminf(best_err, error_with(enc_e4m3<kHW>(amax / S6)));
    float f_min = f[0], f_max = f[0], f_sum = 0.0f;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        f_min = fminf(f_min, f[i]);
        f_max = fmaxf(f_max, f[i]);
        f_sum += f[i];   // (minimum and maximum skip a NaN)
    }
    // (B / F_i >= 1e-30: the clipped element's error and its square are ordinary numbers)
    const bool nothing_less = best_err == 0.0f && f_min >= 0.0f && f_sum == f_sum;   // (a block of zeros)
    const bool bounded = bound > 1e-35f && bound > 1e-30f * f_max && bound < 1e25f && f_min >= 0.0f && f_max < 1e30f && f_sum == f_sum &&
                         amax < 1e15f && p.S > 1e-20f && p.S < 1e20f;
    float inv_root[16];   // reciprocal roots of the sensitivities
    if (bounded) {
        float d_low = 0.0f, d_high = 4.0f * amax;   // (beyond: all zeros, the error of code 0)
        const float root_bound = __builtin_amdgcn_sqrtf(bound) * 1.00001f;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const float ax = fabsf(x[i]);
            // (a vanishing sensitivity gives an infinite root, and no bound; of -0.0, too, whose own reciprocal root is -inf)
            inv_root[i] = __builtin_amdgcn_rsqf(fabsf(f[i]));
            d_low = fmaxf(d_low, __builtin_fmaf(-root_bound, inv_root[i], ax * 0.99999f) * (1.0f / 6.0f));
            if (lost[i] > bound) d_high = fminf(d_high, 4.0f * ax);
        }
        const uint32_t low = enc_e4m3<kHW>(fminf(d_low * 0.99999f * inv_S, 448.0f)), high = enc_e4m3<kHW>(fminf(d_high * 1.00001f * inv_S, 448.0f));
        first = low > 2u ? low - 1u : 1u;
        last = high < 0x7Du ? high + 1u : 0x7Eu;
        // all the elements that are rounded to zero together
#pragma unroll
        for (uint32_t step = 8u; step > 0u; step >>= 1) {
            const uint32_t sc = last > step ? last - step + 1u : 1u;
            // (1 - |x| / (d / 4), times 2^30, clamped to 0 .. 1: no more than 1, 0 for an element that is not lost)
            const float inv_d4 = tbl[sc].y * (4.0001f * 0x1p30f);
            float err = 0.0f;
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const float is_lost = __builtin_amdgcn_fmed3f(__builtin_fmaf(-fabsf(x[i]), inv_d4, 0x1p30f), 0.0f, 1.0f);
                err = __builtin_fmaf(is_lost, lost[i], err);
            }
            if (err * 0.9999f > bound) last = sc - 1u;
        }
    }
    if (!inside || nothing_less) last = 0u;
    // a block's x and f in LDS (of one wave: its accesses complete in order; nothing to wait for but the compiler)
    const float4 *const mine = reinterpret_cast<const float4 *>(&blocks[wave][lane * kStride]);
    auto fetch = [&](const float4 *from) {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float4 vx = from[i], vf = from[4 + i];
            x[4 * i] = vx.x; x[4 * i + 1] = vx.y; x[4 * i + 2] = vx.z; x[4 * i + 3] = vx.w;
            f[4 * i] = vf.x; f[4 * i + 1] = vf.y; f[4 * i + 2] = vf.z; f[4 * i + 3] = vf.w;
        }
    };
    // codes from .. to of the block in x, f
    auto search = [&](uint32_t from, uint32_t to) {
#pragma unroll 1
        for (uint32_t sc = from; sc <= to; ++sc) {
            const float err = error_with(sc);
            if (err < best_err) {
                best_err = err;
                best = sc;
            }
        }
    };
    // The first `own` codes (wave-uniform) of a range that ends at `to`, by estimates: codes 8 apart share a mantissa, so the block
    // is multiplied by one reciprocal for all of them.  With u = 2^-24, E the error and C that under code 0, estimate and error differ
    // by at most 40 u E + 8 u sqrt(C E) (the errors' own sums 6 u E, the estimate's 9 u E, the root 6 u E; per element u |x|, 2 u |v d| and
    // 2 u |e|, weighted and summed by Cauchy-Schwarz), so the code with the smallest error is among those whose estimate is within twice
    // that of the smallest one; `limit` allows another factor of two and the seven bits that the code replaces in a key.  Up to three
    // of them are compared by their errors; false where there are more.
    auto search_by_estimate = [&](uint32_t start, uint32_t to, uint32_t own) -> bool {
        const float c0_err = best_err;
        uint32_t k1 = ~0u, k2 = ~0u, k3 = ~0u, k4 = ~0u;   // the four smallest: estimate, code in the low seven bits
        float g[16], y[16];   // root of the sensitivity
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            g[i] = f[i] * fminf(inv_root[i], 1e30f);
            y[i] = g[i] * x[i];
        }
#pragma unroll 1
        for (uint32_t j = 0; j < 8u && j < own; ++j) {
            const float2 s = tbl[start + j < 127u ? start + j : 127u];
            float t[16], gd[16];
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                t[i] = x[i] * s.y;
                gd[i] = g[i] * s.x;
            }
            float up = 1.0f;
#pragma unroll 1
            for (uint32_t k = j; k < own; k += 8u) {
                const uint32_t sc = start + k;
                const float err = nvfp4_error_estimate(t, gd, y, up);
                const uint32_t key = sc <= to ? (__builtin_bit_cast(uint32_t, err) & ~127u) | sc : ~0u;
                const uint32_t l1 = max(k1, key), l2 = max(k2, l1), l3 = max(k3, l2);
                k1 = min(k1, key);
                k2 = min(k2, l1);
                k3 = min(k3, l2);
                k4 = min(k4, l3);
                up *= 2.0f;
            }
        }
        fetch(mine);   // (x and f need no registers in the loop above)
        auto estimate = [](uint32_t key) { return __builtin_bit_cast(float, key & ~127u); };
        const float least = estimate(k1);
        // (C E itself is below FP32's range for small sensitivities, and the root takes no subnormal number)
        const float root_ce = __builtin_amdgcn_sqrtf(c0_err) * __builtin_amdgcn_sqrtf(fmaxf(least, 0x1p-126f));
        const float limit = least * 1.00004f + 2e-6f * root_ce + 1e-12f * c0_err;
        auto close = [&](uint32_t key) { return key != ~0u && estimate(key) <= limit; };
        if (close(k4)) return false;
        auto consider = [&](uint32_t key) {
            const uint32_t sc = key & 127u;
            const float err = error_with(sc);
            if (err < best_err || (err == best_err && sc < best)) {
                best_err = err;
                best = sc;
            }
        };
        if (k1 != ~0u) consider(k1);
        if (close(k2)) consider(k2);
        if (close(k3)) consider(k3);
        return true;
    };
    if (__ballot(inside && !bounded && !nothing_less) != 0ull) {
        search(first, last);
    } else {
        // A lane tries up to `own` codes of its block.  What is left of the longer ranges -- and all of a range that estimates have
        // not narrowed down -- is cut in pieces of `rest` codes, at most one for each lane: rounding up to whole pieces adds less
        // than one piece to each of the n blocks with something left, so rest >= left / (64 - n) is enough (n = 64: one piece each).
        auto wave_sum = [](uint32_t v) {
#pragma unroll
            for (int d = 32; d > 0; d >>= 1) v += __shfl_xor(v, d);
            return (uint32_t)__builtin_amdgcn_readfirstlane((int)v);
        };
        const uint32_t width = last >= first ? last - first + 1u : 0u;
        auto stage = [&]() {
            float4 *to = reinterpret_cast<float4 *>(&blocks[wave][lane * kStride]);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                to[i] = make_float4(x[4 * i], x[4 * i + 1], x[4 * i + 2], x[4 * i + 3]);
                to[4 + i] = make_float4(f[4 * i], f[4 * i + 1], f[4 * i + 2], f[4 * i + 3]);
            }
        };
        // The estimate takes the root of a sensitivity and squares what is weighted with it: ordinary numbers as well, or zero.
        auto estimable = [&]() {
            uint32_t f_least = ~0u;
#pragma unroll
            for (int i = 0; i < 16; ++i) f_least = min(f_least, __builtin_bit_cast(uint32_t, f[i]) - 1u);
            return bounded && bound > 1e-30f && f_least >= __builtin_bit_cast(uint32_t, 1e-30f);
        };
        // (The estimates' preparation and the final comparison cost as much as eight codes save; the start of a second search a few
        // more.  Below code 8 scales are not normal numbers.)
        const uint32_t mean = (wave_sum(width) + 63u) / 64u;
        const bool by_estimate = kHW && mean >= 14u && __ballot(width != 0u && first < 8u) == 0ull && __ballot(width != 0u && !estimable()) == 0ull;
        const uint32_t own = mean + (by_estimate ? kOwnMore : 0u);
        uint32_t left = width > own ? width - own : 0u, left_from = first + own;
        const uint32_t own_last = left != 0u ? first + own - 1u : last;
        if (by_estimate) {
            stage();
            if (!search_by_estimate(first, own_last, own)) {
                left = width;
                left_from = first;
            }
        } else {
            search(first, own_last);
        }
        const uint64_t longer = __ballot(left != 0u);
        if (longer != 0ull) {
            if (!by_estimate) stage();
            const uint32_t spare = longer != ~0ull ? 64u - (uint32_t)__popcll(longer) : 1u;
            const uint32_t rest = (wave_sum(left) + spare - 1u) / spare;
            const uint32_t n_pieces = (left + rest - 1u) / rest;
            uint32_t at = n_pieces;   // inclusive prefix sum
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) {
                const uint32_t v = __shfl_up(at, d);
                at += lane >= d ? v : 0u;
            }
            const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)at, 63);
            at -= n_pieces;
            // errors are sums of non-negative numbers here: their bit patterns order them, the code decides between equal ones
            auto key = [&]() { return ((uint64_t)__builtin_bit_cast(uint32_t, best_err) << 32) | best; };
            answer[wave][lane] = key();
            for (uint32_t k = 0; k < n_pieces; ++k) {
                const uint32_t from = left_from + k * rest, to = from + rest - 1u < last ? from + rest - 1u : last;
                pieces[wave][at + k] = (uint32_t)lane | (from << 8) | (to << 16);
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            if ((uint32_t)lane < total) {
                const uint32_t piece = pieces[wave][lane];
                const uint32_t from_lane = piece & 0xFFu;
                fetch(reinterpret_cast<const float4 *>(&blocks[wave][from_lane * kStride]));
                best = 0xFFu;
                best_err = __builtin_inff();
                search((piece >> 8) & 0xFFu, piece >> 16);
                atomicMin(reinterpret_cast<unsigned long long *>(&answer[wave][from_lane]), (unsigned long long)key());
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            best = (uint32_t)answer[wave][lane];
            fetch(mine);
        }
    }

    // the block under the scale that was found, exactly as quantize_kernel writes it
    BlockCodes bc;
    quantize_block_math<kHW, false>(x, f, amax, p.S, inv_S, S6, (int)best, false, bc);
    const bool hi = inside && bc.score > p.T;
    if (p.scores != nullptr && inside) p.scores[row * p.nb + kb] = bc.score;
    store_tile<kHW, kModeCompact, false>(p, rt * p.n_kt + kt, lane, hi, __ballot(hi), bc, x, amax, inv_S);
}

// Second and last pass of packing weights (compact; none with a threshold of +inf): plane T -- the exclusive prefix sum over the tiles of
// their numbers of FP8 slots, from plane M --, plane H, and the header fields that depend on the total.  The
// FP8 upper halves are encoded from W once more, which touches only the rows' FP8 blocks: at 10% a fifth of
// W and none of the sensitivities, where a counting pass ahead of the packing pass reads all of both.
//
// A workgroup owns a run of consecutive tiles.  It finds the entries before its run by itself, counting the
// bits of all earlier mask words (8 bytes per tile out of the L2, half of the plane on average): no counter,
// no scan launch, no workgroup waits for another.  That reads 8 x kPackWgs / 2 bytes per tile out of the L2 -- as much as a
// bf16 tile of W -- whatever the size, 13% of the first pass below.  One wave per tile, one slot per lane.
// 22016 x 4096 bf16 with per-element sensitivities: counting pass 94 us, one-workgroup scan of plane T (a strided
// walk: 160 us) and packing pass 110 us before; packing pass 114 us and this kernel 15 us (no FP8 block) or 29 us (10%).
constexpr int kPackWaves = 16, kPackWgs = 512;

template <typename Tin>
__global__ __launch_bounds__(64 * kPackWaves) void pack_upper_halves_kernel(QuantParams p, uint32_t tiles_per_wave)
{
    __shared__ uint32_t before_part[kPackWaves], count_part[kPackWaves];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t n_tiles = (uint32_t)p.layout.n_tiles, n_kt = (uint32_t)p.n_kt;
    const uint32_t wg_tiles = tiles_per_wave * kPackWaves;
    const uint32_t wg_first = blockIdx.x * wg_tiles;   // (under 2^32 blocks of 16 in all: the tiles fit 32 bits with room)
    const uint32_t first = wg_first + wave * tiles_per_wave < n_tiles ? wg_first + wave * tiles_per_wave : n_tiles;
    const uint32_t last = first + tiles_per_wave < n_tiles ? first + tiles_per_wave : n_tiles;
    const uint64_t *masks = p.out.M;

    auto wave_sum = [](uint32_t v) {
#pragma unroll
        for (int d = 32; d > 0; d >>= 1) v += __shfl_xor(v, d);
        return v;
    };
    uint32_t before = 0, count = 0;
    {
        // two words per load; wg_first is even (16 waves)
        const uint4 *m2 = reinterpret_cast<const uint4 *>(masks);
        constexpr uint32_t kStep = 64 * kPackWaves, kFlight = 8;   // loads in flight per thread (one at a time: 20 us for 88064 tiles)
        auto bits = [](const uint4 &v) { return (uint32_t)(__popc(v.x) + __popc(v.y) + __popc(v.z) + __popc(v.w)); };
        uint32_t i = tid;
        for (; i + (kFlight - 1) * kStep < wg_first / 2; i += kFlight * kStep) {
            uint4 v[kFlight];
#pragma unroll
            for (uint32_t u = 0; u < kFlight; ++u) v[u] = m2[i + u * kStep];
#pragma unroll
            for (uint32_t u = 0; u < kFlight; ++u) before += bits(v[u]);
        }
        for (; i < wg_first / 2; i += kStep) before += bits(m2[i]);
        for (uint32_t i = first + lane; i < last; i += 64) count += (uint32_t)__popcll(masks[i]);
    }
    before = wave_sum(before);
    count = wave_sum(count);
    if (lane == 0) {
        before_part[wave] = before;
        count_part[wave] = count;
    }
    __syncthreads();
    uint32_t at = 0;   // entries before the wave's first tile
#pragma unroll
    for (int w = 0; w < kPackWaves; ++w) at += before_part[w] + (w < wave ? count_part[w] : 0u);

    const Tin *X = static_cast<const Tin *>(p.X);
    const float inv_S = 1.0f / p.S;
    uint32_t rt = first / n_kt, kt = first % n_kt;
    constexpr int kAhead = 4;   // tiles whose inputs are in flight together
    constexpr int kVec = (int)(8 * sizeof(Tin) / sizeof(uint4));
    for (uint32_t t0 = first; t0 < last; t0 += 64) {
        const uint32_t mine = t0 + lane;
        const uint64_t m = mine < last ? masks[mine] : 0ull;
        uint32_t incl = (uint32_t)__popcll(m);
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const uint32_t v = __shfl_up(incl, d);
            incl += lane >= d ? v : 0u;
        }
        const uint32_t start = at + incl - (uint32_t)__popcll(m);
        if (mine < last) p.out.T[mine] = start;
        at += __shfl(incl, 63);
        const int n = (int)(last - t0 < 64 ? last - t0 : 64);
        for (int j = 0; j < n; j += kAhead) {
            uint4 raw[kAhead][kVec];
            uint32_t dst[kAhead];
            bool hi[kAhead];
#pragma unroll
            for (int u = 0; u < kAhead; ++u) {
                const int src = j + u < 64 ? j + u : 63;   // (tiles past the run hold an empty mask)
                const uint64_t mu = j + u < n ? (((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(m >> 32), src) << 32) | (uint32_t)__builtin_amdgcn_readlane((int)m, src)) : 0ull;
                hi[u] = (mu >> lane) & 1ull;
                dst[u] = (uint32_t)__builtin_amdgcn_readlane((int)start, src) +
                         __builtin_amdgcn_mbcnt_hi((uint32_t)(mu >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mu, 0u));
                if (hi[u]) {
                    const int64_t row = (int64_t)rt * kTileRows + (lane >> 3), kb = (int64_t)kt * kTileBlocks + (lane & 7);
                    const uint4 *s = reinterpret_cast<const uint4 *>(X + row * p.ldx + kb * kBlock + 8);
#pragma unroll
                    for (int v = 0; v < kVec; ++v) raw[u][v] = s[v];
                }
                if (++kt == n_kt) {
                    kt = 0;
                    ++rt;
                }
            }
#pragma unroll
            for (int u = 0; u < kAhead; ++u)
                if (hi[u]) {
                    float r[16];
                    if constexpr (kVec == 1) {
                        const uint32_t w[4] = {raw[u][0].x, raw[u][0].y, raw[u][0].z, raw[u][0].w};
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            r[2 * i] = u2f(w[i] << 16);
                            r[2 * i + 1] = u2f(w[i] & 0xFFFF0000u);
                        }
                    } else {
#pragma unroll
                        for (int v = 0; v < kVec; ++v) {
                            r[4 * v] = u2f(raw[u][v].x);
                            r[4 * v + 1] = u2f(raw[u][v].y);
                            r[4 * v + 2] = u2f(raw[u][v].z);
                            r[4 * v + 3] = u2f(raw[u][v].w);
                        }
                    }
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        r[i] *= inv_S;
                        r[8 + i] = 0.0f;
                    }
                    uint32_t c[4];
                    encode_fp8_block<kUseHwCvt, true>(r, c);   // (the clamp changes nothing where it is not needed)
                    p.out.H[dst[u]] = make_uint2(c[0], c[1]);
                }
        }
    }
    // the wave that ends the tensor knows the total
    if (last == n_tiles && first < last && lane == 0) {
        p.out.hdr->h_entries = at;
        p.out.hdr->bytes_used = compact_bytes(p.layout, at);
    }
}

// One wave per tile, one slot per lane: packed -> canonical arrays.
__global__ __launch_bounds__(256) void unpack_kernel(PackedView v, PackedLayout l, uint8_t *codes,
                                                      uint8_t *scales, uint8_t *mask)
{
    const int lane = threadIdx.x & 63;
    const int64_t tile = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (tile >= l.n_tiles) return;
    const int64_t rt = tile / l.n_kt, kt = tile % l.n_kt;
    const int64_t row = rt * kTileRows + (lane >> 3);
    const int64_t kb = kt * kTileBlocks + (lane & 7);
    if (row >= l.rows || kb >= l.nb) return;
    const bool hi = (v.M[tile] >> lane) & 1ull;
    const uint2 lw = v.L[tile * kTileSlots + lane];
    const uint32_t sb = v.S[tile * kTileSlots + lane];
    uint4 out;
    if (hi) {
        const uint2 hw = v.H[(uint64_t)v.T[tile] + sb];
        out = make_uint4(lw.x, lw.y, hw.x, hw.y);
    } else {
        // spread 16 nibbles to 16 bytes
        uint32_t w[4];
        const uint32_t src[2] = {lw.x, lw.y};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint32_t h = (src[j >> 1] >> (16 * (j & 1))) & 0xFFFFu;  // 4 nibbles
            w[j] = (h & 0xFu) | ((h & 0xF0u) << 4) | ((h & 0xF00u) << 8) | ((h & 0xF000u) << 12);
        }
        out = make_uint4(w[0], w[1], w[2], w[3]);
    }
    if (codes) *reinterpret_cast<uint4 *>(codes + row * l.K + kb * kBlock) = out;
    if (scales) scales[row * l.nb + kb] = hi ? 0 : (uint8_t)sb;
    if (mask) mask[row * l.nb + kb] = hi ? 1 : 0;
}

// ---- host side ----

static int pick_rt_per_wave(int64_t n_rt)
{

    // enough work per wave to amortize the sensitivity loads, enough workgroups to fill 256 CUs
    if (n_rt >= 4096) return 4;
    if (n_rt >= 1024) return 2;
    return 1;
}

template <typename Tin, int kMode>
static void launch_quantize_mode(const QuantParams &p, bool per_elem, dim3 grid, hipStream_t st)
{
    if (p.delta) {
        if (per_elem)
            hipLaunchKernelGGL((quantize_kernel<Tin, true, kUseHwCvt, kMode, true>), grid, dim3(256), 0, st, p);
        else
            hipLaunchKernelGGL((quantize_kernel<Tin, false, kUseHwCvt, kMode, true>), grid, dim3(256), 0, st, p);
    } else {
        if (per_elem)
            hipLaunchKernelGGL((quantize_kernel<Tin, true, kUseHwCvt, kMode, false>), grid, dim3(256), 0, st, p);
        else
            hipLaunchKernelGGL((quantize_kernel<Tin, false, kUseHwCvt, kMode, false>), grid, dim3(256), 0, st, p);
    }
}

template <typename Tin>
static void launch_quantize(const QuantParams &p, bool per_elem, dim3 grid, hipStream_t st)
{
    switch (p.mode) {
    case kModeStrided: launch_quantize_mode<Tin, kModeStrided>(p, per_elem, grid, st); break;
    case kModeF16: launch_quantize_mode<Tin, kModeF16>(p, per_elem, grid, st); break;
    default: launch_quantize_mode<Tin, kModeCompact>(p, per_elem, grid, st); break;
    }
}

#ifdef FGMP_MEASUREMENT_HOOKS
// (measurement builds: the next activation tensor that takes the trimmed kernel runs its traffic model instead)
static thread_local bool g_traffic_model = false;
fgmp_status_t quantize_traffic_model(const void *X, fgmp_dtype_t dt, int64_t rows, int64_t K, int64_t ldx, const float *fisher,
                                     void *packed, size_t packed_bytes, hipStream_t st)
{
    if (make_layout(rows, K).n_tiles < kQMinTiles) return FGMP_ERR_UNSUPPORTED;
    g_traffic_model = true;
    const fgmp_status_t rc = quantize_tensor(X, dt, rows, K, ldx, fisher, 0, 0.0f, 1.0f, packed, packed_bytes, nullptr, false, st);
    const bool ran = !g_traffic_model;
    g_traffic_model = false;
    return rc != FGMP_OK ? rc : ran ? FGMP_OK : FGMP_ERR_UNSUPPORTED;
}
#endif

// What every quantizing call asks of its arguments.
fgmp_status_t check_quantizer_input(const void *X, fgmp_dtype_t dt, int64_t rows, int64_t K, int64_t ldx, const float *fisher, float T, float S,
                                    int score_mode, int64_t ld_fisher, const void *packed, const float *scores)
{
    if (score_mode != FGMP_SCORE_NVFP4_ERROR && score_mode != FGMP_SCORE_DELTA) return FGMP_ERR_INVALID_ARG;
    if (!X || !fisher) return FGMP_ERR_INVALID_ARG;
    if (rows <= 0 || K <= 0) return FGMP_ERR_INVALID_ARG;
    if (!(S > 0.0f) || !(S < INFINITY) || T != T) return FGMP_ERR_INVALID_ARG;
    if (dt != FGMP_F32 && dt != FGMP_BF16) return FGMP_ERR_UNSUPPORTED;
    if (K % kBlock != 0 || ldx < K || (ld_fisher != 0 && ld_fisher < K)) return FGMP_ERR_BAD_SHAPE;
    if (rows * (K / kBlock) >= (int64_t)1 << 32) return FGMP_ERR_UNSUPPORTED;
    const int64_t esz = (dt == FGMP_F32) ? 4 : 2;
    if (((uintptr_t)X | (uintptr_t)fisher | (uintptr_t)packed | (uintptr_t)scores) % 16 != 0 ||
        (ldx * esz) % 16 != 0 || (ld_fisher * 4) % 16 != 0)
        return FGMP_ERR_BAD_ALIGN;
    return FGMP_OK;
}

fgmp_status_t quantize_tensor(const void *X, fgmp_dtype_t dt, int64_t rows, int64_t K, int64_t ldx,
                              const float *fisher, int64_t ld_fisher, float T, float S, void *packed,
                              size_t packed_bytes, float *scores, bool compact, hipStream_t st,
                              _Float16 *x16, int64_t ld16, uint32_t *zero, int64_t zero_n, int score_mode,
                              bool clip, bool gated)
{
    if (!packed && !x16) return FGMP_ERR_INVALID_ARG;
    const fgmp_status_t rc = check_quantizer_input(X, dt, rows, K, ldx, fisher, T, S, score_mode, ld_fisher, packed, scores);
    if (rc != FGMP_OK) return rc;
    const PackedLayout l = make_layout(rows, K);
    if (x16 != nullptr) {
        // FP16 output: the packed buffer only receives the header
        if (compact || !kUseHwCvt) return FGMP_ERR_UNSUPPORTED;
        if (packed && packed_bytes < sizeof(PackedHeader)) return FGMP_ERR_BUFFER_TOO_SMALL;
        if (ld16 < l.n_kt * kTileK || (uintptr_t)x16 % 16 != 0 || (ld16 * 2) % 16 != 0) return FGMP_ERR_BAD_SHAPE;
    } else if (packed_bytes < l.total_bytes) {
        return FGMP_ERR_BUFFER_TOO_SMALL;
    }

    QuantParams p;
    p.X = X; p.ldx = ldx; p.rows = rows; p.nb = l.nb;
    p.fisher = fisher; p.ld_fisher = ld_fisher;
    p.T = T; p.S = S;
    if (packed) p.out = make_view(packed, l);
    else p.out = PackedView{};
    p.n_rt = l.n_rt; p.n_kt = l.n_kt;
    p.scores = scores;
    p.rt_per_wave = pick_rt_per_wave(l.n_rt);
    const int64_t rt_per_wg = 4 * (int64_t)p.rt_per_wave;
    const int64_t gy = (l.n_rt + rt_per_wg - 1) / rt_per_wg;
    if (gy > 65535 || l.n_kt > 0x7FFFFFFF) return FGMP_ERR_UNSUPPORTED;
    const dim3 grid((unsigned)l.n_kt, (unsigned)gy);
    const bool per_elem = ld_fisher != 0;

    p.layout = l;
    p.compact = compact ? 1u : 0u;
    p.x16 = x16; p.ld16 = ld16;
    if (zero_n < 0 || zero_n > 0x7FFFFFFF || (zero_n > 0 && !zero)) return FGMP_ERR_INVALID_ARG;
    p.zero = zero; p.zero_n = (int)zero_n;
    p.delta = score_mode == FGMP_SCORE_DELTA;
    p.no_fp8 = compact && T == INFINITY;
    // clipping is defined with the NVFP4-error score, for weights
    const int64_t clip_gy = (l.n_rt + 3) / 4;
    if (clip && (p.delta || !compact || clip_gy > 65535)) return FGMP_ERR_UNSUPPORTED;
    // (a gated product: FP32, quantized into a strided tensor)
    if (gated && (dt != FGMP_F32 || p.delta || compact || x16 != nullptr || per_elem || ldx < 2 * K)) return FGMP_ERR_UNSUPPORTED;
    // The activation hot path (one pass, NVFP4-error score, one sensitivity per channel, dynamic-max
    // scales) runs on the trimmed kernel when its 32-bit offsets and its shortcut division apply.
    const uint64_t x_bytes = (uint64_t)rows * (uint64_t)ldx * (dt == FGMP_F32 ? 4u : 2u);
    // (offsets: the input plus one stride of the resident set past its end must stay below 2^32)
    const bool fast = kUseHwCvt && !compact && !per_elem && !gated &&
                      x_bytes < 0x7FFFFF00ull && l.total_bytes < 0xFFFFFF00ull && S >= 1e-30f && S <= 1e30f &&
                      l.n_tiles >= kQMinTiles;
    if (fast) {
        p.mode = x16 != nullptr ? kModeF16 : kModeStrided;
        // one resident set of workgroups, a multiple of the number of K groups, with the row-tiles dealt out
        // evenly: two workgroups of eight waves per compute unit.  (The kernel's 85-93 registers let five waves
        // share a SIMD, i.e. two such workgroups a compute unit: a grid of three per compute unit ran its last
        // third as a second round, 72.9 us on 16384 x 8192 against 69.3; one per compute unit 81.6; three that
        // do fit -- the sensitivities moved to LDS, 74 registers -- 74.3: more waves only crowd the memory system.)
        constexpr int64_t kQResident = 512;
        const int64_t n_kg = (l.n_kt + kQWaves - 1) / kQWaves;
        int64_t gy = std::max<int64_t>(1, kQResident / n_kg);
        if (gy > l.n_rt) gy = l.n_rt;
        const int64_t its = (l.n_rt + gy - 1) / gy;
        gy = (l.n_rt + its - 1) / its;
        const dim3 fgrid((unsigned)(n_kg * gy));
        const uint32_t out_bytes = packed ? (uint32_t)(x16 != nullptr ? sizeof(PackedHeader) : l.total_bytes) : 0u;
        if (p.delta) {
            // the Eq. 8 score
            if (x16 != nullptr) {
                if (dt == FGMP_F32) hipLaunchKernelGGL((quantize_act_kernel<float, kModeF16, false, true>), fgrid, dim3(64 * kQWaves), 0, st, p, (uint32_t)x_bytes, out_bytes, (int)n_kg);
                else hipLaunchKernelGGL((quantize_act_kernel<uint16_t, kModeF16, false, true>), fgrid, dim3(64 * kQWaves), 0, st, p, (uint32_t)x_bytes, out_bytes, (int)n_kg);
            } else {
                if (dt == FGMP_F32) hipLaunchKernelGGL((quantize_act_kernel<float, kModeStrided, false, true>), fgrid, dim3(64 * kQWaves), 0, st, p, (uint32_t)x_bytes, out_bytes, (int)n_kg);
                else hipLaunchKernelGGL((quantize_act_kernel<uint16_t, kModeStrided, false, true>), fgrid, dim3(64 * kQWaves), 0, st, p, (uint32_t)x_bytes, out_bytes, (int)n_kg);
            }
        } else if (x16 != nullptr) {
            if (dt == FGMP_F32) hipLaunchKernelGGL((quantize_act_kernel<float, kModeF16>), fgrid, dim3(64 * kQWaves), 0, st, p, (uint32_t)x_bytes, out_bytes, (int)n_kg);
            else hipLaunchKernelGGL((quantize_act_kernel<uint16_t, kModeF16>), fgrid, dim3(64 * kQWaves), 0, st, p, (uint32_t)x_bytes, out_bytes, (int)n_kg);
#ifdef FGMP_MEASUREMENT_HOOKS
        } else if (g_traffic_model) {
            g_traffic_model = false;
            if (dt == FGMP_F32) hipLaunchKernelGGL((quantize_act_kernel<float, kModeStrided, true>), fgrid, dim3(64 * kQWaves), 0, st, p, (uint32_t)x_bytes, out_bytes, (int)n_kg);
            else hipLaunchKernelGGL((quantize_act_kernel<uint16_t, kModeStrided, true>), fgrid, dim3(64 * kQWaves), 0, st, p, (uint32_t)x_bytes, out_bytes, (int)n_kg);
#endif
        } else {
            if (dt == FGMP_F32) hipLaunchKernelGGL((quantize_act_kernel<float, kModeStrided>), fgrid, dim3(64 * kQWaves), 0, st, p, (uint32_t)x_bytes, out_bytes, (int)n_kg);
            else hipLaunchKernelGGL((quantize_act_kernel<uint16_t, kModeStrided>), fgrid, dim3(64 * kQWaves), 0, st, p, (uint32_t)x_bytes, out_bytes, (int)n_kg);
        }
    } else if (x16 != nullptr) {
        p.mode = kModeF16;
        if (dt == FGMP_F32) launch_quantize<float>(p, per_elem, grid, st);
        else launch_quantize<uint16_t>(p, per_elem, grid, st);
    } else if (gated) {
        p.mode = kModeStrided;
        hipLaunchKernelGGL((quantize_kernel<Gated, false, kUseHwCvt, kModeStrided, false>), grid, dim3(256), 0, st, p);
    } else if (!compact) {
        p.mode = kModeStrided;
        if (dt == FGMP_F32) launch_quantize<float>(p, per_elem, grid, st);
        else launch_quantize<uint16_t>(p, per_elem, grid, st);
    } else {
        p.mode = kModeCompact;
        const dim3 cgrid((unsigned)l.n_kt, (unsigned)clip_gy);
        if (clip && dt == FGMP_F32) {
            if (per_elem) hipLaunchKernelGGL((clip_kernel<float, true, kUseHwCvt>), cgrid, dim3(256), 0, st, p);
            else hipLaunchKernelGGL((clip_kernel<float, false, kUseHwCvt>), cgrid, dim3(256), 0, st, p);
        } else if (clip) {
            if (per_elem) hipLaunchKernelGGL((clip_kernel<uint16_t, true, kUseHwCvt>), cgrid, dim3(256), 0, st, p);
            else hipLaunchKernelGGL((clip_kernel<uint16_t, false, kUseHwCvt>), cgrid, dim3(256), 0, st, p);
        } else if (dt == FGMP_F32) launch_quantize<float>(p, per_elem, grid, st);
        else launch_quantize<uint16_t>(p, per_elem, grid, st);
        // Scoring a tensor before its threshold is known: no block is kept in FP8, and the pass above has written what follows
        // from that.  22016 x 4096 bf16 with per-element sensitivities: 114 us instead of 114 + 22.
        if (p.no_fp8) return hipGetLastError() == hipSuccess ? FGMP_OK : FGMP_ERR_HIP;
        const int64_t waves = (int64_t)kPackWgs * kPackWaves;
        const uint32_t tiles_per_wave = (uint32_t)((l.n_tiles + waves - 1) / waves);
        const int64_t wg_tiles = (int64_t)tiles_per_wave * kPackWaves;
        const dim3 pgrid((unsigned)((l.n_tiles + wg_tiles - 1) / wg_tiles));
        if (dt == FGMP_F32) hipLaunchKernelGGL((pack_upper_halves_kernel<float>), pgrid, dim3(64 * kPackWaves), 0, st, p, tiles_per_wave);
        else hipLaunchKernelGGL((pack_upper_halves_kernel<uint16_t>), pgrid, dim3(64 * kPackWaves), 0, st, p, tiles_per_wave);
    }
    return hipGetLastError() == hipSuccess ? FGMP_OK : FGMP_ERR_HIP;
}

fgmp_status_t unpack_tensor(const void *packed, int64_t rows, int64_t K, uint8_t *codes, uint8_t *scales,
                            uint8_t *mask, hipStream_t st)
{
    if (!packed || rows <= 0 || K <= 0) return FGMP_ERR_INVALID_ARG;
    if (K % kBlock != 0) return FGMP_ERR_BAD_SHAPE;
    if (((uintptr_t)packed | (uintptr_t)codes) % 16 != 0) return FGMP_ERR_BAD_ALIGN;
    const PackedLayout l = make_layout(rows, K);
    const PackedView v = make_view(const_cast<void *>(packed), l);
    const int64_t nwg = (l.n_tiles + 3) / 4;
    if (nwg > 0x7FFFFFFF) return FGMP_ERR_UNSUPPORTED;
    hipLaunchKernelGGL(unpack_kernel, dim3((unsigned)nwg), dim3(256), 0, st, v, l, codes, scales, mask);
    return hipGetLastError() == hipSuccess ? FGMP_OK : FGMP_ERR_HIP;
}

// ---- conversion self-test kernels ----

template <int kFormat> __device__ __forceinline__ uint32_t selftest_encode(float r)
{
    if constexpr (kFormat == 2) return e2m1_encode_int(r);
    else if constexpr (kFormat == 3) return e4m3_encode_int(r);
    else if constexpr (kFormat == 4) return e2m1_encode_pair_hw(r, 0.0f) & 0xFu;
    else return e4m3_encode_pair_hw(r, 0.0f) & 0xFFu;
}

constexpr uint32_t kLastPattern = 0x7F800000u;   // +INF
constexpr uint32_t kRunLength = 4096;

template <int kFormat>
__global__ __launch_bounds__(256) void encode_ranges_kernel(uint32_t *min_bits, uint32_t *max_bits,
                                                             uint32_t *violations)
{
    const uint64_t first = ((uint64_t)blockIdx.x * 256 + threadIdx.x) * kRunLength;
    if (first > kLastPattern) return;
    uint64_t last = first + kRunLength - 1;
    if (last > kLastPattern) last = kLastPattern;
    uint32_t cur = selftest_encode<kFormat>(u2f((uint32_t)first)) & 0xFFu;
    uint32_t start = (uint32_t)first;
    for (uint64_t b = first + 1; b <= last; ++b) {
        const uint32_t c = selftest_encode<kFormat>(u2f((uint32_t)b)) & 0xFFu;
        if (c != cur) {
            atomicMin(&min_bits[cur], start);
            atomicMax(&max_bits[cur], (uint32_t)(b - 1));
            if (c < cur) atomicAdd(violations, 1u);
            cur = c;
            start = (uint32_t)b;
        }
    }
    atomicMin(&min_bits[cur], start);
    atomicMax(&max_bits[cur], (uint32_t)last);
}

__global__ void init_ranges_kernel(uint32_t *min_bits, uint32_t *max_bits, uint32_t *violations)
{
    min_bits[threadIdx.x] = 0xFFFFFFFFu;
    max_bits[threadIdx.x] = 0u;
    if (threadIdx.x == 0) *violations = 0u;
}

__global__ void decode_table_kernel(int format, float *out)
{
    const uint32_t c = threadIdx.x;
    float v;
    switch (format) {
    case 2: v = e2m1_decode_int(c & 0xFu); break;
    case 3: v = e4m3_decode_int(c); break;
    case 4: v = e2m1_decode_pair_hw(c & 0xFu)[0]; break;
    default: v = e4m3_decode_pair_hw(c)[0]; break;
    }
    out[c] = v;
}

fgmp_status_t selftest_encode_ranges(int format, uint32_t *min_bits, uint32_t *max_bits,
                                     uint32_t *violations, hipStream_t st)
{
    if (!min_bits || !max_bits || !violations) return FGMP_ERR_INVALID_ARG;
    if (format < 0 || format > 5) return FGMP_ERR_INVALID_ARG;
    if (format < 2) format += kUseHwCvt ? 4 : 2;   // the form the quantizer uses
    hipLaunchKernelGGL(init_ranges_kernel, dim3(1), dim3(256), 0, st, min_bits, max_bits, violations);
    const uint64_t n_threads = ((uint64_t)kLastPattern + kRunLength) / kRunLength;
    const dim3 grid((unsigned)((n_threads + 255) / 256));
    switch (format) {
    case 2: hipLaunchKernelGGL((encode_ranges_kernel<2>), grid, dim3(256), 0, st, min_bits, max_bits, violations); break;
    case 3: hipLaunchKernelGGL((encode_ranges_kernel<3>), grid, dim3(256), 0, st, min_bits, max_bits, violations); break;
    case 4: hipLaunchKernelGGL((encode_ranges_kernel<4>), grid, dim3(256), 0, st, min_bits, max_bits, violations); break;
    default: hipLaunchKernelGGL((encode_ranges_kernel<5>), grid, dim3(256), 0, st, min_bits, max_bits, violations); break;
    }
    return hipGetLastError() == hipSuccess ? FGMP_OK : FGMP_ERR_HIP;
}

fgmp_status_t selftest_decode_table(int format, float *out, hipStream_t st)
{
    if (!out || format < 0 || format > 5) return FGMP_ERR_INVALID_ARG;
    if (format < 2) format += kUseHwCvt ? 4 : 2;
    hipLaunchKernelGGL(decode_table_kernel, dim3(1), dim3(256), 0, st, format, out);
    return hipGetLastError() == hipSuccess ? FGMP_OK : FGMP_ERR_HIP;
}

}  // namespace fgmp
