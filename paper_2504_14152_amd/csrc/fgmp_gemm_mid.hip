// Block-mixed-precision GEMM (Sec. 4.1) for tens to hundreds of activation rows, and up to 4096 over few columns or a short
// K: between the decode step that streams the weights past a handful of rows and the prefill kernel whose 256 x 256
// tiles are too few to fill the chip here.
//
// What bounds it: at 64 rows the weights' bytes, the activations' way to the compute units, the decode and the
// matrix instructions take about the same time (3-4 us each for a Llama-2-7B QKV product), there are never enough
// tiles to occupy 256 compute units, and every pass over memory that is not an operand -- partial sums -- costs as
// much as the operands do.  Hence:
//   * K is split inside the workgroup first.  A workgroup of eight waves covers 16 MT rows x 16 NT WN columns; its
//     WK groups of WN waves take WK consecutive K-tiles (128 elements each) of a "round" and add their
//     accumulators through LDS at the end: an output tile a quarter of the prefill kernel's, with as much
//     matrix work per barrier.  Only where that leaves compute units idle, K is split over workgroups as well.
//   * The weights never touch LDS.  A wave decodes the blocks of its own 16 NT columns straight into the B
//     operands of 16x16x32 matrix instructions; no other wave of the workgroup needs them, so nothing is
//     decoded twice.  Lane (n = lane % 16, g = lane / 16) owns blocks 2g, 2g+1 of weight row n of a K-tile;
//     matrix instruction j reduces over elements 8 (j % 2) .. + 7 of block 2g + j / 2 for g = 0..3.  The first or
//     second blocks of a K-tile ("half" of it) are decoded between the matrix instructions of the half before: with the
//     decode in a stretch of its own the two waves of a SIMD decode at the same time and the matrix pipe idles (a round
//     of MT = 8, NT = 3 took 3.1 us, the sum of both, against 1.5 us of matrix instructions).  The decode has no branch for the
//     same reason: value = fma(4-bit value, scale, 8-bit value) with the scale, or the 8-bit codes, masked to zero.
//   * The activations (FP16 values, written by the quantizer) go to LDS directly, two rounds deep, one barrier
//     per round.  A row of a K-tile is 256 bytes = 16 chunks; stored in an order that
//     makes the 16-byte operand reads free of bank conflicts.
//   * Where the activations are at most one block per thread of the launch, the launch quantizes them (kQuantize): workgroups that
//     hold a share (mid_units) make its FP16 values and say so; all ask for their first weights and wait for the other shares.  A quantizer
//     launch costs 4 us of which 1.5 are work, this 2 us more before the first round: 64 rows 4096 x 12288 18.3 / 16.7, 77 rows 2064
//     x 5003 13.2 / 11.5, 120 rows 368 x 603 8.5 / 7.2, 200 rows 4096 x 22016 44.7 / 43.7 us.  With two blocks per thread the
//     shares take as long as the launch they replace (872 x 3408 x 764 (M, K, N) 22.8 / 23.2, 512 x 11008 x 4096 with three 56.8 /
//     58.0), and workgroups beyond the first 256 would wait again (663 x 4096 x 22016 127 / 130).
//   * Workgroups that run at the same time on an XCD work on the same rows and the same part of K, tile by tile along
//     N, so the activations come from that XCD's L2.
// All loads of the loop are assembly with hand-counted waits, two per round: while a direct load to LDS is pending the
// compiler waits for every load wherever it needs one, and where it does not know of the direct loads its waits are as
// bad (1.8 us instead of 1.2 for a round of MT = 4, NT = 2: the first wait after the activations' loads waited for them).
#include <algorithm>
#include <cstdlib>
#include <type_traits>

#include "fgmp_gemm_common.hpp"
#include "fgmp_quant_block.hpp"

namespace fgmp {

// (a build with FGMP_FULL_WAITS waits for every load: nothing to miscount, the same result bit for bit)
#ifdef FGMP_FULL_WAITS
#define FGMP_MID_PENDING(n) 0
#else
#define FGMP_MID_PENDING(n) (n)
#endif

constexpr int kMidThreads = 512;
// Workgroups that share the quantizing, at most; how often one looks whether the others are done (0.7 us a look; the shares take 2
// us) before it makes a share itself that another one has begun.
constexpr uint32_t kMidMaxUnits = 256;
constexpr int kMidPatience = 8;
// Behind the units' words: how many workgroups wait no longer, in sixteen counters on lines of their own (192 additions to one
// word took 2 us), then how many of these are complete.
constexpr uint32_t kMidPassed = kMidMaxUnits, kMidPassedGroups = 16, kMidPassedStep = 16;
constexpr uint32_t kMidPassedAll = kMidPassed + kMidPassedGroups * kMidPassedStep;
// ... and a second word per unit: somebody has begun its share.
constexpr uint32_t kMidBegun = kMidPassedAll + 16, kMidDoneWords = kMidBegun + kMidMaxUnits;
constexpr uint32_t kMidRsrc = 0x00020000;   // raw buffer, 32-bit data format

// division by a constant that the host knows; exact for dividends below 2^16 and divisors below 2^16
struct MidDiv {
    uint32_t d, mul;
    static MidDiv by(uint32_t d) { return MidDiv{d, d > 1 ? (uint32_t)(0x100000000ull / d) + 1u : 0u}; }
    __device__ __forceinline__ uint32_t operator()(uint32_t v) const { return d == 1u ? v : __umulhi(v, mul); }
};

// Activations that the launch quantizes itself.  They are dealt out 64 blocks at a time: chunk c to wave c / n_units of
// workgroup c % n_units.
struct MidQuant {
    const void *X;
    const float *fisher;
    float T, S;
    int f32, delta;             // FP32 input (else bf16); the Eq. 8 score
    uint32_t x_bytes, row_bytes;
    uint32_t nb;                // blocks of a row
    uint32_t row_blocks, row_mul;   // blocks of a row in whole K-tiles, and its divisor's multiplier
    uint32_t n_chunks, n_units, n_own;   // n_own: units whose workgroups make them (all; fewer only in a test)
    int patience;
    uint32_t *done;             // one word per unit, then counters (kMidPassed), words again (kMidBegun); zero between launches
};

struct MidArgs {
    const void *w;              // packed weights (header first)
    const _Float16 *x16;        // [tiles_m * 16 MT][ld16]; rows from M on hold anything
    float *Y;
    uint32_t off_L, off_S, off_M, off_T, off_H;          // layout of the packed weights
    uint32_t ld_bytes;
    int M, N, n_kt, n_rt;
    int rounds, parts;          // rounds of a tile; workgroups that share them
    MidDiv by_tiles_n, by_parts;
    uint32_t n_wgs;
    uint32_t partial_bytes;
    float *partial;
    uint32_t *counters;         // one per tile, 2^counter_shift words apart; zero between launches
    int counter_shift;
    const PackedHeader *xh;     // header of the activations (tensor scale, shape check)
    int64_t ldy;
    int64_t w_rows, w_K, x_rows, x_K;                    // the shapes the headers must state
    MidQuant q;
};

// A block of the activations on its way: chunk c of the launch, a lane's block.
struct MidBlock {
    u32x4_t x[4], f[4];   // (bf16: two of x)
    bool valid;
};
__device__ __forceinline__ void mid_place(const MidQuant &q, uint32_t b, uint32_t &m, uint32_t &kb)
{
    m = __umulhi(b, q.row_mul);
    kb = b - m * q.row_blocks;
}
// (loads outside the tensor: beyond the buffers, zeros)
__device__ __forceinline__ void mid_load_block(const MidArgs &a, uint32_t c, int lane, MidBlock &r)
{
    const MidQuant &q = a.q;
    uint32_t m, kb;
    mid_place(q, c * 64u + (uint32_t)lane, m, kb);
    r.valid = c < q.n_chunks && m < (uint32_t)a.M && kb < q.nb;
    const __amdgpu_buffer_rsrc_t xbuf = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(q.X), 0, (int)q.x_bytes, kMidRsrc);
    const __amdgpu_buffer_rsrc_t fbuf = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(q.fisher), 0, (int)(q.nb * (kBlock * 4u)), kMidRsrc);
    const uint32_t xoff = r.valid ? m * q.row_bytes + kb * (q.f32 ? kBlock * 4u : kBlock * 2u) : 0xFFFFFF00u;
    const uint32_t foff = r.valid ? kb * (kBlock * 4u) : 0xFFFFFF00u;
    r.x[0] = __builtin_amdgcn_raw_buffer_load_b128(xbuf, (int)xoff, 0, 0);
    r.x[1] = __builtin_amdgcn_raw_buffer_load_b128(xbuf, (int)xoff + 16, 0, 0);
    if (q.f32) {
        r.x[2] = __builtin_amdgcn_raw_buffer_load_b128(xbuf, (int)xoff + 32, 0, 0);
        r.x[3] = __builtin_amdgcn_raw_buffer_load_b128(xbuf, (int)xoff + 48, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) r.f[i] = __builtin_amdgcn_raw_buffer_load_b128(fbuf, (int)foff + 16 * i, 0, 0);
}
// FP16 values of the chunk's blocks, in memory when the wave's stores are complete (coherent across XCDs: other workgroups read
// them in this launch).  A lane's block is 32 bytes; through LDS (2 KB of the wave's own) every store instruction writes whole lines.
__device__ __forceinline__ void mid_quantize_block(const MidArgs &a, uint32_t c, int lane, const MidBlock &r, char *lds_wave)
{
    const MidQuant &q = a.q;
    float x[16], f[16];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) f[4 * i + e] = u2f(r.f[i][e]);
    if (q.f32) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) x[4 * i + e] = u2f(r.x[i][e]);
    } else {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) {   // bf16 -> fp32 is a 16-bit shift
                x[8 * i + 2 * e] = u2f(r.x[i][e] << 16);
                x[8 * i + 2 * e + 1] = u2f(r.x[i][e] & 0xFFFF0000u);
            }
    }
    half2_t o[8];
    if (q.delta) quantize_block_f16<true>(x, f, r.valid, q.T, q.S, 1.0f / q.S, 6.0f * q.S, o);
    else quantize_block_f16<false>(x, f, r.valid, q.T, q.S, 1.0f / q.S, 6.0f * q.S, o);
    union { half2_t h[8]; u32x4_t v[2]; } pack;
#pragma unroll
    for (int j = 0; j < 8; ++j) pack.h[j] = o[j];
    u32x4_t *mine = reinterpret_cast<u32x4_t *>(lds_wave + lane * 32);
    mine[0] = pack.v[0];
    mine[1] = pack.v[1];
    // (one wave's LDS accesses are served in order; nobody else uses this part of the LDS)
    const __amdgpu_buffer_rsrc_t out = __builtin_amdgcn_make_buffer_rsrc(const_cast<_Float16 *>(a.x16), 0, (int)((uint32_t)a.M * a.ld_bytes), kMidRsrc);
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        uint32_t m, kb;
        mid_place(q, c * 64u + (uint32_t)(j * 32 + (lane >> 1)), m, kb);
        const u32x4_t v = *reinterpret_cast<const u32x4_t *>(lds_wave + j * 1024 + lane * 16);
        const uint32_t at = m < (uint32_t)a.M ? m * a.ld_bytes + kb * (kBlock * 2u) + (uint32_t)(lane & 1) * 16u : 0xFFFFFF00u;
        __builtin_amdgcn_raw_buffer_store_b128(v, out, (int)at, 0, kCoherent);
    }
}
// kQuantize: the activations are quantized by this launch (Sec. 4.2), a share by every workgroup that holds one; all wait for the others'.
// No workgroup depends on another one running: a share that nobody has begun at its second look it makes itself, one that is begun
// and does not come when its patience ends, too, the same values (two launches that fill the chip together on two streams would
// wait for each other's workgroups to leave).  The values
// are stored past the L2s (system-coherent), complete before the share's word is set, and read through the reader's L2 only after
// that: no L2 holds an older copy, since a launch starts with its L2 lines of earlier launches invalidated and reads none
// of the values before the words say so.
template <int MT, int NT, int WN, int WK, bool kQuantize>
__global__ __launch_bounds__(kMidThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void gemm_mid_kernel(MidArgs a)
{
    static_assert(WN * WK == 8, "eight waves");
    constexpr int kRows = 16 * MT, kCols = 16 * NT * WN;
    constexpr int kRowB = kTileK * 2;                         // 256 bytes of a row per K-tile
    constexpr int kGroupBytes = kRows * kRowB;                // one K-tile of activations
    constexpr int kStage = WK * kGroupBytes;
    constexpr int kALoads = kRows / (4 * WN);                 // direct loads per wave and round: 1 KB = 4 rows of a K-tile each
    constexpr int kWLoads = 5 * NT;                           // loads to registers per wave and round: planes L, H, S, M, T
    constexpr int kRedBytes = (WK - 1) * MT * NT * WN * 1024;
    constexpr int kLds = 2 * kStage > kRedBytes ? 2 * kStage : kRedBytes;
    __shared__ __attribute__((aligned(1024))) char lds[kLds];
    __shared__ uint32_t arrived;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wn = wave % WN, wk = wave / WN;
    const int nl = lane & 15, g = lane >> 4;

    // the arguments span several cache lines: all requested together, one trip instead of one for each
    {
        typedef const uint32_t __attribute__((address_space(4))) *const_words_t;
        const_words_t ka = (const_words_t)__builtin_amdgcn_kernarg_segment_ptr();
        uint32_t touch = 0;
#pragma unroll
        for (size_t off = 0; off < sizeof(MidArgs); off += 64) touch ^= ka[off / 4];
        asm volatile("" ::"s"(touch));
    }

    // dispatch goes round the XCDs: consecutive indices w belong to one of them
    uint32_t w = blockIdx.x;
    if (a.n_wgs % kNumXcd == 0) w = (w % kNumXcd) * (a.n_wgs / kNumXcd) + w / kNumXcd;
    const uint32_t mp = a.by_tiles_n(w), n_idx = w - mp * a.by_tiles_n.d;
    const uint32_t m_idx = a.by_parts(mp), part = mp - m_idx * a.by_parts.d;
    const uint32_t tile = m_idx * a.by_tiles_n.d + n_idx;
    const int m0 = (int)m_idx * kRows, n0 = (int)n_idx * kCols;
    const int r0 = (int)a.by_parts(part * (uint32_t)a.rounds), r1 = (int)a.by_parts((part + 1u) * (uint32_t)a.rounds);

    const int kt_end = r1 * WK < a.n_kt ? r1 * WK : a.n_kt;   // K-tiles of this workgroup end here
    auto k_tile = [&](int r) { return r * WK + wk < a.n_kt ? r * WK + wk : a.n_kt - 1; };   // (past the tensor: never used)
    // Chunk c of row r sits at position c ^ swizzle(r).  A 16-byte read is served 16 lanes at a time -- lanes 0-3, 12-15, 20-23,
    // 24-27 first, i.e. rows 0-3, 12-15 of one chunk column and rows 4-11 of the next but three --: with r % 16 alone half of
    // the LDS cycles were conflicts.
    auto swizzle = [](int row) { return (row & 15) ^ ((row & 4) << 1); };
    // ---- activations, direct to LDS: the WN waves of a K group load its K-tile, 4 rows (1 KB) at a time; lane (row lane / 16,
    // position lane % 16) fetches the chunk that belongs at its position
    const char *x_wave = reinterpret_cast<const char *>(a.x16) + (int64_t)(m0 + 4 * wn) * a.ld_bytes;
    const uint32_t x_row = (uint32_t)(lane >> 4) * a.ld_bytes, x_swz = (uint32_t)(nl ^ swizzle(((wn & 3) << 2) | (lane >> 4))) << 4;
    const uint32_t x_off[2] = {x_row + x_swz, x_row + (WN == 2 ? x_swz ^ 128u : x_swz)};   // (with WN = 2 every second load is 8 rows on)
    const int64_t x_step = (int64_t)a.ld_bytes * (4 * WN);
    auto issue_a = [&](int r, int stage, int i) {
        const char *base = x_wave + (int64_t)k_tile(r) * kRowB + i * x_step;
        const uint32_t dst = (uint32_t)(uintptr_t)(lds_void_t *)&lds[stage * kStage + wk * kGroupBytes + wn * 1024 + i * (WN * 1024)];
        load_direct16(dst, x_off[i & 1], base);
    };
    // operand reads: row nl of a 16-row group, chunk 4 g + j
    const uint32_t f_lds = (uint32_t)(wk * kGroupBytes + nl * kRowB + (((4 * g) ^ swizzle(nl)) << 4));

    // ---- weights: row of the lane in each column group, as the slot of its first block in the first tile of its row-tile
    // (rows beyond the tensor read a valid tile; their products only reach columns that are never stored)
    // (of rounds past the workgroup's last one the same loads are issued, since the waits count them, through a buffer of no bytes:
    // zeros come back at once, where the loads themselves were waited for by the sums: 0.9 us)
    auto wbuf_of = [&](int r) { return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(a.w), 0, r < r1 ? (int)a.off_H : 0, kMidRsrc); };
    uint32_t e0[NT], t0[NT];
#pragma unroll
    for (int q = 0; q < NT; ++q) {
        const int row = n0 + (wn * NT + q) * 16 + nl;
        const int rt = (row >> 3) < a.n_rt ? row >> 3 : a.n_rt - 1;
        t0[q] = (uint32_t)rt * (uint32_t)a.n_kt;
        e0[q] = t0[q] * kTileSlots + (uint32_t)((row & 7) * kTileBlocks + 2 * g);
    }
    u32x4_t wl[2][NT], wu[2][NT];   // planes L and H of a round's K-tile
    uint32_t ws[2][NT];             // plane-S bytes of the lane's two blocks
    uint64_t is8[2][NT][2];         // lanes whose first, second block is FP8
    uint32_t ns[NT], nm[NT], nt[NT];
    auto load_meta = [&](__amdgpu_buffer_rsrc_t wbuf, int r, int q) {
        const uint32_t kt = (uint32_t)__builtin_amdgcn_readfirstlane(k_tile(r));
        asm volatile("buffer_load_ushort %0, %1, %2, %3 offen" : "=v"(ns[q]) : "v"(a.off_S + e0[q]), "s"(wbuf), "s"(kt * kTileSlots));
        asm volatile("buffer_load_ubyte %0, %1, %2, %3 offen" : "=v"(nm[q]) : "v"(a.off_M + t0[q] * 8u + (uint32_t)(nl & 7)), "s"(wbuf), "s"(kt * 8u));
        asm volatile("buffer_load_dword %0, %1, %2, %3 offen" : "=v"(nt[q]) : "v"(a.off_T + t0[q] * 4u), "s"(wbuf), "s"(kt * 4u));
    };
    auto load_l = [&](__amdgpu_buffer_rsrc_t wbuf, int r, int set, int q) {
        const uint32_t kt = (uint32_t)__builtin_amdgcn_readfirstlane(k_tile(r));
        asm volatile("buffer_load_dwordx4 %0, %1, %2, %3 offen" : "=v"(wl[set][q]) : "v"(a.off_L + e0[q] * 8u), "s"(wbuf), "s"(kt * (kTileSlots * 8u)));
    };
    // At most kPending loads outstanding; the named registers hold what was loaded from here on.  (Until the wait that
    // names it a register must not be touched; every register is named again at the end, so none is reused early.)
    auto wait_meta = [&](auto pending_c) {
        (void)ns, (void)nm, (void)nt;
        if constexpr (NT == 2)
            asm volatile("s_waitcnt vmcnt(%6)" : "+v"(ns[0]), "+v"(nm[0]), "+v"(nt[0]), "+v"(ns[1]), "+v"(nm[1]), "+v"(nt[1]) : "n"(FGMP_MID_PENDING(decltype(pending_c)::value)) : "memory");
        else if constexpr (NT == 3)
            asm volatile("s_waitcnt vmcnt(%9)" : "+v"(ns[0]), "+v"(nm[0]), "+v"(nt[0]), "+v"(ns[1]), "+v"(nm[1]), "+v"(nt[1]), "+v"(ns[2]), "+v"(nm[2]), "+v"(nt[2])
                         : "n"(FGMP_MID_PENDING(decltype(pending_c)::value)) : "memory");
        else
            asm volatile("s_waitcnt vmcnt(%12)" : "+v"(ns[0]), "+v"(nm[0]), "+v"(nt[0]), "+v"(ns[1]), "+v"(nm[1]), "+v"(nt[1]), "+v"(ns[2]), "+v"(nm[2]), "+v"(nt[2]),
                         "+v"(ns[NT - 1]), "+v"(nm[NT - 1]), "+v"(nt[NT - 1]) : "n"(FGMP_MID_PENDING(decltype(pending_c)::value)) : "memory");
    };
    auto landed = [&](u32x4_t (&l)[NT], u32x4_t (&u)[NT]) {   // (no instruction: the wait before it was for younger loads)
        if constexpr (NT == 2) asm volatile("" : "+v"(l[0]), "+v"(l[1]), "+v"(u[0]), "+v"(u[1]));
        else if constexpr (NT == 3) asm volatile("" : "+v"(l[0]), "+v"(l[1]), "+v"(l[2]), "+v"(u[0]), "+v"(u[1]), "+v"(u[2]));
        else asm volatile("" : "+v"(l[0]), "+v"(l[1]), "+v"(l[2]), "+v"(l[NT - 1]), "+v"(u[0]), "+v"(u[1]), "+v"(u[2]), "+v"(u[NT - 1]));
    };
    auto words = [&](uint32_t from) { return __builtin_amdgcn_make_buffer_rsrc(a.q.done + from, 0, (int)(kMidMaxUnits * 4u), kMidRsrc); };
    if constexpr (kQuantize) {
        const uint32_t c = blockIdx.x < a.q.n_own ? (uint32_t)wave * a.q.n_units + blockIdx.x : a.q.n_chunks;
        if (c < a.q.n_chunks) {
            MidBlock b;
            mid_load_block(a, c, lane, b);
            // (by the first lane, the others' beyond the buffer: no branch, behind which a wait for the loads would be one for the store, too;
            // in front of the loads it is what they wait for, 0.3 us)
            __builtin_amdgcn_raw_buffer_store_b32(1u, words(kMidBegun), (int)(tid == 0 ? blockIdx.x * 4u : 0xFFFFFF00u), 0, kCoherent);
            mid_quantize_block(a, c, lane, b, lds + wave * 2048);
        }
        asm volatile("" ::: "memory");   // (its stores are older than the loads that follow: a wait counts on it)
    }
#pragma unroll
    for (int q = 0; q < NT; ++q) load_meta(wbuf_of(r0), r0, q);
    if constexpr (!kQuantize) {
#pragma unroll
        for (int i = 0; i < kALoads; ++i) issue_a(r0, 0, i);
    }
#pragma unroll
    for (int q = 0; q < NT; ++q) load_l(wbuf_of(r0), r0, 0, q);
    // The weights' header, needed for the first plane-H entries: asked for behind the loads above (scalar loads in front of them
    // held all of them up for a memory round trip, 0.9 us).
    uintptr_t wh_at = reinterpret_cast<uintptr_t>(a.w);
    asm volatile("" : "+s"(wh_at));
    const auto wh = (const PackedHeader __attribute__((address_space(4))) *)wh_at;
    const uint32_t w_magic = wh->magic, w_bytes = (uint32_t)wh->bytes_used;
    const int64_t w_rows = wh->rows, w_K = wh->K;
    const float w_scale = wh->tensor_scale;
    // plane H ends where the header says (a compact tensor may live in a buffer of exactly that size)
    const bool w_ok = (w_magic == kMagic) & (w_rows == a.w_rows) & (w_K == a.w_K);   // (no branches: one trip for all fields)
    const uint32_t w_used = w_ok ? (uint32_t)__builtin_amdgcn_readfirstlane((int)w_bytes) : 0u;
    const __amdgpu_buffer_rsrc_t hbuf = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(a.w), 0, (int)w_used, kMidRsrc);
    // plane H of the K-tile whose small fields have landed: two consecutive entries, the first block's in the low
    // half where that is FP8, the second block's in the high half (lanes without an FP8 block ask for nothing).  A K-tile
    // past the tensor (the K groups of a tile's last round may outnumber its K-tiles) or past the workgroup's rounds gets zero
    // scales and no FP8 blocks.
    auto load_h = [&](int r, int set, int q) {
        // (masks instead of conditions: no branch)
        const uint32_t inside = (uint32_t)((r * WK + wk - kt_end) >> 31);
        const uint32_t bits = __builtin_amdgcn_ubfe(nm[q], 2u * (uint32_t)g, 2u & inside);
        // the entry before the second block's where that is FP8, else the first block's
        const uint32_t entry = nt[q] + __builtin_amdgcn_ubfe(ns[q], (bits & 2u) << 2, 8u) - (bits >> 1);
        const uint32_t none = (uint32_t)((int)(bits - 1u) >> 31) & 0xFFFFFF00u;
        asm volatile("buffer_load_dwordx4 %0, %1, %2, 0 offen" : "=v"(wu[set][q]) : "v"((a.off_H + entry * 8u) | none), "s"(hbuf));
        ws[set][q] = ns[q] & inside;
        is8[set][q][0] = __builtin_amdgcn_ballot_w64((bits & 1u) != 0u);
        is8[set][q][1] = __builtin_amdgcn_ballot_w64(bits > 1u);
    };

    float4_t acc[MT][NT];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int q = 0; q < NT; ++q) acc[i][q] = float4_t{0.0f, 0.0f, 0.0f, 0.0f};

    // Quarter j of a K-tile: eight values of block 2g + j / 2 of each column group, the operands of matrix instruction j.
    // Every lane takes the 4-bit route; then the lanes whose block is FP8 overwrite the result, with the other lanes switched
    // off around the four conversions (a branch would end the stretch that the matrix instructions are scheduled in, and
    // selecting or adding the two routes' results costs a third more vector instructions).  All exact.
    // (piece 3 q + p: a third of column group q's eight values)
    auto decode = [&](int set, auto quarter_c, half2_t (&b)[NT][4], int piece) {
        constexpr int j = decltype(quarter_c)::value, hb = j / 2;
        const int q = piece / 3, p = piece % 3;
        const uint32_t c4 = wl[set][q][j];   // (the lane's eight 4-bit codes; of an FP8 block, half of its first or second 8 bytes)
        const half2_t sc = __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(ws[set][q], 1.0f, false);
        const half2_t s = half2_t{sc[hb], sc[hb]};
        if (p == 0) {
            b[q][0] = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(c4, 1.0f, 0) * s;
            b[q][1] = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(c4, 1.0f, 1) * s;
            asm volatile("" : "+v"(b[q][0]), "+v"(b[q][1]));
        } else if (p == 1) {
            b[q][2] = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(c4, 1.0f, 2) * s;
            b[q][3] = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(c4, 1.0f, 3) * s;
            asm volatile("" : "+v"(b[q][2]), "+v"(b[q][3]));
        } else {
            const uint32_t x8 = (j & 1) ? wu[set][q][2 * hb] : wl[set][q][2 * hb];
            const uint32_t y8 = (j & 1) ? wu[set][q][2 * hb + 1] : wl[set][q][2 * hb + 1];
            const uint64_t lanes8 = is8[set][q][hb];
            asm volatile("s_mov_b64 exec, %6\n\t"
                         "v_cvt_scalef32_pk_f16_fp8 %0, %4, 1.0\n\t"
                         "v_cvt_scalef32_pk_f16_fp8 %1, %4, 1.0 op_sel:[1,0,0]\n\t"
                         "v_cvt_scalef32_pk_f16_fp8 %2, %5, 1.0\n\t"
                         "v_cvt_scalef32_pk_f16_fp8 %3, %5, 1.0 op_sel:[1,0,0]\n\t"
                         "s_mov_b64 exec, -1"
                         : "+v"(b[q][0]), "+v"(b[q][1]), "+v"(b[q][2]), "+v"(b[q][3])
                         : "v"(x8), "v"(y8), "s"(lanes8));
        }
    };
    // operands of a 16-row group, read kAhead groups ahead of their matrix instructions (a quarter reads the first ones of the
    // next, except across the barrier)
    constexpr int kAhead = MT < 3 ? MT : 3;
    half8_t af[kAhead + 1];
    auto read_a = [&](int stage, int n) {   // n = MT quarter + row group
        af[n % (kAhead + 1)] = *reinterpret_cast<const half8_t *>(&lds[stage * kStage + (n % MT) * 16 * kRowB + (f_lds ^ ((n / MT) << 4))]);
    };
    // One quarter, in the order it is written here (the scheduler is kept from moving anything across a row group): the matrix
    // instructions of a row group, a share of the next quarter's decode, a share of the loads that are due.
    auto quarter = [&](int stage, auto j_c, const half2_t (&now)[NT][4], int set, auto next_c, half2_t (&next)[NT][4], auto loads) {
        constexpr int j = decltype(j_c)::value;
#pragma unroll
        for (int i = 0; i < MT; ++i) {
            const int n = j * MT + i;
            if (n + kAhead < 4 * MT) read_a(stage, n + kAhead);
#pragma unroll
            for (int q = 0; q < NT; ++q)
                acc[i][q] = __builtin_amdgcn_mfma_f32_16x16x32_f16(af[n % (kAhead + 1)], *reinterpret_cast<const half8_t *>(&now[q][0]), acc[i][q], 0, 0, 0);
#pragma unroll
            for (int piece = 0; piece < 3 * NT; ++piece)
                if (piece * MT / (3 * NT) == i) decode(set, next_c, next, piece);
            loads(i);
            __builtin_amdgcn_sched_barrier(0);
        }
        // (the compiler does not know what the conversions' assembly writes: no matrix instruction right behind)
        asm volatile("s_nop 1");
    };
    // LDS operations of this wave are done and visible after the barrier; its loads stay in flight across it
    auto barrier = [&]() {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
    };
    auto set_word = [&](uint32_t from, uint32_t unit) { __builtin_amdgcn_raw_buffer_store_b32(1u, words(from), (int)unit * 4, 0, kCoherent); };
    constexpr std::integral_constant<int, 0> h0{};
    constexpr std::integral_constant<int, 1> h1{};
    constexpr std::integral_constant<int, 2> h2{};
    constexpr std::integral_constant<int, 3> h3{};

    if constexpr (kQuantize) {
        // this wave's values are in memory when only the loads above are outstanding; then the workgroup says so
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(FGMP_MID_PENDING(4 * NT)) : "memory");
        barrier();
        if (tid == 0 && blockIdx.x < a.q.n_own) set_word(0, blockIdx.x);
    }
    wait_meta(std::integral_constant<int, (kQuantize ? 0 : kALoads) + NT>{});
#pragma unroll
    for (int q = 0; q < NT; ++q) load_h(r0, 0, q);
#pragma unroll
    for (int q = 0; q < NT; ++q) load_meta(wbuf_of(r0 + 1), r0 + 1, q);
#pragma unroll
    for (int q = 0; q < NT; ++q) load_l(wbuf_of(r0 + 1), r0 + 1, 1, q);
    uint32_t passed = 0u;
    if constexpr (kQuantize) {
        // Looking is what delays the others most -- hundreds of workgroups that read the same few lines hold up the stores to them --,
        // so those with nothing to quantize sleep first (40 x 64 clocks: about as long as a chunk takes), and all let the stores
        // through (us with no sleep / first sleeps only where there is no share / both: 132 x 496 x 5069 (M, K, N) 9.6 / 8.1 / 7.8, 77 x
        // 2064 x 5003 12.0 / 12.0 / 11.6; bytes instead of words, on fewer lines: 11.3, 13.4).  The last wave looks: it has the
        // least to quantize, so its own loads are the first to be out of the way.
        if (wave == 7) {
            if (blockIdx.x >= a.q.n_units) __builtin_amdgcn_s_sleep(40);
            __builtin_amdgcn_s_sleep(12);
        }
        auto load_words = [&](uint32_t from) { return __builtin_amdgcn_raw_buffer_load_b128(words(from), lane * 16, 0, kCoherent); };
        auto unset = [&](const u32x4_t &d, int e) { return d[e] == 0u && (uint32_t)(lane * 4 + e) < a.q.n_units; };
        auto any_unset = [&](const u32x4_t &d) { return __builtin_amdgcn_ballot_w64(unset(d, 0) || unset(d, 1) || unset(d, 2) || unset(d, 3)) != 0ull; };
        // a unit whose word is not set (there is one), the last ones first, since workgroups start in the order of their numbers, and
        // another one for each workgroup as far as there are several
        auto pick = [&](const u32x4_t &d) {
            uint32_t below = 0u, n = 0u;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const uint64_t m = __builtin_amdgcn_ballot_w64(unset(d, e));
                below = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, below));
                n += (uint32_t)__builtin_popcountll(m);
            }
            uint32_t skip = n - 1u - blockIdx.x % n - below, mine = kMidMaxUnits;   // (unset words of lower lanes: skipped, or, wrapped, past it)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (unset(d, e) && skip-- == 0u) mine = (uint32_t)(lane * 4 + e);
            return (uint32_t)__builtin_amdgcn_readlane((int)mine, __builtin_ctzll(__builtin_amdgcn_ballot_w64(mine != kMidMaxUnits)));
        };
        for (int look = 0;; ++look) {
            if (wave == 7) {
                uint32_t unit = kMidMaxUnits;
                for (;; ++look) {
                    asm volatile("" ::: "memory");   // (loaded again every time)
                    const u32x4_t d = load_words(0);
                    u32x4_t begun = {1u, 1u, 1u, 1u};
                    if (look > 0) begun = load_words(kMidBegun);
                    if (!any_unset(d)) {
                        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // (the words it set itself have landed, too)
                        break;
                    }
                    if (look >= a.q.patience) begun = d;
                    if (__builtin_expect(any_unset(begun), 0)) {
                        unit = pick(begun);
                        break;
                    }
                    __builtin_amdgcn_s_sleep(4);
                }
                if (lane == 0) {
                    arrived = unit;
                    if (unit != kMidMaxUnits) set_word(kMidBegun, unit);
                }
            } else if (wave == 0) {
                // (the word it set has landed before this workgroup counts as past the wait, whoever else has set it, too)
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            }
            barrier();
            const uint32_t unit = (uint32_t)__builtin_amdgcn_readfirstlane((int)arrived);
            if (__builtin_expect(unit >= kMidMaxUnits, 1)) break;
            // its workgroup has not started, for other kernels' sake perhaps: its share is made here, and there again, the same values
            // (all loads have landed; named here, in a loop, the registers would be other ones in front of it, copied from those in flight)
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            const uint32_t c = (uint32_t)wave * a.q.n_units + unit;
            if (c < a.q.n_chunks) {
                MidBlock b;
                mid_load_block(a, c, lane, b);
                mid_quantize_block(a, c, lane, b, lds + wave * 2048);
            }
            __builtin_amdgcn_s_waitcnt(0);
            barrier();
            if (tid == 448) set_word(0, unit);   // (by the wave that looks)
        }
#pragma unroll
        for (int i = 0; i < kALoads; ++i) issue_a(r0, 0, i);
        if (tid == 448) passed = __hip_atomic_fetch_add(&a.q.done[kMidPassed + blockIdx.x % kMidPassedGroups * kMidPassedStep], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    wait_meta(std::integral_constant<int, kQuantize ? 0 : NT>{});   // ... and all that is older: the first round's activations and weights
    // (this workgroup was the last of its group to pass the wait)
    bool last_of_group = false;
    if constexpr (kQuantize)
        last_of_group = wave == 7 && (uint32_t)__builtin_amdgcn_readfirstlane((int)passed) == (a.n_wgs - blockIdx.x % kMidPassedGroups - 1u) / kMidPassedGroups;
    landed(wl[0], wu[0]);
#pragma unroll
    for (int q = 0; q < NT; ++q) load_h(r0 + 1, 1, q);
#pragma unroll
    for (int q = 0; q < NT; ++q) load_meta(wbuf_of(r0 + 2), r0 + 2, q);
    half2_t b0[NT][4], b1[NT][4];
#pragma unroll
    for (int piece = 0; piece < 3 * NT; ++piece) decode(0, h0, b0, piece);
    asm volatile("s_nop 1");
    barrier();

    // Round r multiplies the K-tiles r WK ... from stage r % 2, a quarter at a time, and decodes the next quarter meanwhile (the
    // last one: the first of the next round's).  Its first quarter asks for the activations of round r + 1 -- their stage
    // has been free since the barrier --, its last quarter for the weights of round r + 2, whose registers are free by then.
    auto round = [&](int r, auto st_c) {
        constexpr int st = decltype(st_c)::value;
        auto nothing = [](int) {};
#pragma unroll
        for (int n = 0; n < kAhead; ++n) read_a(st, n);
        __builtin_amdgcn_sched_barrier(0);
        quarter(st, h0, b0, st, h1, b1, [&](int i) {
#pragma unroll
            for (int k = 0; k < kALoads; ++k)
                if (k * MT / kALoads == i) issue_a(r + 1, st ^ 1, k);
        });
        quarter(st, h1, b1, st, h2, b0, nothing);
        quarter(st, h2, b0, st, h3, b1, nothing);
        // the small fields of round r + 2 and, older, planes L and H of round r + 1; the activations may stay in flight
        wait_meta(std::integral_constant<int, kALoads>{});
        landed(wl[st ^ 1], wu[st ^ 1]);
        const __amdgpu_buffer_rsrc_t wbuf = wbuf_of(r + 2);
        quarter(st, h3, b1, st ^ 1, h0, b0, [&](int i) {
#pragma unroll
            for (int q = 0; q < NT; ++q)
                if (q * MT / NT == i) {
                    load_l(wbuf, r + 2, st, q);
                    load_h(r + 2, st, q);
                    load_meta(wbuf, r + 3, q);
                }
        });
        // round r + 1's activations have landed: only the weights' loads above are younger
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(FGMP_MID_PENDING(kWLoads)) : "memory");
        barrier();
    };
    int r = r0;
    for (; r + 2 <= r1; r += 2) {
        round(r, h0);
        round(r + 1, h1);
    }
    if (r < r1) round(r, h0);
    // (loads past the range are still on their way, to registers and to LDS)
    wait_meta(h0);
    landed(wl[0], wu[0]);
    landed(wl[1], wu[1]);
    barrier();

    // (the lane's number is found again, so that nothing of it is kept in registers through the rounds)
    int lane_e = (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
    asm volatile("" : "+v"(lane_e));
    const bool first_lane = wave == 0 && lane_e == 0;
    passed = 0u;
    if constexpr (kQuantize)
        if (last_of_group && lane_e == 0) passed = __hip_atomic_fetch_add(&a.q.done[kMidPassedAll], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);

    uint32_t ticket = 0u;
    if (a.parts > 1 && first_lane) ticket = __hip_atomic_fetch_add(&a.counters[tile << a.counter_shift], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);

    // ---- the K groups' sums: 16-row group i is added up by the waves of K group i % WK, in K order
    float4_t *red = reinterpret_cast<float4_t *>(lds);
#pragma unroll
    for (int i = 0; i < MT; ++i) {
        const int owner = i % WK;
        if (wk != owner) {
            const int from = wk < owner ? wk : wk - 1;
#pragma unroll
            for (int q = 0; q < NT; ++q) red[(((from * MT + i) * WN + wn) * NT + q) * 64 + lane_e] = acc[i][q];
        }
    }
    barrier();
    // (in registers of their own: 16-row groups wk, wk + WK, ...)
    constexpr int kMine = (MT + WK - 1) / WK;
    float4_t own[kMine][NT];
#pragma unroll
    for (int i = 0; i < MT; ++i) {
        if (wk != i % WK) continue;
#pragma unroll
        for (int q = 0; q < NT; ++q) {
            float4_t sum = float4_t{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int k = 0; k < WK; ++k) {
                if (k == i % WK) sum += acc[i][q];
                else sum += red[((((k < i % WK ? k : k - 1) * MT + i) * WN + wn) * NT + q) * 64 + lane_e];
            }
            own[i / WK][q] = sum;
        }
    }

    if constexpr (kQuantize) {
        // every workgroup has passed its wait: all words back to zero
        const uint32_t groups = a.n_wgs < kMidPassedGroups ? a.n_wgs : kMidPassedGroups;
        if (last_of_group && (uint32_t)__builtin_amdgcn_readfirstlane((int)passed) == groups - 1u) {
            const __amdgpu_buffer_rsrc_t dbuf = __builtin_amdgcn_make_buffer_rsrc(a.q.done, 0, (int)(kMidDoneWords * 4u), kMidRsrc);
#pragma unroll
            for (uint32_t at = 0; at < kMidDoneWords * 4u; at += 1024u)   // (beyond the words: outside the buffer)
                __builtin_amdgcn_raw_buffer_store_b128(u32x4_t{0u, 0u, 0u, 0u}, dbuf, (int)(at + lane_e * 16u), 0, kCoherent);
        }
    }
    bool x_ok = true;
    float x_scale;
    if constexpr (kQuantize) {
        x_scale = a.q.S;
    } else {
        x_ok = a.xh->magic == kMagic && a.xh->rows == a.x_rows && a.xh->K == a.x_K;
        x_scale = a.xh->tensor_scale;
    }
    const float ss = w_ok && x_ok ? x_scale * w_scale : 0.0f;
    if (a.parts > 1) {
        // Partials and counters cross XCDs: system-coherent accesses that bypass the per-XCD L2.  The tile's word counts tickets
        // in its low half and parts that are complete in memory in its high half.  All but the workgroup with the last ticket store
        // their sums and leave.  That one keeps its own in registers and waits for the others' -- which are all past their
        // tickets, running, and wait for nothing --, adds in K order (the result does not depend on who it is) and puts the word back
        // to zero.  us with all parts stored before the counting, the last to arrive reading every one back, its own too / now:
        // 512 x 11008 x 4096 (M, K, N, two parts) 57.6 / 55.4, 512 x 4096 x 4096 (two) 29.9 / 28.1, 667 x 2464 x 1248 (five)
        // 23.6 / 22.1, 326 x 9104 x 996 (six) 23.0 / 22.7.  Words on lines of their own: side by side, tickets and looks hold
        // each other up (50 x 10880 x 1291 16.2, with lines 12.9).
        constexpr uint32_t kSlotBytes = (uint32_t)kRows * kCols * 4u;
        const __amdgpu_buffer_rsrc_t pbuf = __builtin_amdgcn_make_buffer_rsrc(a.partial, 0, (int)a.partial_bytes, kMidRsrc);
        const uint32_t tile_at = tile * (uint32_t)a.parts * kSlotBytes + (uint32_t)(wn * NT) * 1024u + (uint32_t)lane_e * 16u;
        if (first_lane) arrived = ticket & 0xFFFFu;
        barrier();
        if (arrived != (uint32_t)a.parts - 1u) {
#pragma unroll
            for (int i = 0; i < kMine; ++i) {
                if (wk + i * WK >= MT) continue;
#pragma unroll
                for (int q = 0; q < NT; ++q)
                    store_coherent16(pbuf, tile_at + part * kSlotBytes + (uint32_t)((wk + i * WK) * WN * NT + q) * 1024u, own[i][q]);
            }
            __builtin_amdgcn_s_waitcnt(0);
            __syncthreads();
            if (first_lane) __hip_atomic_fetch_add(&a.counters[tile << a.counter_shift], 0x10000u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            return;
        }
        if (first_lane) {
            while (__hip_atomic_load(&a.counters[tile << a.counter_shift], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >> 16 != (uint32_t)a.parts - 1u) __builtin_amdgcn_s_sleep(2);
            __hip_atomic_store(&a.counters[tile << a.counter_shift], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        __syncthreads();
        float4_t sum[kMine][NT];
#pragma unroll
        for (int i = 0; i < kMine; ++i)
#pragma unroll
            for (int q = 0; q < NT; ++q) sum[i][q] = float4_t{0.0f, 0.0f, 0.0f, 0.0f};
        for (int c = 0; c < a.parts; c += 2) {   // two parts' loads in flight (its own, or a part past the last one: beyond the buffer, zeros)
            float4_t p[2][kMine][NT];
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int i = 0; i < kMine; ++i)
#pragma unroll
                    for (int q = 0; q < NT; ++q) {
                        const int row_group = wk + i * WK;
                        const bool there = c + u < a.parts && c + u != (int)part && row_group < MT;
                        p[u][i][q] = load_coherent16(pbuf, there ? tile_at + (uint32_t)(c + u) * kSlotBytes + (uint32_t)(row_group * WN * NT + q) * 1024u : 0xFFFFFF00u);
                    }
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int i = 0; i < kMine; ++i)
#pragma unroll
                    for (int q = 0; q < NT; ++q) sum[i][q] += c + u == (int)part ? own[i][q] : p[u][i][q];
        }
#pragma unroll
        for (int i = 0; i < kMine; ++i)
#pragma unroll
            for (int q = 0; q < NT; ++q) own[i][q] = sum[i][q];
    }
    // own[i][q][e] = Y[m0 + 16 (wk + i WK) + 4 g + e][n0 + 16 (NT wn + q) + nl]
#pragma unroll
    for (int i = 0; i < kMine; ++i) {
        if (wk + i * WK >= MT) continue;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int m = m0 + 16 * (wk + i * WK) + 4 * (lane_e >> 4) + e;
            if (m < a.M) {
                float *row = a.Y + (int64_t)m * a.ldy;
#pragma unroll
                for (int q = 0; q < NT; ++q) {
                    const int n = n0 + (wn * NT + q) * 16 + (lane_e & 15);
                    if (n < a.N) row[n] = own[i][q][e] * ss;
                }
            }
        }
    }
}

// ---- host side ----

// column groups per wave that fit the 256 registers of two waves per SIMD (accumulators 4 MT NT, weights 38 NT)
constexpr int mid_most_nt(int mt) { return mt <= 4 ? 4 : 3; }

// Which of the 16 MT x 16 NT WN tiles, and how many workgroups share one: the cheapest by a model of the launch, in
// cycles of a compute unit.  A round costs what its matrix instructions, its vector instructions (two waves to a SIMD) or
// its LDS accesses take, whichever is most -- 1.4 times that is measured --, a workgroup 15000 cycles before its first and
// after its last round, partial sums that meet in memory 6000 and 2000 per part.  A launch took 1.2 times the model
// when it was made (a fused step 3 us more, with a launch of the quantizer in front; both have become faster since, all plans alike): 4096 x 12288, 64 rows, 4 x 2 tiles on 192 workgroups 16 us by the model, 19.6 measured (4 x 3 in
// two parts 21.7, 4 x 4 in two 24.1); 11008 x 4096, 512 rows, 8 x 2 in two parts 52 / 57 (8 x 3 in two 68, 4 x 4 63);
// 4096 x 22016, 200 rows, 7 x 3 38 / 45 (5 x 3 66, 7 x 2 59).
MidPlan gemm_mid_plan(int64_t M, int64_t N, int64_t K, size_t most_bytes)
{
    MidPlan best{};
    best.cycles = INFINITY;
    const int64_t n_kt = (K + kTileK - 1) / kTileK, least_m = (M + 127) / 128;
    for (int64_t tiles_m = least_m; tiles_m <= least_m + 2; ++tiles_m) {
        const int mt = (int)(((M + tiles_m - 1) / tiles_m + 15) / 16);
        for (int nt = 2; nt <= mid_most_nt(mt); ++nt) {
            MidPlan p;
            p.mt = mt;
            p.nt = nt;
            p.wn = mt <= 4 ? 2 : 4;
            p.wk = 8 / p.wn;
            p.tiles_m = (M + 16 * mt - 1) / (16 * mt);
            p.tiles_n = (N + p.cols() - 1) / p.cols();
            p.rounds = (n_kt + p.wk - 1) / p.wk;
            const double matrix = 128.0 * mt * nt, vector = 8.0 * (70.0 * nt + 30.0), lds = 256.0 * mt + 32.0 * mt * p.wk;
            const double per_round = std::max(matrix, std::max(vector, lds)) * 1.4 + 300.0;
            for (int64_t parts = 1; parts <= std::min<int64_t>(16, p.rounds); ++parts) {
                p.parts = parts;
                const int64_t waves = (p.tiles() * parts + 255) / 256;
                p.cycles = (double)waves * (15000.0 + (double)((p.rounds + parts - 1) / parts) * per_round) +
                           (parts > 1 ? 6000.0 + 2000.0 * (double)parts : 0.0);
                if (p.cycles < best.cycles && p.bytes(K) <= most_bytes) best = p;
            }
        }
    }
    return best;
}

// A fused step on this kernel in microseconds, for more than 32 rows: quantizing the activations and storing the results (by their
// numbers), what a workgroup pays around its rounds, its rounds -- the slowest of matrix, vector and LDS work and half of all
// three --, and partial sums that meet in memory.  Fitted, with a quantizer launch in front of every one, to 11000 steps of 1076 products (33 to 4096 rows, K and N of the
// Llama-2-7B linears and 256 .. 11008 by 256 .. 22016, up to nine splits of each, weights in the Infinity Cache): 9% rms.
double gemm_mid_micros(const MidPlan &p, int64_t M, int64_t N, int64_t K)
{
    const int64_t wgs = p.tiles() * p.parts;
    const double matrix = 0.042 * p.mt * p.nt, vector = 0.236 * p.nt, lds = 0.031 * p.mt * p.wk;
    const double per_round = std::max(matrix, std::max(vector, lds)) + 0.51 * (matrix + vector + lds);
    const double meet = p.parts > 1 ? 3.8 + 0.028 * p.mt * p.nt * p.wn * (double)(p.parts - 1) * (double)std::min<int64_t>(wgs, 256) / 256.0 : 0.0;
    return 5.1 + (double)((wgs + 255) / 256) * (3.8 + (double)((p.rounds + p.parts - 1) / p.parts) * per_round) + meet +
           (0.92e-6 * (double)K + 1.52e-6 * (double)N) * (double)M;
}

// The same for 20 to 32 rows with the weights coming from HBM, as those of a model's layers do: 2 to 4 us more than out of the
// Infinity Cache, for the dependent loads before a workgroup's first round.  Fitted to 552 measured steps, a quantizer launch in front
// of every one: 2% rms, 8% at most; steps that quantize in their launch take 1 to 3 us less.
double gemm_mid_few_rows_micros(const MidPlan &p, int64_t N, int64_t K)
{
    const int64_t waves = (p.tiles() * p.parts + 255) / 256, rounds = (p.rounds + p.parts - 1) / p.parts;
    return 9.4 + (0.836 + 0.332 * (p.nt - 2)) * (double)(waves * rounds) + (p.parts > 1 ? 0.5 * (double)p.parts : 0.0) +
           0.073e-6 * (double)N * (double)K;
}

bool gemm_mid_applies(const MidPlan &p, int64_t N, int64_t K)
{
    constexpr uint64_t kLimit = 0xFFFFFF00ull;   // 32-bit buffer offsets
    return p.tiles_m > 0 && make_layout(N, K).total_bytes < kLimit && p.partial_bytes() < 0x7FFFFF00ull && p.tiles() * p.parts < 65536 &&
           p.rounds * (p.parts + 1) < 65536 && p.tiles() <= (int64_t)(kWsCtrlRegion / 4) && align_up(K, kTileK) * 8 < 0x7FFFFFFF;
}

template <int MT, int NT> static void launch_mid(const MidArgs &a, hipStream_t st)
{
    constexpr int WN = MT <= 4 ? 2 : 4;
    if (a.q.X != nullptr) hipLaunchKernelGGL((gemm_mid_kernel<MT, NT, WN, 8 / WN, true>), dim3(a.n_wgs), dim3(kMidThreads), 0, st, a);
    else hipLaunchKernelGGL((gemm_mid_kernel<MT, NT, WN, 8 / WN, false>), dim3(a.n_wgs), dim3(kMidThreads), 0, st, a);
}

template <int MT> static void launch_mid_nt(int nt, const MidArgs &a, hipStream_t st)
{
    if (nt == 2) launch_mid<MT, 2>(a, st);
    if constexpr (mid_most_nt(MT) >= 3)
        if (nt == 3) launch_mid<MT, 3>(a, st);
    if constexpr (mid_most_nt(MT) >= 4)
        if (nt == 4) launch_mid<MT, 4>(a, st);
}

// The words that say whose share of the activations is done lie at the end of the control region, behind the tiles' counters.
constexpr size_t kMidDoneAt = kWsCtrlRegion / 4 - kMidDoneWords;

// Workgroups that hold a share of the quantizing: all, where the chip holds two such launches; else the first ones, a chunk for every
// second wave (one per SIMD), as far as there are so many workgroups.  These are the first to start, so that a workgroup that finds
// shares missing has, as a rule, their holders running beside it: dealt out over all workgroups, a launch that holds part of the
// chip, another stream's the rest, waits for workgroups that have not started.  us per round of one product a stream, on one | two |
// four streams (a quantizer launch in front, all workgroups hold shares and make missing ones after eight looks, now): 64 x 4096 x
// 12288 (M, K, N) 18.8 17.4 17.5 | 29.2 36.8 27.7 | 49.2 80.1 50.6, 77 x 2064 x 5003 12.8 12.2 12.0 | 22.3 30.5 18.9 | 34.1 72.6 31.6, 200 x
// 4096 x 22016 45.2 42.9 43.2 | 83.4 86.3 81.3 | 169 206 176.  On one stream alone four chunks
// to a workgroup cost up to 2.5% (one / four: 16.78 / 16.92, 11.77 / 11.91, 42.5 / 42.5).  Where shares take more than half of all waves, overlapping launches
// still pay more than a quantizer launch (512 x 4096 x 4096 30.6 28.8 29.1 | 49.6 60.4 57.9 | 92 136 110, 207 x 6496 x 720 16.0 14.6 14.6 | 25.1
// 32.8 33.3 | 41.2 91.5 63.9).  Eight chunks a workgroup, half as many: two streams up to 15% faster, one 1 to 10% slower.
static uint32_t mid_units(const MidPlan &p, uint32_t n_chunks)
{
    const uint32_t wgs = (uint32_t)(p.tiles() * p.parts);
    return std::min(wgs, 2 * wgs <= kMidMaxUnits ? n_chunks : (n_chunks + 3) / 4);
}

bool gemm_mid_quantizes(const MidPlan &p, int64_t M, int64_t N, int64_t K, int64_t row_bytes)
{
    constexpr int64_t kLimit = 0x7FFFFF00;   // 32-bit buffer offsets
    const int64_t row_blocks = (K + kTileK - 1) / kTileK * kTileBlocks, blocks = M * row_blocks;
    if (!gemm_mid_applies(p, N, K) || p.tiles() > (int64_t)kMidDoneAt || (blocks + 64) * row_blocks >= (int64_t)1 << 32 ||
        blocks * 32 >= kLimit || row_bytes <= 0 || row_bytes >= kLimit / M)
        return false;
    const int64_t wgs = p.tiles() * p.parts;
    return wgs <= kMidMaxUnits && blocks <= wgs * kMidThreads;
}

uint32_t gemm_mid_shares(const MidPlan &p, int64_t M, int64_t N, int64_t K, int64_t row_bytes)
{
    return gemm_mid_quantizes(p, M, N, K, row_bytes) ? mid_units(p, (uint32_t)((M * ((K + kTileK - 1) / kTileK * kTileBlocks) + 63) / 64)) : 0u;
}

fgmp_status_t gemm_mid(const MidPlan &p, const MidInput &in, _Float16 *x16, int64_t ld16, const void *w, int64_t M, int64_t N, int64_t K, float *Y,
                       int64_t ldy, void *ctrl, void *scratch, hipStream_t st)
{
    if (!gemm_mid_applies(p, N, K)) return FGMP_ERR_UNSUPPORTED;
    const PackedLayout lw = make_layout(N, K);
    MidArgs a{};
    const PackedHeader *const xh = in.packed;
    if (in.X != nullptr) {
        const int64_t row_bytes = in.ldx * (in.f32 ? 4 : 2);
        if (!gemm_mid_quantizes(p, M, N, K, row_bytes)) return FGMP_ERR_UNSUPPORTED;
        MidQuant &q = a.q;
        q.X = in.X; q.fisher = in.fisher; q.T = in.T; q.S = in.S; q.f32 = in.f32; q.delta = in.delta;
        q.x_bytes = (uint32_t)((M - 1) * row_bytes + K * (in.f32 ? 4 : 2));
        q.row_bytes = (uint32_t)row_bytes;
        q.nb = (uint32_t)(K / kBlock);
        q.row_blocks = (uint32_t)(lw.n_kt * kTileBlocks);
        q.row_mul = (uint32_t)(0x100000000ull / q.row_blocks) + 1u;
        q.n_chunks = (uint32_t)((M * q.row_blocks + 63) / 64);
        q.n_own = q.n_units = mid_units(p, q.n_chunks);
        q.done = static_cast<uint32_t *>(ctrl) + kMidDoneAt;
        q.patience = kMidPatience;
#ifdef FGMP_MEASUREMENT_HOOKS
        if (const char *e = getenv("FGMP_MID_PATIENCE")) q.patience = atoi(e);   // (0: every workgroup makes what is missing at its first look)
        // (the last ones make nothing and say nothing, as if they had not started)
        if (const char *e = getenv("FGMP_MID_ABSENT")) q.n_own -= std::min(q.n_units, (uint32_t)atoi(e));
#endif
    }
    a.w = w; a.xh = xh; a.x16 = x16; a.Y = Y; a.ldy = ldy;
    a.partial = static_cast<float *>(scratch); a.partial_bytes = (uint32_t)p.partial_bytes();
    a.counters = static_cast<uint32_t *>(ctrl);
    a.w_rows = N; a.w_K = K; a.x_rows = M; a.x_K = K;
    for (a.counter_shift = 5; a.counter_shift > 0 && p.tiles() << a.counter_shift > (int64_t)kMidDoneAt; --a.counter_shift) {}
    a.off_L = (uint32_t)lw.off_L; a.off_S = (uint32_t)lw.off_S; a.off_M = (uint32_t)lw.off_M;
    a.off_T = (uint32_t)lw.off_T; a.off_H = (uint32_t)lw.off_H;
    a.ld_bytes = (uint32_t)(ld16 * 2);
    a.M = (int)M; a.N = (int)N; a.n_kt = (int)lw.n_kt; a.n_rt = (int)lw.n_rt;
    a.rounds = (int)p.rounds; a.parts = (int)p.parts;
    a.by_tiles_n = MidDiv::by((uint32_t)p.tiles_n); a.by_parts = MidDiv::by((uint32_t)p.parts);
    a.n_wgs = (uint32_t)(p.tiles() * p.parts);
#ifdef FGMP_MEASUREMENT_HOOKS
    record_gemm_kernel_event(false, st);
#endif
    switch (p.mt) {
    case 1: launch_mid_nt<1>(p.nt, a, st); break;
    case 2: launch_mid_nt<2>(p.nt, a, st); break;
    case 3: launch_mid_nt<3>(p.nt, a, st); break;
    case 4: launch_mid_nt<4>(p.nt, a, st); break;
    case 5: launch_mid_nt<5>(p.nt, a, st); break;
    case 6: launch_mid_nt<6>(p.nt, a, st); break;
    case 7: launch_mid_nt<7>(p.nt, a, st); break;
    default: launch_mid_nt<8>(p.nt, a, st); break;
    }
#ifdef FGMP_MEASUREMENT_HOOKS
    record_gemm_kernel_event(true, st);
#endif
    return hipGetLastError() == hipSuccess ? FGMP_OK : FGMP_ERR_HIP;
}

}  // namespace fgmp
