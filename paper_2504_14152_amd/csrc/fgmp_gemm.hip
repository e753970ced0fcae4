// Block-mixed-precision GEMM Y = S_x S_w (X^ W^^T) over packed FGMP operands
// (Sec. 4.1).  Each 16-element block is decoded according to its metadata
// bit -- FP8 value, or E2M1 value times its E4M3 block scale -- into FP16,
// where both kinds of operand are exactly representable (at most 6
// significant bits, magnitudes 2^-10 .. 2688), multiplied on the matrix
// cores and accumulated in FP32, which is what the paper's four dot-product
// units followed by the FP32 partial-sum adder compute.
//
// Prefill path (M > 32): the activations are expanded to FP16 in the caller's
// workspace by a decode pass (small), and the 256x256x64-tiled MFMA kernel of
// fgmp_gemm_mixed.hip decodes the packed weights itself.  This file holds the
// decode pass, the dispatch, and the alternative two-pass path in which both
// operands are expanded first and a plain FP16 kernel multiplies them.
#include <stdlib.h>

#include <algorithm>

#include "fgmp_elementwise.hpp"
#include "fgmp_gemm_common.hpp"

namespace fgmp {

// One wave per 8 x 128 tile of the zero-padded FP16 matrix out[8 n_rt_pad][ld].
// One launch serves up to two tensors (both GEMM operands) and can clear a
// small array of counters on the side.
__global__ __launch_bounds__(256) void decode_f16_kernel(DecodeJob ja, DecodeJob jb, uint32_t *zero, int64_t zero_n)
{
    const int lane = threadIdx.x & 63;
    int64_t id = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    {
        const int64_t gid = (int64_t)blockIdx.x * 256 + threadIdx.x;
        if (gid < zero_n) zero[gid] = 0u;
    }
    const bool second = id >= ja.waves;
    if (second) id -= ja.waves;
    const DecodeJob &j = second ? jb : ja;
    if (id >= j.waves) return;
    const PackedLayout &l = j.l;
    const int64_t rt = id / l.n_kt, kt = id % l.n_kt;
    half2_t vals[8];
    // an operand whose header does not describe the shape this launch assumes decodes to zeros
    const bool header_ok = j.v.hdr->magic == kMagic && j.v.hdr->rows == l.rows && j.v.hdr->K == l.K;
    if (rt < l.n_rt && header_ok) {
        decode_slot(j.v, rt * l.n_kt + kt, lane, vals);
    } else {
#pragma unroll
        for (int i = 0; i < 8; ++i) vals[i] = half2_t{(_Float16)0.0f, (_Float16)0.0f};
    }
    _Float16 *dst = j.out + (rt * kTileRows + (lane >> 3)) * j.ld + kt * kTileK + (lane & 7) * kBlock;
    uint4 *d4 = reinterpret_cast<uint4 *>(dst);
    const uint32_t *w = reinterpret_cast<const uint32_t *>(vals);
    d4[0] = make_uint4(w[0], w[1], w[2], w[3]);
    d4[1] = make_uint4(w[4], w[5], w[6], w[7]);
}

DecodeJob make_decode_job(const PackedView &v, const PackedLayout &l, _Float16 *out, int64_t ld, int64_t n_rt_pad)
{
    DecodeJob j;
    j.v = v;
    j.l = l;
    j.out = out;
    j.ld = ld;
    j.waves = n_rt_pad * l.n_kt;
    return j;
}

fgmp_status_t launch_decode_f16(const DecodeJob &a, const DecodeJob *b, uint32_t *zero, int64_t zero_n,
                                hipStream_t st)
{
    DecodeJob none = a;
    none.waves = 0;
    const DecodeJob &jb = b ? *b : none;
    int64_t blocks = (a.waves + jb.waves + 3) / 4;
    const int64_t zblocks = (zero_n + 255) / 256;
    if (blocks < zblocks) blocks = zblocks;
    if (blocks > 0x7FFFFFFF) return FGMP_ERR_UNSUPPORTED;
    hipLaunchKernelGGL(decode_f16_kernel, dim3((unsigned)blocks), dim3(256), 0, st, a, jb, zero, zero_n);
    return FGMP_OK;
}

// ---------------------------------------------------------------------------
// dense FP16 x FP16 -> FP32 MFMA kernel, A [Mp][ld], B [Np][ld], both K-major
// ---------------------------------------------------------------------------

// kWM x kWN waves per workgroup; each wave owns a (256 / kWM) x (256 / kWN)
// piece of the tile as TM x TN MFMA tiles of 32 x 32.
template <int kWM, int kWN>
__global__ __launch_bounds__(kWM *kWN * 64, 1) void gemm_f16_kernel(const _Float16 *__restrict__ A,
                                                                     const _Float16 *__restrict__ B, int64_t ld,
                                                                     int nk, float *__restrict__ Y, int64_t ldy,
                                                                     int64_t M, int64_t N, int64_t n_tm,
                                                                     int64_t n_tn, const PackedHeader *ha,
                                                                     const PackedHeader *hb)
{
    constexpr int kWaves = kWM * kWN;
    constexpr int TM = kBM / (32 * kWM), TN = kBN / (32 * kWN);
    constexpr int kLoads = 32 / kWaves;          // 1 KB wave-loads per operand per wave per K-step
    __shared__ __attribute__((aligned(1024))) char lds[2][2][kTileBytes];   // [stage][operand]
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / kWN, wn = wave % kWN;
    int64_t tm, tn;
    tile_coords(blockIdx.x, n_tm, n_tn, tm, tn);

    // direct global -> LDS: wave-load j (j = kWaves i + wave) fills tile rows 8 j .. 8 j + 7;
    // lane (lr = lane / 8, c = lane % 8) fetches global chunk c ^ swizzle(row) of its row;
    // rows of successive i differ by a multiple of 16, which leaves the swizzle unchanged
    const int lr = lane >> 3, lc = (lane & 7) ^ (((wave * 8 + lr) >> 1) & 7);
    const char *ga = reinterpret_cast<const char *>(A + (tm * kBM + wave * 8 + lr) * ld) + lc * 16;
    const char *gb = reinterpret_cast<const char *>(B + (tn * kBN + wave * 8 + lr) * ld) + lc * 16;
    const int64_t row_step = kWaves * 8 * ld * 2;   // bytes between wave-loads i and i + 1

    auto issue_loads = [&](int kt, int stage) {
#pragma unroll
        for (int i = 0; i < kLoads; ++i) {
            __builtin_amdgcn_global_load_lds((global_void_t *)(ga + i * row_step + (int64_t)kt * kRowBytes),
                                             (lds_void_t *)&lds[stage][0][(kWaves * i + wave) * 1024], 16, 0, 0);
            __builtin_amdgcn_global_load_lds((global_void_t *)(gb + i * row_step + (int64_t)kt * kRowBytes),
                                             (lds_void_t *)&lds[stage][1][(kWaves * i + wave) * 1024], 16, 0, 0);
        }
    };

    float16_t acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;

    // operand fragment of lane: row (lane & 31) of a 32-row group, K chunk 2 kk + (lane >> 5)
    int frag_off[4];
#pragma unroll
    for (int kk = 0; kk < 4; ++kk)
        frag_off[kk] = (lane & 31) * kRowBytes + (((2 * kk + (lane >> 5)) ^ ((lane >> 1) & 7)) << 4);

    auto read_frags = [&](int stage, int kk, half8_t (&a)[TM], half8_t (&b)[TN]) {
        const char *la = &lds[stage][0][wm * (TM * 32) * kRowBytes], *lb = &lds[stage][1][wn * (TN * 32) * kRowBytes];
#pragma unroll
        for (int i = 0; i < TM; ++i) a[i] = *reinterpret_cast<const half8_t *>(la + i * 32 * kRowBytes + frag_off[kk]);
#pragma unroll
        for (int j = 0; j < TN; ++j) b[j] = *reinterpret_cast<const half8_t *>(lb + j * 32 * kRowBytes + frag_off[kk]);
    };
    auto mfma_block = [&](const half8_t (&a)[TM], const half8_t (&b)[TN]) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[i], b[j], acc[i][j], 0, 0, 0);
    };
    constexpr int kReads = TM + TN, kMfma = TM * TN;

    // Software pipeline.  LDS holds two K-steps; the fragments of the next
    // 16-wide K slice are read while the MFMAs of the current one run.
    // Before the last slice of a K-step every wave has finished reading the
    // current stage, so that is where the barrier sits: after it the other
    // stage (filled by loads issued one K-step earlier) is visible, and the
    // stage just consumed is refilled with the K-step after next.
    half8_t fa[2][TM], fb[2][TN];
    issue_loads(0, 0);
    issue_loads(nk > 1 ? 1 : 0, 1);
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    read_frags(0, 0, fa[0], fb[0]);
    __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0): enter the loop with an empty LDS queue (see its end)
    for (int kt = 0; kt < nk; ++kt) {
        const int st = kt & 1;
        read_frags(st, 1, fa[1], fb[1]);
        mfma_block(fa[0], fb[0]);
        order_phase<kReads, kMfma, 0>();
        read_frags(st, 2, fa[0], fb[0]);
        mfma_block(fa[1], fb[1]);
        order_phase<kReads, kMfma, 0>();
        read_frags(st, 3, fa[1], fb[1]);
        mfma_block(fa[0], fb[0]);
        order_phase<kReads, kMfma, 0>();
        __builtin_amdgcn_s_waitcnt(0);   // own LDS reads done, own global->LDS loads landed
        __syncthreads();
        // the last two iterations reload the final K-step, which nobody reads again
        issue_loads(kt + 2 < nk ? kt + 2 : nk - 1, st);
        read_frags(st ^ 1, 0, fa[0], fb[0]);
        mfma_block(fa[1], fb[1]);
        order_phase<kReads, kMfma, kLoads>();
        // the fragments for the next iteration were requested a phase ago; waiting for them here (LDS
        // counter only) costs nothing and lets the next iteration start with a known-empty LDS queue
        __builtin_amdgcn_s_waitcnt(0xC07F);
    }
    __builtin_amdgcn_s_waitcnt(0);

    // per-tensor scales are applied once, after accumulation
    const float ss = ha->tensor_scale * hb->tensor_scale;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int64_t col = tn * kBN + wn * (TN * 32) + j * 32 + (lane & 31);
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int64_t row = tm * kBM + wm * (TM * 32) + i * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
                if (row < M && col < N) Y[row * ldy + col] = acc[i][j][r] * ss;
            }
        }
}

#ifndef FGMP_GEMM_WM
#define FGMP_GEMM_WM 2
#define FGMP_GEMM_WN 4
#endif

static inline int64_t round_up(int64_t v, int64_t a) { return (v + a - 1) / a * a; }

struct GemmWorkspace {
    int64_t ld, Mp, Np;
    size_t off_a, off_b, off_split, total;   // off_split: partial tiles and counters of a split last round
};

static GemmWorkspace gemm_ws_layout(int64_t M, int64_t N, int64_t K)
{
    GemmWorkspace w;
    w.ld = round_up(K, kTileK);
    w.Mp = round_up(M, kBM);
    w.Np = round_up(N, kBN);
    w.off_a = 0;
    w.off_b = (size_t)align_up((uint64_t)w.Mp * w.ld * 2, 256);
    w.off_split = w.off_b + (size_t)align_up((uint64_t)w.Np * w.ld * 2, 256);
    w.total = w.off_split + gemm_mixed_split_bytes((w.Mp / kBM) * (w.Np / kBN));
    return w;
}

// (the fused call on the prefill kernel: header, FP16 activations, then what a split last round needs)
static size_t fused_prefill_split(const GemmWorkspace &w) { return (size_t)align_up((uint64_t)kHeaderBytes + w.off_b, 256); }

// The prefill kernel decodes the weights inside the MFMA kernel.  Builds with FGMP_MEASUREMENT_HOOKS
// (never the shipped library) can select the two-pass path instead -- both operands expanded to FP16
// in the workspace, then a plain FP16 kernel -- with FGMP_PREFILL_KERNEL=dense in the environment.
static bool prefill_decodes_in_kernel()
{
#ifdef FGMP_MEASUREMENT_HOOKS
    static const bool in_kernel = [] {
        const char *e = getenv("FGMP_PREFILL_KERNEL");
        return !(e && e[0] == 'd');
    }();
    return in_kernel;
#else
    return true;
#endif
}

// The MFMA kernel that decodes the weights itself addresses them with 32-bit buffer offsets; larger
// weight tensors take the two-pass path.
static bool mixed_kernel_applies(int64_t N, int64_t K)
{
    return prefill_decodes_in_kernel() && make_layout(N, K).total_bytes < 0xFFFFFF00ull;
}

// FP16 activations of a decode-shape call: gemm_skinny_x16_rows(M) rows
static size_t skinny_x16_bytes(int64_t M, int64_t K)
{
    return (size_t)align_up((uint64_t)gemm_skinny_x16_rows(M) * round_up(K, kTileK) * 2, 256);
}

// Products of 33 to 4096 rows take the kernel for mid-size products (fgmp_gemm_mid.hip) where the two kernels' estimates say so:
// where 256 x 256 tiles leave the chip part empty, or K is too short for what a tile pays around its K loop.  Calls that quantize
// their results have to quantize exactly what the plain call returns, so both take the same kernel, though only the prefill
// kernel quantizes in its epilogue: staging FP32 results for the quantizer costs what that epilogue costs.  Microseconds per
// call, this kernel / the prefill kernel, with FP32, packed and gated packed results.  On this kernel: 4096 x 4096 (K x N) 844 rows
// 38 / 62, 688 x 640 617 rows 14 / 32, 17 / 41, 18 / 43, 656 x 320 42 rows 11 / 20, 13 / 25, 14 / 29, 3136 x 512 1978 rows 29 / 50,
// 31 / 57, 32 / 59.  On the prefill kernel: 11008 x 4096 1650 rows 198 / 160, 200 / 166, 204 / 168, 272 x 6080 2841 rows 47 / 47, 62 /
// 60, 65 / 63, 3440 x 18112 2025 rows 277 / 243, 288 / 261, 291 / 268.  Of 1014 products measured with both (33 to 4096 rows) 226
// changed kernel, none for one that is more than 2% slower; of 631 others 155, 1.46 times as fast on average with
// either kind of result.  Above 1024 rows, where a wrong choice costs more, the estimate has to win by 15%.  The line holds for
// weights from HBM too, which cost both kernels 1.8 us on average: of 600 products next to it that take this kernel, none is more
// than 2.2% slower than on the other one, either way; of 255 drawn over the whole range, six take the prefill kernel though this
// one is 4 to 18% faster (1041 rows, 4096 x 14115 157 / 132), and none the other way round.
//
// Up to 32 rows the one-launch step (fgmp_gemm_stream.hip) shares K among as many workgroups as keep a part's rows in LDS and runs
// through its row groups in rounds; with two rounds or more the parts meet that often, and this kernel is taken where the
// estimates of both, for weights that come from HBM, are in its favour.  Microseconds per fused step, one launch / this kernel,
// weights from HBM | from the Infinity Cache: 4096 x 22016 (K x N) 20 rows (3 rounds) 28.1 / 25.3 | 27.5 / 21.5, 32 rows (2)
// 25.1 / 25.2 | 24.9 / 22.2; 8192 x 8192 20 rows (1) 19.8 / 22.0 | 20.0 / 19.6, 24 rows (7) 38.7 / 22.2 | 38 / 20; 11008 x 4096 24
// rows (2) 20.4 / 19.9 | 20.8 / 17.9, 32 rows (1) 18.3 / 20.2 | 18.4 / 18.0; 5120 x 11008 20 rows (1) 17.3 / 21.9 | 17.5 / 18.7, 28
// rows (5) 30.1 / 21.9; 8192 x 4096 32 rows (2) 18.9 / 17.2 | 19.2 / 16.0; 6144 x 22016 20 rows (2) 30.9 / 34.3 | 30.7 / 27.0; 16384 x
// 2048 32 rows (2) 24.0 / 18.3 | 24.4 / 17.0.  Over 420 such steps none is more than 1.5% slower than in one launch.  (From
// N K^2 = 2^38 on, and only where it needs no more workspace than the step it replaces.)
//
// Steps that the one-launch step does not serve -- K in more than 16 parts, the Eq. 8 score; on the older kernel they take two
// launches -- are faster on this kernel throughout: 32768 x 256 32 rows 26.1 / 20.8, 11008 x 4096 with the Eq. 8 score 21.3 / 17.6.
//
// All these figures and both estimates are of this kernel behind a launch of the quantizer.  Where it quantizes the activations itself it is 1
// to 3 us faster than they say (gemm_mid_quantizes), so that next to the lines some products stay on the other kernel that would now be faster
// here; none takes this one for that.
//
// An odd number of row-tiles is nothing special to either kernel.  Of 1348 such products from N K^2 = 2^38 on, weights from HBM, the
// estimates leave 511 to the one launch, which all took two: 6352 x 8788 22 rows (one launch / this kernel) 17.2 / 24.2, 6960 x 6195
// 24 rows 17.1 / 18.9, 0.90 times as long on average, eleven of them 3 to 7% longer (8064 x 18835 30 rows 37.6 / 35.3).  Out of the
// Infinity Cache, which these estimates are not made for, 1.06 times (10864 x 12228 24 rows 29.9 / 26.1).
constexpr int64_t kMidMinRows = 20, kMidMaxRows = 4096;

static size_t decode_bytes(int64_t M, int64_t N, int64_t K)
{
    return gemm_skinny_applies(M, N, K) ? skinny_x16_bytes(M, K) + gemm_skinny_workspace_bytes(M, N, K) : 0;
}

// (what a decode step is told to bring: with an odd number of row-tiles, what the two launches use, which once served it)
static bool even_row_tiles(int64_t N) { return (N + kTileRows - 1) / kTileRows % 2 == 0; }

GemmRoute gemm_route(int64_t M, int64_t N, int64_t K)
{
    GemmRoute r{};
    if (!kUseHwCvt || !prefill_decodes_in_kernel() || M < kMidMinRows || M > kMidMaxRows || N <= 0 || K <= 0) return r;
    if (M <= 32 && (double)N * (double)K * (double)K < 0x1p38) return r;
    const GemmWorkspace w = gemm_ws_layout(M, N, K);
    const size_t fused = fused_prefill_split(w) + (w.total - w.off_split);   // what a fused call uses on the prefill kernel
    // 33 to 1024 rows: K in as many parts as the sums have room for where the prefill kernel has its operands and sums, or in the
    // static scratch array (a call asks for no more than on the prefill kernel, and the array serves what it serves there).  Left to
    // the prefill kernel where the best plan has no room, us there / here: 695 x 7808 x 394 (M, K, N) 69.6 / 25.5, 497 x 9744 x 385 76.2 /
    // 29.2 (four parts; 25.5 with the eight that need more), 647 x 7040 x 11796 143 / 120.
    const size_t room = std::min(w.total, std::max(fused, (size_t)FGMP_STATIC_SCRATCH_BYTES - kWsCtrlRegion));
    r.plan = gemm_mid_plan(M, N, K, M > 32 && M <= 1024 ? room : SIZE_MAX);
    if (!gemm_mid_applies(r.plan, N, K)) return r;
    if (M <= 32) {
        const bool stream = gemm_stream_applies(M, N, K);
        r.mid_if_not_one_launch = r.plan.bytes(K) <= (stream && even_row_tiles(N) ? gemm_stream_scratch_bytes(M, N, K) : decode_bytes(M, N, K));
        int rounds = 0;
        r.mid = r.mid_if_not_one_launch && (!stream || (gemm_mid_few_rows_micros(r.plan, N, K) <= gemm_stream_micros(M, N, K, &rounds) && rounds > 1));
    } else {
        const double margin = M > 1024 ? 1.15 : 1.0;
        r.mid = margin * gemm_mid_micros(r.plan, M, N, K) <= gemm_mixed_micros(M, N, K) && (M <= 1024 || r.plan.bytes(K) <= fused);
    }
    return r;
}

// (above 1024 rows a call asks for what the prefill kernel needs, whichever kernel it takes)
static bool mid_asks_less(int64_t M, const GemmRoute &route) { return M > 32 && M <= 1024 && route.mid; }

// what a product of packed operands uses behind the control region
static size_t gemm_only_need(int64_t M, int64_t N, int64_t K, const GemmRoute &route)
{
    if (mid_asks_less(M, route)) return route.plan.bytes(K);
    const size_t other = gemm_skinny_applies(M, N, K) ? decode_bytes(M, N, K) : gemm_ws_layout(M, N, K).total;
    return std::max(other, gemm_stream_scratch_bytes(M, N, K));
}

// what a call must be given
size_t gemm_workspace_need(int64_t M, int64_t N, int64_t K, const GemmRoute &route)
{
    // the fused call also keeps the quantized activations here: packed, or header + FP16 values
    return kWsCtrlRegion + (size_t)make_layout(M, K).total_bytes + gemm_only_need(M, N, K, route);
}

// What callers are told to allocate.  A server allocates for its largest batch and passes smaller ones as well: above 32
// rows, where the kernels differ in what they use, the size covers the prefill kernel's buffers for that many rows and
// whatever 32 rows need (partial sums of K in parts: 8.3 MB for 4096 x 12288, where 64 rows use 0.9 MB themselves).
size_t gemm_workspace_bytes(int64_t M, int64_t N, int64_t K)
{
    const size_t own = gemm_workspace_need(M, N, K, gemm_route(M, N, K));
    if (M <= 32) return own;
    const size_t prefill = kWsCtrlRegion + (size_t)make_layout(M, K).total_bytes + gemm_ws_layout(M, N, K).total;
    return std::max(std::max(own, prefill), gemm_workspace_need(32, N, K, gemm_route(32, N, K)));
}

static bool fused_prefill(int64_t M, int64_t N, int64_t K)
{
    return kUseHwCvt && !gemm_skinny_applies(M, N, K) && mixed_kernel_applies(N, K);
}

size_t quant_gemm_workspace_need(int64_t M, int64_t N, int64_t K, const GemmRoute &route)
{
    // (an odd number of row-tiles: as for the two launches that such a step took before, which need more)
    if (even_row_tiles(N) && gemm_stream_applies(M, N, K)) return kWsCtrlRegion + gemm_stream_scratch_bytes(M, N, K);
    if (mid_asks_less(M, route)) return kWsCtrlRegion + route.plan.bytes(K);
    if (fused_prefill(M, N, K)) {
        const GemmWorkspace w = gemm_ws_layout(M, N, K);
        return kWsCtrlRegion + fused_prefill_split(w) + (w.total - w.off_split);
    }
    return gemm_workspace_need(M, N, K, route);
}

// `skip`: bytes behind the control region that the caller keeps for itself (the fused call's packed activations)
fgmp_status_t gemm_packed(const void *packed_X, int64_t M, const void *packed_W, int64_t N, int64_t K,
                          float *Y, int64_t ldy, void *workspace, size_t workspace_bytes, hipStream_t st, const GemmRoute &route,
                          size_t skip)
{
    if (!packed_X || !packed_W || !Y || !workspace) return FGMP_ERR_INVALID_ARG;
    if (M <= 0 || N <= 0 || K <= 0) return FGMP_ERR_INVALID_ARG;
    if (K % kBlock != 0 || ldy < N) return FGMP_ERR_BAD_SHAPE;
    if (((uintptr_t)packed_X | (uintptr_t)packed_W | (uintptr_t)Y | (uintptr_t)workspace) % 16 != 0)
        return FGMP_ERR_BAD_ALIGN;
    if (workspace_bytes < kWsCtrlRegion + skip + gemm_only_need(M, N, K, route)) return FGMP_ERR_BUFFER_TOO_SMALL;
    const PackedLayout la = make_layout(M, K), lb = make_layout(N, K);
    const PackedView A = make_view(const_cast<void *>(packed_X), la);
    const PackedView B = make_view(const_cast<void *>(packed_W), lb);
    void *const ctrl = workspace;
    workspace = static_cast<char *>(workspace) + kWsCtrlRegion + skip;
    if (!route.mid && gemm_stream_applies(M, N, K))
        return gemm_stream(2, nullptr, 0, nullptr, 0.0f, 1.0f, packed_X, M, packed_W, N, K, Y, ldy, ctrl, workspace, st);
    if (route.mid) {
        const int64_t ld16 = round_up(K, kTileK);
        _Float16 *x16 = reinterpret_cast<_Float16 *>(static_cast<char *>(workspace) + kHeaderBytes);
        const fgmp_status_t rcx = launch_decode_f16(make_decode_job(A, la, x16, ld16, la.n_rt), nullptr, nullptr, 0, st);
        if (rcx != FGMP_OK) return rcx;
        return gemm_mid(route.plan, MidInput{A.hdr}, x16, ld16, packed_W, M, N, K, Y, ldy, ctrl,
                        static_cast<char *>(workspace) + kHeaderBytes + route.plan.x16_bytes(K), st);
    }
    if (gemm_skinny_applies(M, N, K)) {
        // decode shapes: expand the few activation rows to FP16 once, then stream the weights
        _Float16 *x16 = static_cast<_Float16 *>(workspace);
        const int64_t ld16 = round_up(K, kTileK);
        const DecodeJob jx = make_decode_job(A, la, x16, ld16, gemm_skinny_x16_rows(M) / kTileRows);
        char *sws = static_cast<char *>(workspace) + skinny_x16_bytes(M, K);
        const SkinnyCounters ctr = gemm_skinny_counters(M, N, K, sws);
        const fgmp_status_t rcx = launch_decode_f16(jx, nullptr, ctr.ptr, ctr.n, st);
        if (rcx != FGMP_OK) return rcx;
        return gemm_skinny(A.hdr, la, x16, ld16, packed_W, lb, M, N, K, Y, ldy, sws, st);
    }
    const GemmWorkspace w = gemm_ws_layout(M, N, K);
    if (mixed_kernel_applies(N, K)) {
        // activations expanded to FP16 once (M x K is small); weights decoded inside the MFMA kernel
        _Float16 *x16 = reinterpret_cast<_Float16 *>(static_cast<char *>(workspace) + w.off_a);
        const int64_t tiles_m = w.Mp / kBM, tiles_n = w.Np / kBN;
        if (tiles_m * tiles_n > 0x7FFFFFFF) return FGMP_ERR_UNSUPPORTED;
        const DecodeJob jx = make_decode_job(A, la, x16, w.ld, w.Mp / kTileRows);
        const SplitTail sp = plan_split_tail(tiles_m * tiles_n, (int)(w.ld / kBK), static_cast<char *>(workspace) + w.off_split);
        const fgmp_status_t rcx = launch_decode_f16(jx, nullptr, sp.counters, (int64_t)sp.n_counters, st);
        if (rcx != FGMP_OK) return rcx;
        launch_gemm_mixed(x16, w.ld, B, lb, Y, ldy, M, N, tiles_m, tiles_n, A.hdr, st, sp);
        return hipGetLastError() == hipSuccess ? FGMP_OK : FGMP_ERR_HIP;
    }
    _Float16 *a16 = reinterpret_cast<_Float16 *>(static_cast<char *>(workspace) + w.off_a);
    _Float16 *b16 = reinterpret_cast<_Float16 *>(static_cast<char *>(workspace) + w.off_b);
    const int64_t n_tm = w.Mp / kBM, n_tn = w.Np / kBN;
    if (n_tm * n_tn > 0x7FFFFFFF) return FGMP_ERR_UNSUPPORTED;
    const DecodeJob ja = make_decode_job(A, la, a16, w.ld, w.Mp / kTileRows);
    const DecodeJob jb = make_decode_job(B, lb, b16, w.ld, w.Np / kTileRows);
    const fgmp_status_t rc = launch_decode_f16(ja, &jb, nullptr, 0, st);
    if (rc != FGMP_OK) return rc;
    hipLaunchKernelGGL((gemm_f16_kernel<FGMP_GEMM_WM, FGMP_GEMM_WN>), dim3((unsigned)(n_tm * n_tn)),
                       dim3(FGMP_GEMM_WM * FGMP_GEMM_WN * 64), 0, st, a16, b16, w.ld,
                       (int)(w.ld / kBK), Y, ldy, M, N, n_tm, n_tn, A.hdr, B.hdr);
    return hipGetLastError() == hipSuccess ? FGMP_OK : FGMP_ERR_HIP;
}

// Fused call.  Prefill shapes: the quantizer writes the FP16 values of the codes
// it selects straight into the GEMM's A operand (the packed form of X is never
// materialized; only its header, which carries the tensor scale).  Other shapes
// and the two-pass path go through the packed activations.
fgmp_status_t quant_gemm(const void *X, fgmp_dtype_t dt, int64_t M, int64_t K, int64_t ldx, const float *fisher_k,
                         float threshold, float scale_x, const void *packed_W, int64_t N, float *Y, int64_t ldy,
                         void *workspace, size_t workspace_bytes, hipStream_t st, const GemmRoute &route, int score_mode,
                         const PackOut *pack_out, bool tight)
{
    if (!workspace || !packed_W || (!Y && !pack_out)) return FGMP_ERR_INVALID_ARG;
    if (M <= 0 || N <= 0 || K <= 0) return FGMP_ERR_INVALID_ARG;
    if (K % kBlock != 0 || ldy < N) return FGMP_ERR_BAD_SHAPE;
    if (((uintptr_t)workspace | (uintptr_t)packed_W | (uintptr_t)Y) % 16 != 0) return FGMP_ERR_BAD_ALIGN;
    // (the one-launch kernel addresses X with 32-bit byte offsets)
    const bool x_fits = ldx > 0 && ldx < (int64_t)0xFFFFFF00 / (M * 4);
    const bool one_launch = score_mode == FGMP_SCORE_NVFP4_ERROR && x_fits && gemm_stream_applies(M, N, K);
    const bool mid = route.mid || (route.mid_if_not_one_launch && !one_launch);
    // (the decode step quantizes its own results where the caller asks for it -- and where the plain call takes it, too: the
    // packed results are the same bit for bit either way)
    const bool stream_pack = pack_out != nullptr && !pack_out->gate && pack_out->one_launch && !mid && gemm_stream_packs(M, N, K);
    const bool stream_fits = one_launch && (pack_out == nullptr || stream_pack);
    const bool stream = stream_fits && !mid;
    if (workspace_bytes < (stream_fits ? (pack_out ? kWsCtrlRegion + gemm_stream_pack_scratch_bytes(M, N, K) : quant_gemm_workspace_need(M, N, K, route))
                                  : tight && M > 32 ? quant_gemm_workspace_need(M, N, K, route) : gemm_workspace_need(M, N, K, route)))
        return FGMP_ERR_BUFFER_TOO_SMALL;
    char *ws = static_cast<char *>(workspace) + kWsCtrlRegion;
    if (stream) {
        // decode shapes: one launch quantizes the activation rows and streams the weights (and, with
        // `pack_out`, quantizes and packs the results)
        if (!X || !fisher_k || (!Y && !pack_out)) return FGMP_ERR_INVALID_ARG;
        if (dt != FGMP_F32 && dt != FGMP_BF16) return FGMP_ERR_UNSUPPORTED;
        if (!(scale_x > 0.0f) || !(scale_x < INFINITY) || threshold != threshold) return FGMP_ERR_INVALID_ARG;
        const int64_t esz = dt == FGMP_F32 ? 4 : 2;
        if (ldx < K) return FGMP_ERR_BAD_SHAPE;
        if (((uintptr_t)X | (uintptr_t)fisher_k) % 16 != 0 || (ldx * esz) % 16 != 0) return FGMP_ERR_BAD_ALIGN;
        return gemm_stream(dt == FGMP_F32 ? 1 : 0, X, ldx, fisher_k, threshold, scale_x, nullptr, M, packed_W, N, K, Y, ldy,
                           workspace, ws, st, pack_out);
    }
    if (mid) {
        if (pack_out != nullptr) return FGMP_ERR_UNSUPPORTED;   // the caller stages the FP32 results
        // the FP16 values of the codes that the quantizer selects: made by the launch of the product, or by one before it
        const int64_t ld16 = round_up(K, kTileK);
        _Float16 *x16 = reinterpret_cast<_Float16 *>(ws + kHeaderBytes);
        MidInput in{reinterpret_cast<const PackedHeader *>(ws)};
        if (gemm_mid_quantizes(route.plan, M, N, K, ldx > 0 && ldx < INT64_MAX / 4 ? ldx * (dt == FGMP_F32 ? 4 : 2) : 0)) {
            const fgmp_status_t rc = check_quantizer_input(X, dt, M, K, ldx, fisher_k, threshold, scale_x, score_mode);
            if (rc != FGMP_OK) return rc;
            in = MidInput{nullptr, X, ldx, fisher_k, threshold, scale_x, dt == FGMP_F32, score_mode == FGMP_SCORE_DELTA};
        } else {
            const fgmp_status_t rc = quantize_tensor(X, dt, M, K, ldx, fisher_k, 0, threshold, scale_x, ws, sizeof(PackedHeader), nullptr,
                                                     false, st, x16, ld16, nullptr, 0, score_mode);
            if (rc != FGMP_OK) return rc;
        }
        return gemm_mid(route.plan, in, x16, ld16, packed_W, M, N, K, Y, ldy, workspace,
                        ws + kHeaderBytes + route.plan.x16_bytes(K), st);
    }
    const bool in_kernel_prefill = fused_prefill(M, N, K);
    if (pack_out != nullptr && !in_kernel_prefill) return FGMP_ERR_UNSUPPORTED;   // the caller falls back
    if (gemm_skinny_applies(M, N, K) && kUseHwCvt) {
        // decode shapes: FP16 values of X (rows beyond the last 8-row group stay unwritten: they only
        // feed output rows that are never stored), then the weight-streaming kernel
        const int64_t ld16 = round_up(K, kTileK);
        _Float16 *x16 = reinterpret_cast<_Float16 *>(ws + kHeaderBytes);
        char *sws = ws + kHeaderBytes + skinny_x16_bytes(M, K);
        const SkinnyCounters ctr = gemm_skinny_counters(M, N, K, sws);
        const fgmp_status_t rc = quantize_tensor(X, dt, M, K, ldx, fisher_k, 0, threshold, scale_x, ws,
                                                 sizeof(PackedHeader), nullptr, false, st, x16, ld16, ctr.ptr, ctr.n,
                                                 score_mode);
        if (rc != FGMP_OK) return rc;
        return gemm_skinny(reinterpret_cast<const PackedHeader *>(ws), make_layout(M, K), x16, ld16, packed_W,
                           make_layout(N, K), M, N, K, Y, ldy, sws, st);
    }
    if (in_kernel_prefill) {
        const GemmWorkspace w = gemm_ws_layout(M, N, K);
        const int64_t tiles_m = w.Mp / kBM, tiles_n = w.Np / kBN;
        if (tiles_m * tiles_n > 0x7FFFFFFF) return FGMP_ERR_UNSUPPORTED;
        PackedHeader *hx = reinterpret_cast<PackedHeader *>(ws);
        _Float16 *x16 = reinterpret_cast<_Float16 *>(ws + kHeaderBytes);
        // The partial tiles behind the room that the packed activations and both FP16 operands would take, not right behind the
        // activations, where there is room for that: 2048 x 256 x 4096 (M, K, N) 34.2 us there, 37.3 here (two parts).
        const size_t far = (size_t)make_layout(M, K).total_bytes + w.off_split;
        char *split_region = ws + (kWsCtrlRegion + far + (w.total - w.off_split) <= workspace_bytes ? far : fused_prefill_split(w));
        const SplitTail sp = plan_split_tail(tiles_m * tiles_n, (int)(w.ld / kBK), split_region);
        const fgmp_status_t rc = quantize_tensor(X, dt, M, K, ldx, fisher_k, 0, threshold, scale_x, ws,
                                                 sizeof(PackedHeader), nullptr, false, st, x16, w.ld, sp.counters,
                                                 (int64_t)sp.n_counters, score_mode);
        if (rc != FGMP_OK) return rc;
        const PackedLayout lb = make_layout(N, K);
        const PackedView B = make_view(const_cast<void *>(packed_W), lb);
        launch_gemm_mixed(x16, w.ld, B, lb, Y, ldy, M, N, tiles_m, tiles_n, hx, st, sp, pack_out);
        return hipGetLastError() == hipSuccess ? FGMP_OK : FGMP_ERR_HIP;
    }
    const size_t xbytes = (size_t)make_layout(M, K).total_bytes;
    const fgmp_status_t rc = quantize_tensor(X, dt, M, K, ldx, fisher_k, 0, threshold, scale_x, ws, xbytes,
                                             nullptr, false, st, nullptr, 0, nullptr, 0, score_mode);
    if (rc != FGMP_OK) return rc;
    // (the packed activations sit behind the control region; the product's own workspace starts with one)
    return gemm_packed(ws, M, packed_W, N, K, Y, ldy, workspace, workspace_bytes, st, route, xbytes);
}

// Fused call whose results are quantized and packed instead of stored as FP32 (Sec. 4.2).  Prefill
// shapes do it in the GEMM's epilogue, decode steps (M <= 32) inside their one launch when asked to
// (FGMP_EPILOGUE_ONE_LAUNCH); otherwise, for other shapes, the gated epilogue at decode sizes and the
// two-pass path, the FP32 results go to the workspace and the standalone quantizer runs over them -- the
// same arithmetic on the same values.
// (the gated activation is applied as the quantizer reads the product: no room of its own)
static size_t staging_bytes(int64_t M, int64_t N) { return (size_t)align_up((uint64_t)M * N * 4, 256); }

size_t gemm_workspace_bytes_packed_out(int64_t M, int64_t N, int64_t K)
{
    return (size_t)align_up(gemm_workspace_bytes(M, N, K), 256) + staging_bytes(M, N);
}

fgmp_status_t quant_gemm_packed_out(const void *X, fgmp_dtype_t dt, int64_t M, int64_t K, int64_t ldx,
                                    const float *fisher_k, float threshold, float scale_x, const void *packed_W,
                                    int64_t N, const float *fisher_n, float threshold_y, float scale_y,
                                    void *packed_Y, size_t packed_Y_bytes, float *scores_y, void *workspace,
                                    size_t workspace_bytes, hipStream_t st, int epilogue)
{
    if (!fisher_n || !packed_Y || !workspace) return FGMP_ERR_INVALID_ARG;
    if (M <= 0 || N <= 0 || K <= 0) return FGMP_ERR_INVALID_ARG;
    const bool one_launch = (epilogue & FGMP_EPILOGUE_ONE_LAUNCH) != 0;
    epilogue &= ~(int)FGMP_EPILOGUE_ONE_LAUNCH;
    if (epilogue != FGMP_EPILOGUE_NONE && epilogue != FGMP_EPILOGUE_SILU_GATE) return FGMP_ERR_INVALID_ARG;
    if (!(scale_y > 0.0f) || !(scale_y < INFINITY) || threshold_y != threshold_y) return FGMP_ERR_INVALID_ARG;
    const bool gate = epilogue == FGMP_EPILOGUE_SILU_GATE;
    if (N % (gate ? kGateGroup : kBlock) != 0 || K % kBlock != 0) return FGMP_ERR_BAD_SHAPE;
    const int64_t n_out = gate ? N / 2 : N;   // columns of the quantized result
    if (((uintptr_t)fisher_n | (uintptr_t)packed_Y | (uintptr_t)scores_y | (uintptr_t)workspace) % 16 != 0)
        return FGMP_ERR_BAD_ALIGN;
    if (M * (N / kBlock) >= (int64_t)1 << 32) return FGMP_ERR_UNSUPPORTED;
    const PackedLayout ly = make_layout(M, n_out);
    if (packed_Y_bytes < ly.total_bytes) return FGMP_ERR_BUFFER_TOO_SMALL;
    const GemmRoute route = gemm_route(M, N, K);
    const size_t base_bytes = gemm_workspace_need(M, N, K, route);
    if (workspace_bytes < align_up(base_bytes, 256) + staging_bytes(M, N)) return FGMP_ERR_BUFFER_TOO_SMALL;
    PackOut po;
    po.out = make_view(packed_Y, ly);
    po.layout = ly;
    po.fisher = fisher_n;
    po.T = threshold_y;
    po.S = scale_y;
    po.scores = scores_y;
    po.gate = gate ? 1 : 0;
    po.one_launch = one_launch ? 1 : 0;
    // (the whole workspace: the one-launch decode step keeps its row groups' decisions behind its partial sums)
    fgmp_status_t rc = quant_gemm(X, dt, M, K, ldx, fisher_k, threshold, scale_x, packed_W, N, nullptr, N, workspace,
                                  workspace_bytes, st, route, FGMP_SCORE_NVFP4_ERROR, &po);
    if (rc != FGMP_ERR_UNSUPPORTED) return rc;
    float *Yf = reinterpret_cast<float *>(static_cast<char *>(workspace) + align_up(base_bytes, 256));
    rc = quant_gemm(X, dt, M, K, ldx, fisher_k, threshold, scale_x, packed_W, N, Yf, N, workspace, base_bytes, st, route,
                    FGMP_SCORE_NVFP4_ERROR, nullptr);
    if (rc != FGMP_OK) return rc;
    // (the gated activation is applied by the quantizer as it reads the staged product)
    return quantize_tensor(Yf, FGMP_F32, M, n_out, N, fisher_n, 0, threshold_y, scale_y, packed_Y, packed_Y_bytes, scores_y,
                           /*compact=*/false, st, nullptr, 0, nullptr, 0, FGMP_SCORE_NVFP4_ERROR, /*clip=*/false, gate);
}

// The order of quant_gemm's decisions, for tests.
int64_t selftest_quantizing_workgroups(int64_t M, int64_t N, int64_t K)
{
    const GemmRoute r = gemm_route(M, N, K);
    return r.mid ? gemm_mid_shares(r.plan, M, N, K, K * 4) : 0;
}

void selftest_gemm_route(int64_t M, int64_t N, int64_t K, int64_t *route)
{
    std::fill(route, route + 6, (int64_t)0);
    const GemmRoute r = gemm_route(M, N, K);
    if (r.mid) {
        const int64_t v[6] = {2, r.plan.mt, r.plan.nt, r.plan.tiles_m, r.plan.tiles_n, r.plan.parts};
        std::copy(v, v + 6, route);
    } else if (gemm_stream_applies(M, N, K)) {
        route[0] = 0;
    } else if (fused_prefill(M, N, K)) {
        const GemmWorkspace w = gemm_ws_layout(M, N, K);
        const SplitTail sp = plan_split_tail((w.Mp / kBM) * (w.Np / kBN), (int)(w.ld / kBK), route);   // (any address: nothing is written)
        const int64_t v[6] = {3, w.ld / kBK, sp.n_whole, sp.n_split, sp.n_split > 0 ? sp.n_parts : 1, 0};
        std::copy(v, v + 6, route);
    } else {
        route[0] = gemm_skinny_applies(M, N, K) && kUseHwCvt ? 1 : 4;
    }
}

// Measurement reference: independent MFMAs only (8 accumulators per wave, so no instruction waits for
// the previous one's result).
__global__ __launch_bounds__(256) void mfma_rate_kernel(float *sink, int iters)
{
    half8_t a, b;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        a[i] = (_Float16)(0.001f * (float)(threadIdx.x & 63) + (float)i);
        b[i] = (_Float16)(0.5f * (float)i);
    }
    float16_t acc[8];
#pragma unroll
    for (int n = 0; n < 8; ++n)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[n][r] = 0.0f;
    for (int it = 0; it < iters; ++it) {
#pragma unroll
        for (int n = 0; n < 8; ++n) acc[n] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, acc[n], 0, 0, 0);
    }
    float s = 0.0f;
#pragma unroll
    for (int n = 0; n < 8; ++n)
#pragma unroll
        for (int r = 0; r < 16; ++r) s += acc[n][r];
    sink[(size_t)blockIdx.x * 256 + threadIdx.x] = s;
}

fgmp_status_t selftest_mfma_rate(int64_t workgroups, int32_t iters, float *sink, hipStream_t st)
{
    if (!sink || workgroups <= 0 || workgroups > 0x7FFFFFFF || iters <= 0) return FGMP_ERR_INVALID_ARG;
    hipLaunchKernelGGL(mfma_rate_kernel, dim3((unsigned)workgroups), dim3(256), 0, st, sink, (int)iters);
    return hipGetLastError() == hipSuccess ? FGMP_OK : FGMP_ERR_HIP;
}

}  // namespace fgmp
