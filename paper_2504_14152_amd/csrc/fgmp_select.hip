// Threshold for a target fraction of FP8 blocks (Eq. 9; over several tensors, Eq. 10): an exact order
// statistic of the scores, found on the device.  The scores stay where the quantizer wrote them: three
// passes of a radix selection over all tensors (digits of 11, 11 and 10 bits, most significant first) narrow
// the 32-bit key of the wanted element down digit by digit; a pass counts, per value of the current digit, the
// elements whose higher digits equal the prefix found so far, and the workgroup of a pass that finishes last
// walks the bins to the one that holds the wanted rank.  Keys order like the numbers: the bit pattern of a
// non-negative float with the sign bit set, that of a negative one inverted (-0 sorts just below +0; both
// compare equal to either as a threshold).  Every pass reads every score once -- 16 bytes per lane where the
// array allows -- so the selection costs three reads of the scores, against a copy to the host and a partial
// sort there.
//
// What bounds a pass is not the read (22 MB of scores come out of the caches in 4 us) but the counting: the
// scores of a tensor share a few exponents, so with a digit of 8 bits -- sign and seven exponent bits -- nearly
// every lane of a wave added to the same LDS bin in the first pass.  Eleven bits take in two mantissa bits as
// well, every wave counts into bins of its own, and few, large workgroups merge their bins with few global atomics:
// one for every other compute unit, since the merge costs more than the reading gains (a selection from 5.6 M scores, host
// included, 48.9 us with 256 workgroups, 45.3 with 128; 2.8 M 40.5 / 39.7; fewer do not ask for that many).
#include <algorithm>
#include <atomic>
#include <cstring>

#include "fgmp_internal.hpp"

namespace fgmp {

namespace {

constexpr int kSelPasses = 3, kSelBins = 2048;
constexpr int kSelThreads = 1024, kSelCopies = 8, kSelMaxWgs = 128;   // 8 x 2048 bins: 64 KB of LDS; two waves share a copy

struct SelectState {
    unsigned long long hist[kSelPasses][kSelBins];   // zero between selections: the workgroup that reads a pass's bins clears them
    unsigned long long rank;        // wanted element, counted from the smallest among those that match the prefix
    uint32_t prefix;                // digits found so far
    uint32_t arrived;               // workgroups of the pass in progress that have merged their bins; zero between passes
    float result;
};

__host__ __device__ constexpr int sel_shift(int pass) { return pass == 0 ? 21 : pass == 1 ? 10 : 0; }
__host__ __device__ constexpr int sel_bits(int pass) { return pass == 2 ? 10 : 11; }

__device__ __forceinline__ uint32_t key_of(float v)
{
    const uint32_t b = __builtin_bit_cast(uint32_t, v);
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}

__device__ inline float value_of(uint32_t key)
{
    const uint32_t b = (key & 0x80000000u) ? (key & 0x7FFFFFFFu) : ~key;
    return __builtin_bit_cast(float, b);
}

// The workgroup that arrives last (all bins of the pass are merged): the bin that holds the wanted rank becomes
// the next digit of the prefix.
template <int kPass>
__device__ __forceinline__ void narrow(SelectState *st, unsigned long long wanted, float *result_host, unsigned long long *part)
{
    constexpr int kBins = 1 << sel_bits(kPass), kPer = kBins / kSelThreads;
    static_assert(kPer >= 1, "a thread owns at least one bin");
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    unsigned long long h[kPer], sum = 0ull;
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        h[i] = __hip_atomic_load(&st->hist[kPass][tid * kPer + i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        sum += h[i];
    }
#pragma unroll
    for (int i = 0; i < kPer; ++i)
        if (h[i] != 0ull) __hip_atomic_store(&st->hist[kPass][tid * kPer + i], 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    unsigned long long incl = sum;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const unsigned long long v = __shfl_up(incl, d);
        incl += lane >= d ? v : 0ull;
    }
    if (lane == 63) part[wave] = incl;
    const unsigned long long rank = kPass == 0 ? wanted : st->rank;   // (written by the pass before)
    const uint32_t prefix = kPass == 0 ? 0u : st->prefix;
    __syncthreads();
    unsigned long long below = incl - sum;
    for (int w = 0; w < wave; ++w) below += part[w];
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        // exactly one bin of the pass holds the rank
        if (rank >= below && rank < below + h[i]) {
            const uint32_t p = prefix | ((uint32_t)(tid * kPer + i) << sel_shift(kPass));
            st->rank = rank - below;
            st->prefix = p;
            if (kPass == kSelPasses - 1) {
                st->result = value_of(p);
                if (result_host != nullptr) __hip_atomic_store(result_host, value_of(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
            }
        }
        below += h[i];
    }
    if (tid == 0) st->arrived = 0u;
}

// One pass over one array; `n_wgs` workgroups take part in the pass over all arrays together.
template <int kPass>
__global__ __launch_bounds__(kSelThreads) void select_count_kernel(const float *__restrict__ s, int64_t n, uint32_t n_wgs, SelectState *st,
                                                                   unsigned long long wanted, float *result_host)
{
    constexpr int kBins = 1 << sel_bits(kPass), kShift = sel_shift(kPass);
    constexpr uint32_t kHigher = kPass == 0 ? 0u : ~0u << sel_shift(kPass - 1);   // bits of the digits found before
    __shared__ __attribute__((aligned(16))) uint32_t bins[kSelCopies][kBins];
    __shared__ uint32_t last;
    const int tid = threadIdx.x;
    for (int i = tid; i < kSelCopies * kBins / 4; i += kSelThreads) reinterpret_cast<uint4 *>(&bins[0][0])[i] = make_uint4(0u, 0u, 0u, 0u);
    __syncthreads();
    const uint32_t prefix = kPass == 0 ? 0u : st->prefix;
    uint32_t *mine = bins[(tid >> 6) % kSelCopies];
    auto take = [&](float v) {
        const uint32_t k = key_of(v);
        if ((k & kHigher) == prefix) atomicAdd(&mine[(k >> kShift) & (uint32_t)(kBins - 1)], 1u);
    };
    // the part of the array that is aligned to 16 bytes in quads, the rest one by one
    const int64_t to_aligned = (int64_t)((16 - ((uintptr_t)s & 15)) & 15) / 4;
    const int64_t head = to_aligned < n ? to_aligned : n;
    const int64_t quads = (n - head) / 4;
    const float4 *q = reinterpret_cast<const float4 *>(s + head);
    const int64_t stride = (int64_t)gridDim.x * kSelThreads;
    int64_t i = (int64_t)blockIdx.x * kSelThreads + tid;
    for (; i + 3 * stride < quads; i += 4 * stride) {   // four loads in flight
        float4 v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = q[i + u * stride];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            take(v[u].x);
            take(v[u].y);
            take(v[u].z);
            take(v[u].w);
        }
    }
    for (; i < quads; i += stride) {
        const float4 v = q[i];
        take(v.x);
        take(v.y);
        take(v.z);
        take(v.w);
    }
    if (blockIdx.x == 0) {
        for (int64_t j = tid; j < head; j += kSelThreads) take(s[j]);
        for (int64_t j = head + quads * 4 + tid; j < n; j += kSelThreads) take(s[j]);
    }
    __syncthreads();
    for (int b = tid; b < kBins; b += kSelThreads) {
        uint32_t c = 0u;
#pragma unroll
        for (int u = 0; u < kSelCopies; ++u) c += bins[u][b];
        if (c != 0u)
            __hip_atomic_fetch_add(&st->hist[kPass][b], (unsigned long long)c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    // every atomic of the workgroup has been performed before it counts as arrived
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (tid == 0)
        last = __hip_atomic_fetch_add(&st->arrived, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == n_wgs - 1u;
    __syncthreads();
    if (last) narrow<kPass>(st, wanted, result_host, reinterpret_cast<unsigned long long *>(&bins[0][0]));
}

__global__ __launch_bounds__(256) void select_init_kernel(SelectState *st)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < kSelPasses * kSelBins) (&st->hist[0][0])[i] = 0ull;
    if (i == 0) st->arrived = 0u;
}

template <int kPass>
void launch_count(const float *s, int64_t n, unsigned grid, uint32_t n_wgs, SelectState *state, unsigned long long wanted, float *result_host,
                  hipStream_t st)
{
    hipLaunchKernelGGL((select_count_kernel<kPass>), dim3(grid), dim3(kSelThreads), 0, st, s, n, n_wgs, state, wanted, result_host);
}

// States that selections borrow, and a pinned word each for the result.  A state allocated and freed per call, cleared by a
// launch of its own and its result copied to pageable memory: scoring, selecting and packing 1193 x 832 weights 93 us, now 50;
// 3302 x 2560 106 / 66; 22016 x 4096 374 / 320.  Up to kSelSlots selections per GPU run at a time on these (each holds its own
// from before its first launch until its stream has been waited for); a further one allocates its state.  The states are part of
// the module, the result words one allocation of the process.
constexpr int kSelSlots = 8, kMaxDevices = 64;
__device__ SelectState g_states[kSelSlots];   // zero when the library is loaded
std::atomic<uint32_t> g_taken[kMaxDevices];   // slots in use, one bit each

float *result_words()
{
    static float *const words = [] {
        void *p = nullptr;
        return hipHostMalloc(&p, (size_t)kMaxDevices * kSelSlots * 64, hipHostMallocPortable | hipHostMallocMapped) == hipSuccess
                   ? static_cast<float *>(p)
                   : nullptr;
    }();
    return words;
}

struct SelectLease {
    SelectState *state = nullptr;
    float *result_host = nullptr;   // null: the state was allocated, and the result is copied from there
    int dev = -1, slot = -1;
    bool take()
    {
        if (hipGetDevice(&dev) != hipSuccess) return false;
        SelectState *all = nullptr;
        if (dev >= 0 && dev < kMaxDevices && result_words() != nullptr &&
            hipGetSymbolAddress(reinterpret_cast<void **>(&all), HIP_SYMBOL(g_states)) == hipSuccess && all != nullptr) {
            uint32_t seen = g_taken[dev].load(std::memory_order_relaxed);
            while (seen != (1u << kSelSlots) - 1u) {
                const int free = __builtin_ctz(~seen);
                if (g_taken[dev].compare_exchange_weak(seen, seen | (1u << free), std::memory_order_acquire)) {
                    slot = free;
                    state = all + slot;
                    result_host = result_words() + ((size_t)dev * kSelSlots + slot) * 16;
                    return true;
                }
            }
        }
        return hipMalloc(reinterpret_cast<void **>(&state), sizeof(SelectState)) == hipSuccess;
    }
    // (a state that a failed selection may have left other than zero is not used again)
    void give_back(bool clean)
    {
        if (slot < 0) (void)hipFree(state);
        else if (clean) g_taken[dev].fetch_and(~(1u << slot), std::memory_order_release);
    }
};

// kSelMaxWgs at most, and not more than have four quads per thread to read
unsigned count_grid(int64_t n) { return (unsigned)std::min<int64_t>(kSelMaxWgs, (n / 4 + 4 * kSelThreads) / (4 * kSelThreads)); }

}  // namespace

// The element of rank `rank` (0 = smallest) of the union of the arrays; result on the host.  Synchronizes `st`.
fgmp_status_t select_rank(const float *const *scores, const int64_t *counts, int32_t n_tensors, int64_t rank, float *result_host,
                          hipStream_t st)
{
    uint64_t n_wgs = 0;
    for (int32_t i = 0; i < n_tensors; ++i) n_wgs += count_grid(counts[i]);
    if (n_wgs > 0xFFFFFFFFull) return FGMP_ERR_UNSUPPORTED;
    // (a stream that is being captured cannot be waited for)
    hipStreamCaptureStatus capturing = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(st, &capturing) != hipSuccess || capturing != hipStreamCaptureStatusNone) return FGMP_ERR_HIP;
    SelectLease lease;
    if (!lease.take()) return FGMP_ERR_HIP;
    fgmp_status_t rc = FGMP_OK;
    if (lease.result_host != nullptr) *lease.result_host = 0.0f;
    else hipLaunchKernelGGL(select_init_kernel, dim3((kSelPasses * kSelBins + 255) / 256), dim3(256), 0, st, lease.state);
    for (int pass = 0; pass < kSelPasses && rc == FGMP_OK; ++pass) {
        for (int32_t i = 0; i < n_tensors; ++i) {
            const unsigned grid = count_grid(counts[i]);
            const unsigned long long wanted = (unsigned long long)rank;
            if (pass == 0) launch_count<0>(scores[i], counts[i], grid, (uint32_t)n_wgs, lease.state, wanted, lease.result_host, st);
            else if (pass == 1) launch_count<1>(scores[i], counts[i], grid, (uint32_t)n_wgs, lease.state, wanted, lease.result_host, st);
            else launch_count<2>(scores[i], counts[i], grid, (uint32_t)n_wgs, lease.state, wanted, lease.result_host, st);
        }
        if (hipGetLastError() != hipSuccess) rc = FGMP_ERR_HIP;
    }
    if (rc == FGMP_OK && lease.result_host == nullptr &&
        hipMemcpyAsync(result_host, &lease.state->result, sizeof(float), hipMemcpyDeviceToHost, st) != hipSuccess)
        rc = FGMP_ERR_HIP;
    if (hipStreamSynchronize(st) != hipSuccess) rc = FGMP_ERR_HIP;
    if (rc == FGMP_OK && lease.result_host != nullptr) *result_host = *static_cast<volatile float *>(lease.result_host);
    lease.give_back(rc == FGMP_OK);
    return rc;
}

}  // namespace fgmp
