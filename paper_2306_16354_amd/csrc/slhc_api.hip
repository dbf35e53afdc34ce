// C ABI of the library (see include/slhc.h) and the host orchestration of the cuSLINK pipeline:
// Alg. "cuSLINK Algorithm" (k-NN graph -> MST -> connect -> relabel), Alg. "connect_graph",
// Alg. "MST Algorithm" of the paper, restructured as one certified Boruvka loop (see
// forest_kernels.hip for what "certified" means).
#include <hip/hip_runtime.h>
#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <exception>
#include <mutex>
#include <memory>
#include <new>
#include <optional>
#include <vector>

#include "../../include/slhc.h"
#include "cluster_kernels.h"
#include "csr_kernels.h"
#include "dendrogram_kernels.h"
#include "forest_kernels.h"
#include "near_kernels.h"
#include "direct_kernels.h"
#include "order_kernels.h"
#include "static_scratch.h"
#include "sweep_kernels.h"

namespace {

thread_local char g_err[512] = "";

void set_err(const char* fmt, ...)
{
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_err, sizeof(g_err), fmt, ap);
    va_end(ap);
}

int hip_fail(hipError_t e, const char* what)
{
    set_err("%s: %s", what, hipGetErrorString(e));
    return SLHC_HIP_ERROR;
}

#define HIP_TRY(expr)                                                  \
    do {                                                               \
        hipError_t _e = (expr);                                        \
        if (_e != hipSuccess) return hip_fail(_e, #expr);              \
    } while (0)

// Runs the body of an exported function; no C++ exception leaves the library.
template <typename F>
int guarded(F&& body) noexcept
{
    try {
        return body();
    } catch (const std::bad_alloc&) {
        set_err("a host allocation failed");
        return SLHC_HOST_MEMORY;
    } catch (const std::exception& e) {
        set_err("unexpected exception: %s", e.what());
        return SLHC_INTERNAL;
    } catch (...) {
        set_err("unexpected exception");
        return SLHC_INTERNAL;
    }
}

constexpr size_t ALIGN = 256;
inline size_t up(size_t b) { return (b + ALIGN - 1) & ~(ALIGN - 1); }

// Bump allocator over the caller's workspace (layout only; nothing is allocated).
struct Carver {
    unsigned char* base;
    size_t off = 0;
    explicit Carver(void* b) : base(static_cast<unsigned char*>(b)) {}
    template <typename T>
    T* take(size_t count)
    {
        T* p = base ? reinterpret_cast<T*>(base + off) : nullptr;
        off += up(count * sizeof(T));
        return p;
    }
};

int check_shape(int64_t N, int32_t d, int32_t k, bool need_k)
{
    if (N < 2 || d < 1) { set_err("need N >= 2 and d >= 1 (N=%lld d=%d)", (long long)N, d); return SLHC_INVALID_ARG; }
    if (need_k) {
        if (k < 1 || (int64_t)k > N - 1) { set_err("need 1 <= k <= N-1 (k=%d N=%lld)", k, (long long)N); return SLHC_INVALID_ARG; }
        if (k > SLHC_MAX_K) { set_err("k=%d exceeds SLHC_MAX_K=%d", k, SLHC_MAX_K); return SLHC_UNSUPPORTED; }
        if (N * (int64_t)k > 2147483647LL) { set_err("N*k exceeds 2^31-1"); return SLHC_UNSUPPORTED; }
    }
    if (N * (int64_t)d > 2147483647LL) { set_err("N*d exceeds 2^31-1"); return SLHC_UNSUPPORTED; }
    return SLHC_OK;
}

__global__ void k_zero_words(uint32_t* p, int n)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0u;
}

// *sum += a[0] + ... + a[n-1]
__global__ void __launch_bounds__(256) k_sum_words(const int32_t* __restrict__ a, int n, unsigned long long* __restrict__ sum)
{
    __shared__ unsigned long long part[256];
    unsigned long long s = 0;
    for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < n; i += (long long)gridDim.x * 256) s += (unsigned long long)a[i];
    part[threadIdx.x] = s;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) part[threadIdx.x] += part[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0 && part[0]) atomicAdd(sum, part[0]);
}

// Columns the sweeps work on.  A zero column adds fma(0, 0, s) = s to a distance and to a norm, so appending
// zero columns changes no bit of any output; it does change which kernels apply.  Up to 128 features the rows are
// padded to whole chunks of 32 columns (register-resident queries, split bfloat16 products, tile pruning for
// every d), beyond that to a multiple of 4 (vector loads and split products in the streaming kernel).  The
// padded copy lives at the head of the caller's workspace.  d is kept where the padded matrix would pass the
// 2^31-1 element limit.
int32_t working_columns(int64_t N, int32_t d)
{
    const int32_t dw = d <= 128 ? (d + 31) / 32 * 32 : (d + 3) / 4 * 4;
    return N * (int64_t)dw > 2147483647LL ? d : dw;
}
size_t padded_copy_bytes(int64_t N, int32_t d)
{
    const int32_t dw = working_columns(N, d);
    return dw == d ? 0 : up((size_t)N * (size_t)dw * sizeof(float));
}

// out[row][c] = c < d ? X[row][c] : 0 for c < dw (dw a multiple of 4); one thread per four output columns
__global__ void __launch_bounds__(256) k_pad_columns(const float* __restrict__ X, long long quads, int d, int dw,
                                                     float* __restrict__ out)
{
    const long long q = (long long)blockIdx.x * 256 + threadIdx.x;
    if (q >= quads) return;
    const int per_row = dw >> 2;
    const long long row = q / per_row;
    const int c0 = 4 * (int)(q - row * per_row);
    const float* src = X + row * d;
    float4 v;
    v.x = c0 < d ? src[c0] : 0.f;
    v.y = c0 + 1 < d ? src[c0 + 1] : 0.f;
    v.z = c0 + 2 < d ? src[c0 + 2] : 0.f;
    v.w = c0 + 3 < d ? src[c0 + 3] : 0.f;
    *reinterpret_cast<float4*>(out + row * dw + c0) = v;
}

int pad_columns(const float* X, int64_t N, int32_t d, int32_t dw, float* out, hipStream_t s)
{
    const long long quads = (long long)N * (dw >> 2);
    hipLaunchKernelGGL(k_pad_columns, dim3((unsigned)((quads + 255) / 256)), dim3(256), 0, s, X, quads, d, dw, out);
    HIP_TRY(hipGetLastError());
    return SLHC_OK;
}

// Regions of the reordered copy: runs of consecutive tiles whose centres stay close.  boundary[t] = 1 when tile t
// starts a region: the first tile, a tile without valid rows (radius < 0) or next to one, or a tile whose centre lies
// farther from the previous tile's than twice the larger of the two radii.
__global__ void __launch_bounds__(256) k_region_boundaries(const float* __restrict__ tile_c, const float* __restrict__ tile_r,
                                                           int T, int d, int32_t* __restrict__ boundary)
{
    const int t = blockIdx.x * 256 + threadIdx.x;
    if (t >= T) return;
    int b = 1;
    if (t > 0) {
        const float r0 = tile_r[t - 1], r1 = tile_r[t];
        if (r0 >= 0.f && r1 >= 0.f) {
            const float* c0 = tile_c + (size_t)(t - 1) * d;
            const float* c1 = tile_c + (size_t)t * d;
            float s2 = 0.f;
            for (int j = 0; j < d; ++j) { const float e = c1[j] - c0[j]; s2 = __builtin_fmaf(e, e, s2); }
            const float reach = 2.f * fmaxf(r0, r1);
            b = (s2 <= reach * reach) ? 0 : 1;           // NaN: a boundary
        }
    }
    boundary[t] = b;
}
// region[t] = number of the region tile t lies in, first[t] = the first tile of that region (one workgroup)
__global__ void __launch_bounds__(1024) k_region_scan(const int32_t* __restrict__ boundary, int T, int32_t* __restrict__ region,
                                                      int32_t* __restrict__ first)
{
    __shared__ int cnt[1024], last[1024];
    const int tid = threadIdx.x;
    const int per = (T + 1023) / 1024;
    const int t0 = tid * per < T ? tid * per : T, t1 = t0 + per < T ? t0 + per : T;
    int c = 0, l = -1;
    for (int t = t0; t < t1; ++t) if (boundary[t]) { ++c; l = t; }
    cnt[tid] = c; last[tid] = l;
    __syncthreads();
    for (int off = 1; off < 1024; off <<= 1) {
        const int cv = tid >= off ? cnt[tid - off] : 0, lv = tid >= off ? last[tid - off] : -1;
        __syncthreads();
        cnt[tid] += cv; last[tid] = last[tid] > lv ? last[tid] : lv;
        __syncthreads();
    }
    int rc = tid > 0 ? cnt[tid - 1] : 0, rl = tid > 0 ? last[tid - 1] : -1;
    for (int t = t0; t < t1; ++t) {
        if (boundary[t]) { ++rc; rl = t; }
        region[t] = rc > 0 ? rc - 1 : 0;
        first[t] = rl >= 0 ? rl : 0;
    }
}
// last[t] = the last tile of tile t's region: the thread of a region's last tile writes the whole run
__global__ void __launch_bounds__(256) k_region_last(const int32_t* __restrict__ boundary, const int32_t* __restrict__ first, int T,
                                                     int32_t* __restrict__ last)
{
    const int t = blockIdx.x * 256 + threadIdx.x;
    if (t >= T) return;
    if (t == T - 1 || boundary[t + 1] != 0) {
        int u = first[t];
        if (u < 0) u = 0;
        for (; u <= t; ++u) last[u] = t;
    }
}
// local[t], centre[t] = the tile's region and that one's first tile where it is at least REGION_TILES long, else -1; *pairs += the tiles of t's region
constexpr int REGION_TILES = 8;
__global__ void __launch_bounds__(256) k_region_local(const int32_t* __restrict__ region, const int32_t* __restrict__ first,
                                                      const int32_t* __restrict__ last, int T, int32_t* __restrict__ local,
                                                      int32_t* __restrict__ centre, unsigned long long* __restrict__ pairs)
{
    const int t = blockIdx.x * 256 + threadIdx.x;
    int len = 0;
    if (t < T) {
        len = last[t] - first[t] + 1;
        local[t] = len >= REGION_TILES ? region[t] : -1;
        centre[t] = len >= REGION_TILES ? first[t] : -1;
    }
    unsigned long long sum = (unsigned long long)(len > 0 ? len : 0);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o);
    if ((threadIdx.x & 63) == 0 && sum) atomicAdd(pairs, sum);
}

// The listed rows in the order of their positions: slot[position] >= 0 marks them; one wavefront per tile of 128 positions.
__global__ void __launch_bounds__(256) k_slot_counts(const int32_t* __restrict__ slot, int n, int T, int32_t* __restrict__ count)
{
    const int t = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (t >= T) return;
    int c = 0;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int p = t * 128 + h * 64 + lane;
        c += __popcll(__ballot(p < n && slot[p] >= 0));
    }
    if (lane == 0) count[t] = c;
}
__global__ void __launch_bounds__(1024) k_slot_offsets(int32_t* __restrict__ count, int T)
{
    __shared__ int sum[1024];
    const int tid = threadIdx.x, per = (T + 1023) / 1024;
    const int t0 = tid * per < T ? tid * per : T, t1 = t0 + per < T ? t0 + per : T;
    int c = 0;
    for (int t = t0; t < t1; ++t) c += count[t];
    sum[tid] = c;
    __syncthreads();
    for (int off = 1; off < 1024; off <<= 1) {
        const int v = tid >= off ? sum[tid - off] : 0;
        __syncthreads();
        sum[tid] += v;
        __syncthreads();
    }
    int at = sum[tid] - c;
    for (int t = t0; t < t1; ++t) { const int v = count[t]; count[t] = at; at += v; }
}
__global__ void __launch_bounds__(256) k_slot_rows(int32_t* __restrict__ slot, const int32_t* __restrict__ perm, int n, int T,
                                                   const int32_t* __restrict__ offset, int m, int32_t* __restrict__ rows,
                                                   int32_t* __restrict__ pos)
{
    const int t = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (t >= T) return;
    int at = offset[t];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int p = t * 128 + h * 64 + lane;
        const bool marked = p < n && slot[p] >= 0;
        const unsigned long long mask = __ballot(marked);
        const int i = at + __builtin_amdgcn_mbcnt_hi((unsigned int)(mask >> 32), __builtin_amdgcn_mbcnt_lo((unsigned int)mask, 0u));
        if (marked && i < m) { rows[i] = perm[p]; pos[i] = p; slot[p] = i; }
        at += __popcll(mask);
    }
}

// out[row] = the smallest lower bound in row `row` of the table of tile pairs among the tiles of other regions
// (+inf: none; NaN entries mark tiles that are never needed)
__global__ void __launch_bounds__(256) k_region_other_min(const float* __restrict__ tile_gap, const int32_t* __restrict__ region,
                                                          int T, float* __restrict__ out)
{
    __shared__ float part[256];
    const int row = blockIdx.x;
    const int mine = region[row];
    const float* g = tile_gap + (size_t)row * T;
    float m = __builtin_inff();
    for (int t = threadIdx.x; t < T; t += 256) {
        const float v = g[t];
        if (region[t] != mine && v < m) m = v;          // false for NaN
    }
    part[threadIdx.x] = m;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) part[threadIdx.x] = fminf(part[threadIdx.x], part[threadIdx.x + w]);
        __syncthreads();
    }
    if (threadIdx.x == 0) out[row] = part[0];
}
// h[i] = +inf for the padding rows of the reordered copy (perm[i] < 0)
__global__ void __launch_bounds__(256) k_mask_padding(const int32_t* __restrict__ perm, int n, float* __restrict__ h)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < n && perm[i] < 0) h[i] = __builtin_inff();
}

// out[0], out[1] = sums of a[i] and b[i] over at most 16384 evenly spaced i < n (one workgroup, fixed order)
__global__ void __launch_bounds__(256) k_sample_sums(const float* __restrict__ a, const float* __restrict__ b, int n,
                                                     float* __restrict__ out)
{
    __shared__ float sa[256], sb[256];
    const int samples = n < 16384 ? n : 16384;
    float xa = 0.f, xb = 0.f;
    for (int i = threadIdx.x; i < samples; i += 256) {
        const long long at = (long long)i * n / samples;
        xa += a[at]; xb += b[at];
    }
    sa[threadIdx.x] = xa; sb[threadIdx.x] = xb;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) { sa[threadIdx.x] += sa[threadIdx.x + w]; sb[threadIdx.x] += sb[threadIdx.x + w]; }
        __syncthreads();
    }
    if (threadIdx.x == 0) { out[0] = sa[0]; out[1] = sb[0]; }
}

// Pinned host memory, kept between calls: taking it from the runtime and giving it back costs tens of microseconds a
// piece and milliseconds for the staging of a million rows.  At most POOL_LIMIT bytes lie idle; what does not fit goes
// back to the runtime at once, and the rest when the process ends.  Any thread may take and give blocks.
class PinnedPool {
public:
    struct Block { void* p; size_t bytes; };
    hipError_t take(size_t bytes, Block* out)
    {
        size_t want = 4096;
        while (want < bytes && want < ((size_t)1 << 20)) want *= 2;
        if (want < bytes) want = (bytes + ((size_t)1 << 20) - 1) >> 20 << 20;
        {
            std::lock_guard<std::mutex> lock(m_);
            size_t best = idle_.size();
            for (size_t i = 0; i < idle_.size(); ++i)
                if (idle_[i].bytes >= want && idle_[i].bytes <= 4 * want && (best == idle_.size() || idle_[i].bytes < idle_[best].bytes)) best = i;
            if (best < idle_.size()) {
                *out = idle_[best];
                idle_bytes_ -= out->bytes;
                idle_[best] = idle_.back();
                idle_.pop_back();
                return hipSuccess;
            }
        }
        void* p = nullptr;
        const hipError_t e = hipHostMalloc(&p, want, hipHostMallocPortable | hipHostMallocMapped | hipHostMallocCoherent);
        if (e != hipSuccess) return e;
        *out = Block{p, want};
        return hipSuccess;
    }
    void give(Block b)
    {
        {
            std::lock_guard<std::mutex> lock(m_);
            if (idle_bytes_ + b.bytes <= POOL_LIMIT && idle_.size() < 64) {
                try {
                    idle_.push_back(b);
                    idle_bytes_ += b.bytes;
                    return;
                } catch (...) { }
            }
        }
        (void)hipHostFree(b.p);
    }
private:
    static constexpr size_t POOL_LIMIT = (size_t)256 << 20;
    std::mutex m_;
    std::vector<Block> idle_;
    size_t idle_bytes_ = 0;
};
PinnedPool& pinned_pool() { static PinnedPool* pool = new PinnedPool; return *pool; }       // (never destroyed: the runtime may be gone first)

// A block of the pool for the duration of a call.  The stream's work on it must be over when it is given back:
// idle() says that it is; otherwise (an early return) the destructor waits for the stream.
struct PinnedHost {
    void* p = nullptr;
    PinnedPool::Block b{nullptr, 0};
    hipStream_t s;
    bool busy = true;
    explicit PinnedHost(hipStream_t stream) : s(stream) {}
    PinnedHost(const PinnedHost&) = delete;
    PinnedHost& operator=(const PinnedHost&) = delete;
    hipError_t alloc(size_t bytes)
    {
        const hipError_t e = pinned_pool().take(bytes, &b);
        if (e == hipSuccess) p = b.p;
        return e;
    }
    void idle() { busy = false; }
    ~PinnedHost()
    {
        if (!p) return;
        if (busy) (void)hipStreamSynchronize(s);
        pinned_pool().give(b);
    }
};

// words of device memory to host memory, then `seq` to host[0] (one workgroup)
__global__ void __launch_bounds__(256) k_fetch_words(const uint32_t* __restrict__ src, int n, uint32_t* __restrict__ host, uint32_t seq)
{
    for (int i = threadIdx.x; i < n; i += 256) __hip_atomic_store(host + 1 + i, src[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    __threadfence_system();
    __syncthreads();
    if (threadIdx.x == 0) __hip_atomic_store(host, seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// A few words from the device without a copy and a synchronisation (20 us): a kernel behind the work writes them to host
// memory, and the host watches for a sequence number there.  Either the words with the number last, in a word before them, or
// 64-bit words with the number in the high half of each.  Each of the two has memory of its own: the number of one would be looked for
// where the other keeps words of any value.
struct Mailbox {
    PinnedHost box;
    hipStream_t s;
    uint32_t seq = 0;
    static constexpr int WORDS = 4096, TAGGED = 8;
    static constexpr size_t BYTES = TAGGED * sizeof(unsigned long long) + (WORDS + 16) * sizeof(uint32_t);
    explicit Mailbox(hipStream_t stream) : box(stream), s(stream) {}
    hipError_t open()
    {
        const hipError_t e = box.alloc(BYTES);
        if (e != hipSuccess) return e;
        for (int i = 0; i < TAGGED; ++i) static_cast<volatile unsigned long long*>(tagged())[i] = 0ull;         // (another user's sequence numbers)
        for (int i = 0; i < 16; ++i) static_cast<volatile uint32_t*>(words())[i] = 0u;
        return hipSuccess;
    }
    unsigned long long* tagged() { return static_cast<unsigned long long*>(box.p); }
    uint32_t* words() { return reinterpret_cast<uint32_t*>(tagged() + TAGGED); }
    uint32_t next() { return ++seq; }
    // whether the sequence number last handed out has arrived
    bool arrived() { return __atomic_load_n(words(), __ATOMIC_ACQUIRE) == seq; }
    // ... in the first n tagged words
    bool arrived_tagged(int n)
    {
        for (int i = 0; i < n; ++i)
            if ((uint32_t)(__atomic_load_n(tagged() + i, __ATOMIC_ACQUIRE) >> 32) != seq) return false;
        return true;
    }
    hipError_t wait() { return until([&] { return arrived(); }); }
    hipError_t wait_tagged(int n) { return until([&] { return arrived_tagged(n); }); }
    template <typename F>
    hipError_t until(F&& there)
    {
        for (unsigned spins = 0;; ++spins) {
            if (there()) return hipSuccess;
#if defined(__x86_64__)
            __builtin_ia32_pause();
#endif
            if ((spins & 4095u) == 4095u) {
                // an error ends the wait; so does a stream that has run dry without the number
                const hipError_t q = hipStreamQuery(s);
                if (q == hipErrorNotReady) continue;
                if (there()) return hipSuccess;
                if (q != hipSuccess) return q;
                const hipError_t w = hipStreamSynchronize(s);
                if (there()) return hipSuccess;
                return w != hipSuccess ? w : hipErrorUnknown;
            }
        }
    }
    // n words at `src` (device), as of everything enqueued so far, to out
    hipError_t fetch(const void* src, int n, void* out)
    {
        if (n < 1 || n > WORDS) return hipErrorInvalidValue;
        hipLaunchKernelGGL(k_fetch_words, dim3(1), dim3(256), 0, s, static_cast<const uint32_t*>(src), n, words(), next());
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        e = wait();
        if (e != hipSuccess) return e;
        std::memcpy(out, words() + 1, (size_t)n * 4);
        return hipSuccess;
    }
};

// A pair of HIP events bracketing work on a stream.
struct EventPair {
    hipEvent_t a = nullptr, b = nullptr;
    hipError_t create() { hipError_t e = hipEventCreate(&a); return e != hipSuccess ? e : hipEventCreate(&b); }
    ~EventPair() { if (a) (void)hipEventDestroy(a); if (b) (void)hipEventDestroy(b); }
    float ms() const { float t = 0.f; return a && b && hipEventElapsedTime(&t, a, b) == hipSuccess ? t : -1.f; }
};

double now_ms()
{
    using clk = std::chrono::steady_clock;
    return std::chrono::duration<double, std::milli>(clk::now().time_since_epoch()).count();
}

// SLHC_LOG=1 in the environment: phase times and per-round counters on stderr (each mark waits for
// the stream, so the logged run is slower than a normal one).
struct PhaseLog {
    bool on;
    hipStream_t s;
    double t;
    explicit PhaseLog(hipStream_t stream) : s(stream), t(0.0)
    {
        const char* e = std::getenv("SLHC_LOG");
        on = e && e[0] && e[0] != '0';
        if (on) t = now_ms();
    }
    void mark(const char* fmt, ...)
    {
        if (!on) return;
        (void)hipStreamSynchronize(s);
        const double now = now_ms();
        char text[256];
        va_list ap;
        va_start(ap, fmt);
        vsnprintf(text, sizeof(text), fmt, ap);
        va_end(ap);
        std::fprintf(stderr, "[slhc] %8.2f ms  %s\n", now - t, text);
        t = now_ms();
    }
};

// Tile pruning is implemented by the register-resident-query sweep only (d <= 128, d % 4 == 0), and
// pays off only when there are enough rows to form several tiles per cluster.
#ifndef SLHC_PRUNE_MIN_ROWS
#define SLHC_PRUNE_MIN_ROWS 512      // compile-time knob so that small harnesses can exercise the reordered path
#endif
constexpr int64_t PRUNE_MIN_ROWS = SLHC_PRUNE_MIN_ROWS;
// two-phase pruned connection sweeps (see run_slhc): rows, tile steps per panel of the round before
#ifndef SLHC_TWO_PHASE_MIN_ROWS
#define SLHC_TWO_PHASE_MIN_ROWS 262144
#endif
constexpr int64_t TWO_PHASE_MIN_ROWS = SLHC_TWO_PHASE_MIN_ROWS;
#ifndef SLHC_TWO_PHASE_MIN_STEPS
#define SLHC_TWO_PHASE_MIN_STEPS 128.0
#endif
constexpr double TWO_PHASE_MIN_STEPS = SLHC_TWO_PHASE_MIN_STEPS;
constexpr int TWO_PHASE_STRIDE = 16;
// pruned connection sweeps lower a component's shared threshold to this multiple of the lightest edge its
// queries have found so far (squared distance; see SweepParams::comp_lower_factor)
#ifndef SLHC_LOWER_FACTOR
#define SLHC_LOWER_FACTOR 1.0f
#endif
constexpr float LOWER_FACTOR = SLHC_LOWER_FACTOR;
#ifndef SLHC_LOWER_MIN_ROWS
#define SLHC_LOWER_MIN_ROWS 4096
#endif
constexpr int LOWER_MIN_ROWS = SLHC_LOWER_MIN_ROWS;
// ... and components of any size where there are this many rows in all: a row that the falling threshold cuts off costs no evaluation,
// and the row it has met last still bounds its component in the next round.  Large components only / all, in us: 300k x 32 in
// clusters of 100 21 100 and 16 600, 500k x 16 in tight ones of 250 12 400 and 10 300, 150k x 8 8800 and 7400, 2M x 32 in tight
// ones of 100 44 000 and 41 000, 1M x 16 in a thousand zipf ones the same; 60k x 20 and 20k x 64 the same, where which rows are asked
// again then stays the same in every run.
constexpr int64_t LOWER_ALL_ROWS = 131072;
constexpr int NESTED_K = 8;
// pruned connection sweeps: a launch with fewer non-empty panels than this splits every panel's scan into parts
// so that about this many work items result, at most SPLIT_MAX_PARTS per panel
#ifndef SLHC_SPLIT_ITEMS_TARGET
#define SLHC_SPLIT_ITEMS_TARGET 32768
#endif
constexpr int SPLIT_ITEMS_TARGET = SLHC_SPLIT_ITEMS_TARGET;
constexpr int SPLIT_MAX_PARTS = 16;
// ... and only as far as a part still has about this many tiles to multiply, going by the steps per panel of the
// sweep before
#ifndef SLHC_SPLIT_MIN_STEPS
#define SLHC_SPLIT_MIN_STEPS 8.0
#endif
constexpr double SPLIT_MIN_STEPS = SLHC_SPLIT_MIN_STEPS;
// up to this many tiles of the reordered copy the lower bounds between all pairs of tiles are tabulated once
// (T x T floats: 4 GiB at the limit) instead of being computed for every query panel of every pruned sweep
#ifndef SLHC_TILE_GAP_MAX_TILES
#define SLHC_TILE_GAP_MAX_TILES 32768
#endif
constexpr int TILE_GAP_MAX_TILES = SLHC_TILE_GAP_MAX_TILES;
// The dendrogram from this many rows on is made on the device (dendrogram_kernels.hip), below on the host, whose pass over so few rows
// stays in its caches.  Sort and dendrogram, three kinds of data, host / device: 12 000 rows 130 / 172 us, 16 000 152 / 165, 18 000 177 / 188,
// 20 000 215 / 190, 24 000 255 / 190.
constexpr int64_t DENDROGRAM_DEVICE_MIN_ROWS = 19000;
bool prunable(int64_t N, int32_t d) { return d % 4 == 0 && d <= 128 && N >= PRUNE_MIN_ROWS; }
#ifndef SLHC_PIVOT_STRIDE
#define SLHC_PIVOT_STRIDE 64
#endif
int first_level_pivots(int64_t N) { return (int)((N + SLHC_PIVOT_STRIDE - 1) / SLHC_PIVOT_STRIDE); }
// The reordered copy inserts padding rows so that well separated clusters start on a tile
// boundary; padding is limited to N/2 rows.
int64_t padded_rows_limit(int64_t N) { return N + N / 2 + 256; }

constexpr size_t NO_LIMIT = ~(size_t)0;      // of a workspace
// (with_near = false: without the half-precision engine)
size_t slhc_ws_bytes(int64_t N, int32_t d, int32_t k, bool with_order, bool with_near);

// tile products from split bfloat16 halves: whole chunks of 32 columns up to 128 features (the
// register-resident-query kernel); beyond 128 features the streaming kernel takes any multiple of 4 columns,
// its split copy padded to whole chunks
bool split_products_ok(int32_t d) { return (d % 32 == 0 && d >= 32 && d <= 128) || (d > 128 && d % 4 == 0); }
// ... in the pruned sweeps from two chunks on only: at 32 features a tile's multiplies are too short for the
// wider filter to pay (2M x 32: pruned connection sweeps 30 ms with float32 products, 60 ms with split ones)
bool split_products_pruned_ok(int32_t d) { return d % 32 == 0 && d >= 64 && d <= 128; }

// Scratch of the half-precision engine (near_kernels.hip): the float16 copy of the candidates, that of separate
// queries (nq > 0), and the buffers of its passes.
struct NearWs {
    slhc::NearCopy c{}, q{};
    slhc::NearBuffers b{};
    bool ok = false;
    // `most`: where the workspace ends; the batch takes what is left of it, and where that is too little there is no engine
    // and nothing of it in the layout (ok stays false)
    // `ordered`: rows of a padded row order that is searched too (0: none)
    // `lent`: memory for the copy of the queries that the layout has anyway; `spare`: for the lists of all rows
    void carve(Carver& w, int64_t nc, int64_t nq, int32_t d, int32_t kk, bool coloured, size_t most = NO_LIMIT, int64_t ordered = 0,
               const slhc::NearCopy* lent = nullptr, unsigned char* spare = nullptr, size_t spare_bytes = 0)
    {
        const size_t begin = w.off;
        auto copy = [&](slhc::NearCopy& x, int64_t n, bool queries) {
            x.rows = (int)n; x.tiles = slhc::near_tiles(n);
            x.frag = w.take<unsigned char>(slhc::near_frag_bytes(n, d));
            x.negh = w.take<float>((size_t)x.tiles * 128);
            x.negh_best = kk == 1 || coloured ? w.take<float>((size_t)x.tiles * 128) : nullptr;
            x.colour = coloured ? w.take<int32_t>((size_t)x.tiles * 128) : nullptr;
            x.left = nullptr; x.count = nullptr; x.best_at = nullptr;
            if (!queries) return;
            x.left = w.take<int32_t>((size_t)x.tiles * 128 * (kk == 1 ? 4 : 1));      // (one part serves k-NN searches as scratch)
            x.count = w.take<int32_t>((size_t)x.tiles * 128);
            if (coloured) x.best_at = w.take<unsigned long long>((size_t)x.tiles * 128);
        };
        b.scale = w.take<slhc::NearScale>(1);
        b.shift = w.take<float>((size_t)d + 8);
        b.partial = w.take<float>(slhc::near_stats_scratch_floats(d));
        copy(c, nc, false);
        if (lent) {
            q = *lent;
            q.rows = (int)nq; q.tiles = slhc::near_tiles(nq);
            q.left = w.take<int32_t>((size_t)q.tiles * 128);
            q.count = w.take<int32_t>((size_t)q.tiles * 128);
        } else if (nq > 0) copy(q, nq, true);
        else q = c;                                         // (k-NN: no scratch per query)
        const int64_t queries = nq > 0 ? nq : nc;
        b.todo_panels = (std::max(queries, ordered) + 127) / 128;
        b.todo = w.take<int32_t>((size_t)(2 + 2 * b.todo_panels));
        b.todo_mark = b.todo + 2 + b.todo_panels;
        b.batch_bytes = slhc::near_batch_bytes(queries, nc, d, kk);
        size_t least = slhc::near_least_batch_bytes(queries, nc, d, kk);
        if (ordered) {
            b.batch_bytes = std::max({b.batch_bytes, slhc::near_ordered_batch_bytes(ordered, kk), slhc::near_linked_batch_bytes(ordered)});
            least = std::max({least, slhc::near_least_ordered_batch_bytes(ordered, kk), slhc::near_linked_batch_bytes(ordered)});
        }
        // The lists of a search that multiplies every pair once: in the batch's memory, in the spare one, or, where neither holds
        // them, in a batch that may grow to the size of the rows for it.
        const size_t pairs = slhc::near_pairs_bytes(nc, d, kk);
        if (pairs > b.batch_bytes && pairs > spare_bytes && pairs <= (size_t)nc * (size_t)d * sizeof(float)) b.batch_bytes = up(pairs);
        const size_t room = most > w.off ? (most - w.off) / ALIGN * ALIGN : 0;
        if (b.batch_bytes > room) b.batch_bytes = room;
        if (b.batch_bytes < least) {
            *this = NearWs{};
            w.off = begin;
            return;
        }
        b.batch = w.take<unsigned char>(b.batch_bytes);
        b.pairs = b.batch; b.pairs_bytes = b.batch_bytes;
        if (pairs > b.batch_bytes) { b.pairs = spare; b.pairs_bytes = spare_bytes; }
        ok = true;
    }
};

// Buffers of the spatially coherent row order (see build_order).
struct OrderWs {
    float *Xp, *hp, *pdist, *sample, *Xs, *hs, *tile_c, *tile_r, *gap_ws, *tile_gap, *n_w;
    float *Xs_split, *hs_split;      // the reordered copy in split bfloat16 halves and its half norms (nullptr: d does not allow it)
    // a second split copy, every tile relative to the centre of the first tile of its region, with its half norms;
    // region number, first tile and boundary flag per tile (see run_knn; nullptr: the pruned sweeps keep float32 products)
    float *Xs_local, *hs_local, *region_other_min;
    int32_t *tile_region, *tile_first, *tile_last, *tile_boundary, *tile_local;
    int32_t *pid, *perm, *inv, *colour_s, *qslot, *tile_colour, *tile_list, *counts, *rank, *shift, *far_count;
    int32_t *n_src, *n_dst;
    uint32_t *tmp_a, *tmp_b, *tmp_c;
    slhc::NearCopy near_all{}, near_local{};      // float16 copies of the rows in this order (see NearOrder)
    slhc::NearScale* local_scale;
    slhc::NearCopy near_p{};          // that of the pivots, and scratch of the assignment
    unsigned long long* best_at;
    int32_t* near_colour;
    bool near_searched;               // near_all, near_local, near_colour and local_scale exist
    void* sort_temp; size_t sort_temp_bytes;
    void* nested_ws; size_t nested_bytes;      // of the clustering of the pivots, which keeps within it
    unsigned char* spare; size_t spare_bytes;  // what a call that makes no order may use
    int P1, Pmax, Tmax;
    int64_t Nmax;
    int P = 0;        // pivots in use          (set by build_order)
    int Ns = 0;       // rows of the padded copy (set by build_order)
    static constexpr int SAMPLE = 4096;
    void carve(Carver& c, int64_t N, int32_t d, bool with_near)
    {
        const size_t n = (size_t)N;
        P1 = first_level_pivots(N);
        Pmax = 4 * P1;            // budget for pivots added for clusters the first level missed
        Nmax = padded_rows_limit(N);
        Tmax = (int)((Nmax + 127) / 128);
        const size_t nm = (size_t)Nmax, pm = (size_t)Pmax;
        Xp = c.take<float>(pm * d); hp = c.take<float>(pm);
        pdist = c.take<float>(n); sample = c.take<float>(SAMPLE);
        // The copies in the row order are made when the pivots' clustering is over, whose workspace takes the same place.
        const size_t copies_begin = c.off;
        Xs = c.take<float>(nm * d); hs = c.take<float>(nm);
        Xs_split = nullptr; hs_split = nullptr;
        if (split_products_ok(d)) { Xs_split = c.take<float>(nm * d); hs_split = c.take<float>(nm); }
        Xs_local = nullptr; hs_local = nullptr; region_other_min = nullptr;
        if (split_products_ok(d) && d <= 128) { Xs_local = c.take<float>(nm * d); hs_local = c.take<float>(nm); }
        // searches of the half-precision engine in this order need the table of tile pairs
        near_searched = with_near && Tmax <= TILE_GAP_MAX_TILES;
        if (near_searched) {
            for (slhc::NearCopy* x : {&near_all, &near_local}) {
                x->in_order = true;
                x->frag = c.take<unsigned char>(slhc::near_frag_bytes(Nmax, d));
                x->negh = c.take<float>((size_t)Tmax * 128); x->negh_best = c.take<float>((size_t)Tmax * 128);
            }
            near_colour = c.take<int32_t>((size_t)Tmax * 128);
            local_scale = c.take<slhc::NearScale>(1);
        }
        int grid = slhc::sweep_grid_limit();
        if (grid < 1) grid = 512;
        {
            const int32_t kp = Pmax - 1 < NESTED_K ? Pmax - 1 : NESTED_K;
            // (the clustering runs on the pivots in use, fewer than Pmax: a k-NN sweep of few panels then also wants
            // its scratch for candidate ranges, which the layout for Pmax rows may not contain)
            nested_bytes = slhc_ws_bytes(Pmax, d, kp, false, with_near) + (size_t)grid * 128 * (size_t)kp * 8 + 1024;
            nested_ws = c.base ? c.base + copies_begin : nullptr;
            if (c.off < copies_begin + up(nested_bytes)) c.off = copies_begin + up(nested_bytes);
        }
        tile_region = c.take<int32_t>((size_t)Tmax); tile_first = c.take<int32_t>((size_t)Tmax);
        tile_last = c.take<int32_t>((size_t)Tmax);
        tile_boundary = c.take<int32_t>((size_t)Tmax); tile_local = c.take<int32_t>((size_t)Tmax);
        if (split_products_ok(d) && d <= 128) region_other_min = c.take<float>((size_t)Tmax);
        tile_c = c.take<float>((size_t)Tmax * d); tile_r = c.take<float>((size_t)Tmax);
        gap_ws = c.take<float>((size_t)grid * Tmax);
        // lower bounds between all pairs of tiles (order_tile_gaps), as long as the table stays moderate
        tile_gap = Tmax <= TILE_GAP_MAX_TILES ? c.take<float>((size_t)Tmax * Tmax) : nullptr;
        pid = c.take<int32_t>(n); perm = c.take<int32_t>(nm); inv = c.take<int32_t>(n); colour_s = c.take<int32_t>(nm);
        qslot = c.take<int32_t>(nm); tile_colour = c.take<int32_t>((size_t)Tmax); tile_list = c.take<int32_t>((size_t)Tmax);
        counts = c.take<int32_t>(pm); rank = c.take<int32_t>(pm); shift = c.take<int32_t>(pm); far_count = c.take<int32_t>(64);
        if (with_near) {
            near_p.tiles = slhc::near_tiles(Pmax);
            near_p.frag = c.take<unsigned char>(slhc::near_frag_bytes(Pmax, d));
            near_p.negh = c.take<float>((size_t)near_p.tiles * 128); near_p.negh_best = c.take<float>((size_t)near_p.tiles * 128);
            best_at = c.take<unsigned long long>((size_t)slhc::near_tiles(N) * 128);
        }
        tmp_a = c.take<uint32_t>(n); tmp_b = c.take<uint32_t>(n); tmp_c = c.take<uint32_t>(n);
        sort_temp_bytes = slhc::pair_sort_temp_bytes((int)N);
        sort_temp = c.take<unsigned char>(sort_temp_bytes);
        n_src = c.take<int32_t>(pm); n_dst = c.take<int32_t>(pm); n_w = c.take<float>(pm);
        spare = c.base ? c.base + copies_begin : nullptr;
        spare_bytes = c.off - copies_begin;
    }
    // Memory of a copy of listed rows: that of the copy in this order, which is made later and no longer used when the
    // connection rounds come to make one.
    slhc::NearCopy lent_copy() const
    {
        slhc::NearCopy q{};
        q.frag = near_all.frag; q.negh = near_all.negh; q.negh_best = near_all.negh_best;
        q.colour = near_colour; q.best_at = best_at;
        return q;
    }
};

struct KnnWs {
    unsigned long long* counters;    // [0] k-NN survivors [1] connect survivors [2] k-NN tile steps [3] connect tile steps
                                     // [4] non-finite flag (low word) [8] panel hand-out counter (low word)
    float* hn;
    bool has_order;
    OrderWs order;
    // lists per candidate range of a k-NN sweep with few panels (see launch_knn_sweep); k = 0: none
    int32_t* part_idx; float* part_dist; long long part_rows;
    // every-tile sweeps on the bf16 MFMA: X split into bfloat16 halves (see SweepParams::Xq_split) and the half
    // norms with the slack that goes with it; nullptr when d does not allow it
    float* Xsplit; float* hn_split;
    // the split copies hold the rows relative to the column means of X (a sample's): shift [d], and the scratch of
    // the two-pass mean
    float* shift; float* shift_scratch;
    // scratch of the every-tile sweeps that go range by range (see SweepParams::carry_ws): 2 + panels words
    unsigned int* carry_ws; long long carry_ws_words;
    NearWs near;                     // every-tile sweeps in half precision
    bool near_done = false;          // ... made the lists of this call
    bool near_ready = false;         // the float16 copy of X is made
    bool near_order_ready = false;   // those of the row order are
    bool regions_ready = false;
    bool split_ready = false;        // filled in this call
    bool order_split_ready = false;  // likewise the split copy of the reordered rows
    bool offset_heavy = false;       // the rows' norms are mostly a common offset (see run_knn): split products everywhere
    bool order_split_connect = false;   // the pruned connection sweeps multiply the split copy of the reordered rows too
    size_t bytes;
    // `connect`: for connection rounds too.
    // `most`: bytes there are.  Too few for the half-precision engine: the layout without it (whose `bytes` may exceed them too).
    KnnWs(void* ws, int64_t N, int32_t d, bool with_order, int32_t k, bool connect, size_t most = NO_LIMIT)
    {
        lay_out(ws, N, d, with_order, k, connect, k > 0, most);
        if (k > 0 && !near.ok) lay_out(ws, N, d, with_order, k, connect, false, most);
    }
private:
    void lay_out(void* ws, int64_t N, int32_t d, bool with_order, int32_t k, bool connect, bool with_near, size_t most)
    {
        Carver c(ws);
        order = OrderWs();
        near = NearWs();
        counters = c.take<unsigned long long>(32);
        hn = c.take<float>((size_t)N);
        part_idx = nullptr; part_dist = nullptr; part_rows = 0;
        Xsplit = nullptr; hn_split = nullptr; shift = nullptr; shift_scratch = nullptr;
        if (split_products_ok(d) && k > 0) {
            Xsplit = c.take<float>((size_t)N * (size_t)slhc::split_row_stride(d));
            hn_split = c.take<float>((size_t)N);
            shift = c.take<float>((size_t)d);
            shift_scratch = c.take<float>(slhc::column_means_scratch_floats(d));
        }
        {
            // ranges x rows never exceeds the workgroup slots x 128: a sweep is only split while its panels
            // fill less than half the slots
            int grid = slhc::sweep_grid_limit();
            if (grid < 1) grid = 512;
            if (k > 1 && ((N + 127) / 128) * 2 <= grid) {
                part_rows = (long long)grid * 128;
                part_idx = c.take<int32_t>((size_t)part_rows * k);
                part_dist = c.take<float>((size_t)part_rows * k);
            }
        }
        carry_ws_words = 2 + (long long)((N + 127) / 128);
        carry_ws = c.take<unsigned int>((size_t)carry_ws_words);
        has_order = with_order && prunable(N, d);
        if (has_order) order.carve(c, N, d, with_near);
        // (the queries' copy serves the making of the row order and, as the colours, the every-tile connection sweeps)
        if (with_near) {
            const bool searched = has_order && order.near_searched;
            const slhc::NearCopy lent = searched ? order.lent_copy() : slhc::NearCopy{};
            near.carve(c, N, connect || has_order ? N : 0, d, k + 1, connect, most, searched ? order.Nmax : 0, searched ? &lent : nullptr,
                       has_order ? order.spare : nullptr, has_order ? order.spare_bytes : 0);
        }
        bytes = c.off;
    }
};

struct SlhcWs {
    int32_t* nbr_idx; float* nbr_dist;
    int32_t *colour, *ptr, *ext_idx, *cand_u, *hook, *qlist, *q_idx, *counters, *e_lo, *e_hi;
    float *ext_dist, *ext_low, *cand_w, *q_dist, *q_low, *e_w;
    uint32_t *best_w, *vals_a, *vals_b;
    unsigned long long *best_e, *keys_a, *keys_b;
    void* sort_temp; size_t sort_temp_bytes;
    std::optional<KnnWs> knn;        // half norms and row order are reused by the connection sweeps
    size_t bytes;
    SlhcWs(void* ws, int64_t N, int32_t d, int32_t k, bool with_order, size_t most = NO_LIMIT)
    {
        Carver c(ws);
        const size_t n = (size_t)N;
        nbr_idx = c.take<int32_t>(n * k);
        nbr_dist = c.take<float>(n * k);
        colour = c.take<int32_t>(n); ptr = c.take<int32_t>(n); ext_idx = c.take<int32_t>(n);
        cand_u = c.take<int32_t>(n); hook = c.take<int32_t>(n); qlist = c.take<int32_t>(n);
        q_idx = c.take<int32_t>(n); counters = c.take<int32_t>(64);
        e_lo = c.take<int32_t>(n); e_hi = c.take<int32_t>(n);
        ext_dist = c.take<float>(n); ext_low = c.take<float>(n); cand_w = c.take<float>(n); q_dist = c.take<float>(n); e_w = c.take<float>(n);
        best_w = c.take<uint32_t>(n);
        vals_a = c.take<uint32_t>(n); vals_b = c.take<uint32_t>(n);
        best_e = c.take<unsigned long long>(n); keys_a = c.take<unsigned long long>(n); keys_b = c.take<unsigned long long>(n);
        sort_temp_bytes = std::max(slhc::edge_sort_temp_bytes((int)(N - 1)), slhc::pair_sort_temp_bytes((int)N));   // the second: the dendrogram's chains
        sort_temp = c.take<unsigned char>(sort_temp_bytes);
        // the k-NN part takes what is left, without the engine's lower ends of the queries' answers
        const size_t low = up(n * sizeof(float));
        knn.emplace(c.base ? c.base + c.off : nullptr, N, d, with_order, k, true, most == NO_LIMIT ? most : most > c.off + low ? most - c.off - low : 0);
        c.off += knn->bytes;
        q_low = knn->near.ok ? c.take<float>(n) : nullptr;
        bytes = c.off;
    }
};

size_t slhc_ws_bytes(int64_t N, int32_t d, int32_t k, bool with_order, bool with_near) { return SlhcWs(nullptr, N, d, k, with_order, with_near ? NO_LIMIT : 0).bytes; }

int run_slhc(const float* X, int64_t N, int32_t d, int32_t k, int32_t* mst_src, int32_t* mst_dst, float* mst_w,
             int32_t* children, float* heights, int32_t* sizes, slhc_stats* stats, void* workspace, size_t workspace_bytes,
             hipStream_t s, uint32_t flags, bool with_order, const float* X_given, int32_t d_given);

int bits_for(long long n) { int b = 1; while (b < 32 && (1LL << b) < n) ++b; return b; }

// X in split bfloat16 halves, taken relative to the column means of a sample of its rows (a translation changes no
// distance and keeps a common offset of the data out of the filter's slack), with the half norms that go with it.
int make_split_copy(const float* X, int64_t N, int32_t d, KnnWs& ws, hipStream_t s)
{
    HIP_TRY(slhc::launch_column_means(X, (int)N, d, ws.shift_scratch, ws.shift, s));
    HIP_TRY(slhc::launch_split_bf16(X, (int)N, d, ws.Xsplit, s, ws.shift));
    HIP_TRY(slhc::launch_half_norms(X, (int)N, d, ws.hn_split, s, nullptr, true, ws.shift));
    ws.split_ready = true;
    return SLHC_OK;
}

// Nearest pivot of every row by the fused sweep (k = 1 against the P pivot rows).
// `x_split` / `hn_split` / `shift` (optional): X in split bfloat16 halves, the half norms that go with it and the
// shift both were taken relative to; the pivots
// then get a split copy of their own (in the buffers of the reordered copy's, which are free until step 4).
// `near` (optional): the half-precision engine with the copy of X made; the nearest pivot is then one up to the rounding
// of the copies, which is all the order needs, in one pass.
slhc::NearCopy pivot_copy(const OrderWs& o, int P)
{
    slhc::NearCopy c = o.near_p;
    c.rows = P; c.tiles = slhc::near_tiles(P);
    c.finite_padding = true;
    return c;
}
int assign_to_pivots(const float* X, int64_t N, int32_t d, const float* hn, OrderWs& o, int P, hipStream_t s,
                     const NearWs* near, const float* x_split = nullptr, const float* hn_split = nullptr, const float* shift = nullptr)
{
    if (near) {
        const slhc::NearCopy c = pivot_copy(o, P);
        HIP_TRY(slhc::near_make(o.Xp, P, d, nullptr, P, nullptr, near->b, c, nullptr, nullptr, s));
        HIP_TRY(slhc::near_assign(near->c, c, X, nullptr, o.Xp, d, near->b, o.best_at, o.pid, o.pdist, s));
        return SLHC_OK;
    }
    slhc::SweepParams p{};
    p.Xq = X; p.hq = hn; p.NQ = (int)N;
    p.Xc = o.Xp; p.hc = o.hp; p.NC = P;
    p.d = d; p.k = 1;
    p.out_idx = o.pid; p.out_dist = o.pdist;
    if (x_split && hn_split && o.Xs_split && o.hs_split) {
        HIP_TRY(slhc::launch_split_bf16(o.Xp, P, d, o.Xs_split, s, shift));
        HIP_TRY(slhc::launch_half_norms(o.Xp, P, d, o.hs_split, s, nullptr, true, shift));
        p.Xq_split = x_split; p.hq_split = hn_split;
        p.Xc_split = o.Xs_split; p.hc_split = o.hs_split;
    }
    HIP_TRY(slhc::launch_knn_sweep(p, s));
    return SLHC_OK;
}

// Spatially coherent order of the rows (not in the paper, whose sweeps multiply every tile).
//   1. Every 64th row is a pivot; each row is assigned to its nearest pivot by the fused 1-NN sweep.
//      Rows much farther from their pivot than the typical row belong to clusters that received no
//      pivot; a sample of those rows becomes a second set of pivots and the assignment is repeated.
//   2. The pivots are clustered by this library's own single-linkage path (without reordering); the
//      leaf order of their dendrogram puts pivots of one cluster next to each other at every scale.
//   3. Rows are sorted by the position of their pivot in that order.  Where consecutive pivots are
//      joined only far above the typical cell scale, the next row starts a new tile of 128 (padding
//      rows: perm = -1, zero features, +inf half norm), so tiles do not straddle distant clusters.
//   4. One bounding ball per tile of the reordered copy.
// The order only affects which tiles the sweeps can skip, never a result.
// `nonfinite`: device word the norm kernel set when a row is not finite; checked first, because
// nothing below is defined for such rows.
int build_order(const float* X, int64_t N, int32_t d, const float* hn, const unsigned int* nonfinite, OrderWs& o,
                hipStream_t s, const NearWs* near, const float* x_split = nullptr, const float* hn_split = nullptr, const float* shift = nullptr)
{
    const int n = (int)N;
    const int P1 = o.P1;
    PhaseLog log(s);
    Mailbox mail(s);
    HIP_TRY(mail.open());
    PinnedHost pin(s);
    HIP_TRY(pin.alloc(((size_t)OrderWs::SAMPLE + 16 + 6 * (size_t)o.Pmax) * 4));
    float* h_sample = static_cast<float*>(pin.p);
    int32_t* h_count = reinterpret_cast<int32_t*>(h_sample + OrderWs::SAMPLE);
    int32_t* h_src = h_count + 16;
    int32_t* h_dst = h_src + o.Pmax;
    float* h_w = reinterpret_cast<float*>(h_dst + o.Pmax);
    int32_t* h_cells = reinterpret_cast<int32_t*>(h_w + o.Pmax);
    int32_t* h_rank = h_cells + o.Pmax;
    int32_t* h_shift = h_rank + o.Pmax;

    HIP_TRY(mail.fetch(nonfinite, 1, h_count + 8));
    if (h_count[8] != 0) { set_err("a row of X is not finite (NaN, infinity, or a squared norm beyond float32)"); return SLHC_NONFINITE; }

    // ---- 1. pivots and assignment
    HIP_TRY(slhc::order_pick_rows(X, hn, n, d, P1, o.Xp, o.hp, s));
    int rc = assign_to_pivots(X, N, d, hn, o, P1, s, near, x_split, hn_split, shift);
    if (rc != SLHC_OK) return rc;
    const int S = n < OrderWs::SAMPLE ? n : OrderWs::SAMPLE;
    HIP_TRY(slhc::order_pick_f32(o.pdist, n, S, o.sample, s));
    HIP_TRY(mail.fetch(o.sample, S, h_sample));
    log.mark("row order: %d pivots, nearest pivot of every row", P1);
    // Scale of a well-placed cell: 4 x the median positive squared distance to the pivot.  (When the
    // clusters are much smaller than the pivot spacing the median is an inter-cluster distance and no
    // row counts as far; such data cannot be pruned at tile granularity anyway, and the connection
    // sweeps then fall back to multiplying every tile, see run_slhc.)
    float tau = __builtin_inff();
    {
        std::vector<float> v;
        for (int i = 0; i < S; ++i) if (h_sample[i] > 0.f && std::isfinite(h_sample[i])) v.push_back(h_sample[i]);
        if (!v.empty()) {
            std::nth_element(v.begin(), v.begin() + v.size() / 2, v.end());
            tau = 4.f * v[v.size() / 2];
        }
    }
    // Rows much farther from their pivot than the typical row: clusters without a pivot.  Every 16th
    // of them (in row order) becomes a pivot and the far rows alone are re-assigned among the new
    // pivots; repeated until no row is far, the pivot budget is used, or four rounds are done.
    int P = P1;
    for (int round = 0; round < 4 && std::isfinite(tau) && P < o.Pmax; ++round) {
        hipLaunchKernelGGL(k_zero_words, dim3(1), dim3(64), 0, s, reinterpret_cast<uint32_t*>(o.far_count), 64);
        HIP_TRY(hipGetLastError());
        HIP_TRY(slhc::order_mark_far(o.pdist, n, tau, o.tmp_a, o.far_count, s));
        HIP_TRY(mail.fetch(o.far_count, 1, h_count));
        const int far = h_count[0];
        if (far < 0 || far > n) { set_err("row order: bad far-row count %d", far); return SLHC_INTERNAL; }
        if (far == 0) break;
        // far rows first, in row order (stable 1-bit sort)
        uint32_t* far_rows = reinterpret_cast<uint32_t*>(o.perm);
        HIP_TRY(slhc::order_iota(reinterpret_cast<int32_t*>(o.tmp_b), n, s));
        HIP_TRY(slhc::pair_sort_u32(o.tmp_a, o.tmp_c, o.tmp_b, far_rows, n, 1, o.sort_temp, o.sort_temp_bytes, s));
        int P2 = (far + 15) / 16;
        if (P2 > o.Pmax - P) P2 = o.Pmax - P;
        HIP_TRY(slhc::order_pick_listed_rows(X, hn, far_rows, far, n, d, P2, o.Xp + (size_t)P * d, o.hp + P, s));
        if (near) {
            slhc::NearCopy q = near->q;
            q.rows = far; q.tiles = slhc::near_tiles(far); q.colour = nullptr;
            const slhc::NearCopy c = pivot_copy(o, P2);
            HIP_TRY(slhc::near_make(X, n, d, reinterpret_cast<const int32_t*>(far_rows), far, nullptr, near->b, q, nullptr, nullptr, s));
            HIP_TRY(slhc::near_make(o.Xp + (size_t)P * d, P2, d, nullptr, P2, nullptr, near->b, c, nullptr, nullptr, s));
            HIP_TRY(slhc::near_assign(q, c, X, reinterpret_cast<const int32_t*>(far_rows), o.Xp + (size_t)P * d, d, near->b, o.best_at, reinterpret_cast<int32_t*>(o.tmp_b), reinterpret_cast<float*>(o.tmp_c), s));
            HIP_TRY(slhc::order_adopt_pivots(far_rows, far, n, reinterpret_cast<const int32_t*>(o.tmp_b),
                                             reinterpret_cast<const float*>(o.tmp_c), P, P2, o.pid, o.pdist, s));
            P += P2;
            log.mark("row order: %d far rows -> %d more pivots", far, P2);
            continue;
        }
        // the far rows as a compact query matrix (the buffer of the reordered copy is still free)
        HIP_TRY(slhc::order_pick_listed_rows(X, hn, far_rows, far, n, d, far, o.Xs, o.hs, s));
        slhc::SweepParams p{};
        p.Xq = o.Xs; p.hq = o.hs; p.NQ = far;
        p.Xc = o.Xp + (size_t)P * d; p.hc = o.hp + P; p.NC = P2;
        p.d = d; p.k = 1;
        p.out_idx = reinterpret_cast<int32_t*>(o.tmp_b); p.out_dist = reinterpret_cast<float*>(o.tmp_c);
        HIP_TRY(slhc::launch_knn_sweep(p, s));
        HIP_TRY(slhc::order_adopt_pivots(far_rows, far, n, reinterpret_cast<const int32_t*>(o.tmp_b),
                                         reinterpret_cast<const float*>(o.tmp_c), P, P2, o.pid, o.pdist, s));
        P += P2;
        log.mark("row order: %d far rows -> %d more pivots", far, P2);
    }
    o.P = P;

    // ---- 2. hierarchy of the pivots: concatenating the two sides of every merge, in merge order,
    // yields a leaf order of the dendrogram; `joined[i]` is the height at which pivot i's successor
    // in that order was attached.
    std::vector<int32_t> order((size_t)P), head((size_t)P), tail((size_t)P), nxt((size_t)P, -1), up_set((size_t)P);
    std::vector<float> joined((size_t)P, 0.f);
    for (int i = 0; i < P; ++i) head[(size_t)i] = tail[(size_t)i] = up_set[(size_t)i] = i;
    if (P >= 2) {
        const int32_t kp = P - 1 < NESTED_K ? P - 1 : NESTED_K;
        rc = run_slhc(o.Xp, P, d, kp, o.n_src, o.n_dst, o.n_w, nullptr, nullptr, nullptr, nullptr,
                      o.nested_ws, o.nested_bytes, s, 0u, false, o.Xp, d);
        if (rc != SLHC_OK) return rc;
        const size_t E = (size_t)(P - 1);
        HIP_TRY(hipMemcpyAsync(h_src, o.n_src, E * 4, hipMemcpyDeviceToHost, s));
        HIP_TRY(hipMemcpyAsync(h_dst, o.n_dst, E * 4, hipMemcpyDeviceToHost, s));
        HIP_TRY(hipMemcpyAsync(h_w, o.n_w, E * 4, hipMemcpyDeviceToHost, s));
        HIP_TRY(hipStreamSynchronize(s));
        auto top = [&](int32_t a) {
            while (up_set[(size_t)a] != a) {
                up_set[(size_t)a] = up_set[(size_t)up_set[(size_t)a]];
                a = up_set[(size_t)a];
            }
            return a;
        };
        for (size_t e = 0; e < E; ++e) {
            if ((uint32_t)h_src[e] >= (uint32_t)P || (uint32_t)h_dst[e] >= (uint32_t)P) { set_err("row order: bad pivot edge"); return SLHC_INTERNAL; }
            const int32_t a = top(h_src[e]), b = top(h_dst[e]);
            if (a == b) { set_err("row order: pivot tree has a cycle"); return SLHC_INTERNAL; }
            nxt[(size_t)tail[(size_t)a]] = head[(size_t)b];
            joined[(size_t)tail[(size_t)a]] = h_w[e];
            tail[(size_t)a] = tail[(size_t)b];
            up_set[(size_t)b] = a;
        }
        int32_t at = head[(size_t)top(0)];
        for (int r = 0; r < P; ++r) {
            if (at < 0) { set_err("row order: pivot chain ends early"); return SLHC_INTERNAL; }
            order[(size_t)r] = at;
            at = nxt[(size_t)at];
        }
    } else {
        order[0] = 0;
    }
    for (int r = 0; r < P; ++r) h_rank[order[(size_t)r]] = r;
    log.mark("row order: single linkage of %d pivots, leaf order", P);

    // ---- 3. cell sizes and the padded layout
    HIP_TRY(slhc::order_fill_i32(o.counts, P, 0, s));
    HIP_TRY(slhc::order_histogram(o.pid, n, P, o.counts, s));
    HIP_TRY(hipMemcpyAsync(h_cells, o.counts, (size_t)P * 4, hipMemcpyDeviceToHost, s));
    HIP_TRY(hipStreamSynchronize(s));
    {
        long long total = 0;
        for (int i = 0; i < P; ++i) { if (h_cells[i] < 0) { total = -1; break; } total += h_cells[i]; }
        if (total != (long long)N) { set_err("row order: cells hold %lld of %lld rows", total, (long long)N); return SLHC_INTERNAL; }
    }
    const long long budget = (long long)(N / 2);
    float tau_pad = tau;
    long long Ns = 0;
    for (int attempt = 0; attempt < 200; ++attempt) {
        long long pos = 0, plain = 0;
        for (int r = 0; r < P; ++r) {
            const int pv = order[(size_t)r];
            h_shift[r] = (int32_t)(pos - plain);
            pos += h_cells[pv];
            plain += h_cells[pv];
            if (r + 1 < P && joined[(size_t)pv] > tau_pad) pos = (pos + 127) / 128 * 128;
        }
        Ns = pos;
        if (Ns - (long long)N <= budget) break;
        tau_pad = attempt < 190 ? tau_pad * 2.f : __builtin_inff();
    }
    if (Ns < (long long)N || Ns > (long long)o.Nmax) { set_err("row order: padded size %lld out of range", Ns); return SLHC_INTERNAL; }
    o.Ns = (int)Ns;

    // ---- 4. place the rows, gather the copy, bound the tiles
    HIP_TRY(hipMemcpyAsync(o.rank, h_rank, (size_t)P * 4, hipMemcpyHostToDevice, s));
    HIP_TRY(hipMemcpyAsync(o.shift, h_shift, (size_t)P * 4, hipMemcpyHostToDevice, s));
    uint32_t* keys = reinterpret_cast<uint32_t*>(o.colour_s);        // free until the connection rounds
    HIP_TRY(slhc::order_keys(o.pid, o.rank, n, P, keys, s));
    HIP_TRY(slhc::order_iota(reinterpret_cast<int32_t*>(o.tmp_a), n, s));
    HIP_TRY(slhc::pair_sort_u32(keys, o.tmp_b, o.tmp_a, o.tmp_c, n, bits_for(P), o.sort_temp, o.sort_temp_bytes, s));
    HIP_TRY(slhc::order_fill_i32(o.perm, o.Ns, -1, s));
    HIP_TRY(slhc::order_scatter(o.tmp_b, o.tmp_c, o.shift, n, P, o.Ns, o.perm, o.inv, s));
    HIP_TRY(slhc::order_gather_padded(X, hn, o.perm, o.Ns, n, d, o.Xs, o.hs, s));
    HIP_TRY(slhc::order_tile_balls(o.Xs, o.perm, o.Ns, d, o.tile_c, o.tile_r, s));
    if (o.tile_gap) HIP_TRY(slhc::order_tile_gaps(o.tile_c, o.tile_r, (o.Ns + 127) / 128, d, o.tile_gap, s));
    HIP_TRY(hipStreamSynchronize(s));        // the pinned staging buffer is given back on return
    pin.idle();
    mail.box.idle();
    log.mark("row order: %d rows placed in %d (tau %.4g, padding above %.4g), tile balls", n, o.Ns, (double)tau, (double)tau_pad);
    return SLHC_OK;
}

// The every-tile k-NN graph by the half-precision engine: any d, no padded copy, same lists as the list kernels.
bool near_wanted(const NearWs& near, uint32_t flags) { return near.ok && !(flags & (SLHC_FP32_FILTER | SLHC_PANEL_ORDER)); }
// (direct: what direct_knn_wanted says; counted: somebody reads the counters, `hn` and the float16 copy may be missing afterwards all the same, see
// ws.near_ready)
int run_knn_near(const float* X, int64_t N, int32_t d, int32_t k, int32_t* nbr_idx, float* nbr_dist, unsigned long long* counters,
                 float* hn, const NearWs& near, hipStream_t stream, int direct, bool counted, int32_t* evaluated = nullptr, EventPair* ev_norm = nullptr,
                 EventPair* ev_sweep = nullptr)
{
    if (direct > 0) {
        if (counted) {
            hipLaunchKernelGGL(k_zero_words, dim3(1), dim3(64), 0, stream, reinterpret_cast<uint32_t*>(counters), 64);
            HIP_TRY(hipGetLastError());
        }
        if (ev_norm) { HIP_TRY(hipEventRecord(ev_norm->a, stream)); HIP_TRY(hipEventRecord(ev_norm->b, stream)); }
        if (ev_sweep) HIP_TRY(hipEventRecord(ev_sweep->a, stream));
        HIP_TRY(slhc::direct_knn(X, (int)N, d, k, direct, nbr_idx, nbr_dist, counted ? counters : nullptr,
                                 counted ? reinterpret_cast<unsigned int*>(counters + 4) : nullptr, stream));
        if (ev_sweep) HIP_TRY(hipEventRecord(ev_sweep->b, stream));
        return SLHC_OK;
    }
    if (ev_norm) HIP_TRY(hipEventRecord(ev_norm->a, stream));
    HIP_TRY(slhc::near_stats(X, (int)N, d, near.b, reinterpret_cast<uint32_t*>(counters), 64, stream));
    HIP_TRY(slhc::near_make(X, (int)N, d, nullptr, (int)N, nullptr, near.b, near.c, hn, reinterpret_cast<unsigned int*>(counters + 4), stream));
    if (ev_norm) HIP_TRY(hipEventRecord(ev_norm->b, stream));
    if (ev_sweep) HIP_TRY(hipEventRecord(ev_sweep->a, stream));
    slhc::NearProblem a{};
    a.Xq = a.Xc = X; a.d = d; a.k = k;
    a.nq = a.nq_rows = a.nc = (int)N;
    a.exclude_self = 1;
    a.out_idx = nbr_idx; a.out_dist = nbr_dist;
    a.evaluated = evaluated;
    HIP_TRY(slhc::near_search(a, near.c, near.c, near.b, stream));
    slhc::SweepParams p{};                      // the panels it could not finish
    p.Xq = p.Xc = X; p.hq = p.hc = hn; p.NQ = p.NC = (int)N;
    p.d = d; p.k = k;
    p.out_idx = nbr_idx; p.out_dist = nbr_dist;
    p.exclude_self = 1;
    p.survivors = counters;
    p.todo = near.b.todo;
    HIP_TRY(slhc::launch_knn_sweep(p, stream));
    if (ev_sweep) HIP_TRY(hipEventRecord(ev_sweep->b, stream));
    if (evaluated) {
        hipLaunchKernelGGL(k_sum_words, dim3(64), dim3(256), 0, stream, evaluated, (int)N, counters);
        HIP_TRY(hipGetLastError());
    }
    return SLHC_OK;
}

slhc::NearOrder near_order_of(const OrderWs& o)
{
    slhc::NearOrder n{};
    n.gap = o.tile_gap; n.tiles = (o.Ns + 127) / 128; n.perm = o.perm; n.rows = o.Ns;
    n.region = o.tile_local; n.all = o.near_all; n.local = o.near_local; n.local_scale = o.local_scale;
    n.all.tiles = n.local.tiles = n.tiles; n.all.rows = n.local.rows = o.Ns;
    n.tile_colour = o.tile_colour;
    return n;
}
// Pruned k-NN searches, and with them the connection rounds, go to the half-precision engine where a tile's region holds as many
// tiles on average as a region must have for a copy relative to its centre (k_region_local).  Without that copy the rounding is a
// share of the distance from all rows' centre, and in tight clusters (300k x 32, a thousand radii apart) every pair of a tile may
// be the one that is wanted: of 700 rows (7 tiles) the search takes 14.4 ms and the list kernels 1.5 ms, of 1000 rows (8 tiles)
// 1.8 and 1.55 ms, of 100 rows 3.3 and 0.8 ms (2M x 32: 22 and 4.7 ms).  Clusters a few radii apart do not need it, and there the
// search costs little where it does not gain, and the connection rounds gain on both sides of the line: 200k x 64 in clusters of
// 800 rows 1.4 and 1.7 ms, rounds 7.0 and 17.3 ms; of 120 rows 1.2 and 0.7 ms, rounds 5.9 and 11.6 ms.  (Both kinds of rounds have
// become shorter since, by a quarter to a third.)
constexpr unsigned long long NEAR_REGION_TILES = REGION_TILES;
// Connection rounds go there too unless the clusters are tight against their distances: a row of another cluster is then known
// up to a few 1e-4 of the spread of all rows, and where that is as much as a cluster's radius every row of a component may be the
// one that is nearest (2M x 32 in clusters of 100 rows, a thousand radii apart: all rows are left to be searched, 57 ms of
// rounds against the list kernels' 30, which are 13 now).  The spread is about 0.6 sqrt(d) times the largest deviation of a column, so the line is
// drawn where the rounding of two rows reaches a quarter of the radius.
constexpr float NEAR_LINK_SPREAD = 360.f;

// Pruned searches by the half-precision engine, where the table of tile pairs exists; the flags that ask for a form of the
// list kernels' sweeps get those.
bool near_ordered(const KnnWs& ws, uint32_t flags)
{
    return near_wanted(ws.near, flags) && ws.has_order && ws.order.tile_gap &&
           !(flags & (SLHC_NO_TILE_TABLE | SLHC_ONE_SHIFT | SLHC_SPLIT_ROUNDS | SLHC_SPLIT_SCANS));
}

// The regions of the row order: tiles are cut where consecutive centres part (see run_knn).
int make_regions(const OrderWs& o, int32_t d, hipStream_t stream)
{
    const int T = (o.Ns + 127) / 128;
    hipLaunchKernelGGL(k_region_boundaries, dim3((unsigned)((T + 255) / 256)), dim3(256), 0, stream, o.tile_c, o.tile_r, T, d,
                       o.tile_boundary);
    hipLaunchKernelGGL(k_region_scan, dim3(1), dim3(1024), 0, stream, o.tile_boundary, T, o.tile_region, o.tile_first);
    hipLaunchKernelGGL(k_region_last, dim3((unsigned)((T + 255) / 256)), dim3(256), 0, stream, o.tile_boundary, o.tile_first, T,
                       o.tile_last);
    HIP_TRY(hipGetLastError());
    return SLHC_OK;
}

int run_knn(const float* X, int64_t N, int32_t d, int32_t k, int32_t* nbr_idx, float* nbr_dist,
            KnnWs& ws, hipStream_t stream, uint32_t flags, bool* pruned_out = nullptr,
            EventPair* ev_norm = nullptr, EventPair* ev_order = nullptr, EventPair* ev_sweep = nullptr)
{
    if (!((flags & SLHC_PRUNE) && ws.has_order) && near_wanted(ws.near, flags)) {
        if (pruned_out) *pruned_out = false;
        if (ev_order) { HIP_TRY(hipEventRecord(ev_order->a, stream)); HIP_TRY(hipEventRecord(ev_order->b, stream)); }
        ws.near_done = true;
        const int direct = slhc::direct_knn_wanted(N, d, k, pruned_out != nullptr);
        ws.near_ready = direct == 0;
        return run_knn_near(X, N, d, k, nbr_idx, nbr_dist, ws.counters, ws.hn, ws.near, stream, direct, pruned_out != nullptr,
                            ev_sweep ? reinterpret_cast<int32_t*>(ws.hn_split) : nullptr, ev_norm, ev_sweep);
    }
    hipLaunchKernelGGL(k_zero_words, dim3(1), dim3(64), 0, stream, reinterpret_cast<uint32_t*>(ws.counters), 64);
    HIP_TRY(hipGetLastError());
    if (ev_norm) HIP_TRY(hipEventRecord(ev_norm->a, stream));
    if (near_wanted(ws.near, flags)) {
        HIP_TRY(slhc::near_stats(X, (int)N, d, ws.near.b, nullptr, 0, stream));
        HIP_TRY(slhc::near_make(X, (int)N, d, nullptr, (int)N, nullptr, ws.near.b, ws.near.c, ws.hn, reinterpret_cast<unsigned int*>(ws.counters + 4), stream));
        ws.near_ready = true;
    } else
        HIP_TRY(slhc::launch_half_norms(X, (int)N, d, ws.hn, stream, reinterpret_cast<unsigned int*>(ws.counters + 4)));
    if (ev_norm) HIP_TRY(hipEventRecord(ev_norm->b, stream));
    const bool prune = (flags & SLHC_PRUNE) && ws.has_order;
    if (pruned_out) *pruned_out = prune;
    const bool split = prune && ws.Xsplit && ws.hn_split && !(flags & SLHC_FP32_FILTER);
    // X in split halves: for the list kernels' sweeps
    auto make_split = [&]() -> int {
        const int rs = make_split_copy(X, N, d, ws, stream);
        if (rs != SLHC_OK) return rs;
        if (!split_products_pruned_ok(d)) {
            // Below 64 features the pruned sweeps multiply in float32, on the rows as they are: fine unless the
            // rows share an offset far larger than their distances, which then fills the filter's slack and
            // lets every pair of a tile through.  The split copy is taken relative to the column means; when
            // that shrinks the norms eightfold or more, the pruned sweeps multiply it too.
            Mailbox mail(stream);
            HIP_TRY(mail.open());
            float h_sums[2];
            hipLaunchKernelGGL(k_sample_sums, dim3(1), dim3(256), 0, stream, ws.hn, ws.hn_split, (int)N, ws.shift_scratch);
            HIP_TRY(hipGetLastError());
            HIP_TRY(mail.fetch(ws.shift_scratch, 2, h_sums));
            mail.box.idle();
            ws.offset_heavy = h_sums[0] >= 8.f * h_sums[1];          // false when either sum is NaN
        }
    
        return SLHC_OK;
    };
    if (ev_order) HIP_TRY(hipEventRecord(ev_order->a, stream));
    if (prune) {
        const int rc0 = split && !near_ordered(ws, flags) ? make_split() : SLHC_OK;
        if (rc0 != SLHC_OK) return rc0;
        const int rc = build_order(X, N, d, ws.hn, reinterpret_cast<const unsigned int*>(ws.counters + 4), ws.order, stream,
                                   ws.near_ready ? &ws.near : nullptr,
                                   ws.split_ready ? ws.Xsplit : nullptr, ws.split_ready ? ws.hn_split : nullptr, ws.split_ready ? ws.shift : nullptr);
        if (rc != SLHC_OK) return rc;
    }
    if (ev_order) HIP_TRY(hipEventRecord(ev_order->b, stream));
    if (ev_sweep) HIP_TRY(hipEventRecord(ev_sweep->a, stream));
    slhc::SweepParams p{};
    p.d = d; p.k = k;
    p.out_idx = nbr_idx; p.out_dist = nbr_dist;
    p.exclude_self = 1;
    p.survivors = ws.counters;
    p.tiles_done = ws.counters + 2;
    bool by_near = false, by_lists = true;
    if (prune && near_ordered(ws, flags)) {
        const OrderWs& o = ws.order;
        const int T = (o.Ns + 127) / 128;
        const int rr = make_regions(o, d, stream);
        if (rr != SLHC_OK) return rr;
        ws.regions_ready = true;
        hipLaunchKernelGGL(k_region_local, dim3((unsigned)((T + 255) / 256)), dim3(256), 0, stream, o.tile_region, o.tile_first, o.tile_last, T,
                           o.tile_local, o.tile_boundary, ws.counters + 10);       // (the boundaries are used up)
        HIP_TRY(hipGetLastError());
        Mailbox mail(stream);
        HIP_TRY(mail.open());
        unsigned long long pairs = 0;
        HIP_TRY(mail.fetch(ws.counters + 10, 2, &pairs));
        by_near = pairs >= NEAR_REGION_TILES * (unsigned long long)T;
        float ratio[2] = {0.f, 0.f};
        if (by_near) {
            slhc::NearOrder n = near_order_of(o);
            n.ratios = reinterpret_cast<float*>(ws.counters + 11);
            HIP_TRY(slhc::near_make_ordered(X, (int)N, d, n, o.tile_c, o.tile_r, o.tile_boundary, ws.hn, ws.near.b, stream));
            HIP_TRY(mail.fetch(ws.counters + 11, 2, ratio));
            ws.near_order_ready = ratio[0] * sqrtf((float)d) <= NEAR_LINK_SPREAD;
        }
        mail.box.idle();
        // (an offset that most of the norms are: the panels left to the list kernels need the split copy)
        by_lists = !ws.near_order_ready || ratio[1] >= 8.f;
        if (split && by_lists) { const int rs = make_split(); if (rs != SLHC_OK) return rs; }
    }
    if (prune) {
        const OrderWs& o = ws.order;
        p.Xq = p.Xc = o.Xs; p.hq = p.hc = o.hs; p.NQ = p.NC = o.Ns;
        if (by_lists && o.Xs_split && ws.hn_split && (split_products_pruned_ok(d) || ws.offset_heavy || (o.Xs_local && !(flags & SLHC_ONE_SHIFT))) &&
            !(flags & SLHC_FP32_FILTER)) {
            // the reordered copy in split halves too; its half norms are those of the rows (padding: +inf)
            HIP_TRY(slhc::launch_split_bf16(o.Xs, o.Ns, d, o.Xs_split, stream, ws.shift));
            HIP_TRY(slhc::order_gather_f32(ws.hn_split, o.perm, o.Ns, (int)N, __builtin_inff(), o.hs_split, stream));
            p.Xq_split = p.Xc_split = o.Xs_split; p.hq_split = p.hc_split = o.hs_split;
            ws.order_split_ready = true;
            // (at 32 features the connection sweeps keep float32 products unless the data has a large common offset:
            // the wider filter costs them more than the multiplies save; the k-NN sweep, in local coordinates for the
            // tiles that matter, gains)
            ws.order_split_connect = split_products_pruned_ok(d) || ws.offset_heavy;
        }
        p.q_out_row = o.perm; p.c_id = o.perm;
        p.tile_c = o.tile_c; p.tile_r = o.tile_r; p.gap_ws = o.gap_ws;
        p.tile_gap = (flags & SLHC_NO_TILE_TABLE) ? nullptr : o.tile_gap;
        p.own_tile_first = 1;
        p.panel_counter = reinterpret_cast<unsigned int*>(ws.counters + 8);     // zeroed above
#ifdef SLHC_STUDY_PANEL_STEPS
        p.panel_steps = reinterpret_cast<int*>(o.qslot);       // free until the connection rounds
        HIP_TRY(hipMemsetAsync(o.qslot, 0, (size_t)((o.Ns + 127) / 128) * 8, stream));
#endif
#ifdef SLHC_PHASE_TIMERS
        p.phase_cycles = ws.counters + 16;
#endif
    } else {
        p.Xq = p.Xc = X; p.hq = p.hc = ws.hn; p.NQ = p.NC = (int)N;
        p.part_idx = ws.part_idx; p.part_dist = ws.part_dist; p.part_rows = ws.part_rows;
        if (!(flags & SLHC_PANEL_ORDER)) {
            p.carry_ws = ws.carry_ws; p.carry_ws_words = ws.carry_ws_words;
            p.carry_fault = reinterpret_cast<unsigned int*>(ws.counters + 4);
        }
        if (ws.Xsplit && !(flags & SLHC_FP32_FILTER)) {
            const int rs = make_split_copy(X, N, d, ws, stream);
            if (rs != SLHC_OK) return rs;
            p.Xq_split = p.Xc_split = ws.Xsplit; p.hq_split = p.hc_split = ws.hn_split;
        }
#ifdef SLHC_PHASE_TIMERS
        p.phase_cycles = ws.counters + 16;
#endif
    }
    if (by_near) {
        const OrderWs& o = ws.order;
        slhc::NearProblem a{};
        a.Xq = a.Xc = X; a.d = d; a.k = k;
        a.nq = a.nq_rows = a.nc = (int)N;
        a.exclude_self = 1;
        a.out_idx = nbr_idx; a.out_dist = nbr_dist;
        a.evaluated = ev_sweep ? ws.near.q.left : nullptr;      // (free until the connection rounds)
        slhc::NearOrder n = near_order_of(o);
        n.tile_steps = ws.counters + 2;
        HIP_TRY(slhc::near_search_ordered(a, n, ws.near.b, stream));
        ws.near_done = true;
        if (!ws.offset_heavy) { p.Xq_split = p.Xc_split = nullptr; p.hq_split = p.hc_split = nullptr; }
        p.todo = ws.near.b.todo;            // the panels it could not finish
        p.tiles_done = nullptr;
        HIP_TRY(slhc::launch_knn_sweep(p, stream));
        if (ev_sweep) {
            HIP_TRY(hipEventRecord(ev_sweep->b, stream));
            hipLaunchKernelGGL(k_sum_words, dim3(64), dim3(256), 0, stream, a.evaluated, (int)N, ws.counters);
            HIP_TRY(hipGetLastError());
        }
        return SLHC_OK;
    }
    if (prune && ws.order_split_ready && ws.order.Xs_local && !(flags & SLHC_ONE_SHIFT)) {
        // Two launches (see SweepParams::region_mode).  The rows of a cluster share their centre as an offset that
        // the common shift does not remove, and the filter's slack is a fraction of the squared norms: 1M x 128
        // passes 660 pairs per row on to the exact evaluation for 217 list updates.  The row order keeps a cluster
        // in consecutive tiles, so the tiles are cut into regions where consecutive centres part (farther than
        // twice the larger radius), a second split copy takes every tile relative to the centre of its region's
        // first tile, and the first launch multiplies that copy for the tiles of the panel's own region; the
        // second launch starts from those lists and visits the other tiles with the common shift.
        const OrderWs& o = ws.order;
        const int T = (o.Ns + 127) / 128;
        if (!ws.regions_ready) { const int rr = make_regions(o, d, stream); if (rr != SLHC_OK) return rr; }
        HIP_TRY(slhc::launch_split_bf16(o.Xs, o.Ns, d, o.Xs_local, stream, o.tile_c, o.tile_first));
        HIP_TRY(slhc::launch_half_norms(o.Xs, o.Ns, d, o.hs_local, stream, nullptr, true, o.tile_c, o.tile_first));
        hipLaunchKernelGGL(k_mask_padding, dim3((unsigned)((o.Ns + 255) / 256)), dim3(256), 0, stream, o.perm, o.Ns, o.hs_local);
        HIP_TRY(hipGetLastError());
        slhc::SweepParams own = p;
        own.Xq_split = own.Xc_split = o.Xs_local; own.hq_split = own.hc_split = o.hs_local;
        own.tile_region = o.tile_region; own.region_mode = 1;
        own.tile_first = o.tile_first; own.tile_last = o.tile_last;
        HIP_TRY(slhc::launch_knn_sweep(own, stream));
        hipLaunchKernelGGL(k_zero_words, dim3(1), dim3(64), 0, stream, p.panel_counter, 2);
        HIP_TRY(hipGetLastError());
        p.tile_region = o.tile_region; p.region_mode = 2;
        if (p.tile_gap) {
            hipLaunchKernelGGL(k_region_other_min, dim3((unsigned)T), dim3(256), 0, stream, p.tile_gap, o.tile_region, T, o.region_other_min);
            HIP_TRY(hipGetLastError());
            p.region_other_min = o.region_other_min;
        }
    }
    HIP_TRY(slhc::launch_knn_sweep(p, stream));
    if (ev_sweep) HIP_TRY(hipEventRecord(ev_sweep->b, stream));
    return SLHC_OK;
}

// Linkage arrays from weight-sorted tree edges (paper Sec. 3.3.1) of few rows, on the host as in the paper: a union-find over the N points
// (union by size, path halving) in which every set carries the dendrogram node created by its last
// merge; merge i creates node N+i.  The edges arrive in weight order, so their end points are
// scattered over the whole array: one 16-byte record per point keeps a find step to one cache
// line, and the records of the edges a few iterations ahead, then their parents, are prefetched.
// End points outside [0, N) (never produced by a correct caller) are skipped and reported by `false`.
bool build_dendrogram(const int32_t* lo, const int32_t* hi, int64_t N, int32_t* children, int32_t* sizes)
{
    struct PointSet { int32_t up, count, node, unused; };
    constexpr int64_t AHEAD = 16;
    std::unique_ptr<PointSet[]> set(new PointSet[(size_t)N]);
    for (int64_t v = 0; v < N; ++v) set[(size_t)v] = PointSet{(int32_t)v, 1, (int32_t)v, 0};
    auto root = [&](int32_t a) {
        while (set[(size_t)a].up != a) {
            set[(size_t)a].up = set[(size_t)set[(size_t)a].up].up;
            a = set[(size_t)a].up;
        }
        return a;
    };
    bool good = true;
    const uint32_t n = (uint32_t)N;
    const int64_t E = N - 1;
    for (int64_t j = 0; j < E; ++j) {
        if (j + AHEAD < E && (uint32_t)lo[j + AHEAD] < n && (uint32_t)hi[j + AHEAD] < n) {
            __builtin_prefetch(&set[(size_t)lo[j + AHEAD]]);
            __builtin_prefetch(&set[(size_t)hi[j + AHEAD]]);
            // and, half way, the records those point to (their own have arrived by now)
            __builtin_prefetch(&set[(size_t)set[(size_t)lo[j + AHEAD / 2]].up]);
            __builtin_prefetch(&set[(size_t)set[(size_t)hi[j + AHEAD / 2]].up]);
        }
        if ((uint32_t)lo[j] >= n || (uint32_t)hi[j] >= n) { good = false; continue; }
        int32_t ra = root(lo[j]), rb = root(hi[j]);
        const int32_t a = set[(size_t)ra].node, b = set[(size_t)rb].node;
        children[2 * j] = a < b ? a : b;
        children[2 * j + 1] = a < b ? b : a;
        if (set[(size_t)ra].count < set[(size_t)rb].count) std::swap(ra, rb);
        set[(size_t)rb].up = ra;
        set[(size_t)ra].count += set[(size_t)rb].count;
        set[(size_t)ra].node = (int32_t)(N + j);
        sizes[j] = set[(size_t)ra].count;
    }
    return good;
}

// ---- scratch of slhc_knn_graph_static: the workspace of the every-tile k-NN path as a fixed device array
// (static_scratch.hip).  Every GPU that entry point runs on holds its own copy at its own address until the process ends.
using slhc::STATIC_SCRATCH_BYTES;
constexpr int MAX_DEVICES = 64;
std::mutex g_scratch_mutex;
void* g_scratch_ptr[MAX_DEVICES] = {};

// Device address of that array on the current device (looked up once per device).
int static_scratch(void** out)
{
    int dev = -1;
    HIP_TRY(hipGetDevice(&dev));
    if (dev < 0 || dev >= MAX_DEVICES) { set_err("device ordinal %d beyond %d", dev, MAX_DEVICES - 1); return SLHC_UNSUPPORTED; }
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void* ptr = nullptr;
        HIP_TRY(slhc::static_scratch_address(&ptr));
        if (!ptr) { set_err("hipGetSymbolAddress returned a null address"); return SLHC_HIP_ERROR; }
        g_scratch_ptr[dev] = ptr;
    }
    *out = g_scratch_ptr[dev];
    return SLHC_OK;
}

}  // namespace

extern "C" {

int slhc_abi_version(void) { return SLHC_ABI_VERSION; }

const char* slhc_strerror(int status)
{
    switch (status) {
        case SLHC_OK: return "ok";
        case SLHC_INVALID_ARG: return "invalid argument";
        case SLHC_UNSUPPORTED: return "unsupported size";
        case SLHC_WORKSPACE_TOO_SMALL: return "workspace too small";
        case SLHC_HIP_ERROR: return "HIP error";
        case SLHC_NONFINITE: return "input not finite";
        case SLHC_INTERNAL: return "internal error";
        case SLHC_HOST_MEMORY: return "host allocation failed";
        default: return "unknown status";
    }
}

const char* slhc_last_error(void) { return g_err; }

int slhc_knn_workspace_bytes(int64_t N, int32_t d, int32_t k, size_t* bytes)
{
    return guarded([&]() -> int {
        if (!bytes) { set_err("bytes is NULL"); return SLHC_INVALID_ARG; }
        const int rc = check_shape(N, d, k, true);
        if (rc != SLHC_OK) return rc;
        *bytes = padded_copy_bytes(N, d) + KnnWs(nullptr, N, working_columns(N, d), true, k, false).bytes;
        return SLHC_OK;
    });
}

int slhc_probe_knn_products(int64_t N, int32_t d, int32_t k, double* products)
{
    return guarded([&]() -> int {
        if (!products) { set_err("products is NULL"); return SLHC_INVALID_ARG; }
        const int rc = check_shape(N, d, k, true);
        if (rc != SLHC_OK) return rc;
        const int32_t dw = working_columns(N, d);
        const KnnWs ws(nullptr, N, dw, true, k, false);
        bool once = false;
        const size_t pairs = slhc::near_pairs_bytes(N, d, k + 1, &once);
        *products = !ws.near.ok ? 3.0 : slhc::direct_knn_wanted(N, d, k, false) > 0 ? 0.0 : once && pairs <= ws.near.b.pairs_bytes ? 0.5 : 1.0;
        return SLHC_OK;
    });
}

int slhc_knn_graph_opt(const float* X, int64_t N, int32_t d, int32_t k, int32_t* nbr_idx, float* nbr_dist,
                       void* workspace, size_t workspace_bytes, void* stream, uint32_t flags)
{
    return guarded([&]() -> int {
        if (!X || !nbr_idx || !nbr_dist || !workspace) { set_err("NULL pointer argument"); return SLHC_INVALID_ARG; }
        const int rc = check_shape(N, d, k, true);
        if (rc != SLHC_OK) return rc;
        const int32_t dw = working_columns(N, d);
        const size_t head = padded_copy_bytes(N, d);
        KnnWs ws(static_cast<unsigned char*>(workspace) + head, N, dw, true, k, false, workspace_bytes > head ? workspace_bytes - head : 0);
        if (workspace_bytes < head + ws.bytes) { set_err("workspace %zu < %zu bytes", workspace_bytes, head + ws.bytes); return SLHC_WORKSPACE_TOO_SMALL; }
        const bool prune = (flags & SLHC_PRUNE) && ws.has_order;
        if (!prune && near_wanted(ws.near, flags))          // (reads the rows as they are)
            return run_knn(X, N, d, k, nbr_idx, nbr_dist, ws, static_cast<hipStream_t>(stream), flags);
        if (dw != d) {
            const int rp = pad_columns(X, N, d, dw, static_cast<float*>(workspace), static_cast<hipStream_t>(stream));
            if (rp != SLHC_OK) return rp;
            X = static_cast<const float*>(workspace);
        }
        return run_knn(X, N, dw, k, nbr_idx, nbr_dist, ws, static_cast<hipStream_t>(stream), flags);
    });
}

int slhc_knn_graph(const float* X, int64_t N, int32_t d, int32_t k, int32_t* nbr_idx, float* nbr_dist,
                   void* workspace, size_t workspace_bytes, void* stream)
{
    return guarded([&]() -> int {
        return slhc_knn_graph_opt(X, N, d, k, nbr_idx, nbr_dist, workspace, workspace_bytes, stream, 0u);
    });
}

int slhc_knn_graph_static(const float* X, int64_t N, int32_t d, int32_t k, int32_t* nbr_idx, float* nbr_dist,
                          void* stream)
{
    return guarded([&]() -> int {
        if (!X || !nbr_idx || !nbr_dist) { set_err("NULL pointer argument"); return SLHC_INVALID_ARG; }
        const int rc = check_shape(N, d, k, true);
        if (rc != SLHC_OK) return rc;
        if (N > (int64_t)SLHC_STATIC_MAX_ROWS) {
            set_err("N=%lld exceeds SLHC_STATIC_MAX_ROWS=%lld of the fixed scratch array; use slhc_knn_graph with a workspace",
                    (long long)N, (long long)SLHC_STATIC_MAX_ROWS);
            return SLHC_UNSUPPORTED;
        }
        void* ptr = nullptr;
        const int rs = static_scratch(&ptr);
        if (rs != SLHC_OK) return rs;
        {
            // counters, half norms, the float16 copy and its buffers, as far as they fit
            Carver c(ptr);
            unsigned long long* counters = c.take<unsigned long long>(32);
            float* hn = c.take<float>((size_t)N);
            NearWs near;
            near.carve(c, N, 0, d, k + 1, false, STATIC_SCRATCH_BYTES);
            if (near.ok && c.off <= STATIC_SCRATCH_BYTES)
                return run_knn_near(X, N, d, k, nbr_idx, nbr_dist, counters, hn, near, static_cast<hipStream_t>(stream),
                                    slhc::direct_knn_wanted(N, d, k, false), false);
        }
        KnnWs ws(ptr, N, d, false, 0, false);       // counters (cleared by run_knn) + half norms (all N written)
        if (ws.bytes > STATIC_SCRATCH_BYTES) { set_err("scratch layout %zu > %zu bytes", ws.bytes, STATIC_SCRATCH_BYTES); return SLHC_INTERNAL; }
        return run_knn(X, N, d, k, nbr_idx, nbr_dist, ws, static_cast<hipStream_t>(stream), 0u);
    });
}

int slhc_probe_fp32_mfma(double* tflops, void* workspace, size_t workspace_bytes, void* stream)
{
    return guarded([&]() -> int {
        if (!tflops || !workspace) { set_err("NULL pointer argument"); return SLHC_INVALID_ARG; }
        if (workspace_bytes < 256) { set_err("workspace %zu < 256 bytes", workspace_bytes); return SLHC_WORKSPACE_TOO_SMALL; }
        hipStream_t s = static_cast<hipStream_t>(stream);
        EventPair ev;
        HIP_TRY(ev.create());
        double flop = 0.0;
        HIP_TRY(slhc::launch_mfma_probe(2000, static_cast<float*>(workspace), s, &flop));      // warm-up: clocks settle
        HIP_TRY(hipEventRecord(ev.a, s));
        HIP_TRY(slhc::launch_mfma_probe(40000, static_cast<float*>(workspace), s, &flop));     // ~40 ms
        HIP_TRY(hipEventRecord(ev.b, s));
        HIP_TRY(hipStreamSynchronize(s));
        const float ms = ev.ms();
        if (!(ms > 0.f)) { set_err("probe timing failed"); return SLHC_HIP_ERROR; }
        *tflops = flop / (ms * 1e-3) / 1e12;
        return SLHC_OK;
    });
}

static int probe_16bit_mfma(bool half, double* tflops, void* workspace, size_t workspace_bytes, void* stream)
{
    if (!tflops || !workspace) { set_err("NULL pointer argument"); return SLHC_INVALID_ARG; }
    if (workspace_bytes < 256) { set_err("workspace %zu < 256 bytes", workspace_bytes); return SLHC_WORKSPACE_TOO_SMALL; }
    hipStream_t s = static_cast<hipStream_t>(stream);
    EventPair ev;
    HIP_TRY(ev.create());
    double flop = 0.0;
    HIP_TRY(slhc::launch_mfma_16bit_probe(half, 2000, static_cast<float*>(workspace), s, &flop));      // warm-up: clocks settle
    HIP_TRY(hipEventRecord(ev.a, s));
    HIP_TRY(slhc::launch_mfma_16bit_probe(half, 80000, static_cast<float*>(workspace), s, &flop));     // ~40 ms
    HIP_TRY(hipEventRecord(ev.b, s));
    HIP_TRY(hipStreamSynchronize(s));
    const float ms = ev.ms();
    if (!(ms > 0.f)) { set_err("probe timing failed"); return SLHC_HIP_ERROR; }
    *tflops = flop / (ms * 1e-3) / 1e12;
    return SLHC_OK;
}

int slhc_probe_bf16_mfma(double* tflops, void* workspace, size_t workspace_bytes, void* stream)
{
    return guarded([&]() -> int { return probe_16bit_mfma(false, tflops, workspace, workspace_bytes, stream); });
}

int slhc_probe_f16_mfma(double* tflops, void* workspace, size_t workspace_bytes, void* stream)
{
    return guarded([&]() -> int { return probe_16bit_mfma(true, tflops, workspace, workspace_bytes, stream); });
}

static int probe_16bit_values(bool half, const float* A, const float* B, const float* C, float* D, int32_t trials, void* stream)
{
    if (!A || !B || !C || !D) { set_err("NULL pointer argument"); return SLHC_INVALID_ARG; }
    if (trials < 0 || trials > (1 << 24)) { set_err("trials must be 0..2^24 (trials=%d)", trials); return SLHC_INVALID_ARG; }
    HIP_TRY(slhc::launch_mfma_16bit_values(half, A, B, C, D, trials, static_cast<hipStream_t>(stream)));
    return SLHC_OK;
}

int slhc_probe_bf16_mfma_values(const float* A, const float* B, const float* C, float* D, int32_t trials, void* stream)
{
    return guarded([&]() -> int { return probe_16bit_values(false, A, B, C, D, trials, stream); });
}

int slhc_probe_f16_mfma_values(const float* A, const float* B, const float* C, float* D, int32_t trials, void* stream)
{
    return guarded([&]() -> int { return probe_16bit_values(true, A, B, C, D, trials, stream); });
}

int slhc_probe_panel_loop(int32_t steps, double* tflops, void* workspace, size_t workspace_bytes, void* stream)
{
    return guarded([&]() -> int {
        if (!tflops || !workspace) { set_err("NULL pointer argument"); return SLHC_INVALID_ARG; }
        if (steps < 0 || steps > 11) { set_err("steps must be 0..11 (steps=%d)", steps); return SLHC_INVALID_ARG; }
        // a sink word, then the rows to stream from: the largest power of two of 512-byte rows that fits
        if (workspace_bytes < 256 + 512 * 256) { set_err("workspace %zu < %d bytes", workspace_bytes, 256 + 512 * 256); return SLHC_WORKSPACE_TOO_SMALL; }
        int rows = 256;
        while ((size_t)rows * 2 * 512 + 256 <= workspace_bytes && rows < (1 << 22)) rows *= 2;
        float* sink = static_cast<float*>(workspace);
        const float* rows_ptr = reinterpret_cast<const float*>(static_cast<unsigned char*>(workspace) + 256);
        hipStream_t s = static_cast<hipStream_t>(stream);
        EventPair ev;
        HIP_TRY(ev.create());
        double flop = 0.0;
        HIP_TRY(slhc::launch_loop_probe(steps, 500, rows_ptr, rows, sink, s, &flop));           // warm-up: clocks settle
        HIP_TRY(hipEventRecord(ev.a, s));
        HIP_TRY(slhc::launch_loop_probe(steps, 10000, rows_ptr, rows, sink, s, &flop));         // ~40 ms
        HIP_TRY(hipEventRecord(ev.b, s));
        HIP_TRY(hipStreamSynchronize(s));
        const float ms = ev.ms();
        if (!(ms > 0.f)) { set_err("probe timing failed"); return SLHC_HIP_ERROR; }
        *tflops = flop / (ms * 1e-3) / 1e12;
        return SLHC_OK;
    });
}

// Scratch of slhc_cross_1nn, `most` bytes of it.  A search that evaluates every pair needs a word per query besides, one of the
// half-precision engine its copies; the list kernels, which run where neither fits, need nothing else.
struct CrossWs {
    unsigned long long* counters;
    float* hn;
    unsigned long long* keys = nullptr;
    NearWs near;
    size_t bytes;
    CrossWs(void* ws, int64_t N, int32_t d, int64_t m, size_t most = NO_LIMIT)
    {
        Carver c(ws);
        counters = c.take<unsigned long long>(32);
        hn = c.take<float>((size_t)N);
        if (m > 0 && slhc::direct_1nn_alone(m, N, d)) {
            if (most > c.off && up((size_t)m * 8) <= most - c.off) keys = c.take<unsigned long long>((size_t)m);
        } else if (m > 0) {
            near.carve(c, N, m, d, 1, true, most);
            if (near.ok && slhc::direct_1nn_wanted(m, N, d) && near.b.batch_bytes >= (size_t)m * 8) keys = reinterpret_cast<unsigned long long*>(near.b.batch);
        }
        bytes = c.off;
    }
};

int slhc_cross_1nn_workspace_bytes(int64_t N, int32_t d, int64_t m, size_t* bytes)
{
    return guarded([&]() -> int {
        if (!bytes) { set_err("bytes is NULL"); return SLHC_INVALID_ARG; }
        const int rc = check_shape(N, d, 1, false);
        if (rc != SLHC_OK) return rc;
        if (m < 0 || m > 2147483647LL) { set_err("bad m"); return SLHC_INVALID_ARG; }
        *bytes = CrossWs(nullptr, N, d, m).bytes;
        return SLHC_OK;
    });
}

int slhc_cross_1nn(const float* X, int64_t N, int32_t d, const int32_t* colour, const int32_t* rows,
                   int64_t m, int32_t* out_idx, float* out_dist, void* workspace,
                   size_t workspace_bytes, void* stream)
{
    return guarded([&]() -> int {
        if (!X || !colour || !out_idx || !out_dist || !workspace) { set_err("NULL pointer argument"); return SLHC_INVALID_ARG; }
        const int rc = check_shape(N, d, 1, false);
        if (rc != SLHC_OK) return rc;
        if (m < 0 || m > 2147483647LL || (!rows && m > N)) { set_err("bad m=%lld", (long long)m); return SLHC_INVALID_ARG; }
        const CrossWs ws(workspace, N, d, m, workspace_bytes);
        const NearWs& near = ws.near;
        unsigned long long* counters = ws.counters;
        float* hn = ws.hn;
        if (workspace_bytes < ws.bytes) { set_err("workspace %zu < %zu bytes", workspace_bytes, ws.bytes); return SLHC_WORKSPACE_TOO_SMALL; }
        if (m == 0) return SLHC_OK;
        hipStream_t s = static_cast<hipStream_t>(stream);
        slhc::SweepParams p{};
        if (ws.keys) {
            HIP_TRY(slhc::direct_1nn(X, (int)m, (int)N, rows, X, (int)N, d, colour, out_idx, out_dist, ws.keys, s));
            return SLHC_OK;
        }
        if (near.ok) {
            HIP_TRY(slhc::near_stats(X, (int)N, d, near.b, reinterpret_cast<uint32_t*>(counters), 64, s));
            const bool all = !rows && m == N;            // queries are the candidates
            slhc::NearCopy c = near.c;
            if (all) { c.left = near.q.left; c.count = near.q.count; }
            HIP_TRY(slhc::near_make(X, (int)N, d, nullptr, (int)N, colour, near.b, c, hn, nullptr, s));
            if (!all) HIP_TRY(slhc::near_make(X, (int)N, d, rows, (int)m, colour, near.b, near.q, nullptr, nullptr, s));
            slhc::NearProblem a{};
            a.Xq = a.Xc = X; a.d = d; a.k = 1;
            a.q_rows = rows; a.nq = (int)m; a.nq_rows = a.nc = (int)N;
            a.coloured = 1;
            a.out_idx = out_idx; a.out_dist = out_dist;
            HIP_TRY(slhc::near_search(a, all ? c : near.q, c, near.b, s));
            p.todo = near.b.todo;
        } else {
            hipLaunchKernelGGL(k_zero_words, dim3(1), dim3(64), 0, s, reinterpret_cast<uint32_t*>(counters), 64);
            HIP_TRY(hipGetLastError());
            HIP_TRY(slhc::launch_half_norms(X, (int)N, d, hn, s));
        }
        p.Xq = p.Xc = X; p.hq = p.hc = hn; p.NQ = p.NC = (int)N; p.d = d; p.k = 1;
        p.out_idx = out_idx; p.out_dist = out_dist;
        p.qcolour = p.ccolour = colour; p.rows = rows; p.m = (int)m;
        p.survivors = counters;
        HIP_TRY(slhc::launch_cross_1nn_sweep(p, s));
        return SLHC_OK;
    });
}

struct CsrWs {
    int32_t *colour, *ptr, *ext_idx, *rank, *hook, *counters, *e_lo, *e_hi;
    float *ext_dist, *ext_low, *e_w;
    uint32_t *best_w, *vals_a, *vals_b, *number;
    unsigned long long *best_e, *keys_a, *keys_b;
    void* sort_temp; size_t sort_temp_bytes;
    size_t bytes;
    CsrWs(void* ws, int64_t V)
    {
        Carver c(ws);
        const size_t n = (size_t)V;
        colour = c.take<int32_t>(n); ptr = c.take<int32_t>(n); ext_idx = c.take<int32_t>(n);       // (ptr and ext_idx serve as one array in the end)
        rank = c.take<int32_t>(n); hook = c.take<int32_t>(n); counters = c.take<int32_t>(64);
        e_lo = c.take<int32_t>(n); e_hi = c.take<int32_t>(n);
        ext_dist = c.take<float>(n); ext_low = c.take<float>(n); number = c.take<uint32_t>(n); e_w = c.take<float>(n);
        best_w = c.take<uint32_t>(n);
        vals_a = c.take<uint32_t>(n); vals_b = c.take<uint32_t>(n);
        best_e = c.take<unsigned long long>(n); keys_a = c.take<unsigned long long>(n); keys_b = c.take<unsigned long long>(n);
        sort_temp_bytes = slhc::edge_sort_temp_bytes((int)(V > 1 ? V - 1 : 1));
        sort_temp = c.take<unsigned char>(sort_temp_bytes);
        bytes = c.off;
    }
};

static int csr_shape(int64_t V, int64_t E)
{
    if (V < 1 || E < 0) { set_err("need V >= 1 and E >= 0 (V=%lld E=%lld)", (long long)V, (long long)E); return SLHC_INVALID_ARG; }
    if (V > 2147483646LL || E > 2147483647LL) { set_err("V or E exceeds 2^31-1"); return SLHC_UNSUPPORTED; }
    return SLHC_OK;
}

int slhc_csr_msf_workspace_bytes(int64_t V, int64_t E, size_t* bytes)
{
    return guarded([&]() -> int {
        if (!bytes) { set_err("bytes is NULL"); return SLHC_INVALID_ARG; }
        const int rc = csr_shape(V, E);
        if (rc != SLHC_OK) return rc;
        *bytes = CsrWs(nullptr, V).bytes;
        return SLHC_OK;
    });
}

int slhc_csr_msf(const int32_t* offsets, const int32_t* indices, const float* weights, int64_t V, int64_t E,
                 int32_t* mst_src, int32_t* mst_dst, float* mst_w, int64_t* n_edges, int32_t* colours,
                 int32_t* rounds, void* workspace, size_t workspace_bytes, void* stream)
{
    return guarded([&]() -> int {
        if (!offsets || (E > 0 && (!indices || !weights)) || !mst_src || !mst_dst || !mst_w || !n_edges || !colours || !workspace) {
            set_err("NULL pointer argument");
            return SLHC_INVALID_ARG;
        }
        const int rc = csr_shape(V, E);
        if (rc != SLHC_OK) return rc;
        CsrWs ws(workspace, V);
        if (workspace_bytes < ws.bytes) { set_err("workspace %zu < %zu bytes", workspace_bytes, ws.bytes); return SLHC_WORKSPACE_TOO_SMALL; }
        hipStream_t s = static_cast<hipStream_t>(stream);
        slhc::CsrForest f{};
        f.offsets = offsets; f.indices = indices; f.weights = weights; f.V = (int)V; f.E = (int)E;
        f.colour = ws.colour; f.hook = ws.hook; f.cand = ws.keys_b;
        f.best_w[0] = ws.best_w; f.best_w[1] = ws.vals_a; f.best_e[0] = ws.best_e; f.best_e[1] = ws.keys_a;
        f.active[0] = ws.ptr; f.active[1] = ws.ext_idx;
        f.roots[0] = reinterpret_cast<int32_t*>(ws.ext_dist); f.roots[1] = reinterpret_cast<int32_t*>(ws.ext_low);
        f.e_lo = ws.e_lo; f.e_hi = ws.e_hi; f.e_w = ws.e_w;
        f.words = ws.counters;
        // Alg. "MST Algorithm": min edge per vertex, min edge per supervertex, label propagation, until a round adds no edge (the
        // graph's components are then the forest's trees).  Rounds are enqueued one ahead of the host's reading (two mailboxes in
        // turn): the device goes from round to round without waiting for the host.  Once few vertices are active one launch does the
        // rest.
        Mailbox mail[2] = {Mailbox(s), Mailbox(s)};
        HIP_TRY(mail[0].open());
        HIP_TRY(mail[1].open());
        int max_rounds = 2;
        for (int64_t t = 1; t < V; t *= 2) ++max_rounds;
        int edges = 0, nrounds = 0;
        // as far as known: active vertices, and roots, of which a round leaves half at most
        int64_t vertices = V, roots = V;
        auto enqueue_round = [&](int round) -> int {
            Mailbox& m = mail[round & 1];
            roots = roots / 2 + 1;
            HIP_TRY(slhc::csr_round(f, round, (int)vertices, (int)roots, m.tagged(), m.next(), s));
            return SLHC_OK;
        };
        int32_t said[slhc::CSR_TOLD];
        bool ties = false;
        auto state = [&](int32_t check) -> int {
            if (check == 0) return SLHC_OK;
            set_err("forest state check %d failed (is every edge stored in both rows with one weight?)", check);
            return SLHC_INTERNAL;
        };
        auto read = [&](int which) -> int {
            HIP_TRY(mail[which].wait_tagged(slhc::CSR_TOLD));
            for (int i = 0; i < slhc::CSR_TOLD; ++i) said[i] = (int32_t)static_cast<volatile unsigned long long*>(mail[which].tagged())[i];
            ties = ((uint32_t)said[0] & slhc::CSR_MANY_TIES) != 0;
            said[0] = (int32_t)((uint32_t)said[0] & ~slhc::CSR_MANY_TIES);
            if (said[3] >= 20) {
                set_err("CSR input check %d failed (20-22: offsets, 23: index out of range, 24: weight negative or not finite)", said[3]);
                return SLHC_INVALID_ARG;
            }
            return state(said[3]);
        };
        // hook chains of `round` longer than a launch follows: finish them with the host in the loop
        auto finish_chains = [&](int round) -> int {
            int32_t left = 1;
            for (int jumps = 0; left != 0; ++jumps) {
                if (jumps > 64) { set_err("component hooks do not form a forest (is every edge stored in both rows with one weight?)"); return SLHC_INTERNAL; }
                hipLaunchKernelGGL(k_zero_words, dim3(1), dim3(64), 0, s, reinterpret_cast<uint32_t*>(f.words + slhc::CSR_CHAINS), 1);
                HIP_TRY(hipGetLastError());
                HIP_TRY(slhc::csr_follow_again(f, round, (int)vertices, s));
                HIP_TRY(mail[0].fetch(f.words + slhc::CSR_CHAINS, 1, &left));
            }
            return SLHC_OK;
        };
        HIP_TRY(slhc::csr_start(f, s));
        const int64_t tail_most = slhc::csr_tail_most(V, E);
        int rc2 = SLHC_OK, next = 1;                       // the round to enqueue next
        if (V > tail_most) { rc2 = enqueue_round(next++); if (rc2 != SLHC_OK) return rc2; }
        // what round `round - 1` left comes back with round `round`, behind which the next one is enqueued already
        for (int round = 1; vertices > tail_most; ++round) {
            rc2 = enqueue_round(next++);
            if (rc2 == SLHC_OK) rc2 = read(round & 1);
            if (rc2 != SLHC_OK) return rc2;
            if (said[2] != 0) {
                // this round and the one behind it did nothing: take both up again
                rc2 = read((round + 1) & 1);
                if (rc2 == SLHC_OK) rc2 = finish_chains(round - 1);
                roots = V;
                next = round;
                for (int i = 0; i < 2 && rc2 == SLHC_OK; ++i) rc2 = enqueue_round(next++);
                if (rc2 == SLHC_OK) rc2 = read(round & 1);
                if (rc2 != SLHC_OK) return rc2;
            }
            if (said[1] < edges || said[1] > V - 1 || said[0] < 0 || said[0] > V) { set_err("round left %d edges (had %d)", said[1], edges); return SLHC_INTERNAL; }
            const bool added = said[1] > edges;
            edges = said[1];
            vertices = said[0];
            nrounds = round;
            if (!added || edges == V - 1) break;           // steady state: a spanning forest
            if (nrounds > max_rounds) { set_err("no steady state after %d rounds", max_rounds); return SLHC_INTERNAL; }
            nrounds = 0;
        }
        const bool tail = nrounds == 0;
        while (nrounds == 0) {
            HIP_TRY(slhc::csr_tail(f, next, mail[1].tagged(), mail[1].next(), s));
            HIP_TRY(slhc::csr_colours(f, colours, s));         // (while the host waits for the tail)
            rc2 = read(1);
            if (rc2 != SLHC_OK) return rc2;
            if (said[2] != 0) {                            // (of a round before, behind which nothing was done)
                next = said[2];
                rc2 = finish_chains(next - 1);
                if (rc2 != SLHC_OK) return rc2;
                continue;
            }
            nrounds = said[0];
            edges = said[1];
            if (edges < 0 || edges > V - 1 || nrounds < 1) { set_err("rounds left %d edges", edges); return SLHC_INTERNAL; }
        }
        if (V == 1) nrounds = 0;
        if (!tail) HIP_TRY(slhc::csr_colours(f, colours, s));
        if (edges < V - 1) HIP_TRY(slhc::csr_closed(f, colours, s));
        // (the arrays of the rounds are free by now)
        slhc::CsrSortScratch t{};
        t.count = reinterpret_cast<int32_t*>(ws.best_e); t.offset = reinterpret_cast<int32_t*>(ws.keys_a);
        t.rank = ws.rank; t.number = ws.number; t.wbits_a = ws.best_w; t.wbits_b = ws.vals_a; t.ends_a = ws.keys_b;
        t.ends_b = reinterpret_cast<unsigned long long*>(ws.ptr);          // (and ext_idx behind it)
        t.temp = ws.sort_temp; t.temp_bytes = ws.sort_temp_bytes;
        // (up to 65 536 vertices edge_sort needs one sort)
        const bool large = edges > 0 && V > 65536, runs = large && !ties && slhc::csr_sort_in_runs_fits(edges, ws.sort_temp_bytes);
        int32_t ended[2] = {0, 1};                             // the end of all work: a failed check, and edges that the sort has not placed
        if (runs) {
            HIP_TRY(slhc::csr_sort_in_runs(ws.e_lo, ws.e_hi, ws.e_w, edges, t, mst_src, mst_dst, mst_w, f.words + slhc::CSR_FLAG, s));
            HIP_TRY(mail[0].fetch(f.words + slhc::CSR_ERROR, 2, ended));
            if (ended[1] > 0 && ended[1] <= slhc::CSR_LONG_MOST) {
                HIP_TRY(slhc::csr_sort_long_runs(ended[1], edges, t, mst_src, mst_dst, mst_w, s));
                HIP_TRY(mail[0].fetch(f.words + slhc::CSR_ERROR, 1, ended));
                ended[1] = 0;
            }
        }
        if (ended[1] != 0) {
            int32_t many = 1;
            if (large && slhc::csr_sort_fits((int)V, edges, ws.sort_temp_bytes)) {
                HIP_TRY(slhc::csr_sort_ends(ws.e_lo, ws.e_hi, ws.e_w, edges, (int)V, t, f.words + slhc::CSR_FLAG, mail[0].tagged(), mail[0].next(), s));
                HIP_TRY(mail[0].wait_tagged(1));
                many = (int32_t)static_cast<volatile unsigned long long*>(mail[0].tagged())[0];
            }
            if (!many) HIP_TRY(slhc::csr_sort_weights(edges, t, mst_src, mst_dst, mst_w, s));
            else if (edges > 0)
                HIP_TRY(slhc::edge_sort(ws.e_lo, ws.e_hi, ws.e_w, edges, (int)V, ws.keys_a, ws.keys_b, ws.vals_a, ws.vals_b,
                                        ws.sort_temp, ws.sort_temp_bytes, mst_src, mst_dst, mst_w, slhc::EdgeCopies{}, s));
            HIP_TRY(mail[0].fetch(f.words + slhc::CSR_ERROR, 1, ended));
        }
        const int32_t check = ended[0];
        mail[0].box.idle();
        mail[1].box.idle();
        rc2 = state(check);
        if (rc2 != SLHC_OK) return rc2;
        *n_edges = edges;
        if (rounds) *rounds = nrounds;
        return SLHC_OK;
    });
}

// (a search that evaluates every pair, and the list kernels, which run where the half-precision engine does not fit, need no more
// than the words per row)
static size_t fused_1nn_layout(void* ws, int64_t m, int64_t n, int32_t d, float** hq, float** hy, unsigned long long** keys, NearWs* near,
                               size_t most = NO_LIMIT)
{
    Carver c(ws);
    *hq = c.take<float>((size_t)m);
    *hy = c.take<float>((size_t)n);
    *keys = c.take<unsigned long long>((size_t)m);
    if (!slhc::direct_1nn_alone(m, n, d)) near->carve(c, n, m, d, 1, false, most);
    return c.off;
}

int slhc_fused_1nn_workspace_bytes(int64_t m, int64_t n, int32_t d, size_t* bytes)
{
    return guarded([&]() -> int {
        if (!bytes) { set_err("bytes is NULL"); return SLHC_INVALID_ARG; }
        if (m < 1 || n < 1 || d < 1) { set_err("need m >= 1, n >= 1, d >= 1"); return SLHC_INVALID_ARG; }
        if (m * (int64_t)d > 2147483647LL || n * (int64_t)d > 2147483647LL) { set_err("m*d or n*d exceeds 2^31-1"); return SLHC_UNSUPPORTED; }
        float *hq, *hy; unsigned long long* keys;
        NearWs near;
        *bytes = fused_1nn_layout(nullptr, m, n, d, &hq, &hy, &keys, &near);
        return SLHC_OK;
    });
}

int slhc_fused_1nn(const float* Q, int64_t m, const float* Y, int64_t n, int32_t d, int32_t* out_idx,
                   float* out_dist, void* workspace, size_t workspace_bytes, void* stream)
{
    return guarded([&]() -> int {
        if (!Q || !Y || !out_idx || !out_dist || !workspace) { set_err("NULL pointer argument"); return SLHC_INVALID_ARG; }
        if (m < 1 || n < 1 || d < 1) { set_err("need m >= 1, n >= 1, d >= 1"); return SLHC_INVALID_ARG; }
        if (m * (int64_t)d > 2147483647LL || n * (int64_t)d > 2147483647LL) { set_err("m*d or n*d exceeds 2^31-1"); return SLHC_UNSUPPORTED; }
        float *hq, *hy; unsigned long long* keys;
        NearWs near;
        const size_t need = fused_1nn_layout(workspace, m, n, d, &hq, &hy, &keys, &near, workspace_bytes);
        if (workspace_bytes < need) { set_err("workspace %zu < %zu bytes", workspace_bytes, need); return SLHC_WORKSPACE_TOO_SMALL; }
        hipStream_t s = static_cast<hipStream_t>(stream);
        slhc::SweepParams p{};
        if (slhc::direct_1nn_wanted(m, n, d)) {
            HIP_TRY(slhc::direct_1nn(Q, (int)m, (int)m, nullptr, Y, (int)n, d, nullptr, out_idx, out_dist, keys, s));
            return SLHC_OK;
        }
        if (near.ok) {
            HIP_TRY(slhc::near_stats(Y, (int)n, d, near.b, nullptr, 0, s));
            HIP_TRY(slhc::near_make(Y, (int)n, d, nullptr, (int)n, nullptr, near.b, near.c, hy, nullptr, s));
            HIP_TRY(slhc::near_make(Q, (int)m, d, nullptr, (int)m, nullptr, near.b, near.q, hq, nullptr, s));
            slhc::NearProblem a{};
            a.Xq = Q; a.Xc = Y; a.d = d; a.k = 1;
            a.nq = a.nq_rows = (int)m; a.nc = (int)n;
            a.out_idx = out_idx; a.out_dist = out_dist;
            HIP_TRY(slhc::near_search(a, near.q, near.c, near.b, s));
            p.todo = near.b.todo;
        } else {
            HIP_TRY(slhc::launch_half_norms(Q, (int)m, d, hq, s));
            HIP_TRY(slhc::launch_half_norms(Y, (int)n, d, hy, s));
        }
        p.Xq = Q; p.hq = hq; p.NQ = (int)m;
        p.Xc = Y; p.hc = hy; p.NC = (int)n;
        p.d = d; p.k = 1;
        p.out_idx = out_idx; p.out_dist = out_dist;
        if (p.todo) HIP_TRY(slhc::launch_knn_sweep(p, s));
        else HIP_TRY(slhc::launch_segmented_1nn(p, keys, s));
        return SLHC_OK;
    });
}

namespace {
struct FlatWs {
    int32_t *above, *counts;
    unsigned char* joined;
    size_t bytes;
    FlatWs(void* ws, int64_t N)
    {
        Carver c(ws);
        above = c.take<int32_t>((size_t)N + 4);                // (read four words and sixteen marks at a time)
        joined = c.take<unsigned char>((size_t)N + 16);
        counts = c.take<int32_t>(slhc::flat_clusters_counts(N));
        bytes = std::max(c.off, 3 * up(2 * (size_t)N * sizeof(int32_t)));       // (the larger: what is asked for has not changed)
    }
};
}  // namespace

int slhc_flat_clusters_workspace_bytes(int64_t N, size_t* bytes)
{
    return guarded([&]() -> int {
        if (!bytes) { set_err("bytes is NULL"); return SLHC_INVALID_ARG; }
        if (N < 2) { set_err("need N >= 2 (N=%lld)", (long long)N); return SLHC_INVALID_ARG; }
        if (N > 1073741823LL) { set_err("2N exceeds 2^31-1"); return SLHC_UNSUPPORTED; }
        *bytes = FlatWs(nullptr, N).bytes;
        return SLHC_OK;
    });
}

int slhc_flat_clusters(const int32_t* children, int64_t N, int64_t n_clusters, int32_t* labels,
                       void* workspace, size_t workspace_bytes, void* stream)
{
    return guarded([&]() -> int {
        if (!children || !labels || !workspace) { set_err("NULL pointer argument"); return SLHC_INVALID_ARG; }
        if (N < 2) { set_err("need N >= 2 (N=%lld)", (long long)N); return SLHC_INVALID_ARG; }
        if (N > 1073741823LL) { set_err("2N exceeds 2^31-1"); return SLHC_UNSUPPORTED; }
        if (n_clusters < 1 || n_clusters > N) { set_err("need 1 <= n_clusters <= N (n_clusters=%lld)", (long long)n_clusters); return SLHC_INVALID_ARG; }
        const FlatWs w(workspace, N);
        if (workspace_bytes < w.bytes) { set_err("workspace %zu < %zu bytes", workspace_bytes, w.bytes); return SLHC_WORKSPACE_TOO_SMALL; }
        HIP_TRY(slhc::flat_clusters(children, (int)N, (int)n_clusters, labels, w.above, w.joined, w.counts, static_cast<hipStream_t>(stream)));
        return SLHC_OK;
    });
}

int slhc_workspace_bytes(int64_t N, int32_t d, int32_t k, size_t* bytes)
{
    return guarded([&]() -> int {
        if (!bytes) { set_err("bytes is NULL"); return SLHC_INVALID_ARG; }
        const int rc = check_shape(N, d, k, true);
        if (rc != SLHC_OK) return rc;
        *bytes = padded_copy_bytes(N, d) + SlhcWs(nullptr, N, working_columns(N, d), k, true).bytes;
        return SLHC_OK;
    });
}

int slhc_slhc(const float* X, int64_t N, int32_t d, int32_t k, int32_t* mst_src, int32_t* mst_dst,
              float* mst_w, int32_t* children, float* heights, int32_t* sizes, slhc_stats* stats,
              void* workspace, size_t workspace_bytes, void* stream)
{
    return guarded([&]() -> int {
        // Below this size the row order costs more than the skipped tiles save.  The line is where the two paths crossed with the list
        // kernels (four kinds of data between 4096 and 65 536 rows: between 24 000 and 32 000 rows) and part of the interface.  With the
        // half-precision engine they cross later: 24 576 x 64 1.3 to 1.4 ms with every tile and 3.3 to 4.3 ms in the row order, 65 536 x 64
        // 3.7 to 4.5 and 5.1 to 7.4 ms; tight clusters 2.5 and 7.2, 12.3 and 10.3 ms.
        return slhc_slhc_opt(X, N, d, k, mst_src, mst_dst, mst_w, children, heights, sizes, stats, workspace,
                             workspace_bytes, stream, N >= SLHC_AUTO_PRUNE_MIN_ROWS ? SLHC_PRUNE : 0u);
    });
}

int slhc_slhc_opt(const float* X, int64_t N, int32_t d, int32_t k, int32_t* mst_src, int32_t* mst_dst,
                  float* mst_w, int32_t* children, float* heights, int32_t* sizes, slhc_stats* stats,
                  void* workspace, size_t workspace_bytes, void* stream, uint32_t flags)
{
    return guarded([&]() -> int {
        if (!X || !mst_src || !mst_dst || !mst_w || !children || !heights || !sizes || !workspace) {
            set_err("NULL pointer argument");
            return SLHC_INVALID_ARG;
        }
        const int rc = check_shape(N, d, k, true);
        if (rc != SLHC_OK) return rc;
        int32_t dw = working_columns(N, d);
        size_t head = padded_copy_bytes(N, d);
        const size_t need = head + SlhcWs(nullptr, N, dw, k, true, workspace_bytes > head ? workspace_bytes - head : 0).bytes;
        if (workspace_bytes < need) { set_err("workspace %zu < %zu bytes", workspace_bytes, need); return SLHC_WORKSPACE_TOO_SMALL; }
        // Where every pair is evaluated the list kernels see a panel or two at most: the rows as they are.  (Without an engine in the workspace
        // they see all of them.)
        if (!(flags & (SLHC_PRUNE | SLHC_FP32_FILTER | SLHC_PANEL_ORDER)) && slhc::direct_knn_wanted(N, d, k, true) > 0 &&
            SlhcWs(nullptr, N, d, k, true, workspace_bytes).knn->near.ok) { dw = d; head = 0; }
        const float* X_given = X;
        if (dw != d) {
            const int rp = pad_columns(X, N, d, dw, static_cast<float*>(workspace), static_cast<hipStream_t>(stream));
            if (rp != SLHC_OK) return rp;
            X = static_cast<const float*>(workspace);
        }
        return run_slhc(X, N, dw, k, mst_src, mst_dst, mst_w, children, heights, sizes, stats,
                        static_cast<unsigned char*>(workspace) + head, workspace_bytes - head, static_cast<hipStream_t>(stream), flags, true, X_given, d);
    });
}

}  // extern "C"

namespace {

// The whole pipeline on validated arguments.  `with_order` selects the workspace layout (the
// nested call that clusters the pivots of the row order runs without one).  X_given: the rows without columns of zeros.
int run_slhc(const float* X, int64_t N, int32_t d, int32_t k, int32_t* mst_src, int32_t* mst_dst, float* mst_w,
             int32_t* children, float* heights, int32_t* sizes, slhc_stats* stats, void* workspace, size_t workspace_bytes,
             hipStream_t s, uint32_t flags, bool with_order, const float* X_given, int32_t d_given)
{
    int rc = SLHC_OK;
    SlhcWs ws(workspace, N, d, k, with_order, workspace_bytes);
    if (ws.bytes > workspace_bytes) { set_err("workspace %zu < %zu bytes", workspace_bytes, ws.bytes); return SLHC_WORKSPACE_TOO_SMALL; }
    slhc_stats st;
    std::memset(&st, 0, sizeof(st));
    const double t_begin = now_ms();
    PhaseLog log(s);

    // ---- k-NN graph (Alg. "cuSLINK Algorithm", first step)
    EventPair ev_norm, ev_order, ev_knn, ev_conn;
    const bool timed = stats != nullptr || log.on;
    if (timed) {
        HIP_TRY(ev_norm.create());
        HIP_TRY(ev_order.create());
        HIP_TRY(ev_knn.create());
        HIP_TRY(ev_conn.create());
    }
    bool pruned = false;
    KnnWs& kws = *ws.knn;
    rc = run_knn(X, N, d, k, ws.nbr_idx, ws.nbr_dist, kws, s, flags, &pruned, timed ? &ev_norm : nullptr, timed ? &ev_order : nullptr,
                 timed ? &ev_knn : nullptr);
    if (rc != SLHC_OK) return rc;
    // The pinned staging of the host's dendrogram pass is taken here, while the k-NN sweep runs.
    const bool host_dendrogram = children && N < DENDROGRAM_DEVICE_MIN_ROWS;
    PinnedHost pin_edges(s);
    if (host_dendrogram) HIP_TRY(pin_edges.alloc(5 * (size_t)(N - 1) * sizeof(int32_t)));
    Mailbox mail(s);
    HIP_TRY(mail.open());
    unsigned long long h_surv[8];
    HIP_TRY(mail.fetch(kws.counters, 10, h_surv));
    if ((h_surv[4] & 2ull) != 0) { set_err("a work item of the k-NN sweep waited for its predecessor in vain"); return SLHC_INTERNAL; }
    if ((h_surv[4] & 0xffffffffull) != 0) { set_err("a row of X is not finite (NaN, infinity, or a squared norm beyond float32)"); return SLHC_NONFINITE; }
    st.knn_filter_survivors = (int64_t)h_surv[0];
    const unsigned long long tiles_all = (unsigned long long)((N + 127) / 128) * (unsigned long long)((N + 127) / 128);
    st.knn_tile_steps = (int64_t)(kws.near_done && !pruned ? tiles_all : h_surv[2]);
#ifdef SLHC_STUDY_PANEL_STEPS
    if (pruned) {
        const int T_ = (kws.order.Ns + 127) / 128;
        std::vector<int> hs((size_t)T_ * 2);
        HIP_TRY(hipMemcpy(hs.data(), kws.order.qslot, hs.size() * 4, hipMemcpyDeviceToHost));
        long long tot = 0; int longest = 0, most = 0;
        for (int i = 0; i < T_; ++i) { tot += hs[(size_t)T_ + i]; if (hs[(size_t)T_ + i] > longest) longest = hs[(size_t)T_ + i]; if (hs[(size_t)i] > most) most = hs[(size_t)i]; }
        std::fprintf(stderr, "[study] k-NN sweep: %d panels, kcycles %lld (per WG slot %.0f), longest panel %d kcycles, most steps %d, kernel %.2f ms\n",
                     T_, tot, tot / 512.0, longest, most, ev_knn.ms());
    }
#endif
    st.ms_norm_kernel = ev_norm.ms();
    st.ms_order = ev_order.ms();
    st.ms_knn_kernel = ev_knn.ms();
    log.mark("k-NN graph of %lld rows: order %.2f ms, sweep %.2f ms, %llu tile steps", (long long)N, st.ms_order,
             st.ms_knn_kernel, (unsigned long long)st.knn_tile_steps);
    const double t_knn = now_ms();
    st.ms_knn = (float)(t_knn - t_begin);

    // ---- certified Boruvka with connection queries (Alg. "MST Algorithm" + "connect_graph")
    slhc::ForestState f{};
    f.N = (int)N; f.k = k;
    f.nbr_idx = ws.nbr_idx; f.nbr_dist = ws.nbr_dist;
    f.colour = ws.colour; f.ptr = ws.ptr; f.ext_idx = ws.ext_idx; f.ext_dist = ws.ext_dist; f.ext_low = ws.ext_low;
    f.cand_w = ws.cand_w; f.cand_u = ws.cand_u; f.best_w = ws.best_w; f.best_e = ws.best_e;
    f.hook = ws.hook; f.qlist = ws.qlist; f.counters = ws.counters;
    f.e_lo = ws.e_lo; f.e_hi = ws.e_hi; f.e_w = ws.e_w;
    // few vertices: whole rounds in one launch (see k_forest_small), which stops where rows have to be queried
    const bool small_forest = N <= slhc::FOREST_SMALL_MAX;
    if (!small_forest) HIP_TRY(slhc::forest_init(f, s));
    int32_t h_cnt[16] = {0};
    int edges = 0;
    int max_rounds = 2;
    for (int64_t t = 1; t < N; t *= 2) ++max_rounds;
    double ms_connect = 0.0;
    bool first_connect = true;
    unsigned long long near_tile_steps = 0;        // of connection sweeps in half precision
    // cleared when pruning stops paying: at once when the k-NN sweep already had to multiply more
    // than a quarter of all tile pairs (the data has no structure at the scale of a tile), else by
    // the per-round test below
    const unsigned long long tiles_1d = (unsigned long long)((N + 127) / 128);
    bool connect_pruned = (unsigned long long)st.knn_tile_steps * 4 <= tiles_1d * tiles_1d;
    unsigned long long conn_steps_seen = 0;
    double prev_steps_per_panel = 0.0;     // tile steps per query panel in the last pruned round
    // tile steps per panel that holds a queried row, as far as known: the k-NN sweep's at first, then the last
    // pruned round's; decides into how many parts a panel's scan is worth splitting
    double steps_per_used_panel = pruned ? (double)st.knn_tile_steps / (double)((kws.order.Ns + 127) / 128) : 0.0;
    long long used_panels_round = 0;
    st.components_after_knn = 1;
    // One read-back per round: the scan of the lists for round r+1 is enqueued right behind the relabelling
    // of round r, so the counters that come back carry the edges committed so far, whether the hook
    // chains were followed to their end, and the number of rows the next round has to query.
    auto enqueue_scan = [&]() -> int {
        HIP_TRY(slhc::forest_scan_lists(f, s));
        HIP_TRY(slhc::forest_classify(f, s));
        return SLHC_OK;
    };
    auto read_counters = [&]() -> int {
        HIP_TRY(slhc::forest_publish(f, reinterpret_cast<int32_t*>(mail.words()), (int32_t)mail.next(), s));
        HIP_TRY(mail.wait());
        std::memcpy(h_cnt, mail.words() + 1, 8 * sizeof(int32_t));
        if (h_cnt[3] != 0) {
            // what the failed check saw (counters[16..22], written by the thread whose report came first)
            HIP_TRY(mail.fetch(ws.counters + 16, 7, h_cnt + 8));
            set_err("forest state check %d failed in round %d (%s rounds, %d connection rounds): %d %d %d %d %d %d", h_cnt[3],
                    st.boruvka_rounds, pruned ? "pruned" : "every-tile", st.connect_rounds,
                    h_cnt[9], h_cnt[10], h_cnt[11], h_cnt[12], h_cnt[13], h_cnt[14]);
            return SLHC_INTERNAL;
        }
        return SLHC_OK;
    };
    if (small_forest) HIP_TRY(slhc::forest_small(f, true, s));
    else {
        rc = enqueue_scan();
        if (rc != SLHC_OK) return rc;
    }
    bool conn_pending = false;
    for (;;) {
        rc = read_counters();
        if (rc != SLHC_OK) return rc;
        if (conn_pending) {
            conn_pending = false;
            const float ms = ev_conn.ms();
            st.ms_connect_kernels += ms;
            ms_connect += ms;
        }
        if (small_forest) {
            if (h_cnt[1] < edges || h_cnt[1] > N - 1 || (h_cnt[1] < N - 1 && h_cnt[0] == 0)) { set_err("rounds left %d edges (had %d)", h_cnt[1], edges); return SLHC_INTERNAL; }
            edges = h_cnt[1];
            st.boruvka_rounds = h_cnt[6] - 1;            // (counted again below)
            if (edges == N - 1) { ++st.boruvka_rounds; break; }
        } else if (st.boruvka_rounds > 0) {
            if (h_cnt[2] != 0) {
                // a hook chain longer than one launch follows (64 hooks): finish
                // it with the host in the loop, relabel, and scan again under the final colours
                for (int jumps = 0; h_cnt[2] != 0; ++jumps) {
                    if (jumps > 64) { set_err("component hooks do not form a forest"); return SLHC_INTERNAL; }
                    hipLaunchKernelGGL(k_zero_words, dim3(1), dim3(64), 0, s, reinterpret_cast<uint32_t*>(ws.counters + 2), 1);
                    HIP_TRY(hipGetLastError());
                    HIP_TRY(slhc::forest_jump(f, 32, true, s));
                    rc = read_counters();
                    if (rc != SLHC_OK) return rc;
                }
                HIP_TRY(slhc::forest_follow(f, s));
                rc = enqueue_scan();
                if (rc != SLHC_OK) return rc;
                rc = read_counters();
                if (rc != SLHC_OK) return rc;
            }
            if (h_cnt[1] <= edges || h_cnt[1] > N - 1) { set_err("round added %d edges (total %d)", h_cnt[1] - edges, h_cnt[1]); return SLHC_INTERNAL; }
            edges = h_cnt[1];
            if (edges == N - 1) break;
        }
        if (st.boruvka_rounds >= max_rounds) { set_err("no single component after %d rounds", max_rounds); return SLHC_INTERNAL; }
        ++st.boruvka_rounds;
        const int nq = h_cnt[0];
        if (h_cnt[3] != 0 || nq < 0 || nq > N) { set_err("forest state check %d failed (nq=%d)", h_cnt[3], nq); return SLHC_INTERNAL; }
        if (nq > 0) {
            const double tc0 = now_ms();
            if (first_connect) { st.components_after_knn = (int32_t)(N - edges); first_connect = false; }
            ++st.connect_rounds;
            const bool round_pruned = pruned && connect_pruned;
            const bool round_ordered = round_pruned && kws.near_order_ready;       // pruned by the half-precision engine
            if (round_ordered) {
                const OrderWs& o = kws.order;
                HIP_TRY(slhc::order_gather_i32(ws.colour, o.perm, o.Ns, (int)N, -1, o.near_colour, s));
                HIP_TRY(slhc::order_tile_colours(o.near_colour, o.Ns, o.tile_colour, s));
            } else if (round_pruned) {
                // colours in the reordered copy and one colour summary per tile
                const OrderWs& o = kws.order;
                HIP_TRY(slhc::order_gather_i32(ws.colour, o.perm, o.Ns, (int)N, -1, o.colour_s, s));
                HIP_TRY(slhc::order_tile_colours(o.colour_s, o.Ns, o.tile_colour, s));
                // rows per component (vals_b is free until the edge sort): which components may lower
                // their shared threshold during the sweep
                if (N < LOWER_ALL_ROWS) {
                    HIP_TRY(slhc::order_fill_i32(reinterpret_cast<int32_t*>(ws.vals_b), (int)N, 0, s));
                    HIP_TRY(slhc::forest_component_sizes(o.colour_s, o.Ns, (int)N, reinterpret_cast<int32_t*>(ws.vals_b), s));
                }
            }
            float ms_round_kernels = 0.f;
            // one cross-colour 1-NN sweep for `n` listed rows, and its answers applied to the forest
            auto sweep_rows = [&](const int32_t* rows, int n) -> int {
                slhc::SweepParams p{};
                p.d = d; p.k = 1;
                p.out_idx = ws.q_idx; p.out_dist = ws.q_dist;
                p.m = n;
                p.survivors = kws.counters + 1;
                p.tiles_done = kws.counters + 3;
                if (round_pruned) {
                    // the queried rows marked in place so that query panels coincide with candidate tiles
                    const OrderWs& o = kws.order;
                    HIP_TRY(slhc::order_fill_i32(o.qslot, o.Ns, -1, s));
                    HIP_TRY(slhc::order_scatter_slots(o.inv, rows, n, (int)N, o.Ns, o.qslot, s));
                    p.Xq = p.Xc = o.Xs; p.hq = p.hc = o.hs; p.NQ = p.NC = o.Ns;
                    p.qslot = o.qslot;
                    p.c_id = o.perm;
                    p.tile_c = o.tile_c; p.tile_r = o.tile_r; p.gap_ws = o.gap_ws;
                    p.tile_gap = (flags & SLHC_NO_TILE_TABLE) ? nullptr : o.tile_gap;
                    p.tile_colour = o.tile_colour;
                    p.comp_count = (int)N;
                    p.panel_counter = reinterpret_cast<unsigned int*>(kws.counters + 8);
                    hipLaunchKernelGGL(k_zero_words, dim3(1), dim3(64), 0, s, p.panel_counter, 1);
                    HIP_TRY(hipGetLastError());
                    // what the forest already knows of every component's lightest edge; lowered by the search (vals_a is free
                    // until the edge sort)
                    HIP_TRY(hipMemcpyAsync(ws.vals_a, ws.best_w, (size_t)N * sizeof(uint32_t), hipMemcpyDeviceToDevice, s));
                    p.comp_best = ws.vals_a;
                }
                if (round_ordered) {
                    p.qcolour = p.ccolour = kws.order.near_colour;
                } else if (round_pruned) {
                    const OrderWs& o = kws.order;
                    // A launch with few panels is as long as its longest panel, and a panel whose queries admit
                    // thousands of tiles outlasts the others several times over: with fewer non-empty panels
                    // than SPLIT_ITEMS_TARGET, every panel's scan is split into parts (see the kernel).
                    int32_t* used = ws.counters + 12;
                    hipLaunchKernelGGL(k_zero_words, dim3(1), dim3(64), 0, s, reinterpret_cast<uint32_t*>(used), 1);
                    HIP_TRY(hipGetLastError());
                    HIP_TRY(slhc::order_count_used_tiles(o.qslot, o.Ns, used, o.tile_list, s));
                    HIP_TRY(mail.fetch(used, 1, h_cnt + 6));
                    const int used_panels = h_cnt[6] > 0 ? h_cnt[6] : 1;
                    used_panels_round += used_panels;
                    int parts = SPLIT_ITEMS_TARGET / used_panels;
                    const int worth = (int)(steps_per_used_panel / SPLIT_MIN_STEPS);      // a part should have some tiles to multiply
                    if (parts > worth) parts = worth;
                    p.segments = parts < 2 ? 1 : (parts > SPLIT_MAX_PARTS ? SPLIT_MAX_PARTS : parts);
                    if (flags & SLHC_SPLIT_SCANS) p.segments = 5;
                    if (h_cnt[6] < 0 || h_cnt[6] > (o.Ns + 127) / 128) { set_err("bad count of queried tiles %d", h_cnt[6]); return SLHC_INTERNAL; }
                    p.panel_list = o.tile_list; p.panel_list_n = h_cnt[6];
                    if (kws.order_split_connect) { p.Xq_split = p.Xc_split = o.Xs_split; p.hq_split = p.hc_split = o.hs_split; }
                    p.qcolour = p.ccolour = o.colour_s;
                    // thresholds shared by the queries of a component, in a working copy that the sweep lowers further as
                    // its queries find lighter edges
#ifndef SLHC_STUDY_NO_LOWERING
                    p.comp_best_lower = ws.vals_a;      // lowered in place; forest_apply_queries reads the final values
                    p.comp_lower_factor = LOWER_FACTOR;
                    p.comp_size = N < LOWER_ALL_ROWS ? reinterpret_cast<const int32_t*>(ws.vals_b) : nullptr;
                    p.comp_lower_min_size = LOWER_MIN_ROWS;
#endif
#ifdef SLHC_PHASE_TIMERS
                    p.phase_cycles = kws.counters + 24;
#endif
                } else {
                    p.Xq = p.Xc = X; p.hq = p.hc = kws.hn; p.NQ = p.NC = (int)N;
                    p.qcolour = p.ccolour = ws.colour;
                    p.rows = rows;
                    if (!(flags & SLHC_PANEL_ORDER)) {
                        p.carry_ws = kws.carry_ws; p.carry_ws_words = kws.carry_ws_words;
                        p.carry_fault = reinterpret_cast<unsigned int*>(kws.counters + 4);
                    }
                    if (kws.Xsplit && !(flags & SLHC_FP32_FILTER) && !near_wanted(kws.near, flags)) {
                        if (!kws.split_ready) {          // (a pruned k-NN sweep did not need it)
                            const int rs = make_split_copy(X, N, d, kws, s);
                            if (rs != SLHC_OK) return rs;
                        }
                        // (a launch that ends in a kernel with float32 products takes hq / hc)
                        p.Xq_split = p.Xc_split = kws.Xsplit; p.hq_split = p.hc_split = kws.hn_split;
                    }
                }
#ifdef SLHC_STUDY_PANEL_STEPS
                int* study_steps = reinterpret_cast<int*>(kws.order.gap_ws);    // unused while the table of tile pairs serves
                const int study_panels = (kws.order.Ns + 127) / 128;
                if (round_pruned) { HIP_TRY(hipMemsetAsync(study_steps, 0, (size_t)study_panels * 8, s)); p.panel_steps = study_steps; }
#endif
                if (timed) HIP_TRY(hipEventRecord(ev_conn.a, s));
                uint32_t* thresholds = round_pruned ? ws.vals_a : nullptr;
                if (round_ordered) {
                    const OrderWs& o = kws.order;
                    const int T = (o.Ns + 127) / 128;
                    // the listed rows by position (tmp_a .. tmp_c are free since the order was made)
                    int32_t* sorted = const_cast<int32_t*>(rows);
                    int32_t* pos = reinterpret_cast<int32_t*>(o.tmp_b);
                    hipLaunchKernelGGL(k_slot_counts, dim3((unsigned)((T + 3) / 4)), dim3(256), 0, s, o.qslot, o.Ns, T, o.tile_list);
                    hipLaunchKernelGGL(k_slot_offsets, dim3(1), dim3(1024), 0, s, o.tile_list, T);
                    hipLaunchKernelGGL(k_slot_rows, dim3((unsigned)((T + 3) / 4)), dim3(256), 0, s, o.qslot, o.perm, o.Ns, T, o.tile_list, n, sorted, pos);
                    HIP_TRY(hipGetLastError());
                    slhc::NearOrder order = near_order_of(o);
                    order.all.colour = o.near_colour;
                    order.tile_steps = kws.counters + 3;
                    slhc::NearLink a{};
                    a.X = X; a.d = d; a.n_rows = (int)N; a.rows = sorted; a.n = n; a.colour = ws.colour;
                    a.threshold = ws.vals_a;
                    a.out_idx = ws.q_idx; a.out_dist = ws.q_dist; a.out_low = ws.q_low; a.evaluated = reinterpret_cast<int32_t*>(ws.vals_b);
                    a.rows_left = reinterpret_cast<int32_t*>(ws.keys_a); a.slot_left = a.rows_left + N;
                    a.reach_left = reinterpret_cast<float*>(ws.keys_b);
                    a.qpos = pos; a.pos_left = reinterpret_cast<int32_t*>(o.tmp_c); a.counts_left = kws.near.q.count;
                    a.edge_at = kws.near.q.left; a.best_at = o.best_at; a.threshold0 = o.tmp_a;
                    HIP_TRY(slhc::near_link_ordered(a, order, kws.near.b, s));
                    hipLaunchKernelGGL(k_sum_words, dim3(16), dim3(256), 0, s, reinterpret_cast<const int32_t*>(ws.vals_b), n, kws.counters + 1);
                    HIP_TRY(hipGetLastError());
                    p.todo = kws.near.b.todo;
                    p.tiles_done = nullptr;
                    HIP_TRY(slhc::launch_cross_1nn_sweep(p, s));
                } else if (!round_pruned && near_wanted(kws.near, flags) && slhc::direct_near_wanted(n, N, d_given)) {
                    // (keys_a is free until the edge sort)
                    HIP_TRY(slhc::direct_near(X_given, n, (int)N, rows, X_given, (int)N, d_given, ws.colour, ws.q_idx, ws.q_dist, ws.keys_a, kws.counters + 1, s));
                    near_tile_steps += (unsigned long long)((n + 127) / 128) * tiles_1d;
                } else if (!round_pruned && near_wanted(kws.near, flags)) {
                    const NearWs& near = kws.near;
                    if (!kws.near_ready) {
                        HIP_TRY(slhc::near_stats(X, (int)N, d, near.b, nullptr, 0, s));
                        HIP_TRY(slhc::near_make(X, (int)N, d, nullptr, (int)N, nullptr, near.b, near.c, kws.hn, nullptr, s));
                        kws.near_ready = true;
                    }
                    slhc::NearCopy q = near.q;
                    q.rows = n; q.tiles = slhc::near_tiles(n); q.in_order = true;
                    kws.near_order_ready = false;           // (in whose memory the copy of the queries may lie)
                    HIP_TRY(slhc::near_colours(near.c, ws.colour, s));
                    // (the arrays of the edge sort and of the thresholds are free until then)
                    HIP_TRY(hipMemcpyAsync(ws.vals_a, ws.best_w, (size_t)N * sizeof(uint32_t), hipMemcpyDeviceToDevice, s));
                    slhc::NearLink a{};
                    a.X = X; a.d = d; a.n_rows = (int)N; a.rows = rows; a.n = n; a.colour = ws.colour;
                    a.threshold = ws.vals_a;
                    a.out_idx = ws.q_idx; a.out_dist = ws.q_dist; a.out_low = ws.q_low; a.evaluated = reinterpret_cast<int32_t*>(ws.vals_b);
                    a.rows_left = reinterpret_cast<int32_t*>(ws.keys_a); a.slot_left = a.rows_left + N;
                    a.reach_left = reinterpret_cast<float*>(ws.keys_b);
                    HIP_TRY(slhc::near_link(a, q, near.c, near.b, s));
                    thresholds = ws.vals_a;
                    hipLaunchKernelGGL(k_sum_words, dim3(16), dim3(256), 0, s, reinterpret_cast<const int32_t*>(ws.vals_b), n, kws.counters + 1);
                    HIP_TRY(hipGetLastError());
                    near_tile_steps += (unsigned long long)((n + 127) / 128) * tiles_1d;
                    p.todo = near.b.todo;
                    p.carry_ws = nullptr;
                    HIP_TRY(slhc::launch_cross_1nn_sweep(p, s));
                } else
                // keys_a / keys_b are free until the edge sort (the two-phase split above keeps its row lists in keys_a,
                // in pruned rounds only)
                HIP_TRY(slhc::launch_segmented_cross_1nn(p, round_pruned ? ws.keys_b : ws.keys_a, s));
                if (timed) HIP_TRY(hipEventRecord(ev_conn.b, s));
                HIP_TRY(slhc::forest_apply_queries(f, rows, ws.q_idx, ws.q_dist, thresholds && (round_ordered || !round_pruned) ? ws.q_low : nullptr, n, thresholds, s));
                // (every-tile rounds leave the check to the next reading of the counters)
                h_cnt[7] = 0;
                if (round_pruned && !round_ordered) HIP_TRY(mail.fetch(ws.counters + 3, 1, h_cnt + 7));
                if (h_cnt[7] == 14) {
                    // an answer inside the query's own component: say what the sweep was given
                    HIP_TRY(hipMemcpy(h_cnt + 8, ws.counters + 16, 7 * sizeof(int32_t), hipMemcpyDeviceToHost));
                    const int q = h_cnt[9], v = h_cnt[10], u = h_cnt[11];
                    int dv[12] = {-9, -9, -9, -9, -9, -9, -9, -9, -9, -9, -9, -9};
                    auto peek = [&](const void* base, long long index, int* out) {
                        if (base && index >= 0) (void)hipMemcpy(out, static_cast<const int32_t*>(base) + index, 4, hipMemcpyDeviceToHost);
                    };
                    peek(ws.colour, v, &dv[0]); peek(ws.colour, u, &dv[1]);
                    peek(ws.q_idx, q, &dv[2]); peek(rows, q, &dv[3]);
                    if (round_pruned) {
                        const OrderWs& o = kws.order;
                        peek(o.inv, v, &dv[4]); peek(o.inv, u, &dv[5]);
                        if (dv[4] >= 0 && dv[4] < o.Ns) { peek(o.colour_s, dv[4], &dv[6]); peek(o.qslot, dv[4], &dv[8]); peek(o.perm, dv[4], &dv[10]); }
                        if (dv[5] >= 0 && dv[5] < o.Ns) { peek(o.colour_s, dv[5], &dv[7]); peek(o.qslot, dv[5], &dv[9]); peek(o.perm, dv[5], &dv[11]); }
                    }
                    set_err("sweep answer inside the query's component: round %d, %s sweep of %d rows in %d parts, q %d v %d u %d; "
                            "colour v %d u %d, q_idx[q] %d rows[q] %d, position v %d u %d, colour_s %d %d, qslot %d %d, perm %d %d",
                            st.boruvka_rounds, round_pruned ? "pruned" : "every-tile", n, p.segments, q, v, u,
                            dv[0], dv[1], dv[2], dv[3], dv[4], dv[5], dv[6], dv[7], dv[8], dv[9], dv[10], dv[11]);
                    return SLHC_INTERNAL;
                }
#ifdef SLHC_STUDY_PANEL_STEPS
                if (round_pruned) {
                    std::vector<int> hs((size_t)study_panels * 2);
                    HIP_TRY(hipMemcpy(hs.data(), study_steps, hs.size() * 4, hipMemcpyDeviceToHost));
                    std::vector<int> order_((size_t)study_panels);
                    for (int i = 0; i < study_panels; ++i) order_[(size_t)i] = i;
                    std::sort(order_.begin(), order_.end(), [&](int a, int b) { return hs[(size_t)study_panels + a] > hs[(size_t)study_panels + b]; });
                    long long tot_steps = 0, tot_cyc = 0; int used = 0;
                    for (int i = 0; i < study_panels; ++i) { tot_steps += hs[(size_t)i]; tot_cyc += hs[(size_t)study_panels + i]; used += hs[(size_t)study_panels + i] > 0; }
                    std::fprintf(stderr, "[study] %d rows, %d panels used, parts %d, steps %lld, kcycles %lld (per WG slot %.0f), kernel %.2f ms\n", n, used, p.segments, tot_steps, tot_cyc, tot_cyc / 512.0, ev_conn.ms());
                    for (int r = 0; r < 12; ++r) { const int i = order_[(size_t)r]; std::fprintf(stderr, "[study]   panel %d: steps %d kcycles %d\n", i, hs[(size_t)i], hs[(size_t)study_panels + i]); }
                }
#endif
                // (the list kernels' pruned sweeps have been waited for above; others are timed when later counters arrive)
                if (timed && round_pruned && !round_ordered) ms_round_kernels += ev_conn.ms();
                return SLHC_OK;
            };
            int queried = nq;
            const bool split_round = (flags & SLHC_SPLIT_ROUNDS)
                                         ? nq >= 256
                                         : ((int64_t)nq * 2 >= N && (int64_t)nq >= TWO_PHASE_MIN_ROWS &&
                                            prev_steps_per_panel >= TWO_PHASE_MIN_STEPS);
            if (round_pruned && !round_ordered && split_round) {
                // Two phases, for a round that queries most rows while the thresholds the forest has
                // are loose (the last pruned round multiplied hundreds of tiles per panel).  The rows
                // of every 16th panel go first; what they find lowers their components' best
                // weights, and the other rows (those the lower weights still leave on the list) then
                // run under thresholds close to the final ones, which lets their panels skip tiles.
                int32_t* part_a = reinterpret_cast<int32_t*>(ws.keys_a);      // free until the edge sort
                int32_t* part_b = part_a + N;
                int32_t* counts = ws.counters + 8;
                hipLaunchKernelGGL(k_zero_words, dim3(1), dim3(64), 0, s, reinterpret_cast<uint32_t*>(counts), 3);
                HIP_TRY(hipGetLastError());
                HIP_TRY(slhc::forest_split_queries(f, ws.qlist, nq, kws.order.inv, TWO_PHASE_STRIDE, part_a, part_b, counts, s));
                HIP_TRY(mail.fetch(counts, 2, h_cnt + 4));
                const int na = h_cnt[4], nb = h_cnt[5];
                if (na < 0 || nb < 0 || na + nb != nq) { set_err("query split lost rows (%d + %d of %d)", na, nb, nq); return SLHC_INTERNAL; }
                if (na > 0) { const int rc = sweep_rows(part_a, na); if (rc != SLHC_OK) return rc; }
                int nb_left = 0;
                if (nb > 0) {
                    HIP_TRY(slhc::forest_still_needed(f, part_b, nb, ws.qlist, counts + 2, s));
                    HIP_TRY(mail.fetch(counts + 2, 1, h_cnt + 4));
                    nb_left = h_cnt[4];
                    if (nb_left < 0 || nb_left > nb) { set_err("query re-filter kept %d of %d rows", nb_left, nb); return SLHC_INTERNAL; }
                    if (nb_left > 0) { const int rc = sweep_rows(ws.qlist, nb_left); if (rc != SLHC_OK) return rc; }
                }
                queried = na + nb_left;
            } else {
                const int rc = sweep_rows(ws.qlist, nq);
                if (rc != SLHC_OK) return rc;
            }
            st.connect_query_rows += queried;
            if (round_pruned) {
                HIP_TRY(mail.fetch(kws.counters, 8, h_surv));
                if (timed && round_ordered) ms_round_kernels += ev_conn.ms();          // (one sweep, over by now)
            } else conn_pending = timed;        // one sweep: its time is read when the next counters have arrived
            st.ms_connect_kernels += ms_round_kernels;
            if (round_pruned) ms_connect += now_ms() - tc0;
            if (round_pruned) {
                // Did skipping pay?  A pruned tile step costs more than an every-tile one (queries
                // stay aligned with tiles, so panels are partly empty, and the surviving tiles are
                // the dense ones); when a large round still multiplied more than a third of what the
                // every-tile sweep would, the remaining rounds run without pruning.
                const unsigned long long steps = h_surv[3] - conn_steps_seen;
                conn_steps_seen = h_surv[3];
                prev_steps_per_panel = (double)steps / (double)((queried + 127) / 128 > 0 ? (queried + 127) / 128 : 1);
                if (used_panels_round > 0) steps_per_used_panel = (double)steps / (double)used_panels_round;
                used_panels_round = 0;
                const unsigned long long every = (unsigned long long)((nq + 127) / 128) * (unsigned long long)((N + 127) / 128);
                // (tiles that only leave out a component's own already cost less, for lists, than they save)
                if ((int64_t)nq * 8 >= N && (round_ordered ? steps * 10 > every * 9 : steps * 3 > every)) connect_pruned = false;
            }
            if (log.on) {
                HIP_TRY(mail.fetch(kws.counters, 8, h_surv));
                int32_t left[2] = {0, queried};
                if (round_ordered || (!round_pruned && near_wanted(kws.near, flags))) HIP_TRY(mail.fetch(kws.near.b.todo, 2, left));
                log.mark("round %d: %d components, %d of %d listed rows queried, %d searched, %d panels by lists, sweeps %.2f ms, %llu tile steps so far",
                         st.boruvka_rounds, (int)(N - edges), queried, nq, left[1], left[0], ms_round_kernels, h_surv[3]);
            }
        }
        if (small_forest) { HIP_TRY(slhc::forest_small(f, false, s)); continue; }
        HIP_TRY(slhc::forest_select_edges(f, s));
        HIP_TRY(slhc::forest_commit(f, s));
        HIP_TRY(slhc::forest_follow(f, s));           // hooks -> new colours
        rc = enqueue_scan();                                  // next round's scan; its counters are read at the top
        if (rc != SLHC_OK) return rc;
    }
    HIP_TRY(mail.fetch(kws.counters, 10, h_surv));
    if ((h_surv[4] & 2ull) != 0) { set_err("a work item of a connection sweep waited for its predecessor in vain"); return SLHC_INTERNAL; }
#ifdef SLHC_PHASE_TIMERS
    if (log.on) {
        unsigned long long* h_ph = h_surv + 4;           // 64-byte staging buffer: not enough, use two copies
        for (int part = 0; part < 4; ++part) {
            HIP_TRY(hipMemcpyAsync(h_ph, kws.counters + 16 + 4 * part, 4 * sizeof(unsigned long long), hipMemcpyDeviceToHost, s));
            HIP_TRY(hipStreamSynchronize(s));
            std::fprintf(stderr, "[slhc] %s phase cycles %d..%d: %llu %llu %llu %llu\n", part < 2 ? "k-NN" : "connect",
                         4 * (part & 1), 4 * (part & 1) + 3, h_ph[0], h_ph[1], h_ph[2], h_ph[3]);
        }
    }
#endif
    st.connect_filter_survivors = (int64_t)h_surv[1];
    st.connect_tile_steps = (int64_t)(h_surv[3] + near_tile_steps);
    st.pruned = pruned ? 1 : 0;
    st.split_products = (kws.split_ready || kws.order_split_ready || kws.near_done) ? 1 : 0;
    st.half_products = kws.near_done ? 1 : 0;
    if (pruned) { st.order_pivots = kws.order.P; st.order_padded_rows = kws.order.Ns; }
    const double t_forest = now_ms();
    st.ms_connect = (float)ms_connect;
    st.ms_boruvka = (float)(t_forest - t_knn - ms_connect);

    // ---- sort by weight (Sec. 3.3.1), then the linkage arrays
    const size_t E = (size_t)(N - 1);
    // host staging: end points, children and sizes.  Kernels write and read it in place.
    int32_t* h_lo = static_cast<int32_t*>(pin_edges.p);
    int32_t* h_hi = h_lo + E;
    int32_t* h_children = h_hi + E;
    int32_t* h_sizes = h_children + 2 * E;
    slhc::EdgeCopies copies{};
    copies.heights = heights;
    if (host_dendrogram) { copies.host_lo = h_lo; copies.host_hi = h_hi; }
    HIP_TRY(slhc::edge_sort(ws.e_lo, ws.e_hi, ws.e_w, (int)(N - 1), (int)N, ws.keys_a, ws.keys_b, ws.vals_a, ws.vals_b,
                            ws.sort_temp, ws.sort_temp_bytes, mst_src, mst_dst, mst_w, copies, s));
    if (!children) {                                        // (the pivots' tree: its edges are all that is wanted)
        mail.box.idle();
        return SLHC_OK;
    }
    double t_sort = t_forest;
    if (host_dendrogram) {
        HIP_TRY(mail.fetch(ws.counters, 1, h_cnt));         // everything staged is in host memory
        t_sort = now_ms();
        if (!build_dendrogram(h_lo, h_hi, N, h_children, h_sizes)) { set_err("dendrogram: an edge of the sorted tree has an end point outside [0, N)"); return SLHC_INTERNAL; }
        log.mark("dendrogram: union-find on the host");
        HIP_TRY(slhc::linkage_upload(h_children, h_sizes, (int)E, children, sizes, s));
    } else {
        // the arrays of the forest rounds and of the sort are free by now
        slhc::DendrogramWork dw{};
        dw.lightest = reinterpret_cast<uint32_t*>(ws.keys_a);
        dw.up = reinterpret_cast<int32_t*>(ws.keys_b);
        dw.hook = ws.hook;
        const size_t half = E / 2 / 32 * 32;                // (the lists of odd levels hold half the vertices at most, the others a quarter)
        dw.edge[0] = ws.vals_a; dw.edge[1] = reinterpret_cast<uint32_t*>(ws.e_w);
        dw.ends[0] = reinterpret_cast<int2*>(ws.best_e); dw.ends[1] = dw.ends[0] + half;
        dw.key = reinterpret_cast<uint32_t*>(ws.ptr); dw.val = ws.vals_b;
        dw.key_sorted = reinterpret_cast<uint32_t*>(ws.colour); dw.listed = reinterpret_cast<uint32_t*>(ws.qlist);
        dw.chain = reinterpret_cast<int2*>(ws.best_e);
        dw.carry = reinterpret_cast<unsigned long long*>(ws.ext_idx);
        dw.counters = ws.cand_u;
        if (timed) hipLaunchKernelGGL(k_fetch_words, dim3(1), dim3(256), 0, s, reinterpret_cast<const uint32_t*>(ws.counters), 1, mail.words(), mail.next());
        HIP_TRY(slhc::dendrogram_chains(mst_src, mst_dst, (int)N, dw, children, s));
        if (timed) { HIP_TRY(mail.wait()); t_sort = now_ms(); }
        // the merges per level come back while the pairs are sorted
        int32_t h_levels[slhc::DENDRO_WORDS];
        hipLaunchKernelGGL(k_fetch_words, dim3(1), dim3(256), 0, s, reinterpret_cast<const uint32_t*>(dw.counters), slhc::DENDRO_WORDS, mail.words(), mail.next());
        HIP_TRY(hipGetLastError());
        HIP_TRY(slhc::pair_sort_u32(dw.key, dw.key_sorted, dw.val, dw.listed, (int)E, bits_for(N), ws.sort_temp, ws.sort_temp_bytes, s));
        HIP_TRY(mail.wait());
        std::memcpy(h_levels, mail.words() + 1, sizeof(h_levels));
        int64_t merges = 0;
        for (int l = 0; l < slhc::DENDRO_LEVELS; ++l) merges += h_levels[slhc::DENDRO_MERGES + l];
        if (h_levels[slhc::DENDRO_ERROR] != 0 || merges != (int64_t)E) {
            set_err("dendrogram: check %d failed, %lld of %zu merges in chains", h_levels[slhc::DENDRO_ERROR], (long long)merges, E);
            return SLHC_INTERNAL;
        }
        log.mark("dendrogram: %d levels", h_levels[slhc::DENDRO_DEPTH]);
        HIP_TRY(slhc::dendrogram_sizes((int)N, h_levels + slhc::DENDRO_MERGES, dw, children, sizes, s));
    }
    st.ms_sort = (float)(t_sort - t_forest);
    HIP_TRY(hipStreamSynchronize(s));
    pin_edges.idle();
    mail.box.idle();
    const double t_end = now_ms();
    st.ms_dendrogram = (float)(t_end - t_sort);
    st.ms_total = (float)(t_end - t_begin);
    if (stats) *stats = st;
    return SLHC_OK;
}

}  // namespace
