// Passes over the pairs of ONE float16 copy, each pair of rows multiplied once.
//
// The distance of two rows does not depend on which of them asks, so where the queries are the candidates a product serves
// both.  With h the stored half norms and acc = x_q . x_c - h_c the product value of the sweeps,
//     u(q, c) = acc - h_q,   about minus half the squared distance,
// is the same for both, up to rounding (see near_e), and a row's bound on product values becomes a limit on u by taking its own
// half norm off.  A value is held against the limit of its query, a register, and against that of its candidate, which
// comes through LDS with the candidate's norm.
//
// The copy is cut into blocks of consecutive tiles, laid out round a circle; the block at place i meets those at the places i, i + 1, ...
// up to half way round, so every pair of blocks meets once, every block has the same number of meetings, and a launch over a
// range of these offsets has shown every row the same share of all others.  Of those that are like it, too: rows that lie together in the
// matrix lie in neighbouring tiles, so neighbouring blocks are far apart on the circle (near_spread).  With blocks in the order of the copy,
// and rows in its tiles as their numbers give it, the lists of rows in the order of their clusters overflowed: clusters of 500 rows, k = 12,
// 60 000 x 128 5.5 ms, 300 000 x 128 60 ms; 1.4 and 16.6 so (in no order 1.5 and 18.5).
#include <hip/hip_runtime.h>
#include <stdint.h>
#include "near_kernels.h"
#include "near_parts.h"
#include "pairs_kernels.h"

namespace slhc {

constexpr int QUEUE = 192;                 // pairs of a wavefront that wait for their slots in the rows' lists
constexpr int PAIR_TILE_BITS = 17;         // of a tile's number in a queued pair

// Pairs that pass wait in LDS until a wavefront's worth is there; then the limits of both rows are read at one tile, the pairs'
// slots in the rows' lists are asked for at the next and used at the one after that, so nobody waits for memory.
struct PairQueue {
    uint2* at;                             // LDS, QUEUE entries
    int n, records;                        // waiting, and records behind the queue (the same for all lanes)
    bool read, asked;                      // 64 pairs at the first and at the second step (the same for all lanes)
    bool full;                             // some row's list was found to be full (the same for all lanes)
    unsigned int u, code, u2, code2;       // of this lane's at the two steps
    float q_limit, c_limit;
    int q_slot, c_slot;
};
// A pair: tile and place of the candidate, place of the query among the wavefront's 64; bit 1: it is met in the other order too.
constexpr unsigned int PAIR_OWN = 2u;
__device__ inline unsigned int pair_code(int tile, int c, int q, bool own)
{
    return ((unsigned int)tile << 15) | ((unsigned int)c << 8) | ((unsigned int)q << 2) | (own ? PAIR_OWN : 0u);
}
// q0: the wavefront's first query among the rows of the lists
__device__ inline int pair_q(unsigned int code, int q0) { return q0 + (int)((code >> 2) & 63u); }
__device__ inline int pair_c(unsigned int code) { return (int)(code >> 15) * TILE + (int)((code >> 8) & 127u); }
__device__ inline void pair_entry(const NearPairs& p, int row, int slot, unsigned int u, unsigned int other)
{
    if ((unsigned int)slot < (unsigned int)p.cap) p.entries[(size_t)row * (size_t)p.cap + (size_t)slot] = make_uint2(u, other);
}
// Every pair under way goes one step further, and where at least `least` wait the next ones set out.
template <bool ONCE>
__device__ inline void pair_turn(PairQueue& w, const NearPairs& p, int q0, int least)
{
    const int lane = threadIdx.x & 63;
    const bool more = w.n >= least && w.n > 0;
    const int from = w.n > 64 ? w.n - 64 : 0;
    uint2 e = make_uint2(0u, ~0u);
    if (more && from + lane < w.n) e = w.at[from + lane];      // (before anything is under way in memory, see pair_push)
    if (w.asked) {
        const int q = pair_q(w.code2, q0), c = pair_c(w.code2);
        pair_entry(p, q, w.q_slot, w.u2, (unsigned int)c);
        if (ONCE) pair_entry(p, c, w.c_slot, w.u2, (unsigned int)q);
        // A row whose list is full is left to another search and takes no more.  (Where copies are more than a list holds, or rounding does not tell most rows
        // apart, everything passed to the end: 40 000 x 30 of 2000 copies each 4.3 -> 2.7 ms, 40 000 x 24 with norms over orders of magnitude, k = 20, 1.8 -> 0.9.)
        if (__any(w.q_slot >= p.cap || (ONCE && w.c_slot >= p.cap))) {
            if (w.q_slot >= p.cap) p.limit[q] = NEVER;
            if (ONCE && w.c_slot >= p.cap) p.limit[c] = NEVER;
            w.full = true;
        }
        w.asked = false;
    }
    if (w.read) {
        const float u = __uint_as_float(w.u);
        w.u2 = w.u; w.code2 = w.code;
        w.q_slot = w.c_slot = -1;
        if (u >= w.q_limit) w.q_slot = atomicAdd(p.counts + pair_q(w.code, q0), 1);
        if (ONCE && u >= w.c_limit) w.c_slot = atomicAdd(p.counts + pair_c(w.code), 1);
        w.read = false;
        w.asked = true;
    }
    if (!more) return;
    w.u = e.x; w.code = e.y;
    w.q_limit = w.c_limit = NEVER;
    if (e.y != ~0u) {
        w.q_limit = p.limit[pair_q(e.y, q0)];
        if (ONCE && !(e.y & PAIR_OWN)) w.c_limit = p.limit[pair_c(e.y)];
    }
    w.n = from;
    w.read = true;
}
// The queue is empty when this returns.
template <bool ONCE>
__device__ inline void pair_finish(PairQueue& w, const NearPairs& p, int q0)
{
#pragma unroll 1
    while (w.n > 0 || w.read || w.asked) pair_turn<ONCE>(w, p, q0, 1);
}

// (Past the compiler, which would wait for the tile on its way into LDS before it writes there.  LDS instructions of a wavefront
// are done in order.)
__device__ inline void pair_push(uint2* at, unsigned int u, unsigned int code)
{
    const unsigned long long e = ((unsigned long long)code << 32) | u;
    asm volatile("ds_write_b64 %0, %1" ::"v"((unsigned int)(uintptr_t)(__attribute__((address_space(3))) void*)at), "v"(e) : "memory");
}

// A lane's 16 values of a block of which some pass, until the tile they belong to is done with.
constexpr int RECORDS = 16;
constexpr int WAVE_LDS = QUEUE * 8 + RECORDS * 80;             // of a wavefront: pairs that wait, records' values and words
__device__ inline unsigned int lds_word(const void* at)
{
    return (unsigned int)(uintptr_t)(__attribute__((address_space(3))) const void*)at;
}
// The records' values, twice four records at a time, against the limits of both rows; tile_limit: LDS, of the tile's candidates.  (Reads past the compiler
// as well, see pair_push.)  Where lists are long and rows few, most lanes of every block hold something, and it is bound by its waits for LDS: with four
// records at a time, and the queue emptied whenever it was full, 4500 x 128, k = 64, took 139 us, 12 000 x 128 273, 300 000 x 128, k = 32, 24.6 ms; 129,
// 256, 24.4 so.  (Values looked for in registers there, as before whole values went to LDS: 130, 277 and, for its registers and code, 26.7.)
template <bool ONCE>
__device__ inline void pair_sift(PairQueue& w, const NearPairs& p, int q0, const unsigned char* tile_limit)
{
    const int lane = threadIdx.x & 63;
    const unsigned int values = lds_word(w.at + QUEUE) + lane * 4, words = lds_word(w.at + QUEUE) + RECORDS * 64 + (lane >> 4) * 16;
#pragma unroll 1
    for (int at = 0; at < w.records; at += 8) {
        float x[2], limit[2] = {0.f, 0.f};
        v4f word[2];
        asm volatile("ds_read_b32 %0, %4\n\tds_read_b128 %1, %5\n\tds_read_b32 %2, %4 offset:256\n\tds_read_b128 %3, %5 offset:64\n\ts_waitcnt lgkmcnt(0)"
                     : "=&v"(x[0]), "=&v"(word[0]), "=&v"(x[1]), "=&v"(word[1]) : "v"(values + at * 64), "v"(words + at * 16) : "memory");
        const unsigned int place = (((lane & 12u) << 1) | (lane & 3u)) << 8;
        const unsigned int code[2] = {__float_as_uint(word[0][0]) + place, __float_as_uint(word[1][0]) + place};
        if (ONCE)
            asm volatile("ds_read_b32 %0, %2\n\tds_read_b32 %1, %3\n\ts_waitcnt lgkmcnt(0)" : "=&v"(limit[0]), "=&v"(limit[1])
                         : "v"(lds_word(tile_limit) + ((code[0] >> 6) & 508u)), "v"(lds_word(tile_limit) + ((code[1] >> 6) & 508u)) : "memory");
#pragma unroll 1
        while (w.n > QUEUE - 128) pair_turn<ONCE>(w, p, q0, 64);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const bool pass = at + 4 * i + (lane >> 4) < w.records && (x[i] >= word[i][1] || (ONCE && x[i] - limit[i] >= word[i][2]));
            const unsigned long long m = __ballot(pass);
            const int pre = __builtin_amdgcn_mbcnt_hi((unsigned int)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned int)m, 0u));
            if (pass) pair_push(w.at + w.n + pre, __float_as_uint(x[i] - word[i][3]), code[i]);
            w.n += __popcll(m);
        }
    }
    w.records = 0;
}

// One 32 x 32 block of values.  limit: of this lane's 16 candidates; bound: the query's limit plus its half norm h; other: h, or
// NaN where the block's pairs are met in both orders anyway.  code: of the lane's first candidate.
// Bound by the test, 36 instructions for 16 values; of 1M x 128 in clusters by Zipf's law every second block holds something, so what
// follows has to be short: the lane's values go to LDS as they are, and which of them pass is found for four lanes at once.  With
// the wavefront looking for them there and then (a bit per value, the value picked out of 16 registers, a turn per pair of a lane) the
// emission of 1M x 128, k = 32, took 171 ms; 146 so, 115 with nothing after the test, 94 with the products alone (1.37 PFLOP/s at 1.9 GHz).
template <bool ONCE>
__device__ inline void pair_emit(const v16f& v, const float (&limit)[16], float bound, float h, float other, unsigned int code,
                                 PairQueue& w, const NearPairs& p, int q0, const unsigned char* tile_limit)
{
    float f = max3(v[0], v[1], v[2]);
#pragma unroll
    for (int r = 3; r < 15; r += 2) f = max3(f, v[r], v[r + 1]);
    f = fmaxf(f, v[15]);
    bool some = f >= bound;
    if (ONCE) {
        float t = max3(v[0] - limit[0], v[1] - limit[1], v[2] - limit[2]);
#pragma unroll
        for (int r = 3; r < 15; r += 2) t = max3(t, v[r] - limit[r], v[r + 1] - limit[r + 1]);
        t = fmaxf(t, v[15] - limit[15]);
        some = some || t >= other;
    }
    unsigned long long m = __ballot(some);
    while (m) {
        const int at = w.records + __builtin_amdgcn_mbcnt_hi((unsigned int)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned int)m, 0u));
        if (some && at < RECORDS) {
            const unsigned int values = lds_word(w.at + QUEUE) + at * 64, words = lds_word(w.at + QUEUE) + RECORDS * 64 + at * 16;
            const v4f word = {__uint_as_float(code), bound, other, h};
            const v4f v0 = {v[0], v[1], v[2], v[3]}, v1 = {v[4], v[5], v[6], v[7]}, v2 = {v[8], v[9], v[10], v[11]}, v3 = {v[12], v[13], v[14], v[15]};
            asm volatile("ds_write_b128 %0, %2\n\tds_write_b128 %0, %3 offset:16\n\tds_write_b128 %0, %4 offset:32\n\tds_write_b128 %0, %5 offset:48\n\tds_write_b128 %1, %6"
                         ::"v"(values), "v"(words), "v"(v0), "v"(v1), "v"(v2), "v"(v3), "v"(word) : "memory");
            some = false;
        }
        w.records += __popcll(m);
        if (w.records < RECORDS) return;
        w.records = w.records < RECORDS ? w.records : RECORDS;
        pair_sift<ONCE>(w, p, q0, tile_limit);
        m = __ballot(some);
    }
}

// Which blocks a workgroup's block meets: offsets [from, from + len) in an order in which all blocks of one stretch of the circle
// meet the same block at the same time, so that it is in L2.
struct PairRange { int at, block, from, len, j0, j1, turn; };      // at: of the circle, block: of the copy
template <bool ONCE>
__device__ inline PairRange pair_range(const NearPairs& p, int item)
{
    PairRange r;
    r.at = item / p.nseg;
    const int seg = item - r.at * p.nseg;
    // (in either order it is all the same where on the circle a block begins)
    if (!ONCE) r.at += p.first;
    r.block = ONCE ? near_spread_at(r.at, p.spread, p.blocks) : r.at;
    // half way round an even circle two blocks meet from both sides
    const int to = ONCE && 2 * (p.to - 1) == p.blocks && p.to - 1 > 0 && 2 * r.at >= p.blocks ? p.to - 1 : p.to;
    r.from = p.from;
    r.len = to > p.from ? to - p.from : 0;
    r.j0 = (int)((long long)r.len * seg / p.nseg);
    r.j1 = (int)((long long)r.len * (seg + 1) / p.nseg);
    r.turn = r.len > 0 ? r.len - r.at % r.len : 0;
    return r;
}
__device__ inline int pair_offset(const PairRange& r, int j) { return r.from + (j + r.turn) % r.len; }
__device__ inline int pair_other(const NearPairs& p, const PairRange& r, int offset)
{
    const int c = r.at + offset;
    return near_spread_at(c >= p.blocks ? c - p.blocks : c, p.spread, p.blocks);
}

// Up to 128 columns: as near_sweep_kernel, a wavefront keeps the fragments of 64 queries in registers and the candidate tiles pass
// through LDS (double buffered); a block is the tiles of a workgroup's queries.  Products alone take 95 of the 142 ms of 1M x 128, k = 32 (1.35 PFLOP/s, to
// which the card throttles), the test 18, what passes 29, and a wavefront waits for LDS or at a barrier a third of its time: so 32 candidates at a time,
// which leaves room for three wavefronts per SIMD at any width (four up to 48 columns), where 64 took two.  1M x 128, k = 32 146 -> 136 ms, 300 000 x 96, k = 16,
// whole search 15.5 -> 14.2.  (More than a step of fragments read ahead, priorities for multiplies or for tests, two workgroups of four: the same times.)
template <int KS, bool ONCE>
__global__ void __launch_bounds__(ONCE ? 768 : 256, ONCE ? 3 : KS <= 2 ? 5 : KS <= 4 ? 4 : 3) pairs_kernel(NearPairs p)
{
    extern __shared__ __align__(16) unsigned char pairs_smem[];
    constexpr int BUF = KS * FRAG_STEP + (ONCE ? 1024 : 512);        // fragments, minus half norms, limits
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, lhalf = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int waves = blockDim.x >> 6, bt = waves >> 1;
    if (*p.lost > p.lost_most) return;
    const PairRange range = pair_range<ONCE>(p, blockIdx.x);
    const int qtile = range.block * bt + (wave >> 1);
    const bool live = qtile < p.tiles;                   // (whole wavefronts)
    const int row0 = ONCE ? 0 : p.row0;
    const int q_pos = (live ? qtile : row0 / TILE) * TILE + (wave & 1) * 64, q0 = q_pos - row0;        // position, and among the rows of the lists
    float h[2], bound[2];
    v8h qf[2][KS];
#pragma unroll
    for (int qb = 0; qb < 2; ++qb) {
        const int at = q_pos + qb * 32 + l32;
        h[qb] = live ? -p.negh[at] : NEVER;
        bound[qb] = live ? p.limit[at - row0] + h[qb] : NEVER;
        const unsigned char* src = p.frag + (size_t)(at >> 7) * (KS * FRAG_STEP) + ((at >> 5) & 3) * 1024 + lane * 16;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) qf[qb][ks] = *reinterpret_cast<const v8h*>(src + ks * FRAG_STEP);
    }
    PairQueue w;
    w.at = reinterpret_cast<uint2*>(pairs_smem + 2 * BUF + wave * WAVE_LDS);
    w.n = w.records = 0; w.read = w.asked = w.full = false; w.u = w.code = w.u2 = w.code2 = 0u; w.q_limit = w.c_limit = NEVER; w.q_slot = w.c_slot = -1;

    bool ever_full = false;
    const int total = (range.j1 - range.j0) * bt;        // tiles to pass over (some may not be there)
    int step_j = range.j0, step_t = 0;                   // of the tile that is brought in next
    int next_tile = 0;
    bool next_own = false;
    auto advance = [&]() {
        if (step_t == 0) {
            const int off = pair_offset(range, step_j++);
            const int block = pair_other(p, range, off);
            next_tile = block * bt;
            next_own = block == range.block;
        } else ++next_tile;
        if (++step_t == bt) step_t = 0;
    };
    auto stage = [&](int i, int tile) {
        const size_t t = tile < p.tiles ? tile : p.tiles - 1;
        unsigned char* dst = pairs_smem + (i & 1) * BUF;
        const unsigned char* src = p.frag + t * (KS * FRAG_STEP);
        for (int j = wave; j < KS * 4; j += waves) near_lds_load(src, j * 1024, dst + j * 1024, true);
        for (int j = wave; j < (ONCE ? 4 : 2); j += waves) {
            near_lds_load((j < 2 ? p.negh : p.limit) + t * TILE, (j & 1) * 256, dst + KS * FRAG_STEP + j * 256, false);
        }
    };
    if (total > 0) { advance(); stage(0, next_tile); }
    for (int i = 0; i < total; ++i) {
        near_lds_ready();
        const int tile = next_tile;
        const bool own = next_own;
        if (live) pair_turn<ONCE>(w, p, q0, 64);
        if (w.full) {
#pragma unroll
            for (int qb = 0; qb < 2; ++qb) bound[qb] = p.limit[q0 + qb * 32 + l32] + h[qb];
            w.full = false;
            ever_full = true;
        }
        if (i + 1 < total) { advance(); stage(i + 1, next_tile); }
        if (tile >= p.tiles || !live) continue;
        const unsigned char* tb = pairs_smem + (i & 1) * BUF;
        const float other[2] = {own ? NEVER : h[0], own ? NEVER : h[1]};
#pragma unroll 1
        for (int blk = 0; blk < 4; ++blk) {
            v16f acc[2];
            v8h cf[2];
            const unsigned char* hb = tb + blk * 1024 + lane * 16;
            cf[0] = *reinterpret_cast<const v8h*>(hb);
            {
                v16f hv;
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const v4f t4 = *reinterpret_cast<const v4f*>(tb + KS * FRAG_STEP + (blk * 32 + 8 * g + 4 * lhalf) * 4);
                    hv[4 * g] = t4[0]; hv[4 * g + 1] = t4[1]; hv[4 * g + 2] = t4[2]; hv[4 * g + 3] = t4[3];
                }
                acc[0] = hv; acc[1] = hv;
            }
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                // (as in near_sweep_kernel: the next step's reads stay ahead of this step's multiplies)
                if (ks + 1 < KS) {
                    cf[(ks + 1) & 1] = *reinterpret_cast<const v8h*>(hb + (ks + 1) * FRAG_STEP);
                    __builtin_amdgcn_sched_barrier(0);
                }
#pragma unroll
                for (int qb = 0; qb < 2; ++qb)
                    acc[qb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(cf[ks & 1], qf[qb][ks], acc[qb], 0, 0, 0);
            }
            float limit[16];
#pragma unroll
            for (int g = 0; ONCE && g < 4; ++g) {
                const v4f t4 = *reinterpret_cast<const v4f*>(tb + KS * FRAG_STEP + 512 + (blk * 32 + 8 * g + 4 * lhalf) * 4);
#pragma unroll
                for (int e = 0; e < 4; ++e) limit[4 * g + e] = t4[e];
            }
#pragma unroll
            for (int qb = 0; qb < 2; ++qb)
                pair_emit<ONCE>(acc[qb], limit, bound[qb], h[qb], other[qb], pair_code(tile, blk * 32 + 4 * lhalf, qb * 32 + l32, own), w, p, q0,
                          tb + KS * FRAG_STEP + 512);
        }
        pair_sift<ONCE>(w, p, q0, tb + KS * FRAG_STEP + 512);
    }
    if (live) pair_finish<ONCE>(w, p, q0);
    // panels of rows whose lists are full are not looked through (see near_select_kernel); the additions to these rows that this wavefront saw are all made
    if (!ONCE && p.full_gone && (ever_full || w.full) && __hip_atomic_load(p.counts + q0 + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) > p.cap)
        near_panel_gone(p.todo, p.todo_mark, (int)(near_row(q_pos + lane, p.tiles, 0) >> 7));
}

// Beyond 128 columns: 256 x 256 rows per meeting, both sides streamed through LDS, as near_wide_kernel; a block is two tiles.
//   BEST = false  pairs within either row's limit go to that row's list
//   BEST = true   rows of another colour: every row's smallest w = max(0, -u), with the place of the 16 rows about it
constexpr int WIDE_ROWS = 3072;                                         // half norms, limits or smallest w, colours of 256 rows
constexpr int WIDE_LDS = CHUNKS * CHUNK + 2 * WIDE_ROWS;

template <bool BEST>
__global__ void __launch_bounds__(512, 2) pairs_wide_kernel(NearPairs p)
{
    extern __shared__ __align__(16) unsigned char pairs_smem[];
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, lhalf = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int qg = wave >> 1, cg = wave & 1;                            // 64 queries, 128 candidates of the 256 x 256
    if (!BEST && *p.lost > p.lost_most) return;
    int item = blockIdx.x;
    {
        // workgroups b, b + 8, ... share an XCD: they get the shares of neighbouring blocks, whose rows stay in its L2
        const int items = p.blocks * p.nseg, per = items >> 3;
        if (item < per * 8) item = (item & 7) * per + (item >> 3);
    }
    const PairRange range = pair_range<true>(p, item);
    const int qtile = range.block * 2 + (qg >> 1);
    const bool live = qtile < p.tiles;
    const int qsafe = live ? qtile : range.block * 2;
    const int q0 = qsafe * TILE + (qg & 1) * 64;
    float h[2], bound[2], m1[2] = {-INF, -INF};
    int qcol[2] = {0, 0}, m1_at[2] = {-1, -1};
#pragma unroll
    for (int qb = 0; qb < 2; ++qb) {
        const int at = q0 + qb * 32 + l32;
        h[qb] = live ? -p.negh[at] : NEVER;
        bound[qb] = NEVER;
        if (BEST) qcol[qb] = p.colour[at];
        else if (live) bound[qb] = p.limit[at] + h[qb];
    }
    PairQueue w;
    w.at = reinterpret_cast<uint2*>(pairs_smem + WIDE_LDS + wave * WAVE_LDS);
    w.n = w.records = 0; w.read = w.asked = w.full = false; w.u = w.code = w.u2 = w.code2 = 0u; w.q_limit = w.c_limit = NEVER; w.q_slot = w.c_slot = -1;

    const int nchunks = (p.filled + CHUNK_STEPS - 1) / CHUNK_STEPS;     // (at least five, beyond 128 columns)
    const bool odd = (p.filled & 1) != 0;                               // the last chunk has one step
    const int nmine = range.j1 - range.j0;
    const int total = nmine * nchunks;
    auto block_at = [&](int i) { return pair_other(p, range, pair_offset(range, range.j0 + i)); };
    // the next chunk's loads: a wavefront has one step of one tile of one side, four pieces of 1 KiB, and with a meeting's first chunk the rows' words
    int staged = 0, stage_i = 0, stage_chunk = 0, stage_block = nmine > 0 ? block_at(0) : 0;
    auto stage = [&]() {
        const int side = wave >> 2, tile = (wave >> 1) & 1, st = wave & 1;
        const int b2 = (side ? stage_block : range.block) * 2;
        const size_t t = b2 + tile < p.tiles ? b2 + tile : b2;
        const unsigned char* src = p.frag + (t * p.steps + stage_chunk * CHUNK_STEPS + st) * FRAG_STEP;
        unsigned char* dst = pairs_smem + (staged & (CHUNKS - 1)) * CHUNK + wave * FRAG_STEP;
        if (stage_chunk == 0) {
            unsigned char* rows = pairs_smem + CHUNKS * CHUNK + (stage_i & 1) * WIDE_ROWS;
            for (int piece = wave; piece < (BEST ? 12 : 8); piece += 8) {
                const int what = piece >> 2, half = piece & 1;
                const size_t r = (stage_block * 2 + ((piece >> 1) & 1) < p.tiles ? stage_block * 2 + ((piece >> 1) & 1) : stage_block * 2) * (size_t)TILE;
                const void* base = what == 0 ? (const void*)(p.negh + r)
                              : what == 2 ? (const void*)(p.colour + r)
                              : BEST ? (const void*)(reinterpret_cast<const uint32_t*>(p.best + r) + 1) : (const void*)(p.limit + r);
                const int stride = BEST && what == 1 ? 8 : 4;
                near_lds_load(base, half * 64 * stride, rows + piece * 256, false, stride);
            }
        }
#pragma unroll
        for (int blk = 0; blk < 4; ++blk) near_lds_load(src, blk * 1024, dst + blk * 1024, true);
        ++staged;
        if (++stage_chunk == nchunks) {
            stage_chunk = 0;
            if (++stage_i < nmine) stage_block = block_at(stage_i);
        }
    };
    v16f acc[2][4];                                                     // [query block][candidate block]
    v8h qf[2][2], cf[2][4];                                             // [step of the chunk]
    auto read = [&](int at, int st) {
        const unsigned char* qs = pairs_smem + (at & (CHUNKS - 1)) * CHUNK + (qg >> 1) * CHUNK_TILE + st * FRAG_STEP + (qg & 1) * 2048 + lane * 16;
        const unsigned char* cs = pairs_smem + (at & (CHUNKS - 1)) * CHUNK + CHUNK_SIDE + cg * CHUNK_TILE + st * FRAG_STEP + lane * 16;
#pragma unroll
        for (int qb = 0; qb < 2; ++qb) qf[st][qb] = *reinterpret_cast<const v8h*>(qs + qb * 1024);
#pragma unroll
        for (int cb = 0; cb < 4; ++cb) cf[st][cb] = *reinterpret_cast<const v8h*>(cs + cb * 1024);
        __builtin_amdgcn_sched_barrier(0);                              // (ahead of the multiplies that follow)
    };
    auto multiply = [&](int st, int from, int to) {
#pragma unroll
        for (int cb = 0; cb < 4; ++cb)
#pragma unroll
            for (int qb = 0; qb < 2; ++qb)
                if (cb >= from && cb < to) acc[qb][cb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(cf[st][cb], qf[st][qb], acc[qb][cb], 0, 0, 0);
    };
    for (int i = 0; i < CHUNKS - 1 && i < total; ++i) stage();
    near_lds_ready();
    int at = 0, block = nmine > 0 ? block_at(0) : 0;
    for (int i = 0; i < nmine; ++i) {
        const unsigned char* rows = pairs_smem + CHUNKS * CHUNK + (i & 1) * WIDE_ROWS;
        const bool own = block == range.block;
        const int tile = block * 2 + cg;
        // (the chunk and the rows' words have been there since the last barrier)
        read(at, 0);
#pragma unroll
        for (int cb = 0; cb < 4; ++cb) {
            v16f hv;
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const v4f t4 = *reinterpret_cast<const v4f*>(rows + cg * 512 + (cb * 32 + 8 * g + 4 * lhalf) * 4);
                hv[4 * g] = t4[0]; hv[4 * g + 1] = t4[1]; hv[4 * g + 2] = t4[2]; hv[4 * g + 3] = t4[3];
            }
            acc[0][cb] = hv; acc[1][cb] = hv;
        }
#pragma unroll 1
        for (int chunk = 1; chunk < nchunks; ++chunk, ++at) {
            near_chunk_ready(at + 2 < total);
            read(at, 1);
            multiply(0, 0, 2);
            if (staged < total) stage();
            multiply(0, 2, 4);
            __builtin_amdgcn_sched_barrier(0);
            read(at + 1, 0);
            multiply(1, 0, 4);
        }
        near_chunk_ready(at + 2 < total);
        read(at, 1);
        multiply(0, 0, 4);
        if (!odd) multiply(1, 0, 4);
        if (staged < total) stage();
        ++at;
        if (!BEST && live) pair_turn<true>(w, p, q0, 64);
        const int next = i + 1 < nmine ? block_at(i + 1) : block;
        if (live && tile < p.tiles) {
#pragma unroll
            for (int cb = 0; cb < 4; ++cb) {
                float limit[16];
                int col[16];
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const unsigned char* word = rows + 1024 + cg * 512 + (cb * 32 + 8 * g + 4 * lhalf) * 4;
                    const v4f t4 = *reinterpret_cast<const v4f*>(word);
#pragma unroll
                    for (int e = 0; e < 4; ++e) limit[4 * g + e] = t4[e];
                    if (BEST) {
                        const v4i c4 = *reinterpret_cast<const v4i*>(word + 1024);
#pragma unroll
                        for (int e = 0; e < 4; ++e) col[4 * g + e] = c4[e];
                    }
                }
#pragma unroll
                for (int qb = 0; qb < 2; ++qb) {
                    if (!BEST) {
                        pair_emit<true>(acc[qb][cb], limit, bound[qb], h[qb], own ? NEVER : h[qb],
                                  pair_code(tile, cb * 32 + 4 * lhalf, qb * 32 + l32, own), w, p, q0, rows + 1024 + cg * 512);
                        continue;
                    }
                    v16f& v = acc[qb][cb];
                    float best = -INF, gain = -INF;
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        v[r] = col[r] == qcol[qb] ? -INF : v[r];
                        best = fmaxf(best, v[r]);
                        gain = fmaxf(gain, v[r] + limit[r]);
                    }
                    const bool up = best > m1[qb];
                    m1_at[qb] = up ? tile * TILE + cb * 32 + 4 * lhalf : m1_at[qb];
                    m1[qb] = up ? best : m1[qb];
                    // (values seen by another workgroup meanwhile only make an update idle)
                    if (p.both && !own && __any(gain > h[qb])) {
                        const unsigned int q_at = (unsigned int)(q0 + qb * 32 + (l32 & 4));
#pragma unroll
                        for (int r = 0; r < 16; ++r)
                            if (v[r] + limit[r] > h[qb])
                                atomicMin(p.best + (size_t)tile * TILE + cb * 32 + 8 * (r >> 2) + 4 * lhalf + (r & 3),
                                          ((unsigned long long)__float_as_uint(fmaxf(0.f, h[qb] - v[r])) << 32) | q_at);
                    }
                }
            }
            if (!BEST) pair_sift<true>(w, p, q0, rows + 1024 + cg * 512);
        }
        block = next;
    }
    if (!live) return;
    if (!BEST) pair_finish<true>(w, p, q0);
    else {
#pragma unroll
        for (int qb = 0; qb < 2; ++qb)
            if (m1_at[qb] >= 0 && fabsf(h[qb]) < INF && fabsf(m1[qb]) < INF)
                atomicMin(p.best + q0 + qb * 32 + l32, ((unsigned long long)__float_as_uint(fmaxf(0.f, h[qb] - m1[qb])) << 32) | (unsigned int)m1_at[qb]);
    }
}

// (Nearly) the kk-th largest of the first n values of a row's list, in `mine`; LOWEST where fewer are finite.
constexpr int PAIR_WORDS = PAIRS_MOST / 64;
__device__ inline void pair_list(uint2 (&mine)[PAIR_WORDS], const uint2* __restrict__ list, int n)
{
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int j = 0; j < PAIR_WORDS; ++j) {
        mine[j] = make_uint2(__float_as_uint(-INF), 0u);
        if (j * 64 + lane < n) mine[j] = list[j * 64 + lane];
    }
}
__device__ inline float pair_kth(const uint2 (&mine)[PAIR_WORDS], int n, int kk)
{
    float lo = INF, hi = -INF;
    int have = 0;
#pragma unroll
    for (int j = 0; j < PAIR_WORDS; ++j)
        if (j * 64 < n) {
            const float x = __uint_as_float(mine[j].x);
            const bool fine = fabsf(x) < INF;
            have += __popcll(__ballot(fine));
            lo = fine ? fminf(lo, x) : lo;
            hi = fine ? fmaxf(hi, x) : hi;
        }
    if (have < kk) return LOWEST;
    lo = wave_min(lo); hi = wave_max(hi);
    for (int it = 0; it < BISECT_FAR; ++it) {
        const float mid = 0.5f * lo + 0.5f * hi;
        int reach = 0;
#pragma unroll
        for (int j = 0; j < PAIR_WORDS; ++j)
            if (j * 64 < n) {
                const float x = __uint_as_float(mine[j].x);
                reach += __popcll(__ballot(x >= mid && x < INF));
            }
        if (reach >= kk) lo = mid; else hi = mid;
        if (reach == kk) break;
    }
    return lo;
}

constexpr int PAIRS_LOST = 0x40000000;     // the count of a list that overflowed and has been counted among the lost
// Between two launches: of what a row's list holds, kk rows reach the kk-th value; what that leaves is kept, and the row's limit
// follows.  Rows whose list has grown by less than half a list of neighbours since are left as they are (all rows of a tight
// cluster, which rounding does not tell apart).  One wavefront per row, bound by its instructions: n / 64 compares a step.  120 000
// rows, k = 32: 226 us a launch with every row tightened each time, 120 so.
__global__ void __launch_bounds__(256) pairs_tighten_kernel(NearPairs p, int kk, const NearScale* __restrict__ sc, float e, float nu, int d,
                                                            int32_t* __restrict__ last)
{
    const int row = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (row >= p.rows) return;
    const int n = __builtin_amdgcn_readfirstlane(p.counts[row]);
    if (n > p.cap) {                                                    // some were lost: nothing more (see pairs_left)
        if (lane == 0 && n != PAIRS_LOST) {
            p.counts[row] = PAIRS_LOST; p.limit[row] = NEVER;
            // (one word, so no more additions than count)
            if (__hip_atomic_load(p.lost, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) <= p.lost_most) atomicAdd(p.lost, 1);
        }
        return;
    }
    const float h = -p.negh[p.row0 + row];
    if (n <= kk || n < __builtin_amdgcn_readfirstlane(last[row]) + (kk + 1) / 2 || !(fabsf(h) < INF)) return;
    uint2* list = p.entries + (size_t)row * (size_t)p.cap;
    uint2 mine[PAIR_WORDS];
    pair_list(mine, list, n);
    const float kth = pair_kth(mine, n, kk);
    if (kth == LOWEST) return;
    const NearBoundArgs a = near_args(sc, p.steps, d, e, nu);
    const float limit = near_bound_from(kth + h, h, a) - h;
    if (!(limit > p.limit[row])) { if (lane == 0) last[row] = n; return; }
    int kept = 0;
#pragma unroll
    for (int j = 0; j < PAIR_WORDS; ++j)
        if (j * 64 < n) {
            const bool keep = j * 64 + lane < n && __uint_as_float(mine[j].x) >= limit;
            const unsigned long long m = __ballot(keep);
            const int pre = __builtin_amdgcn_mbcnt_hi((unsigned int)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned int)m, 0u));
            if (keep) list[kept + pre] = mine[j];
            kept += __popcll(m);
        }
    if (lane == 0) { p.counts[row] = last[row] = kept; p.limit[row] = limit; }
}

// an upper end of the squared distance (of the rows as they are) behind a product value
__device__ inline float pair_reach(float value, float h, const NearBoundArgs& a, const NearScale* sc, int d)
{
    const float t = value > LOWEST ? near_distance_from(value, h, a) / sc->scale : INF;
    return (t * t * (1.f + a.gamma) + (float)d * 2.350988701644575e-38f) * (1.f + 1e-6f);
}
// (one addition to the word of all rows left for LEFT_ROWS rows: 60 000 of them 0.7 ms with one for each)
constexpr int LEFT_ROWS = 16;
__global__ void __launch_bounds__(64 * LEFT_ROWS) pairs_left_kernel(NearPairs p, int kk, const NearScale* __restrict__ sc, float e, float nu, int d, int n_rows,
                                                         PairsLeft out)
{
    __shared__ int s_here, s_from;
    const int of_list = blockIdx.x * LEFT_ROWS + (threadIdx.x >> 6), pos = p.row0 + of_list, lane = threadIdx.x & 63;
    const bool over = p.counts[of_list] > p.cap;
    const float h = -p.negh[pos];
    const long long row = near_row(pos, p.tiles, 0);
    bool left = (over || *p.lost > p.lost_most) && fabsf(h) < INF && row < n_rows;
    // a value that kk rows reach: of the list, or what the row's limit, itself below such a value, comes from
    const NearBoundArgs a = near_args(sc, p.steps, d, e, nu);
    float value = LOWEST;
    if (left && over) {
        uint2 mine[PAIR_WORDS];
        pair_list(mine, p.entries + (size_t)of_list * (size_t)p.cap, p.cap);
        const float kth = pair_kth(mine, p.cap, kk);
        if (kth != LOWEST) {
            value = kth + h;
            // as many rows as the next search's lists hold that rounding does not tell from the kk-th: it would do no better (150 000 x 30 of 2000
            // copies each 111 -> 71 ms)
            const float limit = near_bound_from(value, h, a) - h;
            int within = 0;
#pragma unroll
            for (int j = 0; j < PAIR_WORDS; ++j)
                if (j * 64 < p.cap) within += __popcll(__ballot(__uint_as_float(mine[j].x) >= limit));
            left = within < p.cap || p.cap < p.cap_again;
            if (!left && lane == 0) near_panel_gone(p.todo, p.todo_mark, (int)(row >> 7));
        }
    } else if (left && p.limit[of_list] > LOWEST) value = p.limit[of_list] + h;
    if (threadIdx.x == 0) s_here = 0;
    __syncthreads();
    int at = 0;
    if (left && lane == 0) at = atomicAdd(&s_here, 1);
    __syncthreads();
    if (threadIdx.x == 0) s_from = s_here > 0 ? atomicAdd(out.count, s_here) : 0;
    __syncthreads();
    if (!left) return;
    if (lane != 0) return;
    const int i = s_from + at;
    out.row[i] = (int)row; out.pos[i] = pos; out.counts[i] = 0;
    out.reach[i] = pair_reach(value, h, a, sc, d);
    p.counts[of_list] = 0;
}
__global__ void __launch_bounds__(256) pairs_again_kernel(NearPairs p, int kk, const NearScale* __restrict__ sc, float e, float nu, int d, int first, int n,
                                                          PairsLeft left)
{
    const int i = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (i >= n || first + i >= *left.count) return;
    const int at = first + i;
    if (left.counts[at] <= p.cap) {
        if (lane == 0) left.reach[at] = -1.f;
        return;
    }
    const float h = -p.negh[left.pos[at]];
    uint2 mine[PAIR_WORDS];
    pair_list(mine, p.entries + (size_t)i * (size_t)p.cap, p.cap);
    const float kth = pair_kth(mine, p.cap, kk);
    if (lane != 0) return;
    const float reach = pair_reach(kth, h, near_args(sc, p.steps, d, e, nu), sc, d);
    const bool news = reach < 0.999f * left.reach[at];
    if (news) left.counts[at] = 0;                                      // (else: overflowed for good, which near_select finds)
    left.reach[at] = news ? reach : -1.f;
}

// ---------------------------------------------------------------------------------------------- launches
hipError_t pairs_emit(const NearPairs& p, int waves, hipStream_t s)
{
    if (p.tiles < 1 || p.tiles >= (1 << PAIR_TILE_BITS) || p.cap < 1 || p.cap > PAIRS_MOST || p.nseg < 1 || p.spread < 1) return hipErrorInvalidValue;
    const bool wide = p.steps > REG_STEPS;
    const int bt = wide ? 2 : waves / 2;
    if (p.blocks != (p.tiles + bt - 1) / bt || p.from < 0 || p.to > (p.once ? p.blocks / 2 + 1 : p.blocks) || (!p.once && (wide || waves > 4)) || waves > 12) return hipErrorInvalidValue;
    if (p.rows < 1 || p.rows % TILE != 0 || p.row0 < 0 || p.row0 != p.first * bt * TILE || p.row0 + p.rows > p.tiles * TILE || (p.once && p.rows != p.tiles * TILE) ||
        (p.row0 + p.rows < p.tiles * TILE && p.rows % (bt * TILE) != 0)) return hipErrorInvalidValue;
    const int blocks = (p.rows / TILE + bt - 1) / bt;
    const dim3 grid((unsigned)(blocks * p.nseg)), block((unsigned)(64 * (wide ? 8 : waves)));
    const size_t lds = (wide ? (size_t)WIDE_LDS : 2 * ((size_t)p.steps * FRAG_STEP + (p.once ? 1024 : 512))) + (size_t)(wide ? 8 : waves) * WAVE_LDS;
    auto run = [&](auto kernel) -> hipError_t {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(kernel, grid, block, lds, s, p);
        return hipGetLastError();
    };
    if (wide) return run(&pairs_wide_kernel<false>);
    switch (p.steps) {
        case 1: return p.once ? hipErrorInvalidValue : run(&pairs_kernel<1, false>);
        case 2: return p.once ? hipErrorInvalidValue : run(&pairs_kernel<2, false>);
        case 3: return p.once ? run(&pairs_kernel<3, true>) : run(&pairs_kernel<3, false>);
        case 4: return p.once ? run(&pairs_kernel<4, true>) : run(&pairs_kernel<4, false>);
        case 5: return p.once ? run(&pairs_kernel<5, true>) : run(&pairs_kernel<5, false>);
        case 6: return p.once ? run(&pairs_kernel<6, true>) : run(&pairs_kernel<6, false>);
        case 7: return p.once ? run(&pairs_kernel<7, true>) : run(&pairs_kernel<7, false>);
        case 8: return p.once ? run(&pairs_kernel<8, true>) : run(&pairs_kernel<8, false>);
        default: return hipErrorInvalidValue;
    }
}

hipError_t pairs_best(const NearPairs& p, hipStream_t s)
{
    if (p.tiles < 1 || p.steps <= REG_STEPS || p.nseg < 1 || p.spread < 1 || p.blocks != (p.tiles + 1) / 2 || p.from < 0 || p.to > p.blocks) return hipErrorInvalidValue;
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&pairs_wide_kernel<true>), hipFuncAttributeMaxDynamicSharedMemorySize, WIDE_LDS);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((pairs_wide_kernel<true>), dim3((unsigned)(p.blocks * p.nseg)), dim3(512), WIDE_LDS, s, p);
    return hipGetLastError();
}

hipError_t pairs_tighten(const NearPairs& p, int kk, const NearScale* sc, float e, float nu, int d, int32_t* last, hipStream_t s)
{
    hipLaunchKernelGGL(pairs_tighten_kernel, dim3((unsigned)(p.rows / 4)), dim3(256), 0, s, p, kk, sc, e, nu, d, last);
    return hipGetLastError();
}

hipError_t pairs_left(const NearPairs& p, int kk, const NearScale* sc, float e, float nu, int d, int n_rows, const PairsLeft& out, hipStream_t s)
{
    hipLaunchKernelGGL(pairs_left_kernel, dim3((unsigned)(p.rows / LEFT_ROWS)), dim3(64 * LEFT_ROWS), 0, s, p, kk, sc, e, nu, d, n_rows, out);
    return hipGetLastError();
}

hipError_t pairs_again(const NearPairs& p, int kk, const NearScale* sc, float e, float nu, int d, int first, int n, const PairsLeft& left, hipStream_t s)
{
    hipLaunchKernelGGL(pairs_again_kernel, dim3((unsigned)((n + 3) / 4)), dim3(256), 0, s, p, kk, sc, e, nu, d, first, n, left);
    return hipGetLastError();
}

}  // namespace slhc
