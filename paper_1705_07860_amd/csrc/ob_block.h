// Scan and stable radix sort of an array by one workgroup, for the device-wide primitives and for the scheduler of
// small graphs.  Written for wave64 (gfx950): ranking inside a wave uses 64-bit ballots.
#pragma once

#include "ob_internal.h"

namespace {

template <typename T> __device__ inline T zero_of();
template <> __device__ inline u32 zero_of<u32>() { return 0u; }
template <> __device__ inline Lay zero_of<Lay>() { Lay z; z.val = 0; z.dx = 0; z.ind = z.p0 = z.p1 = z.p2 = 0; return z; }
template <> __device__ inline Tri zero_of<Tri>() { Tri z; z.a = z.b = z.c = z.d = 0; return z; }
template <> __device__ inline CLay zero_of<CLay>() { CLay z; z.tf = z.wf = z.ta = z.wa = z.tb = z.p0 = z.p1 = z.p2 = 0; return z; }

// the element `off` lanes below (anything in the lanes that have none)
template <typename T>
__device__ inline T lane_below(const T &x, int off)
{
    static_assert(sizeof(T) % 4 == 0, "scan elements are whole words");
    u32 w[sizeof(T) / 4];
    __builtin_memcpy(w, &x, sizeof(T));
#pragma unroll
    for (u32 i = 0; i < sizeof(T) / 4; ++i) w[i] = __shfl_up(w[i], off);
    T r;
    __builtin_memcpy(&r, w, sizeof(T));
    return r;
}

// Exclusive scan of the per-thread values of a block: inside the waves by lane shuffles, across them through one LDS
// entry per wave, two barriers in all (a scan through LDS alone takes two per doubling).
// Returns the exclusive prefix of this thread; *block_total gets the sum over the block.
template <int WAVES, typename T>
__device__ inline T block_exclusive(const T &mine, T *lds, T *block_total)
{
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    T incl = mine;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const T below = lane_below(incl, off);
        if (lane >= off) incl = below + incl;
    }
    T excl = lane_below(incl, 1);
    if (lane == 0) excl = zero_of<T>();
    if (lane == 63) lds[w] = incl;
    __syncthreads();
    T before = zero_of<T>(), total = zero_of<T>();
    for (int i = 0; i < WAVES; ++i) {
        if (i == w) before = total;
        total = total + lds[i];
    }
    __syncthreads();
    *block_total = total;
    return before + excl;
}

// Exclusive scan of up to THREADS * ITEMS elements by one workgroup; lds: an element per wave.  in == out is fine.
template <int THREADS, int ITEMS, typename T>
__device__ inline void scan_one(const T *in, T *out, size_t n, T *total_out, T *lds)
{
    const size_t base = (size_t)threadIdx.x * ITEMS;
    T item[ITEMS];
    T sum = zero_of<T>();
    for (int i = 0; i < ITEMS; ++i) {
        item[i] = (base + i < n) ? in[base + i] : zero_of<T>();
        sum = sum + item[i];
    }
    T total;
    T run = block_exclusive<THREADS / 64, T>(sum, lds, &total);
    for (int i = 0; i < ITEMS; ++i) {
        if (base + i < n) out[base + i] = run;
        run = run + item[i];
    }
    if (threadIdx.x == 0 && total_out) *total_out = total;
}

// ---- radix sort ------------------------------------------------------------------------------
constexpr int RS_BITS = 8;
constexpr int RS_RADIX = 1 << RS_BITS;
constexpr int RS_THREADS = 1024;                 // 16 waves
constexpr int RS_WAVES = RS_THREADS / 64;
constexpr int RS_ROUNDS = 2;                     // keys per lane
constexpr int RS_WAVE_KEYS = 64 * RS_ROUNDS;     // 128 consecutive keys per wave
constexpr int RS_BLOCK = RS_WAVE_KEYS * RS_WAVES;  // 2048 keys per block
constexpr int RS_SEGS = RS_THREADS / RS_RADIX;   // threads per digit when the counts of all blocks are added up
constexpr u32 RS_OWN_BLOCKS = 256;               // up to here every block adds up the counts of the others itself

__device__ inline u32 digit_of(u64 key, int shift, u32 mask) { return (u32)(key >> shift) & mask; }

// lanes of the wave whose digit equals this lane's (0 where the lane holds no key)
__device__ inline u64 digit_peers(u32 d, bool ok)
{
    u64 peers = __ballot(ok);
#pragma unroll
    for (int b = 0; b < RS_BITS; ++b) {
        const bool bit = (d >> b) & 1u;
        const u64 m = __ballot(bit);
        peers &= bit ? m : ~m;
    }
    return ok ? peers : 0;
}

// Exclusive scan over the 256 digits: `mine` belongs to digit threadIdx.x, threads from 256 on only keep step at
// the barrier.  tot: four words of LDS.
__device__ inline u32 digit_exclusive(u32 mine, u32 *tot)
{
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    u32 incl = mine;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const u32 up = __shfl_up(incl, off);
        if (lane >= off) incl += up;
    }
    if (w < RS_RADIX / 64 && lane == 63) tot[w] = incl;
    __syncthreads();
    u32 before = 0;
    for (int i = 0; i < RS_RADIX / 64; ++i) before += i < w ? tot[i] : 0u;
    return before + incl - mine;
}

// Short inputs: the whole sort in one workgroup and one launch, both fields, all passes.  Every wave owns R * 64
// consecutive keys, in registers; a pass ranks them against the wave's own digit counts (lanes with equal digits by
// lane id, rounds in order), turns the counts of the sixteen waves into start positions and hands the pairs
// to their new owners through LDS.  Five barriers a pass whatever the size; memory is read and written once.
// Bound by latency.  The version before kept the pairs in memory and walked tiles of 1024, four barriers each,
// behind a scan of sixteen barriers.
constexpr size_t RS_SMALL_MAX = 8192;
struct RsFields { int lo[2], bits[2]; };
template <size_t N>
struct RsSmall {
    u64 key[N];
    u32 val[N];
    u32 cnt[RS_WAVES][RS_RADIX];
    u32 tot[RS_RADIX / 64];
};
template <int R, size_t N>
__device__ inline void rs_small(RsSmall<N> &S, u64 *keys, u32 *vals, u32 n, const RsFields &F)
{
    const u32 t = threadIdx.x, lane = t & 63u, w = t >> 6;
    const u32 base = w * (64u * R) + lane;
    u64 key[R];
    u32 val[R], rank[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const u32 i = base + 64u * r;
        key[r] = i < n ? keys[i] : 0;
        val[r] = i < n ? vals[i] : 0;
    }
    for (int f = 0; f < 2; ++f)
        for (int b = 0; b < F.bits[f]; b += RS_BITS) {
            const int bits = F.bits[f] - b < RS_BITS ? F.bits[f] - b : RS_BITS;
            const u32 mask = (1u << bits) - 1u;
            const int shift = F.lo[f] + b;
            for (u32 i = lane; i < RS_RADIX; i += 64) S.cnt[w][i] = 0;
            __syncthreads();
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const bool ok = base + 64u * r < n;
                const u32 d = digit_of(key[r], shift, mask);
                const u64 peers = digit_peers(d, ok);
                const int leader = peers ? (__ffsll((unsigned long long)peers) - 1) : (int)lane;
                u32 start = 0;
                if (ok && leader == (int)lane) start = atomicAdd(&S.cnt[w][d], (u32)__popcll(peers));
                rank[r] = __shfl(start, leader) + (u32)__popcll(peers & ((1ull << lane) - 1ull));
            }
            __syncthreads();
            u32 c[RS_WAVES], mine = 0;
            if (t < RS_RADIX) {
#pragma unroll
                for (int i = 0; i < RS_WAVES; ++i) { c[i] = S.cnt[i][t]; mine += c[i]; }
            }
            u32 run = digit_exclusive(mine, S.tot);
            if (t < RS_RADIX) {
#pragma unroll
                for (int i = 0; i < RS_WAVES; ++i) { S.cnt[i][t] = run; run += c[i]; }
            }
            __syncthreads();
#pragma unroll
            for (int r = 0; r < R; ++r)
                if (base + 64u * r < n) {
                    const u32 pos = S.cnt[w][digit_of(key[r], shift, mask)] + rank[r];
                    S.key[pos] = key[r];
                    S.val[pos] = val[r];
                }
            __syncthreads();
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const u32 i = base + 64u * r;
                if (i < n) { key[r] = S.key[i]; val[r] = S.val[i]; }
            }
        }
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const u32 i = base + 64u * r;
        if (i < n) { keys[i] = key[r]; vals[i] = val[r]; }
    }
}
}  // namespace
