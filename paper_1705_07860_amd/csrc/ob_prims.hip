// Device-wide primitives of the GPU scheduler: fill, exclusive scan, stable LSD radix sort.
// Written for wave64 (gfx950): ranking inside a wave uses 64-bit ballots.
#include "../../include/ob.h"
#include "ob_ctx.h"
#include "ob_block.h"

#include <mutex>

namespace {

constexpr int SCAN_THREADS = 256;
constexpr int SCAN_ITEMS = 4;
constexpr int SCAN_BLOCK = SCAN_THREADS * SCAN_ITEMS;  // 1024 elements per block

__global__ void k_fill_u32(u32 *p, u32 v, size_t n)
{
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    size_t stride = (size_t)gridDim.x * blockDim.x;
    for (; i < n; i += stride) p[i] = v;
}

template <typename T>
__global__ __launch_bounds__(SCAN_THREADS) void k_scan_local(const T *in, T *out, T *block_sums, size_t n)
{
    __shared__ T lds[SCAN_THREADS / 64];
    const size_t base = (size_t)blockIdx.x * SCAN_BLOCK + (size_t)threadIdx.x * SCAN_ITEMS;
    T item[SCAN_ITEMS];
    T sum = zero_of<T>();
    for (int i = 0; i < SCAN_ITEMS; ++i) {
        item[i] = (base + i < n) ? in[base + i] : zero_of<T>();
        sum = sum + item[i];
    }
    T total;
    T run = block_exclusive<SCAN_THREADS / 64, T>(sum, lds, &total);
    for (int i = 0; i < SCAN_ITEMS; ++i) {
        if (base + i < n) out[base + i] = run;
        run = run + item[i];
    }
    if (threadIdx.x == 0) block_sums[blockIdx.x] = total;
}

// One block turns the per-block sums into exclusive offsets, chunk by chunk with a carry.
template <typename T>
__global__ __launch_bounds__(SCAN_THREADS) void k_scan_sums(T *block_sums, size_t nblk, T *total_out)
{
    __shared__ T lds[SCAN_THREADS / 64];
    T carry = zero_of<T>();
    for (size_t c0 = 0; c0 < nblk; c0 += SCAN_THREADS) {
        const size_t i = c0 + threadIdx.x;
        T mine = (i < nblk) ? block_sums[i] : zero_of<T>();
        T total;
        T ex = block_exclusive<SCAN_THREADS / 64, T>(mine, lds, &total);
        if (i < nblk) block_sums[i] = carry + ex;
        carry = carry + total;
    }
    if (threadIdx.x == 0 && total_out) *total_out = carry;
}

template <typename T>
__global__ __launch_bounds__(SCAN_THREADS) void k_scan_add(T *out, const T *block_sums, size_t n)
{
    const T add = block_sums[blockIdx.x];
    const size_t base = (size_t)blockIdx.x * SCAN_BLOCK + (size_t)threadIdx.x * SCAN_ITEMS;
    for (int i = 0; i < SCAN_ITEMS; ++i)
        if (base + i < n) out[base + i] = out[base + i] + add;
}

// Up to SCAN_THREADS blocks: every block adds up the sums of the blocks before it itself (a few hundred
// integers), so the launch that scans the block sums is not needed.  Block 0 also leaves the total.
template <typename T>
__device__ inline T block_sum(T mine, T *lds)
{
    const int t = threadIdx.x;
    lds[t] = mine;
    __syncthreads();
    for (int off = SCAN_THREADS / 2; off > 0; off >>= 1) {
        if (t < off) lds[t] = lds[t] + lds[t + off];
        __syncthreads();
    }
    const T r = lds[0];
    __syncthreads();
    return r;
}
template <typename T>
__global__ __launch_bounds__(SCAN_THREADS) void k_scan_add_own(T *out, const T *block_sums, size_t nblk, size_t n, T *total_out)
{
    __shared__ T lds[SCAN_THREADS];
    const size_t t = threadIdx.x;
    const T add = block_sum<T>(t < blockIdx.x ? block_sums[t] : zero_of<T>(), lds);
    const size_t base = (size_t)blockIdx.x * SCAN_BLOCK + t * SCAN_ITEMS;
    for (int i = 0; i < SCAN_ITEMS; ++i)
        if (base + i < n) out[base + i] = out[base + i] + add;
    if (blockIdx.x == 0 && total_out) {
        const T total = block_sum<T>(t < nblk ? block_sums[t] : zero_of<T>(), lds);
        if (t == 0) *total_out = total;
    }
}

// Short inputs: one workgroup, one launch instead of two or three (the scheduler of a small graph is bound by the
// number of its launches).  in == out is fine.
constexpr int SCAN_SMALL_THREADS = 1024;
constexpr size_t SCAN_SMALL_MAX = (size_t)SCAN_SMALL_THREADS * SCAN_ITEMS;
template <typename T>
__global__ __launch_bounds__(SCAN_SMALL_THREADS) void k_scan_small(const T *in, T *out, size_t n, T *total_out)
{
    __shared__ T lds[SCAN_SMALL_THREADS / 64];
    scan_one<SCAN_SMALL_THREADS, SCAN_ITEMS>(in, out, n, total_out, lds);
}

template <typename T>
hipError_t scan_impl(const T *in, T *out, size_t n, T *total_dev, void *scratch, hipStream_t s)
{
    if (n == 0) {
        // total = 0
        if (total_dev) return hipMemsetAsync(total_dev, 0, sizeof(T), s);
        return hipSuccess;
    }
    if (n <= SCAN_SMALL_MAX) {
        hipLaunchKernelGGL(k_scan_small<T>, dim3(1), dim3(SCAN_SMALL_THREADS), 0, s, in, out, n, total_dev);
        return hipGetLastError();
    }
    const size_t nblk = (n + SCAN_BLOCK - 1) / SCAN_BLOCK;
    T *sums = (T *)scratch;
    hipLaunchKernelGGL(k_scan_local<T>, dim3((unsigned)nblk), dim3(SCAN_THREADS), 0, s, in, out, sums, n);
    if (nblk <= (size_t)SCAN_THREADS) {
        hipLaunchKernelGGL(k_scan_add_own<T>, dim3((unsigned)nblk), dim3(SCAN_THREADS), 0, s, out, sums, nblk, n, total_dev);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(k_scan_sums<T>, dim3(1), dim3(SCAN_THREADS), 0, s, sums, nblk, total_dev);
    if (nblk > 1)
        hipLaunchKernelGGL(k_scan_add<T>, dim3((unsigned)nblk), dim3(SCAN_THREADS), 0, s, out, sums, n);
    return hipGetLastError();
}

// number of keys of block blk whose digit is d: table[blk * 256 + d], or (dmajor, many blocks: the
// table is then scanned as it lies) table[d * nblk + blk]
__global__ __launch_bounds__(RS_THREADS) void k_rs_hist(const u64 *keys, size_t n, int shift, u32 mask,
                                                       u32 *table, u32 nblk, u32 dmajor)
{
    __shared__ u32 hist[RS_RADIX];
    const u32 t = threadIdx.x;
    if (t < RS_RADIX) hist[t] = 0;
    __syncthreads();
    const size_t base = (size_t)blockIdx.x * RS_BLOCK;
#pragma unroll
    for (int i = 0; i < RS_ROUNDS; ++i) {
        const size_t idx = base + (size_t)i * RS_THREADS + t;
        if (idx < n) atomicAdd(&hist[digit_of(keys[idx], shift, mask)], 1u);
    }
    __syncthreads();
    if (t < RS_RADIX) table[dmajor ? (size_t)t * nblk + blockIdx.x : (size_t)blockIdx.x * RS_RADIX + t] = hist[t];
}

// Stable scatter.  Wave w of a block owns 128 consecutive keys of the block's chunk and walks them in
// rounds of 64; inside a round lanes with equal digits are ranked by lane id.
// The first output positions come from the table of counts: thread (segment, digit) adds up a quarter of the
// blocks for its digit, once over all of them and once over those before its own.  A pass is bound by its
// launches and by latency (52 000 pairs are 0.6 MB), so every block reads the whole table (26 KB there, 16 loads in
// flight per thread) where one workgroup turned it into positions in a launch of its own, and a block is
// wide and its chunk short: four threads per digit, and few blocks to add up.
__global__ __launch_bounds__(RS_THREADS) void k_rs_scatter(const u64 *keys, const u32 *vals, u64 *keys_out,
                                                          u32 *vals_out, size_t n, int shift, u32 mask,
                                                          const u32 *table, u32 nblk, u32 dmajor)
{
    __shared__ u32 cnt[RS_WAVES][RS_RADIX];
    __shared__ u32 seg_all[RS_SEGS][RS_RADIX], seg_before[RS_SEGS][RS_RADIX], s_tot[RS_RADIX / 64];
    const u32 t = threadIdx.x, lane = t & 63u, w = t >> 6, blk = blockIdx.x;
    for (u32 i = lane; i < RS_RADIX; i += 64) cnt[w][i] = 0;
    const size_t wbase = (size_t)blk * RS_BLOCK + (size_t)w * RS_WAVE_KEYS;
    u64 key[RS_ROUNDS];
    u32 val[RS_ROUNDS];
    bool ok[RS_ROUNDS];
#pragma unroll
    for (int r = 0; r < RS_ROUNDS; ++r) {
        const size_t idx = wbase + (size_t)r * 64 + lane;
        ok[r] = idx < n;
        key[r] = ok[r] ? keys[idx] : 0;
        val[r] = ok[r] ? vals[idx] : 0;
    }
    if (!dmajor) {
        const u32 d = t & (RS_RADIX - 1), seg = t / RS_RADIX;
        const u32 per = (nblk + RS_SEGS - 1) / RS_SEGS;
        const u32 b0 = seg * per < nblk ? seg * per : nblk, b1 = b0 + per < nblk ? b0 + per : nblk;
        u32 all = 0, before = 0;
        for (u32 b = b0; b < b1; b += 16) {
            u32 c[16];
#pragma unroll
            for (u32 q = 0; q < 16; ++q) c[q] = b + q < b1 ? table[(size_t)(b + q) * RS_RADIX + d] : 0u;
#pragma unroll
            for (u32 q = 0; q < 16; ++q) { all += c[q]; before += b + q < blk ? c[q] : 0u; }
        }
        seg_all[seg][d] = all;
        seg_before[seg][d] = before;
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < RS_ROUNDS; ++r)
        if (ok[r]) atomicAdd(&cnt[w][digit_of(key[r], shift, mask)], 1u);
    u32 run = 0, mine = 0;
    if (t < RS_RADIX) {
        if (dmajor) run = table[(size_t)t * nblk + blk];
        else for (int q = 0; q < RS_SEGS; ++q) { mine += seg_all[q][t]; run += seg_before[q][t]; }
    }
    const u32 smaller = digit_exclusive(mine, s_tot);   // (its barrier also closes the counting)
    if (t < RS_RADIX) {   // thread d turns the per-wave counts of digit d into per-wave start positions
        run += smaller;
        u32 c[RS_WAVES];
#pragma unroll
        for (int i = 0; i < RS_WAVES; ++i) c[i] = cnt[i][t];
#pragma unroll
        for (int i = 0; i < RS_WAVES; ++i) { cnt[i][t] = run; run += c[i]; }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < RS_ROUNDS; ++r) {
        const u32 d = digit_of(key[r], shift, mask);
        const u64 peers = digit_peers(d, ok[r]);
        const u32 rank = (u32)__popcll(peers & ((1ull << lane) - 1ull));
        const int leader = peers ? (__ffsll((unsigned long long)peers) - 1) : (int)lane;
        u32 start = 0;
        if (ok[r] && leader == (int)lane) start = atomicAdd(&cnt[w][d], (u32)__popcll(peers));
        start = __shfl(start, leader);
        if (ok[r]) {
            keys_out[start + rank] = key[r];
            vals_out[start + rank] = val[r];
        }
    }
}

__global__ __launch_bounds__(RS_THREADS) void k_rs_small(u64 *keys, u32 *vals, u32 n, RsFields F, const u32 *n_dev)
{
    __shared__ RsSmall<RS_SMALL_MAX> S;
    if (n_dev) n = *n_dev < n ? *n_dev : n;   // the same value for every thread: the barriers stay uniform
    if (n <= 1024) rs_small<1>(S, keys, vals, n, F);
    else if (n <= 2048) rs_small<2>(S, keys, vals, n, F);
    else if (n <= 4096) rs_small<4>(S, keys, vals, n, F);
    else rs_small<8>(S, keys, vals, n, F);
}

}  // namespace

// ---- host wrappers -------------------------------------------------------------------------------

static inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

size_t prim_scan_scratch_bytes(size_t n, size_t elem)
{
    return align256(((n + SCAN_BLOCK - 1) / SCAN_BLOCK + 1) * elem);
}

hipError_t prim_fill_u32(u32 *p, u32 v, size_t n, hipStream_t s)
{
    if (n == 0) return hipSuccess;
    size_t blocks = (n + 1023) / 1024;
    if (blocks > 2048) blocks = 2048;
    hipLaunchKernelGGL(k_fill_u32, dim3((unsigned)blocks), dim3(256), 0, s, p, v, n);
    return hipGetLastError();
}

hipError_t prim_scan_u32(const u32 *in, u32 *out, size_t n, u32 *total_dev, void *scratch, hipStream_t s)
{
    return scan_impl<u32>(in, out, n, total_dev, scratch, s);
}

hipError_t prim_scan_lay(const Lay *in, Lay *out, size_t n, Lay *total_dev, void *scratch, hipStream_t s)
{
    return scan_impl<Lay>(in, out, n, total_dev, scratch, s);
}

hipError_t prim_scan_clay(const CLay *in, CLay *out, size_t n, CLay *total_dev, void *scratch, hipStream_t s)
{
    return scan_impl<CLay>(in, out, n, total_dev, scratch, s);
}

hipError_t prim_scan_tri(const Tri *in, Tri *out, size_t n, Tri *total_dev, void *scratch, hipStream_t s)
{
    return scan_impl<Tri>(in, out, n, total_dev, scratch, s);
}

size_t prim_sort_scratch_bytes(size_t n)
{
    const size_t nblk = (n + RS_BLOCK - 1) / RS_BLOCK;
    const size_t table = align256((size_t)RS_RADIX * (nblk ? nblk : 1) * sizeof(u32));
    return table + prim_scan_scratch_bytes((size_t)RS_RADIX * (nblk ? nblk : 1), sizeof(u32));
}

// Stable sort by the bits [lo, lo + bits) of one or two fields, the less significant field first.
static hipError_t sort_pairs_impl(u64 *keys, u32 *vals, u64 *keys_tmp, u32 *vals_tmp, size_t n, const RsFields &F,
                                  void *scratch, hipStream_t s, int *n_launches, const u32 *n_dev, bool *in_tmp)
{
    if (in_tmp) *in_tmp = false;
    if (n <= 1 || (F.bits[0] <= 0 && F.bits[1] <= 0)) return hipSuccess;
    if (n <= RS_SMALL_MAX) {
        hipLaunchKernelGGL(k_rs_small, dim3(1), dim3(RS_THREADS), 0, s, keys, vals, (u32)n, F, n_dev);
        if (n_launches) *n_launches += 1;
        return hipGetLastError();
    }
    const u32 nblk = (u32)((n + RS_BLOCK - 1) / RS_BLOCK);
    u32 *table = (u32 *)scratch;
    void *scan_scratch = (char *)scratch + align256((size_t)RS_RADIX * nblk * sizeof(u32));
    u64 *kin = keys, *kout = keys_tmp;
    u32 *vin = vals, *vout = vals_tmp;
    int passes = 0;
    // up to RS_OWN_BLOCKS blocks the scatter adds up the counts itself; what its blocks read together grows with the
    // square of their number (64 MB there), so beyond the table is laid out digit-major and scanned
    const u32 dmajor = nblk > RS_OWN_BLOCKS ? 1u : 0u;
    for (int f = 0; f < 2; ++f)
        for (int b = 0; b < F.bits[f]; b += RS_BITS) {
            const int bits = (F.bits[f] - b < RS_BITS) ? (F.bits[f] - b) : RS_BITS;
            const u32 mask = (1u << bits) - 1u;
            const int shift = F.lo[f] + b;
            hipLaunchKernelGGL(k_rs_hist, dim3(nblk), dim3(RS_THREADS), 0, s, kin, n, shift, mask, table, nblk, dmajor);
            if (dmajor) {
                hipError_t e = scan_impl<u32>(table, table, (size_t)RS_RADIX * nblk, (u32 *)nullptr, scan_scratch, s);
                if (e != hipSuccess) return e;
            }
            hipLaunchKernelGGL(k_rs_scatter, dim3(nblk), dim3(RS_THREADS), 0, s, kin, vin, kout, vout, n, shift,
                               mask, table, nblk, dmajor);
            u64 *tk = kin; kin = kout; kout = tk;
            u32 *tv = vin; vin = vout; vout = tv;
            ++passes;
            if (n_launches) *n_launches += !dmajor ? 2 : ((size_t)RS_RADIX * nblk <= (size_t)SCAN_THREADS * SCAN_BLOCK ? 4 : 5);
        }
    if ((passes & 1) && in_tmp) {   // the caller takes the result where it is
        *in_tmp = true;
    } else if (passes & 1) {  // result sits in the tmp arrays: copy back
        hipError_t e = hipMemcpyAsync(keys, kin, n * sizeof(u64), hipMemcpyDeviceToDevice, s);
        if (e != hipSuccess) return e;
        e = hipMemcpyAsync(vals, vin, n * sizeof(u32), hipMemcpyDeviceToDevice, s);
        if (e != hipSuccess) return e;
    }
    return hipGetLastError();
}

hipError_t prim_sort_pairs(u64 *keys, u32 *vals, u64 *keys_tmp, u32 *vals_tmp, size_t n, int lo_bit,
                           int n_bits, void *scratch, hipStream_t s, int *n_launches, const u32 *n_dev)
{
    return sort_pairs_impl(keys, vals, keys_tmp, vals_tmp, n, RsFields{{lo_bit, 0}, {n_bits, 0}}, scratch, s, n_launches, n_dev,
                           nullptr);
}

// The same sort without the copy back after an odd number of passes: the two buffer pairs change
// roles instead (on return keys / vals point at the sorted data, keys_tmp / vals_tmp at the other pair).
// By [lo2, lo2 + bits2), among equals by [lo_bit, lo_bit + n_bits).
hipError_t prim_sort_pairs_swap(u64 *&keys, u32 *&vals, u64 *&keys_tmp, u32 *&vals_tmp, size_t n, int lo_bit, int n_bits,
                                int lo2, int bits2, void *scratch, hipStream_t s, int *n_launches, const u32 *n_dev)
{
    bool in_tmp = false;
    hipError_t e = sort_pairs_impl(keys, vals, keys_tmp, vals_tmp, n, RsFields{{lo_bit, lo2}, {n_bits, bits2}}, scratch, s,
                                   n_launches, n_dev, &in_tmp);
    if (in_tmp) {
        u64 *tk = keys; keys = keys_tmp; keys_tmp = tk;
        u32 *tv = vals; vals = vals_tmp; vals_tmp = tv;
    }
    return e;
}

// ---- the sort for callers that cannot allocate ------------------------------------------------------
// Everything the sort needs beyond the caller's two arrays (the second key / value buffer of the
// ping-pong passes, the per-block digit table and the scan's block sums) lies in one array in the
// library's own device image, so the call reaches no allocator.  Each GPU holds its own copy of
// the array at its own address; the address is looked up once per device and kept.
constexpr size_t NOALLOC_TABLE_BYTES = ((size_t)OB_NOALLOC_MAX_PAIRS / RS_BLOCK + 1) * RS_RADIX * sizeof(u32) + 4096;
constexpr size_t NOALLOC_KEYS_OFF = 0;
constexpr size_t NOALLOC_VALS_OFF = (size_t)OB_NOALLOC_MAX_PAIRS * sizeof(u64);
constexpr size_t NOALLOC_TABLE_OFF = NOALLOC_VALS_OFF + (size_t)OB_NOALLOC_MAX_PAIRS * sizeof(u32);
constexpr size_t NOALLOC_BYTES = NOALLOC_TABLE_OFF + 2 * NOALLOC_TABLE_BYTES;
static_assert(NOALLOC_VALS_OFF % 256 == 0 && NOALLOC_TABLE_OFF % 256 == 0, "sections of the scratch array stay 256-byte aligned");
static __device__ __align__(256) unsigned char scratch[NOALLOC_BYTES];

constexpr int NOALLOC_MAX_DEVICES = 64;
static std::mutex g_noalloc_mutex;
static void *g_noalloc_ptr[NOALLOC_MAX_DEVICES] = {};

// device address of the current device's copy of `scratch` (host code never uses the array's name
// for anything else: on the host it is only a handle for this look-up)
static int noalloc_scratch(char **out)
{
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return ctx_fail(nullptr, OB_E_HIP, "hipGetDevice failed: %s", hipGetErrorString(e));
    if (dev < 0 || dev >= NOALLOC_MAX_DEVICES) return ctx_fail(nullptr, OB_E_RANGE, "device index %d outside 0 .. %d", dev, NOALLOC_MAX_DEVICES - 1);
    std::lock_guard<std::mutex> lock(g_noalloc_mutex);
    if (!g_noalloc_ptr[dev]) {
        void *ptr = nullptr;
        e = hipGetSymbolAddress((void **)&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !ptr)
            return ctx_fail(nullptr, OB_E_HIP, "hipGetSymbolAddress(scratch) failed on device %d: %s", dev, hipGetErrorString(e));
        g_noalloc_ptr[dev] = ptr;
    }
    *out = (char *)g_noalloc_ptr[dev];
    return OB_OK;
}

extern "C" int ob_sort_pairs_noalloc(void *hip_stream, size_t n, uint64_t *keys_dev, uint32_t *vals_dev, int lo_bit, int n_bits)
{
    if (n > (size_t)OB_NOALLOC_MAX_PAIRS)
        return ctx_fail(nullptr, OB_E_RANGE, "ob_sort_pairs_noalloc: %zu pairs, the built-in scratch holds at most %d", n,
                        (int)OB_NOALLOC_MAX_PAIRS);
    if (lo_bit < 0 || n_bits < 0 || lo_bit + n_bits > 64)
        return ctx_fail(nullptr, OB_E_ARG, "ob_sort_pairs_noalloc: bits [%d, %d) outside a 64-bit key", lo_bit, lo_bit + n_bits);
    if (n == 0) return OB_OK;
    if (!keys_dev || !vals_dev) return ctx_fail(nullptr, OB_E_ARG, "ob_sort_pairs_noalloc: null array");
    char *base = nullptr;
    if (int rc = noalloc_scratch(&base)) return rc;
    // Nothing in the scratch has to start at zero: every pass writes each entry of the digit table
    // and of the block sums it reads, and the second buffers are written before they are read, so
    // what an earlier (larger) call left behind is never looked at.
    hipError_t e = prim_sort_pairs(keys_dev, vals_dev, (u64 *)(base + NOALLOC_KEYS_OFF), (u32 *)(base + NOALLOC_VALS_OFF), n, lo_bit,
                                   n_bits, base + NOALLOC_TABLE_OFF, (hipStream_t)hip_stream, nullptr);
    if (e != hipSuccess) return ctx_fail(nullptr, OB_E_HIP, "ob_sort_pairs_noalloc: %s", hipGetErrorString(e));
    return OB_OK;
}
