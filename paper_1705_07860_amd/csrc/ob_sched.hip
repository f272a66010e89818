// GPU scheduler: node signatures as integer hashes (Appendix B), depth (Section 3.2) by ranges of node ids
// that settle side by side (or, as the fallback, by frontier passes of one workgroup over the successor CSR),
// batches = equal (depth, signature) found by a stable radix sort, then the
// memory layout of the batched execution (Section 3.3: operands of a batch must be
// addressable as one matrix; results are laid out contiguously in batch order).
#include "ob_ctx.h"
#include "ob_block.h"

#include <type_traits>

namespace {

constexpr int TPB = 256;
inline unsigned blocks_for(size_t n, int per = TPB) { return (unsigned)((n + per - 1) / per); }

__device__ inline u64 mix64(u64 x)
{
    x ^= x >> 33; x *= 0xff51afd7ed558ccdULL;
    x ^= x >> 33; x *= 0xc4ceb9fe1a85ec53ULL;
    x ^= x >> 33;
    return x;
}
__device__ inline u64 comb(u64 h, u64 x) { return mix64(h ^ (x + 0x9e3779b97f4a7c15ULL + (h << 6) + (h >> 2))); }

// start values: the first `zeros` elements zero, the others all ones
__global__ void k_clear(uint4 *p, size_t zeros, size_t n)
{
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
        const u32 v = i < zeros ? 0u : ~0u;
        p[i] = make_uint4(v, v, v, v);
    }
}

// ---- stage 1: signatures, out-degrees, edges by producer -------------------------------------
// The rows of a workgroup that have too many edges for a thread, as one list of edges that all its threads walk: an entry
// finds its row by bisection in LDS.
template <u32 N> struct WideRows {
    u64 n;                              // rows << 32 | edges: one atomic gives a row its place in both
    u32 row[N], lo[N], at[N];     // row, its first edge, its first entry of the list
};
constexpr u32 WIDE_STEP = 4;            // entries a thread takes at a time: their reads run side by side
template <u32 N> __device__ inline void wide_add(WideRows<N> &S, u32 row, u32 lo, u32 edges)
{
    const u64 was = atomicAdd((unsigned long long *)&S.n, (1ull << 32) | edges);
    const u32 i = (u32)(was >> 32);
    S.row[i] = row; S.lo[i] = lo; S.at[i] = (u32)was;
}
template <u32 N> __device__ inline u32 wide_row(const WideRows<N> &S, u32 rows, u32 x)
{
    u32 lo = 0, hi = rows;              // at[lo] <= x < at[hi]
    while (hi - lo > 1) {
        const u32 mid = (lo + hi) >> 1;
        if (S.at[mid] <= x) lo = mid; else hi = mid;
    }
    return lo;
}

// Signature tuple (Section 3.2 / Appendix A): operation, output dimension, arity, shared
// parameter ids (the A and y of A x + y), slice range, operand dimensions.  LOOKUP's row,
// PICK_NLS's label and INPUT's payload are data and stay out.  The operands' dimensions enter as a
// sum of position-salted hashes, so that a node with many operands can be summed by many threads.
// A thread takes a node with up to INIT_OPS operands, edges included; the edges of nodes with more are shared out over
// the workgroup (WideRows).  (A launch with a thread per edge had to look its node up by bisection in memory and
// meet all operands of a wide sum in atomics on one signature: 23 us for 52 000 edges, 169 us for 480 000 of
// which one node holds 10 000, beside 8 and 16 us of this kernel without the edges; 10.5 and 37 us together now.
// With the wide nodes taken by the workgroup one after the other, 4 096 sums of nine operands side by side took
// 768 us, 18 now.)
// steps: 0 = every node is its own step, 1 = steps come from the depth pass by id ranges, 2 = steps are the
// caller's batch labels, 3 = steps come from the single-workgroup depth pass (leaves are queued here).
constexpr u32 INIT_OPS = 8;
__device__ inline u64 operand_hash(const Tables &T, u32 u, u32 j) { return mix64(comb(0x5bd1e995ULL + j, T.out_dim[u])); }

template <u32 N> struct InitLds {
    WideRows<N> wide;
    u64 sum[N];
    u32 ends[N / 64];
};
// (a workgroup of N threads, the nodes from `base` on.  The nodes that a gated cell may end in are listed in passing: T.cell_ends
// from `base` on, as many as T.cell_ends_n says for the part.)
template <u32 N>
__device__ inline void node_init_part(const Tables &T, int steps, u64 *keys, u32 *vals, InitLds<N> &L, u32 base)
{
    WideRows<N> &S = L.wide;
    u64 *s_sum = L.sum;
    if (threadIdx.x == 0) S.n = 0;
    s_sum[threadIdx.x] = 0;
    __syncthreads();
    const u32 v = base + threadIdx.x;
    bool ends = false;
    if (v < T.n) {
        const u32 lo = T.in_off[v], hi = T.in_off[v + 1];
        const u32 o = T.op[v];
        u64 h = mix64(o + 1);
        h = comb(h, T.out_dim[v]);
        h = comb(h, hi - lo);
        h = comb(h, (u64)(u32)(T.param[v] + 1));
        h = comb(h, (u64)(u32)(T.bias[v] + 1));
        h = comb(h, o == OP_SLICE ? (u64)(u32)T.aux0[v] : 0);
        h = comb(h, o == OP_SLICE ? (u64)(u32)T.aux1[v] : 0);
        if (hi - lo <= INIT_OPS) {
            for (u32 e = lo; e < hi; ++e) {
                const u32 u = T.in_idx[e];
                T.edge_cons[e] = v;
                keys[e] = u;
                vals[e] = e;
                atomicAdd(&T.outdeg[u], 1u);
                h += operand_hash(T, u, e - lo);
            }
        } else {
            wide_add(S, v, lo, hi - lo);
        }
        T.sig[v] = h;
        if (T.cells) {
            const u32 x = hi > lo ? T.in_idx[lo] : 0u, y = hi > lo + 1u ? T.in_idx[lo + 1u] : 0u;
            T.nrec[v] = make_uint4(x, y, o, hi - lo);
            T.cell_rows[v] = T.cell_nodes[v] = T.cell_prods[v] = T.cell_takes[v] = 0;
            T.slot_chains[v] = T.slot_rows[v] = T.slot_cells[v] = T.dx_cell[v] = 0;
            if (o == OP_CMULT) {
                const u32 ox = T.op[x], oy = T.op[y];
                ends = (ox == OP_TANH && oy == OP_SIGMOID) || (ox == OP_SIGMOID && oy == OP_TANH);
            }
        }
        if (steps == 3) {
            T.indeg[v] = hi - lo;
            if (hi == lo) {
                const u32 pos = atomicAdd(&T.qcount[0], 1u);
                T.queue[pos] = v;
                T.step[v] = 0;
            }
        } else if (steps == 2) {
            T.step[v] = T.manual[v];   // manual batching: replaced by the label's rank once batches are cut
        } else if (steps == 0) {
            T.step[v] = v;   // unbatched: every node is its own step, in id order
        }
    }
    const u32 lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
    const u64 with = __ballot(ends);
    if (lane == 0u) L.ends[wave] = (u32)__popcll(with);
    __syncthreads();
    if (T.cells) {
        u32 before = 0;
        for (u32 i = 0; i < wave; ++i) before += L.ends[i];
        if (ends) T.cell_ends[base + before + (u32)__popcll(with & ((1ull << lane) - 1ull))] = v;
        if (threadIdx.x == N - 1u) T.cell_ends_n[base / N] = before + (u32)__popcll(with);
    }
    const u32 rows = (u32)(S.n >> 32), edges = (u32)S.n;
    u32 mine = ~0u;         // row whose sum this thread is adding up
    u64 sum = 0;
    for (u32 x0 = threadIdx.x; x0 < edges; x0 += WIDE_STEP * N) {
        u32 i[WIDE_STEP], j[WIDE_STEP], u[WIDE_STEP];
#pragma unroll
        for (u32 q = 0; q < WIDE_STEP; ++q) {
            const u32 x = x0 + q * N < edges ? x0 + q * N : x0;
            i[q] = wide_row(S, rows, x);
            j[q] = x - S.at[i[q]];
            u[q] = T.in_idx[S.lo[i[q]] + j[q]];
        }
#pragma unroll
        for (u32 q = 0; q < WIDE_STEP; ++q) {
            if (x0 + q * N >= edges) continue;
            const u32 e = S.lo[i[q]] + j[q];
            T.edge_cons[e] = S.row[i[q]];
            keys[e] = u[q];
            vals[e] = e;
            atomicAdd(&T.outdeg[u[q]], 1u);
            if (i[q] != mine) {
                if (mine != ~0u) atomicAdd((unsigned long long *)&s_sum[mine], (unsigned long long)sum);
                mine = i[q]; sum = 0;
            }
            sum += operand_hash(T, u[q], j[q]);
        }
    }
    if (mine != ~0u) atomicAdd((unsigned long long *)&s_sum[mine], (unsigned long long)sum);
    __syncthreads();
    if (threadIdx.x < rows) T.sig[S.row[threadIdx.x]] += s_sum[threadIdx.x];
}
__global__ __launch_bounds__(TPB) void k_node_init(Tables T, int steps, u64 *keys, u32 *vals)
{
    __shared__ InitLds<TPB> L;
    node_init_part<TPB>(T, steps, keys, vals, L, blockIdx.x * TPB);
}

// after the sort: succ_edge[q] = edge id, succ_node[q] = its consumer (which
// saves the single-workgroup depth pass and the agenda a hop)
__device__ inline void succ_finish_at(const Tables &T, const u32 *sorted_edge, u32 *succ_node, u32 q)
{
    if (q >= T.E) return;
    const u32 e = sorted_edge[q];
    T.succ_edge[q] = e;
    succ_node[q] = T.edge_cons[e];
}
__global__ void k_succ_finish(Tables T, const u32 *sorted_edge, u32 *succ_node)
{
    succ_finish_at(T, sorted_edge, succ_node, blockIdx.x * blockDim.x + threadIdx.x);
}

// ---- stage 2: depth by frontier passes (the fallback) --------------------------------------------
// One workgroup walks the graph level by level.  queue[head, tail) is the current frontier
// (all nodes of depth `level`); a node joins the next frontier when its last unresolved
// dependency is resolved, which is exactly when the deepest of its operands has been
// processed, so its depth is level + 1 (depth = longest path from a leaf, Section 3.2).
constexpr int FRONTIER_THREADS = 1024;
__global__ __launch_bounds__(FRONTIER_THREADS) void k_depth_frontier(Tables T, const u32 *succ_node)
{
    __shared__ u32 s_head, s_tail, s_next;
    if (threadIdx.x == 0) { s_head = 0; s_tail = T.qcount[0]; s_next = T.qcount[0]; }
    __syncthreads();
    u32 level = 0;
    while (true) {
        const u32 head = s_head, tail = s_tail;
        if (head == tail) break;
        for (u32 i = head + threadIdx.x; i < tail; i += FRONTIER_THREADS) {
            const u32 u = T.queue[i];
            const u32 q1 = T.succ_off[u + 1];
            for (u32 q = T.succ_off[u]; q < q1; ++q) {
                const u32 s = succ_node[q];
                if (atomicSub(&T.indeg[s], 1u) == 1u) {
                    T.step[s] = level + 1;
                    const u32 pos = atomicAdd(&s_next, 1u);
                    T.queue[pos] = s;
                }
            }
        }
        __syncthreads();
        if (threadIdx.x == 0) { s_head = tail; s_tail = s_next; }
        __syncthreads();
        ++level;
    }
    if (threadIdx.x == 0) {
        T.hdr->frontier_done = s_tail;
        if (s_tail != T.n) atomicOr(&T.hdr->err, (u32)ERR_CYCLE);
    }
}

// Depth by id ranges.  Ids are a topological order, so depth(v) = 1 + the largest operand depth can be
// taken range by range: a workgroup owns DEPTH_PART consecutive ids, a thread DEPTH_NPT of them, with the
// operands of its nodes in registers (an operand inside the range is an LDS word, one of a lower range a word
// of g_dep) and the depths of the range in LDS, one word per node: 0 = not known yet, depth + 1 otherwise.
// A sweep looks at the operand words of all nodes of a wave at once and settles every node whose operands are
// all settled; each word is written once, so waves need no barrier between sweeps and run freely.  A thread's
// nodes are consecutive ids, which programs write along their recurrences, and a node settled in a sweep is
// handed to the thread's later nodes in registers: an LSTM cell of sixteen nodes and eight levels takes four sweeps.  A settled
// depth also goes to g_dep, where higher ranges poll for it: the word is its own flag, so no fence is needed.
// A node with more than DEPTH_OPS operands looks at three of them at a time: a settled one makes room for the next
// of its list, all such nodes of a wave side by side, and the last three are waited for like any others.  That is
// a third of a sweep per operand, so where a wave has few such nodes and they are long (a sum over a whole
// minibatch), the wave walks them instead, one after the other, eight reads per lane at a time, whenever nothing else of
// the wave moves.  A walk step takes about as long as four sweeps, which is where
// DEPTH_WALK puts the line.  (With all of them walked, 64 recurrences of 60 steps with a sum of five operands each took
// 5 100 us for this pass, sequences of 60 states with a sum over all earlier ones 2 280; now 109 and 210.)
// What bounds it: one dependent LDS read plus some forty instructions per level of the longest path, which is
// why a wave holds no more than four nodes per lane and a workgroup one wave per SIMD.  The pass this
// replaces kept a frontier queue per 4 096 ids (queue, counter, successor and queue again: five dependent LDS
// operations per level).
// Only lower ranges are waited for and the lowest waits for nobody; every wait is bounded.  A workgroup takes the lowest
// range that is not taken yet (T.qcount[1] counts them), so what it waits for is done or on the chip, however many ranges
// there are, whatever part of the chip the stream has and in whichever order workgroups start.
constexpr u32 DEPTH_THREADS = 256;
constexpr u32 DEPTH_NPT = 4;          // nodes per thread
constexpr u32 DEPTH_PART = DEPTH_THREADS * DEPTH_NPT;   // ids per workgroup
constexpr u32 DEPTH_OPS = 4;          // operands of a node that are kept in registers
constexpr u32 DEPTH_ONE = DEPTH_PART;         // LDS word that always holds 1: an absent operand
constexpr u32 DEPTH_NEVER = DEPTH_PART + 1;   // LDS word that always holds 0: an operand that cannot be read here (yet)
constexpr u32 DEPTH_WALKED = DEPTH_PART + 2;  // reads as DEPTH_NEVER: the node's wave walks it
constexpr u32 DEPTH_EXT = 0x80000000u;        // operand of a lower range: this bit and its id (reads as DEPTH_NEVER)
constexpr u32 DEPTH_LIST = DEPTH_OPS - 1;     // operands of a longer node that are looked at at a time (its first word holds it back until its list is through)
constexpr u32 DEPTH_WALK = 4 * DEPTH_LIST;    // a wave walks the nodes with more operands than this times the number of its long nodes
constexpr u32 DEPTH_WIDE_READS = 8;   // operands per lane of one step of such a walk
constexpr u32 DEPTH_MAX_ARITY = 60000;   // beyond, the single-workgroup pass counts the operands down instead of walking them

__device__ inline u32 lds_load(const u32 *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP); }
__device__ inline void lds_store(u32 *p, u32 v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP); }
__device__ inline void depth_settle(u32 *s_word, u32 *g_word, u32 d)
{
    __hip_atomic_store(s_word, d, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    __hip_atomic_store(g_word, d, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__global__ __launch_bounds__(DEPTH_THREADS) void k_depth_partitioned(Tables T, u32 *g_dep, u32 spin_limit)
{
    __shared__ u32 s_dep[DEPTH_PART + 2];
    __shared__ unsigned short s_wide[DEPTH_THREADS / 64][64 * DEPTH_NPT];
    __shared__ u32 s_quit, s_range;
    const u32 tid = threadIdx.x, lane = tid & 63u, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const u64 lt_mask = (1ull << lane) - 1ull;
    if (tid == 0) s_range = gridDim.x > 1u ? atomicAdd(&T.qcount[1], 1u) : 0u;
    for (u32 i = tid; i < DEPTH_PART + 2; i += DEPTH_THREADS) s_dep[i] = i == DEPTH_ONE ? 1u : 0u;
    if (tid == 0) s_quit = 0;
    __syncthreads();
    const u32 lo = __builtin_amdgcn_readfirstlane(s_range) * DEPTH_PART;
    // node j of a lane: local id first + j
    const u32 first = tid * DEPTH_NPT;
    bool fwd0[DEPTH_NPT][DEPTH_NPT], fwd1[DEPTH_NPT][DEPTH_NPT];   // operand 0 / 1 of node j is the lane's own node i < j
    u32 op[DEPTH_NPT][DEPTH_OPS], ext[DEPTH_NPT], dep[DEPTH_NPT];   // ext: largest word among settled operands of lower ranges
    u32 in0[DEPTH_NPT], ar[DEPTH_NPT], next[DEPTH_NPT];   // operand list; operands of a long node that have been looked at
    bool wide[DEPTH_NPT], has_ext = false, has_34 = false, has_list = false;
    u32 n_long = 0;
#pragma unroll
    for (u32 j = 0; j < DEPTH_NPT; ++j) {
        const u32 l = first + j, v = lo + l;
        const bool live = v < T.n;
        in0[j] = live ? T.in_off[v] : 0u;
        ar[j] = live ? T.in_off[v + 1] - in0[j] : 0u;
        ext[j] = 0;
        dep[j] = ar[j] ? 0u : 1u;
#pragma unroll
        for (u32 q = 0; q < DEPTH_OPS; ++q) {
            op[j][q] = DEPTH_ONE;
            if (q < ar[j] && ar[j] <= DEPTH_OPS) {
                const u32 u = T.in_idx[in0[j] + q];
                op[j][q] = u >= lo ? u - lo : (DEPTH_EXT | u);
                has_ext = has_ext || u < lo;
            }
        }
#pragma unroll
        for (u32 i = 0; i < DEPTH_NPT; ++i) { fwd0[j][i] = op[j][0] == first + i; fwd1[j][i] = op[j][1] == first + i; }
        if (live && ar[j] == 0) depth_settle(&s_dep[l], &g_dep[v], 1u);
        n_long += (u32)__popcll(__ballot(ar[j] > DEPTH_OPS));
    }
    // (walked in ascending order of ids: such a node never waits for a later one)
    u32 at = 0, n_wide = 0;
#pragma unroll
    for (u32 j = 0; j < DEPTH_NPT; ++j) {
        const bool longer = ar[j] > DEPTH_OPS;
        wide[j] = longer && ar[j] > DEPTH_WALK * n_long;
        if (longer) op[j][0] = wide[j] ? DEPTH_WALKED : DEPTH_NEVER;
        next[j] = longer && !wide[j] ? 0u : ar[j];
        has_list = has_list || next[j] < ar[j];
        has_34 = has_34 || (ar[j] > 2u && !wide[j]);
        const u64 m = __ballot(wide[j]);
        at += (u32)__popcll(m & lt_mask);
        n_wide += (u32)__popcll(m);
    }
#pragma unroll
    for (u32 j = 0; j < DEPTH_NPT; ++j)
        if (wide[j]) s_wide[wave][at++] = (unsigned short)(first + j);
    bool any_ext = __ballot(has_ext) != 0ull, any_list = __ballot(has_list) != 0ull;
    const bool any_34 = __ballot(has_34) != 0ull;
    u32 wide_i = 0, wide_e = 0, wide_max = 0;     // node of the wave's list being walked, operands behind it, their largest word
    u32 idle = 0, sweep = 0, seen = 0;            // seen: nodes of ended waves when last looked
    bool gave_up = false;
    // Nodes not settled yet, as lane masks of their own: asked from dep instead, the compiler knows dep to be 0 in
    // the branch, writes that 0 again, and merges `moved` and `left` node by node (64 sentences 145 us of this kernel, 133 now).
    bool open[DEPTH_NPT];
#pragma unroll
    for (u32 j = 0; j < DEPTH_NPT; ++j) open[j] = dep[j] == 0u;
    // (written out for waves without lists and with: beside the code for lists, sweeps took a sixth longer for everybody)
    auto sweeps = [&](auto with_lists) __attribute__((always_inline)) {
    while (true) {
        u32 w0[DEPTH_NPT], w1[DEPTH_NPT], w2[DEPTH_NPT], w3[DEPTH_NPT];
#pragma unroll
        for (u32 j = 0; j < DEPTH_NPT; ++j) {
            w0[j] = lds_load(&s_dep[op[j][0] < DEPTH_NEVER ? op[j][0] : DEPTH_NEVER]);
            w1[j] = lds_load(&s_dep[op[j][1] < DEPTH_NEVER ? op[j][1] : DEPTH_NEVER]);
            w2[j] = w3[j] = 1u;
        }
        if (any_34) {
#pragma unroll
            for (u32 j = 0; j < DEPTH_NPT; ++j) {
                w2[j] = lds_load(&s_dep[op[j][2] < DEPTH_NEVER ? op[j][2] : DEPTH_NEVER]);
                w3[j] = lds_load(&s_dep[op[j][3] < DEPTH_NEVER ? op[j][3] : DEPTH_NEVER]);
            }
        }
        bool moved = false;
#pragma unroll
        for (u32 j = 0; j < DEPTH_NPT; ++j) {
            if (open[j]) {
                u32 x = w0[j], y = w1[j];
#pragma unroll
                for (u32 i = 0; i < j; ++i) { x = fwd0[j][i] ? dep[i] : x; y = fwd1[j][i] ? dep[i] : y; }
                const u32 a = x < y ? x : y, b = w2[j] < w3[j] ? w2[j] : w3[j];
                if ((a < b ? a : b) != 0u) {
                    const u32 c = x > y ? x : y, d = w2[j] > w3[j] ? w2[j] : w3[j];
                    const u32 e = c > d ? c : d;
                    dep[j] = (e > ext[j] ? e : ext[j]) + 1u;
                    depth_settle(&s_dep[first + j], &g_dep[lo + first + j], dep[j]);
                    moved = true;
                    open[j] = false;
                }
            }
        }
        bool left = false;
#pragma unroll
        for (u32 j = 0; j < DEPTH_NPT; ++j) left = left || open[j];
        if (__ballot(left) == 0ull) break;
        bool progress = __ballot(moved) != 0ull;
        ++sweep;
        if (any_ext && (idle > 1u || (sweep & 15u) == 0u)) {
            // operands of lower ranges that are not known yet
            bool got = false, more = false;
#pragma unroll
            for (u32 j = 0; j < DEPTH_NPT; ++j) {
                u32 w[DEPTH_OPS];
#pragma unroll
                for (u32 q = 0; q < DEPTH_OPS; ++q) {
                    w[q] = 0;
                    if (op[j][q] & DEPTH_EXT)
                        w[q] = __hip_atomic_load(&g_dep[op[j][q] & ~DEPTH_EXT], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
#pragma unroll
                for (u32 q = 0; q < DEPTH_OPS; ++q) {
                    if (w[q]) { ext[j] = w[q] > ext[j] ? w[q] : ext[j]; op[j][q] = DEPTH_ONE; got = true; }
                    more = more || (op[j][q] & DEPTH_EXT);
                }
            }
            any_ext = __ballot(more) != 0ull;
            progress = progress || __ballot(got) != 0ull;
        }
        if (with_lists.value && any_list) {
            // (reads of a step side by side: list entries first, then the words of those in lower ranges)
            u32 id[DEPTH_NPT][DEPTH_LIST], w[DEPTH_NPT][DEPTH_LIST];
            bool got = false, more = false, new_ext = false;
#pragma unroll
            for (u32 j = 0; j < DEPTH_NPT; ++j) {
                const u32 seen[DEPTH_LIST] = {w1[j], w2[j], w3[j]};
#pragma unroll
                for (u32 q = 0; q < DEPTH_LIST; ++q) {
                    id[j][q] = ~0u;
                    if (next[j] >= ar[j] || seen[q] == 0u) continue;
                    ext[j] = seen[q] > ext[j] ? seen[q] : ext[j];
                    id[j][q] = T.in_idx[in0[j] + next[j]];
                    ++next[j];
                    got = true;
                }
            }
#pragma unroll
            for (u32 j = 0; j < DEPTH_NPT; ++j)
#pragma unroll
                for (u32 q = 0; q < DEPTH_LIST; ++q) {
                    w[j][q] = 0;
                    if (id[j][q] < lo)
                        w[j][q] = __hip_atomic_load(&g_dep[id[j][q]], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
#pragma unroll
            for (u32 j = 0; j < DEPTH_NPT; ++j) {
#pragma unroll
                for (u32 q = 0; q < DEPTH_LIST; ++q) {
                    if (id[j][q] == ~0u) continue;
                    ext[j] = w[j][q] > ext[j] ? w[j][q] : ext[j];
                    op[j][1 + q] = id[j][q] >= lo ? id[j][q] - lo : (w[j][q] ? DEPTH_ONE : (DEPTH_EXT | id[j][q]));
                    new_ext = new_ext || (op[j][1 + q] & DEPTH_EXT);
                }
                if (next[j] < ar[j]) more = true;
                else if (op[j][0] == DEPTH_NEVER) op[j][0] = DEPTH_ONE;
            }
            any_list = __ballot(more) != 0ull;
            any_ext = any_ext || __ballot(new_ext) != 0ull;
            progress = progress || __ballot(got) != 0ull;
        }
        if (!progress && wide_i < n_wide) {
            const u32 l = __builtin_amdgcn_readfirstlane((u32)s_wide[wave][wide_i]), v = lo + l;
            const u32 a = T.in_off[v], ar = T.in_off[v + 1] - a;
            u32 id[DEPTH_WIDE_READS], w[DEPTH_WIDE_READS];
#pragma unroll
            for (u32 q = 0; q < DEPTH_WIDE_READS; ++q) {
                const u32 e = wide_e + 64u * q + lane;
                id[q] = e < ar ? T.in_idx[a + e] : 0xffffffffu;
            }
#pragma unroll
            for (u32 q = 0; q < DEPTH_WIDE_READS; ++q) {
                w[q] = 1u;
                if (id[q] < lo) w[q] = __hip_atomic_load(&g_dep[id[q]], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                else if (id[q] < v) w[q] = lds_load(&s_dep[id[q] - lo]);
            }
            bool all = true;
#pragma unroll
            for (u32 q = 0; q < DEPTH_WIDE_READS; ++q) {
                all = all && __ballot(w[q] == 0u) == 0ull;
                if (all) { wide_max = w[q] > wide_max ? w[q] : wide_max; wide_e += 64u; progress = true; }
            }
            if (wide_e >= ar) {
                for (int o = 32; o > 0; o >>= 1) { const u32 t = (u32)__shfl_xor((int)wide_max, o); wide_max = t > wide_max ? t : wide_max; }
                if (lane == 0) depth_settle(&s_dep[l], &g_dep[v], wide_max + 1u);
#pragma unroll
                for (u32 j = 0; j < DEPTH_NPT; ++j) if (first + j == l) { dep[j] = wide_max + 1u; open[j] = false; }
                ++wide_i; wide_e = 0; wide_max = 0;
            }
        }
        if (progress) { idle = 0; continue; }
        if (++idle > spin_limit || lds_load(&s_quit) != 0u) { gave_up = true; break; }
        if (idle > 16u) __builtin_amdgcn_s_sleep(1);
        if ((idle & 1023u) != 0u) continue;
        // (a range that gave up leaves its error flag: ranges waiting for it need not run into their own bound)
        if (__hip_atomic_load(&T.hdr->err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & (u32)ERR_CYCLE) { gave_up = true; break; }
        // The bound is on waiting for nothing: while waves below end, a path that goes through many of them is being
        // worked off, and the wait starts anew.
        const u32 ended = __hip_atomic_load(&T.hdr->frontier_done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (ended != seen) { seen = ended; idle = 0; }
    }
    };
    if (any_list) sweeps(std::true_type{});
    else sweeps(std::false_type{});
    u32 done = 0;
#pragma unroll
    for (u32 j = 0; j < DEPTH_NPT; ++j) {
        const u32 v = lo + first + j;
        // A node that was given up on takes its own id as its step: above the step of every operand (a depth
        // is at most the id), so what the later stages build from it before the host sees the error flag
        // stays inside their tables.
        if (v < T.n) T.step[v] = dep[j] ? dep[j] - 1u : v;
        done += (u32)__popcll(__ballot(v < T.n && dep[j] != 0u));
    }
    if (lane == 0) {
        atomicAdd(&T.hdr->frontier_done, done);
        if (gave_up) { s_quit = 1u; atomicOr(&T.hdr->err, (u32)ERR_CYCLE); }
    }
}

// ---- agenda-based batching (Section 3.2, second strategy) -------------------------------------------
// The agenda holds the nodes whose operands are all resolved.  Each iteration takes every
// available node of one signature as a batch; the signature is the one with the smallest average
// depth over ALL nodes of the graph that carry it (a fixed number per signature), equal averages
// go to the cheaper operation class (leaf < component-wise / copy < per-row reduction < matrix
// product), then to the signature whose first node has the smaller id.  Because the priority of a
// signature never changes, signatures are ranked once; the agenda is then one ready list per rank
// and "select" is the lowest rank with a non-empty list.  The iteration index becomes the node's
// step, and everything downstream (grouping by (step, signature), layout, launch plan) is shared
// with depth-based batching.
constexpr u32 AG_TABLE = 4096;        // open-addressing table of signatures
constexpr u32 AG_MAX_CLASSES = 1024;  // distinct signatures an agenda plan can rank
constexpr u32 AG_NONE = 0xffffffffu;

struct AgendaTables {
    u64 *keys;        // [AG_TABLE] signature hash, 0 = empty
    u64 *sum;         // [AG_TABLE] sum of depths
    u32 *cnt;         // [AG_TABLE] nodes
    u32 *first;       // [AG_TABLE] smallest node id
    u32 *op;          // [AG_TABLE] operation of the signature
    u32 *rank_of;     // [AG_TABLE] rank of the signature in a table slot
    u32 *seg_off;     // [AG_MAX_CLASSES + 1] ready-list segment of each rank inside `seg`
    u32 *n_classes;   // [1]
    u32 *cls;         // [n] rank of each node's signature
    u32 *pending;     // [n] unresolved operands
    u32 *seg;         // [n] ready lists, one segment per rank (each node is appended once)
    // for graphs whose counters fit into LDS
    uint2 *edge_to;   // [E] per entry of the successor lists: consumer (ag_entry) | rank of its signature << AG_RANK
    uint2 *ready;     // [n] ready lists of such entries
};

__device__ inline u32 ag_cost_class(u32 op)
{
    if (op == OP_INPUT || op == OP_LOOKUP) return 0;
    if (op == OP_MATVEC) return 3;
    if (op == OP_PICK_NLS || op == OP_SQNORM) return 2;
    return 1;
}

// per node: find / create the table entry of its signature and add (depth, 1, id) to it.  Lanes
// of a wave that carry the same signature are combined first, so the table sees one update per
// distinct signature per wave.
__global__ void k_class_insert(Tables T, AgendaTables A)
{
    const u32 v = blockIdx.x * blockDim.x + threadIdx.x;
    const u32 lane = threadIdx.x & 63;
    const bool active = v < T.n;
    const u64 sig = active ? (T.sig[v] ? T.sig[v] : 1ull) : 0ull;
    const u32 depth = active ? T.step[v] : 0u;
    u64 todo = __ballot(active);
    u32 my_slot = 0;
    while (todo) {
        const u32 leader = (u32)__builtin_ctzll(todo);
        const u64 lsig = ((u64)(u32)__builtin_amdgcn_readlane((int)(u32)(sig >> 32), leader) << 32) |
                         (u32)__builtin_amdgcn_readlane((int)(u32)sig, leader);
        const bool mine = active && sig == lsig;
        const u64 match = __ballot(mine);
        u32 dsum = mine ? depth : 0u;
        for (int o = 32; o > 0; o >>= 1) dsum += __shfl_xor(dsum, o);
        u32 slot = 0;
        if (lane == leader) {
            slot = (u32)(lsig * 0x9e3779b97f4a7c15ull >> 52) & (AG_TABLE - 1);
            bool placed = false;
            for (u32 probe = 0; probe < AG_TABLE; ++probe) {
                const u64 old = atomicCAS((unsigned long long *)&A.keys[slot], 0ULL, (unsigned long long)lsig);
                if (old == 0 || old == lsig) { placed = true; break; }
                slot = (slot + 1) & (AG_TABLE - 1);
            }
            if (!placed) { atomicOr(&T.hdr->err, (u32)ERR_CLASSES); slot = 0; }
            else {
                atomicAdd(&A.cnt[slot], (u32)__popcll(match));
                atomicAdd((unsigned long long *)&A.sum[slot], (unsigned long long)dsum);
                atomicMin(&A.first[slot], v);     // the leader is the lowest matching lane: the smallest id of the wave
                A.op[slot] = T.op[v];
            }
        }
        slot = (u32)__builtin_amdgcn_readlane((int)slot, leader);
        if (mine) my_slot = slot;
        todo &= ~match;
    }
    if (active) T.ht_slot[v] = my_slot;
}

// One workgroup: collect the used table entries, rank them, lay out the ready-list segments.
__global__ __launch_bounds__(1024) void k_class_rank(Tables T, AgendaTables A)
{
    __shared__ u32 s_n;
    __shared__ u32 s_slot[AG_MAX_CLASSES];
    __shared__ u64 s_sum[AG_MAX_CLASSES];
    __shared__ u32 s_cnt[AG_MAX_CLASSES];
    __shared__ u32 s_key2[AG_MAX_CLASSES];   // cost class
    __shared__ u32 s_first[AG_MAX_CLASSES];
    __shared__ u32 s_cnt_by_rank[AG_MAX_CLASSES];
    const u32 tid = threadIdx.x;
    if (tid == 0) s_n = 0;
    __syncthreads();
    for (u32 slot = tid; slot < AG_TABLE; slot += 1024) {
        if (A.keys[slot] != 0) {
            const u32 i = atomicAdd(&s_n, 1u);
            if (i < AG_MAX_CLASSES) s_slot[i] = slot;
        }
    }
    __syncthreads();
    u32 C = s_n;
    if (C > AG_MAX_CLASSES) { if (tid == 0) atomicOr(&T.hdr->err, (u32)ERR_CLASSES); C = AG_MAX_CLASSES; }
    if (tid < C) {
        const u32 slot = s_slot[tid];
        s_sum[tid] = A.sum[slot]; s_cnt[tid] = A.cnt[slot];
        s_key2[tid] = ag_cost_class(A.op[slot]); s_first[tid] = A.first[slot];
    }
    __syncthreads();
    if (tid < C) {
        // rank = number of signatures taken before this one (first ids differ, so the order is strict)
        const u64 si = s_sum[tid]; const u32 ci = s_cnt[tid], ki = s_key2[tid], fi = s_first[tid];
        u32 rank = 0;
        for (u32 j = 0; j < C; ++j) {
            const u64 lhs = s_sum[j] * ci, rhs = si * s_cnt[j];    // avg_j < avg_i  <=>  sum_j * cnt_i < sum_i * cnt_j
            bool before = lhs < rhs;
            if (lhs == rhs) before = s_key2[j] < ki || (s_key2[j] == ki && s_first[j] < fi);
            rank += before ? 1u : 0u;
        }
        A.rank_of[s_slot[tid]] = rank;
        s_cnt_by_rank[rank] = ci;
    }
    __syncthreads();
    if (tid == 0) {
        u32 acc = 0;
        for (u32 r = 0; r < C; ++r) { A.seg_off[r] = acc; acc += s_cnt_by_rank[r]; }
        A.seg_off[C] = acc;
        A.n_classes[0] = C;
    }
}

// per node: rank of its signature, and one word holding that rank above the count of unresolved
// operands ((rank << 22) | count), so that the decrement that resolves the last operand also
// tells which ready list the node joins
constexpr u32 AG_COUNT_BITS = 22;
__global__ void k_class_of(Tables T, AgendaTables A)
{
    const u32 v = blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= T.n) return;
    const u32 rank = A.rank_of[T.ht_slot[v]];
    A.cls[v] = rank;
    // the operand count comes from the graph itself: the single-workgroup depth pass counts T.indeg down to zero
    const u32 arity = T.in_off[v + 1] - T.in_off[v];
    if (arity >> AG_COUNT_BITS) atomicOr(&T.hdr->err, (u32)ERR_CLASSES);
    A.pending[v] = (rank << AG_COUNT_BITS) | arity;
}

// One workgroup runs the agenda.  head / tail of every rank's ready list live in LDS; the lists
// themselves, the dependency counters and the successor lists are in global memory (this
// workgroup's L2).  Nodes that become available while a batch is being taken are appended behind
// the batch's end, so a node never joins the batch of one of its own operands.
constexpr int AGENDA_THREADS = 1024;
__global__ __launch_bounds__(AGENDA_THREADS) void k_agenda(Tables T, AgendaTables A, const u32 *succ_node)
{
    __shared__ u32 s_head[AG_MAX_CLASSES], s_tail[AG_MAX_CLASSES], s_off[AG_MAX_CLASSES + 1];
    __shared__ u32 s_min, s_done, s_t;
    const u32 tid = threadIdx.x;
    const u32 C = A.n_classes[0] < AG_MAX_CLASSES ? A.n_classes[0] : AG_MAX_CLASSES;
    for (u32 c = tid; c < C; c += AGENDA_THREADS) { s_head[c] = 0; s_tail[c] = 0; }
    for (u32 c = tid; c <= C; c += AGENDA_THREADS) s_off[c] = A.seg_off[c];
    if (tid == 0) { s_min = AG_NONE; s_done = 0; s_t = 0; }
    __syncthreads();
    for (u32 v = tid; v < T.n; v += AGENDA_THREADS) {
        const u32 w = A.pending[v];
        if ((w & ((1u << AG_COUNT_BITS) - 1u)) == 0) {
            const u32 c = w >> AG_COUNT_BITS;
            A.seg[s_off[c] + atomicAdd(&s_tail[c], 1u)] = v;
        }
    }
    __syncthreads();
    while (true) {
        for (u32 c = tid; c < C; c += AGENDA_THREADS)
            if (s_tail[c] > s_head[c]) atomicMin(&s_min, c);
        __syncthreads();
        const u32 c = s_min;
        if (c == AG_NONE) break;          // nothing available: all done, or a cycle
        const u32 lo = s_head[c], hi = s_tail[c], base = s_off[c], t = s_t;
        __syncthreads();
        for (u32 i = lo + tid; i < hi; i += AGENDA_THREADS) {
            const u32 v = A.seg[base + i];
            T.step[v] = t;
            const u32 e1 = T.succ_off[v + 1];
            // (four consumers side by side: one after the other each costs a read and an atomic that returns:
            // 64 parsed sentences 1 396 us of this kernel, 1 270 now)
            for (u32 e = T.succ_off[v]; e < e1; e += 4) {
                u32 sn[4], was[4];
#pragma unroll
                for (u32 q = 0; q < 4; ++q) sn[q] = e + q < e1 ? succ_node[e + q] : 0u;
#pragma unroll
                for (u32 q = 0; q < 4; ++q) was[q] = e + q < e1 ? atomicSub(&A.pending[sn[q]], 1u) : 0u;
#pragma unroll
                for (u32 q = 0; q < 4; ++q) {
                    if ((was[q] & ((1u << AG_COUNT_BITS) - 1u)) != 1u) continue;
                    const u32 cs = was[q] >> AG_COUNT_BITS;
                    A.seg[s_off[cs] + atomicAdd(&s_tail[cs], 1u)] = sn[q];
                }
            }
        }
        __syncthreads();
        if (tid == 0) { s_head[c] = hi; s_done += hi - lo; s_t = t + 1; s_min = AG_NONE; }
        __syncthreads();
    }
    if (tid == 0 && s_done != T.n) atomicOr(&T.hdr->err, (u32)ERR_CYCLE);
}

// The same agenda for up to AG_LDS_NODES nodes.  Batches of few nodes are bound by the chain of dependent reads of an iteration, so the
// counters of unresolved operands are in LDS, four bits a node (a node with more than AG_FEW operands keeps its word in memory), an
// entry of a successor list brings the consumer's rank and successor list with it, and so does an entry of a ready list: a batch reads
// its entries, then their successors, then counts, where it read entry, list bounds, successors and counters in turn.  Every wave finds
// the lowest rank for itself, which takes two barriers an iteration instead of four.  Batches of many nodes are bound by the bytes this
// one workgroup moves, so an entry is eight bytes (entries of 16 in two arrays and ready lists of 16: 4.2 ns a node in batches of
// 40 000, where the agenda over memory takes 1.6), and by sums over everything, whose counter all lanes want at once.  Kernel
// over memory / with entries of 16 bytes / now: 64 parsed sentences, 662 batches, 1 323, 989, 965 us; 512 chains of a tanh network
// 97, 103, 83; 5 000 chains 747, 1 002, 632; 40 000 rows of five operations and their sum 1 025, 1 695, 723.  (A schedule with 1 024
// threads 0 to 3 % slower up to 64 sentences and 1 to 3 % faster from 500 rows on; four consumers side by side 1 to 4 % slower, as half of
// all nodes have one.)
constexpr u32 AG_LDS_THREADS = 512, AG_SIDE = 2;
constexpr u32 AG_LDS_WORDS = 32768, AG_LDS_NODES = 8 * AG_LDS_WORDS, AG_FEW = 14;
// An entry names a node and its successor list in eight bytes: id, number of successors (AG_MANY: look it up), whether the
// node has more operands than AG_FEW, rank of its signature | first successor.
constexpr u32 AG_ID = 18, AG_MANY = 7, AG_LONG = 1u << 21, AG_RANK = 22;
static_assert(AG_LDS_NODES <= 1u << AG_ID && AG_MAX_CLASSES <= 1u << (32 - AG_RANK), "entry layout");
__device__ inline uint2 ag_entry(u32 v, u32 lo, u32 hi) { return make_uint2(v | (hi - lo < AG_MANY ? hi - lo : AG_MANY) << AG_ID, lo); }
__device__ inline u32 ag_id(uint2 e) { return e.x & ((1u << AG_ID) - 1u); }
__device__ inline u32 ag_end(const Tables &T, uint2 e)
{
    const u32 deg = (e.x >> AG_ID) & AG_MANY;
    return deg < AG_MANY ? e.y + deg : T.succ_off[ag_id(e) + 1u];
}
__global__ void k_agenda_edges(Tables T, AgendaTables A, const u32 *succ_node)
{
    const u32 q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= T.E) return;
    const u32 v = succ_node[q];
    uint2 e = ag_entry(v, T.succ_off[v], T.succ_off[v + 1]);
    e.x |= A.cls[v] << AG_RANK | (T.in_off[v + 1] - T.in_off[v] > AG_FEW ? AG_LONG : 0u);
    A.edge_to[q] = e;
}
__global__ __launch_bounds__(AG_LDS_THREADS) void k_agenda_lds(Tables T, AgendaTables A)
{
    __shared__ u32 s_head[AG_MAX_CLASSES], s_tail[AG_MAX_CLASSES], s_off[AG_MAX_CLASSES + 1], s_count[AG_LDS_WORDS];
    constexpr u32 COUNT = (1u << AG_COUNT_BITS) - 1u;
    if (T.hdr->err & ERR_CLASSES) return;      // (not every node has a rank)
    const u32 tid = threadIdx.x, lane = tid & 63u;
    const u32 C = A.n_classes[0] < AG_MAX_CLASSES ? A.n_classes[0] : AG_MAX_CLASSES;
    for (u32 c = tid; c < C; c += AG_LDS_THREADS) { s_head[c] = 0; s_tail[c] = 0; }
    for (u32 c = tid; c <= C; c += AG_LDS_THREADS) s_off[c] = A.seg_off[c];
    __syncthreads();
    for (u32 w = tid; 8u * w < T.n; w += AG_LDS_THREADS) {
        u32 p[8], bound[9], word = 0;
#pragma unroll
        for (u32 k = 0; k < 8; ++k) p[k] = 8u * w + k < T.n ? A.pending[8u * w + k] : 1u;
#pragma unroll
        for (u32 k = 0; k < 9; ++k) bound[k] = T.succ_off[8u * w + k < T.n ? 8u * w + k : T.n];
#pragma unroll
        for (u32 k = 0; k < 8; ++k) {
            const u32 count = p[k] & COUNT, c = p[k] >> AG_COUNT_BITS;
            word |= (count <= AG_FEW ? count : AG_FEW + 1u) << (4u * k);
            if (count == 0u) A.ready[s_off[c] + atomicAdd(&s_tail[c], 1u)] = ag_entry(8u * w + k, bound[k], bound[k + 1]);
        }
        s_count[w] = word;
    }
    // The lists of successors were written all over the chip: brought into this XCD's L2 first, side by side.
    u32 sink = 0;
    for (u32 x0 = tid; x0 < T.E; x0 += 8u * AG_LDS_THREADS) {
        u32 a[8];
#pragma unroll
        for (u32 k = 0; k < 8; ++k) a[k] = A.edge_to[x0 + k * AG_LDS_THREADS < T.E ? x0 + k * AG_LDS_THREADS : x0].x;
#pragma unroll
        for (u32 k = 0; k < 8; ++k) sink |= a[k];
    }
    asm volatile("" :: "v"(sink));
    // One operand less of a node whose counter is in memory, for each lane that gets here; how many there were.  Lanes of one node, a sum of
    // all losses in the first place, are counted by one of them.
    auto count_long = [&](u32 v) __attribute__((always_inline)) {
        u32 was = 0;
        for (u64 todo = __ballot(true); todo;) {
            const u32 leader = (u32)__builtin_ctzll(todo), vl = (u32)__builtin_amdgcn_readlane((int)v, (int)leader);
            const u64 same = __ballot(v == vl) & todo;
            u32 had = 0;
            if (lane == leader) had = atomicSub(&A.pending[vl], (u32)__popcll(same)) & COUNT;
            had = (u32)__builtin_amdgcn_readlane((int)had, (int)leader);
            if (v == vl) was = had - (u32)__popcll(same & ((1ull << lane) - 1ull));
            todo &= ~same;
        }
        return was;
    };
    u32 done = 0, prev = AG_NONE, prev_hi = 0;
    for (u32 t = 0;; ++t) {
        __syncthreads();
        u32 c = AG_NONE, lo = 0, hi = 0;
        for (u32 c0 = 0; c0 < C && c == AG_NONE; c0 += 64u) {
            const u32 k = c0 + lane;
            const u32 head = k == prev ? prev_hi : (k < C ? s_head[k] : 0u), tail = k < C ? s_tail[k] : 0u;
            const u64 some = __ballot(tail > head);
            if (!some) continue;
            const int l = __builtin_ctzll(some);
            c = c0 + (u32)l; lo = (u32)__builtin_amdgcn_readlane((int)head, l); hi = (u32)__builtin_amdgcn_readlane((int)tail, l);
        }
        __syncthreads();                  // (every wave has looked: heads and tails may move)
        if (c == AG_NONE) break;          // nothing available: all done, or a cycle
        if (tid == 0 && prev != AG_NONE) s_head[prev] = prev_hi;
        const u32 base = s_off[c];
        for (u32 i = lo + tid; i < hi; i += AG_LDS_THREADS) {
            const uint2 e = A.ready[base + i];
            const u32 end = ag_end(T, e);
            for (u32 q = e.y; q < end; q += AG_SIDE) {
                uint2 to[AG_SIDE];
                u32 left[AG_SIDE];
#pragma unroll
                for (u32 k = 0; k < AG_SIDE; ++k) to[k] = A.edge_to[q + k < end ? q + k : q];
#pragma unroll
                for (u32 k = 0; k < AG_SIDE; ++k) {
                    left[k] = 0u;
                    if (q + k >= end) continue;
                    const u32 v = ag_id(to[k]), at = 4u * (v & 7u);
                    left[k] = to[k].x & AG_LONG ? count_long(v) : (atomicSub(&s_count[v >> 3], 1u << at) >> at) & 15u;
                }
#pragma unroll
                for (u32 k = 0; k < AG_SIDE; ++k) {
                    if (left[k] != 1u) continue;
                    const u32 cs = to[k].x >> AG_RANK;
                    A.ready[s_off[cs] + atomicAdd(&s_tail[cs], 1u)] = to[k];
                }
            }
            T.step[ag_id(e)] = t;
        }
        prev = c; prev_hi = hi;
        done += hi - lo;
    }
    if (tid == 0 && done != T.n) atomicOr(&T.hdr->err, (u32)ERR_CYCLE);
}

// ---- stage 3: batch representative = smallest node id with the same (depth, signature) ------
__device__ inline u64 batch_key(u64 sig, u32 step)
{
    u64 k = comb(sig, step);
    return k ? k : 1;
}

// Thousands of nodes share a key (all leaves of one kind, in the first place), and reads and atomics of one word from
// all over the chip pass one after the other, about 10 ns each.  So the workgroup's nodes first meet in LDS, and one node
// per distinct key goes to the table, with the smallest id; there it looks before it writes (keys never change once
// set, values only fall, so whatever a look returns is safe to act on).
constexpr u32 REP_THREADS = 1024, REP_SLOTS = 2048;
__global__ __launch_bounds__(REP_THREADS) void k_rep_insert(Tables T)
{
    __shared__ u64 s_key[REP_SLOTS];
    __shared__ u32 s_min[REP_SLOTS], s_at[REP_SLOTS];
    for (u32 i = threadIdx.x; i < REP_SLOTS; i += REP_THREADS) { s_key[i] = 0; s_min[i] = 0xffffffffu; }
    __syncthreads();
    const u32 v = blockIdx.x * REP_THREADS + threadIdx.x;
    const bool live = v < T.n;
    u64 k = 0;
    u32 at = 0;
    bool first = false;      // this node's key is new to the workgroup
    if (live) {
        k = batch_key(T.sig[v], T.step[v]);
        for (at = (u32)(k >> 32) & (REP_SLOTS - 1);; at = (at + 1) & (REP_SLOTS - 1)) {   // (twice as many slots as nodes)
            const u64 cur = atomicCAS((unsigned long long *)&s_key[at], 0ULL, (unsigned long long)k);
            first = cur == 0;
            if (first || cur == k) break;
        }
        atomicMin(&s_min[at], v);
    }
    __syncthreads();
    if (first) {
        const u32 low = s_min[at];
        u32 slot = (u32)k & T.ht_mask, probe = 0;
        for (; probe <= T.ht_mask; ++probe, slot = (slot + 1) & T.ht_mask) {
            u64 cur = __hip_atomic_load(&T.ht_keys[slot], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (cur == 0) {
                cur = atomicCAS((unsigned long long *)&T.ht_keys[slot], 0ULL, (unsigned long long)k);
                if (cur == 0) cur = k;
            }
            if (cur == k) {
                if (__hip_atomic_load(&T.ht_vals[slot], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) > low) atomicMin(&T.ht_vals[slot], low);
                break;
            }
        }
        if (probe > T.ht_mask) { atomicOr(&T.hdr->err, (u32)ERR_TABLE_FULL); slot = 0; }
        s_at[at] = slot;
    }
    __syncthreads();
    if (live) T.ht_slot[v] = s_at[at];
}

// rep_src: 0 = the node itself (unbatched), 1 = the representative found by k_rep_insert,
// 2 = none (manual batching: one batch per step, the stable sort keeps ids ascending)
__device__ inline void sort_keys_at(const Tables &T, u64 *keys, u32 *vals, int rep_src, u32 v)
{
    if (v >= T.n) return;
    const u32 rep = rep_src == 1 ? T.ht_vals[T.ht_slot[v]] : (rep_src == 2 ? 0u : v);
    keys[v] = ((u64)T.step[v] << 32) | rep;
    vals[v] = v;
}
__global__ void k_sort_keys(Tables T, u64 *keys, u32 *vals, int rep_src)
{
    sort_keys_at(T, keys, vals, rep_src, blockIdx.x * blockDim.x + threadIdx.x);
}

// ---- stage 4: batches from the sorted order -----------------------------------------------------
__device__ inline void heads_at(const Tables &T, const u64 *skey, const u32 *sval, u32 *head_flag, Tri *counts, u32 p)
{
    if (p >= T.n) return;
    const u32 v = sval[p];
    T.order[p] = v;
    T.pos_of[v] = p;
    T.s_aux0[p] = (u32)T.aux0[v];
    Tri c;
    c.a = (p == 0 || skey[p] != skey[p - 1]) ? 1u : 0u;
    const u32 o = T.op[v];
    c.b = (o == OP_MATVEC) ? XP_MAX : T.in_off[v + 1] - T.in_off[v];   // a product's operand may be listed in up to XP_MAX pieces
    c.c = (o == OP_MATVEC) ? (1u + (T.bias[v] >= 0 ? 1u : 0u)) : (o == OP_LOOKUP ? 1u : 0u);
    c.d = 0;
    head_flag[p] = c.a;
    counts[p] = c;
}
__global__ void k_heads(Tables T, const u64 *skey, const u32 *sval, u32 *head_flag, Tri *counts)
{
    heads_at(T, skey, sval, head_flag, counts, blockIdx.x * blockDim.x + threadIdx.x);
}

__device__ inline void batch_off_at(const Tables &T, const u32 *head_flag, const Tri *before, u32 *item_base, int manual, u32 p)
{
    if (p >= T.n) return;
    const Tri ex = before[p];          // batch heads, operand references and parameter uses before position p
    const u32 b = ex.a + head_flag[p] - 1;
    T.s_in_off[p] = ex.b;
    item_base[p] = ex.c;
    T.batch_of_pos[p] = b;
    if (manual) T.step[T.order[p]] = b;   // labels need not be dense: a batch's step is its rank
    if (head_flag[p]) T.batch_off[b] = p;
    if (p == T.n - 1) {
        T.batch_off[b + 1] = T.n;
        T.hdr->n_batches = b + 1;
    }
}
__global__ void k_batch_off(Tables T, const u32 *head_flag, const Tri *before, u32 *item_base, int manual)
{
    batch_off_at(T, head_flag, before, item_base, manual, blockIdx.x * blockDim.x + threadIdx.x);
}

// Takes bits off a batch's flags.  Flags only fall, so whatever a look returns is safe to act on, and all
// members of a batch mostly take off the same bits: only the first pay for an atomic on the one word.
__device__ inline void flags_off(BatchRec &r, u32 bits)
{
    if (__hip_atomic_load(&r.vec4, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & bits) atomicAnd(&r.vec4, ~bits);
}

__host__ __device__ inline u32 cdiv(u64 a, u32 b) { return (u32)((a + b - 1) / b); }

// one thread per batch: record + sizes for the layout scan (entries b >= n_batches are zero)
__device__ inline void batch_layout_at(const Tables &T, Lay *lay_in, int virt, u32 b)
{
    if (b >= T.n) return;
    Lay L; L.val = 0; L.dx = 0; L.ind = L.p0 = L.p1 = L.p2 = 0;
    if (b < T.hdr->n_batches) {
        const u32 p0 = T.batch_off[b], B = T.batch_off[b + 1] - p0;
        const u32 h = T.order[p0];
        BatchRec r;
        r.pos0 = p0; r.B = B; r.op = T.op[h]; r.d = T.out_dim[h];
        r.arity = T.in_off[h + 1] - T.in_off[h];
        r.param = T.param[h]; r.bias = T.bias[h];
        r.aux0 = T.aux0[h]; r.aux1 = T.aux1[h];
        if (r.op == OP_MATVEC) { r.aux0 = -1; r.aux1 = 0; }
        r.step = T.step[h];
        r.k = r.arity ? T.out_dim[T.in_idx[T.in_off[h]]] : 0;
        r.val_off = r.dx_off = r.indim = 0;
        r.opnd = T.s_in_off[p0];
        r.vec4 = TF_VEC4 | TF_ALIGNED | TF_G_ALIAS;   // cleared below by whatever a member violates
        if (r.op == OP_MATVEC && B >= WIDE_MIN_ROWS && r.d >= (u32)GTW) r.vec4 |= TF_WIDE;
        if (r.op == OP_SLICE) r.vec4 |= TF_VIEW;
        if (r.op == OP_CONCAT && virt) r.vec4 |= TF_VIRT;   // taken back by k_node_offsets / k_opnd
        if (r.op == OP_MATVEC && virt) r.vec4 |= TF_XP;     // taken back by k_xp_check
        T.batches[b] = r;
        const u64 vs = (u64)B * r.d;
        L.val = (vs + VAL_ALIGN - 1) / VAL_ALIGN * VAL_ALIGN;
        if (r.op == OP_MATVEC) {
            const u64 xs = (u64)B * r.k;
            L.dx = (xs + VAL_ALIGN - 1) / VAL_ALIGN * VAL_ALIGN;
        }
        L.ind = r.op == OP_MATVEC ? XP_MAX : r.arity;
    }
    lay_in[b] = L;
}
__global__ void k_batch_layout(Tables T, Lay *lay_in, int virt)
{
    batch_layout_at(T, lay_in, virt, blockIdx.x * blockDim.x + threadIdx.x);
}

__device__ inline void batch_finish_at(const Tables &T, const Lay *lay_ex, const Lay *total, u32 b)
{
    const u32 nb = T.hdr->n_batches;
    if (b >= nb) return;
    const Lay L = lay_ex[b];
    const Lay tot = *total;
    BatchRec &r = T.batches[b];
    r.val_off = (u32)L.val;
    r.dx_off = (u32)(tot.val + L.dx);
    r.indim = L.ind;
    if (b == nb - 1) {
        T.hdr->n_steps = r.step + 1;
        T.hdr->val_floats = tot.val;
        T.hdr->grad_floats = tot.val + tot.dx;
        if (tot.val + tot.dx >= 0xffffffffULL) atomicOr(&T.hdr->err, (u32)ERR_OVERFLOW);
    }
}
__global__ void k_batch_finish(Tables T, const Lay *lay_ex, const Lay *total)
{
    batch_finish_at(T, lay_ex, total, blockIdx.x * blockDim.x + threadIdx.x);
}

__device__ inline void node_offsets_at(const Tables &T, u32 p)
{
    if (p >= T.n) return;
    BatchRec &r = T.batches[T.batch_of_pos[p]];
    const u32 row = p - r.pos0;
    const u32 v = T.order[p];
    T.val_off[v] = T.nat_off[v] = r.val_off + row * r.d;
    T.dx_off[v] = (r.op == OP_MATVEC) ? r.dx_off + row * r.k : 0u;
    T.slot_dx[p] = 0;
    // a CONCAT batch can stay uncopied only with at most XP_MAX pieces whose dimensions are multiples of 4
    if (r.op == OP_CONCAT && (r.vec4 & TF_VIRT)) {
        const u32 ar = T.in_off[v + 1] - T.in_off[v];
        bool ok = ar <= XP_MAX;
        for (u32 j = 0; ok && j < ar; ++j) ok = (T.out_dim[T.in_idx[T.in_off[v] + j]] & 3u) == 0;
        if (!ok) flags_off(r, TF_VIRT);
    }
    // a product whose operand is a CONCAT node: the lowest such CONCAT batch gives the piece structure of the batch
    if (r.op == OP_MATVEC && (r.vec4 & TF_XP)) {
        const u32 x = T.in_idx[T.in_off[v]];
        if (T.op[x] == OP_CONCAT) atomicMin((u32 *)&r.aux0, T.batch_of_pos[T.pos_of[x]]);
    }
}
__global__ void k_node_offsets(Tables T)
{
    node_offsets_at(T, blockIdx.x * blockDim.x + threadIdx.x);
}

// SLICE nodes are views: their value is the range [lo, hi) of the operand's row where it lies
// (through any number of slices of slices), so nothing is copied forward and every reader of the
// node is pointed there.  Their gradient rows stay in their own batch's block (nat_off).
__device__ inline void view_offsets_at(const Tables &T, u32 v)
{
    if (v >= T.n || T.op[v] != OP_SLICE) return;
    u32 x = v, acc = 0;
    while (T.op[x] == OP_SLICE) { acc += (u32)T.aux0[x]; x = T.in_idx[T.in_off[x]]; }   // ids fall: ends at a node that owns its row
    T.val_off[v] = T.nat_off[x] + acc;
}
__global__ void k_view_offsets(Tables T)
{
    view_offsets_at(T, blockIdx.x * blockDim.x + threadIdx.x);
}

// CONCAT batches that only matrix products read are not copied (Section 3.3: operands that already lie in
// memory are used where they are): the product reads each row's pieces from their producers' rows.  This needs
// one piece structure per product batch.  Per product row whose operand is a CONCAT node: its pieces must
// have the dimensions of the batch's reference CONCAT batch (aux0), which must itself qualify; rows with any
// other operand are read whole, which every piece structure allows.  (The reference batch and the CONCAT batches
// that qualify at all were settled by k_node_offsets.)
__device__ inline void xp_check(const Tables &T, u32 p, BatchRec &r)
{
    if (r.op != OP_MATVEC || !(r.vec4 & TF_XP) || r.aux0 < 0) return;
    const u32 x = T.in_idx[T.in_off[T.order[p]]];
    if (T.op[x] != OP_CONCAT) return;
    const BatchRec &rr = T.batches[r.aux0];
    const u32 hr = T.order[rr.pos0];
    const u32 P = rr.arity;
    bool ok = (rr.vec4 & TF_VIRT) && T.in_off[x + 1] - T.in_off[x] == P;
    for (u32 j = 0; ok && j < P; ++j) ok = T.out_dim[T.in_idx[T.in_off[x] + j]] == T.out_dim[T.in_idx[T.in_off[hr] + j]];
    if (!ok) { flags_off(r, TF_XP); return; }
    if (T.batch_of_pos[T.pos_of[x]] == (u32)r.aux0) {   // (every such row writes the same values)
        r.aux1 = (i32)P;
        for (u32 j = 0; j < P; ++j) T.b_indim[r.indim + j] = T.out_dim[T.in_idx[T.in_off[x] + j]];
    }
}

// Per node: the check that every member of a batch really has the signature tuple of the batch
// head (a 64-bit hash collision would otherwise merge incompatible nodes), and whether the
// float4 component-wise path is allowed.
__device__ inline void member_check_at(const Tables &T, u32 p)
{
    if (p >= T.n) return;
    BatchRec &r = T.batches[T.batch_of_pos[p]];
    const u32 v = T.order[p];
    const u32 ar = T.in_off[v + 1] - T.in_off[v];
    bool same = T.op[v] == r.op && T.out_dim[v] == r.d && ar == r.arity && T.param[v] == r.param &&
                T.bias[v] == r.bias && T.step[v] == r.step;
    if (r.op == OP_SLICE) same = same && T.aux0[v] == r.aux0 && T.aux1[v] == r.aux1;
    bool vec = (r.d & 3u) == 0;
    if (r.op == OP_SLICE) vec = vec && ((u32)r.aux0 & 3u) == 0;
    if (r.op == OP_INPUT) vec = vec && ((u32)T.aux0[v] & 3u) == 0;
    if (!same) atomicOr(&T.hdr->err, (u32)ERR_COLLISION);
    if (!vec) flags_off(r, TF_VEC4);
    // A one-element MATVEC node may become the backward root (chosen after scheduling): its gradient is
    // the seed, not its consumer's row, so such batches never alias.
    if (r.op == OP_MATVEC && (T.outdeg[v] != 1 || r.d == 1)) flags_off(r, TF_G_ALIAS);
    xp_check(T, p, r);
}
__global__ void k_member_check(Tables T)
{
    member_check_at(T, blockIdx.x * blockDim.x + threadIdx.x);
}

__device__ inline bool batch_xp(const BatchRec &r) { return r.op == OP_MATVEC && (r.vec4 & TF_XP) && r.aux1 > 0; }

// Per edge: operand row offsets per batch (slot-major), operand dimensions of the batch, the
// operand part of the membership check, and the alignment flags.
__device__ inline void opnd_at(const Tables &T, u32 e)
{
    if (e >= T.E) return;
    const u32 v = T.edge_cons[e];
    const u32 j = e - T.in_off[v];
    const u32 p = T.pos_of[v];
    BatchRec &r = T.batches[T.batch_of_pos[p]];
    const u32 row = p - r.pos0;
    const u32 h = T.order[r.pos0];
    const u32 u = T.in_idx[e];
    const u32 du = T.out_dim[u];
    if (j >= r.arity || du != T.out_dim[T.in_idx[T.in_off[h] + j]]) {
        atomicOr(&T.hdr->err, (u32)ERR_COLLISION);
        return;
    }
    const bool xp = batch_xp(r);
    // an edge into a CONCAT node: any reader that is not a product reading in pieces needs the row in place
    if (T.op[u] == OP_CONCAT && !xp) {
        BatchRec &ru = T.batches[T.batch_of_pos[T.pos_of[u]]];
        if (ru.vec4 & TF_VIRT) flags_off(ru, TF_VIRT);
    }
    if (xp) {
        // the operand in pieces: the rows of a CONCAT node's operands (where the producers left them, whether or
        // not the CONCAT batch ends up copied for another reader's sake), or the whole row once per piece
        const u32 P = (u32)r.aux1;
        const bool pieces = T.op[u] == OP_CONCAT;
        u32 start = 0;
        for (u32 q = 0; q < P; ++q) {
            u32 off = T.val_off[u];
            if (pieces) { const u32 w = T.in_idx[T.in_off[u] + q]; off = T.val_off[w] - start; start += T.out_dim[w]; }
            T.opnd_off[r.opnd + q * r.B + row] = off;
            if (off & 3u) flags_off(r, (TF_VEC4 | TF_ALIGNED));
        }
        return;
    }
    const u32 off = T.val_off[u];
    T.opnd_off[r.opnd + j * r.B + row] = off;
    if (row == 0) T.b_indim[r.indim + j] = du;
    if (off & 3u) flags_off(r, (TF_VEC4 | TF_ALIGNED));
    else if (r.op == OP_CONCAT && (du & 3u)) flags_off(r, TF_VEC4);
}
__global__ void k_opnd(Tables T)
{
    opnd_at(T, blockIdx.x * blockDim.x + threadIdx.x);
}

// ---- launch planning ---------------------------------------------------------------------------------
// The schedule (which nodes form a batch, and the order of batches) is fixed above.  What follows
// only decides which batches share a kernel launch.  Component-wise batches whose operands are
// row-aligned with their producer (row r reads row r) can run in the producer's launch: a
// workgroup that owns a block of rows walks such a chain with workgroup barriers, no grid-wide
// synchronisation is needed.  Every other dependency costs one launch boundary.

__device__ inline bool op_chainable(u32 op, u32 arity)
{
    switch (op) {
    case OP_ADD: return arity < (u32)WIDE_ADD_ARITY;
    case OP_CMULT: case OP_TANH: case OP_SIGMOID: case OP_CONCAT: case OP_SLICE: return true;
    default: return false;
    }
}
__device__ inline bool op_chain_source(u32 op, u32 arity)
{
    return op == OP_INPUT || op == OP_LOOKUP || op_chainable(op, arity);
}

constexpr u32 FUSE_MAX_MULT = 4;
__device__ inline u32 gcd_u32(u32 a, u32 b) { while (b) { const u32 t = a % b; a = b; b = t; } return a; }

// Batch-level dependencies.  Per graph edge: consumer batch, producer batch, and whether a launch
// boundary is needed.  The edge can be fused (weight 0) when both batches are component-wise (the
// producer may also be a leaf) and, with G = gcd of the two row counts, the consumer row and the
// producer row lie in the same group (consumer group = row / (B_cons / G), producer group =
// row / (B_prod / G)).  A group may hold at most FUSE_MAX_MULT rows of a batch: fusing must keep
// that many independent groups, or a fused launch would serialise what a launch per level runs
// wide.  Two batches end up in one slot only if every edge between them is fusable (any other
// edge pushes the consumer to a later slot), so the test is per edge.  Distinct (consumer,
// producer, weight) triples are collected once each through a hash set.
constexpr u32 SLOT_MAX_NB = 4096;     // batches a fused plan can hold (12-bit ids)
constexpr u32 BSET_SIZE = 1u << 16;   // open-addressing set of packed triples
constexpr u32 BLIST_MAX = 20480;      // distinct triples the slot kernel keeps in LDS (80 KB)
constexpr int SLOT_BITS = 13;         // bits of a slot or a label when the plan is fused

// the dependency of the row at schedule position p (batch b) on operand u, packed; never 0
__device__ inline u32 bedge_key(const Tables &T, u32 p, u32 b, const BatchRec &r, u32 u)
{
    const u32 pu = T.pos_of[u];
    const u32 by = T.batch_of_pos[pu];
    const BatchRec &y = T.batches[by];
    bool ok = op_chainable(r.op, r.arity) && op_chain_source(y.op, y.arity);
    if (ok) {
        const u32 G = gcd_u32(r.B, y.B);
        const u32 mc = r.B / G, mp = y.B / G;
        ok = mc <= FUSE_MAX_MULT && mp <= FUSE_MAX_MULT && (p - r.pos0) / mc == (pu - y.pos0) / mp;
    }
    return ((b << 13) | (by << 1) | (ok ? 0u : 1u)) + 1u;
}

// puts a triple into the set, and into the list if it is new there
__device__ inline void bedge_insert(const Tables &T, u32 *bset, u32 *blist, u32 key)
{
    u32 h = (key * 2654435761u) & (BSET_SIZE - 1);
    for (u32 probe = 0; probe < BSET_SIZE; ++probe) {
        u32 old = __hip_atomic_load(&bset[h], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (old == 0u) old = atomicCAS(&bset[h], 0u, key);
        if (old == key) return;
        if (old == 0u) {
            const u32 i = atomicAdd(&T.hdr->n_bedges, 1u);
            if (i < BLIST_MAX) blist[i] = key;
            return;
        }
        h = (h + 1) & (BSET_SIZE - 1);
    }
    atomicAdd(&T.hdr->n_bedges, BLIST_MAX);   // table full: forces the unfused plan
}

// A thread takes a row in schedule order with its operands: the rows of a batch lie side by side and mostly carry the
// same triples, so a small set in LDS lets one of a workgroup's rows through to the set in memory (a thread
// per edge in id order brought every edge there).  The operands of rows with more than BEDGE_OPS of them are shared out
// over the workgroup (WideRows): rows of one batch have the same number of operands and lie side by side here, so taken
// one after the other they were as many rounds of one workgroup as it has threads (4 096 sums of nine operands 175 us, 17
// now; 2 000 of 64 operands 181 and 66).
constexpr u32 BEDGE_SLOTS = 1024, BEDGE_PROBES = 8, BEDGE_OPS = 8;
__device__ inline void bedge_add(const Tables &T, u32 *s_set, u32 *bset, u32 *blist, u32 key)
{
    u32 h = (key * 2654435761u) >> 22;
    static_assert(BEDGE_SLOTS == 1u << (32 - 22), "the hash gives as many bits as the set has slots");
    for (u32 probe = 0; probe < BEDGE_PROBES; ++probe) {
        u32 old = lds_load(&s_set[h]);
        if (old == 0u) old = atomicCAS(&s_set[h], 0u, key);
        if (old == key) return;
        if (old == 0u) break;
        h = (h + 1) & (BEDGE_SLOTS - 1);
    }
    bedge_insert(T, bset, blist, key);   // new here, or the neighbourhood of its place is full
}
__global__ __launch_bounds__(TPB) void k_bedges(Tables T, u32 *bset, u32 *blist)
{
    __shared__ u32 s_set[BEDGE_SLOTS];
    __shared__ WideRows<TPB> S;
    if (T.hdr->n_batches > SLOT_MAX_NB) return;
    for (u32 i = threadIdx.x; i < BEDGE_SLOTS; i += TPB) s_set[i] = 0;
    if (threadIdx.x == 0) S.n = 0;
    __syncthreads();
    const u32 p = blockIdx.x * TPB + threadIdx.x;
    if (p < T.n) {
        const u32 v = T.order[p], b = T.batch_of_pos[p];
        const u32 lo = T.in_off[v], hi = T.in_off[v + 1];
        if (hi - lo <= BEDGE_OPS) {
            const BatchRec &r = T.batches[b];
            for (u32 e = lo; e < hi; e += 2) {       // two operands at a time: their reads run side by side
                const u32 k0 = bedge_key(T, p, b, r, T.in_idx[e]);
                const u32 k1 = bedge_key(T, p, b, r, T.in_idx[e + 1 < hi ? e + 1 : e]);
                bedge_add(T, s_set, bset, blist, k0);
                if (k1 != k0) bedge_add(T, s_set, bset, blist, k1);
            }
        } else {
            wide_add(S, p, lo, hi - lo);
        }
    }
    __syncthreads();
    const u32 rows = (u32)(S.n >> 32), edges = (u32)S.n;
    for (u32 x0 = threadIdx.x; x0 < edges; x0 += WIDE_STEP * TPB) {
        u32 key[WIDE_STEP];
#pragma unroll
        for (u32 k = 0; k < WIDE_STEP; ++k) {
            const u32 x = x0 + k * TPB < edges ? x0 + k * TPB : x0;
            const u32 i = wide_row(S, rows, x), q = S.row[i], b = T.batch_of_pos[q];
            key[k] = bedge_key(T, q, b, T.batches[b], T.in_idx[S.lo[i] + (x - S.at[i])]);
        }
#pragma unroll
        for (u32 k = 0; k < WIDE_STEP; ++k)
            if (k == 0 || key[k] != key[k - 1]) bedge_add(T, s_set, bset, blist, key[k]);
    }
}

// ---- gated cells --------------------------------------------------------------------------------------
// Nearly every run of an LSTM or tree-LSTM network is one computation: gates from slices of a sum, products, their sum, tanh, a
// product.  Worked tile by tile from descriptors a level of it costs 1 400 to 2 600 cycles of one wave whatever it
// computes (a wave issues an instruction every four or five cycles, a taken branch costs thirty: addresses, flags and
// branches of a tile are 150 to 250 instructions).  So the cells of a plan are looked for in the graph, and
// a chain that consists of them is worked a thread per column, in registers, from one record a row, forward and backward
// (launches in kernel traces: 64 trees, forward 8.2 -> 4.2 us, backward 12.4 -> 5.5; 64 sentences, backward 9.8 -> 4.8).
// Does a cell end in product h (of a tanh and a sigmoid)?  Everything that the record relies on is checked here, edge by edge: every
// node of a cell but its output and c is read inside the cell only.  That the nodes lie in one chain is checked by cell_in_chain, and
// that they are all of the chain by k_chain_recs, which counts.  What bounds it is the chain of reads from the output back to the
// operands of S, so each step asks for the records of all nodes at once (first two operands, operation, arity), whether they turn
// out to be what they should or not, and it runs beside the one workgroup that works out the slots (64 trees: 56 us as a launch
// of its own, read one by one, k_slots 18; both together 19 now).
__device__ inline void find_cell(const Tables &T, u32 h)
{
    constexpr u32 NT = CELL_FORGET + 1, NG = NT + 2;      // terms of c; gates: one a term, o, the candidate
    const u32 p = T.pos_of[h];
    const uint4 rh = T.nrec[h];            // first two operands, operation, arity
    u32 tc = rh.x, o = rh.y;
    uint4 rtc = T.nrec[tc], ro = T.nrec[o];
    if (rtc.z == OP_SIGMOID) { const u32 x = tc; tc = o; o = x; const uint4 y = rtc; rtc = ro; ro = y; }
    if (rtc.z != OP_TANH || ro.z != OP_SIGMOID) return;
    const u32 c = rtc.x;
    const uint4 rc = T.nrec[c];
    const u32 nt = rc.z == OP_ADD ? rc.w : 1u;
    if ((rc.z != OP_ADD && rc.z != OP_CMULT) || nt > NT || (rc.z == OP_ADD && nt < 2u)) return;
    const u32 b = T.batch_of_pos[p], H = T.out_dim[h];
    const u32 h0 = T.succ_off[h], nh = T.succ_off[h + 1] - h0, r0 = T.succ_off[c], nc = T.succ_off[c + 1] - r0;
    bool ok = H > 1u && T.outdeg[tc] == 1u && nh <= CELL_H_EDGES && nc >= 1u && nc <= 2u;
    // the terms of c, the gate of each and what it is multiplied by (absent terms: the first once more)
    u32 t[NT], gate[NT], with[NT], ic_at = NT;
    uint4 rt[NT], rgate[NT], rwith[NT];
    static_assert(NT == 3, "terms of c");
    t[0] = rc.z == OP_ADD ? rc.x : c;
    t[1] = nt > 1u ? rc.y : t[0];
    t[2] = nt > 2u ? T.in_idx[T.in_off[c] + 2u] : t[0];
#pragma unroll
    for (u32 q = 0; q < NT; ++q) rt[q] = T.nrec[t[q]];
#pragma unroll
    for (u32 q = 0; q < NT; ++q) {
        gate[q] = rt[q].x; with[q] = rt[q].y;
        rgate[q] = T.nrec[gate[q]]; rwith[q] = T.nrec[with[q]];
    }
    u32 cand = h;
    uint4 rcand = rh;
#pragma unroll
    for (u32 q = NT; q-- > 0;) {
        if (rgate[q].z != OP_SIGMOID) {
            const u32 x = gate[q]; gate[q] = with[q]; with[q] = x;
            const uint4 y = rgate[q]; rgate[q] = rwith[q]; rwith[q] = y;
        }
        const bool fine = rt[q].z == OP_CMULT && (t[q] == c || T.outdeg[t[q]] == 1u);
        ok = ok && (q >= nt || fine);
        if (q < nt && rwith[q].z == OP_TANH) { ic_at = q; cand = with[q]; rcand = rwith[q]; }
    }
    ok = ok && ic_at < NT;
    // gates: one a term, o, the candidate; each the activation of a slice of S, and read nowhere else
    u32 node[NG], sl[NG], at[NG], S = 0;
    uint4 rsl[NG];
#pragma unroll
    for (u32 k = 0; k < NG; ++k) {
        node[k] = k < NT ? gate[k < nt ? k : 0u] : (k == NT ? o : cand);
        sl[k] = k < NT ? rgate[k < nt ? k : 0u].x : (k == NT ? ro.x : rcand.x);
    }
#pragma unroll
    for (u32 k = 0; k < NG; ++k) rsl[k] = T.nrec[sl[k]];
    u32 seen = 0;
#pragma unroll
    for (u32 k = 0; k < NG; ++k) {
        const u32 op = k < NT ? rgate[k < nt ? k : 0u].z : (k == NT ? ro.z : rcand.z);
        if (k == 0) S = rsl[k].x;
        const bool fine = op == (k == NT + 1u ? OP_TANH : OP_SIGMOID) && T.outdeg[node[k]] == 1u &&
                          T.out_dim[node[k]] == H && rsl[k].z == OP_SLICE && T.outdeg[sl[k]] == 1u && rsl[k].x == S;
        at[k] = (u32)T.aux0[sl[k]];
        if (k >= nt && k < NT) continue;       // (no such term)
        ok = ok && fine && at[k] % H == 0u;
        seen |= 1u << (at[k] / H & 31u);
    }
    const u32 gates = nt + 2u;
    ok = ok && seen == (1u << gates) - 1u && T.out_dim[S] == gates * H;
    // S: a sum of two rows that nobody else reads belongs to the cell, any other row does not
    const uint4 rS = T.nrec[S];
    const bool sums = rS.z == OP_ADD && rS.w == 2u && T.outdeg[S] == gates;
    const u32 a = sums ? rS.x : h, a2 = sums ? rS.y : h;
    if (!ok) return;
    // what reads h and c (c is read by its tanh first)
    CellRec R;
    auto edge = [&](u32 q, CellEdge &to) {
        const EdgeRec e = T.edges[q];
        to = CellEdge{e.kind, e.goff, e.voff};
        ok = ok && (e.kind == EK_PLAIN || (e.kind >= EK_MUL && e.kind <= EK_DSIGM));
    };
#pragma unroll
    for (u32 k = 0; k < CELL_H_EDGES; ++k) {
        R.he[k] = CellEdge{0u, 0u, 0u};
        if (k < nh) edge(h0 + k, R.he[k]);
    }
    R.ce = CellEdge{0u, 0u, 0u};
    if (nc == 2u) edge(r0 + 1u, R.ce);
    if (!ok || T.edge_cons[T.succ_edge[r0]] != tc) return;
    R.mark = CELL_MARK; R.H = H; R.nf = nt - 1u; R.ic_at = ic_at; R.taken = 0;
    R.n_edges = nh | (nc - 1u) << 8;
    R.h = T.val_off[h]; R.tc = T.val_off[tc]; R.o = T.val_off[o]; R.c = T.val_off[c];
    R.S = T.val_off[S]; R.sums = sums ? 1u : 0u;
    R.a = sums ? T.val_off[a] : 0u; R.b = sums ? T.val_off[a2] : 0u;
    R.at_o = at[NT]; R.sl_o = T.nat_off[sl[NT]];
    R.g = T.val_off[cand]; R.at_g = at[NT + 1]; R.sl_g = T.nat_off[sl[NT + 1]];
    R.ic = R.i = R.at_i = R.sl_i = 0;
#pragma unroll
    for (u32 k = 0; k < CELL_FORGET; ++k) {
        const bool past = k >= ic_at;       // the k-th term that is not i g
        R.f[k] = R.fp[k] = R.prev[k] = R.at_f[k] = R.sl_f[k] = 0;
        if ((past ? k + 1u : k) >= nt) continue;
        R.f[k] = T.val_off[past ? node[k + 1] : node[k]]; R.fp[k] = T.val_off[past ? t[k + 1] : t[k]];
        R.prev[k] = T.val_off[past ? with[k + 1] : with[k]];
        R.at_f[k] = past ? at[k + 1] : at[k]; R.sl_f[k] = T.nat_off[past ? sl[k + 1] : sl[k]];
    }
#pragma unroll
    for (u32 q = 0; q < NT; ++q)
        if (q == ic_at) { R.ic = T.val_off[t[q]]; R.i = T.val_off[node[q]]; R.at_i = at[q]; R.sl_i = T.nat_off[sl[q]]; }
    const u32 cell = atomicAdd(&T.hdr->n_cells, 1u);
    if (cell >= T.cells_cap) return;
    T.cells[cell] = R;
    T.cell_of[p] = cell;
    // the batches of its nodes (what there is less than CELL_NODES of is filled up with the output's own)
    CellNodes N;
    N.batch[0] = b | (3u + (nt - 1u ? nt : 0u) + 2u * gates + (sums ? 1u : 0u)) << 16;
    auto batch = [&](u32 u) { return T.batch_of_pos[T.pos_of[u]]; };
    N.batch[1] = batch(tc); N.batch[2] = batch(c); N.batch[3] = sums ? batch(S) : b;
#pragma unroll
    for (u32 q = 0; q < NT; ++q) N.batch[4 + q] = q < nt ? batch(t[q]) : b;
#pragma unroll
    for (u32 k = 0; k < NG; ++k) {
        const bool is = k < nt || k >= NT;
        N.batch[4 + NT + 2 * k] = is ? batch(node[k]) : b;
        N.batch[5 + NT + 2 * k] = is ? batch(sl[k]) : b;
    }
    // products that only this cell reads
    N.prod[0] = N.prod[1] = 0;
    if (sums && nt == 2u) {
#pragma unroll
        for (u32 k = 0; k < 2; ++k) {
            const u32 u = k == 0 ? a : a2;
            if (T.op[u] != OP_MATVEC || T.outdeg[u] != 1u) continue;
            const u32 pu = T.pos_of[u];
            N.prod[k] = T.batch_of_pos[pu] + 1u;
            T.prod_cell[pu] = cell;
        }
    }
    // who reads h and c
#pragma unroll
    for (u32 k = 0; k < CELL_H_EDGES + 1; ++k) {
        N.next[k] = 0;
        if (k < CELL_H_EDGES) N.at[k] = 0;
        if (k < CELL_H_EDGES ? k >= nh : nc != 2u) continue;
        const u32 v = T.edge_cons[T.succ_edge[k < CELL_H_EDGES ? h0 + k : r0 + 1u]], pv = T.pos_of[v];
        N.next[k] = T.batch_of_pos[pv] + 1u;
        if (k < CELL_H_EDGES && T.op[v] == OP_MATVEC) N.at[k] = pv + 1u;
    }
    T.cell_nodes_of[cell] = N;
}

// The cells among PARTS parts of `nodes` nodes each, from part `first` on: thread i of `threads`.
template <u32 PARTS>
__device__ inline void find_cells(const Tables &T, u32 nodes, u32 first, u32 i, u32 threads)
{
    u32 count[PARTS], total = 0;
#pragma unroll
    for (u32 q = 0; q < PARTS; ++q) {
        count[q] = (first + q) * nodes < T.n ? T.cell_ends_n[first + q] : 0u;
        total += count[q];
    }
    for (; i < total; i += threads) {
        u32 x = i, part = 0;
#pragma unroll
        for (u32 q = 0; q < PARTS; ++q)
            if (part == q && x >= count[q]) { x -= count[q]; part = q + 1u; }
        find_cell(T, T.cell_ends[(first + part) * nodes + x]);
    }
}

// A cell counts for its output's batch when all its nodes have been placed in one chain.  Called by whole waves: cells of a
// batch mostly lie side by side, and a wave adds them up before it goes to the batch's counters (an atomic per cell kept
// the counters of 64 trees' largest batches busy for 20 us).
__device__ inline void cell_in_chain(const Tables &T, u32 cell)
{
    const u32 lane = threadIdx.x & 63u;
    CellNodes N;
    N.batch[0] = 0;
    bool taken = false, takes = false, hold = false;
    bool one = cell < T.hdr->n_cells && cell < T.cells_cap;
    if (one) {
        N = T.cell_nodes_of[cell];
        const u32 b = N.batch[0] & 0xffffu, slot = T.slot_of[b], label = T.label_of[b];
#pragma unroll
        for (u32 k = 1; k < CELL_NODES; ++k) one = one && T.slot_of[N.batch[k]] == slot && T.label_of[N.batch[k]] == label;
#pragma unroll
        for (u32 k = 0; k < 2; ++k) {
            if (!N.prod[k]) continue;
            const BatchRec &rp = T.batches[N.prod[k] - 1u];
            taken = taken || (T.slot_of[N.prod[k] - 1u] + 1u == slot && !(rp.vec4 & TF_WIDE) && !batch_xp(rp) && rp.d == 4u * T.batches[b].d);
        }
        u32 reader = 0;
#pragma unroll
        for (u32 k = 0; k < CELL_H_EDGES + 1; ++k) {
            if (!N.next[k] || T.slot_of[N.next[k] - 1u] != slot + 1u) continue;
            // (a product's dX tiles work the cells whose outputs are its operands: one that reads c holds them like any other reader)
            const u32 product = k < CELL_H_EDGES ? N.at[k] : 0u;
            hold = hold || takes || !product;
            takes = true;
            reader = product;
        }
        if (one && takes && !hold) T.cells[cell].taken = reader;
    }
    for (u64 todo = __ballot(one); todo;) {
        const u32 leader = (u32)__builtin_ctzll(todo), word = (u32)__shfl((int)N.batch[0], (int)leader);
        const u64 same = __ballot(one && N.batch[0] == word), with = __ballot(one && N.batch[0] == word && taken);
        const u64 reads = __ballot(one && N.batch[0] == word && takes), held = __ballot(one && N.batch[0] == word && hold);
        if (lane == leader) {
            const u32 rows = (u32)__popcll(same);
            atomicAdd(&T.cell_rows[word & 0xffffu], rows);
            atomicAdd(&T.cell_nodes[word & 0xffffu], rows * (word >> 16));
            if (with) atomicAdd(&T.cell_prods[word & 0xffffu], (u32)__popcll(with));
            if (reads) atomicAdd(&T.cell_takes[word & 0xffffu], (u32)__popcll(reads));
            if (held) atomicOr(&T.cell_takes[word & 0xffffu], CELL_HOLD);
        }
        todo &= ~same;
    }
}

// One workgroup.  Over the batch dependencies, where a fusable edge costs 0 and any other edge one
// launch boundary: head(b) = longest path from any source to b, tail(b) = longest path from b to any
// sink.  Batch ids are a topological order (a batch's operands lie in earlier batches in every batching
// mode), so the distinct dependencies are first put in the order of their consumer (a counting sort in
// LDS) and then walked once by a wave, 64 at a time: forward for the heads (every producer of a chunk's
// consumers was settled by an earlier chunk or is settled inside the chunk, which is passed over until
// nothing changes), and by a second wave beside it backward for the tails.  That is as many dependent steps as the list has chunks
// instead of as many as the longest path has edges.  The
// plan has L + 1 slots, L = max head.  fuse == 1 places a batch as early as possible (slot =
// head), fuse == 2 as late as possible (slot = L - tail): batches off the critical path then
// gather in the slots next to their consumers instead of trailing the recurrence one small
// launch at a time.  Batches joined by fusable edges inside one slot then get a common chain
// label (the smallest batch id of the chain).  The workgroups behind the first look for gated cells meanwhile:
// each fills a CU's LDS like the first, so there are few, 2 048 nodes to one.  (With all nodes looked at here, 256 to a workgroup, the 740
// of a graph of 189 000 nodes took 24 rounds on the 32 CUs of a schedule stream: 216 us of this kernel, 101 now, 71 and 70 on the
// whole chip; schedules of that graph there 1 198 and 1 088 us, 650 on the whole chip.  Listing the nodes takes the launch that sets
// nodes up nothing that shows.  4 096 nodes to a workgroup: the same; 8 192: 1 061 us, but 64 trees 356 where they take 332.)
constexpr int SLOT_THREADS = 1024;
constexpr u32 CELL_PARTS = 8;          // parts of TPB nodes
struct SlotsLds {
    u32 slot[SLOT_MAX_NB];
    u32 label[SLOT_MAX_NB];      // tail lengths first, chain labels afterwards
    u32 edge[BLIST_MAX];
    u32 changed;
    u32 flag[3];
    u32 wsum[SLOT_THREADS / 64];
};
// beside(i, k): work of the k threads that have none while two waves walk the dependencies, i = 0 .. k - 1
template <typename Beside>
__device__ inline void slots_of(const Tables &T, int fuse, const u32 *blist, SlotsLds &L, Beside beside)
{
    u32 *s_slot = L.slot, *s_label = L.label, *s_edge = L.edge, *s_flag = L.flag, *s_wsum = L.wsum;
    u32 &s_changed = L.changed;
    const u32 nb = T.hdr->n_batches;
    const u32 ne = T.hdr->n_bedges;
    const u32 tid = threadIdx.x;
    if (!fuse || nb > SLOT_MAX_NB || ne > BLIST_MAX) {   // one slot per step, no fusion
        for (u32 b = tid; b < nb; b += SLOT_THREADS) { T.slot_of[b] = T.batches[b].step; T.label_of[b] = b; }
        if (tid == 0) { T.hdr->n_slots = T.hdr->n_steps; T.hdr->slot_sweeps = 0; T.hdr->p0 = 1; }
        return;
    }
    // ---- the dependencies in the order of their consumer: count per consumer (in s_label), exclusive scan,
    // scatter (the order among one consumer's entries does not matter: only maxima and minima are taken)
    for (u32 b = tid; b < SLOT_MAX_NB; b += SLOT_THREADS) { s_slot[b] = 0; s_label[b] = 0; }
    __syncthreads();
    for (u32 e = tid; e < ne; e += SLOT_THREADS) atomicAdd(&s_label[(blist[e] - 1u) >> 13], 1u);
    __syncthreads();
    {
        constexpr u32 PER = SLOT_MAX_NB / SLOT_THREADS;   // consecutive counters per thread
        u32 c[PER], sum = 0;
        for (u32 i = 0; i < PER; ++i) { c[i] = s_label[tid * PER + i]; sum += c[i]; }
        u32 inc = sum;                                     // inclusive scan over the wave
        for (u32 o = 1; o < 64; o <<= 1) { const u32 v = (u32)__shfl_up((int)inc, o); if ((tid & 63u) >= o) inc += v; }
        if ((tid & 63u) == 63u) s_wsum[tid >> 6] = inc;
        __syncthreads();
        u32 before = inc - sum;
        for (u32 w = 0; w < (tid >> 6); ++w) before += s_wsum[w];
        for (u32 i = 0; i < PER; ++i) { s_label[tid * PER + i] = before; before += c[i]; }
    }
    __syncthreads();
    for (u32 e = tid; e < ne; e += SLOT_THREADS) {
        const u32 k = blist[e] - 1u;
        s_edge[atomicAdd(&s_label[k >> 13], 1u)] = k;
    }
    __syncthreads();
    for (u32 b = tid; b < SLOT_MAX_NB; b += SLOT_THREADS) s_label[b] = 0;
    __syncthreads();
    // ---- heads forward (wave 0, in s_slot) and tails backward (wave 1, in s_label), which know nothing of each
    // other: chunk by chunk (a wave's LDS operations complete in order)
    const u32 lane = tid & 63u;
    u32 walked = 0;      // passes over chunks, for the statistics
    if (tid < 128) {
        const bool tails = __builtin_amdgcn_readfirstlane(tid) >= 64u;
        u32 *len = tails ? s_label : s_slot;
        const u32 n_chunks = (ne + 63u) / 64u;
        for (u32 i = 0; i < n_chunks; ++i) {
            const u32 e = (tails ? n_chunks - 1u - i : i) * 64u + lane;
            const bool valid = e < ne;
            const u32 k = valid ? s_edge[e] : 0u;
            const u32 c = k >> 13, y = (k >> 1) & 0xfffu, cost = k & 1u;
            const u32 *from = &len[tails ? c : y];
            u32 *to = &len[tails ? y : c];
            for (u32 rep = 0; rep < 66u; ++rep) {          // (a chain inside a chunk has at most 64 links)
                bool changed = false;
                if (valid) {
                    const u32 want = lds_load(from) + cost;
                    if (want > lds_load(to)) { atomicMax(to, want); changed = true; }
                }
                ++walked;
                if (__ballot(changed) == 0ull) break;
            }
        }
    }
    else beside(tid - 128u, (u32)SLOT_THREADS - 128u);
    if (tid == 64) s_wsum[0] = walked;
    __syncthreads();
    walked += s_wsum[0];
    {   // number of slots; late placement; labels start as the batch's own id
        u32 mx = 0;
        for (u32 b = tid; b < nb; b += SLOT_THREADS) mx = s_slot[b] > mx ? s_slot[b] : mx;
        if (tid == 0) s_changed = 0;
        __syncthreads();
        atomicMax(&s_changed, mx);
        __syncthreads();
        const u32 L = s_changed;
        __syncthreads();
        for (u32 b = tid; b < nb; b += SLOT_THREADS) {
            if (fuse == 2) s_slot[b] = L - s_label[b];
            s_label[b] = b;
        }
        if (tid == 0) T.hdr->n_slots = L + 1;
        __syncthreads();
    }
    // One barrier per sweep: sweep k raises s_flag[k % 3] when it changes anything, everybody reads
    // it behind the sweep's barrier, and the flag of sweep k + 1 is cleared during sweep k (its last
    // readers were those of sweep k - 2, who have all passed the barrier of sweep k - 1).
    if (tid < 3) s_flag[tid] = 0;
    __syncthreads();
    u32 sweeps = 0;
    while (true) {
        const u32 f = sweeps % 3u;
        if (tid == 0) s_flag[(sweeps + 1u) % 3u] = 0;
        for (u32 e = tid; e < ne; e += SLOT_THREADS) {
            const u32 k = s_edge[e];
            if (k & 1u) continue;
            const u32 c = k >> 13, y = (k >> 1) & 0xfffu;
            if (s_slot[c] != s_slot[y]) continue;
            const u32 a = s_label[c], bb = s_label[y];
            if (a != bb) {
                const u32 m = a < bb ? a : bb;
                atomicMin(&s_label[c], m);
                atomicMin(&s_label[y], m);
                s_flag[f] = 1;
            }
        }
        __syncthreads();
        ++sweeps;
        if (!s_flag[f] || sweeps > 2 * nb + 2) break;
    }
    for (u32 b = tid; b < nb; b += SLOT_THREADS) { T.slot_of[b] = s_slot[b]; T.label_of[b] = s_label[b]; }
    if (tid == 0) T.hdr->slot_sweeps = walked + sweeps;
}
__global__ __launch_bounds__(SLOT_THREADS) void k_slots(Tables T, int fuse, const u32 *blist)
{
    __shared__ SlotsLds L;
    if (blockIdx.x == 0) slots_of(T, fuse, blist, L, [](u32, u32) {});
    else if (T.hdr->n_batches <= SLOT_MAX_NB) find_cells<CELL_PARTS>(T, TPB, (blockIdx.x - 1u) * CELL_PARTS, threadIdx.x, SLOT_THREADS);
}

__device__ inline void launch_keys_at(const Tables &T, u64 *keys, u32 *vals, u32 n_pad, u32 b)
{
    const bool in = b < n_pad;
    if (T.cells) cell_in_chain(T, b);
    if (in) vals[b] = b;
    // batches without forward work, counted for the statistics: summed over the wave first (every lane takes
    // part), one atomic per wave
    const bool live = in && b < T.hdr->n_batches;
    u32 cnt[4] = {0u, 0u, 0u, 0u};
    if (live) {
        const BatchRec &r = T.batches[b];
        if (r.op == OP_MATVEC) atomicAdd(&T.slot_dx[T.slot_of[b]], r.B * r.k);
        if (r.vec4 & TF_VIEW) { cnt[0] = 1u; cnt[1] = r.B * r.d; }
        if (r.vec4 & TF_VIRT) { cnt[2] = 1u; cnt[3] = r.B * r.d; }
    }
    if (__ballot(cnt[0] | cnt[2]) != 0ull) {
        for (int q = 0; q < 4; ++q)
            for (int o = 32; o > 0; o >>= 1) cnt[q] += __shfl_xor(cnt[q], o);
        if ((threadIdx.x & 63u) == 0u) {
            if (cnt[0]) { atomicAdd(&T.hdr->view_batches, cnt[0]); atomicAdd(&T.hdr->view_floats, cnt[1]); }
            if (cnt[2]) { atomicAdd(&T.hdr->virt_batches, cnt[2]); atomicAdd(&T.hdr->virt_floats, cnt[3]); }
        }
    }
    if (!in) return;
    if (!live) { keys[b] = ~0ull; return; }
    // unfused plans are already in launch order (slot = step): equal keys keep that order
    keys[b] = T.hdr->p0 ? 0ull : (((u64)T.slot_of[b] << SLOT_BITS) | T.label_of[b]);
}
__global__ void k_launch_keys(Tables T, u64 *keys, u32 *vals, u32 n_pad)
{
    launch_keys_at(T, keys, vals, n_pad, blockIdx.x * blockDim.x + threadIdx.x);
}

__device__ inline u32 rows_per_block(u32 d) { return d >= (u32)EW_TILE ? 1u : (u32)EW_TILE / d; }

// chains from the launch order: head flags, then one thread per chain head fills the record
__device__ inline u64 chain_key(const Tables &T, u32 b) { return ((u64)T.slot_of[b] << 32) | T.label_of[b]; }

// (and the start values of the tables that the next kernels fill in: every slot entry a plan can use,
// n_slots + 1 <= n + 2, starts out as "no batch here", every chain's layout as empty)
__device__ inline void chain_flags_at(const Tables &T, const u32 *sval, u32 *flag, CLay *clay_in, u32 n_pad, u32 i)
{
    if (i <= T.hdr->n_slots) {
        SlotRec r; r.wf = r.wa = r.tb = r.tf = r.ta = r.lmin = r.nlmax = r.dx_free = 0xffffffffu;
        r.lds_need = 0;
        r.lminf = r.nlmaxf = 0xffffffffu;
        r.plain = 0xffffffffu;
        T.slots[i] = r;
    }
    if (i >= n_pad) return;
    CLay L; L.tf = L.wf = L.ta = L.wa = L.tb = L.p0 = L.p1 = L.p2 = 0;
    clay_in[i] = L;
    const u32 nb = T.hdr->n_batches;
    if (i < nb) T.lorder[i] = sval[i];
    flag[i] = (i < nb && (i == 0 || chain_key(T, sval[i]) != chain_key(T, sval[i - 1]))) ? 1u : 0u;
}
__global__ void k_chain_flags(Tables T, const u32 *sval, u32 *flag, CLay *clay_in, u32 n_pad)
{
    chain_flags_at(T, sval, flag, clay_in, n_pad, blockIdx.x * blockDim.x + threadIdx.x);
}

// whether batch c reads a result of batch y through a fusable dependency (the set k_bedges filled)
__device__ inline bool bset_has(const u32 *bset, u32 c, u32 y)
{
    const u32 key = ((c << 13) | (y << 1)) + 1u;
    u32 h = (key * 2654435761u) & (BSET_SIZE - 1);
    for (u32 probe = 0; probe < BSET_SIZE; ++probe) {
        const u32 k = bset[h];
        if (k == key) return true;
        if (k == 0u) return false;
        h = (h + 1) & (BSET_SIZE - 1);
    }
    return false;
}

constexpr u32 LEVEL_MAX_MEMBERS = 32;   // chains with more members keep their step order and one tile group per member

__device__ inline void chain_recs_at(const Tables &T, int agenda, const u32 *bset, const u32 *flag, const u32 *flag_excl, CLay *clay_in, u32 n_pad, u32 i)
{
    if (i >= n_pad) return;
    const u32 nb = T.hdr->n_batches;
    CLay L; L.tf = L.wf = L.ta = L.wa = L.tb = L.p0 = L.p1 = L.p2 = 0;
    if (i < nb) {
        const u32 c = flag_excl[i] + flag[i] - 1;
        T.chain_of_lpos[i] = c;
        T.chain_of_batch[T.lorder[i]] = c;   // (a chain's members may still be reordered below: same chain)
        if (i == nb - 1) T.hdr->n_chains = c + 1;
    }
    if (i < nb && flag[i]) {
        const u32 c = flag_excl[i];
        u32 k = 1;
        while (true) {          // (eight flags at a time; beyond the last batch they are 0)
            u32 f = 8;
#pragma unroll
            for (u32 q = 8; q-- > 0;) if (i + k + q >= nb || flag[i + k + q]) f = q;
            k += f;
            if (f < 8) break;
        }
        // Members of a chain run level by level, the tiles of one level without a barrier between
        // them.  In depth mode a member's level is its depth.  Agenda batches are steps of their
        // own, so there the levels come from the dependencies inside the chain (level = 1 + the
        // largest level of the members it reads), and the members are put in (level, batch) order.
        const bool by_step = !agenda || T.hdr->p0;
        if (by_step) {
            // (set below)
        } else if (k > LEVEL_MAX_MEMBERS) {
            for (u32 m = 0; m < k; ++m) T.blevel[T.lorder[i + m]] = m;
        } else {
            u32 ids[LEVEL_MAX_MEMBERS], lv[LEVEL_MAX_MEMBERS];
            for (u32 m = 0; m < k; ++m) {
                ids[m] = T.lorder[i + m];
                u32 l = 0;
                for (u32 mm = 0; mm < m; ++mm)
                    if (lv[mm] + 1 > l && bset_has(bset, ids[m], ids[mm])) l = lv[mm] + 1;
                lv[m] = l;
            }
            for (u32 m = 1; m < k; ++m) {   // stable insertion sort by level
                const u32 id = ids[m], l = lv[m];
                u32 j = m;
                while (j > 0 && lv[j - 1] > l) { ids[j] = ids[j - 1]; lv[j] = lv[j - 1]; --j; }
                ids[j] = id; lv[j] = l;
            }
            for (u32 m = 0; m < k; ++m) { T.lorder[i + m] = ids[m]; T.blevel[ids[m]] = lv[m]; }
        }
        const BatchRec r0 = T.batches[T.lorder[i]];
        ChainRec cr;
        cr.first = i; cr.k = k; cr.slot = T.slot_of[T.lorder[i]];
        cr.fused = op_chain_source(r0.op, r0.arity) ? 1u : 0u;
        // one walk over the members, eight side by side (their reads depend on each other in pairs only): a thread that
        // walked them one read after the other, three times, took 11 us for the longest chain of a graph of a thousand nodes
        u32 dmax = 0, G = 0, rows = 0, rows_f = 0;
        u32 floats = 0;         // (a plan of 2^32 and more is refused)
        u32 out = 0xffffffffu, cells = 0, cell_nodes = 0, cell_d = 0;   // the member that gated cells end in
        const bool look = T.cells && T.hdr->n_cells > 0;
        for (u32 m0 = 0; m0 < k; m0 += 8) {
            u32 id[8], B[8], d[8], step[8], flags[8], found[8];
#pragma unroll
            for (u32 q = 0; q < 8; ++q) id[q] = T.lorder[i + (m0 + q < k ? m0 + q : m0)];
#pragma unroll
            for (u32 q = 0; q < 8; ++q) {
                const BatchRec &rm = T.batches[id[q]];
                B[q] = rm.B; d[q] = rm.d; step[q] = rm.step; flags[q] = rm.vec4;
                found[q] = look ? T.cell_rows[id[q]] : 0u;
            }
#pragma unroll
            for (u32 q = 0; q < 8; ++q) {
                if (m0 + q >= k) break;
                if (by_step) T.blevel[id[q]] = step[q];
                dmax = d[q] > dmax ? d[q] : dmax;
                if (B[q] != G) G = gcd_u32(G, B[q]);
                rows += B[q];
                if (!(flags[q] & TF_NOFWD)) rows_f += B[q];
                floats += B[q] * d[q];
                if (found[q]) { out = id[q]; cells = found[q]; cell_d = d[q]; }
            }
        }
        if (out != 0xffffffffu) cell_nodes = T.cell_nodes[out];
        // tiles per block (all members / members with forward work); floats one group of every member takes
        u32 kt = rows / G, ktf = rows_f / G;
        const u32 per_group = floats / G;
        cr.G = G; cr.Rg = rows_per_block(dmax);
        if (cr.fused && k > 1) {
            // hand results from member to member through LDS when a block of groups fits (each
            // member's region is rounded up to 4 floats); fewer groups per block if that is what it takes
            const u32 fit = (CHAIN_LDS_FLOATS - 3u * k) / per_group;
            if (fit >= 1) { cr.fused = 2u; if (fit < cr.Rg) cr.Rg = fit; }
        }
        cr.pad0 = cr.pad1 = cr.pad2 = 0;
        // gated cells and nothing else (cells so wide that a group of all their rows, 17 H floats for an LSTM's, does not fit the LDS copy
        // stay an interpreted run, as do those of plans without room for the tables)
        if (cr.fused == 2u && cells == G && cell_nodes == kt * G) {
            cr.fused = 3u; cr.pad0 = out;
            cr.Rg = CELL_WAVES / cell_row_waves(cell_d);
            kt = ktf = cr.Rg;      // a tile a row; the last block's may be left over
            const u32 takes = T.cell_takes[out];
            if (!(takes & CELL_HOLD)) atomicAdd(&T.slot_cells[cr.slot], 1u);
            if (!(takes & CELL_HOLD) && takes) atomicOr(&T.slot_cells[cr.slot], CELL_HOLD);
        }
        cr.nrb = cdiv(G, cr.Rg); cr.kt = cr.fused ? kt : 1u;
        cr.ktf = cr.fused ? ktf : 1u;
        if (cr.fused) {
            L.ta = cr.nrb * kt; L.wa = cr.nrb;
            L.tf = cr.nrb * ktf; L.wf = ktf ? cr.nrb : 0u;     // a chain of views only has no forward work
        } else {
            switch (r0.op) {
            case OP_MATVEC: {
                const u32 gt = (r0.vec4 & TF_WIDE) ? (u32)GTW : (u32)GT;
                const bool large = T.slot_dx[cr.slot] >= DX_LARGE_SLOT;
                if (large) T.batches[T.lorder[i]].vec4 |= TF_DX_LARGE;
                const u32 dt = dx_tile_edge(r0.vec4 | (large ? (u32)TF_DX_LARGE : 0u), r0.k);
                L.tf = cdiv(r0.B, gt) * cdiv(r0.d, gt); L.tb = cdiv(r0.B, dt) * cdiv(r0.k, dt);
                break;
            }
            case OP_PICK_NLS:
            case OP_SQNORM: L.tf = cdiv(r0.B, ROWS_PER_RED_TILE); break;
            default: L.tf = r0.B; break;   // wide sum: one workgroup per row
            }
            L.wf = L.tf;
            L.ta = L.wa = cr.nrb;          // pull tiles are row blocks of the batch
        }
        if (T.cells) { atomicAdd(&T.slot_chains[cr.slot], 1u); atomicAdd(&T.slot_rows[cr.slot], rows); }
        T.chains[c] = cr;
        clay_in[c] = L;
    }
}
__global__ void k_chain_recs(Tables T, int agenda, const u32 *bset, const u32 *flag, const u32 *flag_excl, CLay *clay_in, u32 n_pad)
{
    chain_recs_at(T, agenda, bset, flag, flag_excl, clay_in, n_pad, blockIdx.x * blockDim.x + threadIdx.x);
}

// floats of a fused chain's LDS copy taken by one member: its rows of a block of groups, rounded up to 4
__device__ inline u32 chain_region(const ChainRec &cr, const BatchRec &r) { return (cr.Rg * (r.B / cr.G) * r.d + 3u) & ~3u; }

// per chain: first work item / tile of every launch slot and its run lengths, totals in the header
__device__ inline void slot_tables_at(const Tables &T, const CLay *clay_ex, const CLay *total, u32 c)
{
    const u32 nc = T.hdr->n_chains;
    if (c >= nc) return;
    const ChainRec cr = T.chains[c];
    const u32 s = cr.slot;
    const CLay L = clay_ex[c];
    SlotRec &S = T.slots[s];
    if (c == 0 || T.chains[c - 1].slot != s) { S.wf = L.wf; S.wa = L.wa; S.tb = L.tb; S.tf = L.tf; S.ta = L.ta; }
    const BatchRec &hb = T.batches[T.lorder[cr.first]];
    if (hb.op == OP_MATVEC && !(hb.vec4 & TF_G_ALIAS)) S.dx_free = 0;   // this slot's dX tiles need the slot's own pull first
    if (cr.fused == 3u) atomicAnd(&S.plain, ~8u);
    if (hb.op != OP_MATVEC || !(hb.vec4 & TF_G_ALIAS)) atomicAnd(&S.plain, ~16u);
    // (every row of a product taken up has one reader, so as many rows as cells are all rows of the slot before)
    if (cr.fused == 3u && s > 0 && T.slot_chains[s] == 1u && T.cell_prods[cr.pad0] == cr.G && T.slot_rows[s - 1u] == cr.G) atomicAnd(&S.plain, ~4u);
    if (cr.fused == 3u && T.slot_cells[s] == (T.slot_chains[s] | CELL_HOLD)) atomicAnd(&S.plain, ~32u);
    if (!cr.fused) atomicAnd(&S.plain, ~1u);     // a GEMM, reduction or wide-sum batch runs in this slot
    if (batch_xp(hb) && hb.aux1 > 1) atomicAnd(&S.plain, ~2u);   // a product that reads its operand rows in pieces
    if (cr.fused == 2u) {
        u32 need = 0;
        for (u32 m = 0; m < cr.k; ++m) need += chain_region(cr, T.batches[T.lorder[cr.first + m]]);
        atomicMax(&S.lds_need, need);
    }
    const u32 cells = cr.fused == 3u ? CELL_ITEM : 0u;
    const u32 len = cr.fused ? cr.kt | cells : 1u;
    atomicMin(&S.lmin, len);
    atomicMin(&S.nlmax, ~len);
    const u32 lenf = cr.fused ? cr.ktf | cells : 1u;
    if (lenf) {   // (a chain of views has no forward work item)
        atomicMin(&S.lminf, lenf);
        atomicMin(&S.nlmaxf, ~lenf);
    }
    if (c == nc - 1) {
        const CLay t = *total;
        SlotRec &E = T.slots[s + 1];
        E.wf = t.wf; E.wa = t.wa; E.tb = t.tb; E.tf = t.tf; E.ta = t.ta;
        T.hdr->tiles_fwd = t.tf; T.hdr->tiles_pull = t.ta; T.hdr->tiles_dx = t.tb;
        T.hdr->works_fwd = t.wf; T.hdr->works_pull = t.wa;
    }
}
__global__ void k_slot_tables(Tables T, const CLay *clay_ex, const CLay *total)
{
    slot_tables_at(T, clay_ex, total, blockIdx.x * blockDim.x + threadIdx.x);
}

// launch slots that hold no batch (neither placement produces one today; the launch tables
// simply do not rely on it) inherit the offsets of the next slot that does, so that their launch
// range is empty
__device__ inline void slot_fill_at(const Tables &T, u32 s)
{
    if (s >= T.hdr->n_slots) return;
    u32 t = s;
    while (T.slots[t].wf == 0xffffffffu) ++t;   // entry n_slots is always set
    if (t != s) {
        const SlotRec N = T.slots[t];
        SlotRec &S = T.slots[s];
        S.wf = N.wf; S.wa = N.wa; S.tb = N.tb; S.tf = N.tf; S.ta = N.ta;
    }
}
__global__ void k_slot_fill(Tables T)
{
    slot_fill_at(T, blockIdx.x * blockDim.x + threadIdx.x);
}

// ---- tile descriptors ------------------------------------------------------------------------------
constexpr u32 CONTIG_MAX_ROWS = 64;   // tiles with more rows skip the even-spacing test

// Where a tile of a fused chain sits: chain, member, block of groups [g0, g0 + ng).  (Handed on by reference with a flag
// beside it: a pointer that may be null would keep it in scratch memory.)
struct ChainCtx { ChainRec cr; u32 m, g0, ng; };


// For up to four row-offset ranges [lo[j], hi[j]] (first element of the lowest / highest row read
// through slot j; offsets in the value arena, which the gradient arena mirrors): state 0 = no
// member of the chain produces these rows, 1 = all of them lie in this block's rows of one member
// (LDS index = offset + delta[j]), 2 = produced in the chain but not covered by one region.
// (Loops over slots and edges run to four with the count as a guard, here and below: an array that is indexed by
// a counter the compiler cannot unroll lives in scratch memory, and these kernels are bound by their reads as it is.)
__device__ inline void chain_lookup(const Tables &T, const ChainCtx &cc, u32 ns, const u32 (&lo)[4], const u32 (&hi)[4],
                                    u32 (&state)[4], u32 (&delta)[4])
{
#pragma unroll
    for (u32 j = 0; j < 4; ++j) { state[j] = 0; delta[j] = 0; }
    u32 lds = 0;
    for (u32 mm = 0; mm < cc.cr.k; ++mm) {
        const BatchRec &y = T.batches[T.lorder[cc.cr.first + mm]];
        const u32 mult = y.B / cc.cr.G;
        const u32 full_lo = y.val_off, full_hi = y.val_off + y.B * y.d;
        const u32 ch_lo = y.val_off + cc.g0 * mult * y.d, ch_hi = ch_lo + cc.ng * mult * y.d;
        if (mm != cc.m) {
#pragma unroll
            for (u32 j = 0; j < 4; ++j) {
                if (j >= ns || hi[j] < full_lo || lo[j] >= full_hi) continue;
                if (state[j] == 0 && cc.cr.fused == 2u && lo[j] >= ch_lo && hi[j] < ch_hi) { state[j] = 1; delta[j] = lds - ch_lo; }
                else state[j] = 2;
            }
        }
        lds += chain_region(cc.cr, y);
    }
}

// LDS index offset of the block's own rows of member cc.m (index = arena offset + result)
__device__ inline u32 chain_own_delta(const Tables &T, const ChainCtx &cc, const BatchRec &r)
{
    u32 lds = 0;
    for (u32 mm = 0; mm < cc.m; ++mm) lds += chain_region(cc.cr, T.batches[T.lorder[cc.cr.first + mm]]);
    return lds - (r.val_off + cc.g0 * (r.B / cc.cr.G) * r.d);
}

// Which tile of a product the t-th of its workgroups takes.  Workgroup g of a launch runs on XCD g % 8 (a product that starts at another
// multiple finds the XCDs renamed, and a workgroup's next tile is a multiple of eight further on), every XCD has its own L2, and all L2s
// are cold when a launch starts, so what an XCD reads is the rows and the columns of its tiles.  The eight XCDs are therefore laid out as
// pr x pc over the tiles, whichever reads least: rows / pr + columns / pc, both as long as the contraction.  (With pr = 1
// throughout, dX of 512 rows a direction had every XCD read all 4 MB of gradients.)
__device__ inline u32 xcd_tile(u32 t, u32 ntr, u32 ntn, u32 rows, u32 cols)
{
    u32 best = 0xffffffffu, pr = 0;
#pragma unroll
    for (u32 p = 1; p <= 8; p *= 2) {
        const u32 reads = rows / p + cols / (8u / p);
        if (p <= ntr && ntn % (8u / p) == 0u && reads < best) { best = reads; pr = p; }
    }
    if (!pr) return t;
    const u32 pc = 8u / pr, npc = ntn / pc;
    if (t >= ntr / pr * pr * ntn) return t;       // rows of tiles that are left over
    const u32 x = t & 7u, j = t >> 3;
    return ((j / npc) * pr + x % pr) * ntn + (j % npc) * pc + x / pr;
}

// descriptor of a forward or dX tile of batch r.  Component-wise tiles (row_block) cover the rows
// row0 + i * rstride, i < nrows; the other kinds derive their rows from the tile index t.
__device__ inline void fill_tile_desc(const Tables &T, const BatchRec &r, u32 t, bool dx, bool row_block, u32 row0,
                                      u32 nrows, u32 rstride, TileDesc &d, bool in_chain, const ChainCtx &cc)
{
    if (r.op == OP_MATVEC && !row_block) {
        const u32 edge = dx ? dx_tile_edge(r.vec4, r.k) : (r.vec4 & TF_WIDE) ? (u32)GTW : (u32)GT, cols = dx ? r.k : r.d;
        t = xcd_tile(t, cdiv(r.B, edge), cdiv(cols, edge), r.B, cols);
    }
    d.op = r.op; d.B = r.B; d.d = r.d; d.arity = r.arity;
    d.pos0 = r.pos0; d.val_off = r.val_off; d.dx_off = r.dx_off; d.k = r.k;
    d.aux0 = r.aux0; d.rstride = rstride;
    d.w = r.param >= 0 ? T.params[r.param].data : nullptr;
    d.b = r.bias >= 0 ? T.params[r.bias].data : nullptr;
    d.lds_out = 0;
    for (int j = 0; j < 4; ++j) d.lds_src[j] = 0;
    d.pad = 0;
    d.opnd = r.opnd; d.indim = r.indim; d.flags = r.vec4; d.t = t;
    d.contig = 0; d.row0 = row0; d.nrows = nrows; d.depth = r.step;
    for (int j = 0; j < 4; ++j) { d.base[j] = 0; d.sdim[j] = 0; d.sstride[j] = 0; }
    if (dx) {
        // dX tile: rows (t / ntn) * DXT ...; with TF_G_ALIAS the gradient rows are read where the
        // consumer left them, evenly spaced or through the per-row list
        if (r.vec4 & TF_G_ALIAS) {
            const u32 dt = dx_tile_edge(r.vec4, r.k);
            const u32 ntn = (r.k + dt - 1) / dt;
            const u32 r_lo = (t / ntn) * dt;
            u32 r_hi = r_lo + dt - 1;
            if (r_hi >= r.B) r_hi = r.B - 1;
            const u32 *gs = T.dx_gsrc + r.pos0;
            const u32 base = gs[r_lo];
            bool ok = true;
            u32 ss = 0;
            if (r_hi > r_lo) {
                ss = gs[r_lo + 1] - base;
                for (u32 i0 = 2; r_lo + i0 <= r_hi; i0 += 8) {      // eight reads in flight
                    u32 o[8];
#pragma unroll
                    for (u32 q = 0; q < 8; ++q) o[q] = gs[r_lo + (r_lo + i0 + q <= r_hi ? i0 + q : 0u)];
#pragma unroll
                    for (u32 q = 0; q < 8; ++q) ok = ok && (r_lo + i0 + q > r_hi || o[q] == base + (i0 + q) * ss);
                }
            }
            d.base[0] = base; d.sstride[0] = ss;
            if (ok) d.contig |= 1u;
        }
        return;
    }
    if (!row_block && r.arity == 0) return;
    if (!row_block) {
        u32 r_lo, r_hi;
        if (r.op == OP_MATVEC) {
            const u32 gt = (r.vec4 & TF_WIDE) ? (u32)GTW : (u32)GT;
            const u32 ntn = (r.d + gt - 1) / gt;
            r_lo = (t / ntn) * gt; r_hi = r_lo + gt - 1;
        } else if (r.op == OP_PICK_NLS || r.op == OP_SQNORM) {
            r_lo = t * ROWS_PER_RED_TILE; r_hi = r_lo + ROWS_PER_RED_TILE - 1;
        } else {
            r_lo = r_hi = t;   // wide sum
        }
        if (r_hi >= r.B) r_hi = r.B - 1;
        d.row0 = row0 = r_lo; d.nrows = nrows = r_hi - r_lo + 1; d.rstride = rstride = 1;
    }
    const bool xp = batch_xp(r);
    const u32 ns = xp ? (u32)r.aux1 : (r.arity < 4 ? r.arity : 4);   // a product reading in pieces: one operand slot per piece
    if (xp) d.arity = ns;
    u32 lo[4], hi[4];
#pragma unroll
    for (u32 j = 0; j < 4; ++j) {
        lo[j] = hi[j] = 0;
        if (j >= ns) continue;
        const u32 *op = T.opnd_off + r.opnd + j * r.B;
        const u32 base = op[row0];
        d.base[j] = base; d.sdim[j] = T.b_indim[r.indim + j];
        bool ok = nrows <= CONTIG_MAX_ROWS;
        u32 ss = 0;
        lo[j] = hi[j] = base;
        if (ok && nrows > 1) {
            ss = op[row0 + rstride] - base;
            for (u32 i0 = 1; i0 < nrows; i0 += 8) {      // eight reads in flight
                u32 o[8];
#pragma unroll
                for (u32 q = 0; q < 8; ++q) o[q] = op[row0 + (i0 + q < nrows ? i0 + q : 0u) * rstride];
#pragma unroll
                for (u32 q = 0; q < 8; ++q) {
                    if (i0 + q >= nrows) continue;
                    ok = ok && o[q] == base + (i0 + q) * ss;
                    lo[j] = o[q] < lo[j] ? o[q] : lo[j]; hi[j] = o[q] > hi[j] ? o[q] : hi[j];
                }
            }
        }
        d.sstride[j] = ss;
        if (ok) d.contig |= 1u << j;
    }
    if (row_block && (d.flags & TF_VEC4) && r.arity >= 1 && r.arity <= 4 && (d.contig & 0xfu) == (1u << r.arity) - 1u &&
        (r.op == OP_ADD || r.op == OP_CMULT || r.op == OP_TANH || r.op == OP_SIGMOID || r.op == OP_SLICE))
        d.flags |= TF_SIMPLE;
    if (!in_chain) return;
    // tile of a fused chain: which operands come from the chain's LDS copy, and whether any
    // operand produced earlier in the same launch still has to come from global memory
    if (cc.cr.fused != 2u || nrows > CONTIG_MAX_ROWS || r.arity > 4) { d.flags |= TF_GLOBAL_DEP; }
    if (cc.cr.fused != 2u) return;
    d.lds_out = chain_own_delta(T, cc, r);
    d.flags |= TF_OUT_LDS;
    if (d.lds_out & 3u) d.flags &= ~(u32)(TF_VEC4 | TF_SIMPLE);   // (never with d % 4 == 0: regions and block rows start at multiples of 4)
    if (nrows > CONTIG_MAX_ROWS) return;
    u32 state[4], delta[4];
    chain_lookup(T, cc, ns, lo, hi, state, delta);
#pragma unroll
    for (u32 j = 0; j < 4; ++j) {
        if (j >= ns) continue;
        if (state[j] == 1 && (!(d.flags & TF_VEC4) || (delta[j] & 3u) == 0)) { d.flags |= TF_SRC_LDS << j; d.lds_src[j] = delta[j]; }
        else if (state[j] != 0) d.flags |= TF_GLOBAL_DEP;
    }
}

constexpr u32 PULL_MAX_ROWS = 16;

// The other rows of a pull tile must have the edges of its first row, shifted by constant strides.  Every step is a
// read that depends on the one before (row -> node -> its consumer list -> the edge records), so each step is
// taken for MAXR rows at once (rows past the tile's last repeat row 0: no read leaves the lists).
template <u32 MAXR>
__device__ inline bool pull_rows_uniform(const Tables &T, const BatchRec &r, u32 row0, u32 nrows, u32 rstride, u32 cnt,
                                         PullDesc &d)
{
    u32 qs[MAXR];
    bool same = true;
#pragma unroll
    for (u32 i = 1; i < MAXR; ++i) {
        const u32 u = T.order[r.pos0 + row0 + (i < nrows ? i : 0u) * rstride];
        qs[i] = T.succ_off[u];
        same = same && T.succ_off[u + 1] - qs[i] == cnt;
    }
    if (!same) return false;
#pragma unroll
    for (u32 j = 0; j < 4; ++j) {
        if (j >= cnt) continue;
        EdgeRec er[MAXR];
#pragma unroll
        for (u32 i = 1; i < MAXR; ++i) er[i] = T.edges[qs[i] + j];
        UEdge &f = d.e[j];
        const u32 gs = er[1].goff - f.goff, vs = er[1].voff - f.voff;
        bool ok = true;
#pragma unroll
        for (u32 i = 1; i < MAXR; ++i) {
            if (i >= nrows) continue;
            ok = ok && er[i].kind == f.kind && er[i].a0 == f.a0 && er[i].a1 == f.a1 && er[i].goff - f.goff == gs * i &&
                 er[i].voff - f.voff == vs * i;
        }
        if (!ok) return false;
        f.gs = gs; f.vs = vs;
    }
    return true;
}

__device__ inline void fill_pull_base(const Tables &T, const BatchRec &r, u32 row0, u32 nrows, u32 rstride, PullDesc &d)
{
    d.lflags = 0; d.lds_out = 0;
    d.own0 = r.val_off + row0 * r.d; d.rowstep = rstride * r.d;
    d.dshift = (r.d & (r.d - 1u)) == 0u && r.d ? (u32)__ffs(r.d) - 1u : PULL_NO_SHIFT;
    d.pos0 = r.pos0; d.B = r.B; d.d = r.d; d.val_off = r.val_off;
    d.depth = r.step; d.row0 = row0; d.nrows = nrows; d.n_uni = PULL_GENERIC; d.rstride = rstride;
#pragma unroll
    for (u32 j = 0; j < 4; ++j) { UEdge z; z.kind = 0; z.goff = z.voff = z.gs = z.vs = 0; z.a0 = z.a1 = 0; z.dl = 0; d.e[j] = z; }
    d.grp_len = 1; d.vec4 = (r.vec4 & TF_VIEW) ? 2u : 0u;   // bit 1: the batch is a view (its values lie in its operands' rows)
    if (nrows > PULL_MAX_ROWS) return;
    const u32 u0 = T.order[r.pos0 + row0];
    const u32 q0 = T.succ_off[u0];
    const u32 cnt = T.succ_off[u0 + 1] - q0;
    if (cnt > 4) return;
#pragma unroll
    for (u32 j = 0; j < 4; ++j) {
        if (j >= cnt) continue;
        const EdgeRec first = T.edges[q0 + j];
        if (first.kind == EK_NLS) return;     // the label is per-row data
        if (first.kind == EK_SQN && (r.vec4 & TF_VIEW)) return;   // needs the rows' own values, which a view keeps elsewhere
        UEdge ue; ue.kind = first.kind; ue.goff = first.goff; ue.voff = first.voff;
        ue.gs = ue.vs = 0; ue.a0 = first.a0; ue.a1 = first.a1; ue.dl = 0;
        d.e[j] = ue;
    }
    // (a tile of rows of 256 columns has four of them: sixteen rows' reads for four rows' use were most of this kernel)
    if (nrows > 4u) { if (!pull_rows_uniform<PULL_MAX_ROWS>(T, r, row0, nrows, rstride, cnt, d)) return; }
    else if (nrows > 1u) { if (!pull_rows_uniform<4>(T, r, row0, nrows, rstride, cnt, d)) return; }
    d.n_uni = cnt;
    bool vec = (r.d & 3u) == 0;
    u32 worst = 0;
#pragma unroll
    for (u32 j = 0; j < 4; ++j) {
        if (j >= cnt) continue;
        const UEdge &ue = d.e[j];
        const bool scalar_g = ue.kind == EK_SQN;                 // these read one gradient scalar per row
        if (!scalar_g && ((ue.goff | ue.gs) & 3u)) vec = false;
        if ((ue.kind == EK_MUL || ue.kind == EK_DTANH || ue.kind == EK_DSIGM) && ((ue.voff | ue.vs) & 3u)) vec = false;
        if (ue.kind == EK_RANGE && (((u32)ue.a0 | (u32)ue.a1) & 3u)) vec = false;
        worst = ue.kind > worst ? ue.kind : worst;
    }
    // (the short routine finds rows and columns by shifting: one row, or a power of two of columns)
    const bool shifts = nrows == 1u || d.dshift != PULL_NO_SHIFT;
    d.vec4 = (d.vec4 & 2u) | (vec ? 1u : 0u) | (vec && shifts && worst <= (u32)EK_DSIGM ? 4u : 0u);
}

__device__ inline void fill_pull_desc(const Tables &T, const BatchRec &r, u32 row0, u32 nrows, u32 rstride, PullDesc &d,
                                      bool in_chain, const ChainCtx &cc)
{
    fill_pull_base(T, r, row0, nrows, rstride, d);
    if (!in_chain) return;
    // tile of a fused chain: consumer gradients computed earlier in the same launch come from the
    // chain's LDS copy where the whole tile finds them in one member's region
    if (cc.cr.fused != 2u) { d.lflags = TF_GLOBAL_DEP; return; }
    d.lds_out = chain_own_delta(T, cc, r);
    d.lflags = TF_OUT_LDS;
    if (d.lds_out & 3u) d.vec4 &= ~5u;
    if (d.n_uni == PULL_GENERIC) { d.lflags |= TF_GLOBAL_DEP; return; }
    u32 lo[4], hi[4], state[4], delta[4];
#pragma unroll
    for (u32 j = 0; j < 4; ++j) {
        const u32 a = d.e[j].goff, b = d.e[j].goff + (nrows - 1) * d.e[j].gs;
        lo[j] = a < b ? a : b; hi[j] = a < b ? b : a;
    }
    chain_lookup(T, cc, d.n_uni, lo, hi, state, delta);
#pragma unroll
    for (u32 j = 0; j < 4; ++j) {
        if (j >= d.n_uni) continue;
        if (state[j] == 1 && (!(d.vec4 & 1u) || (delta[j] & 3u) == 0)) { d.lflags |= TF_SRC_LDS << j; d.e[j].dl = delta[j]; }
        else if (state[j] != 0) d.lflags |= TF_GLOBAL_DEP;
    }
}

// Tiles with uniform edges carry them resolved (see PullDesc).
__device__ inline void resolve_pull_desc(PullDesc &d)
{
    if (d.n_uni == PULL_GENERIC) return;
#pragma unroll
    for (u32 j = 0; j < 4; ++j) {
        if (j >= d.n_uni) continue;
        if (d.e[j].kind == EK_RANGE) d.e[j].goff -= (u32)d.e[j].a0;
        if (d.lflags & (TF_SRC_LDS << j)) d.e[j].goff += d.e[j].dl;
    }
}

// chain that owns global tile / work index x of list `which` (0 fwd tiles, 1 pull tiles, 2 dX tiles,
// 3 fwd works, 4 pull works): the largest c with offset(c) <= x
__device__ inline u32 clay_field(const CLay &L, int which)
{
    switch (which) { case 0: return L.tf; case 1: return L.ta; case 2: return L.tb; case 3: return L.wf; default: return L.wa; }
}
__device__ inline u32 chain_of_index(const CLay *clay_ex, u32 nc, int which, u32 x)
{
    u32 lo = 0, hi = nc;
    while (hi - lo > 1) {
        const u32 mid = (lo + hi) >> 1;
        if (clay_field(clay_ex[mid], which) <= x) lo = mid; else hi = mid;
    }
    return lo;
}

// Bound by the chains of dependent reads behind an entry.  Everything an entry is put together from stays in registers
// (151 of them, three waves a SIMD; with 400 bytes of scratch a lane it had four): 59 -> 27 us on the tagger, 200 -> 100 us
// at 512 sentences, together with reading four rows' edges where a tile has at most four rows.
__global__ __launch_bounds__(TPB) void k_tiles(Tables T, const CLay *clay_ex, const CLay *total, u32 cap_f, u32 cap_a, u32 cap_b)
{
    const u32 nc = T.hdr->n_chains;
    const u32 gtid = blockIdx.x * blockDim.x + threadIdx.x, gsz = gridDim.x * blockDim.x;
    // the five lists laid end to end, one entry per thread and pass: an entry is a chain of dependent reads
    // (chain, batch, operand rows), so a thread that took one entry of each list in turn would take five
    // times as long as the slowest entry
    u32 nts[5];
#pragma unroll
    for (int which = 0; which < 5; ++which) {
        u32 nt = clay_field(*total, which);
        const u32 cap = (which == 0 || which == 3) ? cap_f : ((which == 1 || which == 4) ? cap_a : cap_b);
        if (nt > cap) {   // cannot happen with the host's bound; never write past the lists
            if (gtid == 0) atomicOr(&T.hdr->err, (u32)ERR_OVERFLOW);
            nt = cap;
        }
        nts[which] = nt;
    }
    const u32 f1 = nts[0], f2 = f1 + nts[1], f3 = f2 + nts[2], f4 = f3 + nts[3], f5 = f4 + nts[4];
    for (u32 idx = gtid; idx < f5; idx += gsz) {
        const int which = (idx >= f1) + (idx >= f2) + (idx >= f3) + (idx >= f4);
        {
            const u32 x = idx - (which == 0 ? 0u : (which == 1 ? f1 : (which == 2 ? f2 : (which == 3 ? f3 : f4))));
            const u32 c = chain_of_index(clay_ex, nc, which, x);
            const ChainRec cr = T.chains[c];
            const u32 xx = x - clay_field(clay_ex[c], which);
            if (which >= 3) {   // work item = one block of a fused chain, or one tile
                WorkRec w;
                const bool fwd = which == 3;
                const u32 len = cr.fused ? (fwd ? cr.ktf : cr.kt) : 1u;
                w.first = (fwd ? clay_ex[c].tf : clay_ex[c].ta) + xx * len;
                w.len = len | (cr.fused == 3u ? CELL_ITEM : 0u);
                (fwd ? T.works_f : T.works_a)[x] = w;
            } else if (cr.fused == 3u) {
                const uint4 *from = nullptr;
                if (xx < cr.G) {
                    u32 cell;
                    if (which == 0 && !(T.slots[cr.slot].plain & 4u)) {     // in the order of the products' rows
                        u32 q = c - 1, row = xx;
                        for (; row >= T.chains[q].G; --q) row -= T.chains[q].G;
                        cell = T.prod_cell[T.batches[T.lorder[T.chains[q].first]].pos0 + row];
                    } else {
                        cell = T.cell_of[T.batches[cr.pad0].pos0 + xx];
                    }
                    from = (const uint4 *)&T.cells[cell];
                }
                if (which == 0) {
                    uint4 *to = (uint4 *)&T.tiles_f[x];
                    if (from) {
#pragma unroll
                        for (u32 q = 0; q < sizeof(TileDesc) / 16; ++q) to[q] = from[q];
                    } else to[0] = make_uint4(0u, 0u, 0u, 0u);
                } else {
                    uint4 *to = (uint4 *)&T.tiles_a[x];
                    if (from) {
#pragma unroll
                        for (u32 q = 0; q < sizeof(PullDesc) / 16; ++q) to[q] = from[q];
                        if (const u32 taken = ((const CellRec *)from)->taken) T.dx_cell[taken - 1u] = x + 1u;
                    } else to[0] = make_uint4(0u, 0u, 0u, 0u);
                }
            } else if (which == 2 || (which == 0 && !cr.fused)) {
                const BatchRec r = T.batches[T.lorder[cr.first]];
                TileDesc d;
                fill_tile_desc(T, r, xx, which == 2, false, 0, 0, 1, d, false, ChainCtx{});
                if (T.cells && which == 0 && r.op == OP_MATVEC && cr.slot + 1u < T.hdr->n_slots && !(T.slots[cr.slot + 1u].plain & 4u)) {
                    // where the records of the batch's cells begin: they lie batch by batch, the last chain of the slot first
                    u32 q = c + 1, before = 0;
                    for (; T.chains[q].slot == cr.slot; ++q) before += T.chains[q].G;
                    d.pad = clay_ex[q].tf + before + 1u;
                }
                (which == 0 ? T.tiles_f : T.tiles_b)[x] = d;
            } else {
                // tile `it` of block rb: member m, its q-th row of every group in the block
                // (pull tiles walk the members deepest first)
                // (forward: members that are views have no tiles and are stepped over)
                const u32 ktx = which == 0 ? cr.ktf : cr.kt;
                const u32 rb = xx / ktx;
                u32 it = xx % ktx;
                if (which == 1) it = ktx - 1 - it;
                u32 m = 0, mult = 1;
                if (cr.fused) {
                    for (;; ++m) {
                        const BatchRec &rq = T.batches[T.lorder[cr.first + m]];
                        if (which == 0 && (rq.vec4 & TF_NOFWD)) continue;
                        mult = rq.B / cr.G;
                        if (it < mult) break;
                        it -= mult;
                    }
                } else {
                    it = 0;
                }
                const BatchRec r = T.batches[T.lorder[cr.first + m]];
                const u32 g0 = rb * cr.Rg;
                const u32 ng = (g0 + cr.Rg <= cr.G) ? cr.Rg : cr.G - g0;
                const u32 row0 = g0 * mult + it;
                // tiles of the same level that follow this one in run order (this one included)
                u32 glen = 1;
                const u32 my_level = T.blevel[T.lorder[cr.first + m]];
                if (cr.fused) {
                    if (which == 0) {
                        glen = mult - it;
                        for (u32 mm = m + 1; mm < cr.k; ++mm) {
                            const BatchRec &rn = T.batches[T.lorder[cr.first + mm]];
                            if (T.blevel[T.lorder[cr.first + mm]] != my_level) break;
                            if (!(rn.vec4 & TF_NOFWD)) glen += rn.B / cr.G;
                        }
                    } else {
                        glen = it + 1;
                        for (u32 mm = m; mm-- > 0;) {
                            const BatchRec &rn = T.batches[T.lorder[cr.first + mm]];
                            if (T.blevel[T.lorder[cr.first + mm]] != my_level) break;
                            glen += rn.B / cr.G;
                        }
                    }
                }
                ChainCtx cc; cc.cr = cr; cc.m = m; cc.g0 = g0; cc.ng = ng;
                const bool in_chain = cr.fused && ktx > 1;
                if (which == 1) {
                    PullDesc d;
                    fill_pull_desc(T, r, row0, ng, mult, d, in_chain, cc);
                    resolve_pull_desc(d);
                    d.grp_len = glen;
                    T.tiles_a[x] = d;
                } else {
                    TileDesc d;
                    fill_tile_desc(T, r, xx, false, true, row0, ng, mult, d, in_chain, cc);
                    d.contig |= (glen > 0xffffu ? 0xffffu : glen) << 16;
                    T.tiles_f[x] = d;
                }
            }
        }
    }
}

// consumer-edge records in (producer, consumer, slot) order: what the producer adds to its
// gradient for this use, as one of a few plain formulas over the value / gradient arenas
__device__ inline void edges_at(const Tables &T, u32 q)
{
    if (q >= T.E) return;
    const u32 e = T.succ_edge[q];
    const u32 v = T.edge_cons[e];
    const u32 lo = T.in_off[v];
    const u32 j = e - lo;
    EdgeRec r; r.kind = EK_PLAIN; r.goff = T.nat_off[v]; r.voff = 0; r.a0 = 0; r.a1 = 0;
    switch (T.op[v]) {
    case OP_MATVEC: r.goff = T.dx_off[v]; break;
    case OP_ADD: break;
    case OP_CMULT: r.kind = EK_MUL; r.voff = T.val_off[T.in_idx[lo + (1 - j)]]; break;
    case OP_TANH: r.kind = EK_DTANH; r.voff = T.val_off[v]; break;
    case OP_SIGMOID: r.kind = EK_DSIGM; r.voff = T.val_off[v]; break;
    case OP_CONCAT: {
        u32 o = 0;
        for (u32 jj = 0; jj < j; ++jj) o += T.out_dim[T.in_idx[lo + jj]];
        r.goff += o;
        break;
    }
    case OP_SLICE: r.kind = EK_RANGE; r.a0 = T.aux0[v]; r.a1 = T.aux1[v]; break;
    case OP_PICK_NLS: r.kind = EK_NLS; r.voff = T.val_off[v]; r.a0 = T.aux0[v]; r.a1 = (i32)T.out_dim[T.in_idx[e]]; break;
    case OP_SQNORM: r.kind = EK_SQN; break;
    default: break;
    }
    T.edges[q] = r;
    // a MATVEC node's own gradient row: with one plain consumer it is that consumer's row as it is
    const u32 u = T.in_idx[e];
    if (T.op[u] == OP_MATVEC) {
        const u32 pu = T.pos_of[u];
        T.dx_gsrc[pu] = r.goff;
        if (r.kind != EK_PLAIN || (r.goff & 3u)) flags_off(T.batches[T.batch_of_pos[pu]], TF_G_ALIAS);
    }
}
__global__ void k_edges(Tables T)
{
    edges_at(T, blockIdx.x * blockDim.x + threadIdx.x);
}

// ---- parameter-use items: every MATVEC is a use of W (kind 0) and of its bias (kind 1), every
// LOOKUP a use of (table, row) (kind 2).  Sorted by (parameter, kind, row), stably from
// schedule order, they give each deferred parameter-gradient reduction a fixed summation order.
__device__ inline void item_emit_at(const Tables &T, const u32 *item_base, u64 *keys, u32 *vals, u32 p)
{
    if (p >= T.n) return;
    const u32 v = T.order[p];
    const u32 o = T.op[v];
    u32 i = item_base[p];
    if (o == OP_MATVEC) {
        keys[i] = ((u64)((u32)T.param[v] * 4u + 0u)) << 32; vals[i] = p; ++i;
        if (T.bias[v] >= 0) { keys[i] = ((u64)((u32)T.bias[v] * 4u + 1u)) << 32; vals[i] = p; }
    } else if (o == OP_LOOKUP) {
        keys[i] = (((u64)((u32)T.param[v] * 4u + 2u)) << 32) | (u32)T.aux0[v]; vals[i] = p;
    }
}
__global__ void k_item_emit(Tables T, const u32 *item_base, u64 *keys, u32 *vals)
{
    item_emit_at(T, item_base, keys, vals, blockIdx.x * blockDim.x + threadIdx.x);
}

__device__ inline void item_finish_at(const Tables &T, const u64 *keys, const u32 *vals, u32 n_items, u32 i)
{
    if (i >= n_items) return;
    const u64 k = keys[i];
    const u32 slot = (u32)(k >> 32);
    const u32 p = vals[i];
    const u32 v = T.order[p];
    T.it_key[i] = k;
    u32 gsrc = T.nat_off[v];
    T.it_goff[i] = gsrc;
    u32 xoff = 0;
    if (T.op[v] == OP_MATVEC) {
        const BatchRec &r = T.batches[T.batch_of_pos[p]];
        if (r.vec4 & TF_G_ALIAS) gsrc = T.dx_gsrc[p];
        xoff = T.val_off[T.in_idx[T.in_off[v]]];
        if (batch_xp(r)) {
            // the operand row in pieces: the row's offsets from the batch's operand list and the cuts between pieces
            xoff = XP_LIST;
            const u32 P = (u32)r.aux1, row = p - r.pos0;
            u32 o[XP_MAX], c[XP_MAX];
            u32 end = 0;
            for (u32 q = 0; q < XP_MAX; ++q) {
                o[q] = T.opnd_off[r.opnd + (q < P ? q : P - 1) * r.B + row];
                end += q < P ? T.b_indim[r.indim + q] : 0u;
                c[q] = q + 1 < P ? end : 0xffffffffu;
            }
            T.it_xrec[2 * (size_t)i] = make_uint4(o[0], o[1], o[2], o[3]);
            T.it_xrec[2 * (size_t)i + 1] = make_uint4(c[0], c[1], c[2], 0u);
        }
    }
    T.it_xoff[i] = xoff;
    T.it_gsrc[i] = gsrc;
    if (i == 0 || (u32)(keys[i - 1] >> 32) != slot) T.pu_start[slot] = i;
    if (i == n_items - 1 || (u32)(keys[i + 1] >> 32) != slot) T.pu_end[slot] = i + 1;
}
__global__ void k_item_finish(Tables T, const u64 *keys, const u32 *vals, u32 n_items)
{
    item_finish_at(T, keys, vals, n_items, blockIdx.x * blockDim.x + threadIdx.x);
}

// ---- the plan of a small graph, in one launch ---------------------------------------------------------
// Some forty launches of a few microseconds each plan a graph of a few hundred nodes: what bounds them is the launch (2.4 us
// when empty) and the first reads of whatever the launch before wrote (2 us each, out of another part of the
// chip's caches).  So up to SMALL_NODES nodes one workgroup runs the same stages one behind the other, with a
// barrier where a launch ended, its data in its own cache.  What bounds it now is the chain of dependent reads and barriers
// of its stages, 0.2 to 6 us each: in kernel traces 81 us for some 260 nodes of recurrent networks, 94 for a tree of 944 nodes
// and 133 for 1 344 of a growing graph (whole schedules, by one launch and by many, at the rule in sched_enqueue).
// Only what takes the whole chip stays a launch of its own: the tile descriptors after it.
constexpr u32 SMALL_THREADS = 1024;
constexpr u32 SMALL_NODES = 2 * SMALL_THREADS;
constexpr u32 SMALL_EDGES = 4096;               // edges and parameter uses: what the sort keeps in LDS
struct SmallArgs {
    Tables T;
    uint4 *clear;           // tables that start at zero
    u64 *keys; u32 *vals;
    u32 *succ_node, *head_flag, *s_items, *blist, *cflag, *cflag_excl;
    Tri *tri_in, *tri_ex;
    Lay *lay_in, *lay_total;
    CLay *clay_in, *clay_total;
    u32 clear_words, spin_limit, n_items, row_bits, use_bits;
    int fuse, virt;
};
// The depth of every node by one workgroup: a thread has the nodes tid, tid + SMALL_THREADS, ..., looks at two operands of each at
// a time and settles a node when its list is through.  The operand lists and the depths are in LDS, 0 = not known yet.
// A sweep of a wave is one dependent LDS read and a dozen instructions for each of its nodes, where the pass by ranges, made for four
// nodes a lane and few waves, takes some hundred: 27 -> 6 us for 252 nodes.
// A settled operand of a longer list makes room for the next, so what is known early is through before the last is, and a
// list that is long for its wave is walked by the whole wave, 512 entries at a time, whenever nothing else of the wave moves,
// by the rule of the pass by ranges.  (Two by two in list order by their threads, the schedule of a sum of 2 046 rows
// took 361 us and that of 140 steps over sums of twelve rows 534; now 116 and 295, by the launches for large graphs 169 and 380.)
// Ids are a topological order, so the lowest node that is not settled can be, and every wave comes to look at it (lists are
// walked in ascending order): the bound on idle looks only guards against damaged tables.
struct SmallDepth {
    u32 dep[SMALL_NODES + 2];                // [SMALL_ONE] holds 1: an absent operand; [SMALL_NEVER] 0: of a list that is walked
    unsigned short op[SMALL_EDGES + 2];
    u32 quit;
};
constexpr u32 SMALL_ONE = SMALL_NODES, SMALL_NEVER = SMALL_NODES + 1;
template <u32 NPT>
__device__ inline void small_depths(const Tables &T, u32 spin_limit, SmallDepth &S)
{
    const u32 tid = threadIdx.x, lane = tid & 63u, n = T.n;
    u32 at[NPT], end[NPT], top[NPT], x[NPT], y[NPT];
    bool open[NPT];
    u32 n_long = 0;
#pragma unroll
    for (u32 j = 0; j < NPT; ++j) {
        const u32 v = tid + j * SMALL_THREADS;
        open[j] = v < n;
        at[j] = open[j] ? T.in_off[v] : 0u;
        end[j] = open[j] ? T.in_off[v + 1] : 0u;
        top[j] = 0;
        S.dep[v] = 0;
        n_long += (u32)__popcll(__ballot(end[j] - at[j] > DEPTH_OPS));
    }
    for (u32 e = tid; e < T.E; e += SMALL_THREADS) S.op[e] = (unsigned short)T.in_idx[e];
    if (tid == 0) { S.dep[SMALL_ONE] = 1; S.dep[SMALL_NEVER] = 0; S.quit = 0; }
    __syncthreads();
    auto next = [&](u32 j) __attribute__((always_inline)) { return at[j] < end[j] ? (u32)S.op[at[j]++] : SMALL_ONE; };
    u64 walks[NPT];         // lanes whose node j is walked by the wave
    bool lists = false;
#pragma unroll
    for (u32 j = 0; j < NPT; ++j) {
        const u32 ar = end[j] - at[j];
        const bool walked = ar > DEPTH_OPS && ar > DEPTH_WALK * n_long;
        walks[j] = __ballot(walked);
        lists = lists || ar > 2u;
        if (ar == 0u) { if (open[j]) lds_store(&S.dep[tid + j * SMALL_THREADS], 1u); open[j] = false; }
        x[j] = y[j] = SMALL_NEVER;
        if (!walked) { x[j] = next(j); y[j] = next(j); }
    }
    u32 idle = 0, walk_e = 0, walk_max = 0;     // entries of the list being walked that are through, their largest word
    bool gave_up = false;
    auto sweeps = [&](auto with_lists) __attribute__((always_inline)) {
    while (true) {
        u32 dx[NPT], dy[NPT];
        bool moved = false, left = false;
#pragma unroll
        for (u32 j = 0; j < NPT; ++j) { dx[j] = lds_load(&S.dep[x[j]]); dy[j] = lds_load(&S.dep[y[j]]); }
#pragma unroll
        for (u32 j = 0; j < NPT; ++j) {
            const bool last = !with_lists.value || at[j] == end[j];
            if (open[j] && last && dx[j] != 0u && dy[j] != 0u) {
                const u32 d = dx[j] > dy[j] ? dx[j] : dy[j];
                top[j] = d > top[j] ? d : top[j];
                moved = true;
                open[j] = false;
                lds_store(&S.dep[tid + j * SMALL_THREADS], top[j] + 1u);
            }
            if (with_lists.value && !last) {
                if (dx[j] != 0u) { top[j] = dx[j] > top[j] ? dx[j] : top[j]; x[j] = next(j); moved = true; }
                if (dy[j] != 0u) { top[j] = dy[j] > top[j] ? dy[j] : top[j]; y[j] = next(j); moved = true; }
            }
            left = left || open[j];
        }
        if (__ballot(left) == 0ull) break;
        bool progress = __ballot(moved) != 0ull;
        if (with_lists.value && !progress) {
            u32 a = 0, ar = 0, owner = 0, node = 0;     // the wave's lowest node whose list is walked
#pragma unroll
            for (u32 j = NPT; j-- > 0;)
                if (walks[j]) {
                    owner = (u32)__builtin_ctzll(walks[j]);
                    a = (u32)__builtin_amdgcn_readlane((int)at[j], (int)owner);
                    ar = (u32)__builtin_amdgcn_readlane((int)end[j], (int)owner) - a;
                    node = (tid & ~63u) + owner + j * SMALL_THREADS;
                }
            if (ar) {
                u32 id[DEPTH_WIDE_READS], w[DEPTH_WIDE_READS];
#pragma unroll
                for (u32 q = 0; q < DEPTH_WIDE_READS; ++q) {
                    const u32 e = walk_e + 64u * q + lane;
                    id[q] = e < ar ? (u32)S.op[a + e] : SMALL_ONE;
                }
#pragma unroll
                for (u32 q = 0; q < DEPTH_WIDE_READS; ++q) w[q] = lds_load(&S.dep[id[q]]);
                bool all = true;
#pragma unroll
                for (u32 q = 0; q < DEPTH_WIDE_READS; ++q) {
                    all = all && __ballot(w[q] == 0u) == 0ull;
                    if (all) { walk_max = w[q] > walk_max ? w[q] : walk_max; walk_e += 64u; progress = true; }
                }
                if (walk_e >= ar) {
                    for (int o = 32; o > 0; o >>= 1) { const u32 t = (u32)__shfl_xor((int)walk_max, o); walk_max = t > walk_max ? t : walk_max; }
                    if (lane == 0) lds_store(&S.dep[node], walk_max + 1u);
                    bool found = false;
#pragma unroll
                    for (u32 j = 0; j < NPT; ++j) {
                        if (found || !walks[j]) continue;
                        found = true;
                        if (lane == owner) { top[j] = walk_max; open[j] = false; }
                        walks[j] &= walks[j] - 1ull;
                    }
                    walk_e = walk_max = 0;
                }
            }
        }
        if (progress) { idle = 0; continue; }
        if (++idle > spin_limit || lds_load(&S.quit) != 0u) { gave_up = true; break; }
        if (idle > 8u) __builtin_amdgcn_s_sleep(1);      // (what this wave waits for is some levels off: the others need the LDS)
    }
    };
    if (__ballot(lists) != 0ull) sweeps(std::true_type{});
    else sweeps(std::false_type{});
    u32 done = 0;
#pragma unroll
    for (u32 j = 0; j < NPT; ++j) {
        const u32 v = tid + j * SMALL_THREADS;
        // (a node that was given up on takes its own id as its step, above the step of every operand)
        if (v < n) T.step[v] = open[j] ? v : top[j];
        done += (u32)__popcll(__ballot(v < n && !open[j]));
    }
    if (lane == 0u) {
        atomicAdd(&T.hdr->frontier_done, done);
        if (gave_up) { lds_store(&S.quit, 1u); atomicOr(&T.hdr->err, (u32)ERR_CYCLE); }
    }
}

// Sort keys: the step and the smallest node id with the same step and signature, by way of a table in LDS.
// Returns the largest step.
struct SmallReps {
    u64 key[2 * SMALL_NODES];
    u32 min[2 * SMALL_NODES], top;
};
__device__ inline u32 small_reps(const Tables &T, u64 *keys, u32 *vals, SmallReps &S)
{
    constexpr u32 NPT = SMALL_NODES / SMALL_THREADS, SLOTS = 2 * SMALL_NODES;
    const u32 tid = threadIdx.x;
    for (u32 i = tid; i < SLOTS; i += SMALL_THREADS) { S.key[i] = 0; S.min[i] = ~0u; }
    if (tid == 0) S.top = 0;
    u32 at[NPT], step[NPT];
    u64 k[NPT];
#pragma unroll
    for (u32 j = 0; j < NPT; ++j) {
        const u32 v = tid + j * SMALL_THREADS;
        step[j] = v < T.n ? T.step[v] : 0u;
        k[j] = v < T.n ? batch_key(T.sig[v], step[j]) : 0;
    }
    __syncthreads();
    u32 top = 0;
#pragma unroll
    for (u32 j = 0; j < NPT; ++j) {
        const u32 v = tid + j * SMALL_THREADS;
        if (v >= T.n) continue;
        top = step[j] > top ? step[j] : top;
        for (at[j] = (u32)(k[j] >> 32) & (SLOTS - 1);; at[j] = (at[j] + 1) & (SLOTS - 1)) {   // (twice as many slots as nodes)
            const u64 cur = atomicCAS((unsigned long long *)&S.key[at[j]], 0ULL, (unsigned long long)k[j]);
            if (cur == 0 || cur == k[j]) break;
        }
        atomicMin(&S.min[at[j]], v);
    }
    atomicMax(&S.top, top);
    __syncthreads();
#pragma unroll
    for (u32 j = 0; j < NPT; ++j) {
        const u32 v = tid + j * SMALL_THREADS;
        if (v >= T.n) continue;
        keys[v] = ((u64)step[j] << 32) | S.min[at[j]];
        vals[v] = v;
    }
    top = __builtin_amdgcn_readfirstlane(S.top);
    __syncthreads();
    return top;
}

// The distinct batch dependencies, through a set in LDS that holds all of them; a thread takes an edge.
struct SmallBedges {
    u32 set[2 * SMALL_EDGES];
    u32 count;
};
__device__ inline void small_bedges(const Tables &T, u32 *blist, SmallBedges &S)
{
    const u32 tid = threadIdx.x;
    for (u32 i = tid; i < 2 * SMALL_EDGES; i += SMALL_THREADS) S.set[i] = 0;
    if (tid == 0) S.count = 0;
    __syncthreads();
    for (u32 e = tid; e < T.E; e += SMALL_THREADS) {
        const u32 p = T.pos_of[T.edge_cons[e]], b = T.batch_of_pos[p];
        const u32 key = bedge_key(T, p, b, T.batches[b], T.in_idx[e]);
        for (u32 h = (key * 2654435761u) >> 19;; h = (h + 1) & (2 * SMALL_EDGES - 1)) {     // (twice as many slots as edges)
            static_assert(2 * SMALL_EDGES == 1u << (32 - 19), "the hash gives as many bits as the set has slots");
            u32 old = lds_load(&S.set[h]);
            if (old == 0u) old = atomicCAS(&S.set[h], 0u, key);
            if (old == key) break;
            if (old == 0u) { blist[atomicAdd(&S.count, 1u)] = key; break; }
        }
    }
    __syncthreads();
    if (tid == 0) T.hdr->n_bedges = S.count;
}

union SmallLds {
    InitLds<SMALL_THREADS> init;
    RsSmall<SMALL_EDGES> sort;
    SmallDepth depth;
    SmallReps reps;
    SmallBedges small_bedges;
    SlotsLds slots;
    u32 scan_u32[SMALL_THREADS / 64];
    Tri scan_tri[SMALL_THREADS / 64];
    Lay scan_lay[SMALL_THREADS / 64];
    CLay scan_clay[SMALL_THREADS / 64];
};
static_assert(SMALL_THREADS == RS_THREADS && SMALL_THREADS == (u32)SLOT_THREADS, "one workgroup runs all stages");
static_assert(SMALL_EDGES <= BLIST_MAX && SMALL_NODES <= SLOT_MAX_NB, "a small graph has a fused plan");

__device__ inline void sort_here(SmallLds &L, u64 *keys, u32 *vals, u32 n, const RsFields &F)
{
    if (n <= 2048) rs_small<2>(L.sort, keys, vals, n, F);
    else rs_small<4>(L.sort, keys, vals, n, F);
    __syncthreads();
}
__device__ inline int bits_of(u32 x) { return x ? 32 - __builtin_clz(x) : 0; }

__global__ __launch_bounds__(SMALL_THREADS) void k_plan_small(SmallArgs)
{
    __shared__ SmallLds L;
    // The arguments are read anew in every stage: kept in scalar registers from the first stage that names one to the last,
    // most of them would be spilt.
    using Args = const SmallArgs __attribute__((address_space(4)));
    auto args = []() __attribute__((always_inline)) -> const SmallArgs & {
        Args *p = (Args *)__builtin_amdgcn_kernarg_segment_ptr();
        asm volatile("" : "+s"(p));
        return *(const SmallArgs *)p;
    };
    const u32 tid = threadIdx.x;
#define STAGE if (const SmallArgs &A = args(); true)
#define EACH(count, call)                                                        \
    STAGE {                                                                      \
        const Tables &T = A.T;                                                   \
        for (u32 i = tid; i < (u32)(count); i += SMALL_THREADS) call;            \
    }                                                                            \
    __syncthreads()
#define SCAN(kind, in, out, count, total)                                                            \
    STAGE scan_one<SMALL_THREADS, SMALL_NODES / SMALL_THREADS + 1>(in, out, (size_t)(count), total, L.kind); \
    __syncthreads()

    STAGE {
        for (u32 i = tid; i < A.clear_words; i += SMALL_THREADS) A.clear[i] = make_uint4(0u, 0u, 0u, 0u);
    }
    __syncthreads();
    // signatures, edges by producer
    STAGE {
        for (u32 base = 0; base < A.T.n; base += SMALL_THREADS) {
            node_init_part<SMALL_THREADS>(A.T, 1, A.keys, A.vals, L.init, base);
            __syncthreads();
        }
    }
    SCAN(scan_u32, A.T.outdeg, A.T.succ_off, A.T.n + 1, (u32 *)nullptr);
    STAGE sort_here(L, A.keys, A.vals, A.T.E, RsFields{{0, 0}, {bits_of(A.T.n - 1), 0}});
    EACH(T.E, succ_finish_at(T, A.vals, A.succ_node, i));
    // depth, batches
    STAGE {
        if (A.T.n <= SMALL_THREADS) small_depths<1>(A.T, A.spin_limit, L.depth);
        else small_depths<SMALL_NODES / SMALL_THREADS>(A.T, A.spin_limit, L.depth);
        __syncthreads();
    }
    STAGE {
        // (the bits above those of the largest step need no sorting)
        const u32 top = small_reps(A.T, A.keys, A.vals, L.reps);
        sort_here(L, A.keys, A.vals, A.T.n, RsFields{{0, 32}, {bits_of(A.T.n - 1), bits_of(top)}});
    }
    EACH(T.n, heads_at(T, A.keys, A.vals, A.head_flag, A.tri_in, i));
    SCAN(scan_tri, A.tri_in, A.tri_ex, A.T.n, (Tri *)nullptr);
    EACH(T.n, batch_off_at(T, A.head_flag, A.tri_ex, A.s_items, 0, i));
    EACH(T.n, batch_layout_at(T, A.lay_in, A.virt, i));
    SCAN(scan_lay, A.lay_in, A.T.lay, A.T.n, A.lay_total);
    EACH(T.n, batch_finish_at(T, T.lay, A.lay_total, i));
    EACH(T.n, node_offsets_at(T, i));
    EACH(T.n, view_offsets_at(T, i));
    EACH(T.n, member_check_at(T, i));
    EACH(T.E, opnd_at(T, i));
    EACH(T.E, edges_at(T, i));
    // launch plan
    STAGE {
        small_bedges(A.T, A.blist, L.small_bedges);
        __syncthreads();
    }
    STAGE slots_of(A.T, A.fuse, A.blist, L.slots, [&](u32 i, u32 step) __attribute__((always_inline)) {
        if (A.T.cells) find_cells<SMALL_NODES / SMALL_THREADS>(A.T, SMALL_THREADS, 0, i, step);
    });
    __syncthreads();
    EACH((T.n + SMALL_THREADS - 1) & ~(SMALL_THREADS - 1), launch_keys_at(T, A.keys, A.vals, T.n, i));   // (whole waves)
    STAGE {
        const u32 nb = A.T.hdr->n_batches;
        sort_here(L, A.keys, A.vals, nb, RsFields{{0, SLOT_BITS}, {bits_of(nb - 1), bits_of(A.T.hdr->n_slots - 1)}});
    }
    EACH(T.n + 2, chain_flags_at(T, A.vals, A.cflag, A.clay_in, T.n, i));
    SCAN(scan_u32, A.cflag, A.cflag_excl, A.T.n, (u32 *)nullptr);
    EACH(T.n, chain_recs_at(T, 0, (const u32 *)nullptr, A.cflag, A.cflag_excl, A.clay_in, T.n, i));
    SCAN(scan_clay, A.clay_in, A.T.clay, A.T.n, A.clay_total);
    EACH(T.n, slot_tables_at(T, T.clay, A.clay_total, i));
    EACH(T.n + 2, slot_fill_at(T, i));
    // parameter uses
    STAGE {
        if (A.n_items > 0) {
            for (u32 i = tid; i < A.T.n; i += SMALL_THREADS) item_emit_at(A.T, A.s_items, A.keys, A.vals, i);
            __syncthreads();
            sort_here(L, A.keys, A.vals, A.n_items, RsFields{{0, 32}, {(int)A.row_bits, (int)A.use_bits}});
            for (u32 i = tid; i < A.n_items; i += SMALL_THREADS) item_finish_at(A.T, A.keys, A.vals, A.n_items, i);
        }
    }
#undef SCAN
#undef EACH
#undef STAGE
}

// The header and the slot entries in use, written straight to page-locked host memory: one launch where two
// copies in a row (the second of the whole window, 96 KB) each had a start of their own.
constexpr int READ_BACK_THREADS = 1024;
__global__ __launch_bounds__(READ_BACK_THREADS) void k_read_back(Tables T, u32 *hdr, u32 *slots, u32 window, u32 number)
{
    const u32 i = threadIdx.x, all = READ_BACK_THREADS;
    if (i < sizeof(SchedHeader) / 4) hdr[i] = ((const u32 *)T.hdr)[i];
    const u32 used = T.hdr->n_slots + 1, count = (used < window ? used : window) * (u32)(sizeof(SlotRec) / 4);
    for (u32 k = i; k < count; k += all) slots[k] = ((const u32 *)T.slots)[k];
    pinned_release(hdr + PLAN_DONE_AT / 4, number);
}

inline int bit_width_u32(u32 x) { int b = 0; while (x) { ++b; x >>= 1; } return b; }

}  // namespace

#define K(kern, n_threads, ...)                                                                         \
    do {                                                                                                \
        if ((n_threads) > 0) {                                                                          \
            hipLaunchKernelGGL(kern, dim3(blocks_for(n_threads)), dim3(TPB), 0, s, __VA_ARGS__);        \
            ++ctx->n_launch_sched;                                                                      \
        }                                                                                               \
    } while (0)


// First half of scheduling: allocates the scheduler tables for n nodes / E edges in the arena and
// queues every stage on the schedule stream, ending with the launch that writes the header
// and the per-slot launch tables.  Does not wait.
int sched_enqueue(ob_ctx *ctx)
{
    Tables &T = ctx->T;
    hipStream_t s = ctx->sched_stream;
    const u32 n = T.n, E = T.E;
    const int manual = ctx->mode == 3;     // the caller's batches: no depth pass, no signatures to group by
    const int by_depth = ctx->mode == 1 || ctx->mode == 2;   // steps are depths (mode 1) or agenda iterations (mode 2)
    const int batched = ctx->mode != 0;
    const int agenda = ctx->mode == 2;
    ctx->n_launch_sched = 0;

    u32 n_items = ctx->n_items_total;
    if ((size_t)n != ctx->op.size()) {   // a prefix of the graph: count its parameter uses
        n_items = 0;
        for (u32 v = 0; v < n; ++v)
            n_items += ctx->op[v] == OP_MATVEC ? 1u + (ctx->bias[v] >= 0 ? 1u : 0u) : (ctx->op[v] == OP_LOOKUP ? 1u : 0u);
    }
    // pairs that are sorted: edges, nodes, parameter uses (a product with a bias is two, so there may be more of them than of either)
    const u32 most = n > E ? n : E;
    const size_t max_pairs = (size_t)(most > n_items ? most : n_items) + 1;
    const size_t n_slots = (size_t)ctx->params.size() * 4 + 4;

    const int fuse = batched && ctx->fuse;
    const bool part_depth = by_depth && ctx->max_arity < DEPTH_MAX_ARITY && !ctx->force_frontier;
    ctx->depth_partitioned = part_depth;
    // One workgroup plans a graph of up to 2 048 nodes.  Schedules of one launch and of many, in us: recurrences of 48, 473
    // and 1 617 nodes 92 and 142, 111 and 167, 147 and 187; a tagger's 461, 921 and 1 841 nodes 149 and 257, 165 and 221,
    // 216 and 240; trees of 1 214 and 2 033 nodes 189 and 223, 217 and 231; a sum of 2 046 rows 116 and 169; a chain of 500
    // operations 1 255 and 1 300, of 2 000 5 460 and 5 410: the two meet where the rule ends.
    const bool small = fuse && E > 0 && !agenda && part_depth && !ctx->wide_plan && n <= SMALL_NODES &&
                       E <= SMALL_EDGES && n_items <= SMALL_EDGES;

    // ---- allocation (all from the caller's arena) ----
    u32 ht_size = 1;
    while (ht_size < 2 * n) ht_size <<= 1;
    if (!by_depth) ht_size = 1;
    // upper bounds of the three tile lists from sums the host keeps while nodes are added
    // (a node contributes at most one component-wise / reduction tile; MATVEC nodes their GEMM tiles)
    const size_t cap_f = (size_t)n + (size_t)ctx->sum_mv_d32 + 16;
    const size_t cap_a = (size_t)n + 16;
    const size_t cap_b = (size_t)ctx->sum_mv_k32 + 16;
#define A(field, type, count)                                               \
    do {                                                                    \
        field = arena_array<type>(ctx, (count));                            \
        if (!field) return ctx_fail(ctx, -5, "arena too small for scheduler tables (%s)", #field); \
    } while (0)
    // Tables that must start at zero lie next to each other, those that start as all ones behind them: k_clear sets
    // both in one launch.
    u32 *g_dep;
    u32 *bset, *blist;
    AgendaTables AG{};
    char *zero_lo = (char *)ctx->arena + ctx->top;
    A(T.hdr, SchedHeader, 1);
    A(T.outdeg, u32, n + 1); A(T.qcount, u32, 64);
    A(T.pu_start, u32, n_slots); A(T.pu_end, u32, n_slots);
    char *small_hi = (char *)ctx->arena + ctx->top;     // (the plan of a small graph keeps the others in LDS)
    A(g_dep, u32, n + 1); A(T.ht_keys, u64, ht_size); A(bset, u32, BSET_SIZE);
    if (agenda) { A(AG.keys, u64, AG_TABLE); A(AG.sum, u64, AG_TABLE); A(AG.cnt, u32, AG_TABLE); }
    char *zero_hi = (char *)ctx->arena + ctx->top;
    A(T.ht_vals, u32, ht_size);
    if (agenda) A(AG.first, u32, AG_TABLE);
    char *ones_hi = (char *)ctx->arena + ctx->top;
    A(T.sig, u64, n); A(T.step, u32, n); A(T.indeg, u32, n);
    A(T.succ_off, u32, n + 1); A(T.succ_edge, u32, E + 1); A(T.edge_cons, u32, E + 1);
    A(T.queue, u32, n);
    A(T.ht_slot, u32, n);
    T.ht_mask = ht_size - 1;
    T.slot_dx = T.queue;            // (one depth pass and the agenda list nodes there; both are done when batches have their place)
    T.dx_cell = T.indeg;            // (plans with cells are fused ones, and those of them that count operands down do so before they look for cells)
    A(T.order, u32, n); A(T.pos_of, u32, n); A(T.batch_of_pos, u32, n); A(T.s_aux0, u32, n);
    A(T.s_in_off, u32, n + 1);
    A(T.batch_off, u32, n + 1); A(T.batches, BatchRec, n); A(T.lay, Lay, n); A(T.b_indim, u32, E + (size_t)XP_MAX * n + 1);
    A(T.val_off, u32, n); A(T.nat_off, u32, n); A(T.dx_off, u32, n); A(T.opnd_off, u32, E + (size_t)XP_MAX * n + 1); A(T.dx_gsrc, u32, n);
    A(T.slot_of, u32, n); A(T.label_of, u32, n); A(T.blevel, u32, n);
    A(T.chain_of_batch, u32, n);
    A(T.lorder, u32, n); A(T.chains, ChainRec, n); A(T.clay, CLay, n); A(T.chain_of_lpos, u32, n);
    // a plan has at most one slot per node; twice that leaves room for plans that insert slots
    const size_t slot_cap = 2 * (size_t)n + 4;
    A(T.slots, SlotRec, slot_cap);
    A(T.works_f, WorkRec, cap_f); A(T.works_a, WorkRec, cap_a);
    A(T.tiles_f, TileDesc, cap_f); A(T.tiles_a, PullDesc, cap_a); A(T.tiles_b, TileDesc, cap_b);
    A(T.root_pos, u32, 64);
    A(T.edges, EdgeRec, E + 1);
    A(T.it_key, u64, n_items + 1); A(T.it_gsrc, u32, n_items + 1); A(T.it_goff, u32, n_items + 1);
    A(T.it_xoff, u32, n_items + 1);
    T.it_xrec = nullptr;
    if (ctx->concat_views && ctx->n_concat > 0) A(T.it_xrec, uint4, 2 * ((size_t)n_items + 1));
    // What only the plan itself needs lies behind everything else, and sched_finish puts values and gradients in its place.
    ctx->plan_top = ctx->top;
    u32 *succ_node;
    A(succ_node, u32, E + 1);
    A(ctx->key_a, u64, max_pairs); A(ctx->key_b, u64, max_pairs); A(ctx->val_a, u32, max_pairs); A(ctx->val_b, u32, max_pairs);
    A(ctx->tmp_u32_a, u32, n + 1); A(ctx->tmp_u32_b, u32, n + 1);
    u32 *tmp_d;
    A(tmp_d, u32, n + 1);
    Tri *tri_in, *tri_ex;
    A(tri_in, Tri, n); A(tri_ex, Tri, n);
    A(ctx->lay_in, Lay, n); A(ctx->lay_total, Lay, 1);
    CLay *clay_in, *clay_total;
    A(clay_in, CLay, n); A(clay_total, CLay, 1);
    A(blist, u32, BLIST_MAX);
    if (agenda) {
        A(AG.op, u32, AG_TABLE); A(AG.rank_of, u32, AG_TABLE); A(AG.seg_off, u32, AG_MAX_CLASSES + 1);
        A(AG.n_classes, u32, 64);
        AG.cls = ctx->tmp_u32_a; AG.pending = ctx->tmp_u32_b; AG.seg = T.queue;
    }
    {
        size_t sb = prim_sort_scratch_bytes(max_pairs);
        size_t sc = prim_scan_scratch_bytes(max_pairs, sizeof(Lay));
        ctx->scratch = arena_alloc(ctx, sb > sc ? sb : sc);
        if (!ctx->scratch) return ctx_fail(ctx, -5, "arena too small for scheduler scratch");
    }
#undef A
    // A fused plan of a graph with slices may hold gated cells.  Where there is no room for their tables it holds none: its
    // values and gradients are the same, and an arena that is large enough for the plan stays large enough.
    T.cells = nullptr;
    if (fuse && ctx->n_slice > 0) {
        const size_t before = ctx->top;
        T.cells_cap = n / 8 + 1;        // (a cell holds more than eight nodes)
        bool room = true;
        auto table = [&](auto *&field, size_t count) {
            field = arena_array<std::remove_reference_t<decltype(*field)>>(ctx, count);
            room = room && field;
        };
        table(T.nrec, n); table(T.cell_nodes_of, T.cells_cap); table(T.cell_of, n); table(T.prod_cell, n);
        table(T.cell_ends, n); table(T.cell_ends_n, blocks_for(n));
        table(T.cell_rows, n); table(T.cell_nodes, n); table(T.cell_prods, n); table(T.cell_takes, n); table(T.slot_cells, n);
        table(T.slot_chains, n); table(T.slot_rows, n);
        table(T.cells, T.cells_cap);
        if (!room) { T.cells = nullptr; ctx->top = before; }
    }
    ctx->plan_end = ctx->top;

    // ---- stage 1 ----
    if (!small) {   // (sections of the arena start at multiples of 256 bytes)
        const size_t words = (size_t)(ones_hi - zero_lo) / 16, zeros = (size_t)(zero_hi - zero_lo) / 16;
        const size_t bx = (words + 4 * TPB - 1) / (4 * TPB);
        hipLaunchKernelGGL(k_clear, dim3((unsigned)(bx < 2048 ? bx : 2048)), dim3(TPB), 0, s, (uint4 *)zero_lo, zeros, words);
        ++ctx->n_launch_sched;
    }
    u32 *head_flag = ctx->tmp_u32_a, *s_items = tmp_d, *cflag = ctx->tmp_u32_a, *cflag_excl = ctx->tmp_u32_b;
    const int virt = ctx->concat_views && ctx->n_concat > 0;   // CONCAT batches that only products read stay uncopied
    if (small) {
        SmallArgs a{T, (uint4 *)zero_lo, ctx->key_a, ctx->val_a, succ_node, head_flag, s_items, blist, cflag, cflag_excl, tri_in, tri_ex,
                    ctx->lay_in, ctx->lay_total, clay_in, clay_total, (u32)((small_hi - zero_lo) / 16), ctx->depth_spin_limit, n_items,
                    (u32)bit_width_u32((u32)ctx->max_param_rows), (u32)bit_width_u32((u32)n_slots), ctx->fuse, virt};
        hipLaunchKernelGGL(k_plan_small, dim3(1), dim3(SMALL_THREADS), 0, s, a);
        ++ctx->n_launch_sched;
    } else {
        K(k_node_init, n, T, manual ? 2 : (by_depth ? (part_depth ? 1 : 3) : 0), ctx->key_a, ctx->val_a);
        HIP_TRY(ctx, prim_scan_u32(T.outdeg, T.succ_off, (size_t)n + 1, nullptr, ctx->scratch, s));
        // a scan of a short array is one launch, up to 256 blocks of 1024 elements two, beyond that three
        const int scan_launches = (size_t)n + 1 <= 4096 ? 1 : ((size_t)n + 1 <= 256 * 1024 ? 2 : 3);
        ctx->n_launch_sched += scan_launches;
        if (E > 0) {
            HIP_TRY(ctx, prim_sort_pairs_swap(ctx->key_a, ctx->val_a, ctx->key_b, ctx->val_b, E, 0,
                                         bit_width_u32(n - 1), 0, 0, ctx->scratch, s, &ctx->n_launch_sched));
            K(k_succ_finish, E, T, ctx->val_a, succ_node);
        }

        // ---- stage 2 / 3 ----
        if (by_depth) {
            if (part_depth)
                hipLaunchKernelGGL(k_depth_partitioned, dim3(blocks_for(n, DEPTH_PART)), dim3(DEPTH_THREADS), 0, s, T, g_dep,
                                   ctx->depth_spin_limit);
            else
                hipLaunchKernelGGL(k_depth_frontier, dim3(1), dim3(FRONTIER_THREADS), 0, s, T, succ_node);
            ++ctx->n_launch_sched;
            if (agenda) {   // steps become agenda iterations; T.step holds the depths until k_agenda rewrites it
                K(k_class_insert, n, T, AG);
                hipLaunchKernelGGL(k_class_rank, dim3(1), dim3(1024), 0, s, T, AG);
                K(k_class_of, n, T, AG);
                if (n <= AG_LDS_NODES && E > 0) {
                    // (the sort's buffers and the scans' counts are not in use yet)
                    AG.edge_to = (uint2 *)ctx->key_a; AG.ready = (uint2 *)tri_in;
                    K(k_agenda_edges, E, T, AG, succ_node);
                    hipLaunchKernelGGL(k_agenda_lds, dim3(1), dim3(AG_LDS_THREADS), 0, s, T, AG);
                } else {
                    hipLaunchKernelGGL(k_agenda, dim3(1), dim3(AGENDA_THREADS), 0, s, T, AG, succ_node);
                }
                ctx->n_launch_sched += 2;
            }
            hipLaunchKernelGGL(k_rep_insert, dim3(blocks_for(n, REP_THREADS)), dim3(REP_THREADS), 0, s, T);
            ++ctx->n_launch_sched;
        }
        K(k_sort_keys, n, T, ctx->key_a, ctx->val_a, manual ? 2 : by_depth);
        if (manual) {
            HIP_TRY(ctx, prim_sort_pairs_swap(ctx->key_a, ctx->val_a, ctx->key_b, ctx->val_b, n, 32, bit_width_u32(ctx->manual_max | 1u),
                                         0, 0, ctx->scratch, s, &ctx->n_launch_sched));
        } else if (by_depth) {
            const int lb = bit_width_u32(n - 1);
            HIP_TRY(ctx, prim_sort_pairs_swap(ctx->key_a, ctx->val_a, ctx->key_b, ctx->val_b, n, 0, lb, 32, lb,
                                         ctx->scratch, s, &ctx->n_launch_sched));
        }

        // ---- stage 4 ----
        K(k_heads, n, T, ctx->key_a, ctx->val_a, head_flag, tri_in);
        HIP_TRY(ctx, prim_scan_tri(tri_in, tri_ex, n, nullptr, ctx->scratch, s));
        ctx->n_launch_sched += scan_launches;
        K(k_batch_off, n, T, head_flag, tri_ex, s_items, manual);
        K(k_batch_layout, n, T, ctx->lay_in, virt);
        HIP_TRY(ctx, prim_scan_lay(ctx->lay_in, T.lay, n, ctx->lay_total, ctx->scratch, s));
        ctx->n_launch_sched += scan_launches;
        K(k_batch_finish, n, T, T.lay, ctx->lay_total);
        K(k_node_offsets, n, T);
        K(k_view_offsets, n, T);
        K(k_member_check, n, T);
        if (E > 0) K(k_opnd, E, T);
        if (E > 0) K(k_edges, E, T);

        // ---- launch planning: slots, chains, tile descriptors ----
        if (fuse && E > 0) K(k_bedges, n, T, bset, blist);
        hipLaunchKernelGGL(k_slots, dim3(T.cells ? 1 + blocks_for(n, TPB * CELL_PARTS) : 1), dim3(SLOT_THREADS), 0, s, T, (fuse && E > 0) ? ctx->fuse : 0, blist);
        ++ctx->n_launch_sched;
        K(k_launch_keys, n, T, ctx->key_a, ctx->val_a, n);
        if (fuse && E > 0) {
            const size_t n_sort = n < SLOT_MAX_NB + 1 ? n : SLOT_MAX_NB + 1;
            // entries from n_batches on carry the largest key and stay where they are
            HIP_TRY(ctx, prim_sort_pairs_swap(ctx->key_a, ctx->val_a, ctx->key_b, ctx->val_b, n_sort, 0, 2 * SLOT_BITS,
                                         0, 0, ctx->scratch, s, &ctx->n_launch_sched, &T.hdr->n_batches));
        }
        K(k_chain_flags, (size_t)n + 2, T, ctx->val_a, cflag, clay_in, n);
        HIP_TRY(ctx, prim_scan_u32(cflag, cflag_excl, n, nullptr, ctx->scratch, s));
        K(k_chain_recs, n, T, agenda || manual, bset, cflag, cflag_excl, clay_in, n);
        HIP_TRY(ctx, prim_scan_clay(clay_in, T.clay, n, clay_total, ctx->scratch, s));
        ctx->n_launch_sched += 2 * scan_launches;
        K(k_slot_tables, n, T, T.clay, clay_total);
        if (fuse) K(k_slot_fill, (size_t)n + 2, T);
        if (n_items > 0) {
            K(k_item_emit, n, T, s_items, ctx->key_a, ctx->val_a);
            HIP_TRY(ctx, prim_sort_pairs_swap(ctx->key_a, ctx->val_a, ctx->key_b, ctx->val_b, n_items, 0,
                                         bit_width_u32((u32)ctx->max_param_rows), 32, bit_width_u32((u32)n_slots), ctx->scratch, s,
                                         &ctx->n_launch_sched));
            K(k_item_finish, n_items, T, ctx->key_a, ctx->val_a, n_items);
        }
    }
    hipLaunchKernelGGL(k_tiles, dim3(1024), dim3(TPB), 0, s, T, T.clay, clay_total, (u32)cap_f, (u32)cap_a,
                       (u32)cap_b);
    ++ctx->n_launch_sched;
    HIP_TRY(ctx, hipGetLastError());

    // ---- the header and a first window of the per-slot tables go to the host ----
    // pinned layout: [header 256 B][first hdr_window entries of the slot table]
    ctx->hdr_window = (u32)(slot_cap < SLOT_WINDOW ? slot_cap : SLOT_WINDOW);
    char *hp = (char *)ctx->hdr_pinned;
    hipLaunchKernelGGL(k_read_back, dim3(1), dim3(READ_BACK_THREADS), 0, s, T, (u32 *)hp, (u32 *)(hp + 256), ctx->hdr_window, ++ctx->plan_number);
    HIP_TRY(ctx, hipGetLastError());
    ++ctx->n_launch_sched;
    ctx->n_items_sched = n_items;
    return 0;
}

// Second half of scheduling: waits for the queued work, checks the error flags, takes the
// per-slot launch tables and carves the value and gradient arenas.
int sched_finish(ob_ctx *ctx)
{
    Tables &T = ctx->T;
    hipStream_t s = ctx->sched_stream;
    // wait for this context's own scheduling work only (its event was recorded behind the launch
    // that writes the header): other contexts may already have queued theirs on the same stream
    // (scheduled on a stream of its own, the plan is waited for by the runtime: of an event that the runtime has not seen end, the wait of
    // the execution stream becomes a dependency between two queues; loops of four minibatches of two and eight chains 715 -> 703,
    // 906 -> 898 us, tagged sentences by fours 1 765 -> 1 754)
    const char *hp = (const char *)ctx->hdr_pinned;
    if (s != ctx->stream || !pinned_done((const u32 *)(hp + PLAN_DONE_AT), ctx->plan_number)) HIP_TRY(ctx, hipEventSynchronize(ctx->ev[9]));
    ctx->hdr = *(const SchedHeader *)hp;
    if ((ctx->hdr.err & ERR_CYCLE) && ctx->depth_partitioned) {
        // A range of the partitioned depth pass ran into the bound on its wait for another range.
        // Node ids are a topological order (checked when nodes are added), so the graph has no
        // cycle: schedule once more with the single-workgroup pass, which waits for nothing.
        ++ctx->n_depth_retries;
        ctx->force_frontier = true;
        ctx->top = ctx->graph_top;
        int rc = sched_enqueue(ctx);
        ctx->force_frontier = false;
        if (rc) return rc;
        HIP_TRY(ctx, hipEventRecord(ctx->ev[9], s));
        HIP_TRY(ctx, hipEventSynchronize(ctx->ev[9]));
        hp = (const char *)ctx->hdr_pinned;
        ctx->hdr = *(const SchedHeader *)hp;
    }
    ctx->hdr.n_items = ctx->n_items_sched;
    if (ctx->hdr.err & ERR_CYCLE)
        return ctx_fail(ctx, -6, "%s resolved %u of %u nodes: the graph on the device is cyclic or damaged",
                        ctx->mode == 2 ? "the single-workgroup depth pass / the agenda" : "the single-workgroup depth pass",
                        ctx->hdr.frontier_done, T.n);
    if (ctx->hdr.err & ERR_COLLISION) return ctx_fail(ctx, -6, "signature hash collision detected");
    if (ctx->hdr.err & ERR_TABLE_FULL) return ctx_fail(ctx, -6, "signature table full");
    if (ctx->hdr.err & ERR_OVERFLOW) return ctx_fail(ctx, -5, "value arena exceeds 2^32 elements");
    if (ctx->hdr.err & ERR_CLASSES) return ctx_fail(ctx, -6, "more than 1024 distinct signatures (or a node with more than 4 million operands): agenda-based batching cannot handle the graph");
    const size_t words = (size_t)ctx->hdr.n_slots + 1;
    if (words <= ctx->hdr_window) {
        const SlotRec *sr = (const SlotRec *)(hp + 256);
        ctx->slots.assign(sr, sr + words);
    } else {   // more launch slots than the window (unbatched mode): a plain copy
        ctx->slots.resize(words);
        HIP_TRY(ctx, hipMemcpyAsync(ctx->slots.data(), T.slots, words * sizeof(SlotRec), hipMemcpyDeviceToHost, s));
        HIP_TRY(ctx, hipStreamSynchronize(s));
    }

    // ---- value and gradient arenas ----
    ctx->top = ctx->plan_top;      // (the plan is made and read)
    T.V = arena_array<float>(ctx, ctx->hdr.val_floats + VAL_ALIGN);
    T.G = arena_array<float>(ctx, ctx->hdr.grad_floats + VAL_ALIGN);
    if (!T.V || !T.G)
        return ctx_fail(ctx, -5, "arena too small: values need %llu floats, gradients %llu",
                        (unsigned long long)ctx->hdr.val_floats, (unsigned long long)ctx->hdr.grad_floats);
    return 0;
}
