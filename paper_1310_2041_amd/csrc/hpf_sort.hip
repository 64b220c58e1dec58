// Canonical cell-list order of the beads (the paper reorders particle data for
// cache hits and bins beads into a cell list, Algorithm 1 Kernel 1).
//
// The key of a bead is the brick of B^3 cells holding its cell (one more key
// for beads that cannot be binned); the order is ascending (key, tag), where
// the tags are a permutation of [0, N) (the beads' original indices). Inside
// a brick the beads of a chain (consecutive tags) then stay neighbours, so
// most bond partners are adjacent in memory. The order is produced by a
// stable counting sort of the beads taken in tag order, so beads of one key
// come out in tag order with no sorting inside a key:
//   1. in storage order: by_tag[tag[i]] = (the key of bead i, i);
//   2. the tag sequence is cut into chunks of S tags; per chunk a key
//      histogram is counted in LDS and stored as one row of a chunk x key
//      table;
//   3. a column-wise exclusive scan of that table, taken in key-major order,
//      gives every (chunk, key) pair its first output slot, and the key
//      starts (cell_start);
//   4. per chunk the beads are placed in tag order: each wavefront takes a
//      contiguous part of the chunk with its own row of running slots, and its
//      lanes that share a key take consecutive slots;
//   5. the permutation's inverse, in storage order.
// No step needs a global atomic, and the result does not depend on the input
// order. Finally one pass gathers the bead arrays and the renumbered bond table
// into the output buffers.
#include <algorithm>
#include <type_traits>

#include "hpf_common.hpp"

namespace hpf {

struct SortK {
    MeshK m;
    int32_t B;
    int32_t nb[3];
    uint32_t NK;        // number of bricks; key NK = "cannot be binned"
};

constexpr int kSortThreads = 256;
constexpr int kScanThreads = 1024;
constexpr int kChunkThreads = 256;                    // histogram workgroups
constexpr uint32_t kRangeKeys = 2048;                 // keys above which a chunk's key range is looked up
constexpr int kPlaceRows = 16;                        // 64-tag rows a placing wavefront loads at once
constexpr int kKeyUnroll = 4;                         // keys a placing thread reads at once
constexpr int64_t kMinChunk = 4096;
constexpr int64_t kSmallChunk = kChunkThreads * 4;                    // 1024 tags
constexpr int64_t kChunksWanted = 2048;     // chunks that keep the histogram and placement passes busy
constexpr int kColBlock = 64;                         // chunks per column-scan block
constexpr int64_t kMaxSortKeys = 36864;               // one chunk's histogram in LDS (144 KiB)
constexpr int64_t kMaxTable = 64LL << 20;             // chunk x key table entries
constexpr uint32_t kNoKey = 0xffffffffu;              // a tag that names no bead

__global__ __launch_bounds__(kSortThreads) void k_fill_u32(uint32_t* __restrict__ p, int64_t n, uint32_t v)
{
    for (int64_t i = (int64_t)blockIdx.x * kSortThreads + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * kSortThreads)
        p[i] = v;
}

// ------------------------------------------------------------ scan (u32) --

// A broken permutation leaves beads out, which the placement gives no slot, and as many slots
// at the end: perm and inv are -1 there, so that no output depends on what the workspace held.
// (By one workgroup, the first to know: slow, but free where nothing is broken.)
__device__ __forceinline__ void clear_if_broken(uint32_t placed, int64_t N, int32_t* __restrict__ perm,
                                                int32_t* __restrict__ inv)
{
    if (placed < N)
        for (int64_t i = threadIdx.x; i < N; i += kScanThreads) {
            inv[i] = -1;
            if (i >= placed)
                perm[i] = -1;
        }
}

// In-place exclusive scan of a[0, n) by one workgroup; a[n] receives the total. n is at
// most kMaxSortKeys, so one workgroup reads at most 36 entries per thread, and a single
// launch replaces three (tiles, tops, add), each of which cost its ~4 us start.
__global__ __launch_bounds__(kScanThreads) void k_scan_keys(uint32_t* __restrict__ a, uint32_t n, int64_t N,
                                                            int32_t* __restrict__ perm, int32_t* __restrict__ inv)
{
    __shared__ uint32_t sh[kScanThreads / kWave + 1];
    uint32_t run = 0;
    for (uint32_t k0 = 0; k0 < n; k0 += kScanThreads) {
        const uint32_t k = k0 + threadIdx.x;
        const uint32_t v = k < n ? a[k] : 0u;
        uint32_t total;
        const uint32_t r = block_excl_scan<kScanThreads>(v, sh, &total);
        if (k < n)
            a[k] = run + r;
        run += total;
    }
    if (threadIdx.x == 0)
        a[n] = run;
    clear_if_broken(run, N, perm, inv);
}

// ------------------------------------------------------------------ keys --

// Sort key of bead i, at position r, of one system.
struct CellKeyer {
    SortK sk;
    const float3* R;
    __device__ __forceinline__ uint32_t operator()(int32_t, const float3& r) const
    {
        BeadCell b;
        return bead_cell(r, sk.m, b) ? brick_of(b.c[0], b.c[1], b.c[2], sk.B, sk.nb) : sk.NK;
    }
};

// ------------------------------------------ 1. tag -> index, and the keys --

// In storage order (coalesced reads of the positions): by_tag[tag] = key << 32 | i. Tags that a
// broken permutation leaves out keep the fill (all ones), whose key is kNoKey. Bound by the
// scattered stores, one of 8 bytes a bead: 3M beads, mostly solvent, 49 us, 10M chain beads 74
// (as two of 4 bytes, index and key apart, 94 and 79).
template <class Keyer>
__global__ __launch_bounds__(kSortThreads) void k_tag_index(Keyer keyer, const int32_t* __restrict__ tag,
                                                            int64_t N, unsigned long long* __restrict__ by_tag)
{
    const int64_t i = xcd_block(blockIdx.x, gridDim.x) * kSortThreads + threadIdx.x;
    if (i >= N)
        return;
    const int32_t t = tag ? tag[i] : (int32_t)i;
    if (t < 0 || t >= N)
        raise_flag(HPF_FLAG_SORT_ORDER);
    else
        by_tag[t] = (unsigned long long)keyer((int32_t)i, keyer.R[i]) << 32 | (unsigned long long)(uint32_t)i;
}

__global__ __launch_bounds__(kSortThreads) void k_fill_u64(unsigned long long* __restrict__ p, int64_t n,
                                                           unsigned long long v)
{
    for (int64_t i = (int64_t)blockIdx.x * kSortThreads + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * kSortThreads)
        p[i] = v;
}

// ------------------------------------------------------ 2. chunk histograms --

// Adds one per lane with a key to slot[key]: equal keys of consecutive tags come in runs
// (chain neighbours), and each run is one LDS add.
__device__ __forceinline__ void count_runs(uint32_t* slot, uint32_t key)
{
    const int lane = threadIdx.x & (kWave - 1);
    const uint32_t before = __shfl_up(key, 1, kWave);
    const uint64_t heads = __ballot(lane == 0 || before != key);
    if (((heads >> lane) & 1ull) && key != kNoKey) {
        const uint64_t after = lane == kWave - 1 ? 0ull : heads >> (lane + 1);
        atomicAdd(slot + key, after ? (uint32_t)__builtin_ctzll(after) + 1u : (uint32_t)(kWave - lane));
    }
}

__global__ __launch_bounds__(kChunkThreads) void k_sort_hist(const unsigned long long* __restrict__ by_tag,
                                                             int64_t N, int64_t S, uint32_t nkeys,
                                                             uint32_t* __restrict__ table)
{
    extern __shared__ uint32_t hist[];
    const int64_t c = blockIdx.x;
    for (uint32_t k = threadIdx.x; k < nkeys; k += kChunkThreads)
        hist[k] = 0u;
    __syncthreads();
    const int64_t t0 = c * S, t1 = min(N, t0 + S);
    bool missing = false;
    for (int64_t base = t0; base < t1; base += kChunkThreads) {
        const int64_t t = base + threadIdx.x;
        uint32_t key = kNoKey;
        if (t < t1) {
            key = (uint32_t)(by_tag[t] >> 32);
            missing |= key == kNoKey;
        }
        count_runs(hist, key);
    }
    if (missing)
        raise_flag(HPF_FLAG_SORT_ORDER);
    __syncthreads();
    uint32_t* row = table + c * (int64_t)nkeys;
    for (uint32_t k = threadIdx.x; k < nkeys; k += kChunkThreads)
        row[k] = hist[k];
}

// ------------------------------------------------ 3. column-wise scan --

// The loops below read kColUnroll rows at once: one row after the other each waited out a
// memory latency (64 rows took 17 us whatever the number of keys).
constexpr int kColUnroll = 16;

// part[cb][k] = sum of table[c][k] over the chunks c of column block cb
__global__ __launch_bounds__(kSortThreads) void k_col_partial(const uint32_t* __restrict__ table, int64_t nchunks,
                                                              uint32_t nkeys, uint32_t* __restrict__ part)
{
    const uint32_t k = blockIdx.x * kSortThreads + threadIdx.x;
    if (k >= nkeys)
        return;
    const int64_t c0 = (int64_t)blockIdx.y * kColBlock, c1 = min(nchunks, c0 + kColBlock);
    uint32_t s = 0;
    for (int64_t c = c0; c < c1; c += kColUnroll) {
        uint32_t v[kColUnroll];
#pragma unroll
        for (int j = 0; j < kColUnroll; ++j)
            v[j] = c + j < c1 ? table[(c + j) * nkeys + k] : 0u;
#pragma unroll
        for (int j = 0; j < kColUnroll; ++j)
            s += v[j];
    }
    part[(int64_t)blockIdx.y * nkeys + k] = s;
}

// a[r][k] -> run + the sum of the rows before r, r in [r0, r1); returns the run after r1
__device__ __forceinline__ uint32_t col_scan(uint32_t* __restrict__ a, int64_t r0, int64_t r1, uint32_t nkeys,
                                             uint32_t k, uint32_t run)
{
    for (int64_t r = r0; r < r1; r += kColUnroll) {
        uint32_t v[kColUnroll];
#pragma unroll
        for (int j = 0; j < kColUnroll; ++j)
            v[j] = r + j < r1 ? a[(r + j) * nkeys + k] : 0u;
#pragma unroll
        for (int j = 0; j < kColUnroll; ++j) {
            if (r + j < r1)
                a[(r + j) * nkeys + k] = run;
            run += v[j];
        }
    }
    return run;
}

// part[cb][k] -> exclusive prefix over cb; tot[k] = key total
__global__ __launch_bounds__(kSortThreads) void k_col_prefix(uint32_t* __restrict__ part, int64_t ncb,
                                                             uint32_t nkeys, uint32_t* __restrict__ tot)
{
    const uint32_t k = blockIdx.x * kSortThreads + threadIdx.x;
    if (k < nkeys)
        tot[k] = col_scan(part, 0, ncb, nkeys, k, 0u);
}

// table[c][k] -> first output slot of chunk c's beads with key k
__global__ __launch_bounds__(kSortThreads) void k_col_apply(uint32_t* __restrict__ table,
                                                            const uint32_t* __restrict__ part,
                                                            const uint32_t* __restrict__ start, int64_t nchunks,
                                                            uint32_t nkeys)
{
    const uint32_t k = blockIdx.x * kSortThreads + threadIdx.x;
    if (k >= nkeys)
        return;
    const int64_t c0 = (int64_t)blockIdx.y * kColBlock, c1 = min(nchunks, c0 + kColBlock);
    col_scan(table, c0, c1, nkeys, k, start[k] + part[(int64_t)blockIdx.y * nkeys + k]);
}

// Step 3 for few chunks (one column block) in one workgroup and one launch: key totals,
// their scan (start, with the total in start[nkeys]) and the slots. Below 64 chunks (65,000
// beads) the four launches it replaces are nothing but their start-up times.
constexpr uint32_t kSmallKeys = 4096;

__global__ __launch_bounds__(kScanThreads) void k_col_small(uint32_t* __restrict__ table, int64_t nchunks,
                                                            uint32_t nkeys, uint32_t* __restrict__ start,
                                                            int64_t N, int32_t* __restrict__ perm,
                                                            int32_t* __restrict__ inv)
{
    __shared__ uint32_t sh[kScanThreads / kWave + 1];
    uint32_t base = 0;
    for (uint32_t k0 = 0; k0 < nkeys; k0 += kScanThreads) {
        const uint32_t k = k0 + threadIdx.x;
        uint32_t tot = 0;
        if (k < nkeys)
            tot = col_scan(table, 0, nchunks, nkeys, k, 0u);
        uint32_t total;
        const uint32_t first = base + block_excl_scan<kScanThreads>(tot, sh, &total);
        if (k < nkeys) {
            start[k] = first;
            for (int64_t c = 0; c < nchunks; ++c)
                table[c * nkeys + k] += first;
        }
        base += total;
    }
    if (threadIdx.x == 0)
        start[nkeys] = base;
    clear_if_broken(base, N, perm, inv);
}

// ------------------------------------------------------ 4. placement --

// Active lanes that hold this lane's key (0 for an inactive lane): up to `rounds` distinct keys
// one after the other, then, if lanes are left, one ballot per key bit, whatever the number of
// keys. The rounds pay where a wavefront holds a few keys: at 20,000 beads a key (10M beads in
// 16-cell bricks) the placement takes 70 us with six rounds and 105 us without; at 2000
// (8-cell bricks, a dozen keys a wavefront) 27 with and 21 without, a sweep of replicas 155 and
// 119; solvent beads hold up to 64 keys.
constexpr int kMatchRounds = 6;
constexpr int64_t kMatchBeads = 6000;                 // beads per key from which they are taken

__device__ __forceinline__ uint64_t wave_same_key(uint32_t key, bool active, int rounds, int nbits)
{
    uint64_t left = __ballot(active), mine = 0;
    for (int j = 0; j < rounds && left; ++j) {
        const uint32_t k = __builtin_amdgcn_readlane(key, __builtin_ctzll(left));
        const uint64_t m = __ballot(active && key == k);
        if (key == k)
            mine = m;
        left &= ~m;
    }
    if (left) {
        uint64_t m = left;
        for (int b = 0; b < nbits; ++b) {
            const bool set = (key >> b) & 1u;
            const uint64_t v = __ballot(set);
            m &= set ? v : ~v;
        }
        if ((left >> (threadIdx.x & (kWave - 1))) & 1ull)
            mine = m;
    }
    return active ? mine : 0ull;
}

// The first `rows` wavefronts of a workgroup place one chunk; wavefront w owns the w-th part of
// the chunk and row w of the LDS slots (further ones only help with the rows' keys). The rows are first counted, then turned into each
// wavefront's first slots (chunk slot + the earlier wavefronts' counts); from there on a
// wavefront needs no barrier. With many keys only the chunk's own key range is cleared and
// summed (the replicas of a batch follow each other in tag order, so a chunk sees few).
// Bound by its scattered 4-byte stores; the inverse is therefore left to a pass in storage
// order, where it is nearly in sequence. 3M beads, mostly solvent, in 1729 keys: 50 us, 10M
// chain beads in 513: 59. Before, the wavefronts of a workgroup took turns on one row, a
// barrier per turn, and grouped their lanes one distinct key at a time: 169 and 66 us.
__global__ __launch_bounds__(4 * kWave) void k_sort_place(const unsigned long long* __restrict__ by_tag, int64_t N,
                                                          int64_t S,
                                                          uint32_t nkeys, int rows, int rounds, int nbits,
                                                          const uint32_t* __restrict__ table,
                                                          int32_t* __restrict__ perm)
{
    extern __shared__ uint32_t slots[];                  // place_lds(nkeys, rows) bytes
    uint32_t* range = slots + (size_t)rows * nkeys;
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    const int64_t c = blockIdx.x;
    const int64_t part = S / rows;
    const int64_t t0 = min(N, c * S + wave * part), t1 = wave < rows ? min(N, t0 + part) : t0;
    uint32_t key[kPlaceRows];
    int32_t src[kPlaceRows];
    auto load = [&](int64_t g0) {
#pragma unroll
        for (int b = 0; b < kPlaceRows; ++b) {
            const int64_t t = g0 + b * kWave + lane;
            const unsigned long long e = t < t1 ? by_tag[t] : ~0ull;
            key[b] = (uint32_t)(e >> 32);
            src[b] = (int32_t)(uint32_t)e;
        }
    };
    // a part of one round of rows is read once and stays in registers
    const bool one = part <= kPlaceRows * kWave;
    load(t0);
    uint32_t ka = 0, kb = nkeys;
    if (nkeys > kRangeKeys) {
        if (threadIdx.x == 0) {
            range[0] = nkeys;
            range[1] = 0u;
        }
        __syncthreads();
        int lo = 0x7fffffff, hi = -1;
        for (int64_t g0 = t0; g0 < t1; g0 += kPlaceRows * kWave) {
            if (!one)
                load(g0);
#pragma unroll
            for (int b = 0; b < kPlaceRows; ++b)
                if (key[b] != kNoKey) {
                    lo = min(lo, (int)key[b]);
                    hi = max(hi, (int)key[b]);
                }
        }
        lo = wave_min(lo);
        hi = wave_max(hi);
        if (lane == 0 && hi >= 0) {
            atomicMin(&range[0], (uint32_t)lo);
            atomicMax(&range[1], (uint32_t)hi + 1u);
        }
        __syncthreads();
        ka = range[0];                                // ka >= kb: no tag of the chunk has a key
        kb = range[1];
    }
    uint32_t* mine = slots + (wave < rows ? wave : 0) * nkeys;
    for (uint32_t k = ka + threadIdx.x; k < kb; k += blockDim.x)
        for (int w = 0; w < rows; ++w)
            slots[w * nkeys + k] = 0u;
    __syncthreads();
    for (int64_t g0 = t0; g0 < t1; g0 += kPlaceRows * kWave) {
        if (!one)
            load(g0);
#pragma unroll
        for (int b = 0; b < kPlaceRows; ++b)
            if (g0 + b * kWave < t1)                 // uniform
                count_runs(mine, key[b]);
    }
    __syncthreads();
    const uint32_t* first = table + c * (int64_t)nkeys;
    for (uint32_t k0 = ka + threadIdx.x; k0 < kb; k0 += kKeyUnroll * blockDim.x) {
        uint32_t run[kKeyUnroll];
#pragma unroll
        for (int u = 0; u < kKeyUnroll; ++u)
            run[u] = first[min(k0 + u * blockDim.x, kb - 1)];
#pragma unroll
        for (int u = 0; u < kKeyUnroll; ++u) {
            const uint32_t k = k0 + u * blockDim.x;
            for (int w = 0; k < kb && w < rows; ++w) {
                const uint32_t v = slots[w * nkeys + k];
                slots[w * nkeys + k] = run[u];
                run[u] += v;
            }
        }
    }
    __syncthreads();
    volatile uint32_t* next = mine;            // lanes of one wavefront follow each other in order
    for (int64_t g0 = t0; g0 < t1; g0 += kPlaceRows * kWave) {
        if (!one)
            load(g0);
#pragma unroll
        for (int b = 0; b < kPlaceRows; ++b) {
            if (g0 + b * kWave >= t1)                // uniform: the row holds no tags
                break;
            const bool act = key[b] != kNoKey;
            const uint64_t grp = wave_same_key(key[b], act, rounds, nbits);
            if (act) {
                const uint32_t base = next[key[b]];
                if (__builtin_ctzll(grp) == lane)
                    next[key[b]] = base + (uint32_t)__builtin_popcountll(grp);
                perm[base + (uint32_t)__builtin_popcountll(grp & ((1ull << lane) - 1))] = src[b];
            }
        }
    }
}

// ------------------------------------------------ gather and bond table --

// Old storage index of output slot p. One out of range, in a slot that a broken permutation or
// broken key starts left, stands for the slot itself.
__device__ __forceinline__ int32_t source_of(const int32_t* __restrict__ perm, int64_t p, int64_t N)
{
    const int32_t o = perm[p];
    return o >= 0 && o < N ? o : (int32_t)p;
}

// New storage index of partner j (-1: none, or outside [-1, N), which is flagged, or a bead
// that a broken permutation left out).
__device__ __forceinline__ int32_t renumbered(int32_t j, const int32_t* __restrict__ inv, int64_t N, bool& bad)
{
    if (j >= 0 && j < N) {
        const int32_t nj = inv[j];
        return nj >= 0 && nj < N ? nj : -1;
    }
    bad |= j != -1;
    return -1;
}

__global__ __launch_bounds__(kSortThreads) void k_sort_inverse(const int32_t* __restrict__ perm, int64_t N,
                                                               int32_t* __restrict__ inv)
{
    const int64_t p = xcd_block(blockIdx.x, gridDim.x) * kSortThreads + threadIdx.x;
    if (p >= N)
        return;
    const int32_t o = perm[p];
    if (o >= 0 && o < N)                 // not a slot that a broken permutation left
        inv[o] = (int32_t)p;
}

// Bead rows and bond rows in the new order, in one pass (HBM-bound).
__global__ __launch_bounds__(kSortThreads) void k_sort_permute(const int32_t* __restrict__ perm,
                                                               const int32_t* __restrict__ inv, int64_t N,
                                                               const float3* __restrict__ R_in,
                                                               const float3* __restrict__ V_in,
                                                               const uint8_t* __restrict__ T_in,
                                                               const int32_t* __restrict__ tag_in,
                                                               const int32_t* __restrict__ bonds_in, int D,
                                                               float3* __restrict__ R_out,
                                                               float3* __restrict__ V_out,
                                                               uint8_t* __restrict__ T_out,
                                                               int32_t* __restrict__ tag_out,
                                                               int32_t* __restrict__ bonds_out)
{
    const int64_t p = xcd_block(blockIdx.x, gridDim.x) * kSortThreads + threadIdx.x;
    if (p >= N)
        return;
    const int32_t o = source_of(perm, p, N);
    R_out[p] = R_in[o];
    if (V_in)
        V_out[p] = V_in[o];
    T_out[p] = T_in[o];
    if (tag_in)
        tag_out[p] = tag_in[o];
    bool bad = false;
    for (int b = 0; b < D; ++b)
        bonds_out[(int64_t)b * N + p] = renumbered(bonds_in[(int64_t)b * N + o], inv, N, bad);
    if (bad)
        raise_flag(HPF_FLAG_BAD_BOND);
}

// Per-bead angle table in the new order: partner rows (3a, 3a + 1) renumbered
// like the bond table, code rows (3a + 2) moved with their bead unchanged.
__global__ __launch_bounds__(kSortThreads) void k_sort_angles(const int32_t* __restrict__ perm,
                                                              const int32_t* __restrict__ inv, int64_t N,
                                                              const int32_t* __restrict__ ang_in, int A,
                                                              int32_t* __restrict__ ang_out)
{
    const int64_t p = xcd_block(blockIdx.x, gridDim.x) * kSortThreads + threadIdx.x;
    if (p >= N)
        return;
    const int32_t o = source_of(perm, p, N);
    bool bad = false;
    for (int r = 0; r < 3 * A; ++r) {
        const int32_t j = ang_in[(int64_t)r * N + o];
        ang_out[(int64_t)r * N + p] = r % 3 == 2 ? j : renumbered(j, inv, N, bad);
    }
    if (bad)
        raise_flag(HPF_FLAG_BAD_BOND);
}

// ------------------------------------------- re-sort from a previous order --
//
// Between sorts most beads stay in their brick. When the input is in the order an
// earlier sort produced (ascending (key, tag) for the positions of that time) and
// that sort's key starts are given, the new order is built per key instead of over
// the whole tag sequence:
//   1. per old key range, in storage order (coalesced): every bead's new key; the
//      beads that keep their key ("stayers") are compacted to the front of the
//      range, still in tag order, and the others ("movers") to its end, each with
//      its new key and its rank among that key's movers;
//   2. one scan gives the new key starts and each key's slot range for its movers;
//   3. every mover is written (tag, index) to its slot;
//   4. per new key: its movers are sorted by tag, and the stayers and the movers
//      are merged by tag: a stayer's position is its rank among the stayers plus the
//      number of movers with a smaller tag (a binary search in LDS), and where that
//      number steps up between two stayers, the movers in between take their rank
//      among the stayers from it.
// The result equals the stable counting sort's exactly: (key, tag) order.
// Step 1 reads 16 B a bead and writes 4; only movers cost more. A workgroup reads 4096 beads
// between barriers, all rows before the first key, and counts its movers in an LDS table of
// the few keys they go to, with one global atomic per key. 42M beads in 13,824 bricks, 10 steps
// after their sort: keys 277 us, movers 46, placement 415 with the inverse, rows 827. (With 256
// beads between barriers, every bead's key written and read again and the stayers' tags searched
// in global memory: 350, 290, 581, and 1060 for the rows, bonds and inverse.) A single round of bricks
// (1M beads in 512) takes 95 us, as the full sort does.
// Small bricks take workgroups of 128 threads in the key pass, one row a thread, and a wavefront
// each in the placement, where a workgroup of 512 threads spends its time on barriers and on
// rows past the brick's end: 36,000 bricks of 6 beads 500 us, now 150, of 120 beads 815 and
// 330. Both passes loop, so that a large brick among small ones (a droplet) is only slower: 1M
// beads of a 24^3-cell droplet in 256^3 cells 490 us against 375 with 512 threads.
constexpr int kResortThreads = 512;
constexpr int kResortWaves = kResortThreads / kWave;
constexpr int kSmallThreads = 128;       // key pass of small bricks
constexpr int kResortPer = 8;            // rows a thread of the key pass reads at once
constexpr int kPlacePer = 4;             // stayers a thread reads at once
constexpr int kMoverCap = kPlacePer * kResortThreads;   // movers of one key sorted in LDS (16 KiB)
constexpr uint32_t kWaveBeads = 1024;    // stayers of a key that one wavefront places
template <int n>
using Rows = std::integral_constant<int, n>;
constexpr uint32_t kMoveKeys = 128;      // keys an old range's movers are counted under in LDS
constexpr int kMoveProbes = 16;

__device__ __forceinline__ int32_t tag_of(const int32_t* __restrict__ tag, int64_t i)
{
    return tag ? tag[i] : (int32_t)i;
}

template <int kThreads, class Keyer>
__global__ __launch_bounds__(kThreads) void k_resort_keys(Keyer keyer, const int32_t* __restrict__ tag,
                                                          const uint32_t* __restrict__ cs_old, int64_t N,
                                                          int32_t* __restrict__ order,
                                                          uint32_t* __restrict__ mkey,
                                                          uint32_t* __restrict__ mslot,
                                                          uint32_t* __restrict__ mrank,
                                                          uint32_t* __restrict__ cnt_stay,
                                                          uint32_t* __restrict__ cnt_move)
{
    constexpr int kWaves = kThreads / kWave;
    static_assert(kResortPer * kWaves <= kWave && kThreads >= (int)kMoveKeys, "one wave scans pre; a thread a table entry");
    __shared__ uint32_t hkey[kMoveKeys], hcnt[kMoveKeys];
    __shared__ uint32_t pre[kResortPer * kWaves + 1];
    const uint32_t k = (uint32_t)xcd_block(blockIdx.x, gridDim.x);
    const int64_t a = min((int64_t)cs_old[k], N), b = min((int64_t)cs_old[k + 1], N);
    if (a >= b) {
        if (threadIdx.x == 0)
            cnt_stay[k] = 0u;
        return;
    }
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    if (threadIdx.x < kMoveKeys) {
        hkey[threadIdx.x] = kNoKey;
        hcnt[threadIdx.x] = 0u;
    }
    int64_t run = 0;                     // stayers so far
    bool bad = false;
    // kPer rows of a tile from base on
    auto tile = [&](auto per, int64_t base) {
        constexpr int kPer = decltype(per)::value;
        // all rows first: a key's branches between them would have each wait for its own
        float3 r[kPer];
        int32_t tg[kPer], tb[kPer];
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const int64_t i = min(base + u * kThreads + threadIdx.x, b - 1);
            r[u] = keyer.R[i];
            tg[u] = tag_of(tag, i);
            tb[u] = i > a ? tag_of(tag, i - 1) : -1;
        }
        uint32_t key[kPer];
        uint64_t stay[kPer];
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const int64_t i = base + u * kThreads + threadIdx.x;
            key[u] = kNoKey;
            if (i < b) {
                key[u] = keyer((int32_t)i, r[u]);
                bad |= tg[u] <= tb[u];   // the precondition: every old key range in ascending tag order
            }
        }
        __syncthreads();                 // pre is read out; the table is cleared
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            stay[u] = __ballot(key[u] == k);
            if (lane == 0)
                pre[u * kWaves + wave] = (uint32_t)__builtin_popcountll(stay[u]);
        }
        __syncthreads();
        if (wave == 0) {
            const uint32_t v = lane < kPer * kWaves ? pre[lane] : 0u;
            const uint32_t inc = wave_incl_scan(v);
            if (lane < kPer * kWaves)
                pre[lane] = inc - v;
            if (lane == kPer * kWaves - 1)
                pre[lane + 1] = inc;
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const int64_t i = base + u * kThreads + threadIdx.x;
            if (i >= b)
                continue;
            const int64_t before = run + pre[u * kWaves + wave] +
                                   (uint32_t)__builtin_popcountll(stay[u] & ((1ull << lane) - 1));
            if (key[u] == k) {
                order[a + before] = (int32_t)i;
                continue;
            }
            const int64_t pos = b - 1 - (i - a - before);
            order[pos] = (int32_t)i;
            mkey[pos] = key[u];
        }
        run += pre[kPer * kWaves];
    };
    for (int64_t base = a; base < b;) {
        if (b - base > 2 * kThreads) {
            tile(Rows<kResortPer>(), base);
            base += kResortPer * kThreads;
        } else {
            tile(Rows<1>(), base);
            base += kThreads;
        }
    }
    if (bad) {
        raise_flag(HPF_FLAG_SORT_ORDER);
        cnt_move[gridDim.x] = 1u;        // for k_resort_movers
    }
    if (threadIdx.x == 0)
        cnt_stay[k] = (uint32_t)run;
    if (a + run == b)                    // uniform
        return;
    __syncthreads();
    // the movers, now side by side, are counted per key
    for (int64_t pos = a + run + threadIdx.x; pos < b; pos += kThreads) {
        const uint32_t key = mkey[pos];
        uint32_t h = (key * 2654435761u) >> 25, slot = kMoveKeys, rank = 0;
        for (int q = 0; q < kMoveProbes; ++q, h = (h + 1) % kMoveKeys) {
            const uint32_t old = atomicCAS(&hkey[h], kNoKey, key);
            if (old == kNoKey || old == key) {
                slot = h;
                rank = atomicAdd(&hcnt[h], 1u);
                break;
            }
        }
        if (slot == kMoveKeys)           // table full
            rank = atomicAdd(cnt_move + key, 1u);
        mslot[pos] = slot;
        mrank[pos] = rank;
    }
    __syncthreads();
    // each key's ranks follow those other ranges have reserved
    if (threadIdx.x < kMoveKeys && hcnt[threadIdx.x])
        hcnt[threadIdx.x] = atomicAdd(cnt_move + hkey[threadIdx.x], hcnt[threadIdx.x]);
    __syncthreads();
    for (int64_t pos = a + run + threadIdx.x; pos < b; pos += kThreads)
        if (mslot[pos] < kMoveKeys)
            mrank[pos] += hcnt[mslot[pos]];
}
static_assert(kMoveKeys == 1u << (32 - 25), "hash bits");

// One block: new key starts (stayers + movers per key, exclusive scan; the last entry the
// total) and the movers' slot offsets (exclusive scan of the mover counts).
__global__ __launch_bounds__(kScanThreads) void k_resort_scan(const uint32_t* __restrict__ cnt_stay,
                                                              const uint32_t* __restrict__ cnt_move, uint32_t nkeys,
                                                              uint32_t* __restrict__ start,
                                                              uint32_t* __restrict__ moff)
{
    __shared__ uint32_t sh[kScanThreads / kWave + 1];
    uint32_t run_st = 0, run_mv = 0;
    for (uint32_t k0 = 0; k0 < nkeys; k0 += kScanThreads) {
        const uint32_t k = k0 + threadIdx.x;
        const uint32_t mv = k < nkeys ? cnt_move[k] : 0u;
        const uint32_t st = k < nkeys ? cnt_stay[k] + mv : 0u;
        uint32_t tot_st, tot_mv;
        const uint32_t r_st = block_excl_scan<kScanThreads>(st, sh, &tot_st);
        const uint32_t r_mv = block_excl_scan<kScanThreads>(mv, sh, &tot_mv);
        if (k < nkeys) {
            start[k] = run_st + r_st;
            moff[k] = run_mv + r_mv;
        }
        run_st += tot_st;
        run_mv += tot_mv;
    }
    if (threadIdx.x == 0) {
        start[nkeys] = run_st;
        moff[nkeys] = run_mv;
    }
}

// Movers written to their new key's slots as (tag << 32 | index); their order inside
// a key's slots is arbitrary (sorted in the placement). Where a key range was out of tag order
// (cnt_move[nkeys] set), the placement may leave slots and beads out: perm and inv, which the
// ranks are read out of by then, are -1 beforehand.
__global__ __launch_bounds__(kSortThreads) void k_resort_movers(const int32_t* __restrict__ tag,
                                                                const uint32_t* __restrict__ cs_old, int64_t N,
                                                                const uint32_t* __restrict__ cnt_stay,
                                                                const uint32_t* __restrict__ cnt_move,
                                                                const int32_t* __restrict__ order,
                                                                const uint32_t* __restrict__ mkey,
                                                                const uint32_t* __restrict__ moff,
                                                                unsigned long long* __restrict__ movers,
                                                                int32_t* __restrict__ perm, int32_t* inv)
{
    const uint32_t* mrank = reinterpret_cast<const uint32_t*>(inv);
    const uint32_t k = blockIdx.x;
    const int64_t a = min((int64_t)cs_old[k], N), b = min((int64_t)cs_old[k + 1], N);
    for (int64_t pos = a + cnt_stay[k] + threadIdx.x; pos < b; pos += kSortThreads) {
        const int32_t i = order[pos];
        const int64_t dst = (int64_t)moff[mkey[pos]] + mrank[pos];
        if (dst < N)
            movers[dst] = ((unsigned long long)(uint32_t)tag_of(tag, i) << 32) | (unsigned long long)(uint32_t)i;
    }
    if (cnt_move[gridDim.x]) {
        __syncthreads();
        for (int64_t pos = a + threadIdx.x; pos < b; pos += kSortThreads) {
            perm[pos] = -1;
            inv[pos] = -1;
        }
    }
}

// Ascending sort of v[0, n) padded with +inf to p (a power of two): a bitonic network
// whose comparators all put the smaller value first (the first step of every merge
// compares mirrored positions), so the padding never moves forward. All threads call.
template <class Load, class Store>
__device__ __forceinline__ void sort_padded(int64_t n, int64_t p, Load load, Store store)
{
    for (int size = 1; (int64_t)1 << size <= p; ++size) {
        for (int stride = size - 1; stride >= 0; --stride) {
            for (int64_t q = threadIdx.x; q < p / 2; q += blockDim.x) {
                // the q-th comparator of this step: elements i < j
                const int64_t i = (q >> stride << (stride + 1)) + (q & (((int64_t)1 << stride) - 1));
                int64_t j = i + ((int64_t)1 << stride);
                if (stride == size - 1)
                    j = i ^ (((int64_t)1 << size) - 1);              // mirrored partner
                if (j < n) {
                    const unsigned long long a = load(i), c = load(j);
                    if (c < a) {
                        store(i, c);
                        store(j, a);
                    }
                }
            }
            __syncthreads();
        }
    }
}

// Number of the movers v[0, n) (ascending) below key.
template <class Load>
__device__ __forceinline__ int64_t movers_below(unsigned long long key, int64_t n, Load load)
{
    int64_t lo = 0, hi = n;
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if (load(mid) < key)
            lo = mid + 1;
        else
            hi = mid;
    }
    return lo;
}

// Number of entries of v[0, n) (ascending) below each of the keys e[0, kPer): one binary
// search each, their steps side by side. p2 is a power of two above n.
template <int kPer>
__device__ __forceinline__ void lds_below(const unsigned long long* v, int n, int p2,
                                          const unsigned long long (&e)[kPer], int (&pos)[kPer])
{
#pragma unroll
    for (int u = 0; u < kPer; ++u)
        pos[u] = 0;
    for (int s = p2 >> 1; s > 0; s >>= 1) {
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const int q = pos[u] + s;
            if (q <= n && v[q - 1] < e[u])
                pos[u] = q;
        }
    }
}

// Ascending sort of one value per lane of a wavefront (bitonic).
__device__ __forceinline__ unsigned long long wave_sort(unsigned long long v)
{
    const int lane = threadIdx.x & (kWave - 1);
#pragma unroll
    for (int size = 2; size <= kWave; size <<= 1)
#pragma unroll
        for (int stride = size >> 1; stride > 0; stride >>= 1) {
            const unsigned long long o = __shfl_xor(v, stride, kWave);
            const bool keep_min = ((lane & stride) == 0) == ((lane & size) == 0);
            v = (o < v) == keep_min ? o : v;
        }
    return v;
}

// Ascending sort of v[0, n) in LDS, n <= kMoverCap, v filled up with +inf to whole runs of 64;
// all values different. Each wavefront sorts runs in its registers; a value's place is its
// place in its run plus the number of smaller values in every other run. (A bitonic network
// over all of them took a barrier for each of its 55 steps at 600 values.)
__device__ __forceinline__ void sort_movers(int n, unsigned long long* v)
{
    constexpr int kWaves = kResortWaves, kPer = kPlacePer;
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    const int runs = (n + kWave - 1) / kWave;
    unsigned long long e[kPer];
    int rank[kPer];
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        const int r = u * kWaves + wave;
        e[u] = ~0ull;
        rank[u] = lane;
        if (r < runs) {
            e[u] = wave_sort(v[r * kWave + lane]);
            v[r * kWave + lane] = e[u];
        }
    }
    __syncthreads();
    if (wave < runs)
        for (int q = 0; q < runs; ++q) {
            int pos[kPer];
            lds_below(v + q * kWave, kWave, 2 * kWave, e, pos);
#pragma unroll
            for (int u = 0; u < kPer; ++u)
                rank[u] += q == u * kWaves + wave ? 0 : pos[u];
        }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kPer; ++u)
        if (u * kWaves + wave < runs && e[u] != ~0ull)
            v[rank[u]] = e[u];
    __syncthreads();
}

// Per new key: movers sorted by tag (in LDS when they fit, else in place in their
// slots), then stayers and movers merged by tag into the key's output range. kGroup: a
// wavefront per key, kResortWaves keys a workgroup, which then takes those that are too large
// for one together; else a workgroup per key.
template <bool kGroup>
__global__ __launch_bounds__(kResortThreads) void k_resort_place(const int32_t* __restrict__ tag,
                                                                 const uint32_t* __restrict__ cs_old, int64_t N,
                                                                 const int32_t* __restrict__ order,
                                                                 const uint32_t* __restrict__ cnt_stay,
                                                                 const uint32_t* __restrict__ cnt_move,
                                                                 const uint32_t* __restrict__ moff,
                                                                 const uint32_t* __restrict__ start, uint32_t nkeys,
                                                                 unsigned long long* __restrict__ movers,
                                                                 int32_t* __restrict__ perm,
                                                                 int32_t* __restrict__ inv)
{
    __shared__ unsigned long long smv[kMoverCap];
    __shared__ uint32_t below[kMoverCap];          // stayers below each mover
    const int lane = threadIdx.x & (kWave - 1);
    auto put = [&](int64_t dst, int32_t i) {
        // always, unless the key starts handed in were broken: where their ranges overlap, slots lie
        // beyond N and movers' entries are left as the workspace had them
        if (dst < N && i >= 0 && i < N) {
            perm[dst] = i;
            inv[i] = (int32_t)dst;
        }
    };
    auto n_movers = [&](uint32_t k) { return max((int64_t)0, min((int64_t)cnt_move[k], N - moff[k])); };
    // up to a wavefront's lanes of movers, by one wavefront
    auto by_wave = [&](uint32_t k) {
        const int64_t nmv = n_movers(k), ns = cnt_stay[k], base = start[k];
        const int32_t* st = order + min((int64_t)cs_old[k], N);
        volatile uint32_t* mine = below + threadIdx.x / kWave * kWave;   // one wavefront's, in order
        unsigned long long e = lane < nmv ? movers[moff[k] + lane] : ~0ull;
        if (nmv > 1)
            e = wave_sort(e);
        mine[lane] = (uint32_t)ns;
        int last = 0;                    // movers below the stayer before these
        for (int64_t q0 = 0; q0 < ns; q0 += kWave) {
            const int64_t q = q0 + lane;
            const int32_t idx = q < ns ? st[q] : 0;
            int c = 0;
            if (nmv) {
                const unsigned long long t = (unsigned long long)(uint32_t)tag_of(tag, idx) << 32;
#pragma unroll
                for (int step = kWave / 2; step > 0; step >>= 1)
                    c += __shfl(e, c + step - 1, kWave) < t ? step : 0;
                c += __shfl(e, c, kWave) < t;
            }
            if (q < ns)
                put(base + q + c, idx);
            const int up = __shfl_up(c, 1, kWave);
            if (q < ns)
                for (int j = lane ? up : last; j < c; ++j)
                    mine[j] = (uint32_t)q;
            last = __shfl(c, kWave - 1, kWave);
        }
        if (lane < nmv)
            put(base + lane + mine[lane], (int32_t)(uint32_t)e);
    };
    auto by_block = [&](uint32_t k) {
        const int64_t nmv = n_movers(k), ns = cnt_stay[k];
        const int64_t base = start[k];
        unsigned long long* mv = movers + moff[k];
        const int32_t* st = order + min((int64_t)cs_old[k], N);
        int64_t p2 = 1, p2above = 1;
        while (p2 < nmv)
            p2 <<= 1;
        while (p2above <= nmv)
            p2above <<= 1;
        const bool in_lds = nmv <= kMoverCap;
        auto lds = [&](int64_t q) { return smv[q]; };
        auto glob = [&](int64_t q) { return mv[q]; };
        if (in_lds) {
            for (int64_t q = threadIdx.x; q < (nmv + kWave - 1) / kWave * kWave; q += kResortThreads) {
                smv[q] = q < nmv ? mv[q] : ~0ull;
                below[q] = (uint32_t)ns;
            }
            __syncthreads();
            sort_movers((int)nmv, smv);
        } else {
            sort_padded(nmv, p2, glob, [&](int64_t q, unsigned long long v) { mv[q] = v; });
        }
        // stayers: rank among stayers + movers with a smaller tag; the movers between a stayer
        // and the one before it have that stayer's rank of stayers below them
        for (int64_t q0 = 0; q0 < ns; q0 += kPlacePer * kResortThreads) {
            int32_t idx[kPlacePer], tg[kPlacePer];
#pragma unroll
            for (int u = 0; u < kPlacePer; ++u) {
                const int64_t q = q0 + u * kResortThreads + threadIdx.x;
                idx[u] = q < ns ? st[q] : 0;
            }
#pragma unroll
            for (int u = 0; u < kPlacePer; ++u)
                tg[u] = tag_of(tag, idx[u]);
            unsigned long long e[kPlacePer];
            int c[kPlacePer];
#pragma unroll
            for (int u = 0; u < kPlacePer; ++u) {
                e[u] = (unsigned long long)(uint32_t)tg[u] << 32;
                c[u] = in_lds ? 0 : (int)movers_below(e[u], nmv, glob);
            }
            if (in_lds)
                lds_below(smv, (int)nmv, (int)p2above, e, c);
#pragma unroll
            for (int u = 0; u < kPlacePer; ++u) {
                const int64_t q = q0 + u * kResortThreads + threadIdx.x;
                if (q < ns)
                    put(base + q + c[u], idx[u]);
                if (!in_lds)
                    continue;
                int prev = __shfl_up(c[u], 1, kWave);
                if (lane == 0)
                    prev = q > 0 && q < ns
                               ? (int)movers_below((unsigned long long)(uint32_t)tag_of(tag, st[q - 1]) << 32, nmv, lds)
                               : 0;
                if (q < ns)
                    for (int j = prev; j < c[u]; ++j)
                        below[j] = (uint32_t)q;
            }
        }
        __syncthreads();
        for (int64_t q = threadIdx.x; q < nmv; q += kResortThreads) {
            const unsigned long long e = in_lds ? smv[q] : mv[q];
            int64_t lo = 0;
            if (in_lds) {
                lo = below[q];
            } else {
                const int32_t t = (int32_t)(e >> 32);
                int64_t hi = ns;
                while (lo < hi) {
                    const int64_t mid = (lo + hi) >> 1;
                    if (tag_of(tag, st[mid]) < t)
                        lo = mid + 1;
                    else
                        hi = mid;
                }
            }
            put(base + q + lo, (int32_t)(uint32_t)e);
        }
    };
    const uint32_t b = (uint32_t)xcd_block(blockIdx.x, gridDim.x);
    if constexpr (!kGroup) {
        by_block(b);
    } else {
        __shared__ bool large[kResortWaves];
        const int wave = threadIdx.x / kWave;
        const uint32_t k = b + wave * gridDim.x;           // far from each other: large keys tend not to be
        const bool too_large = k < nkeys && (cnt_move[k] > kWave || cnt_stay[k] > kWaveBeads);
        if (k < nkeys && !too_large)
            by_wave(k);
        if (lane == 0)
            large[wave] = too_large;
        __syncthreads();
        for (int w = 0; w < kResortWaves; ++w)
            if (large[w]) {
                by_block(b + w * gridDim.x);
                __syncthreads();
            }
    }
}

// ------------------------------------------------------------------ host --

static size_t align_up(size_t x) { return (x + 255) & ~(size_t)255; }

// Sizes and workspace layout of one sort of N beads over nkeys keys.
struct SortPlan {
    int64_t N = 0;
    uint32_t nkeys = 0;
    int64_t S = 0, nchunks = 0, ncb = 0;
    size_t off_key = 0, off_perm = 0, off_inv = 0, off_table = 0, off_part = 0, off_start = 0;
    // re-sort from a previous order: compacted stayers and movers, the movers by key (the full
    // sort keeps its keys and indices by tag there), per-key counts and offsets
    size_t off_stay = 0, off_movers = 0, off_cstay = 0, off_cmove = 0, off_moff = 0;
    size_t bytes = 0;
};

bool sort_plan(int64_t N, int64_t nkeys, SortPlan* p)
{
    if (N < 0 || N > 0x7ffffff0LL || nkeys < 1 || nkeys > kMaxSortKeys)
        return false;
    // Chunks of 4096 tags (one placement round), or of 1024 when that leaves fewer
    // than kChunksWanted chunks and the chunk x key table stays within 4 entries
    // per bead; larger while the table exceeds kMaxTable.
    int64_t S = kMinChunk;
    if ((N + S - 1) / S < kChunksWanted && ((N + kSmallChunk - 1) / kSmallChunk) * nkeys <= 4 * std::max<int64_t>(N, 1))
        S = kSmallChunk;
    while (((N + S - 1) / S) * nkeys > kMaxTable)
        S *= 2;
    p->N = N;
    p->nkeys = (uint32_t)nkeys;
    p->S = S;
    p->nchunks = std::max<int64_t>(1, (N + S - 1) / S);
    p->ncb = (p->nchunks + kColBlock - 1) / kColBlock;
    const size_t N1 = (size_t)(N > 0 ? N : 1);
    size_t o = 0;
    p->off_key = o; o += align_up(sizeof(uint32_t) * N1);
    p->off_perm = o; o += align_up(sizeof(int32_t) * N1);
    p->off_inv = o; o += align_up(sizeof(int32_t) * N1);
    p->off_table = o; o += align_up(sizeof(uint32_t) * (size_t)p->nchunks * (size_t)nkeys);
    p->off_part = o; o += align_up(sizeof(uint32_t) * (size_t)p->ncb * (size_t)nkeys);
    p->off_start = o; o += align_up(sizeof(uint32_t) * (size_t)(nkeys + 2));
    p->off_stay = o; o += align_up(sizeof(int32_t) * N1);
    p->off_movers = o; o += align_up(sizeof(uint64_t) * N1);
    p->off_cstay = o; o += align_up(sizeof(uint32_t) * (size_t)nkeys);
    p->off_cmove = o; o += align_up(sizeof(uint32_t) * (size_t)(nkeys + 1));
    p->off_moff = o; o += align_up(sizeof(uint32_t) * (size_t)(nkeys + 1));
    p->bytes = o;
    return true;
}

bool sort_layout(int64_t N, const int32_t M[3], int B, SortK* sk_out, SortPlan* plan)
{
    if (B == 0)
        B = 8;
    if (B < 1 || B > 16)
        return false;
    int64_t nk = 1;
    int32_t nb[3];
    for (int d = 0; d < 3; ++d) {
        nb[d] = (M[d] + B - 1) / B;
        nk *= nb[d];
    }
    if (!sort_plan(N, nk + 1, plan))
        return false;
    if (sk_out) {
        sk_out->B = B;
        for (int d = 0; d < 3; ++d)
            sk_out->nb[d] = nb[d];
        sk_out->NK = (uint32_t)nk;
    }
    return true;
}

static unsigned grid_for(int64_t n) { return (unsigned)((n + kSortThreads - 1) / kSortThreads); }

static void launch_permute(int64_t N, const int32_t* perm, const int32_t* inv, const float* R_in, const float* V_in,
                           const uint8_t* T_in, const int32_t* tag_in, const int32_t* bonds_in, int D, float* R_out,
                           float* V_out, uint8_t* T_out, int32_t* tag_out, int32_t* bonds_out, hipStream_t s)
{
    hipLaunchKernelGGL(k_sort_permute, dim3(grid_for(N)), dim3(kSortThreads), 0, s, perm, inv, N,
                       reinterpret_cast<const float3*>(R_in), reinterpret_cast<const float3*>(V_in), T_in, tag_in,
                       bonds_in, bonds_in ? D : 0, reinterpret_cast<float3*>(R_out), reinterpret_cast<float3*>(V_out),
                       T_out, tag_out, bonds_out);
}

// LDS of a placement workgroup: its slot rows of nkeys u32 and the two ends of its key range.
// The kernel has none besides, so this is all that a launch asks for.
static constexpr size_t place_lds(uint32_t nkeys, int rows)
{
    return sizeof(uint32_t) * ((size_t)nkeys * rows + 2);
}

// Wavefronts of a placement workgroup: 4, 2 or 1, whichever number of slot rows packs the most
// rows into a CU's LDS, and the larger of equals. A number whose workgroup does not fit is out:
// 4 above 10,239 keys, 2 above 20,479. One row fits at every key count.
static_assert(place_lds(kMaxSortKeys, 1) <= kLdsPerCu, "one slot row of the largest key count fits a CU");

static int place_rows(uint32_t nkeys)
{
    const size_t row = sizeof(uint32_t) * (size_t)nkeys;
    int best = 1;
    for (int rows = 2; rows <= 4; rows *= 2)
        if (place_lds(nkeys, rows) <= kLdsPerCu && rows * (kLdsPerCu / (row * rows)) >= best * (kLdsPerCu / (row * best)))
            best = rows;
    return best;
}

// Threads of a placement workgroup. Where a CU has room for at most eight slot rows, they are long,
// and the workgroup has four wavefronts whatever their number, which takes no other's place: 200,000
// beads over 35,938 keys, one row, sort 326 us with one wavefront, 173 with four.
static int place_threads(uint32_t nkeys, int rows)
{
    return rows * (kLdsPerCu / place_lds(nkeys, rows)) <= 8 ? 4 * kWave : rows * kWave;
}

// The four steps and the gather for any key function; `start` receives the
// key starts (nkeys + 1 entries, the last = number of placed beads).
template <class Keyer>
hpf_status_t run_sort(const SortPlan& pl, Keyer keyer, int64_t N, const float* R_in, const float* V_in,
                      const uint8_t* T_in, const int32_t* tag_in, const int32_t* bonds_in, int D, float* R_out,
                      float* V_out, uint8_t* T_out, int32_t* tag_out, int32_t* bonds_out, uint32_t* start,
                      char* work, hipStream_t s)
{
    auto* by_tag = reinterpret_cast<unsigned long long*>(work + pl.off_movers);
    int32_t* perm = reinterpret_cast<int32_t*>(work + pl.off_perm);
    int32_t* inv = reinterpret_cast<int32_t*>(work + pl.off_inv);
    uint32_t* table = reinterpret_cast<uint32_t*>(work + pl.off_table);
    uint32_t* part = reinterpret_cast<uint32_t*>(work + pl.off_part);
    const uint32_t nk = pl.nkeys;
    if (N == 0) {
        hipLaunchKernelGGL(k_fill_u32, dim3((unsigned)std::min<int64_t>(grid_for(nk + 1), 4096)), dim3(kSortThreads),
                           0, s, start, (int64_t)nk + 1, 0u);
        return hipGetLastError() == hipSuccess ? HPF_OK : HPF_EHIP;
    }
    const size_t smem = sizeof(uint32_t) * nk;
    const int rows = place_rows(nk);
    const size_t smem_place = place_lds(nk, rows);
    if ((smem > 65536 && hipFuncSetAttribute(reinterpret_cast<const void*>(k_sort_hist),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem) != hipSuccess) ||
        (smem_place > 65536 &&
         hipFuncSetAttribute(reinterpret_cast<const void*>(k_sort_place), hipFuncAttributeMaxDynamicSharedMemorySize,
                             (int)smem_place) != hipSuccess))
        return HPF_EINVAL;
    hipLaunchKernelGGL(k_fill_u64, dim3((unsigned)std::min<int64_t>(grid_for(N), 8192)), dim3(kSortThreads), 0, s,
                       by_tag, N, ~0ull);
    hipLaunchKernelGGL(k_tag_index<Keyer>, dim3(grid_for(N)), dim3(kSortThreads), 0, s, keyer, tag_in, N, by_tag);
    hipLaunchKernelGGL(k_sort_hist, dim3((unsigned)pl.nchunks), dim3(kChunkThreads), smem, s, by_tag, N, pl.S, nk,
                       table);
    if (pl.ncb == 1 && nk <= kSmallKeys) {
        hipLaunchKernelGGL(k_col_small, dim3(1), dim3(kScanThreads), 0, s, table, pl.nchunks, nk, start, N, perm,
                           inv);
    } else {
        const unsigned gk = (nk + kSortThreads - 1) / kSortThreads;
        const dim3 gcol(gk, (unsigned)pl.ncb);
        hipLaunchKernelGGL(k_col_partial, gcol, dim3(kSortThreads), 0, s, table, pl.nchunks, nk, part);
        hipLaunchKernelGGL(k_col_prefix, dim3(gk), dim3(kSortThreads), 0, s, part, pl.ncb, nk, start);
        hipLaunchKernelGGL(k_scan_keys, dim3(1), dim3(kScanThreads), 0, s, start, nk, N, perm, inv);
        hipLaunchKernelGGL(k_col_apply, gcol, dim3(kSortThreads), 0, s, table, part, start, pl.nchunks, nk);
    }
    int nbits = 1;
    while ((1u << nbits) < nk)
        ++nbits;
    hipLaunchKernelGGL(k_sort_place, dim3((unsigned)pl.nchunks), dim3(place_threads(nk, rows)), smem_place, s, by_tag,
                       N, pl.S, nk, rows, N / nk >= kMatchBeads ? kMatchRounds : 0, nbits, table, perm);
    hipLaunchKernelGGL(k_sort_inverse, dim3(grid_for(N)), dim3(kSortThreads), 0, s, perm, N, inv);
    launch_permute(N, perm, inv, R_in, V_in, T_in, tag_in, bonds_in, D, R_out, V_out, T_out, tag_out, bonds_out, s);
    return hipGetLastError() == hipSuccess ? HPF_OK : HPF_EHIP;
}

hpf_status_t launch_sort(const SortK& sk, const SortPlan& pl, int64_t N, const float* R_in, const float* V_in,
                         const uint8_t* T_in, const int32_t* tag_in, const int32_t* bonds_in, int D, float* R_out,
                         float* V_out, uint8_t* T_out, int32_t* tag_out, int32_t* bonds_out, uint32_t* cell_start,
                         char* work, hipStream_t s)
{
    CellKeyer keyer{sk, reinterpret_cast<const float3*>(R_in)};
    uint32_t* start = cell_start ? cell_start : reinterpret_cast<uint32_t*>(work + pl.off_start);
    return run_sort(pl, keyer, N, R_in, V_in, T_in, tag_in, bonds_in, D, R_out, V_out, T_out, tag_out, bonds_out,
                    start, work, s);
}

// Whether the re-sort takes the passes for small bricks. The line lies where they stop being the
// faster ones (with / without, a tenth of a cell moved and half a cell: 4,096 bricks of 400 beads
// 74 / 110 and 127 / 126 us, of 600 91 / 131 and 163 / 152). A few hundred bricks fill the chip
// only a workgroup each: 27 of 111 beads, every bead moving, 85 and 30 us.
static bool small_bricks(int64_t N, uint32_t nkeys) { return nkeys >= 2048 && N <= 400 * (int64_t)nkeys; }

// The re-sort (steps 1-4 above), then the gather and the bond renumbering of run_sort. The
// movers' table slots and ranks stand in perm and inv until the placement writes those.
template <class Keyer>
hpf_status_t run_resort(const SortPlan& pl, Keyer keyer, int64_t N, const float* R_in, const float* V_in,
                        const uint8_t* T_in, const int32_t* tag_in, const int32_t* bonds_in, int D, float* R_out,
                        float* V_out, uint8_t* T_out, int32_t* tag_out, int32_t* bonds_out, const uint32_t* cs_old,
                        uint32_t* cs_new, char* work, hipStream_t s)
{
    const uint32_t nk = pl.nkeys;
    auto* mkey = reinterpret_cast<uint32_t*>(work + pl.off_key);
    auto* perm = reinterpret_cast<int32_t*>(work + pl.off_perm);
    auto* inv = reinterpret_cast<int32_t*>(work + pl.off_inv);
    auto* order = reinterpret_cast<int32_t*>(work + pl.off_stay);
    auto* movers = reinterpret_cast<unsigned long long*>(work + pl.off_movers);
    auto* cstay = reinterpret_cast<uint32_t*>(work + pl.off_cstay);
    auto* cmove = reinterpret_cast<uint32_t*>(work + pl.off_cmove);
    auto* moff = reinterpret_cast<uint32_t*>(work + pl.off_moff);
    if (N == 0) {
        hipLaunchKernelGGL(k_fill_u32, dim3((unsigned)std::min<int64_t>(grid_for(nk + 1), 4096)), dim3(kSortThreads),
                           0, s, cs_new, (int64_t)nk + 1, 0u);
        return hipGetLastError() == hipSuccess ? HPF_OK : HPF_EHIP;
    }
    hipLaunchKernelGGL(k_fill_u32, dim3((unsigned)std::min<int64_t>(grid_for(nk), 4096)), dim3(kSortThreads), 0, s,
                       cmove, (int64_t)nk + 1, 0u);
    const bool small = small_bricks(N, nk);
    hipLaunchKernelGGL((small ? k_resort_keys<kSmallThreads, Keyer> : k_resort_keys<kResortThreads, Keyer>), dim3(nk),
                       dim3(small ? kSmallThreads : kResortThreads), 0, s, keyer, tag_in, cs_old, N, order, mkey, reinterpret_cast<uint32_t*>(perm),
                       reinterpret_cast<uint32_t*>(inv), cstay, cmove);
    hipLaunchKernelGGL(k_resort_scan, dim3(1), dim3(kScanThreads), 0, s, cstay, cmove, nk, cs_new, moff);
    hipLaunchKernelGGL(k_resort_movers, dim3(nk), dim3(kSortThreads), 0, s, tag_in, cs_old, N, cstay, cmove,
                       order, mkey, moff, movers, perm, inv);
    hipLaunchKernelGGL((small ? k_resort_place<true> : k_resort_place<false>),
                       dim3(small ? (nk + kResortWaves - 1) / kResortWaves : nk), dim3(kResortThreads), 0, s, tag_in, cs_old, N, order, cstay, cmove,
                       moff, cs_new, nk, movers, perm, inv);
    launch_permute(N, perm, inv, R_in, V_in, T_in, tag_in, bonds_in, D, R_out, V_out, T_out, tag_out, bonds_out, s);
    return hipGetLastError() == hipSuccess ? HPF_OK : HPF_EHIP;
}

hpf_status_t launch_resort(const SortK& sk, const SortPlan& pl, int64_t N, const float* R_in, const float* V_in,
                           const uint8_t* T_in, const int32_t* tag_in, const int32_t* bonds_in, int D, float* R_out,
                           float* V_out, uint8_t* T_out, int32_t* tag_out, int32_t* bonds_out,
                           const uint32_t* cs_old, uint32_t* cs_new, char* work, hipStream_t s)
{
    CellKeyer keyer{sk, reinterpret_cast<const float3*>(R_in)};
    return run_resort(pl, keyer, N, R_in, V_in, T_in, tag_in, bonds_in, D, R_out, V_out, T_out, tag_out, bonds_out,
                      cs_old, cs_new, work, s);
}

hpf_status_t launch_sort_angles(const SortPlan& pl, int64_t N, const int32_t* ang_in, int A, int32_t* ang_out,
                                const char* work, hipStream_t s)
{
    if (N == 0 || A == 0)
        return HPF_OK;
    const int32_t* perm = reinterpret_cast<const int32_t*>(work + pl.off_perm);
    const int32_t* inv = reinterpret_cast<const int32_t*>(work + pl.off_inv);
    hipLaunchKernelGGL(k_sort_angles, dim3(grid_for(N)), dim3(kSortThreads), 0, s, perm, inv, N, ang_in, A, ang_out);
    return hipGetLastError() == hipSuccess ? HPF_OK : HPF_EHIP;
}

}  // namespace hpf
