// abi.hip -- status handling, block-hash chains and table construction.
#include <hip/hip_runtime.h>

#include <atomic>
#include <mutex>
#include <stdarg.h>
#include <stdio.h>
#include <string.h>

#include "rk_internal.h"

namespace rk {

static thread_local char g_last_error[512] = "";

int fail(int status, const char* fmt, ...)
{
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_last_error, sizeof g_last_error, fmt, ap);
    va_end(ap);
    return status;
}

int hip_check(hipError_t e, const char* what)
{
    if (e == hipSuccess) return RK_OK;
    return fail(RK_EHIP, "%s: %s", what, hipGetErrorString(e));
}

// One status word per device.  Kernels OR RK_DEV_* bits into it; the host
// finds its address per device once and reads it in rk_device_status.
static __device__ int32_t g_status;

static std::mutex g_status_mu;
static int32_t* g_status_addr[64];

int32_t* status_word()
{
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return nullptr;
    std::lock_guard<std::mutex> lk(g_status_mu);
    if (!g_status_addr[dev]) {
        void* p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(g_status)) != hipSuccess) return nullptr;
        g_status_addr[dev] = (int32_t*)p;
    }
    return g_status_addr[dev];
}

bool event_done(hipEvent_t e)
{
    // the query is a call that a capture elsewhere in the process would otherwise be ended by
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    const bool changed = hipThreadExchangeStreamCaptureMode(&mode) == hipSuccess;
    const hipError_t before = hipPeekAtLastError(), q = hipEventQuery(e);
    if (q != hipSuccess && before == hipSuccess) (void)hipGetLastError();     // "not ready" is no failure
    if (changed) (void)hipThreadExchangeStreamCaptureMode(&mode);
    return q == hipSuccess;
}

// The current device's compute units, asked for once per device (0 if unknown).
int32_t compute_units()
{
    static std::atomic<int32_t> known[64];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 0;
    int32_t n = known[dev].load(std::memory_order_relaxed);
    if (n == 0) {
        int v = 0;
        if (hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
        n = v;
        known[dev].store(n, std::memory_order_relaxed);
    }
    return n;
}

EpisodeLayout episode_layout(int32_t W, int32_t cache_blocks, int32_t max_blocks, int32_t max_conv,
                             int32_t max_routes)
{
    EpisodeLayout L;
    uint64_t live_max = (uint64_t)cache_blocks + (uint64_t)max_blocks;
    L.slots = next_pow2(2 * live_max);
    L.ring = next_pow2(2 * live_max);
    // run index entries: a run's first block and its checkpoints, at most 2 per route plus one per
    // 2^kCkptLog cached blocks of each worker, at load <= 1/2
    L.runs = next_pow2(2 * (2 * (uint64_t)(max_routes > 2 ? max_routes : 2) +
                            (uint64_t)W * ((live_max >> kCkptLog) + 1)));
    size_t o = 0;
    L.off_slots = o;   o = align_up(o + (size_t)W * L.slots * sizeof(Slot), 256);
    L.off_log = o;     o = align_up(o + (size_t)W * L.ring * sizeof(uint32_t), 256);
    L.off_scratch = o; o = align_up(o + live_max * sizeof(uint64_t), 256);
    L.off_scratch_f = o; o = align_up(o + live_max * sizeof(uint32_t), 256);
    L.off_queue = o;   o = align_up(o + ((size_t)max_conv + 1) * sizeof(int32_t), 256);
    L.off_next = o;    o = align_up(o + ((size_t)max_conv + 1) * sizeof(int32_t), 256);
    L.off_hist = o;    o = align_up(o + ((size_t)max_routes + 1) * 2 * sizeof(int32_t), 256);
    L.off_replay = o;  o = align_up(o + (size_t)kEpisodeThreadsMax * 16, 256);
    L.off_later = o;   o = align_up(o + ((size_t)max_conv + 1) * sizeof(int32_t), 256);
    L.off_ctl = o;     o = align_up(o + 256, 256);     // launch control (episode queue counter)
    L.off_runs = o;    o = align_up(o + L.runs * sizeof(RunSlot), 256);
    L.per_episode = o;
    return L;
}

// ------------------------------------------------------------------ hashing

// FNV-1a of every block: one wavefront per sequence, lanes over blocks.  The
// per-block values are written in place of the chain and chained afterwards.
__global__ __launch_bounds__(256) void block_fnv_kernel(int64_t n_seq, const int32_t* __restrict__ tokens,
                                                        const int64_t* __restrict__ tok_off,
                                                        const int64_t* __restrict__ chain_off,
                                                        uint64_t* __restrict__ chains, int32_t* status)
{
    const int lane = threadIdx.x & 63;
    const int64_t nwaves = (int64_t)gridDim.x * (blockDim.x >> 6);
    for (int64_t s = (int64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6); s < n_seq; s += nwaves) {
        const int64_t t0 = tok_off[s], t1 = tok_off[s + 1];
        const int64_t c0 = chain_off[s], c1 = chain_off[s + 1];
        if (t1 < t0 || c1 < c0) {
            if (lane == 0) atomicOr(status, RK_DEV_BAD_OFFSETS);
            continue;
        }
        const int64_t nb = c1 - c0;
        const int64_t avail = (t1 - t0) / 16;
        if (nb > avail && lane == 0) atomicOr(status, RK_DEV_SHORT_INPUT);
        for (int64_t k = lane; k < nb; k += 64) {
            uint64_t h = 0;
            if (k < avail) {
                const int32_t* tk = tokens + t0 + 16 * k;
                h = 0xcbf29ce484222325ull;
#pragma unroll
                for (int q = 0; q < 16; ++q) h = fnv_word(h, (uint32_t)tk[q]);
            }
            chains[c0 + k] = h;
        }
    }
}

// Serial chaining of each sequence: one lane per sequence.  A wavefront runs
// as long as its longest sequence, so each 1024-thread workgroup first ranks
// its sequences by length (classes of 32 blocks, longest first) and hands
// them to lanes in that order: the sequences of one wavefront then have
// similar lengths.  The per-block values move through registers kChainChunk
// at a time, and the next chunk's reads are issued before the current chunk
// is chained, so a lane's memory latency overlaps its arithmetic.  Reads and
// writes past a sequence's end are clamped to its last block (a write there
// stores that block's final value), which keeps every memory instruction
// unconditional.
constexpr int kChainChunk = 16;
// two chained values, 8-byte aligned (a 16-byte access needs only the element alignment)
typedef uint64_t u64x2 __attribute__((ext_vector_type(2), aligned(8)));
constexpr int kChainWG = 1024;
constexpr int kChainClasses = 32;

__device__ __forceinline__ int64_t chain_length(int64_t s, const int64_t* __restrict__ tok_off,
                                                const int64_t* __restrict__ chain_off, int64_t& c0)
{
    c0 = chain_off[s];
    const int64_t c1 = chain_off[s + 1], t0 = tok_off[s], t1 = tok_off[s + 1];
    if (c1 < c0 || t1 < t0) return 0;
    return min(c1 - c0, (t1 - t0) / 16);
}

__global__ __launch_bounds__(kChainWG) void chain_kernel(int64_t n_seq, const int64_t* __restrict__ tok_off,
                                                         const int64_t* __restrict__ chain_off,
                                                         uint64_t* __restrict__ chains)
{
    __shared__ int32_t cnt[kChainClasses], base[kChainClasses];
    __shared__ int32_t order[kChainWG];
    const int tid = threadIdx.x;
    const int64_t s0 = (int64_t)blockIdx.x * kChainWG;
    const int32_t m = (int32_t)min((int64_t)kChainWG, n_seq - s0);
    if (tid < kChainClasses) cnt[tid] = 0;
    __syncthreads();
    int cls = 0;
    if (tid < m) {
        int64_t c0;
        const int64_t n = chain_length(s0 + tid, tok_off, chain_off, c0);
        cls = (int)min(n / 32, (int64_t)(kChainClasses - 1));
        atomicAdd(&cnt[cls], 1);
    }
    __syncthreads();
    if (tid == 0) {
        int32_t o = 0;
        for (int c = kChainClasses - 1; c >= 0; --c) {
            base[c] = o;
            o += cnt[c];
        }
    }
    __syncthreads();
    if (tid < m) order[atomicAdd(&base[cls], 1)] = tid;
    __syncthreads();
    if (tid >= m) return;
    const int64_t s = s0 + order[tid];
    int64_t c0;
    const int64_t n = chain_length(s, tok_off, chain_off, c0);
    if (n <= 0) return;
    const int64_t last = c0 + n - 1;
    uint64_t cur[kChainChunk], nxt[kChainChunk];
    // whole chunks move as pairs of values (16-byte accesses); a chunk that reaches past the
    // sequence's last block moves value by value, clamped to it
    auto load_chunk = [&](int64_t k, uint64_t* v) {
        if (k + kChainChunk - 1 <= last - c0) {
#pragma unroll
            for (int u = 0; u < kChainChunk; u += 2) {
                const u64x2 q = *reinterpret_cast<const u64x2*>(chains + c0 + k + u);
                v[u] = q.x;
                v[u + 1] = q.y;
            }
        } else {
#pragma unroll
            for (int u = 0; u < kChainChunk; ++u) v[u] = chains[min(c0 + k + u, last)];
        }
    };
    load_chunk(0, cur);
    uint64_t h = 0;
    for (int64_t k0 = 0; k0 < n; k0 += kChainChunk) {
        load_chunk(k0 + kChainChunk, nxt);
#pragma unroll
        for (int u = 0; u < kChainChunk; ++u) {
            const uint64_t hn = chain_next(h, cur[u]);
            h = k0 + u < n ? hn : h;
            cur[u] = h;
        }
        if (k0 + kChainChunk - 1 <= last - c0) {
#pragma unroll
            for (int u = 0; u < kChainChunk; u += 2) {
                u64x2 q;
                q.x = cur[u];
                q.y = cur[u + 1];
                *reinterpret_cast<u64x2*>(chains + c0 + k0 + u) = q;
            }
        } else {
#pragma unroll
            for (int u = 0; u < kChainChunk; ++u) chains[min(c0 + k0 + u, last)] = cur[u];
        }
#pragma unroll
        for (int u = 0; u < kChainChunk; ++u) cur[u] = nxt[u];
    }
}

// FNV-1a and chain of few sequences, a workgroup per sequence.  What bounds a
// small call is the chain, one splitmix64 step after another; a wavefront that
// chains one sequence does it in scalar registers (about 28 scalar
// instructions a block), with no memory access in between: wavefront 0 takes 64
// block values from LDS, one per lane, chains them by readlane and keeps the
// results in the lanes for one coalesced store, while the other wavefronts hash
// the blocks kFewSpan further on.  A block takes 73 ns along the chain
// (lane-per-sequence: about 0.4 us, its loads and stores in between), but a
// CU's scalar unit chains no more than 25 G blocks/s over the chip, so it is
// the path of up to kFewSeqs sequences (a workgroup / a lane each, 128 blocks
// on average: 4,096 sequences 61 / 118 us, 8,192 98 / 128, 16,384 169 / 147;
// 600 blocks: 271 / 451, 422 / 509, 737 / 700).
constexpr int64_t kFewSeqs = 8192;
constexpr int kFewThreads = 256;
constexpr int kFewSpan = kFewThreads;    // blocks hashed ahead of the chain

__device__ __forceinline__ uint64_t block_fnv(const int32_t* __restrict__ tk)
{
    uint64_t h = 0xcbf29ce484222325ull;
#pragma unroll
    for (int q = 0; q < 16; ++q) h = fnv_word(h, (uint32_t)tk[q]);
    return h;
}

__global__ __launch_bounds__(kFewThreads) void hash_few_kernel(int64_t n_seq, const int32_t* __restrict__ tokens,
                                                               const int64_t* __restrict__ tok_off,
                                                               const int64_t* __restrict__ chain_off,
                                                               uint64_t* __restrict__ chains, int32_t* status)
{
    __shared__ uint64_t s_f[2][kFewSpan];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    for (int64_t s = blockIdx.x; s < n_seq; s += gridDim.x) {
        const int64_t t0 = tok_off[s], t1 = tok_off[s + 1];
        const int64_t c0 = chain_off[s], c1 = chain_off[s + 1];
        if (t1 < t0 || c1 < c0) {
            if (tid == 0) atomicOr(status, RK_DEV_BAD_OFFSETS);
            continue;
        }
        const int64_t nb = c1 - c0, avail = (t1 - t0) / 16;
        if (nb > avail && tid == 0) atomicOr(status, RK_DEV_SHORT_INPUT);
        const int64_t n = nb < avail ? nb : avail;
        for (int64_t k = n + tid; k < nb; k += kFewThreads) chains[c0 + k] = 0ull;
        const int32_t* __restrict__ tk = tokens + t0;
        if (tid < n) s_f[0][tid] = block_fnv(tk + 16 * (int64_t)tid);
        __syncthreads();
        uint64_t h = 0;
        int cur = 0;
        for (int64_t k0 = 0; k0 < n; k0 += kFewSpan) {
            if (wave > 0) {
                for (int x = tid - 64; x < kFewSpan; x += kFewThreads - 64) {
                    const int64_t k = k0 + kFewSpan + x;
                    if (k < n) s_f[cur ^ 1][x] = block_fnv(tk + 16 * k);
                }
            } else {
                for (int64_t k1 = k0; k1 < k0 + kFewSpan && k1 < n; k1 += 64) {
                    const int m = (int)(n - k1 < 64 ? n - k1 : 64);
                    const uint64_t f = s_f[cur][(int)(k1 - k0) + lane];
                    int lo = 0, hi = 0;
                    auto step = [&](int x) {
                        h = chain_next(h, readlane64(f, x));
                        lo = writelane32((int)(uint32_t)h, x, lo);       // lane x keeps the value
                        hi = writelane32((int)(uint32_t)(h >> 32), x, hi);
                    };
                    int x = 0;
                    for (; x + 4 <= m; x += 4) {
                        step(x);
                        step(x + 1);
                        step(x + 2);
                        step(x + 3);
                    }
                    for (; x < m; ++x) step(x);
                    if (lane < m) chains[c0 + k1 + lane] = ((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo;
                }
            }
            __syncthreads();
            cur ^= 1;
        }
    }
}

// ------------------------------------------------------------------ tables
//
// As for the block index (index.hip): tables of 2^kTabLogMin .. 2^kTabLogMax
// slots are cut into bins of kTabBin consecutive slots, a workgroup sorts a tile
// of a worker's keys by bin in LDS and appends each run to the bin's list, which
// lies in the bin itself, and a workgroup per bin then loads the list, builds the
// bin in LDS and writes it over the list.  Keys that probe past a bin's end wait
// in a side buffer until every bin is built; what does not fit sets a flag that
// makes the last two launches build the tables by atomics.
// 64 tables of 2^20 slots from 33.6 M keys: 2.87 -> 0.43 ms; a quarter full, 1.19 -> 0.20 ms.  One launch for
// all workers, by atomics or not, takes the place of one for each (64 tables of 2^14 slots: 678 -> 47 us).
constexpr int kTabBinLog = 14, kTabBin = 1 << kTabBinLog;
constexpr int kTabLogMin = 15, kTabLogMax = 22;
constexpr int kTabBins = 1 << (kTabLogMax - kTabBinLog);      // at most, of a table
constexpr int kTabAllBins = 1 << 16;                          // at most, of a call
constexpr int kTabSpills = 1 << 15;
constexpr int64_t kTabSlotsMin = 1ll << 21;   // smaller calls: atomics (2^20 slots: 22-48 us against 34-43)

struct TableSide {
    int32_t overrun, n_spill, pad[30];
    uint32_t refilled[kTabAllBins >> (kTabLogMin - kTabBinLog + 6)];    // of every 64 tables: chunks of keys taken
    uint32_t cursor[kTabAllBins];
    uint64_t spill_key[kTabSpills];
    uint64_t spill_at[kTabSpills];                            // first slot to try (over all tables)
};
static __device__ TableSide g_table_side[kBuildSides];

static std::mutex g_table_mu;
static SidePool<TableSide> g_table_sides[64];

__global__ __launch_bounds__(256) void table_clear_kernel(uint64_t* __restrict__ t, uint64_t n, const int32_t* run)
{
    if (run && *run == 0) return;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (uint64_t)gridDim.x * blockDim.x)
        t[i] = kEmpty;
}

// Key into table t from slot s on, by atomics; false when there is no slot.  After kReads slots the walk
// reads a slot first: a slot read as taken stays so, and one read as empty may be taken by now, as the
// exchange tells.
constexpr uint64_t kNoReads = ~0ull;
template <uint64_t kReads>
__device__ __forceinline__ bool table_insert(uint64_t* t, uint64_t mask, uint64_t s, uint64_t key)
{
    for (uint64_t probe = 0; probe <= mask; ++probe) {
        uint64_t seen = kEmpty;
        if constexpr (kReads != kNoReads)
            if (probe >= kReads) seen = __hip_atomic_load(&t[s], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        if (seen == key) return true;
        if (seen == kEmpty) {
            const unsigned long long prev = atomicCAS((unsigned long long*)&t[s], (unsigned long long)kEmpty,
                                                      (unsigned long long)key);
            if (prev == kEmpty || prev == key) return true;
        }
        s = (s + 1) & mask;
    }
    return false;
}

template <uint64_t kReads>
__device__ __forceinline__ void table_insert_key(uint64_t* tables, int32_t log2_slots, int32_t j, uint64_t key,
                                                 int32_t* status)
{
    const uint64_t mask = (1ull << log2_slots) - 1;
    if (key == kEmpty) atomicOr(status, RK_DEV_ZERO_KEY);
    else if (!table_insert<kReads>(tables + ((uint64_t)j << log2_slots), mask, key & mask, key))
        atomicOr(status, RK_DEV_TABLE_FULL);
}

// blockIdx.y: the table, from j0 on
__global__ __launch_bounds__(256) void table_insert_kernel(const uint64_t* __restrict__ keys, KeyRanges r, int32_t j0,
                                                           uint64_t* __restrict__ tables, int32_t log2_slots,
                                                           int32_t* status)
{
    const int64_t n = r.off[blockIdx.y + 1];
    for (int64_t i = r.off[blockIdx.y] + (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        table_insert_key<kNoReads>(tables, log2_slots, j0 + (int32_t)blockIdx.y, keys[i], status);
}

// The keys of m <= 64 tables, from j0 on, if the partition did not fit.
__global__ __launch_bounds__(kRefillKeys) void table_refill_kernel(const uint64_t* __restrict__ keys, KeyRanges r,
                                                                   int32_t j0, int32_t m, uint64_t* __restrict__ tables,
                                                                   int32_t log2_slots, int32_t* status,
                                                                   TableSide* __restrict__ side)
{
    if (side->overrun == 0) return;
    refill(r, m, &side->refilled[j0 / 64],
           [&](int64_t i, int32_t j) { table_insert_key<8>(tables, log2_slots, j0 + j, keys[i], status); });
}

__global__ __launch_bounds__(256) void table_side_kernel(TableSide* __restrict__ side, int32_t bins)
{
    const int32_t i = (int32_t)(blockIdx.x * blockDim.x + threadIdx.x);
    if (i == 0) {
        side->overrun = 0;
        side->n_spill = 0;
    }
    if (i < bins) side->cursor[i] = 0u;
    if (i < (int32_t)(sizeof side->refilled / sizeof side->refilled[0])) side->refilled[i] = 0u;
}

// Keys to the bins' lists.  blockIdx.x: the table, from j0 on, of m, then the tile of its keys: all
// tables' first keys go first, as they did by atomics, so that keys given early lie close to their
// home slots (scoring 65,536 x 64 with the prefixes' keys first: 398 us; 413 with the workers one
// after another).  A table has at most 2^21 keys here, so a launch has at most 2^14 workgroups.
__global__ __launch_bounds__(kBuildThreads) void table_scatter_kernel(const uint64_t* __restrict__ keys, KeyRanges r,
                                                                      int32_t j0, int32_t m, uint64_t* __restrict__ tables,
                                                                      int32_t log2_slots, TableSide* __restrict__ side,
                                                                      int32_t* status)
{
    __shared__ uint64_t s_ent[kTile];
    __shared__ uint8_t s_bin[kTile];
    __shared__ uint32_t s_cnt[kTabBins], s_off[kTabBins], s_gbase[kTabBins], s_tmp[16];
    const int tid = threadIdx.x;
    const int32_t jr = (int32_t)(blockIdx.x % (uint32_t)m), j = j0 + jr;
    const int64_t n0 = r.off[jr] + (int64_t)(blockIdx.x / (uint32_t)m) * kTile, n1 = r.off[jr + 1];
    if (n0 >= n1) return;
    const uint32_t bins = 1u << (log2_slots - kTabBinLog);
    if (tid < kTabBins) s_cnt[tid] = 0u;
    __syncthreads();
    uint64_t key[kTile / kBuildThreads];
    uint32_t rank[kTile / kBuildThreads];
#pragma unroll
    for (int u = 0; u < kTile / kBuildThreads; ++u) {
        const int64_t i = n0 + u * kBuildThreads + tid;
        key[u] = i < n1 ? keys[i] : kEmpty;
        if (i < n1 && key[u] == kEmpty) atomicOr(status, RK_DEV_ZERO_KEY);
    }
#pragma unroll
    for (int u = 0; u < kTile / kBuildThreads; ++u) {
        const uint32_t b = (uint32_t)(key[u] >> kTabBinLog) & (bins - 1);
        rank[u] = key[u] != kEmpty ? atomicAdd(&s_cnt[b], 1u) : 0u;
    }
    __syncthreads();
    if (tid < kTabBins) {
        const uint32_t c = s_cnt[tid];
        s_off[tid] = c;
        uint32_t g = 0;
        if (c) {
            g = atomicAdd(&side->cursor[(uint32_t)j * bins + (uint32_t)tid], c);
            if (g + c > (uint32_t)kTabBin) {
                atomicOr(&side->overrun, 1);
                g = 0xFFFFFFFFu;                             // no room: not written
            }
        }
        s_gbase[tid] = g;
    }
    __syncthreads();
    build_scan(s_off, kTabBins, s_tmp);
#pragma unroll
    for (int u = 0; u < kTile / kBuildThreads; ++u) {
        if (key[u] == kEmpty) continue;
        const uint32_t b = (uint32_t)(key[u] >> kTabBinLog) & (bins - 1);
        const uint32_t p = s_off[b] + rank[u];
        s_ent[p] = key[u];
        s_bin[p] = (uint8_t)b;
    }
    __syncthreads();
    const uint32_t total = s_off[kTabBins - 1] + s_cnt[kTabBins - 1];
    for (uint32_t p = tid; p < total; p += kBuildThreads) {
        const uint32_t b = s_bin[p], g = s_gbase[b];
        if (g == 0xFFFFFFFFu) continue;
        tables[((uint64_t)j << log2_slots) + ((uint64_t)b << kTabBinLog) + g + (p - s_off[b])] = s_ent[p];
    }
}

// A bin from its list.  blockIdx.x: the bin, over all tables.
template <bool PastCaches>
__global__ __launch_bounds__(kBuildThreads) void table_bin_kernel(uint64_t* __restrict__ tables, int32_t log2_slots,
                                                                  TableSide* __restrict__ side)
{
    extern __shared__ __align__(16) uint64_t s_key[];        // [kTabBin]
    __shared__ int32_t s_over;
    const int tid = threadIdx.x;
    if (tid == 0) s_over = side->overrun;
    __syncthreads();
    if (s_over) return;
    const uint32_t n = side->cursor[blockIdx.x];
    uint64_t* bin = tables + ((uint64_t)blockIdx.x << kTabBinLog);
    for (int i = tid; i < kTabBin; i += kBuildThreads) s_key[i] = kEmpty;
    __syncthreads();
    for (uint32_t i = tid; i < n; i += kBuildThreads) {
        const uint64_t key = bin[i];
        uint32_t s = (uint32_t)key & (kTabBin - 1);
        for (; s < (uint32_t)kTabBin; ++s) {
            const unsigned long long prev = atomicCAS((unsigned long long*)&s_key[s], (unsigned long long)kEmpty,
                                                      (unsigned long long)key);
            if (prev == kEmpty || prev == key) break;
        }
        if (s == (uint32_t)kTabBin) {
            const int32_t x = atomicAdd(&side->n_spill, 1);
            if (x < kTabSpills) {
                // the next bin's first slot, within the table
                const uint64_t mask = (1ull << log2_slots) - 1, at = (uint64_t)(blockIdx.x + 1) << kTabBinLog;
                side->spill_key[x] = key;
                side->spill_at[x] = (((uint64_t)blockIdx.x << kTabBinLog) & ~mask) | (at & mask);
            } else {
                atomicOr(&side->overrun, 1);
            }
        }
    }
    __syncthreads();
    for (int i = tid; i < kTabBin; i += kBuildThreads) {
        if constexpr (PastCaches) __builtin_nontemporal_store(s_key[i], bin + i);
        else bin[i] = s_key[i];
    }
}

__global__ __launch_bounds__(256) void table_spill_kernel(uint64_t* __restrict__ tables, int32_t log2_slots,
                                                          TableSide* __restrict__ side, int32_t* status)
{
    if (side->overrun) return;
    const uint64_t mask = (1ull << log2_slots) - 1;
    for (int32_t x = (int32_t)(blockIdx.x * blockDim.x + threadIdx.x); x < side->n_spill; x += gridDim.x * blockDim.x) {
        const uint64_t at = side->spill_at[x];
        if (!table_insert<kNoReads>(tables + (at & ~mask), mask, at & mask, side->spill_key[x])) atomicOr(status, RK_DEV_TABLE_FULL);
    }
}

}  // namespace rk

using namespace rk;

// The partitioned build of tables with `total` slots in all (scatter and refill launch the keys' kernels);
// RK_OK with *done = false when it is not for this call.
template <class Scatter, class Refill>
static int table_build_parts(uint64_t total, int32_t log2_slots, uint64_t* tables, hipStream_t s, const Scatter& scatter,
                             const Refill& refill, int32_t* st, bool* done)
{
    *done = false;
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &cap) != hipSuccess) {
        (void)hipGetLastError();
        return RK_OK;
    }
    if (cap != hipStreamCaptureStatusNone) return RK_OK;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return RK_OK;
    std::lock_guard<std::mutex> lk(g_table_mu);
    SidePool<TableSide>& b = g_table_sides[dev];
    if (!b.addr) {
        void* p = nullptr;
        int rc = hip_check(hipGetSymbolAddress(&p, HIP_SYMBOL(g_table_side)), "rk_table_build side buffers");
        if (!rc) rc = b.make_events("rk_table_build event");
        if (rc) return rc;
        b.addr = (TableSide*)p;
    }
    const int k = b.take(s);
    if (k < 0) return RK_OK;
    TableSide* side = b.addr + k;
    // (a stream's handle may be that of a stream destroyed with its work under way)
    int rc = b.once[k] ? hip_check(hipStreamWaitEvent(s, b.used[k], 0), "rk_table_build wait") : RK_OK;
    if (rc) return rc;
    *done = true;
    const unsigned bins = (unsigned)(total >> kTabBinLog);
    hipLaunchKernelGGL(table_side_kernel, dim3((bins + 255) / 256), dim3(256), 0, s, side, (int32_t)bins);
    scatter(side);
    if (total * sizeof(uint64_t) > kCacheBytes)
        hipLaunchKernelGGL(table_bin_kernel<true>, dim3(bins), dim3(kBuildThreads), 8 * kTabBin, s, tables, log2_slots, side);
    else
        hipLaunchKernelGGL(table_bin_kernel<false>, dim3(bins), dim3(kBuildThreads), 8 * kTabBin, s, tables, log2_slots, side);
    hipLaunchKernelGGL(table_spill_kernel, dim3(16), dim3(256), 0, s, tables, log2_slots, side, st);
    hipLaunchKernelGGL(table_clear_kernel, dim3(1024), dim3(256), 0, s, tables, total, &side->overrun);
    refill(side);
    rc = hip_check(hipGetLastError(), "rk_table_build launch");
    const int re = b.record(k, s, "rk_table_build record");
    return rc ? rc : re;
}

extern "C" {

const char* rk_status_string(int status)
{
    switch (status) {
    case RK_OK: return "ok";
    case RK_EINVAL: return "invalid argument";
    case RK_ENOMEM: return "workspace too small";
    case RK_EHIP: return "HIP runtime error";
    case RK_ETABLEFULL: return "table full";
    case RK_EUNSUPPORTED: return "unsupported size";
    default: return "unknown status";
    }
}

const char* rk_last_error(void) { return g_last_error; }

int rk_device_status(int reset, int32_t* bits, void* stream)
{
    if (!bits) return fail(RK_EINVAL, "rk_device_status: bits is NULL");
    int32_t* p = status_word();
    if (!p) return fail(RK_EHIP, "rk_device_status: no status word on this device");
    hipStream_t st = (hipStream_t)stream;
    int rc = hip_check(hipMemcpyAsync(bits, p, sizeof(int32_t), hipMemcpyDeviceToHost, st),
                       "rk_device_status copy");
    if (rc) return rc;
    rc = hip_check(hipStreamSynchronize(st), "rk_device_status sync");
    if (rc) return rc;
    if (reset) {
        rc = hip_check(hipMemsetAsync(p, 0, sizeof(int32_t), st), "rk_device_status reset");
        if (rc) return rc;
        rc = hip_check(hipStreamSynchronize(st), "rk_device_status sync");
    }
    return rc;
}

int rk_hash_chains(int64_t n_seq, const int32_t* tokens, const int64_t* tok_off,
                   const int64_t* chain_off, uint64_t* chains, void* stream)
{
    if (n_seq < 0) return fail(RK_EINVAL, "rk_hash_chains: n_seq < 0");
    if (n_seq == 0) return RK_OK;
    if (!tokens || !tok_off || !chain_off || !chains)
        return fail(RK_EINVAL, "rk_hash_chains: NULL array");
    int32_t* st = status_word();
    if (!st) return fail(RK_EHIP, "rk_hash_chains: no status word");
    hipStream_t s = (hipStream_t)stream;
    if (n_seq <= kFewSeqs) {
        hipLaunchKernelGGL(hash_few_kernel, dim3((unsigned)n_seq), dim3(kFewThreads), 0, s, n_seq, tokens, tok_off,
                           chain_off, chains, st);
        return hip_check(hipGetLastError(), "rk_hash_chains launch");
    }
    const int64_t waves_per_block = 4;
    int64_t blocks = (n_seq + waves_per_block - 1) / waves_per_block;
    if (blocks > 65536) blocks = 65536;
    hipLaunchKernelGGL(block_fnv_kernel, dim3((unsigned)blocks), dim3(256), 0, s, n_seq, tokens, tok_off,
                       chain_off, chains, st);
    int rc = hip_check(hipGetLastError(), "rk_hash_chains fnv launch");
    if (rc) return rc;
    const int64_t cblocks = (n_seq + kChainWG - 1) / kChainWG;
    hipLaunchKernelGGL(chain_kernel, dim3((unsigned)cblocks), dim3(kChainWG), 0, s, n_seq, tok_off, chain_off,
                       chains);
    return hip_check(hipGetLastError(), "rk_hash_chains chain launch");
}

int rk_table_build(int32_t W, const uint64_t* keys, const int64_t* key_off, uint64_t* tables,
                   int32_t log2_slots, void* stream)
{
    if (W < 1) return fail(RK_EINVAL, "rk_table_build: W < 1");
    if (log2_slots < 4 || log2_slots > 30) return fail(RK_EINVAL, "rk_table_build: log2_slots out of 4..30");
    if (!key_off || !tables) return fail(RK_EINVAL, "rk_table_build: NULL array");
    const uint64_t slots = 1ull << log2_slots;
    for (int32_t j = 0; j < W; ++j) {
        const int64_t n = key_off[j + 1] - key_off[j];
        if (n < 0) return fail(RK_EINVAL, "rk_table_build: key_off not monotone at %d", j);
        if ((uint64_t)n > slots / 2)
            return fail(RK_ETABLEFULL, "rk_table_build: table %d gets %lld keys for %llu slots", j,
                        (long long)n, (unsigned long long)slots);
    }
    if (key_off[W] > 0 && !keys) return fail(RK_EINVAL, "rk_table_build: keys is NULL");
    int32_t* st = status_word();
    if (!st) return fail(RK_EHIP, "rk_table_build: no status word");
    hipStream_t s = (hipStream_t)stream;
    const uint64_t total = slots * (uint64_t)W;
    // the workers' keys, 64 at a time
    auto chunk = [&](int32_t j0, KeyRanges& r, int64_t& longest) {
        const int32_t m = W - j0 < 64 ? W - j0 : 64;
        longest = 0;
        for (int32_t k = 0; k <= m; ++k) r.off[k] = key_off[j0 + k];
        for (int32_t k = 0; k < m; ++k) longest = r.off[k + 1] - r.off[k] > longest ? r.off[k + 1] - r.off[k] : longest;
        return m;
    };
    bool done = false;
    if (log2_slots >= kTabLogMin && log2_slots <= kTabLogMax && total >= (uint64_t)kTabSlotsMin &&
        total >> kTabBinLog <= (uint64_t)kTabAllBins) {
        const int rc = table_build_parts(total, log2_slots, tables, s, [&](TableSide* side) {
            for (int32_t j0 = 0; j0 < W; j0 += 64) {
                KeyRanges r;
                int64_t longest;
                const int32_t m = chunk(j0, r, longest);
                if (longest == 0) continue;
                hipLaunchKernelGGL(table_scatter_kernel, dim3((unsigned)((longest + kTile - 1) / kTile * m)),
                                   dim3(kBuildThreads), 0, s, keys, r, j0, m, tables, log2_slots, side, st);
            }
        }, [&](TableSide* side) {
            for (int32_t j0 = 0; j0 < W; j0 += 64) {
                KeyRanges r;
                int64_t longest;
                const int32_t m = chunk(j0, r, longest);
                if (longest == 0) continue;
                hipLaunchKernelGGL(table_refill_kernel, dim3(refill_blocks(r.off[m] - r.off[0])), dim3(kRefillKeys), 0, s,
                                   keys, r, j0, m, tables, log2_slots, st, side);
            }
        }, st, &done);
        if (rc || done) return rc;
    }
    uint64_t blocks = (total + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    hipLaunchKernelGGL(table_clear_kernel, dim3((unsigned)blocks), dim3(256), 0, s, tables, total, (const int32_t*)nullptr);
    int rc = hip_check(hipGetLastError(), "rk_table_build clear launch");
    if (rc) return rc;
    for (int32_t j0 = 0; j0 < W; j0 += 64) {
        KeyRanges r;
        int64_t longest;
        const int32_t m = chunk(j0, r, longest);
        if (longest == 0) continue;
        int64_t b = (longest + 255) / 256;
        if (b > 65536) b = 65536;
        hipLaunchKernelGGL(table_insert_kernel, dim3((unsigned)b, (unsigned)m), dim3(256), 0, s, keys, r, j0, tables,
                           log2_slots, st);
    }
    return hip_check(hipGetLastError(), "rk_table_build insert launch");
}

}  // extern "C"
