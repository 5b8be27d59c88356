// index.hip -- the router's global block index (block hash -> set of workers
// caching that block) and batched routing-cost evaluation against it.
//
// The router the paper studies answers "which workers hold this prefix" from
// one index over all workers (the global radix tree of the Smart Router in the
// Dynamo architecture background section, queried by best_worker in
// Alg. adaptive-router).  Chained block hashes name prefixes uniquely, so the radix tree
// becomes one open-addressing table of 16-byte slots (key, worker mask) and a
// single probe answers membership on all W <= 64 workers at once.  Scoring a
// request then costs a few lane-parallel probe rounds per request instead of
// a search per (request, worker) pair:
//   - PREFIX mode (every worker's set is prefix-closed along the chains):
//     worker masks along a chain only lose bits.  A coarse round (16
//     samples) bounds the region [0, U) where any worker may still hold the
//     chain, a second round samples it with 64 lanes (every position when
//     U <= 64), and a third probes the inside of the sample intervals where
//     some worker's bit disappears.  Worker j's overlap is the first
//     position whose mask lacks bit j.
//   - SCAN mode (any sets): positions from block 0 in rounds of 64; a
//     running AND of the masks gives each worker's first miss exactly, and
//     the scan stops once no worker is left.
// One wavefront scores two consecutive requests; lane j owns worker j's
// overlap and cost.
#include <hip/hip_runtime.h>

#include <mutex>

#include "rk_internal.h"

namespace rk {

struct __align__(16) IndexSlot {
    uint64_t key;
    uint64_t mask;
};

__device__ __forceinline__ void load_slot(const IndexSlot* t, uint64_t s, uint64_t& k, uint64_t& m)
{
    const uint4 v = *reinterpret_cast<const uint4*>(t + s);
    k = (uint64_t)v.x | ((uint64_t)v.y << 32);
    m = (uint64_t)v.z | ((uint64_t)v.w << 32);
}

// Worker mask of block hash h (0 when no worker holds it): linear probing
// one 16-byte slot per access from the home slot h & smask.  At the loads the
// index is sized for, the home slot settles almost every lookup, and one slot
// costs the smallest read the memory system serves; wider windows (an aligned
// 32- or 64-byte group per access) moved more bytes per lookup and ran slower.
__device__ __forceinline__ uint64_t index_lookup(const IndexSlot* __restrict__ t, uint64_t smask, uint64_t h)
{
    uint64_t s = h & smask;
    for (uint64_t n = 0; n <= smask; ++n) {
        uint64_t k, m;
        load_slot(t, s, k, m);
        if (k == h) return m;
        if (k == kEmpty) return 0ull;
        s = (s + 1) & smask;
    }
    return 0ull;
}

// First index in [lo, hi) whose mask lacks bit j, for masks in which bit j
// never comes back once cleared; hi if none.
__device__ __forceinline__ int32_t first_clear(const uint64_t* m, int32_t lo, int32_t hi, int32_t j)
{
    while (lo < hi) {
        const int32_t mid = (lo + hi) >> 1;
        if ((m[mid] >> j) & 1ull) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

__device__ __forceinline__ uint32_t next_pow2_dev(uint32_t x)
{
    return x <= 1u ? 1u : 1u << (32 - __clz((int)(x - 1u)));
}

// LDS writes of one wavefront made visible to the other lanes of that wavefront.
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

constexpr int kRPW = 2;           // requests per wavefront: their offsets and chains are loaded together
constexpr int kRound1Min = 64;    // chains longer than this get the coarse first round
constexpr int kStage = 256;       // leading chain blocks staged in LDS, read in one coalesced pass
constexpr int kStageRegs = kStage / 64;

struct IdxLds {
    uint64_t ch[kRPW][kStage];   // the first kStage chain hashes of each of the wavefront's requests
    uint64_t m[64];              // masks of the current round (prefix ANDs in rounds 1-2)
    int32_t ioff[65];            // start of each sample interval's positions in the third round
};

constexpr int kFewBounds = 8;     // boundaries handled by a scalar loop; more take the LDS search
constexpr int kDppWaveShr1 = 0x138;   // DPP: every lane takes lane - 1's value (lane 0 keeps old)

__device__ __forceinline__ uint32_t wave_min_u32(uint32_t v)
{
    auto mn = [](uint32_t a, uint32_t b) { return b < a ? b : a; };
    v = mn(v, dpp32<kDppQuadSwap1>(v, v));
    v = mn(v, dpp32<kDppQuadSwap2>(v, v));
    v = mn(v, dpp32<kDppRowHalfMirror>(v, v));
    v = mn(v, dpp32<kDppRowMirror>(v, v));
    const auto rl = [&](int l) { return (uint32_t)__builtin_amdgcn_readlane((int)v, l); };
    return mn(mn(rl(0), rl(16)), mn(rl(32), rl(48)));
}

// The router cost (Section 2.2, Eq. router-cost) in the operation order of
// route_cost; when cap is a power of two, (A + P) / cap is the exact product
// with 1 / cap.
__device__ __forceinline__ float index_route_cost(const rk_cost_params& p, float inv_cap, int32_t P, int32_t o,
                                                  int32_t A)
{
    const float t1 = __fmul_rn(p.w_ov, (float)(P - o));
    const float t2 = __fmul_rn(p.w_act, (float)A);
    const float L = (float)((int64_t)A + (int64_t)P);
    const float r = inv_cap != 0.0f ? __fmul_rn(L, inv_cap) : __fdiv_rn(L, (float)p.cap_blocks);
    const float x = fmaxf(__fsub_rn(r, 1.0f), 0.0f);
    const float t3 = __fmul_rn(p.w_sat, __fmul_rn(x, x));
    return __fadd_rn(__fadd_rn(t1, t2), t3);
}

// Position of second-round sample k: every position when the round is exact,
// else the power-of-two grid of step st2, clamped to U - 1.
__device__ __forceinline__ int32_t round2_pos(int32_t k, bool exact, int64_t st2, int32_t U)
{
    return exact ? k : (int32_t)min((int64_t)(k + 1) * st2, (int64_t)U) - 1;
}

// One wavefront scores kRPW consecutive requests; lane j owns worker j.  The
// requests' chain offsets come in one load and their leading chain blocks in
// one coalesced pass into LDS, so only the first request waits for them.
template <int MODE>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(8))) void score_index_kernel(
    int32_t B, int32_t W, const uint64_t* __restrict__ chains, const int64_t* __restrict__ chain_off,
    const IndexSlot* __restrict__ index, int32_t log2_slots, const int32_t* __restrict__ active, rk_cost_params p,
    int32_t* __restrict__ ov_out, float* __restrict__ cost_out, int32_t* __restrict__ am_out, int32_t* status)
{
    __shared__ IdxLds L;
    const int32_t lane = threadIdx.x & 63;
    const uint64_t smask = (1ull << log2_slots) - 1;
    const int32_t A = lane < W ? active[lane] : 0;
    const uint64_t all = W == 64 ? ~0ull : ((1ull << W) - 1ull);
    const float inv_cap = (p.cap_blocks & (p.cap_blocks - 1)) == 0 ? 1.0f / (float)p.cap_blocks : 0.0f;
    const int64_t npairs = ((int64_t)B + kRPW - 1) / kRPW;

    // Workgroups are handed to the 8 XCDs round-robin; renumber them so each
    // XCD walks one contiguous range of requests (gridDim.x is a multiple of 8).
    const uint32_t nb8 = gridDim.x >> 3;
    const uint32_t lb = (blockIdx.x & 7u) * nb8 + (blockIdx.x >> 3);
    for (int64_t g = lb; g < npairs; g += gridDim.x) {
        const int64_t i0 = g * kRPW;
        const int32_t nr = (int32_t)min((int64_t)kRPW, (int64_t)B - i0);
        const int64_t offv = lane <= nr ? chain_off[i0 + lane] : 0;
        int64_t c[kRPW + 1];
#pragma unroll
        for (int r = 0; r <= kRPW; ++r) c[r] = (int64_t)readlane64((uint64_t)offv, r);
        int32_t Pr[kRPW];
#pragma unroll
        for (int r = 0; r < kRPW; ++r) {
            Pr[r] = 0;
            if (r < nr) {
                if (c[r + 1] < c[r] || c[r + 1] - c[r] > 0x7fffffff) {
                    if (lane == 0) atomicOr(status, RK_DEV_BAD_OFFSETS);
                } else {
                    Pr[r] = (int32_t)(c[r + 1] - c[r]);
                }
            }
        }
        wave_sync();   // the previous requests' reads of L.ch are done
        {
            uint64_t v[kRPW][kStageRegs];
#pragma unroll
            for (int r = 0; r < kRPW; ++r) {
                const int32_t n = min(Pr[r], kStage);
                const uint64_t* __restrict__ hg = chains + c[r];
#pragma unroll
                for (int k = 0; k < kStageRegs; ++k) v[r][k] = lane + 64 * k < n ? hg[lane + 64 * k] : 0ull;
            }
#pragma unroll
            for (int r = 0; r < kRPW; ++r)
#pragma unroll
                for (int k = 0; k < kStageRegs; ++k) L.ch[r][lane + 64 * k] = v[r][k];
        }
        wave_sync();

        for (int32_t r = 0; r < nr; ++r) {
            const int64_t i = i0 + r;
            const int32_t P = Pr[r];
            const uint64_t* __restrict__ hg = chains + c[r];
            const uint64_t* ch = L.ch[r];
            auto h = [&](int32_t x) -> uint64_t { return x < kStage ? ch[x] : hg[x]; };
            int32_t o = 0;   // lane j: overlap on worker j

            if (MODE == RK_PROBE_SCAN) {
                uint64_t carry = all;
                bool done = false;
                for (int32_t base = 0; base < P && carry != 0ull; base += 64) {
                    const int32_t n = min(64, P - base);
                    const uint64_t m = lane < n ? index_lookup(index, smask, h(base + lane)) : 0ull;
                    const uint64_t pa = wave_scan_and_u64(m) & carry;
                    L.m[lane] = pa;
                    wave_sync();
                    if (lane < W && !done) {
                        const int32_t f = first_clear(L.m, 0, n, lane);
                        o += f;
                        done = f < n;
                    }
                    carry = readlane64(pa, n - 1);
                    wave_sync();
                }
            } else {
                // ---- round 1: every worker's first miss lies in [0, U).  Sample
                // positions sit on a power-of-two grid (clamped to the chain's end)
                // so requests of one prefix group probe the same index slots.
                // Masks along a chain only lose bits, so the first sample with an
                // empty mask bounds every worker.
                int32_t U = P;
                if (P > kRound1Min) {
                    const int64_t st1 = (int64_t)next_pow2_dev((uint32_t)P) >> 4;
                    const int32_t q1 = (int32_t)min((int64_t)(lane + 1) * st1, (int64_t)P) - 1;
                    const uint64_t m1 = lane < 16 ? index_lookup(index, smask, h(q1)) & all : all;
                    const uint64_t z = __ballot(m1 == 0ull);
                    if (z) U = __builtin_amdgcn_readlane(q1, __ffsll((unsigned long long)z) - 1) + 1;
                }
                // ---- round 2: every position of [0, U) when U <= 64, else 64 samples
                // on the power-of-two grid of step next_pow2(U) / 64, clamped to U - 1.
                // Sample k is a boundary when its mask lacks bits its predecessor's
                // had (all W bits before sample 0); worker j's first missing sample
                // t is the boundary that drops bit j.  A request has few boundaries
                // (one per distinct overlap), so a loop over them costs a few scalar
                // steps; many boundaries fall back to a search per worker in LDS.
                const bool exact = U <= 64;
                const int32_t nq = exact ? U : 64;
                const int64_t st2 = (int64_t)next_pow2_dev((uint32_t)U) >> 6;
                const int32_t q = round2_pos(lane, exact, st2, U);
                const uint64_t m = lane < nq ? index_lookup(index, smask, h(q)) & all : 0ull;
                const uint64_t mp = dpp64<kDppWaveShr1>(all, m);   // sample lane - 1's mask
                const uint64_t bnd = __ballot(lane < nq && mp != m);
                const bool few = __popcll(bnd) <= kFewBounds;
                int32_t t = nq;
                if (few) {
                    for (uint64_t b = bnd; b; b &= b - 1) {
                        const int k = __ffsll((unsigned long long)b) - 1;
                        if ((((readlane64(mp, k) & ~readlane64(m, k)) >> lane) & 1ull)) t = k;
                    }
                } else {
                    L.m[lane] = m;
                    wave_sync();
                    if (lane < W) t = first_clear(L.m, 0, nq, lane);
                    wave_sync();
                }
                if (exact) {
                    o = t;   // t == U only when U == P: every position is cached
                } else {
                    // ---- round 3: worker j's first miss is in (q[t-1], q[t]]; probe the
                    // inside of the boundary intervals, laid out one after another.
                    const int32_t qprev = (int32_t)dpp32<kDppWaveShr1>(0xffffffffu, (uint32_t)q);
                    const bool mine = lane < W && t < 64;
                    o = mine ? round2_pos(t, false, st2, U) : P;
                    int32_t pos = -1, a0 = 0, a1 = 0, pb = 0, nb3 = 0;
                    uint64_t pstart = 0ull;   // the mask before the lane's position when it opens an interval
                    bool opens = false;
                    if (few) {
                        for (uint64_t b = bnd; b; b &= b - 1) {
                            const int k = __ffsll((unsigned long long)b) - 1;
                            const int32_t qk = __builtin_amdgcn_readlane(q, k), qpk = __builtin_amdgcn_readlane(qprev, k);
                            const int32_t w = max(qk - qpk - 1, 0);
                            if (lane >= nb3 && lane < nb3 + w) pos = qpk + 1 + (lane - nb3);
                            if (w > 0 && lane == nb3) {
                                opens = true;
                                pstart = readlane64(mp, k);
                            }
                            if (t == k) {
                                a0 = nb3;
                                a1 = nb3 + w;
                                pb = qpk + 1;
                            }
                            nb3 += w;
                        }
                    }
                    if (few && nb3 <= 64) {
                        const uint64_t mm = pos >= 0 ? index_lookup(index, smask, h(pos)) & all : 0ull;
                        // the shift runs on every lane (a lane whose source lane sat out
                        // would receive the fill value), then the lanes that open an
                        // interval take the mask before it instead
                        const uint64_t left = dpp64<kDppWaveShr1>(all, mm);
                        const uint64_t pv = opens ? pstart : left;
                        const uint64_t b3 = __ballot(pos >= 0 && pv != mm);
                        if (__popcll(b3) <= kFewBounds) {
                            for (uint64_t b = b3; b; b &= b - 1) {
                                const int x = __ffsll((unsigned long long)b) - 1;
                                if ((((readlane64(pv, x) & ~readlane64(mm, x)) >> lane) & 1ull))
                                    o = __builtin_amdgcn_readlane(pos, x);
                            }
                        } else {
                            L.m[lane] = mm;
                            wave_sync();
                            if (mine && a1 > a0) {
                                const int32_t f = first_clear(L.m, a0, a1, lane);
                                if (f < a1) o = pb + (f - a0);
                            }
                            wave_sync();
                        }
                    } else {
                        // many boundaries or more than 64 positions: chunks of 64
                        // positions, each lane finding its interval by binary search
                        const int32_t width = ((bnd >> lane) & 1ull) ? max(q - qprev - 1, 0) : 0;
                        int32_t total;
                        const int32_t off = wave_excl_sum_dpp(width, total);
                        L.ioff[lane] = off;
                        if (lane == 63) L.ioff[64] = total;
                        wave_sync();
                        const int32_t c0 = mine ? L.ioff[t] : 0, c1 = mine ? L.ioff[t + 1] : 0;
                        const int32_t pbase = mine ? (t == 0 ? 0 : round2_pos(t - 1, false, st2, U) + 1) : 0;
                        bool found = !mine;
                        for (int32_t b3 = 0; b3 < total; b3 += 64) {
                            const int32_t idx = b3 + lane;
                            uint64_t mm = 0ull;
                            if (idx < total) {
                                int32_t lo = 0, hi = 63;   // largest k with ioff[k] <= idx
                                while (lo < hi) {
                                    const int32_t mid = (lo + hi + 1) >> 1;
                                    if (L.ioff[mid] <= idx) lo = mid;
                                    else hi = mid - 1;
                                }
                                const int32_t p3 = (lo == 0 ? 0 : round2_pos(lo - 1, false, st2, U) + 1) +
                                                   (idx - L.ioff[lo]);
                                mm = index_lookup(index, smask, h(p3)) & all;
                            }
                            wave_sync();   // the previous chunk's masks have been read
                            L.m[lane] = mm;
                            wave_sync();
                            if (!found) {
                                const int32_t lo = max(c0, b3), hi = min(c1, b3 + 64);
                                if (lo < hi) {
                                    const int32_t x = first_clear(L.m, lo - b3, hi - b3, lane) + b3;
                                    if (x < hi) {
                                        o = pbase + (x - c0);
                                        found = true;
                                    }
                                }
                            }
                        }
                        wave_sync();   // L.m and L.ioff are free for the next request
                    }
                }
            }

            // cost per worker; argmin = the lowest worker among those of minimal
            // cost (non-negative floats order as their bit patterns)
            uint32_t cb = 0xffffffffu;
            if (lane < W) {
                const float cst = index_route_cost(p, inv_cap, P, o, A);
                if (ov_out) ov_out[i * W + lane] = o;
                if (cost_out) cost_out[i * W + lane] = cst;
                cb = __float_as_uint(__fadd_rn(cst, 0.0f));
            }
            const uint32_t cmin = wave_min_u32(cb);
            const uint64_t win = __ballot(lane < W && cb == cmin);
            if (lane == 0 && am_out) am_out[i] = __ffsll((unsigned long long)win) - 1;
        }
    }
}

// ---------------------------------------------------------------- building the index
//
// Inserting every key where it belongs costs two atomics and a line of memory
// read and written back per key, at random.  From 2^kPartLog slots on the keys
// are partitioned first and each part of the index is built in LDS and written
// once, in order:
//   1. index_scatter_kernel: the index is cut into kBins bins of consecutive
//      slots; a workgroup sorts a tile of kTile keys by bin in LDS and appends
//      each bin's run to the bin's list.  The lists lie in the index itself, a
//      bin's in the upper half of its slots.  An entry is the key with the bin's
//      bits of its home slot (known from the list) replaced by the worker.
//   2. index_bin_kernel, a workgroup per bin: the list is sorted by sub-bin of
//      kSub slots into the bin's lower half, then each sub-bin, from the last to
//      the first, is built in LDS (linear probing with LDS atomics, as in the
//      index) and written out over lists that are done with.  Keys that probe
//      past a sub-bin's end (each counted once, however many workers hold it: a
//      prefix cached everywhere comes 64 times) go on by global atomics in the
//      next ones, which are final by then, and those that leave the bin wait in
//      a side buffer.
//   3. index_spill_kernel inserts the waiting ones.
// Whatever does not fit this (a list or a side buffer that runs over, from keys
// whose low bits are far from uniform) sets a flag that makes the last two
// launches, otherwise empty, clear the index and insert every key by atomics.
// The side buffers belong to the library, kBuildSides per device (SidePool).  When
// other streams' calls have all of them in use, and while the stream is captured
// (its graph may run at any time), the keys are inserted by atomics, all workers
// in one launch.
//
// 33.6 M keys of 64 workers into 2^27 slots (2 GiB): 4.22 -> 0.81 ms (the keys read twice and written twice, the
// index written once: 3.5 GB, 4.3 TB/s; a large copy moves 4.8); twice the keys 9.90 -> 1.49 ms.
constexpr int kPartLog = 20;              // smallest index that is partitioned (below: 20-40 us by atomics)
constexpr int kBinLog = 8, kBins = 1 << kBinLog;
constexpr int kSubLog = 13, kSub = 1 << kSubLog;
constexpr int kSpills = 64;               // keys that may probe past a sub-bin's end, and past a bin's
constexpr int kMaxSubs = 1 << (31 - kBinLog - kSubLog);

struct BuildSide {
    int32_t overrun;                      // the partition does not fit: insert by atomics
    uint32_t refilled;                    // and the chunks of keys taken for that
    int32_t n_spill[kBins];
    uint32_t cursor[kBins * 32];          // one per 128-byte line
    uint64_t spill_key[kBins * kSpills];
    uint64_t spill_mask[kBins * kSpills];
};
static __device__ BuildSide g_build_side[kBuildSides];

__global__ __launch_bounds__(256) void index_clear_kernel(IndexSlot* __restrict__ t, uint64_t n, const int32_t* run)
{
    if (run && *run == 0) return;
    const uint4 zero = make_uint4(0u, 0u, 0u, 0u);
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x)
        *reinterpret_cast<uint4*>(t + i) = zero;
}

// Key into the index from slot s on (bits of the mask added), by atomics; false when there is no slot.
__device__ __forceinline__ bool index_insert(IndexSlot* t, uint64_t smask, uint64_t s, uint64_t key, uint64_t mask)
{
    for (uint64_t probe = 0; probe <= smask; ++probe) {
        const unsigned long long prev = atomicCAS((unsigned long long*)&t[s].key, (unsigned long long)kEmpty,
                                                  (unsigned long long)key);
        if (prev == kEmpty || prev == key) {
            atomicOr((unsigned long long*)&t[s].mask, (unsigned long long)mask);
            return true;
        }
        s = (s + 1) & smask;
    }
    return false;
}

__device__ __forceinline__ void index_insert_key(IndexSlot* t, uint64_t smask, uint64_t key, int32_t j, int32_t* status)
{
    if (key == kEmpty) atomicOr(status, RK_DEV_ZERO_KEY);
    else if (!index_insert(t, smask, key & smask, key, 1ull << j)) atomicOr(status, RK_DEV_TABLE_FULL);
}

// blockIdx.y: the worker
__global__ __launch_bounds__(256) void index_insert_kernel(const uint64_t* __restrict__ keys, KeyRanges r,
                                                           IndexSlot* __restrict__ t, uint64_t smask, int32_t* status)
{
    const int32_t j = (int32_t)blockIdx.y;
    const int64_t n = r.off[j + 1];
    for (int64_t i = r.off[j] + (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        index_insert_key(t, smask, keys[i], j, status);
}

// The keys of all W workers, if the partition did not fit.
__global__ __launch_bounds__(kRefillKeys) void index_refill_kernel(const uint64_t* __restrict__ keys, KeyRanges r,
                                                                   int32_t W, IndexSlot* __restrict__ t, uint64_t smask,
                                                                   int32_t* status, BuildSide* __restrict__ side)
{
    if (side->overrun == 0) return;
    refill(r, W, &side->refilled,
           [&](int64_t i, int32_t j) { index_insert_key(t, smask, keys[i], j, status); });
}

__global__ __launch_bounds__(kBins) void index_side_kernel(BuildSide* __restrict__ side)
{
    if (threadIdx.x == 0) {
        side->overrun = 0;
        side->refilled = 0u;
    }
    side->n_spill[threadIdx.x] = 0;
    side->cursor[threadIdx.x * 32] = 0u;
}

// Keys to the bins' lists.  blockIdx.y: the worker; blockIdx.x: the tile of its keys.
__global__ __launch_bounds__(kBuildThreads) void index_scatter_kernel(const uint64_t* __restrict__ keys, KeyRanges r,
                                                                      IndexSlot* __restrict__ t, int32_t log2_slots,
                                                                      BuildSide* __restrict__ side, int32_t* status)
{
    __shared__ uint64_t s_ent[kTile];
    __shared__ uint8_t s_bin[kTile];
    __shared__ uint32_t s_cnt[kBins], s_off[kBins], s_gbase[kBins], s_tmp[16];
    const int tid = threadIdx.x;
    const int32_t j = (int32_t)blockIdx.y;
    const int64_t n0 = r.off[j] + (int64_t)blockIdx.x * kTile, n1 = r.off[j + 1];
    if (n0 >= n1) return;
    const int shift = log2_slots - kBinLog;                  // slots of a bin, and the bin's bits of a key
    const uint64_t cap = 1ull << shift;                      // entries (8 bytes) in the upper half of a bin
    if (tid < kBins) s_cnt[tid] = 0u;
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
        const uint32_t b = (uint32_t)(key[u] >> shift) & (kBins - 1);
        rank[u] = key[u] != kEmpty ? atomicAdd(&s_cnt[b], 1u) : 0u;
    }
    __syncthreads();
    if (tid < kBins) {
        const uint32_t c = s_cnt[tid];
        s_off[tid] = c;
        uint32_t g = 0;
        if (c) {
            g = atomicAdd(&side->cursor[tid * 32], c);
            if ((uint64_t)g + c > cap) {
                atomicOr(&side->overrun, 1);
                g = 0xFFFFFFFFu;                             // no room: not written
            }
        }
        s_gbase[tid] = g;
    }
    __syncthreads();
    build_scan(s_off, kBins, s_tmp);
    const uint64_t bits = (uint64_t)(kBins - 1) << shift;
#pragma unroll
    for (int u = 0; u < kTile / kBuildThreads; ++u) {
        if (key[u] == kEmpty) continue;
        const uint32_t b = (uint32_t)(key[u] >> shift) & (kBins - 1);
        const uint32_t p = s_off[b] + rank[u];
        s_ent[p] = (key[u] & ~bits) | ((uint64_t)j << shift);
        s_bin[p] = (uint8_t)b;
    }
    __syncthreads();
    const uint32_t total = s_off[kBins - 1] + s_cnt[kBins - 1];
    for (uint32_t p = tid; p < total; p += kBuildThreads) {
        const uint32_t b = s_bin[p], g = s_gbase[b];
        if (g == 0xFFFFFFFFu) continue;
        uint64_t* list = reinterpret_cast<uint64_t*>(t + (((uint64_t)b << shift) + (cap >> 1)));
        list[g + (p - s_off[b])] = s_ent[p];
    }
}

// A bin of the index from its list.
template <bool PastCaches>
__global__ __launch_bounds__(kBuildThreads) void index_bin_kernel(IndexSlot* __restrict__ t, int32_t log2_slots,
                                                                  BuildSide* __restrict__ side)
{
    extern __shared__ __align__(16) unsigned char smem[];
    constexpr int kStageEnt = 8 * kBuildThreads;             // entries sorted by sub-bin at a time
    uint64_t* s_key = reinterpret_cast<uint64_t*>(smem);     // [kSub]; the sort's entries
    uint64_t* s_mask = s_key + kSub;                         // [kSub]; the sort's sub-bins
    uint16_t* s_sb = reinterpret_cast<uint16_t*>(s_mask);
    __shared__ uint32_t s_cnt[kMaxSubs], s_off[kMaxSubs], s_cur[kMaxSubs], s_tmp[16];
    __shared__ uint64_t s_spk[kSpills], s_spm[kSpills];
    __shared__ int32_t s_full, s_over;
    static_assert(kStageEnt <= kSub && kMaxSubs <= kBuildThreads, "the sort's arrays fit the table's");
    const int tid = threadIdx.x;
    const int32_t bin = (int32_t)blockIdx.x;
    const int shift = log2_slots - kBinLog;
    const uint64_t slots = 1ull << shift, first = (uint64_t)bin << shift, smask = (1ull << log2_slots) - 1;
    const uint64_t bits = (uint64_t)(kBins - 1) << shift;
    const int subs = 1 << (shift > kSubLog ? shift - kSubLog : 0);
    const int nscan = subs < 64 ? 64 : subs;                 // the scan takes whole wavefronts
    const int sub_log = shift < kSubLog ? shift : kSubLog;
    // (other bins may set the flag meanwhile: one read decides for the workgroup)
    if (tid == 0) {
        s_over = side->overrun;
        s_full = 0;
    }
    __syncthreads();
    if (s_over) return;
    const uint32_t n = side->cursor[bin * 32];
    const uint64_t* list = reinterpret_cast<const uint64_t*>(t + (first + (slots >> 1)));
    uint64_t* sorted = reinterpret_cast<uint64_t*>(t + first);
    if (tid < nscan) s_cnt[tid] = 0u;
    __syncthreads();
    // ---- entries per sub-bin, then the list sorted by sub-bin, stage by stage
    auto sub_of = [&](uint64_t e) { return (uint32_t)(e >> sub_log) & (uint32_t)(subs - 1); };
    for (uint32_t i = tid; i < n; i += kBuildThreads) atomicAdd(&s_cnt[sub_of(list[i])], 1u);
    __syncthreads();
    if (tid < nscan) s_cur[tid] = s_cnt[tid];
    __syncthreads();
    build_scan(s_cur, nscan, s_tmp);
    // the entries before sub-bin k must lie below its slots (16 bytes each): they are still unread when
    // it is written
    if (tid < subs && (uint64_t)s_cur[tid] > (uint64_t)tid * 2 * kSub) s_over = 1;
    __shared__ uint32_t s_beg[kMaxSubs];
    if (tid < nscan) s_beg[tid] = s_cur[tid];
    __syncthreads();
    if (s_over || (uint64_t)n > slots) {
        if (tid == 0) atomicOr(&side->overrun, 1);
        return;
    }
    if (subs > 1) {
        for (uint32_t i0 = 0; i0 < n; i0 += kStageEnt) {
            uint64_t e[kStageEnt / kBuildThreads];
            uint32_t rank[kStageEnt / kBuildThreads];
            if (tid < nscan) s_cnt[tid] = 0u;
#pragma unroll
            for (int u = 0; u < kStageEnt / kBuildThreads; ++u) {
                const uint32_t i = i0 + u * kBuildThreads + tid;
                e[u] = i < n ? list[i] : 0ull;
            }
            __syncthreads();
#pragma unroll
            for (int u = 0; u < kStageEnt / kBuildThreads; ++u)
                if (i0 + u * kBuildThreads + tid < n) rank[u] = atomicAdd(&s_cnt[sub_of(e[u])], 1u);
            __syncthreads();
            if (tid < nscan) s_off[tid] = s_cnt[tid];
            __syncthreads();
            build_scan(s_off, nscan, s_tmp);
#pragma unroll
            for (int u = 0; u < kStageEnt / kBuildThreads; ++u) {
                if (i0 + u * kBuildThreads + tid >= n) continue;
                const uint32_t sb = sub_of(e[u]), p = s_off[sb] + rank[u];
                s_key[p] = e[u];
                s_sb[p] = (uint16_t)sb;
            }
            __syncthreads();
            const uint32_t m = n - i0 < (uint32_t)kStageEnt ? n - i0 : (uint32_t)kStageEnt;
            for (uint32_t p = tid; p < m; p += kBuildThreads) {
                const uint32_t sb = s_sb[p];
                sorted[s_cur[sb] + (p - s_off[sb])] = s_key[p];
            }
            __syncthreads();
            if (tid < subs) s_cur[tid] += s_cnt[tid];
            __syncthreads();
        }
    }
    const uint64_t* from = subs > 1 ? sorted : list;
    // ---- the sub-bins, from the last to the first
    const uint32_t sub_slots = 1u << sub_log;
    for (int sb = subs - 1; sb >= 0; --sb) {
        const uint32_t beg = s_beg[sb], end = sb + 1 < subs ? s_beg[sb + 1] : n;
        for (uint32_t i = tid; i < sub_slots; i += kBuildThreads) {
            s_key[i] = kEmpty;
            s_mask[i] = 0ull;
        }
        if (tid < kSpills) {
            s_spk[tid] = kEmpty;
            s_spm[tid] = 0ull;
        }
        __syncthreads();
        for (uint32_t i = beg + tid; i < end; i += kBuildThreads) {
            const uint64_t e = from[i];
            const uint64_t key = (e & ~bits) | ((uint64_t)bin << shift), mask = 1ull << ((e & bits) >> shift);
            uint32_t s = (uint32_t)key & (sub_slots - 1);
            for (; s < sub_slots; ++s) {
                const unsigned long long prev = atomicCAS((unsigned long long*)&s_key[s], (unsigned long long)kEmpty,
                                                          (unsigned long long)key);
                if (prev == kEmpty || prev == key) {
                    atomicOr((unsigned long long*)&s_mask[s], (unsigned long long)mask);
                    break;
                }
            }
            if (s == sub_slots) {
                // kept once, whichever workers hold it
                int32_t x = 0;
                for (; x < kSpills; ++x) {
                    const unsigned long long prev = atomicCAS((unsigned long long*)&s_spk[x], (unsigned long long)kEmpty,
                                                              (unsigned long long)key);
                    if (prev == kEmpty || prev == key) break;
                }
                if (x < kSpills) atomicOr((unsigned long long*)&s_spm[x], (unsigned long long)mask);
                else s_full = 1;
            }
        }
        __syncthreads();
        if (s_full) {
            if (tid == 0) atomicOr(&side->overrun, 1);
            return;
        }
        u32x4* out = reinterpret_cast<u32x4*>(t + first + ((uint64_t)sb << sub_log));
        for (uint32_t i = tid; i < sub_slots; i += kBuildThreads) {
            const uint64_t k = s_key[i], m = s_mask[i];
            const u32x4 v = {(uint32_t)k, (uint32_t)(k >> 32), (uint32_t)m, (uint32_t)(m >> 32)};
            if constexpr (PastCaches) __builtin_nontemporal_store(v, out + i);
            else out[i] = v;
        }
        // keys past the sub-bin's end: on through the sub-bins after it, final by now, or out of the bin
        if (tid < kSpills && s_spk[tid] != kEmpty) {
            const uint64_t key = s_spk[tid], mask = s_spm[tid];
            uint64_t s = first + ((uint64_t)(sb + 1) << sub_log);
            const uint64_t stop = first + slots;
            for (; s < stop; ++s) {
                const unsigned long long prev = atomicCAS((unsigned long long*)&t[s].key, (unsigned long long)kEmpty,
                                                          (unsigned long long)key);
                if (prev == kEmpty || prev == key) {
                    atomicOr((unsigned long long*)&t[s].mask, (unsigned long long)mask);
                    break;
                }
            }
            if (s == stop) {
                const int32_t x = atomicAdd(&side->n_spill[bin], 1);
                if (x < kSpills) {
                    side->spill_key[bin * kSpills + x] = key;
                    side->spill_mask[bin * kSpills + x] = mask;
                } else {
                    atomicOr(&side->overrun, 1);
                }
            }
        }
        __syncthreads();
    }
}

// Keys that left their bin, from the next bin's first slot on.
__global__ __launch_bounds__(kBins) void index_spill_kernel(IndexSlot* __restrict__ t, int32_t log2_slots,
                                                            BuildSide* __restrict__ side, int32_t* status)
{
    const int32_t bin = threadIdx.x;
    const uint64_t smask = (1ull << log2_slots) - 1;
    if (side->overrun) return;
    const int32_t n = side->n_spill[bin];
    for (int32_t x = 0; x < n; ++x)
        if (!index_insert(t, smask, ((uint64_t)(bin + 1) << (log2_slots - kBinLog)) & smask,
                          side->spill_key[bin * kSpills + x], side->spill_mask[bin * kSpills + x]))
            atomicOr(status, RK_DEV_TABLE_FULL);
}

static std::mutex g_sides_mu;
static SidePool<BuildSide> g_sides[64];

}  // namespace rk

using namespace rk;

// The partitioned build; RK_OK with *done = false when it is not for this call.
static int index_build_parts(int32_t W, const uint64_t* keys, const KeyRanges& r, int64_t longest, IndexSlot* t,
                             int32_t log2_slots, int32_t* st, hipStream_t s, bool* done)
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
    std::lock_guard<std::mutex> lk(g_sides_mu);
    SidePool<BuildSide>& b = g_sides[dev];
    if (!b.addr) {
        void* p = nullptr;
        int rc = hip_check(hipGetSymbolAddress(&p, HIP_SYMBOL(g_build_side)), "rk_index_build side buffers");
        if (!rc) rc = b.make_events("rk_index_build event");
        if (rc) return rc;
        b.addr = (BuildSide*)p;
    }
    const int k = b.take(s);
    if (k < 0) return RK_OK;
    BuildSide* side = b.addr + k;
    // (a stream's handle may be that of a stream destroyed with its work under way)
    int rc = b.once[k] ? hip_check(hipStreamWaitEvent(s, b.used[k], 0), "rk_index_build wait") : RK_OK;
    if (rc) return rc;
    *done = true;
    hipLaunchKernelGGL(index_side_kernel, dim3(1), dim3(kBins), 0, s, side);
    hipLaunchKernelGGL(index_scatter_kernel, dim3((unsigned)((longest + kTile - 1) / kTile), (unsigned)W),
                       dim3(kBuildThreads), 0, s, keys, r, t, log2_slots, side, st);
    if (sizeof(IndexSlot) << log2_slots > kCacheBytes)
        hipLaunchKernelGGL(index_bin_kernel<true>, dim3(kBins), dim3(kBuildThreads), 16 * kSub, s, t, log2_slots, side);
    else
        hipLaunchKernelGGL(index_bin_kernel<false>, dim3(kBins), dim3(kBuildThreads), 16 * kSub, s, t, log2_slots, side);
    hipLaunchKernelGGL(index_spill_kernel, dim3(1), dim3(kBins), 0, s, t, log2_slots, side, st);
    hipLaunchKernelGGL(index_clear_kernel, dim3(1024), dim3(256), 0, s, t, 1ull << log2_slots, &side->overrun);
    hipLaunchKernelGGL(index_refill_kernel, dim3(refill_blocks(r.off[W] - r.off[0])), dim3(kRefillKeys), 0, s, keys, r, W,
                       t, (1ull << log2_slots) - 1, st, side);
    rc = hip_check(hipGetLastError(), "rk_index_build launch");
    const int re = b.record(k, s, "rk_index_build record");
    return rc ? rc : re;
}

extern "C" int rk_index_build(int32_t W, const uint64_t* keys, const int64_t* key_off, void* index,
                              int32_t log2_slots, void* stream)
{
    if (W < 1 || W > 64) return fail(RK_EUNSUPPORTED, "rk_index_build: W outside 1..64");
    if (log2_slots < 4 || log2_slots > 31) return fail(RK_EINVAL, "rk_index_build: log2_slots outside 4..31");
    if (!key_off || !index) return fail(RK_EINVAL, "rk_index_build: NULL array");
    const uint64_t slots = 1ull << log2_slots;
    KeyRanges r;
    int64_t longest = 0;
    for (int32_t j = 0; j < W; ++j) {
        if (key_off[j + 1] < key_off[j]) return fail(RK_EINVAL, "rk_index_build: key_off not monotone at %d", j);
        r.off[j] = key_off[j];
        r.off[j + 1] = key_off[j + 1];
        longest = key_off[j + 1] - key_off[j] > longest ? key_off[j + 1] - key_off[j] : longest;
    }
    const int64_t total = key_off[W] - key_off[0];
    if ((uint64_t)total > slots / 2)
        return fail(RK_ETABLEFULL, "rk_index_build: %lld keys for %llu slots (load above 0.5)", (long long)total,
                    (unsigned long long)slots);
    if (total > 0 && !keys) return fail(RK_EINVAL, "rk_index_build: keys is NULL");
    int32_t* st = status_word();
    if (!st) return fail(RK_EHIP, "rk_index_build: no status word");
    hipStream_t s = (hipStream_t)stream;
    IndexSlot* t = (IndexSlot*)index;
    if (log2_slots >= kPartLog && total > 0) {
        bool done = false;
        const int rc = index_build_parts(W, keys, r, longest, t, log2_slots, st, s, &done);
        if (rc || done) return rc;
    }
    uint64_t blocks = (slots + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    hipLaunchKernelGGL(index_clear_kernel, dim3((unsigned)blocks), dim3(256), 0, s, t, slots, (const int32_t*)nullptr);
    int rc = hip_check(hipGetLastError(), "rk_index_build clear launch");
    if (rc || longest == 0) return rc;
    int64_t b = (longest + 255) / 256;
    if (b > 65536) b = 65536;
    hipLaunchKernelGGL(index_insert_kernel, dim3((unsigned)b, (unsigned)W), dim3(256), 0, s, keys, r, t, slots - 1, st);
    return hip_check(hipGetLastError(), "rk_index_build insert launch");
}

extern "C" int rk_route_score_index(int32_t B, int32_t W, const uint64_t* chains, const int64_t* chain_off,
                                    const void* index, int32_t log2_slots, const int32_t* active_blocks,
                                    rk_cost_params params, int32_t probe_mode, int32_t* overlap_out, float* cost_out,
                                    int32_t* argmin_out, void* stream)
{
    if (B < 0) return fail(RK_EINVAL, "rk_route_score_index: B < 0");
    if (W < 1 || W > 64) return fail(RK_EUNSUPPORTED, "rk_route_score_index: W outside 1..64");
    if (log2_slots < 4 || log2_slots > 31) return fail(RK_EINVAL, "rk_route_score_index: log2_slots outside 4..31");
    if (!(params.w_ov >= 0.0f) || !(params.w_act >= 0.0f) || !(params.w_sat >= 0.0f))
        return fail(RK_EINVAL, "rk_route_score_index: weights must be >= 0");
    if (params.cap_blocks < 1) return fail(RK_EINVAL, "rk_route_score_index: cap_blocks < 1");
    if (probe_mode != RK_PROBE_PREFIX && probe_mode != RK_PROBE_SCAN)
        return fail(RK_EINVAL, "rk_route_score_index: unknown probe_mode");
    if (B == 0) return RK_OK;
    if (!chain_off || !index || !active_blocks) return fail(RK_EINVAL, "rk_route_score_index: NULL array");
    int32_t* st = status_word();
    if (!st) return fail(RK_EHIP, "rk_route_score_index: no status word");
    hipStream_t s = (hipStream_t)stream;
    int64_t blocks = ((int64_t)B + kRPW - 1) / kRPW;
    if (blocks > 1 << 20) blocks = 1 << 20;
    blocks = (blocks + 7) / 8 * 8;
    const IndexSlot* t = (const IndexSlot*)index;
    if (probe_mode == RK_PROBE_SCAN)
        hipLaunchKernelGGL(score_index_kernel<RK_PROBE_SCAN>, dim3((unsigned)blocks), dim3(64), 0, s, B, W,
                           chains, chain_off, t, log2_slots, active_blocks, params, overlap_out, cost_out, argmin_out,
                           st);
    else
        hipLaunchKernelGGL(score_index_kernel<RK_PROBE_PREFIX>, dim3((unsigned)blocks), dim3(64), 0, s, B,
                           W, chains, chain_off, t, log2_slots, active_blocks, params, overlap_out, cost_out,
                           argmin_out, st);
    return hip_check(hipGetLastError(), "rk_route_score_index launch");
}
