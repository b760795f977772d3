// gfx950 kernels of the sketch hot path.
//
// All arithmetic is integer / GF(2): the sketch is a set of 64-bit words
// combined by XOR (App. A.1.1 of arXiv 2509.14433), so there is no matrix
// work and no floating point.  What bounds these kernels is HBM (and L2/LDS)
// traffic and, for the staged scatter, the 64-bit integer hashing.
//
// Bucket layout in HBM: bucket (w, d, c) at word ((w*D + d)*C + c)*2, alpha
// then gamma.  A vertex's shallow depth rows, which receive almost all
// updates (depth d is hit with probability 2^-(d+1)), are contiguous.
#include "kernels.hpp"

#include <mutex>
#include <type_traits>
#include <utility>

namespace cupk {

#define DEVI __device__ __forceinline__

constexpr uint32_t kCus = 256;
constexpr size_t kCuLds = 163840;  // LDS per CU, bytes

// two words of a bucket; the caller's sketch memory may be 8-byte aligned
typedef uint64_t Bucket2 __attribute__((ext_vector_type(2), aligned(8)));

// SplitMix64 output finalizer (Steele, Lea, Flood 2014).
DEVI uint64_t mix64(uint64_t z)
{
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

// The same finalizer after its first step.  That step, z ^ (z >> 30), is
// linear over XOR, so for z = x ^ seed it equals (x ^ (x >> 30)) ^
// (seed ^ (seed >> 30)): callers hashing one x under many seeds compute
// the two halves once each.
DEVI uint64_t mix64_tail(uint64_t z)
{
    z *= 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

DEVI uint64_t mix64_head(uint64_t z) { return z ^ (z >> 30); }

// Depth of a column hash: trailing zero count, capped at D-1.
DEVI uint32_t depth_of(uint64_t h, uint32_t D)
{
    uint32_t z = h ? (uint32_t)__builtin_ctzll(h) : 64u;
    return z < D - 1 ? z : D - 1;
}

// Packed update: lo32 = one endpoint, bits 32..62 = the other, bit 63 = delete.
DEVI bool unpack(uint64_t p, uint32_t V, uint32_t &u, uint32_t &v, bool &del)
{
    uint32_t a = (uint32_t)p;
    uint32_t b = (uint32_t)(p >> 32) & 0x7fffffffu;
    del = (p >> 63) != 0;
    u = a < b ? a : b;
    v = a < b ? b : a;
    return a != b && v < V;
}

// Number of set bits of m below this lane.
DEVI uint32_t lanes_below(uint64_t m)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                     __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

DEVI void gxor(uint64_t *p, uint64_t v)
{
    __hip_atomic_fetch_xor(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

DEVI void lxor(uint64_t *p, uint64_t v)
{
    __hip_atomic_fetch_xor(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// ---------------------------------------------------------------------------
// Classification: validate the batch, flag structural candidates and count
// endpoint records per vertex tile.
//
// Flagged (using the forest as it stood at the start of the batch):
//   insert {u,v} with lbl[u] != lbl[v]               (may join two trees)
//   delete {u,v} that is a forest edge (par[u]==v or par[v]==u), or with
//   lbl[u] != lbl[v] (an edge linked earlier in this same batch)
// Everything else can only touch the sketch.  Block b covers positions
// [b*4096, (b+1)*4096) with 512 threads; each thread issues the loads of
// all its 8 updates (and their label words) before using any, since the
// kernel is bound by the latency of those dependent loads and by the requests
// that they make to L2.  The launch bound holds it at 78 registers (three
// blocks per CU) where the compiler takes 235 (one block) by itself: 6.7e7
// inserts at V = 2^20 in 0.26 ms instead of 0.44, 3.0e6 deletes at V =
// 200,003 in 37 us instead of 53.  The block writes its flagged updates in
// stream order into its own region of the flag buffers (same offsets), at
// positions from one prefix over (step, wave) counts; cnt[b] gets their
// number.  k_flag_compact later packs the regions into one ordered list.
// ---------------------------------------------------------------------------
constexpr uint32_t kClsThreads = 512;  // 8 updates per thread: 16 label loads in flight
constexpr uint32_t kClsPerBlock = 4096;
constexpr uint32_t kClsPerThread = kClsPerBlock / kClsThreads;
constexpr uint32_t kClsWaves = kClsThreads / 64;
static_assert(kClsPerThread * kClsWaves == 64, "one wave scans the (step, wave) counts");

constexpr uint32_t kScanThreads = 1024;

// Block-wide exclusive scan of one value per thread; returns the prefix and
// sets `total`.
template <uint32_t NT>
DEVI uint32_t block_exscan(uint32_t x, uint32_t &total, uint32_t *sh)
{
    const uint32_t lane = __lane_id();
    const uint32_t wid = threadIdx.x / 64;
    uint32_t inc = x;
#pragma unroll
    for (uint32_t o = 1; o < 64; o <<= 1) {
        const uint32_t y = __shfl_up(inc, o);
        if (lane >= o) inc += y;
    }
    if (lane == 63) sh[wid] = inc;
    __syncthreads();
    if (threadIdx.x < 64) {
        uint32_t w = threadIdx.x < NT / 64 ? sh[threadIdx.x] : 0u;
        uint32_t wi = w;
#pragma unroll
        for (uint32_t o = 1; o < 64; o <<= 1) {
            const uint32_t y = __shfl_up(wi, o);
            if (lane >= o) wi += y;
        }
        if (threadIdx.x < NT / 64) sh[64 + threadIdx.x] = wi - w;
        if (threadIdx.x == NT / 64 - 1) sh[128] = wi;
    }
    __syncthreads();
    const uint32_t ex = sh[64 + wid] + inc - x;
    total = sh[128];
    __syncthreads();
    return ex;
}

// Tile scan (one block, after the classify kernel): publishes the header
// to the host, then (staged path, a.off set) scans the per-tile record
// counts into bin offsets (and fill cursors) and lists the work items
// (tile, chunk), a chunk being at most `chunk` records of one tile's bin.
// The counts are zeroed for the next batch.
__global__ __launch_bounds__(kScanThreads) void k_tile_scan(uint32_t *__restrict__ cnt,
                                                            uint32_t ntiles, ScanArgs a,
                                                            uint32_t *__restrict__ hdr,
                                                            uint32_t *__restrict__ hout,
                                                            FlagInline fi)
{
    __shared__ uint32_t sh[160];
    __shared__ uint32_t boff[kInlineMaxBlocks];
    static_assert(kInlineFlags < 65536 && kClsPerBlock < 65536, "packed region words");
    // the batch's verdict moves to HDR_REJ, which every later kernel of the
    // pass reads, and ERR is cleared for the next classification
    const bool err = hdr[fi.checked ? HDR_REJ : HDR_ERR] != 0;
    __syncthreads();
    if (threadIdx.x == 0 && !fi.checked) {
        hdr[HDR_REJ] = err ? 1u : 0u;
        hdr[HDR_ERR] = 0;
    }
    if (!fi.tiles_only) {
        // the batch's flag counts: sums of the classify blocks' counts
        uint32_t nflag, nflag_del;
        {
            uint32_t a = 0, b = 0;
            for (uint32_t i = threadIdx.x; i < fi.nb; i += kScanThreads) {
                a += fi.fcnt[i];
                b += fi.fdel[i];
            }
            block_exscan<kScanThreads>(a, nflag, sh);
            block_exscan<kScanThreads>(b, nflag_del, sh);
        }
        // few flagged updates: compact them into host memory in stream order
        // (one wave per classify block's region)
        const bool inl = fi.hflags && !err && nflag <= kInlineFlags && fi.nb <= kInlineMaxBlocks;
        if (inl && nflag) {
            uint32_t carry = 0;
            for (uint32_t base = 0; base < fi.nb; base += kScanThreads) {
                const uint32_t b = base + threadIdx.x;
                const uint32_t c = b < fi.nb ? fi.fcnt[b] : 0u;
                uint32_t tot;
                const uint32_t ex = block_exscan<kScanThreads>(c, tot, sh);
                // count (<= 4096) and start (<= kInlineFlags) of the region,
                // packed: the copy below reads no global count again
                if (b < fi.nb) boff[b] = c << 16 | (carry + ex);
                carry += tot;
            }
            __syncthreads();
            const uint32_t lane = __lane_id();
            for (uint32_t b = threadIdx.x / 64; b < fi.nb; b += kScanThreads / 64) {
                const uint32_t w = boff[b];
                const uint32_t c = w >> 16, o = w & 0xffffu;
                for (uint32_t k = lane; k < c; k += 64)
                    fi.hflags[o + k] = fi.fupd[(size_t)b * kClsPerBlock + k];
            }
            // every wave waits until its stores have been acknowledged; thread
            // 0's system-scope release of the sequence number below then writes
            // back L2 once for the whole block (a system fence in every wave
            // would write it back once per wave)
            __atomic_signal_fence(__ATOMIC_SEQ_CST);
            __builtin_amdgcn_s_waitcnt(0);
            __syncthreads();
        }
        // the header goes straight to host memory (no copy, no event): words
        // first, then the sequence number with release semantics
        if (threadIdx.x == 0) {
            hout[HDR_ERR] = err ? 1u : 0u;
            hout[HDR_NFLAG] = nflag;
            hout[HDR_NFLAG_DEL] = nflag_del;
            hout[HDR_INLINE] = inl ? 1u : 0u;
            const uint32_t seq = hdr[HDR_SEQ] + 1;
            hdr[HDR_SEQ] = seq;
            __hip_atomic_store(&hout[HDR_SEQ], seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
        }
    }
    if (!a.off || a.sums) return;  // no tile counts, or the multi-block kernels scan them
    const uint32_t ng = a.groups;  // count copies (1 or kCntGroups)
    if (err) {
        // rejected batch: leave the counts zeroed for the next one
        for (uint32_t t = threadIdx.x; t < ng * ntiles; t += blockDim.x) cnt[t] = 0;
        if (threadIdx.x == 0) *a.nitems = 0;
        return;
    }
    const uint32_t chunk = a.chunk, items_cap = a.items_cap;
    uint32_t *off = a.off, *cur = a.cur, *items = a.items;
    uint32_t carry_r = 0, carry_i = 0;
    for (uint32_t base = 0; base < ntiles; base += kScanThreads) {
        const uint32_t t = base + threadIdx.x;
        uint32_t c = 0;
        uint32_t cg[kCntGroups];
#pragma unroll
        for (uint32_t g = 0; g < kCntGroups; g++) {
            cg[g] = 0;
            if (t < ntiles && g < ng) {
                cg[g] = cnt[g * ntiles + t];
                cnt[g * ntiles + t] = 0;  // ready for the next batch's counts
                c += cg[g];
            }
        }
        const uint32_t k = (c + chunk - 1) / chunk;
        uint32_t tot_c, tot_k;
        const uint32_t ex_c = block_exscan<kScanThreads>(c, tot_c, sh);
        const uint32_t ex_k = block_exscan<kScanThreads>(k, tot_k, sh);
        if (t < ntiles) {
            off[t] = carry_r + ex_c;
            cur[t] = carry_r + ex_c;
            if (a.goff) {
                // where each copy's records start: after the copies before it
                uint32_t o = carry_r + ex_c;
#pragma unroll
                for (uint32_t g = 0; g < kCntGroups; g++)
                    if (g < ng) {
                        a.goff[g * ntiles + t] = o;
                        o += cg[g];
                    }
            }
        }
        // a thread lists the items of its tile, a wave those of a tile that
        // has many
        constexpr uint32_t kMany = 8;
        auto list = [&](uint32_t tile, uint32_t first, uint32_t j) {
            if (first + j < items_cap) ((uint2 *)items)[first + j] = make_uint2(tile, j);
        };
        if (k <= kMany)
            for (uint32_t j = 0; j < k; j++) list(t, carry_i + ex_k, j);
        for (uint64_t m = __ballot(k > kMany); m; m &= m - 1) {
            const uint32_t l = (uint32_t)__builtin_ctzll(m);
            const uint32_t kl = __shfl(k, l), tl = __shfl(t, l), fl = __shfl(carry_i + ex_k, l);
            for (uint32_t j = __lane_id(); j < kl; j += 64) list(tl, fl, j);
        }
        carry_r += tot_c;
        carry_i += tot_k;
    }
    if (threadIdx.x == 0) {
        off[ntiles] = carry_r;
        *a.nitems = min(carry_i, items_cap);
    }
}

// Multi-block tile scan (more than kScanOneBlockTiles tiles, one count
// copy): block b covers tiles [b*kScanChunk, (b+1)*kScanChunk).
// k_tile_sums writes each chunk's record total and work-item total;
// k_tile_offsets adds the totals of the chunks before its own, scans its
// chunk (kScanChunk / kScanThreads consecutive tiles per thread) into bin
// offsets, fill cursors and work items, and zeroes the counts for the next
// batch.  A rejected batch (header error) gets no work items.
constexpr uint32_t kScanChunk = 4096;
constexpr uint32_t kScanPer = kScanChunk / kScanThreads;
static_assert(kScanPer * kScanThreads == kScanChunk, "whole tiles per thread");

__global__ __launch_bounds__(kScanThreads) void k_tile_sums(const uint32_t *__restrict__ cnt,
                                                            uint32_t ntiles, uint32_t chunk,
                                                            uint32_t *__restrict__ sums)
{
    __shared__ uint32_t sh[160];
    const uint32_t t0 = blockIdx.x * kScanChunk + threadIdx.x * kScanPer;
    uint32_t c = 0, k = 0;
#pragma unroll
    for (uint32_t j = 0; j < kScanPer; j++) {
        const uint32_t t = t0 + j;
        const uint32_t x = t < ntiles ? cnt[t] : 0u;
        c += x;
        k += (x + chunk - 1) / chunk;
    }
    uint32_t tc, tk;
    block_exscan<kScanThreads>(c, tc, sh);
    block_exscan<kScanThreads>(k, tk, sh);
    if (threadIdx.x == 0) {
        sums[2 * blockIdx.x] = tc;
        sums[2 * blockIdx.x + 1] = tk;
    }
}

__global__ __launch_bounds__(kScanThreads) void k_tile_offsets(uint32_t *__restrict__ cnt,
                                                               uint32_t ntiles, ScanArgs a,
                                                               const uint32_t *__restrict__ hdr)
{
    __shared__ uint32_t sh[160];
    const bool err = hdr[HDR_REJ] != 0;
    const uint32_t b = blockIdx.x;
    // totals of the chunks before this one
    uint32_t pc = 0, pk = 0;
    for (uint32_t i = threadIdx.x; i < b; i += kScanThreads) {
        pc += a.sums[2 * i];
        pk += a.sums[2 * i + 1];
    }
    uint32_t carry_r, carry_i;
    block_exscan<kScanThreads>(pc, carry_r, sh);
    block_exscan<kScanThreads>(pk, carry_i, sh);
    const uint32_t t0 = b * kScanChunk + threadIdx.x * kScanPer;
    uint32_t c[kScanPer], k[kScanPer], lc = 0, lk = 0;
#pragma unroll
    for (uint32_t j = 0; j < kScanPer; j++) {
        const uint32_t t = t0 + j;
        c[j] = t < ntiles ? cnt[t] : 0u;
        if (t < ntiles) cnt[t] = 0;  // ready for the next batch's counts
        k[j] = err ? 0u : (c[j] + a.chunk - 1) / a.chunk;
        lc += c[j];
        lk += k[j];
    }
    uint32_t tot_c, tot_k;
    const uint32_t ex_c = block_exscan<kScanThreads>(lc, tot_c, sh);
    const uint32_t ex_k = block_exscan<kScanThreads>(lk, tot_k, sh);
    uint32_t o = carry_r + ex_c, q = carry_i + ex_k;
#pragma unroll
    for (uint32_t j = 0; j < kScanPer; j++) {
        const uint32_t t = t0 + j;
        if (t < ntiles) {
            a.off[t] = o;
            a.cur[t] = o;
            for (uint32_t i = 0; i < k[j]; i++, q++)
                if (q < a.items_cap) {
                    a.items[2 * q] = t;
                    a.items[2 * q + 1] = i;
                }
        }
        o += c[j];
    }
    if (b == gridDim.x - 1 && threadIdx.x == 0) {
        a.off[ntiles] = carry_r + tot_c;
        *a.nitems = err ? 0u : min(carry_i + tot_k, a.items_cap);
    }
}

__global__ __launch_bounds__(kClsThreads, 4) void k_classify(
    const BatchDesc *__restrict__ desc, BatchDesc dv, uint32_t V, const uint64_t *__restrict__ lp,
    const uint32_t *__restrict__ blk, uint32_t *__restrict__ hdr, uint64_t *__restrict__ fupd,
    uint32_t *__restrict__ fpos, uint32_t *__restrict__ fcnt, uint32_t *__restrict__ fdel,
    uint32_t *__restrict__ tile_cnt, uint32_t tile_shift, uint32_t ntiles,
    uint32_t *__restrict__ tile_rel)
{
    __shared__ uint32_t hist[kLdsHistMax];
    __shared__ uint32_t pre[64 + 1];  // flagged per (step, wave) -> exclusive prefix; total
    __shared__ uint32_t wdel[kClsWaves];  // flagged deletes per wave
    const bool count = tile_cnt != nullptr;
    const bool use_lds = count && ntiles <= kLdsHistMax;
    if (use_lds)
        for (uint32_t t = threadIdx.x; t < ntiles; t += blockDim.x) hist[t] = 0;

    const uint64_t *__restrict__ upd = desc ? desc->upd : dv.upd;
    const uint32_t n = desc ? desc->n : dv.n;
    const uint32_t begin = blockIdx.x * kClsPerBlock;
    const uint32_t lane = __lane_id();
    const uint32_t wid = threadIdx.x / 64;
    uint64_t p[kClsPerThread];
    uint64_t lu[kClsPerThread], lv[kClsPerThread];  // label | parent << 32
    uint32_t bu[kClsPerThread], bv[kClsPerThread];  // block labels (inserts)
#pragma unroll
    for (uint32_t k = 0; k < kClsPerThread; k++) {
        const uint32_t i = begin + k * kClsThreads + threadIdx.x;
        p[k] = i < n ? upd[i] : 0;
    }
    // bit k of `ok`: update k exists and is valid.  An insert whose
    // endpoints both lie in blocks of one label each is decided by those
    // labels (a table of V/64 words); the others load both forest words.
    uint32_t ok = 0;
#pragma unroll
    for (uint32_t k = 0; k < kClsPerThread; k++) {
        const uint32_t i = begin + k * kClsThreads + threadIdx.x;
        uint32_t u, v;
        bool del;
        bu[k] = bv[k] = kBlkMixed;
        if (i < n && unpack(p[k], V, u, v, del)) {
            ok |= 1u << k;
            if (blk && !del) {
                bu[k] = blk[u >> kBlkShift];
                bv[k] = blk[v >> kBlkShift];
            }
        }
    }
    uint32_t gath = 0;  // bit k: update k is decided by its forest words
#pragma unroll
    for (uint32_t k = 0; k < kClsPerThread; k++) {
        lu[k] = lv[k] = 0;
        if (!((ok >> k) & 1u)) continue;
        if (bu[k] != kBlkMixed && bv[k] != kBlkMixed) continue;
        uint32_t u, v;
        bool del;
        unpack(p[k], V, u, v, del);
        gath |= 1u << k;
        lu[k] = lp[u];
        lv[k] = lp[v];
    }
    bool bad = false;
#pragma unroll
    for (uint32_t k = 0; k < kClsPerThread; k++) {
        const uint32_t i = begin + k * kClsThreads + threadIdx.x;
        if (i < n && !((ok >> k) & 1u)) bad = true;
    }
    uint32_t fl = 0;  // bit k: update k flagged
#pragma unroll
    for (uint32_t k = 0; k < kClsPerThread; k++) {
        if (!((ok >> k) & 1u)) continue;
        bool f;
        if (!((gath >> k) & 1u)) {
            f = bu[k] != bv[k];  // an insert between two uniform blocks
        } else {
            uint32_t u, v;
            bool del;
            unpack(p[k], V, u, v, del);
            f = (uint32_t)lu[k] != (uint32_t)lv[k];
            if (!f && del) f = (uint32_t)(lu[k] >> 32) == v || (uint32_t)(lv[k] >> 32) == u;
        }
        if (f) fl |= 1u << k;
    }
    __syncthreads();  // hist zeroed
    if (count) {
        uint32_t *h = use_lds ? hist : tile_cnt;
#pragma unroll
        for (uint32_t k = 0; k < kClsPerThread; k++) {
            if (!((ok >> k) & 1u)) continue;
            uint32_t u, v;
            bool del;
            unpack(p[k], V, u, v, del);
            atomicAdd(&h[u >> tile_shift], 1u);
            atomicAdd(&h[v >> tile_shift], 1u);
        }
    }
    uint32_t ndel = 0;  // flagged deletes of this lane, then of this wave
#pragma unroll
    for (uint32_t k = 0; k < kClsPerThread; k++) {
        const bool f = (fl >> k) & 1u;
        const uint64_t m = __ballot(f);
        if (lane == 0) pre[k * kClsWaves + wid] = (uint32_t)__popcll(m);
        ndel += (f && (p[k] >> 63)) ? 1u : 0u;
    }
#pragma unroll
    for (uint32_t o = 32; o > 0; o >>= 1) ndel += __shfl_xor(ndel, o);
    if (lane == 0) wdel[wid] = ndel;
    const uint64_t mb = __ballot(bad);
    if (mb && lane == (uint32_t)__builtin_ctzll(mb)) atomicOr(&hdr[HDR_ERR], 1u);
    __syncthreads();
    if (threadIdx.x < 64) {
        const uint32_t x = pre[threadIdx.x];
        uint32_t inc = x;
#pragma unroll
        for (uint32_t o = 1; o < 64; o <<= 1) {
            const uint32_t y = __shfl_up(inc, o);
            if (lane >= o) inc += y;
        }
        pre[threadIdx.x] = inc - x;
        if (threadIdx.x == 63) pre[64] = inc;
    }
    __syncthreads();
#pragma unroll
    for (uint32_t k = 0; k < kClsPerThread; k++) {
        const bool f = (fl >> k) & 1u;
        const uint64_t m = __ballot(f);
        if (f) {
            const uint32_t q = begin + pre[k * kClsWaves + wid] + lanes_below(m);
            fupd[q] = p[k];
            if (fpos) fpos[q] = begin + k * kClsThreads + threadIdx.x;
        }
    }
    // per-block counts only: the one-block scan after this kernel sums them
    // (device atomics of every block on one header word would serialize)
    const uint32_t total = pre[64];
    if (threadIdx.x == 0) {
        uint32_t dsum = 0;
#pragma unroll
        for (uint32_t w = 0; w < kClsWaves; w++) dsum += wdel[w];
        fcnt[blockIdx.x] = total;
        fdel[blockIdx.x] = dsum;
    }
    if (use_lds) {
        __syncthreads();
        if (tile_rel) {
            // the returned count is where this block's records start among
            // its count copy's records in the tile's bin
            uint32_t *rb = tile_rel + (size_t)blockIdx.x * ntiles;
            uint32_t *tc = tile_cnt + (blockIdx.x % kCntGroups) * ntiles;
            for (uint32_t t = threadIdx.x; t < ntiles; t += blockDim.x) {
                const uint32_t h = hist[t];
                if (h) rb[t] = atomicAdd(&tc[t], h);
            }
        } else {
            for (uint32_t t = threadIdx.x; t < ntiles; t += blockDim.x)
                if (hist[t]) atomicAdd(&tile_cnt[t], hist[t]);
        }
    }
}

uint32_t classify_blocks(uint32_t n) { return (n + kClsPerBlock - 1) / kClsPerBlock; }

// Refresh of the device forest, one block per page of 2^pshift vertex ids
// (pages null: page i is block i): packed words lp[w] = label | parent << 32
// and the label that all 64 ids of a vertex block share, or kBlkMixed.  Bound
// by latency: lbl and par may be the host forest's own pinned arrays, so that
// a few pages (or a small forest) take this one launch, which reads them over
// the host link, instead of copies through a staging block and two or three
// kernels (a replacement in exact mode took 20 us more).
__global__ __launch_bounds__(256) void k_load_forest(const uint32_t *__restrict__ lbl,
                                                     const uint32_t *__restrict__ par, uint32_t V,
                                                     const uint32_t *__restrict__ pages,
                                                     uint32_t pshift, uint64_t *__restrict__ lp,
                                                     uint32_t *__restrict__ blk)
{
    const uint32_t base = (pages ? pages[blockIdx.x] : blockIdx.x) << pshift;
    const uint32_t lane = __lane_id();
    constexpr uint32_t kAhead = 4;  // vertex blocks of a wave in flight
    for (uint32_t i0 = threadIdx.x / 64; i0 < 1u << (pshift - kBlkShift); i0 += 4 * kAhead) {
        uint32_t l[kAhead], q[kAhead];
#pragma unroll
        for (uint32_t k = 0; k < kAhead; k++) {
            const uint32_t i = i0 + 4 * k, w = base + (i << kBlkShift) + lane;
            l[k] = q[k] = 0;
            if (i < 1u << (pshift - kBlkShift) && w < V) {
                l[k] = lbl[w];
                q[k] = par[w];
            }
        }
#pragma unroll
        for (uint32_t k = 0; k < kAhead; k++) {
            const uint32_t i = i0 + 4 * k, w = base + (i << kBlkShift) + lane;
            const bool in = i < 1u << (pshift - kBlkShift) && w < V;
            if (in) lp[w] = (uint64_t)l[k] | (uint64_t)q[k] << 32;
            const uint32_t first = __shfl(l[k], 0);
            const uint64_t differ = __ballot(in && l[k] != first);
            if (in && lane == 0) blk[w >> kBlkShift] = differ ? kBlkMixed : first;
        }
    }
}

hipError_t launch_load_forest(hipStream_t s, const uint32_t *lbl, const uint32_t *par, uint32_t V,
                              const uint32_t *pages, uint32_t np, uint32_t pshift, uint64_t *lp,
                              uint32_t *blk)
{
    if (np == 0 || V == 0) return hipSuccess;
    if (pshift < kBlkShift || pshift > 16 || ((size_t)(V - 1) >> pshift) >= (1u << 31))
        return hipErrorInvalidValue;
    k_load_forest<<<np, 256, 0, s>>>(lbl, par, V, pages, pshift, lp, blk);
    return hipGetLastError();
}

hipError_t launch_classify(hipStream_t s, const BatchDesc *desc, BatchDesc dv, uint32_t grid_n,
                           uint32_t V, const uint64_t *lp, const uint32_t *blk, uint32_t *hdr,
                           uint64_t *fupd, uint32_t *fpos, uint32_t *fcnt, uint32_t *tile_cnt,
                           uint32_t tile_shift, uint32_t ntiles, const ScanArgs &sa,
                           uint32_t *hout, const FlagInline &fi, uint32_t *tile_rel)
{
    if (!fi.fdel || fi.fcnt != fcnt || fi.nb != classify_blocks(grid_n)) return hipErrorInvalidValue;
    if (grid_n == 0) return hipSuccess;
    if (tile_rel && (!tile_cnt || ntiles > kRelMaxTiles || sa.groups != kCntGroups || !sa.goff))
        return hipErrorInvalidValue;
    if (!tile_rel && tile_cnt && sa.groups != 1) return hipErrorInvalidValue;
    if (sa.sums && (tile_rel || sa.groups != 1 || ntiles <= kScanOneBlockTiles))
        return hipErrorInvalidValue;
    k_classify<<<classify_blocks(grid_n), kClsThreads, 0, s>>>(
        desc, dv, V, lp, blk, hdr, fupd, fpos, fcnt, fi.fdel, tile_cnt, tile_shift, ntiles,
        tile_rel);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    k_tile_scan<<<1, kScanThreads, 0, s>>>(tile_cnt, ntiles, sa, hdr, hout, fi);
    e = hipGetLastError();
    if (e != hipSuccess || !tile_cnt || !sa.sums) return e;
    const uint32_t nch = tile_scan_chunks(ntiles);
    k_tile_sums<<<nch, kScanThreads, 0, s>>>(tile_cnt, ntiles, sa.chunk, sa.sums);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    k_tile_offsets<<<nch, kScanThreads, 0, s>>>(tile_cnt, ntiles, sa, hdr);
    return hipGetLastError();
}

uint32_t tile_scan_chunks(uint32_t ntiles) { return (ntiles + kScanChunk - 1) / kScanChunk; }

// ---------------------------------------------------------------------------
// Direct scatter: every bucket change straight to HBM with device-scope
// atomics.  One thread per (update, column, word): the two words of a bucket,
// and the columns of one update whose depths agree, are neighbouring lanes on
// neighbouring addresses, so the memory system sees one request per touched
// line of an instruction instead of one per word, and an update's columns run
// beside each other instead of one after the other.  Each lane hashes its
// (update, column) once and changes both endpoints.  Bound by the requests of
// device-scope atomics, which execute past L2.  Against one thread per update
// that walks its columns: 1,000 updates at C = 14 in 4 us instead of 31, 1e6
// on 16,384 vertices in 0.71 ms instead of 2.24, on 2^20 (C = 20) in 1.17
// instead of 3.16.
// ---------------------------------------------------------------------------
constexpr uint32_t kDirThreads = 256;

// The updates [0, n) of a grid-stride share: kDirThreads / 2 pairs of lanes
// per block step, R = that over C updates.
DEVI void scatter_direct(const DevSketch &sk, const uint64_t *__restrict__ upd, uint32_t n)
{
    const uint32_t C = sk.C;
    const uint32_t R = (kDirThreads / 2) / C;
    const uint32_t pair = threadIdx.x >> 1, w = threadIdx.x & 1;
    const uint32_t i0 = pair / C, c = pair - i0 * C;
    if (i0 >= R) return;
    const uint64_t seed = sk.seeds[c];
    for (uint64_t i = (uint64_t)blockIdx.x * R + i0; i < n; i += (uint64_t)gridDim.x * R) {
        uint32_t u, v;
        bool del;
        unpack(upd[i], sk.V, u, v, del);
        const uint64_t x = (uint64_t)u * sk.V + v;
        const uint64_t h = mix64(x ^ seed);
        const uint32_t d = depth_of(h, sk.D);
        const uint64_t q = (uint64_t)d * C + c, val = w ? h : x;
        const uint64_t DC = (uint64_t)sk.D * C;
        gxor(sk.b + (u * DC + q) * 2 + w, val);
        gxor(sk.b + (v * DC + q) * 2 + w, val);
    }
}

static uint32_t direct_blocks(uint32_t n, uint32_t C)
{
    const uint32_t R = (kDirThreads / 2) / C;
    return (n + R - 1) / R;
}

__global__ __launch_bounds__(kDirThreads) void k_scatter_atomic(const BatchDesc *__restrict__ desc,
                                                                BatchDesc dv, DevSketch sk,
                                                                const uint32_t *__restrict__ hdr)
{
    const bool err = hdr[HDR_REJ] != 0;
    const uint32_t n = desc ? desc->n : dv.n;
    const uint64_t *upd = desc ? desc->upd : dv.upd;
    if (!err) scatter_direct(sk, upd, n);
}

// ---------------------------------------------------------------------------
// Small batches: one block classifies the whole batch (PT updates per thread)
// and writes the header and the flagged updates (with positions) straight
// into a result block in coherent pinned host memory, then publishes the next
// sequence number; a direct scatter follows.  The batch comes in the
// arguments, so no descriptor copy, header clearing, compaction, binning, copy
// or event is needed: the latency of a small batch is two launches.  A few
// vertices whose forest words changed since the last pass come along (delta):
// a launch of its own for them made exact mode's chain of passes 7% longer
// (10,000 updates with 64 cuts: 3.74 instead of 3.49 ms).
// ---------------------------------------------------------------------------
constexpr uint32_t kSmallThreads = 1024;

template <uint32_t PT>
__global__ __launch_bounds__(kSmallThreads) void k_small_classify(
    const uint64_t *__restrict__ upd, uint32_t n, uint32_t V, uint64_t *lp,
    const uint32_t *__restrict__ delta, uint32_t nd, SmallResult *__restrict__ out,
    uint32_t *__restrict__ derr, uint32_t *__restrict__ seqp, uint32_t with_pos)
{
    constexpr uint32_t kWaves = kSmallThreads / 64;
    constexpr uint32_t kCounts = PT * kWaves;  // (step, wave) flag counts
    static_assert(kCounts <= kSmallThreads && kCounts % 64 == 0, "one thread per count");
    __shared__ uint32_t pre[kCounts];
    __shared__ uint32_t sh[160];
    __shared__ uint32_t s_bad, s_del, s_flag;
    const uint32_t lane = __lane_id();
    const uint32_t wid = threadIdx.x / 64;
    uint32_t seq = 0;
    if (threadIdx.x == 0) {
        s_bad = 0;
        s_del = 0;
        s_flag = 0;
        seq = *seqp + 1;
    }
    uint64_t p[PT];
    uint32_t fl = 0, bad = 0, ndel = 0;
#pragma unroll
    for (uint32_t k = 0; k < PT; k++) {
        const uint32_t i = k * kSmallThreads + threadIdx.x;
        p[k] = i < n ? upd[i] : 0;
    }
    if (nd) {  // (repeats of a vertex write the same word)
        if (threadIdx.x < nd) {
            const uint32_t *e = delta + 3 * threadIdx.x;
            const uint32_t w = e[0];
            if (w < V) lp[w] = (uint64_t)e[1] | (uint64_t)e[2] << 32;
        }
        __syncthreads();
    }
    // a few updates' forest words are in flight together
    constexpr uint32_t kGather = 4;
#pragma unroll
    for (uint32_t k0 = 0; k0 < PT; k0 += kGather) {
        uint64_t lu[kGather], lv[kGather];
#pragma unroll
        for (uint32_t g = 0; g < kGather; g++) {
            const uint32_t k = k0 + g, i = k * kSmallThreads + threadIdx.x;
            uint32_t u, v;
            bool del;
            lu[g] = lv[g] = 0;
            if (i < n && unpack(p[k], V, u, v, del)) {
                lu[g] = lp[u];
                lv[g] = lp[v];
            }
        }
#pragma unroll
        for (uint32_t g = 0; g < kGather; g++) {
            const uint32_t k = k0 + g, i = k * kSmallThreads + threadIdx.x;
            if (i >= n) continue;
            uint32_t u, v;
            bool del;
            if (!unpack(p[k], V, u, v, del)) {
                bad = 1;
                continue;
            }
            bool f = (uint32_t)lu[g] != (uint32_t)lv[g];
            if (!f && del) f = (uint32_t)(lu[g] >> 32) == v || (uint32_t)(lv[g] >> 32) == u;
            if (f) {
                fl |= 1u << k;
                ndel += del ? 1u : 0u;
            }
        }
    }
    __syncthreads();  // the counts cleared
    if (bad) atomicOr(&s_bad, 1u);
    if (ndel) atomicAdd(&s_del, ndel);
    if (fl) atomicAdd(&s_flag, (uint32_t)__popc(fl));
    __syncthreads();
    const uint32_t total = s_flag;
    // Places of the flagged updates.  Most small batches have none: without the
    // scan (and with the sequence number loaded ahead) one update takes 13.3
    // us from host memory instead of 14.0.
    if (total) {  // (block-uniform)
#pragma unroll
        for (uint32_t k = 0; k < PT; k++) {
            const uint64_t m = __ballot((fl >> k) & 1u);
            if (lane == 0) pre[k * kWaves + wid] = (uint32_t)__popcll(m);
        }
        __syncthreads();
        const uint32_t x = threadIdx.x < kCounts ? pre[threadIdx.x] : 0u;
        uint32_t tot;
        const uint32_t ex = block_exscan<kSmallThreads>(x, tot, sh);
        if (threadIdx.x < kCounts) pre[threadIdx.x] = ex;
        __syncthreads();
#pragma unroll
        for (uint32_t k = 0; k < PT; k++) {
            const bool f = (fl >> k) & 1u;
            const uint64_t m = __ballot(f);
            if (f) {
                const uint32_t q = pre[k * kWaves + wid] + lanes_below(m);
                out->fupd[q] = p[k];
                if (with_pos) out->fpos[q] = k * kSmallThreads + threadIdx.x;
            }
        }
        // the result is in host memory before the sequence number says so:
        // every wave waits until its stores have been acknowledged, and thread
        // 0's system-scope release below writes back L2 once for the block
        __atomic_signal_fence(__ATOMIC_SEQ_CST);
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        *derr = s_bad;  // for the scatter
        out->hdr[HDR_ERR] = s_bad;
        out->hdr[HDR_NFLAG] = s_bad ? 0u : total;
        out->hdr[HDR_NFLAG_DEL] = s_bad ? 0u : s_del;
        *seqp = seq;
        __hip_atomic_store(&out->hdr[HDR_SEQ], seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

__global__ __launch_bounds__(kDirThreads) void k_small_scatter(const uint64_t *__restrict__ upd,
                                                               uint32_t n, DevSketch sk,
                                                               const uint32_t *__restrict__ derr)
{
    if (*derr) return;
    scatter_direct(sk, upd, n);
}

// The buckets a block's threads changed, added to *touched (timed launches;
// all threads of a block, the same `touched`).  One atomic per block: 4,000 of
// them on one word take 50 us.  sum: a word per wave of the block's dynamic
// LDS, overwritten; words of its own would take a fourth block off a CU from
// k_tile_scatter at 40 KiB of dynamic LDS (124 us instead of 150 for 2.0e6
// records on 65,536 vertices, C = 28).
DEVI void add_touched(unsigned long long *touched, uint32_t t, uint32_t *sum)
{
    if (!touched) return;
#pragma unroll
    for (uint32_t o = 32; o > 0; o >>= 1) t += __shfl_xor(t, o);
    __syncthreads();  // the last use of the delta
    if (__lane_id() == 0) sum[threadIdx.x / 64] = t;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (uint32_t w = 1; w < blockDim.x / 64; w++) t += sum[w];
        if (t) atomicAdd(touched, (unsigned long long)t);
    }
}

// Direct scatter of medium batches: as scatter_direct, but a block takes `per`
// updates (a power of two up to kMidMax), counts their endpoints in an LDS
// hash table, and gathers the changes to up to eight vertices that many of
// them share in LDS (rows below kMidRows), sent once.  Bound by the requests of
// device-scope atomics; one per update on the words of a vertex that takes a
// large share of a batch would serialize at about 17 ns each.  131,072 updates
// at V = 131,072, C = 4, a tenth of them at one vertex: 58 us, 139 when only
// the endpoints of four updates in 32 were looked at; uniform ones 42 and 41.
constexpr uint32_t kMidMax = kDirThreads;  // one update per thread when counting
constexpr uint32_t kMidRows = 8;
constexpr uint32_t kMidVerts = 8;
constexpr uint32_t kMidTable = 4 * kMidMax;  // hash entries: at most half are used

__global__ __launch_bounds__(kDirThreads) void k_mid_scatter(const uint64_t *__restrict__ upd,
                                                             uint32_t n, DevSketch sk,
                                                             const uint32_t *__restrict__ derr,
                                                             uint32_t per,
                                                             unsigned long long *__restrict__ touched)
{
    extern __shared__ uint64_t lds[];  // [vertex][row][column][alpha, gamma]
    __shared__ uint32_t key[kMidTable], cnt[kMidTable];
    __shared__ uint32_t hot[kMidVerts], nhot;
    __shared__ uint8_t slot[2 * kMidMax];
    if (*derr) return;
    const uint32_t C = sk.C;
    const uint32_t per_v = kMidRows * 2 * C;
    const uint32_t begin = blockIdx.x * per, m = min(n - begin, per);
    const uint32_t tab = 4 * per;
    for (uint32_t t = threadIdx.x; t < tab; t += kDirThreads) {
        key[t] = 0xffffffffu;  // no vertex (V <= 2^31)
        cnt[t] = 0;
    }
    if (threadIdx.x == 0) nhot = 0;
    uint32_t e[2] = {0, 0}, at[2] = {0, 0};
    bool del;
    if (threadIdx.x < m) unpack(upd[begin + threadIdx.x], sk.V, e[0], e[1], del);
    __syncthreads();
    if (threadIdx.x < m) {
        const uint32_t shift = (uint32_t)__builtin_clz(tab) + 1;  // 32 - log2(tab)
#pragma unroll
        for (uint32_t k = 0; k < 2; k++) {
            uint32_t h = (e[k] * 0x9E3779B1u) >> shift;
            for (;; h = (h + 1) & (tab - 1)) {
                const uint32_t old = atomicCAS(&key[h], 0xffffffffu, e[k]);
                if (old == 0xffffffffu || old == e[k]) break;
            }
            at[k] = h;
            atomicAdd(&cnt[h], 1u);
        }
    }
    // places for the vertices with the most updates: first those with a
    // sixteenth of the block's or more, then any with three
    constexpr uint32_t kPlaced = 1u << 31;
    for (uint32_t many = max(per / 16, 4u); many; many = many > 3 ? 3 : 0) {
        __syncthreads();
        for (uint32_t t = threadIdx.x; t < tab; t += kDirThreads) {
            const uint32_t c = cnt[t];
            if (c < many || c >= kPlaced) continue;
            const uint32_t p = atomicAdd(&nhot, 1u);
            if (p >= kMidVerts) continue;
            hot[p] = key[t];
            cnt[t] = kPlaced | p;
        }
    }
    __syncthreads();
    const uint32_t nh = min(nhot, kMidVerts);
    if (threadIdx.x < m) {
#pragma unroll
        for (uint32_t k = 0; k < 2; k++) {
            const uint32_t c = cnt[at[k]];
            slot[2 * threadIdx.x + k] = (uint8_t)(c >= kPlaced ? c & 0xffu : kMidVerts);
        }
    }
    for (uint32_t q = threadIdx.x; q < nh * per_v; q += kDirThreads) lds[q] = 0;
    __syncthreads();
    const uint32_t R = (kDirThreads / 2) / C;
    const uint32_t pair = threadIdx.x >> 1, w = threadIdx.x & 1;
    const uint32_t i0 = pair / C, c = pair - i0 * C;
    const uint64_t DC = (uint64_t)sk.D * C;
    uint32_t nchanged = 0;
    if (i0 < R) {
        const uint64_t seed = sk.seeds[c];
        for (uint32_t i = i0; i < m; i += R) {
            unpack(upd[begin + i], sk.V, e[0], e[1], del);
            const uint64_t x = (uint64_t)e[0] * sk.V + e[1];
            const uint64_t h = mix64(x ^ seed);
            const uint32_t d = depth_of(h, sk.D);
            const uint64_t val = w ? h : x;
            const uint32_t q = (d * C + c) * 2 + w;
#pragma unroll
            for (uint32_t k = 0; k < 2; k++) {
                const uint32_t p = slot[2 * i + k];
                if (p < kMidVerts && d < kMidRows) {
                    lxor(&lds[p * per_v + q], val);
                } else {
                    gxor(sk.b + e[k] * DC * 2 + q, val);
                    nchanged += 1 - w;
                }
            }
        }
    }
    __syncthreads();
    for (uint32_t q = threadIdx.x; q < nh * per_v; q += kDirThreads) {
        const uint64_t val = lds[q];
        if (val == 0) continue;
        const uint32_t p = q / per_v;
        gxor(sk.b + hot[p] * DC * 2 + (q - p * per_v), val);
        nchanged += 1 - (q & 1);
    }
    add_touched(touched, nchanged, (uint32_t *)lds);
}

hipError_t launch_mid_scatter(hipStream_t s, const uint64_t *upd, uint32_t n, DevSketch sk,
                              const uint32_t *derr, unsigned long long *touched)
{
    if (n == 0) return hipSuccess;
    // updates per block: as many as leave 1,024 blocks (a vertex in every block
    // serializes one atomic per block), at least 32 and enough for all lanes
    uint32_t per = 32;
    while (per < kMidMax && (per * sk.C < kDirThreads / 2 || (uint64_t)per * 1024 < n)) per *= 2;
    const size_t lds = (size_t)kMidVerts * kMidRows * sk.C * 16;
    k_mid_scatter<<<(n + per - 1) / per, kDirThreads, lds, s>>>(upd, n, sk, derr, per, touched);
    return hipGetLastError();
}

hipError_t launch_small_classify(hipStream_t s, const uint64_t *upd, uint32_t n, uint32_t V,
                                 uint64_t *lp, const uint32_t *delta, uint32_t nd,
                                 SmallResult *out, uint32_t *derr, uint32_t *seqp, bool with_pos)
{
    if (n == 0 || n > kOneBlockMax || nd > kSmallThreads) return hipErrorInvalidValue;
    const uint32_t wp = with_pos ? 1u : 0u;
    if (n <= kSmallMax)
        k_small_classify<kSmallMax / kSmallThreads>
            <<<1, kSmallThreads, 0, s>>>(upd, n, V, lp, delta, nd, out, derr, seqp, wp);
    else if (n <= kOneBlockMax / 2)
        k_small_classify<kOneBlockMax / 2 / kSmallThreads>
            <<<1, kSmallThreads, 0, s>>>(upd, n, V, lp, delta, nd, out, derr, seqp, wp);
    else
        k_small_classify<kOneBlockMax / kSmallThreads>
            <<<1, kSmallThreads, 0, s>>>(upd, n, V, lp, delta, nd, out, derr, seqp, wp);
    return hipGetLastError();
}

hipError_t launch_small_scatter(hipStream_t s, const uint64_t *upd, uint32_t n, DevSketch sk,
                                const uint32_t *derr)
{
    if (n == 0 || n > kSmallMax) return hipErrorInvalidValue;
    k_small_scatter<<<direct_blocks(n, sk.C), kDirThreads, 0, s>>>(upd, n, sk, derr);
    return hipGetLastError();
}

hipError_t launch_scatter_atomic(hipStream_t s, const BatchDesc *desc, BatchDesc dv,
                                 uint32_t grid_n, DevSketch sk, const uint32_t *hdr)
{
    if (grid_n == 0) return hipSuccess;
    const uint32_t grid = min(direct_blocks(grid_n, sk.C), 16u * kCus);
    k_scatter_atomic<<<grid, kDirThreads, 0, s>>>(desc, dv, sk, hdr);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Staged scatter.
//
// 1. tile scan (one block, once all counts are in):
//    exclusive scan of the per-tile record counts into bin offsets, and a
//    list of work items (tile, chunk) where a chunk is at most `chunk`
//    records of one tile's bin.
// 2. k_tile_fill: each update writes one record per endpoint into the bin
//    of that endpoint's tile (make_rec).  Slots are reserved per block in LDS
//    first, so global atomics are per (block, tile), not per record.
// 3. k_tile_scatter_stag (up to kStagMaxC columns) or k_tile_scatter: one
//    work item per block iteration.  The block keeps a zeroed LDS delta of
//    depth rows 0..rows-1 for the tile's vertices, XORs every (record,
//    column) pair into it (LDS atomics; depths >= rows go straight to HBM
//    with device atomics), then folds the nonzero delta words into HBM: a
//    plain read-XOR-write when the item is the tile's whole bin (no other
//    block touches these vertices), a device atomic XOR otherwise.
// ---------------------------------------------------------------------------

// The record of endpoint w of an update {w, o} in a bin of 2^shift vertices.
// The binning is bound by HBM, so records are 32 bits where that holds them:
// w's place in the bin, then o (rec_wide otherwise).  The bin gives the rest
// of w, and the update's two endpoints are told apart by their order.  Wide
// records hold the update itself: u | v << 32 with u < v, bit 63 (kRecV) set
// in the record of v.  6.7e7 updates in two levels (16-vertex tiles, V =
// 2^20): 0.63 ms for the two fills and the count against 1.30 with wide ones
// in items of 4,096 and 8,192 records.
constexpr uint64_t kRecV = 1ull << 63;

bool rec_wide(uint32_t V, uint32_t shift)
{
    return V > 1 && 32u - (uint32_t)__builtin_clz(V - 1) + shift > 32u;
}

template <class R>
DEVI R make_rec(uint32_t w, uint32_t o, uint32_t shift)
{
    if constexpr (sizeof(R) == 4)
        return (w & ((1u << shift) - 1)) | o << shift;
    else
        return w < o ? w | (uint64_t)o << 32 : o | (uint64_t)w << 32 | kRecV;
}

// w and o of a record in the bin whose first vertex is w0
template <class R>
DEVI void read_rec(R r, uint32_t w0, uint32_t shift, uint32_t &w, uint32_t &o)
{
    if constexpr (sizeof(R) == 4) {
        w = w0 + ((uint32_t)r & ((1u << shift) - 1));
        o = (uint32_t)r >> shift;
    } else {
        const uint32_t u = (uint32_t)r, v = (uint32_t)(r >> 32) & 0x7fffffffu;
        w = r & kRecV ? v : u;
        o = r & kRecV ? u : v;
    }
}

constexpr uint32_t kFillThreads = 1024;
constexpr uint32_t kFillPerBlock = 4096;
constexpr uint32_t kFillPerThread = kFillPerBlock / kFillThreads;

template <class R>
__global__ __launch_bounds__(kFillThreads) void k_tile_fill(
    const BatchDesc *__restrict__ desc, BatchDesc dv, uint32_t V, uint32_t tile_shift,
    uint32_t ntiles, uint32_t *__restrict__ cur, R *__restrict__ bins,
    const uint32_t *__restrict__ hdr)
{
    __shared__ uint32_t lcnt[kLdsHistMax];
    if (hdr[HDR_REJ]) return;
    const uint64_t *__restrict__ upd = desc ? desc->upd : dv.upd;
    const uint32_t n = desc ? desc->n : dv.n;
    const uint32_t begin = blockIdx.x * kFillPerBlock;
    if (begin >= n) return;
    // all of this thread's updates are loaded once, up front
    uint64_t p[kFillPerThread];
#pragma unroll
    for (uint32_t k = 0; k < kFillPerThread; k++) {
        const uint32_t i = begin + k * kFillThreads + threadIdx.x;
        p[k] = i < n ? upd[i] : 0;
    }
    if (ntiles > kLdsHistMax) {
        // Many small tiles: contention is low, reserve per record.
#pragma unroll
        for (uint32_t k = 0; k < kFillPerThread; k++) {
            if (begin + k * kFillThreads + threadIdx.x >= n) continue;
            uint32_t u, v;
            bool del;
            unpack(p[k], V, u, v, del);
            bins[atomicAdd(&cur[u >> tile_shift], 1u)] = make_rec<R>(u, v, tile_shift);
            bins[atomicAdd(&cur[v >> tile_shift], 1u)] = make_rec<R>(v, u, tile_shift);
        }
        return;
    }
    for (uint32_t t = threadIdx.x; t < ntiles; t += blockDim.x) lcnt[t] = 0;
    __syncthreads();
    // ranks of each record inside its tile's share of this block
    uint32_t ru[kFillPerThread], rv[kFillPerThread];
#pragma unroll
    for (uint32_t k = 0; k < kFillPerThread; k++) {
        ru[k] = rv[k] = 0;
        if (begin + k * kFillThreads + threadIdx.x >= n) continue;
        uint32_t u, v;
        bool del;
        unpack(p[k], V, u, v, del);
        ru[k] = atomicAdd(&lcnt[u >> tile_shift], 1u);
        rv[k] = atomicAdd(&lcnt[v >> tile_shift], 1u);
    }
    __syncthreads();
    // reserve one contiguous range per tile present in this block
    for (uint32_t t = threadIdx.x; t < ntiles; t += blockDim.x) {
        const uint32_t c = lcnt[t];
        if (c) lcnt[t] = atomicAdd(&cur[t], c);
    }
    __syncthreads();
#pragma unroll
    for (uint32_t k = 0; k < kFillPerThread; k++) {
        if (begin + k * kFillThreads + threadIdx.x >= n) continue;
        uint32_t u, v;
        bool del;
        unpack(p[k], V, u, v, del);
        bins[lcnt[u >> tile_shift] + ru[k]] = make_rec<R>(u, v, tile_shift);
        bins[lcnt[v >> tile_shift] + rv[k]] = make_rec<R>(v, u, tile_shift);
    }
}

// Fill for up to kFillStageTiles tiles: the block's 2*kFillPerBlock records
// are first counting-sorted by tile in LDS, then written out in that order,
// so that the lanes of a wave store one (block, tile) run after another into
// consecutive bin words (coalesced) instead of single words scattered over
// all tiles.  A 32-bit record's tile is staged beside it.  Dynamic LDS:
// fill_stage_lds bytes.
static_assert(kFillStageTiles == 2 * kFillThreads, "two tiles per fill thread");
static size_t fill_stage_lds(uint32_t ntiles, bool wide)
{
    return (size_t)2 * kFillPerBlock * (wide ? 8 : 6) + (size_t)2 * ntiles * 4 + 160 * 4;
}

template <class R>
__global__ __launch_bounds__(kFillThreads) void k_tile_fill_staged(
    const BatchDesc *__restrict__ desc, BatchDesc dv, uint32_t V, uint32_t tile_shift,
    uint32_t ntiles, uint32_t *__restrict__ cur, R *__restrict__ bins,
    const uint32_t *__restrict__ hdr, const uint32_t *__restrict__ goff,
    const uint32_t *__restrict__ rel)
{
    extern __shared__ uint64_t fsm[];
    R *stage = (R *)fsm;                                     // records in tile order
    uint32_t *lcnt = (uint32_t *)(stage + 2 * kFillPerBlock);  // per tile: count, then bin base
    uint32_t *lpre = lcnt + ntiles;                          // per tile: first stage slot
    uint32_t *sh = lpre + ntiles;                            // scan scratch (160 words)
    uint16_t *stile = (uint16_t *)(sh + 160);                // 32-bit records: their tiles
    if (hdr[HDR_REJ]) return;
    const uint64_t *__restrict__ upd = desc ? desc->upd : dv.upd;
    const uint32_t n = desc ? desc->n : dv.n;
    const uint32_t begin = blockIdx.x * kFillPerBlock;
    if (begin >= n) return;
    uint64_t p[kFillPerThread];
#pragma unroll
    for (uint32_t k = 0; k < kFillPerThread; k++) {
        const uint32_t i = begin + k * kFillThreads + threadIdx.x;
        p[k] = i < n ? upd[i] : 0;
    }
    for (uint32_t t = threadIdx.x; t < ntiles; t += blockDim.x) lcnt[t] = 0;
    __syncthreads();
    // ranks of each record inside its tile's share of this block
    uint32_t ru[kFillPerThread], rv[kFillPerThread];
#pragma unroll
    for (uint32_t k = 0; k < kFillPerThread; k++) {
        ru[k] = rv[k] = 0;
        if (begin + k * kFillThreads + threadIdx.x >= n) continue;
        uint32_t u, v;
        bool del;
        unpack(p[k], V, u, v, del);
        ru[k] = atomicAdd(&lcnt[u >> tile_shift], 1u);
        rv[k] = atomicAdd(&lcnt[v >> tile_shift], 1u);
    }
    __syncthreads();
    // first stage slot of each tile (two tiles per thread), and one
    // contiguous bin range per tile present in this block
    const uint32_t t0 = 2 * threadIdx.x;
    const uint32_t c0 = t0 < ntiles ? lcnt[t0] : 0u;
    const uint32_t c1 = t0 + 1 < ntiles ? lcnt[t0 + 1] : 0u;
    uint32_t tot;
    const uint32_t ex = block_exscan<kFillThreads>(c0 + c1, tot, sh);
    // with `rel`, the classify block of the same updates has already taken
    // this block's place in every tile, among the records of its count copy
    const uint32_t *rb = rel ? rel + (size_t)blockIdx.x * ntiles : nullptr;
    const uint32_t *go = rel ? goff + (blockIdx.x % kCntGroups) * ntiles : nullptr;
    if (t0 < ntiles) {
        lpre[t0] = ex;
        lcnt[t0] = c0 ? (rb ? go[t0] + rb[t0] : atomicAdd(&cur[t0], c0)) : 0u;
    }
    if (t0 + 1 < ntiles) {
        lpre[t0 + 1] = ex + c0;
        lcnt[t0 + 1] = c1 ? (rb ? go[t0 + 1] + rb[t0 + 1] : atomicAdd(&cur[t0 + 1], c1)) : 0u;
    }
    __syncthreads();
#pragma unroll
    for (uint32_t k = 0; k < kFillPerThread; k++) {
        if (begin + k * kFillThreads + threadIdx.x >= n) continue;
        uint32_t u, v;
        bool del;
        unpack(p[k], V, u, v, del);
        const uint32_t tu = u >> tile_shift, tv = v >> tile_shift;
        const uint32_t ju = lpre[tu] + ru[k], jv = lpre[tv] + rv[k];
        stage[ju] = make_rec<R>(u, v, tile_shift);
        stage[jv] = make_rec<R>(v, u, tile_shift);
        if constexpr (sizeof(R) == 4) {
            stile[ju] = (uint16_t)tu;
            stile[jv] = (uint16_t)tv;
        }
    }
    __syncthreads();
    for (uint32_t j = threadIdx.x; j < tot; j += blockDim.x) {
        const R rec = stage[j];
        uint32_t t;
        if constexpr (sizeof(R) == 4) {
            t = stile[j];
        } else {
            uint32_t w, o;
            read_rec(rec, 0, tile_shift, w, o);
            t = w >> tile_shift;
        }
        bins[lcnt[t] + (j - lpre[t])] = rec;
    }
}

// ---------------------------------------------------------------------------
// Two-level binning, for more tiles than one block's LDS histogram serves.
// The classify kernel counts records per coarse bin (2^fshift consecutive
// tiles), its scan lists work items (coarse bin, part of at most
// fine_chunk records), and the fill bins the records by coarse bin into
// `bins1` (k_tile_fill_staged on coarse bins).  k_fine_count counts an item's
// records per tile in LDS and adds the counts to the tile counts (one global
// atomic per (item, tile)), the multi-block tile scan turns them into bin
// offsets and work items, and k_fine_fill ranks each item's records per tile
// in LDS, reserves one range per (item, tile) from the tile's cursor and
// writes the records there, staged in tile order in LDS so that each (item,
// tile) run is written as consecutive words.  Bound by HBM: the items are as
// large as the staged records leave LDS for two blocks of a CU, which keeps
// the runs long and has few reservations and barriers per record.
// ---------------------------------------------------------------------------
constexpr uint32_t kFineThreads = 1024;
template <class R>
constexpr uint32_t kFinePer = sizeof(R) == 4 ? 16 : 8;  // records per thread

uint32_t fine_chunk(bool wide)
{
    return kFineThreads * (wide ? kFinePer<uint64_t> : kFinePer<uint32_t>);
}

// Block b's item: consecutive items to the blocks of one XCD (blocks go round
// robin over the 8 XCDs), whose L2 then joins the runs that neighbouring
// items write next to each other.
DEVI uint32_t fine_item(uint32_t b, uint32_t n)
{
    const uint32_t x = b % 8, q = n / 8, r = n % 8;
    return x * q + min(x, r) + b / 8;
}

template <class R>
__global__ __launch_bounds__(kFineThreads) void k_fine_count(
    const R *__restrict__ bins1, const uint32_t *__restrict__ coff,
    const uint32_t *__restrict__ citems, const uint32_t *__restrict__ ncitems,
    uint32_t tile_shift, uint32_t fshift, uint32_t *__restrict__ cnt,
    const uint32_t *__restrict__ hdr)
{
    extern __shared__ uint32_t fine_sm[];
    uint32_t *hist = fine_sm;  // per tile of the coarse bin
    constexpr uint32_t P = kFinePer<R>;
    const uint32_t nit = hdr[HDR_REJ] ? 0u : *ncitems;
    if (blockIdx.x >= nit) return;
    const uint32_t it = fine_item(blockIdx.x, nit);
    const uint32_t bin = citems[2 * it];
    const uint32_t cb = coff[bin] + citems[2 * it + 1] * (kFineThreads * P);
    const uint32_t n = min(coff[bin + 1] - cb, kFineThreads * P);
    const uint32_t T = 1u << fshift, t_lo = bin << fshift;
    R rec[P];
#pragma unroll
    for (uint32_t k = 0; k < P; k++) {
        const uint32_t i = k * kFineThreads + threadIdx.x;
        rec[k] = i < n ? bins1[cb + i] : 0;
    }
    for (uint32_t t = threadIdx.x; t < T; t += kFineThreads) hist[t] = 0;
    __syncthreads();
#pragma unroll
    for (uint32_t k = 0; k < P; k++) {
        if (k * kFineThreads + threadIdx.x >= n) continue;
        uint32_t w, o;
        read_rec(rec[k], 0, tile_shift + fshift, w, o);
        atomicAdd(&hist[(w >> tile_shift) & (T - 1)], 1u);
    }
    __syncthreads();
    for (uint32_t t = threadIdx.x; t < T; t += kFineThreads) {
        const uint32_t c = hist[t];
        if (c) atomicAdd(&cnt[t_lo + t], c);
    }
}

template <class R>
static size_t fine_fill_lds(uint32_t fshift)
{
    return (size_t)kFineThreads * kFinePer<R> * sizeof(R) + ((size_t)8 << fshift);
}

template <class R, class R2>
__global__ __launch_bounds__(kFineThreads, 8) void k_fine_fill(
    const R *__restrict__ bins1, const uint32_t *__restrict__ coff,
    const uint32_t *__restrict__ citems, const uint32_t *__restrict__ ncitems,
    uint32_t tile_shift, uint32_t fshift, uint32_t *__restrict__ cur, R2 *__restrict__ bins,
    const uint32_t *__restrict__ hdr)
{
    extern __shared__ uint32_t fine_sm[];
    __shared__ uint32_t sh[160];
    constexpr uint32_t P = kFinePer<R>;
    const uint32_t nit = hdr[HDR_REJ] ? 0u : *ncitems;
    if (blockIdx.x >= nit) return;
    const uint32_t it = fine_item(blockIdx.x, nit);
    const uint32_t bin = citems[2 * it];
    const uint32_t cb = coff[bin] + citems[2 * it + 1] * (kFineThreads * P);
    const uint32_t n = min(coff[bin + 1] - cb, kFineThreads * P);
    const uint32_t cs = tile_shift + fshift;
    const uint32_t T = 1u << fshift, t_lo = bin << fshift;
    R *stage = (R *)fine_sm;                               // the item's records in tile order
    uint32_t *lcnt = (uint32_t *)(stage + kFineThreads * P);  // per tile: count, then bin base
    uint32_t *lpre = lcnt + T;                             // per tile: first stage slot
    R rec[P];
#pragma unroll
    for (uint32_t k = 0; k < P; k++) {
        const uint32_t i = k * kFineThreads + threadIdx.x;
        rec[k] = i < n ? bins1[cb + i] : 0;
    }
    for (uint32_t t = threadIdx.x; t < T; t += kFineThreads) lcnt[t] = 0;
    __syncthreads();
    static_assert(kFineThreads * P < 65536, "two ranks per register");
    uint32_t rk[P / 2];  // ranks in the item's shares of the records' tiles
#pragma unroll
    for (uint32_t k = 0; k < P; k++) {
        uint32_t q = 0;
        if (k * kFineThreads + threadIdx.x < n) {
            uint32_t w, o;
            read_rec(rec[k], 0, cs, w, o);
            q = atomicAdd(&lcnt[(w >> tile_shift) & (T - 1)], 1u);
        }
        rk[k / 2] = k % 2 ? rk[k / 2] | q << 16 : q;
    }
    __syncthreads();
    uint32_t carry = 0;
    for (uint32_t t0 = 0; t0 < T; t0 += kFineThreads) {
        const uint32_t t = t0 + threadIdx.x;
        const uint32_t c = t < T ? lcnt[t] : 0u;
        uint32_t tot;
        const uint32_t ex = carry + block_exscan<kFineThreads>(c, tot, sh);
        carry += tot;
        if (t < T) {
            lpre[t] = ex;
            // (mod 2^32) stage slot j of the tile goes to word lcnt + j
            if (c) lcnt[t] = atomicAdd(&cur[t_lo + t], c) - ex;
        }
    }
    __syncthreads();
#pragma unroll
    for (uint32_t k = 0; k < P; k++) {
        if (k * kFineThreads + threadIdx.x >= n) continue;
        uint32_t w, o;
        read_rec(rec[k], 0, cs, w, o);
        const uint32_t q = k % 2 ? rk[k / 2] >> 16 : rk[k / 2] & 0xffffu;
        stage[lpre[(w >> tile_shift) & (T - 1)] + q] = rec[k];
    }
    __syncthreads();
    // out in tile order: the lanes of a wave store runs of consecutive words
    for (uint32_t j = threadIdx.x; j < n; j += kFineThreads) {
        uint32_t w, o;
        read_rec(stage[j], 0, cs, w, o);
        R2 out;
        if constexpr (sizeof(R) == 8 && sizeof(R2) == 8)
            out = stage[j];
        else
            out = make_rec<R2>(w, o, tile_shift);
        bins[lcnt[(w >> tile_shift) & (T - 1)] + j] = out;
    }
}

hipError_t launch_fine(hipStream_t s, uint32_t grid_n, uint32_t V, const uint32_t *hdr,
                       const uint32_t *bins1, const uint32_t *coff, const uint32_t *citems,
                       const uint32_t *ncitems, uint32_t tile_shift, uint32_t fshift,
                       uint32_t ntiles, uint32_t *tile_cnt, const ScanArgs &sa, uint32_t *bins)
{
    if (grid_n == 0) return hipSuccess;
    if (!sa.sums || sa.groups != 1 || fshift == 0 || (1u << fshift) > kFineLdsTiles)
        return hipErrorInvalidValue;
    const uint32_t ncoarse = (ntiles + (1u << fshift) - 1) >> fshift;
    auto go = [&](auto *b1, auto *b2) {
        using R = std::remove_pointer_t<decltype(b1)>;
        using R2 = std::remove_pointer_t<decltype(b2)>;
        const uint32_t nb = (uint32_t)(2 * (uint64_t)grid_n / fine_chunk(sizeof(R) == 8)) + ncoarse;
        k_fine_count<R><<<nb, kFineThreads, (size_t)4 << fshift, s>>>(
            b1, coff, citems, ncitems, tile_shift, fshift, tile_cnt, hdr);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        const uint32_t nch = tile_scan_chunks(ntiles);
        k_tile_sums<<<nch, kScanThreads, 0, s>>>(tile_cnt, ntiles, sa.chunk, sa.sums);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
        k_tile_offsets<<<nch, kScanThreads, 0, s>>>(tile_cnt, ntiles, sa, hdr);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
        k_fine_fill<R, R2><<<nb, kFineThreads, fine_fill_lds<R>(fshift), s>>>(
            b1, coff, citems, ncitems, tile_shift, fshift, sa.cur, b2, hdr);
        return hipGetLastError();
    };
    uint32_t *b1 = const_cast<uint32_t *>(bins1);
    if (!rec_wide(V, tile_shift + fshift)) return go(b1, bins);
    if (!rec_wide(V, tile_shift)) return go((uint64_t *)b1, bins);
    return go((uint64_t *)b1, (uint64_t *)bins);
}

// ---------------------------------------------------------------------------
// Staged scatter, up to kStagMaxC columns: one lane per record, all C columns
// in turn, each lane starting at a column of its own (lane l at l mod C), so
// that the lanes of a wave hit different columns of the LDS delta at every
// step: 64 lanes on one column of a 4- to 16-vertex tile would meet on few
// words, and the LDS serializes atomics to one word (a 64-lane ds_xor_b64 on
// one word takes 128 clocks per CU, on 64 words 7, on a staggered wave 8-11).
//
// What bounds it.  Dense batches: VALU issue (busy all the time), 19
// instructions per (record, column), 8 of them the two 64-bit products.  The
// two LDS atomics beside them keep the LDS busy for 80 to 93% of the time;
// fewer bank conflicts (rows padded to 16 words: 8 clocks per atomic instead of
// 10) changed nothing.  Against one lane per (record, column) pair the record is
// decoded once instead of read back from LDS (24 B) by each of its C lanes,
// no lane idles (64 mod C did), the column seeds are C registers, the column
// offset is the instruction's offset field, and the finalizer's last step
// z ^ (z >> 31) is left to the fold: it is linear over XOR, so the planes
// hold XORs of z and only the low word of the hash is formed, for its depth.
// Sparse batches (few records per vertex): HBM, the lines of the changed
// buckets read and written; the fold issues the loads of several buckets
// before their stores, clears the delta as it reads it, and the next item's
// descriptor and first records are loaded under the current item.
//
// Deep pairs (depth >= rows; odds 2^-rows each) fall into one extra LDS row
// that is never folded, and after every two columns the wave branches if it
// has one, to send it to HBM with device atomics.  Against a bit per column
// and a loop over them after the columns, which hashed them again: 1.75 ms
// instead of 1.82 for 1.3e8 records on 131,072 of 2^20 vertices, C = 20.
//
// Measured on one MI355X (records, vertices, C: this kernel / the pair
// layout / one lane per record without the stagger, each at its best tile):
//   3.4e7 records on 32,768 vertices, C = 20: 0.41 / 0.57 / 0.73 ms
//   8.0e6 on 65,536, C = 16:                  0.107 / 0.139 / 0.165 ms
//   2.0e6 on 16,384, C = 14:                  0.033 / 0.041 / 0.046 ms
//   6.0e6 on 200,003, C = 18:                 0.252 / 0.260 / 0.260 ms
//   2.0e5 on 131,072, C = 17:                 0.058 / 0.073 / 0.084 ms
// (with 64-bit records and before the two changes below; 0.238 ms for the
// fourth after them)
// ---------------------------------------------------------------------------
typedef __attribute__((address_space(3))) uint64_t *LdsWords;
DEVI void lds_xor(LdsWords p, uint64_t v)
{
    __hip_atomic_fetch_xor(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// The finalizer between its first and its last step, and the low word of
// the hash given that.
DEVI uint64_t mix64_mid(uint64_t z)
{
    z *= 0xBF58476D1CE4E5B9ull;
    return (z ^ (z >> 27)) * 0x94D049BB133111EBull;
}

DEVI uint32_t mix64_low(uint64_t z)
{
    return (uint32_t)z ^ __builtin_amdgcn_alignbit((uint32_t)(z >> 32), (uint32_t)z, 31);
}

// f(integral_constant<uint32_t, T>) for T = 0 .. N-1
template <uint32_t T, uint32_t N, class F>
DEVI void static_for(F &&f)
{
    if constexpr (T < N) {
        f(std::integral_constant<uint32_t, T>{});
        static_for<T + 1, N>(f);
    }
}

constexpr uint32_t kStagThreads = 512;
constexpr uint32_t kStagWaves = kStagThreads / 64;
// Buckets a lane folds at a time.  Their loads are issued together, without a
// branch between them (lanes with nothing to fold load the tile's first
// bucket): behind branches the compiler waits for each load before the next.
// 6.0e6 records on 200,003 vertices, C = 18: 0.238 instead of 0.247 ms, where
// reading and writing the first 7 to 9 of 36 depth rows of every vertex takes
// 0.19 to 0.26 by itself; 4 or 6 buckets at a time are no faster.
constexpr uint32_t kStagFold = 3;
// Items of at most this many records go one (record, column) pair per
// thread, which fills the block; beyond two passes of that, one lane per
// record is faster even with idle lanes (24 records per tile: 0.058 against
// 0.067 ms; 240 per tile: 0.35 against 0.29 ms).
template <uint32_t C>
constexpr uint32_t kStagFew = 2 * (kStagThreads / C);

template <uint32_t C>
__global__ __launch_bounds__(kStagThreads, C <= 20 ? 6 : 4) void k_tile_scatter_stag(
    DevSketch sk, const uint32_t *__restrict__ bins, const uint32_t *__restrict__ off,
    const uint32_t *__restrict__ items, const uint32_t *__restrict__ nitems_p, uint32_t tile_shift,
    uint32_t rows, uint32_t chunk, const uint32_t *__restrict__ hdr,
    unsigned long long *__restrict__ touched)
{
    extern __shared__ uint64_t lds[];
    uint32_t nchanged = 0;  // buckets this thread changed in HBM
    const bool err = hdr[HDR_REJ] != 0;
    const uint32_t TV = 1u << tile_shift;
    const uint32_t V = sk.V, D = sk.D;
    constexpr uint32_t RS = 2 * C;             // words per vertex and row: alpha, then gamma
    const uint32_t rfast = min(rows, D - 1);   // <= 31
    const uint32_t VS = (rfast + 1) * RS;      // words per vertex; last row: deep pairs, if any
    const uint32_t words = VS << tile_shift;
    const uint64_t DC2 = (uint64_t)D * C * 2;  // words per vertex in HBM
    const uint32_t stop = 1u << rfast;
    const uint32_t deep = rows == D ? 64u : rfast;  // depth of a deep pair in LDS (64: none)
    const uint32_t nitems = err ? 0u : *nitems_p;
    const uint32_t s = threadIdx.x % C;        // first column of this lane
    const uint32_t few_i = threadIdx.x / C;    // its record in an item of few records
    const uint32_t lane = __lane_id();
    const uint32_t wid = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
    const LdsWords L = (LdsWords)lds;
    const uint32_t lbase = (uint32_t)(uintptr_t)L;
    const LdsWords seedt = L + words;          // the column seeds, twice over
    if (threadIdx.x < 2 * C)
        seedt[threadIdx.x] = mix64_head(sk.seeds[threadIdx.x < C ? threadIdx.x : threadIdx.x - C]);
    // lanes whose t-th column wraps to the first ones (scalar registers)
    uint64_t wrap[C];
    static_for<0, C>([&](auto tt) {
        constexpr uint32_t t = decltype(tt)::value;
        wrap[t] = __ballot(s + t >= C);
    });
    const uint32_t G = gridDim.x;
    uint32_t it = blockIdx.x, it1 = it + G;
    uint32_t tile = 0, rb = 0, re = 0, j = 0, tile1 = 0, j1 = 0;
    if (it < nitems) {
        tile = items[2 * it];
        j = items[2 * it + 1];
        rb = off[tile];
        re = off[tile + 1];
    }
    if (it1 < nitems) {
        tile1 = items[2 * it1];
        j1 = items[2 * it1 + 1];
    }
    for (uint32_t q = threadIdx.x; q < words; q += kStagThreads) L[q] = 0;
    uint32_t cb, ce;  // the item's records: part `part` of its tile's, in equal parts
    auto range = [&](uint32_t part) {
        const uint32_t n = re - rb;
        uint32_t per = n;
        if (n > chunk) {
            const uint32_t k = (n + chunk - 1) / chunk;
            per = (n + k - 1) / k;
        }
        cb = min(re, rb + part * per);
        ce = min(re, cb + per);
    };
    range(j);
    uint32_t r = cb + (ce - cb <= kStagFew<C> ? few_i : threadIdx.x);
    uint32_t rec = r < ce ? bins[r] : 0;
    while (it < nitems) {
        const bool single = re - rb <= chunk;
        const uint32_t w0 = tile << tile_shift;
        uint32_t rb1 = 0, re1 = 0;
        if (it1 < nitems) {
            rb1 = off[tile1];
            re1 = off[tile1 + 1];
        }
        const uint32_t it2 = it1 + G;
        uint32_t tile2 = 0, j2 = 0;
        if (it2 < nitems) {
            tile2 = items[2 * it2];
            j2 = items[2 * it2 + 1];
        }
        __syncthreads();  // delta cleared (and, first, the seeds stored)
        if (ce - cb <= kStagFew<C>) {
            const uint64_t seed1 = seedt[s];
            while (r < ce && few_i < kStagThreads / C) {
                const uint32_t vl = rec & (TV - 1), w = w0 + vl, o = rec >> tile_shift;
                r += kStagThreads / C;
                if (r < ce) rec = bins[r];
                const uint64_t x = (uint64_t)min(w, o) * V + max(w, o);
                const uint64_t z = mix64_mid(mix64_head(x) ^ seed1);
                const uint32_t d0 = (uint32_t)__builtin_ctz(mix64_low(z) | stop);
                const LdsWords p = L + (vl * VS + d0 * RS + s);
                lds_xor(p, x);
                lds_xor(p + C, z);
                if (d0 == deep) {
                    const uint64_t h = z ^ (z >> 31);
                    uint64_t *bp =
                        sk.b + (uint64_t)(w0 + vl) * DC2 + 2 * (depth_of(h, D) * C + s);
                    gxor(bp, x);
                    gxor(bp + 1, h);
                    nchanged++;
                }
            }
        } else {
            uint64_t seed1[C];
            static_for<0, C>([&](auto tt) {
                constexpr uint32_t t = decltype(tt)::value;
                seed1[t] = seedt[s + t];
            });
            while (r < ce) {
                const uint32_t vl = rec & (TV - 1), w = w0 + vl, o = rec >> tile_shift;
                r += kStagThreads;
                if (r < ce) rec = bins[r];  // in flight while this one is hashed
                const uint64_t x = (uint64_t)min(w, o) * V + max(w, o);
                const uint64_t y = mix64_head(x);
                const uint32_t a0 = lbase + __umul24(vl, VS * 8) + s * 8, a1 = a0 - C * 8;
                // columns t and t + 1 (t + 1 < C) of the record
                auto columns = [&](auto tt) {
                    constexpr uint32_t t = decltype(tt)::value * 2;
                    constexpr uint32_t N = t + 1 < C ? 2 : 1;
                    uint64_t z[2];
                    uint32_t d0[2];
                    static_for<0, N>([&](auto kk) {
                        constexpr uint32_t k = decltype(kk)::value;
                        z[k] = mix64_mid(y ^ seed1[t + k]);
                        d0[k] = (uint32_t)__builtin_ctz(mix64_low(z[k]) | stop);
                        uint32_t a = a0;
                        if (t + k > 0)
                            asm("v_cndmask_b32_e64 %0, %1, %2, %3"
                                : "=v"(a)
                                : "v"(a0), "v"(a1), "s"(wrap[t + k]));
                        const LdsWords p = (LdsWords)(__umul24(d0[k], RS * 8) + a) + t + k;
                        lds_xor(p, x);
                        lds_xor(p + C, z[k]);
                    });
                    if (d0[0] == deep || (N > 1 && d0[1] == deep)) {
                        static_for<0, N>([&](auto kk) {
                            constexpr uint32_t k = decltype(kk)::value;
                            if (d0[k] != deep) return;
                            uint32_t c = s;
                            asm volatile("" : "+v"(c));  // (not a register per column)
                            c += t + k;
                            if (c >= C) c -= C;
                            const uint64_t h = z[k] ^ (z[k] >> 31);
                            uint64_t *bp = sk.b + (uint64_t)(w0 + vl) * DC2 +
                                           2 * (depth_of(h, D) * C + c);
                            gxor(bp, x);
                            gxor(bp + 1, h);
                            nchanged++;
                        });
                    }
                    // keep the unrolled columns in order: interleaving all of
                    // them takes 60 more registers
                    __builtin_amdgcn_sched_barrier(0);
                };
                static_for<0, (C + 1) / 2>(columns);
            }
        }
        // the next item's first records, in flight during the fold
        rb = rb1;
        re = re1;
        range(j1);
        r = cb + (ce - cb <= kStagFew<C> ? few_i : threadIdx.x);
        if (it1 < nitems && r < ce) rec = bins[r];
        tile = tile1;
        j1 = j2;
        tile1 = tile2;
        it = it1;
        it1 = it2;
        __syncthreads();
        // Fold: a wave takes 64 consecutive buckets of one vertex at a time,
        // F of those units together.
        constexpr uint32_t F = kStagFold;
        const uint32_t per_v = rows * C;
        const uint32_t units = ((per_v + 63) / 64) << tile_shift;
        uint8_t *g0 = (uint8_t *)(sk.b + (uint64_t)w0 * DC2);
        for (uint32_t u0 = wid; u0 < units; u0 += F * kStagWaves) {
            uint64_t da[F], z[F];
            uint32_t at[F];  // byte offset of the bucket, the tile's first one if it stays
#pragma unroll
            for (uint32_t k = 0; k < F; k++) {
                const uint32_t un = u0 + k * kStagWaves;
                const uint32_t vl = un & (TV - 1), rc = (un >> tile_shift) * 64 + lane;
                da[k] = z[k] = 0;
                at[k] = 0;
                if (un < units && rc < per_v && w0 + vl < V) {
                    const LdsWords p = L + vl * VS + rc + (rc / C) * C;
                    da[k] = p[0];
                    z[k] = p[C];
                    if (da[k] | z[k]) {
                        p[0] = 0;
                        p[C] = 0;
                        at[k] = vl * (uint32_t)DC2 * 8 + rc * 16;
                        nchanged++;
                    }
                }
            }
            if (single) {
                Bucket2 b[F];
#pragma unroll
                for (uint32_t k = 0; k < F; k++) b[k] = *(const Bucket2 *)(g0 + at[k]);
#pragma unroll
                for (uint32_t k = 0; k < F; k++) {
                    b[k].x ^= da[k];
                    b[k].y ^= z[k] ^ (z[k] >> 31);
                }
#pragma unroll
                for (uint32_t k = 0; k < F; k++)
                    if (da[k] | z[k]) *(Bucket2 *)(g0 + at[k]) = b[k];
            } else {
#pragma unroll
                for (uint32_t k = 0; k < F; k++) {
                    const uint64_t dg = z[k] ^ (z[k] >> 31);
                    if (da[k]) gxor((uint64_t *)(g0 + at[k]), da[k]);
                    if (dg) gxor((uint64_t *)(g0 + at[k]) + 1, dg);
                }
            }
        }
    }
    add_touched(touched, nchanged, (uint32_t *)lds);
}

constexpr uint32_t kTileThreads = 512;
constexpr uint32_t kTileWaves = kTileThreads / 64;
constexpr uint32_t kTileLdsMax = 65536;  // dynamic LDS per block, bytes
constexpr uint32_t kTileStage = 512;     // records staged per pass

// The staged records (24 B each: edge index and the first step of its
// hash, byte offset of the endpoint's words in an LDS depth row, local
// vertex) must fit beside the LDS delta.
constexpr uint32_t kStagedRecBytes = 24;
static bool tile_stage_fits(size_t delta_bytes)
{
    return delta_bytes + (size_t)kTileStage * kStagedRecBytes <= kTileLdsMax;
}

bool tile_geometry_fits(uint32_t rows, uint32_t C, uint32_t tv, uint32_t layout)
{
    const size_t delta = (size_t)2 * rows * C * tv * sizeof(uint64_t);
    if (C < 1 || C > 64 || rows < 1) return false;
    return layout == kLayoutRecord ? delta <= kTileLdsMax : tile_stage_fits(delta);
}

struct StagedRec {
    uint64_t x;   // edge index u*V + v of the record's update
    uint64_t y;   // mix64_head(x)
    uint32_t qb;  // vl*C*8: byte offset of the endpoint's words in a depth row
    uint32_t vl;  // endpoint - first vertex of the tile
};

// XOR one (record, column) pair into the LDS delta (or HBM for a deep row).
// colb = column * 8; RSB = bytes per LDS depth row; pg = gamma plane offset
// in bytes; seed1 = mix64_head(column seed).  The depth is ctz of the hash's
// low word with a stop bit at rfast = min(rows, D-1, 31); only when no bit
// below rfast is set (odds 2^-rfast) is the full depth taken, and a depth >=
// rows goes to HBM with device atomics.
DEVI void tile_pair(uint8_t *lds8, uint32_t RSB, uint32_t pg, uint32_t rows, uint32_t rfast,
                    uint32_t stop, uint32_t colb, uint64_t seed1, const StagedRec &r,
                    const DevSketch &sk, uint32_t w0, uint64_t DC2, uint32_t &nchanged)
{
    const uint64_t h = mix64_tail(r.y ^ seed1);
    const uint32_t d0 = (uint32_t)__builtin_ctz((uint32_t)h | stop);  // <= 31
    if (d0 != rfast) {
        const uint32_t a = __umul24(d0, RSB) + r.qb + colb;
        lxor((uint64_t *)(lds8 + a), r.x);
        lxor((uint64_t *)(lds8 + a + pg), h);
        return;
    }
    const uint32_t d = depth_of(h, sk.D);
    if (d < rows) {
        // (d < 64 and RSB < 2^24: the masks let the compiler use the
        // 24-bit multiply)
        const uint32_t a = __umul24(d & 63u, RSB & 0xffffffu) + r.qb + colb;
        lxor((uint64_t *)(lds8 + a), r.x);
        lxor((uint64_t *)(lds8 + a + pg), h);
    } else {
        uint64_t *bp = sk.b + (uint64_t)(w0 + r.vl) * DC2 + 2 * (uint64_t)d * sk.C + colb / 4;
        gxor(bp, r.x);
        gxor(bp + 1, h);
        nchanged++;
    }
}

// More than kStagMaxC columns, or wide records.  One (record, column) pair per
// lane: the edge index x = u*V + v of the record's update is hashed for column
// c and (x, h) is XOR-ed into bucket (d, c) of its endpoint.  Lane l of a wave
// takes column l mod C of record l / C (G = 64 / C records per wave step,
// lanes l >= G*C idle), so
// the C lanes of a record hit C consecutive LDS words and the hash seed is a
// per-lane constant.
//
// LDS: the delta's alpha and gamma planes, word d*TV*C + vl*C + c for depth
// row d < rows, local vertex vl, column c; then the staged records.
//
// touched (may be null) receives the number of buckets the launch changes
// in HBM: folded buckets with a nonzero delta, plus one per pair that goes
// to a deep row directly.
template <class R>
__global__ __launch_bounds__(kTileThreads) void k_tile_scatter(
    DevSketch sk, const R *__restrict__ bins, const uint32_t *__restrict__ off,
    const uint32_t *__restrict__ items, const uint32_t *__restrict__ nitems_p, uint32_t tile_shift,
    uint32_t rows, uint32_t chunk, const uint32_t *__restrict__ hdr,
    unsigned long long *__restrict__ touched)
{
    uint32_t nchanged = 0;  // buckets this thread changed in HBM
    extern __shared__ uint64_t lds[];
    uint8_t *lds8 = (uint8_t *)lds;
    const bool err = hdr[HDR_REJ] != 0;
    const uint32_t TV = 1u << tile_shift;
    const uint32_t C = sk.C, V = sk.V;
    const uint32_t RS = TV * C;             // words per LDS depth row (< 2^12)
    const uint32_t plane = rows * RS;       // words per LDS plane
    const uint64_t DC2 = (uint64_t)sk.D * C * 2;  // words per vertex in HBM
    const uint32_t rfast = min(min(rows, sk.D - 1), 31u);
    const uint32_t stop = 1u << rfast;
    const uint64_t *la = lds;               // alpha plane
    const uint64_t *lg = lds + plane;       // gamma plane
    StagedRec *st = (StagedRec *)(lds + 2 * plane);
    const uint32_t nitems = err ? 0u : *nitems_p;

    const uint32_t lane = __lane_id(), wid = threadIdx.x / 64;
    const uint32_t G = 64 / C;              // records (or rows) per wave step
    const uint32_t WG = kTileWaves * G;     // records per block step
    const uint32_t slot = lane / C;
    const uint32_t col = lane - slot * C;
    const bool active = slot < G;
    const uint32_t colb = col * 8;
    const uint64_t seed1 = active ? mix64_head(sk.seeds[col]) : 0;

    for (uint32_t it = blockIdx.x; it < nitems; it += gridDim.x) {
        const uint32_t tile = items[2 * it];
        const uint32_t j = items[2 * it + 1];
        const uint32_t rb = off[tile], re = off[tile + 1];
        const uint32_t cb = rb + j * chunk;
        const uint32_t ce = min(re, cb + chunk);
        const bool single = (re - rb) <= chunk;
        const uint32_t w0 = tile << tile_shift;
        if (cb >= ce) continue;  // (block-uniform) nothing to fold

        for (uint32_t q = threadIdx.x; q < 2 * plane; q += kTileThreads) lds[q] = 0;

        for (uint32_t sb = cb; sb < ce; sb += kTileStage) {
            const uint32_t ns = min(kTileStage, ce - sb);
            // stage: decode each record once
            for (uint32_t i = threadIdx.x; i < ns; i += kTileThreads) {
                uint32_t w, o;
                read_rec(bins[sb + i], w0, tile_shift, w, o);
                const uint32_t vl = w - w0;
                StagedRec r;
                r.x = (uint64_t)min(w, o) * V + max(w, o);
                r.y = mix64_head(r.x);
                r.qb = __umul24(vl, C) * 8;
                r.vl = vl;
                st[i] = r;
            }
            __syncthreads();
            if (active) {
                // full block steps need no bound check; the last one does
                const uint32_t full = ns / WG * WG;
                uint32_t i = wid * G + slot;
                for (; i + WG < full; i += 2 * WG) {
                    const StagedRec r0 = st[i], r1 = st[i + WG];
                    tile_pair(lds8, RS * 8, plane * 8, rows, rfast, stop, colb, seed1, r0, sk,
                              w0, DC2, nchanged);
                    tile_pair(lds8, RS * 8, plane * 8, rows, rfast, stop, colb, seed1, r1, sk,
                              w0, DC2, nchanged);
                }
                if (i < full) {
                    tile_pair(lds8, RS * 8, plane * 8, rows, rfast, stop, colb, seed1, st[i], sk,
                              w0, DC2, nchanged);
                    i += WG;
                }
                if (i < ns)
                    tile_pair(lds8, RS * 8, plane * 8, rows, rfast, stop, colb, seed1, st[i], sk,
                              w0, DC2, nchanged);
            }
            __syncthreads();
        }

        // Fold the delta into HBM: lanes (slot, column) of a wave take G
        // vertices at a time and walk their depth rows, so each step reads
        // C consecutive words per row in LDS and C consecutive buckets
        // (16 B each) per row in HBM.
        if (active) {
            const uint32_t nvt = min(TV, V - w0);
            for (uint32_t vl = wid * G + slot; vl < nvt; vl += WG) {
                uint32_t q = __umul24(vl, C) + col;
                uint64_t *g = sk.b + (uint64_t)(w0 + vl) * DC2 + 2 * col;
                for (uint32_t d = 0; d < rows; d++, q += RS, g += 2 * C) {
                    const uint64_t da = la[q], dg = lg[q];
                    if ((da | dg) == 0) continue;
                    nchanged++;
                    if (single) {
                        ulonglong2 *g2 = (ulonglong2 *)g;
                        ulonglong2 b = *g2;
                        b.x ^= da;
                        b.y ^= dg;
                        *g2 = b;
                    } else {
                        if (da) gxor(g, da);
                        if (dg) gxor(g + 1, dg);
                    }
                }
            }
        }
        __syncthreads();
    }
    add_touched(touched, nchanged, (uint32_t *)lds);
}

hipError_t launch_bin(hipStream_t s, const BatchDesc *desc, BatchDesc dv, uint32_t grid_n,
                      DevSketch sk, const uint32_t *hdr, const StagedParams &p,
                      uint32_t *tile_cur, uint32_t *bins, const uint32_t *tile_goff,
                      const uint32_t *tile_rel)
{
    if (grid_n == 0) return hipSuccess;
    const uint32_t fb = (grid_n + kFillPerBlock - 1) / kFillPerBlock;
    // the fill's blocks cover the same updates as the classify blocks
    static_assert(kFillPerBlock == kClsPerBlock,
                  "fill and classify blocks must cover the same updates");
    static_assert(kRelMaxTiles <= kFillStageTiles && kRelMaxTiles <= kLdsHistMax,
                  "tile_rel needs the classify's LDS counts and the staged fill");
    if (tile_rel && (p.ntiles > kRelMaxTiles || !tile_goff)) return hipErrorInvalidValue;
    auto go = [&](auto *b) {
        using R = std::remove_pointer_t<decltype(b)>;
        if (p.ntiles <= kFillStageTiles)
            k_tile_fill_staged<R>
                <<<fb, kFillThreads, fill_stage_lds(p.ntiles, sizeof(R) == 8), s>>>(
                    desc, dv, sk.V, p.tile_shift, p.ntiles, tile_cur, b, hdr, tile_goff, tile_rel);
        else
            k_tile_fill<R><<<fb, kFillThreads, 0, s>>>(desc, dv, sk.V, p.tile_shift, p.ntiles,
                                                       tile_cur, b, hdr);
        return hipGetLastError();
    };
    return rec_wide(sk.V, p.tile_shift) ? go((uint64_t *)bins) : go(bins);
}

// f(integral_constant<uint32_t, C - 1>) for C = 1 .. kStagMaxC (host)
template <class F, uint32_t... T>
static void for_columns_impl(F &f, std::integer_sequence<uint32_t, T...>)
{
    (f(std::integral_constant<uint32_t, T>{}), ...);
}
template <class F>
static void for_columns(F &f)
{
    for_columns_impl(f, std::make_integer_sequence<uint32_t, kStagMaxC>{});
}

hipError_t launch_tile(hipStream_t s, DevSketch sk, const uint32_t *hdr, const StagedParams &p,
                       const uint32_t *tile_off, const uint32_t *bins, const uint32_t *items,
                       const uint32_t *nitems, unsigned long long *touched)
{
    const size_t delta = (size_t)2 * p.rows * sk.C * (1u << p.tile_shift) * sizeof(uint64_t);
    if (!tile_geometry_fits(p.rows, sk.C, 1u << p.tile_shift, p.layout))
        return hipErrorInvalidValue;
    const bool wide = rec_wide(sk.V, p.tile_shift);
    if (sk.C <= kStagMaxC && !wide) {
        // (rows beyond what one word's trailing zero count tells would hold a
        // pair in 2^31: it goes to HBM like any deep one, 167 us against 326
        // in the pair kernel with 36 rows, 1,000,000 updates on 65,536
        // vertices, C = 20)
        const uint32_t rows = min(p.rows, 31u), rfast = min(rows, sk.D - 1);
        const size_t lds = ((size_t)(rfast + 1) * sk.C * 16 << p.tile_shift) + (size_t)sk.C * 16;
        if (lds > kCuLds) return hipErrorInvalidValue;
        // Dense batches (64 records per vertex and more) have heavy items:
        // more blocks than fit, handed out by the hardware, even out what
        // the items differ by (0.44 against 0.50 ms for 3.4e7 records on
        // 32,768 vertices).  Light items: as many blocks as fit, each
        // prefetching its next item (0.252 against 0.266 ms for 6.0e6
        // records on 200,003 vertices, 0.058 against 0.073 ms for 2.0e5 on
        // 131,072).
        const uint32_t fit = kCus * max(1u, min(3u, (uint32_t)(kCuLds / (lds + 1280))));
        const uint32_t def = p.records >= (uint64_t)64 * sk.V ? 16 * kCus : fit;
        const uint32_t grid = min(p.items_cap, p.grid ? p.grid : def);
        hipError_t e = hipErrorInvalidValue;
        auto go = [&](auto cc) {
            constexpr uint32_t C = decltype(cc)::value + 1;
            if (sk.C != C) return;
            k_tile_scatter_stag<C><<<grid, kStagThreads, lds, s>>>(
                sk, bins, tile_off, items, nitems, p.tile_shift, rows, p.chunk, hdr, touched);
            e = hipGetLastError();
        };
        for_columns(go);
        return e;
    }
    // Persistent grid: a few blocks per CU, each looping over work items.
    const uint32_t grid = min(p.items_cap, p.grid ? p.grid : 256u * 8u);
    const size_t lds = delta + (size_t)kTileStage * kStagedRecBytes;
    if (wide)
        k_tile_scatter<<<grid, kTileThreads, lds, s>>>(sk, (const uint64_t *)bins, tile_off, items,
                                                       nitems, p.tile_shift, p.rows, p.chunk, hdr,
                                                       touched);
    else
        k_tile_scatter<<<grid, kTileThreads, lds, s>>>(sk, bins, tile_off, items, nitems,
                                                       p.tile_shift, p.rows, p.chunk, hdr, touched);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Flag compaction: exclusive scan of the per-block flag counts (one block),
// then every classify block's region is copied to its offset, giving the
// flagged updates of the batch in stream order.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kScanThreads) void k_flag_scan(const uint32_t *__restrict__ fcnt,
                                                            uint32_t nb,
                                                            uint32_t *__restrict__ foff)
{
    __shared__ uint32_t sh[160];
    uint32_t carry = 0;
    for (uint32_t base = 0; base < nb; base += kScanThreads) {
        const uint32_t b = base + threadIdx.x;
        const uint32_t c = b < nb ? fcnt[b] : 0u;
        uint32_t tot;
        const uint32_t ex = block_exscan<kScanThreads>(c, tot, sh);
        if (b < nb) foff[b] = carry + ex;
        carry += tot;
    }
}

__global__ __launch_bounds__(256) void k_flag_compact(const uint64_t *__restrict__ fupd,
                                                      const uint32_t *__restrict__ fpos,
                                                      const uint32_t *__restrict__ fcnt,
                                                      const uint32_t *__restrict__ foff,
                                                      uint64_t *__restrict__ oupd,
                                                      uint32_t *__restrict__ opos)
{
    const uint32_t b = blockIdx.x;
    const uint32_t c = fcnt[b], o = foff[b];
    const uint32_t src = b * kClsPerBlock;
    for (uint32_t k = threadIdx.x; k < c; k += blockDim.x) {
        oupd[o + k] = fupd[src + k];
        if (opos) opos[o + k] = fpos[src + k];
    }
}

hipError_t launch_flag_compact(hipStream_t s, uint32_t n, const uint64_t *fupd,
                               const uint32_t *fpos, const uint32_t *fcnt, uint32_t *foff,
                               uint64_t *oupd, uint32_t *opos)
{
    const uint32_t nb = classify_blocks(n);
    if (nb == 0) return hipSuccess;
    k_flag_scan<<<1, kScanThreads, 0, s>>>(fcnt, nb, foff);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    k_flag_compact<<<nb, 256, 0, s>>>(fupd, fpos, fcnt, foff, oupd, opos);
    return hipGetLastError();
}

// Flag check against a newer forest, one wave per classify block's region:
// each step reads 64 flagged updates, keeps those the classify rule still
// flags against `lp`, and writes them back packed at the front of the
// region (a step writes below the next step's reads: in place is safe).
constexpr uint32_t kReflagThreads = 256;

__global__ __launch_bounds__(kReflagThreads) void k_reflag(uint32_t V, const uint64_t *__restrict__ lp,
                                                           const uint32_t *__restrict__ hdr,
                                                           uint64_t *__restrict__ fupd,
                                                           uint32_t *__restrict__ fcnt,
                                                           uint32_t *__restrict__ fdel, uint32_t nb)
{
    const uint32_t b = blockIdx.x * (kReflagThreads / 64) + threadIdx.x / 64;
    if (b >= nb || hdr[HDR_REJ] != 0) return;  // whole waves
    const uint32_t lane = __lane_id();
    const uint32_t c = fcnt[b];
    uint64_t *r = fupd + (size_t)b * kClsPerBlock;
    uint32_t w = 0, nd = 0;
    for (uint32_t k0 = 0; k0 < c; k0 += 64) {
        const uint32_t k = k0 + lane;
        bool keep = false, del = false;
        uint64_t p = 0;
        if (k < c) {
            p = r[k];
            uint32_t u, v;
            unpack(p, V, u, v, del);
            const uint64_t lu = lp[u], lv = lp[v];
            keep = (uint32_t)lu != (uint32_t)lv;
            if (!keep && del) keep = (uint32_t)(lu >> 32) == v || (uint32_t)(lv >> 32) == u;
        }
        const uint64_t m = __ballot(keep);
        if (keep) r[w + lanes_below(m)] = p;
        w += (uint32_t)__popcll(m);
        nd += (uint32_t)__popcll(__ballot(keep && del));
    }
    if (lane == 0) {
        fcnt[b] = w;
        fdel[b] = nd;
    }
}

hipError_t launch_reflag(hipStream_t s, uint32_t V, const uint64_t *lp, uint32_t *hdr,
                         uint64_t *fupd, uint32_t *hout, const FlagInline &fi, uint32_t *foff,
                         uint64_t *oupd, bool check)
{
    if (!fi.fdel || !fi.fcnt || fi.fupd != fupd || fi.tiles_only || !foff || !oupd)
        return hipErrorInvalidValue;
    if (fi.nb) {
        hipError_t e = hipSuccess;
        if (check) {
            const uint32_t per = kReflagThreads / 64;
            k_reflag<<<(fi.nb + per - 1) / per, kReflagThreads, 0, s>>>(
                V, lp, hdr, fupd, const_cast<uint32_t *>(fi.fcnt), fi.fdel, fi.nb);
            e = hipGetLastError();
            if (e != hipSuccess) return e;
        }
        // the ordered list, before the header: the host only copies it
        k_flag_scan<<<1, kScanThreads, 0, s>>>(fi.fcnt, fi.nb, foff);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
        k_flag_compact<<<fi.nb, 256, 0, s>>>(fupd, nullptr, fi.fcnt, foff, oupd, nullptr);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    // header only: no tile counts, and the verdict of the first scan
    FlagInline f2 = fi;
    f2.checked = 1;
    k_tile_scan<<<1, kScanThreads, 0, s>>>(nullptr, 0, ScanArgs{}, hdr, hout, f2);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Utility fills.
// ---------------------------------------------------------------------------
__global__ void k_zero64(uint64_t *p, size_t n)
{
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n;
         i += (size_t)gridDim.x * blockDim.x)
        p[i] = 0;
}

__global__ void k_zero32(uint32_t *p, size_t n)
{
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n;
         i += (size_t)gridDim.x * blockDim.x)
        p[i] = 0;
}

hipError_t launch_zero(hipStream_t s, uint64_t *p, size_t n)
{
    if (n == 0) return hipSuccess;
    size_t blocks = (n + 255) / 256;
    if (blocks > 8192) blocks = 8192;
    k_zero64<<<(uint32_t)blocks, 256, 0, s>>>(p, n);
    return hipGetLastError();
}

hipError_t launch_zero32(hipStream_t s, uint32_t *p, size_t n)
{
    if (n == 0) return hipSuccess;
    size_t blocks = (n + 255) / 256;
    if (blocks > 8192) blocks = 8192;
    k_zero32<<<(uint32_t)blocks, 256, 0, s>>>(p, n);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Segmented XOR reduction (component sketches) with the query of every set in
// the same launch.  A work item is (set, begin, end, items of the set), at
// most kRedChunk members of one set.  A block takes an item: NG groups of 256
// threads stream every NG-th member's slab, one 16-byte bucket per lane and
// load, several members' loads in flight, XOR them into registers and add up
// in LDS.  A set of one item is then queried from registers.  A set of
// several items adds up in its aggregate with device atomics; the block that
// takes the set's last ticket reads it back and queries it.
//
// Query of an aggregate: every lane checks its buckets (alpha != 0, checksum
// and depth derived again from alpha, alpha decodes to u < v < V), the block
// takes the minimum canonical rank c*D + (D-1-d) among the good ones, and the
// lane that holds it writes the edge; an OR over all words tells EMPTY.
//
// Large sets are bound by HBM (the slabs read once); small ones by latency,
// hence one launch where there were a zero fill, a reduction, a query and a
// copy in either direction: members and items come from pinned host memory
// when they are few, results go there, and a lone item publishes them itself.
// ---------------------------------------------------------------------------
constexpr uint32_t kRedThreads = 256;  // per group

// KB buckets per lane: C*D <= KB * kRedThreads.  Dynamic LDS: (NG - 1) slabs.
template <uint32_t KB, uint32_t NG>
__global__ __launch_bounds__(NG *kRedThreads) void k_reduce_sample(ReduceArgs a)
{
    extern __shared__ uint64_t lds[];
    Bucket2 *part = (Bucket2 *)lds;  // slabs of groups 1 .. NG-1
    __shared__ uint32_t s_item[4], s_mem[kRedChunk];
    __shared__ uint32_t s_best[kRedThreads / 64], s_any[kRedThreads / 64];
    __shared__ uint32_t s_last;
    const uint32_t C = a.C, D = a.D, nb = C * D;
    const uint32_t tid = threadIdx.x % kRedThreads;
    const uint32_t grp = __builtin_amdgcn_readfirstlane(threadIdx.x / kRedThreads);
    for (uint32_t it = blockIdx.x; it < a.nitems; it += gridDim.x) {
        uint32_t set = it, n = 1, parts = 1;
        bool frag = false;
        if (a.items) {
            // one wave fetches the item and its members (host memory, maybe;
            // an only item comes in the arguments: two reads over the host
            // link, one after the other, less, 2 of 39 us for the cut of 37
            // vertices)
            if (threadIdx.x < 64) {
                uint32_t w = 0;
                const uint32_t *item = a.nitems == 1 ? a.one : a.items + 4 * it;
                if (threadIdx.x < 4) w = item[threadIdx.x];
                const uint32_t b = __shfl(w, 1), e = __shfl(w, 2);
                if (threadIdx.x < 4) s_item[threadIdx.x] = w;
                if (threadIdx.x < e - b)
                    s_mem[threadIdx.x] =
                        a.nitems == 1 ? a.mem[threadIdx.x] : a.idx[b + threadIdx.x];
            }
            __syncthreads();
            set = s_item[0];
            n = s_item[2] - s_item[1];
            parts = s_item[3];
            frag = set >> 31;
            set &= 0x7fffffffu;
        }
        const Bucket2 *src = (const Bucket2 *)(frag ? a.src1 : a.src0);
        Bucket2 acc[KB];
#pragma unroll
        for (uint32_t k = 0; k < KB; k++) acc[k] = Bucket2{0, 0};
        constexpr uint32_t kAhead = KB <= 4 ? 4 : KB <= 8 ? 2 : 1;  // members in flight
        for (uint32_t j = grp; j < n; j += kAhead * NG) {
            Bucket2 t[kAhead][KB];
#pragma unroll
            for (uint32_t g = 0; g < kAhead; g++) {
                const bool in = j + g * NG < n;
                const uint32_t m =
                    !a.items ? it
                             : (uint32_t)__builtin_amdgcn_readfirstlane(s_mem[in ? j + g * NG : j]);
                const Bucket2 *s0 = src + (uint64_t)m * nb;
#pragma unroll
                for (uint32_t k = 0; k < KB; k++) {
                    const uint32_t q = k * kRedThreads + tid;
                    t[g][k] = in && q < nb ? s0[q] : Bucket2{0, 0};
                }
            }
#pragma unroll
            for (uint32_t g = 0; g < kAhead; g++)
#pragma unroll
                for (uint32_t k = 0; k < KB; k++) acc[k] ^= t[g][k];
        }
        if (NG > 1 && n > 1) {  // (block-uniform)
            if (grp) {
#pragma unroll
                for (uint32_t k = 0; k < KB; k++) {
                    const uint32_t q = k * kRedThreads + tid;
                    if (q < nb) part[(grp - 1) * nb + q] = acc[k];
                }
            }
            __syncthreads();
            if (!grp) {
#pragma unroll
                for (uint32_t g = 1; g < NG; g++)
#pragma unroll
                    for (uint32_t k = 0; k < KB; k++) {
                        const uint32_t q = k * kRedThreads + tid;
                        if (q < nb) acc[k] ^= part[(g - 1) * nb + q];
                    }
            }
        }
        // group 0 holds the item's sum; the others take part in barriers only
        bool last = grp == 0;
        if (parts == 1) {
            if (a.sig && !a.canon && !grp) {
                Bucket2 *o = (Bucket2 *)a.sig + (uint64_t)set * nb;
#pragma unroll
                for (uint32_t k = 0; k < KB; k++) {
                    const uint32_t q = k * kRedThreads + tid;
                    if (q < nb) o[q] = acc[k];
                }
            }
        } else {
            uint64_t *o = a.sig + (uint64_t)set * nb * 2;
#pragma unroll
            for (uint32_t k = 0; k < KB; k++) {
                const uint32_t q = k * kRedThreads + tid;
                if (q < nb && !grp) {
                    if (acc[k].x) gxor(&o[2 * q], acc[k].x);
                    if (acc[k].y) gxor(&o[2 * q + 1], acc[k].y);
                }
            }
            // every wave's atomics have been performed (they and the reads
            // below bypass the caches that are not coherent) before the ticket
            __atomic_signal_fence(__ATOMIC_SEQ_CST);
            __builtin_amdgcn_s_waitcnt(0);
            __syncthreads();
            if (threadIdx.x == 0)
                s_last = __hip_atomic_fetch_add(&a.tick[set], 1u, __ATOMIC_RELAXED,
                                                __HIP_MEMORY_SCOPE_AGENT) == parts - 1;
            __syncthreads();
            last = last && s_last != 0;
            if (last) {
#pragma unroll
                for (uint32_t k = 0; k < KB; k++) {
                    const uint32_t q = k * kRedThreads + tid;
                    if (q < nb) {
                        acc[k].x = __hip_atomic_load(&o[2 * q], __ATOMIC_RELAXED,
                                                     __HIP_MEMORY_SCOPE_AGENT);
                        acc[k].y = __hip_atomic_load(&o[2 * q + 1], __ATOMIC_RELAXED,
                                                     __HIP_MEMORY_SCOPE_AGENT);
                    }
                }
            }
        }
        if (last && a.canon) {
            Bucket2 *o = (Bucket2 *)a.canon + (uint64_t)set * nb;
#pragma unroll
            for (uint32_t k = 0; k < KB; k++) {
                const uint32_t q = k * kRedThreads + tid;
                const uint32_t d = q / C, c = q - d * C;
                if (q < nb) o[c * D + d] = acc[k];
            }
        }
        uint32_t best = 0xffffffffu, mine = best;
        uint64_t pick = 0;
        if (last && a.res) {
            uint64_t any = 0;
#pragma unroll
            for (uint32_t k = 0; k < KB; k++) {
                const uint32_t q = k * kRedThreads + tid;
                const uint64_t x = acc[k].x, g = acc[k].y;
                any |= x | g;
                if (q >= nb || x == 0) continue;
                const uint32_t d = q / C, c = q - d * C;
                const uint64_t h = mix64(x ^ a.seeds[c]);
                if (h != g || depth_of(h, D) != d) continue;
                const uint64_t uu = x / a.V, vv = x - uu * a.V;
                if (!(uu < vv)) continue;
                const uint32_t key = c * D + (D - 1 - d);
                if (key < best) {
                    best = key;
                    pick = x;
                }
            }
            mine = best;
            for (uint32_t o = 32; o > 0; o >>= 1) {
                const uint32_t ob = __shfl_xor(best, o);
                best = ob < best ? ob : best;
            }
            const bool wany = __ballot(any != 0) != 0;
            if (__lane_id() == 0) {
                s_best[tid / 64] = best;
                s_any[tid / 64] = wany ? 1u : 0u;
            }
        }
        __syncthreads();
        if (last && a.res) {
            uint32_t some = 0;
            for (uint32_t w = 0; w < kRedThreads / 64; w++) {
                best = s_best[w] < best ? s_best[w] : best;
                some |= s_any[w];
            }
            int32_t *r = a.res + 3 * (uint64_t)set;
            if (best != 0xffffffffu) {
                if (mine == best) {
                    r[0] = 0;
                    r[1] = (int32_t)(uint32_t)(pick / a.V);
                    r[2] = (int32_t)(uint32_t)(pick % a.V);
                }
            } else if (tid == 0) {
                r[0] = some ? 2 : 1;
                r[1] = 0;
                r[2] = 0;
            }
        }
        __syncthreads();  // the shared words are used again
    }
    if (a.seq_out && gridDim.x == 1) {
        // one block: its results are in host memory before the number is
        __atomic_signal_fence(__ATOMIC_SEQ_CST);
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        if (threadIdx.x == 0)
            __hip_atomic_store(a.seq_out, a.seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

// Publishes a sequence number once the kernels before it on the stream have
// finished (and their stores to host memory with them).
__global__ void k_publish(uint32_t *seq_out, uint32_t seq)
{
    __hip_atomic_store(seq_out, seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Zero the aggregates (W words each) and tickets of the sets listed.
__global__ __launch_bounds__(256) void k_zero_sets(const uint32_t *__restrict__ list, uint32_t W,
                                                   uint64_t *__restrict__ sig,
                                                   uint32_t *__restrict__ tick)
{
    const uint32_t set = list[blockIdx.x];
    uint64_t *o = sig + (uint64_t)set * W;
    for (uint32_t q = threadIdx.x; q < W; q += blockDim.x) o[q] = 0;
    if (threadIdx.x == 0) tick[set] = 0;
}

hipError_t launch_reduce_sample(hipStream_t s, const ReduceArgs &a, const uint32_t *zero_list,
                                uint32_t nzero)
{
    if (a.nitems == 0) return hipSuccess;
    const uint32_t nb = a.C * a.D;
    if (nzero) {
        if (!a.sig || !a.tick) return hipErrorInvalidValue;
        k_zero_sets<<<nzero, 256, 0, s>>>(zero_list, 2 * nb, a.sig, a.tick);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    const uint32_t grid = min(a.nitems, 8192u);
    // Two or four groups share an item; one group each where there are items
    // enough to fill the chip and few members to share (or, without items,
    // one): 65,536 members in 18,000 sets take 150 us instead of 212.
#define CUPK_RED(KB, NG)                                                                     \
    k_reduce_sample<KB, NG><<<grid, NG * kRedThreads, (size_t)(NG - 1) * nb * 16, s>>>(a)
    if (!a.items || (a.nitems >= 4 * kCus && a.members <= 16 * (uint64_t)a.nitems)) {
        if (nb <= 2 * kRedThreads) CUPK_RED(2, 1);
        else if (nb <= 4 * kRedThreads) CUPK_RED(4, 1);
        else if (nb <= 16 * kRedThreads) CUPK_RED(16, 1);
        else return hipErrorInvalidValue;
    }
    else if (nb <= kRedThreads) CUPK_RED(1, 4);
    else if (nb <= 2 * kRedThreads) CUPK_RED(2, 4);
    else if (nb <= 3 * kRedThreads) CUPK_RED(3, 2);
    else if (nb <= 4 * kRedThreads) CUPK_RED(4, 2);
    else if (nb <= 8 * kRedThreads) CUPK_RED(8, 2);
    else if (nb <= 16 * kRedThreads) CUPK_RED(16, 1);
    else return hipErrorInvalidValue;
#undef CUPK_RED
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || !a.seq_out || grid == 1) return e;
    k_publish<<<1, 1, 0, s>>>(a.seq_out, a.seq);
    return hipGetLastError();
}

// Reduction over CSR sets for the allocation-free entry point: a block takes
// members [16q, 16q + 16) of the concatenated member list, finds the set of
// the first one by binary search over the offsets (sets may be empty), and
// walks forward, folding its accumulator into a set's aggregate whenever it
// leaves that set.
constexpr uint32_t kCsrChunk = 16;

template <uint32_t KMAX>
__global__ __launch_bounds__(kRedThreads) void k_reduce_csr(const uint64_t *__restrict__ src,
                                                            uint32_t W,
                                                            const uint32_t *__restrict__ mem,
                                                            const uint64_t *__restrict__ offs,
                                                            uint32_t k, uint32_t nv,
                                                            uint64_t *__restrict__ out)
{
    const uint32_t nchunks = (nv + kCsrChunk - 1) / kCsrChunk;
    for (uint32_t q = blockIdx.x; q < nchunks; q += gridDim.x) {
        const uint32_t b = q * kCsrChunk, e = min(nv, b + kCsrChunk);
        // the last set j with offs[j] <= b; offs[0] = 0 <= b < nv = offs[k]
        uint32_t lo = 0, hi = k;
        while (hi - lo > 1) {
            const uint32_t mid = (lo + hi) / 2;
            if (offs[mid] <= b) lo = mid;
            else hi = mid;
        }
        uint32_t j = lo;
        uint64_t end = offs[j + 1];
        uint64_t acc[KMAX];
#pragma unroll
        for (uint32_t t = 0; t < KMAX; t++) acc[t] = 0;
        for (uint32_t m = b; m < e; m++) {
            if (m >= end) {
                uint64_t *o = out + (uint64_t)j * W;
#pragma unroll
                for (uint32_t t = 0; t < KMAX; t++) {
                    const uint32_t w = t * kRedThreads + threadIdx.x;
                    if (w < W && acc[t]) gxor(&o[w], acc[t]);
                    acc[t] = 0;
                }
                do {
                    j++;
                    end = offs[j + 1];
                } while (m >= end);
            }
            const uint64_t *s0 = src + (uint64_t)mem[m] * W;
#pragma unroll
            for (uint32_t t = 0; t < KMAX; t++) {
                const uint32_t w = t * kRedThreads + threadIdx.x;
                if (w < W) acc[t] ^= s0[w];
            }
        }
        uint64_t *o = out + (uint64_t)j * W;
#pragma unroll
        for (uint32_t t = 0; t < KMAX; t++) {
            const uint32_t w = t * kRedThreads + threadIdx.x;
            if (w < W && acc[t]) gxor(&o[w], acc[t]);
        }
    }
}

hipError_t launch_reduce_csr(hipStream_t s, const uint64_t *src, uint32_t W,
                             const uint32_t *mem, const uint64_t *offs, uint32_t k,
                             uint32_t nv, uint64_t *out)
{
    if (k == 0 || nv == 0) return hipSuccess;
    const uint32_t grid = min((nv + kCsrChunk - 1) / kCsrChunk, 8192u);
    if (W <= 4 * kRedThreads)
        k_reduce_csr<4><<<grid, kRedThreads, 0, s>>>(src, W, mem, offs, k, nv, out);
    else if (W <= 8 * kRedThreads)
        k_reduce_csr<8><<<grid, kRedThreads, 0, s>>>(src, W, mem, offs, k, nv, out);
    else if (W <= 16 * kRedThreads)
        k_reduce_csr<16><<<grid, kRedThreads, 0, s>>>(src, W, mem, offs, k, nv, out);
    else if (W <= 32 * kRedThreads)
        k_reduce_csr<32><<<grid, kRedThreads, 0, s>>>(src, W, mem, offs, k, nv, out);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

// Scratch of the allocation-free entry point: one array per GPU, held until
// the process ends.  In host code its name is a host-side stand-in, not a
// device address: host code uses only the address hipGetSymbolAddress
// returns for the current device, kept per device below.
static __device__ __align__(256) uint64_t scratch[kNoAllocScratchWords];

constexpr int kMaxDevices = 64;
static std::mutex g_scratch_mu;
static uint64_t *g_scratch_addr[kMaxDevices];

hipError_t noalloc_scratch_address(int device, uint64_t **out)
{
    if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_addr[device]) {
        uint64_t *p = nullptr;
        const hipError_t e = hipGetSymbolAddress((void **)&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        g_scratch_addr[device] = p;
    }
    *out = g_scratch_addr[device];
    return hipSuccess;
}

// ---------------------------------------------------------------------------
// Queries of sketches in canonical order (bucket (c, d) at c*D + d), one block
// each, in device or pinned host memory: as the query of k_reduce_sample.
// ---------------------------------------------------------------------------
constexpr uint32_t kSmpThreads = 256;

__global__ __launch_bounds__(kSmpThreads) void k_sample(const uint64_t *__restrict__ sig,
                                                        uint32_t V, uint32_t C, uint32_t D,
                                                        const uint64_t *__restrict__ seeds,
                                                        int32_t *__restrict__ res,
                                                        uint32_t *__restrict__ seq_out,
                                                        uint32_t seq)
{
    __shared__ uint32_t s_best[kSmpThreads / 64];
    __shared__ uint32_t s_any[kSmpThreads / 64];
    const uint32_t nb = C * D;
    const Bucket2 *S = (const Bucket2 *)sig + (uint64_t)blockIdx.x * nb;
    uint32_t best = 0xffffffffu;
    uint64_t any = 0, pick = 0;
    for (uint32_t q = threadIdx.x; q < nb; q += kSmpThreads) {
        const Bucket2 bk = S[q];
        const uint32_t c = q / D, d = q - c * D;
        any |= bk.x | bk.y;
        if (bk.x == 0) continue;
        const uint64_t h = mix64(bk.x ^ seeds[c]);
        if (h != bk.y || depth_of(h, D) != d) continue;
        const uint64_t uu = bk.x / V, vv = bk.x - uu * V;
        if (!(uu < vv)) continue;
        const uint32_t key = c * D + (D - 1 - d);
        if (key < best) {
            best = key;
            pick = bk.x;
        }
    }
    const uint32_t mine = best;
    for (uint32_t o = 32; o > 0; o >>= 1) {
        const uint32_t ob = __shfl_xor(best, o);
        best = ob < best ? ob : best;
    }
    const bool wany = __ballot(any != 0) != 0;
    if (__lane_id() == 0) {
        s_best[threadIdx.x / 64] = best;
        s_any[threadIdx.x / 64] = wany ? 1u : 0u;
    }
    __syncthreads();
    uint32_t some = 0;
    for (uint32_t w = 0; w < kSmpThreads / 64; w++) {
        best = s_best[w] < best ? s_best[w] : best;
        some |= s_any[w];
    }
    int32_t *r = res + 3 * (uint64_t)blockIdx.x;
    if (best != 0xffffffffu) {
        if (mine == best) {
            r[0] = 0;
            r[1] = (int32_t)(uint32_t)(pick / V);
            r[2] = (int32_t)(uint32_t)(pick % V);
        }
    } else if (threadIdx.x == 0) {
        r[0] = some ? 2 : 1;
        r[1] = 0;
        r[2] = 0;
    }
    if (seq_out && gridDim.x == 1) {
        __atomic_signal_fence(__ATOMIC_SEQ_CST);
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        if (threadIdx.x == 0)
            __hip_atomic_store(seq_out, seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

hipError_t launch_sample(hipStream_t s, const uint64_t *sig, uint32_t k, uint32_t V, uint32_t C,
                         uint32_t D, const uint64_t *seeds, int32_t *res, uint32_t *seq_out,
                         uint32_t seq)
{
    if (k == 0) return hipSuccess;
    k_sample<<<k, kSmpThreads, 0, s>>>(sig, V, C, D, seeds, res, seq_out, seq);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || !seq_out || k == 1) return e;
    k_publish<<<1, 1, 0, s>>>(seq_out, seq);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// One-column aggregates for the multi-level hierarchy, each queried in the
// same launch: as k_reduce_sample, but a wave takes a work item and lane d
// holds depth d's bucket of the set's column, so that a set of one item never
// leaves registers.  The deepest good bucket wins (depths are scanned from D-1
// down).  Bound by latency and by the lines of the members' buckets, one per
// depth; several members' loads are in flight.
// ---------------------------------------------------------------------------
constexpr uint32_t kColThreads = 256;

__global__ __launch_bounds__(kColThreads) void k_reduce_sample_col(ReduceArgs a)
{
    const uint32_t C = a.C, D = a.D;
    const uint32_t lane = __lane_id();
    const uint32_t wave = blockIdx.x * (kColThreads / 64) + threadIdx.x / 64;
    const uint32_t nwaves = gridDim.x * (kColThreads / 64);
    for (uint32_t it = wave; it < a.nitems; it += nwaves) {
        const uint32_t w = lane < 4 ? a.items[4 * it + lane] : 0u;
        const uint32_t set = __builtin_amdgcn_readlane(w, 0);
        const uint32_t b = __builtin_amdgcn_readlane(w, 1), e = __builtin_amdgcn_readlane(w, 2);
        const uint32_t pc = __builtin_amdgcn_readlane(w, 3);
        const uint32_t parts = pc & 0xffffffu, c = pc >> 24;
        const uint32_t mem = lane < e - b ? a.idx[b + lane] : 0u;
        const Bucket2 *sk = (const Bucket2 *)a.src0 + (uint64_t)(lane < D ? lane : 0) * C + c;
        Bucket2 acc{0, 0};
        constexpr uint32_t kAhead = 8;
        for (uint32_t j = 0; j < e - b; j += kAhead) {
            Bucket2 t[kAhead];
#pragma unroll
            for (uint32_t g = 0; g < kAhead; g++) {
                const bool in = j + g < e - b;
                const uint64_t m = (uint32_t)__builtin_amdgcn_readlane(mem, in ? j + g : 0);
                t[g] = in && lane < D ? sk[m * D * C] : Bucket2{0, 0};
            }
#pragma unroll
            for (uint32_t g = 0; g < kAhead; g++) acc ^= t[g];
        }
        if (parts > 1) {  // (wave-uniform)
            uint64_t *o = a.sig + ((uint64_t)set * D + lane) * 2;
            if (lane < D) {
                if (acc.x) gxor(o, acc.x);
                if (acc.y) gxor(o + 1, acc.y);
            }
            // the wave's atomics have been performed before its ticket
            __atomic_signal_fence(__ATOMIC_SEQ_CST);
            __builtin_amdgcn_s_waitcnt(0);
            __atomic_signal_fence(__ATOMIC_SEQ_CST);
            uint32_t t = 0;
            if (lane == 0)
                t = __hip_atomic_fetch_add(&a.tick[set], 1u, __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_AGENT);
            if (__builtin_amdgcn_readlane(t, 0) != parts - 1) continue;
            if (lane < D) {
                acc.x = __hip_atomic_load(o, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                acc.y = __hip_atomic_load(o + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
        bool good = false;
        if (lane < D && acc.x != 0) {
            const uint64_t h = mix64(acc.x ^ a.seeds[c]);
            const uint64_t uu = acc.x / a.V, vv = acc.x - uu * a.V;
            good = h == acc.y && depth_of(h, D) == lane && uu < vv;
        }
        const uint64_t mg = __ballot(good);
        const uint64_t mz = __ballot(lane < D && (acc.x | acc.y) != 0);
        const uint32_t top = mg ? 63u - (uint32_t)__builtin_clzll(mg) : 0u;
        if (lane == top) {
            int32_t *r = a.res + 3 * (uint64_t)set;
            r[0] = mg ? 0 : mz ? 2 : 1;
            r[1] = mg ? (int32_t)(uint32_t)(acc.x / a.V) : 0;
            r[2] = mg ? (int32_t)(uint32_t)(acc.x % a.V) : 0;
        }
    }
}

hipError_t launch_reduce_sample_col(hipStream_t s, const ReduceArgs &a, const uint32_t *zero_list,
                                    uint32_t nzero)
{
    if (a.nitems == 0) return hipSuccess;
    if (a.D > 64 || !a.items || !a.res) return hipErrorInvalidValue;
    if (nzero) {
        if (!a.sig || !a.tick) return hipErrorInvalidValue;
        k_zero_sets<<<nzero, 64, 0, s>>>(zero_list, 2 * a.D, a.sig, a.tick);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    const uint32_t waves = kColThreads / 64;
    const uint32_t grid = min((a.nitems + waves - 1) / waves, 8192u);
    k_reduce_sample_col<<<grid, kColThreads, 0, s>>>(a);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess || !a.seq_out) return e;
    k_publish<<<1, 1, 0, s>>>(a.seq_out, a.seq);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Digest: order-independent sum over all buckets of
// mix(alpha ^ rotl(gamma, 32) ^ mix(canonical_position ^ seed)).
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_digest(DevSketch sk, uint64_t S, uint64_t *out)
{
    const uint32_t C = sk.C, D = sk.D;
    const uint32_t per_v = C * D;
    uint64_t acc = 0;
    for (uint32_t w = blockIdx.x; w < sk.V; w += gridDim.x) {
        const uint64_t *b = sk.b + (uint64_t)w * per_v * 2;
        for (uint32_t r = threadIdx.x; r < per_v; r += blockDim.x) {
            const uint32_t d = r / C, c = r - d * C;
            const uint64_t pos = ((uint64_t)w * C + c) * D + d;
            const uint64_t a = b[2 * r], g = b[2 * r + 1];
            const uint64_t rg = (g << 32) | (g >> 32);
            acc += mix64(a ^ rg ^ mix64(pos ^ S));
        }
    }
    for (uint32_t o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o);
    if (__lane_id() == 0) atomicAdd((unsigned long long *)out, (unsigned long long)acc);
}

hipError_t launch_digest(hipStream_t s, DevSketch sk, uint64_t master_seed, uint64_t *out)
{
    const uint32_t grid = min(sk.V, 8192u);
    k_digest<<<grid, 256, 0, s>>>(sk, master_seed, out);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Internal layout -> canonical (c, d) order.
// ---------------------------------------------------------------------------
__global__ void k_to_canonical(const uint64_t *__restrict__ src, uint32_t C, uint32_t D,
                               uint64_t nv, uint64_t *__restrict__ dst)
{
    const uint32_t per_v = C * D;
    const uint64_t total = nv * per_v;
    for (uint64_t q = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; q < total;
         q += (uint64_t)gridDim.x * blockDim.x) {
        const uint64_t i = q / per_v;
        const uint32_t r = (uint32_t)(q - i * per_v);
        const uint32_t c = r / D, d = r - c * D;
        const uint64_t s = (i * per_v + (uint64_t)d * C + c) * 2;
        dst[2 * q] = src[s];
        dst[2 * q + 1] = src[s + 1];
    }
}

hipError_t launch_to_canonical(hipStream_t s, const uint64_t *src, uint32_t C, uint32_t D,
                               uint64_t nv, uint64_t *dst)
{
    const uint64_t total = nv * C * D;
    if (total == 0) return hipSuccess;
    uint64_t blocks = (total + 255) / 256;
    if (blocks > 8192) blocks = 8192;
    k_to_canonical<<<(uint32_t)blocks, 256, 0, s>>>(src, C, D, nv, dst);
    return hipGetLastError();
}

}  // namespace cupk
