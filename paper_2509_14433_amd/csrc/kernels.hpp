// Launch wrappers of the gfx950 kernels.  Host code calls only these.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace cupk {

// Device view of the resident sketch.
// Internal layout: bucket (w, d, c) of vertex w at word ((w*D + d)*C + c)*2,
// alpha at +0 and gamma at +1 ("depth-major inside a vertex": the shallow
// rows that take most updates are contiguous at the front of a vertex).
struct DevSketch {
    uint64_t *b;           // 2*V*C*D words
    const uint64_t *seeds; // C column seeds
    uint32_t V, C, D;
};

// The batch a step works on, read by the kernels from device memory so that
// one captured graph serves batches of any size up to its capacity.
struct BatchDesc {
    const uint64_t *upd;  // packed updates
    uint32_t n;           // number of updates
    uint32_t pad;
};

// Header words.  The classify kernel ORs ERR (a rejected batch); the
// one-block kernel after it moves ERR to REJ, where the rest of the pass
// reads it, and clears it for the next batch (the scatter leaves the header
// alone: a ticket per block on one word took 12 ns each, 12 us behind a
// launch of 1,024 blocks that finish together).  NFLAG and NFLAG_DEL exist
// in the host copy only.  SEQ counts published headers: the one-block kernel
// writes the verdict and the flag counts to the host, then the incremented
// SEQ (release store), which the host waits for.
enum {
    HDR_ERR = 0,
    HDR_NFLAG = 1,
    HDR_NFLAG_DEL = 2,
    HDR_REJ = 3,
    HDR_SEQ = 4,
    HDR_INLINE = 5,  // host copy only: the flagged updates came with the header
    HDR_WORDS = 8
};

// Flagged updates of a batch with at most kInlineFlags of them (and at most
// kInlineMaxBlocks classify blocks) are compacted in stream order straight
// into host memory by the one-block kernel after classification, before it
// publishes the header (HDR_INLINE set): no compaction kernels, no copy.
constexpr uint32_t kInlineFlags = 16384;
constexpr uint32_t kInlineMaxBlocks = 8192;
struct FlagInline {
    const uint64_t *fupd;  // per-block regions (the classify kernel's output)
    const uint32_t *fcnt;  // flags per classify block
    uint32_t *fdel;        // flagged deletes per classify block
    uint32_t nb;           // classify blocks
    uint64_t *hflags;      // coherent pinned host memory; null: never inline
    // 1: the scan after the classify kernel leaves the flags and the header
    // alone (launch_reflag checks the flags against a newer forest and
    // publishes them later); 0: it publishes them
    uint32_t tiles_only;
    uint32_t checked;  // 1: ERR has been moved to REJ already (launch_reflag)
};

// Where the one-block tile scan writes: bin offsets and fill cursors
// (ntiles + 1 words each), work items (tile, chunk) and their number.
// Tile counts are kept in `groups` copies of ntiles words (1, or
// kCntGroups when classify blocks also store where their records start:
// block b adds to copy b % kCntGroups, so that fewer blocks meet on one
// counter).  goff (groups * ntiles words, may be null) receives where each
// copy's records start in every tile's bin.
constexpr uint32_t kCntGroups = 4;
// sums (2 * tile_scan_chunks(ntiles) words, may be null): scratch of the
// multi-block scan, used (and required) when ntiles > kScanOneBlockTiles:
// the one-block kernel then only publishes the header and two multi-block
// kernels scan the counts (one count copy only).
constexpr uint32_t kScanOneBlockTiles = 4096;
struct ScanArgs {
    uint32_t *off, *cur, *items, *nitems;
    uint32_t chunk, items_cap;
    uint32_t groups;
    uint32_t *goff;
    uint32_t *sums;
};
uint32_t tile_scan_chunks(uint32_t ntiles);

// Staged-scatter lane layouts a caller may name.  Up to kStagMaxC columns
// both run k_tile_scatter_stag (one lane per record, staggered columns),
// which is the faster one at every size measured; beyond, k_tile_scatter
// (one lane per (record, column) pair, any number of columns).  They only
// differ in the geometry they admit (tile_geometry_fits).
constexpr uint32_t kLayoutRecord = 1;
constexpr uint32_t kLayoutPair = 2;
constexpr uint32_t kStagMaxC = 24;

struct StagedParams {
    uint32_t tile_shift;   // vertices per tile = 1 << tile_shift
    uint32_t rows;         // depth rows held in LDS (d < rows)
    uint32_t layout;       // kLayoutRecord or kLayoutPair
    uint32_t ntiles;
    uint32_t chunk;        // max records per work item
    uint32_t items_cap;    // capacity of the work-item array
    uint32_t grid;         // blocks of the persistent tile kernel (0 = default)
    uint64_t records;      // endpoint records of the batch (two per update), at most
};

// Per-batch: validation, structural classification and compaction of the
// flagged updates.  hdr's ERR word must be zero (as the one-block kernel of
// the previous batch leaves it).  A one-block kernel after it writes the
// verdict and the flag counts to `hout` (coherent pinned host memory,
// HDR_WORDS words: no copy needed), then the next sequence number at
// hout[HDR_SEQ].  When `tile_cnt` is non-null the classify kernel
// also counts how many endpoint records each vertex tile gets, and the
// one-block kernel scans the counts into `sa` (sa.off set).  Flagged updates of
// classify block b (positions [b*4096, (b+1)*4096)) land in stream order at
// offsets b*4096.. of fupd (capacity: the batch rounded up to a multiple of
// 4096); fcnt[b] receives their number.  fpos (may be null) receives each
// flagged update's position in the batch, alongside.  grid_n sizes the
// grids (the batch size, or the capacity of a captured graph); the kernels
// read the batch from device memory at `desc` (captured graphs) or, when
// desc is null, from `dv`.  When `tile_rel` is non-null (tile counts on, at
// most kRelMaxTiles tiles; classify_blocks(grid_n) * ntiles words; tile_cnt
// of kCntGroups * ntiles words and sa.groups == kCntGroups), block b also
// stores at tile_rel[b*ntiles + t] where its records start among the
// records of count copy b % kCntGroups in tile t (written only for tiles it
// has records in), so that the fill reserves nothing.
// blk (may be null): the block labels (launch_load_forest) of the forest in
// lp; inserts between two uniform blocks then skip the forest words.
constexpr uint32_t kRelMaxTiles = 2048;
hipError_t launch_classify(hipStream_t s, const BatchDesc *desc, BatchDesc dv, uint32_t grid_n,
                           uint32_t V, const uint64_t *lp, const uint32_t *blk, uint32_t *hdr,
                           uint64_t *fupd, uint32_t *fpos, uint32_t *fcnt, uint32_t *tile_cnt,
                           uint32_t tile_shift, uint32_t ntiles, const ScanArgs &sa,
                           uint32_t *hout, const FlagInline &fi, uint32_t *tile_rel);
uint32_t classify_blocks(uint32_t n);
// The device forest as the classify kernels read it: lp[w] = label | parent
// << 32 (one 8-byte load per endpoint) and the block labels blk[b] (b <
// ceil(V / 64)): the label that all vertex ids [64 b, 64 b + 64) below V
// share, or kBlkMixed; the classify kernel (blk non-null) decides an insert
// whose endpoints both lie in uniform blocks by them.  Refreshes np pages of
// 2^pshift ids (pshift in [6, 16]): those listed in `pages`, or, when it is
// null, pages 0 .. np-1.  lbl, par (indexed by vertex) and pages: device or
// pinned host memory.
constexpr uint32_t kBlkShift = 6;
constexpr uint32_t kBlkMixed = 0xffffffffu;
hipError_t launch_load_forest(hipStream_t s, const uint32_t *lbl, const uint32_t *par, uint32_t V,
                              const uint32_t *pages, uint32_t np, uint32_t pshift, uint64_t *lp,
                              uint32_t *blk);
// Second half of a classification launched with fi.tiles_only = 1: with
// `check`, keep, in each classify block's region of fi.fupd (in place,
// stream order kept), only the updates the classify kernel's rule flags
// against the forest in `lp`, and rewrite fi.fcnt and fi.fdel; pack the
// regions into one ordered list at oupd (foff: fi.nb words of scratch), as
// launch_flag_compact does; then publish the flag counts, the short flag
// lists and the header as launch_classify does otherwise.  Exact when `lp`
// is a coarsening of the forest the regions were flagged against that keeps
// all its edges (it then flags a subset of what that forest flagged).  A
// rejected batch (header error) keeps its regions.
hipError_t launch_reflag(hipStream_t s, uint32_t V, const uint64_t *lp, uint32_t *hdr,
                         uint64_t *fupd, uint32_t *hout, const FlagInline &fi, uint32_t *foff,
                         uint64_t *oupd, bool check);

// Pack the per-block flag regions into one list in stream order (foff:
// classify_blocks(n) words of scratch); positions too when fpos and opos
// are not null.
hipError_t launch_flag_compact(hipStream_t s, uint32_t n, const uint64_t *fupd,
                               const uint32_t *fpos, const uint32_t *fcnt, uint32_t *foff,
                               uint64_t *oupd, uint32_t *opos);

// Small batches: header, flagged updates (stream order) and their positions
// of one batch of at most kOneBlockMax updates, written by one kernel straight
// into host memory.  Batches of at most kSmallMax updates always go this way;
// up to kOneBlockMax those that the direct scatter suits (direct_pays in
// api.cpp).
constexpr uint32_t kSmallMax = 4096;
constexpr uint32_t kOneBlockMax = 16384;
struct SmallResult {
    uint32_t hdr[HDR_WORDS];
    uint64_t fupd[kOneBlockMax];
    uint32_t fpos[kOneBlockMax];
};
// First bring the forest words lp of nd (at most 1,024) vertices up to date:
// (vertex, label, parent) each at `delta` (pinned host memory).  Then
// classify (one block) a batch of 1..kOneBlockMax packed updates given in the
// arguments into `out` (coherent pinned host memory; with_pos: also
// positions), set *derr (device) to the error flag, and publish the next
// value of the counter *seqp at out->hdr[HDR_SEQ] (release store) once the
// rest of `out` is written.
hipError_t launch_small_classify(hipStream_t s, const uint64_t *upd, uint32_t n, uint32_t V,
                                 uint64_t *lp, const uint32_t *delta, uint32_t nd,
                                 SmallResult *out, uint32_t *derr, uint32_t *seqp, bool with_pos);
// Direct scatters, with device atomics, of a classified batch; they do nothing
// if an update was invalid (*derr set).  Small: at most kSmallMax updates.
// Mid: any number; a vertex that takes a large share of the batch is gathered
// per block; touched as for launch_tile.
hipError_t launch_small_scatter(hipStream_t s, const uint64_t *upd, uint32_t n, DevSketch sk,
                                const uint32_t *derr);
hipError_t launch_mid_scatter(hipStream_t s, const uint64_t *upd, uint32_t n, DevSketch sk,
                              const uint32_t *derr, unsigned long long *touched);

// Plain scatter: device-scope atomic XOR of (x, h) into both endpoints.
hipError_t launch_scatter_atomic(hipStream_t s, const BatchDesc *desc, BatchDesc dv,
                                 uint32_t grid_n, DevSketch sk, const uint32_t *hdr);

// Staged scatter: launch_bin = fill of the per-tile bins (at the offsets
// the classify kernel's tile scan wrote: the count copy's start in
// tile_goff plus the classify block's tile_rel entry when tile_rel is
// non-null, else reserved from tile_cur);
// launch_tile = LDS-staged XOR per work item; touched (may be null) is
// incremented by the number of buckets the launch changes in HBM.
hipError_t launch_bin(hipStream_t s, const BatchDesc *desc, BatchDesc dv, uint32_t grid_n,
                      DevSketch sk, const uint32_t *hdr, const StagedParams &p,
                      uint32_t *tile_cur, uint32_t *bins, const uint32_t *tile_goff,
                      const uint32_t *tile_rel);
hipError_t launch_tile(hipStream_t s, DevSketch sk, const uint32_t *hdr, const StagedParams &p,
                       const uint32_t *tile_off, const uint32_t *bins, const uint32_t *items,
                       const uint32_t *nitems, unsigned long long *touched);
// Whether the records of bins of 2^shift vertices take 64 bits: two words of
// bins per record instead of one.
bool rec_wide(uint32_t V, uint32_t shift);
// Second level of the two-level binning (used when there are more tiles
// than kFillStageTiles): bins1 holds the batch's records binned by coarse
// bin (2^fshift tiles each; the classify kernel counted them and the fill
// wrote them) at the coarse scan's offsets coff, and citems its work items
// (coarse bin, part of at most fine_chunk(rec_wide(V, tile_shift + fshift))
// records), *ncitems of them.  Counts the records per tile into tile_cnt,
// scans with the multi-block tile scan into sa (one count copy, sa.sums set)
// and writes them into their tile bins in `bins`.
constexpr uint32_t kFillStageTiles = 2048;
// Most bins the classify kernel counts in LDS (beyond, with device atomics),
// and most tiles per coarse bin (launch_fine).
constexpr uint32_t kLdsHistMax = 8192;
constexpr uint32_t kFineLdsTiles = 8192;
uint32_t fine_chunk(bool wide);
hipError_t launch_fine(hipStream_t s, uint32_t grid_n, uint32_t V, const uint32_t *hdr,
                       const uint32_t *bins1, const uint32_t *coff, const uint32_t *citems,
                       const uint32_t *ncitems, uint32_t tile_shift, uint32_t fshift,
                       uint32_t ntiles, uint32_t *tile_cnt, const ScanArgs &sa, uint32_t *bins);
// Whether a staged-scatter geometry fits one block's LDS: the delta of
// `rows` depth rows x C columns x tv vertices (alpha and gamma), plus, in
// the pair layout, room to stage one block's worth of decoded records.
bool tile_geometry_fits(uint32_t rows, uint32_t C, uint32_t tv, uint32_t layout);

// Fill n words with zero.
hipError_t launch_zero(hipStream_t s, uint64_t *p, size_t n);
hipError_t launch_zero32(hipStream_t s, uint32_t *p, size_t n);

// Segmented XOR reduction of vertex sketches or fragment sketches into one
// aggregate per set, and the query of each (see k_reduce_sample).
constexpr uint32_t kRedChunk = 64;  // most members per work item
struct ReduceArgs {
    const uint64_t *src0, *src1;  // slabs of vertices, of the previous round's fragments
    // (set, begin, end, items of the set) per work item; bit 31 of set: the
    // members are fragments.  null: item i is set i, vertex i alone.
    const uint32_t *items;
    const uint32_t *idx;          // members
    uint32_t nitems;
    uint32_t members;             // in all items (chooses the block shape)
    uint32_t V, C, D;
    const uint64_t *seeds;
    uint64_t *sig;    // aggregates, internal layout (may be null when every set has one item)
    uint32_t *tick;   // one word per set, used by sets of several items
    uint64_t *canon;  // aggregates in canonical order, or null
    int32_t *res;     // (status, u, v) per set, or null; device or pinned host memory
    uint32_t *seq_out;  // null, or where to publish seq once all is written
    uint32_t seq;
    // an only item (items set, nitems 1) and its members, read instead of
    // items and idx (launch_reduce_sample)
    uint32_t one[4], mem[kRedChunk];
};
// zero_list: the sets of several items (nzero of them), whose aggregates and
// tickets are zeroed first.  Every set must have an item (an empty one for an
// empty set).
hipError_t launch_reduce_sample(hipStream_t s, const ReduceArgs &a, const uint32_t *zero_list,
                                uint32_t nzero);

// Allocation-free aggregates (cupk_component_sketch_batch_noalloc): the
// members, set offsets and aggregates of one call live in a file-scope
// device array of kNoAllocScratchWords words, one per GPU for the life of
// the process.  Layout in words: aggregates [0, kNoAllocAggWords), then the
// kNoAllocMaxSets + 1 set offsets (uint64), then the members (uint32, two
// per word).
constexpr uint32_t kNoAllocMaxMembers = 1u << 20;
constexpr uint32_t kNoAllocMaxSets = 4096;
constexpr uint32_t kNoAllocAggWords = 1u << 21;  // 16 MiB of aggregates
constexpr size_t kNoAllocOffsWord = kNoAllocAggWords;
constexpr size_t kNoAllocMemWord = kNoAllocOffsWord + kNoAllocMaxSets + 1;
constexpr size_t kNoAllocScratchWords = kNoAllocMemWord + kNoAllocMaxMembers / 2;
// Device address of the scratch array on `device`, which must be current.
// Taken with hipGetSymbolAddress on the first call per device and kept.
hipError_t noalloc_scratch_address(int device, uint64_t **out);

// Segmented XOR reduction over CSR sets: out[j] = XOR of the slabs of
// mem[offs[j] .. offs[j+1]) for j < k (nv = offs[k] members).  Blocks take
// 16 consecutive members at a time and find their set by binary search, so
// no work-item list is needed.  out (k*W words) must be zeroed first.
hipError_t launch_reduce_csr(hipStream_t s, const uint64_t *src, uint32_t W,
                             const uint32_t *mem, const uint64_t *offs, uint32_t k,
                             uint32_t nv, uint64_t *out);

// Query each of k sketches in canonical order, in device or pinned host
// memory.  res: 3 words per set (status, u, v); seq_out as in ReduceArgs.
hipError_t launch_sample(hipStream_t s, const uint64_t *sig, uint32_t k, uint32_t V, uint32_t C,
                         uint32_t D, const uint64_t *seeds, int32_t *res, uint32_t *seq_out,
                         uint32_t seq);

// Digest of the whole sketch, added into *out (zero it first).
hipError_t launch_digest(hipStream_t s, DevSketch sk, uint64_t master_seed, uint64_t *out);

// Copy nv sketches from internal layout (first vertex w0) or from an
// internal-layout aggregate array (w0 ignored when `agg` is set) into
// canonical (c, d) order.
hipError_t launch_to_canonical(hipStream_t s, const uint64_t *src, uint32_t C, uint32_t D,
                               uint64_t nv, uint64_t *dst);

// Multi-level hierarchy: every set reduced over one column only and queried.
// Items: (set, begin, end, items of the set | column << 24), at most kRedChunk
// members each; sig: 2*D words per set ([depth][alpha, gamma]), used by sets
// of several items, listed in zero_list.  src1, canon and members are not
// used; seq_out is published by a kernel of its own.  D <= 64.
hipError_t launch_reduce_sample_col(hipStream_t s, const ReduceArgs &a, const uint32_t *zero_list,
                                    uint32_t nzero);

}  // namespace cupk
