// Dependency resolution of a global switch by sorting (edge key, tag) tuples
// by edge key -- an HBM-atomic-free form of Alg. 1's dependency table T.
//
// Every switch k that survives its local checks emits four tuples: an ERASE
// tuple for each source edge (Def. 3.1 / Alg. 1 "erase") and an INSERT tuple
// for each target edge ("insert"); a switch rejected locally (loop, a target
// equal to one of its own sources, P_L) and the idle position of odd m emit
// ERASE tuples marked STAYS (those edges survive the superstep).  Tuples are
// partitioned by a hash of the key with the same LDS-staged radix scatter as
// the permutation (its first pass computes them from the pair records, see
// emit_switch), so all tuples of one key meet in one workgroup, which
// sorts its partition in LDS and derives for every INSERT tuple (k, X):
//   eraser(X)  : the switch whose source X is (or STAYS / none)   -- lookup
//   pred(k, X) : the next smaller inserter of X                    -- the
//                chain behind lookup_min over non-illegal inserters.
// Only targets with an eraser or a predecessor have a record (rare); a bit in
// the switch's status byte says so, and the rounds read no other record.  (With
// a "free" record written by the emit for every target, the emit wrote and the
// first round read 16 bytes a switch: n = 2^22, d = 32, 45.2 -> 44.0 ms per
// call of ten supersteps without them.)
//
// Decision of switch k (same rule as Alg. 1): illegal if a target is erased
// by a later switch / stays / is erased by an illegal switch, or if an
// earlier inserter of a target is legal; delayed if it depends on an
// undecided switch; else legal.  The predecessor chain of (k, X) lists every
// earlier inserter of X from the nearest down, so walking it until a legal
// (-> illegal) or undecided (-> delayed) switch, or its end (-> free),
// evaluates "no earlier legal inserter of X".
#pragma once

#include "device_common.h"
#include "perm_kernels.h"
#include "switch_kernels.h"

namespace gesmc {

// per-target record: x = eraser (kNoEraser / kStays / switch), y = predecessor (k' << 1 | h') or kNoPred
constexpr uint32_t kNoPred = 0xFFFFFFFFu;
constexpr uint32_t kWalked = 0xFFFFFFFEu;  // every predecessor rejected (a walk that reached the chain's end)
__device__ __forceinline__ bool chain_end(uint32_t p) { return p >= kWalked; }  // kWalked or kNoPred

// The legal inserter of each key.  A key gains at most one legal inserter in
// a superstep: once inserted it stays (a position is a source once), and
// inserters before its eraser saw it present.  head[s] (s a target record
// with a predecessor) names the record of the key's first inserter, and
// win[head] receives the legal inserter if that is a later one (the first
// one's own status tells otherwise).  A switch whose nearest undecided
// predecessor still waits is then rejected as soon as any earlier inserter
// is legal, so the rounds follow the dependency depth instead of the length
// of a hub key's inserter chain: on Pld([1..16000], 2.05), n = 2^19, a
// superstep's rounds fell from about 300 to 8 and the call (10 supersteps)
// from 8.9 to 3.8 ms.
struct Winners {
    uint32_t *head, *win;  // per target record 2k+h; written by k_resolve where a predecessor exists
};
constexpr uint32_t kNoWinner = 0xFFFFFFFFu;
constexpr uint32_t kListEnd = 0xFFFFu;  // end of a cell list in k_resolve (slots are < 2^16)
constexpr uint32_t kEpochNone = 0xFFFFu;  // k_resolve: no list partition yet (epochs are 0 .. 0xFFFE)
static_assert(kLdsCap < kListEnd, "k_resolve slots fit 16 bits");

// ---------------------------------------------------------------------------
// Emit: one thread per switch (+ one for the idle record of odd m).  The
// local outcome of every switch (switch_local) goes to its status; a switch
// decided locally also gets its records (unchanged) and its count, an
// undecided one nothing else.  Workgroup 0
// clears the undecided-list counters of the rounds that follow.  This kernel
// serves the unfused schedule; by default the same work runs inside the
// first tuple count pass (k_emit_counts below), and the switches' tuples are
// never stored: the first partition pass computes them from the same pair
// records (emit_switch).
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kBlock) void k_emit(const uint32_t *__restrict__ s_idx,
                                                 const unsigned long long *__restrict__ s_key, uint32_t t, uint32_t k0,
                                                 uint32_t k1, SrcArgs sa, uint8_t *__restrict__ st,
                                                 uint32_t *__restrict__ out_idx,
                                                 unsigned long long *__restrict__ out_key, uint4 *__restrict__ bslot,
                                                 uint32_t *__restrict__ ucount) {
    __shared__ BlockCounts bc;
    const uint32_t tid = threadIdx.x;
    if (tid == 0) bc = BlockCounts{0, 0, 0, 0};
    if (blockIdx.x == 0 && tid < 4) ucount[tid] = 0;  // the undecided-list counters of the rounds, arrivals
    __syncthreads();
    const uint32_t m = sa.m, ell = m >> 1;
    const uint32_t stride = gridDim.x * kBlock;
    for (uint32_t k = blockIdx.x * kBlock + tid; k <= ell; k += stride) {
        if (k == ell) {
            if (m & 1u) {
                out_idx[m - 1] = s_idx[m - 1];
                out_key[m - 1] = s_key[m - 1];
            }
            continue;
        }
        const uint2 ij = reinterpret_cast<const uint2 *>(s_idx)[k];
        const ulonglong2 ee = reinterpret_cast<const ulonglong2 *>(s_key)[k];
        Targets T{0, 0, false};
        const uint8_t status = switch_local(k, ij, ee, t, k0, k1, sa, &T);
        st[k] = status;
        if (status != ST_UNDECIDED) {
            reinterpret_cast<uint2 *>(out_idx)[k] = ij;
            reinterpret_cast<ulonglong2 *>(out_key)[k] = ee;
            if (status == ST_PL) atomicAdd(&bc.pl, 1u);
            if (status == ST_LOOP) atomicAdd(&bc.loop, 1u);
            if (status == ST_EXISTS) atomicAdd(&bc.exists, 1u);
        }
    }
    store_counts(&bc, bslot + blockIdx.x);
}

// A superstep of a multi-edge class (Sec. 1): no target is rejected for
// being present, so each switch's outcome follows from its own pair records
// alone (P_L skip, else a loop where loops are not allowed, else legal) and
// the whole superstep is decided here, one thread per switch plus one for
// the idle record of odd m.  Writes every record of buffer 0, the status
// array and the superstep's counts.
__global__ __launch_bounds__(kBlock) void k_decide_local(const uint32_t *__restrict__ s_idx,
                                                         const unsigned long long *__restrict__ s_key, uint32_t m,
                                                         uint32_t t, uint32_t k0, uint32_t k1, uint32_t pl,
                                                         uint32_t cls, uint8_t *__restrict__ st,
                                                         uint32_t *__restrict__ out_idx,
                                                         unsigned long long *__restrict__ out_key,
                                                         StepCounters *ctr) {
    __shared__ BlockCounts bc;
    if (threadIdx.x == 0) bc = BlockCounts{0, 0, 0, 0};
    __syncthreads();
    const uint32_t ell = m >> 1;
    const uint32_t stride = gridDim.x * kBlock;
    for (uint32_t k = blockIdx.x * kBlock + threadIdx.x; k <= ell; k += stride) {
        if (k == ell) {
            if (m & 1u) {
                out_idx[m - 1] = s_idx[m - 1];
                out_key[m - 1] = s_key[m - 1];
            }
            continue;
        }
        const uint2 ij = reinterpret_cast<const uint2 *>(s_idx)[k];
        const ulonglong2 ee = reinterpret_cast<const ulonglong2 *>(s_key)[k];
        uint8_t status = ST_LEGAL;
        ulonglong2 out = ee;
        if (pl_skip(k, t, pl, k0, k1)) {
            status = ST_PL;
        } else {
            const Targets T = switch_targets_cls(ee.x, ee.y, ij.x < ij.y, cls);
            if (T.loop)
                status = ST_LOOP;
            else
                out = make_ulonglong2(T.A, T.B);
        }
        st[k] = status;
        reinterpret_cast<uint2 *>(out_idx)[k] = ij;
        reinterpret_cast<ulonglong2 *>(out_key)[k] = out;
        if (status == ST_LEGAL) atomicAdd(&bc.legal, 1u);
        if (status == ST_LOOP) atomicAdd(&bc.loop, 1u);
        if (status == ST_PL) atomicAdd(&bc.pl, 1u);
    }
    flush_counts(&bc, ctr);
}

// The next superstep's first radix level: the records' positions do not change
// in a superstep (the sorted records of position p keep their index), so the
// level-1 digit counts of superstep t + 1 over tiles of `tile` positions need
// only the indices.  They are taken where the indices are read anyway: in the
// emit (k_emit_counts) when the first round scatters the records itself
// (k_decide_scatter), else in the first round.  A batch (gr != nullptr) counts
// the global buckets of its next step's prefix of m positions (each
// position's graph from pg).
struct NextCounts {
    uint32_t *counts;  // [tile][digit], nullptr: none
    uint32_t t, k0, k1;
    int shift, dbits;
    uint32_t tile, m;
    const BatchGraph *gr;  // batch: graph records, the graph of each position,
    const uint32_t *pg;    // the next step and its bucket bits
    uint32_t step;
    int bbits;
};

__device__ __forceinline__ uint32_t next_digit(const NextCounts &nc, uint32_t i, uint32_t pos) {
    const uint32_t dmask = (1u << nc.dbits) - 1;
    if (!nc.gr) return (uint32_t)(perm_key(i, nc.t, nc.k0, nc.k1) >> nc.shift) & dmask;
    const BatchGraph &g = nc.gr[nc.pg[pos]];
    const uint64_t word = (uint64_t)batch_bucket(g, batch_perm_key(g, i, nc.step)) << (64 - nc.bbits);
    return (uint32_t)(word >> nc.shift) & dmask;
}

// k_emit fused into the first tuple partition pass's counts (kSrcEmit or
// kSrcEmitPacked, one segment [0, nslots) of kTile-slot tiles): the pair
// records of a switch are read once, for its status, its records and
// counts (as k_emit) and for its four tuples' digit counts (as
// k_tile_counts).  Tiles are taken grid-stride; each workgroup stores its
// outcome counts in bslot[blockIdx.x].  The per-tile digit counts equal
// k_tile_counts' (the same tiles, tuples and radix words).  With nc.counts
// also the next superstep's first-level counts; without out_idx no record is
// written (k_decide_scatter moves them all).
template <int kSrc, int kTile>
__global__ __launch_bounds__(kBlock) void k_emit_counts(const uint32_t *__restrict__ s_idx,
                                                        const unsigned long long *__restrict__ s_key, uint32_t t,
                                                        uint32_t k0, uint32_t k1, int shift, int dbits, uint32_t nslots,
                                                        uint32_t *__restrict__ counts, SrcArgs sa,
                                                        uint8_t *__restrict__ st, uint32_t *__restrict__ out_idx,
                                                        unsigned long long *__restrict__ out_key,
                                                        uint4 *__restrict__ bslot, uint32_t *__restrict__ ucount,
                                                        NextCounts nc) {
    static_assert(src_emits<kSrc>(), "tuples emitted from the pair records");
    extern __shared__ uint32_t hs[];
    __shared__ BlockCounts bc;
    __shared__ uint32_t hn[1u << kMaxCoarseBits];
    constexpr int kSwitches = kTile / kBlock / 4;  // switches per thread and tile
    constexpr bool kPacked = src_emits_packed<kSrc>();
    const uint32_t nt = max(1u, (nslots + kTile - 1) / kTile);
    const uint32_t nd = 1u << dbits, dmask = nd - 1, tid = threadIdx.x;
    const uint32_t m = sa.m, ell = m >> 1;
    if (tid == 0) bc = BlockCounts{0, 0, 0, 0};
    if (blockIdx.x == 0 && tid < 4) ucount[tid] = 0;  // the undecided-list counters of the rounds, arrivals
    // nc.counts: nc.tile positions (2 nc.tile slots) a trip, which are whole tiles here
    const uint32_t per = nc.counts ? 2 * nc.tile / kTile : 1u, nnext = nc.counts ? 1u << nc.dbits : 0u;
    for (uint32_t w0 = blockIdx.x * per; w0 < nt; w0 += gridDim.x * per) {
        for (uint32_t d = tid; d < nnext; d += kBlock) hn[d] = 0;  // (before the tile's first barrier)
    for (uint32_t w = w0; w < min(w0 + per, nt); ++w) {
        const uint32_t begin = w * kTile;
        const uint32_t cnt = begin < nslots ? min((uint32_t)kTile, nslots - begin) : 0u;
        for (uint32_t d = tid; d < nd; d += kBlock) hs[d] = 0;
        lds_barrier();
#pragma unroll
        for (int j = 0; j < kSwitches; ++j) {
            const uint32_t sl = 4 * (tid + j * kBlock);  // first local slot of this thread's switch
            Tuple tp[4] = {{0u, kEmptyKey}, {0u, kEmptyKey}, {0u, kEmptyKey}, {0u, kEmptyKey}};
            if (sl < cnt) {
                const uint32_t k = (begin + sl) >> 2;
                if (k < ell) {
                    const uint2 ij = reinterpret_cast<const uint2 *>(s_idx)[k];
                    const ulonglong2 ee = reinterpret_cast<const ulonglong2 *>(s_key)[k];
                    Targets T{0, 0, false};
                    const uint8_t status = switch_local(k, ij, ee, t, k0, k1, sa, &T);
                    st[k] = status;
                    if (nnext) {
                        atomicAdd(&hn[next_digit(nc, ij.x, 2 * k)], 1u);
                        atomicAdd(&hn[next_digit(nc, ij.y, 2 * k)], 1u);
                    }
                    if (status != ST_UNDECIDED) {
                        if (out_idx) {
                            reinterpret_cast<uint2 *>(out_idx)[k] = ij;
                            reinterpret_cast<ulonglong2 *>(out_key)[k] = ee;
                        }
                        if (status == ST_PL) atomicAdd(&bc.pl, 1u);
                        if (status == ST_LOOP) atomicAdd(&bc.loop, 1u);
                        if (status == ST_EXISTS) atomicAdd(&bc.exists, 1u);
                    }
                    switch_tuples(k, ij, ee, status, T, tp);
                } else if (k == ell && (m & 1u)) {  // the idle record of odd m stays
                    if (out_idx) {
                        out_idx[m - 1] = s_idx[m - 1];
                        out_key[m - 1] = s_key[m - 1];
                    }
                    if (nnext) atomicAdd(&hn[next_digit(nc, s_idx[m - 1], m - 1)], 1u);
                    tp[0] = Tuple{kTagStays, s_key[m - 1]};
                }
            }
#pragma unroll
            for (int h = 0; h < 4; ++h) {
                if (sl + h >= cnt) continue;
                const unsigned long long word = emitted_word<kPacked>(tp[h].key, sa);
                if (word != kEmptyKey) atomicAdd(&hs[(uint32_t)(word >> shift) & dmask], 1u);
            }
        }
        lds_barrier();
        for (uint32_t d = tid; d < nd; d += kBlock) counts[(size_t)w * nd + d] = hs[d];
        lds_barrier();
    }
        for (uint32_t d = tid; d < nnext; d += kBlock) nc.counts[(size_t)(w0 / per) * nnext + d] = hn[d];
        if (nnext) lds_barrier();
    }
    store_counts(&bc, bslot + blockIdx.x);
}

// The tuples of every slot written out flat (tuple buffer 0), for the
// unfused schedule (GESMC_OPT_FUSE_EMIT 0): one thread per switch.
__global__ __launch_bounds__(kBlock) void k_emit_tuples(const uint32_t *__restrict__ s_idx,
                                                        const unsigned long long *__restrict__ s_key, uint32_t t,
                                                        uint32_t k0, uint32_t k1, SrcArgs sa, uint32_t nslots,
                                                        uint32_t *__restrict__ tu_tag,
                                                        unsigned long long *__restrict__ tu_key) {
    const uint32_t stride = gridDim.x * kBlock;
    for (uint32_t k = blockIdx.x * kBlock + threadIdx.x; 4 * (uint64_t)k < nslots; k += stride) {
        Tuple tp[4];
        emit_switch(k, s_idx, s_key, t, k0, k1, sa, tp);
        for (uint32_t h = 0; h < 4 && 4 * k + h < nslots; ++h) {
            tu_tag[4 * k + h] = tp[h].tag;
            tu_key[4 * k + h] = tp[h].key;
        }
    }
}

// Validation only (no superstep): one STAYS tuple per input edge, so that a
// duplicate edge shows up as two ERASE tuples of one key.
__global__ __launch_bounds__(kBlock) void k_emit_sources(const unsigned long long *__restrict__ key, uint32_t m,
                                                         uint32_t *__restrict__ tu_tag,
                                                         unsigned long long *__restrict__ tu_key) {
    for (uint32_t i = blockIdx.x * kBlock + threadIdx.x; i < m; i += gridDim.x * kBlock) {
        tu_tag[i] = kTagStays;
        tu_key[i] = key[i];
    }
}

// Graph attribution of errors in a batch: the graph owning a key is the one
// whose vertex range holds its smaller endpoint.
struct GraphErr {
    const BatchGraph *gr;  // nullptr: no attribution
    uint32_t ngraphs;
    uint32_t *gerr;        // per graph error bits
};

// `key` is a tuple hash, or (pk.w > 0) a packed word with its tag code
// cleared; f is the tuple's partition, whose first-level digit restores the
// hash bits the packed word dropped.
// The rank of the graph holding the key of a tuple of fine partition f
// (ge.gr must be set): its smaller endpoint, by inverting the hash with the
// first level's digit restored, then the graph whose vertex range holds it.
__device__ __forceinline__ uint32_t graph_of_tuple(unsigned long long key, uint32_t f, const TuplePack &pk,
                                                   const GraphErr &ge) {
    uint32_t v;
    if (pk.w) {
        const uint64_t h = ((uint64_t)(f >> pk.b2) << (pk.w - pk.b1)) | (key >> (64 - pk.w + pk.b1));
        v = key_hash_w_vertex(h, pk.db, pk.w);
    } else {
        v = (uint32_t)(tuple_key_of(key) >> 32);
    }
    uint32_t lo = 0, hi = ge.ngraphs - 1;
    while (lo < hi) {
        const uint32_t mid = (lo + hi + 1) >> 1;
        if (ge.gr[mid].vbase <= v)
            lo = mid;
        else
            hi = mid - 1;
    }
    return lo;
}

__device__ __forceinline__ void flag_duplicate(unsigned long long key, uint32_t f, const TuplePack &pk, uint32_t *err,
                                               uint32_t dup_bit, const GraphErr &ge) {
    if (dup_bit) atomicOr(err, dup_bit);
    if (ge.gr) atomicOr(&ge.gerr[graph_of_tuple(key, f, pk, ge)], ERR_DUP);
}

// Writes the records of the tuple at sorted position p, given the position
// of the first tuple of its key and the smallest INSERT tag of its key.  A
// second ERASE tuple means the edge occurs twice: dup_bit is raised (and the graph flagged in a batch).
__device__ __forceinline__ void resolve_one(uint32_t tag, uint32_t first_tag, uint32_t first_ins, uint32_t p,
                                            uint32_t first, uint32_t prev_tag, unsigned long long key, uint32_t f,
                                            const TuplePack &pk, uint2 *info, uint32_t *st4, const Winners &wn,
                                            uint32_t *err, uint32_t dup_bit, const GraphErr &ge) {
    const bool ins = (tag & kTagInsert) != 0;
    if (!ins) {
        if (p != first) flag_duplicate(key, f, pk, err, dup_bit, ge);
        return;
    }
    uint32_t eraser = kNoEraser;
    if (!(first_tag & kTagInsert)) eraser = (first_tag == kTagStays) ? kStays : first_tag;
    uint32_t pred = (p > first && (prev_tag & kTagInsert)) ? (prev_tag & ~kTagInsert) : kNoPred;
    if (eraser == kNoEraser && pred == kNoPred) return;
    uint32_t slot = tag & ~kTagInsert;
    uint32_t head = first_ins & ~kTagInsert;
    if (pk.local) {  // graph-local tags (all of one key): back to batch-wide switch ids
        const uint32_t kbase = ge.gr[graph_of_tuple(key, f, pk, ge)].poff >> 1;
        slot += 2 * kbase;
        head += 2 * kbase;
        if (eraser != kStays && eraser != kNoEraser) eraser += kbase;
        if (pred != kNoPred) pred += 2 * kbase;
    }
    info[slot] = make_uint2(eraser, pred);
    // bytes of other switches share the word
    atomicOr(st4 + (slot >> 3), (uint32_t)(kStRecord << (slot & 1u)) << (8 * ((slot >> 1) & 3u)));
    if (pred != kNoPred) {
        wn.head[slot] = head;
        wn.win[head] = kNoWinner;  // every inserter after the first writes the same value
    }
}

// One workgroup per fine partition (grid-stride if the grid is smaller).
// LDS path: counting sort on kCellBits hash bits below the partition bits;
// each tuple then reads its own cell.  Partitions above `cap` (hub
// keys with many inserters) take an exact global-memory merge sort.
// Dynamic LDS: 2^kCellBits cell words + cap * 14 bytes
// (keys, tags and the 16-bit cell-list links), or cap * 10 bytes for packed
// words with the cell lists (the tags stay in the words).  kPacked: the tuples are
// packed words (no tag array); pbits is then the second level's bits only,
// the first level's having been dropped from the words.
// Seven waves per SIMD (72 registers): the walks wait on LDS, and at the 74 the
// compiler takes by itself a wave per SIMD is lost (n = 2^22: 38.2 -> 37.9 ms
// per call of ten supersteps; at eight waves 38.6).
template <bool kPacked>
__global__ __launch_bounds__(kBlock, 7) void k_resolve(uint32_t *__restrict__ tu_tag, unsigned long long *__restrict__ tu_key,
                                                    uint32_t *__restrict__ sc_tag,
                                                    unsigned long long *__restrict__ sc_key, int pbits,
                                                    const uint32_t *__restrict__ part_off, uint32_t np, uint32_t cap,
                                                    uint2 *__restrict__ info, uint32_t *__restrict__ err,
                                                    uint32_t dup_bit, StepCounters *ctr, GraphErr ge, TuplePack pk,
                                                    Winners wn, uint32_t *__restrict__ st4) {
    extern __shared__ __attribute__((aligned(16))) uint32_t lds[];
    constexpr uint32_t kCells = 1u << kCellBits;
    uint32_t *cell = lds;
    unsigned long long *sK = reinterpret_cast<unsigned long long *>(cell + kCells);
    uint32_t *sT = reinterpret_cast<uint32_t *>(sK + cap);
    const uint32_t tid = threadIdx.x;
    const int sub_shift = 64 - kCellBits;
    const uint32_t lds_cap = min(cap, (uint32_t)(kSortMaxItems * kBlock));
    const uint64_t code_mask = kPacked ? low_mask(pk.kb + 1) : 0ull;

    // cell lists: each cell word is (epoch << 16) | head slot, where the
    // epoch counts this workgroup's list-resolved partitions; a word of an
    // older epoch is an empty list, so no partition clears the cells
    uint32_t epoch = kEpochNone;
    // partition g's tuples (raw packed words, decoded at their first use)
    uint32_t c_tag[kSortMaxItems];
    unsigned long long c_key[kSortMaxItems];
    uint32_t begin = 0, end = 0;
    auto load_part = [&](uint32_t g) {
        begin = part_off[g];
        end = part_off[g + 1];
#pragma unroll
        for (int q = 0; q < kSortMaxItems; ++q) {
            const uint32_t p = begin + tid + q * kBlock;
            c_tag[q] = (!kPacked && p < end) ? tu_tag[p] : 0u;
            c_key[q] = p < end ? tu_key[p] : 0ull;
        }
    };
    if (blockIdx.x < np) load_part(blockIdx.x);
    for (uint32_t f = blockIdx.x; f < np; f += gridDim.x) {
        const uint32_t c = end > begin ? end - begin : 0;
        if (kPacked && c > lds_cap) {
            // exact slow path over packed words: their order is (key, tag)
            // order, so a merge sort of the words is the sort by (key, tag)
            unsigned long long *ak = tu_key + begin, *bk = sc_key + begin;
            for (uint32_t width = 1; width < c; width <<= 1) {
                for (uint32_t p = tid; p < c; p += kBlock) {
                    const uint32_t run = p / (2 * width);
                    const uint32_t lo = run * 2 * width, mid = min(lo + width, c), hi = min(lo + 2 * width, c);
                    const unsigned long long kp = ak[p];
                    uint32_t pos;
                    if (p < mid) {  // rank among the right run: words strictly smaller
                        uint32_t a = mid, b = hi;
                        while (a < b) {
                            const uint32_t x = (a + b) >> 1;
                            if (ak[x] < kp)
                                a = x + 1;
                            else
                                b = x;
                        }
                        pos = lo + (p - lo) + (a - mid);
                    } else {  // rank among the left run: words smaller or equal
                        uint32_t a = lo, b = mid;
                        while (a < b) {
                            const uint32_t x = (a + b) >> 1;
                            if (ak[x] <= kp)
                                a = x + 1;
                            else
                                b = x;
                        }
                        pos = lo + (p - mid) + (a - lo);
                    }
                    bk[pos] = kp;
                }
                __threadfence_block();
                __syncthreads();
                unsigned long long *xk = ak;
                ak = bk;
                bk = xk;
            }
            for (uint32_t p = tid; p < c; p += kBlock) {
                const unsigned long long kp = ak[p] & ~code_mask;
                uint32_t a = 0, b = p;
                while (a < b) {
                    const uint32_t x = (a + b) >> 1;
                    if ((ak[x] & ~code_mask) < kp)
                        a = x + 1;
                    else
                        b = x;
                }
                const auto tag_at = [&](uint32_t x) { return tag_of_code((uint32_t)(ak[x] & code_mask), pk.kb); };
                const uint32_t tp = tag_at(p), ta = tag_at(a);
                // a group holds one ERASE tuple at most (two are an input error)
                const uint32_t fi = (ta & kTagInsert) ? ta : a < p ? tag_at(a + 1) : tp;
                resolve_one(tp, ta, (fi & kTagInsert) ? fi : tp, p, a, p > 0 ? tag_at(p - 1) : 0u, kp, f, pk, info,
                            st4, wn, err, dup_bit, ge);
            }
            if (tid == 0) atomicAdd(&ctr->fallback_buckets, 1ull);
            __syncthreads();
        } else if (c > lds_cap) {
            // exact slow path: bottom-up merge sort by (key, tag) between the
            // partition's range and the scratch range, then binary searches.
            uint32_t *at = tu_tag + begin, *bt = sc_tag + begin;
            unsigned long long *ak = tu_key + begin, *bk = sc_key + begin;
            for (uint32_t width = 1; width < c; width <<= 1) {
                for (uint32_t p = tid; p < c; p += kBlock) {
                    const uint32_t run = p / (2 * width);
                    const uint32_t lo = run * 2 * width, mid = min(lo + width, c), hi = min(lo + 2 * width, c);
                    const unsigned long long kp = ak[p];
                    const uint32_t tp = at[p];
                    uint32_t pos;
                    if (p < mid) {  // rank among the right run: elements strictly smaller
                        uint32_t a = mid, b = hi;
                        while (a < b) {
                            const uint32_t x = (a + b) >> 1;
                            if (ak[x] < kp || (ak[x] == kp && at[x] < tp))
                                a = x + 1;
                            else
                                b = x;
                        }
                        pos = lo + (p - lo) + (a - mid);
                    } else {  // rank among the left run: elements smaller or equal
                        uint32_t a = lo, b = mid;
                        while (a < b) {
                            const uint32_t x = (a + b) >> 1;
                            if (ak[x] < kp || (ak[x] == kp && at[x] <= tp))
                                a = x + 1;
                            else
                                b = x;
                        }
                        pos = lo + (p - mid) + (a - lo);
                    }
                    bt[pos] = tp;
                    bk[pos] = kp;
                }
                __threadfence_block();
                __syncthreads();
                uint32_t *xt = at;
                at = bt;
                bt = xt;
                unsigned long long *xk = ak;
                ak = bk;
                bk = xk;
            }
            for (uint32_t p = tid; p < c; p += kBlock) {
                const unsigned long long kp = ak[p];
                uint32_t a = 0, b = p;
                while (a < b) {
                    const uint32_t x = (a + b) >> 1;
                    if (ak[x] < kp)
                        a = x + 1;
                    else
                        b = x;
                }
                const uint32_t fi = (at[a] & kTagInsert) ? at[a] : a < p ? at[a + 1] : at[p];
                resolve_one(at[p], at[a], (fi & kTagInsert) ? fi : at[p], p, a, p > 0 ? at[p - 1] : 0u, kp, f, pk,
                            info, st4, wn, err, dup_bit, ge);
            }
            if (tid == 0) atomicAdd(&ctr->fallback_buckets, 1ull);
            __syncthreads();
        } else if (c > 0) {
            // Tuples stay in their own slots p (contiguous writes); each cell
            // keeps a list of its slots, linked by one LDS exchange per tuple.
            // Packed words stay whole in sK (key bits and tag code), with no
            // tag array: 10 bytes of LDS per tuple instead of 14.
            uint16_t *nxt = reinterpret_cast<uint16_t *>(kPacked ? reinterpret_cast<uint32_t *>(sK + cap) : sT + cap);
            if (epoch >= kEpochNone - 1) {  // first list partition, or the epochs wrap: every list empty
                for (uint32_t q = tid; q < kCells; q += kBlock) cell[q] = 0xFFFFFFFFu;
                lds_barrier();
                epoch = 0;
            } else {
                ++epoch;
            }
            const uint32_t ep = epoch << 16;
            uint32_t r_cell[kSortMaxItems];
#pragma unroll
            for (int q = 0; q < kSortMaxItems; ++q) {
                const uint32_t p = tid + q * kBlock;
                if (p < c) {
                    const unsigned long long raw = c_key[q];
                    if (kPacked) {  // the key bits stay in place (cells, equality); the code is the tag
                        c_tag[q] = tag_of_code((uint32_t)(raw & code_mask), pk.kb);
                        c_key[q] = raw & ~code_mask;
                    }
                    const uint64_t hsh = c_key[q];  // tuple words are tuple hashes
                    r_cell[q] = (uint32_t)((pbits >= 64 ? 0ull : (hsh << pbits)) >> sub_shift);
                    sK[p] = raw;
                    if (!kPacked) sT[p] = c_tag[q];
                    const uint32_t old = atomicExch(&cell[r_cell[q]], ep | p);
                    nxt[p] = (old & 0xFFFF0000u) == ep ? (uint16_t)old : (uint16_t)kListEnd;
                }
            }
            lds_barrier();
            // All tuples of one key share a cell.  Each tuple walks its cell's
            // list for what the walk over the sorted group would give: the
            // group's smallest tag, whether a tuple precedes it in (key, tag,
            // slot) order and the largest preceding tag.
#pragma unroll
            for (int q = 0; q < kSortMaxItems; ++q) {
                const uint32_t p = tid + q * kBlock;
                if (p >= c) continue;
                const unsigned long long kx = c_key[q];
                const uint32_t tx = c_tag[q];
                uint32_t first_tag = tx, first_ins = tx, prev_tag = 0;
                bool before = false;
                for (uint32_t y = cell[r_cell[q]] & 0xFFFFu; y != kListEnd; y = nxt[y]) {
                    const unsigned long long wy = sK[y];
                    if (y == p || (kPacked ? (wy & ~code_mask) : wy) != kx) continue;
                    const uint32_t ty = kPacked ? tag_of_code((uint32_t)(wy & code_mask), pk.kb) : sT[y];
                    first_tag = min(first_tag, ty);
                    if (ty & kTagInsert) first_ins = min(first_ins, ty);
                    if (ty < tx || (ty == tx && y < p)) {
                        prev_tag = before ? max(prev_tag, ty) : ty;
                        before = true;
                    }
                }
                resolve_one(tx, first_tag, first_ins, before ? 1u : 0u, 0u, prev_tag, kx, f, pk, info, st4, wn, err,
                            dup_bit, ge);
            }
        }
        // the next partition's loads are issued before the barrier that ends
        // this one (every walk done before the cells are linked again), so
        // they are in flight while the slowest wave finishes
        if (f + gridDim.x < np) load_part(f + gridDim.x);
        lds_barrier();
    }
}

// ---------------------------------------------------------------------------
// Decisions
// ---------------------------------------------------------------------------
// Where a judgement reads statuses: from memory while other workgroups write
// them too, from memory while only this one does (its CU's cache serves the
// loads), or from a copy in LDS.
struct GridStatus {
    static constexpr int kScope = __HIP_MEMORY_SCOPE_AGENT;
    const uint8_t *st;
    __device__ __forceinline__ uint8_t operator()(uint32_t k) const { return load_status(st, k); }
};
struct GroupStatus {
    static constexpr int kScope = __HIP_MEMORY_SCOPE_WORKGROUP;
    const uint8_t *st;
    __device__ __forceinline__ uint8_t operator()(uint32_t k) const { return load_status<true>(st, k); }
};
struct LdsStatus {
    static constexpr int kScope = __HIP_MEMORY_SCOPE_WORKGROUP;
    const volatile uint8_t *st;  // (in LDS; every id is below the switches copied)
    __device__ __forceinline__ uint8_t operator()(uint32_t k) const { return st[k] & kStOutcome; }
};

// Two shortcuts keep long chains (many switches inserting one hub edge)
// linear: inserters older than the target's eraser saw the target present,
// so they were rejected and the walk stops there; and a walk that passed
// decided-rejected inserters stores the first one it stopped at in its own
// record's predecessor link (`self`), so later walks through this switch
// skip them.  Any value so written skips only decided-rejected inserters of
// the same target, so concurrent writers are harmless.
//
// from (nullable): the walk resumes at *from (kNoPred: the first predecessor,
// rec.y) and leaves there the predecessor it waits for: decided predecessors
// never change, so a repeated judgement of the same switch walks each link
// once.
template <typename St>
__device__ __forceinline__ int judge_target_chain(uint2 *info, const Winners &wn, uint2 rec, uint32_t self, uint32_t k,
                                                  St st, uint32_t *from = nullptr) {
    int v = V_OK;
    const uint32_t e = rec.x;
    if (e != kNoEraser) {
        if (e == kStays || e >= k) return V_ILLEGAL;
        const uint8_t se = st(e);
        if (se == ST_UNDECIDED)
            v = V_WAIT;
        else if (se != ST_LEGAL)
            return V_ILLEGAL;
    }
    // earlier inserters of the same target, nearest first; switch ids strictly
    // decrease along the chain (checked, so a corrupt record cannot loop)
    uint32_t p = rec.y, below = k;
    if (from && *from != kNoPred) {
        p = *from;
        if (!chain_end(p)) below = (p >> 1) + 1;
    }
    const uint32_t p0 = p;
    const uint32_t first = chain_end(p) ? kNoPred : wn.head[self];  // ends the chain (it may have no record)
    int out = v;
    while (!chain_end(p)) {
        const uint32_t pk = p >> 1;
        if (pk >= below) return V_ILLEGAL;
        if (e != kNoEraser && pk < e) {  // inserted while the target was still there
            p = kWalked;
            break;
        }
        const uint8_t sp = st(pk);
        if (sp == ST_LEGAL) {
            out = V_ILLEGAL;
            break;
        }
        if (sp == ST_UNDECIDED) {
            // an inserter before it may have won already
            out = st(first >> 1) == ST_LEGAL ||
                          __hip_atomic_load(wn.win + first, __ATOMIC_RELAXED,
                                            St::kScope) != kNoWinner
                      ? V_ILLEGAL
                      : V_WAIT;
            break;
        }
        below = pk;
        const uint32_t q = p == first ? kWalked : info[p].y;
        p = chain_end(q) ? kWalked : q;
    }
    if (p != p0) info[self].y = p;
    if (from) *from = p == kNoPred ? kWalked : p;
    return out;
}

// Leaves the legal switch k as the winner of its targets' keys (records recs).
__device__ __forceinline__ void post_winner(const Winners &wn, uint4 recs, uint32_t k) {
    if (recs.y != kNoPred)
        __hip_atomic_store(wn.win + wn.head[2 * k], k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (recs.w != kNoPred)
        __hip_atomic_store(wn.win + wn.head[2 * k + 1], k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The target records of a switch with undecided status byte s.
__device__ __forceinline__ uint4 target_records(const uint2 *info, uint32_t k, uint8_t s) {
    uint4 r = make_uint4(kNoEraser, kNoPred, kNoEraser, kNoPred);
    if (s & kStRecord) {
        const uint2 a = info[2 * k];
        r.x = a.x;
        r.y = a.y;
    }
    if (s & (kStRecord << 1)) {
        const uint2 b = info[2 * k + 1];
        r.z = b.x;
        r.w = b.y;
    }
    return r;
}

// Verdict on switch k from its two target records.
template <typename St>
__device__ __forceinline__ int judge_switch_chain(uint32_t k, uint4 recs, uint2 *info, const Winners &wn, St st,
                                                  uint2 *from = nullptr) {
    return max(judge_target_chain(info, wn, make_uint2(recs.x, recs.y), 2 * k, k, st, from ? &from->x : nullptr),
               judge_target_chain(info, wn, make_uint2(recs.z, recs.w), 2 * k + 1, k, st,
                                        from ? &from->y : nullptr));
}

// Carries out verdict v on switch k; true if it has to wait.  The pair's
// records (ij, ee) are passed in so that callers can issue every load of the
// switch at once.  pos (nullable): the pair's records stand at pos[k] with the
// sources' keys (k_decide_scatter), else they go to slots 2k, 2k + 1.
__device__ __forceinline__ bool commit_switch_chain(int v, uint32_t k, uint4 recs, uint2 ij, ulonglong2 ee,
                                                    const Winners &wn, uint8_t *st, uint32_t *out_idx,
                                                    unsigned long long *out_key, const uint2 *pos, BlockCounts *bc,
                                                    uint32_t cls) {
    if (v == V_WAIT) return true;
    if (!pos) reinterpret_cast<uint2 *>(out_idx)[k] = ij;
    if (v == V_OK) {
        const Targets T = switch_targets_cls(ee.x, ee.y, ij.x < ij.y, cls);
        if (pos) {
            const uint2 g = pos[k];
            out_key[g.x] = T.A;
            out_key[g.y] = T.B;
        } else {
            reinterpret_cast<ulonglong2 *>(out_key)[k] = make_ulonglong2(T.A, T.B);
        }
        post_winner(wn, recs, k);
        st[k] = ST_LEGAL;
        atomicAdd(&bc->legal, 1u);
    } else {
        if (!pos) reinterpret_cast<ulonglong2 *>(out_key)[k] = ee;
        st[k] = ST_EXISTS;
        atomicAdd(&bc->exists, 1u);
    }
    return false;
}

// Undecided switches staged per workgroup of k_decide_chain: the switches of
// one 4096-record tile.
constexpr uint32_t kWaitStage = kTileLarge / 2;
static_assert(kTileTiny % (2 * kBlock) == 0 && kWaitStage % kBlock == 0, "stage flushes cover whole trips");

// Round 1 (list == nullptr: every switch) or a later round over a list.
// With fold, also sums the nfold per-block counts of the emit and of round 1
// (256 a workgroup: the finisher's one workgroup took 5 us for the 10,240 of a
// large graph).  With nc.counts (round 1 only), each workgroup takes whole tiles of
// nc.tile / 2 switches and also writes their counts.
__global__ __launch_bounds__(kBlock) void k_decide_chain(const uint32_t *__restrict__ s_idx,
                                                         const unsigned long long *__restrict__ s_key, uint32_t ell,
                                                         uint2 *info, uint8_t *st,
                                                         uint32_t *__restrict__ out_idx,
                                                         unsigned long long *__restrict__ out_key,
                                                         const uint32_t *__restrict__ list,
                                                         const uint32_t *__restrict__ count,
                                                         uint32_t *__restrict__ next_list,
                                                         uint32_t *__restrict__ next_count,
                                                         uint32_t *__restrict__ zero_count,
                                                         uint4 *__restrict__ bslot, StepCounters *ctr,
                                                         uint32_t cls, NextCounts nc, Winners wn,
                                                         const uint4 *__restrict__ fold, uint32_t nfold,
                                                         const uint2 *__restrict__ pos) {
    __shared__ BlockCounts bc;
    __shared__ uint32_t hs[1u << kMaxCoarseBits];
    __shared__ uint32_t s_wait[kWaitStage], s_nwait, s_wbase;
    if (threadIdx.x == 0) {
        bc = BlockCounts{0, 0, 0, 0};
        s_nwait = 0;
    }
    __syncthreads();
    // Undecided switches are staged in LDS and leave with one device atomic
    // per kWaitStage switches: an atomic per wave on the one list counter
    // (and one on its tally) serialises memory-side, and on graphs whose
    // switches depend on each other nearly every wave holds an undecided one.
    auto stage_undecided = [&](bool want, uint32_t k) {
        const unsigned long long mask = __ballot(want);
        if (mask == 0) return;
        const uint32_t leader = __ffsll((long long)mask) - 1;
        uint32_t base = 0;
        if (__lane_id() == leader) base = atomicAdd(&s_nwait, (uint32_t)__popcll(mask));
        base = __shfl(base, leader);
        if (want) s_wait[base + __popcll(mask & ((1ull << __lane_id()) - 1ull))] = k;
    };
    // every thread of the workgroup; at most kWaitStage switches since the last call
    auto flush_undecided = [&]() {
        __syncthreads();
        const uint32_t c = s_nwait;
        __syncthreads();  // read by every wave before the next trip may stage again
        if (c == 0) return;
        if (threadIdx.x == 0) s_wbase = atomicAdd(next_count, c);
        __syncthreads();
        for (uint32_t q = threadIdx.x; q < c; q += kBlock) next_list[s_wbase + q] = s_wait[q];
        if (threadIdx.x == 0) s_nwait = 0;
        __syncthreads();
    };
    // the counter cleared here is the one the round after next fills
    if (zero_count && blockIdx.x == 0 && threadIdx.x == 0) *zero_count = 0;
    auto decide_one = [&](uint32_t k, bool *wait, uint2 *ij_out) {
        const uint8_t sk = st[k];
        const uint2 ij = reinterpret_cast<const uint2 *>(s_idx)[k];
        const ulonglong2 ee = reinterpret_cast<const ulonglong2 *>(s_key)[k];
        *ij_out = ij;
        if ((sk & kStOutcome) != ST_UNDECIDED) return;
        const uint4 recs = target_records(info, k, sk);
        *wait = commit_switch_chain(judge_switch_chain(k, recs, info, wn, GridStatus{st}), k, recs, ij, ee, wn, st,
                                    out_idx, out_key,
                                    pos, &bc, cls);
    };
    const uint32_t n = list ? min(*count, ell) : ell;
    for (uint32_t q = blockIdx.x * kBlock + threadIdx.x; q < nfold; q += gridDim.x * kBlock) {
        const uint4 v = fold[q];
        if (v.x) atomicAdd(&bc.legal, v.x);
        if (v.y) atomicAdd(&bc.loop, v.y);
        if (v.z) atomicAdd(&bc.exists, v.z);
        if (v.w) atomicAdd(&bc.pl, v.w);
    }
    if (nc.counts) {
        const uint32_t nd = 1u << nc.dbits, half = nc.tile / 2;
        // tiles of the next step's positions (a batch's prefix may shrink: the
        // tiles then also cover this step's remaining switches, uncounted)
        const uint32_t ncount = (nc.m + nc.tile - 1) / nc.tile;
        const uint32_t ntiles = max(ncount, (ell + half - 1) / half);
        auto digit = [&](uint32_t i, uint32_t pos) { return next_digit(nc, i, pos); };
        for (uint32_t w = blockIdx.x; w < ntiles; w += gridDim.x) {
            for (uint32_t d = threadIdx.x; d < nd; d += kBlock) hs[d] = 0;
            __syncthreads();
            for (uint32_t j = 0; j < half; j += kBlock) {
                const uint32_t k = w * half + j + threadIdx.x;
                bool wait = false;
                if (k < ell) {
                    uint2 ij;
                    decide_one(k, &wait, &ij);
                    if (2 * k + 1 < nc.m) {  // both positions of a pair lie in one graph
                        atomicAdd(&hs[digit(ij.x, 2 * k)], 1u);
                        atomicAdd(&hs[digit(ij.y, 2 * k)], 1u);
                    }
                }
                stage_undecided(wait, k);
            }
            if ((nc.m & 1u) && threadIdx.x == 0 && (nc.m - 1) / nc.tile == w)  // the idle record of odd m
                atomicAdd(&hs[digit(s_idx[nc.m - 1], nc.m - 1)], 1u);
            flush_undecided();
            if (w < ncount)
                for (uint32_t d = threadIdx.x; d < nd; d += kBlock) nc.counts[(size_t)w * nd + d] = hs[d];
            __syncthreads();
        }
    } else {
        const uint32_t stride = gridDim.x * kBlock;
        const uint32_t trips = (n + stride - 1) / stride;
        for (uint32_t r = 0; r < trips; ++r) {
            const uint32_t q = r * stride + blockIdx.x * kBlock + threadIdx.x;
            bool wait = false;
            uint32_t k = 0;
            if (q < n) {
                k = list ? list[q] : q;
                uint2 ij;
                if (k < ell) decide_one(k, &wait, &ij);
            }
            stage_undecided(wait, k);
            if ((r + 1) % (kWaitStage / kBlock) == 0 || r + 1 == trips) flush_undecided();
        }
    }
    // the list of round 1 is counted by whoever reads it first (and sums its counts)
    if (nfold && blockIdx.x == 0 && threadIdx.x == 0) ctr->undecided_round1 = n;
    if (bslot)
        store_counts(&bc, bslot + blockIdx.x);
    else
        flush_counts(&bc, ctr);
    if (blockIdx.x == 0 && threadIdx.x == 0 && n > 0) atomicAdd(&ctr->rounds, 1ull);
}

// Round 1 and the next superstep's first radix scatter in one pass over the
// pair records: a tile's switches are judged as by k_decide_chain, and its
// records -- accepted switches with their targets, all others as they are --
// leave through the LDS stage of k_scatter in the order of the next
// permutation's first level (run bases in offs, counted by k_emit_counts).
// A switch that waits leaves its sources there and its two places in pos; the
// later rounds write its targets over them.  The two passes apart wrote the
// records and read them back, 48 of 114 bytes a switch; both are bound by
// memory: n = 2^22, d = 32, 467 + 382 us a superstep apart, 370 together (5.3
// TB/s in loads and stores; the emit takes 90 us more for the counts).
// One workgroup per tile; its counts go to bslot[blockIdx.x].
template <int kSrc, int kTile, int kThreads, bool kSelf>
__global__ __launch_bounds__(kThreads) void k_decide_scatter(
    const uint32_t *__restrict__ s_idx, const unsigned long long *__restrict__ s_key, uint32_t m, uint2 *info,
    uint8_t *st, Winners wn, uint32_t *__restrict__ dst_idx, unsigned long long *__restrict__ dst_key,
    uint2 *__restrict__ pos, uint32_t *__restrict__ next_list, uint32_t *__restrict__ next_count,
    uint4 *__restrict__ bslot, StepCounters *ctr, uint32_t cls, uint32_t t, uint32_t k0, uint32_t k1, int shift,
    int dbits, const uint32_t *__restrict__ offs, uint32_t *__restrict__ err, SrcArgs ba) {
    static_assert(kSrc == kSrcPerm || kSrc == kSrcBatch, "edge records");
    extern __shared__ __attribute__((aligned(16))) uint32_t lds[];
    __shared__ uint32_t s_nwait, s_wbase, s_legal, s_exists;
    constexpr int kPairs = kTile / kThreads / 2;
    constexpr uint32_t kScanWords = kThreads / 64 + 1;
    const bool dik = kSrc == kSrcPerm && ba.dig_in_key != 0;
    constexpr unsigned long long kKeyLow56 = 0x00FFFFFFFFFFFFFFull;
    const uint32_t nd = 1u << dbits, dmask = nd - 1;
    uint32_t *cnt = lds, *start = cnt + nd, *base = start + nd, *tmp = base + nd;
    uint32_t *l_idx = tmp + kScanWords;
    unsigned long long *l_key =
        reinterpret_cast<unsigned long long *>(l_idx + kTile + ((kScanWords + 3 * nd + kTile) & 1));
    uint16_t *l_dig = reinterpret_cast<uint16_t *>(l_key + kTile);
    uint32_t *l_bkt = reinterpret_cast<uint32_t *>(l_dig + kTile);  // kSrcBatch only
    const uint32_t nt = (m + kTile - 1) / kTile, w = xcd_tile(blockIdx.x, nt), tid = threadIdx.x, ell = m >> 1;
    const uint32_t begin = w * kTile, staged = min((uint32_t)kTile, m - begin);
    // a thread's pairs: k = begin / 2 + tid + j kThreads (the idle record of odd m is half a pair)
    uint2 ij[kPairs];
    ulonglong2 ee[kPairs];
    uint8_t sk[kPairs];
    uint32_t aux[kPairs];
#pragma unroll
    for (int j = 0; j < kPairs; ++j) {
        const uint32_t k = (begin >> 1) + tid + j * kThreads;
        ij[j] = make_uint2(0, 0);
        ee[j] = make_ulonglong2(0, 0);
        sk[j] = ST_IDLE;
        aux[j] = 0;
        if (k < ell) {
            ij[j] = reinterpret_cast<const uint2 *>(s_idx)[k];
            ee[j] = reinterpret_cast<const ulonglong2 *>(s_key)[k];
            sk[j] = st[k];
            if (kSrc == kSrcBatch) aux[j] = ba.aux_in[2 * k];  // both records of a pair belong to one graph
        } else if (k == ell && (m & 1u)) {
            ij[j].x = s_idx[m - 1];
            ee[j].x = s_key[m - 1];
            if (kSrc == kSrcBatch) aux[j] = ba.aux_in[m - 1];
        }
    }
    if (tid == 0) s_nwait = s_legal = s_exists = 0;
    if (kSelf) tile_bases<kThreads>(offs, ba.self_off, w, nt, nd, cnt, start, base, tmp);
    for (uint32_t d = tid; d < nd; d += kThreads) {
        cnt[d] = 0;
        if (!kSelf) base[d] = offs[(size_t)w * nd + d];
    }
    lds_barrier();
    uint32_t legal = 0, exists = 0, slot[kPairs];
    uint32_t waits = 0;
#pragma unroll
    for (int j = 0; j < kPairs; ++j) {
        const uint32_t k = (begin >> 1) + tid + j * kThreads;
        slot[j] = 0;
        if (k >= ell || (sk[j] & kStOutcome) != ST_UNDECIDED) continue;
        const uint4 recs = target_records(info, k, sk[j]);
        const int v = judge_switch_chain(k, recs, info, wn, GridStatus{st});
        if (v == V_WAIT) {
            waits |= 1u << j;
            slot[j] = atomicAdd(&s_nwait, 1u);
        } else if (v == V_OK) {
            const Targets T = switch_targets_cls(ee[j].x, ee[j].y, ij[j].x < ij[j].y, cls);
            ee[j] = make_ulonglong2(T.A, T.B);
            post_winner(wn, recs, k);
            st[k] = ST_LEGAL;
            ++legal;
        } else {
            st[k] = ST_EXISTS;
            ++exists;
        }
    }
    if (legal) atomicAdd(&s_legal, legal);
    if (exists) atomicAdd(&s_exists, exists);
    // (from here on as k_scatter)
    uint32_t r_dig[2 * kPairs], r_rank[2 * kPairs], r_bkt[2 * kPairs];
#pragma unroll
    for (int q = 0; q < 2 * kPairs; ++q) {
        const uint32_t p = begin + 2 * (tid + (q >> 1) * kThreads) + (q & 1);
        r_dig[q] = 0xFFFFFFFFu;
        r_bkt[q] = 0;
        if (p < m) {
            const uint32_t i = (q & 1) ? ij[q >> 1].y : ij[q >> 1].x;
            const uint64_t word = radix_word<kSrc>(i, 0ull, aux[q >> 1], t, k0, k1, ba, &r_bkt[q]);
            r_dig[q] = (uint32_t)(word >> shift) & dmask;
            r_rank[q] = atomicAdd(&cnt[r_dig[q]], 1u);
        }
    }
    lds_barrier();
    for (uint32_t d = tid; d < nd; d += kThreads) start[d] = cnt[d];
    if (tid == 0) {
        if (s_nwait) s_wbase = atomicAdd(next_count, s_nwait);
        bslot[blockIdx.x] = make_uint4(s_legal, 0u, s_exists, 0u);
        if (blockIdx.x == 0) atomicAdd(&ctr->rounds, 1ull);
    }
    lds_barrier();
    block_exclusive_scan<kThreads>(start, nd, tmp);
#pragma unroll
    for (int q = 0; q < 2 * kPairs; ++q) {
        if (r_dig[q] == 0xFFFFFFFFu) continue;
        const uint32_t lp = start[r_dig[q]] + r_rank[q];
        const unsigned long long key = (q & 1) ? ee[q >> 1].y : ee[q >> 1].x;
        l_idx[lp] = (q & 1) ? ij[q >> 1].y : ij[q >> 1].x;
        if (dik) {
            l_key[lp] = (key & kKeyLow56) | ((unsigned long long)r_dig[q] << 56);
        } else {
            l_key[lp] = key;
            l_dig[lp] = (uint16_t)r_dig[q];
        }
        if (kSrc == kSrcBatch) l_bkt[lp] = r_bkt[q];
    }
#pragma unroll
    for (int j = 0; j < kPairs; ++j) {
        if (!(waits & (1u << j))) continue;
        const uint32_t k = (begin >> 1) + tid + j * kThreads;
        const uint2 g = make_uint2(base[r_dig[2 * j]] + r_rank[2 * j], base[r_dig[2 * j + 1]] + r_rank[2 * j + 1]);
        if (g.x < m && g.y < m) {
            pos[k] = g;
            next_list[s_wbase + slot[j]] = k;
        } else {  // never for consistent counts
            pos[k] = make_uint2(0, 0);
            next_list[s_wbase + slot[j]] = k;
            atomicOr(err, ERR_INTERNAL);
        }
    }
    lds_barrier();
    for (uint32_t lp = tid; lp < staged; lp += kThreads) {
        const unsigned long long word = l_key[lp];
        const uint32_t d = dik ? (uint32_t)(word >> 56) : (uint32_t)l_dig[lp];
        const uint32_t g = base[d] + (lp - start[d]);
        if (g < m) {
            dst_idx[g] = l_idx[lp];
            dst_key[g] = dik ? word & kKeyLow56 : word;
            if (kSrc == kSrcBatch) ba.aux_out[g] = l_bkt[lp];
        } else {
            atomicOr(err, ERR_INTERNAL);
        }
    }
}

// Remaining rounds in one workgroup; the next round's list counter is cleared
// by the round that fills it.  Every pass of the workgroup over kChainFinish
// switches of the list counts as a round in ctr (a later pass of the same sweep over
// the list already sees what the earlier ones decided); round_limit is charged
// one for a whole sweep, as for a round of the whole chip, so that what it allows
// does not depend on the workgroup's width.  After kSweepAfter rounds with switches still
// undecided (long dependency chains: hub edges that many switches erase and
// insert), the rest is decided by a sweep in ascending switch id: a switch
// depends on smaller ids only, so chunks of kSweepChunk ids are taken in
// order, each repeated until it holds no undecided switch; earlier chunks
// are then final and only chains inside a chunk cost repeats.  Each repeat
// counts as a round.
constexpr int kChainFinish = 512;
// Undecided switches, of so many in all, whose list and statuses go to LDS: as
// many as the sweep's array holds.  us per superstep without and with the copy:
// 15,000 switches, 290 undecided 65.9 and 59.4; 22,600, 63 of them 58.0 and 56.1,
// 410 69.9 and 63.0; 45,200, 55 64.1 and 63.1, 860 83.4 and 77.1; 60,000, 58
// 69.6 and 68.9, 1,113 91.7 and 88.0.
constexpr uint32_t kFinishList = 2048, kFinishSwitches = 65536;
constexpr uint32_t kSweepAfter = 8;
constexpr uint32_t kSweepChunk = 1024;
constexpr uint32_t kSweepWords = 16384;  // chunk marks: ids below 2^29 (m < 2^30)
static_assert(kFinishSwitches <= 4 * kSweepWords, "the statuses fit the chunk marks' array");

// The first sweep over a longer list than this (but one that fits LDS) is shared
// by the launch's kFinishGrid workgroups, as a round of the whole chip, and the
// last of them to arrive is the finishing workgroup; those of a shorter list leave
// at once.  No list round runs before it on smaller graphs (decision_rounds), and
// on a dense one most switches are still undecided: G(500, 0.9), m = 1.1e5, 20,000
// of 56,000, us per superstep with one workgroup for all passes 399, shared 150,
// after two list rounds 167; power law of gamma = 2.01, n = 40,000 707 and 520.
constexpr uint32_t kFinishShared = 1024, kFinishGrid = 64;

__global__ __launch_bounds__(kChainFinish) void k_finish_chain(const uint32_t *__restrict__ s_idx,
                                                               const unsigned long long *__restrict__ s_key,
                                                               uint32_t ell, uint2 *info,
                                                               uint8_t *st, uint32_t *__restrict__ out_idx,
                                                               unsigned long long *__restrict__ out_key,
                                                               uint32_t *list_a, uint32_t *count_a, uint32_t *list_b,
                                                               uint32_t *count_b, const uint4 *__restrict__ bslot,
                                                               uint32_t nbslot, StepCounters *ctr,
                                                               uint32_t *__restrict__ err, uint32_t round_limit,
                                                               uint32_t cls, Winners wn,
                                                               const uint2 *__restrict__ pos,
                                                               uint32_t *__restrict__ arrived) {
    __shared__ BlockCounts bc;
    __shared__ uint32_t s_n, s_first;
    const uint32_t tid = threadIdx.x;
    unsigned long long charged = 0;  // rounds that count against round_limit (thread 0)
    if (tid == 0) s_first = min(*count_a, ell);
    __syncthreads();
    // (a count that the finishing workgroup of a short list has overwritten is shorter still)
    const uint32_t first = s_first;
    const bool share = gridDim.x > 1 && first > kFinishShared && !(first <= kFinishList && ell <= kFinishSwitches);
    if (!share && blockIdx.x != 0) return;
    if (tid == 0) {
        bc = BlockCounts{0, 0, 0, 0};
        s_n = first;
        if (nbslot && blockIdx.x == 0) ctr->undecided_round1 = first;
        // a caller's round budget (0: none), counted over the superstep's rounds so
        // far (the multi-workgroup rounds before this kernel included)
        charged = round_limit ? atomicAdd(&ctr->rounds, 0ull) : 0ull;
        if (round_limit && (charged > round_limit || (charged == round_limit && first > 0))) {
            atomicOr(err, ERR_ROUNDS);
            s_n = 0;
        }
    }
    __syncthreads();
    uint32_t *cur = list_a, *nxt = list_b, *ccur = count_a, *cnxt = count_b;
    if (share && s_n == 0 && blockIdx.x != 0) return;  // (every workgroup found the budget spent)
    if (share && s_n > 0) {
        __shared__ uint32_t s_here, s_base, s_last;
        for (uint32_t q0 = blockIdx.x * kChainFinish; q0 < first; q0 += gridDim.x * kChainFinish) {
            const uint32_t q = q0 + tid;
            bool wait = false;
            uint32_t k = 0;
            if (tid == 0) s_here = 0;
            if (q < first) {
                k = list_a[q];
                const uint8_t sk = k < ell ? st[k] : (uint8_t)ST_LEGAL;
                if ((sk & kStOutcome) == ST_UNDECIDED) {
                    const uint4 recs = target_records(info, k, sk);
                    wait = commit_switch_chain(judge_switch_chain(k, recs, info, wn, GridStatus{st}), k, recs,
                                               reinterpret_cast<const uint2 *>(s_idx)[k],
                                               reinterpret_cast<const ulonglong2 *>(s_key)[k], wn, st, out_idx,
                                               out_key, pos, &bc, cls);
                }
            }
            __syncthreads();
            const uint32_t slot = wait ? atomicAdd(&s_here, 1u) : 0u;
            __syncthreads();
            if (tid == 0 && s_here) s_base = atomicAdd(count_b, s_here);
            __syncthreads();
            if (wait) list_b[s_base + slot] = k;
        }
        flush_counts(&bc, ctr);
        __threadfence();
        __syncthreads();
        if (tid == 0) s_last = atomicAdd(arrived, 1u) == gridDim.x - 1;
        __syncthreads();
        if (!s_last) return;
        __threadfence();
        if (tid == 0) {
            *arrived = 0;
            bc = BlockCounts{0, 0, 0, 0};
            const uint32_t nn = min(atomicAdd(count_b, 0u), ell);
            if (nn >= first) atomicOr(err, ERR_INTERNAL);  // the smallest undecided switch always decides
            s_n = nn >= first ? 0 : nn;
            atomicAdd(&ctr->rounds, (unsigned long long)((first + kChainFinish - 1) / kChainFinish));
            if (round_limit && ++charged >= round_limit && s_n > 0) {
                atomicOr(err, ERR_ROUNDS);
                s_n = 0;
            }
        }
        __syncthreads();
        cur = list_b;
        nxt = list_a;
        ccur = count_b;
        cnxt = count_a;
    }
    if (nbslot) {  // fold the per-block counts of the emit and first round (no list round did; eight loads in flight)
        constexpr uint32_t kFold = 8;
        uint4 acc = make_uint4(0, 0, 0, 0);
        for (uint32_t q0 = tid; q0 < nbslot; q0 += kFold * kChainFinish) {
            uint4 v[kFold];
#pragma unroll
            for (uint32_t j = 0; j < kFold; ++j) {
                const uint32_t q = q0 + j * kChainFinish;
                v[j] = q < nbslot ? bslot[q] : make_uint4(0, 0, 0, 0);
            }
#pragma unroll
            for (uint32_t j = 0; j < kFold; ++j) {
                acc.x += v[j].x;
                acc.y += v[j].y;
                acc.z += v[j].z;
                acc.w += v[j].w;
            }
        }
        if (acc.x) atomicAdd(&bc.legal, acc.x);
        if (acc.y) atomicAdd(&bc.loop, acc.y);
        if (acc.z) atomicAdd(&bc.exists, acc.z);
        if (acc.w) atomicAdd(&bc.pl, acc.w);
    }
    uint32_t n = s_n, here = 0;
    __shared__ __align__(16) uint32_t s_chunks[kSweepWords];  // the sweep's chunk marks; statuses before it
    if (n > 0 && n <= kFinishList && ell <= kFinishSwitches) {
        // few enough switches: statuses and list in LDS.  A pass from memory is
        // a chain of eight dependent loads and two atomics on the list counter.
        __shared__ uint32_t l_list[2][kFinishList], l_n;
        uint8_t *ls = reinterpret_cast<uint8_t *>(s_chunks);
        for (uint32_t w = tid; 16 * w < ell; w += kChainFinish)  // (st has 64 bytes to spare)
            reinterpret_cast<uint4 *>(s_chunks)[w] = reinterpret_cast<const uint4 *>(st)[w];
        for (uint32_t q = tid; q < n; q += kChainFinish) l_list[0][q] = cur[q];
        for (; n > 0 && here < kSweepAfter; ++here) {
            const uint32_t *in = l_list[here & 1u];
            uint32_t *out = l_list[(here + 1) & 1u];
            if (tid == 0) l_n = 0;
            __syncthreads();
            const uint32_t trips = (n + kChainFinish - 1) / kChainFinish;
            for (uint32_t r = 0; r < trips; ++r) {
                const uint32_t q = r * kChainFinish + tid;
                const uint32_t k = q < n ? in[q] : 0u;
                const bool todo = q < n && k < ell && (ls[k] & kStOutcome) == ST_UNDECIDED;
                uint4 recs = make_uint4(0, 0, 0, 0);
                int v = V_WAIT;
                if (todo) {
                    recs = target_records(info, k, ls[k]);
                    v = judge_switch_chain(k, recs, info, wn, LdsStatus{ls});
                }
                __syncthreads();  // (as below)
                if (todo) {
                    if (commit_switch_chain(v, k, recs, reinterpret_cast<const uint2 *>(s_idx)[k],
                                            reinterpret_cast<const ulonglong2 *>(s_key)[k], wn, st, out_idx, out_key,
                                            pos, &bc, cls))
                        out[atomicAdd(&l_n, 1u)] = k;
                    else
                        ls[k] = v == V_OK ? ST_LEGAL : ST_EXISTS;
                }
                __syncthreads();
            }
            if (tid == 0) {
                const uint32_t nn = l_n;
                if (nn >= n) atomicOr(err, ERR_INTERNAL);  // the smallest undecided switch always decides
                s_n = nn >= n ? 0 : nn;
                atomicAdd(&ctr->rounds, (unsigned long long)trips);
                if (round_limit && ++charged >= round_limit && s_n > 0) {
                    atomicOr(err, ERR_ROUNDS);
                    s_n = 0;
                }
            }
            __syncthreads();
            n = s_n;
        }
        for (uint32_t q = tid; q < n; q += kChainFinish) cur[q] = l_list[here & 1u][q];  // (the sweep's)
        __syncthreads();
    }
    for (; n > 0 && here < kSweepAfter; ++here) {
        if (tid == 0) *cnxt = 0;
        __threadfence();
        __syncthreads();
        const uint32_t trips = (n + kChainFinish - 1) / kChainFinish;
        for (uint32_t r = 0; r < trips; ++r) {
            const uint32_t q = r * kChainFinish + tid;
            bool wait = false, todo = false;
            uint32_t k = 0;
            uint4 recs = make_uint4(0, 0, 0, 0);
            int v = V_WAIT;
            if (q < n) {
                k = cur[q];
                const uint8_t sk = k < ell ? st[k] : (uint8_t)ST_LEGAL;
                todo = (sk & kStOutcome) == ST_UNDECIDED;
                if (todo) {
                    recs = target_records(info, k, sk);
                    v = judge_switch_chain(k, recs, info, wn, GroupStatus{st});
                }
            }
            // a pass judges by what earlier passes decided, so its round count
            // does not depend on which wave runs first
            __syncthreads();
            if (todo)
                wait = commit_switch_chain(v, k, recs, reinterpret_cast<const uint2 *>(s_idx)[k],
                                           reinterpret_cast<const ulonglong2 *>(s_key)[k], wn, st, out_idx, out_key,
                                           pos, &bc, cls);
            __syncthreads();
            append_undecided(wait, k, nxt, cnxt);
        }
        __threadfence();
        __syncthreads();
        if (tid == 0) {
            const uint32_t nn = min(*cnxt, ell);
            if (nn >= n) atomicOr(err, ERR_INTERNAL);  // the smallest undecided switch always decides
            s_n = nn >= n ? 0 : nn;
            atomicAdd(&ctr->rounds, (unsigned long long)trips);
            if (round_limit && ++charged >= round_limit && s_n > 0) {
                atomicOr(err, ERR_ROUNDS);
                s_n = 0;
            }
        }
        __syncthreads();
        n = s_n;
        uint32_t *tl = cur;
        cur = nxt;
        nxt = tl;
        uint32_t *tc = ccur;
        ccur = cnxt;
        cnxt = tc;
    }
    if (n > 0) {
        __shared__ uint32_t s_wait, s_done, s_stop;
        const uint32_t nwords = ((ell + kSweepChunk - 1) / kSweepChunk + 31) / 32;
        for (uint32_t w = tid; w < nwords; w += kChainFinish) s_chunks[w] = 0;
        if (tid == 0) s_stop = 0;
        __syncthreads();
        for (uint32_t q = tid; q < n; q += kChainFinish) {
            const uint32_t k = cur[q];
            if (k < ell) atomicOr(&s_chunks[(k / kSweepChunk) >> 5], 1u << ((k / kSweepChunk) & 31));
        }
        __syncthreads();
        unsigned long long added = 0;
        for (uint32_t w = 0; w < nwords && !s_stop; ++w) {
            uint32_t bits = s_chunks[w];
            while (bits && !s_stop) {
                const uint32_t c = w * 32 + (uint32_t)(__ffs(bits) - 1);
                bits &= bits - 1;
                const uint32_t kb = c * kSweepChunk, ke = min(kb + kSweepChunk, ell);
                constexpr uint32_t kPer = kSweepChunk / kChainFinish;
                uint2 from[kPer];  // resume points of the two predecessor walks
#pragma unroll
                for (uint32_t j = 0; j < kPer; ++j) from[j] = make_uint2(kNoPred, kNoPred);
                for (;;) {
                    if (tid == 0) {
                        s_wait = 0;
                        s_done = 0;
                    }
                    __syncthreads();
                    uint32_t waits = 0, dones = 0;
#pragma unroll
                    for (uint32_t j = 0; j < kPer; ++j) {
                        const uint32_t k = kb + tid + j * kChainFinish;
                        if (k >= ke || load_status<true>(st, k) != ST_UNDECIDED) continue;
                        const uint4 recs = target_records(info, k, st[k]);
                        if (commit_switch_chain(judge_switch_chain(k, recs, info, wn, GroupStatus{st}, &from[j]), k, recs,
                                                reinterpret_cast<const uint2 *>(s_idx)[k],
                                                reinterpret_cast<const ulonglong2 *>(s_key)[k], wn, st, out_idx,
                                                out_key, pos, &bc, cls))
                            ++waits;
                        else
                            ++dones;
                    }
                    if (waits) atomicAdd(&s_wait, waits);
                    if (dones) atomicAdd(&s_done, dones);
                    __syncthreads();
                    const uint32_t W = s_wait, D = s_done;
                    if (tid == 0) {
                        ++added;
                        // the smallest undecided switch of the chunk always decides
                        if (W > 0 && D == 0) {
                            atomicOr(err, ERR_INTERNAL);
                            s_stop = 1;
                        } else if (W > 0 && round_limit && charged + added >= round_limit) {
                            atomicOr(err, ERR_ROUNDS);
                            s_stop = 1;
                        }
                    }
                    __syncthreads();
                    if (W == 0 || s_stop) break;
                }
            }
        }
        if (tid == 0 && added) atomicAdd(&ctr->rounds, added);
    }
    flush_counts(&bc, ctr);
}

}  // namespace gesmc
