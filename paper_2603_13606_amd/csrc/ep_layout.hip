// Routing layout kernels: per-expert / per-destination-rank counts, prefix
// offsets and the stable slot map (Sec. IV-A index algebra; Sec. IV-C "Token
// Count"; the slot rule of Sec. IV-B made deterministic).
//
// The slot of entry i = t*K + k is the number of entries j < i naming the same
// expert: a stable counting sort.  No atomic decides an order anywhere (atomics
// only add counts or set bits), so the output is a pure function of the input.
//
// The flattened entry list is cut into chunks, one per workgroup of up
// to 16 wavefronts, and every chunk into wave-chunks of 64*passes consecutive entries,
// one per wavefront.  ONE launch (Sec. IV-C "Token Count": the count runs next to the
// send, not as a phase of its own):
//   rows        a pass of a wave is a row of 64 entries; per row and bin -- E experts, masked,
//               invalid, R destination ranks -- a 64-bit word of LDS gets the bits of the lanes
//               that hold the bin: the lower bits of an entry's word are its rank in the row.
//               (Large inputs and tables: a histogram per wave, and ballots, see layout_chunk.)
//   publish     one thread per bin sums the row counts of the chunk and stores
//               the sum, tagged with the number of this launch, to global memory;
//   look across one thread per bin reads that bin's sums of ALL chunks (it waits, a
//               bounded number of polls, until each carries this launch's tag): entries
//               in earlier chunks (the prefix) and in all chunks (the totals, hence
//               the expert offsets).  Only sums of counts cross between workgroups,
//               so the result does not depend on which chunk is published first;
//   scan        one exclusive scan of the totals over all bins by one wavefront, and one per
//               block of the walk list by others;
//   emit        slot = prefix of earlier chunks + in-chunk rank, the destination row,
//               the expert-sorted entry list and the walk list.
// The chunks wait for each other, so all of them must be resident at the same time:
// there are at most 256 of them (64 when entries go by rows) and one for the tables, the part has 256
// compute units, they are the lowest workgroup ids of the launch, and every
// wait gives up after a fixed number of polls (status bit, never a hang).
// The work is latency bound (a chain of dependent LDS and global round trips per
// wave), so every phase issues all of its global loads before it waits for any of
// them and the workgroup barriers order LDS traffic only.
#include "ep_internal.h"
#include "ep_fp8.h"

#include <algorithm>

namespace ep {
namespace {

constexpr int PU = 2;  // passes whose loads are issued together and whose entries stay in registers

// Workgroup barrier that orders LDS traffic only: the LDS operations of this wave have
// completed when it arrives (s_waitcnt lgkmcnt(0)), and the compiler moves no memory access
// across it, but global loads and stores issued before it stay in flight (a
// __syncthreads(), or a workgroup-scope fence, would wait for them: a round trip to
// memory at every barrier of a latency-bound kernel).  Global memory written by one wave
// is never read by another wave of the workgroup in these kernels.
__device__ __forceinline__ void lds_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

__device__ __forceinline__ int lane_id() {
    return __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
}

// Data-parallel-primitive controls of the cross-lane moves below (CDNA ISA, DPP_CTRL).
constexpr int kDppRowShr = 0x110;      // + n: lane i reads lane i-n of its row of 16
constexpr int kDppWaveShr1 = 0x138;    // lane i reads lane i-1 of the wavefront
constexpr int kDppRowBcast15 = 0x142;  // lane 15 of each row to every lane of the next row
constexpr int kDppRowBcast31 = 0x143;  // lane 31 to every lane of rows 2 and 3

// The value of the lane below; lane 0 gets `fill`.
__device__ __forceinline__ int lane_below(int v, int fill) {
    return __builtin_amdgcn_update_dpp(fill, v, kDppWaveShr1, 0xf, 0xf, false);
}

// Inclusive prefix sum over the 64 lanes: within rows of 16 by shifted adds, then the
// row sums are carried into the rows above.  A lane whose source lies outside its row
// (or whose row is masked out) adds 0.
__device__ __forceinline__ int wave_inclusive_scan(int v) {
    v += __builtin_amdgcn_update_dpp(0, v, kDppRowShr + 1, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, kDppRowShr + 2, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, kDppRowShr + 4, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, kDppRowShr + 8, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, kDppRowBcast15, 0xa, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, kDppRowBcast31, 0xc, 0xf, false);
    return v;
}

__device__ __forceinline__ int wave_max(int v) {
    for (int off = kWave / 2; off > 0; off >>= 1) v = max(v, __shfl_xor(v, off, kWave));
    return v;
}

// Lanes (among those with valid == true) that hold the same key as this lane.
__device__ __forceinline__ uint64_t match_key(int key, bool valid, int nbits) {
    uint64_t peers = __ballot(valid);
    for (int b = 0; b < nbits; ++b) {
        const bool bit = (key >> b) & 1;
        const uint64_t bal = __ballot(valid && bit);
        peers &= bit ? bal : ~bal;
    }
    return valid ? peers : 0ull;
}

// Token index of flattened entry i (i / K), with a shift when K is a power of two.
__device__ __forceinline__ int token_of(const LayoutArgs& a, int i) {
    return a.K_shift >= 0 ? (i >> a.K_shift) : (int)(__umulhi((uint32_t)i, a.K_magic) >> (31 - __builtin_clz(a.K)));
}

__device__ __forceinline__ int owner_of(const LayoutArgs& a, int e) {
    return a.L_shift >= 0 ? (e >> a.L_shift) : (int)(__umulhi((uint32_t)e, a.L_magic) >> (31 - __builtin_clz(a.L)));
}

struct Entry {
    int i;         // flattened index, or -1 beyond the input
    int t, k, e, d;
    bool ok;       // names an expert that gets a row
    bool masked;   // id == -1
    bool invalid;  // any other id outside [0, E)
    bool lead;     // first k of its token that names destination rank d
};

// LDS carve-up shared by the kernels: the per-wave or per-pass tables, then
struct Lds {
    int32_t *wh;      // layout_chunk: [nw+1][W] per-wave histograms, later "entries of the bin in the earlier waves of the
                      //     chunk"; row nw stands in for the rows a smaller workgroup does not have, so that
                      //     sweeps over kLayoutWavesPerBlock rows need no branch: it reads as 0 and is never used
    int32_t *tot;     // [W] totals over the whole input
    int32_t *S;       // [W] exclusive scan of tot over all bins.  S[e], e <= E, is the first position of expert
                      //     e in the expert-sorted list (S[E] = routed entries), and its first row in the
                      //     concatenated layout unless the caller gave the first rows; the rank bins are the
                      //     last R bins: for compact staging windows rank_offset[d] = S[E+2+d] - S[E+2]
    int32_t *before;  // [W] entries of each bin in earlier chunks (several chunks only)
    int32_t *flag;    // [1] set when a thread of the workgroup gave up waiting for another chunk
    // with a walk list only
    int32_t *first;   // [kLayoutWavesPerBlock] where each block of the chunk starts in the list
    int32_t *bstart;  // [E] entries of the expert before the block of this chunk (before the chunk, if it holds several blocks)
    int32_t *bcount;  // [E] entries of the expert in the block (in the chunk)
    int32_t *walk;    // [blocks of the chunk][E] place of an entry in the list, less its slot and the block's start
};

__device__ __forceinline__ Lds carve_lds(int32_t* base, const LayoutArgs& a, int tables) {
    Lds l;
    l.wh = base;
    l.tot = l.wh + tables;
    l.S = l.tot + a.W;
    l.before = l.S + a.W;
    l.flag = l.before + a.W;
    l.first = l.flag + 1;
    l.bstart = l.first + kLayoutWavesPerBlock;
    l.bcount = l.bstart + a.E;
    l.walk = l.bcount + a.E;
    return l;
}

// Row-by-row layouts (layout_rows): a workgroup of 16 / passes wavefronts has 16 rows of 64 entries, and LDS holds one 64-bit
// word per row and bin.  Rows start on 16-byte boundaries.
constexpr int kRows = 16;
__host__ __device__ constexpr int row_words(int W) { return (W + 1) & ~1; }

// The low half of such a word, which holds a count in place of the bits later on: the compiler must not take accesses to the half for
// independent of those to the word.
typedef int32_t __attribute__((may_alias)) half_word;

constexpr int lds_ints(int W, int nw) { return (nw + 1) * W + 3 * W + 1; }
constexpr int rows_lds_ints(int W) { return 2 * kRows * row_words(W) + 3 * W + 1; }
// What the walk list adds, with blocks of `group` wave-chunks.
constexpr int walk_lds_ints(int E, int nw, int group) { return kLayoutWavesPerBlock + (2 + (nw > group ? nw / group : 1)) * E; }

// How a layout is cut into workgroups, and what LDS they take.
struct LayoutCut {
    bool rows;    // layout_rows
    int waves;    // wavefronts per workgroup
    size_t lds;   // bytes
};

// Of layout_chunk: half of a compute unit's.  With 64 KiB the tables of the walk list took the workgroups of 1024 experts from 8 waves
// to 4 (on 64 ranks) and 2 (on 128; layout of 8800 entries 30.3 us, now 17.0; 1024 ranks 109 and 47, without the list 92 and 41).
constexpr size_t kLdsLimit = 80 * 1024;
constexpr size_t kLdsUnit = 160 * 1024;   // of a compute unit: what a workgroup of layout_rows may take

// group: wave-chunks per block of the walk list, 0 without one.  A wave keeps its entries in registers for up to PU passes;
// the tables of 1024 experts on up to 128 ranks fit.
LayoutCut cut_layout(int E, int R, int passes, int group) {
    const int W = E + 2 + R;
    LayoutCut c;
    c.rows = true;
    c.waves = kRows / std::min(passes, PU);
    c.lds = sizeof(int32_t) * (size_t)(rows_lds_ints(W) + (group ? walk_lds_ints(E, c.waves, group) : 0));
    if (passes <= PU && c.lds <= kLdsUnit) return c;
    c.rows = false;
    for (c.waves = kLayoutWavesPerBlock;; c.waves >>= 1) {  // fewer waves when the bin tables are large
        c.lds = sizeof(int32_t) * (size_t)(lds_ints(W, c.waves) + (group ? walk_lds_ints(E, c.waves, group) : 0));
        if (c.lds <= kLdsLimit || c.waves == 1) return c;
    }
}

// Marks the entries that are the first of their token to name their destination
// rank.  The entries of a token sit in consecutive lanes, so lane l compares its
// rank with the ranks held by lanes l-1 .. l-k (one shift of the wave per step); only
// when a token began before lane 0 are its earlier entries read from memory.
// Must be called by all 64 lanes.
//
// With K a power of two up to 16 tokens do not straddle the rows of 16 lanes: key ^ (key of lane l-j), j < K, by shifts
// inside the row, is 0 for an earlier entry of the same token and rank (two instructions per step where the
// general walk takes five).  Lanes shifted in from outside the row read 0, which is no key.
template <int K>
__device__ __forceinline__ uint32_t closest_key(uint32_t key) {
    uint32_t m = ~0u;
#define EP_STEP(j) if (j < K) m = min(m, key ^ (uint32_t)__builtin_amdgcn_update_dpp(0, (int)key, kDppRowShr + j, 0xf, 0xf, true));
    EP_STEP(1) EP_STEP(2) EP_STEP(3) EP_STEP(4) EP_STEP(5) EP_STEP(6) EP_STEP(7) EP_STEP(8)
    EP_STEP(9) EP_STEP(10) EP_STEP(11) EP_STEP(12) EP_STEP(13) EP_STEP(14) EP_STEP(15)
#undef EP_STEP
    return m;
}

__device__ __forceinline__ void mark_leaders(const LayoutArgs& a, Entry& en, int lane) {
    if (a.K_shift >= 0 && a.K_shift <= 4) {  // uniform
        // token of the row of lanes (at most 16), rank; no two lanes without a rank share a key
        const uint32_t key = 0x40000000u | ((uint32_t)(lane >> a.K_shift) << 16) | (uint32_t)(en.ok ? en.d : 0x8000 + lane);
        uint32_t m = ~0u;
        if (a.K_shift == 1) m = closest_key<2>(key);
        else if (a.K_shift == 2) m = closest_key<4>(key);
        else if (a.K_shift == 3) m = closest_key<8>(key);
        else if (a.K_shift == 4) m = closest_key<16>(key);
        en.lead = en.ok && m != 0;
        return;
    }
    const int dkey = en.ok ? en.d : -1;
    bool lead = en.ok;
    int prev = dkey;
    for (int j = 1; j < a.K; ++j) {
        prev = lane_below(prev, -2);  // the key of lane l-j; -2 (no key) below lane 0
        if (j <= en.k && prev == dkey) lead = false;
    }
    if (en.ok && en.k > lane) {  // entries of this token that precede lane 0 of this pass
        const int32_t* row = a.topk + (int64_t)en.t * a.topk_stride;
        for (int k2 = 0; k2 < en.k - lane; ++k2) {
            const int e2 = row[k2];
            if ((unsigned)e2 < (unsigned)a.E && owner_of(a, e2) == en.d) lead = false;
        }
    }
    en.lead = lead;
}

// Issues the global loads of the ids of passes p0 .. p0+N-1 of wave-chunk wc
// (nothing waits on them here).
template <int N>
__device__ __forceinline__ void issue_group(const LayoutArgs& a, int wc, int p0, int lane, int (&raw)[N]) {
#pragma unroll
    for (int j = 0; j < N; ++j) {
        const int p = p0 + j;
        const int i = (wc * a.passes + p) * kWave + lane;
        raw[j] = 0;
        if (p < a.passes && i < a.n) {
            const int t = token_of(a, i), k = i - t * a.K;
            raw[j] = a.topk[(int64_t)t * a.topk_stride + k];
        }
    }
}

// Classifies the ids loaded by issue_group.  Must be called by all 64 lanes.
template <int N>
__device__ __forceinline__ void classify_group(const LayoutArgs& a, int wc, int p0, int lane,
                                               const int (&raw)[N], Entry (&en)[N]) {
#pragma unroll
    for (int j = 0; j < N; ++j) {
        Entry& x = en[j];
        const int p = p0 + j;
        const int i = (wc * a.passes + p) * kWave + lane;
        const bool in = p < a.passes && i < a.n;
        x.i = in ? i : -1;
        x.t = in ? token_of(a, i) : 0;
        x.k = in ? i - x.t * a.K : 0;
        const int e = raw[j];
        const bool inrange = (unsigned)e < (unsigned)a.E;
        x.d = inrange ? owner_of(a, e) : 0;
        x.ok = in && inrange;
        x.masked = in && e == -1;
        x.invalid = in && !inrange && e != -1;
        if (p < a.passes) mark_leaders(a, x, lane);  // wave-uniform condition
        else x.lead = false;
        x.e = x.ok ? e : 0;
    }
}

__device__ __forceinline__ void load_group(const LayoutArgs& a, int wc, int p0, int lane, Entry (&en)[PU]) {
    int raw[PU];
    issue_group(a, wc, p0, lane, raw);
    classify_group(a, wc, p0, lane, raw, en);
}

// Histogram of a loaded group into h[0..W) with LDS atomics (integer adds: the
// result does not depend on their order).
__device__ __forceinline__ void hist_group(const LayoutArgs& a, const Entry (&en)[PU], int32_t* h) {
#pragma unroll
    for (int j = 0; j < PU; ++j) {
        if (en[j].ok) atomicAdd(&h[en[j].e], 1);
        if (en[j].masked) atomicAdd(&h[a.E], 1);
        if (en[j].invalid) atomicAdd(&h[a.E + 1], 1);
        if (en[j].lead) atomicAdd(&h[a.E + 2 + en[j].d], 1);
    }
}

// First row of expert e in the receiver's tensor.
__device__ __forceinline__ int first_row(const LayoutArgs& a, const Lds& l, int e) {
    if (a.padded) return e * a.C;
    return a.expert_base ? a.expert_base[e] : l.S[e];
}

// First staging slot of destination rank d (d == R: one past the last).
__device__ __forceinline__ int first_slot(const LayoutArgs& a, const Lds& l, int d) {
    if (a.padded) return d * a.C_rank;
    const int end = d < a.R ? l.S[a.E + 2 + d] : l.S[a.W - 1] + l.tot[a.W - 1];
    return end - l.S[a.E + 2];
}

// p[i] = v for arrays of less than 2^30 words: a 32-bit offset goes into the store instruction, a 64-bit index
// takes four more to add up.
__device__ __forceinline__ void put(int32_t* p, int i, int32_t v) { *(int32_t*)((uint8_t*)p + ((uint32_t)i << 2)) = v; }

// Writes what the layout records for one entry, given its rank inside the chunk among the
// entries of its expert and (for a leader) among the tokens of its destination rank; the
// entries of earlier chunks (l.before) turn the ranks into slots.
// walk: the places of the wave's block, walk_base: where the block starts in the walk list.
template <bool MULTI, bool WALK>
__device__ __forceinline__ void emit_entry(const LayoutArgs& a, const Entry& x, int slot, int rslot, const Lds& l,
                                           const int32_t* walk, int walk_base) {
    int row = -1, rrow = -1;
    if (x.ok) {
        if (MULTI) slot += l.before[x.e];
        if (a.padded) row = slot < a.C ? x.e * a.C + slot : -1;
        else row = first_row(a, l, x.e) + slot;
        if (a.sorted_token) {
            const int pos = l.S[x.e] + slot;
            put(a.sorted_token, pos, x.t);
            put(a.sorted_k, pos, x.k);
            put(a.sorted_row, pos, row);
        }
        if (WALK && row >= 0) a.walk[walk_base + walk[x.e] + slot] = make_int2(x.t, row);
    }
    if (x.lead) rrow = first_slot(a, l, x.d) + (MULTI ? l.before[a.E + 2 + x.d] : 0) + rslot;
    if (x.i >= 0) {
        if (a.slot) put(a.slot, x.i, slot);
        put(a.dst_row, x.i, row);
        if (a.rank_row) put(a.rank_row, x.i, rrow);
        if (a.entry_rank) put(a.entry_rank, x.i, x.ok ? x.d : -1);
    }
}

// Where an entry stands among the entries of its wave that hold the same key, for the expert
// key and (for a leader) the destination-rank key: entries below it and entries in all.
struct InWave {
    int below, all;      // among the lanes naming the same expert
    int below_r, all_r;  // among the leader lanes naming the same destination rank
};

// The in-wave standing of a loaded group: ballots only, no memory.  Must be called by all
// 64 lanes.
__device__ __forceinline__ void rank_group(const LayoutArgs& a, const Entry (&en)[PU], int p0, int lane, InWave (&iw)[PU]) {
    const uint64_t lt = (1ull << lane) - 1ull;
#pragma unroll
    for (int j = 0; j < PU; ++j) {
        iw[j] = InWave{0, 0, 0, 0};
        if (p0 + j >= a.passes) continue;  // wave-uniform
        const uint64_t peers = match_key(en[j].e, en[j].ok, a.bits_e);
        const uint64_t peers_r = match_key(en[j].d, en[j].lead, a.bits_r);
        iw[j] = InWave{(int)__popcll(peers & lt), (int)__popcll(peers), (int)__popcll(peers_r & lt), (int)__popcll(peers_r)};
    }
}

// Ranks of a loaded group inside its chunk: h holds, per bin, the number of entries of that
// bin in the earlier waves of the chunk and in the earlier groups of this wave; it is
// advanced as the group is walked.  LDS accesses of one wavefront are performed in program
// order, and the wave barriers keep the compiler from moving them across each other.
// Must be called by all 64 lanes.
__device__ __forceinline__ void place_group(const LayoutArgs& a, const Entry (&en)[PU], const InWave (&iw)[PU], int p0,
                                            int32_t* h, int (&slot)[PU], int (&rslot)[PU]) {
#pragma unroll
    for (int j = 0; j < PU; ++j) {
        slot[j] = -1;
        rslot[j] = -1;
        if (p0 + j >= a.passes) continue;  // wave-uniform
        const Entry& x = en[j];
        if (x.ok) slot[j] = h[x.e] + iw[j].below;
        if (x.lead) rslot[j] = h[a.E + 2 + x.d] + iw[j].below_r;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
        __builtin_amdgcn_wave_barrier();
        if (x.ok && iw[j].below == 0) h[x.e] += iw[j].all;
        if (x.lead && iw[j].below_r == 0) h[a.E + 2 + x.d] += iw[j].all_r;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
        __builtin_amdgcn_wave_barrier();
    }
}

template <bool MULTI, bool WALK, int N>
__device__ __forceinline__ void emit_group(const LayoutArgs& a, const Entry (&en)[N], int p0, const int (&slot)[N],
                                           const int (&rslot)[N], const Lds& l, const int32_t* walk, int walk_base) {
#pragma unroll
    for (int j = 0; j < N; ++j)  // wave-uniform condition
        if (p0 + j < a.passes) emit_entry<MULTI, WALK>(a, en[j], slot[j], rslot[j], l, walk, walk_base);
}

// The scans over the bins are done by one wavefront each, while the others wait: done by all 16, every wave adds up the
// sums of all waves, and 16 waves share the four instruction streams of a compute unit (0.3 us of the layout).
constexpr int kScanRows = 4;  // rows of 64 bins whose loads are issued together

// Exclusive scan of the totals tot[0..W) over all bins into S.
__device__ void scan_totals(const LayoutArgs& a, const Lds& l, int lane) {
    int carry = 0;
    for (int c0 = 0; c0 < a.W; c0 += kScanRows * kWave) {
        int v[kScanRows];
#pragma unroll
        for (int r = 0; r < kScanRows; ++r) {
            const int c = c0 + r * kWave + lane;
            v[r] = c < a.W ? l.tot[c] : 0;
        }
#pragma unroll
        for (int r = 0; r < kScanRows; ++r) {
            const int c = c0 + r * kWave + lane;
            const int inc = wave_inclusive_scan(v[r]);
            if (c < a.W) l.S[c] = carry + inc - v[r];
            carry += __builtin_amdgcn_readlane(inc, kWave - 1);
        }
    }
}

// The places of block sb of this chunk (the only one, or one of several) in the walk list:
// l.walk[sb][e] + slot is the place, counted from the start of the block, of the entry of expert e with that slot;
// l.first[sb] is where the block starts: the rows of all earlier blocks.  A row count of an expert is its entry count
// cut at the capacity.
// before0: of block 0's first wave, the entries of every bin in the waves of the chunk before it, a word every `step`,
// then the next waves' at `pitch`.
__device__ void scan_walk(const LayoutArgs& a, const Lds& l, const half_word* before0, int pitch, int step, int sb, int nsub, int lane) {
    const int E = a.E, cap = a.padded ? a.C : 0x7fffffff;
    const half_word* lo = before0 + sb * a.walk_group * pitch;
    const half_word* hi = lo + a.walk_group * pitch;
    int base = 0, carry = 0;
    for (int c0 = 0; c0 < E; c0 += kScanRows * kWave) {
        int start[kScanRows], rows[kScanRows];
#pragma unroll
        for (int r = 0; r < kScanRows; ++r) {
            const int c = c0 + r * kWave + lane;
            start[r] = rows[r] = 0;
            if (c < E) {
                const int bstart = l.bstart[c];
                start[r] = bstart + (sb == 0 ? 0 : lo[c * step]);
                rows[r] = bstart + (sb == nsub - 1 ? l.bcount[c] : hi[c * step]);
            }
        }
#pragma unroll
        for (int r = 0; r < kScanRows; ++r) {
            const int c = c0 + r * kWave + lane;
            const int before = min(start[r], cap), n = min(rows[r], cap) - before;
            const int inc = wave_inclusive_scan(n);
            base += __builtin_amdgcn_readlane(wave_inclusive_scan(before), kWave - 1);
            if (c < E) l.walk[sb * E + c] = carry + inc - n - start[r];
            carry += __builtin_amdgcn_readlane(inc, kWave - 1);
        }
    }
    if (lane == 0) l.first[sb] = base;
}

// The per-expert / per-rank arrays and the totals block (all but the status word) in
// global memory, from tot and S in LDS.  By every thread of one workgroup: the experts, the ranks and the sums
// over all experts fall to different waves, which have their share of other work too (by wave 0 alone, one after the
// other, this was the last 1.4 us of a small layout).  STATUS: the status word too (there is one chunk; the caller of a
// fused launch says how many rows its output takes).
// kept: rows of padded windows in use (in the last wave; see sum_kept).
template <bool STATUS>
__device__ __forceinline__ void write_tables(const LayoutArgs& a, const Lds& l, int tid, int lane, int w, int kept) {
    const int32_t* tot = l.tot;
    const int32_t* S = l.S;
    const int E = a.E, R = a.R, threads = blockDim.x;  // a power of two
    for (int e = (tid + threads / 2) & (threads - 1); e < E; e += threads) {
        const int v = tot[e];
        const int kept = a.padded ? min(v, a.C) : v;
        a.expert_count[e] = v;
        a.expert_kept[e] = kept;
        if (a.recv_count) a.recv_count[e] = kept;
        a.expert_offset[e] = first_row(a, l, e);
    }
    if (a.rank_pair_count) {
        for (int d = (tid + threads / 4) & (threads - 1); d <= R; d += threads) {
            if (d < R) {
                a.rank_pair_count[d] = S[(d + 1) * a.L] - S[d * a.L];
                a.rank_token_count[d] = tot[E + 2 + d];
            }
            a.rank_offset[d] = first_slot(a, l, d);
        }
    }
    if (w != threads / kWave - 1) return;
    const int total_e = S[E];
    int rend = 0;
    if (!a.padded) kept = total_e;
    if (!a.padded && a.expert_base) {
        for (int e = lane; e < E; e += kWave)
            if (tot[e] > 0) rend = max(rend, a.expert_base[e] + tot[e]);
        rend = wave_max(rend);
    }
    const int rows_end = a.padded ? E * a.C : (a.expert_base ? rend : total_e);
    if (lane == 0) {
        a.expert_offset[E] = rows_end;
        a.totals[TOT_KEPT] = kept;
        a.totals[TOT_DROPPED] = total_e - kept;
        a.totals[TOT_MASKED] = tot[E];
        a.totals[TOT_INVALID] = tot[E + 1];
        a.totals[TOT_SORTED] = total_e;
        a.totals[TOT_MSGS] = S[a.W - 1] + tot[a.W - 1] - S[E + 2];  // the rank bins are the last R bins
        a.totals[TOT_ROWS_END] = rows_end;
        if (a.drop_hint) *a.drop_hint = (int64_t)kept | ((int64_t)(total_e - kept) << 32);
        if (STATUS)
            a.totals[TOT_STATUS] = (tot[E + 1] ? STATUS_INVALID_IDS : 0) | (kept < total_e ? STATUS_CAPACITY_DROP : 0) |
                                   (!a.padded && a.rows_cap >= 0 && rows_end > a.rows_cap ? STATUS_OUTPUT_OVERFLOW : 0);
    }
}

// One past the highest destination row of the concatenated layout.  One wavefront; must be called
// by all 64 lanes.
__device__ int last_row_end(const LayoutArgs& a, const Lds& l, int lane) {
    if (!a.expert_base) return l.S[a.E];
    int end = 0;
    for (int e = lane; e < a.E; e += kWave)
        if (l.tot[e] > 0) end = max(end, a.expert_base[e] + l.tot[e]);
    return wave_max(end);
}

// The status word of the totals block.  One wavefront; must be called by all 64 lanes.
__device__ void write_status(const LayoutArgs& a, const Lds& l, int lane, int extra_status) {
    int dropped = 0;
    if (a.padded)
        for (int e = lane; e < a.E; e += kWave) dropped |= l.tot[e] > a.C ? 1 : 0;
    const bool any_dropped = __ballot(dropped != 0) != 0;
    if (lane == 0)
        a.totals[TOT_STATUS] = (l.tot[a.E + 1] ? STATUS_INVALID_IDS : 0) | (any_dropped ? STATUS_CAPACITY_DROP : 0) |
                               extra_status;
}

// Extra workgroups of the layout kernel (blockIdx >= nchunks): read the token rows the
// caller announced, with ordinary cached loads, while the layout workgroups -- a few dozen
// on a part with 256 compute units -- do their latency-bound work.  wb of nwb.  Rows
// [0, warm_rows), 16 bytes per load, four loads of a thread in flight.
constexpr int kWarmUnroll = 4;
__device__ void warm_tokens(const LayoutArgs& a, int wb, int nwb) {
    const uint32_t units = (uint32_t)a.warm_units;
    const uint32_t total = (uint32_t)a.warm_rows * units;  // at most 64 MiB / 16
    const uint32_t stride = (uint32_t)nwb * blockDim.x;
    const bool dense = a.warm_stride == (int64_t)units * 8;  // rows back to back: no division
    uint32_t acc = 0;
    for (uint32_t i0 = (uint32_t)wb * blockDim.x + threadIdx.x; i0 < total; i0 += kWarmUnroll * stride) {
        u32x4 v[kWarmUnroll];
#pragma unroll
        for (int q = 0; q < kWarmUnroll; ++q) {
            const uint32_t i = min(i0 + q * stride, total - 1);  // the tail repeats the last unit
            if (dense) {
                v[q] = *((const u32x4*)a.warm_x + i);
            } else {
                const uint32_t t = i / units;
                v[q] = *((const u32x4*)(a.warm_x + (int64_t)t * a.warm_stride) + (i - t * units));
            }
        }
#pragma unroll
        for (int q = 0; q < kWarmUnroll; ++q) acc ^= v[q][0] ^ v[q][1] ^ v[q][2] ^ v[q][3];
    }
    asm volatile("" ::"v"(acc));  // the loads are the point: keep them
}

constexpr int kLookLimit = 1 << 19;  // rounds of polling after which a thread stops waiting (about a second)
constexpr int kTagShift = 24;        // a published word is (tag << 24) | count: a chunk holds fewer than 2^24 entries
constexpr uint32_t kCountMask = (1u << kTagShift) - 1u;
constexpr uint32_t kTags = 255;      // tags 1 .. 255; 0 is what a cleared word holds

// What a word says to launch `tag`: a chunk that has not published counts nothing.
constexpr uint32_t published(uint32_t word, uint32_t tag) { return word >> kTagShift == tag ? word & kCountMask : 0u; }
static_assert(published((7u << kTagShift) | 300u, 7u) == 300u && published((6u << kTagShift) | 300u, 7u) == 0u &&
              published(0u, 1u) == 0u && published((kTags << kTagShift) | kCountMask, kTags) == kCountMask, "stale words count nothing");

// Loads the words chunks r0 .. r0+HB-1 have published for bin c.  Every lane loads from a
// valid address (rows beyond the last chunk repeat it, their words are ignored later):
// no branch, so all HB loads are in flight together.
template <int HB>
__device__ __forceinline__ void look_across(const LayoutArgs& a, int c, int r0, uint32_t (&v)[HB]) {
    const int last = a.nchunks - 1;
    const uint32_t* row = a.pub + (int64_t)min(r0, last) * a.W;  // wave-uniform: the row pointer steps in scalar registers
#pragma unroll
    for (int j = 0; j < HB; ++j) {
        v[j] = __hip_atomic_load(row + c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        row += r0 + j < last ? a.W : 0;
    }
}

// The extra workgroups for a group that quantises ahead: instead of only reading the token
// rows they quantise them (the FP8 dispatch's format, see ep_fp8.h) into a staging copy, row t
// at quant_out + t * quant_pitch: H bytes of codes, then H/128 float scales.  The quantising
// dispatch that follows copies staged rows in destination order and finds them, like the
// tokens, in the caches.  A lane owns 16 consecutive channels, 8 neighbouring lanes one
// 128-channel group; H is a multiple of 128, so a group never straddles rows and the 8 lanes
// of a group are in or out of range together.  Ordinary cached loads and stores: both the
// tokens and the staged rows are wanted in the cache afterwards.
__device__ void quantize_tokens(const LayoutArgs& a, int wb, int nwb) {
    const uint32_t per_row = (uint32_t)a.warm_units >> 1;   // 32-byte lane items per row (H / 16)
    const uint32_t total = (uint32_t)a.warm_rows * per_row;
    const uint32_t stride = (uint32_t)nwb * blockDim.x;
    const uint32_t H = (uint32_t)a.warm_units * 8;
    for (uint32_t i = (uint32_t)wb * blockDim.x + threadIdx.x; i < total; i += stride) {
        const uint32_t t = i / per_row, u = i - t * per_row;
        const u32x4* src = (const u32x4*)(a.warm_x + (int64_t)t * a.warm_stride) + 2 * u;
        const u32x4 in0 = src[0], in1 = src[1];
        float scale;
        const u32x4 q = quantize16(in0, in1, &scale);
        uint8_t* row = a.quant_out + (int64_t)t * a.quant_pitch;
        *((u32x4*)row + u) = q;
        if ((u & 7u) == 0) *(float*)(row + H + 4 * (u >> 3)) = scale;
    }
}

// Chunk b = wave-chunks [b*wpb, (b+1)*wpb); with several chunks workgroup nchunks writes the
// tables; the workgroups after those read tokens ahead.
// With one chunk nothing is published or awaited.
//
// Cross-workgroup state (only with more than one chunk), all in a.pub / a.ctl:
//   pub[r][c]  one word: (tag << 24) | entries of bin c in chunk r, tag = ctl[0] + 1 of the
//              launch that wrote it; written once per launch with one atomic store, so a
//              reader that sees the tag of its own launch also sees the count;
//   ctl[0]     launches completed on this scratch since pub was last cleared (the
//              generation, 0 .. 254); read at the start, advanced by the workgroup that is
//              last to finish looking across, which clears pub when the tags run out;
//   ctl[1]     workgroups of this launch that have finished looking across, in the low 16
//              bits; a workgroup that gave up waiting also adds 1 << 16.  Back to 0 at the end.
// Tags never repeat between two clearings of pub, and the scratch starts out all zero,
// which no launch uses as a tag.
//
// HB: chunks whose published words a thread loads in one batch (at most 32: bit masks), 0 = there
// is one chunk.  FUSED: the launch also dispatches.  In three steps:
//
// (A) per bin: entries in earlier chunks and in all chunks, into LDS (and of the block of the walk list).  A batch of words is
//     polled as a whole until every word of it carries this launch's tag (rows beyond the last
//     chunk repeat its words, and the chunk's own word is among them: no exceptions to
//     test for).  Which words of a batch count, and which belong to earlier chunks, are
//     wave-uniform bit masks.
template <int HB, bool WALK>
__device__ __forceinline__ void gather_chunks(const LayoutArgs& a, const Lds& l, int b, int waves, uint32_t tag) {
    const int nchunks = a.nchunks, W = a.W, tid = threadIdx.x;
    const int gchunks = WALK ? max(a.walk_group / waves, 1) : 1, g0 = WALK ? b / gchunks * gchunks : 0;  // of its block
    int rounds = 0;  // of this thread, over all its batches
    bool gave_up = false;
    for (int c = tid; c < W; c += blockDim.x) {
        int before = 0, total = 0, bstart = 0, bcount = 0;
        for (int r0 = 0; r0 < nchunks; r0 += HB) {
            uint32_t hv[HB];
            for (;;) {
                look_across(a, c, r0, hv);
                bool all = true;
#pragma unroll
                for (int j = 0; j < HB; ++j) all = all && (hv[j] >> kTagShift) == tag;
                if (all) break;
                if (++rounds >= kLookLimit) {  // a chunk has not published: flag it
                    gave_up = true;
                    break;
                }
                __builtin_amdgcn_s_sleep(1);
            }
            auto up_to = [&](int chunk) {  // the chunks of the batch that come before this one
                const int m = min(max(chunk - r0, 0), HB);
                return m >= 32 ? ~0u : (1u << m) - 1u;
            };
            const uint32_t valid = up_to(nchunks), earlier = up_to(b);
            const uint32_t blk_earlier = WALK ? up_to(g0) : 0u, blk = WALK ? up_to(g0 + gchunks) & ~blk_earlier : 0u;
#pragma unroll
            for (int j = 0; j < HB; ++j) {
                const uint32_t cnt = hv[j] & kCountMask & (0u - ((valid >> j) & 1u));
                total += (int)cnt;
                before += (int)(cnt & (0u - ((earlier >> j) & 1u)));
                if (WALK) bstart += (int)(cnt & (0u - ((blk_earlier >> j) & 1u)));
                if (WALK) bcount += (int)(cnt & (0u - ((blk >> j) & 1u)));
            }
        }
        if (__builtin_expect(gave_up, 0)) {
            // Without all of the counts, what this launch has published so far, word by word: the sums are too small then, never too
            // large, and slots and places of the lists come out below the true ones, inside their arrays.  (The words of
            // an earlier, larger launch would point beyond them.)
            before = total = bstart = bcount = 0;
#pragma unroll 1
            for (int r = 0; r < nchunks; ++r) {
                const int cnt = (int)published(__hip_atomic_load(a.pub + (int64_t)r * W + c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT), tag);
                total += cnt;
                if (r < b) before += cnt;
                if (WALK && r < g0) bstart += cnt;
                if (WALK && r >= g0 && r < g0 + gchunks) bcount += cnt;
            }
        }
        if (WALK && c < a.E) {
            l.bstart[c] = bstart;
            l.bcount[c] = bcount;
        }
        l.tot[c] = total;  // the chunk's own sum is one of the words
        l.before[c] = before;
    }
    if (gave_up) atomicOr(l.flag, 1);
}

constexpr uint32_t kGaveUp = 1u << 16;  // of ctl[1]: the low 16 bits count workgroups, the rest flags a time-out

// (B) with several chunks: thread 0 reports for the workgroup; the value it gets back tells wave 0 whether this
//     workgroup is the last to have looked across (then every chunk is done with pub and ctl,
//     and it may advance the generation) and whether any workgroup gave up waiting.
__device__ __forceinline__ uint32_t report_chunk(const LayoutArgs& a, const Lds& l) {
    uint32_t seen = 0;
    const uint32_t mine = 1u + (*l.flag ? kGaveUp : 0u);
    if (threadIdx.x == 0)
        seen = __hip_atomic_fetch_add(&a.ctl[1], mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + mine;
    return seen;
}

// (C) wave 0 of the last workgroup to have reported (lane 0 holds `seen`): the status word, and the cross-workgroup words
//     made ready for the next launch.  All 64 lanes.
template <bool FUSED>
__device__ __forceinline__ void finish_chunks(const LayoutArgs& a, const Lds& l, int lane, uint32_t seen_lane0, uint32_t gen) {
    const uint32_t seen = __builtin_amdgcn_readfirstlane(seen_lane0);
    if ((int)(seen & (kGaveUp - 1u)) != a.nchunks + 1) return;  // the chunks and the workgroup of the tables
    int extra = seen >= kGaveUp ? STATUS_TIMEOUT : 0;
    if (FUSED && !a.padded && last_row_end(a, l, lane) > a.rows_cap) extra |= STATUS_OUTPUT_OVERFLOW;
    write_status(a, l, lane, extra);
    uint32_t next = gen + 1u;
    if (next >= kTags) {  // the tags have run out: clear every published word and start over
        for (int64_t j = lane; j < (int64_t)kMaxChunks * a.W; j += kWave) a.pub[j] = 0u;
        next = 0u;
    }
    if (lane == 0) {
        __hip_atomic_store(&a.ctl[1], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(&a.ctl[0], next, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// Rows of padded windows in use.  One wavefront; must be called by all 64 lanes.
__device__ __forceinline__ int sum_kept(const LayoutArgs& a, const Lds& l, int lane) {
    int kept = 0;
    for (int c0 = 0; c0 < a.E; c0 += kScanRows * kWave) {
        int v[kScanRows];
#pragma unroll
        for (int r = 0; r < kScanRows; ++r) v[r] = l.tot[min(c0 + r * kWave + lane, a.E - 1)];
#pragma unroll
        for (int r = 0; r < kScanRows; ++r) kept += c0 + r * kWave + lane < a.E ? min(v[r], a.C) : 0;
    }
    return __builtin_amdgcn_readlane(wave_inclusive_scan(kept), kWave - 1);
}

// The scans over the bins, between two barriers: the totals by wave 0, the blocks of the walk list by the others
// (the workgroup of the tables has none).  Returns, in the last wave of the workgroup of the tables, the rows of padded
// windows in use.
template <bool MULTI, bool WALK>
__device__ __forceinline__ int scan_bins(const LayoutArgs& a, const Lds& l, int b, int w, int waves, int nsub, const half_word* before0,
                                         int pitch, int step, int lane) {
    int kept = 0;
    lds_barrier();
    if (w == 0) scan_totals(a, l, lane);
    else if (WALK && b < a.nchunks) {
        for (int sb = w - 1; sb < nsub; sb += waves - 1) scan_walk(a, l, before0, pitch, step, sb, nsub, lane);
    }
    if (a.padded && w == waves - 1 && b == (MULTI ? a.nchunks : 0)) kept = sum_kept(a, l, lane);
    lds_barrier();
    return kept;
}

// One workgroup's share of a layout of at most PASSES = PU passes per wavefront (64 K entries), whose entries stay in
// registers: 16 rows of 64 entries, row = a pass of a wave.  The standing of an entry among those of its row with the same bin
// comes from a word of LDS per row and bin in which every entry sets the bit of its lane (an OR: no order is
// decided), and so does the row's count of the bin: 16 waves share the four instruction streams of a compute unit, so what
// bounds a small layout is instructions per wave, and ballots over the bits of the keys, with histograms beside them,
// take several times as many (744 entries of 256 experts in one workgroup: 6.4 us from its first instruction to its last, now
// 3.4; 18 006 entries of 96 experts: 9.3 us, now 7.1).
template <int HB, int PASSES, bool FUSED, bool WALK>
__device__ __forceinline__ void layout_rows(const LayoutArgs& a, int32_t* lds, const int b) {
    constexpr int waves = kRows / PASSES;
    constexpr bool multi = HB > 0;
    const int W = a.W, Wr = row_words(W);
    const Lds l = carve_lds(lds, a, 2 * kRows * Wr);
    const int tid = threadIdx.x, lane = lane_id();
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wc = b * waves + w;
    const bool active = wc < a.nwc;
    uint64_t* rows = (uint64_t*)lds;           // [kRows][Wr]
    uint64_t* mine = rows + w * PASSES * Wr;   // the rows of this wave

    // the loads of the ids, and meanwhile the clearing of the wave's own rows
    int raw[PASSES];
    if (active) issue_group(a, wc, 0, lane, raw);
    uint32_t gen = 0;
    if (multi) gen = __hip_atomic_load(&a.ctl[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    for (int j = lane; j < PASSES * Wr / 2; j += kWave) ((u32x4*)mine)[j] = (u32x4){0u, 0u, 0u, 0u};
    if (multi && tid == 0) *l.flag = 0;

    Entry en[PASSES];
    int sl[PASSES], rsl[PASSES];
    if (active) {
        classify_group(a, wc, 0, lane, raw, en);
        // LDS accesses of one wavefront are performed in program order; the fences keep the compiler to it
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
        const uint64_t bit = 1ull << lane;
#pragma unroll
        for (int p = 0; p < PASSES; ++p) {
            uint64_t* row = mine + p * Wr;
            const int bin = en[p].ok ? en[p].e : en[p].masked ? a.E : a.E + 1;
            if (en[p].i >= 0) __hip_atomic_fetch_or(&row[bin], bit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            if (en[p].lead) __hip_atomic_fetch_or(&row[a.E + 2 + en[p].d], bit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
#pragma unroll
        for (int p = 0; p < PASSES; ++p) {
            const uint64_t* row = mine + p * Wr;
            sl[p] = (int)__popcll(row[en[p].e] & (bit - 1ull));  // lanes without an expert hold e = 0 and use neither
            rsl[p] = (int)__popcll(row[a.E + 2 + en[p].d] & (bit - 1ull));
        }
    }
    lds_barrier();

    // per bin (thread = column): the sum of the chunk, which is published at once, and the running sum down the rows,
    // which takes the place of the bits
    if (multi) asm volatile("" : "+v"(gen));  // the generation is first looked at here
    const uint32_t tag = gen + 1u;
    for (int c = tid; c < W; c += waves * kWave) {
        uint64_t v[kRows];
#pragma unroll
        for (int r = 0; r < kRows; ++r) v[r] = rows[r * Wr + c];
        int run = 0;
#pragma unroll
        for (int r = 0; r < kRows; ++r) {
            *(half_word*)&rows[r * Wr + c] = run;
            run += (int)__popcll(v[r]);
        }
        if (multi && b < a.nchunks)  // the workgroup after the last chunk has no entries: it only writes the tables
            __hip_atomic_store(&a.pub[(int64_t)b * W + c], (tag << kTagShift) | (uint32_t)run, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
        if (!multi) l.tot[c] = run;
    }
    if constexpr (multi) gather_chunks<HB, WALK>(a, l, b, waves, tag);
    const int nsub = WALK && waves > a.walk_group ? waves / a.walk_group : 1;  // blocks of the walk list in this chunk
    const int kept = scan_bins<multi, WALK>(a, l, b, w, waves, nsub, (const half_word*)rows, 2 * PASSES * Wr, 2, lane);
    uint32_t seen = 0;
    if (multi) seen = report_chunk(a, l);

    // slots
    if (active) {
        const int sb = nsub > 1 ? w / a.walk_group : 0;  // the block of this wave
        const int walk_base = WALK ? __builtin_amdgcn_readfirstlane(l.first[sb]) : 0;
#pragma unroll
        for (int p = 0; p < PASSES; ++p) {
            const uint64_t* row = mine + p * Wr;
            sl[p] = en[p].ok ? sl[p] + *(const half_word*)&row[en[p].e] : -1;
            rsl[p] += *(const half_word*)&row[a.E + 2 + en[p].d];
        }
        emit_group<multi, WALK>(a, en, 0, sl, rsl, l, l.walk + sb * a.E, walk_base);
    }
    // the tables: with several chunks from a workgroup of their own, number nchunks, which has no entries: it looks across,
    // scans and writes the tables while the chunks still write theirs
    if (b == (multi ? a.nchunks : 0)) write_tables<!multi>(a, l, tid, lane, w, kept);
    if (multi && w == 0) finish_chunks<FUSED>(a, l, lane, seen, gen);
}

// The same for any number of passes and tables of any size: a wave walks its entries PU passes at a time, twice, with one
// histogram per wave.
template <int HB, bool WALK>
__device__ __forceinline__ void layout_chunk(const LayoutArgs& a, int32_t* lds, const int b) {
    const int wpb = blockDim.x >> 6;
    const Lds l = carve_lds(lds, a, (wpb + 1) * a.W);
    const int W = a.W;
    const int tid = threadIdx.x;
    const int lane = lane_id();
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wc = b * wpb + w;
    const int nchunks = a.nchunks;
    const bool active = wc < a.nwc;
    constexpr bool multi = HB > 0;

    // (1) the global loads this workgroup can issue at once: its own ids and the generation
    //     (first needed in (3): nothing here waits for it)
    int raw[PU];
    if (active) issue_group(a, wc, 0, lane, raw);
    uint32_t gen = __hip_atomic_load(&a.ctl[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    for (int j = tid; j < lds_ints(W, wpb); j += blockDim.x) l.wh[j] = 0;
    lds_barrier();

    // (2) per-wave histograms of this chunk
    Entry en[PU];
    if (active) {
        for (int p0 = 0; p0 < a.passes; p0 += PU) {
            if (p0 > 0) issue_group(a, wc, p0, lane, raw);
            classify_group(a, wc, p0, lane, raw, en);
            hist_group(a, en, l.wh + w * W);
        }
    }
    lds_barrier();

    // (3) per bin (thread = column): the sum of the chunk, which is published at once, and
    //     the running sum down the waves -- row r becomes "entries of the bin in the waves
    //     before r"
    asm volatile("" : "+v"(gen));  // the generation is first looked at here
    const uint32_t tag = gen + 1u;
    for (int c = tid; c < W; c += blockDim.x) {
        int v[kLayoutWavesPerBlock];
#pragma unroll
        for (int r = 0; r < kLayoutWavesPerBlock; ++r) v[r] = l.wh[min(r, wpb) * W + c];  // rows beyond the last: 0
        int run = 0;
#pragma unroll
        for (int r = 0; r < kLayoutWavesPerBlock; ++r) {
            const int x = v[r];
            v[r] = run;
            run += x;
        }
        if (multi && b < nchunks)  // the workgroup after the last chunk has no entries: it only writes the tables
            __hip_atomic_store(&a.pub[(int64_t)b * W + c], (tag << kTagShift) | (uint32_t)run, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
        l.tot[c] = run;
#pragma unroll
        for (int r = 0; r < kLayoutWavesPerBlock; ++r) l.wh[min(r, wpb) * W + c] = v[r];
    }
    // (4) entries of the other chunks, and the scans
    if constexpr (multi) gather_chunks<HB, WALK>(a, l, b, wpb, tag);
    const int nsub = WALK && wpb > a.walk_group ? wpb / a.walk_group : 1;  // blocks of the walk list in this chunk
    const int kept = scan_bins<multi, WALK>(a, l, b, w, wpb, nsub, l.wh, W, 1, lane);
    uint32_t seen = 0;
    if (multi) seen = report_chunk(a, l);

    // (5) ranks inside the chunk, and slots
    if (active) {
        const int sb = nsub > 1 ? w / a.walk_group : 0;  // the block of this wave
        const int walk_base = WALK ? __builtin_amdgcn_readfirstlane(l.first[sb]) : 0;
        InWave iw[PU];
        int sl[PU], rsl[PU];
        for (int p0 = 0; p0 < a.passes; p0 += PU) {
            load_group(a, wc, p0, lane, en);
            rank_group(a, en, p0, lane, iw);
            place_group(a, en, iw, p0, l.wh + w * W, sl, rsl);
            emit_group<multi, WALK>(a, en, p0, sl, rsl, l, l.walk + sb * a.E, walk_base);
        }
    }
    // (6) the tables, as in layout_rows
    if (b == (multi ? nchunks : 0)) write_tables<!multi>(a, l, tid, lane, w, kept);
    if (multi && w == 0) finish_chunks<false>(a, l, lane, seen, gen);
}

// PASSES: of layout_rows; 0: layout_chunk.
template <bool MULTI, int PASSES, bool WALK>
__global__ __launch_bounds__(1024, MULTI ? 4 : 8) void layout_kernel(LayoutArgs a) {
    extern __shared__ __align__(16) int32_t lds[];
    const int nlay = a.nchunks + (MULTI ? 1 : 0);  // workgroups that lay out: the chunks and, with several, the one of the tables
    if ((int)blockIdx.x >= nlay) {  // a whole workgroup: no barrier is reached by part of one
        // a short pause first (about 0.4 us): the chunks' loads of their ids then go ahead of the flood of
        // token reads instead of queueing behind it (1.2 us of the kernel at the prefill shape)
        __builtin_amdgcn_s_sleep(16);
        if (a.quant_out) quantize_tokens(a, blockIdx.x - nlay, gridDim.x - nlay);
        else warm_tokens(a, blockIdx.x - nlay, gridDim.x - nlay);
        return;
    }
    if constexpr (PASSES > 0) layout_rows<MULTI ? 32 : 0, PASSES, false, WALK>(a, lds, blockIdx.x);
    else layout_chunk<MULTI ? 32 : 0, WALK>(a, lds, blockIdx.x);
}

// ---- layout and direct dispatch of a small input in ONE launch (Sec. IV-C: in the
// low-latency kernels the count runs next to the send) ----
//
// The first `nlay` workgroups are the layout above and write the handle's arrays, which combine
// and the queries read later.  Every other workgroup copies `group` tokens (the segments of
// one of `parts` shares of their rows) and needs only the destination rows of these tokens'
// entries, which it counts out of the ids directly: row of an entry naming expert e = first row
// of e + entries before the group that name e + earlier entries of the group that name e, the
// first row being the number of entries that name a lower expert (or e * C, or the caller's).
// All ids (at most 8 per thread) go through one LDS histogram whose words hold the entries of a
// bin in the low half and those before the group in the high half; the entries of the group
// (at most 64) sit in the lanes of every wave and are ranked with one ballot per key bit.  Same
// ids, same arithmetic as the layout: the rows are those it records.  No copying workgroup
// waits for another.
//
// What bounds it: the id loads, three barriers and the random-placement write rate; the layout, a
// chain of latencies of about the same length as a short copy, is hidden behind it.  128 tokens of 14 336 bytes,
// top-8: 6.2 us (9.1 before the layout went by rows of LDS words), 64 tokens of 512 bytes, top-2: 3.4 (5.8).
constexpr int kFusedIds = 8;  // ids per thread
constexpr int kFusedMaxEntries = kFusedIds * kLayoutWavesPerBlock * kWave;

// IDS: ids per thread.
template <int IDS, bool MULTI>
__global__ __launch_bounds__(1024, 8) void layout_dispatch_kernel(LayoutArgs a, DispatchArgs d, int nlay, int nseg, int units,
                                                               int group, int parts, int spp) {
    extern __shared__ __align__(16) int32_t lds[];
    if ((int)blockIdx.x < nlay) {
        layout_rows<MULTI ? kFusedIds : 0, 1, true, false>(a, lds, blockIdx.x);  // at most kFusedIds chunks
        return;
    }
    constexpr int threads = kLayoutWavesPerBlock * kWave;
    uint32_t* bins = (uint32_t*)lds;  // [E]
    const int tid = threadIdx.x;
    const int lane = lane_id();
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wg = blockIdx.x - nlay;
    const int grp = wg / parts;
    const int seg0 = (wg - grp * parts) * spp, segs = min(spp, nseg - seg0);
    const int t0 = grp * group, nt = min(group, a.T - t0);
    const int first = t0 * a.K, m = nt * a.K;  // m <= 64
    const int items = nt * segs;               // segments this workgroup copies, wave w takes w, w + 16, ...
    // the loads this wave needs first, all issued before any is waited for: a segment of a token, the
    // ids of the entries this thread stands for, the group's ids and gate weights
    u32x4 v = {0u, 0u, 0u, 0u};
    int g = w / segs, seg = seg0 + (w - g * segs);
    auto fetch = [&]() {
        const int unit = seg * kWave + lane;
        if (g < nt && unit < units) v = __builtin_nontemporal_load((const u32x4*)(d.x + (int64_t)(t0 + g) * d.x_stride) + unit);
    };
    fetch();
    int id[IDS];
#pragma unroll
    for (int j = 0; j < IDS; ++j) {
        const int i = tid + j * threads;
        id[j] = -1;
        if (j * threads < a.n && i < a.n) {
            const int ti = token_of(a, i);
            id[j] = a.topk[(int64_t)ti * a.topk_stride + (i - ti * a.K)];
        }
    }
    const int my_g = token_of(a, lane), my_k = lane - my_g * a.K;
    const int my_e = lane < m ? a.topk[(int64_t)(t0 + my_g) * a.topk_stride + my_k] : -1;
    const bool routed = (unsigned)my_e < (unsigned)a.E;  // lanes beyond the group hold -1
    float my_w = 1.0f;
    if (d.recv_w && d.w && lane < m) my_w = d.w[(int64_t)(t0 + my_g) * d.w_stride + my_k];
    int my_base = 0;
    if (!a.padded && a.expert_base && routed) my_base = a.expert_base[my_e];
    if (tid < a.E) bins[tid] = 0u;  // E <= 1024
    lds_barrier();
#pragma unroll
    for (int j = 0; j < IDS; ++j)
        if ((unsigned)id[j] < (unsigned)a.E) atomicAdd(&bins[id[j]], tid + j * threads < first ? 0x10001u : 1u);
    lds_barrier();
    if (!a.padded && !a.expert_base) {  // the first row of every expert: entries that name a lower one
        if (w == kLayoutWavesPerBlock - 1) {  // one wave, the one with the fewest segments; the others rank the group's entries
            int carry = 0;
            for (int c0 = 0; c0 < a.E; c0 += kScanRows * kWave) {
                uint32_t word[kScanRows];
#pragma unroll
                for (int r = 0; r < kScanRows; ++r) {
                    const int c = c0 + r * kWave + lane;
                    word[r] = c < a.E ? bins[c] : 0u;
                }
#pragma unroll
                for (int r = 0; r < kScanRows; ++r) {
                    const int c = c0 + r * kWave + lane, count = (int)(word[r] & 0xffffu);
                    const int inc = wave_inclusive_scan(count);
                    if (c < a.E) bins[c] = (word[r] & 0xffff0000u) | (uint32_t)(carry + inc - count);
                    carry += __builtin_amdgcn_readlane(inc, kWave - 1);
                }
            }
        }
    }
    const uint64_t peers = match_key(my_e, routed, a.bits_e);
    if (!a.padded && !a.expert_base) lds_barrier();
    if (w >= items) return;
    const int in_group = (int)__popcll(peers & ((1ull << lane) - 1ull));
    int my_row = -1;
    int64_t my_off = 0;
    if (routed) {
        const uint32_t word = bins[my_e];
        const int slot = (int)(word >> 16) + in_group;
        if (a.padded) {
            if (slot < a.C) my_row = my_e * a.C + slot;
            my_off = (int64_t)my_e * d.win.stride0 + (int64_t)slot * d.win.stride1;
        } else {
            my_row = (a.expert_base ? my_base : (int)(word & 0xffffu)) + slot;
            my_off = (int64_t)my_row * d.win.stride0;
        }
        if (my_row >= d.win.rows_cap) my_row = -1;  // flagged with the layout's status word
    }
    for (int it = w;;) {
        const int unit = seg * kWave + lane;
        const bool active = unit < units;
        if (seg == 0 && my_row >= 0 && my_g == g) {
            if (d.recv_w) d.recv_w[my_row] = my_w;
            if (d.recv_src) d.recv_src[my_row] = t0 + g;
        }
        for (int k = 0; k < a.K; ++k) {
            const int src = g * a.K + k;
            if (__builtin_amdgcn_readlane(my_row, src) < 0) continue;
            const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)my_off, src);
            const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)((uint64_t)my_off >> 32), src);
            uint16_t* dst = d.win.base + (int64_t)(((uint64_t)hi << 32) | lo);
            if (active) __builtin_nontemporal_store(v, (u32x4*)dst + unit);
        }
        it += kLayoutWavesPerBlock;
        if (it >= items) break;
        g = it / segs;
        seg = seg0 + (it - g * segs);
        fetch();
    }
}

}  // namespace

// Wave-chunk plan for n entries: 64*passes consecutive entries per wavefront.  As many wave-chunks as there are passes of
// 64 entries, up to kMaxWaveChunks, so that every wave has as short a chain of dependent steps as possible.  (Up to 1024
// entries are one workgroup's; 4096 of 256 experts in one workgroup of four passes took 18.6 us per call, in four workgroups
// of one 7.9.)
void plan_layout(int n, int* passes, int* nwc) {
    int p = (n + kWave * kMaxWaveChunks - 1) / (kWave * kMaxWaveChunks);
    if (p < 1) p = 1;
    *passes = p;
    *nwc = (n + kWave * p - 1) / (kWave * p);
}

// A block of the walk list is a whole number of chunks (workgroups of the layout) or a whole part of one.
int plan_walk(int E, int R, int passes, int most) {
    int group = 0;
    for (int waves = kLayoutWavesPerBlock; waves >= 1; waves >>= 1) {
        group = most / waves * waves;
        if (group == 0) {
            group = 1;
            while (2 * group <= most) group *= 2;
        }
        // two waves and one block always fit, and 512 wave-chunks allow no fewer
        if (waves == 2) group = std::max(group, 2);
        if (cut_layout(E, R, passes, group).waves >= waves) break;
    }
    return group;
}

// The read-ahead rides on the layout kernel of inputs that are laid out by several workgroups.
bool layout_prefetches(const LayoutArgs& a) {
    return a.warm_x != nullptr && a.warm_rows > 0 && a.n >= kRunOrderMinEntries && a.nwc > kLayoutWavesPerBlock;
}

// The one-launch path takes inputs of at most 8192 entries that are copied by the plain
// token-ordered walk (bf16 rows, the K entries of a token held by the lanes of one wave).  Beyond
// that every workgroup would count more than 8 ids per thread, and the layout is a small part
// of the two launches.  Nor do inputs that move more than kFusedMaxBytes come this way: 512 resident
// workgroups stream a little slower than one wavefront per segment (rows of 14 336 bytes, two launches
// / one: top-8 30.8/18.0 us at 512 tokens, 26.9/19.9 at 611, 33.4/27.6 at 900, 38.1/34.3 at 1023 =
// 132 MB; top-2 40.2/39.6 at 4096 = 176 MB; top-1 47.4/49.8 at 8192 = 235 MB; 8192 rows of 512 bytes
// 13.0/9.8).
constexpr int64_t kFusedMaxBytes = 176ll << 20;
constexpr int kFusedMaxBins = 818;  // 112 KB of tables, one workgroup per compute unit; not tried beyond

bool layout_dispatch_fusable(const LayoutArgs& a, const DispatchArgs& d) {
    if (a.walk) return false;  // goes in destination order
    if (((int64_t)a.n + a.T) * d.H * 2 > kFusedMaxBytes) return false;
    return a.n >= 1 && a.n <= kFusedMaxEntries && a.passes == 1 && a.K <= kWave && a.E <= kLayoutWavesPerBlock * kWave && d.H >= 8 &&
           a.W <= kFusedMaxBins && cut_layout(a.E, a.R, 1, 0).rows;
}

// Copying workgroups of a fused launch: two of 1024 threads fit a compute unit, the layout's come first.
constexpr int kFusedCopyBlocks = 480;

hipError_t launch_layout_dispatch(const LayoutArgs& a_in, const DispatchArgs& d, hipStream_t s) {
    LayoutArgs a = a_in;
    a.nchunks = 1;
    if (!layout_dispatch_fusable(a, d)) return hipErrorInvalidValue;
    a.rows_cap = d.win.rows_cap;
    a.recv_count = d.recv_count;
    // one pass per wave (at most 8192 entries); one workgroup lays out where there is one chunk
    a.nchunks = (a.nwc + kLayoutWavesPerBlock - 1) / kLayoutWavesPerBlock;
    const bool multi = a.nchunks > 1;
    const int nlay = multi ? a.nchunks + 1 : 1;
    const int units = d.H / 8;
    const int nseg = (units + kWave - 1) / kWave;
    // tokens per workgroup: so many that all copying workgroups run at once if a row takes one of them, no more than
    // 64 entries.  Rows of more than 16 segments take several, the later ones after the first have ended (480 tokens of
    // 32 768 bytes, top-8: 29.5 us, in two launches 43.5).
    const int group = std::max(1, std::min((a.T + kFusedCopyBlocks - 1) / kFusedCopyBlocks, kWave / a.K));
    const int ngroups = (a.T + group - 1) / group;
    // workgroups per group: at most 16 segments of a token each, and as many as leave every workgroup of the launch a
    // compute unit of its own (rows of 14 336 bytes, top-8, at 85 tokens 5.1 us in 170 workgroups, 6.2 in 340; at 128 tokens
    // 6.2 us in 128, 6.5 in 256 beside the one of the layout)
    int parts = (nseg + kLayoutWavesPerBlock - 1) / kLayoutWavesPerBlock;
    while (parts < nseg && nlay + (int64_t)ngroups * (parts + 1) <= 256) ++parts;
    const int spp = (nseg + parts - 1) / parts;
    parts = (nseg + spp - 1) / spp;
    const int64_t nblk = nlay + (int64_t)ngroups * parts;
    if (nblk > 0x7fffffffLL) return hipErrorInvalidValue;
    const dim3 grid((unsigned)nblk), block(kLayoutWavesPerBlock * kWave);
    const size_t lds = cut_layout(a.E, a.R, 1, 0).lds;  // holds the copying workgroups' E words as well
    if (a.nchunks > 2) hipLaunchKernelGGL((layout_dispatch_kernel<kFusedIds, true>), grid, block, lds, s, a, d, nlay, nseg, units, group, parts, spp);
    else if (multi) hipLaunchKernelGGL((layout_dispatch_kernel<2, true>), grid, block, lds, s, a, d, nlay, nseg, units, group, parts, spp);
    else hipLaunchKernelGGL((layout_dispatch_kernel<1, false>), grid, block, lds, s, a, d, nlay, nseg, units, group, parts, spp);
    return hipGetLastError();
}

// Extra workgroups of the layout kernel that read tokens.  All of them and the layout's own (33 of 16 waves up to 32 768 entries, 65 of
// 8 or fewer beyond) run from the start, one per compute unit: a unit holds 16 waves of this kernel (its registers), and tables of
// 512 experts take more than half of its LDS.  Layout alone, us, tokens in the memory-side cache / not (us there with the 384 that as
// many waves of 8 per workgroup make; they share units with the chunks or, with large tables, half of them run as a tail):
//   192 of 16 waves: 4096 tokens of 14 336 bytes, 256 experts, 12.1 / 12.7 (128 workgroups 11.1 / 14.4, 224 15.2 / 15.6)
//   160 of 8: 8192 of 14 336 15.1 / 16.5 (384 16.9 / 16.9; 128 14.0 / 18.6; 192 16.5 / 20.9), 8192 of 8192, 128 experts,
//   13.8 / 16.0 (384 15.4 / 15.8; 128 12.4 / 18.0), 512 experts 19.4 / 18.7 (384 20.2 / 21.1), 6000 of 10 240, 1024 experts,
//   27.4 / 27.0 (384 28.4 / 28.7)
constexpr int kWarmBlocks = 192, kWarmBlocksShort = 160;
// Wavefronts where the tokens are quantised ahead, which is bound by arithmetic (8192 tokens of 4096 channels, 256 experts, layout of
// 22.7 us with 384 workgroups of 8 waves, 29.2 with 192; 512 experts, whose tables leave one workgroup per unit, 27.6 and 36.0).
constexpr int kQuantWaves = 192 * 16;

hipError_t launch_layout(const LayoutArgs& a_in, hipStream_t s) {
    LayoutArgs a = a_in;
    a.nchunks = 1;
    const LayoutCut cut = cut_layout(a.E, a.R, a.passes, a.walk ? a.walk_group : 0);
    const int wpb = cut.waves;
    if (cut.lds > kLdsUnit || (!cut.rows && cut.lds > kLdsLimit)) return hipErrorInvalidValue;
    if (a.walk && a.walk_group % wpb != 0 && wpb % a.walk_group != 0) return hipErrorInvalidValue;
    int nblk = (a.nwc + wpb - 1) / wpb;
    if (nblk < 1) nblk = 1;
    if (nblk > kMaxChunks) return hipErrorInvalidValue;
    if ((int64_t)wpb * kWave * a.passes > (int64_t)kCountMask) return hipErrorInvalidValue;  // a chunk's count must fit its word
    a.nchunks = nblk;
    const bool pf = layout_prefetches(a);
    const int nlay = nblk + (nblk > 1 ? 1 : 0);
    const int nwarm = !pf ? 0 : a.quant_out ? kQuantWaves / wpb : wpb == kLayoutWavesPerBlock ? kWarmBlocks : kWarmBlocksShort;
    const dim3 grid(nlay + nwarm), block(wpb * kWave);
    auto launch = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, block, cut.lds, s, a); };
    const int passes = cut.rows ? a.passes : 0;
    if (a.walk && nblk == 1) return hipErrorInvalidValue;  // inputs this small have no walk list
    if (a.walk && passes == 1) launch(layout_kernel<true, 1, true>);
    else if (a.walk && passes == 2) launch(layout_kernel<true, 2, true>);
    else if (a.walk) launch(layout_kernel<true, 0, true>);
    else if (nblk > 1 && passes == 1) launch(layout_kernel<true, 1, false>);
    else if (nblk > 1 && passes == 2) launch(layout_kernel<true, 2, false>);
    else if (nblk > 1) launch(layout_kernel<true, 0, false>);
    else if (passes == 1) launch(layout_kernel<false, 1, false>);
    else launch(layout_kernel<false, 0, false>);
    return hipGetLastError();
}

}  // namespace ep
