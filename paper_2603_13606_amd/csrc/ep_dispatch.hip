// Dispatch pack, direct path (Sec. IV-C "Send Tokens"; row format of Sec. IV-B
// with the source index and gate weight kept in side arrays so rows are pure
// token data, ready for a grouped GEMM as Sec. III-E asks).
//
// Pure data movement, bound by HBM: a token row of 2H bytes is read once and
// written to up to K destination rows.  Work unit = one wavefront moving one
// 1 KiB segment of one token row: every lane loads 16 bytes once and stores
// them K times, so all global accesses are full 64-lane x 16-byte bursts.  The
// routing entries of the token are wave-uniform and come through scalar loads.
#include "ep_internal.h"
#include "ep_fp8.h"

#include <algorithm>

namespace ep {
namespace {

// One wavefront copies one 1 KiB segment (16-byte unit `seg * 64 + lane` of every lane) of
// token t to the token's destination rows, in two halves so that a caller can put other
// work between the loads and the stores.  Both must be called by all 64 lanes.
struct TokenSegment {
    u32x4 v;     // the 16 bytes of this lane
    int my_row;  // lane k: destination row of the token's k-th entry
    float my_w;  // first segment: its gate weight, where one is delivered
};

// Lane k: the gate weight delivered with entry k of token t (1 without gate weights).
__device__ __forceinline__ float entry_weight(const DispatchArgs& a, int t, int lane, bool first) {
    return first && a.recv_w && a.w && lane < a.K ? a.w[(int64_t)t * a.w_stride + lane] : 1.0f;
}

__device__ __forceinline__ TokenSegment load_token_segment(const DispatchArgs& a, int t, int seg, int units, int lane) {
    TokenSegment s;
    const int unit = seg * kWave + lane;
    s.v = (u32x4){0u, 0u, 0u, 0u};
    if (unit < units) s.v = __builtin_nontemporal_load((const u32x4*)(a.x + (int64_t)t * a.x_stride) + unit);
    // lane k fetches the k-th destination row of the token: one load for all K entries
    s.my_row = lane < a.K ? a.dst_row[(int64_t)t * a.K + lane] : -1;
    s.my_w = entry_weight(a, t, lane, seg == 0);
    return s;
}

__device__ __forceinline__ void store_token_segment(const DispatchArgs& a, const TokenSegment& s, int t, int seg, int units,
                                                    int lane) {
    const int unit = seg * kWave + lane;
    const bool active = unit < units;
    const int my_row = deliver_sides(a.win, a.recv_w, a.recv_src, a.totals, seg == 0, s.my_row, s.my_w, t);
    for (int k = 0; k < a.K; ++k) {
        const int row = __builtin_amdgcn_readlane(my_row, k);
        if (row < 0) continue;
        uint16_t* dst = a.win.base + window_offset(a.win, row);
        if (active) __builtin_nontemporal_store(s.v, (u32x4*)dst + unit);
    }
}

__device__ __forceinline__ void copy_token_segment(const DispatchArgs& a, int t, int seg, int units, int lane) {
    const TokenSegment s = load_token_segment(a, t, seg, units, lane);
    store_token_segment(a, s, t, seg, units, lane);
}

__global__ __launch_bounds__(256) void dispatch_direct_kernel(DispatchArgs a, int nseg, int units) {
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t u = (int64_t)blockIdx.x * 4 + wave;
    if (blockIdx.x == 0 && a.recv_count) {
        for (int e = threadIdx.x; e < a.E; e += blockDim.x) a.recv_count[e] = a.expert_kept[e];
    }
    if (u >= (int64_t)a.T * nseg) return;
    const int t = (int)(u / nseg);
    copy_token_segment(a, t, (int)(u - (int64_t)t * nseg), units, lane);
}

// ---- destination-ordered variant for large inputs
//
// Writes that land next to each other within a short time are served much faster by the
// memory system than rows scattered at random (measured on this part: 6.3 TB/s against
// 4.9 TB/s; 4096 tokens of 14 336 bytes, top-8, take 82 us this way and 108 in token order), so large inputs are walked in the order of the destination rows instead of
// the order of the tokens.  The layout has made a walk list for it: {token, row} of every entry
// that has a row, block of the input by block, expert by expert within a block.  The copy
// sweeps over all expert regions once per block and every region grows by about a dozen
// adjacent rows each time.
//
// A row is read once from HBM and up to K-1 more times from the L2 cache: the 16-byte
// units of a row are split into kSlices equal pieces and workgroup index mod kSlices picks
// the piece, which on this part is also the accelerator die the workgroup runs on, so each
// die's L2 only ever holds its own piece of the tokens of the current block.
constexpr int kSlices = 8;
// Rows per thread: how much is on its way at a time.  The writes of all resident workgroups should stay close together
// in memory, and the chain from a workgroup's start to its stores be covered: one row of a piece that takes two
// waves or more (4096 rows of 1792-byte pieces: dispatch of 4096 x 14 336 bytes, top-8, 82 us; with two rows 94, with four
// 94), two of shorter ones (8192 x 1024 bytes, top-8: 26.2 us, with one 28.2; 8192-byte rows 47.4/48.0).
constexpr int walk_unroll(int tpr_shift) { return tpr_shift >= 7 ? 1 : 2; }

// A launch takes fewer than 2^32 work-items.  kMaxEntries is what a group may be made for.
constexpr int64_t kMaxWalkWorkgroups = (1ll << 32) / 256 - 1;
constexpr int64_t kMaxEntries = 1ll << 28;
constexpr int64_t side_workgroups(int64_t entries) { return (entries + 2047) / 2048 * 8; }
// Places of the walk list one launch can cover, `rows` per workgroup.  A block is shorter: at most 2^20 entries where it is two
// wave-chunks of the longest input, and otherwise bounded by its share of L2 (65 536 entries of the longest pieces, one row
// per workgroup, top-64).
constexpr int64_t launch_places(int slices, int rows) {
    return (kMaxWalkWorkgroups - side_workgroups(kMaxEntries)) / slices * rows;
}
constexpr bool launch_fits(int slices, int rows) {  // with the side arrays of the longest input beside it
    const int64_t workgroups = slices * ((launch_places(slices, rows) + rows - 1) / rows);
    return launch_places(slices, rows) >= 1 << 20 && (workgroups + side_workgroups(kMaxEntries)) * 256 < 1ll << 32;
}

struct WalkPlan {
    int piece;      // 16-byte units per slice
    int units;      // 16-byte units per row
    int first, last;  // places of the walk list this launch covers
    int side_blocks;  // leading workgroups that fill the side arrays, a multiple of 8 (the dies stay aligned with the slices)
    int entries;      // routed entries of the input, at most
};

// What the walk copies when the rows were quantised ahead of the dispatch (FP8 codes and scales
// in a staging copy, row t at staged + t * pitch: H bytes of codes, then H/128 floats): unit col
// of a staged row goes to the code row of the output window while col < code_units and to the
// row of the scales array after that.  A staged row is half as long as a token row, so it is cut
// into 4 slices instead of 8 (two dies share a slice): the bytes per workgroup stay what they are
// for bf16 rows.  Window strides are in one-byte elements then.
constexpr int kFp8Slices = 4;

static_assert(launch_fits(kSlices, 1) && launch_fits(kSlices, 2) && launch_fits(kSlices, 32), "bf16 rows");
static_assert(launch_fits(kFp8Slices, 1) && launch_fits(kFp8Slices, 2) && launch_fits(kFp8Slices, 32), "staged FP8 rows");

struct StagedRows {
    const uint8_t* staged;
    int64_t pitch;
    float* recv_scales;  // [rows, groups]
    int code_units;      // H / 16
    int groups;          // H / 128
};

// The token an entry of the layout's lists names.  A layout that ended without all of its counts (STATUS_TIMEOUT) leaves
// places of the lists as they were before it: such an entry may hold anything.
__device__ __forceinline__ int listed_token(const DispatchArgs& a, int t) { return (int)min((uint32_t)t, (uint32_t)a.T - 1u); }

// Fills the side arrays in the order of the expert-sorted list, that is of the rows: 64 neighbouring
// words per store, by workgroups of their own.  Done by the copying workgroups of one slice, one word per row,
// all of it fell to one die, and its workgroups were the last to end (101 us for 82).
__device__ void walk_sides(const DispatchArgs& a, int i, int entries) {
    if (i >= min(entries, a.totals[TOT_SORTED])) return;
    const int row = a.sorted_row[i];
    if (row < 0 || row >= a.win.rows_cap) return;
    const int t = listed_token(a, a.sorted_token[i]);
    if (a.recv_src) a.recv_src[row] = t;
    if (a.recv_w) a.recv_w[row] = a.w ? a.w[(int64_t)t * a.w_stride + min((uint32_t)a.sorted_k[i], (uint32_t)a.K - 1u)] : 1.0f;
}

// TPR_SHIFT = log2(threads that share one row piece); PADDED = window addressing mode; FP8 =
// rows come from a staging copy of quantised rows instead of the bf16 tokens.
//
// A workgroup takes the next 256 / 2^TPR_SHIFT * walk_unroll places of the list: every workgroup but the last has all
// its rows, and the chain from its start to its stores is one list load and one token load.  (Cut by runs -- the
// entries of one expert in one block, at positions read from a table first -- a third of the workgroups had
// fewer rows than they could take, some looped, and the chain was one load longer: 87 us where this takes 82, and 96/80 with
// Zipf routing, 55/45 with rows of 8192 bytes, 32/22 of 5760, 41/17 of 1024; all in us.)
//
// The vector-memory counter of this part counts loads and stores alike, in order, and the
// compiler waits for it to reach zero wherever control flow stands between an access and the
// use of its result -- which, between two row stores, means waiting for the first store to
// reach memory before the second is issued.  So the rows of a step are copied by straight-line
// code (loads, then stores, nothing conditional in between) whenever every lane of the wave has
// all its rows, with the general code kept for the end of the list.
template <int TPR_SHIFT, bool PADDED, bool FP8>
__global__ __launch_bounds__(256) void dispatch_walk_kernel(DispatchArgs a, WalkPlan p, StagedRows f) {
    if (blockIdx.x == 0 && p.first == 0 && a.recv_count) {
        for (int e = threadIdx.x; e < a.E; e += blockDim.x) a.recv_count[e] = a.expert_kept[e];
    }
    if ((int)blockIdx.x < p.side_blocks) {
        walk_sides(a, blockIdx.x * 256 + threadIdx.x, p.entries);
        return;
    }
    constexpr int tpr = 1 << TPR_SHIFT, nsub = 256 >> TPR_SHIFT, U = walk_unroll(TPR_SHIFT);
    constexpr int slices = FP8 ? kFp8Slices : kSlices;
    constexpr int elem_bytes = FP8 ? 1 : 2;  // size of the elements the window strides count
    // workgroups are handed out slice by slice, then along the list
    const int b = blockIdx.x - p.side_blocks;
    const int xs = b & (slices - 1);
    int sub = threadIdx.x >> TPR_SHIFT;
    if (TPR_SHIFT >= 6) sub = __builtin_amdgcn_readfirstlane(sub);  // a row piece takes whole waves: token and row, and with
                                                                    // them the row addresses, live in scalar registers
    const int u = threadIdx.x & (tpr - 1);
    const int pos0 = p.first + ((b / slices) * nsub + sub) * U;
    const int end = min(p.last, a.totals[TOT_KEPT]);
    int2 en[U];
#pragma unroll
    for (int q = 0; q < U; ++q) en[q] = a.walk[pos0 + q];  // the list is followed by kWalkPad unused places
    const int u0 = xs * p.piece, u1 = min(p.units, u0 + p.piece);
    const int cend = FP8 ? min(u1, f.code_units) : u1;  // units of the row proper end here
    const uint8_t* src_base = FP8 ? f.staged : (const uint8_t*)a.x;
    const int64_t src_pitch = FP8 ? f.pitch : a.x_stride * 2;
    int row[U];
    const uint8_t* src[U];
    uint8_t* dst[U];
    bool have_all = true;
#pragma unroll
    for (int q = 0; q < U; ++q) {
        row[q] = pos0 + q < end ? en[q].y : -1;
        if (row[q] >= a.win.rows_cap) {
            if (xs == 0 && u == 0) atomicOr(&a.totals[TOT_STATUS], STATUS_OUTPUT_OVERFLOW);
            row[q] = -1;
        }
        const int t = row[q] >= 0 ? listed_token(a, en[q].x) : 0, r = max(row[q], 0);
        const int64_t off = PADDED ? window_offset(a.win, r) : (int64_t)r * a.win.stride0;
        src[q] = src_base + (int64_t)t * src_pitch;
        dst[q] = (uint8_t*)a.win.base + off * elem_bytes;
        have_all = have_all && row[q] >= 0;
    }
    if (FP8 && u1 > f.code_units) {  // the slice that holds the scales (workgroup-uniform), a few lanes of it
        for (int col = max(u0, f.code_units) + u; col < u1; col += tpr) {
            const int j = (col - f.code_units) * 4;  // up to four scales; the last unit may be part padding
#pragma unroll
            for (int q = 0; q < U; ++q) {
                if (row[q] < 0) continue;
                const u32x4 v = *((const u32x4*)src[q] + col);
                float* sdst = f.recv_scales + (int64_t)row[q] * f.groups + j;
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    if (j + c < f.groups) sdst[c] = __uint_as_float(v[c]);
            }
        }
    }
    if (__builtin_amdgcn_ballot_w64(!have_all) == 0) {
        for (int col = u0 + u; col < cend; col += tpr) {
            u32x4 v[U];
#pragma unroll
            for (int q = 0; q < U; ++q) v[q] = *((const u32x4*)src[q] + col);
#pragma unroll
            for (int q = 0; q < U; ++q) __builtin_nontemporal_store(v[q], (u32x4*)dst[q] + col);
        }
    } else {
        for (int col = u0 + u; col < cend; col += tpr) {
            u32x4 v[U];
#pragma unroll
            for (int q = 0; q < U; ++q)
                if (row[q] >= 0) v[q] = *((const u32x4*)src[q] + col);
#pragma unroll
            for (int q = 0; q < U; ++q)
                if (row[q] >= 0) __builtin_nontemporal_store(v[q], (u32x4*)dst[q] + col);
        }
    }
}

// Reads token rows [t0, t1) (and, when asked, the walk list) once, front
// to back, with ordinary cached loads, so that the run-ordered copy that follows finds
// them in the memory-side cache and the DRAM sees a read phase and then a write phase.
__global__ __launch_bounds__(256) void dispatch_warm_kernel(DispatchArgs a, int units, int t0, int t1, int with_index) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    uint32_t acc = 0;
    const int64_t total = (int64_t)(t1 - t0) * units;
    for (int64_t i = gid; i < total; i += stride) {
        const int64_t t = i / units;
        const int col = (int)(i - t * units);
        const u32x4 v = *((const u32x4*)(a.x + (t0 + t) * a.x_stride) + col);
        acc ^= v[0] ^ v[1] ^ v[2] ^ v[3];
    }
    if (with_index) {
        const int n = a.T * a.K;
        for (int64_t i = gid; i < n; i += stride) acc ^= (uint32_t)(a.walk[i].x ^ a.walk[i].y);
    }
    asm volatile("" ::"v"(acc));  // the loads are the point: keep them
}

// ---- quantising dispatch: FP8 (OCP E4M3) rows with one float scale per 128 channels
//
// The paper lets dispatch quantise tokens (Sec. I) and sizes the FP8 row at H bytes
// plus H/128 float scales (Sec. IV-B payload); format and scale rule are fixed by this
// library: per token and 128-channel group amax = max|x|, scale = amax / 448,
// q = e4m3(float(x) * (448 / amax)) rounded to nearest even and saturated at 448;
// amax == 0 gives scale 1.  Work unit = one wavefront x 1024 channels of one token:
// a lane owns 16 consecutive channels (32 bytes in, 16 bytes out), a group is 8 lanes.
// The row is quantised once and stored K times.
//
// LATE: the destination rows are loaded behind the quantisation, a round trip later, and the stores of a wave begin
// that much apart from those of the others (see launch_dispatch_fp8).
template <bool LATE>
__global__ __launch_bounds__(256) void dispatch_fp8_kernel(DispatchArgs a, float* recv_scales, int nseg) {
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t u = (int64_t)blockIdx.x * 4 + wave;
    if (blockIdx.x == 0 && a.recv_count) {
        for (int e = threadIdx.x; e < a.E; e += blockDim.x) a.recv_count[e] = a.expert_kept[e];
    }
    if (u >= (int64_t)a.T * nseg) return;
    const int t = (int)(u / nseg);
    const int seg = (int)(u - (int64_t)t * nseg);
    const int ch0 = seg * 1024 + lane * 16;  // first channel of this lane
    const bool active = ch0 < a.H;
    u32x4 in0 = {0u, 0u, 0u, 0u}, in1 = {0u, 0u, 0u, 0u};
    if (active) {
        const u32x4* src = (const u32x4*)(a.x + (int64_t)t * a.x_stride + ch0);
        in0 = __builtin_nontemporal_load(src);
        in1 = __builtin_nontemporal_load(src + 1);
    }
    int my_row = -1;
    float my_w = 1.0f;
    if (!LATE) {
        my_row = lane < a.K ? a.dst_row[(int64_t)t * a.K + lane] : -1;
        my_w = entry_weight(a, t, lane, seg == 0);
    }
    float scale;
    const u32x4 q = quantize16(in0, in1, &scale);
    const int groups = a.H >> 7;
    if (LATE) {
        my_row = lane < a.K ? a.dst_row[(int64_t)t * a.K + lane] : -1;
        my_w = entry_weight(a, t, lane, seg == 0);
    }
    my_row = deliver_sides(a.win, a.recv_w, a.recv_src, a.totals, seg == 0, my_row, my_w, t);
    uint8_t* base = (uint8_t*)a.win.base;  // window strides are in one-byte elements here
    for (int k = 0; k < a.K; ++k) {
        const int row = __builtin_amdgcn_readlane(my_row, k);
        if (row < 0) continue;
        if (active) {
            __builtin_nontemporal_store(q, (u32x4*)(base + window_offset(a.win, row) + ch0));
            if ((lane & 7) == 0) recv_scales[(int64_t)row * groups + (ch0 >> 7)] = scale;
        }
    }
}

// Plain streaming copy, 16 bytes per lane, grid-stride: the yardstick the hardware
// counters and the achievable copy bandwidth are calibrated against.
__global__ __launch_bounds__(256) void calibration_copy_kernel(u32x4* dst, const u32x4* src, int64_t n16) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n16; i += stride)
        __builtin_nontemporal_store(__builtin_nontemporal_load(src + i), dst + i);
}

// The two halves of that copy on their own, four 16-byte accesses per lane and trip: what this
// part's memory sustains for reads alone and for writes alone (a row kernel that mostly writes,
// or mostly reads, is bounded by these and not by the mixed copy).
__global__ __launch_bounds__(256) void calibration_fill_kernel(u32x4* dst, int64_t n16) {
    const int64_t stride = (int64_t)gridDim.x * 1024;
    const u32x4 v = {0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u};
    for (int64_t i = (int64_t)blockIdx.x * 1024 + threadIdx.x; i < n16; i += stride) {
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (i + j * 256 < n16) __builtin_nontemporal_store(v, dst + i + j * 256);
    }
}

__global__ __launch_bounds__(256) void calibration_read_kernel(const u32x4* src, int64_t n16, uint32_t* sink) {
    const int64_t stride = (int64_t)gridDim.x * 1024;
    uint32_t acc = 0;
    for (int64_t i = (int64_t)blockIdx.x * 1024 + threadIdx.x; i < n16; i += stride) {
        u32x4 v[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = __builtin_nontemporal_load(src + min(i + j * 256, n16 - 1));
#pragma unroll
        for (int j = 0; j < 4; ++j) acc ^= v[j][0] ^ v[j][1] ^ v[j][2] ^ v[j][3];
    }
    // the loads must not be dropped: the word is written only if the lane's checksum is one particular value
    if (acc == 0x9e3779b9u) *sink = acc;
}

}  // namespace

hipError_t launch_calibration_fill(void* dst, size_t bytes, hipStream_t s) {
    const int64_t n16 = (int64_t)(bytes / 16);
    if (n16 == 0) return hipSuccess;
    int64_t nblk = (n16 + 1023) / 1024;
    if (nblk > 256 * 64) nblk = 256 * 64;
    hipLaunchKernelGGL(calibration_fill_kernel, dim3((unsigned)nblk), dim3(256), 0, s, (u32x4*)dst, n16);
    return hipGetLastError();
}

hipError_t launch_calibration_read(const void* src, size_t bytes, uint32_t* sink, hipStream_t s) {
    const int64_t n16 = (int64_t)(bytes / 16);
    if (n16 == 0) return hipSuccess;
    int64_t nblk = (n16 + 1023) / 1024;
    if (nblk > 256 * 64) nblk = 256 * 64;
    hipLaunchKernelGGL(calibration_read_kernel, dim3((unsigned)nblk), dim3(256), 0, s, (const u32x4*)src, n16, sink);
    return hipGetLastError();
}

hipError_t launch_calibration_copy(void* dst, const void* src, size_t bytes, hipStream_t s) {
    const int64_t n16 = (int64_t)(bytes / 16);
    if (n16 == 0) return hipSuccess;
    int64_t nblk = (n16 + 255) / 256;
    if (nblk > 256 * 64) nblk = 256 * 64;
    hipLaunchKernelGGL(calibration_copy_kernel, dim3((unsigned)nblk), dim3(256), 0, s, (u32x4*)dst,
                       (const u32x4*)src, n16);
    return hipGetLastError();
}

// Inputs from kRunOrderMinEntries entries on can be copied in destination order (when the layout
// made the list); smaller ones are bound by latency and keep the shorter token-ordered
// kernel.  A read pass covers kWarmBytes of tokens: a piece must stay in the 256 MiB
// memory-side cache, next to whatever else lives there, while the copy of that piece runs.
//
// A block holds as many tokens as keep one slice of them (2H/8 bytes each) within 2 MiB, half of an XCD's L2: the
// longer its runs, the closer together the writes (dispatch of 4096 tokens, top-8, of 14 336 bytes, 256 experts: 85.0 us
// with 16 rows per expert and block, 83.0 with 32, 82.3 with 36, which is 2 MiB, and 87 with 64; of 8192 bytes, 128 experts, 47.7
// with 16, 46.6 with 64, 45.3 with 128, 2 MiB).  Blocks end where workgroups of the layout end, or at an even part of one.
// `units` 16-byte units per copied row, cut into `slices` slices; H = channels of a token row
// (what a read pass reads).
static bool plan_rows(int T, int K, int H, int units, int slices, int E, int R, int order, bool have_walk, int prefetched_rows,
                      DispatchPlan* out) {
    DispatchPlan d = {};
    const int64_t n = (int64_t)T * K;
    d.run_order = order != EP_ORDER_TOKEN && have_walk && n >= kRunOrderMinEntries && units >= slices;
    if (!d.run_order) { *out = d; return false; }
    int passes = 0, nwc = 0;
    plan_layout((int)n, &passes, &nwc);
    const int chunk_entries = passes * kWave;
    const int64_t l2_tokens = (2ll << 20) / std::max(16 * units / slices, 1);
    const int64_t most = std::max<int64_t>(768, l2_tokens * K);
    d.group = plan_walk(E, R, passes, (int)std::min<int64_t>(std::max<int64_t>(1, most / chunk_entries), kMaxWaveChunks));
    d.blocks = (nwc + d.group - 1) / d.group;
    d.piece = (units + slices - 1) / slices;
    if (d.piece >= 8) d.piece = (d.piece + 7) / 8 * 8;  // whole 128-byte lines per slice (the last slices get less)
    d.tpr_shift = 4;
    while ((1 << d.tpr_shift) < d.piece && d.tpr_shift < 8) ++d.tpr_shift;
    d.rows = (256 >> d.tpr_shift) * walk_unroll(d.tpr_shift);
    d.block_entries = d.group * chunk_entries;
    // blocks per launch: as many as a grid holds (3.9 million rows of 14 336 bytes), or as cover kWarmBytes of tokens
    int64_t per_launch = launch_places(slices, d.rows) / d.block_entries;
    if (order == EP_ORDER_DESTINATION) {
        const int64_t block_bytes = ((int64_t)d.block_entries + K - 1) / K * H * 2;
        per_launch = std::min(per_launch, kWarmBytes / std::max<int64_t>(block_bytes, 1));
    }
    d.blocks_per_launch = (int)std::max<int64_t>(1, std::min<int64_t>(d.blocks, per_launch));
    for (int b0 = 0; b0 < d.blocks; b0 += d.blocks_per_launch) {
        const int nb = std::min(d.blocks_per_launch, d.blocks - b0);
        const int t1 = (int)std::min<int64_t>(T, ((int64_t)(b0 + nb) * d.block_entries + K - 1) / K);
        d.launches += 1;
        if (order == EP_ORDER_DESTINATION && t1 > prefetched_rows) d.read_passes += 1;
    }
    *out = d;
    return true;
}

// Units of a staged FP8 row: H/16 of codes, then the scales rounded up to whole units.
static int fp8_code_units(int H) { return H / 16; }
static int fp8_row_units(int H) { return H / 16 + (H / 32 + 15) / 16; }

bool plan_dispatch(int T, int K, int H, int E, int R, int order, bool have_walk, int prefetched_rows, DispatchPlan* out) {
    return plan_rows(T, K, H, H / 8, kSlices, E, R, order, have_walk, prefetched_rows, out);
}

bool plan_dispatch_fp8_staged(int T, int K, int H, int E, int R, bool have_walk, DispatchPlan* out) {
    return plan_rows(T, K, H, fp8_row_units(H), kFp8Slices, E, R, EP_ORDER_DESTINATION_RESIDENT, have_walk, 0, out);
}

template <int TPR_SHIFT, bool FP8>
static void launch_walk_kernel(const DispatchArgs& a, const WalkPlan& p, const StagedRows& f, hipStream_t s) {
    const int rows = (256 >> TPR_SHIFT) * walk_unroll(TPR_SHIFT);
    const dim3 grid((unsigned)p.side_blocks + (unsigned)(FP8 ? kFp8Slices : kSlices) * (unsigned)((p.last - p.first + rows - 1) / rows));
    if (a.win.padded) hipLaunchKernelGGL((dispatch_walk_kernel<TPR_SHIFT, true, FP8>), grid, dim3(256), 0, s, a, p, f);
    else hipLaunchKernelGGL((dispatch_walk_kernel<TPR_SHIFT, false, FP8>), grid, dim3(256), 0, s, a, p, f);
}

// One launch of the walk over the places [first, last) of the list.  The first one also fills the side arrays.
template <bool FP8>
static void launch_walk(const DispatchArgs& a, const DispatchPlan& d, int units, int first, int last, const StagedRows& f,
                        hipStream_t s) {
    WalkPlan p;
    p.piece = d.piece; p.units = units; p.first = first; p.last = last;
    p.entries = a.T * a.K;
    p.side_blocks = first == 0 && (a.recv_w || a.recv_src) ? (int)side_workgroups(p.entries) : 0;
    switch (d.tpr_shift) {
        case 4: launch_walk_kernel<4, FP8>(a, p, f, s); break;
        case 5: launch_walk_kernel<5, FP8>(a, p, f, s); break;
        case 6: launch_walk_kernel<6, FP8>(a, p, f, s); break;
        case 7: launch_walk_kernel<7, FP8>(a, p, f, s); break;
        default: launch_walk_kernel<8, FP8>(a, p, f, s); break;
    }
}

// LDS that a workgroup of the token walk reserves and does not use, so that fewer than 8 workgroups share a compute unit.  LDS is
// handed out in units of 1280 bytes of 160 KiB: 21 of them leave 6 workgroups, 25 leave 5 (counted on the card).  The stores on
// their way spread over less memory then, which the memory system rewards where a launch is long and a wave has several
// rows to write.  Elsewhere the waves are needed to keep loads in flight, or the workgroups that do not fit run as a tail.
// Dispatch alone, with 8 / 6 / 5 workgroups, in us, at 128 experts; us before the reserve was introduced (and the side arrays
// were written by lanes) in front:
//   top-1  32.7: 33.5/39.1/43.0 at 134 000 rows of 512 bytes, 91.6: 91.9/95.3/101 at 19 100 of 14 336       -> 8
//   top-2  44.7: 41.1/49.6/56.0 at 128 MB of 512-byte rows (so from 1 KiB rows on), 134: 132/132/128 at 440 MB of 14 336
//   top-4  15.4: 15.6/15.8/16.8 at 64 MB of 14 336, 32.8: 31.3/31.1/31.1 at 128 MB, 109: 109/107/107 at 440 MB
//   top-6  8.9: 8.7/9.6/9.2 at 40 MB of 14 336, 30.0: 30.5/29.3/29.7 at 128 MB, 106: 111/103/103 at 440 MB
//   top-8  9.1: 8.9/9.0/9.8 at 40 MB of 14 336, 15.4: 15.1/14.9/14.6 at 64 MB with side arrays, 31.0: 30.9/29.1/29.2 at 128 MB,
//          106: 112/101/104 at 440 MB; 103: 110/103/107 at 440 MB of 2048
//   top-12 14.3: 14.1/14.0/14.3 at 64 MB of 14 336, 28.4: 28.2/29.0/28.1 at 128 MB, 99.3: 109/104/98.2 at 440 MB
// In between, how evenly the workgroups fill the rounds of resident ones decides, within 5 % either way.
constexpr size_t kLdsGranule = 1280, kSixWorkgroups = 21 * kLdsGranule, kFiveWorkgroups = 25 * kLdsGranule;

static size_t token_walk_reserve(int T, int K, int H) {
    const int64_t bytes = (int64_t)T * K * H * 2;
    if (K < 2 || H < 512) return 0;
    if (bytes >= 112ll << 20) return K > 8 ? kFiveWorkgroups : kSixWorkgroups;
    return K >= 6 && K <= 8 && bytes >= 48ll << 20 ? kFiveWorkgroups : 0;
}

hipError_t launch_dispatch(const DispatchArgs& a, hipStream_t s) {
    const int units = a.H / 8;  // 16-byte units per row
    DispatchPlan d;
    if (plan_dispatch(a.T, a.K, a.H, a.E, a.R, a.order, a.walk != nullptr, a.prefetched_rows, &d)) {
        const int n = a.T * a.K;
        for (int b0 = 0; b0 < d.blocks; b0 += d.blocks_per_launch) {
            const int nb = std::min(d.blocks_per_launch, d.blocks - b0);
            const int64_t e0 = (int64_t)b0 * d.block_entries, e1 = std::min<int64_t>(n, (int64_t)(b0 + nb) * d.block_entries);
            const int t0 = (int)(e0 / a.K), t1 = (int)((e1 + a.K - 1) / a.K);
            // a read pass, unless the layout launch has read these rows already
            if (a.order == EP_ORDER_DESTINATION && t1 > a.prefetched_rows)
                hipLaunchKernelGGL(dispatch_warm_kernel, dim3(2048), dim3(256), 0, s, a, units, t0, t1, b0 == 0 ? 1 : 0);
            launch_walk<false>(a, d, units, (int)e0, (int)e1, StagedRows{}, s);
        }
        return hipGetLastError();
    }
    const int nseg = (units + kWave - 1) / kWave;
    const int64_t nwaves = (int64_t)a.T * nseg;
    int64_t nblk = (nwaves + 3) / 4;
    if (nblk < 1) nblk = 1;  // block 0 also copies the per-expert counts
    if (nblk > 0x7fffffffLL) return hipErrorInvalidValue;
    hipLaunchKernelGGL(dispatch_direct_kernel, dim3((unsigned)nblk), dim3(256), token_walk_reserve(a.T, a.K, a.H), s, a, nseg, units);
    return hipGetLastError();
}

// The quantising dispatch in token order: a row is quantised once for all its destinations.
// (Measured at the prefill shape, 61 us this way.  In the order of the destination rows:
// quantising a row piece again for every destination row is bound by arithmetic, 129 us;
// quantising once into a staging copy by a kernel of its own and copying that in run order,
// 90 us for the two.  Only when the staging copy is made while the layout runs -- see
// launch_dispatch_fp8_staged -- does the copy, 56 us, come out ahead, and the layout launch
// then takes 7 us longer.)
hipError_t launch_dispatch_fp8(const DispatchArgs& a, float* recv_scales, hipStream_t s) {
    const int nseg = (a.H + 1023) / 1024;
    const int64_t nwaves = (int64_t)a.T * nseg;
    int64_t nblk = (nwaves + 3) / 4;
    if (nblk < 1) nblk = 1;
    if (nblk > 0x7fffffffLL) return hipErrorInvalidValue;
    // Rows loaded late where the launch fills the 8192 waves that are resident at a time, or nearly: all of their stores would come at
    // once otherwise.  Dispatch, us, early / late: 8000 waves of 1024 channels, top-8, 18.7/16.5, 8192 waves of 512 12.9/11.1,
    // 8192 of 1024, top-2, 8.3/7.4, 7800 of 1024 to 7168, top-4, 11.8/10.5.  Fewer waves are bound by the round trip (7000 of 7168
    // channels 13.8/14.1, 3500 7.3/7.6), and so are single rows (11 700 of 512, top-1, 7.0/7.3) and short ones (30 000 of 256
    // 24.5/26.6).  In longer launches the waves are apart by themselves: top-4 and more rows of 1 KiB still gain (15 600 waves, top-4,
    // 21.3/20.7, 36 600 48.3/46.4, 30 000, top-8, 63.0/62.5), others lose (15 600 of 512, top-4, 13.1/13.9, 62 500, top-2, 30.7/34.0,
    // 31 000 of 1024, top-2, 26.3/26.7).
    const bool late = nwaves >= 7680 && (nwaves < 12288 ? a.K > 1 && a.H >= 512 : a.K >= 4 && a.H >= 1024);
    if (late) hipLaunchKernelGGL(dispatch_fp8_kernel<true>, dim3((unsigned)nblk), dim3(256), 0, s, a, recv_scales, nseg);
    else hipLaunchKernelGGL(dispatch_fp8_kernel<false>, dim3((unsigned)nblk), dim3(256), 0, s, a, recv_scales, nseg);
    return hipGetLastError();
}

bool dispatch_fp8_staged_possible(const DispatchArgs& a) {
    DispatchPlan d;
    return a.H % 128 == 0 && plan_dispatch_fp8_staged(a.T, a.K, a.H, a.E, a.R, a.walk != nullptr, &d);
}

hipError_t launch_dispatch_fp8_staged(const DispatchArgs& a, float* recv_scales, const uint8_t* staged, int64_t pitch,
                                      hipStream_t s) {
    DispatchPlan d;
    if (a.H % 128 != 0 || !plan_dispatch_fp8_staged(a.T, a.K, a.H, a.E, a.R, a.walk != nullptr, &d)) return hipErrorInvalidValue;
    const StagedRows f = {staged, pitch, recv_scales, fp8_code_units(a.H), a.H / 128};
    // the staged rows were written just before, nothing to read ahead
    const int64_t n = (int64_t)a.T * a.K, step = (int64_t)d.blocks_per_launch * d.block_entries;
    for (int64_t e0 = 0; e0 < n; e0 += step) launch_walk<true>(a, d, fp8_row_units(a.H), (int)e0, (int)std::min(n, e0 + step), f, s);
    return hipGetLastError();
}

}  // namespace ep
