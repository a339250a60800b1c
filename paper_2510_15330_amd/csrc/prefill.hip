// Prompt (prefill) path over the paged KV cache: the write of a prompt's
// keys and values into its pages, and causal prompt attention (each query
// token attends every cached token up to its own position), for gfx950.
//
// The paper's serving loop (Sec. 3 "Our key proposal", Sec. 4 "Setup and
// trace") prefills each queued request's prompt before decoding; the
// prefill's cost sets the time to first token.  The attention is a dense
// contraction (QK^T and PV over head_dim and keys), so it runs on
// v_mfma_f32_32x32x16_bf16, with the keys and values staged through LDS and
// shared by the workgroup's four waves.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <type_traits>

#include "../../include/bellman.h"
#include "internal.h"
#include "wave_scan.h"

namespace bellman {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ float swap_halves(float x) {  // value of lane l ^ 32
    const unsigned u = __float_as_uint(x);
    // the swap exchanges the first operand's lanes 32..63 with the second
    // operand's lanes 0..31: the upper half finds its partner in r[0], the
    // lower half in r[1]
    const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return __uint_as_float((threadIdx.x & 32) ? r[0] : r[1]);
}

// ----------------------------------------------------------- prompt write --
// Work is cut by (request, page the request's new positions touch, KV head):
// write_plan_kernel scans the touched-page counts of the requests into
// page_start[0..B]; kv_write_kernel takes one item per workgroup.  A K page
// [D/x chunks][16 slots][x] takes 16-byte units with consecutive threads on
// consecutive slots; the V rows of the page's tokens go through LDS and
// leave as 16-byte runs of the dim-major V page [D][16 slots] (element by
// element where the page is only partly written).  Lengths are advanced
// afterwards by lens_kernel, so every item sees its request's old length.
// Up to 64 requests there is no such launch: every wave counts the touched
// pages itself, a request a lane.
constexpr int kPlanThreads = 1024;

// Inclusive scan of one value per thread over a kPlanThreads block.
__device__ __forceinline__ int block_scan(int v, int* part) {
    const int tid = threadIdx.x;
    part[tid] = v;
    __syncthreads();
    for (int off = 1; off < kPlanThreads; off <<= 1) {
        const int x = tid >= off ? part[tid - off] : 0;
        __syncthreads();
        part[tid] += x;
        __syncthreads();
    }
    return part[tid];
}

// Pages a request's new positions touch (token rows s0 .. s1 - 1 after L
// cached ones), or -1 for a malformed request (negative or reversed range,
// rows past T, negative length).
__device__ __forceinline__ int pages_touched(const WriteArgs& a, int s0, int s1, int L) {
    if (s0 < 0 || s1 < s0 || s1 > a.T || L < 0) return -1;
    if (s1 == s0) return 0;
    const int64_t last = (int64_t)L + (s1 - s0) - 1;
    return (int)(last / kPage - L / kPage + 1);
}

__global__ void __launch_bounds__(kPlanThreads) write_plan_kernel(WriteArgs a, int32_t* page_start) {
    __shared__ int part[kPlanThreads];
    __shared__ int malformed;
    const int tid = threadIdx.x;
    if (tid == 0) malformed = (a.q_start[0] < 0 || a.q_start[a.B] > a.T) ? 1 : 0;
    __syncthreads();
    const int per = (a.B + kPlanThreads - 1) / kPlanThreads;
    const int b0 = tid * per;
    int sum = 0, bad = 0;
    for (int k = 0; k < per; ++k) {
        const int b = b0 + k;
        if (b >= a.B) break;
        if (a.q_start[b + 1] < a.q_start[b]) atomicOr(&malformed, 1);
        const int t = pages_touched(a, a.q_start[b], a.q_start[b + 1], a.seq_lens[b]);
        if (t < 0) bad = 1;
        else sum += t;
    }
    if (bad) atomicOr(a.err, kErrAppendSlot);
    const int incl = block_scan(sum, part);
    if (malformed) {
        for (int k = 0; k < per; ++k)
            if (b0 + k < a.B) page_start[b0 + k] = 0;
        if (tid == 0) {
            page_start[a.B] = 0;
            atomicOr(a.err, kErrAppendSlot);
        }
        return;
    }
    int run = incl - sum;
    for (int k = 0; k < per; ++k) {
        const int b = b0 + k;
        if (b < a.B) {
            page_start[b] = run;
            run += max(pages_touched(a, a.q_start[b], a.q_start[b + 1], a.seq_lens[b]), 0);
        }
    }
    if (tid == kPlanThreads - 1) {
        page_start[a.B] = incl;
        if (a.q_start[a.B] < a.T) atomicOr(a.err, kErrAppendSlot);   // rows no request owns
    }
}

template <int EB>
__global__ void __launch_bounds__(256) kv_write_kernel(WriteArgs a, const int32_t* page_start) {
    __shared__ __attribute__((aligned(16))) uint8_t vst[kPage * 128 * 2];   // the page's V rows, one head
    const int item = blockIdx.x, tid = threadIdx.x;
    int b, s0, L, n, pi;
    if (a.B <= 64) {
        // the plan, as write_plan_kernel makes it
        const int lane = tid & 63;
        int q0 = 0, q1 = 0, Lb = 0, pages = 0;
        if (lane < a.B) {
            q0 = a.q_start[lane];
            q1 = a.q_start[lane + 1];
            Lb = a.seq_lens[lane];
            pages = pages_touched(a, q0, q1, Lb);
        }
        const int last = __builtin_amdgcn_readlane(q1, a.B - 1);
        const bool malformed = __builtin_amdgcn_readlane(q0, 0) < 0 || last > a.T || __ballot(q1 < q0) != 0;
        if (item == 0 && blockIdx.y == 0 && tid < 64 && (malformed || last < a.T || __ballot(pages < 0) != 0) && lane == 0)
            atomicOr(a.err, kErrAppendSlot);
        if (malformed) return;
        const int end = lane_scan(max(pages, 0));
        if (item >= __builtin_amdgcn_readlane(end, 63)) return;
        b = __ffsll((unsigned long long)__ballot(item < end)) - 1;      // the first whose pages end past item
        s0 = __builtin_amdgcn_readlane(q0, b);
        L = __builtin_amdgcn_readlane(Lb, b);
        n = __builtin_amdgcn_readlane(q1, b) - s0;
        pi = L / kPage + (item - (__builtin_amdgcn_readlane(end, b) - __builtin_amdgcn_readlane(pages, b)));
    } else {
        if (item >= page_start[a.B]) return;
        int lo = 0, hi = a.B - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (page_start[mid] <= item) lo = mid;
            else hi = mid - 1;
        }
        b = lo;
        s0 = a.q_start[b];
        L = a.seq_lens[b];
        n = a.q_start[b + 1] - s0;
        pi = L / kPage + (item - page_start[b]);
    }
    const int64_t first = (int64_t)kPage * pi;              // position of slot 0
    const int slot_lo = (int)(max((int64_t)L, first) - first);
    const int slot_hi = (int)(min((int64_t)L + n, first + kPage) - first);
    int pg = -1;
    if (pi < a.max_pages) pg = a.block_table[(int64_t)b * a.bt_stride + pi];
    if (pg < 0 || pg >= a.num_pages) {
        if (blockIdx.y == 0 && tid == 0) atomicOr(a.err, kErrAppendSlot);
        return;
    }
    const int64_t row0 = s0 + (first - L);                   // token row of slot 0
    constexpr int x = 16 / EB;                               // elements per 16-byte unit
    const int chunks = a.D / x;
    const char* kn = (const char*)a.k_new;
    const char* vn = (const char*)a.v_new;
    for (int g = blockIdx.y; g < a.H_kv; g += gridDim.y) {
        if (g != (int)blockIdx.y) __syncthreads();           // the last head's rows have been read
        char* kp = (char*)a.k_pages + ((int64_t)pg * a.H_kv + g) * (int64_t)a.D * kPage * EB;
        char* vp = (char*)a.v_pages + ((int64_t)pg * a.H_kv + g) * (int64_t)a.D * kPage * EB;
        for (int u = tid; u < chunks * kPage; u += 256) {
            const int c = u / kPage, sl = u % kPage;
            if (sl < slot_lo || sl >= slot_hi) continue;
            const char* src = kn + ((row0 + sl) * a.k_st + (int64_t)g * a.k_sh + (int64_t)c * x) * EB;
            *(u32x4*)(kp + (int64_t)u * 16) = *(const u32x4*)src;
        }
        const int row_units = a.D * EB / 16;                     // 16-byte units of one token's V row
        for (int u = tid; u < kPage * row_units; u += 256) {
            const int sl = u / row_units, k = u % row_units;
            if (sl < slot_lo || sl >= slot_hi) continue;
            *(u32x4*)&vst[u * 16] = *(const u32x4*)(vn + ((row0 + sl) * a.v_st + (int64_t)g * a.v_sh) * EB + k * 16);
        }
        __syncthreads();
        // V page rows: unit (d, h) holds slots h x .. h x + x - 1 of dim d
        const int row_bytes = a.D * EB;
        for (int u = tid; u < a.D * EB; u += 256) {
            const int d = u / EB, h = u % EB;
            const int sa = h * x;
            char* dst = vp + (int64_t)u * 16;
            if (sa >= slot_lo && sa + x <= slot_hi) {
                uint8_t buf[16];
#pragma unroll
                for (int e = 0; e < x; ++e)
#pragma unroll
                    for (int q = 0; q < EB; ++q) buf[e * EB + q] = vst[(sa + e) * row_bytes + d * EB + q];
                *(u32x4*)dst = *(const u32x4*)buf;
            } else {
                for (int sl = max(sa, slot_lo); sl < min(sa + x, slot_hi); ++sl)
                    for (int q = 0; q < EB; ++q) dst[(sl - sa) * EB + q] = (char)vst[sl * row_bytes + d * EB + q];
            }
        }
    }
}

// Each request's length grows by its token count (when its last position
// fits the table).
__global__ void lens_kernel(WriteArgs a) {
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= a.B) return;
    const int n = a.q_start[b + 1] - a.q_start[b];
    const int L = a.seq_lens[b];
    if (n < 0 || L < 0 || (int64_t)L + n > (int64_t)a.max_pages * kPage || a.q_start[b + 1] > a.T) {
        atomicOr(a.err, kErrAppendSlot);
        return;
    }
    a.seq_lens[b] = L + n;
}

// --------------------------------------------------------------- planning --
// A request's query rows are its n_b tokens x the G query heads of a KV
// head, token-major (row r: token r / G, head r % G): tiles of 128 rows,
// whose heads share the KV head's keys.  A request whose range is malformed
// (longer than its length, or a length past the table) gets no tiles and a
// flag; a q_start that is not non-decreasing from a non-negative start up to
// at most T gives no request any tile (so the tiles always fit the grid).
//
// Where the tiles x KV heads are too few to fill the CUs, the keys of a
// tile are cut too: request b's tiles take S_b units each, unit k the steps
// [nt k / S_b, nt (k + 1) / S_b) of the tile's nt, and a second pass merges
// them.  Units per KV head are numbered request by request, within one by
// (key chunk, tile), so that neighbours read the same keys.
//
// Up to 64 requests every wave plans for itself from the lengths, a request
// a lane (a planning launch took 5-6 us, and what a workgroup read back from
// it as many round trips); beyond, prefill_plan_kernel does (no key split: 64
// requests of 30 new tokens after 500 take 56 us, 65 67, as against 100 and
// 102 with rows of one query head each; 100 after 3,000 301 and 312 us).
//
// Measured, whole prompt steps, against rows of one query head each, no key
// split and the planning launch: one 2048-token chunk after 4,900 tokens on
// 4/2 heads (64 tiles: 512 units of 14 steps) 171 -> 56 us, the attention
// alone 141 -> 41 us and 8 us of merge (256 units: 50 + 6 us); eight chats'
// 16-256 new tokens after 2-8k (336 tiles instead of 416, 488 units) 205 ->
// 163 us; four prompts of 6-12k (7584 tiles, never cut) 2017 and 2006 us,
// within the spread of runs.
struct ReqPlan {
    int q0, n, L, tiles, steps;   // steps: 64-key steps of its keys; 0 with no tiles
    bool bad;
};
__device__ __forceinline__ ReqPlan plan_request(const PrefillArgs& a, int b) {
    ReqPlan r;
    r.q0 = a.q_start[b];
    r.n = a.q_start[b + 1] - r.q0;
    r.L = a.seq_lens[b];
    r.bad = r.n < 0 || r.n > r.L || (int64_t)r.L > (int64_t)a.max_pages * kPage;
    r.tiles = r.bad ? 0 : (int)(((int64_t)r.n * a.G + kPrefillRows - 1) / kPrefillRows);
    r.steps = r.tiles > 0 ? (r.L + kPrefillKeys - 1) / kPrefillKeys : 0;
    return r;
}

__device__ __forceinline__ int lane_sum(int v) { return __builtin_amdgcn_readlane(lane_scan(v), 63); }

// The plan of a batch of at most 64 requests, a request a lane.
struct WavePlan {
    ReqPlan r;
    int S;          // units a tile
    int u_end;      // inclusive scan of the requests' units per KV head
    int units;      // units per KV head
    int chunk;      // steps of a key-split unit
    // known: the chunk, 0 to find it (the merge reads what the attention
    // found: the search is a third of its plan); without `cut` the units are
    // not needed
    __device__ __forceinline__ WavePlan(const PrefillArgs& a, bool cut, int known) {
        const int lane = threadIdx.x & 63;
        r = ReqPlan{0, 0, 0, 0, 0, false};
        if (lane < a.B) r = plan_request(a, lane);
        const int first = __builtin_amdgcn_readlane(r.q0, 0);
        const int last = __builtin_amdgcn_readlane(r.q0 + r.n, a.B - 1);
        const bool malformed = first < 0 || last > a.T || __ballot(r.n < 0) != 0;
        if (blockIdx.x == 0 && threadIdx.x < 64 && (malformed || __ballot(r.bad) != 0) && lane == 0)
            atomicOr(a.err, kErrLength);
        if (malformed) r.tiles = r.steps = 0;
        S = 1;
        chunk = known;
        if (cut && chunk == 0) {
            // the smallest chunk of C steps at which the units still run in
            // as few rounds as the tiles do (see the host's rule)
            const int items = lane_sum(r.tiles) * a.H_kv;
            const int target = (items + a.slots - 1) / a.slots * a.slots;
            // from the even deal of all steps up: rounding up costs a unit more
            // for each tile at most (long requests: the deal of their whole
            // 1024 steps, which keeps the sums inside 32 bits)
            const int long_steps = lane_sum(r.tiles * (r.steps >> 10));
            const int64_t steps = long_steps > 0 ? (int64_t)long_steps << 10 : lane_sum(r.tiles * r.steps);
            int lo = max(kPrefillMinChunk, (int)(steps * a.H_kv / max(target, 1))), hi = lo;
            while (lane_sum(r.tiles * ((r.steps + hi - 1) / hi)) * a.H_kv > target) {
                lo = hi + 1;
                hi += (hi >> 2) + 1;
            }
            while (lo < hi) {
                const int mid = (lo + hi) >> 1;
                if (lane_sum(r.tiles * ((r.steps + mid - 1) / mid)) * a.H_kv <= target) hi = mid;
                else lo = mid + 1;
            }
            chunk = lo;
        }
        if (cut) S = max((r.steps + chunk - 1) / chunk, 1);
        u_end = lane_scan(r.tiles * S);
        units = __builtin_amdgcn_readlane(u_end, 63);
    }
};

__global__ void __launch_bounds__(kPlanThreads) prefill_plan_kernel(PrefillArgs a) {
    __shared__ int part[kPlanThreads];
    __shared__ int malformed;
    __shared__ int total_steps;
    const int tid = threadIdx.x;
    if (tid == 0) malformed = (a.q_start[0] < 0 || a.q_start[a.B] > a.T) ? 1 : 0;
    __syncthreads();
    const int per = (a.B + kPlanThreads - 1) / kPlanThreads;
    const int b0 = tid * per;
    int sum = 0, bad = 0;
    for (int k = 0; k < per; ++k) {
        const int b = b0 + k;
        if (b >= a.B) break;
        const ReqPlan r = plan_request(a, b);
        if (r.n < 0) atomicOr(&malformed, 1);
        if (r.bad) bad = 1;
        sum += r.tiles;
    }
    if (bad) atomicOr(a.err, kErrLength);
    const int incl = block_scan(sum, part);
    if (!a.fp8) {
        // bf16 pools: the steps the value copy holds (every step of a request
        // with query tiles, none of the others; none at all when malformed)
        int steps = 0;
        for (int k = 0; k < per; ++k)
            if (b0 + k < a.B && !malformed) steps += plan_request(a, b0 + k).steps;
        const int sincl = block_scan(steps, part);
        int srun = sincl - steps;
        for (int k = 0; k < per; ++k) {
            const int b = b0 + k;
            if (b < a.B) {
                a.step_off[b] = srun;
                srun += malformed ? 0 : plan_request(a, b).steps;
            }
        }
        if (tid == kPlanThreads - 1) {
            a.step_off[a.B] = sincl;
            total_steps = sincl;
        }
        __syncthreads();   // step_off is read back below by every thread
        // the request of every copied step: the last b with step_off[b] <= p
        for (int p = tid; p < total_steps; p += kPlanThreads) {
            int lo = 0, hi = a.B - 1;
            while (lo < hi) {
                const int mid = (lo + hi + 1) >> 1;
                if (a.step_off[mid] <= p) lo = mid;
                else hi = mid - 1;
            }
            a.step_req[p] = lo;
        }
    }
    if (malformed) {
        for (int k = 0; k < per; ++k)
            if (b0 + k < a.B) a.tile_start[b0 + k] = 0;
        if (tid == 0) {
            a.tile_start[a.B] = 0;
            atomicOr(a.err, kErrLength);
        }
        return;
    }
    int run = incl - sum;
    for (int k = 0; k < per; ++k) {
        const int b = b0 + k;
        if (b < a.B) {
            a.tile_start[b] = run;
            run += plan_request(a, b).tiles;
        }
    }
    if (tid == kPlanThreads - 1) a.tile_start[a.B] = incl;
}

// ------------------------------------------------ fp16 copy of bf16 values --
// Over bf16 pools PV runs in fp16, in one pass (P, below 2^8, keeps 11
// significant bits in fp16; rounded to bf16 once it would spend the bf16
// error budget).  The values of every (64-key step, KV head) are copied into
// the workspace as fp16 at a power-of-two scale 2^e of their own that puts
// their largest magnitude M in [2^14, 2^15): bf16's 8 significant bits fit
// fp16's 11, so every value of at least M 2^-28 converts exactly and none
// overflows, and the rest keep an absolute error below M 2^-40.  A step's
// four pages [D][16 slots] are contiguous, a request's steps consecutive,
// slots past its length zero.  A scale a step needs one pass over the values
// (a scale a (request, head) took three: the maximum of every tile, of every
// (request, head), then the copy; 46 against 32 us on 36k tokens of 8 heads);
// the attention holds its output at the finest step's scale and works what a
// coarser step's is below that into its weights.
constexpr int kAnyExp = 1 << 20;   // the step's values are all zero: any scale holds

// the scale exponent e for a largest magnitude whose float bits are mb
// (e = 0 when the maximum is not finite)
__device__ __forceinline__ int vcopy_exp(uint32_t mb) {
    if (mb == 0u) return kAnyExp;
    if (mb >= 0x7f800000u) return 0;
    const int E = max((int)(mb >> 23), 1);          // floor(log2 M) + 127
    return min(max(141 - E, -126), 126);
}
__device__ __forceinline__ float pow2f(int e) {   // 2^e, -126 <= e <= 127
    return __uint_as_float((uint32_t)(e + 127) << 23);
}

// One (step, KV head) at a time per workgroup, wave w its page w; each lane
// takes 4 (D = 128) or 2 16-byte units (8 slots of one dim row) of the page,
// all loaded before any is used.  Bound by memory: V read once, the copy
// written once.
template <int D>
__global__ void __launch_bounds__(256) vcopy_kernel(PrefillArgs a) {
    constexpr int U = 2 * D / 64;   // units per lane
    __shared__ float wmax[2][4];
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const bool self = a.B <= 64;
    int s_end = 0, total, Lb = 0;
    if (self) {
        const WavePlan p(a, false, 0);
        s_end = lane_scan(p.r.steps);
        total = __builtin_amdgcn_readlane(s_end, 63);
        s_end -= p.r.steps;         // first step of this lane's request
        Lb = p.r.steps > 0 ? p.r.L : 0;
    } else {
        total = a.step_off[a.B];
    }
    int par = 0;
    for (int64_t t = blockIdx.x; t < (int64_t)total * a.H_kv; t += gridDim.x, par ^= 1) {
        const int p = (int)(t / a.H_kv), g = (int)(t % a.H_kv);
        int b, j, L;
        if (self) {
            // the last request with steps that starts at or before p
            const uint64_t m = __ballot(Lb > 0 && s_end <= p);
            b = 63 - __clzll((long long)m);
            j = p - __builtin_amdgcn_readlane(s_end, b);
            L = __builtin_amdgcn_readlane(Lb, b);
        } else {
            b = a.step_req[p];
            j = p - a.step_off[b];
            L = a.seq_lens[b];
        }
        const int pi = (kPrefillKeys / kPage) * j + w;     // this wave's page of the request
        const bool inside = kPage * (int64_t)pi < L;
        const int pg = inside ? a.block_table[(int64_t)b * a.bt_stride + pi] : -1;
        const bool ok = (unsigned)pg < (unsigned)a.num_pages;
        const uint16_t* src = (const uint16_t*)a.v_pages + ((int64_t)(ok ? pg : 0) * a.H_kv + g) * (D * kPage);
        u32x4 v[U];
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const int r = 64 * k + lane, live = L - kPage * pi - 8 * (r & 1);   // slots below the length
            v[k] = ok && live > 0 ? *(const u32x4*)(src + (r >> 1) * kPage + 8 * (r & 1)) : u32x4{0u, 0u, 0u, 0u};
            if (live < 8) {
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    v[k][i] &= (2 * i + 1 < live ? 0xffffffffu : 2 * i < live ? 0x0000ffffu : 0u);
            }
        }
        float m = 0.f;
#pragma unroll
        for (int k = 0; k < U; ++k)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                m = fmaxf(m, fmaxf(fabsf(__uint_as_float(v[k][i] << 16)), fabsf(__uint_as_float(v[k][i] & 0xffff0000u))));
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) m = fmaxf(m, __shfl_xor(m, o, 64));
        if (lane == 0) wmax[par][w] = m;
        __syncthreads();            // two sets in turn: the next step's writes cannot pass this step's reads
        m = fmaxf(fmaxf(wmax[par][0], wmax[par][1]), fmaxf(wmax[par][2], wmax[par][3]));
        const int e = vcopy_exp(__float_as_uint(m));
        if (threadIdx.x == 0) a.vexp[t] = e;
        const float sc = e == kAnyExp ? 1.f : pow2f(e);
        uint16_t* dst = a.vcopy + (t * (kPrefillKeys / kPage) + w) * (int64_t)(D * kPage);
#pragma unroll
        for (int k = 0; k < U; ++k) {
            u32x4 h;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const f32x2 x = {__uint_as_float(v[k][i] << 16) * sc, __uint_as_float(v[k][i] & 0xffff0000u) * sc};
                h[i] = __builtin_bit_cast(uint32_t, __builtin_convertvector(x, f16x2));   // round to nearest even
            }
            *(u32x4*)(dst + (64 * k + lane) * 8) = h;
        }
    }
}

// -------------------------------------------------------------- attention --
// Workgroup = a unit of the plan: 128 query rows of one request and KV head
// over a range of its keys; wave w owns rows 32w..32w+31.  Keys go by steps
// of 64 (four pages).  The step's K and V tiles are copied from the pool
// (bf16 pools: V from its fp16 copy) straight into LDS (global_load_lds, 16
// bytes a lane) in the pool's own layout (K [page][D/8 chunks][16 slots][8],
// V [page][D][16 slots], both XOR-swizzled against bank conflicts by the
// choice of unit each lane fetches), double-buffered in four separate arrays
// (so no read of one buffer waits on a copy into another), with K one step
// ahead of V, and read by all four waves.
//
// S^T = K Q^T on 32x32x16 MFMAs: A = 32 keys x 16 dims from LDS, B = the
// wave's 32 query columns, held in registers for the whole kernel.  A's row i
// holds key pi(i) = 16 (i / 16) + 8 ((i / 4) % 2) + 4 ((i / 8) % 2) + i % 4,
// which leaves lane (h, c) (h = lane / 32) of the result with query c and the
// keys 16 u + 8 h + 0..7 for u = 0, 1: the row max needs only the partner lane
// c + 32, and the lane's probabilities are exactly the B operand of
// O^T += V^T P^T for the 16 keys of page u, whose V^T elements are one
// 16-byte run of each dim-major V row.  Online softmax in base 2 with a lazy
// max: O and l are rescaled only when some column's max grows by more than
// 2^8, so P stays below 2^8.  P enters as fp16, rounded once (2^-12 of each
// weight above 2^-14, against the output's own 2^-9).
//
// The loop is software-pipelined: step s masks and takes the max of S(s)
// (computed one step earlier), then issues the MFMAs of S(s + 1)
// interleaved with the exponentials of P(s), then the PV MFMAs of step s.
constexpr float kLazyMax = 8.0f;
// bf16 pools: O is held at a scale 2^eref, never coarser than the step at
// hand, so that no weight is made smaller before it is rounded to fp16 (whose
// numbers below 2^-14 lose a bit a factor of two): O moves up to a finer
// step's scale, and a coarser step's weights are multiplied by up to 2^7 (P,
// below 2^8, stays inside fp16) before O moves down to it.  Holding O at the
// first step's scale and multiplying finer steps' weights by 2^-d instead
// left them 11 - (d - 14) bits: rows made of values 2^20 finer than a large
// step of small weight came out 0.1 to 0.3 off, and now 2e-3 (their bf16
// rounding); four prompts of 6-12k tokens 2017 and 2021 us, runs 1.3% apart.
// O stays within 2^64 of the coarsest step seen (2^64 2^15 values at weights
// of 2^8 from 2^24 keys stay inside fp32); values finer still, below M 2^-63,
// take smaller weights.
constexpr int kMaxCoarser = 7, kMaxRise = 64;
constexpr int kPageWindow = 1024;   // block-table entries staged in LDS
constexpr int kXcds = 8;            // accelerator complexes; workgroup i runs on XCD i % 8
// VALU instructions of the softmax placed between consecutive S MFMAs
constexpr int kValuPerMfma = 7;

// FP8: pools of e4m3fn codes with per-(request, KV head) dequantisation
// scales.  The tiles reach LDS as codes (half the bytes) and each operand is
// widened exactly to bf16 before the same bf16 MFMAs; the K scale folds into
// the score scale and the V scale into the final normalisation.  A lane
// reads one whole 16-byte unit and feeds two MFMAs with its halves:
//  * S: A row i holds key pi8(i) = 16 ((i / 4) % 2) + 8 (i / 16) +
//    4 ((i / 8) % 2) + i % 4, so lane (h, c) of the result holds the keys
//    16 h + 8 e + 0..7 (e = 0, 1) of each 32-key half: page h of the half.
//    MFMA pair (2 m, 2 m + 1) reads, in lane (h, c), the unit of chunk
//    2 m + h of key pi8(c) and takes its codes 8 e .. 8 e + 7 into MFMA
//    2 m + e; the query operand of MFMA 2 m + e holds dims 32 m + 16 h + 8 e.
//  * PV: lane (h, c) reads row 32 t + c of page h of the half (16 keys) and
//    takes keys 8 e .. 8 e + 7 into MFMA e, whose P operand is then exactly
//    the lane's probabilities of group e.  PV runs in fp16, one pass: the
//    codes (at most 448 in magnitude, subnormals from 2^-9) are exact in
//    fp16, and P (below 2^8 with the lazy max) keeps 11 significant bits
//    there, against the bf16 hi + lo pair's two passes.
// Pages sit PB + 128 bytes apart in LDS and odd pages hold K slot s at
// s ^ 4, so every 8 (and 16) consecutive lanes of a read touch distinct
// banks.
template <int D, int NH, bool FP8>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2)))
prefill_attn_kernel(PrefillArgs a) {
    constexpr int KS = 32 * NH;         // keys per step
    constexpr int PPS = KS / kPage;     // pages per step
    constexpr int EB = FP8 ? 1 : 2;     // bytes per pool element
    constexpr int PE = D * kPage;       // elements of one page of one head (K or V)
    constexpr int PB = PE * EB;         // its bytes
    constexpr int KT = PPS * PE;        // a step's K (or V) tile, elements
    constexpr int PBP = FP8 ? PB + 128 : PB;   // LDS bytes from one page of a tile to the next
    constexpr int KTW = PPS * PBP / 2;  // the tile in 16-bit words
    constexpr int UPP = PB / 16;        // 16-byte units per page
    constexpr int PER = 2 * PPS * UPP / 256;   // units of K + V per thread per step
    constexpr int WIN = kPageWindow / PPS;     // steps per block-table window
    __shared__ __attribute__((aligned(16))) uint16_t kb0[KTW];
    __shared__ __attribute__((aligned(16))) uint16_t kb1[KTW];
    __shared__ __attribute__((aligned(16))) uint16_t vb0[KTW];
    __shared__ __attribute__((aligned(16))) uint16_t vb1[KTW];
    __shared__ int pages[kPageWindow];
    __shared__ int vexps[FP8 ? 1 : WIN];

    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 31, hl = lane >> 5;
    // work item r = g * units + i: KV head g, its i-th unit from the end (the
    // longest first).  Each of the 8 XCDs (workgroups go to XCD blockIdx % 8)
    // takes a contiguous share of the items, so the neighbouring tiles that
    // stream the same keys and values run together and share that XCD's L2.
    int units, b = 0, u0 = 0, S = 1, vstep0 = 0;
    ReqPlan rq;
    const int kq = (int)blockIdx.x / kXcds, xcd = (int)blockIdx.x % kXcds;
    int r, g;
    if (a.B <= 64) {
        const WavePlan p(a, a.split, 0);
        units = p.units;
        if (a.split && blockIdx.x == 0 && tid == 0) *a.chunk = p.chunk;
        const int items = units * a.H_kv, share = (items + kXcds - 1) / kXcds;
        r = xcd * share + kq;
        if (kq >= share || r >= items) return;
        g = r / units;
        const int x = units - 1 - (r - g * units);
        const int mine = p.r.tiles * p.S;
        b = __ffsll((unsigned long long)__ballot(x < p.u_end)) - 1;    // the first whose units end past x
        u0 = x - (__builtin_amdgcn_readlane(p.u_end, b) - __builtin_amdgcn_readlane(mine, b));
        S = __builtin_amdgcn_readlane(p.S, b);
        rq.q0 = __builtin_amdgcn_readlane(p.r.q0, b);
        rq.n = __builtin_amdgcn_readlane(p.r.n, b);
        rq.L = __builtin_amdgcn_readlane(p.r.L, b);
        rq.tiles = __builtin_amdgcn_readlane(p.r.tiles, b);
        if (!FP8) vstep0 = __builtin_amdgcn_readlane(lane_scan(p.r.steps) - p.r.steps, b);
    } else {
        units = a.tile_start[a.B];
        const int items = units * a.H_kv, share = (items + kXcds - 1) / kXcds;
        r = xcd * share + kq;
        if (kq >= share || r >= items) return;
        g = r / units;
        const int x = units - 1 - (r - g * units);
        int lo = 0, hi = a.B - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (a.tile_start[mid] <= x) lo = mid;
            else hi = mid - 1;
        }
        b = lo;
        rq = plan_request(a, b);
        u0 = x - a.tile_start[b];
        if (!FP8) vstep0 = a.step_off[b];
    }
    const int chunk = u0 / rq.tiles, tile = u0 - chunk * rq.tiles;
    const int t0 = rq.q0, n = rq.n, L = rq.L;
    const int p0 = L - n;                          // position of query token 0
    // rows tile 128 .. of the request's n G: the tile's first token and head
    const int64_t rows_b = (int64_t)n * a.G, row_t = (int64_t)tile * kPrefillRows;
    const int rows = (int)min(rows_b - row_t, (int64_t)kPrefillRows);
    const int tok0 = (int)(row_t / a.G), head0 = (int)(row_t - (int64_t)tok0 * a.G);
    auto token_of = [&](int i) { return tok0 + (int)((unsigned)(head0 + i) / (unsigned)a.G); };
    const int kv_end = p0 + token_of(rows - 1) + 1;   // the tile's keys [0, kv_end)
    const int nsteps = (kv_end + KS - 1) / KS;
    // this unit's steps
    const int s_lo = (int)((int64_t)nsteps * chunk / S), s_hi = (int)((int64_t)nsteps * (chunk + 1) / S);
    const int np = (L + kPage - 1) / kPage;
    const int32_t* bt = a.block_table + (int64_t)b * a.bt_stride;

    const int rw = 32 * w;                         // this wave's first row of the tile
    const int row = min(rw + c, rows - 1);         // padding columns repeat the last row
    const int tok = token_of(row);
    const int h = g * a.G + (head0 + row) - (tok - tok0) * a.G;
    const int pos = p0 + tok;                      // keys 0..pos are visible to this column
    const int pos_w = p0 + token_of(min(rw, rows - 1));   // the wave's first position
    const int wave_steps = rw < rows ? min((p0 + token_of(min(rw + 31, rows - 1))) / KS + 1, s_hi) : 0;

    // softmax(scale * s) = softmax(|scale| * (-s)): for a negative scale the
    // query's sign bits are flipped (the host keeps |scale| >= FLT_MIN).
    // fp8 pools: the scores are dequantised by the (request, head)'s K scale.
    float s_eff = a.scale_log2, v_scale = 1.f;
    if constexpr (FP8) {
        s_eff *= a.k_scale[(int64_t)b * a.H_kv + g];
        v_scale = a.v_scale[(int64_t)b * a.H_kv + g];
    }
    const float sl = fabsf(s_eff);
    bf16x8 qv[D / 16];
    {
        const uint32_t flip = s_eff < 0.f ? 0x80008000u : 0u;
        // the B operand of MFMA kb: dims 16 kb + 8 hl (fp8: 32 (kb / 2) + 16 hl + 8 (kb % 2))
        const uint16_t* qrow = a.q + (int64_t)(t0 + tok) * a.q_st + (int64_t)h * a.q_sh + (FP8 ? 16 : 8) * hl;
#pragma unroll
        for (int kb = 0; kb < D / 16; ++kb) {
            u32x4 v = *(const u32x4*)(qrow + (FP8 ? 32 * (kb >> 1) + 8 * (kb & 1) : 16 * kb));
            v ^= flip;
            qv[kb] = __builtin_bit_cast(bf16x8, v);
        }
    }
    f32x16 o[D / 32];
#pragma unroll
    for (int t = 0; t < D / 32; ++t) o[t] = f32x16{};
    // m starts at the lowest finite value: scores of -inf alone weigh nothing
    // (l = 0), and only a NaN makes l one
    float m = -__FLT_MAX__, l = 0.f;
    bool bad = false;

    // the block-table entries (and value scales) of WIN steps at a time sit in
    // LDS, refilled when no copy is in flight, so a step's pages cost LDS
    // reads only; j a multiple of WIN
    auto refill = [&](int j) {
        // the entries the unit reads, all loads out before any is stored
        const int e0 = max(0, PPS * (s_lo - j)), e1 = min(kPageWindow, PPS * (s_hi - j));
        int pe[kPageWindow / 256], ve = 0;
#pragma unroll
        for (int k = 0; k < kPageWindow / 256; ++k) {
            const int e = 256 * k + tid;
            if (e >= e0 && e < e1) pe[k] = bt[min(PPS * j + e, np - 1)];
        }
        const bool mine = !FP8 && PPS * tid >= e0 && PPS * tid < e1;
        if (mine) ve = a.vexp[(int64_t)(vstep0 + j + tid) * a.H_kv + g];
#pragma unroll
        for (int k = 0; k < kPageWindow / 256; ++k) {
            const int e = 256 * k + tid;
            if (e >= e0 && e < e1) pages[e] = pe[k];
        }
        if (mine) vexps[tid] = ve;
        __syncthreads();
    };
    // unit u = 256 k + tid of a step: tensor u / (PPS UPP) (K, V), page
    // (u / UPP) % PPS, 16-byte unit u % UPP of that page; a wave's 64 units
    // are consecutive and lie in one page.  K runs one step ahead of V: while
    // step s computes, K of step s + 2 and V of step s + 1 are loaded into
    // registers, and written to LDS after it.
    constexpr int PERH = PER / 2;      // units of one tensor per thread per step
    const char* kbase = (const char*)a.k_pages + (int64_t)g * PB;
    const char* vbase = (const char*)a.v_pages + (int64_t)g * PB;
    const int64_t page_bytes = (int64_t)a.H_kv * PB;
    // bf16 pools: the values come from the fp16 copy, whose steps of request b
    // are consecutive from vstep0
    const char* vbase16 = FP8 ? nullptr : (const char*)a.vcopy + ((int64_t)vstep0 * a.H_kv + g) * (PPS * PB);
    int64_t off1[PPS], off2[PPS];      // page byte offsets of steps s + 1 and s + 2
    auto pages_of = [&](int j, int64_t (&off)[PPS]) {
        const int e = PPS * (j % WIN);
#pragma unroll
        for (int q = 0; q < PPS; ++q) {
            int pg = pages[e + q];
            if ((unsigned)pg >= (unsigned)a.num_pages) {
                pg = 0;
                bad = true;
            }
            off[q] = (int64_t)pg * page_bytes;
        }
    };
    // direct copies into LDS: lane l of a wave lands at unit (wave base + l);
    // it fetches the global unit the swizzle maps there (the swizzles are
    // involutions within a page; fp8 tiles are not swizzled)
    auto dma = [&](const char* base, const int64_t (&off)[PPS], uint16_t* dst, bool isv) {
#pragma unroll
        for (int k = 0; k < PERH; ++k) {
            int64_t o_pg;
            if constexpr (FP8) {
                const int u0 = 256 * k + 64 * w;    // this wave's 64 units: one page's units u0 % UPP ..
                const int pp = u0 / UPP;
                // page (256 k) / UPP + (w / (4 / BPP)) of the step, chosen by
                // selects on the wave's bits (no indexed access of off[],
                // which the compiler would stage through memory)
                constexpr int BPP = 256 / UPP;  // pages a round of 256 units covers: 2 (D 128) or 4 (D 64)
                const int p0k = (256 * k) / UPP;
                if constexpr (BPP == 2) {
                    o_pg = (w >> 1) ? off[p0k + 1] : off[p0k];
                } else {
                    const int64_t lo2 = (w & 1) ? off[p0k + 1] : off[p0k];
                    const int64_t hi2 = (w & 1) ? off[p0k + 3] : off[p0k + 2];
                    o_pg = (w & 2) ? hi2 : lo2;
                }
                const int v = u0 % UPP + lane;
                const int vg = (!isv && (pp & 1)) ? v ^ 4 : v;
                __builtin_amdgcn_global_load_lds(base + o_pg + vg * 16, dst + (pp * PBP + (u0 % UPP) * 16) / 2, 16, 0,
                                                 0);
                continue;
            } else {
                constexpr int BPP = 256 / UPP;
                const int pp = (256 * k) / UPP;
                o_pg = off[pp];
                if constexpr (BPP == 2) o_pg = (w >> 1) ? off[pp + 1] : o_pg;
            }
            const int v = ((256 * k + 64 * w) % UPP) + lane;          // LDS unit within its page
            const int vg = FP8 ? v : isv ? v ^ (((v >> 3) ^ (v >> 4)) & 1) : v ^ (((v >> 3) & 1) << 2);
            __builtin_amdgcn_global_load_lds(base + o_pg + vg * 16, dst + 8 * (256 * k + 64 * w), 16, 0, 0);
        }
    };
    // the fp16 value copy of step j (bf16 pools), laid out and swizzled as V
    auto dma_v16 = [&](int j, uint16_t* dst) {
        const char* src = vbase16 + (int64_t)j * a.H_kv * (PPS * PB);
#pragma unroll
        for (int k = 0; k < PERH; ++k) {
            const int v = ((256 * k + 64 * w) % UPP) + lane;
            const int vg = v ^ (((v >> 3) ^ (v >> 4)) & 1);
            __builtin_amdgcn_global_load_lds(src + (256 * k + 64 * w - v + lane + vg) * 16, dst + 8 * (256 * k + 64 * w), 16,
                                             0, 0);
        }
    };
    // fp8: V slots of keys >= L hold no token (NaN in a pool); P is 0 there,
    // and 0 * NaN must not reach O, so the tail step's slots are cleared (the
    // fp16 copy holds zeros there)
    auto clear_tail = [&](int s, uint16_t* V) {
        // codes [page][D][16 slots], pages PBP bytes apart
        uint8_t* Vb = (uint8_t*)V;
        for (int e = tid; e < KT; e += 256) {
            const int key = KS * s + 16 * (e / PE) + (e & 15);
            if (key >= L) Vb[(e / PE) * PBP + e % PE] = 0;
        }
    };

    // lane (h, c) reads A row c = key pi(c) of each 32-key half
    const int kk = 16 * (c >> 4) + 8 * ((c >> 2) & 1) + 4 * ((c >> 3) & 1) + (c & 3);
    const int kslot = (kk & 15) ^ (((kk >> 3) & 1) << 2);
    const int k_off = (kk >> 4) * PE + hl * (kPage * 8) + kslot * 8;
    const int v_off = c * kPage + 8 * (hl ^ (((c >> 2) ^ (c >> 3)) & 1));
    // fp8 (byte offsets): the K unit (chunk 2 m + hl, slot) of key pi8(c),
    // and row c of V page hl, of each 32-key half
    const int kk8 = 16 * ((c >> 2) & 1) + 8 * ((c >> 4) & 1) + 4 * ((c >> 3) & 1) + (c & 3);
    const int k_off8 = (kk8 >> 4) * PBP + hl * 256 + ((kk8 & 15) ^ (4 * (kk8 >> 4))) * 16;
    const int v_off8 = hl * PBP + c * 16;
    // eight codes -> eight bf16, exactly
    auto widen = [](const u32x2 w8) -> bf16x8 {
        const bf16x2 p0 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w8.x, 1.0f, false);
        const bf16x2 p1 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w8.x, 1.0f, true);
        const bf16x2 p2 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w8.y, 1.0f, false);
        const bf16x2 p3 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w8.y, 1.0f, true);
        return __builtin_bit_cast(bf16x8, u32x4{__builtin_bit_cast(uint32_t, p0), __builtin_bit_cast(uint32_t, p1),
                                                __builtin_bit_cast(uint32_t, p2), __builtin_bit_cast(uint32_t, p3)});
    };
    // eight codes -> eight fp16, exactly
    auto widen16 = [](const u32x2 w8) -> f16x8 {
        const f16x2 p0 = __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(w8.x, 1.0f, false);
        const f16x2 p1 = __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(w8.x, 1.0f, true);
        const f16x2 p2 = __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(w8.y, 1.0f, false);
        const f16x2 p3 = __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(w8.y, 1.0f, true);
        return __builtin_bit_cast(f16x8, u32x4{__builtin_bit_cast(uint32_t, p0), __builtin_bit_cast(uint32_t, p1),
                                               __builtin_bit_cast(uint32_t, p2), __builtin_bit_cast(uint32_t, p3)});
    };
    auto k_operand = [&](const uint16_t* Kt, int hh, int kb) -> bf16x8 {
        return *(const bf16x8*)(Kt + k_off + hh * 2 * PE + kb * (2 * kPage * 8));
    };
    auto v_operand = [&](const uint16_t* Vt0, int hh, int u, int t) -> bf16x8 {
        return *(const bf16x8*)(Vt0 + v_off + hh * 2 * PE + (u * D + 32 * t) * kPage);
    };
    // fp8: the 16-byte unit of K pair m, and row 32 t + c of V, of half hh
    auto k_unit8 = [&](const uint16_t* Kt, int hh, int m) -> u32x4 {
        return *(const u32x4*)((const char*)Kt + hh * 2 * PBP + m * 512 + k_off8);
    };
    auto v_row8 = [&](const uint16_t* Vt0, int hh, int t) -> u32x4 {
        return *(const u32x4*)((const char*)Vt0 + hh * 2 * PBP + (32 * t) * 16 + v_off8);
    };

    auto qk = [&](const uint16_t* Kt, f32x16 (&sc)[NH]) {
#pragma unroll
        for (int hh = 0; hh < NH; ++hh) sc[hh] = f32x16{};
        if constexpr (FP8) {
#pragma unroll
            for (int m = 0; m < D / 32; ++m) {
                u32x4 ku[NH];
#pragma unroll
                for (int hh = 0; hh < NH; ++hh) ku[hh] = k_unit8(Kt, hh, m);
#pragma unroll
                for (int e = 0; e < 2; ++e)
#pragma unroll
                    for (int hh = 0; hh < NH; ++hh) {
                        const bf16x8 ka = widen(e ? u32x2{ku[hh].z, ku[hh].w} : u32x2{ku[hh].x, ku[hh].y});
                        sc[hh] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka, qv[2 * m + e], sc[hh], 0, 0, 0);
                    }
            }
        } else {
#pragma unroll
            for (int kb = 0; kb < D / 16; ++kb)
#pragma unroll
                for (int hh = 0; hh < NH; ++hh) {
                    const bf16x8 ka = k_operand(Kt, hh, kb);
                    sc[hh] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka, qv[kb], sc[hh], 0, 0, 0);
                }
        }
    };

    // bf16 pools: the scale exponent of O (kAnyExp while every value was
    // zero), the same in all waves, and the lowest of the steps so far.  e1,
    // e2: the scales of steps s, s + 1 (before step s + 2's is read)
    int eref = kAnyExp, elow = kAnyExp, e1 = kAnyExp, e2 = kAnyExp;
    auto vexp_of = [&](int j) {
        if constexpr (FP8) return 0;
        else return __builtin_amdgcn_readfirstlane(vexps[j % WIN]);
    };

    // prologue: K and V of the first step, K of the next, S of the first
    if (s_lo < s_hi) {
        refill(s_lo / WIN * WIN);
        pages_of(s_lo, off2);
        e1 = vexp_of(s_lo);
        dma(kbase, off2, kb0, false);
        if constexpr (FP8) dma(vbase, off2, vb0, true);
        else dma_v16(s_lo, vb0);
        if (s_lo + 1 < s_hi) {
            if ((s_lo + 1) % WIN == 0) {
                __syncthreads();       // every wave has read the first step's pages
                refill(s_lo + 1);
            }
            pages_of(s_lo + 1, off1);
            e2 = vexp_of(s_lo + 1);
            dma(kbase, off1, kb1, false);
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (FP8 && KS * (s_lo + 1) > L) {
            clear_tail(s_lo, vb0);
            __syncthreads();
        }
    }
    f32x16 sca[NH], scb[NH];
    if (s_lo < wave_steps) qk(kb0, sca);
    // the first step copies K(s + 2) over K(s): every wave's reads of it come first
    __syncthreads();

    // one step; sc holds S(s), scn receives S(s + 1)
    auto step = [&](auto par, const int s, f32x16 (&sc)[NH], f32x16 (&scn)[NH]) {
        constexpr int P = decltype(par)::value;   // (s - s_lo) % 2
        uint16_t* k_rd = P ? kb0 : kb1;   // K(s + 1)
        uint16_t* k_wr = P ? kb1 : kb0;   // K(s + 2), over K(s)
        uint16_t* v_rd = P ? vb1 : vb0;   // V(s)
        uint16_t* v_wr = P ? vb0 : vb1;   // V(s + 1), over V(s - 1)
        const bool more_k = s + 2 < s_hi, more_v = s + 1 < s_hi;
        int e3 = kAnyExp;
        if (more_v) {
            if constexpr (FP8) dma(vbase, off1, v_wr, true);
            else dma_v16(s + 1, v_wr);
        }
        if (more_k) {
            if ((s + 2) % WIN == 0) refill(s + 2);
            pages_of(s + 2, off2);
            e3 = vexp_of(s + 2);
            dma(kbase, off2, k_wr, false);
        }
        // the weights' factor 2^-d of this step, as the exponent's offset, and
        // 2^d, which takes their sum back (d in [-7, 0], above 0 only past
        // kMaxRise)
        float d = 0.f, pd = 1.f;
        if constexpr (!FP8) {
            if (e1 != kAnyExp) {
                elow = min(elow, e1);
                if (eref == kAnyExp) eref = e1;    // O is zero so far
                const int to = min(e1, elow + kMaxRise);
                if (to > eref || to < eref - kMaxCoarser) {
                    const float f = to - eref < -126 ? 0.f : pow2f(to - eref);
#pragma unroll
                    for (int t = 0; t < D / 32; ++t) o[t] *= f;
                    eref = to;
                }
                const int di = min(e1 - eref, kMaxRise);
                d = (float)di;
                pd = pow2f(di);
            }
        }
        uint32_t ph[NH][8];   // P as fp16 pairs
        if (s < wave_steps) {
            // keys above a column's position are masked only on the steps
            // the wave's diagonal crosses
            if (KS * s + KS - 1 > pos_w) {
#pragma unroll
                for (int hh = 0; hh < NH; ++hh)
#pragma unroll
                    for (int j = 0; j < 16; ++j) {
                        const int key = KS * s + 32 * hh + (j & 7) + (FP8 ? 16 * hl + 8 * (j >> 3) : 16 * (j >> 3) + 8 * hl);
                        sc[hh][j] = key <= pos ? sc[hh][j] : -INFINITY;
                    }
            }
            float mx = -INFINITY;
#pragma unroll
            for (int hh = 0; hh < NH; ++hh)
#pragma unroll
                for (int j = 0; j < 16; ++j) mx = fmaxf(mx, sc[hh][j]);
            mx = fmaxf(mx, swap_halves(mx));
            const float m_new = fmaxf(m, mx * sl);     // scaled units
            if (__any(m_new > m + kLazyMax)) {
                const float alpha = __builtin_amdgcn_exp2f(m - m_new);
                l *= alpha;
#pragma unroll
                for (int t = 0; t < D / 32; ++t) o[t] *= alpha;
                m = m_new;
            }
            // S of step s + 1 on the matrix cores while P of step s is formed
            // (past a wave's last step the result is not used)
            qk(k_rd, scn);
            float psum = 0.f;
            const float md = FP8 ? m : m + d;
#pragma unroll
            for (int hh = 0; hh < NH; ++hh)
#pragma unroll
                for (int j = 0; j < 16; j += 2) {
                    const f32x2 pq = {__builtin_amdgcn_exp2f(__builtin_fmaf(sc[hh][j], sl, -md)),
                                      __builtin_amdgcn_exp2f(__builtin_fmaf(sc[hh][j + 1], sl, -md))};
                    psum += pq.x + pq.y;
                    ph[hh][j / 2] = __builtin_bit_cast(uint32_t, __builtin_convertvector(pq, f16x2));   // RNE
                }
            l = FP8 ? l + psum : __builtin_fmaf(psum, pd, l);
            // K reads run two MFMAs ahead of the S MFMAs, with the softmax
            // VALU work spread between them
            // (fp8: one K read per two MFMAs)
            constexpr int KR = FP8 ? 2 : 1;
            __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
#pragma unroll
            for (int i = 0; i < 8 * NH; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);        // an MFMA of S
                if (i % KR == KR - 1 && i / KR + 2 < 8 * NH / KR)
                    __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);   // a K read
                __builtin_amdgcn_sched_group_barrier(0x002, kValuPerMfma, 0);   // softmax VALU
            }
            // O^T += V^T P^T, per 16-key group u of each half and 32-dim tile t
            // (bf16: group u is page u; fp8: keys 8 u .. 8 u + 7 of the
            // lane's page, both groups from one 16-byte V row)
            auto p_operand = [](const uint32_t (&p)[8], int u) {
                return __builtin_bit_cast(f16x8, u32x4{p[4 * u], p[4 * u + 1], p[4 * u + 2], p[4 * u + 3]});
            };
            if constexpr (FP8) {
#pragma unroll
                for (int hh = 0; hh < NH; ++hh)
#pragma unroll
                    for (int t = 0; t < D / 32; ++t) {
                        const u32x4 vr = v_row8(v_rd, hh, t);
#pragma unroll
                        for (int u = 0; u < 2; ++u) {
                            const f16x8 va = widen16(u ? u32x2{vr.z, vr.w} : u32x2{vr.x, vr.y});
                            o[t] = __builtin_amdgcn_mfma_f32_32x32x16_f16(va, p_operand(ph[hh], u), o[t], 0, 0, 0);
                        }
                    }
            } else {
#pragma unroll
                for (int hh = 0; hh < NH; ++hh)
#pragma unroll
                    for (int u = 0; u < 2; ++u) {
                        const f16x8 pa = p_operand(ph[hh], u);
#pragma unroll
                        for (int t = 0; t < D / 32; ++t) {
                            const f16x8 va = __builtin_bit_cast(f16x8, v_operand(v_rd, hh, u, t));
                            o[t] = __builtin_amdgcn_mfma_f32_32x32x16_f16(va, pa, o[t], 0, 0, 0);
                        }
                    }
            }
            // V reads run four MFMAs ahead of the PV MFMAs (fp8: two reads
            // ahead, each feeding two)
            constexpr int MF = FP8 ? 2 : 1;
            constexpr int NV = (FP8 ? 1 : 2) * NH * (D / 32);
            constexpr int VA = FP8 ? 2 : 4;
            __builtin_amdgcn_sched_group_barrier(0x100, VA, 0);
#pragma unroll
            for (int i = 0; i < NV; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x008, MF, 0);
                if (i + VA < NV) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
            }
        }
        if (more_v) {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __syncthreads();
            if (FP8 && KS * (s + 2) > L) {
                clear_tail(s + 1, v_wr);
                __syncthreads();
            }
        }
#pragma unroll
        for (int q = 0; q < PPS; ++q) off1[q] = off2[q];
        e1 = e2;
        e2 = e3;
    };
    // unrolled by two so that S(s) and S(s + 1) alternate between register sets
    for (int s = s_lo; s < s_hi; s += 2) {
        step(std::integral_constant<int, 0>{}, s, sca, scb);
        if (s + 1 < s_hi) step(std::integral_constant<int, 1>{}, s + 1, scb, sca);
    }
    if (bad && lane == 0) atomicOr(a.err, kErrPage);
    if (rw >= rows) return;
    const float l_tot = l + swap_halves(l);
    // fp8: the V scale; bf16: undo the values' scale, in a multiplication of
    // its own (2^-eref / l may be subnormal where the output is not)
    const float f = (FP8 ? v_scale : 1.f) / l_tot, unscale = FP8 || eref == kAnyExp ? 1.f : pow2f(-eref);
    auto out_of = [&](float x) { return FP8 ? x * f : x * f * unscale; };
    if (S > 1) {
        // a piece: its rows' (m, l) and normalised O, in the lanes' own order
        // (dead, m = -inf, where the row sees no key of this unit or scores of
        // -inf alone; a NaN sum stays and poisons the row)
        const int64_t piece = (int64_t)r * 4 + w;
        const bool dead = s_lo >= s_hi || pos < KS * s_lo || l_tot == 0.f;
        if (hl == 0) a.part_ml[piece * 32 + c] = make_float2(dead ? -INFINITY : m, l_tot);
        f32x4* po = (f32x4*)a.part_o + piece * (D / 8) * 64 + lane;
#pragma unroll
        for (int t = 0; t < D / 32; ++t)
#pragma unroll
            for (int r4 = 0; r4 < 4; ++r4)
                po[(4 * t + r4) * 64] = f32x4{out_of(o[t][4 * r4]), out_of(o[t][4 * r4 + 1]), out_of(o[t][4 * r4 + 2]),
                                              out_of(o[t][4 * r4 + 3])};
        return;
    }
    if (rw + c < rows) {
        uint16_t* orow = a.out + (int64_t)(t0 + tok) * a.o_st + (int64_t)h * a.o_sh;
#pragma unroll
        for (int t = 0; t < D / 32; ++t)
#pragma unroll
            for (int r4 = 0; r4 < 4; ++r4) {
                const f32x2 v01 = {out_of(o[t][4 * r4]), out_of(o[t][4 * r4 + 1])};
                const f32x2 v23 = {out_of(o[t][4 * r4 + 2]), out_of(o[t][4 * r4 + 3])};
                u32x2 pk;
                pk.x = __builtin_bit_cast(uint32_t, __builtin_convertvector(v01, bf16x2));
                pk.y = __builtin_bit_cast(uint32_t, __builtin_convertvector(v23, bf16x2));
                *(u32x2*)(orow + 32 * t + 8 * r4 + 4 * hl) = pk;
            }
    }
}

// Merge of the key-split tiles' pieces: a wave takes 32 dims (t) of 32 rows
// (w) of a tile, in the lane order the attention kernel wrote them:
//   M = max_i m_i,  out = sum_i 2^(m_i - M) l_i O_i / sum_i 2^(m_i - M) l_i
// Bound by reading the pieces; every piece's loads are independent.
template <int D>
__global__ void __launch_bounds__(256) prefill_merge_kernel(PrefillArgs a) {
    constexpr int NT = D / 32, WPT = 4 * NT;      // waves a tile
    const int lane = threadIdx.x & 63, c = lane & 31, hl = lane >> 5;
    const WavePlan p(a, true, __builtin_amdgcn_readfirstlane(*a.chunk));
    const int t_end = lane_scan(p.r.tiles);
    const int tiles = __builtin_amdgcn_readlane(t_end, 63);
    const int64_t j = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int item = __builtin_amdgcn_readfirstlane((int)(j / WPT)), q = __builtin_amdgcn_readfirstlane((int)(j % WPT));
    if (tiles == 0 || item >= tiles * a.H_kv) return;
    const int g = item / tiles, x = item - g * tiles;
    const int b = __ffsll((unsigned long long)__ballot(x < t_end)) - 1;
    const int S = __builtin_amdgcn_readlane(p.S, b);
    if (S == 1) return;
    const int tiles_b = __builtin_amdgcn_readlane(p.r.tiles, b), n = __builtin_amdgcn_readlane(p.r.n, b);
    const int tile = x - (__builtin_amdgcn_readlane(t_end, b) - tiles_b);
    const int u0 = __builtin_amdgcn_readlane(p.u_end, b) - tiles_b * S + tile;   // chunk k: u0 + k tiles_b
    const int64_t row_t = (int64_t)tile * kPrefillRows;
    const int rows = (int)min((int64_t)n * a.G - row_t, (int64_t)kPrefillRows);
    const int w = q / NT, t = q - w * NT;
    if (32 * w >= rows) return;
    auto piece = [&](int k) { return ((int64_t)g * p.units + (p.units - 1 - (u0 + k * tiles_b))) * 4 + w; };
    float M = -INFINITY, l = 0.f;
    f32x4 acc[4] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f},
                    f32x4{0.f, 0.f, 0.f, 0.f}};
    constexpr int K = 4;                           // pieces a batch
    for (int k0 = 0; k0 < S; k0 += K) {
        float2 ml[K];
        f32x4 o[K][4];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int64_t pc = piece(min(k0 + k, S - 1));
            ml[k] = a.part_ml[pc * 32 + c];
            if (k0 + k >= S) ml[k].x = -INFINITY;
#pragma unroll
            for (int r4 = 0; r4 < 4; ++r4) o[k][r4] = *((const f32x4*)a.part_o + (pc * (D / 8) + 4 * t + r4) * 64 + lane);
        }
        float Mb = M;
#pragma unroll
        for (int k = 0; k < K; ++k) Mb = fmaxf(Mb, ml[k].x);
        const float f = Mb > M ? __builtin_amdgcn_exp2f(M - Mb) : 1.f;
        l *= f;
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) acc[r4] *= f;
        M = Mb;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const bool live = ml[k].x != -INFINITY;
            const float wt = live ? __builtin_amdgcn_exp2f(ml[k].x - M) * ml[k].y : 0.f;
            l += wt;
#pragma unroll
            for (int r4 = 0; r4 < 4; ++r4) acc[r4] += live ? wt * o[k][r4] : f32x4{0.f, 0.f, 0.f, 0.f};
        }
    }
    const int row = 32 * w + c;
    if (row >= rows) return;
    const float f = 1.f / l;
    const int tok0 = (int)(row_t / a.G), head0 = (int)(row_t - (int64_t)tok0 * a.G);
    const int dt = (int)((unsigned)(head0 + row) / (unsigned)a.G);
    const int h = g * a.G + head0 + row - dt * a.G;
    uint16_t* orow = a.out + (int64_t)(__builtin_amdgcn_readlane(p.r.q0, b) + tok0 + dt) * a.o_st + (int64_t)h * a.o_sh;
#pragma unroll
    for (int r4 = 0; r4 < 4; ++r4) {
        const f32x2 v01 = {acc[r4][0] * f, acc[r4][1] * f}, v23 = {acc[r4][2] * f, acc[r4][3] * f};
        u32x2 pk;
        pk.x = __builtin_bit_cast(uint32_t, __builtin_convertvector(v01, bf16x2));
        pk.y = __builtin_bit_cast(uint32_t, __builtin_convertvector(v23, bf16x2));
        *(u32x2*)(orow + 32 * t + 8 * r4 + 4 * hl) = pk;
    }
}

}  // namespace

void launch_kv_write(const WriteArgs& a, int32_t* page_start, hipStream_t s) {
    if (a.B > 64) hipLaunchKernelGGL(write_plan_kernel, dim3(1), dim3(kPlanThreads), 0, s, a, page_start);
    // an upper bound on the pages touched: ceil(n_b / 16) + 1 per request
    const unsigned items = (unsigned)(a.T / kPage + 2 * a.B + 1);
    // the heads of a page go over as many workgroups as it takes to have 4096,
    // so that the plan each makes is spread over the rest: 30k tokens of 8
    // heads 48.5 us with a workgroup a head, 42.6 us with three heads each
    // (planning launch and a workgroup a head before: 4.8 + 41.3 us; eight
    // chats' 1.1k tokens 4.6 + 6.0 -> 6.0 us)
    const unsigned ny = std::min((unsigned)a.H_kv, 4096u / std::min(items, 4096u) + 1);
    const dim3 grid(items, ny);
    if (a.elem_bytes == 2) hipLaunchKernelGGL(kv_write_kernel<2>, grid, dim3(256), 0, s, a, (const int32_t*)page_start);
    else hipLaunchKernelGGL(kv_write_kernel<1>, grid, dim3(256), 0, s, a, (const int32_t*)page_start);
    hipLaunchKernelGGL(lens_kernel, dim3((a.B + 255) / 256), dim3(256), 0, s, a);
}

void launch_prefill_prep(const PrefillArgs& a, hipStream_t s) {
    if (a.B > 64) hipLaunchKernelGGL(prefill_plan_kernel, dim3(1), dim3(kPlanThreads), 0, s, a);
    if (a.fp8) return;
    if (a.D == 128) hipLaunchKernelGGL(vcopy_kernel<128>, dim3((unsigned)a.vgrid), dim3(256), 0, s, a);
    else hipLaunchKernelGGL(vcopy_kernel<64>, dim3((unsigned)a.vgrid), dim3(256), 0, s, a);
}

void launch_prefill_attn(const PrefillArgs& a, hipStream_t s) {
    constexpr int NH = kPrefillKeys / 32;
    const dim3 grid((unsigned)((a.max_units + kXcds - 1) / kXcds * kXcds));
    if (a.fp8) {
        if (a.D == 128)
            hipLaunchKernelGGL((prefill_attn_kernel<128, NH, true>), grid, dim3(256), 0, s, a);
        else
            hipLaunchKernelGGL((prefill_attn_kernel<64, NH, true>), grid, dim3(256), 0, s, a);
    } else if (a.D == 128) {
        hipLaunchKernelGGL((prefill_attn_kernel<128, NH, false>), grid, dim3(256), 0, s, a);
    } else {
        hipLaunchKernelGGL((prefill_attn_kernel<64, NH, false>), grid, dim3(256), 0, s, a);
    }
    if (!a.split) return;
    // a wave for every 32 rows x 32 dims of a tile
    const dim3 mgrid((unsigned)(a.max_tiles * (a.D / 32)));
    if (a.D == 128) hipLaunchKernelGGL(prefill_merge_kernel<128>, mgrid, dim3(256), 0, s, a);
    else hipLaunchKernelGGL(prefill_merge_kernel<64>, mgrid, dim3(256), 0, s, a);
}

}  // namespace bellman
