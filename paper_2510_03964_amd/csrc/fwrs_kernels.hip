// HIP kernels of the weighted-reservoir-sampling pass for gfx950.
//
// Store layout (per context, N pixels, k slots): a w_sum plane w_sum[N],
// one record of k slots per pixel, rec[p * k + j] = {w, r, g, b} (16k bytes,
// so at k = 4 a pixel's record is exactly one 64-byte sector), the slots'
// frame indices idx[p * k + j], and the resolve plane res[N][3] (each pixel's
// resolve as of its last change).  A slot replacement therefore dirties only
// the sector of the pixel that replaced it, not one sector in each of k * 4
// planes; reads of whole records stay contiguous across a wave.  Alg. 2's
// candidate count m is the same for every pixel (each pixel receives exactly
// one candidate per frame), so it is the context's frame count, not a plane.
//
// A block of 256 threads covers one work item of 256 pixels, laid out as 1, 2
// or 4 tiles of tile_x pixels by tile_y rows (the tile shape changes the access
// pattern, never the results).  Decisions run with one lane per pixel, the work
// on records with one lane per slot (stream_tiles, whole_tile, per_slot_tile), except
// where one lane per pixel measured faster (resolve_pixel, pixel_per_slot,
// pixel_group).  The passes are bound by their traffic to memory; there is no
// contraction anywhere, so no matrix cores.
//
// Per pixel and frame (Sec. 4.1-4.2 of the paper):
//   w    = Eq. 4 weight from the eccentricity to the gaze (level 0 -> 1)
//   W1'  = Eq. 6 biased w_sum (BERNOULLI) or w_sum (NONE); under FULL every
//          slot has its own w_sum, biased by Eq. 7 against its own sample
//   slot j takes (colour, w, t) when u_j * (W1' + w) > W1'   (Alg. 2)
//   w_sum <- W1' + w
//   out  = sum_j wt_j col_j / sum_j wt_j                      (resolve)
// The new colour is read only by pixels in which some slot takes it (per-slot
// modes: by every pixel).
#include "fwrs_device.hpp"
#include "fwrs_internal.hpp"

// Which streams use non-temporal loads / stores (bits, see kNt* below); a
// launch-shape tuning constant that never changes results.  Level, colour,
// w_sum and the output are streamed once a frame.  The resolve plane is a choice of
// the op (kCachedNt), the incremental output's scattered stores one of scattered_nt.
#ifndef FWRS_NT_MASK
#define FWRS_NT_MASK 0x0C7u
#endif

namespace fwrs {

// kPush: update only; kResolve: resolve only; kFused: update + resolve of every
// pixel from its slots; kIncremental: update + resolve of the pixels whose record
// changed (the output already holds the previous frame's resolve everywhere
// else); kCached: update + resolve of every pixel, where a pixel without a
// replacement copies its resolve from the store's resolve plane (which holds it
// unchanged since the pixel last changed) and a changed pixel recomputes it and
// refreshes the plane; kCachedNt: kCached with non-temporal accesses to the plane;
// kFill: kFused that also writes every pixel's resolve into the plane, making it
// valid for the kCached frames that follow.
enum Op : int {
    kPush = kOpPush, kResolve = kOpResolve, kFused = kOpFused, kIncremental = kOpIncremental, kCached = kOpCached,
    kCachedNt = kOpCachedNt, kFill = kOpFill, kGroup = kOpGroup,
};

enum : uint32_t {
    kNtLevel = 1u, kNtWsumLd = 2u, kNtWsumSt = 4u, kNtRecLd = 8u, kNtRecSt = 16u, kNtIdxSt = 32u,
    kNtColor = 64u, kNtOut = 128u, kNtResLd = 256u, kNtResSt = 512u,
};
constexpr uint32_t kNt = FWRS_NT_MASK;

typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v2f __attribute__((ext_vector_type(2)));

// Every access of the pass goes through these helpers, which address global
// memory explicitly: a descriptor read from a table in device memory (the
// batched kernel) yields generic pointers, which would otherwise compile to
// flat instructions.
#define FWRS_GLOBAL __attribute__((address_space(1)))

template <typename T>
__device__ __forceinline__ const FWRS_GLOBAL T* gbl(const T* p)
{
    return (const FWRS_GLOBAL T*)p;
}

template <typename T>
__device__ __forceinline__ FWRS_GLOBAL T* gbl(T* p)
{
    return (FWRS_GLOBAL T*)p;
}

template <uint32_t BIT, typename T>
__device__ __forceinline__ T ld(const T* p)
{
    if constexpr ((kNt & BIT) != 0u) return __builtin_nontemporal_load(gbl(p));
    return *gbl(p);
}

template <uint32_t BIT, typename T>
__device__ __forceinline__ void st(T* p, T v)
{
    if constexpr ((kNt & BIT) != 0u) __builtin_nontemporal_store(v, gbl(p));
    else *gbl(p) = v;
}

// ... by a value instead of a stream's bit.
template <uint32_t NT, typename T>
__device__ __forceinline__ T ld_as(const T* p)
{
    if constexpr (NT != 0u) return __builtin_nontemporal_load(gbl(p));
    return *gbl(p);
}

template <uint32_t NT, typename T>
__device__ __forceinline__ void st_as(T* p, T v)
{
    if constexpr (NT != 0u) __builtin_nontemporal_store(v, gbl(p));
    else *gbl(p) = v;
}

template <uint32_t BIT>
__device__ __forceinline__ float4 ld4(const float4* p)
{
    const v4f v = ld<BIT>(reinterpret_cast<const v4f*>(p));
    return make_float4(v.x, v.y, v.z, v.w);
}

template <uint32_t BIT>
__device__ __forceinline__ float2 ld2(const float* p)
{
    const v2f v = ld<BIT>(reinterpret_cast<const v2f*>(p));
    return make_float2(v.x, v.y);
}

template <uint32_t BIT>
__device__ __forceinline__ void st4(float4* p, const float4& v)
{
    st<BIT>(reinterpret_cast<v4f*>(p), v4f{v.x, v.y, v.z, v.w});
}

// ---------------------------------------------------------------------------
// Variates and decisions of one pixel.  The Philox words depend only on the
// pixel index and the frame, so they are computed while the pixel's loads are
// in flight; the decision (bit j set when slot j takes the new candidate)
// needs the loaded w_sum.  K > 0: compile-time slot count; K == 0: d.k.
// ---------------------------------------------------------------------------
template <int K>
struct Words {
    uint32_t w[K ? 4 * ((K + 3) / 4) : 4];
};

template <int K>
__device__ __forceinline__ Words<K> philox_words(const FrameDesc& d, uint32_t p)
{
    static_assert(K > 0, "compile-time slot count");
    Words<K> out;
#pragma unroll
    for (int b = 0; b < (K + 3) / 4; ++b) {
        const uint4 r = philox4x32_10(p, d.t, (uint32_t)b, d.seed, d.stream_id);
        out.w[4 * b + 0] = r.x;
        out.w[4 * b + 1] = r.y;
        out.w[4 * b + 2] = r.z;
        out.w[4 * b + 3] = r.w;
    }
    return out;
}

template <int K, bool TAME>
__device__ __forceinline__ uint32_t decide_words(const Words<K>& words, float W1b, float s)
{
    uint32_t mask = 0u;
#pragma unroll
    for (int j = 0; j < K; ++j)
        if (takes<TAME>(words.w[j], s, W1b)) mask |= 1u << j;
    return mask;
}

// Run-time slot count: blocks drawn as needed.
template <bool TAME>
__device__ __forceinline__ uint32_t decide_any(const FrameDesc& d, uint32_t p, float W1b, float s)
{
    const int kk = (int)d.k;
    uint32_t mask = 0u;
    for (int b = 0; 4 * b < kk; ++b) {
        const uint4 r = philox4x32_10(p, d.t, (uint32_t)b, d.seed, d.stream_id);
        const uint32_t words[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int j = 4 * b + q;
            if (j < kk && takes<TAME>(words[q], s, W1b)) mask |= 1u << j;
        }
    }
    return mask;
}

// The Eq. 4 weight in two parts, as weight_outside and select_eq4.
//
// The frames of a context that is not tame (frame_tame) take the general
// division, root and variate test in the same kernels, behind branches on a
// uniform value, so they run at the compiled slot counts like any other frame.
// The branches stand where no load is waited for: one around the arithmetic
// before the level is needed, one after w_sum is there.
__device__ __forceinline__ float weight_part(const FrameDesc& d, uint32_t x, uint32_t y, float& e)
{
    const float dx = ((float)x + 0.5f) - d.gx;
    const float dy = ((float)y + 0.5f) - d.gy;
    if (d.tame) return weight_outside<true>(d.c, dx * dx + dy * dy, e);
    return weight_outside<false>(d.c, dx * dx + dy * dy, e);
}

__device__ __forceinline__ float frame_weight(const FrameDesc& d, uint32_t x, uint32_t y, uint32_t lv)
{
    float e;
    const float o = weight_part(d, x, y, e);
    return select_eq4(d.c, o, e, lv);
}

// The bias of the sum W for a candidate of weight w, the sum s after the frame and
// the slots that take the candidate.
template <int K, bool TAME>
__device__ __forceinline__ uint32_t decide_as(const FrameDesc& d, uint32_t p, const Words<K ? K : 1>& words, float W,
                                              float w, float& s)
{
    const float W1b = bias_shared<TAME>(W, w, d.bias, d.c.decay);
    s = W1b + w;
    if constexpr (K > 0) return decide_words<K, TAME>(words, W1b, s);
    else return decide_any<TAME>(d, p, W1b, s);
}

// A pixel's decision: from its sum W before the frame to the weight w, the sum s
// after it and the slots that take the candidate.
template <int K>
__device__ __forceinline__ uint32_t decide(const FrameDesc& d, uint32_t x, uint32_t y, uint32_t p, uint32_t lv,
                                           float W, float& w, float& s)
{
    Words<K ? K : 1> words;
    if constexpr (K > 0) words = philox_words<K>(d, p);
    w = frame_weight(d, x, y, lv);
    if (d.tame) return decide_as<K, true>(d, p, words, W, w, s);
    return decide_as<K, false>(d, p, words, W, w, s);
}

// 1 / S for the resolve sum_j w_j col_j / sum_j w_j, the sums taken in slot
// order; 0 for a record with no weight (only the empty reservoir: every kept
// weight is > 0).
template <bool TAME>
__device__ __forceinline__ float resolve_scale_as(float S)
{
    const float rs = TAME ? rcp_rn(S) : 1.0f / S;
    return S > 0.0f ? rs : 0.0f;
}

__device__ __forceinline__ float resolve_scale(const FrameDesc& d, float S)
{
    if (d.tame) return resolve_scale_as<true>(S);
    return resolve_scale_as<false>(S);
}

// The resolve of a record held in registers.
template <int R>
__device__ __forceinline__ void resolve_slots(const FrameDesc& d, const float4 (&r)[R], float& q0, float& q1, float& q2)
{
    float S = 0.f, a0 = 0.f, a1 = 0.f, a2 = 0.f;
#pragma unroll
    for (int j = 0; j < R; ++j) {
        S = S + r[j].x;
        a0 = a0 + r[j].x * r[j].y;
        a1 = a1 + r[j].x * r[j].z;
        a2 = a2 + r[j].x * r[j].w;
    }
    const float rs = resolve_scale(d, S);
    q0 = a0 * rs;
    q1 = a1 * rs;
    q2 = a2 * rs;
}

// ---------------------------------------------------------------------------
// One pixel over a group of consecutive frames of one context (batched ticks;
// K > 0 slots, one w_sum per pixel): d0 is the group's first frame, later[f - 1]
// its frame f.  The pixel's state stays in registers from the group's first
// frame to its last -- w_sum, the pixel's resolve (read from the resolve plane
// where that holds it, else computed from the record, which is then read up
// front) and, from the first replacement on, the whole record -- so the store
// is read once and written once per group.  Each frame runs the single-frame
// arithmetic in the same order (the Philox words of its own frame index, the
// Eq. 4 weight at its own gaze, the bias, the Alg. 2 decision per slot, the
// resolve of a changed pixel in slot order) and writes its own output; at the
// end go w_sum, the replaced slots' records and frame indices, and the
// resolve plane (where the pixel changed, or everywhere if it did not hold the
// resolve), so the results are those of the frames run one by one, bit for bit.
//
// The frames are software-pipelined so that no frame waits for its own loads:
// a frame's level is read one frame ahead, and a frame is applied (slots
// replaced, resolve, output) one frame after its decision, once the next
// frame's loads are in flight.  The decision chain needs only w_sum and the
// level, so deciding frame f before applying frame f - 1 changes nothing.
// The colour load is issued by every pixel (those that take nothing read the
// frame's first texel, one line per wave), so no load sits in a branch and
// each wait covers exactly the loads it needs.
// Adds the replaced slots and the frames in which the pixel changed.
// ---------------------------------------------------------------------------
template <int K>
struct GroupPixel {
    float4 r[K];
    uint32_t tj[K];                             // the replaced slots' last frame index
    uint32_t dirty = 0u;                        // slots replaced in the group
    float q0 = 0.f, q1 = 0.f, q2 = 0.f;         // the resolve as of the last applied frame

    // Frame d's decision tk (weight w, colour c) becomes part of the record.
    __device__ __forceinline__ void apply(const FrameDesc& d, uint32_t p, uint32_t tk, float w, float c0, float c1,
                                          float c2, uint32_t& slots, uint32_t& changed)
    {
        if (tk) {
            const float4 fresh = make_float4(w, c0, c1, c2);
#pragma unroll
            for (int j = 0; j < K; ++j)
                if ((tk >> j) & 1u) {
                    r[j] = fresh;
                    tj[j] = d.t;
                }
            dirty |= tk;
            resolve_slots<K>(d, r, q0, q1, q2);
            slots += (uint32_t)__popc(tk);
            changed += 1u;
        }
        float* o = d.out + 3 * (size_t)p;
        st<kNtOut>(o + 0, q0);
        st<kNtOut>(o + 1, q1);
        st<kNtOut>(o + 2, q2);
    }
};

template <int K>
__device__ __forceinline__ void pixel_group(const FrameDesc& d0, const FrameDesc* __restrict__ later, uint32_t x,
                                            uint32_t y, uint32_t& slots, uint32_t& changed)
{
    const uint32_t p = y * d0.width + x;
    const uint32_t nf = d0.nf;
    float4* rec = reinterpret_cast<float4*>(d0.rec) + (size_t)p * K;
    uint32_t* idx = d0.idx + (size_t)p * K;
    float* res = d0.res + 3 * (size_t)p;
    const bool keep = d0.res != nullptr;
    const bool empty = d0.t == 0u;              // the empty store: every slot zero, nothing to read
    const bool from_plane = keep && d0.res_ok != 0u && !empty;

    GroupPixel<K> g;
    float W1 = ld<kNtWsumLd>(d0.wsum + p);
    uint32_t lv = ld<kNtLevel>(d0.level + p);
#pragma unroll
    for (int j = 0; j < K; ++j) {
        g.r[j] = make_float4(0.f, 0.f, 0.f, 0.f);
        g.tj[j] = 0u;
    }
    bool have = true;                           // the record is in registers (or on its way)
    if (from_plane) {
        g.q0 = ld<kNtResLd>(res + 0);
        g.q1 = ld<kNtResLd>(res + 1);
        g.q2 = ld<kNtResLd>(res + 2);
        have = false;
    } else if (!empty) {
#pragma unroll
        for (int j = 0; j < K; ++j) g.r[j] = ld4<kNtRecLd>(rec + j);
        resolve_slots<K>(d0, g.r, g.q0, g.q1, g.q2);
    }

    // the decided frame still to apply
    uint32_t ptk = 0u;
    float pw = 0.f, pc0 = 0.f, pc1 = 0.f, pc2 = 0.f;
    for (uint32_t f = 0; f < nf; ++f) {
        const FrameDesc& d = f == 0u ? d0 : later[f - 1u];
        uint32_t lv_next = 0u;
        if (f + 1u < nf) lv_next = ld<kNtLevel>(later[f].level + p);
        // the decision: Eq. 4 weight, bias, Alg. 2 per slot
        float w, s;
        const uint32_t tk = decide<K>(d, x, y, p, lv, W1, w, s);
        W1 = s;
        // its colour, and at the pixel's first replacement the slots it keeps
        const float* cp = d.color + (tk ? 3 * (size_t)p : 0);
        const float c0 = ld<kNtColor>(cp + 0), c1 = ld<kNtColor>(cp + 1), c2 = ld<kNtColor>(cp + 2);
        // the previous frame
        if (f) g.apply(f == 1u ? d0 : later[f - 2u], p, ptk, pw, pc0, pc1, pc2, slots, changed);
        if (tk && !have) {
#pragma unroll
            for (int j = 0; j < K; ++j)
                if (!((tk >> j) & 1u)) g.r[j] = ld4<kNtRecLd>(rec + j);
            have = true;
        }
        ptk = tk;
        pw = w;
        pc0 = c0;
        pc1 = c1;
        pc2 = c2;
        lv = lv_next;
    }
    g.apply(nf == 1u ? d0 : later[nf - 2u], p, ptk, pw, pc0, pc1, pc2, slots, changed);

    st<kNtWsumSt>(d0.wsum + p, W1);
#pragma unroll
    for (int j = 0; j < K; ++j)
        if ((g.dirty >> j) & 1u) {
            st4<kNtRecSt>(rec + j, g.r[j]);
            st<kNtIdxSt>(idx + j, g.tj[j]);
        }
    if (keep && (g.dirty != 0u || !from_plane)) {
        st<kNtResSt>(res + 0, g.q0);
        st<kNtResSt>(res + 1, g.q1);
        st<kNtResSt>(res + 2, g.q2);
    }
}

// ---------------------------------------------------------------------------
// Pixel of a lane of wave `wave` in work item `item` (256 pixels); false outside
// the image (or past the frame's last item).  The wave index is a uniform value,
// so the tile arithmetic runs on the scalar unit.
// ---------------------------------------------------------------------------
__device__ __forceinline__ bool item_pixel_of(const FrameDesc& d, uint32_t item, uint32_t wave, uint32_t lane,
                                              uint32_t& x, uint32_t& y)
{
    const uint32_t tlog = d.tile_x_log2 + d.tile_y_log2;            // log2(threads per tile): 6..8
    const uint32_t waves_per_tile_log2 = tlog - 6u;
    const uint32_t tiles_per_item_log2 = 8u - tlog;
    const uint32_t tile = (item << tiles_per_item_log2) + (wave >> waves_per_tile_log2);
    const uint32_t local = ((wave & ((1u << waves_per_tile_log2) - 1u)) << 6) | lane;
    const uint32_t ty = d.div_m ? __umulhi(tile, d.div_m) >> d.div_s : tile;
    const uint32_t tx = tile - ty * d.tiles_x;
    x = (tx << d.tile_x_log2) + (local & ((1u << d.tile_x_log2) - 1u));
    y = (ty << d.tile_y_log2) + (local >> d.tile_x_log2);
    return item < d.items && y < d.height && x < d.width;
}

// Sum of v over the wave, in every lane: five row-wise steps by data-parallel
// moves (no LDS traffic) and the last lane's total as a scalar.
__device__ __forceinline__ uint32_t wave_sum(uint32_t v)
{
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xF, 0xF, true);    // row_shr:1
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xF, 0xF, true);    // row_shr:2
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xF, 0xF, true);    // row_shr:4
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xF, 0xF, true);    // row_shr:8
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xA, 0xF, false);   // row_bcast:15, rows 1 and 3
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xC, 0xF, false);   // row_bcast:31, rows 2 and 3
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// The wave's counts go to a triple chosen by the wave's id, lane c adding
// counter c: one atomic instruction per wave.
__device__ __forceinline__ void add_counts(unsigned long long* stats, uint32_t slots, uint32_t changed,
                                           uint32_t flushed)
{
    const uint32_t lane = threadIdx.x & 63u;
    if (lane < (flushed ? 3u : 2u)) {
        const uint32_t slot = (blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6)) & (kStatSlots - 1);
        atomicAdd(stats + 3 * slot + lane, (unsigned long long)(lane == 0u ? slots : lane == 1u ? changed : flushed));
    }
}

// add_stats for counts beyond its packed fields' range (a group of frames):
// replaced slots and changed pixel-frames as separate wave sums.
__device__ __forceinline__ void add_stats_wide(unsigned long long* stats, uint32_t slots, uint32_t changed)
{
    changed = wave_sum(changed);
    if (changed) add_counts(stats, wave_sum(slots), changed, 0u);
}

// The counts of stream_tiles, uniform over the wave.
__device__ __forceinline__ void add_stats_uniform(unsigned long long* stats, uint32_t v)
{
    if (v) add_counts(stats, v & 0xFFFFu, v >> 16, 0u);
}

__device__ __forceinline__ void add_stats(unsigned long long* stats, uint32_t v)
{
    // v = replaced slots + 2^16 * (pixel changed) + 2^24 * (pixel flushed); the wave sum
    // has at most 1024 slots and 64 pixels per field
    v = wave_sum(v);
    if (v) add_counts(stats, v & 0xFFFFu, (v >> 16) & 0xFFu, v >> 24);
}

// ---------------------------------------------------------------------------
// A frame of a mode with one w_sum per pixel: T tiles of 64 pixels per wave.
//  1. One lane per pixel: the loads every pixel needs (level, w_sum, for kCached
//     its resolve from the plane), then the decision.  The pixels that replace a
//     slot go on a list in LDS.
//  2. One lane per slot: groups of lanes work through the list, so a record
//     (16k bytes) is one coalesced access instead of k accesses 16k bytes apart,
//     and a wave holds only pixels that have work.
//  3. One lane per pixel: w_sum and (kCached) the output row, a listed pixel's
//     resolve read back from the list, so rows leave whole.
// The list is the wave's own, so no barrier is needed.  Stores come after the
// loads of the same step, because vector-memory operations are waited for in
// order.
//
// Why: the passes are bound by their requests to the memory side (128-byte reads,
// 64-byte writes, about 6 TB/s of them) and by waiting; one lane per pixel with k
// loads per record kept every line's requests pending in L1 k times.  Measured
// against that form, per frame: k = 8 at 1280x720 after 45 frames 38 -> 32.5 us, k = 16 at
// 1920x1080 276 -> 173, incremental 2560x1440 at frame 1200, k = 4 37.5 -> 28 and k = 2
// 31.5 -> 20, update-only 3840x2160, k = 2 53 -> 34.5.
// ---------------------------------------------------------------------------
// T, the tiles per wave: the ops without the plane's row (kIncremental, kPush) have
// few loads in flight per tile and take two where lists are short enough for one
// round, that is up to 4 slots and where the records fit the Infinity Cache or, beyond,
// once few pixels change (us, one tile / two: incremental k = 4 at 2560x1440, frame 1200
// 31 / 28, at 3840x2160, frame 50 184 / 189, frame 1200 72.8 / 76; k = 3 at frame 100
// 134.7 / 139, 400 91.6 / 94, 800 78 / 70; k = 1 at 7680x4320, frame 45 274 / 288, 400
// 212 / 150; update-only k = 4 at 3840x2160, frame 50 134 / 138, 400 74.5 / 77, 1200
// 55.8 / 51.6; k = 8 at 1920x1080 incremental 59 / 63.8 with either list), and where
// that still leaves a whole round of resident waves (2 x 8192; 800x600, less than one:
// 10.3 / 11.0).
inline bool takes_two_tiles(const FrameDesc& d, int op)
{
    const uint64_t records = (uint64_t)d.width * d.height * d.k * 16u;
    return d.k <= 4u && d.items >= 4096u &&
           (records <= kCacheBytes || d.t >= (op == kPush ? 128u : 256u) * d.k);
}

// Whether the scattered stores of a changed pixel's resolve are non-temporal.
// kCached (the plane): no; rewriting 12 bytes of a line that was just read
// is cheaper through L2 once the records are larger than the Infinity Cache (3840x2160,
// k = 4, frame 80: 196 us against 214).  While they fit, the cache is better left to them:
// kCachedNt 1920x1080, k = 4 44.7 -> 41.5, k = 8 1280x720 32.5 -> 30, behind the
// mip generator at 1920x1080, k = 4 58.5 -> 50.  kIncremental (the output) up to 4
// slots: 3840x2160, k = 2 95 -> 79.6, 1280x720, k = 4 while filling 30.4 -> 28; at 8
// 145 -> 150 (2560x1440).
constexpr uint32_t scattered_nt(int k, int op) { return op == kCachedNt || (op == kIncremental && k >= 1 && k <= 4); }

__device__ __forceinline__ void wave_lds_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Data-parallel moves within quads of lanes: lane a, b, c, d of the quad to its
// four lanes.
template <int A, int B, int C, int D>
__device__ __forceinline__ float quad_perm(float v)
{
    constexpr int sel = A | (B << 2) | (C << 4) | (D << 6);
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), sel, 0xF, 0xF, true));
}

// Lanes of a pixel's group: one per slot, a power of two, whole quads from 3
// slots on.
template <int K>
__device__ __forceinline__ uint32_t group_log2(uint32_t kk)
{
    return K == 1 ? 0u : K == 2 ? 1u : kk <= 4u ? 2u : kk <= 8u ? 3u : 4u;
}

// The group's first lane that has group_sum's result: lane 0, beyond 4 slots the
// first lane of the last slot's quad.
template <int K>
__device__ __forceinline__ uint32_t group_first(uint32_t kk)
{
    return K == 1 || K == 2 ? 0u : (kk - 1u) & ~3u;
}

// 0 + v_0 + v_1 + ... + v_(kk-1) over a group of lanes, added in lane order (K: as
// kk where known, else 0).  Lanes past the slots hold +0, which leaves a sum that
// started at +0 as it is.  Valid in the quad of group_first.
template <int K>
__device__ __forceinline__ float group_sum(float v, uint32_t kk)
{
    float s = 0.f;
    if constexpr (K == 1) {
        s = s + v;
    } else if constexpr (K == 2) {
        s = s + quad_perm<0, 0, 2, 2>(v);
        s = s + quad_perm<1, 1, 3, 3>(v);
    } else {
        const float v0 = quad_perm<0, 0, 0, 0>(v), v1 = quad_perm<1, 1, 1, 1>(v);
        const float v2 = quad_perm<2, 2, 2, 2>(v), v3 = quad_perm<3, 3, 3, 3>(v);
#pragma unroll
        for (uint32_t j = 0; j < (K ? (uint32_t)K : (uint32_t)kMaxK); j += 4u) {
            if (!K && j >= kk) break;
            // the sum so far, from the quad below (row_shr:4)
            if (j) s = __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, s), 0x114, 0xF, 0xF, true));
            s = s + v0;
            s = s + v1;
            s = s + v2;
            s = s + v3;
        }
    }
    return s;
}

template <int T>
struct ListShare {                              // one wave's listed pixels
    uint4 pixel[64 * T];                        // {x, y, weight, replaced slots | level << 16}
    float4 colour[64 * T];                      // the new colour (colours_first), then the resolve (kCached)
};

// Whether the listed pixels' colours are loaded with one lane per pixel, before the
// rounds, instead of in each round: beyond 4 slots, where a list takes many rounds,
// a wave waits for them once (incremental k = 16 at 640x360 27.0 -> 21.8 us, update-only k = 8
// at 1920x1080 38.5 -> 33.6, 640x360 steps at k = 8 13.0 -> 10.8); with few rounds it is
// one access more (1279x719, k = 3, frame 2000 11.0 us, and 11.8 with this).
template <int K>
__device__ __forceinline__ bool colours_first(uint32_t kk)
{
    return K ? K > 4 : kk > 4u;
}

// The list's n pixels.  A group of lanes takes a pixel, 64 / group pixels a round.
// Kept slots are read, replaced slots stored (whole records, as whole_tile has them:
// 6% slower here, where few pixels change).  The resolve goes to the list and the plane
// (kCached) or to the output (kIncremental).  Returns the lane's replaced slots.
template <int K, int OP, int T, bool FOV, uint32_t NT, bool TAME>
__device__ __forceinline__ uint32_t listed_pixels(const FrameDesc& d, const FovSrc* fs, ListShare<T>& sh, uint32_t n,
                                                  uint32_t lane)
{
    constexpr bool kResolves = OP != kPush;
    const uint32_t kk = K ? (uint32_t)K : d.k;
    const uint32_t lg = group_log2<K>(kk), first = group_first<K>(kk);
    const uint32_t j = lane & ((1u << lg) - 1u), per = 64u >> lg;
    const bool slot = K || j < kk;
    const bool empty = d.t == 0u;                   // frame 0 meets the empty store: nothing to read
    uint32_t taken = 0u;
    for (uint32_t b = 0; b < n; b += per) {
        const uint32_t at = b + (lane >> lg);
        const bool own = at < n;
        const uint32_t e = own ? at : b;            // past the end: the round's first entry
        const uint4 entry = sh.pixel[e];
        const uint32_t p = entry.y * d.width + entry.x;
        const size_t s = (size_t)p * kk + (slot ? j : 0u);
        const bool take = slot && ((entry.w >> j) & 1u) != 0u;
        float4 r = make_float4(0.f, 0.f, 0.f, 0.f);
        if (kResolves && !empty && slot && !take) r = ld4<kNtRecLd>(reinterpret_cast<const float4*>(d.rec) + s);
        float c0, c1, c2;
        if (colours_first<K>(kk)) {
            const float4 c = sh.colour[e];
            c0 = c.x;
            c1 = c.y;
            c2 = c.z;
        } else if constexpr (K == 1 || K == 2) {
            if constexpr (FOV) {
                const float3 c = fov_colour(*fs, entry.x, entry.y, p, entry.w >> 16);
                c0 = c.x;
                c1 = c.y;
                c2 = c.z;
            } else {
                const float* color = d.color + 3 * (size_t)p;
                c0 = ld<kNtColor>(color + 0);
                c1 = ld<kNtColor>(color + 1);
                c2 = ld<kNtColor>(color + 2);
            }
        } else {                                    // each lane of a quad loads one channel
            const uint32_t ch = (j & 3u) < 3u ? (j & 3u) : 2u;
            float c;
            if constexpr (FOV) c = fov_channel(*fs, entry.x, entry.y, p, entry.w >> 16, ch);
            else c = ld<kNtColor>(d.color + 3 * (size_t)p + ch);
            c0 = quad_perm<0, 0, 0, 0>(c);
            c1 = quad_perm<1, 1, 1, 1>(c);
            c2 = quad_perm<2, 2, 2, 2>(c);
        }
        if (take) r = make_float4(__builtin_bit_cast(float, entry.z), c0, c1, c2);
        float q0 = 0.f, q1 = 0.f, q2 = 0.f;
        if constexpr (kResolves) {
            const float rs = resolve_scale_as<TAME>(group_sum<K>(r.x, kk));
            q0 = group_sum<K>(r.x * r.y, kk) * rs;
            q1 = group_sum<K>(r.x * r.z, kk) * rs;
            q2 = group_sum<K>(r.x * r.w, kk) * rs;
        }
        if (own) {
            if (take) {
                st4<kNtRecSt>(reinterpret_cast<float4*>(d.rec) + s, r);
                st<kNtIdxSt>(d.idx + s, d.t);
                taken += 1u;
            }
            if constexpr (kResolves) {
                float* to = (OP == kCached ? d.res : d.out) + 3 * (size_t)p;
                if constexpr (K == 1 || K == 2) {
                    if (j == 0u) {
                        st_as<NT>(to + 0, q0);
                        st_as<NT>(to + 1, q1);
                        st_as<NT>(to + 2, q2);
                    }
                } else if (j >= first && j < first + 3u) {
                    st_as<NT>(to + (j - first), j == first ? q0 : j == first + 1u ? q1 : q2);
                }
            }
            if (OP == kCached && j == first) sh.colour[at] = make_float4(q0, q1, q2, 0.f);
        }
    }
    return taken;
}

// The wave's 64 T pixels of work items item0 .. item0 + T - 1.  Returns the wave's
// (uniform) replaced slots + 2^16 x changed pixels.
template <int K, int OPV, int T, bool FOV = false>
__device__ __forceinline__ uint32_t stream_tiles(const FrameDesc& d, uint32_t item0, uint32_t wave, uint32_t lane,
                                                 ListShare<T>& sh, const FovSrc* fs = nullptr)
{
    constexpr int OP = OPV == kCachedNt ? kCached : OPV;
    constexpr uint32_t NT = scattered_nt(K, OPV);
    static_assert(OP == kPush || OP == kIncremental || OP == kCached, "the ops that need few records");

    uint32_t x[T], y[T], p[T], lv[T], at[T];
    bool in[T];
    float W[T], q0[T], q1[T], q2[T];
#pragma unroll
    for (int t = 0; t < T; ++t) {
        in[t] = item_pixel_of(d, item0 + t, wave, lane, x[t], y[t]);
        p[t] = in[t] ? y[t] * d.width + x[t] : 0u;          // lanes outside read pixel 0 and store nothing
        if constexpr (FOV) lv[t] = fov_level(*fs, d.gx, d.gy, x[t], y[t]);
        else lv[t] = ld<kNtLevel>(d.level + p[t]);
        W[t] = ld<kNtWsumLd>(d.wsum + p[t]);
        if constexpr (OP == kCached) {
            const float* res = d.res + 3 * (size_t)p[t];
            q0[t] = ld_as<NT>(res + 0);
            q1[t] = ld_as<NT>(res + 1);
            q2[t] = ld_as<NT>(res + 2);
        }
    }
    uint32_t n = 0u;
#pragma unroll
    for (int t = 0; t < T; ++t) {
        float w, s;
        uint32_t tk = decide<K>(d, x[t], y[t], p[t], lv[t], W[t], w, s);
        if (!in[t]) tk = 0u;
        W[t] = s;
        const uint64_t took = __ballot(tk != 0u);
        at[t] = 0xFFFFFFFFu;
        if (tk) {
            at[t] = n + __builtin_amdgcn_mbcnt_hi((uint32_t)(took >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)took, 0u));
            sh.pixel[at[t]] = make_uint4(x[t], y[t], __builtin_bit_cast(uint32_t, w), tk | (lv[t] << 16));
            if (colours_first<K>(d.k)) {
                float3 c;
                if constexpr (FOV) {
                    c = fov_colour(*fs, x[t], y[t], p[t], lv[t]);
                } else {
                    const float* color = d.color + 3 * (size_t)p[t];
                    c = make_float3(ld<kNtColor>(color + 0), ld<kNtColor>(color + 1), ld<kNtColor>(color + 2));
                }
                sh.colour[at[t]] = make_float4(c.x, c.y, c.z, 0.f);
            }
        }
        n += (uint32_t)__builtin_popcountll(took);
    }
    wave_lds_fence();
    uint32_t slots = 0u;
    if (n) {
        if (OP == kPush || d.tame) slots = listed_pixels<K, OP, T, FOV, NT, true>(d, fs, sh, n, lane);
        else slots = listed_pixels<K, OP, T, FOV, NT, false>(d, fs, sh, n, lane);
        slots = wave_sum(slots);
    }
    wave_lds_fence();
#pragma unroll
    for (int t = 0; t < T; ++t) {
        if (!in[t]) continue;
        st<kNtWsumSt>(d.wsum + p[t], W[t]);
        if constexpr (OP == kCached) {
            if (at[t] != 0xFFFFFFFFu) {
                const float4 v = sh.colour[at[t]];
                q0[t] = v.x;
                q1[t] = v.y;
                q2[t] = v.z;
            }
            float* o = d.out + 3 * (size_t)p[t];
            st<kNtOut>(o + 0, q0[t]);
            st<kNtOut>(o + 1, q1[t]);
            st<kNtOut>(o + 2, q2[t]);
        }
    }
    return slots + (n << 16);
}

// ---------------------------------------------------------------------------
// The ops that take every pixel's resolve from its record (kFused, kFill; kResolve
// for a run-time slot count), 64 pixels a wave: no list is needed, so the first
// rounds' records are loaded with the pixels' own inputs, ahead of the decisions,
// and the colours, of the pixels that replace a slot, with one lane per pixel.
// Where many pixels replace slots, whole records are stored (below).  Against
// the list with every pixel on it, whose rounds each wait for a record and a
// colour: while a store fills 53 -> 45 us at 1280x720, k = 8, and 96.5 -> 94 at
// 2560x1440, k = 4; without a resolve plane at frame 600 37.5 -> 36.2 at 1920x1080,
// k = 4, and 332 -> 315 at 3840x2160, k = 8 (one lane per pixel with its k loads:
// 62, 120, 35.8 and 317).  Rounds loaded ahead: at k = 4 two (four: 28 us against
// 26.5 at 1280x720 while filling), at k = 8 one (two: 28.8 against 27.2 at frame 600).
// ---------------------------------------------------------------------------
// kResolve at a compiled slot count: one lane per pixel, its record in registers (the
// rounds of whole_tile: 188 us against 202 at 3840x2160, k = 8).
template <int K>
__device__ __forceinline__ void resolve_pixel(const FrameDesc& d, uint32_t item, uint32_t wave)
{
    uint32_t x, y;
    if (!item_pixel_of(d, item, wave, threadIdx.x & 63u, x, y)) return;
    const uint32_t p = y * d.width + x;
    const float4* rec = reinterpret_cast<const float4*>(d.rec) + (size_t)p * K;
    float4 r[K];
#pragma unroll
    for (int j = 0; j < K; ++j) r[j] = make_float4(0.f, 0.f, 0.f, 0.f);
    if (d.t != 0u) {                            // the empty store: every slot zero, nothing to read
#pragma unroll
        for (int j = 0; j < K; ++j) r[j] = ld4<kNtRecLd>(rec + j);
    }
    float q0, q1, q2;
    resolve_slots<K>(d, r, q0, q1, q2);
    float* o = d.out + 3 * (size_t)p;
    st<kNtOut>(o + 0, q0);
    st<kNtOut>(o + 1, q1);
    st<kNtOut>(o + 2, q2);
}

struct WholeShare {                             // one wave's pixels
    uint2 pixel[64];                            // {p, inside | replaced slots << 1}
    float4 colour[64];                          // the new colour, weight; then the resolve
};

template <int K, int OP, bool FOV = false>
__device__ __forceinline__ uint32_t whole_tile(const FrameDesc& d, uint32_t item, uint32_t wave, uint32_t lane, WholeShare& sh,
                                               const FovSrc* fs = nullptr)
{
    static_assert(OP == kFused || OP == kFill || OP == kResolve, "the ops that read every record");
    constexpr bool kUpdates = OP != kResolve;
    constexpr uint32_t D = K == 0 || K == 2 || K == 4 ? 2u : 1u;    // rounds loaded ahead
    const uint32_t kk = K ? (uint32_t)K : d.k;
    const uint32_t lg = group_log2<K>(kk), first = group_first<K>(kk);
    const uint32_t j = lane & ((1u << lg) - 1u), per = 64u >> lg;
    const bool slot = K || j < kk;
    const bool empty = d.t == 0u;               // frame 0 meets the empty store: nothing to read

    uint32_t x, y;
    const bool in = item_pixel_of(d, item, wave, lane, x, y);
    const uint32_t p = in ? y * d.width + x : 0u;           // lanes outside read pixel 0 and store nothing
    sh.pixel[lane] = make_uint2(p, in ? 1u : 0u);
    uint32_t lv = 0u;
    float W = 0.f;
    if constexpr (kUpdates) {
        if constexpr (FOV) lv = fov_level(*fs, d.gx, d.gy, x, y);
        else lv = ld<kNtLevel>(d.level + p);
        W = ld<kNtWsumLd>(d.wsum + p);
    }
    wave_lds_fence();
    float4 v[D];
    auto load = [&](uint32_t b) {
        const size_t at = (size_t)sh.pixel[b + (lane >> lg)].x * kk + (slot ? j : 0u);
        return ld4<kNtRecLd>(reinterpret_cast<const float4*>(d.rec) + at);
    };
#pragma unroll
    for (uint32_t u = 0; u < D; ++u) {
        v[u] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (u * per < 64u && !empty) v[u] = load(u * per);
    }
    uint32_t slots = 0u, changed = 0u;
    if constexpr (kUpdates) {
        float w, s;
        uint32_t tk = decide<K>(d, x, y, p, lv, W, w, s);
        if (!in) tk = 0u;
        W = s;
        changed = (uint32_t)__builtin_popcountll(__ballot(tk != 0u));
        if (changed) slots = wave_sum((uint32_t)__popc(tk));
        if (tk) {
            float c0, c1, c2;
            if constexpr (FOV) {
                const float3 c = fov_colour(*fs, x, y, p, lv);
                c0 = c.x;
                c1 = c.y;
                c2 = c.z;
            } else {
                const float* color = d.color + 3 * (size_t)p;
                c0 = ld<kNtColor>(color + 0);
                c1 = ld<kNtColor>(color + 1);
                c2 = ld<kNtColor>(color + 2);
            }
            sh.pixel[lane] = make_uint2(p, 1u | (tk << 1));
            sh.colour[lane] = make_float4(c0, c1, c2, w);
        }
        wave_lds_fence();
    }

    // one lane per slot
    for (uint32_t b0 = 0; b0 < 64u; b0 += D * per)
#pragma unroll
    for (uint32_t u = 0; u < D; ++u) {
        const uint32_t b = b0 + u * per;
        if (b >= 64u) break;
        const uint32_t e = b + (lane >> lg);
        const uint2 px = sh.pixel[e];
        float4 r = v[u];
        if (b + D * per < 64u && !empty) v[u] = load(b + D * per);
        bool take = false;
        if constexpr (kUpdates) {
            take = slot && ((px.y >> (1u + j)) & 1u) != 0u;
            if (take) {
                const float4 c = sh.colour[e];
                r = make_float4(c.w, c.x, c.y, c.z);
            }
        }
        if (!slot) r = make_float4(0.f, 0.f, 0.f, 0.f);
        const float rs = resolve_scale(d, group_sum<K>(r.x, kk));
        const float q0 = group_sum<K>(r.x * r.y, kk) * rs;
        const float q1 = group_sum<K>(r.x * r.z, kk) * rs;
        const float q2 = group_sum<K>(r.x * r.w, kk) * rs;
        if constexpr (kUpdates) {
            const size_t at = (size_t)px.x * kk + (slot ? j : 0u);
            // full lines are written faster than parts of them (k = 8 while filling 108.9
            // -> 106.1 us a 1920x1080 frame, k = 4 at 3840x2160 258 -> 250.6)
            const bool whole = slot && 4u * (uint32_t)__popc(px.y >> 1) >= kk;
            if (take || whole) st4<kNtRecSt>(reinterpret_cast<float4*>(d.rec) + at, r);
            if (take) st<kNtIdxSt>(d.idx + at, d.t);
        }
        if (j == first) sh.colour[e] = make_float4(q0, q1, q2, 0.f);
    }
    wave_lds_fence();
    if (in) {
        if constexpr (kUpdates) st<kNtWsumSt>(d.wsum + p, W);
        const float4 q = sh.colour[lane];
        float* o = d.out + 3 * (size_t)p;
        st<kNtOut>(o + 0, q.x);
        st<kNtOut>(o + 1, q.y);
        st<kNtOut>(o + 2, q.z);
        if constexpr (OP == kFill) {
            float* res = d.res + 3 * (size_t)p;
            st<kNtResSt>(res + 0, q.x);
            st<kNtResSt>(res + 1, q.y);
            st<kNtResSt>(res + 2, q.z);
        }
    }
    return slots + (changed << 16);
}

// The A-ES key log2(u) / w of a candidate.
__device__ __forceinline__ float aes_key(const FrameDesc& d, uint32_t word, float w)
{
    const float l = log2_unit(word);
    if (d.tame) return div_rn(l, w);
    return l / w;
}

// Eq. 7 and the slot's Alg. 2 decision: s is the slot's sum after the frame.
template <bool TAME>
__device__ __forceinline__ bool decide_eq7_as(uint32_t word, float W, float w, float dl, float& s)
{
    const float W1b = bias_eq7<TAME>(W, w, dl);
    s = W1b + w;
    return takes<TAME>(word, s, W1b);
}

__device__ __forceinline__ bool decide_eq7(const FrameDesc& d, uint32_t word, float W, float w, float dl, float& s)
{
    if (d.tame) return decide_eq7_as<true>(word, W, w, dl, s);
    return decide_eq7_as<false>(word, W, w, dl, s);
}

// rgb_to_lab of a colour that all lanes of a quad hold, one curve per lane.  The whole
// quad is active.
__device__ __forceinline__ float3 rgb_to_lab_quad(float r, float g, float b, uint32_t lane)
{
    const uint32_t q = lane & 3u;
    const float m0 = q == 0u ? 0.4124564f : q == 1u ? 0.2126729f : 0.0193339f;
    const float m1 = q == 0u ? 0.3575761f : q == 1u ? 0.7151522f : 0.1191920f;
    const float m2 = q == 0u ? 0.1804375f : q == 1u ? 0.0721750f : 0.9503041f;
    const float c = q == 0u ? 0.95047f : q == 1u ? 1.0f : 1.08883f;
    const float rc = q == 0u ? 0x1.0d5728p+0f : q == 1u ? 1.0f : 0x1.d63ac2p-1f;
    const float f = lab_curve(div_const((m0 * r + m1 * g) + m2 * b, c, rc));     // x / 1 is x
    const float fx = quad_perm<0, 0, 0, 0>(f), fy = quad_perm<1, 1, 1, 1>(f), fz = quad_perm<2, 2, 2, 2>(f);
    return make_float3(116.0f * fy - 16.0f, 500.0f * (fx - fy), 200.0f * (fy - fz));
}

// Eq. 7's |dL| of a slot's sample against its pixel's new colour, every lane of the wave
// active.  A sample with the new colour has |dL| = 0 exactly (same_colour): Lab and
// CIE94 are evaluated only where some slot of the wave differs, the new colour's Lab
// once per quad from 3 slots on.
template <int K>
__device__ __forceinline__ float slot_delta(const float4& s, const float4& c, uint32_t lane)
{
    const bool differs = !(lab_bounded(c.x, c.y, c.z) && same_colour(s, c.x, c.y, c.z));
    float dl = 0.0f;
    if (__ballot(differs) != 0u) {
        float3 lab;
        if constexpr (K == 1 || K == 2) lab = rgb_to_lab(c.x, c.y, c.z);
        else lab = rgb_to_lab_quad(c.x, c.y, c.z, lane);
        if (differs) dl = delta_l(s.y, s.z, s.w, lab);
    }
    return dl;
}

// ---------------------------------------------------------------------------
// A frame of a per-slot mode, one value per slot in wsum[p * k + j]:
//  - Eq. 7 (FULL): the slot's own w_sum, biased by the slot's colour
//    difference to the new pixel before its Alg. 2 decision;
//  - A-ES: the log2 key of the slot's sample; the candidate's key log2(u) / w
//    replaces it when larger (Sec. 3.1).
// Every slot's record and value are read by every op that updates, so the wave
// goes through its 64 pixels with one lane per slot: the pixel's weight, colour
// and Philox words are computed with one lane per pixel and handed over in LDS,
// records and values are coalesced accesses, a round's being loaded while the
// one before is worked on, and Lab and CIE94 run only in the rounds (16 pixels at
// k = 4) that hold a slot whose colour differs.  The resolve goes back through
// LDS to leave by rows.  Against one lane per pixel streaming its record slot by
// slot, as ticks and slot counts other than 4 and 8 had it: four 900x600 Eq. 7
// sessions in a tick 82.4 -> 44.5 us, five 700x500 A-ES k = 8 sessions 170 -> 54,
// 1600x1000 Eq. 7 k = 1 21.2 -> 15.4, 1920x1080 k = 16 1283 -> 248.
// Non-temporal record loads gain 10% where other sessions' frames come in between (three
// 2560x1440 sessions, Eq. 7, k = 4: 89 us against 99) and lose 20 to 40% where one session
// runs frame after frame, whose next frame finds part of its store in the Infinity
// Cache (109 us against 87), so they are plain.
// ---------------------------------------------------------------------------
template <int K>
struct PerSlotShare {                           // one wave's pixels
    static constexpr int kBlocks = K ? (K + 3) / 4 : (kMaxK + 3) / 4;
    uint2 pixel[64];                            // {p, inside}
    float4 colour[64];                          // the new colour, weight; then the resolve, changed
    uint32_t words[64][4 * kBlocks];            // Philox words, one per slot
};

template <int K, int OP, bool FOV = false>
__device__ __forceinline__ uint32_t per_slot_tile(const FrameDesc& d, uint32_t item, uint32_t wave, uint32_t lane,
                                                  PerSlotShare<K>& sh, const FovSrc* fs = nullptr)
{
    static_assert(OP == kPush || OP == kFused || OP == kIncremental, "the resolve-only pass is the same under every mode");
    constexpr bool kResolves = OP != kPush;
    const uint32_t kk = K ? (uint32_t)K : d.k;
    const uint32_t lg = group_log2<K>(kk), first = group_first<K>(kk);
    const uint32_t j = lane & ((1u << lg) - 1u), per = 64u >> lg;
    const bool slot = K || j < kk;
    const bool aes = d.bias == kAes;
    constexpr uint32_t D = K == 4 ? 4u : 1u;      // rounds loaded ahead

    // 1. one lane per pixel
    uint32_t x, y;
    const bool in = item_pixel_of(d, item, wave, lane, x, y);
    if (!in) x = y = 0u;                        // lanes outside read pixel 0 and store nothing
    const uint32_t p = y * d.width + x;
    sh.pixel[lane] = make_uint2(p, in ? 1u : 0u);
    uint32_t lv;
    float c0, c1, c2;
    if constexpr (FOV) {
        lv = fov_level(*fs, d.gx, d.gy, x, y);
        const float3 c = fov_colour(*fs, x, y, p, lv);
        c0 = c.x;
        c1 = c.y;
        c2 = c.z;
    } else {
        lv = ld<kNtLevel>(d.level + p);
        const float* color = d.color + 3 * (size_t)p;
        c0 = ld<kNtColor>(color + 0);
        c1 = ld<kNtColor>(color + 1);
        c2 = ld<kNtColor>(color + 2);
    }
    wave_lds_fence();

    // the records and values of the first rounds, in flight over the pixels' arithmetic
    float4 v[D];
    float W1[D];
    auto load = [&](uint32_t b, float4& rec, float& val) {
        const uint32_t q = sh.pixel[b + (lane >> lg)].x;
        const size_t at = (size_t)q * kk + (slot ? j : 0u);
        rec = ld4<kNtRecLd>(reinterpret_cast<const float4*>(d.rec) + at);
        val = ld<kNtWsumLd>(d.wsum + at);
    };
#pragma unroll
    for (uint32_t q = 0; q < D; ++q)
        if (q * per < 64u) load(q * per, v[q], W1[q]);

    for (uint32_t b = 0; 4u * b < kk; ++b) {
        const uint4 r = philox4x32_10(p, d.t, b, d.seed, d.stream_id);
        *reinterpret_cast<uint4*>(&sh.words[lane][4u * b]) = r;
    }
    sh.colour[lane] = make_float4(c0, c1, c2, frame_weight(d, x, y, lv));
    wave_lds_fence();

    // 2. one lane per slot
    uint32_t slots = 0u, changed = 0u;
    for (uint32_t b0 = 0; b0 < 64u; b0 += D * per)
#pragma unroll
    for (uint32_t q = 0; q < D; ++q) {
        const uint32_t b = b0 + q * per;
        if (b >= 64u) break;
        const uint32_t e = b + (lane >> lg);
        const uint2 now = sh.pixel[e];
        const size_t s_at = (size_t)now.x * kk + (slot ? j : 0u);
        float4 r = v[q];
        const float Wj = W1[q];
        if (b + D * per < 64u) load(b + D * per, v[q], W1[q]);
        const float4 c = sh.colour[e];
        const float w = c.w;
        const uint32_t word = sh.words[e][slot ? j : 0u];
        bool take;
        float s;
        if (aes) {
            // A-ES: the larger key log2(u) / w wins; the slot keeps its sample's key
            const float kn = aes_key(d, word, w);
            take = kn > Wj;
            s = take ? kn : Wj;
        } else {
            // Eq. 7 against this slot's sample, then the slot's Alg. 2 decision
            take = decide_eq7(d, word, Wj, w, slot_delta<K>(r, c, lane), s);
        }
        const bool own = slot && now.y != 0u;
        take = take && own;
        if (take) r = make_float4(w, c.x, c.y, c.z);
        if (!slot) r = make_float4(0.f, 0.f, 0.f, 0.f);
        const uint64_t took = __ballot(take);
        slots += (uint32_t)__builtin_popcountll(took);
        const bool any = ((took >> (lane & ~((1u << lg) - 1u))) & ((1ull << (1u << lg)) - 1ull)) != 0u;
        changed += (uint32_t)__builtin_popcountll(__ballot(any && j == 0u));
        float q0 = 0.f, q1 = 0.f, q2 = 0.f;
        if constexpr (kResolves) {
            const float rs = resolve_scale(d, group_sum<K>(r.x, kk));
            q0 = group_sum<K>(r.x * r.y, kk) * rs;
            q1 = group_sum<K>(r.x * r.z, kk) * rs;
            q2 = group_sum<K>(r.x * r.w, kk) * rs;
        }
        if (own) st<kNtWsumSt>(d.wsum + s_at, s);
        if (take) {
            st4<kNtRecSt>(reinterpret_cast<float4*>(d.rec) + s_at, r);
            st<kNtIdxSt>(d.idx + s_at, d.t);
        }
        if (kResolves && j == first) sh.colour[e] = make_float4(q0, q1, q2, any ? 1.f : 0.f);
    }
    wave_lds_fence();

    // 3. one lane per pixel: the output rows
    if constexpr (kResolves) {
        const float4 q = sh.colour[lane];
        if (in && (OP != kIncremental || q.w != 0.f)) {
            float* o = d.out + 3 * (size_t)p;
            st<OP == kIncremental ? 0u : kNtOut>(o + 0, q.x);
            st<OP == kIncremental ? 0u : kNtOut>(o + 1, q.y);
            st<OP == kIncremental ? 0u : kNtOut>(o + 2, q.z);
        }
    }
    return slots + (changed << 16);
}

// The same with one lane per pixel, the record and values in registers: fewer
// instructions per pixel, which counts where colours differ everywhere (k = 3 and 4 at
// 3840x2160 with every colour changing: 210 and 267 us, one lane per slot 307 and 297;
// k = 8 at 1920x1080 137 and 148).  For the slot counts it is compiled for, but not 1 and
// 2, where one lane per slot is as short and reads whole lines (k = 2 at 1920x1080 32 us
// against 43).
template <int K, int OP, bool FOV = false>
__device__ __forceinline__ uint32_t pixel_per_slot(const FrameDesc& d, uint32_t x, uint32_t y,
                                                   const FovSrc* fs = nullptr)
{
    const uint32_t p = y * d.width + x;
    constexpr bool kUpdates = OP == kPush || OP == kFused || OP == kIncremental;
    constexpr bool kResolves = OP == kFused || OP == kIncremental;
    float4* rec = reinterpret_cast<float4*>(d.rec) + (size_t)p * K;
    uint32_t* idx = d.idx + (size_t)p * K;
    float* wslot = d.wsum + (size_t)p * K;

    // every slot's record and sum up front, then the pixel's own inputs
    float4 r[K];
    float W[K];
#pragma unroll
    for (int j = 0; j < K; ++j) r[j] = ld4<kNtRecLd>(rec + j);
    if constexpr (K % 4 == 0) {
#pragma unroll
        for (int j = 0; j < K; j += 4) {
            const float4 v = ld4<kNtWsumLd>(reinterpret_cast<const float4*>(wslot + j));
            W[j] = v.x;
            W[j + 1] = v.y;
            W[j + 2] = v.z;
            W[j + 3] = v.w;
        }
    } else {
#pragma unroll
        for (int j = 0; j < K; ++j) W[j] = ld<kNtWsumLd>(wslot + j);
    }
    uint32_t lv;
    float c0, c1, c2;
    if constexpr (FOV) {
        lv = fov_level(*fs, d.gx, d.gy, x, y);
        const float3 c = fov_colour(*fs, x, y, p, lv);
        c0 = c.x;
        c1 = c.y;
        c2 = c.z;
    } else {
        lv = ld<kNtLevel>(d.level + p);
        const float* color = d.color + 3 * (size_t)p;
        c0 = ld<kNtColor>(color + 0);
        c1 = ld<kNtColor>(color + 1);
        c2 = ld<kNtColor>(color + 2);
    }
    const float w = frame_weight(d, x, y, lv);
    const bool aes = d.bias == kAes;
    // Eq. 7: a slot whose sample has the new pixel's colour has |dL| = 0 exactly
    // (same_colour), so its Lab and CIE94 are not evaluated, nor the new
    // pixel's Lab when that holds for every slot.
    const bool bounded = lab_bounded(c0, c1, c2);
    uint32_t same = 0u;
    if (!aes) {
#pragma unroll
        for (int j = 0; j < K; ++j)
            if (bounded && same_colour(r[j], c0, c1, c2)) same |= 1u << j;
    }
    float3 lab_new = make_float3(0.f, 0.f, 0.f);
    if (!aes && same != (1u << K) - 1u) lab_new = rgb_to_lab(c0, c1, c2);
    const float4 fresh = make_float4(w, c0, c1, c2);

    float S = 0.f, a0 = 0.f, a1 = 0.f, a2 = 0.f;
    uint32_t tk = 0u;
    uint4 words = make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
    for (int j = 0; j < K; ++j) {
        float4 v = r[j];
        const float W1 = W[j];
        if ((j & 3) == 0) words = philox4x32_10(p, d.t, (uint32_t)(j >> 2), d.seed, d.stream_id);
        const uint32_t word = (j & 3) == 0 ? words.x : (j & 3) == 1 ? words.y : (j & 3) == 2 ? words.z : words.w;
        bool take;
        float s;
        if (aes) {
            // A-ES: the larger key log2(u) / w wins; the slot keeps its sample's key
            const float kn = aes_key(d, word, w);
            take = kn > W1;
            s = take ? kn : W1;
        } else {
            // Eq. 7 against this slot's sample, then the slot's Alg. 2 decision
            float dl = 0.0f;
            if (((same >> j) & 1u) == 0u) dl = delta_l(v.y, v.z, v.w, lab_new);
            take = decide_eq7(d, word, W1, w, dl, s);
        }
        if (take) {
            tk |= 1u << j;
            v = fresh;
            st4<kNtRecSt>(rec + j, fresh);
            st<kNtIdxSt>(idx + j, d.t);
        }
        W[j] = s;
        S = S + v.x;
        a0 = a0 + v.x * v.y;
        a1 = a1 + v.x * v.z;
        a2 = a2 + v.x * v.w;
    }
    if constexpr (K % 4 == 0) {
#pragma unroll
        for (int j = 0; j < K; j += 4)
            st4<kNtWsumSt>(reinterpret_cast<float4*>(wslot + j), make_float4(W[j], W[j + 1], W[j + 2], W[j + 3]));
    } else {
#pragma unroll
        for (int j = 0; j < K; ++j) st<kNtWsumSt>(wslot + j, W[j]);
    }
    if (kResolves && (OP != kIncremental || tk)) {
        const float rs = resolve_scale(d, S);
        float* o = d.out + 3 * (size_t)p;
        st<kNtOut>(o + 0, a0 * rs);
        st<kNtOut>(o + 1, a1 * rs);
        st<kNtOut>(o + 2, a2 * rs);
    }
    static_assert(kUpdates, "the resolve-only pass is the same under every bias mode");
    return __popc(tk) + (tk ? 0x10000u : 0u);
}

// Work items are visited in reverse order on odd frames, so each frame starts
// where the previous one ended: the store it touched last is still in the
// 256 MB Infinity Cache (a third of a 4K, k = 4 store) when it is read again.
// The order never changes a result.
__device__ __forceinline__ uint32_t frame_item(uint32_t block, uint32_t items, uint32_t t)
{
    return (t & 1u) ? items - 1u - block : block;
}

// Work items [T block, T block + T) of a frame.  Per-slot modes, an item per block:
// T = 0 one lane per pixel, 1 one lane per slot.
template <int K, int OP, bool PER_SLOT, int T, bool FOV>
__device__ __forceinline__ void frame_block(const FrameDesc& d, uint32_t block, const FovSrc* fs)
{
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63u;
    if constexpr (PER_SLOT && T == 0) {
        uint32_t x, y, n = 0u;
        if (item_pixel_of(d, block, wave, lane, x, y)) n = pixel_per_slot<K, OP, FOV>(d, x, y, fs);
        if (d.stats) add_stats(d.stats, n);
    } else if constexpr (PER_SLOT) {
        __shared__ PerSlotShare<K> share[kBlock / 64];
        const uint32_t n = per_slot_tile<K, OP, FOV>(d, block, wave, lane, share[wave], fs);
        if (d.stats) add_stats_uniform(d.stats, n);
    } else if constexpr (OP == kResolve && K > 0) {
        resolve_pixel<K>(d, block, wave);
    } else if constexpr (OP == kFused || OP == kFill || OP == kResolve) {
        __shared__ WholeShare share[kBlock / 64];
        const uint32_t n = whole_tile<K, OP, FOV>(d, block, wave, lane, share[wave], fs);
        if (OP != kResolve && d.stats) add_stats_uniform(d.stats, n);
    } else {
        __shared__ ListShare<T> share[kBlock / 64];
        const uint32_t n = stream_tiles<K, OP, T, FOV>(d, T * block, wave, lane, share[wave], fs);
        if (d.stats) add_stats_uniform(d.stats, n);
    }
}

// Waves per SIMD the frame kernels are compiled for and the most they run with.
// One lane per pixel reads a record in k accesses, which eight waves a SIMD push out
// of L1 between the first and the last.  resolve_pixel at 3840x2160: k = 8 213 us with 8
// waves, 191 with 6, 188 with 4, 216 with 2; k = 4 107, 106, 103 and 110; k = 2 49.5, 50.7,
// 52.5 and 69.  pixel_per_slot (T = 0), Eq. 7 and k = 4 at 3840x2160: 238.5 us with 8, 233.8
// with 5, 229 with 3; with every colour changing 263, 268 and 294.  (Foveated frames,
// which wait for samples of the frame first, are not held to 5: behind the mips, Eq. 7
// and k = 4 at 3840x2160 312 us with 5, 302 with 8.)
struct Waves {
    int least, most;
};
constexpr Waves frame_waves(int k, int op, int t)
{
    return op == kResolve && k >= 4 ? Waves{4, 4} : t == 0 ? Waves{5, 5} : Waves{8, 8};
}

template <int K, int OP, bool PER_SLOT = false, int T = 1>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(frame_waves(K, OP, T).least, frame_waves(K, OP, T).most)))
void frame_kernel(FrameDesc d)
{
    frame_block<K, OP, PER_SLOT, T, false>(d, frame_item(blockIdx.x, gridDim.x, d.t), nullptr);
}

// ---------------------------------------------------------------------------
// Batched tick: one launch for all the frames of a tick, any number of them.
// The frames' descriptors are a table in device memory or in the kernel's
// arguments (uniform data, read with scalar loads).  The consecutive frames of
// one context in a tick form a group, whose first frame (the leader) stands for
// it among the table's leaders, in the order the tick visits them; the tick's
// 256-pixel work items are numbered leader after leader, and a leader whose
// `rev` is set visits its own items last first (the host reverses the group
// order and sets `rev` on every other tick, so such a tick runs entirely
// backwards).  The grid has one block per work item (blocks past the last item
// exit): this measured faster than a persistent grid of resident blocks looping
// over the items -- the hardware's block dispatch balances the uneven per-item
// cost of the pass better than a fixed stride -- and without a loop over items
// the kernel keeps fewer values live (one more wave per SIMD).  A block finds
// its item's leader by binary search over the leaders' first items.  An item of
// a lone frame runs the single-frame per-pixel code for the frame's slot count
// and op (kFused, kCached, kCachedNt or kFill); an item of a group runs pixel_group (op
// kGroup), or else (run-time slot counts, per-slot modes) each of the group's
// frames in turn through the store, every pixel in the same wave, so each
// frame reads what the one before wrote.
// ---------------------------------------------------------------------------
// A wave's LDS in the batched kernel: a list (stream_tiles), in ticks with
// per-slot modes (PS) also a share (per_slot_tile).
template <bool PS>
union TickShare {
    ListShare<1> list;
    WholeShare whole;
};
template <>
union TickShare<true> {
    ListShare<1> list;
    WholeShare whole;
    PerSlotShare<0> slots;
    PerSlotShare<1> slots1;
    PerSlotShare<2> slots2;
    PerSlotShare<4> slots4;
};

// One wave's share of a lone frame's work item; counts its replaced slots and
// changed pixels.
template <bool PS>
__device__ __forceinline__ void tick_item(const FrameDesc& d, uint32_t local, uint32_t wave, uint32_t lane, TickShare<PS>& sh)
{
    if constexpr (PS) {
        if (per_slot_mode(d.bias)) {
            const uint32_t n = d.k == 1u   ? per_slot_tile<1, kFused>(d, local, wave, lane, sh.slots1)
                               : d.k == 2u ? per_slot_tile<2, kFused>(d, local, wave, lane, sh.slots2)
                               : d.k == 4u ? per_slot_tile<4, kFused>(d, local, wave, lane, sh.slots4)
                                           : per_slot_tile<0, kFused>(d, local, wave, lane, sh.slots);
            if (d.stats) add_stats_uniform(d.stats, n);
            return;
        }
    }
    uint32_t n = 0u;
#define FWRS_TICK_OPS(KK)                                                        \
    n = d.op == kCached ? stream_tiles<KK, kCached, 1>(d, local, wave, lane, sh.list)  \
      : d.op == kCachedNt ? stream_tiles<KK, kCachedNt, 1>(d, local, wave, lane, sh.list) \
      : d.op == kFill ? whole_tile<KK, kFill>(d, local, wave, lane, sh.whole)          \
                      : whole_tile<KK, kFused>(d, local, wave, lane, sh.whole)
    switch (d.k) {
        case 1: FWRS_TICK_OPS(1); break;
        case 2: FWRS_TICK_OPS(2); break;
        case 4: FWRS_TICK_OPS(4); break;
        case 8: FWRS_TICK_OPS(8); break;
        default: FWRS_TICK_OPS(0); break;
    }
#undef FWRS_TICK_OPS
    if (d.stats) add_stats_uniform(d.stats, n);
}

// One work item of a group run by pixel_group (d its leader); G as tick_blocks'.
template <int G>
__device__ __forceinline__ void tick_group_item(const FrameDesc& d, const FrameDesc* __restrict__ descs,
                                                uint32_t local, uint32_t wave)
{
    const FrameDesc* later = descs + d.more;
    uint32_t x, y, slots = 0u, changed = 0u;
    if (item_pixel_of(d, local, wave, threadIdx.x & 63u, x, y)) {
        switch (d.k) {
            case 1: pixel_group<1>(d, later, x, y, slots, changed); break;
            case 2: pixel_group<2>(d, later, x, y, slots, changed); break;
            case 4: pixel_group<4>(d, later, x, y, slots, changed); break;
            default:                                     // the host sets kGroup only for k in {1, 2, 4, 8}
                if constexpr (G == kTickGroups8) pixel_group<8>(d, later, x, y, slots, changed);
                break;
        }
    }
    if (d.stats) add_stats_wide(d.stats, slots, changed);
}

// The tick of table (head, descs), block by block; KIND: what the tick holds (G =
// kTickAlone: no groups; kTickStored: groups, all of them through the store; kTickGroups:
// groups, some run as kGroup, none of these with k = 8; kTickGroups8: some with k = 8;
// PS, + kTickPerSlot: frames of per-slot modes).  A group holds its pixels' whole
// records across its frames, which takes more registers than the single-frame paths
// (at k = 8 far more), and so does a per-slot frame's round, so each kind of tick
// runs the instantiation with only the paths it needs, at the best occupancy they
// allow without spilling registers.
template <int KIND>
__device__ __forceinline__ void tick_blocks(const TickHead& head, const FrameDesc* __restrict__ descs)
{
    constexpr int G = KIND % kTickPerSlot;
    constexpr bool PS = KIND >= kTickPerSlot;
    const uint32_t item = blockIdx.x;
    if (item >= head.total) return;
    uint32_t f = 0u, hi = head.n - 1u;               // last leader whose first item <= item
    while (f < hi) {
        const uint32_t mid = (f + hi + 1u) >> 1;
        if (descs[mid].first <= item) f = mid;
        else hi = mid - 1u;
    }
    const FrameDesc& d = descs[f];
    uint32_t local = item - d.first;
    if (d.rev) local = d.items - 1u - local;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if constexpr (G == kTickGroups || G == kTickGroups8) {
        if (d.op == kGroup) {
            tick_group_item<G>(d, descs, local, wave);
            return;
        }
    }
    __shared__ TickShare<PS> share[kBlock / 64];
    if constexpr (G == kTickAlone) {
        tick_item<PS>(d, local, wave, threadIdx.x & 63u, share[wave]);
    } else {
#pragma nounroll
        for (uint32_t f = 0; f < d.nf; ++f) {
            // A pixel's record may pass from one lane of the wave to another between
            // frames: no load may move above the stores of the frame before.  The wave's
            // accesses then go through its compute unit's cache in that order.
            if (f) {
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
            }
            // opaque, so that what the paths of every slot count derive from it is not
            // kept in registers over the loop
            uint32_t lane = threadIdx.x & 63u;
            asm volatile("" : "+v"(lane));
            tick_item<PS>(f ? descs[d.more + f - 1u] : d, local, wave, lane, share[wave]);
        }
    }
}

// Waves per SIMD the kernels are compiled for: the most that spill no register.
constexpr int tick_waves(int kind)
{
    constexpr int shared[] = {8, 8, 7, 5}, per_slot[] = {7, 7, 7, 5};
    return kind < kTickPerSlot ? shared[kind] : per_slot[kind - kTickPerSlot];
}

// The table in device memory.
template <int G>
__global__ __launch_bounds__(kBlock, tick_waves(G)) void tick_kernel(const TickHead* __restrict__ head,
                                                      const FrameDesc* __restrict__ descs)
{
    tick_blocks<G>(*head, descs);
}

// The table carried in the kernel's arguments (a tick of at most kArgFrames
// frames), read in place from the kernel-argument segment: indexing the
// by-value parameter itself would copy it to private memory first.
template <int G>
__global__ __launch_bounds__(kBlock, tick_waves(G)) void tick_args_kernel(const TickArgs a)
{
    (void)a;
    const TickArgs* in = (const TickArgs*)__builtin_amdgcn_kernarg_segment_ptr();
    tick_blocks<G>(in->head, in->descs);
}

// Writes descriptors carried as kernel arguments into a tick table.
__global__ __launch_bounds__(64) void tick_fill_kernel(uint32_t* __restrict__ table, const TickFill f)
{
    constexpr uint32_t kDescWords = sizeof(FrameDesc) / 4;
    static_assert(sizeof(FrameDesc) % 4 == 0, "descriptors are copied as words");
    const uint32_t* src = reinterpret_cast<const uint32_t*>(f.descs);
    uint32_t* dst = table + kTickDescOffset / 4 + (size_t)f.at * kDescWords;
    for (uint32_t i = threadIdx.x; i < f.count * kDescWords; i += blockDim.x) st<0u>(dst + i, src[i]);
    if (f.write_head && threadIdx.x < 4u) st<0u>(table + threadIdx.x, reinterpret_cast<const uint32_t*>(&f.head)[threadIdx.x]);
}

// ---------------------------------------------------------------------------
// Reprojected frame (Sec. 4.3).  Pixel p continues the reservoir of the pixel
// containing its centre moved back by its motion vector, if that point is in
// the image and its previous depth agrees with p's depth within the relative
// tolerance; otherwise p starts from the empty reservoir (flush).  Then the
// frame's update as in the other kernels (Eq. 4, the bias, Alg. 2 per slot),
// written densely to this frame's bank, and the resolve.  A gather from the
// previous bank, so the banks alternate; every slot is rewritten.
// Bound by its bytes (61 + 40k a pixel).  Sources, depth test and decisions run
// with one lane per pixel, the records with one lane per slot, so gathers and the
// dense stores are whole lines; those stores are non-temporal (nothing reads them
// before the next frame).  Against one lane per pixel: 3840x2160 k = 4 370 -> 307 us
// (322 with cached stores) = 6.0 TB/s, 1920x1080 k = 8 225 -> 139, Eq. 7 k = 4
// 141 -> 101, 640x360 14.8 -> 11.0.
// ---------------------------------------------------------------------------
template <int K, bool PER_SLOT>
struct ReprojShare {                            // one wave's pixels
    static constexpr int kBlocks = K ? (K + 3) / 4 : (kMaxK + 3) / 4;
    uint4 pixel[64];                            // {p, source, inside | history kept << 1, replaced slots (shared w_sum)}
    float4 colour[64];                          // the new colour, weight; then the resolve
    uint32_t words[PER_SLOT ? 64 : 1][4 * kBlocks];    // Philox words, one per slot (per-slot modes)
};

template <int K, bool PER_SLOT>
__device__ __forceinline__ void reproject_tile(const ReprojDesc& r, uint32_t item, uint32_t wave,
                                               ReprojShare<K, PER_SLOT>& sh)
{
    const FrameDesc& d = r.f;
    constexpr uint32_t D = K == 4 ? 4u : K == 8 ? 2u : 1u;      // rounds loaded ahead
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t kk = K ? (uint32_t)K : d.k;
    const uint32_t lg = group_log2<K>(kk), first = group_first<K>(kk);
    const uint32_t j = lane & ((1u << lg) - 1u), per = 64u >> lg;
    const bool slot = K || j < kk;
    const bool aes = d.bias == kAes;
    const float empty_slot = aes ? -INFINITY : 0.f;     // A-ES key / Eq. 7 sum of an empty slot

    // 1. one lane per pixel: the motion-compensated source
    uint32_t x, y;
    const bool in = item_pixel_of(d, item, wave, lane, x, y);
    if (!in) x = y = 0u;                                // lanes outside read pixel 0 and store nothing
    const uint32_t p = y * d.width + x;
    const float2 mv = ld2<kNtColor>(r.motion + 2 * (size_t)p);
    const float dc = ld<kNtColor>(r.depth + p);
    const uint32_t lv = ld<kNtLevel>(d.level + p);
    const float* color = d.color + 3 * (size_t)p;
    const float c0 = ld<kNtColor>(color + 0);
    const float c1 = ld<kNtColor>(color + 1);
    const float c2 = ld<kNtColor>(color + 2);
    const float sx = ((float)x + 0.5f) - mv.x;
    const float sy = ((float)y + 0.5f) - mv.y;
    const bool inside = sx >= 0.0f && sx < (float)d.width && sy >= 0.0f && sy < (float)d.height;
    uint32_t q = 0u;                                    // a valid pixel where there is no source
    if (inside) q = (uint32_t)floorf(sy) * d.width + (uint32_t)floorf(sx);
    sh.pixel[lane] = make_uint4(p, q, 0u, 0u);
    wave_lds_fence();

    // the first rounds' source records, in flight over the pixels' arithmetic
    // (unconditional; an empty history is selected afterwards)
    float4 v[D];
    uint32_t vi[D];
    float vw[D];
    auto load = [&](uint32_t b, float4& rec, uint32_t& idx, float& val) {
        const size_t at = (size_t)sh.pixel[b + (lane >> lg)].y * kk + (slot ? j : 0u);
        rec = ld4<0u>(reinterpret_cast<const float4*>(r.src_rec) + at);
        idx = ld<0u>(r.src_idx + at);
        val = PER_SLOT ? ld<kNtWsumLd>(r.src_wsum + at) : 0.f;
    };
#pragma unroll
    for (uint32_t u = 0; u < D; ++u)
        if (u * per < 64u) load(u * per, v[u], vi[u], vw[u]);

    // the depth test, the frame's candidate and (shared w_sum) the decisions
    const float dp = r.src_depth[q];
    const float ws = PER_SLOT ? 0.f : r.src_wsum[q];
    const uint32_t mc = r.src_cnt[q];
    const bool keep = inside && fabsf(dc - dp) <= r.tol * dc;      // NaN (no previous frame) compares false
    const uint32_t m = keep ? mc : 0u;
    float s = 0.f, w;
    uint32_t tk = 0u;
    if constexpr (PER_SLOT) {
        w = frame_weight(d, x, y, lv);
        for (uint32_t b = 0; 4u * b < kk; ++b) {
            const uint4 t = philox4x32_10(p, d.t, b, d.seed, d.stream_id);
            *reinterpret_cast<uint4*>(&sh.words[lane][4u * b]) = t;
        }
    } else {
        tk = decide<K>(d, x, y, p, lv, keep ? ws : 0.f, w, s);
    }
    sh.pixel[lane] = make_uint4(p, q, (in ? 1u : 0u) | (keep ? 2u : 0u), tk);
    sh.colour[lane] = make_float4(c0, c1, c2, w);
    const uint32_t flushed = (uint32_t)__builtin_popcountll(__ballot(in && !keep));
    wave_lds_fence();

    // 2. one lane per slot: Alg. 2, dense stores to this frame's bank, resolve sums
    uint32_t slots = 0u, changed = 0u;
    for (uint32_t b0 = 0; b0 < 64u; b0 += D * per)
#pragma unroll
    for (uint32_t u = 0; u < D; ++u) {
        const uint32_t b = b0 + u * per;
        if (b >= 64u) break;
        const uint32_t e = b + (lane >> lg);
        const uint4 px = sh.pixel[e];
        const float4 c = sh.colour[e];
        const size_t at = (size_t)px.x * kk + (slot ? j : 0u);
        const bool kept = (px.z & 2u) != 0u;
        float4 t = kept ? v[u] : make_float4(0.f, 0.f, 0.f, 0.f);
        uint32_t ti = kept ? vi[u] : 0xFFFFFFFFu;
        const float Wj = kept ? vw[u] : empty_slot;
        if (b + D * per < 64u) load(b + D * per, v[u], vi[u], vw[u]);
        bool take;
        float sj = 0.f;
        if constexpr (!PER_SLOT) {
            take = ((px.w >> j) & 1u) != 0u;
        } else {
            const uint32_t word = sh.words[e][slot ? j : 0u];
            if (aes) {
                const float kn = aes_key(d, word, c.w);
                take = kn > Wj;
                sj = take ? kn : Wj;
            } else {
                take = decide_eq7(d, word, Wj, c.w, slot_delta<K>(t, c, lane), sj);
            }
        }
        const bool own = slot && (px.z & 1u) != 0u;
        take = take && own;
        if (take) {
            t = make_float4(c.w, c.x, c.y, c.z);
            ti = d.t;
        }
        if (!slot) t = make_float4(0.f, 0.f, 0.f, 0.f);
        const uint64_t took = __ballot(take);
        slots += (uint32_t)__builtin_popcountll(took);
        const bool any = ((took >> (lane & ~((1u << lg) - 1u))) & ((1ull << (1u << lg)) - 1ull)) != 0u;
        changed += (uint32_t)__builtin_popcountll(__ballot(any && j == 0u));
        if (d.out) {                                    // uniform
            const float rs = resolve_scale(d, group_sum<K>(t.x, kk));
            const float q0 = group_sum<K>(t.x * t.y, kk) * rs;
            const float q1 = group_sum<K>(t.x * t.z, kk) * rs;
            const float q2 = group_sum<K>(t.x * t.w, kk) * rs;
            if (j == first) sh.colour[e] = make_float4(q0, q1, q2, 0.f);
        }
        if (own) {
            st4<kNtOut>(reinterpret_cast<float4*>(d.rec) + at, t);
            st<kNtOut>(d.idx + at, ti);
            if (PER_SLOT) st<kNtWsumSt>(d.wsum + at, sj);
        }
    }
    wave_lds_fence();

    // 3. one lane per pixel
    if (in) {
        if (!PER_SLOT) st<kNtWsumSt>(d.wsum + p, s);
        st<kNtWsumSt>(r.cnt + p, m + 1u);
        st<kNtWsumSt>(r.depth_out + p, dc);
        if (d.out) {
            const float4 o4 = sh.colour[lane];
            float* o = d.out + 3 * (size_t)p;
            st<kNtOut>(o + 0, o4.x);
            st<kNtOut>(o + 1, o4.y);
            st<kNtOut>(o + 2, o4.z);
        }
    }
    if (d.stats && (changed || flushed)) add_counts(d.stats, slots, changed, flushed);
}

template <int K, bool PER_SLOT>
__global__ __launch_bounds__(kBlock, 6) void reproject_kernel(ReprojDesc r)
{
    __shared__ ReprojShare<K, PER_SLOT> share[kBlock / 64];
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // forward order every frame: this dense pass (221 B per pixel) gains nothing
    // from the Infinity Cache and streams slightly slower backwards
    reproject_tile<K, PER_SLOT>(r, blockIdx.x, wave, share[wave]);
}

// ---------------------------------------------------------------------------
// Foveation generator (Sec. 4.3).  mip_kernel: one lane per mip-1 texel, the
// mip-2 texels from their mip-1 children by wave shuffles; each texel the mean
// of the children that exist, summed in row-major order.
// gauss_levels_kernel: the separable Gaussian levels, clamp to edge,
// accumulation in offset order.  foveate_kernel: the degraded frame and level map on their own;
// foveated_kernel: the same sampling fused into the reservoir pass.
// ---------------------------------------------------------------------------
struct MipArgs {
    const float* full;
    float* m1;
    float* m2;
    uint32_t w, h, w1, h1, w2, h2;
};

// 1 / n for the child counts a texel can have (1, 2 or 4): a power of two, so
// s * (1 / n) is exactly the correctly rounded s / n.
__device__ __forceinline__ float inv_count(uint32_t n)
{
    return n == 4u ? 0.25f : (n == 2u ? 0.5f : 1.0f);
}

// Mean of the children (2i + dx, 2j + dy) of a texel; every load is issued
// before the sums (children outside the source read the texel's first child
// and are not added).
__device__ __forceinline__ float3 texel_mean(const float* src, uint32_t sw, uint32_t sh, uint32_t i, uint32_t j)
{
    float3 v[4];
    bool in[4];
#pragma unroll
    for (uint32_t q = 0; q < 4; ++q) {
        const uint32_t x = 2 * i + (q & 1u), y = 2 * j + (q >> 1);
        in[q] = x < sw && y < sh;
        const float* c = src + ((size_t)(in[q] ? y : 2 * j) * sw + (in[q] ? x : 2 * i)) * 3;
        v[q] = make_float3(c[0], c[1], c[2]);
    }
    float s0 = 0.f, s1 = 0.f, s2 = 0.f;
    uint32_t n = 0u;
#pragma unroll
    for (uint32_t q = 0; q < 4; ++q)
        if (in[q]) {
            s0 = s0 + v[q].x;
            s1 = s1 + v[q].y;
            s2 = s2 + v[q].z;
            n = n + 1u;
        }
    const float r = inv_count(n);
    return make_float3(s0 * r, s1 * r, s2 * r);
}

__global__ __launch_bounds__(kBlock) void mip_kernel(MipArgs a)
{
    // One lane per mip-1 texel: a wave covers 32 mip-1 columns of the two
    // mip-1 rows under one mip-2 row (lanes 0-31 the upper row, 32-63 the
    // lower); lane pairs (2m, 2m + 1) of each half are the children of one
    // mip-2 texel, gathered by wave shuffles in row-major order.
    const uint32_t wave = (blockIdx.x * kBlock + threadIdx.x) >> 6, lane = threadIdx.x & 63u;
    const uint32_t strips = (a.w1 + 31u) / 32u;
    if (wave >= strips * a.h2) return;                 // whole waves only
    const uint32_t i1 = (wave % strips) * 32u + (lane & 31u), j2 = wave / strips;
    const uint32_t j1 = 2u * j2 + (lane >> 5);
    const bool own = i1 < a.w1 && j1 < a.h1;
    const float3 m = texel_mean(a.full, a.w, a.h, own ? i1 : 0u, own ? j1 : 0u);
    if (own) {
        float* o = a.m1 + ((size_t)j1 * a.w1 + i1) * 3;
        o[0] = m.x;
        o[1] = m.y;
        o[2] = m.z;
    }
    // children of mip-2 texel (i1 / 2, j2) for the even lanes of the upper row
    const int src[3] = {(int)(lane ^ 1u), (int)(lane + 32u) & 63, (int)((lane ^ 1u) + 32u) & 63};
    float v[4][3] = {{m.x, m.y, m.z}};
    bool in[4] = {own};
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        v[q + 1][0] = __shfl(m.x, src[q]);
        v[q + 1][1] = __shfl(m.y, src[q]);
        v[q + 1][2] = __shfl(m.z, src[q]);
        in[q + 1] = __shfl((int)own, src[q]) != 0;
    }
    if ((lane & 33u) == 0u && own) {                   // even lane of the upper row, texel exists
        float s0 = 0.f, s1 = 0.f, s2 = 0.f;
        uint32_t n = 0u;
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (in[q]) {
                s0 = s0 + v[q][0];
                s1 = s1 + v[q][1];
                s2 = s2 + v[q][2];
                n = n + 1u;
            }
        const float r = inv_count(n);
        float* o = a.m2 + ((size_t)j2 * a.w2 + i1 / 2u) * 3;
        o[0] = s0 * r;
        o[1] = s1 * r;
        o[2] = s2 * r;
    }
}

// Gaussian levels from one read of the frame, into one plane: every pixel of
// level l >= 1 gets the frame blurred with sigma 2^(l-1) (radius kGaussR1 or
// kGaussR2) at that pixel; level-0 pixels are not written.  The channels are
// independent, so a row is W * 3 floats and a thread owns one float column: a
// block owns kGaussCols of them and a strip of ROWS output rows, and walks the
// strip's rows and a halo of kGaussR2 rows above and below (clamped to the
// image) in batches of kGaussBatch: a batch is staged in LDS with its halo of
// 3 kGaussR2 floats on either side (pixels clamped) while the next one is being
// loaded, one barrier a batch.
//
// Sums start at zero and add the taps in offset order, horizontally, then
// vertically, each product rounded.  The vertical sums are kept per output row
// in progress: when a row's horizontal sum h arrives, it is tap i of the output
// row i rows further up for every i, so acc[i] = acc[i - 1] + g[i] h moves every
// sum one tap on (no register moves), and the weights' symmetry leaves 7 products
// for the 13 taps.  A column thread thus takes 13 + 13 operations across and
// 7 + 13 down per row.  Which levels a block needs comes from its rectangle's
// distances to the gaze, widened by 2^-10 relative so that rounding can only make
// it need more.
//
// Bound by the vector ALU (a fused multiply-add would round differently), at
// about 60% of its issue rate: 84 registers leave 5 waves per SIMD, and 6 spill (51
// -> 61 us).  One thread per pixel column with a window of row sums took 276
// instructions per pixel and walked row, and its few waves left the chip idle
// below 4K.  The generator call at 2560x1440 went from 68 to 51 us (these levels 53
// to 36), at 1920x1080 from 42 to 33, at 256x256 from 20 to 9.5, at 3840x2160 from
// 121 to 104.  Four neighbouring floats per lane read 2.6 times less LDS but leave
// 1.3 waves per SIMD at 2560x1440 (52 us; 99 at 3840x2160); two floats: 57 and 117;
// the two levels in blocks of their own: 51 and 108; two rows a batch: 50 and 107.
struct GaussArgs {
    const float* src;
    float* dst;
    uint32_t w, h, cols;                               // cols: blocks per strip
    float gx, gy, r0sq, r1sq;
    float g1[kGaussR1 + 1];                            // weights of offsets 0 .. R (symmetric)
    float g2[kGaussR2 + 1];
};

constexpr int kGaussBatch = 4;

// The vertical sums of radius R after one more row: acc[i] is the sum, taps 0 to
// i, of the output row for which this row is tap i; returns the one that is
// complete.
template <int R>
__device__ __forceinline__ float gauss_down(float (&acc)[2 * R], const float (&g)[R + 1], float h)
{
    float m[R + 1];
#pragma unroll
    for (int i = 0; i <= R; ++i) m[i] = g[i] * h;      // offset -i and i
    const float done = acc[2 * R - 1] + m[R];
#pragma unroll
    for (int i = 2 * R - 1; i > 0; --i) acc[i] = acc[i - 1] + m[i < R ? R - i : i - R];
    acc[0] = 0.0f + m[R];
    return done;
}

// The horizontal sums of radius R of a batch's rows around float c of each
// (floats of one channel are 3 apart), the rows' chains of additions side by side.
template <int R, int B, int SEG>
__device__ __forceinline__ void gauss_across(const float (*rows)[SEG], int c, const float (&g)[R + 1], float (&t)[B])
{
#pragma unroll
    for (int u = 0; u < B; ++u) t[u] = 0.0f;
#pragma unroll
    for (int i = -R; i <= R; ++i)
#pragma unroll
        for (int u = 0; u < B; ++u) t[u] = t[u] + g[i < 0 ? -i : i] * rows[u][c + 3 * i];
}

template <int ROWS>
__global__ __launch_bounds__(kGaussCols) void gauss_levels_kernel(GaussArgs a)
{
    constexpr int R1 = kGaussR1, R2 = kGaussR2, B = kGaussBatch;
    constexpr int SEG = kGaussCols + 6 * R2;           // floats of a staged row
    constexpr int NV = ROWS + 2 * R2;                  // rows walked (halo included)
    static_assert(NV % B == 0 && 6 * R2 <= kGaussCols, "whole batches; the halo is one extra float per thread at most");
    __shared__ float seg[2][B][SEG];

    const int tid = (int)threadIdx.x;
    const int W = (int)a.w, H = (int)a.h;
    const uint32_t bx = blockIdx.x % a.cols, by = blockIdx.x / a.cols;   // one-dimensional grid, row-major
    const int f0 = (int)bx * kGaussCols, y0 = (int)by * ROWS;
    const int x = (f0 + tid) / 3;
    const bool own = x < W;

    // Levels present in the block's pixels (block-uniform, conservative).
    bool need1, need2;
    {
        const float xa = (float)(f0 / 3) + 0.5f, xb = (float)min((f0 + kGaussCols - 1) / 3, W - 1) + 0.5f;
        const float ya = (float)y0 + 0.5f, yb = (float)min(y0 + ROWS, H) - 0.5f;
        const float nx = fminf(fmaxf(a.gx, xa), xb) - a.gx, ny = fminf(fmaxf(a.gy, ya), yb) - a.gy;
        const float fx = fmaxf(fabsf(xa - a.gx), fabsf(xb - a.gx)), fy = fmaxf(fabsf(ya - a.gy), fabsf(yb - a.gy));
        const float dmin = nx * nx + ny * ny, dmax = fx * fx + fy * fy;
        need1 = dmin * (1.0f - 0x1p-10f) <= a.r1sq && dmax * (1.0f + 0x1p-10f) > a.r0sq;
        need2 = dmax * (1.0f + 0x1p-10f) > a.r1sq;
    }
    if (!need1 && !need2) return;                      // every pixel at level 0

    // Staged float e = tid (and kGaussCols + tid in the halo) is float f0 - 3 R2 + e
    // of the row, its pixel clamped.
    auto column = [&](int e) {
        const int fs = f0 + e, px = fs / 3 - R2;
        return min(max(px, 0), W - 1) * 3 + fs % 3;
    };
    const int off0 = column(tid);
    const bool extra = tid < 6 * R2;
    const int off1 = extra ? column(kGaussCols + tid) : off0;
    float stage[B], halo[B];
    auto fetch = [&](int vb) {
#pragma unroll
        for (int u = 0; u < B; ++u) {
            const int yy = min(max(y0 - R2 + vb + u, 0), H - 1);
            const float* row = a.src + (size_t)yy * (size_t)W * 3;
            stage[u] = row[off0];
            halo[u] = extra ? row[off1] : 0.f;
        }
    };

    const float dx = ((float)x + 0.5f) - a.gx;
    const float dx2 = dx * dx;
    // The finished sum o of image row y goes out where the pixel is at this level.
    auto store = [&](int y, uint32_t level, float o) {
        const float dy = ((float)y + 0.5f) - a.gy;     // ring_level
        const float d2 = dx2 + dy * dy;
        const uint32_t at = d2 <= a.r0sq ? 0u : (d2 <= a.r1sq ? 1u : 2u);
        if (own && at == level) (a.dst + (size_t)y * (size_t)W * 3 + f0)[tid] = o;
    };

    float acc1[2 * R1], acc2[2 * R2];
#pragma unroll
    for (int i = 0; i < 2 * R1; ++i) acc1[i] = 0.f;
#pragma unroll
    for (int i = 0; i < 2 * R2; ++i) acc2[i] = 0.f;
    fetch(0);
    for (int vb = 0; vb < NV; vb += B) {
        float(*s)[SEG] = seg[(vb / B) & 1];
#pragma unroll
        for (int u = 0; u < B; ++u) {
            s[u][tid] = stage[u];
            if (extra) s[u][kGaussCols + tid] = halo[u];
        }
        __syncthreads();                               // also: the other buffer's readers are done with it
        if (vb + B < NV) fetch(vb + B);
        // walked row v is image row y0 - R2 + v (clamped), the last tap of the row R further up
        float h[B];
        if (need2) {
            gauss_across<R2, B, SEG>(s, tid + 3 * R2, a.g2, h);
#pragma unroll
            for (int u = 0; u < B; ++u) h[u] = gauss_down<R2>(acc2, a.g2, h[u]);
#pragma unroll
            for (int u = 0; u < B; ++u) {
                const int v = vb + u, y = y0 + v - 2 * R2;
                if (v >= 2 * R2 && y < H) store(y, 2u, h[u]);
            }
        }
        if (need1) {
            gauss_across<R1, B, SEG>(s, tid + 3 * R2, a.g1, h);
#pragma unroll
            for (int u = 0; u < B; ++u) h[u] = gauss_down<R1>(acc1, a.g1, h[u]);
#pragma unroll
            for (int u = 0; u < B; ++u) {
                const int v = vb + u, y = y0 + v - R1 - R2;
                if (v >= R1 + R2 && v < R1 + R2 + ROWS && y < H) store(y, 1u, h[u]);
            }
        }
    }
}

struct FoveateArgs {
    FovSrc s;
    float* color;
    uint8_t* level;
    uint32_t w, h;
    float gx, gy;
};

__global__ __launch_bounds__(kBlock) void foveate_kernel(FoveateArgs a)
{
    const uint32_t p = blockIdx.x * kBlock + threadIdx.x;
    if (p >= a.w * a.h) return;
    const uint32_t x = p % a.w, y = p / a.w;
    const uint32_t lv = fov_level(a.s, a.gx, a.gy, x, y);
    const float3 c = fov_colour(a.s, x, y, p, lv);
    float* o = a.color + (size_t)p * 3;
    o[0] = c.x;
    o[1] = c.y;
    o[2] = c.z;
    a.level[p] = (uint8_t)lv;
}

template <int K, bool PER_SLOT, int OP, int T = 1>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(frame_waves(K, OP, T).least, 8)))
void foveated_kernel(FovDesc fd)
{
    frame_block<K, OP, PER_SLOT, T, true>(fd.f, frame_item(blockIdx.x, gridDim.x, fd.f.t), &fd.s);
}

__global__ void fill_u32_kernel(uint32_t* __restrict__ p, size_t n, uint32_t v)
{
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
        p[i] = v;
}

// ---------------------------------------------------------------------------
// Host-side launchers.
// ---------------------------------------------------------------------------
template <int OP, int T>
static hipError_t launch_shared(const FrameDesc& d, hipStream_t stream)
{
    const dim3 grid((d.items + (uint32_t)T - 1u) / (uint32_t)T), block(kBlock);
    switch (d.k) {
        case 1: hipLaunchKernelGGL((frame_kernel<1, OP, false, T>), grid, block, 0, stream, d); break;
        case 2: hipLaunchKernelGGL((frame_kernel<2, OP, false, T>), grid, block, 0, stream, d); break;
        case 4: hipLaunchKernelGGL((frame_kernel<4, OP, false, T>), grid, block, 0, stream, d); break;
        case 8:                                         // two tiles: up to 4 slots (takes_two_tiles)
            if constexpr (T == 1) hipLaunchKernelGGL((frame_kernel<8, OP, false, T>), grid, block, 0, stream, d);
            break;
        default: hipLaunchKernelGGL((frame_kernel<0, OP, false, T>), grid, block, 0, stream, d); break;
    }
    return hipGetLastError();
}

template <int OP>
static hipError_t launch_frame_op(const FrameDesc& d, hipStream_t stream)
{
    // the per-slot modes keep no resolve plane: they run kPush, kFused or kIncremental
    if constexpr (OP == kPush || OP == kFused || OP == kIncremental) {
        if (per_slot_mode(d.bias)) {
            const dim3 grid(d.items), block(kBlock);
            switch (d.k) {
                case 1: hipLaunchKernelGGL((frame_kernel<1, OP, true, 1>), grid, block, 0, stream, d); break;
                case 2: hipLaunchKernelGGL((frame_kernel<2, OP, true, 1>), grid, block, 0, stream, d); break;
                case 3: hipLaunchKernelGGL((frame_kernel<3, OP, true, 0>), grid, block, 0, stream, d); break;
                case 4: hipLaunchKernelGGL((frame_kernel<4, OP, true, 0>), grid, block, 0, stream, d); break;
                case 5: hipLaunchKernelGGL((frame_kernel<5, OP, true, 0>), grid, block, 0, stream, d); break;
                case 8: hipLaunchKernelGGL((frame_kernel<8, OP, true, 0>), grid, block, 0, stream, d); break;
                default: hipLaunchKernelGGL((frame_kernel<0, OP, true, 1>), grid, block, 0, stream, d); break;
            }
            return hipGetLastError();
        }
    }
    if constexpr (OP == kIncremental || OP == kPush) {
        if (takes_two_tiles(d, OP)) return launch_shared<OP, 2>(d, stream);
    }
    return launch_shared<OP, 1>(d, stream);
}

hipError_t launch_frame(const FrameDesc& d, int op, hipStream_t stream)
{
    if (d.items == 0u) return hipSuccess;
    switch (op) {
        case kPush: return launch_frame_op<kPush>(d, stream);
        case kResolve: return launch_frame_op<kResolve>(d, stream);
        case kIncremental: return launch_frame_op<kIncremental>(d, stream);
        case kCached: return launch_frame_op<kCached>(d, stream);
        case kCachedNt: return launch_frame_op<kCachedNt>(d, stream);
        case kFill: return launch_frame_op<kFill>(d, stream);
        default: return launch_frame_op<kFused>(d, stream);
    }
}

// One of a table of kernels, one per kind of tick.
#define FWRS_TICK_KINDS(f) {f<0>, f<1>, f<2>, f<3>, f<4>, f<5>, f<6>, f<7>}
static_assert(kTickKinds == 8, "a kernel per kind");
static void (*const kTickKernels[])(const TickHead*, const FrameDesc*) = FWRS_TICK_KINDS(tick_kernel);
static void (*const kTickArgsKernels[])(TickArgs) = FWRS_TICK_KINDS(tick_args_kernel);
#undef FWRS_TICK_KINDS

hipError_t launch_tick(const void* table, uint32_t grid, int kind, hipStream_t stream)
{
    if (grid == 0u) return hipSuccess;
    const TickHead* head = static_cast<const TickHead*>(table);
    const FrameDesc* descs = reinterpret_cast<const FrameDesc*>(static_cast<const char*>(table) + kTickDescOffset);
    hipLaunchKernelGGL(kTickKernels[kind], dim3(grid), dim3(kBlock), 0, stream, head, descs);
    return hipGetLastError();
}

hipError_t launch_tick_fill(void* table, const TickFill& f, hipStream_t stream)
{
    hipLaunchKernelGGL(tick_fill_kernel, dim3(1), dim3(64), 0, stream, static_cast<uint32_t*>(table), f);
    return hipGetLastError();
}

hipError_t launch_reproject(const ReprojDesc& r, hipStream_t stream)
{
    const dim3 grid(r.f.items), block(kBlock);
    const bool eq7 = per_slot_mode(r.f.bias);
    switch (r.f.k) {
        case 1:
            if (eq7) hipLaunchKernelGGL((reproject_kernel<1, true>), grid, block, 0, stream, r);
            else hipLaunchKernelGGL((reproject_kernel<1, false>), grid, block, 0, stream, r);
            break;
        case 2:
            if (eq7) hipLaunchKernelGGL((reproject_kernel<2, true>), grid, block, 0, stream, r);
            else hipLaunchKernelGGL((reproject_kernel<2, false>), grid, block, 0, stream, r);
            break;
        case 4:
            if (eq7) hipLaunchKernelGGL((reproject_kernel<4, true>), grid, block, 0, stream, r);
            else hipLaunchKernelGGL((reproject_kernel<4, false>), grid, block, 0, stream, r);
            break;
        case 8:
            if (eq7) hipLaunchKernelGGL((reproject_kernel<8, true>), grid, block, 0, stream, r);
            else hipLaunchKernelGGL((reproject_kernel<8, false>), grid, block, 0, stream, r);
            break;
        default:
            if (eq7) hipLaunchKernelGGL((reproject_kernel<0, true>), grid, block, 0, stream, r);
            else hipLaunchKernelGGL((reproject_kernel<0, false>), grid, block, 0, stream, r);
            break;
    }
    return hipGetLastError();
}

hipError_t launch_mips(const float* full, float* m1, float* m2, uint32_t w, uint32_t h, hipStream_t stream)
{
    MipArgs a{full, m1, m2, w, h, (w + 1) / 2, (h + 1) / 2, 0u, 0u};
    a.w2 = (a.w1 + 1) / 2;
    a.h2 = (a.h1 + 1) / 2;
    const uint64_t threads = (uint64_t)((a.w1 + 31u) / 32u) * a.h2 * 64u;   // whole waves
    hipLaunchKernelGGL(mip_kernel, dim3((uint32_t)((threads + kBlock - 1) / kBlock)), dim3(kBlock), 0, stream, a);
    return hipGetLastError();
}

hipError_t launch_gauss_levels(const float* full, float* dst, uint32_t w, uint32_t h, float gx, float gy, float r0sq,
                               float r1sq, const float* g1, const float* g2, hipStream_t stream)
{
    GaussArgs a{};
    a.src = full;
    a.dst = dst;
    a.w = w;
    a.h = h;
    a.gx = gx;
    a.gy = gy;
    a.r0sq = r0sq;
    a.r1sq = r1sq;
    for (int i = 0; i <= kGaussR1; ++i) a.g1[i] = g1[kGaussR1 + i];
    for (int i = 0; i <= kGaussR2; ++i) a.g2[i] = g2[kGaussR2 + i];
    // The tallest strip (the halo costs 12 walked rows per strip) whose grid still
    // gives every compute unit four blocks: at 1920x1080 a generator call takes 33 us
    // with 16 rows (1564 blocks), 35 with 32 (782); at 3840x2160 104 us with 64 rows,
    // 107 with 32.
    a.cols = (uint32_t)(((uint64_t)w * 3u + kGaussCols - 1u) / kGaussCols);
    auto blocks = [&](uint32_t rows) { return (uint64_t)a.cols * ((h + rows - 1) / rows); };
    const dim3 block(kGaussCols);
    const uint64_t enough = 1024u;
    if (blocks(64) >= enough)
        hipLaunchKernelGGL(gauss_levels_kernel<64>, dim3((uint32_t)blocks(64)), block, 0, stream, a);
    else if (blocks(32) >= enough)
        hipLaunchKernelGGL(gauss_levels_kernel<32>, dim3((uint32_t)blocks(32)), block, 0, stream, a);
    else if (blocks(16) >= enough)
        hipLaunchKernelGGL(gauss_levels_kernel<16>, dim3((uint32_t)blocks(16)), block, 0, stream, a);
    else if (blocks(8) >= enough)
        hipLaunchKernelGGL(gauss_levels_kernel<8>, dim3((uint32_t)blocks(8)), block, 0, stream, a);
    else
        hipLaunchKernelGGL(gauss_levels_kernel<4>, dim3((uint32_t)blocks(4)), block, 0, stream, a);
    return hipGetLastError();
}

hipError_t launch_foveate(const FovSrc& s, float* color, uint8_t* level, uint32_t w, uint32_t h, float gx, float gy,
                          hipStream_t stream)
{
    FoveateArgs a{s, color, level, w, h, gx, gy};
    const uint32_t n = w * h;
    hipLaunchKernelGGL(foveate_kernel, dim3((n + kBlock - 1) / kBlock), dim3(kBlock), 0, stream, a);
    return hipGetLastError();
}

hipError_t launch_foveated(const FovDesc& fd, int op, hipStream_t stream)
{
    if (fd.f.items == 0u) return hipSuccess;
    const bool ps = per_slot_mode(fd.f.bias);
    const dim3 grid(fd.f.items), block(kBlock);
#define FWRS_FOV_LAUNCH(KK, PS, OPV) hipLaunchKernelGGL((foveated_kernel<KK, PS, OPV>), grid, block, 0, stream, fd)
#define FWRS_FOV_OPS(KK)                                      \
    do {                                                      \
        if (op == kCached) FWRS_FOV_LAUNCH(KK, false, kCached);   \
        else if (op == kCachedNt) FWRS_FOV_LAUNCH(KK, false, kCachedNt); \
        else if (op == kFill) FWRS_FOV_LAUNCH(KK, false, kFill);  \
        else if (op == kPush) FWRS_FOV_LAUNCH(KK, false, kPush);  \
        else FWRS_FOV_LAUNCH(KK, false, kFused);              \
    } while (0)
    if (ps) {
#define FWRS_FOV_PER_SLOT(KK, T)                                                                                 \
    do {                                                                                                         \
        if (op == kPush) hipLaunchKernelGGL((foveated_kernel<KK, true, kPush, T>), grid, block, 0, stream, fd);  \
        else hipLaunchKernelGGL((foveated_kernel<KK, true, kFused, T>), grid, block, 0, stream, fd);             \
    } while (0)
        switch (fd.f.k) {
            case 1: FWRS_FOV_PER_SLOT(1, 1); break;
            case 2: FWRS_FOV_PER_SLOT(2, 1); break;
            case 3: FWRS_FOV_PER_SLOT(3, 0); break;
            case 4: FWRS_FOV_PER_SLOT(4, 0); break;
            case 5: FWRS_FOV_PER_SLOT(5, 0); break;
            default: FWRS_FOV_PER_SLOT(0, 1); break;
        }
#undef FWRS_FOV_PER_SLOT
    } else {
        switch (fd.f.k) {
            case 4: FWRS_FOV_OPS(4); break;
            case 8: FWRS_FOV_OPS(8); break;
            default: FWRS_FOV_OPS(0); break;
        }
    }
#undef FWRS_FOV_OPS
#undef FWRS_FOV_LAUNCH
    return hipGetLastError();
}

hipError_t launch_fill_u32(uint32_t* p, size_t n, uint32_t v, hipStream_t stream)
{
    if (n == 0) return hipSuccess;
    size_t blocks = (n + kBlock - 1) / kBlock;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(fill_u32_kernel, dim3((uint32_t)blocks), dim3(kBlock), 0, stream, p, n, v);
    return hipGetLastError();
}

hipError_t launch_tick_args(const TickArgs& a, int kind, hipStream_t stream)
{
    const uint32_t grid = a.head.total;
    if (grid == 0u) return hipSuccess;
    hipLaunchKernelGGL(kTickArgsKernels[kind], dim3(grid), dim3(kBlock), 0, stream, a);
    return hipGetLastError();
}

void* tick_kernel_entry(int kind) { return reinterpret_cast<void*>(kTickKernels[kind]); }

}  // namespace fwrs
