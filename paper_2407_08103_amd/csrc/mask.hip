// Decode step: loop body of Algorithm 2 after ComputeLogits (allowed set, -inf penalty, greedy
// token choice, edge traversal), batched over sequences, for gfx950.
//
// The allowed set of a state is its row of allowed bits (1 bit per token, written by the compile
// stage), so a step has |V| logits and |V|/8 mask bytes per sequence before it, and one table
// entry for the chosen token.  Nothing here is a contraction: the kernels stream logits with
// 16-byte loads and reduce (value, position) pairs across lanes; `parts` workgroups share a row
// and meet through two device-scope atomics per workgroup.  A logit whose token is not allowed
// cannot matter, so a wavefront whose part of the row allows few tokens reads the mask bytes
// first and then only the groups of eight logits that hold an allowed token (unless the masked
// row is to be written, which takes every logit).
//
// Ordering of candidates (exact path).  Each allowed logit is mapped to an unsigned key that
// preserves the order of the floating-point values, with every NaN mapped to the key of -inf and
// -0 to +0.  Candidates are compared as the 64-bit number (key << 32) | (0xFFFFFFFF - token), so
// the largest value wins and the lowest token id wins ties; 0 means "nothing allowed" (the
// smallest key of an allowed token, that of -inf, is above 0).
//
// bf16 fast path.  Two logits per 32-bit register are turned into 16-bit unsigned keys with
// packed instructions (arithmetic shift, one three-input bit operation), multiplied by their
// allowed bit (0 or 1), and folded with packed max; a lane remembers its best key and the group
// of eight tokens that holds it.  The packed keys do not treat NaN and -0 specially, so a row
// whose winning key is NaN-like, not above -inf, or a zero is handed to the exact path, which the
// last workgroup of the row runs over the whole row.
#include "pda_device.h"
#include "tdfa_internal.h"

#include <algorithm>
#include <type_traits>

namespace tdfa {
namespace {

constexpr int kMaxThreads = 1024;      // workgroup sizes used: 256 .. 1024
constexpr int kMaxWaves = kMaxThreads / 64;

typedef short s16x2 __attribute__((ext_vector_type(2)));
typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ uint32_t key_bf16(uint32_t h)
{
    if ((h & 0x7FFFu) > 0x7F80u) h = 0xFF80u;                 // NaN ranks as -inf
    if ((h & 0x7FFFu) == 0) h = 0;                            // -0 equals +0
    return (h & 0x8000u) ? (~h & 0xFFFFu) : (h | 0x8000u);
}

__device__ __forceinline__ uint32_t key_f32(uint32_t u)
{
    if ((u & 0x7FFFFFFFu) > 0x7F800000u) u = 0xFF800000u;     // NaN ranks as -inf
    if ((u & 0x7FFFFFFFu) == 0) u = 0;                        // -0 equals +0
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// Maximum of a 32-bit value over the 64 lanes of a wavefront (all lanes must be active); the result
// is uniform.  Four cross-lane steps inside each row of 16 lanes (data-parallel primitives, no LDS
// traffic), then the four row results are read as scalars.
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v)
{
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, true));    // quad_perm [1,0,3,2]
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, true));    // quad_perm [2,3,0,1]
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xF, 0xF, true));   // row_half_mirror
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x140, 0xF, 0xF, true));   // row_mirror
    const uint32_t r0 = (uint32_t)__builtin_amdgcn_readlane((int)v, 0), r1 = (uint32_t)__builtin_amdgcn_readlane((int)v, 16);
    const uint32_t r2 = (uint32_t)__builtin_amdgcn_readlane((int)v, 32), r3 = (uint32_t)__builtin_amdgcn_readlane((int)v, 48);
    return max(max(r0, r1), max(r2, r3));
}

// 64-bit maximum over a wavefront: the high words first, then the low words of the lanes that hold
// the highest high word.
__device__ __forceinline__ unsigned long long wave_max_u64(unsigned long long v)
{
    const uint32_t hi = (uint32_t)(v >> 32), lo = (uint32_t)v;
    const uint32_t mh = wave_max_u32(hi);
    const uint32_t ml = wave_max_u32(hi == mh ? lo : 0u);
    return ((unsigned long long)mh << 32) | ml;
}

// Maximum over the workgroup; the result is valid in thread 0.  Ends with a barrier-free read, so
// callers that reuse `wave_best` must synchronise first.
__device__ __forceinline__ unsigned long long block_max_u64(unsigned long long v, unsigned long long* wave_best)
{
    v = wave_max_u64(v);
    if ((threadIdx.x & 63) == 0) wave_best[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        const int n_waves = (int)blockDim.x >> 6;
        for (int w = 1; w < n_waves; ++w) v = wave_best[w] > v ? wave_best[w] : v;
    }
    return v;
}

template <int DTYPE> struct ElemOf { using type = uint32_t; };
template <> struct ElemOf<TDFA_BF16> { using type = uint16_t; };

template <int DTYPE>
__device__ __forceinline__ void load_group(const typename ElemOf<DTYPE>::type* row, int t, int V,
                                           typename ElemOf<DTYPE>::type (&e)[8])
{
    using Elem = typename ElemOf<DTYPE>::type;
    constexpr Elem NEG_INF = DTYPE == TDFA_F32 ? (Elem)0xFF800000u : (Elem)0xFF80u;
    if (t + 8 <= V) {
        if constexpr (DTYPE == TDFA_F32) {
            const uint4 x0 = *reinterpret_cast<const uint4*>(row + t);
            const uint4 x1 = *reinterpret_cast<const uint4*>(row + t + 4);
            e[0] = x0.x; e[1] = x0.y; e[2] = x0.z; e[3] = x0.w;
            e[4] = x1.x; e[5] = x1.y; e[6] = x1.z; e[7] = x1.w;
        } else {
            const uint4 x = *reinterpret_cast<const uint4*>(row + t);
            e[0] = (Elem)(x.x & 0xFFFFu); e[1] = (Elem)(x.x >> 16);
            e[2] = (Elem)(x.y & 0xFFFFu); e[3] = (Elem)(x.y >> 16);
            e[4] = (Elem)(x.z & 0xFFFFu); e[5] = (Elem)(x.z >> 16);
            e[6] = (Elem)(x.w & 0xFFFFu); e[7] = (Elem)(x.w >> 16);
        }
    } else {
#pragma unroll
        for (int j = 0; j < 8; ++j) e[j] = t + j < V ? row[t + j] : NEG_INF;
    }
}

template <int DTYPE>
__device__ __forceinline__ void store_group(typename ElemOf<DTYPE>::type* orow, int t, int V,
                                            const typename ElemOf<DTYPE>::type (&e)[8])
{
    if (t + 8 <= V) {
        if constexpr (DTYPE == TDFA_F32) {
            *reinterpret_cast<uint4*>(orow + t) = make_uint4(e[0], e[1], e[2], e[3]);
            *reinterpret_cast<uint4*>(orow + t + 4) = make_uint4(e[4], e[5], e[6], e[7]);
        } else {
            *reinterpret_cast<uint4*>(orow + t) =
                make_uint4((uint32_t)e[0] | ((uint32_t)e[1] << 16), (uint32_t)e[2] | ((uint32_t)e[3] << 16),
                           (uint32_t)e[4] | ((uint32_t)e[5] << 16), (uint32_t)e[6] | ((uint32_t)e[7] << 16));
        }
    } else {
#pragma unroll
        for (int j = 0; j < 8; ++j)
            if (t + j < V) orow[t + j] = e[j];
    }
}

// Exact scan of groups [g_lo, g_hi) of one row by the whole workgroup: this thread's best
// candidate (key << 32 | ~token), 0 if it saw nothing allowed.  Writes the masked row if orow.
// (bits_at(g): the allowed bits of group g.)
template <int DTYPE, class BitsAt>
__device__ __forceinline__ unsigned long long exact_scan_with(const typename ElemOf<DTYPE>::type* row,
                                                              typename ElemOf<DTYPE>::type* orow, BitsAt bits_at,
                                                              bool valid, int V, int g_lo, int g_hi)
{
    using Elem = typename ElemOf<DTYPE>::type;
    constexpr Elem NEG_INF = DTYPE == TDFA_F32 ? (Elem)0xFF800000u : (Elem)0xFF80u;
    uint32_t best_key = 0, best_idx = 0;
    for (int g = g_lo + (int)threadIdx.x; g < g_hi; g += (int)blockDim.x) {
        const int t = g << 3;
        const uint32_t m = valid ? bits_at(g) : 0u;
        Elem e[8];
        load_group<DTYPE>(row, t, V, e);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const bool ok = (m >> j) & 1u;
            const uint32_t key = DTYPE == TDFA_F32 ? key_f32((uint32_t)e[j]) : key_bf16((uint32_t)e[j]);
            if (ok && key > best_key) { best_key = key; best_idx = (uint32_t)(t + j); }
            if (!ok) e[j] = NEG_INF;
        }
        if (orow) store_group<DTYPE>(orow, t, V, e);
    }
    return best_key ? ((unsigned long long)best_key << 32) | (0xFFFFFFFFu - best_idx) : 0ull;
}

template <int DTYPE>
__device__ __forceinline__ unsigned long long exact_scan(const typename ElemOf<DTYPE>::type* row,
                                                         typename ElemOf<DTYPE>::type* orow, const uint8_t* bits,
                                                         bool valid, int V, int g_lo, int g_hi)
{
    return exact_scan_with<DTYPE>(row, orow, [bits](int g) { return (uint32_t)bits[g]; }, valid, V, g_lo, g_hi);
}

// Thread 0 of each of the `parts` workgroups of row b brings its candidate; returns true in the
// workgroup that arrives last, with the row's maximum in `cand`.  Both scratch words are zero
// again when it returns true.  All traffic on the two words is device-scope atomics, which
// execute at one place in arrival order; the counter update carries a dependency on the value
// the max returned, so it cannot be issued before the max has been performed.
__device__ __forceinline__ bool combine_parts(const MaskArgs& a, int b, int parts, unsigned long long& cand)
{
    if (parts == 1) return true;
    unsigned int inc = 1u;
    if (cand) {
        const unsigned long long old = __hip_atomic_fetch_max(&a.scratch_best[b], cand, __ATOMIC_RELAXED,
                                                              __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("" : "+v"(inc) : "v"((uint32_t)old), "v"((uint32_t)(old >> 32)));
    }
    const unsigned done = __hip_atomic_fetch_add(&a.scratch_count[b], inc, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (done != (unsigned)parts - 1) return false;
    cand = __hip_atomic_exchange(&a.scratch_best[b], 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(&a.scratch_count[b], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return true;
}

// delta_T[q][token] for a row q and a token id; DEAD if the token has no edge.  A packed table
// keeps only the targets of the edges, in token order: the position of the edge is the number of
// allowed bits of the row below the token (a per-128-token directory plus the bits of one block).
struct PackedBlock {          // what a lookup in a packed row needs, for one block of 128 tokens
    uint32_t w[4];            // the allowed bits of the block
    uint32_t base;            // edges of the row below the block
    int64_t begin;            // first edge of the row
};

__device__ __forceinline__ PackedBlock packed_block(const MaskArgs& a, int q, int blk)
{
    PackedBlock pb;
    const uint32_t* words = a.allow + (int64_t)q * a.row_words + 4 * blk;
    pb.w[0] = words[0]; pb.w[1] = words[1]; pb.w[2] = words[2]; pb.w[3] = words[3];
    pb.base = a.dir[(int64_t)q * (a.row_words >> 2) + blk];
    pb.begin = a.row_begin[q];
    return pb;
}

__device__ __forceinline__ int32_t packed_entry(const MaskArgs& a, const PackedBlock& pb, int token)
{
    const int wi = (token >> 5) & 3, bit = token & 31;
    const uint32_t w = wi == 0 ? pb.w[0] : (wi == 1 ? pb.w[1] : (wi == 2 ? pb.w[2] : pb.w[3]));
    if (!((w >> bit) & 1u)) return TDFA_DEAD;
    const uint32_t below = (wi > 0 ? __popc(pb.w[0]) : 0) + (wi > 1 ? __popc(pb.w[1]) : 0) + (wi > 2 ? __popc(pb.w[2]) : 0) +
                           __popc(w & ((1u << bit) - 1u));
    return a.targets[pb.begin + pb.base + below];
}

__device__ __forceinline__ int32_t table_entry(const MaskArgs& a, int q, int token)
{
    if (a.delta) return a.delta[(int64_t)q * a.n_tokens + token];
    if (!a.targets) return q;                                  // no table: the caller traverses the edge
    return packed_entry(a, packed_block(a, q, token >> 7), token);
}

// How many tokens row q of the table allows: a count the library keeps beside a table it has written, or the
// edges of a packed row; kUnknown where neither is there.
constexpr uint32_t kUnknown = 0xFFFFFFFFu;
__device__ __forceinline__ uint32_t allowed_count(const MaskArgs& a, int q)
{
    if (a.row_allowed) return a.row_allowed[q];
    if (a.row_begin) return (uint32_t)(a.row_begin[q + 1] - a.row_begin[q]);
    return kUnknown;
}

__device__ __forceinline__ void write_result(const MaskArgs& a, int b, int q, bool valid, unsigned long long cand)
{
    int32_t token = TDFA_NO_TOKEN, next = valid ? q : TDFA_DEAD;
    if (cand) {
        token = (int32_t)(0xFFFFFFFFu - (uint32_t)cand);
        next = table_entry(a, q, token);
    }
    a.tokens[b] = token;
    a.new_states[b] = next;
}

// Exact kernel: fp32 rows that the kernels below do not take, 16-bit rows beyond 32-bit offsets.
template <int DTYPE>
__global__ void __launch_bounds__(kMaxThreads)
mask_step_exact_kernel(MaskArgs a, int parts, int groups_per_part)
{
    using Elem = typename ElemOf<DTYPE>::type;
    __shared__ unsigned long long wave_best[kMaxWaves];
    const int b = blockIdx.x / parts, p = blockIdx.x % parts;
    const int V = a.n_tokens;
    const int q = a.states[b];
    const bool valid = q >= 0 && (int64_t)q < a.n_rows;
    const uint8_t* bits = reinterpret_cast<const uint8_t*>(a.allow + (valid ? (int64_t)q * a.row_words : 0));
    const Elem* row = static_cast<const Elem*>(a.logits) + (int64_t)b * a.row_stride;
    Elem* orow = a.masked_out ? static_cast<Elem*>(a.masked_out) + (int64_t)b * a.row_stride : nullptr;
    const int n_groups = (V + 7) >> 3;
    const int g_lo = p * groups_per_part;
    const int g_hi = min(n_groups, g_lo + groups_per_part);
    unsigned long long cand = exact_scan<DTYPE>(row, orow, bits, valid, V, g_lo, g_hi);
    cand = block_max_u64(cand, wave_best);
    if (threadIdx.x != 0) return;
    if (combine_parts(a, b, parts, cand)) write_result(a, b, q, valid, cand);
}

// 16-bit unsigned order keys of two bf16 values: x ^ 0x8000 for non-negative x, ~x for negative.
__device__ __forceinline__ uint32_t keys2(uint32_t d)
{
    const s16x2 s = __builtin_bit_cast(s16x2, d) >> (s16x2){15, 15};
    return d ^ (__builtin_bit_cast(uint32_t, s) | 0x80008000u);
}

// Buffer descriptors for raw byte-offset access (no structure, 32-bit data format) and the cache
// policy of data that is read once and never again (non-temporal).
constexpr int kRawBuffer = 0x00020000;
constexpr int kReadOnce = 2;
constexpr int kMaxBitRowBytes = 128 * 1024;    // the most allowed bits (a byte per eight tokens) a workgroup keeps in LDS:
                                               // vocabularies of up to about a million tokens
constexpr int kPlainLdsBytes = 40 * 1024;      // what a launch may ask for without the kernel's limit being raised first

// fp32 logits with the penalised row written: every logit is read and written once.  A lane takes four logits at a
// time, so that a wavefront's accesses are whole kilobytes, and has kExactAhead such loads in flight before it compares
// and writes the first; the loads and stores go through buffer descriptors that end with the row's whole groups, so that
// none sits under a branch.
//
// Bound by the memory: 64 rows of 128,256 tokens, 65.7 MB, 16.3 us with one group of eight in flight per lane (two loads
// that skip over each other's halves), 15.0 us so (a plain copy of as much: 13.3 us); 256 rows 50.4 -> 47.4 us, 1,024
// rows 226 -> 208 us.  Non-temporal accesses: 14.4, 52.7 and 202 us.
constexpr int kExactAhead = 4;

__global__ void __launch_bounds__(kMaxThreads)
mask_write_f32_kernel(MaskArgs a, int parts, int groups_per_part)
{
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    constexpr uint32_t NEG_INF = 0xFF800000u;
    __shared__ unsigned long long wave_best[kMaxWaves];
    const int b = blockIdx.x / parts, p = blockIdx.x % parts;
    const int V = a.n_tokens;
    const int q = a.states[b];
    const bool valid = q >= 0 && (int64_t)q < a.n_rows;
    const uint8_t* bits = reinterpret_cast<const uint8_t*>(a.allow + (valid ? (int64_t)q * a.row_words : 0));
    const uint32_t* row = static_cast<const uint32_t*>(a.logits) + (int64_t)b * a.row_stride;
    uint32_t* orow = static_cast<uint32_t*>(a.masked_out) + (int64_t)b * a.row_stride;
    const int n_groups = (V + 7) >> 3, n_full = V >> 3;
    const int g_lo = p * groups_per_part;
    const int g_hi = min(n_full, g_lo + groups_per_part);
    const int T = (int)blockDim.x, tid = (int)threadIdx.x;
    uint32_t best_key = 0, best_idx = 0;
    auto take = [&](uint32_t x, uint32_t tok, bool ok) {       // (a thread meets its tokens in ascending order)
        const uint32_t key = ok ? key_f32(x) : 0u;
        if (key > best_key) { best_key = key; best_idx = tok; }
    };
    const int q_hi = 2 * g_hi;                                 // in quads: four logits, 16 bytes
    for (int q0 = 2 * g_lo; q0 < q_hi; q0 += kExactAhead * T) {             // (uniform)
        u32x4 x[kExactAhead];
        uint32_t m[kExactAhead];
#pragma unroll
        for (int u = 0; u < kExactAhead; ++u) {
            const int qs = q0 + u * T, n = min(max(q_hi - qs, 0), T);
            const __amdgpu_buffer_rsrc_t r_x = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t*>(row) + (int64_t)qs * 4, 0, n * 16, kRawBuffer);
            const __amdgpu_buffer_rsrc_t r_m = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(bits) + (qs >> 1), 0, valid ? n >> 1 : 0, kRawBuffer);
            x[u] = __builtin_amdgcn_raw_buffer_load_b128(r_x, tid * 16, 0, 0);
            m[u] = __builtin_amdgcn_raw_buffer_load_b8(r_m, tid >> 1, 0, 0);
        }
#pragma unroll
        for (int u = 0; u < kExactAhead; ++u) {
            const int qs = q0 + u * T, n = min(max(q_hi - qs, 0), T);
            const __amdgpu_buffer_rsrc_t r_o = __builtin_amdgcn_make_buffer_rsrc(orow + (int64_t)qs * 4, 0, n * 16, kRawBuffer);
            const uint32_t e[4] = {x[u].x, x[u].y, x[u].z, x[u].w}, mq = m[u] >> (4 * (tid & 1));
            uint32_t o[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const bool ok = (mq >> j) & 1u;
                take(e[j], (uint32_t)((qs + tid) * 4 + j), ok);
                o[j] = ok ? e[j] : NEG_INF;
            }
            __builtin_amdgcn_raw_buffer_store_b128(u32x4{o[0], o[1], o[2], o[3]}, r_o, tid * 16, 0, 0);
        }
    }
    if (n_groups > n_full && p == parts - 1 && tid < V - 8 * n_full) {      // the row's partial group, a token per thread
        const int t = 8 * n_full + tid;
        const bool ok = valid && ((bits[n_full] >> tid) & 1u);
        const uint32_t x = row[t];
        take(x, (uint32_t)t, ok);
        orow[t] = ok ? x : NEG_INF;
    }
    unsigned long long cand = best_key ? ((unsigned long long)best_key << 32) | (0xFFFFFFFFu - best_idx) : 0ull;
    cand = block_max_u64(cand, wave_best);
    if (tid != 0) return;
    if (combine_parts(a, b, parts, cand)) write_result(a, b, q, valid, cand);
}

constexpr uint32_t KU_POS_INF = 0xFF80u;   // key of +inf: anything above is a NaN pattern
constexpr uint32_t KU_NEG_INF = 0x007Fu;   // key of -inf: anything below is a negative-sign NaN
constexpr uint32_t KU_POS_ZERO = 0x8000u, KU_NEG_ZERO = 0x7FFFu;

// Sum of a 32-bit value over the 64 lanes of a wavefront (all lanes active); the result is uniform.
__device__ __forceinline__ uint32_t wave_sum_u32(uint32_t v)
{
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, true);     // quad_perm [1,0,3,2]
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, true);     // quad_perm [2,3,0,1]
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xF, 0xF, true);    // row_half_mirror
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x140, 0xF, 0xF, true);    // row_mirror
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 0) + (uint32_t)__builtin_amdgcn_readlane((int)v, 16) +
           (uint32_t)__builtin_amdgcn_readlane((int)v, 32) + (uint32_t)__builtin_amdgcn_readlane((int)v, 48);
}

// Sums over the lanes up to and including this one (all lanes active).
__device__ __forceinline__ uint32_t wave_prefix_u32(uint32_t v)
{
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xF, 0xF, false);   // row_shr:1
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xF, 0xF, false);   // row_shr:2
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xF, 0xF, false);   // row_shr:4
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xF, 0xF, false);   // row_shr:8
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xA, 0xF, false);   // row_bcast:15, rows 1 and 3
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xC, 0xF, false);   // row_bcast:31, rows 2 and 3
    return v;
}

// Number of lanes below this one for which `flag` holds (all lanes active).
__device__ __forceinline__ uint32_t lanes_below(bool flag)
{
    const unsigned long long mask = __builtin_amdgcn_ballot_w64(flag);
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// Number of non-zero bytes of a word.
__device__ __forceinline__ uint32_t nonzero_bytes(uint32_t w)
{
    return (uint32_t)__builtin_popcount((((w & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | w) & 0x80808080u);
}

constexpr int kListCap = 256;          // groups a wavefront may fetch one by one instead of reading its stretch
constexpr int kEarlyWaves = 8;         // wavefronts of a workgroup that request their first group of logits before the state is known

// A state known to allow less than this part of the vocabulary (one in ...) is gathered by the workgroup instead of
// each wavefront finding out about its own stretch.  1,024 rows of 128,256 tokens whose states allow few tokens:
// 19.7 -> 16.4 us (50 signatures), 17.8 -> 14.0 us (16 schemas); states anywhere in the texts of 16 schemas 30.0 -> 28.8
// us (with two workgroups per compute unit, below: 12.9, 10.6 and 24.7 us).  With 8 instead of 32 the states that allow 4 to 12 % are gathered too, and streaming them is faster (the
// same signatures 36 -> 51 us); 64 is as good as 32.
constexpr uint32_t kSparseShare = 32;
// Gathering pays where rows share a compute unit, and so does the form of the step kernel that does it, two of whose
// workgroups a compute unit holds (below): rows of a dense table take it from one and a half per compute unit on.  States
// anywhere in the texts, rows of states that allow few tokens, and rows of states that allow most of 128,256 tokens,
// without -> with: 300 rows 17.0 -> 15.8, 9.4 -> 8.7 and 19.1 -> 18.0 us for 50 signatures, but 13.3 -> 14.6 us for the texts
// of 16 schemas; 257 rows 12.1 -> 14.2 us for those of the signatures; 380 rows 17.5 -> 16.2, 9.8 -> 8.7 and 19.7 -> 18.5 us,
// 16.6 -> 15.1 us for the schemas; 511 rows 18.6 -> 17.2, 10.8 -> 8.7 and 23.3 -> 21.6 us.  Packed tables take it at any size.
constexpr int kGatherRows = 384;

constexpr int kGatherQueue = 128;      // groups a wavefront's ring holds (a power of two; 64 are fetched at a time)

// Greedy choice over groups [g_lo, g_hi) of a row that allows few tokens, by the whole workgroup: this thread's
// best candidate.  A thread reads the allowed bits of four groups per load, four loads in flight; a wavefront
// whose 256 groups allow nothing is done with them after one ballot, and the groups that hold an allowed token
// wait in its ring in LDS (`ring`, kGatherQueue entries of (group, bits)) until 64 of them are fetched at once,
// one per lane, a batch ahead of the one that is compared.  Bound by instructions where several such rows share a
// compute unit and by latency where they do not; logits of groups without an allowed token are never read.
template <int DTYPE>
__device__ __forceinline__ unsigned long long gather_scan(const typename ElemOf<DTYPE>::type* row, const uint8_t* bits, int V,
                                                          int g_lo, int g_hi, uint2* ring)
{
    using Elem = typename ElemOf<DTYPE>::type;
    const uint32_t lane = threadIdx.x & 63u;
    auto wave_sync = []() {                                    // LDS written by some lanes, read by others
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    uint32_t best_key = 0, best_idx = 0xFFFFFFFFu;             // key 0: no candidate yet
    uint32_t head = 0, tail = 0;                               // ring positions, the same in all lanes
    uint32_t m = 0;                                            // allowed bits of this lane's group; 0: none
    int t = 0;                                                 // its first token
    Elem e[8] = {};
    auto compare = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const uint32_t x = (uint32_t)e[j], key = key_f32(DTYPE == TDFA_F32 ? x : x << 16), tok = (uint32_t)(t + j);
            if (((m >> j) & 1u) && (key > best_key || (key == best_key && tok < best_idx))) {
                best_key = key;
                best_idx = tok;
            }
        }
    };
    auto fetch = [&](uint32_t n) __attribute__((always_inline)) {        // n <= 64 waiting groups: request them, compare the batch before
        wave_sync();
        uint32_t m_next = 0;
        int t_next = 0;
        Elem e_next[8] = {};
        if (lane < n) {
            const uint2 en = ring[(head + lane) & (kGatherQueue - 1)];
            t_next = (int)en.x << 3;
            m_next = en.y;
            load_group<DTYPE>(row, t_next, V, e_next);
        }
        head += n;
        wave_sync();
        compare();
        m = m_next;
        t = t_next;
#pragma unroll
        for (int j = 0; j < 8; ++j) e[j] = e_next[j];
    };
    const uint32_t* words = reinterpret_cast<const uint32_t*>(bits);
    const int w_lo = g_lo >> 2, w_hi = (g_hi + 3) >> 2;                    // (g_lo is a multiple of four groups)
    const int NT = (int)blockDim.x;
    auto load_word = [&](int wi) { return wi < w_hi ? words[wi] : 0u; };
    int wi = w_lo + (int)threadIdx.x;
    uint32_t w0 = load_word(wi), w1 = load_word(wi + NT), w2 = load_word(wi + 2 * NT), w3 = load_word(wi + 3 * NT);
    for (int base = w_lo; base < w_hi; base += NT, wi += NT) {               // trip count uniform in the workgroup
        const uint32_t w = w0;
        w0 = w1;
        w1 = w2;
        w2 = w3;
        w3 = load_word(wi + 4 * NT);
        const int left = g_hi - (wi << 2);                                   // groups of this word inside the part
        const uint32_t wm = left >= 4 ? w : (left > 0 ? w & ((1u << (8 * left)) - 1u) : 0u);
        if (__builtin_amdgcn_ballot_w64(wm != 0) == 0) continue;
        // 64 consecutive groups at a time (lane L takes byte L mod 4 of the word of lane 16 i + L / 4), so that
        // neighbouring lanes fetch neighbouring logits
#pragma unroll 1
        for (int i = 0; i < 4; ++i) {
            const int src = 16 * i + (int)(lane >> 2);
            const uint32_t ws = (uint32_t)__shfl((int)wm, src, 64);
            const uint32_t mg = (ws >> (8 * (lane & 3u))) & 0xFFu;
            const unsigned long long bal = __builtin_amdgcn_ballot_w64(mg != 0);
            if (bal == 0) continue;
            const uint32_t at = tail + __builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0u));
            const int g = ((wi - (int)lane + src) << 2) + (int)(lane & 3u);
            if (mg != 0) ring[at & (kGatherQueue - 1)] = make_uint2((uint32_t)g, mg);
            tail += (uint32_t)__popcll(bal);
            if (tail - head >= 64u) fetch(64u);
        }
    }
    if (tail != head) fetch(tail - head);
    compare();
    return best_key ? ((unsigned long long)best_key << 32) | (0xFFFFFFFFu - best_idx) : 0ull;
}

// One step on 16-bit logits.  The groups [g_lo, g_hi) of a workgroup are cut into one stretch of
// `stretch` groups (a multiple of 16) per wavefront, read 64 consecutive groups per load.
//
// SKIP: a wavefront first reads the allowed bits of its whole stretch, 16 bytes (16 groups) per
// lane and pass, into its part of `s_pieces`.  If at most one group in 16 (and at most kListCap)
// holds an allowed token, only those groups' logits are fetched: a decode spends most steps in
// states that allow a few hundred of 10^5 tokens, and the logits of a group without an allowed
// token cannot matter.  Otherwise, and always when the masked row is written, the stretch is
// streamed.  The choice is a wavefront's own; the result does not depend on it.
//
// PDA: the step of a push-down constraint.  The allowed bits of a sequence are not one row but
// the OR of the rows of its state's classes of edges whose pops its stack ends with; the wavefront
// finds those classes (one per lane) before it reads its stretch of bits, and ORs the rows as it
// reads them.  At the end the wavefront that finishes the row traverses the chosen token's edge, which also moves
// the stack (every workgroup of the row has read it by then).
template <bool WRITE, int kUnroll, bool SKIP, int kBuf, bool PDA, bool GATHER>
__device__ __forceinline__ void mask_step_bf16(const std::conditional_t<PDA, PdaMaskArgs, MaskArgs>& a, int parts, int groups_per_part,
                                               int stretch)
{
    static_assert(!PDA || (SKIP && !WRITE), "the push-down step reads its bits into LDS");
    static_assert(!GATHER || (SKIP && !PDA), "the rings of a gathered row lie in the lists' room");
    extern __shared__ uint4 s_pieces[];
    __shared__ __attribute__((aligned(8))) uint32_t s_list[SKIP ? kMaxWaves * kListCap : 1];
    static_assert(kListCap >= 2 * kGatherQueue, "the rings of a sparse row share the lists' room");
    __shared__ unsigned long long wave_best[kMaxWaves], wave_best_exact[kMaxWaves];
    __shared__ int s_exact;
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    const int b = blockIdx.x / parts, p = blockIdx.x % parts;
    const int V = a.n_tokens;
    const uint16_t* row = static_cast<const uint16_t*>(a.logits) + (int64_t)b * a.row_stride;
    uint16_t* orow = WRITE ? static_cast<uint16_t*>(a.masked_out) + (int64_t)b * a.row_stride : nullptr;

    const int n_groups = (V + 7) >> 3;
    const int n_full = V >> 3;                                 // groups with all eight tokens inside the row
    const int g_lo = p * groups_per_part;
    const int g_hi = min(n_groups, g_lo + groups_per_part);
    const int g_hi_full = min(g_hi, n_full);
    const int lane = (int)threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);    // the same in every lane: kept in a scalar register
    const int w_lo = min(g_lo + wave * stretch, g_hi_full);    // this wavefront's full groups
    const int w_hi = min(w_lo + stretch, g_hi_full);

    // kBuf register buffers of kUnroll groups each: the loads of the next batches are in flight while
    // one is folded.  Logits and allowed bits are read through buffer descriptors that end
    // with the stretch: a group past the end reads as zeros without touching memory, so no load
    // sits under a branch and every lane runs the same number of passes.  Logits are requested
    // before the state is read, since they do not depend on it: every buffer where the wavefront
    // will stream for certain, one group per lane (1 KB per wavefront) where it may turn out to
    // fetch single groups instead, the rest then follows when it knows.  There the allowed bytes
    // of the stretch are in LDS by then, and the stream reads them from there.
    const __amdgpu_buffer_rsrc_t r_logits =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(row), 0, w_hi * 16, kRawBuffer);
    const __amdgpu_buffer_rsrc_t r_out =
        __builtin_amdgcn_make_buffer_rsrc(orow, 0, WRITE ? w_hi * 16 : 0, kRawBuffer);
    auto load_x = [&](int gb, uint4 (&x)[kUnroll]) {
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(r_logits, (gb + u * 64) * 16, 0, kReadOnce);
            x[u] = make_uint4(v.x, v.y, v.z, v.w);
        }
    };
    constexpr int step = 64 * kUnroll;
    int g0 = w_lo + lane;
    uint4 xr[kBuf][kUnroll];
    uint32_t mr[kBuf][kUnroll];
    constexpr bool kMaySkip = SKIP && !WRITE;
    auto load_x1 = [&](int g, uint4& x) {
        const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(r_logits, g * 16, 0, kReadOnce);
        x = make_uint4(v.x, v.y, v.z, v.w);
    };
    if constexpr (!kMaySkip) {
#pragma unroll
        for (int r = 0; r < kBuf; ++r) load_x(g0 + r * step, xr[r]);
    } else {
        // (the first kEarlyWaves wavefronts of a workgroup only: the early request costs the rows that turn out to
        // allow little or nothing, and half of it serves the rows that stream as well as all of it)
        if (wave < kEarlyWaves) load_x1(g0, xr[0][0]);         // (the rest once the wavefront knows that it streams)
    }
    const int q = a.states[b];
    bool valid = q >= 0 && (int64_t)q < a.n_rows;
    bool surely_wide = false;                         // the state allows so many tokens that the row is streamed whatever the bits say
    if constexpr (!WRITE && !PDA) {
        // (packed tables do not come to the form with SKIP alone, which need not ask for the edges of a packed row)
        uint32_t n_allowed = kUnknown;
        if constexpr (GATHER || !SKIP) {
            if (valid) n_allowed = allowed_count(a, q);
        } else if (a.row_allowed != nullptr && valid) {
            n_allowed = a.row_allowed[q];
        }
        if (n_allowed != kUnknown) {
            // A state that allows no token (a sequence whose text is complete): no token, the state stays.
            if (n_allowed == 0u) {
                if (threadIdx.x == 0) {
                    unsigned long long none = 0ull;
                    if (combine_parts(a, b, parts, none)) write_result(a, b, q, valid, none);
                }
                return;
            }
            if constexpr (GATHER) {
                // A state known to allow few tokens.
                if (n_allowed < (uint32_t)V / kSparseShare) {
                    unsigned long long c = gather_scan<TDFA_BF16>(row, reinterpret_cast<const uint8_t*>(a.allow + (int64_t)q * a.row_words),
                                                                  V, g_lo, g_hi, reinterpret_cast<uint2*>(s_list) + wave * kGatherQueue);
                    c = block_max_u64(c, wave_best);
                    if (threadIdx.x == 0 && combine_parts(a, b, parts, c)) write_result(a, b, q, valid, c);
                    return;
                }
            }
            surely_wide = n_allowed >= (uint32_t)V / 4u;
        }
    }
    unsigned long long classes = 0;                   // PDA: the classes of q (bit j: row class_row0 + j) the stack matches
    int32_t class_row0 = 0;
    int32_t depth = 0;                                // PDA: of the sequence's stack
    if constexpr (PDA) {
        depth = a.pda.depths[b];
        valid = q >= 0 && q < a.pda.n_states && depth >= 0 && depth <= a.pda.stack_cap;
        class_row0 = valid ? a.pda.class_first[q] : 0;
        const int n_classes = valid ? a.pda.class_first[q + 1] - class_row0 : 0;
        // the top symbols of the stack and a class's pops are read whole (top first), so that no read
        // waits for the outcome of a comparison
        const int32_t* stack = a.pda.stacks + (int64_t)b * a.pda.stack_cap;
        int32_t top[kPdaPops];
#pragma unroll
        for (int j = 0; j < kPdaPops; ++j) top[j] = valid && depth - 1 - j >= 0 ? stack[depth - 1 - j] : -1;
        bool ok = false;
        if (lane < n_classes) {
            const int np = a.pda.class_n_pops[class_row0 + lane];
            const int4* pp = reinterpret_cast<const int4*>(a.pda.class_pops + (int64_t)(class_row0 + lane) * kPdaPops);
            const int4 p0 = pp[0], p1 = pp[1], p2 = pp[2];
            const int32_t pops[kPdaPops] = {p0.x, p0.y, p0.z, p0.w, p1.x, p1.y, p1.z, p1.w, p2.x, p2.y, p2.z, p2.w};
            ok = np <= depth;
#pragma unroll
            for (int j = 0; j < kPdaPops; ++j)
                if (j < np) ok = ok && pops[j] == top[j];
        }
        classes = __builtin_amdgcn_ballot_w64(ok);
    }
    const uint8_t* bits = reinterpret_cast<const uint8_t*>(a.allow + (valid && !PDA ? (int64_t)q * a.row_words : 0));
    // the allowed bits of group g, from memory: (PDA: of every matching class)
    auto bits_at = [&](int g) -> uint32_t {
        if constexpr (PDA) {
            uint32_t m = 0;
            for (unsigned long long c = classes; c; c &= c - 1)
                m |= reinterpret_cast<const uint8_t*>(a.allow + (int64_t)(class_row0 + __builtin_ctzll(c)) * a.row_words)[g];
            return m;
        } else {
            return bits[g];
        }
    };
    const __amdgpu_buffer_rsrc_t r_bits =          // one byte per full group; empty for a state outside the table
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(bits), 0, valid ? w_hi : 0, kRawBuffer);
    const uint8_t* my_bits = nullptr;                 // kMaySkip: the stretch's allowed bytes in LDS (set below)
    auto load_m = [&](int gb, uint32_t (&m)[kUnroll]) {
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            if constexpr (kMaySkip) m[u] = my_bits[gb + u * 64 - w_lo];
            else m[u] = __builtin_amdgcn_raw_buffer_load_b8(r_bits, gb + u * 64, 0, 0);
        }
    };
    if constexpr (!kMaySkip) {
#pragma unroll
        for (int r = 0; r < kBuf; ++r) load_m(g0 + r * step, mr[r]);
    }

    // A lane remembers its best key and the group of eight in which its maximum rose to it (the
    // lowest such group; the maximum rises a few times per row at most), with the group's logits
    // and allowed bits, so that the token inside the group is found from registers when needed.
    // (No key may rise above 0, that of the NaN pattern 0xFFFF: the group is then the stretch's first, so that the
    // wavefronts' candidates differ all the same.)
    uint32_t best = 0, best_g = (uint32_t)w_lo, best_m = 0, any = 0;
    uint4 best_x = make_uint4(0, 0, 0, 0);
    // `ANY_ORDER`: groups may come in any order, so an equal key from a lower group takes over.
    auto fold_one = [&](auto any_order, int g, const uint4& x, uint32_t m) {
        const uint32_t d[4] = {x.x, x.y, x.z, x.w};
        const uint32_t y = m | (m << 15);                      // allowed bit 2j at bit 2j, bit 2j+1 at bit 16+2j
        u16x2 acc = {0, 0};
        uint32_t o[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint32_t pj = (y >> (2 * j)) & 0x00010001u;
            const u16x2 km = __builtin_bit_cast(u16x2, keys2(d[j])) * __builtin_bit_cast(u16x2, pj);
            acc = __builtin_elementwise_max(acc, km);
            if constexpr (WRITE) {
                const uint32_t md = __builtin_bit_cast(uint32_t, __builtin_bit_cast(u16x2, pj) * (u16x2){0xFFFF, 0xFFFF});
                o[j] = (d[j] & md) | (0xFF80FF80u & ~md);
            }
        }
        if constexpr (WRITE) {
            // written once, not read again by this step: a streaming store (dropped past the end of the stretch)
            const u32x4 pack = {o[0], o[1], o[2], o[3]};
            __builtin_amdgcn_raw_buffer_store_b128(pack, r_out, g * 16, 0, kReadOnce);
        }
        const uint32_t a2 = __builtin_bit_cast(uint32_t, acc);
        const uint32_t top = max(a2 & 0xFFFFu, a2 >> 16);
        any |= m;
        if (top > best || (decltype(any_order)::value && top == best && (uint32_t)g < best_g)) {
            best = top;
            best_g = (uint32_t)g;
            best_m = m;
            best_x = x;
        }
    };
    auto fold = [&](int gb, const uint4 (&x)[kUnroll], const uint32_t (&m)[kUnroll]) {
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) fold_one(std::false_type{}, gb + u * 64, x[u], m[u]);
    };
    // The lane's candidate, exactly: (has an allowed token, key, lowest token id first).
    auto candidate = [&]() -> unsigned long long {
        const uint32_t d[4] = {best_x.x, best_x.y, best_x.z, best_x.w};
        int j = 7;
#pragma unroll
        for (int pr = 3; pr >= 0; --pr) {
            const uint32_t k2 = keys2(d[pr]);
            if ((best_m >> (2 * pr + 1) & 1u) && (k2 >> 16) == best) j = 2 * pr + 1;
            if ((best_m >> (2 * pr) & 1u) && (k2 & 0xFFFFu) == best) j = 2 * pr;
        }
        const uint32_t tok = best_g * 8 + (uint32_t)j;
        return any ? (1ull << 63) | ((unsigned long long)best << 32) | (0xFFFFFFFFu - tok) : 0ull;
    };

    // Which way this wavefront goes: count the groups of the stretch that hold an allowed token.
    bool skip = false;
    uint32_t n_listed = 0;
    constexpr int kPad16 = 4 * step / 16;                          // zero bytes behind a stretch: the four batches read past its end
    uint4* my_pieces = s_pieces + wave * ((stretch >> 4) + kPad16);
    const int n_pieces = (w_hi - w_lo + 15) >> 4;              // (w_lo is a multiple of 16 unless the stretch is empty)
    my_bits = reinterpret_cast<const uint8_t*>(my_pieces);
    if constexpr (SKIP && !WRITE) {
        const __amdgpu_buffer_rsrc_t r_row =       // the whole bit row, a multiple of 16 bytes
            __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(bits), 0, valid ? a.row_words * 4 : 0, kRawBuffer);
        uint32_t nz = 0;
        // A state known to allow a quarter of the vocabulary or more is streamed: the rest of the buffers is
        // requested right behind the first bits, without waiting for them to be counted.
        u32x4 v_first = {0, 0, 0, 0};
        if constexpr (!PDA) {
            v_first = __builtin_amdgcn_raw_buffer_load_b128(r_row, w_lo + lane * 16, 0, 0);
            if (surely_wide) {
                if (wave >= kEarlyWaves) load_x1(g0, xr[0][0]);
#pragma unroll
                for (int u = 1; u < kUnroll; ++u) load_x1(g0 + u * 64, xr[0][u]);
#pragma unroll
                for (int r = 1; r < kBuf; ++r) load_x(g0 + r * step, xr[r]);
            }
        }
        for (int i = lane; i < n_pieces; i += 64) {
            u32x4 v = {0, 0, 0, 0};
            if constexpr (PDA) {
                for (unsigned long long c = classes; c; c &= c - 1) {       // (the same classes in every lane)
                    const uint32_t* class_row = a.allow + (int64_t)(class_row0 + __builtin_ctzll(c)) * a.row_words;
                    v |= __builtin_amdgcn_raw_buffer_load_b128(
                        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t*>(class_row), 0, a.row_words * 4, kRawBuffer),
                        w_lo + i * 16, 0, 0);
                }
            } else {
                v = i == lane ? v_first : __builtin_amdgcn_raw_buffer_load_b128(r_row, w_lo + i * 16, 0, 0);
            }
            uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                const int left = w_hi - (w_lo + i * 16 + d * 4);       // bytes of this word inside the stretch
                if (left <= 0) w[d] = 0;
                else if (left < 4) w[d] &= (1u << (8 * left)) - 1u;
                nz += nonzero_bytes(w[d]);
            }
            my_pieces[i] = make_uint4(w[0], w[1], w[2], w[3]);
        }
        for (int i = n_pieces + lane; i < (stretch >> 4) + kPad16; i += 64) my_pieces[i] = make_uint4(0, 0, 0, 0);
        n_listed = wave_sum_u32(nz);
        skip = !surely_wide && n_listed <= (uint32_t)kListCap && n_listed * 16u <= (uint32_t)(w_hi - w_lo);
        if (skip) {
            // Every lane lists the groups of its pieces: (group within the stretch) << 8 | bits.
            uint32_t slot = 0;
#pragma unroll
            for (int bit = 0; bit < 9; ++bit) slot += lanes_below((nz >> bit) & 1u) << bit;   // lanes' counts below this one's
            uint32_t* list = s_list + wave * kListCap;
            for (int i = lane; i < n_pieces; i += 64) {
                const uint4 pc = my_pieces[i];
                const uint32_t w[4] = {pc.x, pc.y, pc.z, pc.w};
#pragma unroll
                for (int d = 0; d < 4; ++d) {
                    uint32_t rest = w[d];
                    while (rest) {
                        const int byte = (__builtin_ctz(rest)) >> 3;
                        list[slot++] = (uint32_t)((i * 16 + d * 4 + byte) << 8) | ((rest >> (8 * byte)) & 0xFFu);
                        rest &= ~(0xFFu << (8 * byte));
                    }
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            // One listed group per lane, four loads in flight; a lane without one reads past the end.
            for (uint32_t r0 = 0; r0 < n_listed; r0 += 256) {
                uint4 x[4];
                uint32_t m[4];
                int g[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const uint32_t idx = r0 + (uint32_t)(u * 64 + lane);
                    const uint32_t e = idx < n_listed ? list[idx] : 0u;
                    g[u] = w_lo + (int)(e >> 8);
                    m[u] = e & 0xFFu;
                    const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(r_logits, idx < n_listed ? g[u] * 16 : 0x7FFFFFF0, 0, kReadOnce);
                    x[u] = make_uint4(v.x, v.y, v.z, v.w);
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) fold_one(std::true_type{}, g[u], x[u], m[u]);
            }
        }
    }

    // The traversal of the chosen edge (Algorithm 2, last statement) is one dependent read of the
    // table at the very end of the step.  It is taken off the critical path: after about three
    // quarters of a stretch, the wavefront requests the table entry of its best token so far; the
    // token that wins in the end has most often been seen by then, and its entry has long arrived
    // when the workgroup's maximum is known.
    const bool ahead = parts == 1 && a.delta != nullptr && a.n_rows > 0;       // (packed tables and split rows look the entry up at the end)
    uint32_t tok_ahead = 0xFFFFFFFFu;                                          // an id no token has
    int32_t val_ahead = TDFA_DEAD;
    if (!skip) {
        if constexpr (kMaySkip) {
            if (!surely_wide) {
                if (wave >= kEarlyWaves) load_x1(g0, xr[0][0]);
#pragma unroll
                for (int u = 1; u < kUnroll; ++u) load_x1(g0 + u * 64, xr[0][u]);
#pragma unroll
                for (int r = 1; r < kBuf; ++r) load_x(g0 + r * step, xr[r]);
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
            for (int r = 0; r < kBuf; ++r) load_m(g0 + r * step, mr[r]);
        }
        int base = w_lo;
        auto stream_until = [&](int limit) {           // every buffer is loaded on entry
            for (; base < limit; base += kBuf * step, g0 += kBuf * step) {
#pragma unroll
                for (int r = 0; r < kBuf; ++r) {
                    fold(g0 + r * step, xr[r], mr[r]);
                    load_x(g0 + (kBuf + r) * step, xr[r]);
                    load_m(g0 + (kBuf + r) * step, mr[r]);
                }
            }
        };
        const int span = w_hi - w_lo;
        stream_until(w_lo + span - span / 4);
        if (ahead) {
            const unsigned long long w = wave_max_u64(candidate());
            tok_ahead = 0xFFFFFFFFu - (uint32_t)w;
            // w != 0: a token is allowed, so q is a row of the table; otherwise its first entry is read and not used
            const int64_t row_first = w != 0 ? (int64_t)q * V : 0;
            uint32_t col = w != 0 ? tok_ahead : 0u;
            asm volatile("" : "+v"(col));                  // a vector load: the LDS reads of the loop do not wait for it
            val_ahead = a.delta[row_first + col];
        }
        stream_until(w_hi);
    }
    if (g_hi > g_hi_full && threadIdx.x == 0) {
        // the row's last, partial group: element loads, same 16-bit keys
        const int g = n_full, t = g << 3;
        const uint32_t m = (valid ? bits_at(g) : 0u) & ((1u << (V - t)) - 1u);
        uint32_t d[4] = {0, 0, 0, 0}, top = 0;
        for (int j = 0; j < V - t; ++j) {
            const uint32_t h = row[t + j];
            const bool ok = (m >> j) & 1u;
            d[j >> 1] |= h << (16 * (j & 1));
            if (ok) top = max(top, (h & 0x8000u) ? (~h & 0xFFFFu) : (h ^ 0x8000u));
            if (WRITE) orow[t + j] = ok ? (uint16_t)h : (uint16_t)0xFF80u;
        }
        any |= m;
        if (top > best) {
            best = top;
            best_g = (uint32_t)g;
            best_m = m;
            best_x = make_uint4(d[0], d[1], d[2], d[3]);
        }
    }
    // The wavefront that holds the workgroup's maximum finishes the row (the first one if nothing is allowed; one
    // wavefront, since candidates differ in their tokens): each reads the wavefronts' candidates one per lane and folds
    // them across lanes.
    const unsigned long long wmax = wave_max_u64(candidate());         // the wavefront's final candidate
    if (lane == 0) wave_best[wave] = wmax;
    __syncthreads();
    unsigned long long cand = wave_max_u64(lane < ((int)blockDim.x >> 6) ? wave_best[lane] : 0ull);
    auto needs_exact = [](unsigned long long c) {
        const uint32_t ku = (uint32_t)(c >> 32) & 0xFFFFu;
        return ku > KU_POS_INF || ku <= KU_NEG_INF || ku == KU_POS_ZERO || ku == KU_NEG_ZERO;
    };
    // what lane 0 has, in every lane
    auto from_lane0 = [](unsigned long long c) {
        return ((unsigned long long)(uint32_t)__builtin_amdgcn_readfirstlane((int)(c >> 32)) << 32) |
               (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)c);
    };
    // PDA, by a whole wavefront: the row's token is taken (0: none)
    auto traverse = [&](unsigned long long c) {
        if (c == 0) {
            if (lane == 0) write_result(a, b, q, valid, 0ull);
        } else if constexpr (PDA) {
            pda_traverse(a.pda.edges, a.pda.stacks + (int64_t)b * a.pda.stack_cap, a.pda.depths + b, depth, a.pda.stack_cap, q,
                         (int)(0xFFFFFFFFu - (uint32_t)c), a.tokens + b, a.new_states + b);
        }
    };
    if constexpr (PDA) {
        if (cand == 0 ? wave == 0 : wmax == cand) {
            int last = 0;
            if (lane == 0) last = combine_parts(a, b, parts, cand) ? 1 : 0;
            last = __builtin_amdgcn_readfirstlane(last);
            cand = from_lane0(cand);
            const bool exact = last && cand != 0 && needs_exact(cand);
            if (last && !exact) traverse(cand);
            if (lane == 0) s_exact = exact ? 1 : 0;
        }
    } else {
    const bool finisher = lane == 0 && (cand == 0 ? threadIdx.x == 0 : wmax == cand);
    if (finisher) {
        int exact = 0;
        if (combine_parts(a, b, parts, cand)) {
            if (cand == 0) {
                write_result(a, b, q, valid, 0ull);
            } else if (needs_exact(cand)) {
                exact = 1;
            } else {
                const uint32_t token = 0xFFFFFFFFu - (uint32_t)cand;
                int32_t next;
                if (ahead && token == tok_ahead) next = val_ahead;
                else next = table_entry(a, q, (int)token);
                a.tokens[b] = (int32_t)token;
                a.new_states[b] = next;
            }
        }
        s_exact = exact;
    }
    }
    __syncthreads();
    if (!s_exact) return;
    // Rare: NaN, zeros or nothing above -inf at the top of the row.  The masked row is already
    // written, so this pass only chooses the token.
    unsigned long long c = exact_scan_with<TDFA_BF16>(row, nullptr, bits_at, valid, V, 0, n_groups);
    c = block_max_u64(c, wave_best_exact);
    if constexpr (PDA) {
        if (wave == 0) traverse(from_lane0(c));
    } else {
        if (threadIdx.x == 0) write_result(a, b, q, valid, c);
    }
}

template <bool WRITE, int kUnroll, bool SKIP, int kBuf = 2, bool PDA = false>
__global__ void __launch_bounds__(kMaxThreads)
mask_step_bf16_kernel(std::conditional_t<PDA, PdaMaskArgs, MaskArgs> a, int parts, int groups_per_part, int stretch)
{
    mask_step_bf16<WRITE, kUnroll, SKIP, kBuf, PDA, false>(a, parts, groups_per_part, stretch);
}

// The same for launches of more workgroups than compute units: at most 80 scalar registers, or eight wavefronts of a
// SIMD do not find room and a compute unit holds one workgroup of 1,024 threads at a time, not two (the compiler counts up
// to 100 as room for eight; the counters show half the wavefronts in flight from 94 on).  128,256 tokens, packed
// tables, every row sparse: 1,024 rows 16.7 -> 13.5 us (50 signatures) and 14.4 -> 11.2 us (16 schemas), 512 rows 11.3 ->
// 8.5 us; 1,024 rows of 64 schemas' states on a dense table 31.8 -> 26.4 us.  The registers that are kept in lanes for that cost launches that fill the chip once 0.2 to 0.5 us.
template <int kUnroll>
__global__ void __launch_bounds__(kMaxThreads) __attribute__((amdgpu_num_sgpr(80)))
mask_step_bf16_many_kernel(MaskArgs a, int parts, int groups_per_part, int stretch)
{
    mask_step_bf16<false, kUnroll, true, 2, false, true>(a, parts, groups_per_part, stretch);
}

// One step on fp32 logits.  Like the 16-bit kernel, every wavefront first reads the allowed bytes of
// its stretch and lists the groups that hold an allowed token; if all wavefronts of the workgroup
// find at most one such group in 16, they fetch just those groups (32 bytes each) and compare their
// allowed logits exactly.  Otherwise the workgroup scans its part of the row as the exact kernel
// does.  Candidates are (key, lowest token) as everywhere, so the order of the groups does not matter.
__global__ void __launch_bounds__(kMaxThreads)
mask_step_f32_kernel(MaskArgs a, int parts, int groups_per_part, int stretch)
{
    extern __shared__ uint4 s_pieces[];
    __shared__ uint32_t s_list[kMaxWaves * kListCap];
    __shared__ unsigned long long wave_best[kMaxWaves];
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    const int b = blockIdx.x / parts, p = blockIdx.x % parts;
    const int V = a.n_tokens;
    const int q = a.states[b];
    const bool valid = q >= 0 && (int64_t)q < a.n_rows;
    if (a.row_allowed != nullptr && valid && a.row_allowed[q] == 0u) {          // nothing allowed: no token, the state stays
        if (threadIdx.x == 0) {
            unsigned long long none = 0ull;
            if (combine_parts(a, b, parts, none)) write_result(a, b, q, valid, none);
        }
        return;
    }
    const uint8_t* bits = reinterpret_cast<const uint8_t*>(a.allow + (valid ? (int64_t)q * a.row_words : 0));
    const uint32_t* row = static_cast<const uint32_t*>(a.logits) + (int64_t)b * a.row_stride;
    const int n_groups = (V + 7) >> 3;
    const int n_full = V >> 3;
    const int g_lo = p * groups_per_part;
    const int g_hi = min(n_groups, g_lo + groups_per_part);
    const int g_hi_full = min(g_hi, n_full);
    const int lane = (int)threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int w_lo = min(g_lo + wave * stretch, g_hi_full);
    const int w_hi = min(w_lo + stretch, g_hi_full);

    // the allowed bytes of the stretch, 16 per lane and pass, and how many of them are not zero
    uint4* my_pieces = s_pieces + wave * (stretch >> 4);
    const int n_pieces = (w_hi - w_lo + 15) >> 4;
    const __amdgpu_buffer_rsrc_t r_row =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(bits), 0, valid ? a.row_words * 4 : 0, kRawBuffer);
    uint32_t nz = 0;
    for (int i = lane; i < n_pieces; i += 64) {
        const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(r_row, w_lo + i * 16, 0, 0);
        uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            const int left = w_hi - (w_lo + i * 16 + d * 4);
            if (left <= 0) w[d] = 0;
            else if (left < 4) w[d] &= (1u << (8 * left)) - 1u;
            nz += nonzero_bytes(w[d]);
        }
        my_pieces[i] = make_uint4(w[0], w[1], w[2], w[3]);
    }
    const uint32_t n_listed = wave_sum_u32(nz);
    const bool few = n_listed <= (uint32_t)kListCap && n_listed * 16u <= (uint32_t)(w_hi - w_lo);
    unsigned long long best = 0;
    if (__syncthreads_and(few)) {
        uint32_t slot = 0;
#pragma unroll
        for (int bit = 0; bit < 9; ++bit) slot += lanes_below((nz >> bit) & 1u) << bit;
        uint32_t* list = s_list + wave * kListCap;
        for (int i = lane; i < n_pieces; i += 64) {
            const uint4 pc = my_pieces[i];
            const uint32_t w[4] = {pc.x, pc.y, pc.z, pc.w};
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                uint32_t rest = w[d];
                while (rest) {
                    const int byte = (__builtin_ctz(rest)) >> 3;
                    list[slot++] = (uint32_t)((i * 16 + d * 4 + byte) << 8) | ((rest >> (8 * byte)) & 0xFFu);
                    rest &= ~(0xFFu << (8 * byte));
                }
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        const __amdgpu_buffer_rsrc_t r_logits =
            __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t*>(row), 0, w_hi * 32, kRawBuffer);
        // one listed group per lane, two at a time
        for (uint32_t r0 = 0; r0 < n_listed; r0 += 128) {
            u32x4 lo[2], hi[2];
            uint32_t m[2];
            int g[2];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const uint32_t idx = r0 + (uint32_t)(u * 64 + lane);
                const uint32_t e = idx < n_listed ? list[idx] : 0u;
                g[u] = w_lo + (int)(e >> 8);
                m[u] = e & 0xFFu;
                lo[u] = __builtin_amdgcn_raw_buffer_load_b128(r_logits, idx < n_listed ? g[u] * 32 : 0x7FFFFFF0, 0, kReadOnce);
                hi[u] = __builtin_amdgcn_raw_buffer_load_b128(r_logits, idx < n_listed ? g[u] * 32 + 16 : 0x7FFFFFF0, 0, kReadOnce);
            }
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const uint32_t e8[8] = {lo[u].x, lo[u].y, lo[u].z, lo[u].w, hi[u].x, hi[u].y, hi[u].z, hi[u].w};
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const unsigned long long c = ((unsigned long long)key_f32(e8[j]) << 32) | (0xFFFFFFFFu - (uint32_t)(g[u] * 8 + j));
                    if (((m[u] >> j) & 1u) && c > best) best = c;
                }
            }
        }
        if (g_hi > g_hi_full && threadIdx.x == 0 && valid) {
            // the row's last, partial group
            const int t = n_full << 3;
            const uint32_t m = bits[n_full];
            for (int j = 0; j < V - t; ++j) {
                const unsigned long long c = ((unsigned long long)key_f32(row[t + j]) << 32) | (0xFFFFFFFFu - (uint32_t)(t + j));
                if (((m >> j) & 1u) && c > best) best = c;
            }
        }
    } else {
        best = exact_scan<TDFA_F32>(row, nullptr, bits, valid, V, g_lo, g_hi);
    }
    best = block_max_u64(best, wave_best);
    if (threadIdx.x != 0) return;
    if (combine_parts(a, b, parts, best)) write_result(a, b, q, valid, best);
}

// ---------------------------------------------------------------------------------------------
// Sampling step: SampleNextToken of Algorithm 2 as a draw from softmax(l / T) over the allowed
// set, by the Gumbel-max rule: the allowed token with the largest fma(l_t, 1/T, g_t) wins, g_t
// standard Gumbel noise made from one word of Philox4x32-10 (Salmon et al. 2011) per token.  The
// chosen token is an integer decided by floating point, so the noise is defined operation by
// operation in IEEE-754 binary32 (see the declaration of tdfa_sample_step); nothing below may be
// contracted, reassociated or replaced by an approximate instruction.
// ---------------------------------------------------------------------------------------------
#pragma clang fp contract(off)

struct SampleParams {
    float inv_t;
    uint32_t seed_lo, seed_hi, off_lo, off_hi;
    const unsigned long long* off_dev;   // if not NULL: the offset is read from here by the kernel (off_lo / off_hi unused)
};

// counter (c0, c1, c2, c3), key (k0, k1) -> four words, ten rounds.  Where c1, c2, c3 and the key are the same in all
// lanes, half of the first three rounds is scalar: their exclusive-ors are grouped for that, the later ones take one
// three-input instruction.
__device__ __forceinline__ void philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3, uint32_t k0,
                                              uint32_t k1, uint32_t (&w)[4])
{
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const unsigned long long p0 = (unsigned long long)0xD2511F53u * c0;
        const unsigned long long p1 = (unsigned long long)0xCD9E8D57u * c2;
        const uint32_t h0 = (uint32_t)(p0 >> 32), h1 = (uint32_t)(p1 >> 32);
        c0 = r < 2 ? h1 ^ (c1 ^ k0) : __builtin_amdgcn_bitop3_b32(h1, c1, k0, 0x96);
        c2 = r == 1 ? c3 ^ (h0 ^ k1) : r < 3 ? h0 ^ (c3 ^ k1) : __builtin_amdgcn_bitop3_b32(h0, c3, k1, 0x96);
        c1 = (uint32_t)p1;
        c3 = (uint32_t)p0;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    w[0] = c0; w[1] = c1; w[2] = c2; w[3] = c3;
}

// Natural logarithm of a positive normal number: x = 2^e m, m in (sqrt(1/2), sqrt(2)],
// ln m = 2 atanh(s) with s = (m - 1) / (m + 1), five terms of the series by Horner's rule.
__device__ __forceinline__ float ln32(float x)
{
    const uint32_t i = __float_as_uint(x);
    int e = (int)(i >> 23) - 127;
    const uint32_t frac = i & 0x7FFFFFu;
    float m = __uint_as_float(frac | 0x3F800000u);
    if (frac > 0x3504F3u) {                                  // above sqrt(2): halve (exact)
        m = m * 0.5f;
        e += 1;
    }
    const float f = m - 1.0f;                                 // exact
    const float s = __fdiv_rn(f, 2.0f + f);
    const float z = s * s;
    float p = __builtin_fmaf(z, 2.0f / 9.0f, 2.0f / 7.0f);
    p = __builtin_fmaf(z, p, 2.0f / 5.0f);
    p = __builtin_fmaf(z, p, 2.0f / 3.0f);
    p = __builtin_fmaf(z, p, 2.0f);
    return __builtin_fmaf((float)e, 0.693147180559945309f, s * p);
}

// Standard Gumbel variate from one generator word: u = ((x >> 9) + 1/2) 2^-23, g = -ln(-ln u).
__device__ __forceinline__ float gumbel_of(uint32_t x)
{
    const float u = __builtin_fmaf((float)(x >> 9), 0x1p-23f, 0x1p-24f);
    return -ln32(-ln32(u));
}

constexpr float kNoiseMax = 16.64f;    // above every noise value: -ln(-ln(1 - 2^-24)) = 16.6355...

// Not below the noise that generator word x makes.  With v = 2^32 (1 - u), a multiple of 256 below 2^32 and so exact in
// binary32, g = -ln(-ln u) <= -ln(1 - u) = (32 - log2 v) ln 2, and the bits of v's binary32 pattern, as an integer
// divided by 2^23, less 127, are its logarithm with straight lines between the powers of two: never above log2 v,
// and at most 0.0861 below.  The slack added covers the rounding of the noise as computed and of this bound.  fma is monotonic in its addend, so a token whose bound stays below a score already reached
// scores below it as well.
__device__ __forceinline__ float noise_bound(uint32_t x)
{
    const uint32_t v = (~x & 0xFFFFFE00u) | 0x100u;
    return __builtin_fmaf((float)(int32_t)__float_as_uint((float)v), -0.693147180559945309f * 0x1p-23f, 159.0f * 0.693147180559945309f + 1.0e-3f);
}

// The noise alone: out[b][t] = g_t of sequence b, for callers that want to reproduce a draw.
__global__ void __launch_bounds__(256)
sample_noise_kernel(SampleParams sp, int32_t n_tokens, int64_t n_quads_total, int32_t quads_per_row, float* __restrict__ out)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n_quads_total) return;
    const int32_t b = (int32_t)(i / quads_per_row), k = (int32_t)(i % quads_per_row);
    uint32_t w[4];
    philox4x32_10((uint32_t)k, (uint32_t)b, sp.off_lo, sp.off_hi, sp.seed_lo, sp.seed_hi, w);
#pragma unroll
    for (int j = 0; j < 4; ++j)
        if (4 * k + j < n_tokens) out[(int64_t)b * n_tokens + 4 * k + j] = gumbel_of(w[j]);
}

// Draw under a top-k cut: one workgroup per sequence finds the order key of the k-th largest allowed logit and draws
// among the tokens that reach it (fewer than k allowed tokens: among all).
//
// The row is read once.  Every thread keeps 16 groups of eight tokens (kRowGroups; 1,024 threads: 131,072 tokens) in
// registers as 16-bit order keys, a token that is not allowed as key 0, all loads in flight at once:
//   1. the k-th largest of the threads' maxima, L, is selected from two 256-bin histograms in LDS: at least k allowed
//      logits reach L, so the k-th largest of the row does too;
//   2. the tokens that reach L (little more than k of them) are collected in LDS from the registers, and the k-th
//      largest of the collected keys is the cut;
//   3. the collected tokens at or above the cut, one per thread, get their noise and compete.
// A state that allows at most kKeep tokens is collected whole, reading only its groups.  Where the shortcut does not
// hold (k above the number of threads that saw a token, masses of equal logits, NaN or -inf at the cut) the cut is
// selected over the row, most significant digit first, and a scan of the row draws (`slow` below).
//
// What bounds it: a compute unit streams its 256 KB row at what one unit gets from memory (9 to 10 us), then five
// barriers and two dependent reads follow.  k = 50, T = 0.7, 256 sequences, 128,256 tokens in bf16: states anywhere in
// their texts 73.6 -> 17.6 us, all in states that allow most tokens 75.7 -> 19.3 us, all in states that allow few
// 22.6 -> 9.1 us (fp32: 78.5 -> 31.5 us where most are allowed), against a kernel that made the cut, which read the row
// one and an eighth times, and the gathering scan for the draw, which read it again.
constexpr int kKeep = 2048;            // collected tokens that fit in LDS
constexpr int kRowGroups = 16;         // groups of eight tokens that a thread holds in registers

template <int DTYPE, bool WRITE, bool RESIDENT>
__global__ void __launch_bounds__(kMaxThreads)
topk_step_kernel(MaskArgs a, SampleParams sp, int32_t top_k)
{
    using Elem = typename ElemOf<DTYPE>::type;
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    __shared__ __attribute__((aligned(16))) uint32_t s_keys[kKeep];
    __shared__ __attribute__((aligned(16))) uint32_t hist[4 * 256];        // a histogram of 256 bins per digit of a key
    __shared__ uint2 s_cand[kKeep];                                        // (token, logit as binary32)
    __shared__ uint2 s_list[kKeep];                                        // few: (group << 8 | bits, place of its first token)
    __shared__ unsigned long long wave_best[kMaxWaves];
    __shared__ uint32_t s_scan[kMaxWaves];
    __shared__ uint32_t s_bin, s_n, s_groups, s_special;
    const int b = blockIdx.x;
    const int V = a.n_tokens;
    const int q = a.states[b];
    const bool valid = q >= 0 && (int64_t)q < a.n_rows;
    const uint8_t* bits = reinterpret_cast<const uint8_t*>(a.allow + (valid ? (int64_t)q * a.row_words : 0));
    const Elem* row = static_cast<const Elem*>(a.logits) + (int64_t)b * a.row_stride;
    Elem* orow = WRITE ? static_cast<Elem*>(a.masked_out) + (int64_t)b * a.row_stride : nullptr;
    const int n_groups = (V + 7) >> 3, n_full = V >> 3;
    const int T = (int)blockDim.x, tid = (int)threadIdx.x, lane = tid & 63;     // T is 256 or 1024
    const uint32_t k = (uint32_t)top_k;
    if (sp.off_dev) {                                              // the same word for every thread
        const unsigned long long o = *sp.off_dev;
        sp.off_lo = (uint32_t)o;
        sp.off_hi = (uint32_t)(o >> 32);
    }
    if (tid == 0) {
        s_n = 0;
        s_groups = 0;
        s_special = 0;
    }
    for (int i = tid; i < 512; i += T) hist[i] = 0;

    // how many tokens the state allows
    uint32_t n_allowed = valid ? allowed_count(a, q) : 0u;
    __syncthreads();
    if (n_allowed == kUnknown) {                                   // the bit row tells
        const uint32_t* words = reinterpret_cast<const uint32_t*>(bits);
        const int n_words = (V + 31) >> 5;
        uint32_t c = 0;
        for (int i = tid; i < n_words; i += T) c += __popc(words[i]);
        c = wave_sum_u32(c);
        if (lane == 0) s_scan[tid >> 6] = c;
        __syncthreads();
        n_allowed = 0;
        for (int w = 0; w < (T >> 6); ++w) n_allowed += s_scan[w];
    }
    if (!WRITE && n_allowed == 0) {
        if (tid == 0) write_result(a, b, q, valid, 0ull);
        return;
    }
    const bool few = n_allowed <= (uint32_t)kKeep;
    // rows beyond the reach of 32-bit byte offsets are scanned through pointers
    const bool huge = V > (1 << 26);

    // f(u, group, its eight logits, the words they came in, its allowed bits) for the thread's whole groups of chunk c:
    // kRowGroups loads in flight (fp32: four groups, eight loads).  The tokens of the row's last, partial group are
    // for the first threads: for_tail.
    constexpr int kAhead = DTYPE == TDFA_F32 ? (WRITE ? 2 : 4) : kRowGroups;
    auto for_chunk = [&](int c, auto&& f) __attribute__((always_inline)) {
        const int g0 = c * kRowGroups * T + tid;
#pragma unroll
        for (int u0 = 0; u0 < kRowGroups; u0 += kAhead) {
            if (DTYPE == TDFA_F32) __builtin_amdgcn_sched_barrier(0);      // (loads of later batches moved up here would spill)
            u32x4 lo[kAhead], hi[DTYPE == TDFA_F32 ? kAhead : 1];
            uint32_t m[kAhead];
#pragma unroll
            for (int u = 0; u < kAhead; ++u) {
                // a descriptor of its own per pass over the threads, made of scalars: the lane's offsets are the same in
                // all of them.  (A group past the end reads zeros, without a memory access.)
                const int gs = (c * kRowGroups + u0 + u) * T;
                const __amdgpu_buffer_rsrc_t r_x = __builtin_amdgcn_make_buffer_rsrc(
                    const_cast<Elem*>(row) + (int64_t)gs * 8, 0, max(n_full - gs, 0) * 8 * (int)sizeof(Elem), kRawBuffer);
                const __amdgpu_buffer_rsrc_t r_m =
                    __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(bits) + gs, 0, valid ? max(n_full - gs, 0) : 0, kRawBuffer);
                lo[u] = __builtin_amdgcn_raw_buffer_load_b128(r_x, tid * 8 * (int)sizeof(Elem), 0, kReadOnce);
                if constexpr (DTYPE == TDFA_F32) hi[u] = __builtin_amdgcn_raw_buffer_load_b128(r_x, tid * 32 + 16, 0, kReadOnce);
                m[u] = __builtin_amdgcn_raw_buffer_load_b8(r_m, tid, 0, 0);
            }
#pragma unroll
            for (int u = 0; u < kAhead; ++u) {
                const int g = g0 + (u0 + u) * T;
                Elem e[8];
                if constexpr (DTYPE == TDFA_F32) {
                    e[0] = lo[u].x; e[1] = lo[u].y; e[2] = lo[u].z; e[3] = lo[u].w;
                    e[4] = hi[u].x; e[5] = hi[u].y; e[6] = hi[u].z; e[7] = hi[u].w;
                } else {
                    e[0] = (Elem)lo[u].x; e[1] = (Elem)(lo[u].x >> 16); e[2] = (Elem)lo[u].y; e[3] = (Elem)(lo[u].y >> 16);
                    e[4] = (Elem)lo[u].z; e[5] = (Elem)(lo[u].z >> 16); e[6] = (Elem)lo[u].w; e[7] = (Elem)(lo[u].w >> 16);
                }
                f(u0 + u, g, e, lo[u], m[u]);
            }
        }
    };
    const int n_chunks = RESIDENT ? 1 : (n_full + kRowGroups * T - 1) / (kRowGroups * T);
    auto as_f32 = [](uint32_t x) {                                 // NaN counts as -inf
        uint32_t lb = DTYPE == TDFA_F32 ? x : x << 16;
        if ((lb & 0x7FFFFFFFu) > 0x7F800000u) lb = 0xFF800000u;
        return lb;
    };
    auto push = [&](int t, uint32_t lb) {
        const uint32_t i = atomicAdd(&s_n, 1u);
        if (i < (uint32_t)kKeep) {
            s_cand[i] = make_uint2((uint32_t)t, lb);
            s_keys[i] = key_f32(lb);
        }
    };
    // the penalised logits of group gs + tid (gs: scalar); nothing past the whole groups
    auto store_masked = [&](int gs, const Elem (&e)[8], uint32_t mg) {
        if constexpr (WRITE) {
            constexpr Elem NEG_INF = DTYPE == TDFA_F32 ? (Elem)0xFF800000u : (Elem)0xFF80u;
            uint32_t o[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) o[j] = (mg >> j) & 1u ? e[j] : NEG_INF;
            const __amdgpu_buffer_rsrc_t r_o = __builtin_amdgcn_make_buffer_rsrc(
                orow + (int64_t)gs * 8, 0, max(n_full - gs, 0) * 8 * (int)sizeof(Elem), kRawBuffer);
            if constexpr (DTYPE == TDFA_F32) {
                __builtin_amdgcn_raw_buffer_store_b128(u32x4{o[0], o[1], o[2], o[3]}, r_o, tid * 32, 0, kReadOnce);
                __builtin_amdgcn_raw_buffer_store_b128(u32x4{o[4], o[5], o[6], o[7]}, r_o, tid * 32 + 16, 0, kReadOnce);
            } else {
                __builtin_amdgcn_raw_buffer_store_b128(u32x4{o[0] | o[1] << 16, o[2] | o[3] << 16, o[4] | o[5] << 16, o[6] | o[7] << 16}, r_o,
                                                       tid * 16, 0, kReadOnce);
            }
        }
    };
    // f(token, its logit, whether it is allowed) for the tokens of the partial group
    auto for_tail = [&](auto&& f) {
        const int t = (n_full << 3) + tid;
        if (t < V) f(t, row[t], valid && ((bits[n_full] >> tid) & 1u));
    };
    auto store_tail = [&]() {
        if constexpr (WRITE) {
            constexpr Elem NEG_INF = DTYPE == TDFA_F32 ? (Elem)0xFF800000u : (Elem)0xFF80u;
            for_tail([&](int t, Elem x, bool ok) { orow[t] = ok ? x : NEG_INF; });
        }
    };

    // The bin of a 256-bin histogram that holds the want-th entry from the top, and which entry of the bin it is; false
    // if there are fewer.  Every wavefront reads the histogram for itself, four bins per lane.
    auto find_bin = [&](const uint32_t* h, uint32_t want, uint32_t* bin, uint32_t* left) -> bool {
        const uint4 v = *reinterpret_cast<const uint4*>(h + 4 * lane);
        const uint32_t mine = v.x + v.y + v.z + v.w;
        uint32_t incl = mine;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const uint32_t other = __shfl_down(incl, d, 64);
            if (lane + d < 64) incl += other;
        }
        const uint32_t a3 = incl - mine, a2 = a3 + v.w, a1 = a2 + v.z, a0 = a1 + v.y;        // counts above the lane's bins
        const uint32_t sub = want <= a2 ? 3u : want <= a1 ? 2u : want <= a0 ? 1u : 0u;
        const uint32_t above = want <= a2 ? a3 : want <= a1 ? a2 : want <= a0 ? a1 : a0;
        const unsigned long long at = __builtin_amdgcn_ballot_w64(a3 < want && want <= incl);
        if (at == 0) return false;
        const int src = __builtin_ctzll(at);
        *bin = 4u * (uint32_t)src + (uint32_t)__builtin_amdgcn_readlane((int)sub, src);
        *left = want - (uint32_t)__builtin_amdgcn_readlane((int)above, src);
        return true;
    };
    // The want-th largest of the keys that `each` enumerates, or a number between it and the next smaller key; false if
    // there are fewer keys.  Eight bits per pass from the top; the upper half of a bf16 logit's key tells all of it.
    auto select = [&](auto&& each, uint32_t want, uint32_t* result) -> bool {
        __syncthreads();
        for (int i = tid; i < 4 * 256; i += T) hist[i] = 0;
        __syncthreads();
        uint32_t prefix = 0, fixed_mask = 0;
        for (int pass = 0; pass < (DTYPE == TDFA_F32 ? 4 : 2); ++pass) {
            const int shift = 24 - 8 * pass;
            each([&](uint32_t key) {
                if ((key & fixed_mask) == prefix) atomicAdd(&hist[256 * pass + ((key >> shift) & 255u)], 1u);
            });
            __syncthreads();
            uint32_t bin = 0;
            if (!find_bin(hist + 256 * pass, want, &bin, &want)) return false;
            prefix |= bin << shift;
            fixed_mask |= 255u << shift;
        }
        *result = prefix;
        return true;
    };

    uint32_t best_key = 0, best_idx = 0xFFFFFFFFu;                 // key 0: no candidate yet
    auto consider = [&](uint32_t tok, uint32_t lb, uint32_t word) {
        const uint32_t key = key_f32(__float_as_uint(__builtin_fmaf(__uint_as_float(lb), sp.inv_t, gumbel_of(word))));
        if (key > best_key || (key == best_key && tok < best_idx)) {
            best_key = key;
            best_idx = tok;
        }
    };

    bool slow = huge;
    uint32_t floor_key = 0;                                        // k allowed tokens or more are known to reach it
    if (few && !huge) {
        // The groups with an allowed token, and where their tokens go among the collected ones: 16 groups per thread
        // and pass, a prefix over the lanes, one addition per wavefront to the two counts.  Then a group per thread.
        const uint4* pieces = reinterpret_cast<const uint4*>(bits);
        const int n_pieces = (n_groups + 15) >> 4;
        for (int i0 = 0; i0 < n_pieces; i0 += T) {                 // (uniform trip count)
            const int i = i0 + tid;
            uint4 pc = make_uint4(0, 0, 0, 0);
            if (valid && i < n_pieces) pc = pieces[i];
            uint32_t w[4] = {pc.x, pc.y, pc.z, pc.w};
            uint32_t n_here = 0, g_here = 0;
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                const int rem = V - (i * 16 + d * 4) * 8;          // tokens from this word on
                if (rem < 32) w[d] = rem <= 0 ? 0u : w[d] & ((1u << rem) - 1u);
                n_here += __popc(w[d]);
                g_here += nonzero_bytes(w[d]);
            }
            // both counts in one word: at most 128 tokens and 16 groups a lane
            const uint32_t both = n_here | (g_here << 16);
            uint32_t incl = both;
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) {
                const uint32_t other = __shfl_up(incl, d, 64);
                if (lane >= d) incl += other;
            }
            const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
            if (total == 0) continue;                              // (uniform in the wavefront)
            uint32_t n_base = 0, g_base = 0;
            if (lane == 0) {
                n_base = atomicAdd(&s_n, total & 0xFFFFu);
                g_base = atomicAdd(&s_groups, total >> 16);
            }
            n_base = (uint32_t)__builtin_amdgcn_readfirstlane((int)n_base) + ((incl - both) & 0xFFFFu);
            g_base = (uint32_t)__builtin_amdgcn_readfirstlane((int)g_base) + ((incl - both) >> 16);
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                uint32_t rest = w[d];
                while (rest) {
                    const int at = __builtin_ctz(rest) & 24;
                    const uint32_t m = (rest >> at) & 0xFFu;
                    if (g_base < (uint32_t)kKeep) s_list[g_base] = make_uint2((uint32_t)(i * 16 + d * 4 + (at >> 3)) << 8 | m, n_base);
                    ++g_base;
                    n_base += __popc(m);
                    rest &= ~(0xFFu << at);
                }
            }
        }
        __syncthreads();
        if (s_n <= (uint32_t)kKeep) {                              // (always, unless the count beside the table is not the row's)
            for (uint32_t i = tid; i < s_groups; i += (uint32_t)T) {
                const uint2 en = s_list[i];
                const int t = (int)(en.x >> 8) << 3;
                Elem e[8];
                load_group<DTYPE>(row, t, V, e);
                uint32_t at = en.y;
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    if ((en.x >> j) & 1u) {
                        const uint32_t lb = as_f32((uint32_t)e[j]);
                        s_cand[at] = make_uint2((uint32_t)(t + j), lb);
                        s_keys[at] = key_f32(lb);
                        ++at;
                    }
            }
        }
        if constexpr (WRITE) {
            __syncthreads();                                       // (the rows may be the same memory)
            for (int c = 0; c < n_chunks; ++c)
                for_chunk(c, [&](int u, int, const Elem (&e)[8], const u32x4&, uint32_t mg) {
                    store_masked((c * kRowGroups + u) * T, e, mg);
                });
            store_tail();
        }
    } else if (!huge) {
        // 16-bit order keys, two per word, 0 for a token that is not allowed: of a bf16 logit the whole key, of an fp32
        // logit its upper half (NaN and -0 as their patterns)
        uint32_t kk[RESIDENT ? kRowGroups : 1][4];
        auto keys_of = [&](const Elem (&e)[8], const u32x4& raw, uint32_t mg, uint32_t (&o)[4]) {
            const uint32_t d[4] = {raw.x, raw.y, raw.z, raw.w};
            const uint32_t y = mg | (mg << 15);                    // allowed bit 2j at bit 2j, bit 2j + 1 at bit 16 + 2j
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                uint32_t two;
                if constexpr (DTYPE == TDFA_F32) {
                    const uint32_t x0 = (uint32_t)e[2 * i], x1 = (uint32_t)e[2 * i + 1];
                    const uint32_t k0 = x0 ^ ((uint32_t)((int32_t)x0 >> 31) | 0x80000000u), k1 = x1 ^ ((uint32_t)((int32_t)x1 >> 31) | 0x80000000u);
                    two = __builtin_amdgcn_perm(k1, k0, 0x07060302u);          // the upper halves
                } else {
                    two = keys2(d[i]);
                }
                const uint32_t pj = (y >> (2 * i)) & 0x00010001u;
                o[i] = __builtin_bit_cast(uint32_t, __builtin_bit_cast(u16x2, two) * __builtin_bit_cast(u16x2, pj));
            }
        };
        u16x2 acc = {0, 0};
        for (int c = 0; c < n_chunks; ++c)
            for_chunk(c, [&](int u, int g, const Elem (&e)[8], const u32x4& raw, uint32_t mg) {
                uint32_t o[4];
                keys_of(e, raw, mg, o);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    acc = __builtin_elementwise_max(acc, __builtin_bit_cast(u16x2, o[i]));
                    if constexpr (RESIDENT) kk[u][i] = o[i];
                }
                store_masked((c * kRowGroups + u) * T, e, mg);
            });
        store_tail();
        const uint32_t a2 = __builtin_bit_cast(uint32_t, acc);
        const uint32_t top = max(a2 & 0xFFFFu, a2 >> 16);
        // the k-th largest of the threads' maxima
        if (top != 0) atomicAdd(&hist[top >> 8], 1u);
        if (top > KU_POS_INF || (DTYPE == TDFA_F32 && top == KU_POS_INF)) s_special = 1;         // perhaps NaN
        __syncthreads();
        uint32_t hi8 = 0, lo8 = 0, left = 0;
        bool found = find_bin(hist, k, &hi8, &left);
        if (found && top != 0 && (top >> 8) == hi8) atomicAdd(&hist[256 + (top & 255u)], 1u);
        __syncthreads();
        found = found && find_bin(hist + 256, left, &lo8, &left);
        uint32_t L = (hi8 << 8) | lo8;
        if (!found || s_special || L <= KU_NEG_INF) {
            slow = true;                                           // the same in every thread
        } else {
            if (L == KU_POS_ZERO) L = KU_NEG_ZERO;                 // -0 equals +0
            floor_key = L << 16;
            for_tail([&](int t, Elem x, bool ok) {
                if (ok && key_f32(as_f32((uint32_t)x)) >> 16 >= L) push(t, as_f32((uint32_t)x));
            });
            if constexpr (RESIDENT) {
                if (__builtin_amdgcn_ballot_w64(top >= L) != 0) {
#pragma unroll
                    for (int u = 0; u < kRowGroups; ++u) {
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            const uint32_t k0 = kk[u][i] & 0xFFFFu, k1 = kk[u][i] >> 16;
                            if (k0 >= L || k1 >= L) {
                                const int t = ((u * T + tid) << 3) + 2 * i;
                                auto put = [&](uint32_t key, int tok) {
                                    if (key < L) return;
                                    if constexpr (DTYPE == TDFA_F32) push(tok, as_f32((uint32_t)row[tok]));
                                    else push(tok, as_f32(key & 0x8000u ? key ^ 0x8000u : ~key & 0xFFFFu));
                                };
                                put(k0, t);
                                put(k1, t + 1);
                            }
                        }
                    }
                }
            } else {
                for (int c = 0; c < n_chunks; ++c)
                    for_chunk(c, [&](int, int g, const Elem (&e)[8], const u32x4& raw, uint32_t mg) {
                        uint32_t o[4];
                        keys_of(e, raw, mg, o);
                        u16x2 ga = {0, 0};
#pragma unroll
                        for (int i = 0; i < 4; ++i) ga = __builtin_elementwise_max(ga, __builtin_bit_cast(u16x2, o[i]));
                        const uint32_t g2 = __builtin_bit_cast(uint32_t, ga);
                        if (__builtin_amdgcn_ballot_w64(max(g2 & 0xFFFFu, g2 >> 16) >= L) == 0) return;
#pragma unroll
                        for (int j = 0; j < 8; ++j)
                            if ((o[j >> 1] >> (16 * (j & 1)) & 0xFFFFu) >= L) push((g << 3) + j, as_f32((uint32_t)e[j]));
                    });
            }
        }
    }
    __syncthreads();
    const uint32_t n = s_n;
    slow = slow || n > (uint32_t)kKeep;
    uint32_t cut = 0;
    if (!slow) {
        // the k-th largest of the collected keys (fewer than k, so fewer than k allowed tokens: no cut)
        if (n >= k) {
            if (n <= 128u) {
                // by counting: a key is the answer if fewer than k keys are greater and at least k are greater or equal
                for (uint32_t i = n + tid; i < ((n + 3u) & ~3u); i += (uint32_t)T) s_keys[i] = 0;   // pad to whole uint4
                if (tid == 0) s_bin = 0;
                __syncthreads();
                for (uint32_t i = tid; i < n; i += (uint32_t)T) {
                    const uint32_t mine = s_keys[i];
                    uint32_t gt = 0, ge = 0;
                    for (uint32_t j = 0; j < n; j += 4) {
                        const uint4 o = *reinterpret_cast<const uint4*>(&s_keys[j]);
                        gt += (o.x > mine) + (o.y > mine) + (o.z > mine) + (o.w > mine);
                        ge += (o.x >= mine) + (o.y >= mine) + (o.z >= mine) + (o.w >= mine);
                    }
                    if (gt < k && k <= ge) s_bin = mine;            // equal keys all write the same value
                }
                __syncthreads();
                cut = s_bin;
            } else if (!select([&](auto&& f) { for (uint32_t i = tid; i < n; i += (uint32_t)T) f(s_keys[i]); }, k, &cut)) {
                cut = 0;
            }
        }
        for (uint32_t i = tid; i < n; i += (uint32_t)T) {
            if (s_keys[i] < cut) continue;
            const uint2 en = s_cand[i];
            uint32_t w[4];
            philox4x32_10(en.x >> 2, (uint32_t)b, sp.off_lo, sp.off_hi, sp.seed_lo, sp.seed_hi, w);
            const uint32_t lo = (en.x & 1u) ? w[1] : w[0], hi = (en.x & 1u) ? w[3] : w[2];
            consider(en.x, en.y, (en.x & 2u) ? hi : lo);
        }
    } else {
        auto for_row = [&](auto&& f) {                             // f(key) for every allowed logit of the row that may be at the cut
            for (int g = tid; g < n_groups; g += T) {
                const uint32_t mg = valid ? bits[g] : 0u;
                if (mg == 0) continue;
                Elem e[8];
                load_group<DTYPE>(row, g << 3, V, e);
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const uint32_t key = key_f32(as_f32((uint32_t)e[j]));
                    if (((mg >> j) & 1u) && key >= floor_key) f(key);
                }
            }
        };
        if (!select(for_row, k, &cut)) cut = 0;                    // fewer than k allowed tokens: no cut
        float reached = -__builtin_inff();                         // a score some token of this wavefront has reached
        for (int base = 0; base < n_groups; base += T) {
            const int g = base + tid;
            const uint32_t mg = valid && g < n_groups ? bits[g] : 0u;
            uint32_t take = 0;
            Elem e[8] = {};
            if (mg != 0 || (WRITE && huge && g < n_groups)) load_group<DTYPE>(row, g << 3, V, e);
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const uint32_t lb = as_f32((uint32_t)e[j]);
                // no noise value exceeds kNoiseMax: a token that cannot reach the best score is not drawn for
                const bool may = __builtin_fmaf(__uint_as_float(lb), sp.inv_t, kNoiseMax) >= reached;
                take |= (uint32_t)(((mg >> j) & 1u) && key_f32(lb) >= cut && may) << j;
            }
            if (WRITE && huge && g < n_groups) {
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const int64_t t = (int64_t)g * 8 + j;
                    if (t < V) orow[t] = (mg >> j) & 1u ? e[j] : (Elem)(DTYPE == TDFA_F32 ? 0xFF800000u : 0xFF80u);
                }
            }
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                if (((take >> (4 * h)) & 15u) == 0) continue;
                uint32_t w[4];
                philox4x32_10(((uint32_t)g << 1) + h, (uint32_t)b, sp.off_lo, sp.off_hi, sp.seed_lo, sp.seed_hi, w);
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    if (!((take >> (4 * h + j)) & 1u)) continue;
                    const uint32_t lb = as_f32((uint32_t)e[4 * h + j]);
                    if (__builtin_fmaf(__uint_as_float(lb), sp.inv_t, noise_bound(w[j])) >= reached) consider((uint32_t)((g << 3) + 4 * h + j), lb, w[j]);
                }
            }
            const uint32_t wave_top = wave_max_u32(best_key);      // 0: nothing scored yet
            if (wave_top != 0) reached = __uint_as_float((wave_top & 0x80000000u) ? wave_top & 0x7FFFFFFFu : ~wave_top);
        }
    }
    unsigned long long cand = best_key ? ((unsigned long long)best_key << 32) | (0xFFFFFFFFu - best_idx) : 0ull;
    cand = block_max_u64(cand, wave_best);
    if (tid == 0) write_result(a, b, q, valid, cand);
}

// Greedy step on a packed table whose logits are fp32 (or whose rows the step kernel cannot address): the
// gathering scan of sparse rows, and an element by element comparison of the rows that allow an eighth of the
// vocabulary or more.
template <int DTYPE>
__global__ void __launch_bounds__(kMaxThreads)
packed_step_kernel(MaskArgs a, int parts, int groups_per_part)
{
    using Elem = typename ElemOf<DTYPE>::type;
    __shared__ unsigned long long wave_best[kMaxWaves];
    __shared__ uint2 s_ring[kMaxWaves][kGatherQueue];
    const int b = blockIdx.x / parts, p = blockIdx.x % parts;
    const int V = a.n_tokens;
    const int q = a.states[b];
    const bool valid = q >= 0 && (int64_t)q < a.n_rows;
    const uint8_t* bits = reinterpret_cast<const uint8_t*>(a.allow + (valid ? (int64_t)q * a.row_words : 0));
    const Elem* row = static_cast<const Elem*>(a.logits) + (int64_t)b * a.row_stride;
    const int g_lo = p * groups_per_part;
    const int g_hi = min((V + 7) >> 3, g_lo + groups_per_part);
    const uint32_t n_allowed = valid ? allowed_count(a, q) : 0u;
    unsigned long long cand = 0ull;
    if (n_allowed != 0u) {                                     // uniform in the workgroup
        if ((uint64_t)n_allowed * 8u >= (uint64_t)V) cand = exact_scan<DTYPE>(row, nullptr, bits, true, V, g_lo, g_hi);
        else cand = gather_scan<DTYPE>(row, bits, V, g_lo, g_hi, s_ring[threadIdx.x >> 6]);
        cand = block_max_u64(cand, wave_best);
    }
    if (threadIdx.x == 0 && combine_parts(a, b, parts, cand)) write_result(a, b, q, valid, cand);
}

constexpr int kDrawThreads = 256, kDrawWaves = kDrawThreads / 64;      // workgroup of the draw
constexpr int kDrawGroups = 1024;      // workgroups that a draw of a smaller batch is split into: four to a compute unit (1,536: 128 and 256 rows anywhere in
                                       // their texts 15.5 and 23.1 -> 15.8 and 23.8 us, all wide 16.1 and 22.3 -> 17.4 and 24.0; 2,048: 16.7, 23.4, 19.6 and 27.1)
constexpr int kScratchWords = 4096;    // that the step's scratch holds at least
constexpr int kLineWords = 32;         // words of a cache line
constexpr int kDrawPartGroups = 1 << 24;    // groups of a part at most: its offsets and its quads' numbers have 32 bits
// noise_bound is above the noise by at most 0.0861 ln 2 + 0.001 and what -ln(1 - u) exceeds -ln(-ln u) by, which is no more
// than -ln u: from u = 0.9 on by less than 0.168.  With scores of magnitude kTightScore at most, whose sums are rounded
// by less than 0.002 each, a score is never below its bound less kBoundSlack.
constexpr uint32_t kTightWord = 0xE6666800u;    // generator words from here on have u >= 0.9
constexpr float kBoundSlack = 0.2f, kTightScore = 32768.0f;
constexpr int kDrawList = 2048;        // quads that a wavefront lists at once
constexpr int kDrawPieces = 4;         // 16-byte pieces of allowed bits that a lane has in flight
constexpr int kWordGroups = 64 * kDrawPieces * kDrawWaves * 4;     // groups of a part whose allowed bits are read by words of 32 tokens, at most
constexpr uint32_t kDrawDense = 10;    // a state that allows one token in so many or more has every quad drawn (7: the same within 0.5 us; 14: 256 rows 0.9 us
                                       // slower, 128 rows 1.4, 512 rows 4.5 and 1,024 rows 4)

struct DrawShared {
    unsigned long long wave_best[kDrawWaves];
    uint4 cands[kDrawWaves][64];                               // tokens that may win: id, logit, generator word, bound of the score
    uint32_t sums[kDrawWaves];
    uint32_t reached;                                          // order key of the best score any wavefront has reached
};

// The draw from the whole allowed set.  A workgroup takes one part of a row, all parts of the same length.  What a token costs is
// its generator block, made for four neighbouring tokens (a quad) at a time, one quad per lane.
//   A state known to allow one token in kDrawDense or more, a part with an allowed token in half of its quads where
//     nothing is known of the state, and a masked row to be written have every quad drawn, in the order it lies in:
//     one bound for the quad, from its largest logit, allowed or not, and its largest generator word.
//   Else the quads with an allowed token are listed from the bits, 64 and more at a time, and drawn from the list; or the allowed
//     tokens, where a wavefront has no more of them than lanes: each scored at once.
// Where a quad's bound reaches the best score so far its tokens are bounded one by one; those that may win are kept, the
// tightest of them raises the best score by its bound less kBoundSlack, and only what is left at the end (or fills the
// wavefront's 64 places) gets its two logarithms.  The maximum does not depend on the order: candidates are compared as
// (score, lowest id).
//
// Bound by the instructions issued where states allow many tokens: 75 vector instructions per quad, 18 of them 64-bit products (counters,
// 256 rows of 128,256 tokens all in such states: the vector units are busy in 75 % of the cycles), so 256 rows with every
// quad drawn take 15 us of every SIMD; and by some 20 dependent steps, 5 us, where states allow few.  The scheduler
// serves the oldest wavefront first, so that the last one of a SIMD would run alone: a wavefront that draws every quad lowers its
// priority as it gets on.  (Without: 256 rows 22.1 and 26.2 instead of 20.9 and 23.7 us.)  One that works from a list mostly waits, for
// memory and for itself, so it goes first (128, 256 and 512 rows anywhere in their texts 15.5, 23.1 and 34.0 -> 14.2, 21.4 and 32.1 us).
//
// T = 1, bf16, rows anywhere in the texts of 50 signatures / all in states that allow most / all that allow few, replayed, against rows in
// parts of equal length and two queues per wavefront: 128,256 tokens, 1 row 10.2, 10.1 and 5.8 -> 8.4, 8.5 and 5.9 us, 16 rows 10.6, 11.6 and 7.1 ->
// 8.9, 9.3 and 5.4, 64 rows 14.3, 16.1 and 9.1 -> 12.2, 13.1 and 6.9, 128 rows 19.0, 24.2 and 11.2 -> 14.1, 16.1 and 7.0, 256 rows 27.8, 35.1 and 10.8 -> 21.4, 21.6
// and 7.2, 512 rows 43.0, 54.1 and 12.7 -> 32.5, 40.4 and 9.9, 1,024 rows 77.7, 94.5 and 17.1 -> 56.1, 62.0 and 10.7; 9,000 tokens, 256 rows 11.0, 11.1 and 6.2 ->
// 9.1, 9.2 and 5.8, 4,096 rows 34.0, 41.8 and 13.9 -> 29.0, 33.8 and 13.9; 2,000 tokens, 1,024 rows 10.8, 11.2 and 5.4 -> 7.4, 7.4 and 6.0, 4,096 rows 22.9, 27.6 and
// 12.2 -> 17.7, 19.1 and 13.3.  States advanced in place take as long, and tables of which no count is known, 256 rows of 128,256 tokens, 27.4, 34.9
// and 10.9 -> 21.4, 22.0 and 7.3 (every row from the list: 38.5, 43.6 and 10.5); the masked row as well, 256 rows 35.8, 40.1 and 28.3 -> 29.6, 29.6 and 29.9.
//
// Rows shared out over 720 workgroups by what their states allow, each workgroup working the plan out for itself from all states: 128, 256, 512 and
// 1,024 rows anywhere in their texts 15.0, 22.0, 34.4 and 48.7 us, 128 and 256 rows that allow few 7.9 and 8.3.  Not done: the plan reads states that a call
// in place writes, and holds only as long as nobody changes them.
template <int DTYPE, bool WRITE, bool WORDS>
__device__ __forceinline__ unsigned long long draw_part(const MaskArgs& a, SampleParams sp, int b, int p, int groups_per_part, int q,
                                                        uint32_t* s_lists, int list_cap, DrawShared& s)
{
    using Elem = typename ElemOf<DTYPE>::type;
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
    constexpr int kSize = (int)sizeof(Elem);
    constexpr uint32_t NEG_INF = DTYPE == TDFA_F32 ? 0xFF800000u : 0xFF80u;
    constexpr int kWaves = kDrawWaves;
    const int V = a.n_tokens, n_groups = (V + 7) >> 3;
    const int lane = (int)threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const bool valid = q >= 0 && (int64_t)q < a.n_rows;
    if (!WRITE && !valid) return 0ull;                         // no token; (uniform in the workgroup)
    if (sp.off_dev) {                                          // the same word for every thread
        const unsigned long long o = *sp.off_dev;
        sp.off_lo = (uint32_t)o;
        sp.off_hi = (uint32_t)(o >> 32);
    }
    // the workgroup's part of the row: tokens 8 g_lo .. 8 g_lo + n_tok
    const int64_t g_lo = min((int64_t)p * groups_per_part, (int64_t)n_groups);
    const int n_part = (int)min((int64_t)groups_per_part, n_groups - g_lo);
    const int n_tok = (int)max(min((int64_t)n_part * 8, V - g_lo * 8), (int64_t)0);
    const int n_full = n_tok >> 3;
    const uint32_t quad0 = (uint32_t)(g_lo * 2);
    const Elem* row = static_cast<const Elem*>(a.logits) + (int64_t)b * a.row_stride + g_lo * 8;
    Elem* orow = WRITE ? static_cast<Elem*>(a.masked_out) + (int64_t)b * a.row_stride + g_lo * 8 : nullptr;
    const uint8_t* bits = reinterpret_cast<const uint8_t*>(a.allow + (valid ? (int64_t)q * a.row_words : 0)) + g_lo;

    // The allowed bits by wavefronts, each a stretch of its own: a lane reads those of 128 tokens at a time, or of 32 in a part of
    // 4,096 groups or less, so that every lane has some; kDrawPieces such pieces in flight, the first ones requested with the
    // count of the state and used unless every quad is drawn.
    // (WORDS: no part of the launch is longer; 79 vector registers instead of 114, so that a SIMD holds six wavefronts: 16 rows that allow
    // few 6.0 -> 5.5 us, 256 rows anywhere in their texts 24.8 -> 23.1, 2,000 tokens, 4,096 rows that allow few 17.7 -> 13.3.)
    constexpr int kDims = WORDS ? 1 : 4;
    const bool by_word = WORDS || n_part <= kWordGroups;
    const int unit = by_word ? 32 : 128, n_units = (n_tok + unit - 1) / unit, per_wave = (n_units + kWaves - 1) / kWaves;
    const int lo = wave * per_wave, hi = min(n_units, lo + per_wave);
    const __amdgpu_buffer_rsrc_t r_bits = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint8_t*>(bits), 0, (int)min(a.row_words * 4 - g_lo, (int64_t)((n_part + 15) & ~15)), kRawBuffer);
    uint32_t v[kDrawPieces][kDims];
    auto load_pieces = [&](int i0) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < kDrawPieces; ++k) {
#pragma unroll
            for (int d = 0; d < kDims; ++d) v[k][d] = 0u;
            if (i0 + 64 * k >= hi) continue;                   // (uniform: a short part has fewer)
            const int i = i0 + 64 * k + lane;
            if constexpr (!WORDS) {
                if (!by_word) {
                    const u32x4 x = __builtin_amdgcn_raw_buffer_load_b128(r_bits, i < hi ? i * 16 : 0x7FFFFFF0, 0, 0);
                    v[k][0] = x.x, v[k][1] = x.y, v[k][2] = x.z, v[k][3] = x.w;
                    continue;
                }
            }
            v[k][0] = __builtin_amdgcn_raw_buffer_load_b32(r_bits, i < hi ? i * 4 : 0x7FFFFFF0, 0, 0);
        }
    };
    // What lies behind the row's last token leaves the pieces.
    auto trim_pieces = [&](int i0) __attribute__((always_inline)) {
        if (min(i0 + 64 * kDrawPieces, hi) * unit <= n_tok) return;        // (uniform)
#pragma unroll
        for (int k = 0; k < kDrawPieces; ++k) {
            const int left = n_tok - (i0 + 64 * k + lane) * unit;
#pragma unroll
            for (int d = 0; d < kDims; ++d) {
                const uint32_t rem = (uint32_t)min(max(left - 32 * d, 0), 32);
                v[k][d] &= (uint32_t)((1ull << rem) - 1ull);
            }
        }
    };
    uint32_t mine[kDrawPieces];                                // what a lane's pieces hold
    auto count_tokens = [&]() __attribute__((always_inline)) {
        uint32_t n = 0;
#pragma unroll
        for (int k = 0; k < kDrawPieces; ++k) {
            mine[k] = 0;
#pragma unroll
            for (int d = 0; d < kDims; ++d)
                if (d == 0 || !by_word) mine[k] += (uint32_t)__builtin_popcount(v[k][d]);
            n += mine[k];
        }
        return n;
    };
    auto count_quads = [&]() __attribute__((always_inline)) {
        uint32_t n = 0;
#pragma unroll
        for (int k = 0; k < kDrawPieces; ++k) {
            mine[k] = 0;
#pragma unroll
            for (int d = 0; d < kDims; ++d) {
                if (d != 0 && by_word) continue;
                uint32_t x = v[k][d] | v[k][d] >> 1;
                x = (x | x >> 2) & 0x11111111u;
                mine[k] += (uint32_t)__builtin_popcount(x);
            }
            n += mine[k];
        }
        return n;
    };
    const uint32_t n_allowed = WRITE ? kUnknown : allowed_count(a, q);
    const bool counted = !WRITE && n_allowed == kUnknown;
    uint32_t all = 0, total = 0;                               // of the pieces at hand: quads of the lane, of the wavefront
    bool dense = WRITE;
    if (!WRITE && n_allowed == 0u) return 0ull;
    if (!WRITE && n_allowed != kUnknown) dense = n_allowed >= (uint32_t)V / kDrawDense;
    if (!dense) load_pieces(lo);
    // (No count: half of the part's quads, or of the first pieces of a long one.  At 3/4 256 rows anywhere in their texts take 28.4 instead of 25.3 us.)
    if (counted) {
        trim_pieces(lo);
        all = count_quads();
        total = wave_sum_u32(all);
        if (lane == 0) s.sums[wave] = total;
        __syncthreads();
        uint32_t sum = 0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) sum += s.sums[w];
        dense = sum >= (uint32_t)min(n_tok, kWaves * 64 * kDrawPieces * unit) / 8u;
    } else {
        __syncthreads();                                       // (s.reached)
    }

    uint32_t best_key = 0, best_idx = 0xFFFFFFFFu;             // key 0: no candidate yet
    float reached = -__builtin_inff();                         // a score that some token of the workgroup has reached
    auto reach = [&](uint32_t key) {                           // (key 0: nothing scored yet)
        const float r = __uint_as_float((key & 0x80000000u) ? key & 0x7FFFFFFFu : ~key);
        if (key != 0 && r > reached) reached = r;
    };
    auto look = [&]() {
        reach((uint32_t)__builtin_amdgcn_readfirstlane((int)__hip_atomic_load(&s.reached, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)));
    };
    // The largest score a token of the quad may have; NaN if one of its logits is.
    auto quad_bound = [&](const float (&l)[4], const uint32_t (&w)[4]) {
        const float most = __builtin_elementwise_maximum(__builtin_elementwise_maximum(l[0], l[1]), __builtin_elementwise_maximum(l[2], l[3]));
        return __builtin_fmaf(most, sp.inv_t, noise_bound(max(max(w[0], w[1]), max(w[2], w[3]))));
    };
    auto publish = [&](uint32_t key) {
        if (lane == 0) atomicMax(&s.reached, key);               // the other wavefronts prune by it too
        reach(key);
    };
    // The candidates of this wavefront: those that may still win compete.
    uint32_t n_cand = 0;
    uint4* cands = s.cands[wave];
    auto compete = [&]() __attribute__((always_inline)) {
        if (n_cand == 0) return;
        wave_lds_sync();
        look();
        const uint4 c = cands[lane];
        const bool live = (uint32_t)lane < n_cand && !(__uint_as_float(c.w) < reached);
        n_cand = 0;
        wave_lds_sync();
        if (__builtin_amdgcn_ballot_w64(live) == 0) return;
        if (live) {
            const uint32_t lb = (c.y & 0x7FFFFFFFu) > 0x7F800000u ? 0xFF800000u : c.y;       // NaN counts as -inf
            const uint32_t key = key_f32(__float_as_uint(__builtin_fmaf(__uint_as_float(lb), sp.inv_t, gumbel_of(c.z))));
            if (key > best_key || (key == best_key && c.x < best_idx)) {
                best_key = key;
                best_idx = c.x;
            }
        }
        publish(wave_max_u32(best_key));
    };
    // One quad per lane (all lanes active; take: its allowed tokens, 0: none): those that may win become candidates.
    auto settle = [&](uint32_t quad, uint32_t take, const float (&l)[4], const uint32_t (&w)[4]) __attribute__((always_inline)) {
        float bd[4], low = -__builtin_inff();
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            bd[j] = __builtin_fmaf(l[j], sp.inv_t, noise_bound(w[j]));
            if (bd[j] < reached) take &= ~(1u << j);
        }
        if (__builtin_amdgcn_ballot_w64(take != 0) == 0) return;
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if ((take >> j & 1u) && w[j] >= kTightWord && fabsf(bd[j]) <= kTightScore && bd[j] > low) low = bd[j];
        publish(wave_max_u32(key_f32(__float_as_uint(low - kBoundSlack))));
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const bool may = (take >> j & 1u) && !(bd[j] < reached);
            const unsigned long long bal = __builtin_amdgcn_ballot_w64(may);
            if (bal == 0) continue;
            if (n_cand + (uint32_t)__popcll(bal) > 64u) compete();
            if (may)
                cands[n_cand + __builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0u))] =
                    make_uint4((quad0 + quad) * 4u + (uint32_t)j, __float_as_uint(l[j]), w[j], __float_as_uint(bd[j]));
            n_cand += (uint32_t)__popcll(bal);
        }
    };
    auto generate = [&](uint32_t quad, uint32_t (&w)[4]) {
        philox4x32_10(quad0 + quad, (uint32_t)b, sp.off_lo, sp.off_hi, sp.seed_lo, sp.seed_hi, w);
    };
    uint32_t* list = s_lists + wave * list_cap;
    const bool ragged = (n_tok & 3) != 0;
    const __amdgpu_buffer_rsrc_t r_quads =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<Elem*>(row), 0, (n_tok & ~3) * kSize, kRawBuffer);
    // The n quads of the wavefront's list, 64 at a time, their logits requested a batch ahead.
    struct Quad {
        uint32_t e;
        float l[4];
    };
    auto fetch = [&](uint32_t i, uint32_t n, Quad& k) __attribute__((always_inline)) {
        k.e = i < n ? list[i] : 0u;
        const int quad = (int)(k.e >> 4);
        if constexpr (DTYPE == TDFA_F32) {
            const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(r_quads, k.e ? quad * 16 : 0x7FFFFFF0, 0, 0);
            k.l[0] = __uint_as_float(v.x); k.l[1] = __uint_as_float(v.y); k.l[2] = __uint_as_float(v.z); k.l[3] = __uint_as_float(v.w);
        } else {
            const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(r_quads, k.e ? quad * 8 : 0x7FFFFFF0, 0, 0);
            k.l[0] = __uint_as_float(v.x << 16); k.l[1] = __uint_as_float(v.x & 0xFFFF0000u);
            k.l[2] = __uint_as_float(v.y << 16); k.l[3] = __uint_as_float(v.y & 0xFFFF0000u);
        }
        if (ragged && k.e != 0u && quad * 4 + 4 > n_tok) {     // the row's last quad, not whole
#pragma unroll
            for (int j = 0; j < 4; ++j)
                k.l[j] = quad * 4 + j < n_tok ? __uint_as_float(DTYPE == TDFA_F32 ? (uint32_t)row[quad * 4 + j] : (uint32_t)row[quad * 4 + j] << 16) : 0.0f;
        }
    };
    auto draw_list = [&](uint32_t n) __attribute__((always_inline)) {
        wave_lds_sync();
        Quad k, next;
        fetch((uint32_t)lane, n, k);
        for (uint32_t i = 0; i < n; i += 64) {
            fetch(i + 64 + (uint32_t)lane, n, next);
            uint32_t w[4];
            generate(k.e >> 4, w);
            look();
            if (__builtin_amdgcn_ballot_w64(!(quad_bound(k.l, w) < reached)) != 0) settle(k.e >> 4, k.e & 15u, k.l, w);
            k = next;
        }
        wave_lds_sync();
    };

    // The n tokens of the wavefront's list, at most 64: each scored at once.
    auto draw_tokens = [&](uint32_t n) __attribute__((always_inline)) {
        wave_lds_sync();
        const bool has = (uint32_t)lane < n;
        const uint32_t t = has ? list[lane] : 0u;
        uint32_t x = (uint32_t)row[t], w[4];
        if constexpr (DTYPE == TDFA_BF16) x <<= 16;
        generate(t >> 2, w);
        const uint32_t word = (t & 2u) ? (t & 1u ? w[3] : w[2]) : (t & 1u ? w[1] : w[0]);
        if ((x & 0x7FFFFFFFu) > 0x7F800000u) x = 0xFF800000u;                                // NaN counts as -inf
        const uint32_t key = key_f32(__float_as_uint(__builtin_fmaf(__uint_as_float(x), sp.inv_t, gumbel_of(word))));
        const uint32_t idx = quad0 * 4u + t;
        if (has && (key > best_key || (key == best_key && idx < best_idx))) {
            best_key = key;
            best_idx = idx;
        }
        wave_lds_sync();
    };

    if (dense) {
        constexpr int kLoads = DTYPE == TDFA_F32 ? 2 : 1;
        const __amdgpu_buffer_rsrc_t r_x = __builtin_amdgcn_make_buffer_rsrc(const_cast<Elem*>(row), 0, n_full * 8 * kSize, kRawBuffer);
        const __amdgpu_buffer_rsrc_t r_o = __builtin_amdgcn_make_buffer_rsrc(orow, 0, WRITE ? n_full * 8 * kSize : 0, kRawBuffer);
        const __amdgpu_buffer_rsrc_t r_m = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(bits), 0, valid ? n_full : 0, kRawBuffer);
        struct Chunk {                                         // 64 groups: two quads per lane, and their allowed bits
            u32x4 x[kLoads];
            uint32_t m[kLoads];
        };
        // bf16: a lane takes a group; fp32: quad `lane` of either half, so that a load covers a whole kilobyte
        auto load = [&](int g, Chunk& c) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < kLoads; ++i) {
                c.x[i] = __builtin_amdgcn_raw_buffer_load_b128(r_x, lane * 16 + g * 8 * kSize + i * 1024, 0, kReadOnce);
                c.m[i] = __builtin_amdgcn_raw_buffer_load_b8(r_m, (DTYPE == TDFA_F32 ? lane >> 1 : lane) + g + i * 32, 0, 0);
            }
            __builtin_amdgcn_sched_barrier(0);                 // (the loads return in the order they are used in; an offset of its own per
                                                               // lane: the range check wraps where the scalar offset lies past the end)
        };
        auto draw_chunk = [&](int g, const Chunk& c) __attribute__((always_inline)) {
            float l[2][4];
            uint32_t w[2][4], quad[2], ok[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                if constexpr (DTYPE == TDFA_F32) {
                    const u32x4 x = c.x[h];
                    l[h][0] = __uint_as_float(x.x); l[h][1] = __uint_as_float(x.y); l[h][2] = __uint_as_float(x.z); l[h][3] = __uint_as_float(x.w);
                    quad[h] = 2u * (uint32_t)g + 64u * (uint32_t)h + (uint32_t)lane;
                    ok[h] = c.m[h] >> (4 * (lane & 1)) & 15u;
                } else {
                    const uint32_t x0 = h ? c.x[0].z : c.x[0].x, x1 = h ? c.x[0].w : c.x[0].y;
                    l[h][0] = __uint_as_float(x0 << 16); l[h][1] = __uint_as_float(x0 & 0xFFFF0000u);
                    l[h][2] = __uint_as_float(x1 << 16); l[h][3] = __uint_as_float(x1 & 0xFFFF0000u);
                    quad[h] = 2u * (uint32_t)(g + lane) + (uint32_t)h;
                    ok[h] = c.m[0] >> (4 * h) & 15u;
                }
            }
            if constexpr (WRITE) {
                uint32_t o[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const uint32_t x = DTYPE == TDFA_F32 ? __float_as_uint(l[i >> 2][i & 3]) : __float_as_uint(l[i >> 2][i & 3]) >> 16;
                    o[i] = ok[i >> 2] >> (i & 3) & 1u ? x : NEG_INF;
                }
                if constexpr (DTYPE == TDFA_F32) {
                    __builtin_amdgcn_raw_buffer_store_b128(u32x4{o[0], o[1], o[2], o[3]}, r_o, lane * 16 + g * 32, 0, kReadOnce);
                    __builtin_amdgcn_raw_buffer_store_b128(u32x4{o[4], o[5], o[6], o[7]}, r_o, lane * 16 + g * 32 + 1024, 0, kReadOnce);
                } else {
                    __builtin_amdgcn_raw_buffer_store_b128(u32x4{o[0] | o[1] << 16, o[2] | o[3] << 16, o[4] | o[5] << 16, o[6] | o[7] << 16},
                                                           r_o, lane * 16 + g * 16, 0, kReadOnce);
                }
                if (__builtin_amdgcn_ballot_w64((ok[0] | ok[1]) != 0) == 0) return;
            }
            generate(quad[0], w[0]);
            generate(quad[1], w[1]);
            look();
            const float top0 = quad_bound(l[0], w[0]), top1 = quad_bound(l[1], w[1]);
            if (__builtin_amdgcn_ballot_w64(!(top0 < reached) | !(top1 < reached)) == 0) return;
#pragma unroll 1
            for (int h = 0; h < 2; ++h) {
                if (__builtin_amdgcn_ballot_w64(!((h ? top1 : top0) < reached)) == 0) continue;
                float lh[4];
                uint32_t wh[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    lh[j] = h ? l[1][j] : l[0][j];
                    wh[j] = h ? w[1][j] : w[0][j];
                }
                settle(h ? quad[1] : quad[0], h ? ok[1] : ok[0], lh, wh);
            }
        };
        constexpr int step = 64 * kWaves;
        int g = 64 * wave;
        constexpr int kDepth = 4 / kLoads;
        Chunk c[kDepth];
#pragma unroll
        for (int d = 0; d < kDepth; ++d) load(g + d * step, c[d]);
        const int g_2 = n_full >> 2, g_1 = n_full >> 1, g_0 = n_full - g_2;
        __builtin_amdgcn_s_setprio(3);                         // (so that the wavefronts of a SIMD end together)
        for (; g < n_full; g += kDepth * step) {               // (a chunk past the end is all zeros: nothing allowed)
            if (g >= g_0) __builtin_amdgcn_s_setprio(0);
            else if (g >= g_1) __builtin_amdgcn_s_setprio(1);
            else if (g >= g_2) __builtin_amdgcn_s_setprio(2);
#pragma unroll
            for (int d = 0; d < kDepth; ++d) {
                if (g + d * step < n_full) draw_chunk(g + d * step, c[d]);
                load(g + (kDepth + d) * step, c[d]);
            }
        }
        if (n_tok > 8 * n_full && wave == 0) {                 // the row's last, partial group
            const uint32_t m = valid ? (uint32_t)bits[n_full] & ((1u << (n_tok - 8 * n_full)) - 1u) : 0u;
            Elem x = (Elem)0;
            const int t = 8 * n_full + lane;
            if (WRITE && t < n_tok) x = row[t];
            if (lane < 8 && (m >> lane & 1u)) list[__builtin_popcount(m & ((1u << lane) - 1u))] = (uint32_t)t;
            draw_tokens((uint32_t)__builtin_popcount(m));
            if (WRITE && t < n_tok) orow[t] = m >> lane & 1u ? x : (Elem)NEG_INF;
        }
    } else {
        // What is allowed is listed: single tokens if a wavefront's pieces hold no more of them than it has lanes, else quads.
        __builtin_amdgcn_s_setprio(3);
        for (int i0 = lo; i0 < hi; i0 += 64 * kDrawPieces) {
            if (i0 != lo) load_pieces(i0);
            if (i0 != lo || !counted) {
                trim_pieces(i0);
                all = count_quads();
                total = wave_sum_u32(all);
            }
            if (total == 0) continue;
            bool single = false;
            if (total <= 64u) {
                const uint32_t tokens = count_tokens();
                single = wave_sum_u32(tokens) <= 64u;
                if (single) all = tokens;
                else all = count_quads();
            }
            // all pieces at once, or one after the other where the list would not hold them
            const int rounds = total <= (uint32_t)list_cap ? 1 : kDrawPieces;
            for (int r = 0; r < rounds; ++r) {
                uint32_t here = all;
                if (rounds != 1) here = r == 0 ? mine[0] : r == 1 ? mine[1] : r == 2 ? mine[2] : mine[3];
                const uint32_t incl = wave_prefix_u32(here);
                const uint32_t n = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
                uint32_t at = incl - here;
                auto list_pieces = [&](auto tokens) __attribute__((always_inline)) {
                    constexpr bool kTokens = decltype(tokens)::value;
#pragma unroll
                    for (int k = 0; k < kDrawPieces; ++k) {
                        if ((rounds != 1 && k != r) || __builtin_amdgcn_ballot_w64(mine[k] != 0) == 0) continue;
                        const uint32_t first = (uint32_t)((i0 + 64 * k + lane) * (kTokens ? unit : unit >> 2));
#pragma unroll
                        for (int d = 0; d < kDims; ++d) {
                            if (d != 0 && by_word) continue;
                            uint32_t rest = v[k][d];
                            while (rest) {
                                const uint32_t bit = (uint32_t)__builtin_ctz(rest), nib = bit & 28u;
                                if constexpr (kTokens) {
                                    list[at++] = first + 32u * (uint32_t)d + bit;
                                    rest &= rest - 1u;
                                } else {
                                    list[at++] = (first + 8u * (uint32_t)d + (nib >> 2)) << 4 | (rest >> nib & 15u);
                                    rest &= ~(15u << nib);
                                }
                            }
                        }
                    }
                };
                if (single) list_pieces(std::true_type{});
                else list_pieces(std::false_type{});
                if (single) draw_tokens(n);
                else draw_list(n);
            }
        }
    }
    compete();
    const unsigned long long cand = best_key ? ((unsigned long long)best_key << 32) | (0xFFFFFFFFu - best_idx) : 0ull;
    return block_max_u64(cand, s.wave_best);
}

template <int DTYPE, bool WRITE, bool WORDS>
__global__ void __launch_bounds__(kDrawThreads, WORDS || WRITE ? 6 : 4)
draw_step_kernel(MaskArgs a, SampleParams sp, int parts, int groups_per_part, int list_cap, int spread)
{
    extern __shared__ uint32_t s_lists[];                      // [kDrawWaves][list_cap]
    __shared__ DrawShared s;
    if (threadIdx.x == 0) s.reached = 0;
    const int b = blockIdx.x / parts, q = __builtin_amdgcn_readfirstlane(a.states[b]);
    unsigned long long cand = draw_part<DTYPE, WRITE, WORDS>(a, sp, b, blockIdx.x % parts, groups_per_part, q, s_lists, list_cap, s);
    if (threadIdx.x != 0) return;
    // (read again, the kernel's first argument: kept all along, its pointers spill, and with them the compiler reserves private
    // memory that every launch next to other kernels pays for, 0.3 to 0.5 us)
    const __attribute__((address_space(4))) MaskArgs* args = (const __attribute__((address_space(4))) MaskArgs*)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(args));
    const MaskArgs& z = *(const MaskArgs*)args;
    if (combine_parts(z, b * spread, parts, cand)) write_result(z, b, q, q >= 0 && (int64_t)q < z.n_rows, cand);
}

// Runs of speculated tokens (Section 5.3): one lane per sequence follows its k tokens through the
// table and records every state on the way.  The lookups of a sequence depend on one another;
// the sequences are independent.
__global__ void __launch_bounds__(64)
advance_tokens_kernel(MaskArgs a, int32_t batch, int32_t k, const int32_t* __restrict__ states,
                      const int32_t* __restrict__ tokens, int32_t* __restrict__ history, int32_t* __restrict__ n_valid)
{
    const int b = blockIdx.x * 64 + threadIdx.x;
    if (b >= batch) return;
    int32_t s = states[b];
    if (s < 0 || (int64_t)s >= a.n_rows) s = TDFA_DEAD;
    int32_t* h = history + (int64_t)b * (k + 1);
    const int32_t* run = tokens + (int64_t)b * k;
    h[0] = s;
    int32_t ok = 0;
    for (int32_t i = 0; i < k; ++i) {
        const int32_t t = run[i];
        s = (s != TDFA_DEAD && t >= 0 && t < a.n_tokens) ? table_entry(a, s, t) : TDFA_DEAD;
        h[i + 1] = s;
        if (s != TDFA_DEAD && ok == i) ok = i + 1;
    }
    if (n_valid) n_valid[b] = ok;
}

// best[0 .. n) <- 0, count[0 .. n) <- 0
__global__ void __launch_bounds__(256)
clear_scratch_kernel(unsigned long long* __restrict__ best, unsigned int* __restrict__ count, int32_t n)
{
    const int i = (int)(blockIdx.x * 256 + threadIdx.x);
    if (i < n) {
        best[i] = 0ull;
        count[i] = 0u;
    }
}

// Launch shape of the packed step kernel: a row per workgroup of 1024 threads when the batch fills the
// chip, else rows split over `parts` workgroups of 256, each part a whole number of 32-bit words
// of allowed bits.
void gather_shape(const MaskArgs& a, int* parts_out, int* threads_out, int* gpp_out)
{
    const int n_groups = (a.n_tokens + 7) >> 3;
    int parts = 1, threads = 1024;
    if (a.batch < 192 || n_groups < 4096) {
        threads = 256;
        parts = (2048 + a.batch - 1) / a.batch;
        const int max_parts = (n_groups + 1023) / 1024;
        if (parts > max_parts) parts = max_parts;
    }
    if (parts < 1) parts = 1;
    int gpp = ((n_groups + parts - 1) / parts + 3) / 4 * 4;
    if (gpp < 4) gpp = 4;
    *parts_out = parts;
    *threads_out = threads;
    *gpp_out = gpp;
}

}  // namespace

namespace {
constexpr int kPieceGroups = 4096;     // groups of a row that a workgroup takes where rows are split
constexpr int kBitsGroups = kMaxBitRowBytes - 8192;     // groups of a workgroup whose allowed bits are sure to fit its LDS, beside the loads in flight
constexpr int kSmallBatch = 16;        // rows from which on that is the better split (1 to 8 rows: 4.8 to 6.0 us in 16 parts of 256 threads, 5.9 to 6.4 us so)

// Rows that one workgroup of 512 threads streams with four groups per lane and buffer, not one of 1,024 with two: as much in
// flight, and the workgroup starts, matches the stack and ends sooner.  Push-down step, 128,256 tokens, replayed from a graph, 192, 257,
// 512, 768, 1,024 and 2,048 rows anywhere in their texts 13.2, 15.1, 20.9, 34.0, 38.6 and 70.1 -> 13.3, 13.6, 20.2, 28.0, 40.4 and 65.3 us,
// 1,024 rows that allow little 23.5 -> 17.5 (against the form with 1,024 threads held to 80 scalar registers, which only 896 to 1,088
// rows of 100,000 tokens and more anywhere in their texts would prefer, by 2 to 9 %; this form held to 80: 2 to 4 % slower); greedy,
// where some compute units hold two rows, 300 and 383 rows 17.6 and 18.0 -> 16.4 and 16.3 (256 rows 9.8 -> 10.0, 257 rows 12.3 -> 13.7,
// 512 rows 18.3 -> 18.6, 1,024 rows 32.8 -> 33.6, so not).
bool takes_deep(const MaskArgs& a, bool pda)
{
    if (a.dtype == TDFA_F32 || a.masked_out) return false;
    const int n_groups = (a.n_tokens + 7) >> 3;
    if (n_groups > kBitsGroups) return false;
    return pda ? n_groups >= kPieceGroups && a.batch > 128 : n_groups >= 2 * kPieceGroups && a.delta && a.batch >= 288 && a.batch < kGatherRows;
}

// Launch shape of the streaming kernels: `parts` workgroups of `threads` threads to a row.
//
// Rows whose bits would not fit the LDS of a few large workgroups are cut as small batches are: in parts of 256 threads, or
// one of 1,024 (without the bits the push-down step makes a row per sequence first, and the others stream rows they could skip).
//
// What it weighs: a compute unit streams at what one unit gets from memory (a 256 KB row in 6.5 us), so few rows are split;
// every workgroup costs its launch and its own look at state and bits, and workgroups of a row meet at the end; a workgroup
// of 512 threads starts and ends a microsecond sooner than one of 1,024, which has more loads in flight.  The times are of steps
// replayed from a graph, rows anywhere in their texts where nothing else is said (a call of its own costs the host 8 us).
void stream_shape(const MaskArgs& a, bool pda, bool alone, int* parts_out, int* threads_out, int* gpp_out)
{
    const int n_groups = (a.n_tokens + 7) >> 3;
    const int64_t batch = a.batch, pieces = (n_groups + kPieceGroups - 1) / kPieceGroups;
    const bool plain = a.dtype != TDFA_F32 && !a.masked_out;             // 16-bit logits that are only read
    int64_t parts = 1;
    int threads = 1024;
    if (plain && !pda && n_groups > 1024 && n_groups < kPieceGroups) {
        // a short row, 8,193 to 32,767 tokens.  32,000 tokens, 16, 64, 256 and 1,024 rows: in parts of 256 threads 5.2, 6.0, 8.2
        // and 12.9 us; so 4.9, 5.9, 6.4 and 11.9 us (9,000 tokens 5.1, -, 6.3 and 9.4 -> 4.4, -, 5.1 and 8.8)
        threads = 512;
    } else if (plain && !pda && n_groups >= kPieceGroups && n_groups < 2 * kPieceGroups && (a.delta ? batch >= 320 || (batch > 128 && batch < 192 && n_groups <= (batch <= 170 ? 7000 : 6000)) : batch >= 768)) {
        // rows of middle length, enough to fill the chip.  50,000 tokens, 384, 512 and 1,024 rows: 10.5, 11.6 and 20.1 -> 9.5, 10.8 and
        // 16.4 us (200 rows that allow most 7.5 -> 8.1, so not; 384 rows of a packed table 10.1 -> 10.5; 1,024 rows of 128,256 tokens
        // that allow most 42.4 -> 43.6).  129 to 191 rows, if they are no longer than what the pieces below take as fast: 40,000
        // tokens, 160 and 191 rows 7.9 and 7.6 -> 7.3 and 7.2 us, 50,000 tokens, 160 rows 8.6 -> 8.4 (all that allow little 7.4 -> 5.4), but 191
        // rows 7.7 -> 8.4, 60,000 tokens, 160 and 191 rows 8.6 and 7.8 -> 9.2 and 9.0
        threads = 512;
    } else if (plain && n_groups >= kPieceGroups && batch >= kSmallBatch &&
               (pda ? batch <= 128 && batch * (n_groups - kPieceGroups) >= 300000 && n_groups <= 2 * kBitsGroups :
                      batch < 192 && (batch <= 170 || pieces <= 4) && (a.delta || pieces > 2) && n_groups <= 512 / batch * kBitsGroups)) {
        // as many pieces as the chip holds at once.  128,256 tokens, 16, 64 and 128 rows: in parts of 256 threads 7.5, 10.7 and 13.4
        // us, in one piece 8.3, 9.3 and 9.1; so 7.2, 7.8 and 8.7 us (16 rows that allow little 6.9 -> 6.0).  In fewer than three pieces one
        // workgroup of 1,024 threads is better: 191 rows 14.0 in parts of 256 threads, 11.6 in two pieces, 10.2 us so; rows too long
        // for that stay as they were (250,000 tokens, 180 rows: 15.6, in two pieces 20.3), as do the shorter ones of packed tables
        // (50,000 tokens, 64 rows: 6.9, in two pieces 7.4).  Rows of two pieces gain from 64 rows on (60,000 tokens, 128 rows 8.5 -> 7.7;
        // 33,000 tokens, 32 rows 5.8 -> 6.0).
        // The push-down step matches its stack in every workgroup: two large ones at most, where what lies beyond the first piece of
        // each row is work enough for them.  128,256 tokens, 48, 64 and 128 rows 11.6, 13.2 and 18.3 -> 10.7, 11.0 and 11.7 us, 24 rows 9.9 ->
        // 10.2; 80,000 tokens, 64 and 128 rows 10.8 and 12.3 -> 10.6 and 10.9, 48 rows 9.5 -> 10.3; 65,600 tokens, 96 rows 11.1 -> 10.9, 48 rows
        // 9.4 -> 10.5; 45,000 tokens, 32 and 128 rows 8.6 and 10.1 -> 9.6 and 10.5; 33,000 tokens, 16 and 64 rows 8.1 and 8.8 -> 9.4 and 9.7.
        parts = pda ? 2 : batch <= 170 ? std::min<int64_t>(pieces, 512 / batch) : 1;
        threads = pda || batch > 170 ? 1024 : 512;
    } else if (!plain && pieces > 3 &&
               (a.dtype != TDFA_F32 ? batch >= kSmallBatch && batch <= 64 :
                a.masked_out ? (alone && mask_step_wants_scratch(a)) || (batch >= 48 && batch * pieces <= 256) : batch >= 48 && batch * pieces <= 512)) {
        // Long rows that are written as well, or of fp32: larger workgroups keep the memory busy with fewer of them, while all of them
        // are in flight: one to a compute unit where rows are written, two where they are only read.  fp32, in parts of 256 threads
        // and so: 128,256 tokens, 64, 96 and 128 rows 11.5, 13.8 and 15.1 -> 9.9, 13.2 and 13.5 us, 160 and 191 rows 16.0 and 18.1 -> 19.8
        // and 21.1; 250,000 tokens, 64 rows 18.3 -> 14.0, 96 rows 19.1 -> 21.1 (32 rows of 128,256 8.9 -> 9.2).  With the
        // penalised row 64 rows 15.5 -> 14.1, 65 rows 16.7 -> 18.1, 100,000 tokens, 65 and 160 rows 13.4 and 23.3 -> 15.6 and 25.1.  From
        // 256 rows on, which otherwise are one workgroup each, need no scratch and leave compute units idle at the end: 256, 320, 512
        // and 1,024 rows 48.6, 82.4, 109 and 207 -> 46.9, 63.7, 101 and 192 us, where the scratch is this step's alone.  bf16 with the row 16 and 64 rows 7.2 and 11.0 -> 6.3 and 8.5 us (100
        // rows 13.7 -> 14.0, so not).
        parts = pieces;
    } else if (takes_deep(a, pda)) {
        threads = 512;
    } else if (batch < 192 || n_groups < kPieceGroups) {
        threads = 256;
        parts = std::min<int64_t>((2048 + batch - 1) / batch, (n_groups + 1023) / 1024);
    }
    if (parts < 1) parts = 1;
    int gpp = (int)((n_groups + parts - 1) / parts);
    if (gpp < 1) gpp = 1;
    gpp = (gpp + 15) & ~15;                    // the bits of 16 groups are read at once
    *parts_out = (int)parts;
    *threads_out = threads;
    *gpp_out = gpp;
}
}  // namespace

namespace {
// A packed table takes the step kernel of the dense ones on 16-bit logits without a penalised row (512 rows of a
// constraint's states at 128,256 tokens: 29.8 us by the gathering scan alone, whose wide rows are compared element
// by element, 15.6 us by the step kernel); fp32 logits, where that scan reads wide rows as fast and sparse ones faster
// (1,024 rows: 67 against 87 us), and penalised rows stay with it, as do rows beyond the step kernel's 32-bit offsets.
bool packed_takes_gather(const MaskArgs& a)
{
    return !a.delta && a.targets && !a.masked_out && (a.dtype == TDFA_F32 || a.n_tokens > (1 << 27));
}
}  // namespace

bool mask_step_uses_scratch(const MaskArgs& a)
{
    if (a.batch <= 0) return false;
    int parts, threads, gpp;
    if (packed_takes_gather(a)) gather_shape(a, &parts, &threads, &gpp);
    else stream_shape(a, false, false, &parts, &threads, &gpp);
    return parts > 1;
}

// Written rows of fp32, as many as there are compute units or more.
bool mask_step_wants_scratch(const MaskArgs& a)
{
    return a.dtype == TDFA_F32 && a.masked_out && a.batch >= 256;
}

int launch_clear_scratch(unsigned long long* best, unsigned int* count, int32_t n, hipStream_t stream)
{
    if (n <= 0) return TDFA_OK;
    clear_scratch_kernel<<<(unsigned)((n + 255) / 256), 256, 0, stream>>>(best, count, n);
    TDFA_HIP(hipGetLastError());
    return TDFA_OK;
}

namespace {
// The launch of the 16-bit kernel that keeps a stretch's bits in LDS: shape, LDS bytes, and whether they fit.
struct BitsInLds {
    int parts, threads, gpp, unroll, stretch;
    size_t lds;
    bool fits;
};
BitsInLds bits_in_lds(const MaskArgs& a, bool pda, bool alone)
{
    BitsInLds r;
    stream_shape(a, pda, alone, &r.parts, &r.threads, &r.gpp);
    // groups per load batch: one for the few small workgroups of a small batch, four where half as many wavefronts stream a row
    r.unroll = takes_deep(a, pda) ? 4 : r.threads < 1024 && (int64_t)a.batch * r.parts <= 384 ? 1 : 2;
    // A stretch of the row per wavefront, in whole 16-group pieces; the bits of the stretches fit
    // in LDS for any vocabulary of a few hundred thousand tokens, else every stretch is streamed.
    const int n_waves = r.threads / 64;
    r.stretch = ((r.gpp + n_waves - 1) / n_waves + 15) & ~15;
    r.lds = (size_t)n_waves * ((size_t)r.stretch + 4 * 64 * (size_t)r.unroll);
    r.fits = !a.masked_out && r.lds <= (size_t)kMaxBitRowBytes;
    return r;
}

// Lets the kernels that keep the bits in LDS take more than the default 64 KB, once per device.
int raise_lds_limit(size_t lds)
{
    if (lds <= (size_t)kPlainLdsBytes) return TDFA_OK;
    static bool raised[64] = {};
    int dev = 0;
    TDFA_HIP(hipGetDevice(&dev));
    if (dev >= 0 && dev < 64 && !raised[dev]) {
        for (const void* k : {reinterpret_cast<const void*>(mask_step_bf16_kernel<false, 1, true>),
                              reinterpret_cast<const void*>(mask_step_bf16_kernel<false, 2, true>),
                              reinterpret_cast<const void*>(mask_step_bf16_many_kernel<1>),
                              reinterpret_cast<const void*>(mask_step_bf16_many_kernel<2>),
                              reinterpret_cast<const void*>(mask_step_bf16_kernel<false, 1, true, 2, true>),
                              reinterpret_cast<const void*>(mask_step_bf16_kernel<false, 2, true, 2, true>),
                              reinterpret_cast<const void*>(mask_step_bf16_kernel<false, 4, true>),
                              reinterpret_cast<const void*>(mask_step_bf16_kernel<false, 4, true, 2, true>)})
            TDFA_HIP(hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, kMaxBitRowBytes));
        raised[dev] = true;
    }
    return TDFA_OK;
}
}  // namespace

bool mask_step_takes_pda(const PdaMaskArgs& a)
{
    return a.batch > 0 && a.dtype != TDFA_F32 && !a.delta && !a.targets && a.n_tokens <= (1 << 27) && bits_in_lds(a, true, false).fits;
}

int launch_mask_step(const MaskArgs& a, hipStream_t stream, bool alone)
{
    if (a.batch <= 0) return TDFA_OK;
    if (packed_takes_gather(a)) {
        // a packed table: the scan that reads only the groups with allowed tokens
        int g_parts, g_threads, g_gpp;
        gather_shape(a, &g_parts, &g_threads, &g_gpp);
        if ((int64_t)a.batch * g_parts > 0x7FFFFFFFll) return fail(TDFA_E_UNSUPPORTED, "batch too large for one launch");
        const dim3 grid((unsigned)(a.batch * g_parts));
        if (a.dtype == TDFA_F32) packed_step_kernel<TDFA_F32><<<grid, (unsigned)g_threads, 0, stream>>>(a, g_parts, g_gpp);
        else packed_step_kernel<TDFA_BF16><<<grid, (unsigned)g_threads, 0, stream>>>(a, g_parts, g_gpp);
        TDFA_HIP(hipGetLastError());
        return TDFA_OK;
    }
    const BitsInLds sh = bits_in_lds(a, false, alone);
    const int parts = sh.parts, threads = sh.threads, gpp = sh.gpp, unroll = sh.unroll, stretch = sh.stretch;
    const size_t lds = sh.lds;
    const bool skip = sh.fits;
    if ((int64_t)a.batch * parts > 0x7FFFFFFFll) return fail(TDFA_E_UNSUPPORTED, "batch too large for one launch");
    // the 16-bit kernel addresses a row through 32-bit byte offsets
    const dim3 grid((unsigned)(a.batch * parts));
    const unsigned kThreads = (unsigned)threads;
    if (a.dtype != TDFA_F32 && a.n_tokens > (1 << 27)) {
        if (a.delta || !a.targets) return fail(TDFA_E_UNSUPPORTED, "more than 2^27 tokens in a 16-bit row");
        mask_step_exact_kernel<TDFA_BF16><<<grid, kThreads, 0, stream>>>(a, parts, gpp);     // (packed rows have no such limit)
        TDFA_HIP(hipGetLastError());
        return TDFA_OK;
    }
    const int n_waves = threads / 64;
    if (skip && a.dtype != TDFA_F32) {
        const int rc = raise_lds_limit(lds);
        if (rc != TDFA_OK) return rc;
    }
    if (a.dtype == TDFA_F32 && !a.masked_out && (size_t)n_waves * (size_t)stretch <= (size_t)kPlainLdsBytes)
        mask_step_f32_kernel<<<grid, kThreads, (size_t)n_waves * (size_t)stretch, stream>>>(a, parts, gpp, stretch);
    else if (a.dtype == TDFA_F32 && a.masked_out && a.n_tokens <= (1 << 26))      // (32-bit byte offsets)
        mask_write_f32_kernel<<<grid, kThreads, 0, stream>>>(a, parts, gpp);
    else if (a.dtype == TDFA_F32)
        mask_step_exact_kernel<TDFA_F32><<<grid, kThreads, 0, stream>>>(a, parts, gpp);
    else if (a.masked_out)
        mask_step_bf16_kernel<true, 2, false><<<grid, kThreads, 0, stream>>>(a, parts, gpp, stretch);
    else if (skip && (a.batch >= kGatherRows || !a.delta)) {
        if (unroll == 1) mask_step_bf16_many_kernel<1><<<grid, kThreads, lds, stream>>>(a, parts, gpp, stretch);
        else mask_step_bf16_many_kernel<2><<<grid, kThreads, lds, stream>>>(a, parts, gpp, stretch);
    } else if (skip && unroll == 4)
        mask_step_bf16_kernel<false, 4, true><<<grid, kThreads, lds, stream>>>(a, parts, gpp, stretch);
    else if (skip && unroll == 1)
        mask_step_bf16_kernel<false, 1, true><<<grid, kThreads, lds, stream>>>(a, parts, gpp, stretch);
    else if (skip)
        mask_step_bf16_kernel<false, 2, true><<<grid, kThreads, lds, stream>>>(a, parts, gpp, stretch);
    else if (unroll == 1)
        mask_step_bf16_kernel<false, 1, false><<<grid, kThreads, 0, stream>>>(a, parts, gpp, stretch);
    else
        mask_step_bf16_kernel<false, 2, false><<<grid, kThreads, 0, stream>>>(a, parts, gpp, stretch);
    TDFA_HIP(hipGetLastError());
    return TDFA_OK;
}

int launch_pda_mask_step(const PdaMaskArgs& a, hipStream_t stream)
{
    if (a.batch <= 0) return TDFA_OK;
    if (!mask_step_takes_pda(a)) return fail(TDFA_E_UNSUPPORTED, "this step wants one row of allowed bits per sequence");
    const BitsInLds sh = bits_in_lds(a, true, false);
    if ((int64_t)a.batch * sh.parts > 0x7FFFFFFFll) return fail(TDFA_E_UNSUPPORTED, "batch too large for one launch");
    const int rc = raise_lds_limit(sh.lds);
    if (rc != TDFA_OK) return rc;
    const dim3 grid((unsigned)(a.batch * sh.parts));
    const unsigned threads = (unsigned)sh.threads;
    if (sh.unroll == 4) mask_step_bf16_kernel<false, 4, true, 2, true><<<grid, threads, sh.lds, stream>>>(a, sh.parts, sh.gpp, sh.stretch);
    else if (sh.unroll == 1) mask_step_bf16_kernel<false, 1, true, 2, true><<<grid, threads, sh.lds, stream>>>(a, sh.parts, sh.gpp, sh.stretch);
    else mask_step_bf16_kernel<false, 2, true, 2, true><<<grid, threads, sh.lds, stream>>>(a, sh.parts, sh.gpp, sh.stretch);
    TDFA_HIP(hipGetLastError());
    return TDFA_OK;
}

int launch_sample_step(const MaskArgs& a, float inv_t, int32_t top_k, uint64_t seed, uint64_t offset, const uint64_t* offset_dev,
                       hipStream_t stream)
{
    if (a.batch <= 0) return TDFA_OK;
    SampleParams sp;
    sp.inv_t = inv_t;
    sp.seed_lo = (uint32_t)seed;
    sp.seed_hi = (uint32_t)(seed >> 32);
    sp.off_lo = (uint32_t)offset;
    sp.off_hi = (uint32_t)(offset >> 32);
    sp.off_dev = reinterpret_cast<const unsigned long long*>(offset_dev);
    if (top_k > 0) {
        // a workgroup per sequence: as many threads as hold the row in registers, 1,024 at most
        const unsigned t = a.n_tokens > kRowGroups * 8 * 256 ? 1024u : 256u;
        const bool resident = a.n_tokens <= (int32_t)t * kRowGroups * 8;
        auto launch = [&](auto dtype, auto write) {
            constexpr int kType = decltype(dtype)::value;
            constexpr bool kWrite = decltype(write)::value;
            // (with the penalised row written, keys and stores together would not fit the registers: the row is read twice)
            if (resident && !kWrite) topk_step_kernel<kType, kWrite, !kWrite><<<(unsigned)a.batch, t, 0, stream>>>(a, sp, top_k);
            else topk_step_kernel<kType, kWrite, false><<<(unsigned)a.batch, t, 0, stream>>>(a, sp, top_k);
        };
        using F32 = std::integral_constant<int, TDFA_F32>;
        using Bf16 = std::integral_constant<int, TDFA_BF16>;
        if (a.dtype == TDFA_F32 && a.masked_out) launch(F32{}, std::true_type{});
        else if (a.dtype == TDFA_F32) launch(F32{}, std::false_type{});
        else if (a.masked_out) launch(Bf16{}, std::true_type{});
        else launch(Bf16{}, std::false_type{});
        TDFA_HIP(hipGetLastError());
        return TDFA_OK;
    }
    // Workgroups of 256 threads, kDrawGroups of them (rows in parts of at least 1,024 groups), and up to twice as many where parts whose
    // bits are read by words take that: anywhere in the texts / all wide / all few, 384 rows of 128,256 tokens 31.5, 30.7 and 7.9 -> 25.7,
    // 30.1 and 8.1 us, 512 rows 38.3, 37.7 and 8.7 -> 32.6, 41.0 and 9.9, 256 of 256,000 37.2, 38.5 and 8.6 -> 34.1, 42.0 and 9.8.  Not for rows
    // that are not cut otherwise: 768 rows of 128,256 45.8, 53.4 and 9.4 -> 45.1, 56.9 and 12.6, 1,024 rows of 64,000 32.8, 38.1 and 7.9 -> 35.6, 44.1 and 10.2.
    const int n_groups = (a.n_tokens + 7) >> 3;
    const int64_t batch = a.batch;
    int64_t parts = std::min<int64_t>(kDrawGroups / batch, (n_groups + 1023) / 1024);
    const int64_t by_words = ((int64_t)n_groups + kWordGroups - 1) / kWordGroups;
    if (parts > 1 && !a.masked_out && batch * by_words <= 2 * kDrawGroups) parts = std::max(parts, by_words);
    parts = std::max<int64_t>({parts, ((int64_t)n_groups + kDrawPartGroups - 1) / kDrawPartGroups, 1});
    const int gpp = (int)(((n_groups + parts - 1) / parts + 63) & ~63);
    const int64_t grid = batch * parts;
    // A wavefront's list holds half of its quads where their bits are read by words (more of them, or of the whole part's where no count is
    // known, are rarely listed; if so, a piece of 512 at a time), so that a compute unit has room for six workgroups: 2,000 tokens, 4,096 rows
    // that allow few 26 -> 13 us.
    const bool words = gpp <= kWordGroups && !a.masked_out;
    int cap = kDrawList;
    if (words) {
        const int quads = (gpp / 4 + kDrawWaves - 1) / kDrawWaves * 8;
        cap = std::max(quads <= 512 ? quads : std::max(512, quads / 2), 64);
    }
    const size_t lds = (size_t)cap * kDrawWaves * 4;
    // The words that the parts of a row meet through lie as far apart as there is room for, up to a cache line: atomics on one line wait
    // for each other, some 10 ns each (16 rows that allow few, 16 parts each, 8.2 -> 6.3 us).
    int spread = 1;
    while (spread < kLineWords && 2 * spread * batch <= kScratchWords) spread *= 2;
    if (grid > 0x7FFFFFFFll) return fail(TDFA_E_UNSUPPORTED, "batch too large for one launch");
    const dim3 blocks((unsigned)grid);
    auto launch = [&](auto write, auto by_word) {
        constexpr bool kWrite = decltype(write)::value, kWords = decltype(by_word)::value;
        if (a.dtype == TDFA_F32) draw_step_kernel<TDFA_F32, kWrite, kWords><<<blocks, kDrawThreads, lds, stream>>>(a, sp, (int)parts, gpp, cap, spread);
        else draw_step_kernel<TDFA_BF16, kWrite, kWords><<<blocks, kDrawThreads, lds, stream>>>(a, sp, (int)parts, gpp, cap, spread);
    };
    if (a.masked_out) launch(std::true_type{}, std::false_type{});
    else if (words) launch(std::false_type{}, std::true_type{});
    else launch(std::false_type{}, std::false_type{});
    TDFA_HIP(hipGetLastError());
    return TDFA_OK;
}

int launch_sample_noise(int32_t batch, int32_t n_tokens, uint64_t seed, uint64_t offset, float* out, hipStream_t stream)
{
    if (batch <= 0 || n_tokens <= 0) return TDFA_OK;
    const int32_t quads_per_row = (n_tokens + 3) / 4;
    const int64_t total = (int64_t)batch * quads_per_row;
    if ((total + 255) / 256 > 0x7FFFFFFFll) return fail(TDFA_E_UNSUPPORTED, "batch * n_tokens too large for one launch");
    SampleParams sp;
    sp.inv_t = 1.0f;
    sp.off_dev = nullptr;
    sp.seed_lo = (uint32_t)seed;
    sp.seed_hi = (uint32_t)(seed >> 32);
    sp.off_lo = (uint32_t)offset;
    sp.off_hi = (uint32_t)(offset >> 32);
    sample_noise_kernel<<<(unsigned)((total + 255) / 256), 256, 0, stream>>>(sp, n_tokens, total, quads_per_row, out);
    TDFA_HIP(hipGetLastError());
    return TDFA_OK;
}

int launch_advance_tokens(const MaskArgs& table, int32_t batch, int32_t k, const int32_t* states, const int32_t* tokens,
                          int32_t* history, int32_t* n_valid, hipStream_t stream)
{
    if (batch <= 0) return TDFA_OK;
    advance_tokens_kernel<<<(batch + 63) / 64, 64, 0, stream>>>(table, batch, k, states, tokens, history, n_valid);
    TDFA_HIP(hipGetLastError());
    return TDFA_OK;
}

}  // namespace tdfa
