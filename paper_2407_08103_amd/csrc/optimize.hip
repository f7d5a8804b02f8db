// Token-level optimisation of a compiled table (Appendix C.2, the fourth of the compile operations it
// times, applied to the composed automaton).  The paper does not name the optimisation; the reading taken is the
// classical one for a deterministic automaton: keep the states that some token sequence reaches
// from a start state and from which a final state can be reached, and merge the states that accept
// the same token sequences (Moore's partition refinement).  A set-up call.
//
// A row of a token table has many entries but few distinct targets (the character states one
// token away).  One pass over the table therefore reduces every row to its distinct targets r,
// each with the weight F(q, r) = sum of w(t) over the tokens t with delta_T[q][t] = r (w: a mixed,
// odd 64-bit number per token); all the rounds then run on these short lists:
//
//   reach      rounds from the start states: the targets of a marked row are marked
//   co-reach   rounds over the rows not yet known to reach a final state: a row with a target
//              that does becomes one
//   refine     a class is named by its smallest state.  A round gives every kept row the
//              signature sum of g(class of r) * F(q, r) (= the sum over its tokens of
//              w(t) * g(class of the target), in any order), rows with the same (class,
//              signature) find each other in a hash table on the device and take their smallest
//              row as the new name.  The host only reads the number of classes of each round.
//              Equal rows always get equal signatures, so a signature never splits wrongly; when
//              no class splits any more every row that joined another is compared with it entry
//              by entry over the dense table, so a signature never decides that rows are equal.
//   compact    the first row of each class, its entries renamed, is a row of the new table
//
// A row with more distinct targets than the workgroup's table in LDS holds (a table that is not
// sparse in this sense), or a failed comparison, sends the whole call down the dense path: the same
// steps with the host driving rounds of kernels that stream the table's rows.
//
// Two entries in three of an ordinary table are DEAD, and most of them lie in long runs (states that allow a few
// hundred tokens).  The first pass over the rows (lists) reads every entry and holds the table's allowed bits against them; if
// they agree, the passes after it (comparison, renaming) read the bits, an entry's 32nd part, and then only the entries
// behind a set bit.  If they do not (bits or entries that a caller has edited, which the result follows), every pass reads every entry.
#include <algorithm>
#include <cstring>
#include <new>
#include <vector>

#include "tdfa_internal.h"

namespace tdfa {
namespace {

constexpr int kThreads = 256;

// A wavefront takes a row in spans of 64 * CHUNKS tokens: 2 * CHUNKS words of bits, a word in each of the first lanes, that
// say which entries are read.  BITS: the row's allowed bits; otherwise every token of the row counts as one to read.
template <bool BITS, int CHUNKS>
__device__ __forceinline__ uint32_t span_word(const uint32_t* bits, int64_t w0, int lane, int32_t n_tokens)
{
    const int64_t wi = w0 + lane;
    const int64_t rem = (int64_t)n_tokens - 32 * wi;
    if (lane >= 2 * CHUNKS || rem <= 0) return 0u;
    const uint32_t w = BITS ? bits[wi] : 0xFFFFFFFFu;
    return rem >= 32 ? w : w & ((1u << rem) - 1u);
}

// the bits of the span's chunk c: an execution mask
__device__ __forceinline__ unsigned long long span_mask(uint32_t w, int c)
{
    return ((unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)w, 2 * c + 1) << 32) | (uint32_t)__builtin_amdgcn_readlane((int)w, 2 * c);
}

// the entries of the span's tokens whose bit is set, a token per lane and chunk, all loads in flight; DEAD for the others
template <int CHUNKS>
__device__ __forceinline__ void span_load(const int32_t* row, int64_t w0, int lane, uint32_t w, int32_t (&v)[CHUNKS])
{
#pragma unroll
    for (int c = 0; c < CHUNKS; ++c) {
        v[c] = TDFA_DEAD;
        if (__builtin_amdgcn_inverse_ballot_w64(span_mask(w, c))) v[c] = __builtin_nontemporal_load(row + 32 * w0 + 64 * c + lane);
    }
}

// rows[i] is scanned: every live entry marks its target in `mark` (bytes; equal stores may race).
__global__ void __launch_bounds__(kThreads)
mark_targets_kernel(const int32_t* __restrict__ delta, int32_t n_tokens, const int32_t* __restrict__ rows,
                    uint8_t* __restrict__ mark)
{
    const int32_t* row = delta + (size_t)rows[blockIdx.y] * n_tokens;
    for (int t = blockIdx.x * kThreads + threadIdx.x; t < n_tokens; t += gridDim.x * kThreads) {
        const int32_t v = row[t];
        if (v >= 0 && !mark[v]) mark[v] = 1;
    }
}

// rows[i] becomes good (can reach a final state) if one of its entries leads to a good state.
__global__ void __launch_bounds__(kThreads)
reach_final_kernel(const int32_t* __restrict__ delta, int32_t n_tokens, const int32_t* __restrict__ rows,
                   const uint8_t* __restrict__ kept, uint8_t* __restrict__ good, int32_t* __restrict__ changed)
{
    const int32_t q = rows[blockIdx.y];
    const int32_t* row = delta + (size_t)q * n_tokens;
    bool hit = false;
    for (int t = blockIdx.x * kThreads + threadIdx.x; t < n_tokens && !hit; t += gridDim.x * kThreads) {
        const int32_t v = row[t];
        hit = v >= 0 && kept[v] && good[v];
    }
    if (hit && !good[q]) {
        good[q] = 1;
        *changed = 1;
    }
}

__device__ __forceinline__ unsigned long long mix64(unsigned long long x)
{
    x ^= x >> 30;
    x *= 0xBF58476D1CE4E5B9ull;
    x ^= x >> 27;
    x *= 0x94D049BB133111EBull;
    x ^= x >> 31;
    return x;
}

// hash[i] of rows[i]: sum over the tokens of mix(token, class of the entry's target); cls is -1
// for a state that is not kept, and a DEAD entry counts like one.
__global__ void __launch_bounds__(kThreads)
row_hash_kernel(const int32_t* __restrict__ delta, int32_t n_tokens, const int32_t* __restrict__ rows,
                const int32_t* __restrict__ cls, unsigned long long seed, unsigned long long* __restrict__ hash)
{
    __shared__ unsigned long long part[kThreads / 64];
    const int32_t* row = delta + (size_t)rows[blockIdx.x] * n_tokens;
    unsigned long long h = 0;
    for (int t = threadIdx.x; t < n_tokens; t += kThreads) {
        const int32_t v = row[t];
        const int32_t c = v >= 0 ? cls[v] : -1;
        if (c >= 0) h += mix64(seed + (unsigned long long)t * 0x9E3779B97F4A7C15ull + (unsigned long long)(unsigned)c);
    }
    for (int off = 32; off > 0; off >>= 1) h += __shfl_xor(h, off, 64);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = h;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < kThreads / 64; ++w) h += part[w];
        hash[blockIdx.x] = h;
    }
}

// rows[i] and first_of[i] (the first row of its class) must agree, entry by entry, on the class of the target: the
// dense path's comparison of n pairs, and the sparse path's (BITS where the table's allowed bits agree with its entries).
//
// Workgroups take pairs in turn, with the classes in LDS where they fit (LDS_CLS), and a wavefront has the entries of
// kVerifyChunks * 64 tokens of both rows in flight.  Pieces of rows and not whole ones, because there are about as many pairs
// as workgroups.  1,142 pairs of 128,256 tokens: 317 us with every entry read and the classes in memory, 180 us by the bits
// with a workgroup per pair, 135 us so.
constexpr int kVerifyThreads = 512;
constexpr int kVerifyChunks = 8;
constexpr int kPieceWords = 128;       // words of bits of a piece of a row (4,096 tokens): what a wavefront takes at a time
constexpr size_t kMapLdsBytes = 64 * 1024;

template <bool BITS, bool LDS_CLS>
__global__ void __launch_bounds__(kVerifyThreads)
verify_classes_kernel(const int32_t* __restrict__ delta, const uint32_t* __restrict__ allow, int32_t n_tokens, int64_t row_words, int64_t n,
                      int32_t n_old, const int32_t* __restrict__ rows, const int32_t* __restrict__ first_of, const int32_t* __restrict__ cls,
                      int32_t* __restrict__ mismatch)
{
    extern __shared__ int32_t s_cls[];
    if constexpr (LDS_CLS) {
        for (int i = threadIdx.x; i < n_old; i += kVerifyThreads) s_cls[i] = cls[i];
        __syncthreads();
    }
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    constexpr int kSpan = 2 * kVerifyChunks;                       // in words of bits
    bool bad = false;
    // a wavefront takes pieces of pairs in turn
    const int64_t per_row = (row_words + kPieceWords - 1) / kPieceWords, n_waves = (int64_t)gridDim.x * (kVerifyThreads / 64);
    for (int64_t j = (int64_t)blockIdx.x * (kVerifyThreads / 64) + wave; j < n * per_row; j += n_waves) {
        const int64_t i = j / per_row, lo = (j - i * per_row) * kPieceWords, hi = min(row_words, lo + kPieceWords);
        const int32_t *a = delta + (size_t)rows[i] * n_tokens, *b = delta + (size_t)first_of[i] * n_tokens;
        const uint32_t *a_bits = allow + (size_t)rows[i] * row_words, *b_bits = allow + (size_t)first_of[i] * row_words;
        auto either = [&](int64_t w0) {
            const uint32_t w = span_word<BITS, kVerifyChunks>(a_bits, w0, lane, n_tokens);
            return BITS ? w | span_word<BITS, kVerifyChunks>(b_bits, w0, lane, n_tokens) : w;
        };
        uint32_t w_next = either(lo);
        for (int64_t w0 = lo; w0 < hi; w0 += kSpan) {
            const uint32_t w = w_next;
            w_next = either(w0 + kSpan);
            if (__builtin_amdgcn_ballot_w64(w != 0) == 0) continue;
            int32_t x[kVerifyChunks], y[kVerifyChunks];
            span_load<kVerifyChunks>(a, w0, lane, w, x);
            span_load<kVerifyChunks>(b, w0, lane, w, y);
#pragma unroll
            for (int u = 0; u < kVerifyChunks; ++u) {
                const int32_t cx = x[u] >= 0 ? (LDS_CLS ? s_cls[x[u]] : cls[x[u]]) : -1;
                const int32_t cy = y[u] >= 0 ? (LDS_CLS ? s_cls[y[u]] : cls[y[u]]) : -1;
                bad |= cx != cy;
            }
        }
    }
    if (bad) *mismatch = 1;
}

// New row c = row first_row[c] of the old table with its entries renamed by `map` (-1 for a state
// that was dropped); allowed words from the new entries.
//
// A workgroup of a grid that fills the chip takes rows in turn and keeps the map in LDS where it fits (LDS_MAP; 16,384
// states: 64 KB): looked up in memory, the 64 lanes' scattered entries cost a compute unit more than two cycles each.
// A wavefront renames kRenameChunks * 64 tokens at a time, so that as many loads are in flight, and writes their allowed
// words side by side.
//
// Wavefronts take pieces of rows (kPieceWords), so that none waits for another's row, and have the next span's entries
// in flight while they rename one.  Bound by the memory: 4,245 rows of 128,256 tokens are 2.2 GB written and, without the
// bits, as much read: 890 us; by the bits, which leave about 40 % of the entries to be read, 750 us (writing rows of which
// a third are copied takes 565 us on this card, only writing them 395; without the non-temporal stores 800 us).
constexpr int kRenameThreads = 512;
constexpr int kRenameChunks = 8;

template <bool BITS, bool LDS_MAP>
__global__ void __launch_bounds__(kRenameThreads)
compact_rows_kernel(const int32_t* __restrict__ delta, const uint32_t* __restrict__ allow, int32_t n_tokens, int64_t row_words, int64_t n_new,
                    int32_t n_old, const int32_t* __restrict__ first_row, const int32_t* __restrict__ map,
                    int32_t* __restrict__ out_delta, uint32_t* __restrict__ out_allow)
{
    extern __shared__ int32_t s_map[];
    if constexpr (LDS_MAP) {
        for (int i = threadIdx.x; i < n_old; i += kRenameThreads) s_map[i] = map[i];
        __syncthreads();
    }
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    constexpr int kSpan = 2 * kRenameChunks;                       // in words of bits
    // a wavefront takes pieces of rows in turn
    const int64_t per_row = (row_words + kPieceWords - 1) / kPieceWords, n_waves = (int64_t)gridDim.x * (kRenameThreads / 64);
    for (int64_t i = (int64_t)blockIdx.x * (kRenameThreads / 64) + wave; i < n_new * per_row; i += n_waves) {
        const int64_t c = i / per_row, lo = (i - c * per_row) * kPieceWords, hi = min(row_words, lo + kPieceWords);
        const int32_t* row = delta + (size_t)first_row[c] * n_tokens;
        const uint32_t* bits = allow + (size_t)first_row[c] * row_words;
        int32_t* out = out_delta + (size_t)c * n_tokens;
        // the next span's entries are requested before this one's are renamed, and the bits of the one after it
        int32_t v_next[kRenameChunks];
        span_load<kRenameChunks>(row, lo, lane, span_word<BITS, kRenameChunks>(bits, lo, lane, n_tokens), v_next);
        uint32_t w_next = span_word<BITS, kRenameChunks>(bits, lo + kSpan, lane, n_tokens);
        for (int64_t w0 = lo; w0 < hi; w0 += kSpan) {
            int32_t v[kRenameChunks];
#pragma unroll
            for (int u = 0; u < kRenameChunks; ++u) v[u] = v_next[u];
            if (w0 + kSpan < hi) {
                span_load<kRenameChunks>(row, w0 + kSpan, lane, w_next, v_next);
                w_next = span_word<BITS, kRenameChunks>(bits, w0 + 2 * kSpan, lane, n_tokens);
            }
            uint32_t word = 0;                                     // lanes 2 u, 2 u + 1: the allowed words of chunk u
#pragma unroll
            for (int u = 0; u < kRenameChunks; ++u) {
                const int64_t t = 32 * w0 + u * 64 + lane;
                if (v[u] >= 0) v[u] = LDS_MAP ? s_map[v[u]] : map[v[u]];
                else v[u] = TDFA_DEAD;
                if (t < n_tokens) __builtin_nontemporal_store(v[u], out + t);
                const uint64_t m = __builtin_amdgcn_ballot_w64(v[u] != TDFA_DEAD);
                if (lane == 2 * u) word = (uint32_t)m;
                if (lane == 2 * u + 1) word = (uint32_t)(m >> 32);
            }
            const int64_t wi = w0 + lane;
            if (lane < kSpan && wi < row_words) out_allow[(size_t)c * row_words + wi] = word;
        }
    }
}

struct DeviceBuffers {
    int32_t* rows = nullptr;
    int32_t* aux = nullptr;       // first_of
    int32_t* cls = nullptr;
    uint8_t* mark = nullptr;
    uint8_t* good = nullptr;
    unsigned long long* hash = nullptr;
    int32_t* flag = nullptr;
};

// Device memory of one call, given back to the library's cache when it ends.
struct Arena {
    std::vector<DeviceBlock> blocks;
    template <class T>
    int get(T** p, size_t n)
    {
        try {
            blocks.emplace_back();
        } catch (const std::bad_alloc&) {
            return fail(TDFA_E_OOM, "host allocation failed");
        }
        const int rc = block_alloc(&blocks.back(), std::max<size_t>(n, 1) * sizeof(T));
        *p = static_cast<T*>(blocks.back().ptr);
        return rc;
    }
    ~Arena()
    {
        int dev = 0;
        (void)hipGetDevice(&dev);
        for (const DeviceBlock& b : blocks) block_free(b, dev);
    }
};
#define TDFA_GET(expr)                                                                            \
    do {                                                                                          \
        const int rc_ = (expr);                                                                   \
        if (rc_ != TDFA_OK) return rc_;                                                           \
    } while (0)

constexpr size_t kMaxGridY = 65535;

unsigned grid_x(int32_t n_tokens) { return (unsigned)std::max(1, std::min(64, (n_tokens + kThreads * 8 - 1) / (kThreads * 8))); }


// ---------------------------------------------------------------------------------------------
// The sparse path: rows as lists of distinct targets.

constexpr int kListThreads = 1024;      // workgroup of the pass that builds a row's list
constexpr int kSlots = 4096;           // its table of targets in LDS (open addressing, 48 KB)
constexpr int kMaxTargets = 3072;      // more distinct targets in one row: the dense path
constexpr int kListChunks = 8;         // 64 entries each that a wavefront has in flight

// w(t), odd: three products of 32 bits, each half of the one before folded into the next.
__device__ __forceinline__ unsigned long long token_weight(unsigned long long seed, int t)
{
    const unsigned long long p = (unsigned long long)((uint32_t)t ^ (uint32_t)seed) * 0x9E3779B1u + seed;
    const unsigned long long r = (unsigned long long)((uint32_t)p ^ (uint32_t)(p >> 32)) * 0x85EBCA77u + p;
    const unsigned long long u = (unsigned long long)((uint32_t)r ^ (uint32_t)(r >> 32)) * 0xC2B2AE3Du;
    return (((unsigned long long)((uint32_t)(u >> 32) ^ (uint32_t)r) << 32) | ((uint32_t)u ^ (uint32_t)(r >> 32))) | 1ull;
}

__global__ void __launch_bounds__(kThreads)
token_weights_kernel(unsigned long long seed, int32_t n_tokens, unsigned long long* __restrict__ weight)
{
    const int32_t t = blockIdx.x * kThreads + threadIdx.x;
    if (t < n_tokens) weight[t] = token_weight(seed, t);
}

__device__ __forceinline__ void add_target(int32_t* key, unsigned long long* sum, int* n_used, int32_t v, unsigned long long w)
{
    unsigned slot = ((unsigned)v * 0x9E3779B1u) >> 20;
    // (mostly the target is there already, in its first place)
    if (key[slot] == v) {
        atomicAdd(&sum[slot], w);
        return;
    }
    for (int probe = 0; probe < kSlots; ++probe, slot = (slot + 1) & (kSlots - 1)) {
        int32_t k = key[slot];
        if (k == -1) {
            k = atomicCAS(&key[slot], -1, v);
            if (k == -1) {
                atomicAdd(n_used, 1);
                k = v;
            }
        }
        if (k == v) {
            atomicAdd(&sum[slot], w);
            return;
        }
    }
    atomicAdd(n_used, kSlots);          // the table is full of other targets: counts as too many
}

// Row blockIdx.x: its distinct targets and their weights, appended to (e_target, e_weight) at a
// position taken from `counter` (which keeps counting past e_cap, so that a second attempt knows the
// size).  *overflow is set when a row has more than kMaxTargets targets, *differ where a bit of `allow` and its entry
// disagree: the bits may be the caller's, and its entries may have changed since, so they lead no pass before this one
// has held them against every entry.
//
// Bound by instructions and by the waits of each update (the target's place in LDS, then the atomic): 5,387 rows of 128,256
// tokens took 690 us with each entry's weight made in place (a dozen instructions), 660 us with the weights from memory (1 MB,
// in every L2) and the bits compared; led by the bits it would take 525 us, and believe them.  More than 80 scalar registers
// leave room for one workgroup on a compute unit (870 us); 16 loads in flight take 900 us, 4 with the next span's requested
// beforehand 745 us, 8 of those 670 us, workgroups of 512 threads 710 us.
__global__ void __launch_bounds__(kListThreads) __attribute__((amdgpu_num_sgpr(80)))
row_targets_kernel(const int32_t* __restrict__ delta, const uint32_t* __restrict__ allow, int32_t n_tokens, int64_t row_words,
                   const unsigned long long* __restrict__ weight, unsigned long long e_cap,
                   unsigned long long* __restrict__ counter, unsigned long long* __restrict__ row_begin,
                   int32_t* __restrict__ row_n, int32_t* __restrict__ e_target, unsigned long long* __restrict__ e_weight,
                   int32_t* overflow, int32_t* differ)
{
    __shared__ int32_t key[kSlots];
    __shared__ unsigned long long sum[kSlots];
    __shared__ int n_used, n_out, stop;
    __shared__ unsigned long long base;
    for (int i = threadIdx.x; i < kSlots; i += kListThreads) {
        key[i] = -1;
        sum[i] = 0;
    }
    if (threadIdx.x == 0) {
        n_used = 0;
        n_out = 0;
        stop = *(volatile int32_t*)overflow;        // another row has too many: the lists will not be used
    }
    __syncthreads();
    if (stop) return;
    const int32_t* row = delta + (size_t)blockIdx.x * n_tokens;
    const uint32_t* bits = allow + (size_t)blockIdx.x * row_words;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    constexpr int kSpan = 2 * kListChunks, kStep = kListThreads / 64 * kSpan;            // in words of bits
    int32_t last = TDFA_DEAD;
    unsigned long long acc = 0;
    bool wrong = false;                             // (the same in every lane)
    for (int64_t w0 = (int64_t)wave * kSpan; w0 < row_words; w0 += kStep) {
        int32_t v[kListChunks];
        span_load<kListChunks>(row, w0, lane, span_word<false, kListChunks>(bits, w0, lane, n_tokens), v);
        const uint32_t w = span_word<true, kListChunks>(bits, w0, lane, n_tokens);
        unsigned long long any = 0;
#pragma unroll
        for (int u = 0; u < kListChunks; ++u) {
            const unsigned long long edges = __builtin_amdgcn_ballot_w64(v[u] >= 0);
            any |= edges;
            wrong |= edges != span_mask(w, u);
        }
        if (any == 0) continue;
        unsigned long long tw[kListChunks];
#pragma unroll
        for (int u = 0; u < kListChunks; ++u)
            if (v[u] >= 0) tw[u] = weight[32 * w0 + 64 * u + lane];
#pragma unroll
        for (int u = 0; u < kListChunks; ++u) {
            if (v[u] < 0) continue;
            if (v[u] != last) {             // runs of one target (a state that mostly loops) cost one update
                if (last >= 0) add_target(key, sum, &n_used, last, acc);
                last = v[u];
                acc = 0;
            }
            acc += tw[u];
        }
        if (*(volatile int*)&n_used > kMaxTargets) break;
    }
    if (wrong && lane == 0) *differ = 1;
    if (last >= 0) add_target(key, sum, &n_used, last, acc);
    __syncthreads();
    const int n = n_used;
    if (n > kMaxTargets) {
        if (threadIdx.x == 0) *overflow = 1;
        return;
    }
    if (threadIdx.x == 0) {
        base = atomicAdd(counter, (unsigned long long)n);
        row_begin[blockIdx.x] = base;
        row_n[blockIdx.x] = n;
    }
    __syncthreads();
    if (base + (unsigned long long)n > e_cap) return;
    for (int i = threadIdx.x; i < kSlots; i += kListThreads)
        if (key[i] != -1) {
            const int p = atomicAdd(&n_out, 1);
            e_target[base + p] = key[i];
            e_weight[base + p] = sum[i];
        }
}

// The kernels below give a wavefront to a row's list.
constexpr int kRowsPerBlock = kThreads / 64;

struct Lists {
    const unsigned long long* row_begin;
    const int32_t* row_n;
    const int32_t* e_target;
    const unsigned long long* e_weight;
    int32_t n_rows;
};

// Marks are bytes that only ever rise from 0 to 1, so a wavefront need not wait for a round of all rows to end: it looks
// at its row several times in a launch, and what another wavefront has marked meanwhile counts.  (Loads and stores of the
// marks at device scope; the wavefronts wait for nothing, and launches that have marked nothing end the rounds.)  A look is
// a trip to the L2 or beyond, a third of a microsecond; a launch per round took 3 us and its gap as much.  5,387 rows, both
// searches: 96 launches of a round each, 12 between two looks of the host: 270 us of kernels and 380 us of gaps; 32 sweeps 13
// launches, 192 sweeps 5 launches and 120 us of kernels.
//
// A row that is never marked takes all the sweeps of a launch, though, and those of the search for final states each read
// its list; and where the rows outnumber the wavefronts in flight, waiting ones hold the places of those they wait for.  So
// the sweeps of a launch fall with the trips a row's list takes, and beyond kSearchRows rows, where the host looks every
// kSearchLaunches launches, with the rows; what is spent between two looks stays near that of twelve plain rounds.
// 20,000 rows of 1,000 targets that reach no final state, the whole call: 2.0 ms with plain rounds, 14.4 with 192 sweeps for all,
// 2.3 so; 16,000 rows, 40 % of them traps of
// 150 targets: 1.2, 3.2 and 1.4 ms; 12,000 rows in a chain of random order: 1,190, 620 and 510 ms.  With a look only behind both searches
// and the refinement, whose rounds take two launches and not four (the same calls 1.2, 0.7 and 490 ms), 5,387 rows of 128,256 tokens
// are minimised in 1.9 ms (2.1 before), 7,300 of 10,001 in 1.25 (1.65) and a few hundred of 2,000 in 0.37 (0.69).
constexpr int kSweeps = 192;
constexpr int kSearchRows = 8192, kSearchLaunches = 12;

struct SearchShape {
    int launches, sweeps;
};
SearchShape search_shape(int32_t n_rows)
{
    if (n_rows <= kSearchRows) return {1, kSweeps};
    return {kSearchLaunches, std::max<int>(1, (int)((int64_t)kSweeps * kSearchRows / n_rows / kSearchLaunches))};
}

__device__ __forceinline__ bool marked(const uint8_t* mark, int32_t q)
{
    return __hip_atomic_load(mark + q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0;
}

__device__ __forceinline__ void set_mark(uint8_t* mark, int32_t q)
{
    __hip_atomic_store(mark + q, (uint8_t)1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// A launch says in *changed whether it marked anything; one whose predecessor did not (*before, NULL for the first) has nothing to do.
__global__ void __launch_bounds__(kThreads)
list_reach_kernel(Lists g, int sweeps, uint8_t* mark, uint8_t* done, const int32_t* before, int32_t* changed)
{
    if (before && *before == 0) return;
    const int32_t q = blockIdx.x * kRowsPerBlock + __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    if (q >= g.n_rows || done[q]) return;
    const int lane = threadIdx.x & 63;
    int sweep = 0;
    while (sweep < sweeps && !marked(mark, q)) ++sweep;
    if (sweep == sweeps) return;
    if (lane == 0) done[q] = 1;
    const int32_t* e = g.e_target + g.row_begin[q];
    for (int i = lane; i < g.row_n[q]; i += 64)
        if (!marked(mark, e[i])) {
            set_mark(mark, e[i]);
            *changed = 1;
        }
}

__global__ void __launch_bounds__(kThreads)
list_good_start_kernel(int32_t n_rows, const uint8_t* __restrict__ mark, const uint8_t* __restrict__ accept, uint8_t* __restrict__ good)
{
    const int32_t q = blockIdx.x * kThreads + threadIdx.x;
    if (q < n_rows) good[q] = mark[q] && accept[q];
}

__global__ void __launch_bounds__(kThreads)
list_reach_final_kernel(Lists g, int sweeps, const uint8_t* mark, uint8_t* good, const int32_t* before, int32_t* changed)
{
    if (before && *before == 0) return;
    const int32_t q = blockIdx.x * kRowsPerBlock + __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    if (q >= g.n_rows || !mark[q] || good[q]) return;
    const int lane = threadIdx.x & 63;
    const int32_t* e = g.e_target + g.row_begin[q];
    const int32_t n = g.row_n[q];
    if (n == 0) return;
    const int most = max(1, sweeps / ((n + 63) >> 6));
    for (int sweep = 0; sweep < most; ++sweep) {
        bool hit = false;
        // (every target of a marked row is marked)
        for (int i = lane; i < n; i += 64) hit |= marked(good, e[i]);
        if (__builtin_amdgcn_ballot_w64(hit) == 0) continue;
        if (lane == 0) {
            set_mark(good, q);
            *changed = 1;
        }
        return;
    }
}

// What the searches and the refinement begin with: no row looked at, nothing changed, two empty hash tables.
struct HashTable {
    unsigned long long* key;            // 0: free
    int32_t* min;
};
__global__ void __launch_bounds__(kThreads)
list_init_kernel(int32_t n_rows, uint8_t* __restrict__ done, uint32_t* __restrict__ slot_of, int32_t* __restrict__ flags, int n_flags,
                 HashTable a, HashTable b, uint32_t ht_size)
{
    const size_t i = (size_t)blockIdx.x * kThreads + threadIdx.x;
    if (i < (size_t)n_rows) {
        done[i] = 0;
        slot_of[i] = 0;
    }
    if (i < (size_t)n_flags) flags[i] = 0;
    if (i < ht_size) {
        a.key[i] = b.key[i] = 0ull;
        a.min[i] = b.min[i] = 0x7FFFFFFF;
    }
}

// A round of the refinement, first half: the key of each kept row, which is its class and the signature of its targets'
// classes, mixed (never 0; in the first round, which also tells the kept rows, its final flag), and the slot of the table that rows
// with this key meet in, where they leave their smallest row.  In the early rounds thousands of rows share a key: the rows of
// a workgroup go to the table as one per key.
//
// Nothing is done once a round has split no class (counts[0] is the number of classes of this round, counts[-1] that of the
// one before; `round` counts from 0): rounds are launched ahead of the host's look.
constexpr int kKeyThreads = 1024, kKeyRows = kKeyThreads / 64;

__device__ __forceinline__ bool no_class_split(const int32_t* counts, int round) { return round >= 2 && counts[-1] == counts[-2]; }

__global__ void __launch_bounds__(kKeyThreads)
list_keys_kernel(Lists g, int round, const int32_t* __restrict__ counts, const uint8_t* __restrict__ mark, const uint8_t* __restrict__ good,
                 const uint8_t* __restrict__ accept, int32_t* __restrict__ cls, unsigned long long seed, HashTable ht, uint32_t ht_mask,
                 uint32_t* __restrict__ slot_of)
{
    __shared__ unsigned long long s_key[kKeyRows];
    if (no_class_split(counts, round)) return;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int32_t q0 = blockIdx.x * kKeyRows, q = q0 + wave;
    unsigned long long key = 0;                                    // 0: the row is not kept
    if (q < g.n_rows) {
        if (round == 0) {
            const bool kept = mark[q] && good[q];
            if (kept) key = mix64(seed + (accept[q] ? 1 : 2)) | 1ull;
            if (lane == 0) cls[q] = kept ? 0 : -1;
        } else if (cls[q] >= 0) {
            const unsigned long long b = g.row_begin[q];
            unsigned long long h = 0;
            for (int i = lane; i < g.row_n[q]; i += 64) {
                const int32_t c = cls[g.e_target[b + i]];
                if (c >= 0) h += mix64(seed ^ (unsigned long long)(unsigned)c) * g.e_weight[b + i];
            }
            for (int off = 32; off > 0; off >>= 1) h += __shfl_xor(h, off, 64);
            key = mix64(h ^ mix64(seed + 0x632BE59BD9B4E019ull + (unsigned long long)(unsigned)cls[q])) | 1ull;
        }
    }
    if (lane == 0) s_key[wave] = key;
    __syncthreads();
    if (wave != 0) return;
    const unsigned long long k = lane < kKeyRows ? s_key[lane] : 0ull;
    int first = lane;                                              // the first row of the workgroup with this key
    for (int i = kKeyRows - 1; i >= 0; --i)
        if (s_key[i] == k && i < lane) first = i;
    uint32_t slot = 0;
    if (k != 0ull && first == lane) {
        slot = (uint32_t)(k >> 20) & ht_mask;
        for (uint32_t probe = 0; probe <= ht_mask; ++probe, slot = (slot + 1) & ht_mask) {
            // (a look first: most rows need not change the slot)
            unsigned long long was = __hip_atomic_load(&ht.key[slot], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (was == 0ull) was = atomicCAS(&ht.key[slot], 0ull, k);
            if (was == 0ull || was == k) {
                if (__hip_atomic_load(&ht.min[slot], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) > q0 + lane) atomicMin(&ht.min[slot], q0 + lane);
                break;
            }
        }
    }
    slot = (uint32_t)__shfl((int)slot, first, 64);
    if (k != 0ull) slot_of[q0 + lane] = slot;
}

// Second half: a class is named by the smallest row that met there; the table of the round before is emptied for the next.
__global__ void __launch_bounds__(kThreads)
list_assign_kernel(int32_t n_rows, int round, const int32_t* __restrict__ cls, const uint32_t* __restrict__ slot_of, const int32_t* __restrict__ ht_min,
                   HashTable other, uint32_t ht_size, int32_t* __restrict__ cls_out, int32_t* counts)
{
    const uint32_t i = blockIdx.x * kThreads + threadIdx.x;
    if (no_class_split(counts, round)) {                           // (the two arrays of classes are the same by now)
        if (i == 0) counts[0] = counts[-1];
        return;
    }
    if (i < ht_size) {
        other.key[i] = 0ull;
        other.min[i] = 0x7FFFFFFF;
    }
    bool first = false;
    if (i < (uint32_t)n_rows) {
        const int32_t c = cls[i] < 0 ? -1 : ht_min[slot_of[i]];
        cls_out[i] = c;
        first = c == (int32_t)i;
    }
    const uint64_t m = __builtin_amdgcn_ballot_w64(first);
    if ((threadIdx.x & 63) == 0 && m != 0) atomicAdd(&counts[0], __builtin_popcountll(m));
}

// The comparison of n pairs of rows (allow: the table's bits, or NULL where only the entries count).
int launch_verify(const int32_t* delta, const uint32_t* allow, int32_t n_tokens, int64_t row_words, int64_t n, int32_t n_old,
                  const int32_t* rows, const int32_t* first_of, const int32_t* cls, int32_t* mismatch, hipStream_t s)
{
    const int64_t pieces = n * ((row_words + kPieceWords - 1) / kPieceWords);
    const unsigned grid = (unsigned)std::min<int64_t>((pieces + kVerifyThreads / 64 - 1) / (kVerifyThreads / 64), 256 * 4);
    const size_t lds = (size_t)n_old * 4;
    auto launch = [&](auto kernel, size_t bytes) {
        kernel<<<grid, kVerifyThreads, bytes, s>>>(delta, allow, n_tokens, row_words, n, n_old, rows, first_of, cls, mismatch);
    };
    if (lds <= kMapLdsBytes) launch(allow ? verify_classes_kernel<true, true> : verify_classes_kernel<false, true>, lds);
    else launch(allow ? verify_classes_kernel<true, false> : verify_classes_kernel<false, false>, 0);
    TDFA_HIP(hipGetLastError());
    return TDFA_OK;
}

// The dense path: every round streams rows of the table.
int minimize_dense(const int32_t* delta, int64_t row_words, int32_t n_rows, int32_t n_tokens, const uint8_t* accept, const int32_t* starts,
                   int32_t n_starts, hipStream_t s, std::vector<int32_t>* first_rows, std::vector<int32_t>* map_out)
{
    DeviceBuffers d;
    Arena mem;
    TDFA_GET(mem.get(&d.rows, (size_t)n_rows));
    TDFA_GET(mem.get(&d.aux, (size_t)n_rows));
    TDFA_GET(mem.get(&d.cls, (size_t)n_rows));
    TDFA_GET(mem.get(&d.mark, (size_t)n_rows));
    TDFA_GET(mem.get(&d.good, (size_t)n_rows));
    TDFA_GET(mem.get(&d.hash, (size_t)n_rows));
    TDFA_GET(mem.get(&d.flag, 1));
    std::vector<uint8_t> mark((size_t)n_rows, 0), good((size_t)n_rows, 0), seen((size_t)n_rows, 0);
    std::vector<int32_t> rows;
    const unsigned gx = grid_x(n_tokens);

    // ---- states that a token sequence reaches
    for (int32_t i = 0; i < n_starts; ++i)
        if (!mark[(size_t)starts[i]]) {
            mark[(size_t)starts[i]] = 1;
            rows.push_back(starts[i]);
        }
    seen = mark;
    TDFA_HIP(hipMemcpyAsync(d.mark, mark.data(), (size_t)n_rows, hipMemcpyHostToDevice, s));
    while (!rows.empty() && n_tokens > 0) {
        TDFA_HIP(hipMemcpyAsync(d.rows, rows.data(), rows.size() * 4, hipMemcpyHostToDevice, s));
        for (size_t lo = 0; lo < rows.size(); lo += kMaxGridY) {
            mark_targets_kernel<<<dim3(gx, (unsigned)std::min(kMaxGridY, rows.size() - lo)), kThreads, 0, s>>>(delta, n_tokens, d.rows + lo,
                                                                                                          d.mark);
            TDFA_HIP(hipGetLastError());
        }
        TDFA_HIP(hipMemcpyAsync(mark.data(), d.mark, (size_t)n_rows, hipMemcpyDeviceToHost, s));
        TDFA_HIP(hipStreamSynchronize(s));
        rows.clear();
        for (int32_t q = 0; q < n_rows; ++q)
            if (mark[(size_t)q] && !seen[(size_t)q]) {
                seen[(size_t)q] = 1;
                rows.push_back(q);
            }
    }
    // ---- of those, the states that can reach a final state
    for (int32_t q = 0; q < n_rows; ++q) good[(size_t)q] = mark[(size_t)q] && accept[q];
    TDFA_HIP(hipMemcpyAsync(d.good, good.data(), (size_t)n_rows, hipMemcpyHostToDevice, s));
    for (bool changed = n_tokens > 0; changed;) {
        rows.clear();
        for (int32_t q = 0; q < n_rows; ++q)
            if (mark[(size_t)q] && !good[(size_t)q]) rows.push_back(q);
        if (rows.empty()) break;
        int32_t zero = 0, flag = 0;
        TDFA_HIP(hipMemcpyAsync(d.flag, &zero, 4, hipMemcpyHostToDevice, s));
        TDFA_HIP(hipMemcpyAsync(d.rows, rows.data(), rows.size() * 4, hipMemcpyHostToDevice, s));
        for (size_t lo = 0; lo < rows.size(); lo += kMaxGridY) {
            reach_final_kernel<<<dim3(gx, (unsigned)std::min(kMaxGridY, rows.size() - lo)), kThreads, 0, s>>>(delta, n_tokens, d.rows + lo,
                                                                                                         d.mark, d.good, d.flag);
            TDFA_HIP(hipGetLastError());
        }
        TDFA_HIP(hipMemcpyAsync(&flag, d.flag, 4, hipMemcpyDeviceToHost, s));
        TDFA_HIP(hipMemcpyAsync(good.data(), d.good, (size_t)n_rows, hipMemcpyDeviceToHost, s));
        TDFA_HIP(hipStreamSynchronize(s));
        changed = flag != 0;
    }
    // ---- refinement over the kept states
    rows.clear();
    std::vector<int32_t> cls((size_t)n_rows, -1);
    for (int32_t q = 0; q < n_rows; ++q)
        if (mark[(size_t)q] && good[(size_t)q]) {
            rows.push_back(q);
            cls[(size_t)q] = accept[q] ? 1 : 0;
        }
    const size_t n = rows.size();
    map_out->assign((size_t)n_rows, TDFA_DEAD);
    first_rows->clear();
    if (n == 0) return TDFA_OK;
    TDFA_HIP(hipMemcpyAsync(d.rows, rows.data(), n * 4, hipMemcpyHostToDevice, s));
    std::vector<unsigned long long> hash(n);
    std::vector<int32_t> by(n), first_of(n);
    size_t n_cls = 0;
    for (unsigned attempt = 0;; ++attempt) {
        if (attempt == 4) return fail(TDFA_E_DEVICE, "row hashes collided in four attempts");
        for (size_t prev = 0;;) {
            TDFA_HIP(hipMemcpyAsync(d.cls, cls.data(), (size_t)n_rows * 4, hipMemcpyHostToDevice, s));
            row_hash_kernel<<<(unsigned)n, kThreads, 0, s>>>(delta, n_tokens, d.rows, d.cls, 0x243F6A8885A308D3ull * (attempt + 1), d.hash);
            TDFA_HIP(hipGetLastError());
            TDFA_HIP(hipMemcpyAsync(hash.data(), d.hash, n * 8, hipMemcpyDeviceToHost, s));
            TDFA_HIP(hipStreamSynchronize(s));
            for (size_t i = 0; i < n; ++i) by[i] = (int32_t)i;
            std::sort(by.begin(), by.end(), [&](int32_t x, int32_t y) {
                const int32_t cx = cls[(size_t)rows[(size_t)x]], cy = cls[(size_t)rows[(size_t)y]];
                if (cx != cy) return cx < cy;
                if (hash[(size_t)x] != hash[(size_t)y]) return hash[(size_t)x] < hash[(size_t)y];
                return x < y;
            });
            std::vector<int32_t> next(n);
            n_cls = 0;
            for (size_t i = 0; i < n; ++i) {
                const bool same = i > 0 && cls[(size_t)rows[(size_t)by[i]]] == cls[(size_t)rows[(size_t)by[i - 1]]] &&
                                  hash[(size_t)by[i]] == hash[(size_t)by[i - 1]];
                if (!same) {
                    ++n_cls;
                    first_of[n_cls - 1] = rows[(size_t)by[i]];          // the smallest row of the class (ties sorted by index)
                }
                next[(size_t)by[i]] = (int32_t)(n_cls - 1);
            }
            for (size_t i = 0; i < n; ++i) cls[(size_t)rows[i]] = next[i];
            if (n_cls == prev) break;
            prev = n_cls;
        }
        // no class splits any more: compare every row with the first row of its class
        std::vector<int32_t> first_of_row(n);
        for (size_t i = 0; i < n; ++i) first_of_row[i] = first_of[(size_t)cls[(size_t)rows[i]]];
        int32_t zero = 0, bad = 0;
        TDFA_HIP(hipMemcpyAsync(d.flag, &zero, 4, hipMemcpyHostToDevice, s));
        TDFA_HIP(hipMemcpyAsync(d.aux, first_of_row.data(), n * 4, hipMemcpyHostToDevice, s));
        TDFA_HIP(hipMemcpyAsync(d.cls, cls.data(), (size_t)n_rows * 4, hipMemcpyHostToDevice, s));
        if (n_tokens > 0) {
            TDFA_GET(launch_verify(delta, nullptr, n_tokens, row_words, (int64_t)n, n_rows, d.rows, d.aux, d.cls, d.flag, s));
        }
        TDFA_HIP(hipMemcpyAsync(&bad, d.flag, 4, hipMemcpyDeviceToHost, s));
        TDFA_HIP(hipStreamSynchronize(s));
        if (!bad) break;
        // a collision merged rows that differ: start over from {final, not final} with other hashes
        for (size_t i = 0; i < n; ++i) cls[(size_t)rows[i]] = accept[rows[i]] ? 1 : 0;
    }
    // ---- number the classes by their smallest state
    std::vector<int32_t> order(n_cls);
    for (size_t c = 0; c < n_cls; ++c) order[c] = (int32_t)c;
    std::sort(order.begin(), order.end(), [&](int32_t x, int32_t y) { return first_of[(size_t)x] < first_of[(size_t)y]; });
    std::vector<int32_t> new_id(n_cls);
    first_rows->resize(n_cls);
    for (size_t k = 0; k < n_cls; ++k) {
        new_id[(size_t)order[k]] = (int32_t)k;
        (*first_rows)[k] = first_of[(size_t)order[k]];
    }
    for (size_t i = 0; i < n; ++i) (*map_out)[(size_t)rows[i]] = new_id[(size_t)cls[(size_t)rows[i]]];
    return TDFA_OK;
}

constexpr int kNotSparse = -1000;       // minimize_lists: take the dense path

// The sparse path.  Returns kNotSparse when a row has too many distinct targets or the final
// comparison fails (two different rows with one signature).  *bits_agree: every bit has been seen to mark its entry.
int minimize_lists(const int32_t* delta, const uint32_t* allow, int64_t row_words, int32_t n_rows, int32_t n_tokens, const uint8_t* accept, const int32_t* starts,
                   int32_t n_starts, hipStream_t s, std::vector<int32_t>* first_rows, std::vector<int32_t>* map_out, bool* bits_agree)
{
    const unsigned long long seed = 0x243F6A8885A308D3ull;
    const SearchShape search = search_shape(n_rows);
    // Launches between two looks of the host, which cost as much as half a dozen of them (a copy and a wait, some 25 us); those
    // behind the last one that changes anything end at once.  The first look comes behind both searches and the refinement,
    // each with launches enough for most tables; only a search that is not through by then is looked at by itself, and then the
    // refinement begins anew.  (8, 4 and 8: 179 rows of 2,000 tokens 352 us, 224 of a schema 433, 2,204 of eight schemas 831, 5,387 of 128,256 tokens 1,894;
    // 4 launches of the first search 354, 684, 1,188 and 1,865, 12 359, 434, 849 and 1,870; 2 of the second 354, 501, 996 and 1,879, 8 366, 435, 836 and
    // 1,905; 4 rounds 419, 476, 905 and 1,932, 12 370, 442, 773 and 1,909.)
    const int reaches = search.launches > 1 ? search.launches : 8, finals = search.launches > 1 ? search.launches : 4;
    const int rounds = search.launches > 1 ? 4 : 8;    // (even: the hash tables take turns)
    // what the host looks at, side by side: the size of the lists; [0] a row with too many targets, [1] bits that differ, [2] mismatch, then a
    // flag for each launch of the searches, the number of classes after each round (behind that of the two before), and the classes of the rows
    const int at_reach = 3, at_final = at_reach + reaches, at_rounds = at_final + finals + 2, n_flags = (at_rounds + rounds + 1) & ~1;
    Arena mem;
    unsigned long long *counter, *row_begin, *weight, *e_weight = nullptr, *ht_keys;
    int32_t *row_n, *e_target = nullptr, *flags, *ht_mins, *pairs_dev, *cls_b;
    uint32_t* slot_of;
    uint8_t *mark, *done, *good, *accept_dev;
    uint32_t ht_size = 1024;
    while (ht_size < 2u * (uint32_t)n_rows && ht_size < 0x80000000u) ht_size <<= 1;
    // (the flags apart from the counter: every row looks at them, and adds to it)
    constexpr int kApart = 64;                     // in ints: two cache lines
    TDFA_GET(mem.get(&counter, ((size_t)kApart + (size_t)n_flags + (size_t)n_rows + 1) / 2));
    flags = reinterpret_cast<int32_t*>(counter) + kApart;
    int32_t* const cls_a = flags + n_flags;
    TDFA_GET(mem.get(&row_begin, n_rows));
    TDFA_GET(mem.get(&weight, n_tokens));
    TDFA_GET(mem.get(&row_n, n_rows));
    TDFA_GET(mem.get(&ht_keys, (size_t)2 * ht_size));
    TDFA_GET(mem.get(&ht_mins, (size_t)2 * ht_size));
    TDFA_GET(mem.get(&slot_of, n_rows));
    TDFA_GET(mem.get(&cls_b, n_rows));
    TDFA_GET(mem.get(&mark, (size_t)2 * n_rows));
    accept_dev = mark + n_rows;
    TDFA_GET(mem.get(&done, n_rows));
    TDFA_GET(mem.get(&good, n_rows));
    const HashTable ht[2] = {{ht_keys, ht_mins}, {ht_keys + ht_size, ht_mins + ht_size}};
    std::vector<uint8_t> mark_h((size_t)2 * n_rows, 0);
    for (int32_t i = 0; i < n_starts; ++i) mark_h[(size_t)starts[i]] = 1;
    std::copy(accept, accept + n_rows, mark_h.begin() + n_rows);
    TDFA_HIP(hipMemcpyAsync(mark, mark_h.data(), mark_h.size(), hipMemcpyHostToDevice, s));

    // ---- the lists: one pass over the table (a second one when they need more room than guessed)
    unsigned long long e_cap = std::max<unsigned long long>(1u << 20, std::min<unsigned long long>((unsigned long long)n_rows * 512, 1ull << 26));
    if (n_tokens > 0) token_weights_kernel<<<(unsigned)((n_tokens + kThreads - 1) / kThreads), kThreads, 0, s>>>(seed, n_tokens, weight);
    TDFA_HIP(hipGetLastError());
    const size_t n_init = std::max<size_t>({(size_t)n_rows, (size_t)(kApart + n_flags), ht_size});
    std::vector<int32_t> look((size_t)kApart + (size_t)n_flags + (size_t)n_rows);        // the counter, the flags, the classes
    int32_t* const seen = look.data() + kApart;
    for (int attempt = 0;; ++attempt) {
        TDFA_GET(mem.get(&e_target, e_cap));
        TDFA_GET(mem.get(&e_weight, e_cap));
        list_init_kernel<<<(unsigned)((n_init + kThreads - 1) / kThreads), kThreads, 0, s>>>(n_rows, done, slot_of, reinterpret_cast<int32_t*>(counter),
                                                                                             kApart + n_flags, ht[0], ht[1], ht_size);
        row_targets_kernel<<<(unsigned)n_rows, kListThreads, 0, s>>>(delta, allow, n_tokens, row_words, weight, e_cap, counter, row_begin,
                                                                     row_n, e_target, e_weight, flags, flags + 1);
        TDFA_HIP(hipGetLastError());
        TDFA_HIP(hipMemcpyAsync(look.data(), counter, (kApart + 2) * 4, hipMemcpyDeviceToHost, s));
        TDFA_HIP(hipStreamSynchronize(s));
        unsigned long long total;
        std::memcpy(&total, look.data(), 8);
        if (seen[0]) return kNotSparse;
        *bits_agree = seen[1] == 0;
        if (total <= e_cap) break;
        if (attempt == 1) return fail(TDFA_E_DEVICE, "the lists of targets changed size between two passes");
        e_cap = total;
    }
    const Lists g = {row_begin, row_n, e_target, e_weight, n_rows};
    const unsigned by_wave = (unsigned)(((size_t)n_rows + kRowsPerBlock - 1) / kRowsPerBlock);
    const unsigned by_thread = (unsigned)(((size_t)n_rows + kThreads - 1) / kThreads);
    const unsigned by_key = (unsigned)(((size_t)n_rows + kKeyRows - 1) / kKeyRows);
    const unsigned by_slot = (unsigned)((std::max<size_t>((size_t)n_rows, ht_size) + kThreads - 1) / kThreads);
    auto reach = [&](int i) { list_reach_kernel<<<by_wave, kThreads, 0, s>>>(g, search.sweeps, mark, done, i ? flags + at_reach + i - 1 : nullptr, flags + at_reach + i); };
    auto reach_final = [&](int i) {
        list_reach_final_kernel<<<by_wave, kThreads, 0, s>>>(g, search.sweeps, mark, good, i ? flags + at_final + i - 1 : nullptr, flags + at_final + i);
    };
    // n launches of a search, again and again, until one has changed nothing
    auto search_on = [&](auto launch, int at, int n) -> int {
        do {
            TDFA_HIP(hipMemsetAsync(flags + at, 0, (size_t)n * 4, s));
            for (int i = 0; i < n; ++i) launch(i);
            TDFA_HIP(hipGetLastError());
            TDFA_HIP(hipMemcpyAsync(seen + at, flags + at, (size_t)n * 4, hipMemcpyDeviceToHost, s));
            TDFA_HIP(hipStreamSynchronize(s));
        } while (seen[at + n - 1]);
        return TDFA_OK;
    };

    // ---- states that a token sequence reaches, and of those the ones that reach a final state
    auto reach_anew = [&]() { list_good_start_kernel<<<by_thread, kThreads, 0, s>>>(n_rows, mark, accept_dev, good); };
    for (int i = 0; i < reaches; ++i) reach(i);
    reach_anew();
    for (int i = 0; i < finals; ++i) reach_final(i);
    // ---- refinement: classes named by their smallest row
    int round = 0;
    auto refine = [&]() {
        for (int r = 0; r < rounds; ++r, ++round) {
            int32_t *in = r & 1 ? cls_b : cls_a, *out = r & 1 ? cls_a : cls_b, *counts = flags + at_rounds + r;
            list_keys_kernel<<<by_key, kKeyThreads, 0, s>>>(g, round, counts, mark, good, accept_dev, in, seed, ht[r & 1], ht_size - 1, slot_of);
            list_assign_kernel<<<by_slot, kThreads, 0, s>>>(n_rows, round, in, slot_of, ht[r & 1].min, ht[~r & 1], ht_size, out, counts);
        }
    };
    refine();
    for (bool searched = false, stable = false; !stable;) {
        TDFA_HIP(hipGetLastError());
        TDFA_HIP(hipMemcpyAsync(seen, flags, ((size_t)n_flags + (size_t)n_rows) * 4, hipMemcpyDeviceToHost, s));
        TDFA_HIP(hipStreamSynchronize(s));
        if (!searched && (seen[at_reach + reaches - 1] || seen[at_final + finals - 1])) {
            // a search was not through: it goes on, and the refinement begins anew
            if (seen[at_reach + reaches - 1]) {
                TDFA_GET(search_on(reach, at_reach, reaches));
                reach_anew();
            }
            TDFA_GET(search_on(reach_final, at_final, finals));
            list_init_kernel<<<(unsigned)((n_init + kThreads - 1) / kThreads), kThreads, 0, s>>>(n_rows, done, slot_of, flags, n_flags, ht[0], ht[1], ht_size);
            searched = true;
            round = 0;
            refine();
            continue;
        }
        searched = true;
        // no class split in some round: none did after it either
        for (int r = round == rounds ? 1 : 0; r < rounds; ++r) stable = stable || seen[at_rounds + r] == seen[at_rounds + r - 1];
        if (stable) break;
        TDFA_HIP(hipMemcpyAsync(flags + at_rounds - 2, flags + at_rounds + rounds - 2, 8, hipMemcpyDeviceToDevice, s));
        TDFA_HIP(hipMemsetAsync(flags + at_rounds, 0, rounds * 4, s));
        refine();
    }
    const int32_t* const cls_h = seen + n_flags;

    // ---- every row that joined another one is compared with it
    std::vector<int32_t> joined, with;
    for (int32_t q = 0; q < n_rows; ++q) {
        const int32_t c = cls_h[q];
        if (c < 0 || c == q) continue;
        if (c > q || cls_h[c] != c || (accept[q] != 0) != (accept[c] != 0)) return kNotSparse;
        joined.push_back(q);
        with.push_back(c);
    }
    if (!joined.empty() && n_tokens > 0) {
        const size_t n = joined.size();
        TDFA_GET(mem.get(&pairs_dev, 2 * n));
        joined.insert(joined.end(), with.begin(), with.end());
        TDFA_HIP(hipMemcpyAsync(pairs_dev, joined.data(), joined.size() * 4, hipMemcpyHostToDevice, s));
        TDFA_GET(launch_verify(delta, *bits_agree ? allow : nullptr, n_tokens, row_words, (int64_t)n, n_rows, pairs_dev, pairs_dev + n, cls_a, flags + 2, s));
        TDFA_HIP(hipMemcpyAsync(seen + 2, flags + 2, 4, hipMemcpyDeviceToHost, s));
        TDFA_HIP(hipStreamSynchronize(s));
        if (seen[2]) return kNotSparse;
    }

    // ---- the classes in the order of their smallest states
    map_out->assign((size_t)n_rows, TDFA_DEAD);
    first_rows->clear();
    for (int32_t q = 0; q < n_rows; ++q)
        if (cls_h[q] == q) {
            (*map_out)[(size_t)q] = (int32_t)first_rows->size();
            first_rows->push_back(q);
        }
    for (int32_t q = 0; q < n_rows; ++q)
        if (cls_h[q] >= 0) (*map_out)[(size_t)q] = (*map_out)[(size_t)cls_h[q]];
    return TDFA_OK;
}

}  // namespace

int minimize_table(const int32_t* delta, const uint32_t* allow, int64_t row_words, int64_t n_rows64, int32_t n_tokens, const uint8_t* accept, const int32_t* starts,
                   int32_t n_starts, hipStream_t s, std::vector<int32_t>* first_rows, std::vector<int32_t>* map_out, bool* bits_agree)
{
    const int32_t n_rows = (int32_t)n_rows64;
    *bits_agree = false;
    const int rc = minimize_lists(delta, allow, row_words, n_rows, n_tokens, accept, starts, n_starts, s, first_rows, map_out, bits_agree);
    if (rc != kNotSparse) return rc;
    return minimize_dense(delta, row_words, n_rows, n_tokens, accept, starts, n_starts, s, first_rows, map_out);
}

int launch_compact_rows(const int32_t* delta, const uint32_t* allow, int32_t n_tokens, int64_t row_words, const std::vector<int32_t>& first_rows,
                        const std::vector<int32_t>& map, int32_t* out_delta, uint32_t* out_allow, hipStream_t s)
{
    // (no row kept, or rows without tokens: nothing to write, and nothing is sent that would have to be waited for)
    const int64_t n_new = (int64_t)first_rows.size();
    const int64_t pieces = n_new * ((row_words + kPieceWords - 1) / kPieceWords);
    if (pieces == 0) return TDFA_OK;
    Arena mem;
    int32_t *rows = nullptr, *map_dev = nullptr;
    std::vector<int32_t> both;
    try {
        both.reserve(first_rows.size() + map.size());
    } catch (const std::bad_alloc&) {
        return fail(TDFA_E_OOM, "host allocation failed");
    }
    both.insert(both.end(), first_rows.begin(), first_rows.end());
    both.insert(both.end(), map.begin(), map.end());
    TDFA_GET(mem.get(&rows, both.size()));
    map_dev = rows + first_rows.size();
    TDFA_HIP(hipMemcpyAsync(rows, both.data(), both.size() * 4, hipMemcpyHostToDevice, s));
    // four workgroups of eight wavefronts per compute unit (two where the map is at its largest)
    const size_t lds = map.size() * 4;
    const unsigned grid = (unsigned)std::min<int64_t>((pieces + kRenameThreads / 64 - 1) / (kRenameThreads / 64), 256 * 4);
    auto launch = [&](auto kernel, size_t bytes) {
        kernel<<<grid, kRenameThreads, bytes, s>>>(delta, allow, n_tokens, row_words, n_new, (int32_t)map.size(), rows, map_dev, out_delta,
                                                   out_allow);
    };
    if (lds <= kMapLdsBytes) launch(allow ? compact_rows_kernel<true, true> : compact_rows_kernel<false, true>, lds);
    else launch(allow ? compact_rows_kernel<true, false> : compact_rows_kernel<false, false>, 0);
    TDFA_HIP(hipGetLastError());
    TDFA_HIP(hipStreamSynchronize(s));
    return TDFA_OK;
}

}  // namespace tdfa
