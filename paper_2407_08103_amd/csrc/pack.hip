// Edge-list form of a compiled table.  The paper keeps A_{R o V} as a list of edges and remarks
// (Section 2.5.1) that it is the states with near-|V| out-degree that make this costly; the dense
// table pays |V| entries for every state instead, though most states of a constraint automaton
// allow a handful of tokens.  The packed form keeps what both need: the allowed-bit row of every
// state (the decode step streams it as before) and, in place of the dense row, only the targets
// of its edges, in token order.  The token of an edge is not stored: it is the position of the
// edge among the set bits of the row, found with a directory of per-128-token counts:
//
//   delta_T[q][t] = targets[row_begin[q] + dir[q][t / 128] + popcount(bits of q in [128 (t / 128), t))]
//
// Size: 4 B per edge + |V| (1/8 + 1/32) B per state; never more than the dense row plus 4 %.
// A set-up call: the host sums the per-state counts between the two kernels and waits for them.
#include <new>
#include <vector>

#include "tdfa_internal.h"

namespace tdfa {
namespace {

constexpr int kThreads = 256;

// The bits of word `wi` of a row that stand for tokens: padding bits never count as edges.
__device__ __forceinline__ uint32_t token_bits(uint32_t w, int wi, int32_t n_tokens)
{
    const int rem = n_tokens - 32 * wi;
    return rem >= 32 ? w : (rem <= 0 ? 0u : w & ((1u << rem) - 1u));
}

__device__ __forceinline__ uint32_t block_count(uint4 w, int k, int32_t n_tokens)
{
    return __popc(token_bits(w.x, 4 * k, n_tokens)) + __popc(token_bits(w.y, 4 * k + 1, n_tokens)) +
           __popc(token_bits(w.z, 4 * k + 2, n_tokens)) + __popc(token_bits(w.w, 4 * k + 3, n_tokens));
}

// One workgroup per state: dir[q][k] for every block of 128 tokens, the state's edge count, and a copy of its bits.  A
// thread takes one block of every kThreads, so that a wavefront reads and writes whole kilobytes; bound by the memory.
// 4,245 rows of 128,256 tokens: 46 us and a copy of 28 us with the blocks of a thread side by side, 24 us so.
__global__ void __launch_bounds__(kThreads)
pack_count_kernel(const uint32_t* __restrict__ allow, int32_t n_tokens, int64_t row_words, int32_t n_blocks,
                  uint32_t* __restrict__ dir, uint32_t* __restrict__ row_count, uint32_t* __restrict__ allow_out)
{
    __shared__ uint32_t s_sum[2][kThreads / 64];
    const int64_t q = blockIdx.x;
    const uint4* row = reinterpret_cast<const uint4*>(allow + q * row_words);
    uint4* row_out = reinterpret_cast<uint4*>(allow_out + q * row_words);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t before = 0;                                   // edges in the blocks of the passes done
    int turn = 0;
    for (int k0 = 0; k0 < n_blocks; k0 += kThreads, turn ^= 1) {
        const int k = k0 + (int)threadIdx.x;
        uint4 w = make_uint4(0, 0, 0, 0);
        if (k < n_blocks) {
            w = row[k];
            row_out[k] = w;
        }
        const uint32_t mine = k < n_blocks ? block_count(w, k, n_tokens) : 0u;
        uint32_t incl = mine;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const uint32_t other = __shfl_up(incl, d, 64);
            if (lane >= d) incl += other;
        }
        if (lane == 63) s_sum[turn][wave] = incl;
        __syncthreads();                                   // (the next pass writes the other half of s_sum)
        uint32_t below = before, all = 0;
#pragma unroll
        for (int v = 0; v < kThreads / 64; ++v) {
            const uint32_t n = s_sum[turn][v];
            if (v < wave) below += n;
            all += n;
        }
        if (k < n_blocks) dir[q * n_blocks + k] = below + incl - mine;
        before += all;
    }
    if (threadIdx.x == 0) row_count[q] = before;
}

// One workgroup per state: the targets of its edges in token order.  A wavefront takes kChunks * 64 tokens at a time:
// their bits are read by the lanes side by side, a prefix over the lanes' counts and the directory's count of the first
// block place every 64 tokens, and then kChunks loads of entries are in flight, one token per lane (the entries are
// read and the targets written side by side; 64 tokens without an edge cost a branch).
//
// Bound by the memory: the entries of 4,245 rows of 128,256 tokens of which a quarter are edges, 0.55 GB written and about
// as much read: 1,490 us when a wavefront took 64 tokens at a time, each a chain of three dependent reads, 433 us with
// kChunks, 405 us with the next span's entries requested before one's are written.
constexpr int kPackThreads = 512;
constexpr int kChunks = 16;                                      // 32 words of bits, one per lane of half a wavefront

__global__ void __launch_bounds__(kPackThreads)
pack_targets_kernel(const int32_t* __restrict__ delta, const uint32_t* __restrict__ allow, int32_t n_tokens,
                    int64_t row_words, int32_t n_blocks, const uint32_t* __restrict__ dir,
                    const int64_t* __restrict__ row_begin, int32_t* __restrict__ targets)
{
    const int64_t q = blockIdx.x;
    const uint32_t* bits = allow + q * row_words;
    const int32_t* row = delta + q * n_tokens;
    int32_t* out = targets + row_begin[q];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    constexpr int kStep = kPackThreads / 64 * 2 * kChunks;          // words of bits
    auto load_word = [&](int w0) {
        const int wi = w0 + lane;
        return lane < 2 * kChunks && wi < (int)row_words ? token_bits(bits[wi], wi, n_tokens) : 0u;
    };
    auto load_dir = [&](int w0) { return w0 < (int)row_words ? dir[q * n_blocks + (w0 >> 2)] : 0u; };
    auto mask_of = [](uint32_t w, int c) {
        return ((unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)w, 2 * c + 1) << 32) | (uint32_t)__builtin_amdgcn_readlane((int)w, 2 * c);
    };
    auto load_entries = [&](int w0, uint32_t w, int32_t (&v)[kChunks]) {
#pragma unroll
        for (int c = 0; c < kChunks; ++c)
            if (__builtin_amdgcn_inverse_ballot_w64(mask_of(w, c))) v[c] = __builtin_nontemporal_load(row + 32 * w0 + 64 * c + lane);
    };
    // the next span's entries are requested before this one's are written, and the bits of the one after it
    int w0 = wave * 2 * kChunks;
    uint32_t w_next = load_word(w0), d_next = load_dir(w0), w_after = load_word(w0 + kStep), d_after = load_dir(w0 + kStep);
    int32_t v_next[kChunks];
    load_entries(w0, w_next, v_next);
    for (; w0 < (int)row_words; w0 += kStep) {
        const uint32_t w = w_next, d = d_next;
        int32_t v[kChunks];
#pragma unroll
        for (int c = 0; c < kChunks; ++c) v[c] = v_next[c];
        w_next = w_after;
        d_next = d_after;
        load_entries(w0 + kStep, w_next, v_next);
        w_after = load_word(w0 + 2 * kStep);
        d_after = load_dir(w0 + 2 * kStep);
        if (__builtin_amdgcn_ballot_w64(w != 0) == 0) continue;
        uint32_t incl = __popc(w);
#pragma unroll
        for (int s = 1; s < 2 * kChunks; s <<= 1) {
            const uint32_t other = __shfl_up(incl, s, 64);
            if (lane >= s) incl += other;
        }
        const uint32_t before = incl - __popc(w) + d;               // edges of the row below the lane's word
#pragma unroll
        for (int c = 0; c < kChunks; ++c) {
            const unsigned long long mask = mask_of(w, c);
            const uint32_t base = (uint32_t)__builtin_amdgcn_readlane((int)before, 2 * c);
            const uint32_t at = base + __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
            if (__builtin_amdgcn_inverse_ballot_w64(mask)) __builtin_nontemporal_store(v[c], out + at);
        }
    }
}

// One workgroup per state: how many tokens it allows.
__global__ void __launch_bounds__(kThreads)
row_allowed_kernel(const uint32_t* __restrict__ allow, int32_t n_tokens, int64_t row_words, uint32_t* __restrict__ out)
{
    __shared__ uint32_t s_part[kThreads / 64];
    const int64_t q = blockIdx.x;
    const uint4* row = reinterpret_cast<const uint4*>(allow + q * row_words);
    uint32_t mine = 0;
    for (int k = threadIdx.x; k < (int)(row_words / 4); k += kThreads) mine += block_count(row[k], k, n_tokens);
    for (int off = 32; off > 0; off >>= 1) mine += __shfl_xor(mine, off, 64);
    if ((threadIdx.x & 63) == 0) s_part[threadIdx.x >> 6] = mine;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t total = 0;
        for (int w = 0; w < kThreads / 64; ++w) total += s_part[w];
        out[q] = total;
    }
}

}  // namespace

int launch_row_allowed(const uint32_t* allow, int64_t n_rows, int32_t n_tokens, int64_t row_words, uint32_t* out, hipStream_t stream)
{
    if (n_rows <= 0) return TDFA_OK;
    row_allowed_kernel<<<(unsigned)n_rows, kThreads, 0, stream>>>(allow, n_tokens, row_words, out);
    TDFA_HIP(hipGetLastError());
    return TDFA_OK;
}

int pack_table(const int32_t* delta, const uint32_t* allow, int64_t n_rows, int32_t n_tokens, int64_t row_words,
               uint32_t* allow_out, hipStream_t stream, DeviceBlock* dir_block, DeviceBlock* begin_block, DeviceBlock* targets_block, int64_t* n_edges_out)
{
    const int32_t n_blocks = (int32_t)(row_words / 4);
    const size_t rows = (size_t)(n_rows > 0 ? n_rows : 1);
    int rc = block_alloc(dir_block, rows * (size_t)(n_blocks > 0 ? n_blocks : 1) * sizeof(uint32_t));
    if (rc == TDFA_OK) rc = block_alloc(begin_block, (rows + 1) * sizeof(int64_t));
    // the counts of the states share the block of row_begin until that is known: they are read before it is written
    if (rc != TDFA_OK) return rc;
    uint32_t* dir = static_cast<uint32_t*>(dir_block->ptr);
    int64_t* row_begin = static_cast<int64_t*>(begin_block->ptr);
    uint32_t* counts = static_cast<uint32_t*>(begin_block->ptr);
    std::vector<uint32_t> h_counts;
    std::vector<int64_t> h_begin;
    try {
        h_counts.resize((size_t)n_rows);
        h_begin.resize((size_t)n_rows + 1);
    } catch (const std::bad_alloc&) {
        return fail(TDFA_E_OOM, "host allocation failed");
    }
    // grids of at most 2^31 - 1 workgroups: one per state
    if (n_rows > 0) {
        pack_count_kernel<<<(unsigned)n_rows, kThreads, 0, stream>>>(allow, n_tokens, row_words, n_blocks, dir, counts, allow_out);
        TDFA_HIP(hipGetLastError());
        TDFA_HIP(hipMemcpyAsync(h_counts.data(), counts, (size_t)n_rows * sizeof(uint32_t), hipMemcpyDeviceToHost, stream));
    }
    TDFA_HIP(hipStreamSynchronize(stream));
    int64_t n_edges = 0;
    for (int64_t q = 0; q < n_rows; ++q) {
        h_begin[(size_t)q] = n_edges;
        n_edges += h_counts[(size_t)q];
    }
    h_begin[(size_t)n_rows] = n_edges;
    rc = block_alloc(targets_block, (size_t)(n_edges > 0 ? n_edges : 1) * sizeof(int32_t));
    if (rc != TDFA_OK) return rc;
    TDFA_HIP(hipMemcpyAsync(row_begin, h_begin.data(), ((size_t)n_rows + 1) * sizeof(int64_t), hipMemcpyHostToDevice, stream));
    if (n_rows > 0 && n_edges > 0)
        pack_targets_kernel<<<(unsigned)n_rows, kPackThreads, 0, stream>>>(delta, allow, n_tokens, row_words, n_blocks, dir, row_begin,
                                                                         static_cast<int32_t*>(targets_block->ptr));
    const hipError_t launched = hipGetLastError();
    const hipError_t done = hipStreamSynchronize(stream);  // h_begin is read by the copy until here
    TDFA_HIP(launched);
    TDFA_HIP(done);
    *n_edges_out = n_edges;
    return TDFA_OK;
}

}  // namespace tdfa
