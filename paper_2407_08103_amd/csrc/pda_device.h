// The traversal of a token edge of a push-down constraint (Algorithm 3, the last statements of the loop), shared by
// the step kernel, which does it itself, and by the kernel that follows the other forms of the step.
#pragma once

#include "tdfa_internal.h"

namespace tdfa {

// One wavefront (all lanes active, every argument the same in all of them): the edge of state q (a state of the table)
// with token `tok` whose pops the stack ends with is found and traversed.
//
// A chain of three reads: the directory, which holds the place of the first edge of every 64 tokens of a state; the
// edges of those tokens, one per lane, token, pops and the top of the stack together; what the edge pushes and where it
// leads.  (A search that narrows a state's edges 64 probes at a time is three reads longer; in a kernel of its own it took
// 4.0 us.  256 sequences, nested JSON, 128,256 tokens in bf16: the step 18.75 us that way, 16.0 us with the directory and
// the traversal in the step kernel.)
__device__ __forceinline__ void pda_traverse(const PdaEdges& e, int32_t* stack, int32_t* depth_out, int depth, int stack_cap, int q,
                                             int tok, int32_t* token_out, int32_t* state_out)
{
    const int lane = (int)threadIdx.x & 63;
    const int64_t first = e.edge_first[q];
    const uint32_t* dir = e.dir + (int64_t)q * e.dir_stride + (tok >> kPdaDirShift);
    const int64_t lo = first + dir[0], hi = first + dir[1];
    // the top of the stack, the symbol popped first in lane 0
    const int32_t top = lane < kPdaPops && depth - 1 - lane >= 0 ? stack[depth - 1 - lane] : -1;
    long long found = -1;
    for (int64_t base = lo; base < hi && found < 0; base += 64) {
        const int64_t c = base + lane;
        const bool in = c < hi;
        const int64_t at = in ? c : lo;
        const int np = e.n_pops[at];
        const int4* pp = reinterpret_cast<const int4*>(e.pops + at * kPdaPops);
        const int4 p0 = pp[0], p1 = pp[1], p2 = pp[2];
        const int32_t pops[kPdaPops] = {p0.x, p0.y, p0.z, p0.w, p1.x, p1.y, p1.z, p1.w, p2.x, p2.y, p2.z, p2.w};
        bool mine = in && e.token[at] == tok && np <= depth;
#pragma unroll
        for (int j = 0; j < kPdaPops; ++j) {                       // (bottom to top: pops[np - 1] is the top)
            const int32_t s = __shfl(top, np - 1 - j < 0 ? 0 : np - 1 - j, 64);
            if (j < np) mine = mine && pops[j] == s;
        }
        const unsigned long long hit = __builtin_amdgcn_ballot_w64(mine);
        if (hit) found = (long long)(base + (int64_t)__builtin_ctzll(hit));
    }
    const int64_t at = found >= 0 ? found : lo;
    const int np = found >= 0 ? e.n_pops[at] : 0, nu = found >= 0 ? e.n_push[at] : 0;
    const int keep = depth - np;
    // no edge: cannot happen, the token was allowed through one; too many symbols: the sequence ends
    const bool ok = found >= 0 && keep + nu <= stack_cap;
    if (ok && lane < nu) stack[keep + lane] = e.pushes[at * kPdaPops + lane];
    if (lane != 0) return;
    *token_out = ok ? tok : TDFA_NO_TOKEN;
    *state_out = ok ? e.dst[at] : TDFA_DEAD;
    if (ok) *depth_out = keep + nu;
}

}  // namespace tdfa
