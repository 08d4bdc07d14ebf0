// Internal interface between the C-ABI shim and the device kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "bf1_route.h"

namespace bf1 {

struct AttnArgs {
    const void* Q;
    const void* K;
    const void* V;
    void* O;
    float* LSE;             // may be null
    const int32_t* row_ptr; // a caller's table; null: the route of Eq. 1 (or the dense one)
    const int32_t* col_idx;
    int64_t nnz;            // entries of the route's table
    int32_t batch;
    int64_t n;
    int32_t Hq;
    int32_t Hkv;
    int32_t head_dim;       // 64 or 128
    int32_t B;              // block width 64 or 128 (BF1 route)
    int32_t L;              // local width of the route of Eq. 1
    bool dense;             // implicit route {0..j} over 64-token blocks
    int32_t key_split = 0;  // 0 automatic, 1 one key group, 2 two key groups per workgroup
    bool token_major = false;  // O is [batch, n, Hq, head_dim] instead of [batch, Hq, n, head_dim]
};

// Backward (head_dim 64 or 128; G * B >= 128).  All pointers are device memory.
struct BwdArgs {
    const void* Q;
    const void* K;
    const void* V;
    const void* O;
    const void* dO;
    const float* LSE;
    float* dQ;               // [batch, Hq, n, head_dim] fp32
    float* dK;               // [batch, Hkv, n, head_dim] fp32
    float* dV;
    float* delta;            // workspace: [batch, Hq, n] fp32 (D = rowsum(dO * O))
    float* lse2;             // workspace: [batch, Hq, n] fp32 (LSE * log2 e)
    float* part;             // workspace or dQ: [batch * Hkv, nslots, 2, 64, head_dim] fp32
    void* ds;                // workspace: dS units, [batch * Hkv, nusers, B/64, B/64, Hq/Hkv] x 8 KB bf16
    const int32_t* row_ptr;  // forward route (CSR)
    const int32_t* col_idx;
    int64_t nnz;
    const int32_t* users;    // transposed route entries (query blocks per key block)
    const int32_t* uoffs;    // [NB + 1]: first entry of each key block's list in users
    int64_t nusers;          // entries of the transposed route
    const int32_t* segs;     // [nseg][8]: key block, sub-tile, first entry, count, slot
    int32_t nseg;
    const int32_t* reds;     // [nred][4]: key block, sub-tile, first slot, slot count
    int32_t nred;
    int32_t nslots;
    int32_t batch;
    int64_t n;
    int32_t Hq;
    int32_t Hkv;
    int32_t B;               // block width 64 or 128
    int32_t head_dim;        // 64 or 128
    int32_t L;               // local width of the route
};

hipError_t launch_backward(const BwdArgs& a, hipStream_t stream);

// One-token decode over a paged cache (validated arguments only).
struct DecodePlanArgs {
    int32_t batch;
    const int32_t* seq_lens;    // [batch]
    const int32_t* page_table;  // [batch, max_pages]
    int32_t max_pages;
    int32_t num_pages;
    int32_t B;                  // page = block width
    int32_t L;
    int32_t dense;              // 1: every earlier block (dense comparator)
    int32_t* plan;              // [batch, stride]
    int32_t stride;
    int32_t cap;                // stride - 3
};
hipError_t launch_decode_plan(const DecodePlanArgs& a, hipStream_t stream);

struct DecodeArgs {
    const void* Q;              // [batch, Hq, head_dim] bf16
    const void* K;              // [num_pages, Hkv, B, head_dim] bf16
    const void* V;
    const int32_t* seq_lens;
    int32_t num_pages;
    const int32_t* plan;
    int32_t stride;
    int32_t cap;
    void* O;                    // [batch, Hq, head_dim] bf16
    float* LSE;                 // [batch, Hq] or null
    float* ws;                  // [batch * Hkv * nsplit, G * (head_dim + 2)] fp32
    int32_t batch;
    int32_t Hq;
    int32_t Hkv;
    int32_t head_dim;           // 64 or 128
    int32_t B;                  // 64 or 128
    int32_t nsplit;             // most splits per (sequence, kv-head), <= 256
    int32_t ppw;                // pages per split of a list that fills its row
};
// How a long list of decode pages is cut.  Splits are walked side by side, their
// records merged in rounds of 16 loads, for each of `outs` outputs of a merge
// thread; 64 keys take some 1.1 us with heads of 128, 0.85 with 64, a round 1.3.  A
// round more pays while it shortens the longest split by more than it costs:
// keys / 64 >= 25 r (r + 1) outs for round r + 1.  1024 pages of 64, one output: 46 us
// with 32 splits, 32 with 64, 31 with 128, 41 with 256; four outputs: 55 with 32, 51
// with 64, 69 with 128; 256 pages, four outputs: 31 with 16, 29 with 32, 37 with 64.
BF1_HD int32_t decode_rounds(int64_t keys, int32_t outs, int32_t nsplit) {
    int32_t r = 1;
    while (16 * r < nsplit && (int64_t)25 * 64 * r * (r + 1) * outs <= keys) ++r;
    return r;
}
// Pages per split of a list cut into at most nsplit by its own length, for lists
// far shorter than their plan row could hold: 128 pages in a row for 2048, 16/8
// heads, 77 us at the row's split length, 16 at their own.
BF1_HD int32_t decode_pages_per_split(int32_t npages, int32_t page_keys, int32_t outs, int32_t nsplit) {
    const int32_t r = 16 * decode_rounds((int64_t)npages * page_keys, outs, nsplit);
    const int32_t most = r < nsplit ? r : nsplit;
    return (npages + most - 1) / most;
}
hipError_t launch_decode(const DecodeArgs& a, hipStream_t stream);

// Largest route table (row_ptr and col_idx entries) bf1_attn_fwd_noalloc accepts: a
// bound of its interface, no such table is made.
constexpr int64_t kNoallocInts = int64_t(1) << 20;

// Route planner: row_ptr[0..NB], col_idx[0..nnz) on `stream`.
hipError_t launch_plan(int32_t NB, int32_t L, int32_t* row_ptr, int32_t* col_idx,
                       hipStream_t stream);

// Attention forward (validated arguments only).
hipError_t launch_attention(const AttnArgs& a, hipStream_t stream);

}  // namespace bf1
