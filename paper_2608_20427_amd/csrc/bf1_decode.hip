// BF1 one-token decode over a paged key/value cache, for gfx950.
//
// The newest token of a sequence (position t = seq_len - 1, query block
// j = t / B) attends to the keys of row t of the paper's §3.1 mask: every key
// of the earlier selected blocks of P(j) (Eq. 1) and the keys j*B .. t of its
// own block.  §3.2 notes that such a token reads only O(log NB) blocks; here a
// block is one cache page of B tokens, so a step reads |P(j)| pages per
// kv-head.  The selected pages stay the same for all B tokens of block j
// (§5.4: a plan can persist across the 64-token route epoch), so they are
// listed once per epoch by the plan kernel and reused by every step.
//
// Cache layout: K and V pages [num_pages, Hkv, B, D] bf16 (a page holds B
// consecutive tokens of one sequence; one (page, kv-head) slice is contiguous,
// B * D * 2 bytes).  A page table [batch, max_pages] maps each sequence's
// logical block i to its physical page; only the planner reads it.
//
// Plan row of a sequence (int32, `stride` = 3 + cap entries):
//   [0]                 block j the plan was made for (-1: not plannable)
//   [1]                 c, the number of earlier selected pages
//   [2, 2 + c)          their physical pages, ascending logical block
//   [2 + c]             the page of block j itself
// A step reads only its sequence length and this row, two independent loads,
// before it can address the cache.
//
// Split kernel: one workgroup of four waves per (sequence, kv-head, split);
// a split is some consecutive pages of the sequence's list (earlier pages,
// then the self page).  Each wave takes 16 keys of every 64 as one matrix tile
// and keeps an online softmax (log2 units).  The four waves merge in LDS; a
// split that covers the whole list writes O and LSE at once, otherwise it
// writes a partial record
// (per q-head: max, sum, unnormalised O row).  Merge kernel: one workgroup
// per (sequence, kv-head) with more than one split sums the records in split
// order (deterministic).  The kernel boundary orders the records before their
// readers; a single kernel with a completion counter would need device-scope
// release/acquire fences per workgroup, which write back and invalidate the
// whole L2 of an XCD each time and cost far more than the second launch.
// Masked keys (past t in the self page) contribute exactly nothing, whatever
// the page holds there.
#include <hip/hip_runtime.h>
#include <math.h>

#include <type_traits>

#include "bf1_device.h"
#include "bf1_kernels.h"

namespace bf1 {
namespace {

constexpr int DEC_THREADS = 256;
constexpr int DEC_WAVES = DEC_THREADS / 64;
constexpr int PLAN_THREADS = 64;
constexpr float MIN_PART = 0x1p-132f;  // least first part of a weight: its half is the smallest bf16 number
constexpr int MAX_ROUTE = 64;  // bound on |P(j)| - 1 for any j < 2^31 and L <= 32

// ---------------------------------------------------------------------------
// Plan: one workgroup per sequence.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(PLAN_THREADS) void decode_plan_kernel(
    int32_t batch, const int32_t* __restrict__ seq_lens, const int32_t* __restrict__ page_table,
    int32_t max_pages, int32_t num_pages, int32_t B, int32_t L, int32_t dense,
    int32_t* __restrict__ plan, int32_t stride, int32_t cap) {
    __shared__ int32_t blocks[MAX_ROUTE];
    __shared__ int32_t count;
    __shared__ int32_t bad;
    const int b = blockIdx.x;
    const int tid = threadIdx.x;
    if (b >= batch) return;
    int32_t* row = plan + (int64_t)b * stride;
    const int64_t t = (int64_t)seq_lens[b] - 1;
    const int64_t j = t >= 0 ? t / B : -1;
    if (tid == 0) {
        bad = (t < 0 || j >= max_pages) ? 1 : 0;
        int c = 0;
        if (!bad && !dense) {
            // earlier blocks of P(j), ascending: 0, j - 2^r (r from high to
            // low, 2^r > L, skipping j - 2^r = 0), then j-L .. j-1
            if (j > L) blocks[c++] = 0;
            int r = 2;
            while (r < 30 && (int64_t(1) << (r + 1)) <= j) ++r;
            for (; r >= 2; --r) {
                const int64_t off = int64_t(1) << r;
                if (off <= j && off > L && j - off > 0) blocks[c++] = (int32_t)(j - off);
            }
            for (int64_t i = (j - L > 0 ? j - L : 0); i < j; ++i) blocks[c++] = (int32_t)i;
        } else if (!bad) {
            c = (int)j;
        }
        if (c > cap) bad = 1;
        count = c;
    }
    __syncthreads();
    const int c = count;
    const int32_t* pt = page_table + (int64_t)b * max_pages;
    if (!bad) {
        for (int e = tid; e < c; e += PLAN_THREADS) {
            const int32_t i = dense ? e : blocks[e];
            const int32_t p = pt[i];
            if (p < 0 || p >= num_pages) atomicOr(&bad, 1);
            row[2 + e] = p;
        }
        if (tid == 0) {
            const int32_t p = pt[j];  // the self page must exist as well
            if (p < 0 || p >= num_pages) atomicOr(&bad, 1);
            row[2 + c] = p;
        }
    }
    __syncthreads();
    if (tid == 0) {
        row[0] = bad ? -1 : (int32_t)j;
        row[1] = bad ? 0 : c;
    }
}

// ---------------------------------------------------------------------------
// Decode attention.
// ---------------------------------------------------------------------------

template <int D, int G>
constexpr int MERGE_OUTS = (G * D + DEC_THREADS - 1) / DEC_THREADS;  // outputs of a merge thread

// Whether a list is cut by its own length instead of its row's: less than half
// of a row for more than 32 pages (the cut's divisions cost 0.3 us of a step).
__device__ __forceinline__ bool short_list(int npages, int cap) { return cap >= 32 && 2 * (int64_t)npages <= cap; }

// What one step of sequence b reads: its newest position t, block j and the
// number c of earlier pages in its plan row.  False if the plan row was made
// for another block or is not a planner row; both kernels take the same
// decision from the same data.
struct StepView {
    int64_t t, j;
    int c;
};

__device__ __forceinline__ bool step_view(const int32_t* __restrict__ seq_lens, const int32_t* row,
                                          int32_t cap, int PW, int b, StepView* v) {
    const int32_t n = seq_lens[b];
    const int32_t pj = row[0];
    const int32_t pc = row[1];
    v->t = (int64_t)n - 1;
    v->j = v->t >= 0 ? v->t / PW : -1;
    v->c = pc;
    return v->t >= 0 && pj == v->j && pc >= 0 && pc <= cap;
}

template <int D, int G>
__device__ __forceinline__ void write_nan(__bf16* O, float* LSE, int b, int Hq, int h, int tid, int nthreads) {
    for (int x = tid; x < G * D; x += nthreads)
        O[((int64_t)b * Hq + h * G + x / D) * D + x % D] = (__bf16)__builtin_nanf("");
    if (LSE != nullptr && tid < G) LSE[(int64_t)b * Hq + h * G + tid] = __builtin_nanf("");
}

// A unit of decode work for one wave: 16 keys of a page, one 16x16x32 matrix
// tile of scores per 32 dims.  A page has PW / 16 units; wave w takes units w,
// w + 4.  Columns of the score tile are the q-heads of the group, repeated:
// column c is head c % G, and c / G selects a part of that head's weight.
//
// Scores S = K Q^T: A = K rows straight from memory (lane l: key l % 16, 16-byte
// chunk 4 s + l / 16 for k-step s), B = Q rows.  Lane l then holds the scores of
// keys 4 (l / 16) + 0..3 and column l % 16, which is the B operand of
// O^T += V^T P^T as it stands.  That product needs 16-bit weights, so a weight
// goes in as three bf16 parts that add up to the fp32 value (each part the
// rounded rest of the ones before: 24 bits), one part per column group.  G = 8
// has two column groups and a second product: the first group takes the first
// part in two halves, the other the second and the third part.  The rests are
// often zero or negative, so an infinite value would make NaN of them: the first
// group's columns never meet a rest, and the epilogue adds the other columns
// only where the first is finite.  V^T comes from LDS by transpose reads: a V unit
// is staged by direct buffer -> LDS loads, 32-byte slot s of key row r at
// s ^ vslot(r) (conflict-free: the 16 rows of a read hit distinct banks).
// Rows past the valid keys are zeros by the buffer range check, whatever the
// page holds.
//
// Bound by memory: about 40 vector instructions per unit where one fma per head
// and element took 400, which bounded groups of 8 and cost the others their
// overlap.  128 registers (K rows single-buffered, refilled once the scores have
// read them) keep four workgroups per compute unit; three with K double-buffered
// (154 registers) were no faster for G = 8 and 2-12% slower for G <= 2.  Device
// time per step with the same splits, us, before / now: 32 sequences, context
// 64K, 16/8 heads of 128 25.1 / 23.2; 16/2 heads 30.8 / 18.3; 16 sequences of
// 16/8 heads of 64 12.6 / 10.6; four dense lists of 32K 101 / 91.
template <int D>
struct Unit {
    static constexpr int KEYS = 16;
    static constexpr int RB = 2 * D;            // bytes per key row
    static constexpr int KS = D / 32;           // k-steps of the scores = K loads per unit
    static constexpr int DT = D / 16;           // 16-wide d tiles of O
    static constexpr int SEGS = KEYS * RB / 1024;  // direct V loads per unit
    static constexpr int WAIT_NEXT = 0x0F70 | SEGS;  // vmcnt: all but the next unit's V loads
};
template <int D>
__device__ __forceinline__ int vslot(int row) {
    return D == 128 ? (row & 7) : ((row >> 1) & 3);
}

// 16 bytes per lane of a page row, to registers or (in lane order) to LDS;
// non-temporal, for a page row is read once per step.
constexpr int CPOL_NT = 2;
__device__ __forceinline__ u32x4 load_row16_nt(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff) {
    return __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, CPOL_NT);
}
__device__ __forceinline__ void load_lds16_nt(__amdgpu_buffer_rsrc_t r, void* lds_segment, uint32_t voff,
                                              uint32_t soff) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_void*)lds_segment, 16, voff, soff, 0, CPOL_NT);
}

// 16-key V^T operands of four d tiles: four transpose reads at constant offset
// OFF from their lane addresses and the wait for them in one statement (the
// destinations are written asynchronously).
template <int OFF>
__device__ __forceinline__ void read_v_tr(uint32_t a0, uint32_t a1, uint32_t a2, uint32_t a3, u32x2 (&v)[4]) {
    asm volatile(
        "ds_read_b64_tr_b16 %0, %4 offset:%8\n\tds_read_b64_tr_b16 %1, %5 offset:%8\n\t"
        "ds_read_b64_tr_b16 %2, %6 offset:%8\n\tds_read_b64_tr_b16 %3, %7 offset:%8\n\t"
        "s_waitcnt lgkmcnt(0)"
        : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3])
        : "v"(a0), "v"(a1), "v"(a2), "v"(a3), "i"(OFF)
        : "memory");
}

// x combined with the values of the lanes 16, 32 and 48 apart (same column)
__device__ __forceinline__ float col_max(float x) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return pair_max(fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1])));
}
__device__ __forceinline__ float col_sum(float x) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return pair_sum(__uint_as_float(r[0]) + __uint_as_float(r[1]));
}

template <int D, int G, int PW>
__global__ __launch_bounds__(DEC_THREADS, 4) void decode_kernel(
    const __bf16* __restrict__ Q, const __bf16* __restrict__ Kp, const __bf16* __restrict__ Vp,
    const int32_t* __restrict__ seq_lens, int32_t num_pages, const int32_t* __restrict__ plan,
    int32_t stride, int32_t cap, __bf16* __restrict__ O, float* __restrict__ LSE,
    float* __restrict__ ws, int32_t Hkv, int32_t nsplit, int32_t ppw, float c_log2) {
    using U = Unit<D>;
    constexpr int KS = U::KS, DT = U::DT, RB = U::RB;
    constexpr int REC = G * (D + 2);          // floats per partial record
    constexpr int UPW = PW / 16 / DEC_WAVES;  // units of a page per wave
    constexpr int GROUPS = 16 / G < 3 ? 16 / G : 3;  // column groups that carry a part
    constexpr int COLS = GROUPS * G;
    constexpr int OST = D + 4;                // floats per O column in LDS (conflict-free 16-byte stores)

    // V units (two per wave), then the waves' results
    constexpr int V_BYTES = DEC_WAVES * 2 * 16 * RB;
    constexpr int R_BYTES = DEC_WAVES * COLS * (OST + 2) * 4;
    __shared__ __align__(256) u32x4 lds[(V_BYTES > R_BYTES ? V_BYTES : R_BYTES) / 16 + 1];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 15;
    const int quad = lane >> 4;
    const int s = blockIdx.x % nsplit;
    const int bh = blockIdx.x / nsplit;
    const int h = bh % Hkv;
    const int b = bh / Hkv;
    const int Hq = Hkv * G;
    const int32_t* row = plan + (int64_t)b * stride;

    StepView sv;
    if (!step_view(seq_lens, row, cap, PW, b, &sv)) {
        // stale or unplannable: the outputs of this (sequence, kv-head) are NaN
        if (s == 0) write_nan<D, G>(O, LSE, b, Hq, h, tid, DEC_THREADS);
        return;
    }
    const int c = sv.c;
    const int npages = c + 1;
    if (short_list(npages, cap)) ppw = decode_pages_per_split(npages, PW, MERGE_OUTS<D, G>, nsplit);
    const int nsb = (npages + ppw - 1) / ppw;
    if (s >= nsb) return;
    const int p0 = s * ppw;
    const int p1 = min(npages, p0 + ppw);

    // this wave's LDS: two V units
    char* vbuf = reinterpret_cast<char*>(&lds[0]) + wave * (2 * 16 * RB);
    // lane offsets inside a unit: K operand rows, V rows in swizzled lane order
    const uint32_t koff = (uint32_t)(col * RB + quad * 16);
    uint32_t voff[U::SEGS];
#pragma unroll
    for (int i = 0; i < U::SEGS; ++i) {
        const int r = i * (1024 / RB) + lane / (RB / 16), pc = lane % (RB / 16);
        voff[i] = (uint32_t)(r * RB + 16 * (2 * ((pc >> 1) ^ vslot<D>(r)) + (pc & 1)));
    }
    // transpose reads: key row 4 quad + col / 4, dims 16 dt + 4 (col % 4) ..; the
    // slot's address bits are clear in the rest, so tile dt is this ^ 32 dt
    static_assert((16 * RB) % 256 == 0 && RB >= 32 * DT, "slot bits must be clear in unit and row addresses");
    const uint32_t vtr = lds_addr(vbuf) + (4 * quad + (col >> 2)) * RB + 8 * (col & 3) +
                         32 * vslot<D>(4 * quad + (col >> 2));

    // Q rows as the score product's B operand
    bf16x8 qf[KS];
    {
        const u32x4* src = reinterpret_cast<const u32x4*>(Q + ((int64_t)b * Hq + h * G + col % G) * D);
#pragma unroll
        for (int k = 0; k < KS; ++k) qf[k] = __builtin_bit_cast(bf16x8, src[4 * k + quad]);
    }

    f32x4 acc[DT];
#pragma unroll
    for (int t = 0; t < DT; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
    float m_run = -INFINITY, l_run = 0.f;

    // Step st of this wave: page p0 + st / UPW, unit wave + 4 (st % UPW).
    // Pages written by the planner are in range; the clamp only keeps a foreign
    // plan row from addressing memory outside the cache.
    const int nsteps = (p1 - p0) * UPW;
    auto valid_keys = [&](int p) { return p < c ? PW : (int)(sv.t - sv.j * PW + 1); };
    struct Where {
        int64_t base;   // element offset of the page slice
        uint32_t bytes; // its valid keys
        uint32_t soff;  // the unit in it
    };
    auto where = [&](int st) {
        const int p = p0 + st / UPW;
        const int page = __builtin_amdgcn_readfirstlane(min(max(row[2 + p], 0), num_pages - 1));
        return Where{((int64_t)page * Hkv + h) * PW * D, (uint32_t)valid_keys(p) * RB,
                     (uint32_t)(wave + DEC_WAVES * (st % UPW)) * 16 * RB};
    };
    u32x4 kr[KS];
    auto load_k = [&](const Where& a) {
        const __amdgpu_buffer_rsrc_t r = head_rsrc(Kp + a.base, a.bytes);
#pragma unroll
        for (int k = 0; k < KS; ++k) kr[k] = load_row16_nt(r, koff + 64 * k, a.soff);
    };
    auto load_v = [&](const Where& a, int buf) {
        const __amdgpu_buffer_rsrc_t r = head_rsrc(Vp + a.base, a.bytes);
#pragma unroll
        for (int i = 0; i < U::SEGS; ++i) load_lds16_nt(r, vbuf + buf * (16 * RB) + i * 1024, voff[i], a.soff);
    };
    // One unit: its K rows are in flight to kr and its V rows to buffer BUF.  The
    // next unit's V rows are issued before the wait for them, its K rows as soon
    // as the scores have taken kr.
    auto step = [&](int st, auto buf_c) {
        constexpr int BUF = decltype(buf_c)::value;
        const int p = p0 + st / UPW, un = wave + DEC_WAVES * (st % UPW);
        const int nv = valid_keys(p) - 16 * un - 4 * quad;  // valid ones among this lane's keys
        const bool more = st + 1 < nsteps;
        const Where nx = where(more ? st + 1 : st);
        if (more) {
            load_v(nx, BUF ^ 1);
            __builtin_amdgcn_sched_barrier(0);
            __builtin_amdgcn_s_waitcnt(U::WAIT_NEXT);
        } else {
            __builtin_amdgcn_s_waitcnt(VMCNT0);
        }
        f32x4 sc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < KS; ++k)
            sc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kr[k]), qf[k], sc, 0, 0, 0);
        if (more) load_k(nx);
        __builtin_amdgcn_sched_barrier(0);
        float mx = -INFINITY;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            sc[r] = r < nv ? sc[r] * c_log2 : -INFINITY;
            mx = fmaxf(mx, sc[r]);
        }
        const float m_new = fmaxf(m_run, col_max(mx));
        const float m_use = m_new == -INFINITY ? 0.f : m_new;
        if (__any(m_new > m_run)) {
            const float alpha = exp2f(m_run - m_use);
            l_run *= alpha;
#pragma unroll
            for (int t = 0; t < DT; ++t)
#pragma unroll
                for (int r = 0; r < 4; ++r) acc[t][r] *= alpha;
            m_run = m_new;
        }
        bf16x4 pb, pb2;  // this column group's parts in the first product, and (G = 8) in the second
        // Weights and what their first parts are made of.  The exp2 instruction
        // gives 0 below 2^-126: weights there take the library function and a first
        // part above 0, so that an infinite value counts at every weight fp32 holds.
        // Asking costs a step 0.5% with heads of 128, 1.5% with heads of 64.
        float w[4], first[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) w[r] = sc[r] - m_use;
        if (__builtin_expect(__any(fminf(fminf(w[0], w[1]), fminf(w[2], w[3])) < -126.f), 0)) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                w[r] = exp2f(w[r]);
                first[r] = w[r] > 0.f ? fmaxf(w[r], MIN_PART) : w[r];
            }
        } else {
#pragma unroll
            for (int r = 0; r < 4; ++r) first[r] = w[r] = __builtin_amdgcn_exp2f(w[r]);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float pv = w[r];
            l_run += pv;
            const __bf16 p1b = (__bf16)first[r];
            const float r1 = pv - (float)p1b;
            const __bf16 p2b = (__bf16)r1;
            const __bf16 p3b = (__bf16)(r1 - (float)p2b);
            const int part = col / G;
            if constexpr (GROUPS == 3) {
                pb[r] = part == 0 ? p1b : part == 1 ? p2b : part == 2 ? p3b : (__bf16)0.f;
            } else {
                const __bf16 half1 = (__bf16)(0.5f * (float)p1b);
                pb[r] = part == 0 ? half1 : p2b;
                pb2[r] = part == 0 ? half1 : p3b;
            }
        }
#pragma unroll
        for (int t0 = 0; t0 < DT; t0 += 4) {
            u32x2 vt[4];
            read_v_tr<BUF * 16 * RB>(vtr ^ (32 * t0), vtr ^ (32 * t0 + 32), vtr ^ (32 * t0 + 64), vtr ^ (32 * t0 + 96),
                                     vt);
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const s16x4 a = __builtin_bit_cast(s16x4, vt[t]);
                f32x4& o = acc[t0 + t];
                o = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, __builtin_bit_cast(s16x4, pb), o, 0, 0, 0);
                if constexpr (GROUPS < 3)
                    o = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, __builtin_bit_cast(s16x4, pb2), o, 0, 0, 0);
            }
        }
    };

    {
        const Where w0 = where(0);
        load_v(w0, 0);
        load_k(w0);
    }
    for (int st = 0; st < nsteps; st += 2) {
        step(st, std::integral_constant<int, 0>{});
        if (st + 1 < nsteps) step(st + 1, std::integral_constant<int, 1>{});
    }

    // ---- the four waves' results through LDS (over the V units) ----------------
    float* r_o = reinterpret_cast<float*>(&lds[0]);       // [wave][column][OST]
    float* r_m = r_o + DEC_WAVES * COLS * OST;            // [wave][column][max, sum]
    l_run = col_sum(l_run);
    __syncthreads();
    if (col < COLS) {
        float* dst = r_o + (wave * COLS + col) * OST + 4 * quad;
#pragma unroll
        for (int t = 0; t < DT; ++t) *reinterpret_cast<f32x4*>(dst + 16 * t) = acc[t];
        if (quad == 0) {
            r_m[(wave * COLS + col) * 2] = m_run;
            r_m[(wave * COLS + col) * 2 + 1] = l_run;
        }
    }
    __syncthreads();

    const bool single = nsb == 1;
    float* rec = ws + ((int64_t)bh * nsplit + s) * REC;
    for (int x = tid; x < G * D; x += DEC_THREADS) {
        const int e = x / D, d = x % D;
        float M = -INFINITY;
#pragma unroll
        for (int w = 0; w < DEC_WAVES; ++w) M = fmaxf(M, r_m[(w * COLS + e) * 2]);
        float o = 0.f, l = 0.f;
#pragma unroll
        for (int w = 0; w < DEC_WAVES; ++w) {
            const float mw = r_m[(w * COLS + e) * 2];
            const float sw = mw == -INFINITY ? 0.f : exp2f(mw - M);
            float ow = r_o[(w * COLS + e) * OST + d], rest = 0.f;
#pragma unroll
            for (int gr = 1; gr < GROUPS; ++gr) rest += r_o[(w * COLS + gr * G + e) * OST + d];
            ow = fabsf(ow) < INFINITY ? ow + rest : ow;
            o = fmaf(ow, sw, o);
            l = fmaf(r_m[(w * COLS + e) * 2 + 1], sw, l);
        }
        if (single) {
            O[((int64_t)b * Hq + h * G + e) * D + d] = (__bf16)(o / l);
            if (d == 0 && LSE != nullptr) LSE[(int64_t)b * Hq + h * G + e] = (M + log2f(l)) * LN2;
        } else {
            rec[e * (D + 2) + 2 + d] = o;
            if (d == 0) {
                rec[e * (D + 2)] = M;
                rec[e * (D + 2) + 1] = l;
            }
        }
    }
}

// Merge of the split records of one (sequence, kv-head), in split order:
// every thread owns one (q-head, dim) output and folds the records in groups
// of sixteen (their loads issued together, so a selected list of up to 16
// splits costs one load round trip) into a running max / sum / row.
template <int D, int G, int PW>
__global__ __launch_bounds__(DEC_THREADS) void decode_merge_kernel(
    const int32_t* __restrict__ seq_lens, const int32_t* __restrict__ plan, int32_t stride,
    int32_t cap, __bf16* __restrict__ O, float* __restrict__ LSE, const float* __restrict__ ws,
    int32_t Hkv, int32_t nsplit, int32_t ppw) {
    constexpr int REC = G * (D + 2);
    constexpr int U = 16;  // decode_rounds counts in these
    const int tid = threadIdx.x;
    const int bh = blockIdx.x;
    const int h = bh % Hkv;
    const int b = bh / Hkv;
    const int Hq = Hkv * G;
    StepView sv;
    if (!step_view(seq_lens, plan + (int64_t)b * stride, cap, PW, b, &sv))
        return;  // the split kernel wrote NaN
    if (short_list(sv.c + 1, cap)) ppw = decode_pages_per_split(sv.c + 1, PW, MERGE_OUTS<D, G>, nsplit);
    const int nsb = (sv.c + ppw) / ppw;
    if (nsb <= 1) return;  // the split kernel wrote the result
    const float* recs = ws + (int64_t)bh * nsplit * REC;
    for (int x = tid; x < G * D; x += DEC_THREADS) {
        const int e = x / D, d = x % D;
        float M = -INFINITY, l = 0.f, o = 0.f;
        for (int q0 = 0; q0 < nsb; q0 += U) {
            float mq[U], lq[U], oq[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const bool in = q0 + u < nsb;
                const float* r = recs + (int64_t)(in ? q0 + u : 0) * REC + e * (D + 2);
                mq[u] = in ? r[0] : -INFINITY;
                lq[u] = in ? r[1] : 0.f;
                oq[u] = in ? r[2 + d] : 0.f;
            }
            float mm = M;
#pragma unroll
            for (int u = 0; u < U; ++u) mm = fmaxf(mm, mq[u]);
            if (mm == -INFINITY) continue;
            const float a = exp2f(M - mm);  // 0 while nothing is accumulated
            l *= a;
            o *= a;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const float w = mq[u] == -INFINITY ? 0.f : exp2f(mq[u] - mm);
                l = fmaf(lq[u], w, l);
                o = fmaf(oq[u], w, o);
            }
            M = mm;
        }
        O[((int64_t)b * Hq + h * G + e) * D + d] = (__bf16)(o / l);
        if (d == 0 && LSE != nullptr) LSE[(int64_t)b * Hq + h * G + e] = (M + log2f(l)) * LN2;
    }
}

template <int D, int G, int PW>
hipError_t launch_decode_pw(const DecodeArgs& a, hipStream_t st) {
    const float c_log2 = LOG2E / sqrtf((float)D);
    hipLaunchKernelGGL((decode_kernel<D, G, PW>), dim3((unsigned)((int64_t)a.batch * a.Hkv * a.nsplit)),
                       dim3(DEC_THREADS), 0, st, (const __bf16*)a.Q, (const __bf16*)a.K, (const __bf16*)a.V,
                       a.seq_lens, a.num_pages, a.plan, a.stride, a.cap, (__bf16*)a.O, a.LSE, a.ws, a.Hkv,
                       a.nsplit, a.ppw, c_log2);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || a.nsplit <= 1) return e;
    hipLaunchKernelGGL((decode_merge_kernel<D, G, PW>), dim3((unsigned)((int64_t)a.batch * a.Hkv)),
                       dim3(DEC_THREADS), 0, st, a.seq_lens, a.plan, a.stride, a.cap, (__bf16*)a.O, a.LSE,
                       a.ws, a.Hkv, a.nsplit, a.ppw);
    return hipGetLastError();
}

template <int D, int G>
hipError_t launch_decode_g(const DecodeArgs& a, hipStream_t st) {
    return a.B == 64 ? launch_decode_pw<D, G, 64>(a, st) : launch_decode_pw<D, G, 128>(a, st);
}

template <int D>
hipError_t launch_decode_d(const DecodeArgs& a, hipStream_t st) {
    switch (a.Hq / a.Hkv) {
        case 1: return launch_decode_g<D, 1>(a, st);
        case 2: return launch_decode_g<D, 2>(a, st);
        case 4: return launch_decode_g<D, 4>(a, st);
        default: return launch_decode_g<D, 8>(a, st);
    }
}

}  // namespace

hipError_t launch_decode_plan(const DecodePlanArgs& a, hipStream_t st) {
    hipLaunchKernelGGL(decode_plan_kernel, dim3((unsigned)a.batch), dim3(PLAN_THREADS), 0, st, a.batch,
                       a.seq_lens, a.page_table, a.max_pages, a.num_pages, a.B, a.L, a.dense, a.plan,
                       a.stride, a.cap);
    return hipGetLastError();
}

hipError_t launch_decode(const DecodeArgs& a, hipStream_t st) {
    return a.head_dim == 64 ? launch_decode_d<64>(a, st) : launch_decode_d<128>(a, st);
}

}  // namespace bf1
