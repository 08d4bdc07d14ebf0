// C-ABI shim of libbf1.so: argument validation, the plan cache, stream
// handling and the mapping of HIP errors to status codes.  Every argument
// check happens before any HIP call, so invalid calls touch no device.
#include <hip/hip_runtime_api.h>

#include <algorithm>
#include <array>
#include <atomic>
#include <map>
#include <mutex>
#include <tuple>
#include <vector>

#include "../../include/bf1.h"
#include "bf1_kernels.h"
#include "bf1_route.h"

namespace {

constexpr int kVersion = 10200;  // 1.2.0

bool aligned(const void* p, uintptr_t a) { return (reinterpret_cast<uintptr_t>(p) % a) == 0; }

// Route sizes; false if the table would not fit int32 indices.
bool route_sizes(int64_t n, int64_t B, int64_t L, int64_t* NB, int64_t* nnz) {
    *NB = (n + B - 1) / B;
    if (*NB >= 0x7fffffff) return false;
    *nnz = bf1::route_row_start(*NB, L);
    return *nnz >= 0 && *nnz < 0x7fffffff;
}

// ---- plan cache: (device, n, B, L) -> device CSR --------------------------
// A plan is complete before it enters the cache (built on a private stream
// that the host waits for), so later calls use it with no stream ordering at
// all -- which also makes them safe to capture into a HIP graph.  Building a
// plan is refused while the caller's stream is being captured.
struct Plan {
    int32_t* row_ptr = nullptr;
    int32_t* col_idx = nullptr;
    int64_t nnz = 0;
};

std::mutex g_mu;
std::map<std::tuple<int, int64_t, int32_t, int32_t>, Plan> g_plans;
std::map<int, hipStream_t> g_plan_streams;  // per device, created on first use

int status_of(hipError_t e) { return e == hipSuccess ? BF1_OK : BF1_ERR_HIP; }

// Forward key split (bf1_set_forward_key_split): 0 automatic, 1 never, 2 always.
std::atomic<int> g_key_split{0};

// True (and BF1_OK) if `s` is being captured into a graph.
int capturing(hipStream_t s, bool* yes) {
    hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &st) != hipSuccess) return BF1_ERR_HIP;
    *yes = st != hipStreamCaptureStatusNone;
    return BF1_OK;
}

// Validation shared by the attention entry points.
int check_attn(const void* Q, const void* K, const void* V, void* O, float* LSE, int32_t batch,
               int64_t n, int32_t Hq, int32_t Hkv, int32_t head_dim) {
    if (batch < 0 || n < 0 || Hq < 1 || Hkv < 1) return BF1_ERR_INVALID_ARG;
    if (Hq % Hkv != 0) return BF1_ERR_INVALID_ARG;
    if (n > 0x7fffffffLL - 256) return BF1_ERR_INVALID_ARG;
    // one head's K or V rows are addressed through a 32-bit buffer range
    if (n >= (int64_t(1) << 24)) return BF1_ERR_UNSUPPORTED;
    const int32_t G = Hq / Hkv;
    if (head_dim != 64 && head_dim != 128) return BF1_ERR_UNSUPPORTED;
    if (G != 1 && G != 2 && G != 4 && G != 8) return BF1_ERR_UNSUPPORTED;
    if (batch == 0 || n == 0) return BF1_OK;
    if (!Q || !K || !V || !O) return BF1_ERR_INVALID_ARG;
    if (!aligned(Q, 16) || !aligned(K, 16) || !aligned(V, 16) || !aligned(O, 16))
        return BF1_ERR_INVALID_ARG;
    if (LSE && !aligned(LSE, 4)) return BF1_ERR_INVALID_ARG;
    // element counts must fit comfortably in int64 byte offsets
    const double elems = (double)batch * (double)Hq * (double)n * (double)head_dim;
    if (elems > 4.0e18) return BF1_ERR_INVALID_ARG;
    return BF1_OK;
}

// ---- decode ----------------------------------------------------------------
// Earlier selected pages any token of a sequence of at most max_seq_len
// tokens can need: the largest c(j) over j < NB, which is c(NB - 1) because
// c never decreases (j <= L: c = j; beyond, the locals stay L, the dyadic
// count only grows, and where block 0 stops being a separate entry (j a power
// of two) the dyadic count has just grown by one), or NB - 1 if dense.
bool decode_cap(int64_t max_seq_len, int64_t B, int64_t L, bool dense, int64_t* cap) {
    const int64_t NB = (max_seq_len + B - 1) / B;
    if (NB < 1 || NB >= 0x7fffffff) return false;
    *cap = dense ? NB - 1 : bf1::route_pred_count(NB - 1, L);
    return true;
}

// Splits that a workspace of bf1_decode_workspace_size holds records for: lists
// of up to P pages cut for about 1024 workgroups, at most 256, of equal size.
int64_t decode_ws_splits(int64_t batch, int64_t Hkv, int64_t P) {
    const int64_t units = std::max<int64_t>(1, batch * Hkv);
    const int64_t most = std::min<int64_t>(P, std::min<int64_t>((1024 + units - 1) / units, 256));
    const int64_t pages = (P + most - 1) / most;
    return (P + pages - 1) / pages;
}

// Most splits of a step per (sequence, kv-head), never more than
// decode_ws_splits, and pages per split.  units = sequences x kv-heads, for 256
// compute units that hold four workgroups each.  Device time of a step, us, by
// splits:
//
// Lists of up to 16 pages (the selected ones) are walked uncut from a number of
// units on that depends on the instance: an uncut list is a chain of its pages,
// a cut one pays the merge launch, which costs more for more q-heads, while the
// bytes (half with heads of 64) come in at the same rate.  32K tokens, uncut / 2 /
// finest: heads of 128, pages of 64, one q-head: 128 units 17.6 / 15.8 / 15.4, 192
// 18.5 / 21.6 / 19.8, 256 19.4 / 22.5 / 23.0; four: 128 18.1 / 17.8 / 18.2, 160
// 18.6 / 22.6 / 20.4; eight: 64 18.0 / 20.3 / 18.6, 96 18.1 / 20.7 / 22.0, 128 18.5 /
// 21.3 / 22.1.  Pages of 128, one q-head: 192 30.1 / 30.2 / 28.3, 256 32.0 / 33.5 /
// 36.4; eight: 128 29.6 / 27.7 / 29.0, 192 30.9 / 36.1 / 35.1.  Heads of 64, pages of
// 64, one: 192 15.3 / 14.5 / 13.6, 256 15.5 / 15.2 / 15.7, 384 17.7 / 18.7 / 20.0;
// eight: 128 14.8 / 15.0 / 14.3, 192 14.8 / 16.7 / 16.4.  Pages of 128, one: 256 25.0 /
// 20.9 / 22.8, 384 28.3 / 27.5 / 30.0, 512 30.7 / 34.4 / 34.0; eight: 256 24.0 / 23.3 /
// 25.1, 320 27.9 / 28.6 / 29.6.  Below that line two splits from 193 units on, the
// finest cut before; up to 64 units at most 16 splits, one round of the merge, or
// where a merge thread has two or more outputs, one workgroup per compute unit and
// at least four splits.
//
// Longer lists (dense ones) are cut for four workgroups per compute unit into at
// most 32 splits, or for one per compute unit (two with heads of 64) where that
// makes at least 64 and as many merge rounds pay (decode_rounds has the figures):
// 16/8 heads of 128, 1024 pages, 4 units 48.0 / 35.0 / 40.5 with 32 / 64 / 128, 8 units
// 51.8 / 53.3 with 32 / 64, 16 units 92.2 / 88.2 / 93.3 with 16 / 32 / 64; heads of 64, 8
// units 39.6 / 33.4 / 40.3 with 32 / 64 / 128.  The grid has no split that a full list
// leaves empty: workgroups go to the chiplets in turn, and 20 of 32 in use load
// them 3 : 2 (40 pages of 128, 12 units, 18.3 us instead of 15.3).
void decode_splits(int64_t batch, int64_t Hkv, int64_t G, int64_t D, int64_t B, int64_t P, int32_t* nsplit,
                   int32_t* ppw) {
    // by head size, page width and q-heads per kv-head (1, 2, 4, 8)
    static constexpr int uncut_from[2][2][4] = {{{256, 256, 256, 192}, {448, 448, 448, 320}},
                                                {{192, 192, 160, 96}, {256, 256, 192, 192}}};
    const int64_t units = std::max<int64_t>(1, batch * Hkv);
    const int64_t outs = (G * D + 255) / 256;
    int64_t want = (1024 + units - 1) / units;
    if (P > 16) {
        want = std::min<int64_t>(want, 32);
        const int64_t fill = ((D == 64 ? 512 : 256) + units - 1) / units;
        if (fill >= 64)
            want = std::max(want, std::min<int64_t>(fill, 16 * bf1::decode_rounds(P * B, (int32_t)outs, 256)));
    } else if (units >= uncut_from[D == 128][B == 128][G == 8 ? 3 : G / 2]) {
        want = 1;
    } else if (units > 192) {
        want = 2;
    } else if (units <= 64) {
        want = outs == 1 ? 16 : std::max<int64_t>(4, (256 + units - 1) / units);
    }
    const int64_t most = std::min(want, decode_ws_splits(batch, Hkv, P));
    *ppw = (int32_t)((P + most - 1) / most);
    *nsplit = (int32_t)((P + *ppw - 1) / *ppw);
}

int64_t decode_ws_bytes(int64_t batch, int64_t Hq, int64_t Hkv, int64_t D, int64_t nsplit) {
    const int64_t G = Hq / Hkv;
    const int64_t b = batch * Hkv * nsplit * G * (D + 2) * 4;
    return (b + 255) / 256 * 256;
}

int run_attn(bf1::AttnArgs a, hipStream_t s) {
    a.key_split = g_key_split.load(std::memory_order_relaxed);
    return status_of(bf1::launch_attention(a, s));
}

// Cached forward route of (current device, n, B, L), built by the planner
// kernel on first use and complete on return.  `s` is the caller's stream
// (only checked for capture).
int get_plan(int64_t n, int32_t B, int32_t L, hipStream_t s, Plan* out) {
    int64_t NB, nnz;
    if (!route_sizes(n, B, L, &NB, &nnz)) return BF1_ERR_INVALID_ARG;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return BF1_ERR_HIP;
    std::lock_guard<std::mutex> lock(g_mu);
    auto key = std::make_tuple(dev, n, B, L);
    auto it = g_plans.find(key);
    if (it != g_plans.end()) {
        *out = it->second;
        return BF1_OK;
    }
    bool cap = false;
    int st = capturing(s, &cap);
    if (st != BF1_OK) return st;
    if (cap) return BF1_ERR_CAPTURE;
    hipStream_t ps = nullptr;
    auto ps_it = g_plan_streams.find(dev);
    if (ps_it == g_plan_streams.end()) {
        if (hipStreamCreateWithFlags(&ps, hipStreamNonBlocking) != hipSuccess) return BF1_ERR_HIP;
        g_plan_streams.emplace(dev, ps);
    } else {
        ps = ps_it->second;
    }
    Plan p;
    p.nnz = nnz;
    if (hipMalloc((void**)&p.row_ptr, sizeof(int32_t) * (NB + 1)) != hipSuccess) return BF1_ERR_NOMEM;
    if (hipMalloc((void**)&p.col_idx, sizeof(int32_t) * (nnz > 0 ? nnz : 1)) != hipSuccess) {
        (void)hipFree(p.row_ptr);
        return BF1_ERR_NOMEM;
    }
    hipError_t e = bf1::launch_plan((int32_t)NB, L, p.row_ptr, p.col_idx, ps);
    if (e == hipSuccess) e = hipStreamSynchronize(ps);
    if (e != hipSuccess) {
        (void)hipFree(p.row_ptr);
        (void)hipFree(p.col_idx);
        return BF1_ERR_HIP;
    }
    g_plans.emplace(key, p);
    *out = p;
    return BF1_OK;
}

// ---- backward plan: transposed route cut into segments ---------------------
// Every 64-key tile (key block i, sub-tile u, starting before n) gets the list
// of query blocks that select block i.  Lists longer than a segment length are
// cut into segments: the first one writes dK/dV, the others leave partial sums
// in numbered slots, which the reduce kernel adds in order.  Segments are
// ordered longest first.
//
// A workgroup walks one segment, so its length sets the longest chain.  Long
// sequences have work for every compute unit whatever the cut; there only
// block 0's list (every query block) exceeds 16 entries, and its partial tiles
// lie in the workspace (bf1_attn_bwd_workspace_size counts them).  Short ones
// leave most units idle behind that chain, so they are cut to about the
// entries a workgroup slot gets when all slots share the work, and the partial
// tiles lie in dQ, which the dQ kernel overwrites last.  Whole backward on
// MI355X, us, cut at 16 / for half / for exactly / for twice the 512 slots
// there are (16/8 heads of 128 unless said): 1K tokens 75 / 42 / 42 / 42, 2K
// 85 / 55 / 61 / 61, 4K 106 / 105 / 94 / 103, 4K at width 128 167 / 145 / 124 /
// 138, 4 x 1K 95 / 86 / 72 / 88, 2 x 1500 tokens of 8/2 heads of 64 106 / 43 /
// 43 / 43; from 8K on the share exceeds 16 entries and nothing changes.
constexpr int64_t SEG_MAX = 16;
constexpr int64_t SEG_LENGTHS[] = {1, 2, 3, 4, 6, 8, 12, SEG_MAX};
constexpr int SEG_KINDS = sizeof(SEG_LENGTHS) / sizeof(SEG_LENGTHS[0]);
constexpr int64_t BWD_SLOTS = 512;  // two resident dK/dV workgroups on each of 256 compute units

// Entries per workgroup slot of a backward over bh (batch x kv-head) problems
// (a list entry is B/64 query sub-tiles for each of B/64 key tiles).
int64_t seg_wanted(int64_t nusers, int64_t nsub, int64_t bh) {
    return (nusers * nsub * bh + BWD_SLOTS - 1) / BWD_SLOTS;
}

// Transposed route sizes: entries, and partial slots of the cut at SEG_MAX with
// a slot for every segment of a split list.
bool bwd_sizes(int64_t n, int32_t B, int32_t L, int64_t* nusers, int64_t* nslots) {
    const int64_t NB = (n + B - 1) / B;
    int64_t total = 0, slots = 0;
    for (int64_t i = 0; i < NB; ++i) {
        const int64_t cnt = bf1::route_users(NB, L, i, nullptr);
        total += cnt;
        const int64_t nch = (cnt + SEG_MAX - 1) / SEG_MAX;
        if (nch > 1) slots += nch * std::min<int64_t>(B / 64, (n - i * B + 63) / 64);
        if (slots > 0x3fffffff || total > 0x3fffffff) return false;
    }
    *nusers = total;
    *nslots = slots;
    return true;
}

// Segments (int32 x 8: key block, sub-tile, first entry, count, slot, 0, 0, 0)
// and reduce descriptors (int32 x 4: key block, sub-tile, first slot, count) of
// the lists in uoffs cut at `len` entries; returns the number of slots.
int64_t bwd_cut(int64_t n, int32_t B, const std::vector<int32_t>& uoffs, int64_t len, std::vector<int32_t>* segs,
                std::vector<int32_t>* reds) {
    std::vector<std::array<int32_t, 8>> sg;
    int64_t nslots = 0;
    for (int64_t i = 0; i + 1 < (int64_t)uoffs.size(); ++i) {
        const int64_t off = uoffs[i], cnt = uoffs[i + 1] - off;
        const int64_t nch = (cnt + len - 1) / len;
        for (int u = 0; u < B / 64 && i * B + u * 64 < n; ++u) {
            for (int64_t c = 0; c < nch; ++c)
                sg.push_back({(int32_t)i, u, (int32_t)(off + len * c), (int32_t)std::min(len, cnt - len * c),
                              (int32_t)(c > 0 ? nslots + c - 1 : -1), 0, 0, 0});
            if (nch > 1) {
                reds->insert(reds->end(), {(int32_t)i, u, (int32_t)nslots, (int32_t)(nch - 1)});
                nslots += nch - 1;
            }
        }
    }
    std::stable_sort(sg.begin(), sg.end(), [](const std::array<int32_t, 8>& a, const std::array<int32_t, 8>& b) {
        return a[3] > b[3];
    });
    for (auto& x : sg) segs->insert(segs->end(), x.begin(), x.end());
    return nslots;
}

struct BwdCut {
    int64_t len = 0;
    int32_t* segs = nullptr;
    int32_t* reds = nullptr;
    int32_t nseg = 0, nred = 0, nslots = 0;
};
struct BwdPlan {
    int32_t* memory = nullptr;   // one allocation, which the other pointers lie in
    int32_t* users = nullptr;
    int32_t* uoffs = nullptr;
    int64_t nusers = 0;
    int ncuts = 0;               // ascending lengths, SEG_MAX last
    BwdCut cuts[SEG_KINDS];
};
std::map<std::tuple<int, int64_t, int32_t, int32_t>, BwdPlan> g_bwd_plans;

// The cut of a call: the shortest segments that still give every slot its
// share, if their partial tiles fit dQ (nslots x 2 x 64 rows against the G n
// rows of a kv-head).
const BwdCut& pick_cut(const BwdPlan& p, int64_t n, int32_t B, int64_t bh, int64_t G) {
    const int64_t want = seg_wanted(p.nusers, B / 64, bh);
    int c = 0;
    while (c + 1 < p.ncuts && (p.cuts[c].len < want || (int64_t)p.cuts[c].nslots * 128 > G * n)) ++c;
    return p.cuts[c];
}

int bwd_workspace_bytes(int32_t batch, int64_t n, int32_t Hq, int32_t Hkv, int32_t head_dim, int32_t B,
                        int32_t L, int64_t* bytes) {
    int64_t nusers, nslots;
    if (!bwd_sizes(n, B, L, &nusers, &nslots)) return BF1_ERR_INVALID_ARG;
    const int64_t delta = ((int64_t)batch * Hq * n * 4 + 255) / 256 * 256;
    const int64_t part = (int64_t)batch * Hkv * nslots * 2 * 64 * head_dim * 4;
    const int64_t nsub = B / 64;
    const int64_t ds = (int64_t)batch * Hq * nusers * nsub * nsub * 64 * 64 * 2;
    *bytes = 2 * delta + part + ds;  // D, LSE * log2 e, partial tiles, dS units
    return BF1_OK;
}

int get_bwd_plan(int64_t n, int32_t B, int32_t L, hipStream_t s, BwdPlan* out) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return BF1_ERR_HIP;
    std::lock_guard<std::mutex> lock(g_mu);
    auto key = std::make_tuple(dev, n, B, L);
    auto it = g_bwd_plans.find(key);
    if (it == g_bwd_plans.end()) {
        bool cap = false;
        int st = capturing(s, &cap);
        if (st != BF1_OK) return st;
        if (cap) return BF1_ERR_CAPTURE;
        int64_t nslots;
        BwdPlan p;
        if (!bwd_sizes(n, B, L, &p.nusers, &nslots)) return BF1_ERR_INVALID_ARG;
        const int64_t NB = (n + B - 1) / B;
        std::vector<int32_t> users(p.nusers), uoffs, all;
        int64_t at = 0;
        for (int64_t i = 0; i < NB; ++i) {
            uoffs.push_back((int32_t)at);
            at += bf1::route_users(NB, L, i, users.data() + at);
        }
        uoffs.push_back((int32_t)at);
        // One allocation and one copy for all arrays, each 256-byte aligned: the
        // first call of a length waits for them (what it takes more than the next,
        // us, an allocation and a copy per array / one: 1000 tokens 254 / 28, 4K 297 /
        // 53, 16K 189 / 64).
        auto put = [&all](const std::vector<int32_t>& v) -> size_t {
            const size_t off = (all.size() + 63) / 64 * 64;
            all.resize(off);
            all.insert(all.end(), v.begin(), v.end());
            return off;
        };
        const size_t users_at = put(users), uoffs_at = put(uoffs);
        size_t segs_at[SEG_KINDS], reds_at[SEG_KINDS];
        // every cut that some batch and head count can ask for is made now, so
        // that later calls of any of them find it (also under capture)
        for (int k = 0; k < SEG_KINDS; ++k) {
            if (SEG_LENGTHS[k] != SEG_MAX && SEG_LENGTHS[k] < seg_wanted(p.nusers, B / 64, 1)) continue;
            std::vector<int32_t> segs, reds;
            BwdCut& c = p.cuts[p.ncuts];
            c.len = SEG_LENGTHS[k];
            c.nslots = (int32_t)bwd_cut(n, B, uoffs, c.len, &segs, &reds);
            c.nseg = (int32_t)(segs.size() / 8);
            c.nred = (int32_t)(reds.size() / 4);
            segs_at[p.ncuts] = put(segs);
            reds_at[p.ncuts++] = put(reds);
        }
        const size_t bytes = sizeof(int32_t) * all.size();
        if (hipMalloc((void**)&p.memory, bytes) != hipSuccess) return BF1_ERR_NOMEM;
        if (hipMemcpy(p.memory, all.data(), bytes, hipMemcpyHostToDevice) != hipSuccess) {
            (void)hipFree(p.memory);
            return BF1_ERR_NOMEM;
        }
        p.users = p.memory + users_at;
        p.uoffs = p.memory + uoffs_at;
        for (int c = 0; c < p.ncuts; ++c) {
            p.cuts[c].segs = p.memory + segs_at[c];
            p.cuts[c].reds = p.memory + reds_at[c];
        }
        it = g_bwd_plans.emplace(key, p).first;
    }
    *out = it->second;
    return BF1_OK;
}

}  // namespace

extern "C" {

int bf1_version(void) { return kVersion; }

const char* bf1_status_string(int status) {
    switch (status) {
        case BF1_OK: return "BF1_OK";
        case BF1_ERR_INVALID_ARG: return "BF1_ERR_INVALID_ARG: invalid argument";
        case BF1_ERR_UNSUPPORTED: return "BF1_ERR_UNSUPPORTED: configuration not supported";
        case BF1_ERR_BUFFER_TOO_SMALL: return "BF1_ERR_BUFFER_TOO_SMALL: route table capacity too small";
        case BF1_ERR_HIP: return "BF1_ERR_HIP: HIP runtime or launch error";
        case BF1_ERR_NOMEM: return "BF1_ERR_NOMEM: device allocation failed";
        case BF1_ERR_CAPTURE:
            return "BF1_ERR_CAPTURE: the route plan is not built yet and cannot be built while the "
                   "stream is being captured (call once outside capture first)";
        default: return "BF1: unknown status";
    }
}

int bf1_plan_size(int64_t n, int32_t B, int32_t L, int32_t* num_blocks, int64_t* nnz,
                  int64_t* pairs) {
    if (n < 0 || B < 1 || L < 0) return BF1_ERR_INVALID_ARG;
    int64_t NB, z;
    if (!route_sizes(n, B, L, &NB, &z)) return BF1_ERR_INVALID_ARG;
    if (num_blocks) *num_blocks = (int32_t)NB;
    if (nnz) *nnz = z;
    if (pairs) *pairs = bf1::route_selected_pairs(n, B, L);
    return BF1_OK;
}

int bf1_plan(int64_t n, int32_t B, int32_t L, int32_t* row_ptr, int32_t* col_idx,
             int64_t col_capacity, void* stream) {
    if (n < 0 || B < 1 || L < 0 || col_capacity < 0) return BF1_ERR_INVALID_ARG;
    int64_t NB, nnz;
    if (!route_sizes(n, B, L, &NB, &nnz)) return BF1_ERR_INVALID_ARG;
    if (!row_ptr) return BF1_ERR_INVALID_ARG;
    if (nnz > 0 && !col_idx) return BF1_ERR_INVALID_ARG;
    if (!aligned(row_ptr, 4) || (col_idx && !aligned(col_idx, 4))) return BF1_ERR_INVALID_ARG;
    if (col_capacity < nnz) return BF1_ERR_BUFFER_TOO_SMALL;
    return status_of(bf1::launch_plan((int32_t)NB, L, row_ptr, col_idx, (hipStream_t)stream));
}

int bf1_attn_fwd(const void* Q, const void* K, const void* V, void* O, float* LSE, int32_t batch,
                 int64_t n, int32_t Hq, int32_t Hkv, int32_t head_dim, int32_t B, int32_t L,
                 void* stream) {
    int st = check_attn(Q, K, V, O, LSE, batch, n, Hq, Hkv, head_dim);
    if (st != BF1_OK) return st;
    if (L < 0) return BF1_ERR_INVALID_ARG;
    if (B != 64 && B != 128) return BF1_ERR_UNSUPPORTED;
    if (batch == 0 || n == 0) return BF1_OK;
    hipStream_t s = (hipStream_t)stream;
    // The kernel walks Eq. 1 itself; the plan call keeps what the interface says
    // about a route's first use (no such call under capture, sizes, errors).
    Plan plan;
    st = get_plan(n, B, L, s, &plan);
    if (st != BF1_OK) return st;
    bf1::AttnArgs a{Q, K, V, O, LSE, nullptr, nullptr, plan.nnz, batch, n, Hq, Hkv, head_dim, B, L, false};
    return run_attn(a, s);
}

int bf1_attn_fwd_noalloc(const void* Q, const void* K, const void* V, void* O, float* LSE,
                         int32_t batch, int64_t n, int32_t Hq, int32_t Hkv, int32_t head_dim,
                         int32_t B, int32_t L, void* stream) {
    int st = check_attn(Q, K, V, O, LSE, batch, n, Hq, Hkv, head_dim);
    if (st != BF1_OK) return st;
    if (L < 0) return BF1_ERR_INVALID_ARG;
    if (B != 64 && B != 128) return BF1_ERR_UNSUPPORTED;
    if (batch == 0 || n == 0) return BF1_OK;
    int64_t NB, nnz;
    if (!route_sizes(n, B, L, &NB, &nnz)) return BF1_ERR_INVALID_ARG;
    if (NB + 1 + nnz > bf1::kNoallocInts) return BF1_ERR_BUFFER_TOO_SMALL;
    bf1::AttnArgs a{Q, K, V, O, LSE, nullptr, nullptr, nnz, batch, n, Hq, Hkv, head_dim, B, L, false};
    return run_attn(a, (hipStream_t)stream);
}

int bf1_attn_fwd_csr(const void* Q, const void* K, const void* V, void* O, float* LSE,
                     int32_t batch, int64_t n, int32_t Hq, int32_t Hkv, int32_t head_dim,
                     int32_t B, const int32_t* row_ptr, const int32_t* col_idx, int64_t nnz,
                     void* stream) {
    int st = check_attn(Q, K, V, O, LSE, batch, n, Hq, Hkv, head_dim);
    if (st != BF1_OK) return st;
    if (B != 64 && B != 128) return BF1_ERR_UNSUPPORTED;
    if (nnz < 0 || nnz >= 0x7fffffff) return BF1_ERR_INVALID_ARG;
    if (batch == 0 || n == 0) return BF1_OK;
    if (!row_ptr || (nnz > 0 && !col_idx)) return BF1_ERR_INVALID_ARG;
    if (!aligned(row_ptr, 4) || (col_idx && !aligned(col_idx, 4))) return BF1_ERR_INVALID_ARG;
    bf1::AttnArgs a{Q, K, V, O, LSE, row_ptr, col_idx, nnz, batch, n, Hq, Hkv, head_dim, B, 0, false};
    return run_attn(a, (hipStream_t)stream);
}

int bf1_dense_causal_fwd(const void* Q, const void* K, const void* V, void* O, float* LSE,
                         int32_t batch, int64_t n, int32_t Hq, int32_t Hkv, int32_t head_dim,
                         void* stream) {
    int st = check_attn(Q, K, V, O, LSE, batch, n, Hq, Hkv, head_dim);
    if (st != BF1_OK) return st;
    if (batch == 0 || n == 0) return BF1_OK;
    bf1::AttnArgs a{Q, K, V, O, LSE, nullptr, nullptr, 0, batch, n, Hq, Hkv, head_dim, 64, 0, true};
    return run_attn(a, (hipStream_t)stream);
}

int bf1_attn_fwd_token_major(const void* Q, const void* K, const void* V, void* O, int32_t batch, int64_t n,
                             int32_t Hq, int32_t Hkv, int32_t head_dim, int32_t B, int32_t L, int32_t dense,
                             void* stream) {
    int st = check_attn(Q, K, V, O, nullptr, batch, n, Hq, Hkv, head_dim);
    if (st != BF1_OK) return st;
    if (dense != 0 && dense != 1) return BF1_ERR_INVALID_ARG;
    if (!dense && L < 0) return BF1_ERR_INVALID_ARG;
    if (!dense && B != 64 && B != 128) return BF1_ERR_UNSUPPORTED;
    if (batch == 0 || n == 0) return BF1_OK;
    hipStream_t s = (hipStream_t)stream;
    Plan plan;
    if (!dense) {
        st = get_plan(n, B, L, s, &plan);
        if (st != BF1_OK) return st;
    }
    bf1::AttnArgs a{Q, K, V, O, nullptr, nullptr, nullptr, plan.nnz, batch, n, Hq, Hkv, head_dim,
                    dense ? 64 : B, L, dense == 1};
    a.token_major = true;
    return run_attn(a, s);
}

int bf1_plan_transposed(int64_t n, int32_t B, int32_t L, int32_t* row_ptr, int32_t* col_idx,
                        int64_t col_capacity) {
    if (n < 0 || B < 1 || L < 0 || col_capacity < 0 || !row_ptr) return BF1_ERR_INVALID_ARG;
    int64_t NB, nnz;
    if (!route_sizes(n, B, L, &NB, &nnz)) return BF1_ERR_INVALID_ARG;
    if (nnz > 0 && !col_idx) return BF1_ERR_INVALID_ARG;
    if (col_capacity < nnz) return BF1_ERR_BUFFER_TOO_SMALL;
    int64_t e = 0;
    for (int64_t i = 0; i < NB; ++i) {
        row_ptr[i] = (int32_t)e;
        e += bf1::route_users(NB, L, i, col_idx ? col_idx + e : nullptr);
    }
    row_ptr[NB] = (int32_t)e;
    return e == nnz ? BF1_OK : BF1_ERR_INVALID_ARG;
}

int bf1_plan_variant(int32_t kind, int64_t n, int32_t B, int32_t L, uint64_t seed, int32_t* row_ptr,
                     int32_t* col_idx, int64_t col_capacity) {
    if (kind != BF1_ROUTE_BF1 && kind != BF1_ROUTE_SLIDING && kind != BF1_ROUTE_STATIC_RANDOM)
        return BF1_ERR_INVALID_ARG;
    if (n < 0 || B < 1 || L < 0 || col_capacity < 0 || !row_ptr) return BF1_ERR_INVALID_ARG;
    int64_t NB, nnz;
    if (!route_sizes(n, B, L, &NB, &nnz)) return BF1_ERR_INVALID_ARG;
    if (nnz > 0 && !col_idx) return BF1_ERR_INVALID_ARG;
    if (col_capacity < nnz) return BF1_ERR_BUFFER_TOO_SMALL;
    int64_t e = 0;
    for (int64_t j = 0; j < NB; ++j) {
        row_ptr[j] = (int32_t)e;
        if (kind == BF1_ROUTE_BF1) {
            // Eq. 1, ascending: block 0, dyadics from the farthest, locals, self
            const int64_t start = e;
            if (j > L) col_idx[e++] = 0;
            int r = 2;
            while (r < 62 && (int64_t(1) << (r + 1)) <= j) ++r;
            for (; r >= 2; --r) {
                const int64_t off = int64_t(1) << r;
                if (off <= j && off > L && j - off > 0) col_idx[e++] = (int32_t)(j - off);
            }
            for (int64_t t = (j - L > 0 ? j - L : 0); t <= j; ++t) col_idx[e++] = (int32_t)t;
            if (e - start != 1 + bf1::route_pred_count(j, L)) return BF1_ERR_INVALID_ARG;
        } else if (kind == BF1_ROUTE_SLIDING) {
            e += bf1::route_sliding_row(j, L, col_idx + e);
        } else {
            e += bf1::route_static_random_row(j, L, seed, col_idx + e);
        }
    }
    row_ptr[NB] = (int32_t)e;
    return e == nnz ? BF1_OK : BF1_ERR_INVALID_ARG;
}

int bf1_route_depth(const int32_t* row_ptr, const int32_t* col_idx, int32_t num_blocks,
                    int32_t* max_depth) {
    if (num_blocks < 0 || num_blocks > 16384 || !row_ptr || !max_depth) return BF1_ERR_INVALID_ARG;
    const int32_t NB = num_blocks;
    if (row_ptr[0] != 0) return BF1_ERR_INVALID_ARG;
    for (int32_t j = 0; j < NB; ++j)
        if (row_ptr[j + 1] < row_ptr[j]) return BF1_ERR_INVALID_ARG;
    if (row_ptr[NB] > 0 && !col_idx) return BF1_ERR_INVALID_ARG;
    // successor lists: edge i -> j for every earlier block i in row j
    std::vector<int32_t> deg(NB + 1, 0);
    for (int32_t j = 0; j < NB; ++j)
        for (int32_t e = row_ptr[j]; e < row_ptr[j + 1]; ++e) {
            const int32_t i = col_idx[e];
            if (i < 0 || i > j) return BF1_ERR_INVALID_ARG;
            if (i < j) ++deg[i + 1];
        }
    for (int32_t i = 0; i < NB; ++i) deg[i + 1] += deg[i];
    std::vector<int32_t> succ(deg[NB]), fill(deg.begin(), deg.end() - 1);
    for (int32_t j = 0; j < NB; ++j)
        for (int32_t e = row_ptr[j]; e < row_ptr[j + 1]; ++e)
            if (col_idx[e] < j) succ[fill[col_idx[e]]++] = j;
    // breadth-first search from every source; edges only go forward, so a
    // source's search touches blocks src..NB-1 only
    std::vector<int32_t> dist(NB), queue(NB);
    int32_t worst = 0;
    for (int32_t src = 0; src < NB; ++src) {
        std::fill(dist.begin() + src, dist.end(), -1);
        dist[src] = 0;
        int32_t head = 0, tail = 0;
        queue[tail++] = src;
        while (head < tail) {
            const int32_t u = queue[head++];
            for (int32_t e = deg[u]; e < deg[u + 1]; ++e) {
                const int32_t w = succ[e];
                if (dist[w] < 0) {
                    dist[w] = dist[u] + 1;
                    queue[tail++] = w;
                }
            }
        }
        if (tail != NB - src) {
            *max_depth = -1;
            return BF1_OK;
        }
        worst = std::max(worst, dist[queue[tail - 1]]);
    }
    *max_depth = worst;
    return BF1_OK;
}

int bf1_attn_bwd_workspace_size(int32_t batch, int64_t n, int32_t Hq, int32_t Hkv,
                                int32_t head_dim, int32_t B, int32_t L, int64_t* bytes) {
    if (!bytes) return BF1_ERR_INVALID_ARG;
    int st = check_attn(nullptr, nullptr, nullptr, nullptr, nullptr, 0, n, Hq, Hkv, head_dim);
    if (st != BF1_OK) return st;
    if (batch < 0 || L < 0) return BF1_ERR_INVALID_ARG;
    if ((B != 64 && B != 128) || (Hq / Hkv) * B < 128) return BF1_ERR_UNSUPPORTED;
    return bwd_workspace_bytes(batch, n, Hq, Hkv, head_dim, B, L, bytes);
}

int bf1_attn_bwd(const void* Q, const void* K, const void* V, const void* O, const void* dO,
                 const float* LSE, float* dQ, float* dK, float* dV, int32_t batch, int64_t n,
                 int32_t Hq, int32_t Hkv, int32_t head_dim, int32_t B, int32_t L, void* workspace,
                 int64_t workspace_bytes, void* stream) {
    int st = check_attn(Q, K, V, const_cast<void*>(O), nullptr, batch, n, Hq, Hkv, head_dim);
    if (st != BF1_OK) return st;
    if (L < 0 || workspace_bytes < 0) return BF1_ERR_INVALID_ARG;
    if ((B != 64 && B != 128) || (Hq / Hkv) * B < 128) return BF1_ERR_UNSUPPORTED;
    if (batch == 0 || n == 0) return BF1_OK;
    if (!dO || !LSE || !dQ || !dK || !dV || !workspace) return BF1_ERR_INVALID_ARG;
    if (!aligned(dO, 16) || !aligned(dQ, 16) || !aligned(dK, 16) || !aligned(dV, 16) ||
        !aligned(LSE, 4) || !aligned(workspace, 256))
        return BF1_ERR_INVALID_ARG;
    int64_t need = 0;
    st = bwd_workspace_bytes(batch, n, Hq, Hkv, head_dim, B, L, &need);
    if (st != BF1_OK) return st;
    if (workspace_bytes < need) return BF1_ERR_BUFFER_TOO_SMALL;
    hipStream_t s = (hipStream_t)stream;
    Plan plan;
    st = get_plan(n, B, L, s, &plan);
    if (st != BF1_OK) return st;
    BwdPlan bp;
    st = get_bwd_plan(n, B, L, s, &bp);
    if (st != BF1_OK) return st;
    const int64_t delta_bytes = ((int64_t)batch * Hq * n * 4 + 255) / 256 * 256;
    float* delta = (float*)workspace;
    float* lse2 = (float*)((char*)workspace + delta_bytes);
    const int64_t ds_bytes = (int64_t)batch * Hq * bp.nusers * (B / 64) * (B / 64) * 64 * 64 * 2;
    void* ds = (char*)workspace + need - ds_bytes;
    const BwdCut& cut = pick_cut(bp, n, B, (int64_t)batch * Hkv, Hq / Hkv);
    float* part = cut.len == SEG_MAX ? (float*)((char*)workspace + 2 * delta_bytes) : dQ;
    bf1::BwdArgs a{Q, K, V, O, dO, LSE, dQ, dK, dV, delta, lse2, part, ds,
                   plan.row_ptr, plan.col_idx, plan.nnz, bp.users, bp.uoffs, bp.nusers, cut.segs, cut.nseg,
                   cut.reds, cut.nred, cut.nslots, batch, n, Hq, Hkv, B, head_dim, L};
    return status_of(bf1::launch_backward(a, s));
}

int bf1_set_forward_key_split(int32_t mode) {
    if (mode < 0 || mode > 2) return BF1_ERR_INVALID_ARG;
    g_key_split.store(mode, std::memory_order_relaxed);
    return BF1_OK;
}

void bf1_release_plans(void) {
    std::lock_guard<std::mutex> lock(g_mu);
    if (!g_plans.empty() || !g_bwd_plans.empty()) (void)hipDeviceSynchronize();
    for (auto& kv : g_plans) {
        (void)hipFree(kv.second.row_ptr);
        (void)hipFree(kv.second.col_idx);
    }
    g_plans.clear();
    for (auto& kv : g_bwd_plans) (void)hipFree(kv.second.memory);
    g_bwd_plans.clear();
}

int bf1_decode_plan_stride(int64_t max_seq_len, int32_t B, int32_t L, int32_t dense, int32_t* stride) {
    if (!stride || max_seq_len < 1 || L < 0 || L > 32 || (dense != 0 && dense != 1))
        return BF1_ERR_INVALID_ARG;
    if (B != 64 && B != 128) return BF1_ERR_UNSUPPORTED;
    if (max_seq_len >= (int64_t(1) << 31)) return BF1_ERR_INVALID_ARG;
    int64_t cap;
    if (!decode_cap(max_seq_len, B, L, dense != 0, &cap)) return BF1_ERR_INVALID_ARG;
    *stride = (int32_t)(3 + cap);
    return BF1_OK;
}

int bf1_decode_plan(int32_t batch, const int32_t* seq_lens, const int32_t* page_table,
                    int32_t max_pages_per_seq, int32_t num_pages, int32_t B, int32_t L, int32_t dense,
                    int32_t* plan, int32_t plan_stride, void* stream) {
    if (batch < 0 || L < 0 || L > 32 || (dense != 0 && dense != 1)) return BF1_ERR_INVALID_ARG;
    if (B != 64 && B != 128) return BF1_ERR_UNSUPPORTED;
    if (max_pages_per_seq < 1 || num_pages < 1 || plan_stride < 3) return BF1_ERR_INVALID_ARG;
    if (batch == 0) return BF1_OK;
    if (!seq_lens || !page_table || !plan) return BF1_ERR_INVALID_ARG;
    if (!aligned(seq_lens, 4) || !aligned(page_table, 4) || !aligned(plan, 4)) return BF1_ERR_INVALID_ARG;
    bf1::DecodePlanArgs a{batch, seq_lens, page_table, max_pages_per_seq, num_pages, B, L, dense,
                          plan, plan_stride, plan_stride - 3};
    return status_of(bf1::launch_decode_plan(a, (hipStream_t)stream));
}

int bf1_decode_workspace_size(int32_t batch, int32_t Hq, int32_t Hkv, int32_t head_dim,
                              int32_t plan_stride, int64_t* bytes) {
    if (!bytes || batch < 0 || Hq < 1 || Hkv < 1 || Hq % Hkv != 0 || plan_stride < 3)
        return BF1_ERR_INVALID_ARG;
    if (head_dim != 64 && head_dim != 128) return BF1_ERR_UNSUPPORTED;
    *bytes = decode_ws_bytes(batch, Hq, Hkv, head_dim, decode_ws_splits(batch, Hkv, (int64_t)plan_stride - 2));
    return BF1_OK;
}

int bf1_decode_attn(const void* Q, const void* K_pages, const void* V_pages, const int32_t* seq_lens,
                    int32_t num_pages, const int32_t* plan, int32_t plan_stride, void* O, float* LSE,
                    int32_t batch, int32_t Hq, int32_t Hkv, int32_t head_dim, int32_t B,
                    void* workspace, int64_t workspace_bytes, void* stream) {
    if (batch < 0 || Hq < 1 || Hkv < 1 || Hq % Hkv != 0) return BF1_ERR_INVALID_ARG;
    if (num_pages < 1 || plan_stride < 3) return BF1_ERR_INVALID_ARG;
    const int32_t G = Hq / Hkv;
    if (head_dim != 64 && head_dim != 128) return BF1_ERR_UNSUPPORTED;
    if (B != 64 && B != 128) return BF1_ERR_UNSUPPORTED;
    if (G != 1 && G != 2 && G != 4 && G != 8) return BF1_ERR_UNSUPPORTED;
    if ((int64_t)batch * Hkv > (int64_t(1) << 22)) return BF1_ERR_INVALID_ARG;
    if ((double)num_pages * Hkv * B * head_dim > 4.0e18) return BF1_ERR_INVALID_ARG;
    if (batch == 0) return BF1_OK;
    if (!Q || !K_pages || !V_pages || !seq_lens || !plan || !O || !workspace) return BF1_ERR_INVALID_ARG;
    if (!aligned(Q, 16) || !aligned(K_pages, 16) || !aligned(V_pages, 16) || !aligned(O, 16) ||
        !aligned(workspace, 16) || !aligned(seq_lens, 4) || !aligned(plan, 4))
        return BF1_ERR_INVALID_ARG;
    if (LSE && !aligned(LSE, 4)) return BF1_ERR_INVALID_ARG;
    const int64_t P = (int64_t)plan_stride - 2;
    if (workspace_bytes < decode_ws_bytes(batch, Hq, Hkv, head_dim, decode_ws_splits(batch, Hkv, P)))
        return BF1_ERR_BUFFER_TOO_SMALL;
    int32_t nsplit, ppw;
    decode_splits(batch, Hkv, G, head_dim, B, P, &nsplit, &ppw);
    bf1::DecodeArgs a{Q, K_pages, V_pages, seq_lens, num_pages, plan, plan_stride, plan_stride - 3, O,
                      LSE, (float*)workspace, batch, Hq, Hkv, head_dim, B, nsplit, ppw};
    return status_of(bf1::launch_decode(a, (hipStream_t)stream));
}

}  // extern "C"
