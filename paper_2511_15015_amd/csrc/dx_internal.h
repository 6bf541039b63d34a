// Internal declarations shared by the translation units of libdynaexq.so.
#pragma once

#include <hip/hip_runtime.h>

#include <array>
#include <cstdint>
#include <cstdio>
#include <deque>
#include <string>
#include <vector>

#include "dynaexq.h"

typedef uint16_t dx_bf16; // bit pattern

struct dx_block_pool {
    char *base = nullptr;
    size_t block_bytes = 0;
    int n_blocks = 0;
    std::vector<int> free_list;           // LIFO of free block indices
    std::vector<hipEvent_t> reuse_after;  // per block: compute-stream event to pass before reuse (or null)
    void *block_ptr(int i) const { return base + (size_t)i * block_bytes; }
};

struct dx_entry {
    uint8_t state = DX_STATE_EMPTY;
    int8_t pool = -1;        // -1: caller-owned memory, 0: pool_hi, 1: pool_lo
    int32_t block = -1;      // block index of the published version
    int32_t next_block = -1; // block being filled by an in-flight transition
    dx_handle h{};           // host mirror of the published handle
};

struct dx_packed_host {
    const void *p[6] = {nullptr, nullptr, nullptr, nullptr, nullptr, nullptr}; // q_gate q_up q_down s_gate s_up s_down
};

struct dx_request {
    int layer, expert;
    bool promote;
};

struct dx_transition {
    int layer, expert;
    bool promote;
    hipEvent_t done;
};

// Timing events of one profiled forward call.  ev[0..3]: before gate/up, after it, after down, after
// combine; ev[7], ev[4]: two records back to back (what an event pair itself adds).  Calls of the streaming kernels and of
// thin tiles alone set per_kernel: there ev[0]/ev[1], ev[5]/ev[2] and ev[6]/ev[3] are the start and stop stamps of the three
// kernels' own dispatches (attached to the launches), not records between them.  Tiles of several kinds: records between
// the phases.
struct dx_marks {
    hipEvent_t ev[8];
    bool per_kernel;
    bool combined; // the down kernel wrote y: no combine kernel, ev[6] and ev[3] are not recorded
};

struct dx_ctx {
    dx_config cfg{};
    int device = 0;
    int n_cu = 0; // compute units of the device: size of the persistent grids
    hipStream_t compute = nullptr;
    hipStream_t mig = nullptr;
    std::string err;

    // handle tables: routed [L*E] then shared [L]
    dx_handle *d_table = nullptr;
    std::vector<dx_entry> entries; // L*E routed + L shared

    // hotness
    unsigned long long *d_counters = nullptr; // [L*E]
    long long *h_counters = nullptr;          // pinned [L*E]
    std::vector<uint64_t> scores;             // host S, Q16

    // routing scratch (chunks of 64 tokens)
    int n_chunks_max = 0;
    unsigned long long *d_mask = nullptr; // [n_chunks_max, E]
    int32_t *d_mask_sums = nullptr;       // [ceil(n_chunks_max / DX_SUM_CHUNKS), E]

    // forward scratch
    dx_bf16 *d_h = nullptr; // [max_tokens*(k+1), fmax]
    float *d_o = nullptr;   // [max_tokens*(k+1), d]
    struct dx_tile_head *d_tiles = nullptr; // row tiles of the tiled experts of one call (or the experts of its few places)
    int fmax = 0;

    // pools / budget tracker / transitions
    dx_block_pool pool_hi, pool_lo;
    char *staging = nullptr;
    uint64_t b_hi = 0, b_lo = 0, b_shared = 0;
    uint64_t reserved = 0;
    std::vector<int> hi_count; // per layer: Resident-Hi + Promoting
    int n_hi_cap = 0;          // per-layer capacity from the budget rule
    std::deque<dx_transition> inflight;
    std::deque<dx_request> update_q;                       // waiting promotions and demotions, in arrival order
    std::vector<std::array<const void *, 3>> host_master; // per routed entry: pinned bf16 gate/up/down or nulls
    int max_inflight = 0;                                  // 0: unbounded
    // quantized precision pair: pre-packed versions in pinned host memory, [0] high tier, [1] low tier
    std::vector<dx_packed_host> host_packed[2];
    std::vector<hipEvent_t> event_pool;
    dx_stats stats{};

    // optional per-kernel timing of the forward pass
    bool profiling = false;
    std::vector<hipEvent_t> timing_pool;           // free timing-enabled events
    std::vector<dx_marks> marks;                   // one per profiled forward call
};

#define DX_FAIL(ctx, code, ...)                                   \
    do {                                                          \
        char _buf[512];                                           \
        snprintf(_buf, sizeof _buf, __VA_ARGS__);                 \
        if (ctx) (ctx)->err = _buf;                               \
        return (code);                                            \
    } while (0)

#define DX_HIP(ctx, call)                                                                  \
    do {                                                                                   \
        hipError_t _e = (call);                                                            \
        if (_e != hipSuccess)                                                              \
            DX_FAIL(ctx, DX_ERR_HIP, "%s failed: %s (%s:%d)", #call, hipGetErrorString(_e), \
                    __FILE__, __LINE__);                                                   \
    } while (0)

constexpr int DX_ROUTE_CHUNK = 64; // tokens of a routing chunk; calls of one chunk are routed by one kernel
constexpr int DX_SUM_CHUNKS = 32; // chunks whose population counts are added up together in large batches
// What the list of row tiles is made from, beside the segments
struct dx_list_args {
    const dx_handle *table;
    struct dx_tile_head *tiles; // null: no list
    int T, E, k, m_big, n_cu;
    int shared;    // the layer has a shared expert
    int thin_only; // all segments in tiles of DX_THIN_ROWS rows
};
// ---- kernel launchers (each validates nothing; callers validate) ----------
// dx_route.hip
hipError_t dxk_route(const float *logits, int T, int E, int k, int32_t *ids, float *w, int32_t *counts,
                     int32_t *offsets, int32_t *perm, unsigned long long *mask, int32_t *sums,
                     unsigned long long *hotness /* window counters of the layer, or null */,
                     const dx_list_args &list /* of row tiles; batches of several chunks write it too */, hipStream_t s);
hipError_t dxk_router_gemm(const dx_bf16 *x, const dx_bf16 *w_r, const float *bias, int T, int E, int d, float *logits,
                           int n_cu, hipStream_t s);
hipError_t dxk_hotness_add(unsigned long long *counters, const int32_t *counts, int E, hipStream_t s);
hipError_t dxk_fill_u64(unsigned long long *p, size_t n, unsigned long long v, hipStream_t s);
hipError_t dxk_store_handle(dx_handle *slot, const dx_handle &h, hipStream_t s);
hipError_t dxk_probe_read(const void *buf, size_t bytes, int n_cu, hipStream_t s); // bytes: whole MiB are read

// dx_quantize.hip
hipError_t dxk_quantize(const dx_bf16 *w, int rows, int K, int group, uint8_t *q, dx_bf16 *sc, hipStream_t s);
hipError_t dxk_quantize2(const dx_bf16 *w, int rows, int K, int group, uint8_t *q, dx_bf16 *sc, hipStream_t s); // 2-bit

// dx_moe_decode.hip / dx_moe_prefill.hip
// The list of row tiles of a call: a head, then the rows: 128-row tiles of the routed experts, of the shared one, 256-row tiles likewise, thin tiles.
constexpr int DX_TILE_ROWS = 128, DX_BIG_ROWS = 256, DX_THIN_ROWS = 32;
struct dx_tile_row {
    int e, mt;   // expert (E = shared), row tile of the rows below
    int m, seg0; // rows and first pair slot of the segment, or of the part of it that this tile size takes
};
struct dx_tile_head {
    int n_routed, n_shared;  // 128-row tiles of the routed experts, of the shared one
    int n_quant;             // of the former, those of quantized experts
    int n_single;            // and those of experts with one only
    int n_big, n_big_shared; // 256-row tiles
    int n_thin, n_thin_quant, n_thin_shared; // thin tiles' rows: of bf16 experts, of quantized ones, of the shared one
    int n_cu;
};
// most row tiles that segments of more than m_min rows can have in a call of T tokens (a routed expert has ceil(m / 128) of them)
inline long dxk_tile_rows_max(int T, int k, int E, int m_min, bool shared)
{
    const long pairs = (long)T * k, with = pairs / ((long)m_min + 1) < E ? pairs / ((long)m_min + 1) : E;
    // (256 rows in one 256-row tile are fewer tiles than in two of 128)
    return pairs / DX_TILE_ROWS + with + (shared ? (T + DX_TILE_ROWS - 1) / DX_TILE_ROWS : 0);
}
// and most rows of thin tiles when all segments are in them
inline long dxk_thin_rows_max(int T, int k, int E, bool shared)
{
    const long pairs = (long)T * k;
    return pairs / DX_THIN_ROWS + (pairs < E ? pairs : E) + (shared ? (T + DX_THIN_ROWS - 1) / DX_THIN_ROWS : 0);
}
constexpr int DX_FP32_TOKENS = 128; // calls of up to so many tokens (and larger ones on the streaming kernels) keep O in fp32 and never round a quantized weight
// Calls of so few tokens (and top-k up to DX_ROUTED_MAX_TOPK) run the down projection and the combine in one kernel
constexpr int DX_FEW_TOKENS = 2;
struct dx_fwd_args {
    const dx_handle *table;  // E routed entries of the layer
    const dx_handle *shared; // one entry or null
    const dx_bf16 *x;
    dx_bf16 *y;
    const int32_t *ids;
    const float *w;
    const int32_t *offsets;
    const int32_t *perm;
    dx_bf16 *h;  // scratch [T*k (+T), fmax]
    float *o;    // scratch [T*k (+T), d]: fp32, or (tiles) bf16 in the same allocation
    int T, E, k, d, f, group, shared_f, fmax;
    int o_bf16;  // O rows are bf16 (prefill: halves the traffic between the down kernels and the combine), else fp32
    int m_big;   // formats whose segments' whole 256 rows go in 256-row tiles: bit 0 bf16, bit 1 int4 (the values of dx_fmt)
    int any_quantized; // some routed expert of the table may be (a caller's table: unknown)
    // A list for the kernels of a call, or null: calls on tiles: the row tiles; up to DX_FEW_TOKENS tokens on a caller's
    // routing arrays: the expert of every place in the segments, as int32_t, which the gate/up kernel leaves for the down kernel.
    dx_tile_head *tiles;
    bool listed; // the row tiles are listed already (by the routing kernels in front)
};
// Decode batches that the gate/up kernel routes itself (dx_route_forward): what its first block reads and
// writes on top of dx_fwd_args (whose ids, w, offsets and perm point at the same arrays for the kernels
// that follow)
constexpr int DX_ROUTED_MAX_TOKENS = 64, DX_ROUTED_MAX_EXPERTS = 512, DX_ROUTED_MAX_TOPK = 16;
struct dx_route_io {
    const float *logits; // [T, E]
    int32_t *ids;        // [T, k]
    float *w;            // [T, k]
    int32_t *counts;     // [E]
    int32_t *offsets;    // [E + 1]
    int32_t *perm;       // [T * k]
    unsigned long long *hotness; // the layer's window counters, or null
};
// The list that a call's tiles need (tiles null: the call does not run on tiles)
dx_list_args dxk_list_args(const dx_fwd_args &a, int n_cu);
hipError_t dxk_moe_forward(const dx_fwd_args &a, int n_cu, hipStream_t s, dx_marks *marks);
// Routing and forward pass in one call.  Returns true in *routed when the gate/up kernel did the routing
// (small decode batches whose shapes fit); otherwise nothing was launched and the caller runs dxk_route
// and dxk_moe_forward.
hipError_t dxk_route_forward(const dx_fwd_args &a, const dx_route_io &r, int n_cu, hipStream_t s, dx_marks *marks,
                             bool *routed);
// dx_moe_prefill.hip: the list of row tiles of a call, and gate/up and down of its experts
void dxk_tile_list(const dx_list_args &l, const int32_t *offsets, hipStream_t s);
// (start, stop: events for the stamps of the kernel of a call of thin tiles alone, or null)
void dxk_tiles_gate_up(const dx_fwd_args &a, hipStream_t s, hipEvent_t start, hipEvent_t stop);
void dxk_tiles_down(const dx_fwd_args &a, hipStream_t s, hipEvent_t start, hipEvent_t stop);
