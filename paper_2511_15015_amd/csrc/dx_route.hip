// Router top-k, routing weights and the stable permutation of (token, slot)
// pairs into per-expert segments, plus the small table/counter kernels.
//
// Paper: Sec. 3.1 (the worker obtains top-k expert ids from the router and
// indexes the handle table with them); Sec. 3.5 (per-expert selection counts).
//
// Determinism: the order inside an expert segment is by increasing pair
// index p = t*k + j.  Because the k ids of one token are distinct, the rank of
// pair (t, j) inside the segment of expert e equals the number of tokens
// t' < t that selected e.  Tokens are handled in chunks of 64: each chunk
// builds, per expert, a 64-bit mask of the tokens that selected it; ranks are
// population counts of mask prefixes.  No atomics decide any position.
#include "dx_internal.h"
#include "dx_route_core.h"
#include "dx_tile_list.h"

#include <cfloat>
#include <cstdarg>
#include <mutex>

namespace {

constexpr int kChunk = DX_ROUTE_CHUNK;      // tokens per chunk = bits per mask word
constexpr int kRouteThreads = 1024;
constexpr int kWaves = kRouteThreads / 64;

// exclusive scan of one int per thread across a 1024-thread block
__device__ int block_exclusive_scan(int v, int *lds_wave_tot /*[kWaves]*/, int *total)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int inc = dx_route_core::wave_scan_inclusive(v);
    if (lane == 63) lds_wave_tot[wave] = inc;
    __syncthreads();
    int base = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        int t = lds_wave_tot[w];
        if (w < wave) base += t;
        tot += t;
    }
    __syncthreads();
    *total = tot;
    return base + inc - v;
}

// ROWS16 (layers of up to 512 experts): a token per 16-lane row, NV logits per lane of the row (E <= 16*NV), so
// a block's wavefronts take four tokens each in one pass (the selection code of the decode kernels' routing
// prologue).  Otherwise a token per wavefront, NV consecutive logits per lane (E <= 64*NV), four passes.
// WAVES 16: the call is one chunk of 64 tokens and one block, which finishes counts, offsets and permutation as well.
// WAVES 4: a quarter of a chunk per block, which leaves its 16 bits of the chunk's mask words (also where it has no
// tokens).  Four wavefronts share no SIMD, and a compute unit takes in 16 rows of logits instead of 64: with a whole chunk
// to a block of 16 wavefronts 128 experts, 101 tokens 5.5 us against 4.6 now, 4096 tokens 7.5 and 5.3; 512 experts,
// 1000 tokens 11.5 and 7.9.
template <int NV, bool ROWS16, int WAVES>
__global__ __launch_bounds__(64 * WAVES) void k_route_topk(
    const float *__restrict__ logits, int T, int E, int k, int32_t *__restrict__ ids, float *__restrict__ w,
    int32_t *__restrict__ counts, int32_t *__restrict__ offsets, int32_t *__restrict__ perm,
    unsigned long long *__restrict__ mask_out, unsigned long long *__restrict__ hotness, int n_chunks)
{
    constexpr bool fused = WAVES == kWaves;
    constexpr int THREADS = 64 * WAVES, TOKENS = 4 * WAVES;
    static_assert(fused || TOKENS == 16, "a block writes 16 bits of a mask word");
    extern __shared__ unsigned long long lds_mask[]; // [E], then int ids [64*k], then wave totals
    int *lds_ids = reinterpret_cast<int *>(lds_mask + E);
    int *lds_tot = lds_ids + TOKENS * k;

    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    // (the quarters of a chunk on one XCD, where their bits meet in the same lines)
    const int chunk = fused ? 0 : (int)(blockIdx.x >> 5) * 8 + (blockIdx.x & 7), part = fused ? 0 : (blockIdx.x >> 3) & 3;
    if (chunk >= n_chunks) return; // block-uniform
    const int first = chunk * kChunk + part * TOKENS;
    for (int e = threadIdx.x; e < E; e += THREADS) lds_mask[e] = 0ull;
    // single-chunk launch with the hotness update inside: fetch the counter now, it is added to at the end
    unsigned long long hot_before = 0ull;
    if (fused && hotness && (int)threadIdx.x < E) hot_before = hotness[threadIdx.x];
    __syncthreads();

    if constexpr (ROWS16) {
        const int tt = 4 * wave + (lane >> 4), t = first + tt, c = lane & 15;
        if (first + 4 * wave < T) { // wave-uniform: some row of this wavefront has a token (T > 0)
            float v[NV];
            dx_route_core::load_logits_rows16<NV>(logits + (size_t)(t < T ? t : T - 1) * E, c, E, v);
            int my_id;
            float my_w;
            if constexpr (NV <= 8) {
                dx_route_core::topk_rows16<NV>(v, k, lane, my_id, my_w);
            } else { // wide layers: a threshold first, then the selections over the few entries at or above it
                auto scratch = (__attribute__((address_space(3))) int *)(lds_tot + WAVES + (E + 3) / 4 * 4) + wave * 64 * NV;
                dx_route_core::topk_rows16_filtered<NV, 6>(v, k, lane, my_id, my_w, scratch);
            }
            if (t < T && c < k) {
                ids[(size_t)t * k + c] = my_id;
                w[(size_t)t * k + c] = my_w;
                lds_ids[tt * k + c] = my_id;
                atomicOr(&lds_mask[my_id], 1ull << tt);
            }
        }
    } else
    for (int tt = wave; tt < TOKENS; tt += WAVES) {
        const int t = first + tt;
        if (t >= T) break; // wave-uniform
        const float *row = logits + (size_t)t * E;
        float v[1][NV];
        if constexpr (NV >= 4) dx_route_core::load_logits<NV>(row, lane, E, v[0]);
        else {
#pragma unroll
            for (int s = 0; s < NV; ++s) {
                const int e = NV * lane + s;
                v[0][s] = e < E ? row[e < E ? e : E - 1] : -INFINITY;
            }
        }
        int id1[1];
        float wt1[1];
        dx_route_core::topk_rows<NV, 1>(v, k, lane, id1, wt1);
        const int my_id = id1[0];
        if (lane < k) {
            ids[(size_t)t * k + lane] = my_id;
            w[(size_t)t * k + lane] = wt1[0];
            lds_ids[tt * k + lane] = my_id;
            atomicOr(&lds_mask[my_id], 1ull << tt);
        }
    }
    __syncthreads();

    if constexpr (!fused) {
        uint16_t *out = reinterpret_cast<uint16_t *>(mask_out + (size_t)chunk * E) + part;
        for (int e = threadIdx.x; e < E; e += THREADS) out[4 * e] = (uint16_t)lds_mask[e];
        return;
    }
    // single chunk: finish counts, offsets and the permutation here (E <= 1024)
    const int e = threadIdx.x;
    const int c = e < E ? __popcll(lds_mask[e]) : 0;
    int total;
    const int off = block_exclusive_scan(c, lds_tot, &total);
    if (e < E) {
        counts[e] = c;
        offsets[e] = off;
        if (hotness) hotness[e] = hot_before + (unsigned long long)c;
        lds_ids[kChunk * k + kWaves + e] = off; // offsets kept in LDS after the wave totals
    }
    if (e == 0) offsets[E] = total;
    __syncthreads();
    const int *lds_off = lds_ids + kChunk * k + kWaves;
    const int P = T * k;
    for (int p = threadIdx.x; p < P; p += kRouteThreads) {
        const int tt = p / k;
        const int ex_id = lds_ids[p];
        const unsigned long long below = lds_mask[ex_id] & ((1ull << tt) - 1ull);
        perm[lds_off[ex_id] + __popcll(below)] = p;
    }
}

// Batches of several chunks: a block per chunk places the chunk's pairs.  It needs every expert's count and what the
// chunks before its own hold of it.  Every block adds up the population counts of all chunk masks by itself (64 KB from L2
// for 4096 tokens on 128 experts), S threads to an expert, because a kernel in between costs more (30B-shaped layer: a
// pass of 4096 tokens 492 us with a scan kernel, 482 without; of 300 tokens 140 and 138).  That work grows with the square
// of the batch: in large ones k_route_sums adds up groups of kSumChunks chunks first, and a block reads the sums and the
// masks of its own group.
constexpr int kSumChunks = DX_SUM_CHUNKS;

// threads per expert in a block of kRouteThreads (log2)
inline int route_split(int E)
{
    int split = 0;
    while ((E << (split + 1)) <= kRouteThreads && split < 6) ++split;
    return split;
}

__global__ __launch_bounds__(kRouteThreads) void k_route_sums(int E, int split, int n_chunks,
                                                              const unsigned long long *__restrict__ mask,
                                                              int32_t *__restrict__ sums)
{
    const int S = 1 << split, e = threadIdx.x >> split, part = threadIdx.x & (S - 1);
    const int c0 = blockIdx.x * kSumChunks, c1 = min(n_chunks, c0 + kSumChunks);
    int n = 0;
    if (e < E) {
#pragma unroll 8
        for (int c = c0 + part; c < c1; c += S) n += __popcll(mask[(size_t)c * E + e]);
    }
    for (int o = S >> 1; o > 0; o >>= 1) n += __shfl_xor(n, o, 64); // (an expert's threads are neighbours)
    if (part == 0 && e < E) sums[(size_t)blockIdx.x * E + e] = n;
}

// sums: of the groups of chunks (k_route_sums), or null
__global__ __launch_bounds__(kRouteThreads) void k_route_place(
    const int32_t *__restrict__ ids, int T, int E, int k, int split /* log2 of S */, int n_chunks,
    const unsigned long long *__restrict__ mask, const int32_t *__restrict__ sums, int32_t *__restrict__ counts,
    int32_t *__restrict__ offsets, int32_t *__restrict__ perm, unsigned long long *__restrict__ hotness, dx_list_args list)
{
    __shared__ unsigned long long lds_mask[kRouteThreads];
    __shared__ int lds_at[kRouteThreads]; // where the chunk's first pair of the expert goes
    __shared__ int lds_tot[kWaves];
    const bool lists = (int)blockIdx.x == n_chunks; // a block more: the list of row tiles
    const int chunk = lists ? 0 : blockIdx.x, S = 1 << split;
    const int p0 = chunk * kChunk * k, n = min(T - chunk * kChunk, kChunk) * k;
    // asked for here because the masks' way to the first use takes as long as theirs: the first pair's expert, the counter,
    // the expert's format
    const int first_id = ids[p0 + min((int)threadIdx.x, n - 1)];
    const int e = threadIdx.x >> split, part = threadIdx.x & (S - 1);
    const bool counts_hot = blockIdx.x == 0 && part == 0 && e < E && hotness;
    const unsigned long long hot_before = counts_hot ? hotness[e] : 0ull;
    const uint32_t fmt = lists && part == 0 && e < E ? list.table[e].fmt : (uint32_t)DX_FMT_BF16;
    int total = 0, before = 0;
    if (e < E) {
        constexpr int U = 8; // independent loads in flight
        const int group = chunk / kSumChunks;
        if (sums) {
            const int n_groups = (n_chunks + kSumChunks - 1) / kSumChunks;
            for (int g0 = part; g0 < n_groups; g0 += U * S) {
                int m[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int g = g0 + u * S;
                    m[u] = sums[(size_t)(g < n_groups ? g : n_groups - 1) * E + e];
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int g = g0 + u * S;
                    const int n = g < n_groups ? m[u] : 0;
                    total += n;
                    before += g < group ? n : 0;
                }
            }
        }
        const int first = sums ? group * kSumChunks : 0, end = sums ? chunk + 1 : n_chunks; // masks to read
        for (int c0 = first + part; c0 < end; c0 += U * S) {
            unsigned long long m[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int c = c0 + u * S;
                m[u] = mask[(size_t)(c < end ? c : end - 1) * E + e];
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int c = c0 + u * S;
                const int n = c < end ? __popcll(m[u]) : 0;
                if (!sums) total += n;
                before += c < chunk ? n : 0;
                if (c == chunk) lds_mask[e] = m[u];
            }
        }
    }
    for (int o = S >> 1; o > 0; o >>= 1) { // (an expert's threads are neighbours)
        total += __shfl_xor(total, o, 64);
        before += __shfl_xor(before, o, 64);
    }
    int all;
    const int off = block_exclusive_scan(part == 0 && e < E ? total : 0, lds_tot, &all);
    if (lists) { // block-uniform
        __shared__ dx_tile_list::lds<kWaves> of_list;
        const bool owner = part == 0 && e < E;
        dx_tile_list::write<kWaves>(list, owner ? e : E, fmt, off, owner ? total : 0, of_list);
        return;
    }
    if (part == 0 && e < E) {
        lds_at[e] = off + before;
        if (chunk == 0) {
            counts[e] = total;
            offsets[e] = off;
            if (counts_hot) hotness[e] = hot_before + (unsigned long long)total;
            if (e == 0) offsets[E] = all;
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < n; i += kRouteThreads) {
        const int ex = i == (int)threadIdx.x ? first_id : ids[p0 + i];
        const unsigned long long below = lds_mask[ex] & ((1ull << (i / k)) - 1ull);
        perm[lds_at[ex] + __popcll(below)] = p0 + i;
    }
}

__global__ void k_hotness_add(unsigned long long *__restrict__ counters, const int32_t *__restrict__ counts, int E)
{
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e < E) counters[e] += (unsigned long long)counts[e];
}

__global__ void k_fill_u64(unsigned long long *p, size_t n, unsigned long long v)
{
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

// Measurement aid: a streaming read as fast as this chip does one (whole lines per load instruction,
// non-temporal hint, as the decode kernels' weight stream).  Block b reads the 1 MiB units b, b + grid, ...;
// 16 bytes per thread and load, eight loads in flight per thread.  What it reads is folded into a value that
// is never equal to the magic number, so the loads cannot be dropped and nothing is written.
__global__ __launch_bounds__(512) void k_probe_read(const char *__restrict__ p, int n_units, unsigned *sink)
{
    typedef __attribute__((ext_vector_type(4))) unsigned u32x4;
    constexpr size_t kUnit = 1u << 20;
    u32x4 acc = {0u, 0u, 0u, 0u};
    for (int u = blockIdx.x; u < n_units; u += gridDim.x) {
        const char *base = p + (size_t)u * kUnit + threadIdx.x * 16;
        for (size_t o = 0; o < kUnit; o += (size_t)8 * 512 * 16) {
            u32x4 v[8];
#pragma unroll
            for (int i = 0; i < 8; ++i)
                v[i] = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(base + o + (size_t)i * 512 * 16));
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                acc.x ^= v[i].x; acc.y ^= v[i].y; acc.z ^= v[i].z; acc.w ^= v[i].w;
            }
        }
    }
    if ((acc.x ^ acc.y ^ acc.z ^ acc.w) == 0x5EED1E55u && sink) *sink = 1u;
}

__global__ void k_store_handle(dx_handle *slot, dx_handle h)
{
    if (threadIdx.x == 0 && blockIdx.x == 0) *slot = h;
}

// Router gate: logits = x . W_r^T (+ bias).  Bound by latency for decode batches (2 MB of W_r at most: a fraction
// of a microsecond at the HBM rate) and by what a compute unit can take in for prefill batches.  A block
// computes 16*MT tokens x 16*NT experts and its WAVES wavefronts split K, so every operand byte of the tile
// enters the compute unit once and no second kernel or atomic is needed; the partial tiles meet in LDS and are
// added in the order of the wavefronts.
// A compute unit takes in 120 GB/s from L2 when eight neighbouring lanes read one 128-byte line, but only 37 GB/s
// in the operand order of v_mfma_f32_16x16x32_bf16 (lane (r, q): row r, 16 bytes at 64 bytes of 16 rows per
// instruction; the same for lines of 8 rows whose lanes are not neighbours).  So a wavefront loads whole lines
// (8 rows x 128 bytes per instruction, two lines of every row in flight), passes each line through a stage of
// LDS of its own (piece p of row r in slot p ^ ((r >> 1) & 7): no bank conflicts) and reads the operands there.
// Per call, d = 2048: 32 tokens x 512 experts 4.2 us, 4096 x 128 9.5 us (13.4 and 17.0 us with 32 x 32 tiles of 4
// wavefronts straight from global memory).
typedef __attribute__((ext_vector_type(8))) __bf16 rt_bf16x8;
typedef __attribute__((ext_vector_type(4))) float rt_f32x4;
typedef __attribute__((ext_vector_type(4))) uint32_t rt_u32x4;

template <int MT, int NT, int WAVES>
__global__ __launch_bounds__(WAVES * 64) void k_router_gemm(const dx_bf16 *__restrict__ x, const dx_bf16 *__restrict__ w_r,
                                                            const float *__restrict__ bias, int T, int E, int d,
                                                            int by_xcd, float *__restrict__ logits)
{
    constexpr int ROWS = 16 * MT, COLS = 16 * NT, LOADS = 2 * (MT + NT); // LOADS: eight-row groups of a line
    constexpr int kStage = LOADS * 1024;
    constexpr int kPart = MT * NT * 1024;
    __shared__ __attribute__((aligned(128))) char lds[WAVES * (kStage > kPart ? kStage : kPart)];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // by_xcd: block b runs on XCD b % 8; the column tiles of a row tile go to one XCD, so that its x rows are read
    // into one L2 only (row tiles are padded to a multiple of 8).
    const int ncol = (E + COLS - 1) / COLS, at_xcd = blockIdx.x >> 3;
    const int t0 = (by_xcd ? (at_xcd / ncol) * 8 + (blockIdx.x & 7) : blockIdx.x / ncol) * ROWS;
    const int e0 = (by_xcd ? at_xcd % ncol : blockIdx.x % ncol) * COLS;
    if (t0 >= T) return;
    // loader: piece lane % 8 of row lane / 8 of every group.  Rows past the end repeat the last one; never stored.
    const int piece = lane & 7;
    const dx_bf16 *row[LOADS];
#pragma unroll
    for (int i = 0; i < LOADS; ++i) {
        const int rr = 8 * i + (lane >> 3);
        row[i] = i < 2 * MT ? x + (size_t)min(t0 + rr, T - 1) * d : w_r + (size_t)min(e0 + rr - ROWS, E - 1) * d;
    }
    const int nlines = (d + 63) / 64, nsteps = d / 32; // the last line may be half a line: its second step is left out
    const int per = (nlines + WAVES - 1) / WAVES;      // consecutive lines of a row to a wavefront
    const int l0 = wave * per, l1 = min(nlines, l0 + per);
    auto load_line = [&](int l, rt_u32x4 (&v)[LOADS]) {
        l = max(min(l, l1 - 1), 0);
        const int at = l * 64 + (2 * l + 1 < nsteps ? piece : piece & 3) * 8;
#pragma unroll
        for (int i = 0; i < LOADS; ++i) v[i] = *reinterpret_cast<const rt_u32x4 *>(row[i] + at);
    };
    char *stage = lds + wave * kStage;
    const int put = (lane >> 3) * 128 + (piece ^ ((lane >> 4) & 3)) * 16; // + 1024 per group, the swizzle's third bit below
    const int r = lane & 15, q = lane >> 4;
    rt_f32x4 acc[MT][NT];
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int n = 0; n < NT; ++n) acc[m][n] = rt_f32x4{0.f, 0.f, 0.f, 0.f};
    union frag {
        rt_u32x4 u;
        rt_bf16x8 v;
    };
    auto multiply_line = [&](int l, const rt_u32x4 (&v)[LOADS]) {
#pragma unroll
        for (int i = 0; i < LOADS; ++i) // row 8 * i + lane / 8: bit 2 of (row >> 1) & 7 is i & 1
            *reinterpret_cast<rt_u32x4 *>(stage + i * 1024 + (put ^ ((i & 1) * 64))) = v[i];
        // (no instruction: the wavefront's LDS accesses stay in order in the hardware, and here in the compiler, which sees
        // that a lane reads other addresses than it wrote)
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            if (2 * l + h >= nsteps) break; // wavefront-uniform
            frag a[MT], b[NT];
            const int slot = ((q + 4 * h) ^ ((r >> 1) & 7)) * 16;
#pragma unroll
            for (int m = 0; m < MT; ++m) a[m].u = *reinterpret_cast<const rt_u32x4 *>(stage + (16 * m + r) * 128 + slot);
#pragma unroll
            for (int n = 0; n < NT; ++n) b[n].u = *reinterpret_cast<const rt_u32x4 *>(stage + (ROWS + 16 * n + r) * 128 + slot);
#pragma unroll
            for (int m = 0; m < MT; ++m)
#pragma unroll
                for (int n = 0; n < NT; ++n)
                    acc[m][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[m].v, b[n].v, acc[m][n], 0, 0, 0);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    };
    rt_u32x4 v[2][LOADS];
    if (l0 < l1) { // wavefront-uniform
        load_line(l0, v[0]);
        load_line(l0 + 1, v[1]);
        for (int l = l0; l < l1; l += 2) { // loads past the end are duplicates that are not multiplied
            multiply_line(l, v[0]);
            load_line(l + 2, v[0]);
            if (l + 1 < l1) multiply_line(l + 1, v[1]);
            load_line(l + 3, v[1]);
        }
    }
    __syncthreads(); // the stages are free
    float *part = reinterpret_cast<float *>(lds); // [WAVES][MT * NT][4][64]
    // accumulator element v of lane (r, q): token row 4q + v, expert column r
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int n = 0; n < NT; ++n)
#pragma unroll
            for (int i = 0; i < 4; ++i) part[((wave * MT * NT + m * NT + n) * 4 + i) * 64 + lane] = acc[m][n][i];
    __syncthreads();
    for (int i = threadIdx.x; i < ROWS * COLS; i += WAVES * 64) { // in the order of `part`: no bank conflicts
        const int tile = i >> 8, tr = 16 * (tile / NT) + 4 * ((i & 63) >> 4) + ((i >> 6) & 3), ec = 16 * (tile % NT) + (i & 15);
        if (t0 + tr >= T || e0 + ec >= E) continue;
        float s = part[i];
#pragma unroll
        for (int w = 1; w < WAVES; ++w) s += part[w * ROWS * COLS + i];
        if (bias) s += bias[e0 + ec];
        logits[(size_t)(t0 + tr) * E + e0 + ec] = s;
    }
}

template <int NV, bool ROWS16>
hipError_t launch_topk(const float *logits, int T, int E, int k, int32_t *ids, float *w, int32_t *counts,
                       int32_t *offsets, int32_t *perm, unsigned long long *mask, unsigned long long *hotness,
                       int n_chunks, hipStream_t s)
{
    auto run = [&](auto kernel, int blocks, int waves) {
        size_t lds = (size_t)E * 8 + (size_t)(4 * waves * k + waves + (E + 3) / 4 * 4) * 4;
        if (ROWS16 && NV > 8) lds += (size_t)waves * 64 * NV * 4; // the wide selection's keys
        hipLaunchKernelGGL(kernel, dim3(blocks), dim3(64 * waves), lds, s, logits, T, E, k, ids, w, counts, offsets, perm, mask,
                           hotness, n_chunks);
        return hipGetLastError();
    };
    if (n_chunks == 1) return run(k_route_topk<NV, ROWS16, kWaves>, 1, kWaves);
    return run(k_route_topk<NV, ROWS16, 4>, (n_chunks + 7) / 8 * 32, 4);
}

} // namespace

hipError_t dxk_route(const float *logits, int T, int E, int k, int32_t *ids, float *w, int32_t *counts,
                     int32_t *offsets, int32_t *perm, unsigned long long *mask, int32_t *sums, unsigned long long *hotness,
                     const dx_list_args &list, hipStream_t s)
{
    // T == 0 still runs one (empty) chunk so that counts and offsets are written.
    const int n_chunks = T > 0 ? (T + kChunk - 1) / kChunk : 1;
    hipError_t e;
    // (k <= 16: a selected id per lane of the token's row)
    if (k <= 16 && E <= 64) e = launch_topk<4, true>(logits, T, E, k, ids, w, counts, offsets, perm, mask, hotness, n_chunks, s);
    else if (k <= 16 && E <= 128) e = launch_topk<8, true>(logits, T, E, k, ids, w, counts, offsets, perm, mask, hotness, n_chunks, s);
    else if (k <= 16 && E <= 256) e = launch_topk<16, true>(logits, T, E, k, ids, w, counts, offsets, perm, mask, hotness, n_chunks, s);
    else if (k <= 16 && E <= 512) e = launch_topk<32, true>(logits, T, E, k, ids, w, counts, offsets, perm, mask, hotness, n_chunks, s);
    else if (E <= 64) e = launch_topk<1, false>(logits, T, E, k, ids, w, counts, offsets, perm, mask, hotness, n_chunks, s);
    else if (E <= 128) e = launch_topk<2, false>(logits, T, E, k, ids, w, counts, offsets, perm, mask, hotness, n_chunks, s);
    else if (E <= 256) e = launch_topk<4, false>(logits, T, E, k, ids, w, counts, offsets, perm, mask, hotness, n_chunks, s);
    else if (E <= 512) e = launch_topk<8, false>(logits, T, E, k, ids, w, counts, offsets, perm, mask, hotness, n_chunks, s);
    else e = launch_topk<16, false>(logits, T, E, k, ids, w, counts, offsets, perm, mask, hotness, n_chunks, s);
    if (e != hipSuccess || n_chunks == 1) return e;
    const int split = route_split(E);
    // Mask words that all blocks read without the groups' sums: about 3 million of them (24 MB) cost as much as the sums (more
    // where every expert has one thread only, to whom the sums are dear as well).  us without and with them: 128 experts
    // 8192 tokens (2.1 M) 17.5 and 17.3, 16384 tokens 25.3 and 18.8; 256 experts 4096 tokens (1 M) 18.1 and 21.2, 8192 tokens
    // (4.2 M) 25.7 and 20.9; 512 experts 4096 tokens (2.1 M) 22.7 and 25.4, 8192 tokens 30.4 and 27.4; 1024 experts 4096 tokens
    // (4.2 M) 38.7 and 41.9, 8192 tokens 48.5 and 43.8; 65536 tokens on 128 to 1024 experts 248 to 590 and 41 to 160.
    const long long words = (long long)n_chunks * n_chunks * E;
    const bool direct = words <= (split == 0 ? 5000000 : 3000000);
    if (!direct)
        hipLaunchKernelGGL(k_route_sums, dim3((n_chunks + kSumChunks - 1) / kSumChunks), dim3(kRouteThreads), 0, s, E, split,
                           n_chunks, mask, sums);
    hipLaunchKernelGGL(k_route_place, dim3(n_chunks + (list.tiles ? 1 : 0)), dim3(kRouteThreads), 0, s, ids, T, E, k, split, n_chunks, mask,
                       static_cast<const int32_t *>(direct ? nullptr : sums), counts, offsets, perm, hotness, list);
    return hipGetLastError();
}

hipError_t dxk_router_gemm(const dx_bf16 *x, const dx_bf16 *w_r, const float *bias, int T, int E, int d, float *logits,
                           int n_cu, hipStream_t s)
{
    if (T == 0) return hipSuccess;
    // The smallest tile whose blocks run in one round on the chip; beyond that the tile that moves the fewest bytes
    // into the compute units (an x row is read E / 16*NT times, a W_r row T / 16*MT times).  Measured, d = 2048:
    // T = 300, E = 128: 4.0 us (16 x 16), 5.7 (32 x 32); T = 1000, E = 512: 16.8, 9.4, 8.5 (32 x 64), 11.9 (64 x 64);
    // T = 4096, E = 512: 27.0, 28.4 and 18.9 us from 32 x 32 up.
    const long cu = n_cu;
    auto blocks = [&](int rows, int cols) { return (long)((T + rows - 1) / rows) * ((E + cols - 1) / cols); };
    auto run = [&](auto kernel, int rows, int cols, int threads) {
        const int nrow = (T + rows - 1) / rows, ncol = (E + cols - 1) / cols;
        const int by_xcd = nrow >= 16 && ncol > 1;
        hipLaunchKernelGGL(kernel, dim3((by_xcd ? (nrow + 7) / 8 * 8 : nrow) * ncol), dim3(threads), 0, s, x, w_r, bias, T, E,
                           d, by_xcd, logits);
    };
    if (blocks(16, 16) <= cu) run(k_router_gemm<1, 1, 8>, 16, 16, 512);
    else if (blocks(32, 32) <= cu) run(k_router_gemm<2, 2, 8>, 32, 32, 512);
    else if (blocks(32, 64) <= cu) run(k_router_gemm<2, 4, 8>, 32, 64, 512);
    else run(k_router_gemm<4, 4, 4>, 64, 64, 256);
    return hipGetLastError();
}

hipError_t dxk_hotness_add(unsigned long long *counters, const int32_t *counts, int E, hipStream_t s)
{
    hipLaunchKernelGGL(k_hotness_add, dim3((E + 255) / 256), dim3(256), 0, s, counters, counts, E);
    return hipGetLastError();
}

hipError_t dxk_fill_u64(unsigned long long *p, size_t n, unsigned long long v, hipStream_t s)
{
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_fill_u64, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, p, n, v);
    return hipGetLastError();
}

hipError_t dxk_probe_read(const void *buf, size_t bytes, int n_cu, hipStream_t s)
{
    const int n_units = (int)(bytes >> 20);
    if (n_units == 0) return hipSuccess;
    hipLaunchKernelGGL(k_probe_read, dim3(n_cu), dim3(512), 0, s, static_cast<const char *>(buf), n_units,
                       static_cast<unsigned *>(nullptr));
    return hipGetLastError();
}

hipError_t dxk_store_handle(dx_handle *slot, const dx_handle &h, hipStream_t s)
{
    hipLaunchKernelGGL(k_store_handle, dim3(1), dim3(64), 0, s, slot, h);
    return hipGetLastError();
}

// ---- dx_route for callers that cannot allocate ---------------------------------------------------
// The routing scratch (per-chunk token masks, the array dx_create otherwise allocates for a context) lives in a file-scope device array.  Every GPU the library runs
// on holds its own copy at its own address until the process ends; the address is asked for once per
// device, with that device current, and kept.  In host code the array's name is only a stand-in for
// the symbol: kernels get the resolved pointer, never the name.
namespace {

constexpr size_t kStaticEntries = DX_ROUTE_STATIC_MAX_ENTRIES; // (chunks of 64 tokens) x experts
struct route_scratch {
    unsigned long long mask[kStaticEntries];
    int32_t sums[kStaticEntries / kSumChunks + 1024]; // groups of chunks x experts
};
static __device__ __align__(256) route_scratch scratch; // 524 KiB per GPU

constexpr int kMaxDevices = 64;
route_scratch *g_scratch_ptr[kMaxDevices]; // per device, null until resolved
std::mutex g_scratch_lock;
thread_local char g_static_err[256] = "";

dx_status static_fail(dx_status code, const char *fmt, ...)
{
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_static_err, sizeof g_static_err, fmt, ap);
    va_end(ap);
    return code;
}

} // namespace

extern "C" const char *dx_route_static_last_error(void) { return g_static_err; }

extern "C" dx_status dx_route_static(const float *logits, int T, int E, int top_k, int32_t *ids, float *w,
                                     int32_t *counts, int32_t *offsets, int32_t *perm, void *hip_stream)
{
    if (E < 1 || E > 1024) return static_fail(DX_ERR_INVALID, "dx_route_static: E=%d outside [1,1024]", E);
    if (top_k < 1 || top_k > E || top_k > 64)
        return static_fail(DX_ERR_INVALID, "dx_route_static: top_k=%d outside [1,min(E,64)]", top_k);
    if (T < 0) return static_fail(DX_ERR_INVALID, "dx_route_static: T=%d is negative", T);
    const long long n_chunks = T > 0 ? ((long long)T + kChunk - 1) / kChunk : 1;
    if (n_chunks * E > (long long)kStaticEntries)
        return static_fail(DX_ERR_INVALID,
                           "dx_route_static: ceil(T/64)*E = %lld exceeds the static scratch of %zu entries "
                           "(T=%d, E=%d); use dx_route on a context for larger batches",
                           n_chunks * E, kStaticEntries, T, E);
    if (!counts || !offsets || (T > 0 && (!logits || !ids || !w || !perm)))
        return static_fail(DX_ERR_INVALID, "dx_route_static: null pointer");
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return static_fail(DX_ERR_HIP, "dx_route_static: hipGetDevice: %s", hipGetErrorString(e));
    if (dev < 0 || dev >= kMaxDevices) return static_fail(DX_ERR_INVALID, "dx_route_static: device %d not supported", dev);
    route_scratch *sp;
    {
        std::lock_guard<std::mutex> hold(g_scratch_lock);
        if (!g_scratch_ptr[dev]) {
            void *p = nullptr;
            e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
            if (e != hipSuccess || !p)
                return static_fail(DX_ERR_HIP, "dx_route_static: hipGetSymbolAddress: %s", hipGetErrorString(e));
            g_scratch_ptr[dev] = static_cast<route_scratch *>(p);
        }
        sp = g_scratch_ptr[dev];
    }
    // Nothing in the scratch has to start at zero: every chunk's block writes all E masks of its chunk.
    e = dxk_route(logits, T, E, top_k, ids, w, counts, offsets, perm, sp->mask, sp->sums, nullptr, dx_list_args{},
                  static_cast<hipStream_t>(hip_stream));
    if (e != hipSuccess) return static_fail(DX_ERR_HIP, "dx_route_static: launch: %s", hipGetErrorString(e));
    return DX_OK;
}
