// Mixed-precision expert execution for small per-expert token counts
// (decode): SwiGLU gate/up grouped GEMM, down grouped GEMM, weighted combine.
//
// Paper: Sec. 3.2 -- the compute path resolves each expert's stable handle to
// the active version (bf16, or int4 / int2 with its quantization parameters)
// and runs the matching kernel.  The paper gives no kernel; this one is built for
// gfx950.
//
// Regime: every activated expert's weights are streamed from HBM exactly once
// and there are at most a few dozen tokens per expert, so both GEMM kernels are
// bandwidth-bound.  What decides the achieved bandwidth on this chip is that
// every compute unit streams for the whole duration of the kernel, so:
//   - Persistent grid, one block of 8 wavefronts per compute unit.  The work
//     is the list of (activated expert, 32-token block, strip of 16 weight
//     rows: 16 rows of W_down, or 8 rows of W_gate with the same 8 of W_up),
//     weighed in cost units (units_of, kRunUnits below); block b takes the
//     strips that start in units [b*U/G, (b+1)*U/G).  Every block derives
//     the same partition from `offsets` and the handles' formats in its
//     prologue (a block-wide scan): no atomics, no work queue.
//   - The 8 wavefronts of a block split the K extent of a strip between them
//     (wavefront kw owns CPW consecutive K-chunks of 4*LK elements), so a
//     whole strip is in flight at once and the following ones are prefetched
//     into further register stages while this one is multiplied.  Strips go
//     in pairs (two accumulators, one barrier per pair); when K is short,
//     the block works on several pairs side by side.  Partial sums meet in
//     LDS, are added in a fixed order and finished (SwiGLU, or the store of
//     the down output) by all threads of the block.
//   - The token rows (A operand of v_mfma_f32_16x16x32_bf16) only depend on
//     the expert and the K-chunk, so each wavefront keeps its fragments in
//     registers for all strips of a run: after the first strip, weights are
//     the only global traffic.
//   - Lane (r = lane%16, q = lane/16) owns tile row r in the matrix instruction.  Weights and token rows are
//     loaded in another order, eight neighbouring lanes to a 128-byte line, and pass through a small area of
//     LDS of the wavefront on their way to the operands (see line_load).  Contractions that are no multiple
//     of 128 load in operand order (LK = 16, 8).
//   - Quantized weights are expanded to exact small bf16 integers; a step of
//     the matrix instruction never crosses a quantization group, so the
//     group's scale multiplies the group's fp32 partial sums once (q*s is
//     never rounded).
// Segments above 32 tokens go in blocks of 32.  Most calls of more than 128 tokens, and calls of fewer
// on layers whose K takes several rounds here, run on tiles (takes_tiles).
#include "dx_internal.h"
#include "dx_route_core.h"

#include <hip/hip_ext.h>

#include <algorithm>
#include <cmath>
#include <type_traits>

namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4; // 16 bytes in registers
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;

// Pointers that come out of a handle are loaded from memory, so the compiler cannot infer their
// address space and would fall back to FLAT loads (whose wait counters serialise the pipeline).
// Everything the kernels stream is in global memory: say so in the type.
#define DX_GLOBAL __attribute__((address_space(1)))
typedef const DX_GLOBAL char *gbytes;   // weight bytes
typedef const DX_GLOBAL dx_bf16 *gbf16; // bf16 rows (scales, tokens)
typedef const DX_GLOBAL u32x4 *gvec16;
typedef const DX_GLOBAL u32x2 *gvec8;
typedef const DX_GLOBAL uint32_t *gvec4;
typedef const DX_GLOBAL uint32_t __attribute__((aligned(2))) *gscales2; // two scales
typedef const __attribute__((address_space(3))) int *lds_ints; // an int array in LDS

union frag8 {
    u32x4 u;
    bf16x8 v;
};

__device__ __forceinline__ uint32_t float_to_bf16_rne(float f)
{
    uint32_t u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return u >> 16;
}

// int4 -> bf16 without arithmetic.  XOR with 0x8 turns a two's-complement nibble q into u = q + 8 in
// [0, 15]; OR-ing u into the mantissa of bf16 128.0 (0x4300) gives exactly 128 + u = 136 + q.  One
// shift and one and-or yield two such values, elements t and t+4 of the word, so the 8 elements come
// out in the order (0,4,1,5,2,6,3,7); the token fragment is permuted to match once per run, and the
// bias is removed through  sum_k a_k (136 + q_k) - 136 sum_k a_k.
constexpr float kNibbleBias = 136.f;

// The flip, the mask and the OR are one v_bitop3_b32 per register (x is the shifted word): with two
// constant words p and q the result bit is 0, 1, the bit of x or its complement for (p, q) = (0, 0),
// (0, 1), (1, 0), (1, 1) -- truth table 0x6A over (x, p, q).
__device__ __forceinline__ uint32_t keep_flip_set(uint32_t x, uint32_t p, uint32_t q)
{
    return __builtin_amdgcn_bitop3_b32(x, p, q, 0x6A);
}

__device__ __forceinline__ bf16x8 nibbles_to_biased_bf16(uint32_t word)
{
    constexpr uint32_t p = 0x000F000Fu, q = (0x88888888u & p) | 0x43004300u; // ((x ^ 0x8888...) & p) | 0x4300...
    frag8 out;
    out.u = u32x4{keep_flip_set(word, p, q), keep_flip_set(word >> 4, p, q), keep_flip_set(word >> 8, p, q),
                  keep_flip_set(word >> 12, p, q)};
    return out.v;
}

// int2 (the low tier of the int4 / int2 pair): XOR with binary 10 turns a two's-complement code q in
// [-2, 1] into u = q + 2 in [0, 3]; OR-ed into bf16 128.0 it is 130 + q.  A word holds 16 codes; one
// shift and one and-or yield elements t and t+8, so the first MFMA step of a word takes elements
// (0,8,1,9,2,10,3,11) (shifts 0,2,4,6) and the second (4,12,5,13,6,14,7,15) (shifts 8..14).
constexpr float kCrumbBias = 130.f;

template <int HALF>
__device__ __forceinline__ bf16x8 crumbs_to_biased_bf16(uint32_t word)
{
    constexpr uint32_t p = 0x00030003u, q = (0xAAAAAAAAu & p) | 0x43004300u;
    frag8 out;
    out.u = u32x4{keep_flip_set(word >> (8 * HALF), p, q), keep_flip_set(word >> (8 * HALF + 2), p, q),
                  keep_flip_set(word >> (8 * HALF + 4), p, q), keep_flip_set(word >> (8 * HALF + 6), p, q)};
    return out.v;
}

// the matching order for two consecutive token fragments a = (e0..e7), b = (e8..e15):
// lo = (e0,e8,e1,e9,e2,e10,e3,e11), hi = (e4,e12,e5,e13,e6,e14,e7,e15)
__device__ __forceinline__ void zip_fragments(u32x4 &a, u32x4 &b)
{
    const u32x4 lo = u32x4{(a.x & 0x0000FFFFu) | (b.x << 16), (a.x >> 16) | (b.x & 0xFFFF0000u),
                           (a.y & 0x0000FFFFu) | (b.y << 16), (a.y >> 16) | (b.y & 0xFFFF0000u)};
    const u32x4 hi = u32x4{(a.z & 0x0000FFFFu) | (b.z << 16), (a.z >> 16) | (b.z & 0xFFFF0000u),
                           (a.w & 0x0000FFFFu) | (b.w << 16), (a.w >> 16) | (b.w & 0xFFFF0000u)};
    a = lo;
    b = hi;
}

// the same element order for a token fragment: (e0..e7) -> (e0,e4,e1,e5,e2,e6,e3,e7)
__device__ __forceinline__ u32x4 interleave_halves(u32x4 v)
{
    return u32x4{(v.x & 0x0000FFFFu) | (v.z << 16), (v.x >> 16) | (v.z & 0xFFFF0000u),
                 (v.y & 0x0000FFFFu) | (v.w << 16), (v.y >> 16) | (v.w & 0xFFFF0000u)};
}

constexpr int kWaves = 8;             // wavefronts per block
constexpr int kThreads = 64 * kWaves; // 512
constexpr int kMaxExperts = 1024 + 1; // routed + shared
// Cost units of the partition, from a fit of the blocks' measured times (per-block time stamps of a debug
// build, 30B- and 80B-shaped decode layers, a dozen routing draws each) to
//   time = runs * c_run + sum over the block's strips of c(format, token tiles):
// a bf16 strip for up to 16 tokens is 32 units; the same strip for two token tiles multiplies and finishes
// twice as much (1.25x gate/up, 1.35x down); a quantized strip is a quarter of the bytes or less but
// carries the same per-step work (expansion, barrier, reduction), 0.47x for one tile and 0.8x for two --
// weighed by time, not bytes.  int2 strips (an eighth of the bytes, the same per-step work) are taken a
// little below the int4 ones.
// A run that starts on a new expert pays for the token rows and a cold pipeline (3 to 5 us: two to three
// bf16 gate/up strips, five down strips): every expert's range begins with kRunUnits units that carry no
// strips, so the block that holds an expert boundary gets correspondingly fewer strips.
template <bool DOWN>
constexpr uint32_t kRunUnits = DOWN ? 176 : 84;
template <bool DOWN>
__device__ __forceinline__ uint32_t units_of(uint32_t fmt, int m)
{
    const bool two = m > 16;
    if (fmt == DX_FMT_BF16) return two ? (DOWN ? 43 : 40) : 32;
    const uint32_t q = two ? (DOWN ? 26 : 25) : 15;
    return fmt == DX_FMT_INT4G ? q : q - 3;
}

#ifdef DX_TRACE
// Debug build only: per-block start/end time stamps (100 MHz wall clock).
__device__ unsigned long long g_trace[2][8192][4];
__device__ unsigned long long g_steps[2][4][256];
__device__ unsigned int g_nsteps[2][4];
__device__ unsigned int g_mix[2][8192][8]; // per block: runs, then strips by (format != bf16) * 2 + (second token tile)
#endif

// element offset inside a chunk of MFMA step j for lane quarter q
// FMT: 0 bf16, 1 int4, 2 int2 (the values of dx_fmt)
template <int LK, int FMT>
__device__ __forceinline__ int k_of(int j, int q)
{
    return FMT ? q * LK + 8 * j : 32 * j + 8 * q;
}

// weight registers of one wavefront for one 16-row strip: CPW chunks
template <int LK, int CPW, int FMT>
struct wstage {
    static constexpr int JN = LK / 8;
    static constexpr int NQ = FMT == 1 ? JN : (FMT == 2 ? (JN + 1) / 2 : 1);
    u32x4 w[CPW][FMT ? 1 : JN]; // bf16: JN 16-byte pieces per chunk
    uint32_t wq[CPW][NQ];       // int4: JN words of 8 nibbles; int2: JN/2 words of 16 codes
};

// The weight stream of chunks of 128 elements (LK = 32), and the token rows of all formats.  Three measurements on
// this chip decide its shape (a 192 MB stream of cold strips, one 8-wavefront block per compute unit):
//   - a compute unit takes in 120 GB/s (from L2) when eight neighbouring lanes read one 128-byte line, 37 GB/s
//     when the lanes of a line are spread over the wavefront, as the operand order of the matrix instruction
//     (lane (r, q): 16 bytes of row r) wants them;
//   - with the non-temporal hint whole lines in neighbour order stream at 6.2 TB/s, in the spread order (8 rows
//     x 128 bytes per instruction all the same) at 5.75, without the hint at 5.2 to 5.6;
//   - loads to LDS stream at 5.2 TB/s whatever the hint.
// So lane l fetches 16-byte piece l % 8 of row l / 8 into registers, and when a stage is used it passes through a
// small area of LDS that belongs to the wavefront (no barrier; the area is the wavefront's part of the `red`
// buffer that is next to be filled, unused until the sums are parked), from where the operands are read in the
// order they are needed.  Reading from LDS also lets every step of the matrix instruction take its elements
// from one quantization group, whatever the group size: GPC = groups per chunk (1, 2, 4 for groups of 128, 64, 32).
//   Area: bf16 [line][16 rows][128 B], a chunk at a time; int4 [16 rows][64 * CPW B]; int2 in groups of 64
//   [16 rows][32 * CPW B] (in groups of 128 it does not pass through LDS).
//   16-byte piece p of row r sits in slot p ^ ((r >> 1) & 7) of a 128-byte row, p ^ ((r >> 2) & 3) of a 64-byte
//   row: the 16 lanes that read one piece index of 16 rows hit 16 different bank groups.
template <typename T>
__device__ __forceinline__ T line_load(const DX_GLOBAL T *p)
{
    return __builtin_nontemporal_load(p);
}

typedef __attribute__((address_space(3))) char *lds_bytes;
template <typename T>
__device__ __forceinline__ T lds_get(lds_bytes p)
{
    return *reinterpret_cast<const __attribute__((address_space(3))) T *>(p);
}
template <typename T>
__device__ __forceinline__ void lds_put(lds_bytes p, T v)
{
    *reinterpret_cast<__attribute__((address_space(3))) T *>(p) = v;
}

// Lanes of one wavefront hand data to each other through LDS, which the hardware accesses in the wavefront's order.  The
// compiler sees only that a lane reads other addresses than it wrote, and may move such reads: the readers take the area's
// address through this (no instruction), of which it knows nothing, so that every read may be of what was written.  (A
// fence of wavefront scope also holds the loads from memory in place: T = 1 30B-shaped 27.0 -> 27.7 us.)
__device__ __forceinline__ lds_bytes as_other_lanes(lds_bytes p)
{
    uint32_t at = (uint32_t)(uintptr_t)p;
    asm("" : "+v"(at));
    return (lds_bytes)(uintptr_t)at;
}

// weight registers of one wavefront for one 16-row strip of CPW chunks, in the order they were loaded
template <int CPW, int FMT>
struct line_stage {
    static constexpr int N = FMT == 0 ? 4 * CPW : (FMT == 1 ? CPW : 1);
    u32x4 w[N];
};

// `lo`: the strip's first eight rows at the wavefront's first chunk, `hi`: its other eight (in a gate/up strip
// another matrix); `two`: the second chunk of a CPW = 2 stage exists.
template <int GPC, int CPW, int FMT>
__device__ __forceinline__ void issue_lines(line_stage<CPW, FMT> &st, gbytes lo, gbytes hi, uint32_t row_bytes, bool one,
                                            bool two, int lane)
{
    if constexpr (FMT == 0) {
        const uint32_t off = (uint32_t)(lane >> 3) * row_bytes + (lane & 7) * 16;
#pragma unroll
        for (int i = 0; i < CPW; ++i) {
            if (i ? two : one) { // wavefront-uniform
#pragma unroll
                for (int n = 0; n < 4; ++n)
                    st.w[i * 4 + n] = line_load(reinterpret_cast<gvec16>(((n & 1) ? hi : lo) + (i * 256 + 128 * (n >> 1)) + off));
            }
        }
    } else if constexpr (FMT == 1 && CPW == 2) {
        // (without the second chunk the lanes of its half re-read the first)
        const uint32_t off = (uint32_t)(lane >> 3) * row_bytes + (lane & (two ? 7 : 3)) * 16;
        if (one) {
            st.w[0] = line_load(reinterpret_cast<gvec16>(lo + off));
            st.w[1] = line_load(reinterpret_cast<gvec16>(hi + off));
        }
    } else if constexpr (FMT == 2 && GPC == 1) {
        // Codes of 2 bits in one group per chunk: 8 bytes per lane and chunk, in operand order straight to the registers.  A
        // strip is so small that the way through LDS costs more than the loads in whole lines gain (30B-shaped layer, all
        // experts int2, 64 tokens 85.7 us through LDS, 80.7 without).
        const gbytes base = (lane & 8 ? hi : lo) + (uint32_t)(lane & 7) * row_bytes + (lane >> 4) * 8;
        if (one) {
            const u32x2 t = *reinterpret_cast<gvec8>(base);
            st.w[0].x = t.x, st.w[0].y = t.y;
        }
        if (CPW == 2 && two) {
            const u32x2 t = *reinterpret_cast<gvec8>(base + 32);
            st.w[0].z = t.x, st.w[0].w = t.y;
        }
    } else if (one) {
        // all 16 rows in one instruction: 64 (int2, one chunk: 32) bytes of each
        const gbytes base = (lane < 32 ? lo : hi) + (uint32_t)((lane >> 2) & 7) * row_bytes;
        if constexpr (FMT == 2 && CPW == 1) {
            const u32x2 t = line_load(reinterpret_cast<gvec8>(base + (lane & 3) * 8));
            st.w[0] = u32x4{t.x, t.y, 0u, 0u};
        } else {
            st.w[0] = line_load(reinterpret_cast<gvec16>(base + (lane & (CPW == 1 || two ? 3 : 1)) * 16));
        }
    }
}

// byte addresses in the wavefront's area, computed once per run
struct line_lanes {
    int put, get, get64, get32; // 128-byte rows: the loaded piece; pieces q, q / 2 (8 bytes), 0 (4 bytes) of row r
    int put_s, get_s, get64_s, get32_s; // the same for 64-byte rows
    int tok1, tok2;             // tokens: piece 4 * (q % 2) of line q / 2; piece 2q
};
__device__ __forceinline__ line_lanes line_lanes_of(int lane)
{
    const int r = lane & 15, q = lane >> 4, s = (r >> 1) & 7, f = (r >> 2) & 3;
    line_lanes ll;
    ll.put = (lane >> 3) * 128 + ((lane & 7) ^ ((lane >> 4) & 3)) * 16; // rows 8..15: ^ 64 on top
    ll.get = r * 128 + (q ^ s) * 16;
    ll.get64 = r * 128 + ((q >> 1) ^ s) * 16 + 8 * (q & 1);
    ll.get32 = r * 128 + s * 16 + 4 * q;
    ll.put_s = (lane >> 2) * 64 + ((lane & 3) ^ ((lane >> 4) & 3)) * 16;
    ll.get_s = r * 64 + (q ^ f) * 16;
    ll.get64_s = r * 64 + ((q >> 1) ^ f) * 16 + 8 * (q & 1);
    ll.get32_s = r * 64 + f * 16 + 4 * q;
    ll.tok1 = r * 128 + ((4 * (q & 1)) ^ s) * 16 + (q >> 1) * 2048;
    ll.tok2 = r * 128 + ((2 * q) ^ s) * 16;
    return ll;
}

// Which 8 elements of a chunk lane (r, q) takes in step j: bf16 and GPC = 4: 32j + 8q; else
// (128 / GPC) * (j / SPG) + (32 / GPC) * q + 8 * (j % SPG) with SPG = 4 / GPC steps per group.
template <int GPC, int CPW, int FMT, int MT>
__device__ __forceinline__ void load_token_lines(u32x4 (&x)[CPW][MT][4], const gbf16 (&row)[2][2], int c0, int nc, int lane,
                                                 const line_lanes &ll, lds_bytes area)
{
#pragma unroll
    for (int i = 0; i < CPW; ++i) {
        if (c0 + i < nc) {
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int n = 0; n < 4; ++n)
                    x[i][mt][n] = *reinterpret_cast<gvec16>(row[mt][n & 1] + (c0 + i) * 128 + 64 * (n >> 1) + (lane & 7) * 8);
        }
    }
#pragma unroll
    for (int i = 0; i < CPW; ++i) {
        if (c0 + i < nc) {
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
#pragma unroll
                for (int n = 0; n < 4; ++n)
                    lds_put(area + (n >> 1) * 2048 + (n & 1) * 1024 + (ll.put ^ ((n & 1) * 64)), x[i][mt][n]);
                const lds_bytes from = as_other_lanes(area);
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    if constexpr (FMT == 0 || GPC == 4) x[i][mt][j] = lds_get<u32x4>(from + (j >> 1) * 2048 + (ll.get ^ ((j & 1) * 64)));
                    else if constexpr (GPC == 2) x[i][mt][j] = lds_get<u32x4>(from + (j >> 1) * 2048 + (ll.tok2 ^ ((j & 1) * 16)));
                    else x[i][mt][j] = lds_get<u32x4>(from + (ll.tok1 ^ (j * 16)));
                }
            }
        }
    }
}

// Quantized runs: bring the token fragments into the element order of the expanded codes and compute
// nbias[i][g][mt] = -bias * sum over group g of chunk i of the token row (one MFMA against all-ones per step), laid
// out like an accumulator (every column holds the row's sum): what the group's products start from.
template <int GPC, int CPW, int MT, int FMT>
__device__ __forceinline__ void prepare_line_tokens(u32x4 (&x)[CPW][MT][4], f32x4 (&nbias)[CPW][GPC][MT], int c0, int nc)
{
    constexpr int SPG = 4 / GPC;
    frag8 ones;
    ones.u = u32x4{0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u};
#pragma unroll
    for (int i = 0; i < CPW; ++i) {
        if (c0 + i < nc) {
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
#pragma unroll
                for (int g = 0; g < GPC; ++g) {
                    f32x4 sum = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int j = g * SPG; j < (g + 1) * SPG; ++j) {
                        frag8 a;
                        a.u = x[i][mt][j];
                        sum = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.v, ones.v, sum, 0, 0, 0);
                        if constexpr (FMT == 1) x[i][mt][j] = interleave_halves(x[i][mt][j]);
                    }
                    nbias[i][g][mt] = sum * (FMT == 1 ? -kNibbleBias : -kCrumbBias);
                }
                if constexpr (FMT == 2) {
#pragma unroll
                    for (int j = 0; j < 4; j += 2) zip_fragments(x[i][mt][j], x[i][mt][j + 1]);
                }
            }
        }
    }
}

template <int GPC, int CPW, int FMT, int MT>
__device__ __forceinline__ void multiply_lines(const line_stage<CPW, FMT> &st, const u32x4 (&x)[CPW][MT][4],
                                               const f32x4 (&nbias)[CPW][GPC][MT], const uint32_t (&scales)[(CPW * GPC + 1) / 2],
                                               bool one, bool two, const line_lanes &ll, int lane, lds_bytes area,
                                               f32x4 (&acc)[MT])
{
    constexpr int SPG = 4 / GPC;
    if (!one) return; // wavefront-uniform
    if constexpr (FMT == 0) {
        frag8 wv[CPW][4];
#pragma unroll
        for (int i = 0; i < CPW; ++i) {
            if (i == 0 || two) {
#pragma unroll
                for (int n = 0; n < 4; ++n)
                    lds_put(area + (n >> 1) * 2048 + (n & 1) * 1024 + (ll.put ^ ((n & 1) * 64)), st.w[i * 4 + n]);
                const lds_bytes from = as_other_lanes(area);
#pragma unroll
                for (int j = 0; j < 4; ++j) wv[i][j].u = lds_get<u32x4>(from + (j >> 1) * 2048 + (ll.get ^ ((j & 1) * 64)));
            }
        }
#pragma unroll
        for (int i = 0; i < CPW; ++i) {
            if (i == 0 || two) {
#pragma unroll
                for (int j = 0; j < 4; ++j)
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt) {
                        frag8 a;
                        a.u = x[i][mt][j];
                        acc[mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.v, wv[i][j].v, acc[mt], 0, 0, 0);
                    }
            }
        }
    } else {
        constexpr bool wide = FMT == 1 && CPW == 2; // 128-byte rows in the area
        if constexpr (FMT == 2 && GPC == 1) { // in operand order already
        } else if constexpr (wide) {
            lds_put(area + ll.put, st.w[0]);
            lds_put(area + 1024 + (ll.put ^ 64), st.w[1]);
        } else if constexpr (FMT == 2 && CPW == 1) {
            lds_put(area + lane * 8, u32x2{st.w[0].x, st.w[0].y}); // 32-byte rows
        } else {
            lds_put(area + ll.put_s, st.w[0]);
        }
        const lds_bytes from = as_other_lanes(area);
        uint32_t wq[CPW][4]; // int4: a word of 8 codes per step; int2: a word of 16 codes per two steps
#pragma unroll
        for (int i = 0; i < CPW; ++i) {
            if (i && !two) continue;
            if constexpr (FMT == 1) {
                if constexpr (GPC == 1) {
                    const u32x4 t = lds_get<u32x4>(from + (wide ? ll.get ^ (i * 64) : ll.get_s));
                    wq[i][0] = t.x; wq[i][1] = t.y; wq[i][2] = t.z; wq[i][3] = t.w;
                } else if constexpr (GPC == 2) {
#pragma unroll
                    for (int g = 0; g < 2; ++g) {
                        const u32x2 t = lds_get<u32x2>(from + (wide ? ll.get64 ^ (i * 64) ^ (g * 32) : ll.get64_s ^ (g * 32)));
                        wq[i][2 * g] = t.x; wq[i][2 * g + 1] = t.y;
                    }
                } else {
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        wq[i][j] = lds_get<uint32_t>(from + (wide ? ll.get32 ^ (i * 64) ^ (j * 16) : ll.get32_s ^ (j * 16)));
                }
            } else {
                const int r = lane & 15, q = lane >> 4;
                if constexpr (GPC == 1) {
                    wq[i][0] = i ? st.w[0].z : st.w[0].x; wq[i][1] = i ? st.w[0].w : st.w[0].y;
                } else {
#pragma unroll
                    for (int g = 0; g < 2; ++g)
                        wq[i][g] = lds_get<uint32_t>(from + (CPW == 2 ? ll.get32_s ^ (i * 32) ^ (g * 16) : r * 32 + 16 * g + 4 * q));
                }
            }
        }
#pragma unroll
        for (int i = 0; i < CPW; ++i) {
            if (i && !two) continue;
#pragma unroll
            for (int g = 0; g < GPC; ++g) {
                f32x4 part[MT];
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) part[mt] = nbias[i][g][mt];
#pragma unroll
                for (int j = g * SPG; j < (g + 1) * SPG; ++j) {
                    bf16x8 wv;
                    if constexpr (FMT == 1) wv = nibbles_to_biased_bf16(wq[i][j]);
                    else wv = (j & 1) ? crumbs_to_biased_bf16<1>(wq[i][j / 2]) : crumbs_to_biased_bf16<0>(wq[i][j / 2]);
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt) {
                        frag8 a;
                        a.u = x[i][mt][j];
                        part[mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.v, wv, part[mt], 0, 0, 0);
                    }
                }
                // (the bf16 scales of the wavefront's groups, two to a word: even ones in the low half)
                const uint32_t sw = scales[(i * GPC + g) >> 1];
                const float scale = __uint_as_float(((i * GPC + g) & 1) ? sw & 0xFFFF0000u : sw << 16);
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) acc[mt] += part[mt] * scale;
            }
        }
    }
}

// ---- chunks of 64 or 32 elements (LK = 16, 8): contractions that are no multiple of 128, operand order ----
template <int LK, int CPW, int FMT>
__device__ __forceinline__ void issue_weights(wstage<LK, CPW, FMT> &st, gbytes row, int c0, int nc, int q)
{
    constexpr int CHUNK = 4 * LK, JN = LK / 8;
#pragma unroll
    for (int i = 0; i < CPW; ++i) {
        const int c = c0 + i;
        if (c < nc) { // wavefront-uniform
            if constexpr (FMT == 2) {
                gbytes p = row + ((c * CHUNK + q * LK) >> 2);
                if constexpr (LK == 16) {
                    st.wq[i][0] = *reinterpret_cast<gvec4>(p);
                } else { // 8 codes = 2 bytes (handles of this format are refused for group 32; kept in bounds)
                    st.wq[i][0] = *reinterpret_cast<const DX_GLOBAL uint16_t *>(p);
                }
            } else if constexpr (FMT == 1) {
                gbytes p = row + ((c * CHUNK + q * LK) >> 1);
                if constexpr (LK == 16) {
                    const u32x2 t = *reinterpret_cast<gvec8>(p);
                    st.wq[i][0] = t.x; st.wq[i][1] = t.y;
                } else {
                    st.wq[i][0] = *reinterpret_cast<gvec4>(p);
                }
            } else {
#pragma unroll
                for (int j = 0; j < JN; ++j)
                    st.w[i][j] = *reinterpret_cast<gvec16>(row + (size_t)(c * CHUNK + k_of<LK, 0>(j, q)) * 2);
            }
        }
    }
}

template <int LK, int CPW, int FMT, int MT>
__device__ __forceinline__ void load_tokens(u32x4 (&x)[CPW][MT][LK / 8], gbf16 arow0, gbf16 arow1, int c0, int nc,
                                            int q)
{
    constexpr int CHUNK = 4 * LK, JN = LK / 8;
#pragma unroll
    for (int i = 0; i < CPW; ++i) {
        const int c = c0 + i;
        if (c < nc) {
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int j = 0; j < JN; ++j)
                    x[i][mt][j] = *reinterpret_cast<gvec16>((mt ? arow1 : arow0) + c * CHUNK + k_of<LK, FMT>(j, q));
        }
    }
}

// int4 runs: bring the token fragments into the element order of nibbles_to_biased_bf16 and compute
// bias[i][mt] = 136 * sum over chunk i of the token row (one MFMA against all-ones per step), laid out
// like an accumulator (every column holds the row's sum).
template <int LK, int CPW, int MT, int FMT>
__device__ __forceinline__ void prepare_quant_tokens(u32x4 (&x)[CPW][MT][LK / 8], f32x4 (&bias)[CPW][1][MT], int c0, int nc)
{
    constexpr int JN = LK / 8;
    frag8 ones;
    ones.u = u32x4{0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u};
#pragma unroll
    for (int i = 0; i < CPW; ++i) {
        if (c0 + i < nc) {
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                f32x4 sum = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int j = 0; j < JN; ++j) {
                    frag8 a;
                    a.u = x[i][mt][j];
                    sum = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.v, ones.v, sum, 0, 0, 0);
                    if constexpr (FMT == 1) x[i][mt][j] = interleave_halves(x[i][mt][j]);
                }
                if constexpr (FMT == 2) {
#pragma unroll
                    for (int j = 0; j + 1 < JN; j += 2) zip_fragments(x[i][mt][j], x[i][mt][j + 1]);
                }
                bias[i][0][mt] = sum * (FMT == 1 ? kNibbleBias : kCrumbBias);
            }
        }
    }
}

template <int LK, int CPW, int FMT, int MT>
__device__ __forceinline__ void multiply(const wstage<LK, CPW, FMT> &st, const u32x4 (&x)[CPW][MT][LK / 8],
                                         const f32x4 (&bias)[CPW][1][MT], uint32_t scales, int c0, int nc, f32x4 (&acc)[MT])
{
    constexpr int JN = LK / 8;
#pragma unroll
    for (int i = 0; i < CPW; ++i) {
        if (c0 + i < nc) {
            if constexpr (FMT != 0) {
                f32x4 part[MT];
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) part[mt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int j = 0; j < JN; ++j) {
                    bf16x8 wv;
                    if constexpr (FMT == 1) wv = nibbles_to_biased_bf16(st.wq[i][j]);
                    else wv = (j & 1) ? crumbs_to_biased_bf16<1>(st.wq[i][j / 2]) : crumbs_to_biased_bf16<0>(st.wq[i][j / 2]);
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt) {
                        frag8 a;
                        a.u = x[i][mt][j];
                        part[mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.v, wv, part[mt], 0, 0, 0);
                    }
                }
                // (the bf16 scales of the wavefront's chunks, two to a word: chunk 0 in the low half)
                const float scale = __uint_as_float(i == 0 ? scales << 16 : scales & 0xFFFF0000u);
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) acc[mt] += (part[mt] - bias[i][0][mt]) * scale;
            } else {
#pragma unroll
                for (int j = 0; j < JN; ++j) {
                    frag8 wv;
                    wv.u = st.w[i][j];
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt) {
                        frag8 a;
                        a.u = x[i][mt][j];
                        acc[mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.v, wv.v, acc[mt], 0, 0, 0);
                    }
                }
            }
        }
    }
}

// what a block needs to know about the expert it is working on
struct expert_ctx {
    gbytes w0, w1;   // gate/up: the gate and up matrices; down: the down matrix twice
    gbf16 s0, s1;    // their scales (int4)
    uint32_t row_bytes; // of a weight row (a matrix is smaller than 4 GiB)
    int K;           // contraction length
    int G;           // scale groups per row
    int seg0, m;     // segment in the H/O scratch, tokens
    bool shared;
    int fmt;         // dx_fmt of the published version
    lds_ints perm_lds; // the permutation in LDS when the kernel routed itself, else null (a.perm is used)
};

// Strips.  The unit of work is a strip of 16 weight rows against all of K: for the down projection rows
// 16s .. 16s+15 of W_down (16 columns of O); for gate/up the rows 8s .. 8s+7 of W_gate as tile rows 0..7 and
// the same rows of W_up as tile rows 8..15 (8 columns of H: silu(gate) * up pairs column c with column
// c + 8 of the same accumulator).  Strips are worked through in pairs (two accumulators, one barrier and
// one finish per pair); a run of an odd number of strips ends with half a pair.
//
// Add up the partial sums of the pairs that start at strips sb, sb + 2, ... (live_groups of them, side by
// side across the wavefront groups) in a fixed order and finish the strips below h_hi:
// gate/up -> H = silu(gate) * up (bf16); down -> O (fp32).  All threads.
// Element (group gg, tile mt, accumulator lane L, component i) is token 4*(L/16)+i, tile column L%16.
// (slot, row of O) of the output elements a thread finishes: idx = threadIdx.x + n * kThreads has the
// same idx % (MT * 256) for every n, so both are fixed for a whole run and the row lookup in the
// permutation happens once, off the critical path of the first finish.
template <bool DOWN, int MT>
__device__ __forceinline__ void finish_target(const dx_fwd_args &a, const expert_ctx &ex, int mb, int &slot, int &orow)
{
    const int rem = threadIdx.x % (MT * 256);
    const int mt = rem / 256, L = rem & 63, i = (rem >> 6) & 3;
    slot = mb * 32 + 16 * mt + 4 * (L >> 4) + i;
    orow = 0;
    if (DOWN && slot < ex.m) orow = ex.shared ? ex.seg0 + slot : a.perm[ex.seg0 + slot];
}

template <bool DOWN, int MT>
__device__ __forceinline__ void finish_batch(const dx_fwd_args &a, const expert_ctx &ex, int slot, int orow, int sb,
                                             int live_groups, int WPS, int h_hi, const float *redf)
{
    if (slot >= ex.m) return;
    for (int idx = threadIdx.x; idx < live_groups * MT * 256; idx += kThreads) {
        const int gg = idx / (MT * 256), rem = idx % (MT * 256);
        const int mt = rem / 256, L = rem & 63, i = (rem >> 6) & 3;
        // down: the thread adds up column L%16 of both strips of the pair; gate/up: column L%16 of the pair's
        // 16 columns of H lies in strip (L%16)/8, its gate sum in tile column L%8 and its up sum 8 columns on
        const int first = DOWN ? 0 : (L >> 3) & 1, second = DOWN ? 1 : first;
        const int l0 = DOWN ? L : (L & 0x37), l1 = DOWN ? L : l0 + 8;
        // the partial sums are read four wavefronts at a time before they are added (in the order of the
        // wavefronts): one LDS round trip per four instead of one each; past WPS a duplicate is read and
        // not added
        float v0 = 0.f, v1 = 0.f;
        for (int w0 = 0; w0 < WPS; w0 += 4) {
            float p0[4], p1[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int ww = w0 + u < WPS ? w0 + u : WPS - 1;
                const float *base = redf + ((gg * WPS + ww) * 4) * 64 * 4 + i;
                p0[u] = base[((first * 2 + mt) * 64 + l0) * 4];
                p1[u] = base[((second * 2 + mt) * 64 + l1) * 4];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                if (w0 + u < WPS) {
                    v0 += p0[u];
                    v1 += p1[u];
                }
            }
        }
        const int s0 = sb + 2 * gg; // the pair's first strip (below h_hi: the group is live)
        if constexpr (DOWN) {
            const int n = s0 * 16 + (L & 15);
            const bool both = s0 + 1 < h_hi;
            a.o[(size_t)orow * a.d + n] = v0;
            if (both) a.o[(size_t)orow * a.d + n + 16] = v1;
        } else {
            if (s0 + first < h_hi) {
                const float hv = v0 / (1.f + expf(-v0)) * v1;
                a.h[(size_t)(ex.seg0 + slot) * a.fmax + s0 * 8 + (L & 15)] = (dx_bf16)float_to_bf16_rne(hv);
            }
        }
    }
}

// How the K extent of a strip is split (pick_split):
//   kWhole:  one round of whole chunks, K / (4*LK) = WPS * CPW with WPS <= 8;
//   kRagged: one round of CPW = 2 chunks, of which the last wavefront may have one only;
//   kRounds: more chunks than the wavefronts take at once.
enum split_mode { kWhole, kRagged, kRounds };
// One run: strips [h_lo, h_hi) of one expert for one block of up to 32 tokens (mb).
// All kThreads threads of the block execute this with identical arguments.
//
// With one round the steady-state loop is straight-line code -- every iteration issues the next strip pair's loads
// unconditionally (the strip index is clamped, so the last iterations of a ragged run fetch a duplicate) -- which
// lets the compiler wait for exactly the loads it is about to use and keep the prefetch in flight.
template <int LK, int GPC, int CPW, bool DOWN, int FMT, int MT, int MODE>
__device__ __forceinline__ void run_strips(const dx_fwd_args &a, const expert_ctx &ex, int mb, int h_lo, int h_hi,
                                           f32x4 (*red)[kWaves][4][64], int &pb)
{
    constexpr int CHUNK = 4 * LK;
    // (the wavefront's index through readfirstlane: everything derived from it -- its K-part, its strips, the
    // strips' offsets in the matrices -- is then scalar arithmetic, and the loads take a scalar base plus a
    // per-lane offset that is computed once per run)
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, r = lane & 15, q = lane >> 4;
    const int nc = ex.K / CHUNK;
    // wavefronts per strip pair, strip pairs side by side, K rounds
    const int per = (nc + CPW - 1) / CPW;
    const int WPS = per < kWaves ? per : kWaves;
    const int SPP = kWaves / WPS;
    constexpr bool ONE_ROUND = MODE != kRounds;
    const int rounds = ONE_ROUND ? 1 : (per + WPS - 1) / WPS;
    const int g = wave / WPS, kw = wave % WPS;
    const bool idle = g >= SPP;
    const int npairs = (h_hi - h_lo + 1) / 2;
    const int nbatch = (npairs + SPP - 1) / SPP;

    int fin_slot, fin_orow;
    finish_target<DOWN, MT>(a, ex, mb, fin_slot, fin_orow);
    auto finish = [&](int batch) {
        __syncthreads();
        const int sb = h_lo + 2 * batch * SPP;
        const int left = (h_hi - sb + 1) / 2; // pairs from sb on
        const int live_groups = left < SPP ? left : SPP;
        finish_batch<DOWN, MT>(a, ex, fin_slot, fin_orow, sb, live_groups, WPS, h_hi,
                               reinterpret_cast<const float *>(&red[pb][0][0][0]));
        pb ^= 1; // the other half of `red` is free: its readers passed the barrier above
    };

    if (idle) { // wavefronts without a K-part (8 is not a multiple of WPS) only help finishing
        for (int batch = 0; batch < nbatch; ++batch) finish(batch);
        return;
    }

    // kWhole: nc counts as "unbounded" so that every chunk predicate folds away
    const int ncp = MODE == kWhole ? 0x7fffffff : nc;
    constexpr bool LINES = LK == 32;
    constexpr int NSW = (CPW * GPC + 1) / 2; // words of group scales per strip
    u32x4 x[CPW][MT][LK / 8];
    f32x4 bias[CPW][GPC][MT];
    // token rows of this run, looked up after the weight prologue: LINES: the rows the lane loads (lane / 8 and
    // 8 + lane / 8 of every 16-token tile), else row r of tile mt in [mt][0]
    gbf16 arow[2][2];
    const line_lanes ll = line_lanes_of(lane);
    // the wavefront's area of LDS: its part of the half of `red` that is filled next
    auto area = [&]() { return (lds_bytes)(__attribute__((address_space(3))) void *)&red[pb][wave][0][0]; };
    auto fetch_tokens = [&](int c0) {
        if constexpr (LINES) {
            load_token_lines<GPC, CPW, FMT, MT>(x, arow, c0, ncp, lane, ll, area());
            if constexpr (FMT != 0) prepare_line_tokens<GPC, CPW, MT, FMT>(x, bias, c0, ncp);
        } else {
            load_tokens<LK, CPW, FMT, MT>(x, arow[0][0], arow[1][0], c0, ncp, q);
            if constexpr (FMT != 0) prepare_quant_tokens<LK, CPW, MT, FMT>(x, bias, c0, ncp);
        }
    };

    // A step is one strip: b = 0 the first strip of a pair, b = 1 the second; the last pair of a run may lack its
    // second strip (no load, no multiply).  One round: step t = 2 * batch + b.  Otherwise K goes in rounds of 8 * CPW chunks
    // and the tokens are fetched anew in every round, so NB pairs share a round's tokens, each with accumulators
    // of its own: step t = (((batch / NB) * rounds + round) * NB + batch % NB) * 2 + b.  (One pair per fetch moved as
    // many token bytes as weight bytes: 8 tokens of 16 experts of 4096 x 6400, bf16/int4 227 us, now 192.  NB = 4 with two chunks of 128 per
    // wavefront does not fit the registers.)
    // NST register stages: the strip of step t + NST - 1 is fetched while step t is multiplied.  A quantized
    // strip is a quarter of the bytes or less, so it gets a deeper pipeline (four stages; with six or eight
    // the runs of a decode batch, a dozen steps each, spend most of their steps outside the steady loop,
    // which measured slower).  Not so two chunks of four groups each: their scales and sums leave no registers for four
    // stages (18 to 36 of them spilled; 30B-shaped layer in groups of 32, 8 tokens 66 us with four, 60 with two).
    constexpr int NB = ONE_ROUND ? 1 : (LK == 32 && CPW == 2 ? 2 : 4);
    constexpr int NST = FMT && !(GPC == 4 && CPW == 2) ? 4 : 2;
    const int nhalf = (nbatch + NB - 1) / NB * NB * rounds * 2; // steps
    using stage_t = std::conditional_t<LINES, line_stage<CPW, FMT>, wstage<LK, CPW, FMT>>;
    stage_t st[NST];
    const gbytes weight_rows0 = ex.w0, weight_rows1 = ex.w1;
    const uint32_t lane_row8 = (uint32_t)(r & 7) * ex.row_bytes, lane_row16 = (uint32_t)r * ex.row_bytes; // per-lane byte offsets
    // the strip of step t (past the end of the run for the missing half of the last pair and for the pairs of
    // wavefront groups without one in the last batch) and its K round
    auto strip_of = [&](int t) {
        if constexpr (ONE_ROUND) return h_lo + 2 * ((t >> 1) * SPP + g) + (t & 1);
        else return h_lo + 2 * (((t / (2 * NB) / rounds) * NB + ((t >> 1) % NB)) * SPP + g) + (t & 1);
    };
    auto chunk_of_step = [&](int t) { return ONE_ROUND ? kw * CPW : (((t / (2 * NB)) % rounds) * WPS + kw) * CPW; };
    // row r of a strip's tile in the weight (scale) matrices: row index and which of the two matrices
    auto issue_step = [&](int t, stage_t &dst) {
        int s = strip_of(t);
        s = s < h_hi ? s : h_hi - 1; // ragged tail: fetch a duplicate rather than branch
        const int c0 = chunk_of_step(t);
        const size_t strip_at = (size_t)((DOWN ? 16 : 8) * s) * ex.row_bytes; // scalar
        if constexpr (LINES) {
            constexpr int CB = FMT == 0 ? 256 : (FMT == 1 ? 64 : 32); // bytes of a chunk in a row
            const gbytes lo = weight_rows0 + strip_at + c0 * CB;
            const gbytes hi = (DOWN ? weight_rows0 + 8 * (size_t)ex.row_bytes : weight_rows1) + strip_at + c0 * CB;
            issue_lines<GPC, CPW, FMT>(dst, lo, hi, ex.row_bytes, ONE_ROUND || c0 < ncp, c0 + 1 < ncp, lane);
        } else {
            const gbytes p = DOWN ? weight_rows0 + strip_at + lane_row16
                                  : (r < 8 ? weight_rows0 + strip_at : weight_rows1 + strip_at) + lane_row8;
            issue_weights<LK, CPW, FMT>(dst, p, c0, ncp, q);
        }
    };
    // Quantized formats: the group scales of the steps [t0, t0 + NST), one per chunk (a chunk never crosses a
    // group).  They travel apart from the weight stages, a whole loop iteration ahead and issued before that
    // iteration's weight loads: the registers they land in are carried around the loop, which costs a copy
    // at the end of every iteration, and the completion counter is in order -- a copy of a load issued
    // last would wait for every load in flight, a copy of the oldest ones waits for nothing.
    static_assert(CPW <= 2, "two chunk scales to a word");
    uint32_t sc_cur[NST][NSW], sc_next[NST][NSW];
    const gbf16 scale_rows0 = ex.s0, scale_rows1 = ex.s1;
    auto issue_scales = [&](int t0 /* even */, uint32_t (&dst)[NST][NSW]) __attribute__((always_inline)) {
        if constexpr (FMT != 0) {
#pragma unroll
            for (int u = 0; u < NST; ++u) {
                int s = strip_of(t0 + u);
                s = s < h_hi ? s : h_hi - 1;
                const size_t strip_at = (size_t)((DOWN ? 16 : 8) * s) * ex.G; // scalar
                const gbf16 sp = DOWN ? scale_rows0 + strip_at + (uint32_t)(r * ex.G)
                                      : (r < 8 ? scale_rows0 + strip_at : scale_rows1 + strip_at) + (uint32_t)((r & 7) * ex.G);
                const int c0 = chunk_of_step(t0 + u);
                if constexpr (GPC > 1) {
                    // the groups of the wavefront's chunks are neighbours, GPC (even) of them per chunk
#pragma unroll
                    for (int i = 0; i < CPW; ++i)
                        if (c0 + i < ncp) {
#pragma unroll
                            for (int g = 0; g < GPC; g += 2)
                                dst[u][(i * GPC + g) >> 1] = *reinterpret_cast<gvec4>(sp + (c0 + i) * GPC + g);
                        }
                } else if (CPW == 2 && a.group == CHUNK && c0 + 1 < ncp) {
                    // the two chunks' scales are neighbours (a row of an odd number of them may start at any even address)
                    dst[u][0] = *reinterpret_cast<gscales2>(sp + c0);
                } else {
                    uint32_t v = 0;
#pragma unroll
                    for (int i = 0; i < CPW; ++i)
                        if (c0 + i < ncp) v |= (uint32_t)sp[((c0 + i) * CHUNK) / a.group] << (16 * i);
                    dst[u][0] = v;
                }
            }
        }
    };
    auto rotate_scales = [&]() {
        if constexpr (FMT != 0) {
#pragma unroll
            for (int u = 0; u < NST; ++u)
#pragma unroll
                for (int i = 0; i < NSW; ++i) sc_cur[u][i] = sc_next[u][i];
        }
    };

    f32x4 acc[NB][2][MT];
#pragma unroll
    for (int p = 0; p < NB; ++p)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) acc[p][b][mt] = f32x4{0.f, 0.f, 0.f, 0.f};

    auto multiply_step = [&](int t, const stage_t &cur, const uint32_t (&sc)[NSW], f32x4 (&to)[MT]) __attribute__((always_inline)) {
        const int c0 = chunk_of_step(t);
#ifdef DX_TRACE_STEPS
        if (threadIdx.x == 0 && (blockIdx.x & 63) == 37) {
            const unsigned int n = g_nsteps[DOWN][blockIdx.x >> 6]++;
            if (n < 256) g_steps[DOWN][blockIdx.x >> 6][n] = wall_clock64() | ((unsigned long long)FMT << 60) | ((unsigned long long)(t == 0) << 59);
        }
#endif
        if (strip_of(t) < h_hi) { // wavefront-uniform; a strip past the end was not fetched either, or is a duplicate
            if constexpr (LINES) multiply_lines<GPC, CPW, FMT, MT>(cur, x, bias, sc, ONE_ROUND || c0 < ncp, c0 + 1 < ncp, ll, lane, area(), to);
            else multiply<LK, CPW, FMT, MT>(cur, x, bias, sc[0], c0, ncp, to);
        }
    };
    // a batch's strip pairs are complete: park the partial sums (zeros for a missing second strip)
    auto park_and_finish = [&](int batch, f32x4 (&sums)[2][MT]) __attribute__((always_inline)) {
        const bool live = h_lo + 2 * (batch * SPP + g) < h_hi;
#pragma unroll
        for (int bb = 0; bb < 2; ++bb)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                if (live) red[pb][wave][bb * 2 + mt][lane] = sums[bb][mt];
                sums[bb][mt] = f32x4{0.f, 0.f, 0.f, 0.f};
            }
        finish(batch);
    };

    // prologue: the first NST-1 strips (nhalf is even and >= 2) go out before anything that depends on
    // the routing arrays, so that they are in flight while the token rows are looked up
#pragma unroll
    for (int i = 0; i < NST - 1; ++i)
        if (i < nhalf && strip_of(i) < h_hi) issue_step(i, st[i]);
    issue_scales(0, sc_cur);

    // token rows of this run (A operand)
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int h = 0; h < (LINES ? 2 : 1); ++h) {
            int slot = mb * 32 + 16 * mt + (LINES ? 8 * h + (lane >> 3) : r);
            slot = slot < ex.m ? slot : ex.m - 1;
            if constexpr (DOWN) {
                arow[mt][h] = (gbf16)a.h + (size_t)(ex.seg0 + slot) * a.fmax;
            } else {
                int tok = slot;
                if (!ex.shared) {
                    const int p = ex.perm_lds ? ex.perm_lds[ex.seg0 + slot] : a.perm[ex.seg0 + slot];
                    tok = p / a.k;
                }
                arow[mt][h] = (gbf16)a.x + (size_t)tok * ex.K;
            }
        }
    if constexpr (ONE_ROUND) {
        fetch_tokens(kw * CPW);
        auto do_step = [&](int t, const stage_t &cur, const uint32_t (&sc)[NSW],
                           int b /* = t & 1, compile-time at every call */) __attribute__((always_inline)) {
            multiply_step(t, cur, sc, acc[0][b]);
            if (b) park_and_finish(t >> 1, acc[0]);
        };
        int t = 0;
        // steady state: NST strips per iteration, every prefetch unconditional (NST is even, so stage i always
        // holds a strip with b = i & 1)
        for (; t + 2 * NST - 2 < nhalf; t += NST) {
            issue_scales(t + NST, sc_next);
#pragma unroll
            for (int i = 0; i < NST; ++i) {
                issue_step(t + i + NST - 1, st[(i + NST - 1) % NST]);
                do_step(t + i, st[i], sc_cur[i], i & 1);
            }
            rotate_scales();
        }
        // drain: the same, with the prefetch guarded (an unconditional prefetch of duplicates past the end of
        // the run was measured: the next run then starts behind those loads, 72.6 -> 79.1 us per C2 step)
        for (; t < nhalf; t += NST) {
            if (t + NST < nhalf) issue_scales(t + NST, sc_next);
#pragma unroll
            for (int i = 0; i < NST; ++i) {
                if (t + i < nhalf) {
                    if (t + i + NST - 1 < nhalf && strip_of(t + i + NST - 1) < h_hi) issue_step(t + i + NST - 1, st[(i + NST - 1) % NST]);
                    do_step(t + i, st[i], sc_cur[i], i & 1);
                }
            }
            rotate_scales();
        }
    } else {
        // one iteration: NB pairs in one K round (2 * NB steps, a multiple of NST)
        static_assert((2 * NB) % NST == 0, "the stages come round with every iteration");
        for (int t = 0; t < nhalf; t += 2 * NB) {
            fetch_tokens(chunk_of_step(t));
#pragma unroll
            for (int i = 0; i < 2 * NB; ++i) {
                if (i % NST == 0 && t + i + NST < nhalf) issue_scales(t + i + NST, sc_next);
                if (t + i + NST - 1 < nhalf && strip_of(t + i + NST - 1) < h_hi) issue_step(t + i + NST - 1, st[(i + NST - 1) % NST]);
                multiply_step(t + i, st[i % NST], sc_cur[i % NST], acc[i >> 1][i & 1]);
                if (i % NST == NST - 1) rotate_scales();
            }
            const int it = t / (2 * NB);
            if (it % rounds == rounds - 1) {
#pragma unroll
                for (int p = 0; p < NB; ++p) {
                    const int batch = it / rounds * NB + p;
                    if (batch < nbatch) park_and_finish(batch, acc[p]);
                }
            }
        }
    }
}

// LDS of the partition: per expert its tokens, its segment start and the prefix of the cost units
struct partition_lds {
    uint32_t cum[kMaxExperts + 1];
    int seg_start[kMaxExperts], seg_tokens[kMaxExperts];
    uint32_t wave_tot[kWaves];
    int wave_cnt[kWaves];
    int e_first;
};

// The partition: cost units of every expert, exclusive prefix, this block's unit range [ub0, ub1) and the
// first expert in it.  All threads; ends with a barrier.
template <bool DOWN>
__device__ __forceinline__ void build_partition(const dx_fwd_args &a, partition_lds &pl, uint32_t &ub0, uint32_t &ub1)
{
    const int nE = a.E + (a.shared ? 1 : 0);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    auto tokens_of = [&](int e) {
        return e == a.E ? a.T : a.offsets[e + 1] - a.offsets[e];
    };
    auto strips_of = [&](int e) { return DOWN ? a.d / 16 : (e == a.E ? a.shared_f : a.f) / 8; };
    auto fmt_of = [&](int e) { return e == a.E ? (uint32_t)DX_FMT_BF16 : a.table[e].fmt; };
    const int R = (nE + kThreads - 1) / kThreads; // experts per thread, consecutive
    uint32_t mine[3] = {0, 0, 0}, local = 0;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const int e = tid * R + i;
        if (i < R && e < nE) {
            const int m = tokens_of(e);
            pl.seg_tokens[e] = m;
            pl.seg_start[e] = e == a.E ? a.T * a.k : a.offsets[e];
            if (m > 0)
                mine[i] = (uint32_t)((m + 31) / 32) * strips_of(e) * units_of<DOWN>(fmt_of(e), m) + kRunUnits<DOWN>;
            local += mine[i];
        }
    }
    const uint32_t inc = dx_route_core::wave_scan_inclusive(local);
    if (lane == 63) pl.wave_tot[wave] = inc;
    if (tid == 0) pl.e_first = nE;
    __syncthreads();
    uint32_t base = 0, U = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        const uint32_t t = pl.wave_tot[w];
        if (w < wave) base += t;
        U += t;
    }
    uint32_t run = base + inc - local;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const int e = tid * R + i;
        if (i < R && e < nE) {
            pl.cum[e] = run;
            run += mine[i];
        }
    }
    if (tid == 0) pl.cum[nE] = U;
    // this block's unit range (in double: exact for these sizes, no 64-bit integer division, and every
    // block evaluates the same expression for a boundary it shares)
    const double share = (double)U / (double)gridDim.x;
    ub0 = (uint32_t)(share * (double)blockIdx.x);
    ub1 = blockIdx.x + 1 == gridDim.x ? U : (uint32_t)(share * (double)(blockIdx.x + 1));
    __syncthreads();
    // the expert whose unit range contains ub0 (experts without work have empty ranges)
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const int e = tid * R + i;
        if (i < R && e < nE && pl.cum[e] <= ub0 && ub0 < pl.cum[e + 1]) pl.e_first = e;
    }
    __syncthreads();
}

// The expert of every place in the segments, for the down kernel of a call of a few tokens (one block).
__device__ __forceinline__ void write_place_experts(const dx_fwd_args &a)
{
    int32_t *out = reinterpret_cast<int32_t *>(a.tiles);
    for (int e = threadIdx.x; e < a.E; e += kThreads)
        for (int at = a.offsets[e]; at < a.offsets[e + 1] && at < a.T * a.k; ++at) out[at] = e;
}

// This block's share: the strips whose first unit lies in [ub0, ub1), run by run.
template <int LK, int GPC, int CPW, bool DOWN, int MODE>
__device__ __forceinline__ void run_share(const dx_fwd_args &a, const partition_lds &pl, uint32_t ub0, uint32_t ub1,
                                          lds_ints perm_lds, f32x4 (*red)[kWaves][4][64])
{
    const int nE = a.E + (a.shared ? 1 : 0);
    int pb = 0;
    if (ub0 >= ub1) return;
    for (int e = pl.e_first; e < nE && pl.cum[e] < ub1; ++e) {
        const uint32_t ue = pl.cum[e + 1] - pl.cum[e];
        if (ue == 0) continue;
        expert_ctx ex;
        ex.shared = e == a.E;
        ex.m = pl.seg_tokens[e];
        ex.seg0 = pl.seg_start[e];
        ex.perm_lds = perm_lds;
        const dx_handle hd = ex.shared ? *a.shared : a.table[e];
        ex.fmt = (int)hd.fmt;
        const int fe = ex.shared ? a.shared_f : a.f;
        ex.K = DOWN ? fe : a.d;
        ex.G = ex.K / a.group;
        ex.row_bytes = ex.fmt == DX_FMT_BF16 ? (uint32_t)ex.K * 2 : (ex.fmt == DX_FMT_INT4G ? (uint32_t)ex.K / 2 : (uint32_t)ex.K / 4);
        ex.w0 = (gbytes)(DOWN ? hd.w_down : hd.w_gate);
        ex.w1 = (gbytes)(DOWN ? hd.w_down : hd.w_up);
        ex.s0 = (gbf16)(DOWN ? hd.s_down : hd.s_gate);
        ex.s1 = (gbf16)(DOWN ? hd.s_down : hd.s_up);
        const int spe = DOWN ? a.d / 16 : fe / 8; // strips per token block of this expert
        const uint32_t wgt = units_of<DOWN>((uint32_t)ex.fmt, ex.m);
        const uint32_t lo = (ub0 > pl.cum[e] ? ub0 : pl.cum[e]) - pl.cum[e];
        const uint32_t hi = (ub1 < pl.cum[e + 1] ? ub1 : pl.cum[e + 1]) - pl.cum[e];
        // strips (flattened over token blocks) whose first unit lies in [lo, hi); strip i starts
        // kRunUnits + i * wgt units into the expert's range
        constexpr uint32_t kRun = kRunUnits<DOWN>;
        const uint32_t lo_p = lo > kRun ? lo - kRun : 0, hi_p = hi > kRun ? hi - kRun : 0;
        int i = (int)((lo_p + wgt - 1) / wgt);
        const int i1 = (int)((hi_p + wgt - 1) / wgt);
        while (i < i1) {
            const int mb = i / spe;
            const int iend = i1 < (mb + 1) * spe ? i1 : (mb + 1) * spe;
            const int s_lo = i - mb * spe, s_hi = iend - mb * spe;
            const bool two = ex.m - mb * 32 > 16;
#ifdef DX_TRACE
            if (threadIdx.x == 0 && blockIdx.x < 8192) {
                g_mix[DOWN][blockIdx.x][0] += 1;
                g_mix[DOWN][blockIdx.x][1 + (ex.fmt != DX_FMT_BF16) * 2 + two] += s_hi - s_lo;
            }
#endif
            if (ex.fmt == DX_FMT_INT4G) {
                if (two) run_strips<LK, GPC, CPW, DOWN, 1, 2, MODE>(a, ex, mb, s_lo, s_hi, red, pb);
                else run_strips<LK, GPC, CPW, DOWN, 1, 1, MODE>(a, ex, mb, s_lo, s_hi, red, pb);
            } else if (ex.fmt == DX_FMT_INT2G) {
                // (16 codes per word: the library refuses int2 handles when the group is 32)
                if constexpr (LK >= 16 && GPC < 4) {
                    if (two) run_strips<LK, GPC, CPW, DOWN, 2, 2, MODE>(a, ex, mb, s_lo, s_hi, red, pb);
                    else run_strips<LK, GPC, CPW, DOWN, 2, 1, MODE>(a, ex, mb, s_lo, s_hi, red, pb);
                }
            } else {
                if (two) run_strips<LK, GPC, CPW, DOWN, 0, 2, MODE>(a, ex, mb, s_lo, s_hi, red, pb);
                else run_strips<LK, GPC, CPW, DOWN, 0, 1, MODE>(a, ex, mb, s_lo, s_hi, red, pb);
            }
            i = iend;
        }
    }
}

template <int LK, int GPC, int CPW, bool DOWN, int MODE>
__global__ __launch_bounds__(kThreads) void k_stream(dx_fwd_args a)
{
    __shared__ f32x4 red[2][kWaves][4][64]; // 64 KB: partial sums, double buffered
    __shared__ partition_lds pl;
#ifdef DX_TRACE
    const unsigned long long trace_t0 = wall_clock64();
#endif
    uint32_t ub0, ub1;
    build_partition<DOWN>(a, pl, ub0, ub1);
#ifdef DX_TRACE
    const unsigned long long trace_t1 = wall_clock64();
#endif
    if constexpr (!DOWN) {
        if (a.tiles && blockIdx.x + 1 == gridDim.x) write_place_experts(a);
    }
    run_share<LK, GPC, CPW, DOWN, MODE>(a, pl, ub0, ub1, nullptr, red);
#ifdef DX_TRACE
    if (threadIdx.x == 0 && blockIdx.x < 8192) {
        g_trace[DOWN ? 1 : 0][blockIdx.x][0] = trace_t0;
        g_trace[DOWN ? 1 : 0][blockIdx.x][1] = wall_clock64();
        g_trace[DOWN ? 1 : 0][blockIdx.x][2] = ub1 - ub0;
        g_trace[DOWN ? 1 : 0][blockIdx.x][3] = trace_t1;
    }
#endif
}

// Decode batches of at most kRoutedTokens tokens and kRoutedExperts experts: the gate/up kernel routes
// by itself.  Every block repeats the small routing computation (top-k and weights per token, counts,
// offsets and the stable permutation, as dx_route.hip does them) in its prologue and keeps the result in
// LDS, so the forward pass does not wait for a routing kernel and its round trip through memory; block 0
// also writes the routing arrays out for the down and combine kernels and for the caller, and adds the
// counts to the layer's hotness counters.
// NV = logits per lane of a token's 16-lane row (E <= 16 * NV): 8 for up to 128 experts, 32 for up to 512.
// Each thread also owns EPT consecutive experts for the counts, offsets and cost units.
constexpr int kRoutedTokens = DX_ROUTED_MAX_TOKENS, kRoutedExperts = DX_ROUTED_MAX_EXPERTS, kRoutedTopK = DX_ROUTED_MAX_TOPK;

template <int LK, int GPC, int CPW, int NV>
__global__ __launch_bounds__(kThreads) void k_stream_routed(dx_fwd_args a, dx_route_io r)
{
    constexpr int kE = 16 * NV;                 // experts this instance takes
    constexpr int EPT = kE >= kThreads ? 2 : 1; // experts per thread: E + shared <= kThreads * EPT
    __shared__ f32x4 red[2][kWaves][4][64];
    __shared__ partition_lds pl;
    __shared__ unsigned long long lds_mask[kE];
    __shared__ int lds_perm[kRoutedTokens * kRoutedTopK];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const bool writer = blockIdx.x == 0;
    const int nE = a.E + (a.shared ? 1 : 0);
    static_assert(kRoutedTokens == 2 * 4 * kWaves && kE <= kRoutedExperts && kRoutedTopK == 16,
                  "two passes of one token per 16-lane row, NV logits per lane, one selected id per lane of the row");
    static_assert(kE + 1 <= kThreads * EPT, "every expert and the shared one have a thread");
#ifdef DX_TRACE
    const unsigned long long trace_t0 = wall_clock64();
    unsigned long long trace_t1 = 0, trace_t2 = 0, trace_t3 = 0;
#endif

    for (int i = tid; i < kE; i += kThreads) lds_mask[i] = 0ull;
    unsigned long long hot_before[EPT];
    uint32_t fmt[EPT]; // of the experts tid * EPT + i
#pragma unroll
    for (int i = 0; i < EPT; ++i) {
        const int e = tid * EPT + i;
        hot_before[i] = 0ull;
        fmt[i] = DX_FMT_BF16;
        if (writer && r.hotness && e < a.E) hot_before[i] = r.hotness[e];
        if (e < a.E) fmt[i] = a.table[e].fmt;
    }
    // ---- top-k and weights: token 32 * pass + 4 * wavefront + row (rows past T repeat the last token); the
    // second pass runs for batches of more than 32 tokens
    const int c = lane & 15, t0 = 4 * wave + (lane >> 4);
    const bool second = a.T > 32; // block-uniform
    int my_id[2] = {0, 0};
    float my_w[2] = {0.f, 0.f};
    {
        float v[2][NV];
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            if (p == 0 || second) {
                const int t = t0 + 32 * p;
                dx_route_core::load_logits_rows16<NV>(r.logits + (size_t)(t < a.T ? t : a.T - 1) * a.E, c, a.E, v[p]);
            }
        }
        __syncthreads(); // the masks are clear
#ifdef DX_TRACE
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        trace_t1 = wall_clock64();
#endif
        if constexpr (NV <= 8) {
            dx_route_core::topk_rows16<NV>(v[0], a.k, lane, my_id[0], my_w[0]);
            if (second) dx_route_core::topk_rows16<NV>(v[1], a.k, lane, my_id[1], my_w[1]);
        } else {
            // wide layers: a threshold first, then the selections over the few entries at or above it; the keys
            // pass through this wavefront's eighth of `red`, which holds nothing yet
            static_assert(sizeof(red) >= sizeof(int) * 64 * NV * kWaves, "NV * 64 words of LDS per wavefront");
            auto scratch = (__attribute__((address_space(3))) int *)&red[0][0][0][0] + wave * 64 * NV;
            dx_route_core::topk_rows16_filtered<NV, 6>(v[0], a.k, lane, my_id[0], my_w[0], scratch);
            if (second) dx_route_core::topk_rows16_filtered<NV, 6>(v[1], a.k, lane, my_id[1], my_w[1], scratch);
        }
#ifdef DX_TRACE
        trace_t2 = wall_clock64();
#endif
    }
    bool have[2]; // this lane holds pair (t, c) of the pass
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        const int t = t0 + 32 * p;
        have[p] = t < a.T && c < a.k;
        if (have[p]) {
            atomicOr(&lds_mask[my_id[p]], 1ull << t);
            if (writer) {
                r.ids[(size_t)t * a.k + c] = my_id[p];
                r.w[(size_t)t * a.k + c] = my_w[p];
            }
        }
    }
    __syncthreads();
    // ---- counts, offsets (exclusive scan) and the cost units of the partition, EPT consecutive experts per thread
    int cnt[EPT], m[EPT], mine[EPT], cnt_local = 0, mine_local = 0;
#pragma unroll
    for (int i = 0; i < EPT; ++i) {
        const int e = tid * EPT + i;
        cnt[i] = m[i] = mine[i] = 0;
        if (e < a.E) cnt[i] = m[i] = __popcll(lds_mask[e]);
        else if (e == a.E && a.shared) m[i] = a.T;
        if (m[i] > 0)
            mine[i] = ((m[i] + 31) / 32) * ((e == a.E ? a.shared_f : a.f) / 8) * (int)units_of<false>(fmt[i], m[i]) +
                      (int)kRunUnits<false>;
        cnt_local += cnt[i];
        mine_local += mine[i];
    }
    const int inc = dx_route_core::wave_scan_inclusive(mine_local), cinc = dx_route_core::wave_scan_inclusive(cnt_local);
    if (lane == 63) {
        pl.wave_tot[wave] = (uint32_t)inc;
        pl.wave_cnt[wave] = cinc;
    }
    if (tid == 0) pl.e_first = nE;
    __syncthreads();
    uint32_t base = 0, U = 0;
    int cbase = 0, ctot = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        const uint32_t tu = pl.wave_tot[w];
        const int tc = pl.wave_cnt[w];
        if (w < wave) {
            base += tu;
            cbase += tc;
        }
        U += tu;
        ctot += tc;
    }
    // this block's unit range (in double: exact for these sizes, and every block evaluates the same
    // expression for a shared boundary)
    const double share = (double)U / (double)gridDim.x;
    const uint32_t ub0 = (uint32_t)(share * (double)blockIdx.x);
    const uint32_t ub1 = blockIdx.x + 1 == gridDim.x ? U : (uint32_t)(share * (double)(blockIdx.x + 1));
    {
        int off_e = cbase + cinc - cnt_local;
        uint32_t cum_e = base + (uint32_t)(inc - mine_local);
#pragma unroll
        for (int i = 0; i < EPT; ++i) {
            const int e = tid * EPT + i;
            if (e < nE) {
                pl.cum[e] = cum_e;
                pl.seg_tokens[e] = m[i];
                pl.seg_start[e] = e == a.E ? a.T * a.k : off_e;
                if (mine[i] && cum_e <= ub0 && ub0 < cum_e + (uint32_t)mine[i]) pl.e_first = e;
            }
            if (writer && e < a.E) {
                r.counts[e] = cnt[i];
                r.offsets[e] = off_e;
                if (r.hotness) r.hotness[e] = hot_before[i] + (unsigned long long)cnt[i];
            }
            off_e += cnt[i];
            cum_e += (uint32_t)mine[i];
        }
    }
    if (tid == 0) {
        pl.cum[nE] = U;
        if (writer) r.offsets[a.E] = ctot;
    }
    __syncthreads();
    // ---- the permutation: the rank of pair (t, c) inside its segment = tokens below t that chose the expert
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        if (have[p]) {
            const int t = t0 + 32 * p;
            const unsigned long long below = lds_mask[my_id[p]] & ((1ull << t) - 1ull);
            const int at = pl.seg_start[my_id[p]] + __popcll(below);
            lds_perm[at] = t * a.k + c;
            if (writer) r.perm[at] = t * a.k + c;
        }
    }
    __syncthreads();
#ifdef DX_TRACE
    trace_t3 = wall_clock64();
#endif
    run_share<LK, GPC, CPW, false, kWhole>(a, pl, ub0, ub1, (lds_ints)lds_perm, red);
#ifdef DX_TRACE
    if (threadIdx.x == 0 && blockIdx.x < 8192) {
        g_trace[0][blockIdx.x][0] = trace_t0;
        g_trace[0][blockIdx.x][1] = wall_clock64();
        g_trace[0][blockIdx.x][2] = trace_t1 - trace_t0 + ((trace_t2 - trace_t1) << 20) + ((trace_t3 - trace_t2) << 40);
        g_trace[0][blockIdx.x][3] = trace_t3;
    }
#endif
}

// ---- a call of one or two tokens: gate/up, then down and combine ----------------------------------------------
// Bound by latency: k_stream spends as long on the partition, on the starts of its runs and on the strips' meetings
// in LDS as on the few weights, and leaves O to a combine kernel.  With so few pairs there is nothing to partition and
// nothing that a matrix instruction would share: a lane multiplies and adds what it has loaded.  A wavefront asks for all
// its weights before it uses the first; the sums over lanes are DPP steps.
// Whole calls, us, with the streaming kernels and with these, on weights that no cache holds, a quarter of the experts bf16: one token,
// 30B-shaped 27.9 and 17.8 (int4/int2 26.3 and 15.4), 80B-shaped 55 and 18.9, 16 experts of 4096 x 6400 60 and 38.5, 8 of 4096 x 14336 108 and
// 71, 256 of 7168 x 2048 116 and 93; two tokens 31.8 and 25.0, 45.8 and 27.3, 93 and 65.  Three tokens with k_stream for gate/up, k_stream and
// k_down_few behind it: 30B-shaped 36.4 and 32.5, but an expert of all three is read three times: 16 of 4096 x 6400 60.6 and 68.4, 4 of
// 4096 x 4096 70.9 and 80.5.
// Which expert a pair belongs to and where its row of H is: ROUTED (the gate/up kernel writes the routing
// arrays itself): from the ids, whose segments are in increasing order.  Else the arrays are the caller's: from `offsets`
// and `perm` alone, as in the other kernels, in any order inside a segment (the gate/up kernel leaves the expert of every
// place in the list); a pair that is in no segment adds nothing.
constexpr int kFewTokens = DX_FEW_TOKENS, kFewTasks = DX_ROUTED_MAX_TOPK + 1;
static_assert(kFewTokens * DX_ROUTED_MAX_TOPK <= 64, "a pair per lane");

// wavefronts per expert of a token in k_down_few
__host__ __device__ __forceinline__ int few_split(int tasks) { return tasks < kWaves ? kWaves / tasks : 1; }

// ---- gate/up: three rows of W_gate and of W_up per wavefront and round, over all of K in steps of 2048 elements (24 KB of
// bf16, 96 registers: 3 wavefronts to a SIMD).  Groups of rows go round the experts, so that every compute unit has its part of
// the bf16 experts; blocks beyond what the chip holds at once would route again, so wavefronts go on to another group instead
// (30B-shaped, T = 2: 24.6 -> 20.3; with a shared expert of its own width a fixed number of wavefronts per expert is 27.4 against 21.6 of
// k_stream; both tokens' experts listed twice and the second dropped 19.5 against 16.5 where all are shared).  An expert that both tokens select is read once.  K up to what the tokens may take of LDS.
constexpr int kFewWaves = 4, kFewRows = 3, kFewStep = 2048, kFewMaxK = 8192, kFewBlocks = 3;
constexpr int kFewPieces = kFewMaxK / 8; // of eight elements of a token row, in LDS

// (so that reads of neighbouring pieces and of every fourth one both spread over the banks)
__device__ __forceinline__ int few_piece_at(int p) { return p ^ ((p >> 3) & 7); }

// sum[i][0 / 1][n]: this lane's part of rows row0 + i of W_gate / W_up times token n
template <int FMT, int NT>
__device__ __forceinline__ void rows_of_few(gbytes gate, gbytes up, gbf16 s_gate, gbf16 s_up, int row0, int N, int K, int lg,
                                            const u32x4 *x0, const u32x4 *x1, int lane, float (&sum)[kFewRows][2][2])
{
    constexpr int LOADS = FMT == 0 ? 4 : 1;
    constexpr uint32_t kBias = FMT == 1 ? 8 : 2;
    const uint32_t row_bytes = FMT == 0 ? (uint32_t)K * 2 : (FMT == 1 ? (uint32_t)K / 2 : (uint32_t)K / 4), G = (uint32_t)K >> lg;
    for (int c = 0; c < K; c += kFewStep) {
        u32x4 w[kFewRows][2][LOADS];
        uint32_t sc[kFewRows][2];
        const bool ragged = c + kFewStep > K; // wavefront-uniform; lanes past the end read the row's start and count nothing
#pragma unroll
        for (int i = 0; i < kFewRows; ++i)
#pragma unroll
            for (int g = 0; g < 2; ++g) {
                const int row = row0 + i < N ? row0 + i : N - 1;
                const gbytes at = (g ? up : gate) + (size_t)row * row_bytes;
#pragma unroll
                for (int l = 0; l < LOADS; ++l) {
                    const int k0 = FMT == 0 ? c + 512 * l + 8 * lane : c + 32 * lane, k = k0 < K ? k0 : 0;
                    if constexpr (FMT == 0) w[i][g][l] = *reinterpret_cast<gvec16>(at + 2 * k);
                    else if constexpr (FMT == 1) w[i][g][l] = *reinterpret_cast<gvec16>(at + k / 2);
                    else {
                        const u32x2 t = *reinterpret_cast<gvec8>(at + k / 4);
                        w[i][g][l].x = t.x, w[i][g][l].y = t.y;
                    }
                    if constexpr (FMT != 0) sc[i][g] = (g ? s_up : s_gate)[(uint32_t)row * G + ((uint32_t)k >> lg)];
                }
            }
        __builtin_amdgcn_sched_barrier(0);
        // eight elements of the lane's tokens: piece l of its four
        auto load_x = [&](int l, float (&x)[NT][8]) {
#pragma unroll
            for (int n = 0; n < NT; ++n) {
                const u32x4 p = (n ? x1 : x0)[few_piece_at(c / 8 + (FMT == 0 ? 64 * l + lane : 4 * lane + l))];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    x[n][2 * j] = __uint_as_float(p[j] << 16);
                    x[n][2 * j + 1] = __uint_as_float(p[j] & 0xFFFF0000u);
                }
            }
        };
        float part[kFewRows][2][NT];
        if constexpr (FMT == 0) {
#pragma unroll
            for (int l = 0; l < 4; ++l) {
                const bool past = ragged && c + 512 * l + 8 * lane >= K;
                float x[NT][8];
                load_x(l, x);
#pragma unroll
                for (int i = 0; i < kFewRows; ++i)
#pragma unroll
                    for (int g = 0; g < 2; ++g) {
                        u32x4 v = w[i][g][l];
                        if (past) v = u32x4{0u, 0u, 0u, 0u};
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            const float lo = __uint_as_float(v[j] << 16), hi = __uint_as_float(v[j] & 0xFFFF0000u);
#pragma unroll
                            for (int n = 0; n < NT; ++n) sum[i][g][n] = fmaf(hi, x[n][2 * j + 1], fmaf(lo, x[n][2 * j], sum[i][g][n]));
                        }
                    }
            }
        } else {
#pragma unroll
            for (int l = 0; l < 4; ++l) {
                float x[NT][8], bias[NT];
                load_x(l, x);
#pragma unroll
                for (int n = 0; n < NT; ++n) {
                    bias[n] = 0.f;
#pragma unroll
                    for (int j = 0; j < 8; ++j) bias[n] += x[n][j];
                    bias[n] *= -(float)kBias;
                }
#pragma unroll
                for (int i = 0; i < kFewRows; ++i)
#pragma unroll
                    for (int g = 0; g < 2; ++g) {
#pragma unroll
                        for (int n = 0; n < NT; ++n) part[i][g][n] = l == 0 ? bias[n] : part[i][g][n] + bias[n];
                        if constexpr (FMT == 1) { // element 2 b in the low nibble of byte b; flipped: code + 8
                            const uint32_t f = w[i][g][0][l] ^ 0x88888888u, lo = f & 0x0F0F0F0Fu, hi = (f >> 4) & 0x0F0F0F0Fu;
#pragma unroll
                            for (int b = 0; b < 4; ++b)
#pragma unroll
                                for (int n = 0; n < NT; ++n)
                                    part[i][g][n] = fmaf((float)((hi >> (8 * b)) & 255u), x[n][2 * b + 1],
                                                         fmaf((float)((lo >> (8 * b)) & 255u), x[n][2 * b], part[i][g][n]));
                        } else { // element 4 b + q in bits 2 q of byte b of the half word; flipped: code + 2
                            const uint32_t f = (w[i][g][0][l >> 1] ^ 0xAAAAAAAAu) >> (16 * (l & 1));
#pragma unroll
                            for (int q = 0; q < 4; ++q)
#pragma unroll
                                for (int b = 0; b < 2; ++b)
#pragma unroll
                                    for (int n = 0; n < NT; ++n)
                                        part[i][g][n] = fmaf((float)((f >> (8 * b + 2 * q)) & 3u), x[n][4 * b + q], part[i][g][n]);
                        }
                    }
            }
#pragma unroll
            for (int i = 0; i < kFewRows; ++i)
#pragma unroll
                for (int g = 0; g < 2; ++g) {
                    const float scale = ragged && c + 32 * lane >= K ? 0.f : __uint_as_float(sc[i][g] << 16);
#pragma unroll
                    for (int n = 0; n < NT; ++n) sum[i][g][n] = fmaf(scale, part[i][g][n], sum[i][g][n]);
                }
        }
    }
}

template <int NV, bool ROUTED>
__global__ __launch_bounds__(64 * kFewWaves, kFewBlocks) void k_gate_up_few(dx_fwd_args a, dx_route_io r)
{
    constexpr int THREADS = 64 * kFewWaves, HOT = (16 * NV + THREADS - 1) / THREADS;
    __shared__ u32x4 xs[kFewTokens * kFewPieces];
    static_assert(NV <= 8 || sizeof(xs) >= sizeof(int) * kFewWaves * 64 * NV, "the wide selection's keys fit in front of the tokens");
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), P = a.T * a.k;
    const int pieces = (a.d + kFewStep - 1) / kFewStep * (kFewStep / 8); // of a token, with zeros up to a whole step
    const bool writer = ROUTED && blockIdx.x == 0;
    float v[ROUTED ? NV : 1];
    unsigned long long hot_before[HOT] = {};
    if constexpr (ROUTED) {
        const int t = lane >> 4;
        dx_route_core::load_logits_rows16<NV>(r.logits + (size_t)(t < a.T ? t : a.T - 1) * a.E, lane & 15, a.E, v);
        if (writer && r.hotness) {
#pragma unroll
            for (int i = 0; i < HOT; ++i)
                if (tid + i * THREADS < a.E) hot_before[i] = r.hotness[tid + i * THREADS];
        }
    }
    auto piece = [&](int i) { // of token i / pieces
        const int t = i >= pieces, p = t ? i - pieces : i;
        return p * 8 < a.d ? *reinterpret_cast<gvec16>((gbf16)a.x + (size_t)t * a.d + p * 8) : u32x4{0u, 0u, 0u, 0u};
    };
    auto keep = [&](int i, u32x4 x) {
        const int t = i >= pieces, p = t ? i - pieces : i;
        xs[t * kFewPieces + few_piece_at(p)] = x;
    };
    const u32x4 x_first = piece(tid);
    // (the handles' lines into L2, while the routing runs)
    uint32_t touched = 0;
    if constexpr (ROUTED) {
#pragma unroll
        for (int i = 0; i < NV / 8; ++i) touched |= a.table[min(2 * (64 * i + lane), a.E - 1)].fmt;
    }
    // Of this lane's pair (not routed: of the place of this number in the segments): the expert; whether it has one; its token
    // (not routed).  Lanes that stand for an item of work: routed: whose pair is its expert's first; else whose place is the first
    // or at an even distance from it, and those of them with a second place.
    int my_id = 0, my_t = 0;
    float my_w = 0.f;
    bool has_pair = false;
    unsigned long long first = 0, second = 0;
    if constexpr (ROUTED) {
        if constexpr (NV <= 8) dx_route_core::topk_rows16<NV>(v, a.k, lane, my_id, my_w);
        else dx_route_core::topk_rows16_filtered<NV, 6>(v, a.k, lane, my_id, my_w, (__attribute__((address_space(3))) int *)xs + wave * 64 * NV);
        has_pair = (lane >> 4) < a.T && (lane & 15) < a.k;
        bool again = false; // an earlier token has the expert
        if (a.T == 2) {
            for (int j = 0; j < a.k; ++j) again |= lane >= 16 && __builtin_amdgcn_readlane(my_id, j) == my_id;
        }
        first = __ballot(has_pair && !again);
    } else {
        // every expert with a segment tells the lane of its first place (lane 63 stands for none: there are at most 32 places);
        // all loads of a round are asked for before the first is waited for.  (dx_moe_forward, us, with groups of rows dealt out over
        // places, each group looking for its place in the offsets, and now: two tokens with the same experts, 30B-shaped 22.5 and
        // 19.5, 80B-shaped 26.5 and 21.3, 8 of 2048 x 768 21.7 and 19.0; 1024 experts of 2048 x 512, T = 1 17.9 and 14.6.)
        static_assert(kFewTokens * DX_ROUTED_MAX_TOPK < 63, "a place per lane, and one more lane");
        const int pair = a.perm[lane < P ? lane : 0];
        const int last = a.offsets[a.E];
        int told = 0; // 1 + expert
        for (int e0 = 0; e0 < a.E; e0 += 256) { // wavefront-uniform
            int o0[4], o1[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int el = min(e0 + 64 * i + lane, a.E - 1);
                o0[i] = a.offsets[el], o1[i] = a.offsets[el + 1];
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int el = e0 + 64 * i + lane;
                const bool has = (el < a.E) & (0 <= o0[i]) & (o0[i] < o1[i]) & (o0[i] < P);
                told |= __builtin_amdgcn_ds_permute(4 * (has ? o0[i] : 63), has ? el + 1 : 0);
            }
        }
        const int end = min(P, last);
        my_t = pair / a.k;
        const unsigned long long starts = __ballot(told != 0), up_to = starts & (~0ull >> (63 - lane));
        const int begin = up_to ? 63 - __builtin_clzll(up_to) : 0;
        my_id = __shfl(told, begin, 64) - 1;
        has_pair = up_to != 0ull && lane < end;
        first = __ballot(has_pair && ((lane - begin) & 1) == 0);
        second = first & __ballot(lane + 1 < end && ((starts >> (lane + 1 & 63)) & 1) == 0ull);
        if (blockIdx.x == 0 && wave == 0 && has_pair) reinterpret_cast<int32_t *>(a.tiles)[lane] = my_id; // for the down kernel
    }
    const int tasks = __popcll(first);
    // ---- the wavefront's groups of rows: the shared expert's first, then those of the items in turn.  Of a group: the expert, its
    // first place in the segments and its tokens
    const int shared_groups = a.shared ? (a.shared_f + kFewRows - 1) / kFewRows : 0, groups = shared_groups + tasks * ((a.f + kFewRows - 1) / kFewRows);
    int e, pos, n_tok, t0, t1, row0;
    auto take = [&](int group) {
        e = a.E, pos = P, n_tok = a.T, t0 = 0, t1 = a.T - 1, row0 = group * kFewRows;
        if (group < shared_groups) return;
        const int item = (group - shared_groups) % tasks, before = __popcll(first & ((1ull << lane) - 1ull));
        const int src = __builtin_ctzll(__ballot(((first >> lane) & 1ull) != 0ull && before == item));
        row0 = (group - shared_groups) / tasks * kFewRows;
        e = __builtin_amdgcn_readlane(my_id, src);
        if constexpr (ROUTED) {
            pos = __popcll(__ballot(has_pair && my_id < e));
            n_tok = __popcll(__ballot(has_pair && my_id == e));
            t0 = src >> 4;
        } else {
            pos = src;
            n_tok = 1 + (int)((second >> src) & 1ull);
            t0 = __builtin_amdgcn_readlane(my_t, src);
            t1 = __builtin_amdgcn_readlane(my_t, src + n_tok - 1);
        }
    };
    const int stride = (int)gridDim.x * kFewWaves;
    int group = (int)blockIdx.x * kFewWaves + wave;
    if (group < groups) take(group);
    asm volatile("" ::"v"(touched));
    if constexpr (ROUTED && NV > 8) __syncthreads(); // the keys are done with
    keep(tid, x_first);
    for (int i = tid + THREADS; i < a.T * pieces; i += THREADS) keep(i, piece(i));
    if constexpr (ROUTED) { // the routing arrays, for the down kernel and the caller (here, not behind the rows, whose registers are all in use)
        if (writer) {
            int below[HOT] = {}, count[HOT] = {}, at = 0;
            for (int t = 0; t < a.T; ++t)
                for (int j = 0; j < a.k; ++j) {
                    const int id = __builtin_amdgcn_readlane(my_id, 16 * t + j);
                    at += id < my_id || (id == my_id && 16 * t + j < lane);
#pragma unroll
                    for (int i = 0; i < HOT; ++i) {
                        below[i] += id < tid + i * THREADS;
                        count[i] += id == tid + i * THREADS;
                    }
                }
            if (wave == 0 && has_pair) {
                const int p = (lane >> 4) * a.k + (lane & 15);
                r.ids[p] = my_id;
                r.w[p] = my_w;
                r.perm[at] = p;
            }
#pragma unroll
            for (int i = 0; i < HOT; ++i) {
                const int ex = tid + i * THREADS;
                if (ex < a.E) {
                    r.counts[ex] = count[i];
                    r.offsets[ex] = below[i];
                    if (r.hotness) r.hotness[ex] = hot_before[i] + (unsigned long long)count[i];
                }
            }
            if (tid == 0) r.offsets[a.E] = P;
        }
    }
    __syncthreads();
    for (; group < groups;) { // wavefront-uniform
        const int N = e == a.E ? a.shared_f : a.f, lg = __builtin_ctz((unsigned)a.group);
        const dx_handle *h = e == a.E ? a.shared : a.table + e;
        const dx_handle hd = *h;
        const u32x4 *x0 = xs + t0 * kFewPieces, *x1 = xs + t1 * kFewPieces;
        float sum[kFewRows][2][2] = {};
        auto rows = [&](auto fmt, auto nt) {
            rows_of_few<decltype(fmt)::value, decltype(nt)::value>((gbytes)hd.w_gate, (gbytes)hd.w_up, (gbf16)hd.s_gate, (gbf16)hd.s_up,
                                                                   row0, N, a.d, lg, x0, x1, lane, sum);
        };
        auto any = [&](auto nt) {
            if (hd.fmt == DX_FMT_INT4G) rows(std::integral_constant<int, 1>{}, nt);
            else if (hd.fmt == DX_FMT_INT2G) rows(std::integral_constant<int, 2>{}, nt);
            else rows(std::integral_constant<int, 0>{}, nt);
        };
        if (n_tok == 1) any(std::integral_constant<int, 1>{});
        else any(std::integral_constant<int, 2>{});
#pragma unroll
        for (int n = 0; n < 2; ++n) {
            if (n < n_tok) {
                float hv[kFewRows];
#pragma unroll
                for (int i = 0; i < kFewRows; ++i) {
                    const float g = dx_route_core::wave_sum(sum[i][0][n]), u = dx_route_core::wave_sum(sum[i][1][n]);
                    hv[i] = g / (1.f + expf(-g)) * u;
                }
                if (lane == 0) {
                    dx_bf16 *out = a.h + (size_t)(pos + n) * a.fmax + row0;
#pragma unroll
                    for (int i = 0; i < kFewRows; ++i)
                        if (row0 + i < N) out[i] = (dx_bf16)float_to_bf16_rne(hv[i]);
                }
            }
        }
        group += stride;
        if (group < groups) take(group);
    }
}

// ---- down and combine: block (8 columns, token).  Its items, an expert each (or a part of K where there are fewer than eight), go round
// its wavefronts: an expert's rows of W_down times the pair's row of H, a 16-lane row to a row, up to six chunks of 128 elements
// in flight; the results meet in LDS, where they are weighted and added in the order of the slots as k_combine does.  Contractions
// that are multiples of 128.  (8 columns because d / 16 blocks leave half of the chip idle at d = 2048, and a compute unit takes
// in 28 GB/s past L2.  One token of the 30B-shaped layer: 7.7 us for 25 MB, 10.2 with 16 columns.)
constexpr int kFewCols = 8, kFewDownWaves = 16, kFewChunks = 6; // columns of a block, wavefronts at most, chunks in flight

// sum[p]: this lane's part of row 4 p + lane / 16 of eight rows of W_down times a row of H, over the chunks [c0, c1) of 128
// elements, of which a lane has eight
template <int FMT>
__device__ __forceinline__ void columns_of_few(gbf16 h_row, gbytes w, gbf16 sc, int K, int lg, int c0, int c1, int lane, float (&sum)[2])
{
    constexpr uint32_t kBias = FMT == 1 ? 8 : 2;
    const uint32_t row_bytes = FMT == 0 ? (uint32_t)K * 2 : (FMT == 1 ? (uint32_t)K / 2 : (uint32_t)K / 4), G = (uint32_t)K >> lg;
    const int row = lane >> 4, l = lane & 15;
    for (int c = c0; c < c1; c += kFewChunks) { // wavefront-uniform
        u32x4 xp[kFewChunks], wp[kFewChunks][2];
        uint32_t scales[kFewChunks][2];
#pragma unroll
        for (int i = 0; i < kFewChunks; ++i) {
            const int cc = c + i < c1 ? c + i : c1 - 1, k = 128 * cc + 8 * l;
            xp[i] = *reinterpret_cast<gvec16>(h_row + k);
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                const uint32_t r = 4 * p + row;
                const gbytes at = w + r * row_bytes;
                if constexpr (FMT == 0) wp[i][p] = *reinterpret_cast<gvec16>(at + 2 * k);
                else if constexpr (FMT == 1) wp[i][p].x = *reinterpret_cast<gvec4>(at + k / 2);
                else wp[i][p].x = *reinterpret_cast<gbf16>(at + k / 4);
                if constexpr (FMT != 0) scales[i][p] = sc[r * G + ((uint32_t)k >> lg)];
            }
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < kFewChunks; ++i) {
            if (c + i < c1) { // wavefront-uniform
                float x[8], bias = 0.f;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    x[2 * j] = __uint_as_float(xp[i][j] << 16);
                    x[2 * j + 1] = __uint_as_float(xp[i][j] & 0xFFFF0000u);
                }
                if constexpr (FMT != 0) {
#pragma unroll
                    for (int j = 0; j < 8; ++j) bias += x[j];
                    bias *= -(float)kBias;
                }
#pragma unroll
                for (int p = 0; p < 2; ++p) {
                    if constexpr (FMT == 0) {
#pragma unroll
                        for (int j = 0; j < 4; ++j)
                            sum[p] = fmaf(__uint_as_float(wp[i][p][j] & 0xFFFF0000u), x[2 * j + 1],
                                          fmaf(__uint_as_float(wp[i][p][j] << 16), x[2 * j], sum[p]));
                    } else {
                        float part = bias; // code j in bits BITS * j; flipped: code + kBias
                        constexpr int BITS = FMT == 1 ? 4 : 2;
                        const uint32_t f = wp[i][p].x ^ (FMT == 1 ? 0x88888888u : 0xAAAAAAAAu);
#pragma unroll
                        for (int j = 0; j < 8; ++j) part = fmaf((float)((f >> (BITS * j)) & ((1u << BITS) - 1)), x[j], part);
                        sum[p] = fmaf(__uint_as_float(scales[i][p] << 16), part, sum[p]);
                    }
                }
            }
        }
    }
}

template <bool ROUTED>
__global__ __launch_bounds__(64 * kFewDownWaves) void k_down_few(dx_fwd_args a)
{
    __shared__ float part[kFewTasks][kFewCols]; // (a task per item, or at most eight items)
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, waves = blockDim.x >> 6;
    const int t = blockIdx.y, strip = blockIdx.x, P = a.T * a.k;
    const int tasks = a.k + (a.shared ? 1 : 0);
    const int split = few_split(tasks); // wavefronts per expert
    // lane i: routed: the expert of pair i; else the expert and the pair of place i
    const int at_i = lane < P ? lane : 0;
    int expert_i = ROUTED ? a.ids[at_i] : reinterpret_cast<const int32_t *>(a.tiles)[at_i], pair_i = -1;
    const float w_j = a.w[t * a.k + (lane < a.k ? lane : 0)];
    if constexpr (ROUTED) {
        expert_i = lane < P ? expert_i : 0x7fffffff;
    } else { // (places outside the segments are dropped after the loads)
        const int p = a.perm[at_i], first = a.offsets[0], end = a.offsets[a.E];
        pair_i = lane >= first && lane < min(P, end) ? p : -1;
    }
    for (int item = wave; item < tasks * split; item += waves) {
        const int j = item / split, piece = item % split;
        const bool shared = j == a.k;
        // the expert, and the pair's place in the segments
        int e = a.E, pos = P + t;
        if (!shared) {
            if constexpr (ROUTED) { // pairs of lower experts, and of the same expert from tokens in front
                e = __builtin_amdgcn_readlane(expert_i, t * a.k + j);
                pos = __popcll(__ballot(expert_i < e)) + __popcll(__ballot(expert_i == e && lane < t * a.k));
            } else {
                const unsigned long long at = __ballot(pair_i == t * a.k + j);
                if (at == 0ull) {
                    if (lane < kFewCols) part[item][lane] = 0.f;
                    continue;
                }
                pos = __builtin_ctzll(at);
                e = __builtin_amdgcn_readlane(expert_i, pos);
            }
        }
        const dx_handle *h = shared ? a.shared : a.table + e;
        const dx_handle hd = *h;
        const int K = shared ? a.shared_f : a.f, nc = K / 128, per = (nc + split - 1) / split;
        const int c0 = piece * per, c1 = c0 + per < nc ? c0 + per : nc;
        const gbf16 h_row = (gbf16)a.h + (size_t)pos * a.fmax;
        const gbytes w = (gbytes)hd.w_down;
        const int lg = __builtin_ctz((unsigned)a.group), G = K >> lg;
        const gbf16 sc = (gbf16)hd.s_down + (size_t)strip * kFewCols * G;
        const size_t row0 = (size_t)strip * kFewCols;
        float sum[2] = {0.f, 0.f};
        if (c0 < c1) {
            if (hd.fmt == DX_FMT_INT4G) columns_of_few<1>(h_row, w + row0 * (K / 2), sc, K, lg, c0, c1, lane, sum);
            else if (hd.fmt == DX_FMT_INT2G) columns_of_few<2>(h_row, w + row0 * (K / 4), sc, K, lg, c0, c1, lane, sum);
            else columns_of_few<0>(h_row, w + row0 * K * 2, sc, K, lg, c0, c1, lane, sum);
        }
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            const float s = dx_route_core::row_sum(sum[p]);
            if ((lane & 15) == 15) part[item][4 * p + (lane >> 4)] = s;
        }
    }
    __syncthreads();
    if (threadIdx.x < 64) {
        const int col = lane & (kFewCols - 1);
        float acc = 0.f, sh = 0.f;
        for (int j = 0; j < tasks; ++j) {
            float v = 0.f;
            for (int i = 0; i < split; ++i) v += part[j * split + i][col];
            if (j < a.k) acc += __int_as_float(__builtin_amdgcn_readlane(__float_as_int(w_j), j)) * v;
            else sh = v;
        }
        if (a.shared) acc += sh;
        if (lane < kFewCols) a.y[(size_t)t * a.d + strip * kFewCols + lane] = (dx_bf16)float_to_bf16_rne(acc);
    }
}

// ---- combine: y[t] = sum_j w[t,j] * O[t*k+j] (+ O[T*k+t] of the shared expert) ----------
// The rows are fetched eight at a time before they are added (in the order of j), so that a thread has
// its loads in flight together instead of one round trip per row.
__global__ __launch_bounds__(256) void k_combine(dx_fwd_args a)
{
    const int t = blockIdx.y;
    const int c = (blockIdx.x * 256 + threadIdx.x) * 4;
    if (c >= a.d) return;
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    float4 sh = make_float4(0.f, 0.f, 0.f, 0.f);
    if (a.shared) sh = *reinterpret_cast<const float4 *>(a.o + ((size_t)a.T * a.k + t) * a.d + c);
    for (int j0 = 0; j0 < a.k; j0 += 8) {
        float4 o[8];
        float wj[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int j = j0 + u < a.k ? j0 + u : a.k - 1; // past the end: a duplicate that is not added
            wj[u] = a.w[(size_t)t * a.k + j];
            o[u] = *reinterpret_cast<const float4 *>(a.o + ((size_t)t * a.k + j) * a.d + c);
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            if (j0 + u < a.k) {
                acc.x += wj[u] * o[u].x; acc.y += wj[u] * o[u].y; acc.z += wj[u] * o[u].z; acc.w += wj[u] * o[u].w;
            }
        }
    }
    if (a.shared) {
        acc.x += sh.x; acc.y += sh.y; acc.z += sh.z; acc.w += sh.w;
    }
    uint2 out;
    out.x = float_to_bf16_rne(acc.x) | (float_to_bf16_rne(acc.y) << 16);
    out.y = float_to_bf16_rne(acc.z) | (float_to_bf16_rne(acc.w) << 16);
    *reinterpret_cast<uint2 *>(a.y + (size_t)t * a.d + c) = out;
}

// the same with bf16 O rows: 8 columns per thread
__global__ __launch_bounds__(256) void k_combine_bf16(dx_fwd_args a)
{
    const int t = blockIdx.y;
    const int c = (blockIdx.x * 256 + threadIdx.x) * 8;
    if (c >= a.d) return;
    const dx_bf16 *ob = reinterpret_cast<const dx_bf16 *>(a.o);
    float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    auto add_row = [&](const uint4 &o, float wj) {
        const uint32_t p[4] = {o.x, o.y, o.z, o.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            acc[2 * i] += wj * __uint_as_float(p[i] << 16);
            acc[2 * i + 1] += wj * __uint_as_float(p[i] & 0xFFFF0000u);
        }
    };
    uint4 sh = make_uint4(0u, 0u, 0u, 0u);
    if (a.shared) sh = *reinterpret_cast<const uint4 *>(ob + ((size_t)a.T * a.k + t) * a.d + c);
    for (int j0 = 0; j0 < a.k; j0 += 8) { // eight rows in flight, added in the order of j
        uint4 o[8];
        float wj[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int j = j0 + u < a.k ? j0 + u : a.k - 1;
            wj[u] = a.w[(size_t)t * a.k + j];
            o[u] = *reinterpret_cast<const uint4 *>(ob + ((size_t)t * a.k + j) * a.d + c);
        }
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (j0 + u < a.k) add_row(o[u], wj[u]);
    }
    if (a.shared) add_row(sh, 1.f);
    uint4 out;
    out.x = float_to_bf16_rne(acc[0]) | (float_to_bf16_rne(acc[1]) << 16);
    out.y = float_to_bf16_rne(acc[2]) | (float_to_bf16_rne(acc[3]) << 16);
    out.z = float_to_bf16_rne(acc[4]) | (float_to_bf16_rne(acc[5]) << 16);
    out.w = float_to_bf16_rne(acc[6]) | (float_to_bf16_rne(acc[7]) << 16);
    *reinterpret_cast<uint4 *>(a.y + (size_t)t * a.d + c) = out;
}

// Chunks per wavefront for a contraction of nc chunks: the fast path needs nc = WPS * CPW with
// WPS <= 8 wavefronts; prefer the split that leaves the fewest of the 8 wavefronts without a K-part.
struct split_choice {
    int cpw;
    split_mode mode;
};

split_choice pick_split(int nc_a, int nc_b)
{
    int best = 0, best_busy = -1;
    for (int cpw = 1; cpw <= 2; ++cpw) {
        bool ok = true;
        int busy = kWaves;
        for (int nc : {nc_a, nc_b}) {
            if (nc % cpw || nc / cpw > kWaves) ok = false;
            else {
                const int wps = nc / cpw;
                busy = busy < (kWaves / wps) * wps ? busy : (kWaves / wps) * wps;
            }
        }
        if (ok && busy >= best_busy) { // ties go to the larger cpw: more bytes in flight per wavefront
            best = cpw;
            best_busy = busy;
        }
    }
    if (best) return {best, kWhole};
    if (nc_a <= 2 * kWaves && nc_b <= 2 * kWaves) return {2, kRagged};
    // Two chunks per wavefront unless many more wavefronts have work in the rounds with one (the last round of two holds few
    // chunks).  Layers of 32 experts, us with one and with two chunks: 20 chunks (0.83 and 0.63 of the places in use)
    // int4 32 tokens 54.9 and 62.4, 24 chunks (1 and 0.75) 61.2 and 65.7; 28 chunks (0.88 both) 66.5 and 69.6, int2 73.1 and
    // 67.0, 32 chunks int2 80.9 and 70.6, 40 chunks (1 and 0.83) int2 94.6 and 86.8, bf16 141 and 146.
    auto in_use = [&](int cpw) {
        const int nc = nc_a > nc_b ? nc_a : nc_b, per = (nc + cpw - 1) / cpw;
        return (double)per / ((per + kWaves - 1) / kWaves * kWaves);
    };
    return {in_use(2) >= 0.8 * in_use(1) ? 2 : 1, kRounds};
}

// A launch, optionally with events that take the start and stop time stamps of the kernel's own dispatch
// (HIP's extended launch): the duration they give is the kernel's, with no event packets inside it.
template <typename... Args>
void launch(void (*kernel)(Args...), dim3 grid, dim3 block, hipStream_t s, hipEvent_t start, hipEvent_t stop, Args... args)
{
    if (start || stop) hipExtLaunchKernelGGL(kernel, grid, block, 0, s, start, stop, 0, args...);
    else hipLaunchKernelGGL(kernel, grid, block, 0, s, args...);
}

// How a projection's contraction is cut into chunks.  Multiples of 128: chunks of 128 elements in whole lines, with
// 128 / group quantization groups each; other sizes (the group, 32 or 64, still divides them): chunks of one
// group in operand order.
template <int LK_, int GPC_>
struct chunking {
    static constexpr int LK = LK_, GPC = GPC_;
};
template <typename F>
void with_chunking(int group, int K_a, int K_b, F f)
{
    if (K_a % 128 == 0 && K_b % 128 == 0) {
        if (group == 128) f(chunking<32, 1>{});
        else if (group == 64) f(chunking<32, 2>{});
        else f(chunking<32, 4>{});
    } else {
        if (group == 64) f(chunking<16, 1>{});
        else f(chunking<8, 1>{});
    }
}
int chunk_of(int group, int K_a, int K_b) { return K_a % 128 == 0 && K_b % 128 == 0 ? 128 : group; }

// gate/up or down on the streaming kernels; r: the gate/up kernel routes in its prologue (K a fast split)
template <bool DOWN>
void launch_stream(const dx_fwd_args &a, dim3 grid, hipStream_t s, hipEvent_t start = nullptr, hipEvent_t stop = nullptr,
                   const dx_route_io *r = nullptr)
{
    const dim3 block(kThreads);
    const int K_a = DOWN ? a.f : a.d, K_b = DOWN && a.shared ? a.shared_f : K_a;
    const int chunk = chunk_of(a.group, K_a, K_b);
    const split_choice c = pick_split(K_a / chunk, K_b / chunk);
    with_chunking(a.group, K_a, K_b, [&](auto ch) {
        constexpr int LK = decltype(ch)::LK, GPC = decltype(ch)::GPC;
        if constexpr (!DOWN) {
            if (r) {
                if (a.E <= 128) {
                    if (c.cpw == 2) launch(k_stream_routed<LK, GPC, 2, 8>, grid, block, s, start, stop, a, *r);
                    else launch(k_stream_routed<LK, GPC, 1, 8>, grid, block, s, start, stop, a, *r);
                } else {
                    if (c.cpw == 2) launch(k_stream_routed<LK, GPC, 2, 32>, grid, block, s, start, stop, a, *r);
                    else launch(k_stream_routed<LK, GPC, 1, 32>, grid, block, s, start, stop, a, *r);
                }
                return;
            }
        }
        if (c.mode == kRounds) {
            // (a pair of chunks with two or four groups each and its sums do not fit the registers)
            if constexpr (LK < 32) launch(k_stream<LK, GPC, 2, DOWN, kRounds>, grid, block, s, start, stop, a);
            else if constexpr (GPC > 1) launch(k_stream<LK, GPC, 1, DOWN, kRounds>, grid, block, s, start, stop, a);
            else if (c.cpw == 2) launch(k_stream<LK, GPC, 2, DOWN, kRounds>, grid, block, s, start, stop, a);
            else launch(k_stream<LK, GPC, 1, DOWN, kRounds>, grid, block, s, start, stop, a);
        } else if (c.mode == kRagged) launch(k_stream<LK, GPC, 2, DOWN, kRagged>, grid, block, s, start, stop, a);
        else if (c.cpw == 2) launch(k_stream<LK, GPC, 2, DOWN, kWhole>, grid, block, s, start, stop, a);
        else launch(k_stream<LK, GPC, 1, DOWN, kWhole>, grid, block, s, start, stop, a);
    });
}

// groups of rows of k_gate_up_few, at most (no expert of both tokens)
long few_groups(const dx_fwd_args &a)
{
    auto of = [](int f) { return (f + kFewRows - 1) / kFewRows; };
    return (a.shared ? of(a.shared_f) : 0) + (long)a.T * a.k * of(a.f);
}

// Which kernels a call of one or two tokens takes: down, that the down projection and the combine run in k_down_few, and gate_up,
// that k_gate_up_few is in front of it.  Figures: whole calls, us, the streaming kernel and this one, a quarter of the experts bf16.
// down: blocks of 8 columns read W_down by themselves, k_stream spreads the bytes over the whole chip and reads an expert once.  So at
// most 512 chunks of W_down (8 rows of 128) per compute unit where blocks are too few: one token, top-8, f = 4096, d = 1024 (512) 37.2
// and 34.7, d = 512 (1024) 30.6 and 30.7, d = 128 (4096) 24.6 and 25.5.  And two tokens that may well have the same experts (less than
// twice as many as pairs) at most 128 chunks per compute unit: all experts the same, 8 of 2048 x 1024 (128) 28.1 and 25.4, 4 of
// 4096 x 2048, top-2 (128) 30.9 and 29.5, 8 of 4096 x 2048, top-4 (256) 44.9 and 47.2, 16 of 4096 x 1024, top-16 (512) 64 and 84.
// gate_up: where the streaming kernel needs a routing kernel in front or more than one round for K (two tokens: 64 experts of 4096 x 1024,
// top-4 41.8 and 31.5, 1024 of 2048 x 512 40.2 and 25.9), except layers without a quantized expert, whose bytes it streams faster (8 of
// 4096 x 14336 208 and 225).  Else as long as the groups of rows are at most 1.4 times the wavefronts that the chip holds: two tokens,
// 30B-shaped (1.33) 26.2 and 24.9, 64 of 2048 x 1024, top-8 (1.78) 29.7 and 30.6, 64 of 2048 x 2048, top-8 (3.6) 44.4 and 46.8; rows shorter
// than a step, which leave lanes without elements, count for more there (32 of 1024 x 512, top-16 22.7 and 25.8, 64 of 512 x 512, top-8 16.0 and 17.2).
struct few_choice {
    bool gate_up, down;
};
few_choice takes_few(const dx_fwd_args &a, int n_cu)
{
    if (a.T > kFewTokens || a.k >= kFewTasks || a.f % 128 || (a.shared && a.shared_f % 128)) return {false, false};
    const long chunks = (long)a.k * (a.f / 128) + (a.shared ? a.shared_f / 128 : 0), blocks = (long)(a.d / kFewCols) * a.T;
    const bool down = chunks * n_cu <= 512 * blocks && (a.T == 1 || 2 * a.T * a.k <= a.E || chunks * blocks <= 128L * n_cu);
    if (!down || a.d % 128 || a.d > kFewMaxK) return {false, down};
    const int nc = a.d / chunk_of(a.group, a.d, a.d);
    const bool one_launch = pick_split(nc, nc).mode == kWhole && a.E <= kRoutedExperts; // the streaming kernel would route by itself
    if (a.E > kRoutedExperts || (!one_launch && a.any_quantized)) return {true, true};
    const long rows = few_groups(a) * (a.T == 2 && a.d < kFewStep ? kFewStep / a.d : 1);
    return {5 * rows <= 7L * kFewBlocks * kFewWaves * n_cu, true};
}

// Wavefronts of a block of k_down_few: as many as let all blocks run at once (a compute unit holds 20 at 100 registers), in one round
// of items more where that leaves none without work.  T = 2, us, one wavefront to an item (nine to 17 items) and now: 64 experts of
// 2048 x 768, top-16 40.9 and 38.0, 64 of 4096 x 512, top-16 60.0 and 52.1, 64 of 4096 x 1024, top-8 and a shared one 59.3 and 56.8.
int few_down_waves(const dx_fwd_args &a, int n_cu)
{
    const int tasks = a.k + (a.shared ? 1 : 0), items = tasks * few_split(tasks);
    const int per_cu = ((a.d / kFewCols) * a.T + n_cu - 1) / n_cu, most = std::max(4, std::min(kFewDownWaves, 20 / per_cu));
    const int least = (items + most - 1) / most;
    auto waves = [&](int rounds) { return (items + rounds - 1) / rounds; };
    return waves(least) * least <= waves(least + 1) * (least + 1) ? waves(least) : waves(least + 1);
}

void launch_few(const dx_fwd_args &a, int n_cu, hipStream_t s, hipEvent_t start, hipEvent_t stop, const dx_route_io *r)
{
    const long fits = (long)kFewBlocks * n_cu, blocks = (few_groups(a) + kFewWaves - 1) / kFewWaves;
    const dim3 grid((unsigned)(blocks < fits ? blocks : fits)), block(64 * kFewWaves);
    if (!r) launch(k_gate_up_few<8, false>, grid, block, s, start, stop, a, dx_route_io{});
    else if (a.E <= 128) launch(k_gate_up_few<8, true>, grid, block, s, start, stop, a, *r);
    else launch(k_gate_up_few<32, true>, grid, block, s, start, stop, a, *r);
}

// The formats whose segments go in 256-row tiles (bits as in a.m_big).  Shapes: whole tiles of columns; the kernel addresses rows
// with 32-bit byte offsets; it reads the scales of an int4 row as aligned pairs (an even number of groups along both
// contractions).  Size: the tiles of the down projection fill the chip once, and a segment has 1024 rows on average (bf16)
// or 512 (int4, whose tiles gain more: a row of codes is expanded for twice the tokens).  Passes of layers of one format,
// us, 128-row tiles alone and with 256-row ones: bf16, 8 experts of 4096 x 14336, 768 rows on average 2440 and 2560, 1024 rows
// 3330 and 2930, 4096 rows 12170 and 10100; 30B-shaped 512 rows 889 and 932, 1024 rows 1670 and 1558.  int4, 16 experts of
// 4096 x 6400 256 rows 995 and 1055, 512 rows 1816 and 1727, 1024 rows 3480 and 3086; 30B-shaped 768 rows 1461 and 1363.  One expert
// of 4096 x 4096, 1024 rows (64 tiles of the down projection) 122 and 185.
int big_tile_formats(const dx_fwd_args &a, int n_cu)
{
    const uint64_t span_x = (uint64_t)a.T * a.d * 2, span_h = (uint64_t)a.T * (a.k + 1) * a.fmax * 2;
    if (a.d % 256 || a.f % 128 || (a.shared && a.shared_f % 128) || span_x >= (1ull << 32) || span_h >= (1ull << 32)) return 0;
    const long pairs = (long)a.T * a.k;
    if (pairs / DX_BIG_ROWS * (a.d / 256) < n_cu) return 0;
    const bool pairs_of_scales = (a.d / a.group) % 2 == 0 && (a.f / a.group) % 2 == 0;
    return (pairs >= 1024L * a.E ? 1 << DX_FMT_BF16 : 0) | (pairs >= 512L * a.E && pairs_of_scales ? 1 << DX_FMT_INT4G : 0);
}

// Whether a call runs on tiles.  Otherwise the streaming kernels take every expert.  (x starts at a multiple of the 16 bytes that a lane of the
// tiles' memory-to-LDS loads fetches; the streaming kernels' loads to registers take any address.)  Figures: us a layer, streaming and tiles.
// More than 128 tokens: tiles, because the streaming kernels read the weights of a segment once per 32 tokens (30B-shaped, 129 tokens 115 and 98, 190 tokens 143
// and 107; 80B-shaped, 129 tokens 99 and 87), but
// - not where the most row tiles that the pairs can have leave a quarter of the compute units without one, and pairs per expert are few (2048 elements of K and more; Zipf(0.5), 129, 200, 256
//   tokens: 64 experts of 7168 x 256, top-2, 108 and 132, 112 and 134, 124 and 136, 400 tokens 138 and 142; 16 of 5120 x 512, top-1, 59 and 97, 66 and 99, 75 and 100; 32 of 2048 x 256,
//   top-2, 37 and 49, 39 and 51, 42 and 52; 16 of 4096 x 1024, top-1, 256 tokens 80 and 90, 400 tokens, 1.1 tiles per compute unit, 103 and 91; many pairs: 8 of 7168 x 128, top-8, 320 tokens 126 and 121);
// - nor, K in one round and up to 160 tokens, with up to 9/4 tiles per compute unit and 12 pairs per expert (129 and 160 tokens, Zipf(0.5), Zipf(1), Zipf(1.5): 32 experts of 2048 x 1024, top-2, 57 and 67, 60 and
//   78; 57 and 64, 61 and 62; 55 and 60, 58 and 60; 128 of 2048 x 512, top-2, 63 and 66, 67 and 72; 52 and 55, 55 and 53; 45 and 52, 48 and 50; but 16 to 20 pairs, 32 of 2048 x 768, top-4,
//   160 tokens 65 and 68, 69 and 64, 67 and 59).
// With a shared expert always on tiles: all tokens are its segment (16 experts of 4096 x 128 and a shared one of 4096, 129 tokens 158 and 104).
// Up to 128 tokens thin tiles alone, O in fp32, where the streaming gate/up kernel takes K in rounds (more than 16 chunks of 128), each of which fetches the tokens
// anew.  Where K is one round the streaming kernels take all of them (30B-shaped 32 tokens 62 and 70; but 101 tokens 105 and 99, 80B-shaped 101 tokens 88 and 85: a line
// below 128 tokens is still to be found).
// - The tiles have to fill the chip, because each of them goes through all of K one step after the other: by the most row tiles that the pairs can have, two gate/up
//   tiles and three quarters of a down tile per compute unit.  Gate/up: 0.1 (8 experts of 7168 x 256, top-2) 128 tokens 54 and 109; 1.4 (16 of 8192 x 2048, top-2) 90 tokens 220 and 236;
//   1.6 to 2.1 (32 of 8192 x 1536, top-8) 12, 24 and 48 tokens 242 and 249, 260 and 258, 303 and 277.  Down: 0.5 (4 of 4096 x 14336, top-2) 66 tokens 302 and 311; 0.6 to 0.75 (8 of
//   them) 24, 32, 48 and 66 tokens 324 and 344, 348 and 349, 418 and 362, 504 and 375.
// - And a tile has to have tokens: three pairs per expert if both contractions take rounds (16 of 4096 x 6400, top-2, Zipf(1.5), int4/int2, 2 pairs 141 and 140, 3 pairs 152 and 141; 32 of 4096 x
//   2304, top-4, 2 pairs 171 and 146), else four (256 of 7168 x 256 and a shared one, top-8, 2 pairs 212 and 231, 3 pairs 240 and 251, 4 pairs 265 and 241; 64 of 4096 x 1024, top-8, 2 pairs
//   135 and 136, 3 pairs 149 and 141, int4/int2 102 and 107, 115 and 109).
// - Up to 64 tokens, besides, a quantized expert (16 of 4096 x 6400, top-4, all bf16, 48 tokens 442 and 468, 64 tokens 472 and 472, 66 tokens 488 and 474).
// Over 889 calls (41 layers, 4 to 128 tokens) those that the rule puts on tiles are 1.03 to 2 times as fast there.
bool takes_tiles(const dx_fwd_args &a, int n_cu)
{
    const bool fit = a.d % 128 == 0 && a.f % 64 == 0 && (!a.shared || a.shared_f % 64 == 0) && ((uintptr_t)a.x & 15) == 0;
    if (!fit) return false;
    const long pairs = (long)a.T * a.k, cols = (a.f + 127) / 128, rows = dxk_thin_rows_max(a.T, a.k, a.E, false);
    auto in_rounds = [](int K) { return pick_split((K + 127) / 128, (K + 127) / 128).mode == kRounds; };
    if (a.T > DX_FP32_TOKENS) {
        const long tiles = rows * cols;
        const bool idle = 4 * tiles <= 3L * n_cu && (a.T <= 256 ? pairs <= 48L * a.E : a.T <= 400 && pairs <= 24L * a.E);
        const bool one_round = !in_rounds(a.d) && a.T <= 160 && 4 * tiles <= 9L * n_cu && pairs <= 12L * a.E;
        return a.shared || a.d < 2048 || !(idle || one_round);
    }
    if (a.T <= kFewTokens || !in_rounds(a.d) || pairs < (in_rounds(a.f) ? 3L : 4L) * a.E || (a.T <= DX_ROUTE_CHUNK && !a.any_quantized)) return false;
    const long rows_shared = a.shared ? (a.T + DX_THIN_ROWS - 1) / DX_THIN_ROWS : 0;
    const long gate_up = rows * cols + rows_shared * ((a.shared_f + 127) / 128), down = (rows + rows_shared) * (a.d / 256);
    return gate_up >= 2L * n_cu && 4 * down >= 3L * n_cu;
}

// r: null, or the routing inputs and outputs of a call that asks the gate/up kernel to route; *routed
// then tells whether it did (if not, nothing has been launched).
hipError_t launch_all(const dx_fwd_args &a_in, int n_cu, hipStream_t s, dx_marks *mk, const dx_route_io *r,
                      bool *routed)
{
    dx_fwd_args a = a_in;
    const bool tiled = takes_tiles(a, n_cu);
    const few_choice few = tiled ? few_choice{false, false} : takes_few(a, n_cu);
    if (!tiled && (!few.down || r)) a.tiles = nullptr;
    a.o_bf16 = a.T > DX_FP32_TOKENS && tiled; // d % 128 == 0 there, so rows split into 8-column pieces
    a.m_big = a.o_bf16 ? big_tile_formats(a, n_cu) : 0;
    if (r) {
        const int nc = a.d / chunk_of(a.group, a.d, a.d);
        *routed = !tiled && (few.gate_up || pick_split(nc, nc).mode == kWhole) && a.T >= 1 && a.T <= kRoutedTokens && a.E <= kRoutedExperts && a.k <= kRoutedTopK;
        if (!*routed) return hipSuccess;
    }
    hipEvent_t *marks = mk ? mk->ev : nullptr;
    if (mk) mk->per_kernel = !a.o_bf16, mk->combined = false;
    bool combined = false; // y is there already
    // profiled: every kernel's own start and stop stamps; with tiles of several kinds, whose phases may be two kernels, records around the phases
    hipEvent_t ev[8] = {};
    if (marks && !a.o_bf16)
        for (int i = 0; i < 8; ++i) ev[i] = marks[i];
    if (!tiled) {
        const dim3 grid(n_cu);
        if (few.gate_up) launch_few(a, n_cu, s, ev[0], ev[1], r);
        else launch_stream<false>(a, grid, s, ev[0], ev[1], r);
        if (few.down) {
            const dim3 strips(a.d / kFewCols, a.T), block(64 * few_down_waves(a, n_cu));
            if (r) launch(k_down_few<true>, strips, block, s, ev[5], ev[2], a);
            else launch(k_down_few<false>, strips, block, s, ev[5], ev[2], a);
            combined = true;
            if (mk) mk->combined = true;
        } else {
            launch_stream<true>(a, grid, s, ev[5], ev[2]);
        }
    } else {
        const bool records = marks && a.o_bf16;
        if (records) (void)hipEventRecord(marks[0], s);
        if (!a.listed) dxk_tile_list(dxk_list_args(a, n_cu), a.offsets, s);
        dxk_tiles_gate_up(a, s, ev[0], ev[1]);
        if (records) (void)hipEventRecord(marks[1], s);
        dxk_tiles_down(a, s, ev[5], ev[2]);
        if (records) (void)hipEventRecord(marks[2], s);
    }
    if (combined) {
    } else if (a.o_bf16) {
        launch(k_combine_bf16, dim3((a.d / 8 + 255) / 256, a.T), dim3(256), s, ev[6], ev[3], a);
    } else {
        launch(k_combine, dim3((a.d / 4 + 255) / 256, a.T), dim3(256), s, ev[6], ev[3], a);
    }
    if (marks) {
        if (a.o_bf16) (void)hipEventRecord(marks[3], s);
        (void)hipEventRecord(marks[7], s); // two records back to back: the cost of an event pair itself
        (void)hipEventRecord(marks[4], s);
    }
    return hipGetLastError();
}

} // namespace

#ifdef DX_TRACE
extern "C" int dx_debug_read_trace(void *dst, size_t bytes)
{
    return (int)hipMemcpyFromSymbol(dst, HIP_SYMBOL(g_trace), bytes, 0, hipMemcpyDeviceToHost);
}
extern "C" int dx_debug_read_mix(void *dst) // reads and clears
{
    int rc = (int)hipMemcpyFromSymbol(dst, HIP_SYMBOL(g_mix), sizeof(unsigned int) * 2 * 8192 * 8, 0, hipMemcpyDeviceToHost);
    void *p = nullptr;
    rc |= (int)hipGetSymbolAddress(&p, HIP_SYMBOL(g_mix));
    if (p) rc |= (int)hipMemset(p, 0, sizeof(unsigned int) * 2 * 8192 * 8);
    return rc;
}
extern "C" int dx_debug_read_steps(void *dst, void *counts)
{
    unsigned int zero[2][4] = {};
    int rc = (int)hipMemcpyFromSymbol(dst, HIP_SYMBOL(g_steps), sizeof(unsigned long long) * 2 * 4 * 256, 0, hipMemcpyDeviceToHost);
    rc |= (int)hipMemcpyFromSymbol(counts, HIP_SYMBOL(g_nsteps), sizeof zero, 0, hipMemcpyDeviceToHost);
    rc |= (int)hipMemcpyToSymbol(HIP_SYMBOL(g_nsteps), zero, sizeof zero, 0, hipMemcpyHostToDevice);
    return rc;
}
#endif

dx_list_args dxk_list_args(const dx_fwd_args &a, int n_cu)
{
    if (!takes_tiles(a, n_cu)) return dx_list_args{};
    const bool thin_only = a.T <= DX_FP32_TOKENS;
    return dx_list_args{a.table, a.tiles, a.T, a.E, a.k, thin_only ? 0 : big_tile_formats(a, n_cu), n_cu, a.shared != nullptr, thin_only};
}

hipError_t dxk_moe_forward(const dx_fwd_args &a, int n_cu, hipStream_t s, dx_marks *marks)
{
    if (a.T == 0) return hipSuccess;
    return launch_all(a, n_cu, s, marks, nullptr, nullptr);
}

hipError_t dxk_route_forward(const dx_fwd_args &a, const dx_route_io &r, int n_cu, hipStream_t s, dx_marks *marks,
                             bool *routed)
{
    *routed = false;
    if (a.T == 0) return hipSuccess;
    return launch_all(a, n_cu, s, marks, &r, routed);
}
