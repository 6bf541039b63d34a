// Mixed-precision expert execution for large per-expert token counts
// (prefill): LDS-tiled bf16 MFMA grouped GEMMs.
//
// Paper: Sec. 3.2 (the compute path resolves the handle and runs the kernel of
// the active version).  The paper gives no kernel; this one is built for gfx950.
//
// Regime: calls of more than 128 tokens, and fewer on layers with a long K (takes_tiles in dx_moe_decode.hip).  Output tiles with
// v_mfma_f32_32x32x16_bf16, fp32 accumulators and K in steps of 64 (one 128-byte line of a token or weight row).
//   k_tiled: tiles of 128 rows x 128 or 256 columns, any number of rows, all formats, and thin ones for segments of up to 32 rows;
//   k_big:   256 x 256 for the whole 256 rows of large bf16 and int4 segments;
//   k_thin:  thin tiles alone, for calls of up to 128 tokens.
// Quantized weights are expanded on their way to the matrix instructions: code -> fp32 -> times the group's scale -> bf16; in thin tiles the
// codes are multiplied as integers and the scale goes on the fp32 sums.
//   gate/up: half of the tile's columns are gate rows and the other half the up rows of the same
//            indices, and every wavefront owns matching gate/up columns, so SwiGLU happens on the
//            accumulators; H is written once as bf16.
//   down:    plain tiles of O = H . W_down^T, written as rows in pair order for the combine kernel, bf16 (k_thin: fp32).
// Tiles are listed expert-major, in bands of row tiles, inside a band column tile next, row tile innermost, and
// the list is cut into 8 contiguous ranges, one per XCD (block b works in range b % 8), so the tiles that
// share token and weight lines run at the same time on the same L2.
#include "dx_internal.h"
#include "dx_tile_list.h"

#include <hip/hip_ext.h>

#include <type_traits>

namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;

#define DX_GLOBAL __attribute__((address_space(1)))

union frag8 {
    u32x4 u;
    bf16x8 v;
};

constexpr int BN = 128, BNW = 256, BK = 64; // columns of a narrow and of a wide tile, k-values of a step

// silu(g) * u with the hardware exp2 and reciprocal (their error is far below the bf16 rounding of H)
__device__ __forceinline__ float swiglu_fast(float g, float u)
{
    return g * __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(-1.4426950408889634f * g)) * u;
}

// The same as the streaming kernels take it, within 3e-7 of its value: the thin tiles' (segments that those kernels have elsewhere).  swiglu_fast is off by up to
// 3e-6 for large gates, the rounding of the exponent's product, and flushes silu(g) below g = -87.3.
__device__ __forceinline__ float swiglu(float g, float u) { return g / (1.f + expf(-g)) * u; }

typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;

// two fp32 -> two bf16 in one word (the hardware's packed conversion: round to nearest even, the same
// bits as the decode kernels' integer rounding for finite values)
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi)
{
    const f32x2 v{lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

// 8 nibbles of `word` times 16 * scale16 -> 8 bf16 in element order (16ths of a bf16 scale are exact: it has eight significant bits): the
// nibbles as the upper halves of signed bytes, which the conversion takes out of their word by itself.
__device__ __forceinline__ u32x4 dequant8(uint32_t word, float scale16)
{
    const uint32_t even = (word << 4) & 0xF0F0F0F0u, odd = word & 0xF0F0F0F0u;
    uint32_t p[4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
        p[i] = pack_bf16((float)(int8_t)(even >> (8 * i)) * scale16, (float)(int8_t)(odd >> (8 * i)) * scale16);
    return u32x4{p[0], p[1], p[2], p[3]};
}

// The four products of a two-bit code (0, 1, -2, -1) and a bf16 scale, which are bf16 values: their lower and their upper bytes.
struct crumb_products {
    uint32_t lo, hi;
    __device__ __forceinline__ explicit crumb_products(float scale)
    {
        const uint32_t zero = __float_as_uint(0.f * scale), one = __float_as_uint(scale), minus_two = __float_as_uint(-2.f * scale);
        // bytes (zero, one, minus two, one) of what is in the upper halves; then minus one is one with the other sign
        const uint32_t los = __builtin_amdgcn_perm(minus_two, one, 0x02060200u), his = __builtin_amdgcn_perm(minus_two, one, 0x03070300u);
        lo = __builtin_amdgcn_perm(zero, los, 0x03020106u);
        hi = __builtin_amdgcn_perm(zero, his, 0x03020107u) ^ 0x80000000u;
    }
};

// 8 two-bit codes (`half`: 16 bits) times the scale -> 8 bf16 in element order.  A byte selection looks a pair up: its selector is code a, code a + 4, code b,
// code b + 4.  (15 vector instructions; by conversions and products 28.  16 experts of 4096 x 6400, int4/int2, a layer, us: 300 tokens 297 and 282, 1100
// tokens 557 and 542; 30B-shaped, 500 tokens 146 and 141.)
__device__ __forceinline__ u32x4 dequant8_crumbs(uint32_t half, const crumb_products &of)
{
    const uint32_t w = half | (half << 14), v = w >> 4; // codes 2j and 2j + 1 sixteen bits apart: 0 and 4 (in v: 2 and 6) first
    auto two = [&](uint32_t from, uint32_t bytes) {
        const uint32_t sel = (__builtin_amdgcn_perm(from, from, bytes) & 0x03030303u) | 0x04000400u;
        return __builtin_amdgcn_perm(of.hi, of.lo, sel);
    };
    return u32x4{two(w, 0x02020000u), two(v, 0x02020000u), two(w, 0x03030101u), two(v, 0x03030101u)};
}

// Reads of what the kernel never writes at a wave-uniform index, as scalar loads.
template <typename T>
__device__ __forceinline__ T uniform_load(const T *p)
{
    return *reinterpret_cast<const __attribute__((address_space(4))) T *>((uintptr_t)p);
}

struct tile_id {
    int e, mt, nt; // expert (E = shared), row tile, column tile
    int seg0, m;   // first pair slot and number of rows of the segment, or of the part of it that the tile size takes
    bool valid;
};

// column tiles of a projection with fe rows in W_gate (down: d); the last one may be half a tile
template <bool DOWN>
__host__ __device__ __forceinline__ int columns_of(const dx_fwd_args &a, int fe, int width)
{
    return DOWN ? (a.d + width - 1) / width : (2 * fe + width - 1) / width;
}

// Tile number `idx` of the row tiles that are listed from `row` on, `ntn` column tiles each.  The tiles of an expert go in bands of
// BAND row tiles, inside a band column tile next, row tile innermost: with 8 of them and as many columns next to each other
// the tiles that run together on an XCD ask for every line about eight times.  (Bands that run on over the experts' borders:
// 16 experts of 4096 x 6400, 1100 tokens 701 us against 688 -- eight experts' tokens do not stay in an XCD's L2 from
// one column to the next.)
template <int ROWS, int BAND>
__device__ __forceinline__ tile_id tile_of(const dx_tile_row *rows, uint32_t idx, int ntn)
{
    tile_id t;
    const int q = (int)(idx / (uint32_t)ntn); // some row tile of the band that the tile is in
    const dx_tile_row *row = rows + q;
    t.e = uniform_load(&row->e), t.m = uniform_load(&row->m), t.seg0 = uniform_load(&row->seg0);
    const int mt = uniform_load(&row->mt), mt0 = mt / BAND * BAND, nmt = (t.m + ROWS - 1) / ROWS;
    const int band = nmt - mt0 < BAND ? nmt - mt0 : BAND, in_band = (int)idx - (q - (mt - mt0)) * ntn;
    t.nt = in_band / band;
    t.mt = mt0 + in_band % band;
    t.valid = true;
    return t;
}

// This block's tile.  The row tiles of all experts are in a.tiles (written in front, by the routing's placement kernel or by k_tile_list,
// because a prologue that derives the list from the offsets in every block is 3 of a tile's 20 to 35 us): the routed
// experts', the shared one's, the 256-row tiles behind them, the thin tiles.  Each XCD takes an eighth of the former.
// Figures: us a layer.
// Thin tiles are in the launch of the others.  (Streaming kernels for the segments of up to 32 rows, a launch in front in each phase, and this: 30B-shaped 129
// tokens 111 and 98, 300 tokens 137 and 116, 1000 tokens 196 and 184, 4096 tokens 456 and 425, int4/int2 150 tokens 101 and 82; 80B-shaped 150 tokens 115 and 86, 1000
// tokens 200 and 170; 16 experts of 4096 x 6400 150 tokens 397 and 309, 1100 tokens 587 and 532.  But if no segment has more than 32 rows: 30B-shaped, balanced
// routing, 129 tokens 120 and 130, 200 tokens 122 and 130, no bf16 expert 97 and 106; 80B-shaped 129 tokens 225 and 235, 600 tokens 248 and 253: 1.5 rounds of thin tiles in gate/up.)
// Thin tiles go last, because they are short and fill the last round.  They go first where bf16 weights from memory are all there is, up to four narrow tiles per compute
// unit, and with few other tiles (up to one) only if a good part of the thin ones is bf16 as well.
//   First and last: 30B-shaped 130 tokens 96 and 99, 300 tokens 116 and 124, 500 tokens 139 and 146, int4/int2 150 tokens 86 and 81; 80B-shaped 150 tokens 88 and 84, 1000
//   tokens 175 and 162; 16 of 4096 x 6400 150 tokens 329 and 297, int4/int2 266 and 244, 1100 tokens 534 and 522.  Over 55 calls of 19 layers the rule takes 0.93 to 1.09 times as
//   long as last throughout, 0.91 to 1.02 times as long as first; what it gets wrong is a K of 7168 (64 experts of 7168 x 512, top-2, 200 tokens 190 and 176).
// Wide or narrow: a compute unit holds two tiles of either kind.  Figures: the phase's kernels alone, narrow and wide, by narrow tiles
// per compute unit; the same lines hold for both phases.
//   Quantized weights gain by the expansion as soon as there is more than one round: all int4, 128 experts of 2048 x 768, 110 rows each, gate/up
//   2.6 76 and 75, 4.3 123 and 122, 6.0 153 and 134, down 3.4 48 and 40, 8.0 96 and 78; 8 of 4096 x 4096, down 2.0 96 and 102, 3.0 141 and 141.
//   bf16 weights gain by the loads, and a round of wide tiles takes as long as 1.7 to 1.9 of narrow ones: one for two of them (3 to 4) 8 of
//   4096 x 4096, gate/up 4.0 188 and 157, down 2.0 90 and 104, 3.0 126 and 137; two for three (4 to 6) 64 of 2048 x 1536, gate/up 6.0 191 and 224,
//   30B-shaped 4.5 128 and 145, down 4.5 71 and 77; two for four and more (from 6) 30B-shaped 6.8 167 and 162, 10.5 233 and 219, 12.9 273 and 253,
//   down 7.6 100 and 91.
//   Mixed: as quantized ones from 45 % of the row tiles on (half: 4.0 109 and 96, 6.0 162 and 161), and from 20 % on where most experts have several
//   row tiles, which ask for the same weights (80B-shaped, a third, 3.2 123 and 106, 5.2 168 and 149, down 6.4 81 and 70); with one row tile to an expert bf16
//   weights come from memory alone, and narrow tiles take in more (a third, 4.3 132 and 157, 6.0 174 and 185).
enum tile_kind { kNarrow, kWide, kThin };
template <bool DOWN>
__device__ __forceinline__ tile_id find_tile(const dx_fwd_args &a, tile_kind &kind)
{
    const int n = uniform_load(&a.tiles->n_routed), n_shared = uniform_load(&a.tiles->n_shared), n_cu = uniform_load(&a.tiles->n_cu);
    const int narrow_tiles = n * columns_of<DOWN>(a, a.f, BN) + n_shared * columns_of<DOWN>(a, a.shared_f, BN);
    const int quant = uniform_load(&a.tiles->n_quant), single = uniform_load(&a.tiles->n_single);
    const int thin_bf16 = uniform_load(&a.tiles->n_thin), n_thin = thin_bf16 + uniform_load(&a.tiles->n_thin_quant), ntn_thin = columns_of<DOWN>(a, a.f, BNW);
    const bool as_quantized = 20 * quant >= 9 * (n + n_shared) || (5 * quant >= n + n_shared && 5 * single <= 2 * n);
    const bool wide = as_quantized ? 2 * narrow_tiles > 5 * n_cu : narrow_tiles > 6 * n_cu || (narrow_tiles > 3 * n_cu && narrow_tiles <= 4 * n_cu);
    const int width = wide ? BNW : BN, ntn = columns_of<DOWN>(a, a.f, width), ntn_shared = columns_of<DOWN>(a, a.shared_f, width);
    const uint32_t routed = (uint32_t)(n * ntn), total = routed + (uint32_t)(n_shared * ntn_shared), per_xcd = (total + 7) / 8;
    const uint32_t thin = (uint32_t)(n_thin * ntn_thin), thin_per_xcd = (thin + 15) / 16 * 2;
    const dx_tile_row *rows = reinterpret_cast<const dx_tile_row *>(a.tiles + 1);
    const uint32_t xcd = blockIdx.x & 7;
    uint32_t at = blockIdx.x >> 3;
    tile_id t;
    t.valid = false;
    const bool thin_first = !as_quantized && narrow_tiles <= 4 * n_cu && (narrow_tiles > n_cu || 2 * thin_bf16 > n + n_shared);
    const bool is_thin = thin_first ? at < thin_per_xcd : at >= per_xcd;
    if (thin_first != is_thin) at -= thin_first ? thin_per_xcd : per_xcd; // behind the other kind
    if (is_thin) {
        kind = kThin;
        // (two at a time to an XCD, so that every one has its share of the bf16 ones, which are listed first: a list in eight parts of
        // unlike weight 30B-shaped, 130 tokens 104 us a layer against 101)
        const uint32_t idx = ((at >> 1) * 8 + xcd) * 2 + (at & 1);
        if (idx >= thin) return t;
        const dx_tile_row *of = rows + n + n_shared + uniform_load(&a.tiles->n_big) + uniform_load(&a.tiles->n_big_shared) + idx / (uint32_t)ntn_thin;
        t.e = uniform_load(&of->e), t.m = uniform_load(&of->m), t.seg0 = uniform_load(&of->seg0);
        t.mt = 0, t.nt = (int)(idx % (uint32_t)ntn_thin);
        t.valid = true;
        return t;
    }
    kind = wide ? kWide : kNarrow;
    const uint32_t idx = xcd * per_xcd + at;
    if (at < per_xcd && idx < total) t = idx < routed ? tile_of<DX_TILE_ROWS, 8>(rows, idx, ntn) : tile_of<DX_TILE_ROWS, 8>(rows + n, idx - routed, ntn_shared);
    return t;
}

// ---- loads from memory to LDS ---------------------------------------------------------------------
// Inline assembly, so that the compiler does not serialise them against the LDS reads; their completion is
// awaited with explicit vmcnt counts.
typedef __attribute__((address_space(3))) char lds_char;

// a wave-uniform pointer as a scalar pair (the halves go through unsigned 32-bit values: the builtin
// returns int, which must not be sign-extended into the upper half)
__device__ __forceinline__ uint64_t scalar_ptr(const void *p)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(uintptr_t)p);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)((uintptr_t)p >> 32));
    return (uint64_t)lo | ((uint64_t)hi << 32);
}
// one wavefront-wide 16-byte-per-lane load: memory (sbase + voff) -> LDS (m0 + 16 * lane)
__device__ __forceinline__ void load_to_lds(uint32_t m0, uint32_t voff, uint64_t sbase)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(m0), "v"(voff), "s"(sbase)
                 : "memory");
}
// the same from a 64-bit address per lane
__device__ __forceinline__ void load_to_lds(uint32_t m0, uint64_t addr)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(m0), "v"(addr) : "memory");
}
// with 4 bytes per lane: memory -> LDS (m0 + 4 * lane)
__device__ __forceinline__ void load_to_lds4(uint32_t m0, uint32_t voff, uint64_t sbase)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2" ::"s"(m0), "v"(voff), "s"(sbase)
                 : "memory");
}

__device__ __forceinline__ void load_to_lds4(uint32_t m0, uint64_t addr)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, off" ::"s"(m0), "v"(addr) : "memory");
}

// the bare barrier, over which the compiler moves no LDS access
__device__ __forceinline__ void block_barrier()
{
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// A token row's 32 columns (gate/up, after SwiGLU) or 64 (down) of a wavefront, from the accumulators of two MFMA tiles
// (columns 0..31 and 32..63, or gate and up) to memory at dst + 8 * (lane / 32).  The weights were the first MFMA operand:
// accumulator element v of a 32 x 32 tile is output column (v/4)*8 + (lane/32)*4 + v%4 of token lane%32.  One swap of the
// wavefront's halves per pair of words gives every lane eight consecutive columns, 16 bytes.  Both halves of the wavefront
// must store the same rows.
template <bool DOWN>
__device__ __forceinline__ void store_row(const f32x16 &a0, const f32x16 &a1, dx_bf16 *dst)
{
#pragma unroll
    for (int ns = 0; ns < (DOWN ? 2 : 1); ++ns)
#pragma unroll
        for (int qp = 0; qp < 2; ++qp) {
            const f32x16 &acc = ns ? a1 : a0;
            uint32_t w[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) { // words (q = 2qp: columns 0, 2), (q = 2qp + 1: columns 0, 2)
                const int v = 4 * (2 * qp + (u >> 1)) + 2 * (u & 1);
                if constexpr (DOWN) w[u] = pack_bf16(acc[v], acc[v + 1]);
                else w[u] = pack_bf16(swiglu_fast(a0[v], a1[v]), swiglu_fast(a0[v + 1], a1[v + 1]));
            }
            const auto lo = __builtin_amdgcn_permlane32_swap(w[0], w[2], false, false);
            const auto hi = __builtin_amdgcn_permlane32_swap(w[1], w[3], false, false);
            *reinterpret_cast<u32x4 *>(dst + ns * 32 + qp * 16) = u32x4{lo[0], hi[0], lo[1], hi[1]};
        }
}

constexpr int kLine = BK * 2; // 128: bytes of a row per K-step, one line

// ---------------------------------------------------------------------------------------------
// Output tiles of 128 rows x 128 columns, any number of rows, all formats: 4 wavefronts, each a 64 x 64 sub-tile = 2 x 2
// MFMA tiles; two blocks to a compute unit, which multiply in each other's waits.
// What bounds it: the fill.  Most of its lines hit in L2, but the tiles that share a line ask for it at the same
// time, so a step waits as long as a miss takes (1.5 to 2 us in a full launch), and what a compute unit gets is
// the bytes it has in flight over that time.  So the loads must never stop: a wavefront reads all operands of a step (K = 64)
// into registers while it multiplies the step before, which frees the step's LDS stage at once, and STAGES stages
// are in flight nearly all the time.
//   LDS rows are one line (128 bytes), unpadded; piece c of row r sits in slot c ^ ((r >> 1) & 7), which makes
//   the 128-bit operand reads conflict-free.  A load instruction fills 8 rows, neighbouring lanes on a line.
//   bf16 weights arrive like the tokens.  Codes (FMT 1, 2) and scales arrive in a side ring of two slots, one step
//   before the wavefront that loaded them expands its own rows into the weight half of the stage.  A row's
//   scale is the half of an aligned word that (row * groups + group) is in; with groups of 32 a step spans the
//   two groups of an aligned word (K / 32 is even), and the lane takes the half its elements are in.
// Rows past the end of a segment repeat its last row (one line for all of them) and are not stored.
// Measured, 30B-shaped layer, both phases' tiles of 4096 tokens (299 GFLOP, 332 with the padding of the row tiles): 385 us
// (0.86 PFLOP/s; registers -> LDS staging of the same tiles with bf16 segments of 256 rows in a kernel of 256 x 256
// tiles: 470); of 1000 tokens: 115 us against 160.  256-row tiles with three stages and one block of 8 wavefronts
// were slower (4096 tokens 572 us a pass against 506): the block's barriers have nothing beside them.  At this load the
// clock is 1.9 GHz (2.4 idle), i.e. the matrix cores could do 2.0 PFLOP/s.
struct cfg {
    static constexpr int ROWS = DX_TILE_ROWS, WAVES = 4, THREADS = 64 * WAVES;
    static constexpr int STAGES = 2;
    static constexpr int STAGE = (ROWS + BN) * kLine;         // 32 KB: token rows then weight rows
    static constexpr int WROWS = BN / WAVES;                  // weight rows a wavefront loads
    static constexpr int SIDE_WAVE = WROWS * (32 + 4);        // up to 32 bytes of codes and one word of scales per row
    static constexpr int SIDE = WAVES * SIDE_WAVE;
    static constexpr int RING = STAGES * STAGE + 2 * SIDE;
    // wide tiles: two slots of token rows; for every wavefront its 64 weight rows of a step, or (quantized) two slots of the codes of
    // two steps of them (int2: half of it) and of two words of scales per row
    static constexpr int A_SLOT = ROWS * kLine, B_WAVE = 64 * kLine, SIDE_WIDE = 64 * 64 + 2 * 256;
    static_assert(2 * A_SLOT + WAVES * B_WAVE <= RING && 2 * A_SLOT + WAVES * 2 * SIDE_WIDE <= RING, "the ring");
    // thin tiles, quantized: three slots of the token rows and codes of two steps
    static constexpr int THIN_SLOTS = 3, THIN_A = DX_THIN_ROWS * kLine, THIN = THIN_SLOTS * (2 * THIN_A + WAVES * SIDE_WIDE);
    static constexpr int LDS = THIN > RING ? THIN : RING;
    static_assert(2 * (LDS + 256 * WAVES) <= 160 * 1024, "two blocks to a compute unit");
};

template <bool DOWN, int FMT>
__device__ __forceinline__ void narrow_tile(const dx_fwd_args &a, const tile_id &t, const dx_handle *h, char *ring)
{
    constexpr bool quant = FMT != 0;
    constexpr int ROWS = cfg::ROWS, STAGES = cfg::STAGES, STAGE = cfg::STAGE, WROWS = cfg::WROWS;
    // loads per wavefront and step: tokens; weights, or codes and scales
    constexpr int NA = 4, NC = FMT == 0 ? WROWS / 8 : (FMT == 1 ? 2 : WROWS / 16 + 1);
    const bool shared = t.e == a.E;
    const int fe = shared ? a.shared_f : a.f;
    const int K = DOWN ? fe : a.d;
    const int nk = K / BK;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1;

    // ---- loader role: wavefront w fills token rows [32w, 32w + 32) and weight rows [WROWS * w, + WROWS) ----
    // weight-tile row -> matrix row: down: BN consecutive rows; gate/up: 64 gate rows, then the same up rows
    auto wrow = [&](int row) { return DOWN ? t.nt * BN + row : t.nt * (BN / 2) + (row & 63); };
    uint64_t a_at[NA]; // advances by a line with every step that is issued
    uint32_t b_off[4];
    const uint32_t row_bytes = FMT == 0 ? (uint32_t)K * 2 : (FMT == 1 ? (uint32_t)K / 2 : (uint32_t)K / 4);
#pragma unroll
    for (int i = 0; i < NA; ++i) {
        const int row = 32 * wave + 8 * i + (lane >> 3);
        const uint32_t piece = (uint32_t)((lane & 7) ^ ((row >> 1) & 7));
        int slot = t.mt * ROWS + row;
        slot = slot < t.m ? slot : t.m - 1;
        if constexpr (DOWN) {
            a_at[i] = (uint64_t)a.h + (uint64_t)(t.seg0 + slot) * a.fmax * 2 + piece * 16;
        } else {
            const int tok = shared ? t.seg0 - a.T * a.k + slot : a.perm[t.seg0 + slot] / a.k;
            a_at[i] = (uint64_t)a.x + (uint64_t)tok * K * 2 + piece * 16;
        }
    }
    // bf16: the lane's piece of the row; int4: 16 of the row's 32 bytes per step, two lanes to a row; int2: 4 of its 16 bytes,
    // four lanes to a row
    const int w0 = WROWS * wave;
#pragma unroll
    for (int i = 0; i < (FMT == 0 ? WROWS / 8 : (FMT == 1 ? 1 : WROWS / 16)); ++i) {
        if constexpr (FMT == 0) {
            const int row = w0 + 8 * i + (lane >> 3);
            b_off[i] = (uint32_t)wrow(row) * row_bytes + ((lane & 7) ^ ((row >> 1) & 7)) * 16;
        } else if constexpr (FMT == 1) {
            b_off[i] = (uint32_t)wrow(w0 + (lane >> 1)) * row_bytes + (lane & 1) * 16;
        } else {
            b_off[i] = (uint32_t)wrow(w0 + 16 * i + (lane >> 2)) * row_bytes + (lane & 3) * 4;
        }
    }
    const bool up_rows = w0 >= 64; // gate/up: the wavefront's weight rows belong to W_up
    const uint64_t b_base = scalar_ptr(uniform_load(DOWN ? &h->w_down : (up_rows ? &h->w_up : &h->w_gate)));
    const uint64_t s_base = quant ? scalar_ptr(uniform_load(DOWN ? &h->s_down : (up_rows ? &h->s_up : &h->s_gate))) : 0;
    const int lg = __builtin_ctz((unsigned)a.group);
    const uint32_t s_row = quant ? (uint32_t)wrow(w0 + (lane & (WROWS - 1))) * (uint32_t)(K >> lg) : 0; // first scale of the lane's row
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_char *)ring;
    const uint32_t m0_a = lds0 + wave * 32 * kLine, m0_b = lds0 + ROWS * kLine + w0 * kLine;
    const int side_wave = STAGES * STAGE + wave * cfg::SIDE_WAVE; // + slot * SIDE
    auto clamped = [&](int kt) { return kt < nk ? kt : nk - 1; }; // steps past the end: duplicates that are not multiplied
    auto issue_token = [&](int kt, int stage, int i) { // called for kt = 0, 1, 2, ...
        load_to_lds(m0_a + (uint32_t)(stage * STAGE) + 1024 * i, a_at[i]);
        a_at[i] += kt + 1 < nk ? kLine : 0;
    };
    auto issue_tokens = [&](int kt, int stage) {
#pragma unroll
        for (int i = 0; i < NA; ++i) issue_token(kt, stage, i);
    };
    auto issue_weight = [&](int kt, int stage, int i) { // bf16
        load_to_lds(m0_b + (uint32_t)(stage * STAGE) + 1024 * i, b_off[i], b_base + (uint64_t)clamped(kt) * kLine);
    };
    auto issue_weights = [&](int kt, int stage) {
#pragma unroll
        for (int i = 0; i < WROWS / 8; ++i) issue_weight(kt, stage, i);
    };
    auto issue_codes = [&](int kt, int slot) {
        const int kc = clamped(kt);
        const uint32_t m0 = lds0 + (uint32_t)(side_wave + slot * cfg::SIDE);
        if constexpr (FMT == 1) {
            load_to_lds(m0, b_off[0], b_base + (uint64_t)kc * (BK / 2));
        } else {
#pragma unroll
            for (int i = 0; i < WROWS / 16; ++i) load_to_lds4(m0 + 256 * i, b_off[i], b_base + (uint64_t)kc * (BK / 4));
        }
        if (lane < WROWS) load_to_lds4(m0 + 32 * WROWS, ((s_row + (uint32_t)((kc * BK) >> lg)) * 2) & ~3u, s_base);
    };
    // the wavefront's rows of step kt, from side slot `slot` into the weight half of `stage`: LPR lanes to a row, 64 / LPR
    // elements (16-byte pieces of the stage) each.  (The parity of a row's place in its matrix is that of its place
    // in the tile.)
    auto expand = [&](int kt, int slot, int stage) {
        constexpr int LPR = 64 / WROWS, PIECES = 8 / LPR;
        const char *side = ring + side_wave + slot * cfg::SIDE;
        const int row = w0 + lane / LPR, part = lane % LPR;
        const uint32_t word = *reinterpret_cast<const uint32_t *>(side + 32 * WROWS + 4 * (lane / LPR));
        const bool odd = a.group == 32 ? 2 * part >= LPR : ((row & (K >> lg)) ^ ((clamped(kt) * BK) >> lg)) & 1;
        const float scale = __uint_as_float(odd ? word & 0xFFFF0000u : word << 16);
        char *dst = ring + stage * STAGE + (ROWS + row) * kLine;
        const int swz = (row >> 1) & 7;
        auto put = [&](int i, u32x4 v) { *reinterpret_cast<u32x4 *>(dst + (((PIECES * part + i) ^ swz) * 16)) = v; };
        if constexpr (FMT == 1) { // a word of codes per piece
            uint32_t c[PIECES];
            __builtin_memcpy(c, __builtin_assume_aligned(side + 4 * PIECES * lane, 4 * PIECES), 4 * PIECES);
#pragma unroll
            for (int i = 0; i < PIECES; ++i) put(i, dequant8(c[i], scale * 0.0625f));
        } else { // half a word per piece
            const crumb_products products(scale);
            uint32_t c[PIECES / 2];
            __builtin_memcpy(c, __builtin_assume_aligned(side + 2 * PIECES * lane, 2 * PIECES), 2 * PIECES);
#pragma unroll
            for (int i = 0; i < PIECES; ++i) put(i, dequant8_crumbs(i & 1 ? c[i / 2] >> 16 : c[i / 2] & 0xFFFFu, products));
        }
    };

    // ---- MFMA role ----
    const int r = lane & 31, kq = lane >> 5;
    const int r_lane = r * kLine + ((kq ^ ((r >> 1) & 7)) * 16); // piece kq of row r; piece 2 * kk + kq: ^ (32 * kk)
    // down: the pair indices of the wavefront's 64 token rows, where the rows of the tile go (the oldest of its loads)
    if constexpr (DOWN) {
        if (!shared) {
            const int slot = t.mt * ROWS + wm * 64 + lane;
            load_to_lds4(lds0 + cfg::LDS + 256 * wave, (uint32_t)(slot < t.m ? slot : t.m - 1) * 4u, scalar_ptr(a.perm + t.seg0));
        }
    }
    f32x16 acc[2][2];
#pragma unroll
    for (int ms = 0; ms < 2; ++ms)
#pragma unroll
        for (int ns = 0; ns < 2; ++ns)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[ms][ns][v] = 0.f;
    frag8 fa[2][2][4], fb[2][2][4]; // [register set][tile][quarter of the step]
    // two of a step's 16 operands (n = 0 .. 7): quarter n / 2, tokens (n odd) or weights
    auto read_pair = [&](int a_wave, int b_wave, frag8 (&af)[2][4], frag8 (&bf)[2][4], int n) {
        const int kk = n >> 1;
        if (n & 1) {
            const char *p = ring + a_wave + (r_lane ^ (32 * kk));
            af[0][kk].u = *reinterpret_cast<const u32x4 *>(p);
            af[1][kk].u = *reinterpret_cast<const u32x4 *>(p + 32 * kLine);
        } else {
            const char *p = ring + b_wave + (r_lane ^ (32 * kk));
            bf[0][kk].u = *reinterpret_cast<const u32x4 *>(p);
            bf[1][kk].u = *reinterpret_cast<const u32x4 *>(p + (DOWN ? 32 : 64) * kLine);
        }
    };
    auto a_rows = [&](int stage) { return stage * STAGE + wm * 64 * kLine; };
    auto b_rows = [&](int stage) { return stage * STAGE + (ROWS + (DOWN ? wn * 64 : wn * 32)) * kLine; };
    auto mma = [&](const frag8 (&af)[2][4], const frag8 (&bf)[2][4], int n) { // the n-th of a step's 16
        const int kk = n >> 2, ms = (n >> 1) & 1, ns = n & 1;
        acc[ms][ns] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bf[ns][kk].v, af[ms][kk].v, acc[ms][ns], 0, 0, 0);
    };
    // Start: steps 0 .. STAGES - 1, and step STAGES as soon as step 0 has been read.  Order of the loads of a wavefront
    // from there on: bf16: step by step.  Quantized: codes j + 1 and tokens j together, after codes j have been
    // expanded into the stage.
    if constexpr (quant) {
        issue_codes(0, 0), issue_codes(1, 1);
#pragma unroll
        for (int j = 0; j < STAGES; ++j) issue_tokens(j, j);
        asm volatile("s_waitcnt vmcnt(8)" ::: "memory"); // own codes 0, 1
        expand(0, 0, 0);
        expand(1, 1, 1);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); // side slots read
        issue_codes(2, 0);
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory"); // own tokens and codes; expansions written
    } else {
#pragma unroll
        for (int j = 0; j < STAGES; ++j) issue_tokens(j, j), issue_weights(j, j);
        asm volatile("s_waitcnt vmcnt(8)" ::: "memory"); // own loads of step 0
    }
    block_barrier();
#pragma unroll
    for (int n = 0; n < 8; ++n) read_pair(a_rows(0), b_rows(0), fa[0], fb[0], n);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    block_barrier(); // stage 0 has been read by every wavefront
    if constexpr (quant) {
        expand(STAGES, STAGES & 1, 0);
        issue_codes(STAGES + 1, (STAGES + 1) & 1);
        issue_tokens(STAGES, 0);
    } else {
        issue_tokens(STAGES, 0), issue_weights(STAGES, 0);
    }
    int stage = 1; // of step kt + 1
    auto step = [&](int kt, auto parity) __attribute__((always_inline)) {
        constexpr int P = decltype(parity)::value;
        // own loads of step kt + 1 have landed (quantized: and its expansions are written); those of the STAGES - 1 steps
        // after it and the codes of the one after them may be on their way.  After the barrier that holds for every wavefront.
        constexpr int pending = (STAGES - 1) * (NA + NC);
        if constexpr (quant) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(pending) : "memory");
        else asm volatile("s_waitcnt vmcnt(%0)" ::"n"(pending) : "memory");
        block_barrier();
        // A wavefront issues in order, and its reads wait for the compute unit's LDS: reads and matrix instructions take
        // turns (16 reads in a row: 506 us a pass of 4096 tokens against 499), and so do the loads of the refill.
        int a_at_lds = a_rows(stage), b_at_lds = b_rows(stage);
        asm volatile("" : "+s"(a_at_lds), "+s"(b_at_lds)); // (opaque: the addresses are added up here, not kept in a dozen registers)
#pragma unroll
        for (int n = 0; n < 8; ++n) {
            read_pair(a_at_lds, b_at_lds, fa[P ^ 1], fb[P ^ 1], n);
            mma(fa[P], fb[P], n);
            __builtin_amdgcn_sched_barrier(0);
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        block_barrier(); // every wavefront has read the stage: refill it with step kt + 1 + STAGES
        if constexpr (quant) {
            constexpr int SL = (P + 1 + STAGES) & 1; // side slot of step kt + 1 + STAGES (kt has the parity P)
            asm volatile("s_waitcnt vmcnt(4)" ::: "memory"); // own codes of that step
            expand(kt + 1 + STAGES, SL, stage);
            issue_codes(kt + 2 + STAGES, SL ^ 1);
            issue_tokens(kt + 1 + STAGES, stage);
#pragma unroll
            for (int n = 8; n < 16; ++n) mma(fa[P], fb[P], n);
            __builtin_amdgcn_sched_barrier(0);
        } else {
#pragma unroll
            for (int n = 0; n < 8; ++n) {
                if (n < 4) issue_token(kt + 1 + STAGES, stage, n);
                else issue_weight(kt + 1 + STAGES, stage, n - 4);
                mma(fa[P], fb[P], 8 + n);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        stage = stage + 1 < STAGES ? stage + 1 : 0;
    };
    static_assert(NA == 4 && WROWS == 32 && STAGES == 2, "the waits");
    int kt = 0;
    for (; kt + 1 < nk; kt += 2) {
        step(kt, std::integral_constant<int, 0>{});
        step(kt + 1, std::integral_constant<int, 1>{});
    }
    if (kt < nk) step(kt, std::integral_constant<int, 0>{});
    // The tile leaves straight from the registers.  The weights were the first MFMA operand: accumulator element v of a
    // 32 x 32 tile is output column (v/4)*8 + (lane/32)*4 + v%4 of token lane%32.  One swap of the wavefront's halves
    // per pair of words gives every lane eight consecutive columns, 16 bytes.
#pragma unroll
    for (int ms = 0; ms < 2; ++ms) {
        const int slot = t.mt * ROWS + wm * 64 + ms * 32 + r;
        dx_bf16 *dst;
        if constexpr (DOWN) {
            const int orow = shared ? t.seg0 + slot : *reinterpret_cast<const int *>(ring + cfg::LDS + 256 * wave + 4 * (ms * 32 + r));
            dst = reinterpret_cast<dx_bf16 *>(a.o) + (size_t)orow * a.d + t.nt * BN + wn * 64 + 8 * kq;
        } else {
            dst = a.h + (size_t)(t.seg0 + slot) * a.fmax + t.nt * (BN / 2) + wn * 32 + 8 * kq;
        }
        if (slot < t.m) store_row<DOWN>(acc[ms][0], acc[ms][1], dst);
    }
    // the redundant loads issued past the end still target this block's LDS: it must not end before they have landed
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

// ---------------------------------------------------------------------------------------------
// The 64 weight rows of a wavefront in the wide and the thin tiles and their way to the registers: down: 64 consecutive ones;
// gate/up: 32 gate rows, then the same up rows.
template <bool DOWN, int FMT>
struct weight_rows {
    uint64_t lo, hi, s_base = 0; // rows 0 .. 31 and 32 .. 63; scales of the matrix that row `lane` is in
    uint32_t rb, s_row = 0;      // bytes of a row; first scale of row `lane`
    uint32_t off[2] = {0, 0};    // bf16: even and odd groups of eight rows
    uint32_t scale_sel = 0;
    int lg;                      // group = 2^lg
    // The half of the aligned word that a scale is in, as v_perm_b32 wants it: (row * groups + group) odd or even (the parity of a
    // row's place in its matrix is that of its place in the tile); with groups of 32 both groups of a step are in the word.
    static constexpr uint32_t kFirst = 0x01000C0Cu, kOther = 0x02020000u;

    __device__ __forceinline__ weight_rows(const dx_handle *h, int row0, int K, int group, int lane)
    {
        rb = FMT == 0 ? (uint32_t)K * 2 : (FMT == 1 ? (uint32_t)K / 2 : (uint32_t)K / 4);
        lo = scalar_ptr(uniform_load(DOWN ? &h->w_down : &h->w_gate)) + (uint64_t)row0 * rb;
        hi = DOWN ? lo + (uint64_t)32 * rb : scalar_ptr(uniform_load(&h->w_up)) + (uint64_t)row0 * rb;
        lg = __builtin_ctz((unsigned)group);
        const int G = K >> lg;
        if constexpr (FMT != 0) {
            const uint64_t s_lo = scalar_ptr(uniform_load(DOWN ? &h->s_down : &h->s_gate)), s_hi = DOWN ? s_lo : scalar_ptr(uniform_load(&h->s_up));
            s_base = lane < 32 ? s_lo : s_hi;
            s_row = (uint32_t)(row0 + (DOWN ? lane : lane & 31)) * (uint32_t)G;
            scale_sel = kFirst ^ (G & lane & 1 ? kOther : 0u);
        } else {
#pragma unroll
            for (int p = 0; p < 2; ++p) off[p] = (uint32_t)(lane >> 3) * rb + (uint32_t)((lane & 7) ^ (4 * p + (lane >> 4))) * 16;
        }
    }
    // bf16: eight rows (i = 0 .. 7) of step kt, laid out as the token rows: + off[i & 1]
    __device__ __forceinline__ uint64_t rows_base(int kt, int i) const { return (i < 4 ? lo : hi) + (uint64_t)(8 * (i & 3)) * rb + (uint64_t)kt * kLine; }
    // Codes of steps 2c and 2c + 1: int4: 64 bytes of a row, four lanes to it, piece p of row r in slot p ^ ((r >> 2) & 3), i = 0 .. 3; int2: 32 bytes,
    // two lanes, i = 0, 1.  Past the end of an odd number of steps (not `whole`) the first half is read again.
    __device__ __forceinline__ uint64_t codes_base(int i, int c) const
    {
        if constexpr (FMT == 1) return (i < 2 ? lo : hi) + (uint64_t)(16 * (i & 1)) * rb + (uint64_t)c * 64;
        else return (i == 0 ? lo : hi) + (uint64_t)c * 32;
    }
    __device__ __forceinline__ uint32_t codes_off(bool whole, int lane) const
    {
        if constexpr (FMT == 1) {
            const uint32_t piece = (uint32_t)((lane & 3) ^ (lane >> 4)); // row 16 i + lane / 4
            return (uint32_t)(lane >> 2) * rb + (whole ? piece : piece & 1) * 16;
        } else {
            return (uint32_t)(lane >> 1) * rb + (whole ? lane & 1 : 0) * 16;
        }
    }
    // the aligned word that the scale of step kt is in
    __device__ __forceinline__ uint64_t scales_at(int kt) const { return s_base + (((s_row + (uint32_t)((kt * BK) >> lg)) * 2) & ~3u); }
    // both, to LDS
    __device__ __forceinline__ void issue_codes(uint32_t m0, int c, int nk, int lane) const
    {
        const bool whole = 2 * c + 1 < nk; // wave-uniform
#pragma unroll
        for (int i = 0; i < (FMT == 1 ? 4 : 2); ++i) load_to_lds(m0 + 1024 * i, codes_off(whole, lane), codes_base(i, c));
#pragma unroll
        for (int u = 0; u < 2; ++u) load_to_lds4(m0 + 64 * 64 + 256 * u, scales_at(whole ? 2 * c + u : 2 * c));
    }
    // step kt of the codes at p: of each tile of 32 rows the lane's elements 16 q + 8 kq .. + 7 of quarter q (int2: in half kq of word q), and
    // the scales of the first and of the second half of the step
    __device__ __forceinline__ void read_codes(const char *p, int kt, int lane, u32x4 (&codes)[2], float (&scale)[2][2]) const
    {
        const int r = lane & 31, kq = lane >> 5;
        uint32_t sel[2];
        sel[0] = scale_sel ^ (lg != 5 && ((kt * BK) >> lg & 1) ? kOther : 0u);
        sel[1] = sel[0] ^ (lg == 5 ? kOther : 0u);
#pragma unroll
        for (int n = 0; n < 2; ++n) {
            const int row = 32 * n + r;
            const uint32_t word = *reinterpret_cast<const uint32_t *>(p + 64 * 64 + 256 * (kt & 1) + 4 * row);
            if constexpr (FMT == 1) { // lane half kq has words 4 kq .. 4 kq + 3 of the step's eight; it takes words 2 q + kq
                const u32x4 c = *reinterpret_cast<const u32x4 *>(p + row * 64 + (((2 * (kt & 1) + kq) ^ ((r >> 2) & 3)) * 16));
                const auto first = __builtin_amdgcn_permlane32_swap(c.x, c.y, false, false);
                const auto second = __builtin_amdgcn_permlane32_swap(c.z, c.w, false, false);
                codes[n] = u32x4{first[0], second[0], first[1], second[1]};
            } else {
                codes[n] = *reinterpret_cast<const u32x4 *>(p + row * 32 + 16 * (kt & 1));
            }
#pragma unroll
            for (int half = 0; half < 2; ++half) scale[half][n] = __uint_as_float(__builtin_amdgcn_perm(0u, word, sel[half]));
        }
    }
};

// ---------------------------------------------------------------------------------------------
// Output tiles of 128 rows x 256 columns: 4 wavefronts side by side, each all rows x 64 columns of its own (4 x 2 MFMA tiles); two
// blocks to a compute unit.
// Why beside the narrow ones: no weight is shared between wavefronts.  So a wavefront turns its codes into operands in registers,
// in the shadow of the other block's matrix instructions, where the narrow kernel writes them to LDS for two wavefronts between two
// barriers; a row group of 32 without rows costs nothing; and a tile reads 24 KB from LDS per wavefront and 1.05 MFLOP (a 64 x 64
// sub-tile 16 KB per 0.52) and loads three quarters of the bytes per FLOP.  64 int4 experts of 2048 x 1536, 100 rows each: gate/up 148 ->
// 122 us, down 79 -> 64.  What bounds it: the latency of the weights.  A wavefront's 8 KB of a step (bf16) are read to registers at the
// step's start and loaded again at once, so they have one step to arrive: 1.9 us a step for one block or two.
//   LDS: two slots of token rows (laid out as in the other kernel); weights: of the wavefront alone, no barrier.  Codes come for two steps
//   at a time, 64 (int2: 32) bytes of a row, into two slots.  The matrix instructions take the elements of every format in the order
//   of the narrow tiles, so a token's result does not depend on which kind a call has.  What that costs (swaps, shifts, a scale more) the
//   expansion makes up for: nibbles as bytes that the conversion picks, pairs of crumbs that a byte selection looks up.  Calls, us, with the lanes'
//   own order, in order, and in order with this expansion: all int4, 16 experts of 4096 x 6400, 200 rows each 689, 691 and 663, 128 of 2048 x 768,
//   40 rows 166, 168 and 161; int2 616, 614 and 612, 147, 148 and 145.
template <bool DOWN, int FMT>
__device__ __forceinline__ void wide_tile(const dx_fwd_args &a, const tile_id &t, const dx_handle *h, char *ring)
{
    constexpr bool quant = FMT != 0;
    constexpr int ROWS = cfg::ROWS, B0 = 2 * cfg::A_SLOT;
    const bool shared = t.e == a.E;
    const int fe = shared ? a.shared_f : a.f;
    const int K = DOWN ? fe : a.d;
    const int nk = K / BK;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rows = t.m - t.mt * ROWS < ROWS ? t.m - t.mt * ROWS : ROWS;
    const int live = (rows + 31) >> 5; // row groups of 32 with rows
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_char *)ring;

    // ---- loader: wavefront w fills token rows [32w, 32w + 32) and its own 64 weight rows ----
    uint64_t a_at[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int row = 32 * wave + 8 * i + (lane >> 3);
        const uint32_t piece = (uint32_t)((lane & 7) ^ ((row >> 1) & 7));
        int slot = t.mt * ROWS + row;
        slot = slot < t.m ? slot : t.m - 1;
        if constexpr (DOWN) {
            a_at[i] = (uint64_t)a.h + (uint64_t)(t.seg0 + slot) * a.fmax * 2 + piece * 16;
        } else {
            const int tok = shared ? t.seg0 - a.T * a.k + slot : a.perm[t.seg0 + slot] / a.k;
            a_at[i] = (uint64_t)a.x + (uint64_t)tok * K * 2 + piece * 16;
        }
    }
    const bool loads_tokens = wave < live;
    // (the last tile of columns may be half a tile: the wavefronts of the missing half load the last rows again)
    const int N = DOWN ? a.d : fe, first = DOWN ? t.nt * BNW + 64 * wave : t.nt * (BNW / 2) + 32 * wave;
    const int row0 = first < N ? first : N - (DOWN ? 64 : 32);
    const weight_rows<DOWN, FMT> w(h, row0, K, a.group, lane);
    auto issue_token = [&](int slot, int i) { // called for steps 0, 1, 2, ...
        if (loads_tokens) {
            load_to_lds(lds0 + (uint32_t)(slot * cfg::A_SLOT + (32 * wave + 8 * i) * kLine), a_at[i]);
            a_at[i] += kLine;
        }
    };
    auto issue_tokens = [&](int slot) {
#pragma unroll
        for (int i = 0; i < 4; ++i) issue_token(slot, i);
    };
    const uint32_t b_at = lds0 + B0 + wave * cfg::B_WAVE;
    auto issue_weight = [&](int kt, int i) { // bf16
        load_to_lds(b_at + 1024 * i, w.off[i & 1], w.rows_base(kt, i));
    };
    const uint32_t c_at = lds0 + B0 + wave * 2 * cfg::SIDE_WIDE;
    auto issue_codes = [&](int c, int slot) { w.issue_codes(c_at + (uint32_t)(slot * cfg::SIDE_WIDE), c, nk, lane); }; // of steps 2c and 2c + 1

    // ---- MFMA role: all rows x the wavefront's 64 weight rows ----
    const int r = lane & 31, kq = lane >> 5, swz = (r >> 1) & 7;
    if constexpr (DOWN) { // the pair indices of the tile's rows, where they go
        if (!shared && wave < 2) {
            const int slot = t.mt * ROWS + wave * 64 + lane;
            load_to_lds4(lds0 + cfg::LDS + 256 * wave, (uint32_t)(slot < t.m ? slot : t.m - 1) * 4u, scalar_ptr(a.perm + t.seg0));
        }
    }
    f32x16 acc[4][2];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int ns = 0; ns < 2; ++ns)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][ns][v] = 0.f;
    frag8 fa[2][4];
    u32x4 fb[2][quant ? 1 : 4]; // bf16: the step's operands; quantized: the codes of the lane's elements 16 s + 8 kq .. + 7 of quarter s
    uint32_t scales[2] = {0, 0};
    const char *const a_rd = ring + r * kLine;
    auto read_a = [&](int slot, int s, frag8 (&af)[4]) {
        const char *p = a_rd + slot * cfg::A_SLOT + (((2 * s + kq) ^ swz) * 16);
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (i == 0 || i < live) af[i].u = *reinterpret_cast<const u32x4 *>(p + i * 32 * kLine);
    };
    auto read_weights = [&](int kt) {
        if constexpr (!quant) {
            const char *p = ring + B0 + wave * cfg::B_WAVE + r * kLine;
#pragma unroll
            for (int s = 0; s < 4; ++s)
#pragma unroll
                for (int ns = 0; ns < 2; ++ns) fb[ns][s] = *reinterpret_cast<const u32x4 *>(p + ns * 32 * kLine + (((2 * s + kq) ^ swz) * 16));
        } else {
            const char *p = ring + B0 + wave * 2 * cfg::SIDE_WIDE + ((kt >> 1) & 1) * cfg::SIDE_WIDE;
#pragma unroll
            for (int ns = 0; ns < 2; ++ns) {
                const int row = 32 * ns + r;
                scales[ns] = *reinterpret_cast<const uint32_t *>(p + 64 * 64 + 256 * (kt & 1) + 4 * row);
                if constexpr (FMT == 1) {
                    fb[ns][0] = *reinterpret_cast<const u32x4 *>(p + row * 64 + (((2 * (kt & 1) + kq) ^ ((r >> 2) & 3)) * 16));
                } else { // (the lane's half of word s)
                    fb[ns][0] = *reinterpret_cast<const u32x4 *>(p + row * 32 + 16 * (kt & 1));
                }
            }
        }
    };
    // The half of the aligned word that a scale is in, as v_perm_b32 wants it: (row * groups + group) odd or even (the parity of a
    // row's place in its matrix is that of its place in the tile); with groups of 32 both groups of a step are in the word.
    constexpr uint32_t kFirst = 0x01000C0Cu, kOther = 0x02020000u;
    const int lg = w.lg, G = K >> lg;
    const uint32_t scale_sel = kFirst ^ (G & r & 1 ? kOther : 0u);
    float scale[2][2] = {}; // of the first and of the second half of the step's elements
    crumb_products products[2] = {crumb_products(0.f), crumb_products(0.f)}; // int2 (groups of 64 and more: of the whole step)
    auto operand = [&](int ns, int s) {
        frag8 b;
        if constexpr (FMT == 0) b.u = fb[ns][s];
        else if constexpr (FMT == 1) b.u = dequant8(fb[ns][0][s], scale[ns][s >> 1]);
        else b.u = dequant8_crumbs(__builtin_amdgcn_ubfe(fb[ns][0][s], 16 * kq, 16), products[ns]);
        return b;
    };
    if constexpr (quant) {
        issue_codes(0, 0);
        issue_tokens(0);
        if (2 < nk) issue_codes(1, 1);
    } else {
        issue_tokens(0);
#pragma unroll
        for (int i = 0; i < 8; ++i) issue_weight(0, i);
    }
    for (int kt = 0; kt < nk; ++kt) {
        // own loads of step kt have landed; after the barrier that holds for every wavefront, and all have read the tokens of step kt - 1
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        block_barrier();
        const int slot = kt & 1;
        read_weights(kt);
        read_a(slot, 0, fa[0]);
        if (quant && kt + 1 < nk) issue_tokens(slot ^ 1);
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); // own weights are in registers: the next ones may come
        if constexpr (quant) {
            if ((kt & 1) && kt + 3 < nk) issue_codes((kt + 3) >> 1, (kt >> 1) & 1);
            uint32_t sel[2];
            sel[0] = scale_sel ^ (lg != 5 && ((kt * BK) >> lg & 1) ? kOther : 0u);
            sel[1] = sel[0] ^ (lg == 5 ? kOther : 0u);
#pragma unroll
            for (int ns = 0; ns < 2; ++ns) {
                if constexpr (FMT == 1) { // lane half kq has words 4 kq .. 4 kq + 3 of the step's eight; it takes words 2 s + kq
                    const auto first = __builtin_amdgcn_permlane32_swap(fb[ns][0].x, fb[ns][0].y, false, false);
                    const auto second = __builtin_amdgcn_permlane32_swap(fb[ns][0].z, fb[ns][0].w, false, false);
                    fb[ns][0] = u32x4{first[0], second[0], first[1], second[1]};
                }
#pragma unroll
                for (int half = 0; half < 2; ++half) scale[ns][half] = __uint_as_float(__builtin_amdgcn_perm(0u, scales[ns], sel[half])) * (FMT == 1 ? 0.0625f : 1.f);
                if constexpr (FMT == 2) products[ns] = crumb_products(scale[ns][0]);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            if (s < 3) read_a(slot, s + 1, fa[(s + 1) & 1]);
            const frag8 b0 = operand(0, s), b1 = operand(1, s);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (i == 0 || i < live) {
                    acc[i][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b0.v, fa[s & 1][i].v, acc[i][0], 0, 0, 0);
                    acc[i][1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b1.v, fa[s & 1][i].v, acc[i][1], 0, 0, 0);
                }
                if constexpr (!quant) { // the loads of the next step take turns with the first half's matrix instructions
                    if (kt + 1 < nk) {
                        if (s == 0) issue_weight(kt + 1, 2 * i), issue_weight(kt + 1, 2 * i + 1);
                        else if (s == 1) issue_token(slot ^ 1, i);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    // The tile leaves straight from the registers.
    const int col = DOWN ? t.nt * BNW + 64 * wave : t.nt * (BNW / 2) + 32 * wave;
    if (col >= N) return;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int row = 32 * i + r, slot = t.mt * ROWS + row;
        if (row >= rows) continue;
        dx_bf16 *dst;
        if constexpr (DOWN) {
            const int orow = shared ? t.seg0 + slot : *reinterpret_cast<const int *>(ring + cfg::LDS + 4 * row);
            dst = reinterpret_cast<dx_bf16 *>(a.o) + (size_t)orow * a.d + col + 8 * kq;
        } else {
            dst = a.h + (size_t)(t.seg0 + slot) * a.fmax + col + 8 * kq;
        }
        store_row<DOWN>(acc[i][0], acc[i][1], dst);
    }
}

// ---------------------------------------------------------------------------------------------
// Segments of up to 32 rows: 4 wavefronts side by side, each the segment's rows x 64 columns of its own (1 x 2 MFMA tiles); two blocks
// to a compute unit.  What bounds it: the weights, which nothing else asks for, so a compute unit needs enough of them on their way.
// Tokens are the first MFMA operand: accumulator element v is token (v / 4) * 8 + (lane / 32) * 4 + v % 4 of weight row lane % 32.

// ALONE: calls of few tokens, which have no other tiles: segments of more rows in several tiles, the shared expert's among them, and O in fp32.

// the shared expert (bf16) in a call of thin tiles alone
template <bool ALONE>
__device__ __forceinline__ bool thin_shared(const dx_fwd_args &a, const tile_id &t)
{
    return ALONE && t.e == a.E;
}

// where a lane's part of token row 8 * wave + lane / 8 comes from (rows past the end repeat the last one)
template <bool DOWN, bool ALONE>
__device__ __forceinline__ uint64_t thin_token_at(const dx_fwd_args &a, const tile_id &t, int K, int wave, int lane)
{
    const int row = 8 * wave + (lane >> 3), at = (ALONE ? t.mt * DX_THIN_ROWS : 0) + row, slot = at < t.m ? at : t.m - 1;
    const uint32_t piece = (uint32_t)((lane & 7) ^ ((row >> 1) & 7));
    if constexpr (DOWN) return (uint64_t)a.h + (uint64_t)(t.seg0 + slot) * a.fmax * 2 + piece * 16;
    else return (uint64_t)a.x + (uint64_t)(thin_shared<ALONE>(a, t) ? slot : a.perm[t.seg0 + slot] / a.k) * K * 2 + piece * 16;
}

// row of H or O that token lane % 32 goes to
template <bool DOWN, bool ALONE>
__device__ __forceinline__ int thin_row(const dx_fwd_args &a, const tile_id &t, int lane)
{
    const int at = (ALONE ? t.mt * DX_THIN_ROWS : 0) + (lane & 31), place = t.seg0 + (at < t.m ? at : t.m - 1);
    return DOWN && !thin_shared<ALONE>(a, t) ? a.perm[place] : place;
}

template <bool DOWN, bool ALONE>
__device__ __forceinline__ void store_thin(const dx_fwd_args &a, const tile_id &t, const f32x16 (&acc)[2], int row, int first, int lane)
{
    const int rows = t.m - (ALONE ? t.mt * DX_THIN_ROWS : 0);
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        if (8 * (v >> 2) >= rows) break; // wave-uniform: most segments have few rows, and an exact SwiGLU is some thirty instructions
        const int token = (v >> 2) * 8 + 4 * (lane >> 5) + (v & 3);
        const int to = __shfl(row, token);
        if (token >= rows) continue;
        if constexpr (DOWN && ALONE) {
            float *dst = a.o + (size_t)to * a.d + first + (lane & 31);
            dst[0] = acc[0][v], dst[32] = acc[1][v];
        } else if constexpr (DOWN) {
            dx_bf16 *dst = reinterpret_cast<dx_bf16 *>(a.o) + (size_t)to * a.d + first + (lane & 31);
            const uint32_t both = pack_bf16(acc[0][v], acc[1][v]);
            dst[0] = (dx_bf16)both, dst[32] = (dx_bf16)(both >> 16);
        } else {
            a.h[(size_t)to * a.fmax + first + (lane & 31)] = (dx_bf16)pack_bf16(swiglu(acc[0][v], acc[1][v]), 0.f);
        }
    }
}

// Quantized weights.  The codes of two steps (half a line of a row) and their tokens are a slot; two slots are in flight while the third is
// multiplied.  The values are multiplied as integers (int4: 16 times the code), and the group's scale
// multiplies the group's fp32 sums once, as in the streaming kernels.  (By way of registers, as bf16 weights come: 5 to 15 % slower.)
//   LDS: token rows, laid out as in the other kernels, then the codes of each wavefront alone.  One barrier per slot: behind it every
//   wavefront has read the slot that is filled next.
template <bool DOWN, int FMT, bool ALONE>
__device__ __forceinline__ void thin_codes(const dx_fwd_args &a, const tile_id &t, const dx_handle *h, char *ring)
{
    constexpr int SLOTS = cfg::THIN_SLOTS, A_SLOT = 2 * cfg::THIN_A, W_SLOT = cfg::SIDE_WIDE, W0 = SLOTS * A_SLOT;
    constexpr int LOADS = FMT == 1 ? 8 : 6; // of a wavefront per slot
    const int K = DOWN ? a.f : a.d, nk = K / BK, ns = (nk + 1) / 2; // steps, slots
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_char *)ring;

    // ---- loader: wavefront w fills token rows [8w, 8w + 8) and its own 64 weight rows ----
    uint64_t a_at = thin_token_at<DOWN, ALONE>(a, t, K, wave, lane);
    // (the last tile of columns may be half a tile: the wavefronts of the missing half load the last rows again)
    const int N = DOWN ? a.d : a.f, first = DOWN ? t.nt * BNW + 64 * wave : t.nt * (BNW / 2) + 32 * wave;
    const weight_rows<DOWN, FMT> w(h, first < N ? first : N - (DOWN ? 64 : 32), K, a.group, lane);
    auto issue = [&](int s, int slot) { // called for s = 0, 1, 2, ...
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            load_to_lds(lds0 + (uint32_t)(slot * A_SLOT + u * cfg::THIN_A + 1024 * wave), a_at);
            a_at += 2 * s + u + 1 < nk ? kLine : 0;
        }
        w.issue_codes(lds0 + (uint32_t)(W0 + (wave * SLOTS + slot) * W_SLOT), s, nk, lane);
    };

    // ---- MFMA role: all rows x the wavefront's 64 weight rows ----
    const int r = lane & 31, kq = lane >> 5, swz = (r >> 1) & 7;
    const int row = thin_row<DOWN, ALONE>(a, t, lane);
    f32x16 acc[2], part[2];
#pragma unroll
    for (int n = 0; n < 2; ++n)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[n][v] = part[n][v] = 0.f;
    const crumb_products crumbs(1.f);
    constexpr float kUnit = FMT == 1 ? 0.0625f : 1.f; // int4: the integers are 16 times the codes
    auto flush = [&](const float (&scale)[2]) { // a group is complete
#pragma unroll
        for (int n = 0; n < 2; ++n)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                acc[n][v] = fmaf(part[n][v], scale[n] * kUnit, acc[n][v]);
                part[n][v] = 0.f;
            }
    };
    issue(0, 0);
    if (ns > 1) issue(1, 1);
    int slot = 0;
    for (int s = 0; s < ns; ++s) {
        // own loads of the slot have landed; after the barrier that holds for every wavefront, and all have read the slot before it
        if (s + 1 < ns) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(LOADS) : "memory");
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        block_barrier();
        if (s + 2 < ns) issue(s + 2, slot == 0 ? SLOTS - 1 : slot - 1);
        const char *wp = ring + W0 + (wave * SLOTS + slot) * W_SLOT;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int kt = 2 * s + u;
            if (kt >= nk) break; // wave-uniform
            frag8 af[4];
#pragma unroll
            for (int q = 0; q < 4; ++q)
                af[q].u = *reinterpret_cast<const u32x4 *>(ring + slot * A_SLOT + u * cfg::THIN_A + r * kLine + (((2 * q + kq) ^ swz) * 16));
            u32x4 codes[2];
            float scale[2][2]; // [first and second half of the step][tile]
            w.read_codes(wp, kt, lane, codes, scale);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
#pragma unroll
                for (int n = 0; n < 2; ++n) {
                    frag8 b;
                    if constexpr (FMT == 1) b.u = dequant8(codes[n][q], 1.f);
                    else b.u = dequant8_crumbs(__builtin_amdgcn_ubfe(codes[n][q], 16 * kq, 16), crumbs);
                    part[n] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[q].v, b.v, part[n], 0, 0, 0);
                }
                if (q == 1 && w.lg == 5) flush(scale[0]);
            }
            if (w.lg < 7 || u || kt + 1 == nk) flush(scale[1]);
        }
        slot = slot + 1 < SLOTS ? slot + 1 : 0;
    }
    if (first < N) store_thin<DOWN, ALONE>(a, t, acc, row, first, lane);
}

// bf16 weights.  They and the token rows come to registers, and pass through LDS on their way to the operands: with the
// non-temporal hint, from which loads to LDS gain nothing, a cold stream runs at 6.2 TB/s, by loads to LDS at 5.2 (30B-shaped, 130 tokens: a
// layer 107 us by loads to LDS, 101 this way).  Four steps are in flight (250 registers), and every tile starts at another one and goes round: tiles that start together
// would all ask for the same 128 bytes of rows that lie a power of two apart, which are in few of the memory's channels.  128 experts of 2048 x 768, top-8, a
// layer, us, balanced routing, 129, 160 and 256 tokens: two steps and the same start 149, 150 and 153, three steps 147, 147 and 148, and starts of their own 138, 138 and
// 142; Zipf(1.1) 102, 105, 118 and 97, 99, 115.  The fourth step: balanced 129 and 200 tokens 136 -> 130, 138 -> 130, 16 of 4096 x 6400 128 tokens 341 -> 338, the others the same.  (Codes, which are a quarter as much, gain nothing by it: 80B-shaped, 150 tokens 88 and 90.)
//   LDS: two slots of token rows, one barrier per step: behind it every wavefront has read the slot that is filled next; one slot of the
//   weights of each wavefront alone.
template <bool DOWN, bool ALONE>
__device__ __forceinline__ void thin_rows(const dx_fwd_args &a, const tile_id &t, const dx_handle *h, char *ring)
{
    constexpr int DEPTH = 4, W0 = 2 * cfg::THIN_A;
    static_assert(W0 + cfg::WAVES * cfg::B_WAVE <= cfg::LDS, "the ring");
    const int fe = thin_shared<ALONE>(a, t) ? a.shared_f : a.f;
    const int K = DOWN ? fe : a.d, nk = K / BK;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    // ---- loader: wavefront w loads token rows [8w, 8w + 8) and its own 64 weight rows (the last tile of columns may be half a tile: the
    // wavefronts of the missing half load the last rows again) ----
    const DX_GLOBAL char *const a_at = (const DX_GLOBAL char *)thin_token_at<DOWN, ALONE>(a, t, K, wave, lane);
    const int N = DOWN ? a.d : fe, first = DOWN ? t.nt * BNW + 64 * wave : t.nt * (BNW / 2) + 32 * wave;
    const weight_rows<DOWN, 0> w(h, first < N ? first : N - (DOWN ? 64 : 32), K, a.group, lane);
    struct step_regs {
        u32x4 tokens, weights[8];
    } st[DEPTH];
    const int begin = (int)((uint32_t)(7 * t.nt + 13 * t.e) % (uint32_t)nk);
    auto fetch = [&](int step, step_regs &to) __attribute__((always_inline)) { // the tile's step: step 0 is the matrix's step `begin`
        const int kt = step + begin < nk ? step + begin : step + begin - nk;
        to.tokens = *reinterpret_cast<const DX_GLOBAL u32x4 *>(a_at + (uint32_t)(kt * kLine));
#pragma unroll
        for (int i = 0; i < 8; ++i)
            to.weights[i] = __builtin_nontemporal_load(reinterpret_cast<const DX_GLOBAL u32x4 *>(w.rows_base(kt, i) + w.off[i & 1]));
    };

    // ---- MFMA role: all rows x the wavefront's 64 weight rows ----
    const int r = lane & 31, kq = lane >> 5, swz = (r >> 1) & 7;
    const int row = thin_row<DOWN, ALONE>(a, t, lane);
    f32x16 acc[2];
#pragma unroll
    for (int n = 0; n < 2; ++n)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[n][v] = 0.f;
    char *const w_at = ring + W0 + wave * cfg::B_WAVE;
    // step kt: to LDS and, behind the barrier, into the products; its registers take step `next` (negative: none)
    auto consume = [&](int kt, step_regs &from, int next) __attribute__((always_inline)) {
        char *const a_slot = ring + (kt & 1) * cfg::THIN_A;
        *reinterpret_cast<u32x4 *>(a_slot + 1024 * wave + 16 * lane) = from.tokens;
#pragma unroll
        for (int i = 0; i < 8; ++i) *reinterpret_cast<u32x4 *>(w_at + 1024 * i + 16 * lane) = from.weights[i];
        if (next >= 0) fetch(next, from);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); // own stores are in LDS; behind the barrier every wavefront's
        block_barrier();
        frag8 af[4], b[2][4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int at = r * kLine + (((2 * q + kq) ^ swz) * 16);
            af[q].u = *reinterpret_cast<const u32x4 *>(a_slot + at);
#pragma unroll
            for (int n = 0; n < 2; ++n) b[n][q].u = *reinterpret_cast<const u32x4 *>(w_at + 32 * n * kLine + at);
        }
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int n = 0; n < 2; ++n) acc[n] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[q].v, b[n][q].v, acc[n], 0, 0, 0);
    };
#pragma unroll
    for (int i = 0; i < DEPTH; ++i)
        if (i < nk) fetch(i, st[i]);
    // With every load issued without a branch the compiler waits for the step that it stores only; the last steps apart.
    int kt = 0;
    for (; kt + 2 * DEPTH - 1 < nk; kt += DEPTH)
#pragma unroll
        for (int i = 0; i < DEPTH; ++i) consume(kt + i, st[i], kt + i + DEPTH);
    for (; kt < nk; kt += DEPTH)
#pragma unroll
        for (int i = 0; i < DEPTH; ++i)
            if (kt + i < nk) consume(kt + i, st[i], kt + i + DEPTH < nk ? kt + i + DEPTH : -1);
    if (first < N) store_thin<DOWN, ALONE>(a, t, acc, row, first, lane);
}

template <bool DOWN>
__global__ __launch_bounds__(cfg::THREADS, 2) void k_tiled(dx_fwd_args a)
{
    // the ring and (down) the pair indices of the rows: two blocks to a compute unit
    __shared__ __attribute__((aligned(1024))) char ring[cfg::LDS + (DOWN ? 256 * cfg::WAVES : 0)];
    tile_kind kind;
    const tile_id t = find_tile<DOWN>(a, kind);
    if (!t.valid) return; // block-uniform
    const dx_handle *h = t.e == a.E ? a.shared : a.table + t.e;
    const int fmt = (int)uniform_load(&h->fmt);
    if (kind == kThin) {
        if (fmt == DX_FMT_INT4G) thin_codes<DOWN, 1, false>(a, t, h, ring);
        else if (fmt == DX_FMT_INT2G) thin_codes<DOWN, 2, false>(a, t, h, ring);
        else thin_rows<DOWN, false>(a, t, h, ring);
    } else if (kind == kWide) {
        if (fmt == DX_FMT_INT4G) wide_tile<DOWN, 1>(a, t, h, ring);
        else if (fmt == DX_FMT_INT2G) wide_tile<DOWN, 2>(a, t, h, ring);
        else wide_tile<DOWN, 0>(a, t, h, ring);
    } else {
        if (fmt == DX_FMT_INT4G) narrow_tile<DOWN, 1>(a, t, h, ring);
        else if (fmt == DX_FMT_INT2G) narrow_tile<DOWN, 2>(a, t, h, ring);
        else narrow_tile<DOWN, 0>(a, t, h, ring);
    }
}

// Thin tiles alone (calls of few tokens).  The row tiles of a segment, up to four, go next to each other, so that its weights come to one XCD; four tiles at
// a time to an XCD.  A kernel of its own: as part of k_tiled it cost the calls of more tokens 1 to 4 %.
template <bool DOWN>
__global__ __launch_bounds__(cfg::THREADS, 2) void k_thin(dx_fwd_args a)
{
    __shared__ __attribute__((aligned(1024))) char ring[cfg::LDS];
    const int n = uniform_load(&a.tiles->n_thin) + uniform_load(&a.tiles->n_thin_quant), n_shared = uniform_load(&a.tiles->n_thin_shared);
    const int ntn = columns_of<DOWN>(a, a.f, BNW), ntn_shared = columns_of<DOWN>(a, a.shared_f, BNW);
    const uint32_t routed = (uint32_t)(n * ntn), total = routed + (uint32_t)(n_shared * ntn_shared);
    const uint32_t at = blockIdx.x >> 3, idx = ((at >> 2) * 8 + (blockIdx.x & 7)) * 4 + (at & 3);
    if (idx >= total) return; // block-uniform
    const dx_tile_row *rows = reinterpret_cast<const dx_tile_row *>(a.tiles + 1);
    const tile_id t = idx < routed ? tile_of<DX_THIN_ROWS, 4>(rows, idx, ntn) : tile_of<DX_THIN_ROWS, 4>(rows + n, idx - routed, ntn_shared);
    const dx_handle *h = t.e == a.E ? a.shared : a.table + t.e;
    const int fmt = (int)uniform_load(&h->fmt);
    if (fmt == DX_FMT_INT4G) thin_codes<DOWN, 1, true>(a, t, h, ring);
    else if (fmt == DX_FMT_INT2G) thin_codes<DOWN, 2, true>(a, t, h, ring);
    else thin_rows<DOWN, true>(a, t, h, ring);
}

// ---------------------------------------------------------------------------------------------
// Large segments: 256 x 256 output tiles, 8 wavefronts (2 along rows x 4 along columns, each a 128 x 64 sub-tile = 4 x 2
// MFMA tiles), one block to a compute unit, K in steps of 64 through two stages, one barrier per step.
// Why beside the 128-row tiles: their operand reads take as many LDS cycles as the matrix instructions (a 64 x 64 sub-tile
// reads 16 KB per 524 kFLOP) and the fill comes on top; a 128 x 64 sub-tile reads 24 KB per 1.05 MFLOP, and a tile loads half
// the bytes per FLOP.  With few or ragged row tiles the smaller tiles win all the same: no padding, two blocks whose waits
// overlap: large segments only (big_tile_formats, with the passes measured on both sides of its lines).
//   LDS rows and loads as in the other kernel.  Codes (Q4): four bytes per lane into a side ring (per slot and wavefront:
//   4 x 8 rows x 32 bytes of nibbles, 32 rows x one pair of scales), one step before the wavefront that loaded them expands
//   them into the weight half of the stage that has just been freed; it expands only what it loaded itself, so the side ring
//   needs no barrier.
constexpr int TM = 256, TN = 256, TK = 64;
constexpr int kBigThreads = 512;
constexpr int kRowBytes64 = TK * 2;                      // 128: one line of a row per step
constexpr int kStageBytes = (TM + TN) * kRowBytes64;     // 64 KB: token rows then weight rows
constexpr int kStages = 2;
constexpr int kSideWave = 1280;                          // per wavefront: 4 x 256 bytes of nibbles, 256 of scale pairs
constexpr int kSideStage = (kBigThreads / 64) * kSideWave; // 10 KB
constexpr int kRingBytes = kStages * (kStageBytes + kSideStage);

template <bool DOWN, bool Q4>
__device__ __forceinline__ void big_tile(const dx_fwd_args &a, const tile_id &t, const dx_handle *h, char *ring)
{
    const bool shared = t.e == a.E;
    const int fe = shared ? a.shared_f : a.f;
    const int K = DOWN ? fe : a.d;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 2, wn = wave & 3;

    // ---- loader role: wavefront w fills rows [32w, 32w + 32) of the token part and of the weight part ----
    // A load instruction covers 8 rows x one 128-byte line; lane l writes LDS piece l % 8 of row l / 8 and
    // fetches the memory piece that belongs there: piece p of row r sits in slot p ^ ((r >> 1) & 7).
    // weight-tile row -> matrix row: down: TN consecutive rows; gate/up: 128 gate rows, then the same up rows
    auto wrow = [&](int row) { return DOWN ? t.nt * TN + row : t.nt * (TN / 2) + (row & 127); };
    uint32_t a_off[4], b_off[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int row = 32 * wave + 8 * i + (lane >> 3);
        const uint32_t piece = (uint32_t)((lane & 7) ^ ((row >> 1) & 7));
        const int slot = t.mt * TM + row; // big tiles are full: slot < t.m
        if constexpr (DOWN) {
            a_off[i] = (uint32_t)(t.seg0 + slot) * (uint32_t)a.fmax * 2u + piece * 16u;
        } else {
            const int tok = shared ? t.seg0 - a.T * a.k + slot : a.perm[t.seg0 + slot] / a.k;
            a_off[i] = (uint32_t)tok * (uint32_t)K * 2u + piece * 16u;
        }
        // bf16: the lane's 16-byte piece of the row; int4: its four bytes (8 nibbles) of the row's 32 per step
        b_off[i] = Q4 ? (uint32_t)wrow(row) * (uint32_t)(K / 2) + (uint32_t)(lane & 7) * 4u
                      : (uint32_t)wrow(row) * (uint32_t)K * 2u + piece * 16u;
    }
    const uint64_t a_base = (uint64_t)(DOWN ? (const void *)a.h : (const void *)a.x);
    const uint64_t b_base = scalar_ptr(uniform_load(DOWN ? &h->w_down : (wave < 4 ? &h->w_gate : &h->w_up)));
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_char *)ring;
    const uint32_t m0_a = lds0 + wave * 32 * kRowBytes64, m0_b = lds0 + TM * kRowBytes64 + wave * 32 * kRowBytes64;
    const int nk = K / TK;
    // int4: scales of the lane's row (lane & 31 of the wavefront's 32 rows), read as the aligned pair that
    // holds the step's groups (the number of groups per row is even there, so a pair never leaves its row;
    // with groups of 32 a step spans exactly the two groups of its pair)
    const int lg = __builtin_ctz((unsigned)a.group);
    const uint32_t s_off = Q4 ? (uint32_t)wrow(32 * wave + (lane & 31)) * (uint32_t)(K >> lg) * 2u : 0u;
    const uint64_t s_base = Q4 ? scalar_ptr(uniform_load(DOWN ? &h->s_down : (wave < 4 ? &h->s_gate : &h->s_up))) : 0;
    const int side_wave = kStages * kStageBytes + wave * kSideWave; // + slot * kSideStage
    auto clamped = [&](int kt) { return kt < nk ? kt : nk - 1; };
    auto issue_tokens = [&](int kt, int stage) {
        const uint64_t kb = (uint64_t)clamped(kt) * kRowBytes64;
        const uint32_t so = (uint32_t)stage * kStageBytes;
#pragma unroll
        for (int i = 0; i < 4; ++i) load_to_lds(m0_a + so + 1024 * i, a_off[i], a_base + kb);
    };
    auto issue_weights = [&](int kt, int stage) { // bf16
        const uint64_t kb = (uint64_t)clamped(kt) * kRowBytes64;
        const uint32_t so = (uint32_t)stage * kStageBytes;
#pragma unroll
        for (int i = 0; i < 4; ++i) load_to_lds(m0_b + so + 1024 * i, b_off[i], b_base + kb);
    };
    auto issue_codes = [&](int kt, int slot) { // int4: nibbles and scale pairs of step kt -> side slot
        const int kc = clamped(kt);
        const uint32_t m0 = lds0 + (uint32_t)(side_wave + slot * kSideStage);
#pragma unroll
        for (int i = 0; i < 4; ++i) load_to_lds4(m0 + 256 * i, b_off[i], b_base + (uint64_t)kc * (TK / 2));
        load_to_lds4(m0 + 1024, s_off, s_base + (uint64_t)((((kc * TK) >> lg) * 2) & ~3));
    };
    // int4: the wavefront's 32 rows of step kt, from side slot `slot` into the weight half of `stage`
    auto expand = [&](int kt, int slot, int stage) {
        const int odd = ((clamped(kt) * TK + 8 * (lane & 7)) >> lg) & 1; // per lane when a group is 32 wide
        const char *side = ring + side_wave + slot * kSideStage;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t codes = *reinterpret_cast<const uint32_t *>(side + 256 * i + 4 * lane);
            const uint32_t pair = *reinterpret_cast<const uint32_t *>(side + 1024 + 4 * (8 * i + (lane >> 3)));
            const float scale = __uint_as_float(odd ? pair & 0xFFFF0000u : pair << 16);
            const int row = 32 * wave + 8 * i + (lane >> 3);
            const int pos = (lane & 7) ^ ((row >> 1) & 7);
            *reinterpret_cast<u32x4 *>(ring + stage * kStageBytes + TM * kRowBytes64 + row * kRowBytes64 + pos * 16) =
                dequant8(codes, scale * 0.0625f);
        }
    };

    // ---- MFMA role ----
    const int r = lane & 31, kq = lane >> 5, swz = (r >> 1) & 7;
    const int a_lane = (wm * 128 + r) * kRowBytes64;
    const int b_lane0 = TM * kRowBytes64 + (DOWN ? wn * 64 + r : wn * 32 + r) * kRowBytes64;
    const int b_lane1 = TM * kRowBytes64 + (DOWN ? wn * 64 + 32 + r : 128 + wn * 32 + r) * kRowBytes64;

    f32x16 acc[4][2];
#pragma unroll
    for (int ms = 0; ms < 4; ++ms)
#pragma unroll
        for (int ns = 0; ns < 2; ++ns)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[ms][ns][v] = 0.f;

    // Software pipeline.  Each K-step has four quarters (16 k-values each); the fragments of a quarter sit
    // in registers before its MFMAs start.  The barrier comes once the last quarter's fragments have been
    // read, in the shadow of the third quarter's MFMAs: past it every wavefront holds what it needs of
    // stage S, so S is refilled at once with step kt + 2, and the landed stage of step kt + 1 may be read.
    frag8 fa[2][4], fb[2][2];
    auto read_frags = [&](int stage, int quarter, frag8 (&af)[4], frag8 (&bf)[2]) {
        const char *st = ring + stage * kStageBytes;
        const int so = ((2 * quarter + kq) ^ swz) * 16;
#pragma unroll
        for (int ms = 0; ms < 4; ++ms) af[ms].u = *reinterpret_cast<const u32x4 *>(st + a_lane + ms * 32 * kRowBytes64 + so);
        bf[0].u = *reinterpret_cast<const u32x4 *>(st + b_lane0 + so);
        bf[1].u = *reinterpret_cast<const u32x4 *>(st + b_lane1 + so);
    };
    auto mma_quarter = [&](const frag8 (&af)[4], const frag8 (&bf)[2]) {
#pragma unroll
        for (int ms = 0; ms < 4; ++ms)
#pragma unroll
            for (int ns = 0; ns < 2; ++ns)
                acc[ms][ns] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bf[ns].v, af[ms].v, acc[ms][ns], 0, 0, 0);
    };
    if constexpr (Q4) {
        // The codes of step j are loaded with the tokens of step j - 1 and expanded when step j - 2 frees
        // its stage.  Start: codes 0, 1 and tokens 0, 1; expand 0, 1 as soon as the codes are there; then
        // the codes of step 2.
        issue_codes(0, 0);
        issue_codes(1, 1);
        issue_tokens(0, 0);
        issue_tokens(1, 1);
        asm volatile("s_waitcnt vmcnt(8)" ::: "memory"); // own codes 0, 1
        expand(0, 0, 0);
        expand(1, 1, 1);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); // side slot 0 has been read: refill it
        issue_codes(2, 0);
        asm volatile("s_waitcnt vmcnt(9) lgkmcnt(0)" ::: "memory"); // own tokens of step 0; own expansions
    } else {
        issue_tokens(0, 0), issue_weights(0, 0);
        issue_tokens(1, 1), issue_weights(1, 1);
        asm volatile("s_waitcnt vmcnt(8)" ::: "memory"); // own loads of step 0
    }
    block_barrier();
    read_frags(0, 0, fa[0], fb[0]);
    auto step = [&](int kt, auto stage_c) {
        constexpr int S = decltype(stage_c)::value;
        // (the scheduling fences keep the LDS reads ahead of the MFMAs they overlap with)
        read_frags(S, 1, fa[1], fb[1]);
        __builtin_amdgcn_sched_barrier(0);
        mma_quarter(fa[0], fb[0]);
        __builtin_amdgcn_sched_barrier(0);
        read_frags(S, 2, fa[0], fb[0]);
        __builtin_amdgcn_sched_barrier(0);
        mma_quarter(fa[1], fb[1]);
        __builtin_amdgcn_sched_barrier(0);
        read_frags(S, 3, fa[1], fb[1]);
        __builtin_amdgcn_sched_barrier(0);
        mma_quarter(fa[0], fb[0]);
        __builtin_amdgcn_sched_barrier(0);
        // own loads of step kt + 1 (int4: and the codes of step kt + 2) have landed; own LDS reads of stage S
        // have returned and own LDS writes are done; after the barrier that holds for every wavefront
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
        block_barrier();
        issue_tokens(kt + 2, S);
        if constexpr (Q4) {
            issue_codes(kt + 3, S ^ 1);
            expand(kt + 2, S, S);
        } else {
            issue_weights(kt + 2, S);
        }
        read_frags(S ^ 1, 0, fa[0], fb[0]);
        __builtin_amdgcn_sched_barrier(0);
        mma_quarter(fa[1], fb[1]);
        __builtin_amdgcn_sched_barrier(0);
    };
    for (int kt = 0; kt < nk; kt += 2) { // nk is even (K a multiple of 128)
        step(kt, std::integral_constant<int, 0>{});
        step(kt + 1, std::integral_constant<int, 1>{});
    }
    // the redundant loads issued past the end still target this block's LDS: drain them
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");

    // (the tile leaves straight from the registers, as in the other kernel)
    int o_row[4]; // where its rows go
#pragma unroll
    for (int ms = 0; ms < 4; ++ms) {
        const int slot = t.mt * TM + wm * 128 + ms * 32 + r;
        o_row[ms] = DOWN && !shared ? a.perm[t.seg0 + slot] : t.seg0 + slot;
    }
#pragma unroll
    for (int ms = 0; ms < 4; ++ms) {
        dx_bf16 *dst = DOWN ? reinterpret_cast<dx_bf16 *>(a.o) + (size_t)o_row[ms] * a.d + t.nt * TN + wn * 64 + 8 * kq
                            : a.h + (size_t)o_row[ms] * a.fmax + t.nt * (TN / 2) + wn * 32 + 8 * kq;
        store_row<DOWN>(acc[ms][0], acc[ms][1], dst);
    }
}

template <bool DOWN>
__global__ __launch_bounds__(kBigThreads) void k_big(dx_fwd_args a)
{
    __shared__ __attribute__((aligned(1024))) char ring[kRingBytes]; // 128 KB of stages and 20 KB of side ring
    const dx_tile_row *rows = reinterpret_cast<const dx_tile_row *>(a.tiles + 1) + uniform_load(&a.tiles->n_routed) + uniform_load(&a.tiles->n_shared);
    const int n = uniform_load(&a.tiles->n_big), n_shared = uniform_load(&a.tiles->n_big_shared);
    const int ntn = columns_of<DOWN>(a, a.f, TN), ntn_shared = columns_of<DOWN>(a, a.shared_f, TN);
    const uint32_t routed = (uint32_t)(n * ntn), total = routed + (uint32_t)(n_shared * ntn_shared), per_xcd = (total + 7) / 8;
    const uint32_t idx = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if ((blockIdx.x >> 3) >= per_xcd || idx >= total) return; // block-uniform
    const tile_id t = idx < routed ? tile_of<DX_BIG_ROWS, 4>(rows, idx, ntn) : tile_of<DX_BIG_ROWS, 4>(rows + n, idx - routed, ntn_shared);
    const dx_handle *h = t.e == a.E ? a.shared : a.table + t.e;
    if (uniform_load(&h->fmt) == DX_FMT_INT4G) big_tile<DOWN, true>(a, t, h, ring);
    else big_tile<DOWN, false>(a, t, h, ring);
}

// The list of row tiles on a caller's routing arrays (one block).
constexpr int kListThreads = 1024; // an expert to a thread

__global__ __launch_bounds__(kListThreads) void k_tile_list(dx_list_args l, const int32_t *offsets)
{
    __shared__ dx_tile_list::lds<kListThreads / 64> of_list;
    const bool owner = threadIdx.x < (unsigned)l.E;
    const int e = owner ? (int)threadIdx.x : l.E, seg0 = offsets[e];
    dx_tile_list::write<kListThreads / 64>(l, e, owner ? l.table[e].fmt : (uint32_t)DX_FMT_BF16, seg0, owner ? offsets[e + 1] - seg0 : 0, of_list);
}

} // namespace

template <bool DOWN>
static void launch_tiles(const dx_fwd_args &a, hipStream_t s)
{
    // an upper bound on the tile count; surplus blocks find no tile and leave
    const int fe = a.shared && a.shared_f > a.f ? a.shared_f : a.f;
    const long pairs = (long)a.T * a.k, active = pairs < a.E ? pairs : a.E, above = pairs / (DX_THIN_ROWS + 1);
    const long thin = active - (above < active ? above : active); // beside as many of more rows as there can be (a tile less there: one more here at most)
    const long tiles = dxk_tile_rows_max(a.T, a.k, a.E, DX_THIN_ROWS, a.shared != nullptr) * columns_of<DOWN>(a, fe, BN) + thin * columns_of<DOWN>(a, a.f, BNW);
    const long blocks = (tiles + 7 + 15 + 7) / 8 * 8; // the ranges of the XCDs: eighths of the one kind, of thin tiles in twos
    hipLaunchKernelGGL((k_tiled<DOWN>), dim3((unsigned)blocks), dim3(cfg::THREADS), 0, s, a);
}

template <bool DOWN>
static void launch_thin(const dx_fwd_args &a, hipStream_t s, hipEvent_t start, hipEvent_t stop)
{
    const int fe = a.shared && a.shared_f > a.f ? a.shared_f : a.f;
    const long tiles = dxk_thin_rows_max(a.T, a.k, a.E, a.shared != nullptr) * columns_of<DOWN>(a, fe, BNW);
    const dim3 grid((unsigned)((tiles + 31) / 32 * 32)), block(cfg::THREADS);
    if (start || stop) hipExtLaunchKernelGGL((k_thin<DOWN>), grid, block, 0, s, start, stop, 0, a);
    else hipLaunchKernelGGL((k_thin<DOWN>), grid, block, 0, s, a);
}

template <bool DOWN>
static void launch_big_tiles(const dx_fwd_args &a, hipStream_t s)
{
    const int fe = a.shared && a.shared_f > a.f ? a.shared_f : a.f;
    const long rows = (long)a.T * a.k / DX_BIG_ROWS + (a.shared ? a.T / DX_BIG_ROWS : 0), tiles = rows * (DOWN ? a.d / TN : fe / (TN / 2));
    if (a.m_big && tiles) hipLaunchKernelGGL((k_big<DOWN>), dim3((unsigned)((tiles + 7) / 8 * 8)), dim3(kBigThreads), 0, s, a);
}

void dxk_tile_list(const dx_list_args &l, const int32_t *offsets, hipStream_t s)
{
    hipLaunchKernelGGL(k_tile_list, dim3(1), dim3(kListThreads), 0, s, l, offsets);
}
void dxk_tiles_gate_up(const dx_fwd_args &a, hipStream_t s, hipEvent_t start, hipEvent_t stop)
{
    if (!a.o_bf16) return launch_thin<false>(a, s, start, stop);
    launch_big_tiles<false>(a, s);
    launch_tiles<false>(a, s);
}
void dxk_tiles_down(const dx_fwd_args &a, hipStream_t s, hipEvent_t start, hipEvent_t stop)
{
    if (!a.o_bf16) return launch_thin<true>(a, s, start, stop);
    launch_big_tiles<true>(a, s);
    launch_tiles<true>(a, s);
}
