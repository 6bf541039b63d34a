// The list of row tiles of a call that runs on tiles (dx_tile_head and the rows behind it), written by one block: the last one of the
// routing's placement kernel, which has every expert's count by then, or of a kernel of its own on a caller's routing arrays.
#pragma once

#include "dx_internal.h"
#include "dx_route_core.h"

namespace dx_tile_list {

constexpr int kCounts = 6; // row tiles of 128; of them those of quantized experts and of experts with one; row tiles of 256; thin tiles, bf16 and quantized

// All threads of a block of WAVES wavefronts.  A thread whose `e` is below l.E (increasing with the thread) has the expert's segment: m
// pairs from seg0 on; the other threads have l.E and no pairs.
template <int WAVES>
__device__ __forceinline__ void write(const dx_list_args &l, int e, int seg0, int m, int (*sums)[kCounts])
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    auto big_rows = [&](int rows, uint32_t fmt) { // leading rows that go in 256-row tiles
        return (l.m_big >> fmt) & 1 ? rows / DX_BIG_ROWS * DX_BIG_ROWS : 0;
    };
    auto tiles = [](int rows) { return (rows + DX_TILE_ROWS - 1) / DX_TILE_ROWS; };
    const uint32_t fmt = e < l.E ? l.table[e].fmt : (uint32_t)DX_FMT_BF16;
    const bool thin = m > 0 && m <= DX_THIN_ROWS, quant = fmt != DX_FMT_BF16;
    const int lead = m > DX_THIN_ROWS ? big_rows(m, fmt) : 0, t = m > DX_THIN_ROWS ? tiles(m - lead) : 0;
    const int mine[kCounts] = {t, quant ? t : 0, t == 1 && lead == 0, lead / DX_BIG_ROWS, thin && !quant, thin && quant};
    int base[kCounts], total[kCounts];
#pragma unroll
    for (int i = 0; i < kCounts; ++i) {
        const int upto = dx_route_core::wave_scan_inclusive(mine[i]);
        if (lane == 63) sums[wave][i] = upto;
        base[i] = upto - mine[i];
        total[i] = 0;
    }
    __syncthreads();
#pragma unroll
    for (int w = 0; w < WAVES; ++w)
#pragma unroll
        for (int i = 0; i < kCounts; ++i) {
            if (w < wave) base[i] += sums[w][i];
            total[i] += sums[w][i];
        }
    const int T_shared = l.shared ? l.T : 0, lead_shared = big_rows(T_shared, DX_FMT_BF16); // (more than DX_THIN_ROWS tokens)
    const int n_shared = tiles(T_shared - lead_shared), n_big_shared = lead_shared / DX_BIG_ROWS;
    dx_tile_row *rows = reinterpret_cast<dx_tile_row *>(l.tiles + 1), *big = rows + total[0] + n_shared, *thins = big + total[3] + n_big_shared;
    for (int mt = 0; mt < mine[3]; ++mt) big[base[3] + mt] = dx_tile_row{e, mt, lead, seg0};
    for (int mt = 0; mt < t; ++mt) rows[base[0] + mt] = dx_tile_row{e, mt, m - lead, seg0 + lead};
    if (thin) thins[quant ? total[4] + base[5] : base[4]] = dx_tile_row{e, 0, m, seg0};
    const int shared0 = l.T * l.k;
    for (int mt = tid; mt < n_shared; mt += 64 * WAVES) rows[total[0] + mt] = dx_tile_row{l.E, mt, T_shared - lead_shared, shared0 + lead_shared};
    for (int mt = tid; mt < n_big_shared; mt += 64 * WAVES) big[total[3] + mt] = dx_tile_row{l.E, mt, lead_shared, shared0};
    if (tid == 0) *l.tiles = dx_tile_head{total[0], n_shared, total[1], total[2], total[3], n_big_shared, total[4], total[5], l.n_cu};
}

} // namespace dx_tile_list
