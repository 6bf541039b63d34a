// The list of row tiles of a call that runs on tiles (dx_tile_head and the rows behind it), written by one block: the last one of the
// routing's placement kernel, which has every expert's count by then, or of a kernel of its own on a caller's routing arrays.
#pragma once

#include "dx_internal.h"
#include "dx_route_core.h"

namespace dx_tile_list {

constexpr int kCounts = 6; // row tiles of 128; of them those of quantized experts and of experts with one; row tiles of 256; thin tiles, bf16 and quantized

template <int WAVES>
struct lds {
    int of_wave[WAVES][kCounts];
};

// All threads of a block of WAVES wavefronts (16 at most).  A thread whose `e` is below l.E (increasing with the thread) has the expert's segment, m
// pairs from seg0 on, and its format; the other threads have l.E and no pairs.
template <int WAVES>
__device__ __forceinline__ void write(const dx_list_args &l, int e, uint32_t fmt, int seg0, int m, lds<WAVES> &s)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    auto big_rows = [&](int rows, uint32_t fmt) { // leading rows that go in 256-row tiles
        return (l.m_big >> fmt) & 1 ? rows / DX_BIG_ROWS * DX_BIG_ROWS : 0;
    };
    auto tiles = [](int rows) { return (rows + DX_TILE_ROWS - 1) / DX_TILE_ROWS; };
    const bool thin = m > 0 && (m <= DX_THIN_ROWS || l.thin_only), quant = fmt != DX_FMT_BF16;
    const int n_thin = thin ? (m + DX_THIN_ROWS - 1) / DX_THIN_ROWS : 0;
    const int lead = thin ? 0 : big_rows(m, fmt), t = thin ? 0 : tiles(m - lead);
    const int mine[kCounts] = {t, quant ? t : 0, t == 1 && lead == 0, lead / DX_BIG_ROWS, quant ? 0 : n_thin, quant ? n_thin : 0};
    int base[kCounts], total[kCounts];
#pragma unroll
    for (int i = 0; i < kCounts; ++i) {
        const int upto = dx_route_core::wave_scan_inclusive(mine[i]);
        if (lane == 63) s.of_wave[wave][i] = upto;
        base[i] = upto - mine[i];
    }
    __syncthreads();
    const int at = __builtin_amdgcn_readfirstlane(wave);
#pragma unroll
    for (int i = 0; i < kCounts; ++i) { // a wavefront's sum to a lane
        const int of = lane < WAVES ? s.of_wave[lane][i] : 0, upto = dx_route_core::wave_scan_inclusive(of);
        base[i] += __builtin_amdgcn_readlane(upto - of, at);
        total[i] = __builtin_amdgcn_readlane(upto, WAVES - 1);
    }
    const int T_shared = l.shared && !l.thin_only ? l.T : 0, lead_shared = big_rows(T_shared, DX_FMT_BF16); // (more than DX_THIN_ROWS tokens)
    const int n_shared = tiles(T_shared - lead_shared), n_big_shared = lead_shared / DX_BIG_ROWS;
    dx_tile_row *rows = reinterpret_cast<dx_tile_row *>(l.tiles + 1), *big = rows + total[0] + n_shared, *thins = big + total[3] + n_big_shared;
    for (int mt = 0; mt < mine[3]; ++mt) big[base[3] + mt] = dx_tile_row{e, mt, lead, seg0};
    for (int mt = 0; mt < t; ++mt) rows[base[0] + mt] = dx_tile_row{e, mt, m - lead, seg0 + lead};
    thins += quant ? total[4] + base[5] : base[4];
    for (int mt = 0; mt < n_thin; ++mt) thins[mt] = dx_tile_row{e, mt, m, seg0};
    const int shared0 = l.T * l.k, n_thin_shared = l.shared && l.thin_only ? (l.T + DX_THIN_ROWS - 1) / DX_THIN_ROWS : 0;
    thins = big + total[3] + n_big_shared + total[4] + total[5];
    for (int mt = tid; mt < n_thin_shared; mt += 64 * WAVES) thins[mt] = dx_tile_row{l.E, mt, l.T, shared0};
    for (int mt = tid; mt < n_shared; mt += 64 * WAVES) rows[total[0] + mt] = dx_tile_row{l.E, mt, T_shared - lead_shared, shared0 + lead_shared};
    for (int mt = tid; mt < n_big_shared; mt += 64 * WAVES) big[total[3] + mt] = dx_tile_row{l.E, mt, lead_shared, shared0};
    if (tid == 0) *l.tiles = dx_tile_head{total[0], n_shared, total[1], total[2], total[3], n_big_shared, total[4], total[5], n_thin_shared, l.n_cu};
}

} // namespace dx_tile_list
