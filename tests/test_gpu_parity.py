"""GPU parity: the HIP path, called through the C-ABI, against the CPU oracle
on the same seeded inputs.  Integer stages bit-exact; layer outputs within
rel-L2 1e-2 (the bar the build's target states); routing weights within 1e-5."""
import numpy as np
import pytest
import torch

from paper_2511_15015_amd import workloads as W
from paper_2511_15015_amd.workloads import WORKLOADS, bf16_bits_to_f32, f32_to_bf16_bits
from tests.bounds import assert_elementwise

pytestmark = pytest.mark.gpu

REL_L2_TOL = 1e-2
W_TOL = 1e-5


@pytest.fixture(scope="module")
def B():
    from paper_2511_15015_amd import binding
    binding.load()
    assert torch.cuda.is_available()
    return binding


@pytest.fixture(scope="module")
def LY():
    from paper_2511_15015_amd import layer
    return layer


def rel_l2(y_gpu_bits, y_ref):
    y = bf16_bits_to_f32(y_gpu_bits).astype(np.float64)
    return float(np.linalg.norm(y - y_ref) / max(np.linalg.norm(y_ref), 1e-300))


def sync():
    torch.cuda.synchronize()


# ------------------------------------------------------------------ quantizer
@pytest.mark.parametrize("rows,K,group", [(128, 256, 64), (768, 2048, 128), (2048, 768, 128), (37, 96, 32),
                                          (1, 128, 128), (5, 64, 64)])
def test_quantize_bit_exact(B, LY, dxo, rows, K, group):
    print(f"quantize rows={rows} K={K} group={group}", flush=True)
    g = np.random.default_rng(rows * 7 + K)
    w = 0.02 * g.standard_normal((rows, K)).astype(np.float32)
    w[0, :group] = 0.0                       # an all-zero group
    if rows > 2:
        w[1] *= 1e3
        w[2] *= 1e-4
    # exact .5 ties: scale 1 (absmax 7), values k + 0.5
    w[-1, :group] = 0.0
    w[-1, 0] = 7.0
    w[-1, 1:9] = [0.5, 1.5, 2.5, 3.5, -0.5, -1.5, -2.5, -6.5]
    bits = f32_to_bf16_bits(w)
    q_ref, s_ref = dxo.quantize(bits, group)
    ctx = B.Context(L=1, E=4, d=128, f=128, top_k=2, group=group, max_tokens=4)
    wd = LY.bits_to_device(bits)
    q = torch.empty((rows, K // 2), dtype=torch.uint8, device="cuda")
    s = torch.empty((rows, K // group), dtype=torch.bfloat16, device="cuda")
    ctx.dx_quantize_expert(wd, rows, K, group, q, s)
    sync()
    assert np.array_equal(LY.device_to_bits(s), s_ref)
    assert np.array_equal(q.cpu().numpy(), q_ref)
    ctx.close()


@pytest.mark.parametrize("bits", [4, 2])
def test_quantize_exact_ties_and_extreme_scales(B, LY, dxo, bits):
    """Rows built to sit on the quantizer's rounding ties: the group scale is a power of two (absmax = q_max *
    2^k) and the other values are multiples of half a step, so about half of them are exact ties that must go
    to the even code; scales with other mantissas mixed in; groups with tiny and huge scales (the kernel's
    divide shortcut does not cover those) and an all-zero group.  Codes and scales bit for bit."""
    group, rows, K = 128, 96, 1024
    g = np.random.default_rng(1234 + bits)
    q_max = 7 if bits == 4 else 1
    w = np.zeros((rows, K), np.float32)
    for r in range(rows):
        for c0 in range(0, K, group):
            kind = (r + c0 // group) % 6
            if kind == 0:                                   # step 2^k: every multiple of step/2 in range
                step = 2.0 ** int(g.integers(-12, 3))
                vals = g.integers(-2 * q_max, 2 * q_max + 1, group) * (step / 2)
            elif kind == 1:                                 # step 1.5 * 2^k: ties at odd multiples of 0.75 * 2^k
                step = 1.5 * 2.0 ** int(g.integers(-10, 2))
                vals = g.integers(-2 * q_max, 2 * q_max + 1, group) * (step / 2)
            elif kind == 2:                                 # tiny scale (below the shortcut's range)
                step = 2.0 ** -110
                vals = g.integers(-2 * q_max, 2 * q_max + 1, group) * (step / 2)
            elif kind == 3:                                 # huge scale
                step = 2.0 ** 105
                vals = g.integers(-2 * q_max, 2 * q_max + 1, group) * (step / 2)
            elif kind == 4:                                 # ordinary weights
                step = None
                vals = 0.02 * g.standard_normal(group)
            else:
                step = None
                vals = np.zeros(group)
            vals = np.asarray(vals, np.float64)
            if step is not None:
                vals[0] = q_max * step                      # pins absmax, hence the scale
            w[r, c0:c0 + group] = vals
    bits_in = f32_to_bf16_bits(w)
    quant = dxo.quantize if bits == 4 else dxo.quantize2
    q_ref, s_ref = quant(bits_in, group)
    # the rows really are full of ties: the oracle's codes differ from rounding half away from zero
    wf = bf16_bits_to_f32(bits_in).astype(np.float64)
    sf = np.repeat(bf16_bits_to_f32(s_ref).astype(np.float64), group, axis=1)
    with np.errstate(divide="ignore", invalid="ignore"):
        frac = np.where(sf > 0, np.abs(wf / sf) % 1.0, 0.0)
    assert np.count_nonzero(frac == 0.5) > rows * K // 8
    ctx = B.Context(L=1, E=4, d=128, f=128, top_k=2, group=group, max_tokens=4)
    q = torch.empty((rows, K // (8 // bits)), dtype=torch.uint8, device="cuda")
    s = torch.empty((rows, K // group), dtype=torch.bfloat16, device="cuda")
    (ctx.dx_quantize_expert if bits == 4 else ctx.dx_quantize_expert_int2)(LY.bits_to_device(bits_in), rows, K, group, q, s)
    sync()
    assert np.array_equal(LY.device_to_bits(s), s_ref)
    bad = np.argwhere(q.cpu().numpy() != q_ref)
    assert len(bad) == 0, bad[:5]
    ctx.close()


def test_quantize_rejects_bad_arguments(B):
    ctx = B.Context(L=1, E=4, d=128, f=128, top_k=2, group=64, max_tokens=4)
    buf = torch.zeros(4096, dtype=torch.uint8, device="cuda")
    with pytest.raises(B.DxError) as ei:
        ctx.dx_quantize_expert(buf, 2, 96, 64, buf, buf)          # K % group != 0
    assert ei.value.status == B.DX_ERR_INVALID
    with pytest.raises(B.DxError):
        ctx.dx_quantize_expert(buf, 2, 128, 48, buf, buf)         # unsupported group
    with pytest.raises(B.DxError):
        ctx.dx_quantize_expert(None, 2, 128, 64, buf, buf)        # null pointer
    ctx.dx_quantize_expert(buf, 0, 128, 64, buf, buf)             # empty is fine
    ctx.close()


# -------------------------------------------------------------------- routing
def _check_route(B, LY, dxo, logits, k, max_tokens=None):
    T, E = logits.shape
    ctx = B.Context(L=1, E=E, d=64, f=64, top_k=k, group=32, max_tokens=max(max_tokens or T, 1))
    rb = LY.RoutingBuffers(max(T, 1), E, k)
    dl = torch.from_numpy(logits).cuda() if T else torch.empty((1, E), dtype=torch.float32, device="cuda")
    rb.route(ctx, 0, dl, T)
    sync()
    ids_r, w_r, counts_r, offsets_r, perm_r = dxo.route(logits, k)
    assert np.array_equal(rb.counts.cpu().numpy(), counts_r)
    assert np.array_equal(rb.offsets.cpu().numpy(), offsets_r)
    if T:
        assert np.array_equal(rb.ids.cpu().numpy()[:T], ids_r)
        assert np.array_equal(rb.perm.cpu().numpy()[:T * k], perm_r)
        wg = rb.w.cpu().numpy()[:T].astype(np.float64)
        assert np.max(np.abs(wg - w_r) / np.maximum(w_r, 1e-30)) < W_TOL or np.max(np.abs(wg - w_r)) < 1e-7
    ctx.close()


@pytest.mark.parametrize("name", ["C1", "C2", "C3", "C4"])
def test_route_workloads_bit_exact(B, LY, dxo, name):
    wl = WORKLOADS[name]
    print(f"route {name} T={wl.T} E={wl.E} k={wl.k}", flush=True)
    _, logits = W.layer_inputs(wl, seed=0)
    _check_route(B, LY, dxo, logits, wl.k)


@pytest.mark.parametrize("T,E,k", [(0, 8, 2), (1, 8, 2), (63, 16, 4), (64, 16, 4), (65, 16, 4), (130, 200, 6),
                                   (1000, 1024, 3), (5, 8, 8), (3, 1, 1), (257, 64, 64)])
def test_route_edge_shapes_and_ties(B, LY, dxo, T, E, k):
    print(f"route T={T} E={E} k={k}", flush=True)
    g = np.random.default_rng(T * 31 + E)
    # logits on a coarse grid: many exact ties, both signs of zero
    logits = np.round(g.standard_normal((T, E)) * 2).astype(np.float32) / 2
    logits[logits == 0] *= np.where(g.random(np.count_nonzero(logits == 0)) < 0.5, -1.0, 1.0).astype(np.float32)
    _check_route(B, LY, dxo, logits, k)


@pytest.mark.parametrize("T,E,k,coarse", [
    # large batches, the chunks' sums in groups of 32: 72 chunks, the third group of eight, the selection of a token per
    # wavefront; 161 chunks, the sixth group of one, an expert's sums over four threads; 1734 chunks on 64 threads
    (4580, 1000, 17, False), (10304, 130, 2, True), (110930, 1, 1, False),
    (4544, 1000, 3, True),     # 71 chunks: the last size without
    (65, 1, 1, False), (130, 3, 2, True),          # 64 threads per expert in the placement, more than there are chunks
    (1300, 600, 3, True), (1400, 1024, 5, False),  # one thread per expert, more chunks than loads in flight
    (2000, 129, 16, True), (700, 512, 10, False),  # wide layers: the threshold and, on a coarse grid, its fall-back
    (64, 512, 10, False), (40, 200, 16, True),     # the same in a single chunk
])
def test_route_chunks_and_wide_selection(B, LY, dxo, T, E, k, coarse):
    """The placement's thread splits at both ends of the expert count, and the chunk kernel's selection for layers of more
    than 128 experts: ids, weights, counts, offsets and permutation as the oracle has them."""
    g = np.random.default_rng(T + E)
    logits = g.standard_normal((T, E)).astype(np.float32)
    if coarse:
        logits = np.round(logits * 2) / 2
    _check_route(B, LY, dxo, logits, k)


@pytest.mark.parametrize("T,E,k", [(79, 128, 8), (80, 16, 2), (81, 512, 10), (113, 300, 4), (575, 128, 17), (128, 1024, 9)])
def test_route_quarters_of_a_chunk(B, LY, dxo, T, E, k):
    """Several chunks, 16 tokens to a block: last quarters that are full, begun and empty, for every kind of selection."""
    logits = np.random.default_rng(T * E).standard_normal((T, E)).astype(np.float32)
    _check_route(B, LY, dxo, logits, k)


def test_route_rejects_bad_arguments(B, LY):
    ctx = B.Context(L=2, E=8, d=64, f=64, top_k=2, group=32, max_tokens=16)
    rb = LY.RoutingBuffers(16, 8, 2)
    lg = torch.zeros((16, 8), dtype=torch.float32, device="cuda")
    for layer, T in [(2, 4), (-1, 4), (0, 17), (0, -1)]:
        with pytest.raises(B.DxError) as ei:
            ctx.dx_route(layer, lg, T, rb.ids, rb.w, rb.counts, rb.offsets, rb.perm)
        assert ei.value.status == B.DX_ERR_INVALID
    with pytest.raises(B.DxError):
        ctx.dx_route(0, None, 4, rb.ids, rb.w, rb.counts, rb.offsets, rb.perm)
    for bad in [dict(E=0), dict(top_k=9), dict(group=48), dict(d=100), dict(max_tokens=0), dict(alpha_q16=65536)]:
        kw = dict(L=1, E=8, d=64, f=64, top_k=2, group=32, max_tokens=4)
        kw.update(bad)
        with pytest.raises(B.DxError):
            B.Context(**kw)
    ctx.close()


@pytest.mark.parametrize("T,E,d,with_bias", [(32, 128, 2048, True), (1, 8, 64, False), (33, 40, 96, True),
                                             (4096, 128, 2048, True), (70, 512, 2048, False)])
def test_router_logits_match_oracle(B, LY, dxo, T, E, d, with_bias):
    """The router gate on the matrix cores against the fp64 oracle: fp32 accumulation of exact bf16
    products, so the difference stays near d * 2^-24 of the largest partial sum."""
    g = np.random.default_rng(T + E)
    x = W.f32_to_bf16_bits(g.standard_normal((T, d)).astype(np.float32))
    wr = W.f32_to_bf16_bits((0.02 * g.standard_normal((E, d))).astype(np.float32))
    bias = (g.standard_normal(E) * 3).astype(np.float32) if with_bias else None
    ctx = B.Context(L=1, E=E, d=d, f=64, top_k=2, group=32, max_tokens=T)
    out = torch.full((T, E), float("nan"), dtype=torch.float32, device="cuda")
    ctx.dx_router_logits(LY.bits_to_device(x), LY.bits_to_device(wr),
                         torch.from_numpy(bias).cuda() if with_bias else None, T, out)
    sync()
    ref = dxo.router_logits(x, wr, bias)
    got = out.cpu().numpy()
    assert np.isfinite(got).all()
    scale = float(np.abs(ref).max())
    assert np.abs(got - ref).max() <= 2e-5 * max(scale, 1.0), np.abs(got - ref).max()
    with pytest.raises(B.DxError):
        ctx.dx_router_logits(LY.bits_to_device(x), LY.bits_to_device(wr), None, T + 1, out)
    ctx.close()


@pytest.mark.parametrize("T,E,d,with_bias", [
    (20, 20, 32, False),      # 16 x 16 tiles, half a line, more wavefronts than lines
    (16, 16, 2080, True),     # an odd number of lines per wavefront and half a line at the end
    (4097, 17, 64, True),     # 32 x 32 tiles, remainders of one, the XCD order with padded row tiles
    (1000, 500, 96, True),    # 32 x 64 tiles
    (2049, 500, 160, False),  # 64 x 64 tiles
])
def test_router_logits_tile_edges(B, LY, dxo, T, E, d, with_bias):
    """Every tile of the router gate at remainders of rows, columns and K.  Bound per element: fp32 sums of d exact
    products, each addition at most 2^-24 of the sum of the magnitudes."""
    g = np.random.default_rng(T * E + d)
    x = W.f32_to_bf16_bits(g.standard_normal((T, d)).astype(np.float32))
    wr = W.f32_to_bf16_bits((0.02 * g.standard_normal((E, d))).astype(np.float32))
    bias = (g.standard_normal(E) * 3).astype(np.float32) if with_bias else None
    ctx = B.Context(L=1, E=E, d=d, f=64, top_k=2, group=32, max_tokens=T)
    out = torch.full((T, E), float("nan"), dtype=torch.float32, device="cuda")
    ctx.dx_router_logits(LY.bits_to_device(x), LY.bits_to_device(wr),
                         torch.from_numpy(bias).cuda() if with_bias else None, T, out)
    sync()
    ref = dxo.router_logits(x, wr, bias)
    mag = np.abs(W.bf16_bits_to_f32(x)).astype(np.float64) @ np.abs(W.bf16_bits_to_f32(wr)).astype(np.float64).T
    if with_bias:
        mag = mag + np.abs(bias)[None, :]
    assert (np.abs(out.cpu().numpy() - ref) <= (d + 1) * 2.0 ** -24 * mag).all()
    ctx.close()


# ------------------------------------------------------------------ the layer
class Layer:
    """One layer set up on both sides from the same master bits."""

    def __init__(self, B, LY, dxo, wl, resident, seed=0, layer=0, masters=None, T=None, shared=None):
        self.wl, self.B = wl, B
        T = wl.T if T is None else T
        self.T = T
        self.masters = masters if masters is not None else W.layer_masters(wl, seed, layer)
        wg, wu, wd = self.masters
        self.ctx = B.Context(L=1, E=wl.E, d=wl.d, f=wl.f, top_k=wl.k, group=wl.group, max_tokens=max(T, 1),
                             shared_f=wl.shared_f if shared is not None else 0)
        self.dev = [LY.bits_to_device(m) for m in self.masters]
        self.lw = LY.LayerWeights(self.ctx, 0, *self.dev, resident, wl.group)
        self.rb = LY.RoutingBuffers(max(T, 1), wl.E, wl.k)
        self.resident = set(int(e) for e in resident)
        self.versions = [dxo.ExpertVersion.bf16(wg[e], wu[e], wd[e]) if e in self.resident
                         else dxo.ExpertVersion.int4_from_master(wg[e], wu[e], wd[e], wl.group)
                         for e in range(wl.E)]
        self.shared = None
        if shared is not None:
            self.shared_dev = [LY.bits_to_device(m) for m in shared]
            self.ctx.dx_swap_handle(0, wl.E, B.make_handle(B.DX_FMT_BF16, *self.shared_dev))
            self.shared = dxo.ExpertVersion.bf16(*shared)
        self.LY, self.dxo = LY, dxo

    def run(self, x_bits, logits, tokens=None):
        T = x_bits.shape[0]
        xd = self.LY.bits_to_device(x_bits)
        ld = torch.from_numpy(logits).cuda()
        y = torch.empty((T, self.wl.d), dtype=torch.bfloat16, device="cuda")
        self.rb.route(self.ctx, 0, ld, T)
        self.rb.forward(self.ctx, 0, xd, y, None, T)
        sync()
        ids, w, counts, offsets, perm = self.dxo.route(logits, self.wl.k)
        assert np.array_equal(self.rb.ids.cpu().numpy()[:T], ids)
        y_ref = self.dxo.moe_forward(self.versions, self.wl.d, self.wl.f, self.wl.group, x_bits, ids, w,
                                     shared=self.shared, shared_f=self.wl.shared_f if self.shared else 0,
                                     tokens=tokens)
        y_gpu = self.LY.device_to_bits(y)
        if tokens is not None:
            y_gpu = y_gpu[np.asarray(tokens)]
        # next to the norm the caller checks: every element within the bound the bf16 roundings of H, O and y allow
        used = assert_elementwise(self.dxo, y_gpu, y_ref, self.versions, self.wl.group, x_bits, ids, w, shared=self.shared,
                                  tokens=tokens, T_call=T)
        print(f"  element-wise: largest error = {used:.2f} of its bound", flush=True)
        return y_gpu, y_ref


def test_forward_c1_mixed_all_hi_all_lo(B, LY, dxo):
    wl = WORKLOADS["C1"]
    x, logits = W.layer_inputs(wl, seed=0)
    masters = W.layer_masters(wl, 0, 0)
    for resident in ([1, 6], list(range(wl.E)), []):
        print(f"forward C1 resident={resident}", flush=True)
        ly = Layer(B, LY, dxo, wl, resident, masters=masters)
        y_gpu, y_ref = ly.run(x, logits)
        err = rel_l2(y_gpu, y_ref)
        print("  rel-L2", err, flush=True)
        assert err <= REL_L2_TOL
        ly.ctx.close()


@pytest.mark.parametrize("shift", [16, 80, 112])
def test_forward_weights_that_start_inside_a_line(B, LY, dxo, shift):
    """The boundary promises 16-byte alignment only.  The decode kernels fetch weights in pieces that are whole
    128-byte lines when a matrix starts on a line; here every matrix and scale array of every expert starts
    `shift` bytes into one (bf16 and int4 versions, d = 2048 so that the line-shaped loads are the ones that
    run): same bits as with the aligned copies, and the oracle's values."""
    import dataclasses
    wl = dataclasses.replace(WORKLOADS["C1"], T=24, E=8, k=3, d=2048, f=128, group=128)
    print(f"weights shifted by {shift} bytes", flush=True)
    x, logits = W.layer_inputs(wl, seed=41)
    ly = Layer(B, LY, dxo, wl, [1, 4, 6], seed=41)
    y_gpu, y_ref = ly.run(x, logits)
    assert rel_l2(y_gpu, y_ref) <= REL_L2_TOL
    keep = []

    def moved(t):
        n = t.numel() * t.element_size()
        raw = torch.zeros(n + 256, dtype=torch.uint8, device=t.device)
        base = (-raw.data_ptr()) % 128 + shift                      # `shift` bytes past a line boundary
        v = raw[base:base + n].view(t.dtype).view(t.shape)
        v.copy_(t)
        assert v.data_ptr() % 128 == shift % 128 and v.data_ptr() % 16 == 0
        keep.append(raw)
        return v

    lw = ly.lw
    for e in range(wl.E):
        if lw.is_hi[e]:
            h = B.make_handle(B.DX_FMT_BF16, *(moved(m[e]) for m in lw.hi))
        else:
            i = lw.lo_slot[e]
            h = B.make_handle(B.DX_FMT_INT4G, *(moved(q[i]) for q in lw.q), *(moved(sc[i]) for sc in lw.s))
        ly.ctx.dx_swap_handle(0, e, h)
    y_moved, _ = ly.run(x, logits)
    assert np.array_equal(y_moved, y_gpu)
    ly.ctx.close()


@pytest.mark.parametrize("T", [1, 7, 16, 17, 33, 40])
def test_forward_ragged_token_counts(B, LY, dxo, T):
    import dataclasses
    wl = dataclasses.replace(WORKLOADS["C1"], T=T, E=4, k=2)   # few experts: segments longer than one 16-row tile
    print(f"forward ragged T={T}", flush=True)
    x, logits = W.layer_inputs(wl, seed=3)
    ly = Layer(B, LY, dxo, wl, [0, 2], seed=3)
    y_gpu, y_ref = ly.run(x, logits)
    assert rel_l2(y_gpu, y_ref) <= REL_L2_TOL
    # per-token check as well: no token may be far off
    yg = bf16_bits_to_f32(y_gpu).astype(np.float64)
    tok = np.linalg.norm(yg - y_ref, axis=1) / np.linalg.norm(y_ref, axis=1)
    assert tok.max() <= 2 * REL_L2_TOL
    ly.ctx.close()


def test_forward_group32(B, LY, dxo):
    import dataclasses
    wl = dataclasses.replace(WORKLOADS["C1"], group=32, T=9)
    x, logits = W.layer_inputs(wl, seed=4)
    ly = Layer(B, LY, dxo, wl, [3], seed=4)
    y_gpu, y_ref = ly.run(x, logits)
    assert rel_l2(y_gpu, y_ref) <= REL_L2_TOL
    ly.ctx.close()


def test_forward_c2_decode_full(B, LY, dxo):
    """The 30B-shaped decode layer at full size; resident set = top-32 by the oracle's window counts."""
    wl = WORKLOADS["C2"]
    print("forward C2: drawing masters", flush=True)
    masters = W.layer_masters(wl, 0, 0)
    x, logits = W.layer_inputs(wl, seed=0)
    # hotness from a warm-up window of routing only (oracle side decides the set for both)
    c = np.zeros(wl.E, np.int64)
    for step in range(1, 9):
        _, lg = W.layer_inputs(wl, seed=0, step=step)
        _, _, counts, _, _ = dxo.route(lg, wl.k)
        dxo.hotness_update(c, counts)
    S = np.zeros(wl.E, np.uint64)
    dxo.window_end(S, c, 0)
    resident = dxo.select_topn(S, wl.n_hi)
    print("forward C2: running", flush=True)
    ly = Layer(B, LY, dxo, wl, resident, masters=masters)
    y_gpu, y_ref = ly.run(x, logits)
    err = rel_l2(y_gpu, y_ref)
    print("  C2 rel-L2", err, flush=True)
    assert err <= REL_L2_TOL
    ly.ctx.close()


def test_forward_with_shared_expert(B, LY, dxo):
    import dataclasses
    wl = dataclasses.replace(WORKLOADS["C4"], L=1, E=16, k=4, T=19, d=256, f=128, shared_f=256, group=128)
    x, logits = W.layer_inputs(wl, seed=5)
    shared = W.shared_master(wl, 5, 0)
    ly = Layer(B, LY, dxo, wl, [0, 5, 9], seed=5, shared=shared)
    y_gpu, y_ref = ly.run(x, logits)
    err = rel_l2(y_gpu, y_ref)
    print("  shared rel-L2", err, flush=True)
    assert err <= REL_L2_TOL
    ly.ctx.close()


def test_forward_empty_batch_and_bad_arguments(B, LY, dxo):
    wl = WORKLOADS["C1"]
    ly = Layer(B, LY, dxo, wl, [0])
    y = torch.zeros((wl.T, wl.d), dtype=torch.bfloat16, device="cuda")
    x = torch.zeros((wl.T, wl.d), dtype=torch.bfloat16, device="cuda")
    ly.rb.forward(ly.ctx, 0, x, y, None, 0)                      # T = 0: nothing to do
    with pytest.raises(B.DxError):
        ly.rb.forward(ly.ctx, 0, None, y, None, 4)
    with pytest.raises(B.DxError):
        ly.rb.forward(ly.ctx, 1, x, y, None, 4)
    with pytest.raises(B.DxError):
        ly.rb.forward(ly.ctx, 0, x, y, None, wl.T + 1)
    ly.ctx.close()
    # a context whose experts were never published refuses to run
    ctx = B.Context(L=1, E=wl.E, d=wl.d, f=wl.f, top_k=wl.k, group=wl.group, max_tokens=wl.T)
    rb = LY.RoutingBuffers(wl.T, wl.E, wl.k)
    with pytest.raises(B.DxError):
        rb.forward(ctx, 0, x, y, None, 4)
    ctx.close()


# ---------------------------------------------------------- swap / publication
def test_swap_handle_takes_effect_between_forward_passes(B, LY, dxo):
    wl = WORKLOADS["C1"]
    x, logits = W.layer_inputs(wl, seed=0)
    masters = W.layer_masters(wl, 0, 0)
    ly = Layer(B, LY, dxo, wl, [], masters=masters)              # all int4
    y_gpu0, y_ref0 = ly.run(x, logits)
    assert rel_l2(y_gpu0, y_ref0) <= REL_L2_TOL
    fm = ly.ctx.dx_get_formats()
    assert np.all(fm == B.DX_FMT_INT4G)
    # publish bf16 versions of every expert, straight from the master tensors
    v0 = ly.ctx.dx_get_handle(0, 3).version
    for e in range(wl.E):
        ly.ctx.dx_swap_handle(0, e, B.make_handle(B.DX_FMT_BF16, ly.dev[0][e], ly.dev[1][e], ly.dev[2][e]))
    assert ly.ctx.dx_get_handle(0, 3).version == v0 + 1
    assert np.all(ly.ctx.dx_get_formats() == B.DX_FMT_BF16)
    ly.versions = [dxo.ExpertVersion.bf16(masters[0][e], masters[1][e], masters[2][e]) for e in range(wl.E)]
    y_gpu1, y_ref1 = ly.run(x, logits)
    assert rel_l2(y_gpu1, y_ref1) <= REL_L2_TOL
    assert rel_l2(y_gpu1, y_ref0) > rel_l2(y_gpu1, y_ref1)       # it really switched versions
    # a version whose producer has not finished is refused
    ev = torch.cuda.Event()
    side = torch.cuda.Stream()
    big = torch.empty(1 << 28, dtype=torch.float32, device="cuda")
    with torch.cuda.stream(side):
        for _ in range(20):
            big.add_(1.0)
        ev.record(side)
    with pytest.raises(B.DxError) as ei:
        ly.ctx.dx_swap_handle(0, 0, ly.lw.handle(0, B.DX_FMT_INT4G), producer_event=ev.cuda_event)
    assert ei.value.status == B.DX_ERR_BUSY
    ev.synchronize()
    ly.ctx.dx_swap_handle(0, 0, ly.lw.handle(0, B.DX_FMT_INT4G), producer_event=ev.cuda_event)
    assert ly.ctx.dx_get_formats()[0, 0] == B.DX_FMT_INT4G
    with pytest.raises(B.DxError):
        ly.ctx.dx_swap_handle(0, wl.E, ly.lw.handle(0, B.DX_FMT_INT4G))   # no shared expert configured
    ly.ctx.close()


# ------------------------------------------------------- hotness and selection
def test_hotness_window_and_selection_match_oracle(B, LY, dxo):
    wl = WORKLOADS["C2"]
    L = 3
    b_hi, b_lo = dxo.expert_bytes(wl.d, wl.f, wl.group, 0), dxo.expert_bytes(wl.d, wl.f, wl.group, 1)
    ctx = B.Context(L=L, E=wl.E, d=wl.d, f=wl.f, top_k=wl.k, group=wl.group, max_tokens=wl.T, alpha_q16=16384)
    rb = LY.RoutingBuffers(wl.T, wl.E, wl.k)
    c = np.zeros((L, wl.E), np.int64)
    S = np.zeros((L, wl.E), np.uint64)
    for window in range(3):
        for step in range(6):
            for layer in range(L):
                _, lg = W.layer_inputs(wl, seed=1, layer=layer, step=window * 6 + step)
                rb.route(ctx, layer, torch.from_numpy(lg).cuda())
                ctx.dx_hotness_update(layer, rb.counts)
                _, _, counts, _, _ = dxo.route(lg, wl.k)
                dxo.hotness_update(c[layer], counts)
        assert np.array_equal(ctx.dx_get_counters(), c)
        S_gpu = ctx.dx_window_end()
        for layer in range(L):
            dxo.window_end(S[layer], c[layer], 16384)
        assert np.array_equal(S_gpu, S)
        assert not ctx.dx_get_counters().any()
        for layer in range(L):
            budget = 535560192
            ids = ctx.dx_select_resident(layer, budget)
            n = dxo.budget_capacity(budget, wl.E, b_hi, b_lo)
            assert n == 32 and np.array_equal(ids, dxo.select_topn(S[layer], n))
            assert len(ids) * b_hi + (wl.E - len(ids)) * b_lo <= budget
    with pytest.raises(B.DxError) as ei:
        ctx.dx_select_resident(0, wl.E * b_lo - 1)
    assert ei.value.status == B.DX_ERR_BUDGET
    ctx.close()


def test_route_can_update_hotness_itself(B, LY, dxo):
    wl = WORKLOADS["C2"]
    for T in (wl.T, 200):                       # single-chunk and multi-chunk routing paths
        ctx = B.Context(L=2, E=wl.E, d=wl.d, f=wl.f, top_k=wl.k, group=wl.group, max_tokens=T,
                        route_updates_hotness=True)
        rb = LY.RoutingBuffers(T, wl.E, wl.k)
        c = np.zeros((2, wl.E), np.int64)
        g = np.random.default_rng(T)
        for step in range(5):
            for layer in range(2):
                lg = g.standard_normal((T, wl.E)).astype(np.float32)
                rb.route(ctx, layer, torch.from_numpy(lg).cuda())
                _, _, counts, _, _ = dxo.route(lg, wl.k)
                dxo.hotness_update(c[layer], counts)
        assert np.array_equal(ctx.dx_get_counters(), c)
        ctx.close()


# ------------------------------------------------------- prefill-sized batches
@pytest.mark.parametrize("T,E,k,resident", [(65, 4, 2, [0, 2]), (128, 4, 2, [0, 2]), (200, 4, 2, [1]), (300, 8, 3, [0, 5, 6]),
                                            (129, 2, 2, [0]), (400, 4, 1, []),
                                            # segments of several row tiles
                                            (700, 4, 2, [0, 2]), (1100, 2, 2, [0, 1]), (512, 2, 2, [1]),
                                            (256, 1, 1, [0]),
                                            # one bf16 expert with 200, 385 = 3 * 128 + 1, 384 = 3 * 128 rows; two with 641
                                            (200, 1, 1, [0]), (385, 1, 1, [0]), (384, 1, 1, [0]), (641, 2, 2, [0, 1])])
def test_forward_prefill_tiles_small_shapes(B, LY, dxo, T, E, k, resident):
    """Up to 128 tokens per call the streaming kernels walk each segment in blocks of 32 tokens; above,
    segments of more than 32 tokens take 128-row tiles (bf16 and int4), the others thin
    tiles; ragged row tiles; every token checked."""
    import dataclasses
    wl = dataclasses.replace(WORKLOADS["C1"], T=T, E=E, k=k)
    print(f"prefill tiles T={T} E={E} k={k} resident={resident}", flush=True)
    x, logits = W.layer_inputs(wl, seed=6)
    ly = Layer(B, LY, dxo, wl, resident, seed=6)
    y_gpu, y_ref = ly.run(x, logits)
    err = rel_l2(y_gpu, y_ref)
    print("  rel-L2", err, flush=True)
    assert err <= REL_L2_TOL
    yg = bf16_bits_to_f32(y_gpu).astype(np.float64)
    tok = np.linalg.norm(yg - y_ref, axis=1) / np.linalg.norm(y_ref, axis=1)
    assert tok.max() <= 2 * REL_L2_TOL
    ly.ctx.close()


@pytest.mark.parametrize("T,E,k,d,f,group,resident", [
    (600, 2, 2, 256, 128, 32, []),          # both experts int4 with 600 rows: four row tiles and a remainder each
    (1100, 2, 2, 256, 128, 64, []),         # nine tiles each, more than a band; the down contraction is two steps
    (520, 2, 1, 512, 256, 128, []),         # about 260 rows each: two tiles and a few rows
    (700, 4, 2, 512, 256, 128, [0]),        # bf16 and int4 tiles in one launch
    (768, 1, 1, 256, 384, 128, []),         # three groups per row of W_down
    (300, 1, 1, 2048, 768, 128, []),        # the 30B layer's K extents: 32 and 12 steps
])
def test_forward_prefill_int4_segments_of_256_rows_and_more(B, LY, dxo, T, E, k, d, f, group, resident):
    """int4 experts of several row tiles, whose codes the tile kernel expands into its LDS stages; every token, and the same
    bits on a second run.  (The 256-row tiles of larger batches: test_forward_prefill_256_row_tiles.)"""
    import dataclasses
    wl = dataclasses.replace(WORKLOADS["C1"], T=T, E=E, k=k, d=d, f=f, group=group)
    print(f"prefill int4 tiles T={T} E={E} k={k} d={d} f={f} g={group} resident={resident}", flush=True)
    x, logits = W.layer_inputs(wl, seed=31)
    ly = Layer(B, LY, dxo, wl, resident, seed=31)
    y_gpu, y_ref = ly.run(x, logits)
    err = rel_l2(y_gpu, y_ref)
    print("  rel-L2", err, flush=True)
    assert err <= REL_L2_TOL
    yg = bf16_bits_to_f32(y_gpu).astype(np.float64)
    tok = np.linalg.norm(yg - y_ref, axis=1) / np.linalg.norm(y_ref, axis=1)
    assert tok.max() <= 2 * REL_L2_TOL
    again, _ = ly.run(x, logits)
    assert np.array_equal(again, y_gpu)
    ly.ctx.close()


@pytest.mark.parametrize("pair,T,E,k,d,f,group,shared_f", [
    ("bf16-int4", 150, 2, 1, 128, 64, 64, 0),      # one K step of 64 in the down projection; one group per row of W_down
    ("bf16-int4", 150, 2, 1, 128, 64, 32, 0),      # the same with the step's two groups in a word
    ("int4-int2", 150, 2, 1, 128, 64, 64, 0),
    ("bf16-int4", 300, 3, 2, 256, 192, 64, 0),     # three steps and three groups per row, half a column tile in gate/up
    ("int4-int2", 300, 3, 2, 256, 192, 64, 0),
    ("bf16-int4", 300, 3, 2, 256, 192, 32, 0),
    ("bf16-int4", 270, 2, 2, 384, 320, 64, 0),     # five steps
    ("int4-int2", 270, 2, 2, 256, 384, 128, 0),    # three groups of 128 per row: the scale's half by row parity
    ("bf16-int4", 270, 2, 2, 256, 384, 128, 0),
    ("bf16-int4", 200, 2, 1, 128, 128, 64, 192),   # the shared expert with another, odd number of steps
    ("bf16-int4", 200, 2, 1, 128, 192, 64, 64),
])
def test_forward_prefill_tiles_k_steps_and_groups(B, LY, dxo, pair, T, E, k, d, f, group, shared_f):
    """The 128-row tile kernel at one, an odd and an even number of K steps with every format, and at odd numbers of groups
    per row: every token against the oracle."""
    import dataclasses
    wl = dataclasses.replace(WORKLOADS["C1"], T=T, E=E, k=k, d=d, f=f, group=group, shared_f=shared_f)
    x, logits = W.layer_inputs(wl, seed=73)
    shared = None
    if pair == "int4-int2":
        ctx, keep, versions = _quant_pair_layer(B, LY, dxo, wl, [0], 73, T)
    else:
        masters = W.shared_master(wl, 73, 0) if shared_f else None
        ly = Layer(B, LY, dxo, wl, [0], seed=73, shared=masters)
        ctx, keep, versions, shared = ly.ctx, ly, ly.versions, ly.shared
    ids, w, counts, offsets, perm = dxo.route(logits, k)
    assert (counts[1:] > 32).any(), "some quantized expert has to take the tiles"
    rb = LY.RoutingBuffers(T, E, k)
    y = torch.full((T, d), float("nan"), dtype=torch.bfloat16, device="cuda")
    rb.route_forward(ctx, 0, torch.from_numpy(logits).cuda(), LY.bits_to_device(x), y)
    sync()
    assert np.array_equal(rb.perm.cpu().numpy(), perm)
    y_ref = dxo.moe_forward(versions, d, f, group, x, ids, w, shared=shared, shared_f=shared_f if shared else 0)
    yg = bf16_bits_to_f32(LY.device_to_bits(y)).astype(np.float64)
    tok = np.linalg.norm(yg - y_ref, axis=1) / np.linalg.norm(y_ref, axis=1)
    assert rel_l2(LY.device_to_bits(y), y_ref) <= REL_L2_TOL and tok.max() <= 2 * REL_L2_TOL
    del keep
    ctx.close()


@pytest.mark.parametrize("pair,T,E,k,d,f,group,hi", [
    # gate/up: 40.5 column tiles, 2 K steps; then 82 column tiles, 6 steps and an odd number of groups per row
    ("bf16-int4", 320, 4, 2, 128, 5184, 64, [1]),
    ("bf16-int4", 170, 5, 2, 384, 10496, 128, [0, 2]),
    ("int4-int2", 320, 4, 2, 128, 5184, 64, [1]),
    ("int4-int2", 320, 4, 2, 128, 7168, 128, [0, 3]),
    # down: 40.5 column tiles, one and three K steps
    ("bf16-int4", 320, 4, 2, 10368, 64, 32, [1]),
    ("bf16-int4", 320, 4, 2, 10368, 192, 64, [1]),
    ("int4-int2", 320, 4, 2, 10368, 192, 64, [1]),
    # nearly all bf16
    ("bf16-int4", 700, 3, 2, 256, 8256, 64, [0, 1, 2]),
])
def test_forward_prefill_wide_tiles(B, LY, dxo, pair, T, E, k, d, f, group, hi):
    """The 256-column tiles of calls with many tiles, every format: every seventh token against the oracle."""
    import dataclasses
    wl = dataclasses.replace(WORKLOADS["C1"], T=T, E=E, k=k, d=d, f=f, group=group)
    print(f"wide tiles {pair} T={T} E={E} k={k} d={d} f={f} group={group}", flush=True)
    x, logits = W.layer_inputs(wl, seed=13)
    ids, w, counts, offsets, perm = dxo.route(logits, k)
    assert _wide_phases(counts, hi, f, d, T, hi_quantized=pair == "int4-int2") == (f > d, d > f)
    if pair == "int4-int2":
        ctx, keep, versions = _quant_pair_layer(B, LY, dxo, wl, hi, 13, T)
    else:
        keep = Layer(B, LY, dxo, wl, hi, seed=13)
        ctx, versions = keep.ctx, keep.versions
    rb = LY.RoutingBuffers(T, E, k)
    y = torch.full((T, d), float("nan"), dtype=torch.bfloat16, device="cuda")
    rb.route_forward(ctx, 0, torch.from_numpy(logits).cuda(), LY.bits_to_device(x), y)
    sync()
    tokens = np.unique(np.append(np.arange(0, T, 7), T - 1))
    y_ref = dxo.moe_forward(versions, d, f, group, x, ids, w, tokens=tokens)
    bits = LY.device_to_bits(y)
    assert np.isfinite(bf16_bits_to_f32(bits)).all()
    assert rel_l2(bits[tokens], y_ref) <= REL_L2_TOL
    used = assert_elementwise(dxo, bits[tokens], y_ref, versions, group, x, ids, w, tokens=tokens, T_call=T)
    print(f"  element-wise: largest error = {used:.2f} of its bound", flush=True)
    del keep
    ctx.close()


@pytest.mark.parametrize("pair,d,f,group", [
    ("bf16-int4", 128, 64, 32),     # two steps and one; a quarter and half of a tile's columns
    ("bf16-int4", 384, 320, 64),    # six steps and five, odd numbers of groups per row; 2.5 and 1.5 column tiles
    ("bf16-int4", 640, 384, 128),   # ten steps and six, five and three groups
    ("bf16-int4", 256, 448, 64),    # four steps and seven: bf16 tiles start at one of them each, and have four in flight
    ("bf16-int4", 512, 576, 64),    # eight and nine
    ("bf16-int4", 2048, 768, 128),  # the 30B layer's
    ("int4-int2", 384, 320, 64),
    ("int4-int2", 256, 128, 128),
    ("int4-int2", 2048, 768, 128),
])
def test_forward_prefill_thin_segments(B, LY, dxo, pair, d, f, group):
    """Segments of up to 32 rows in a call on tiles: none, 1, 16, 17, 31 and 32 rows and one above, in both formats, every token
    against the oracle; the list of tiles from the routing kernels and from the caller's arrays: the same bits."""
    import dataclasses
    sizes = [0, 1, 16, 17, 31, 32, 33]
    E, T = 2 * len(sizes), 2 * sum(sizes)
    wl = dataclasses.replace(WORKLOADS["C1"], T=T, E=E, k=1, d=d, f=f, group=group)
    x, _ = W.layer_inputs(wl, seed=17)
    logits = np.zeros((T, E), np.float32)
    logits[np.arange(T), np.random.default_rng(3).permutation(np.repeat(np.arange(E), np.repeat(sizes, 2)))] = 4.0
    hi = list(range(0, E, 2))
    print(f"thin segments {pair} d={d} f={f} group={group} T={T}", flush=True)
    if pair == "int4-int2":
        ctx, keep, versions = _quant_pair_layer(B, LY, dxo, wl, hi, 17, T)
    else:
        keep = Layer(B, LY, dxo, wl, hi, seed=17)
        ctx, versions = keep.ctx, keep.versions
    ids, w, counts, offsets, perm = dxo.route(logits, 1)
    assert counts.tolist() == np.repeat(sizes, 2).tolist()
    rb = LY.RoutingBuffers(T, E, 1)
    y = torch.full((T, d), float("nan"), dtype=torch.bfloat16, device="cuda")
    xd, ld = LY.bits_to_device(x), torch.from_numpy(logits).cuda()
    rb.route_forward(ctx, 0, ld, xd, y)
    y1 = torch.full_like(y, float("nan"))
    rb.route(ctx, 0, ld)
    rb.forward(ctx, 0, xd, y1)
    sync()
    y_ref = dxo.moe_forward(versions, d, f, group, x, ids, w)
    bits = LY.device_to_bits(y)
    assert np.array_equal(bits, LY.device_to_bits(y1))
    yg = bf16_bits_to_f32(bits).astype(np.float64)
    tok = np.linalg.norm(yg - y_ref, axis=1) / np.linalg.norm(y_ref, axis=1)
    assert rel_l2(bits, y_ref) <= REL_L2_TOL and tok.max() <= 2 * REL_L2_TOL
    assert_elementwise(dxo, bits, y_ref, versions, group, x, ids, w, T_call=T)
    del keep
    ctx.close()


@pytest.mark.parametrize("pair,d,f,group,shared_f", [
    ("bf16-int4", 2176, 192, 64, 0),    # 34 K steps and three; 1.5 and 8.5 column tiles
    ("bf16-int4", 2304, 256, 128, 384), # a shared expert of another width, in four row tiles
    ("bf16-int4", 2176, 64, 32, 64),
    ("int4-int2", 2176, 192, 64, 0),
    ("int4-int2", 2304, 256, 128, 0),
])
def test_forward_thin_tiles_alone(B, LY, dxo, pair, d, f, group, shared_f):
    """Calls of up to 128 tokens whose K the streaming kernels take in rounds, ragged segments (too few for thin tiles to fill the chip: the streaming
    kernels have them), with O in fp32: every token against the oracle; the same bits from one call and from two."""
    import dataclasses
    sizes = [1, 1, 32, 33, 0, 0, 20, 17, 3, 4]
    E, T = len(sizes), sum(sizes)
    wl = dataclasses.replace(WORKLOADS["C1"], T=T, E=E, k=1, d=d, f=f, group=group, shared_f=shared_f)
    x, _ = W.layer_inputs(wl, seed=19)
    logits = np.zeros((T, E), np.float32)
    logits[np.arange(T), np.random.default_rng(5).permutation(np.repeat(np.arange(E), sizes))] = 4.0
    hi = list(range(0, E, 2))
    print(f"thin tiles alone {pair} d={d} f={f} group={group} shared={shared_f} T={T}", flush=True)
    shared = None
    if pair == "int4-int2":
        ctx, keep, versions = _quant_pair_layer(B, LY, dxo, wl, hi, 19, T)
    else:
        keep = Layer(B, LY, dxo, wl, hi, seed=19, shared=W.shared_master(wl, 19, 0) if shared_f else None)
        ctx, versions, shared = keep.ctx, keep.versions, keep.shared
    ids, w, counts, offsets, perm = dxo.route(logits, 1)
    assert counts.tolist() == sizes and 64 < T <= 128
    rb = LY.RoutingBuffers(T, E, 1)
    xd, ld = LY.bits_to_device(x), torch.from_numpy(logits).cuda()
    y, y1 = (torch.full((T, d), float("nan"), dtype=torch.bfloat16, device="cuda") for _ in range(2))
    rb.route_forward(ctx, 0, ld, xd, y)
    rb.route(ctx, 0, ld)
    rb.forward(ctx, 0, xd, y1)
    sync()
    bits = LY.device_to_bits(y)
    assert np.array_equal(bits, LY.device_to_bits(y1))
    y_ref = dxo.moe_forward(versions, d, f, group, x, ids, w, shared=shared, shared_f=shared_f if shared else 0)
    yg = bf16_bits_to_f32(bits).astype(np.float64)
    tok = np.linalg.norm(yg - y_ref, axis=1) / np.linalg.norm(y_ref, axis=1)
    assert rel_l2(bits, y_ref) <= REL_L2_TOL and tok.max() <= 2 * REL_L2_TOL
    assert_elementwise(dxo, bits, y_ref, versions, group, x, ids, w, shared=shared, T_call=T)
    del keep
    ctx.close()


def _layer_of_few_versions(B, LY, dxo, pair, E, k, d, f, group, T, seed, shared_f=0, n=5, hi=(0, 2)):
    """A layer of E experts that share n versions: context, what it needs kept, the versions, the shared expert's."""
    import dataclasses
    wl = dataclasses.replace(WORKLOADS["C1"], T=1, E=n, k=1, d=d, f=f, group=group, shared_f=shared_f)
    if pair == "int4-int2":
        small, keep, versions = _quant_pair_layer(B, LY, dxo, wl, list(hi), seed, 1)
    else:
        keep = Layer(B, LY, dxo, wl, list(hi), seed=seed)
        small, versions = keep.ctx, keep.versions
    ctx = B.Context(L=1, E=E, d=d, f=f, top_k=k, group=group, max_tokens=T, shared_f=shared_f,
                    hi_fmt=B.DX_FMT_INT4G if pair == "int4-int2" else B.DX_FMT_BF16)
    for e in range(E):
        ctx.dx_swap_handle(0, e, small.dx_get_handle(0, e % n))
    shared, shared_dev = None, None
    if shared_f:
        masters = W.shared_master(wl, seed, 0)
        shared_dev = [LY.bits_to_device(m) for m in masters]
        ctx.dx_swap_handle(0, E, B.make_handle(B.DX_FMT_BF16, *shared_dev))
        shared = dxo.ExpertVersion.bf16(*masters)
    return ctx, (keep, small, shared_dev), [versions[e % n] for e in range(E)], shared


def _logits_of_segments(sizes, T, k, seed):
    """Logits [T, E] whose top-k gives expert e sizes[e] tokens (each at most T, T * k together): the tokens in turn."""
    g = np.random.default_rng(seed)
    logits = np.full((T, len(sizes)), -8.0, np.float32)
    at = 0
    for e, m in enumerate(sizes):
        logits[(at + np.arange(m)) % T, e] = g.uniform(1.0, 3.0, m)
        at += m
    assert at == T * k and max(sizes) <= T
    return logits[g.permutation(T)]


def _moved_by_four_bytes(x):
    """x where the tiles' loads cannot take it: the call runs on the streaming kernels"""
    flat = torch.empty(x.numel() + 8, dtype=x.dtype, device=x.device)
    return flat[2:2 + x.numel()].view_as(x).copy_(x)


def _check_thin_tiles_alone(LY, dxo, ctx, versions, shared, shared_f, x, logits, k, f, group, tokens=None):
    """A call that runs on thin tiles alone: one call and two the same bits, `tokens` (all) against the oracle, and all of them against the streaming
    kernels, from which it differs in some bit (other kernels did run).  Returns y."""
    T, E, d = *logits.shape, x.shape[1]
    ids, w, *_ = dxo.route(logits, k)
    rb = LY.RoutingBuffers(T, E, k)
    xd, ld = LY.bits_to_device(x), torch.from_numpy(logits).cuda()
    y, y1, ys = (torch.full((T, d), float("nan"), dtype=torch.bfloat16, device="cuda") for _ in range(3))
    rb.route_forward(ctx, 0, ld, xd, y)
    rb.route(ctx, 0, ld)
    rb.forward(ctx, 0, xd, y1)
    rb.forward(ctx, 0, _moved_by_four_bytes(xd), ys)
    sync()
    assert np.array_equal(rb.ids.cpu().numpy(), ids)
    bits, streamed = LY.device_to_bits(y), LY.device_to_bits(ys)
    assert np.array_equal(bits, LY.device_to_bits(y1))
    assert not np.array_equal(bits, streamed), "the call did not run on tiles"
    # (both round H and y to bf16 from fp32 sums in another order: of the values of H and y that lie close to a border one may be off by 2^-8)
    assert rel_l2(bits, bf16_bits_to_f32(streamed).astype(np.float64)) <= 2.0 ** -8
    y_ref = dxo.moe_forward(versions, d, f, group, x, ids, w, shared=shared, shared_f=shared_f, tokens=tokens)
    some = bits if tokens is None else bits[tokens]
    tok = np.linalg.norm(bf16_bits_to_f32(some).astype(np.float64) - y_ref, axis=1) / np.linalg.norm(y_ref, axis=1)
    assert rel_l2(some, y_ref) <= REL_L2_TOL and tok.max() <= 2 * REL_L2_TOL
    assert_elementwise(dxo, some, y_ref, versions, group, x, ids, w, shared=shared, tokens=tokens, T_call=T)
    return y


@pytest.mark.parametrize("pair,k,d,f,group,shared_f", [
    ("bf16-int4", 10, 2176, 192, 64, 0),    # 34 K steps and three; 1.5 and 8.5 column tiles
    ("bf16-int4", 10, 2304, 256, 128, 384), # a shared expert of another width, in four row tiles
    ("bf16-int4", 64, 2176, 64, 32, 64),    # one K step in the down projection
    ("int4-int2", 10, 2176, 192, 64, 0),
    ("int4-int2", 10, 2304, 256, 128, 0),
])
def test_forward_thin_tiles_alone_at_the_edges_of_a_tile(B, LY, dxo, pair, k, d, f, group, shared_f):
    """Calls of up to 128 tokens whose K the streaming kernels would take in rounds run on thin tiles if they fill the chip, segments above 32 rows
    in several, with O in fp32: segments at the edges of a tile, every token against the oracle."""
    T, E = 128, 256
    edges = [128, 127, 97, 96, 65, 64, 63, 33, 33, 32, 31, 17, 16, 1]
    n = E - len(edges) - 10
    each, more = divmod(T * k - sum(edges), n)
    sizes = edges + [0] * 10 + [each + (i < more) for i in range(n)]
    print(f"thin tiles alone {pair} k={k} d={d} f={f} group={group} shared={shared_f}", flush=True)
    ctx, keep, versions, shared = _layer_of_few_versions(B, LY, dxo, pair, E, k, d, f, group, T, 19, shared_f)
    sizes = np.random.default_rng(5).permutation(sizes).tolist()
    logits = _logits_of_segments(sizes, T, k, 19)
    assert dxo.route(logits, k)[2].tolist() == sizes
    x = f32_to_bf16_bits(np.random.default_rng(19).standard_normal((T, d)).astype(np.float32))
    _check_thin_tiles_alone(LY, dxo, ctx, versions, shared, shared_f, x, logits, k, f, group)
    ctx.close()
    del keep


@pytest.mark.parametrize("E,k,d,f,T,hi,tiles", [
    (8, 2, 7168, 256, 66, (0, 2), False),       # 12 row tiles of two columns
    (4, 1, 2560, 2048, 128, (0, 2), False),
    (216, 10, 2304, 256, 128, (0, 2), True),    # 512 gate/up tiles
    (215, 10, 2304, 256, 128, (0, 2), False),   # 510
    (256, 8, 2304, 256, 128, (0, 2), True),     # four pairs per expert, the down projection's K in one round
    (256, 8, 2304, 256, 127, (0, 2), False),    # a little less
    (64, 8, 2304, 2176, 24, (0, 2), True),      # three pairs per expert, both contractions in rounds
    (64, 8, 2304, 2176, 23, (0, 2), False),     # a little less
    (16, 8, 2176, 2944, 32, (0, 2), True),      # 192 down tiles
    (16, 8, 2176, 2944, 31, (0, 2), False),     # 184
    (32, 26, 2304, 512, 127, (0, 1, 2, 3, 4), True),    # all bf16
    (16, 15, 2304, 2176, 33, (0, 1, 2, 3, 4), False),   # all bf16, up to 64 tokens
    (16, 15, 2304, 2176, 33, (0, 2), True),
    (16, 15, 2304, 2112, 33, (0, 2), True),     # f in chunks and a half
    (16, 15, 2304, 2048, 64, (0, 2), True),     # the down projection's K in one round
    (16, 15, 2048, 2304, 64, (0, 2), False),    # gate/up's
])
def test_forward_up_to_128_tokens_on_tiles_where_they_fill_the_chip(B, LY, dxo, E, k, d, f, T, hi, tiles):
    """Which calls of up to 128 tokens with K in rounds run on thin tiles: those that do not give the same bits as with an x that only the streaming kernels
    take."""
    assert torch.cuda.get_device_properties(0).multi_processor_count == 256, "the sizes are those of 256 compute units"
    ctx, keep, _, _ = _layer_of_few_versions(B, LY, dxo, "bf16-int4", E, k, d, f, 64, T, 23, hi=hi)
    g = torch.Generator(device="cuda").manual_seed(3)
    logits = torch.randn((T, E), generator=g, device="cuda")
    x = torch.randn((T, d), generator=g, device="cuda").to(torch.bfloat16)
    rb = LY.RoutingBuffers(T, E, k)
    y, ys = torch.empty_like(x), torch.empty_like(x)
    rb.route_forward(ctx, 0, logits, x, y)
    rb.route_forward(ctx, 0, logits, _moved_by_four_bytes(x), ys)
    sync()
    assert torch.equal(y, ys) == (not tiles)
    assert rel_l2(LY.device_to_bits(y), bf16_bits_to_f32(LY.device_to_bits(ys)).astype(np.float64)) <= 2.0 ** -8
    ctx.close()
    del keep


@pytest.mark.parametrize("E,k,d,f,T,shared_f,tiles", [
    (80, 2, 2048, 256, 256, 0, False),      # 192 tiles at most
    (81, 2, 2048, 256, 256, 0, True),       # 194
    (5, 1, 2048, 256, 240, 0, False),       # 48 pairs per expert
    (5, 1, 2048, 256, 241, 0, True),
    (16, 1, 2048, 256, 384, 0, False),      # above 256 tokens 24
    (16, 1, 2048, 256, 385, 0, True),
    (32, 1, 2176, 256, 400, 0, False),
    (32, 1, 2176, 256, 401, 0, True),
    (16, 1, 1920, 256, 200, 0, True),       # a short K
    (16, 1, 2048, 256, 200, 64, True),      # a shared expert
    (128, 2, 2048, 512, 160, 0, False),     # K in one round: 552 tiles
    (128, 2, 2048, 512, 161, 0, True),
    (128, 2, 2048, 640, 160, 0, True),      # 690
    (128, 2, 2176, 512, 160, 0, True),      # K in rounds
    (22, 2, 2048, 1024, 132, 0, False),     # 12 pairs per expert
    (22, 2, 2048, 1024, 133, 0, True),
])
def test_forward_above_128_tokens_on_streaming_kernels_where_tiles_are_few(B, LY, dxo, E, k, d, f, T, shared_f, tiles):
    """Which calls of more than 128 tokens run on the streaming kernels: those that give the same bits as with an x that only they take; a dozen tokens
    against the oracle."""
    assert torch.cuda.get_device_properties(0).multi_processor_count == 256, "the sizes are those of 256 compute units"
    print(f"above 128 tokens E={E} k={k} d={d} f={f} T={T} shared={shared_f}", flush=True)
    ctx, keep, versions, shared = _layer_of_few_versions(B, LY, dxo, "bf16-int4", E, k, d, f, 64, T, 31, shared_f)
    g = np.random.default_rng(T)
    x, logits = f32_to_bf16_bits(g.standard_normal((T, d)).astype(np.float32)), g.standard_normal((T, E)).astype(np.float32)
    ids, w, *_ = dxo.route(logits, k)
    xd, ld = LY.bits_to_device(x), torch.from_numpy(logits).cuda()
    rb = LY.RoutingBuffers(T, E, k)
    y, y1, ys = (torch.full((T, d), float("nan"), dtype=torch.bfloat16, device="cuda") for _ in range(3))
    rb.route_forward(ctx, 0, ld, xd, y)
    rb.route(ctx, 0, ld)
    rb.forward(ctx, 0, xd, y1)
    rb.forward(ctx, 0, _moved_by_four_bytes(xd), ys)
    sync()
    assert np.array_equal(rb.ids.cpu().numpy(), ids)
    bits = LY.device_to_bits(y)
    assert np.array_equal(bits, LY.device_to_bits(y1))
    assert torch.equal(y, ys) == (not tiles)
    tokens = np.sort(g.choice(T, 12, replace=False)).astype(np.int32)
    y_ref = dxo.moe_forward(versions, d, f, 64, x, ids, w, shared=shared, shared_f=shared_f, tokens=tokens)
    assert rel_l2(bits[tokens], y_ref) <= REL_L2_TOL
    assert_elementwise(dxo, bits[tokens], y_ref, versions, 64, x, ids, w, shared=shared, tokens=tokens, T_call=T)
    ctx.close()
    del keep


@pytest.mark.parametrize("pair,T,k", [("bf16-int4", 64, 8), ("bf16-int4", 40, 14), ("int4-int2", 64, 8)])
def test_forward_thin_tiles_alone_of_one_routing_chunk(B, LY, dxo, pair, T, k):
    """Up to 64 tokens the routing is one kernel that lists no tiles: the list of the call, not that of the call of 128 tokens in front of it, and calls of
    few tokens on thin tiles, recorded into a graph and replayed with other calls between."""
    E, d, f, group = 16, 2304, 2176, 128
    print(f"thin tiles alone {pair} T={T} k={k}", flush=True)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        ctx, keep, versions, _ = _layer_of_few_versions(B, LY, dxo, pair, E, k, d, f, group, 128, 29, n=3, hi=(1,))
        g = np.random.default_rng(T)
        inputs = []
        for n in (128, T):
            inputs.append((f32_to_bf16_bits(g.standard_normal((n, d)).astype(np.float32)), (2 * g.standard_normal((n, E))).astype(np.float32)))
        (x0, logits0), (x, logits) = inputs
        rb0, y0 = LY.RoutingBuffers(128, E, k), torch.empty((128, d), dtype=torch.bfloat16, device="cuda")
        x0, logits0 = LY.bits_to_device(x0), torch.from_numpy(logits0).cuda()

        def other_call():
            rb0.route_forward(ctx, 0, logits0, x0, y0)
            stream.synchronize()

        other_call()
        tokens = np.sort(g.choice(T, 10, replace=False)).astype(np.int32)
        eager = _check_thin_tiles_alone(LY, dxo, ctx, versions, None, 0, x, logits, k, f, group, tokens=tokens)
        rb, y = LY.RoutingBuffers(T, E, k), torch.empty_like(eager)
        xd, ld = LY.bits_to_device(x), torch.from_numpy(logits).cuda()
        stream.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            rb.route_forward(ctx, 0, ld, xd, y)
        for rep in range(4):
            y.zero_()
            other_call()
            graph.replay()
            stream.synchronize()
            assert torch.equal(y, eager), rep
        # fewer tokens' worth of segments in the same buffers: the replay follows them
        ld.copy_(torch.where(torch.arange(E, device="cuda") < k, 1.0, -4.0) + ld * 0.1)
        rb.route_forward(ctx, 0, ld, xd, y)
        stream.synchronize()
        assert rb.counts.cpu().tolist() == [T] * k + [0] * (E - k)
        want = y.clone()
        other_call()
        y.zero_()
        graph.replay()
        stream.synchronize()
        assert torch.equal(y, want)
        del graph
    ctx.close()
    del keep


def _hard_gates():
    """bf16 pairs (g, u), g < 0, whose silu(g) * u lies closer than 3e-6 of its value to the border between two bf16 values, but not closer than
    6e-7, and all u with g = -87.5, -88 and -88.5, where 1 / (1 + e^-g) is below the normal range; and the bf16 value each rounds to (bits)."""
    g = -np.unique(bf16_bits_to_f32(np.arange(0x4100, 0x42B2, dtype=np.uint16)))    # -8 .. -88.5
    u = bf16_bits_to_f32(np.arange(0x3F80, 0x4000, dtype=np.uint16))                # 1 .. 2
    g, u = (a.ravel().astype(np.float64) for a in np.meshgrid(g, u))
    h = g / (1.0 + np.exp(-g)) * u
    ulp = 2.0 ** (np.floor(np.log2(np.abs(h))) - 7)
    border = (np.floor(np.abs(h) / ulp) + 0.5) * ulp
    off = np.abs(np.abs(h) - border) / np.abs(h)
    keep = (off > 6e-7) & ((off < 3e-6) | (g < -87.25))
    up = np.abs(h) > border
    value = np.sign(h) * (np.floor(np.abs(h) / ulp) + up) * ulp
    return tuple(f32_to_bf16_bits(a[keep].astype(np.float32)) for a in (g, u, value))


@pytest.mark.parametrize("T,E,k,d,f", [
    (240, 8, 1, 256, 128),      # thin tiles in the launch of the others
    (128, 256, 10, 2176, 192),  # thin tiles alone
])
def test_forward_thin_tiles_swiglu(B, LY, T, E, k, d, f):
    """SwiGLU of the thin tiles to fp32 accuracy: gates and ups given exactly (a token has one element, so they are a column of the matrices),
    W_down the identity, and values that an error of 6e-7 may not but one of a few 1e-6 does round to another bf16 value (the exact form:
    expf one ulp, sum, quotient and product half an ulp each, 3e-7 together)."""
    g, u, h = _hard_gates()
    assert len(h) > 400
    at = (np.arange(f)[:, None] + f * np.arange(d)[None, :]) % len(h)       # pair of (row of W_gate, column)
    wg, wu = (LY.bits_to_device(a[at]) for a in (g, u))
    eye = np.zeros((d, f), np.float32)
    eye[np.arange(f), np.arange(f)] = 1.0
    wd = LY.bits_to_device(f32_to_bf16_bits(eye))
    ctx = B.Context(L=1, E=E, d=d, f=f, top_k=k, group=64, max_tokens=T)
    for e in range(E):
        ctx.dx_swap_handle(0, e, B.make_handle(B.DX_FMT_BF16, wg, wu, wd))
    column = np.random.default_rng(1).permutation(d)[:T]
    x = np.zeros((T, d), np.float32)
    x[np.arange(T), column] = 1.0
    pair = np.arange(T * k)
    expert = (pair // k + pair % k * (E // k)) % E                          # k different ones to a token
    perm = np.argsort(expert, kind="stable").astype(np.int32)
    counts = np.bincount(expert, minlength=E)
    assert counts.max() <= 32
    w = np.zeros((T, k), np.float32)
    w[:, 0] = 1.0
    dev = [torch.from_numpy(a).cuda() for a in (expert.reshape(T, k).astype(np.int32), w, np.r_[0, np.cumsum(counts)].astype(np.int32), perm)]
    y = torch.full((T, d), float("nan"), dtype=torch.bfloat16, device="cuda")
    print(f"thin SwiGLU T={T} E={E} k={k} d={d} f={f}", flush=True)
    ctx.dx_moe_forward(0, None, LY.bits_to_device(f32_to_bf16_bits(x)), T, *dev, y)
    sync()
    got, want = LY.device_to_bits(y)[:, :f], h[at[:, column]].T
    bad = np.argwhere(got != want)
    assert len(bad) == 0, (len(bad), bf16_bits_to_f32(got[tuple(bad[0])][None]), bf16_bits_to_f32(want[tuple(bad[0])][None]))
    ctx.close()


def _wide_phases(counts, hi, f, d, T, shared_f=0, hi_quantized=False):
    """Whether the 128-row tiles of a call (segments below 512 rows, none in 256-row tiles) are 256 columns wide: gate/up, down."""
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    tiles = [-(-int(m) // 128) if m > 32 else 0 for m in counts]
    shared = -(-T // 128) if shared_f else 0
    quant = sum(t for e, t in enumerate(tiles) if hi_quantized or e not in hi)
    all_tiles = sum(tiles) + shared
    as_quantized = 20 * quant >= 9 * all_tiles or (5 * quant >= all_tiles and 5 * tiles.count(1) <= 2 * sum(tiles))
    narrow = [sum(tiles) * -(-columns // 128) + shared * -(-columns_shared // 128)
              for columns, columns_shared in ((2 * f, 2 * shared_f), (d, d))]
    return tuple(2 * n > 5 * n_cu if as_quantized else n > 6 * n_cu or 3 * n_cu < n <= 4 * n_cu for n in narrow)


@pytest.mark.parametrize("pair,d,f,group,shared_f", [
    ("int4-int2", 384, 5184, 64, 0),      # gate/up: 6 K steps, so every slot of codes is filled again
    ("int4-int2", 10368, 512, 128, 0),    # down: 8 steps
    ("int4-int2", 10368, 704, 64, 0),     # 11
    ("bf16-int4", 10368, 704, 32, 0),
    ("bf16-int4", 128, 3840, 64, 5184),   # gate/up with a shared expert of another width, half a tile of columns at its end
    ("bf16-int4", 10368, 192, 64, 320),   # down: 5 steps for the shared expert, 3 for the others
])
def test_forward_prefill_wide_tiles_many_steps_and_shared_expert(B, LY, dxo, pair, d, f, group, shared_f):
    """As above: rings that are filled several times, and the shared expert's tiles behind the routed ones'."""
    import dataclasses
    T, E, k, hi = 320, 4, 2, [1]
    wl = dataclasses.replace(WORKLOADS["C1"], T=T, E=E, k=k, d=d, f=f, group=group, shared_f=shared_f)
    print(f"wide tiles {pair} d={d} f={f} group={group} shared_f={shared_f}", flush=True)
    x = W.activations(wl, seed=19)
    logits = np.random.default_rng(19).standard_normal((T, E)).astype(np.float32)
    ids, w, counts, offsets, perm = dxo.route(logits, k)
    assert _wide_phases(counts, hi, f, d, T, shared_f, hi_quantized=pair == "int4-int2") == (f > d, d > f)
    shared = None
    if pair == "int4-int2":
        ctx, keep, versions = _quant_pair_layer(B, LY, dxo, wl, hi, 19, T)
    else:
        keep = Layer(B, LY, dxo, wl, hi, seed=19, shared=W.shared_master(wl, 19, 0) if shared_f else None)
        ctx, versions, shared = keep.ctx, keep.versions, keep.shared
    y = torch.full((T, d), float("nan"), dtype=torch.bfloat16, device="cuda")
    LY.RoutingBuffers(T, E, k).route_forward(ctx, 0, torch.from_numpy(logits).cuda(), LY.bits_to_device(x), y)
    sync()
    tokens = np.unique(np.append(np.arange(0, T, 7), T - 1))
    y_ref = dxo.moe_forward(versions, d, f, group, x, ids, w, shared=shared, shared_f=shared_f, tokens=tokens)
    bits = LY.device_to_bits(y)
    assert np.isfinite(bf16_bits_to_f32(bits)).all()
    assert rel_l2(bits[tokens], y_ref) <= REL_L2_TOL
    used = assert_elementwise(dxo, bits[tokens], y_ref, versions, group, x, ids, w, shared=shared, tokens=tokens, T_call=T)
    print(f"  element-wise: largest error = {used:.2f} of its bound", flush=True)
    del keep
    ctx.close()


@pytest.mark.parametrize("E,k,T,d,f,hi,wide", [
    (4, 1, 250, 128, 6144, [0, 1, 2, 3], (False, False)),   # bf16, 4 x 96 narrow tiles: 1.5 per compute unit
    (8, 1, 500, 128, 8192, list(range(8)), (True, False)),  # 4
    (8, 1, 500, 128, 8256, list(range(8)), (False, False)), # a little more than 4
    (12, 1, 750, 128, 8192, list(range(12)), (False, False)),  # 6
    (12, 1, 750, 128, 8256, list(range(12)), (True, False)),   # a little more than 6
    (8, 1, 500, 128, 9216, [0, 1, 2, 3, 4, 5], (False, False)),  # a quarter quantized, a row tile each, 4.5
    (4, 1, 900, 128, 9216, [0, 1, 2], (True, False)),          # the same with two row tiles each
])
def test_prefill_lines_between_narrow_and_wide_tiles(B, LY, dxo, E, k, T, d, f, hi, wide):
    """Calls on both sides of every line between the kinds of tiles, rows evenly spread: every 16th token against the oracle."""
    import dataclasses
    wl = dataclasses.replace(WORKLOADS["C1"], T=T, E=E, k=k, d=d, f=f, group=64)
    x = W.activations(wl, seed=23)
    logits = np.random.default_rng(23).standard_normal((T, E)).astype(np.float32)
    logits[np.arange(T), np.arange(T) % E] += 100.0
    ids, w, counts, offsets, perm = dxo.route(logits, k)
    if torch.cuda.get_device_properties(0).multi_processor_count == 256:
        assert _wide_phases(counts, hi, f, d, T) == wide
    ly = Layer(B, LY, dxo, wl, hi, seed=23)
    y = torch.full((T, d), float("nan"), dtype=torch.bfloat16, device="cuda")
    ly.rb.route_forward(ly.ctx, 0, torch.from_numpy(logits).cuda(), LY.bits_to_device(x), y)
    sync()
    tokens = np.arange(0, T, 16)
    y_ref = dxo.moe_forward(ly.versions, d, f, 64, x, ids, w, tokens=tokens)
    assert rel_l2(LY.device_to_bits(y)[tokens], y_ref) <= REL_L2_TOL
    ly.ctx.close()


@pytest.mark.parametrize("pair,d,f,group", [
    ("bf16-int4", 128, 5184, 32),    # gate/up in wide tiles: 2 K steps
    ("bf16-int4", 384, 5184, 64),
    ("bf16-int4", 1152, 5248, 128),  # 18 steps, an odd number of groups
    ("int4-int2", 384, 5184, 64),
    ("int4-int2", 1152, 5248, 128),
    ("bf16-int4", 10368, 192, 32),   # down: 3 steps, then 11
    ("bf16-int4", 10368, 704, 64),
    ("int4-int2", 10368, 704, 64),
])
def test_prefill_outputs_do_not_depend_on_the_kind_of_tile(B, LY, dxo, pair, d, f, group):
    """The same tokens in a call of many tiles (256 columns wide) and in one of few: the same bits, because the sums over K
    have one order."""
    import dataclasses
    T, T_few, E, k = 320, 190, 4, 2
    wl = dataclasses.replace(WORKLOADS["C1"], T=T, E=E, k=k, d=d, f=f, group=group)
    x = W.activations(wl, seed=17)
    logits = np.random.default_rng(17).standard_normal((T, E)).astype(np.float32)
    for n, wide in ((T, True), (T_few, False)):
        counts = dxo.route(logits[:n], k)[2]
        assert counts.min() > 32
        assert _wide_phases(counts, [1], f, d, n, hi_quantized=pair == "int4-int2") == (wide and f > d, wide and d > f)
    if pair == "int4-int2":
        ctx, keep, _ = _quant_pair_layer(B, LY, dxo, wl, [1], 17, T)
    else:
        keep = Layer(B, LY, dxo, wl, [1], seed=17)
        ctx = keep.ctx
    xd, ld = LY.bits_to_device(x), torch.from_numpy(logits).cuda()
    y = torch.full((T, d), float("nan"), dtype=torch.bfloat16, device="cuda")
    y_few = torch.full((T_few, d), float("nan"), dtype=torch.bfloat16, device="cuda")
    LY.RoutingBuffers(T, E, k).route_forward(ctx, 0, ld, xd, y)
    LY.RoutingBuffers(T_few, E, k).route_forward(ctx, 0, ld[:T_few].contiguous(), xd[:T_few].contiguous(), y_few)
    sync()
    assert np.isfinite(bf16_bits_to_f32(LY.device_to_bits(y))).all()
    assert torch.equal(y[:T_few], y_few)
    del keep
    ctx.close()


def test_forward_prefill_tile_list_at_its_bound(B, LY, dxo):
    """Segments of 129 rows in a context of exactly that many tokens: the list of row tiles has as many entries as the
    context holds (two per expert), every one of them in use."""
    import dataclasses
    E, T = 5, 5 * 129
    wl = dataclasses.replace(WORKLOADS["C1"], T=T, E=E, k=1, d=128, f=64, group=64)
    x, logits = W.layer_inputs(wl, seed=79)
    logits = logits.copy()
    logits[np.arange(T), np.arange(T) % E] += 100.0
    ly = Layer(B, LY, dxo, wl, [1, 3], seed=79)
    y_gpu, y_ref = ly.run(x, logits)
    yg = bf16_bits_to_f32(y_gpu).astype(np.float64)
    assert (np.linalg.norm(yg - y_ref, axis=1) / np.linalg.norm(y_ref, axis=1)).max() <= 2 * REL_L2_TOL
    ly.ctx.close()


@pytest.mark.parametrize("T,E,k,d,f,group,shared_f,resident", [
    (8330, 2, 2, 1024, 128, 64, 0, [0]),       # bf16 and int4: 32 tiles of 256 rows each and ten rows of a 128-row tile
    (8192, 1, 1, 2048, 128, 64, 128, []),      # int4, whole tiles only; the shared expert's
    (16400, 1, 1, 1024, 384, 128, 0, []),      # three groups per row of W_down: int4 stays with the 128-row tiles
    (16500, 2, 1, 1024, 384, 64, 256, [1]),    # a shared expert of another size
    (8200, 3, 2, 1024, 128, 32, 0, [1]),       # int4 in groups of 32
    (8200, 14, 1, 2048, 128, 64, 0, [2, 3]),   # 586 rows on average: int4 only
])
def test_forward_prefill_256_row_tiles(B, LY, dxo, T, E, k, d, f, group, shared_f, resident):
    """Segments of 1024 rows and more on average (int4: 512): their whole 256 rows go in 256-row tiles, the rest in 128-row
    ones; every seventh token and the last ones against the oracle."""
    import dataclasses
    wl = dataclasses.replace(WORKLOADS["C1"], T=T, E=E, k=k, d=d, f=f, group=group, shared_f=shared_f)
    x, logits = W.layer_inputs(wl, seed=71)
    shared = W.shared_master(wl, 71, 0) if shared_f else None
    ly = Layer(B, LY, dxo, wl, resident, seed=71, shared=shared)
    y_gpu, y_ref = ly.run(x, logits, tokens=sorted(set(range(0, T, 7)) | set(range(T - 12, T))))
    yg = bf16_bits_to_f32(y_gpu).astype(np.float64)
    tok = np.linalg.norm(yg - y_ref, axis=1) / np.linalg.norm(y_ref, axis=1)
    assert rel_l2(y_gpu, y_ref) <= REL_L2_TOL and tok.max() <= 2 * REL_L2_TOL
    ly.ctx.close()


@pytest.mark.parametrize("T,E,group,resident", [(150, 16, 128, [0, 5, 9]), (600, 16, 128, [0, 5, 9]),
                                               # row tiles of the shared expert, of a bf16 and of int4 experts in one launch
                                               (1100, 4, 64, [1])])
def test_forward_prefill_with_shared_expert(B, LY, dxo, T, E, group, resident):
    import dataclasses
    wl = dataclasses.replace(WORKLOADS["C4"], L=1, E=E, k=min(4, E), T=T, d=256, f=128, shared_f=256, group=group)
    x, logits = W.layer_inputs(wl, seed=8)
    shared = W.shared_master(wl, 8, 0)
    ly = Layer(B, LY, dxo, wl, resident, seed=8, shared=shared)
    y_gpu, y_ref = ly.run(x, logits)
    err = rel_l2(y_gpu, y_ref)
    print("  prefill shared rel-L2", err, flush=True)
    assert err <= REL_L2_TOL
    ly.ctx.close()


@pytest.mark.parametrize("T,n_hi", [(4096, None), (8192, None), (4096, 0)])
def test_forward_c3_prefill_sampled_tokens(B, LY, dxo, T, n_hi):
    """The 30B-shaped prefill layer at full size (T=4096) and at twice that (the largest batch the
    benchmarks use), and with no resident expert (every expert int4):
    routing bit-exact on all tokens, layer output checked on sampled tokens the oracle computes one by one."""
    import dataclasses
    wl = dataclasses.replace(WORKLOADS["C3"], T=T)
    if n_hi is not None:
        wl = dataclasses.replace(wl, n_hi=n_hi)
    print("forward C3: drawing masters", flush=True)
    masters = W.layer_masters(wl, 0, 0)
    x, logits = W.layer_inputs(wl, seed=0)
    ids, w, counts, offsets, perm = dxo.route(logits, wl.k)
    S = counts.astype(np.uint64) << np.uint64(16)
    resident = set(int(e) for e in dxo.select_topn(S, wl.n_hi)) if wl.n_hi else set()
    ctx = B.Context(L=1, E=wl.E, d=wl.d, f=wl.f, top_k=wl.k, group=wl.group, max_tokens=wl.T)
    dev = [LY.bits_to_device(m) for m in masters]
    lw = LY.LayerWeights(ctx, 0, *dev, resident, wl.group)
    rb = LY.RoutingBuffers(wl.T, wl.E, wl.k)
    y = torch.empty((wl.T, wl.d), dtype=torch.bfloat16, device="cuda")
    print("forward C3: running", flush=True)
    rb.route(ctx, 0, torch.from_numpy(logits).cuda())
    rb.forward(ctx, 0, LY.bits_to_device(x), y)
    sync()
    assert np.array_equal(rb.ids.cpu().numpy(), ids)
    assert np.array_equal(rb.perm.cpu().numpy(), perm)
    g = np.random.default_rng(0)
    # sampled tokens: random ones plus tokens routed to the largest and to the smallest segments
    big, small = int(np.argmax(counts)), int(np.argmin(np.where(counts > 0, counts, 1 << 30)))
    forced = [int(perm[offsets[big]] // wl.k), int(perm[offsets[big + 1] - 1] // wl.k), int(perm[offsets[small]] // wl.k)]
    tokens = np.unique(np.concatenate([g.choice(wl.T, 40, replace=False), forced])).astype(np.int32)
    wg, wu, wd = masters
    needed = set(int(e) for e in ids[tokens].ravel())
    filler = None
    versions = [None] * wl.E
    for e in needed:
        versions[e] = (dxo.ExpertVersion.bf16(wg[e], wu[e], wd[e]) if e in resident
                       else dxo.ExpertVersion.int4_from_master(wg[e], wu[e], wd[e], wl.group))
        filler = versions[e]
    versions = [v if v is not None else filler for v in versions]
    y_ref = dxo.moe_forward(versions, wl.d, wl.f, wl.group, x, ids, w, tokens=tokens)
    y_gpu = LY.device_to_bits(y)[tokens]
    err = rel_l2(y_gpu, y_ref)
    print("  C3 sampled rel-L2", err, "segments max/min", counts.max(), counts[counts > 0].min(), flush=True)
    assert err <= REL_L2_TOL
    yg = bf16_bits_to_f32(y_gpu).astype(np.float64)
    tok = np.linalg.norm(yg - y_ref, axis=1) / np.linalg.norm(y_ref, axis=1)
    assert tok.max() <= 2 * REL_L2_TOL
    used = assert_elementwise(dxo, y_gpu, y_ref, versions, wl.group, x, ids, w, tokens=tokens, T_call=wl.T)
    print(f"  element-wise: largest error = {used:.2f} of its bound", flush=True)
    del lw
    ctx.close()


@pytest.mark.parametrize("T,one_call", [(32, False), (300, False), (32, True)])
def test_route_and_forward_replay_from_a_captured_graph(B, LY, dxo, T, one_call):
    """dx_route + dx_moe_forward (or the two as one dx_route_forward call) recorded into a HIP graph (the
    decode pass, and the prefill pass with its tile kernels), replayed several times
    with eager work and synchronisations in between: every replay reproduces the eager result bit for bit."""
    import dataclasses
    wl = dataclasses.replace(WORKLOADS["C1"], T=T, E=4 if T > 64 else 8)
    x, logits = W.layer_inputs(wl, seed=9)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        ly = Layer(B, LY, dxo, wl, [0, 2], seed=9)
        ctx, rb = ly.ctx, ly.rb
        xd, ld = LY.bits_to_device(x), torch.from_numpy(logits).cuda()
        y = torch.empty((T, wl.d), dtype=torch.bfloat16, device="cuda")
        rb.route(ctx, 0, ld, T)
        rb.forward(ctx, 0, xd, y, None, T)
        stream.synchronize()
        eager = y.clone()
        ids, w, *_ = dxo.route(logits, wl.k)
        y_ref = dxo.moe_forward(ly.versions, wl.d, wl.f, wl.group, x, ids, w)
        assert rel_l2(LY.device_to_bits(eager), y_ref) <= REL_L2_TOL
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=stream):
            if one_call:
                rb.route_forward(ctx, 0, ld, xd, y, None, T)
            else:
                rb.route(ctx, 0, ld, T)
                rb.forward(ctx, 0, xd, y, None, T)
        for rep in range(4):
            y.zero_()                                  # eager work between the replays
            rb.perm.zero_()
            stream.synchronize()
            g.replay()
            stream.synchronize()
            assert torch.equal(y, eager), rep
        # new inputs in the same buffers: the replay follows them
        x2, logits2 = W.layer_inputs(wl, seed=10)
        xd.copy_(LY.bits_to_device(x2))
        ld.copy_(torch.from_numpy(logits2).cuda())
        stream.synchronize()
        g.replay()
        stream.synchronize()
        ids2, w2, *_ = dxo.route(logits2, wl.k)
        assert np.array_equal(rb.ids.cpu().numpy()[:T], ids2)
        y_ref2 = dxo.moe_forward(ly.versions, wl.d, wl.f, wl.group, x2, ids2, w2)
        assert rel_l2(LY.device_to_bits(y), y_ref2) <= REL_L2_TOL
        del g
    ly.ctx.close()


# ------------------------------------------- the int4 (high) / int2 (low) precision pair
@pytest.mark.parametrize("rows,K,group", [(128, 256, 64), (768, 2048, 128), (37, 128, 32), (2048, 768, 128)])
def test_int2_quantize_bit_exact(B, LY, dxo, rows, K, group):
    g = np.random.default_rng(rows + K)
    w = (0.02 * g.standard_normal((rows, K))).astype(np.float32)
    w[0, :group] = 0.0
    wb = W.f32_to_bf16_bits(w)
    ctx = B.Context(L=1, E=2, d=64, f=64, top_k=1, group=32, max_tokens=4)
    q = torch.zeros((rows, K // 4), dtype=torch.uint8, device="cuda")
    s = torch.zeros((rows, K // group), dtype=torch.bfloat16, device="cuda")
    ctx.dx_quantize_expert_int2(LY.bits_to_device(wb), rows, K, group, q, s)
    sync()
    q_ref, s_ref = dxo.quantize2(wb, group)
    assert np.array_equal(q.cpu().numpy(), q_ref)
    assert np.array_equal(LY.device_to_bits(s), s_ref)
    ctx.close()


def _quant_pair_layer(B, LY, dxo, wl, hi_ids, seed, T):
    masters = W.layer_masters(wl, seed, 0)
    ctx = B.Context(L=1, E=wl.E, d=wl.d, f=wl.f, top_k=wl.k, group=wl.group, max_tokens=max(T, 1), hi_fmt=B.DX_FMT_INT4G)
    dev = [LY.bits_to_device(m) for m in masters]
    lw = LY.QuantPairLayerWeights(ctx, 0, *dev, hi_ids, wl.group)
    wg, wu, wd = masters
    versions = [dxo.ExpertVersion.int4_from_master(wg[e], wu[e], wd[e], wl.group) if e in set(hi_ids)
                else dxo.ExpertVersion.int2_from_master(wg[e], wu[e], wd[e], wl.group) for e in range(wl.E)]
    return ctx, lw, versions


@pytest.mark.parametrize("T,E,k,d,f,group,hi_ids", [
    (16, 8, 2, 256, 128, 64, [1, 6]),          # decode, K-chunks of 64 (16 codes per lane and chunk)
    (40, 8, 2, 256, 128, 128, [0]),            # two token tiles, chunks of 128
    (7, 4, 2, 512, 256, 128, []),              # every expert int2
    (33, 16, 4, 2048, 768, 128, [2, 3, 5]),    # the 30B layer's K extents
    (300, 4, 2, 256, 128, 64, [0, 2]),         # prefill-sized: 128-row tiles expand int2 on the way to LDS
    (700, 4, 2, 256, 128, 128, [1]),
    (700, 4, 2, 512, 256, 128, [1, 2]),        # int4 segments of several row tiles
])
def test_forward_int4_int2_pair(B, LY, dxo, T, E, k, d, f, group, hi_ids):
    import dataclasses
    wl = dataclasses.replace(WORKLOADS["C1"], T=T, E=E, k=k, d=d, f=f, group=group)
    print(f"int4/int2 pair T={T} E={E} k={k} d={d} f={f} g={group} hi={hi_ids}", flush=True)
    x, logits = W.layer_inputs(wl, seed=13)
    ctx, lw, versions = _quant_pair_layer(B, LY, dxo, wl, hi_ids, 13, T)
    fm = ctx.dx_get_formats()[0]
    st = ctx.dx_get_states()[0]
    for e in range(E):
        assert fm[e] == (B.DX_FMT_INT4G if e in hi_ids else B.DX_FMT_INT2G)
        assert st[e] == (B.DX_STATE_RESIDENT_HI if e in hi_ids else B.DX_STATE_RESIDENT_LO)
    rb = LY.RoutingBuffers(T, E, k)
    y = torch.empty((T, d), dtype=torch.bfloat16, device="cuda")
    rb.route(ctx, 0, torch.from_numpy(logits).cuda())
    rb.forward(ctx, 0, LY.bits_to_device(x), y)
    sync()
    ids, w, *_ = dxo.route(logits, k)
    assert np.array_equal(rb.ids.cpu().numpy(), ids)
    y_ref = dxo.moe_forward(versions, d, f, group, x, ids, w)
    err = rel_l2(LY.device_to_bits(y), y_ref)
    print("  rel-L2", err, flush=True)
    assert err <= REL_L2_TOL
    ctx.close()


def test_int2_handles_need_a_group_of_64_or_more(B, LY):
    with pytest.raises(B.DxError):
        B.Context(L=1, E=4, d=64, f=64, top_k=2, group=32, max_tokens=4, hi_fmt=B.DX_FMT_INT4G)
    ctx = B.Context(L=1, E=4, d=64, f=64, top_k=2, group=32, max_tokens=4)
    buf = torch.zeros(4096, dtype=torch.uint8, device="cuda")
    h = B.make_handle(B.DX_FMT_INT2G, buf, buf, buf, buf, buf, buf)
    with pytest.raises(B.DxError):
        ctx.dx_swap_handle(0, 0, h)
    ctx.close()


@pytest.mark.parametrize("T,E,k,d,f,shared_f,resident", [
    (1, 8, 2, 256, 128, 0, [0, 3]), (7, 8, 2, 256, 128, 0, []), (16, 8, 4, 512, 384, 0, list(range(8))),
    (17, 4, 2, 256, 256, 0, [1]), (32, 4, 3, 512, 384, 0, [0, 2]), (32, 2, 2, 256, 128, 0, [0]),
    (32, 16, 4, 256, 128, 256, [0, 5, 9]), (9, 16, 4, 512, 256, 128, []), (32, 128, 8, 256, 128, 0, list(range(0, 128, 3))),
])
def test_forward_decode_group128_small_shapes(B, LY, dxo, T, E, k, d, f, shared_f, resident):
    """Decode batches of up to 32 tokens with group 128 (K-chunks of 128): one and two token tiles per
    expert, one to three K-chunks, all-bf16 / all-int4 / mixed tables, the shared expert; every token,
    and the same bits on a second run (every sum has a fixed order)."""
    import dataclasses
    wl = dataclasses.replace(WORKLOADS["C1"], T=T, E=E, k=k, d=d, f=f, group=128, shared_f=shared_f)
    print(f"decode g128 T={T} E={E} k={k} d={d} f={f} shared_f={shared_f}", flush=True)
    x, logits = W.layer_inputs(wl, seed=21)
    shared = W.shared_master(wl, 21, 0) if shared_f else None
    ly = Layer(B, LY, dxo, wl, resident, seed=21, shared=shared)
    y_gpu, y_ref = ly.run(x, logits)
    err = rel_l2(y_gpu, y_ref)
    print("  rel-L2", err, flush=True)
    assert err <= REL_L2_TOL
    yg = bf16_bits_to_f32(y_gpu).astype(np.float64)
    tok = np.linalg.norm(yg - y_ref, axis=1) / np.linalg.norm(y_ref, axis=1)
    assert tok.max() <= 2 * REL_L2_TOL
    again, _ = ly.run(x, logits)
    assert np.array_equal(again, y_gpu)                              # a fixed summation order: bit-reproducible
    ly.ctx.close()


@pytest.mark.parametrize("T", [16, 200])
def test_forward_with_a_caller_owned_handle_table(B, LY, dxo, T):
    """dx_moe_forward(handle_table, ...): a table in caller memory (here with the opposite format of
    every expert) is used instead of the context's own; passing the context's table address is the
    same as passing none."""
    import ctypes as C
    import dataclasses
    wl = dataclasses.replace(WORKLOADS["C1"], T=T)
    x, logits = W.layer_inputs(wl, seed=17)
    ly = Layer(B, LY, dxo, wl, [0, 2], seed=17)
    ctx, rb = ly.ctx, ly.rb
    xd, ld = LY.bits_to_device(x), torch.from_numpy(logits).cuda()
    y0 = torch.empty((T, wl.d), dtype=torch.bfloat16, device="cuda")
    y1, y2 = torch.empty_like(y0), torch.empty_like(y0)
    rb.route(ctx, 0, ld, T)
    rb.forward(ctx, 0, xd, y0, None, T)
    rb.forward(ctx, 0, xd, y1, ctx.dx_handle_table(0), T)
    # a second set of versions, formats flipped, in a table the caller owns
    flipped = [e for e in range(wl.E) if e not in (0, 2)]
    lw2 = LY.LayerWeights(ctx, 0, *ly.dev, flipped, wl.group, publish=False)
    raw = b"".join(bytes(lw2.handle(e)) for e in range(wl.E))
    assert len(raw) == 64 * wl.E
    table = torch.frombuffer(bytearray(raw), dtype=torch.uint8).cuda()
    rb.forward(ctx, 0, xd, y2, table, T)
    sync()
    assert torch.equal(y0, y1)
    ids, w, *_ = dxo.route(logits, wl.k)
    wg, wu, wd = ly.masters
    v_flip = [dxo.ExpertVersion.bf16(wg[e], wu[e], wd[e]) if e in flipped
              else dxo.ExpertVersion.int4_from_master(wg[e], wu[e], wd[e], wl.group) for e in range(wl.E)]
    assert rel_l2(LY.device_to_bits(y0), dxo.moe_forward(ly.versions, wl.d, wl.f, wl.group, x, ids, w)) <= REL_L2_TOL
    assert rel_l2(LY.device_to_bits(y2), dxo.moe_forward(v_flip, wl.d, wl.f, wl.group, x, ids, w)) <= REL_L2_TOL
    assert not torch.equal(y0, y2)
    assert np.array_equal(ctx.dx_get_formats()[0], [0 if e in (0, 2) else 1 for e in range(wl.E)])   # own table untouched
    del lw2
    ctx.close()


# --------------------------------------------- routing inside the forward call
def _route_forward_case(B, LY, dxo, wl, resident, seed, shared=None, logits=None, hotness=False):
    """dx_route_forward against the oracle (every routing array bit-exact, y within the bar) and against
    dx_route + dx_moe_forward on the same inputs (the same bits)."""
    x, lg = W.layer_inputs(wl, seed=seed)
    if logits is not None:
        lg = logits
    T = wl.T
    ly = Layer(B, LY, dxo, wl, resident, seed=seed, shared=shared)
    ctx, rb = ly.ctx, ly.rb
    xd, ld = LY.bits_to_device(x), torch.from_numpy(lg).cuda()
    y_sep = torch.empty((T, wl.d), dtype=torch.bfloat16, device="cuda")
    y_one = torch.full_like(y_sep, float("nan"))
    rb.route(ctx, 0, ld, T)
    rb.forward(ctx, 0, xd, y_sep, None, T)
    sync()
    for t in (rb.ids, rb.counts, rb.offsets, rb.perm):
        t.fill_(-1)
    rb.w.fill_(float("nan"))
    rb.route_forward(ctx, 0, ld, xd, y_one, None, T)
    sync()
    ids, w, counts, offsets, perm = dxo.route(lg, wl.k)
    assert np.array_equal(rb.ids.cpu().numpy()[:T], ids)
    assert np.array_equal(rb.counts.cpu().numpy(), counts)
    assert np.array_equal(rb.offsets.cpu().numpy(), offsets)
    assert np.array_equal(rb.perm.cpu().numpy()[:T * wl.k], perm)
    wg = rb.w.cpu().numpy()[:T].astype(np.float64)
    assert np.max(np.abs(wg - w) / np.maximum(w, 1e-30)) < W_TOL or np.max(np.abs(wg - w)) < 1e-7
    assert torch.equal(y_one, y_sep)
    y_ref = dxo.moe_forward(ly.versions, wl.d, wl.f, wl.group, x, ids, w, shared=ly.shared,
                            shared_f=wl.shared_f if ly.shared else 0)
    err = rel_l2(LY.device_to_bits(y_one), y_ref)
    print("  rel-L2", err, flush=True)
    assert err <= REL_L2_TOL
    assert_elementwise(dxo, LY.device_to_bits(y_one), y_ref, ly.versions, wl.group, x, ids, w, shared=ly.shared, T_call=T)
    ctx.close()


@pytest.mark.parametrize("T,E,k,d,f,group,shared_f,resident", [
    (16, 8, 2, 256, 128, 64, 0, [1, 6]),                 # the small configuration
    (1, 8, 2, 256, 128, 128, 0, [0, 3]), (7, 8, 8, 256, 128, 128, 0, []), (17, 4, 2, 256, 256, 128, 0, [1]),
    (32, 128, 8, 256, 128, 128, 0, list(range(0, 128, 3))), (32, 16, 4, 256, 128, 128, 256, [0, 5, 9]),
    (31, 100, 16, 512, 384, 128, 0, list(range(50))), (32, 1, 1, 256, 128, 32, 0, [0]),
    # more than 32 tokens: a second routing pass in the prologue, segments of more than 32 tokens
    (33, 8, 2, 256, 128, 64, 0, [1]), (64, 128, 8, 256, 128, 128, 0, list(range(0, 128, 5))),
    (50, 16, 4, 256, 128, 128, 256, [0, 5, 9]), (63, 4, 4, 256, 128, 128, 0, [2]),
    # more than 128 experts: 32 logits per lane in the routing prologue, two experts per thread in the scans
    (8, 200, 4, 256, 128, 64, 0, [7]), (32, 512, 10, 256, 128, 128, 0, list(range(3, 512, 43))),
    (32, 512, 10, 256, 128, 128, 128, list(range(0, 512, 50))), (64, 300, 16, 256, 128, 128, 0, [0, 299]),
    (33, 511, 10, 256, 128, 64, 128, list(range(100, 140))), (1, 129, 1, 256, 128, 128, 0, []),
    # shapes the self-routing kernel does not take: the call runs the two kernels one after the other
    (65, 8, 2, 256, 128, 64, 0, [1]), (8, 600, 4, 256, 128, 64, 0, [7]), (150, 4, 2, 256, 128, 64, 0, [0]),
    # full-width contractions (8 or 16 K-chunks) at small intermediate sizes, every chunk size, with and
    # without a shared expert, resident sets from none to all
    (32, 16, 4, 2048, 128, 128, 0, [0, 5, 9]), (32, 128, 8, 2048, 128, 128, 0, list(range(0, 128, 4))),
    (17, 12, 3, 2048, 128, 128, 0, []), (5, 8, 2, 2048, 128, 128, 0, list(range(8))), (1, 8, 2, 1024, 128, 128, 0, [2, 3]),
    (32, 16, 4, 2048, 128, 128, 256, [0, 5, 9]), (16, 6, 6, 1024, 128, 128, 128, [4]), (31, 40, 16, 1024, 128, 64, 0, [1, 2, 3, 30]),
    (32, 8, 2, 512, 64, 64, 0, [0, 1]), (9, 8, 3, 512, 64, 32, 64, [6]), (32, 4, 2, 256, 32, 32, 0, [3]),
    (32, 128, 8, 2048, 128, 128, 0, list(range(60, 124))), (3, 128, 8, 2048, 128, 128, 128, [0]),
])
def test_route_forward_matches_oracle_and_separate_calls(B, LY, dxo, T, E, k, d, f, group, shared_f, resident):
    import dataclasses
    wl = dataclasses.replace(WORKLOADS["C1"], T=T, E=E, k=k, d=d, f=f, group=group, shared_f=shared_f)
    print(f"route_forward T={T} E={E} k={k} d={d} f={f} g={group} shared_f={shared_f}", flush=True)
    shared = W.shared_master(wl, 23, 0) if shared_f else None
    _route_forward_case(B, LY, dxo, wl, resident, 23, shared=shared)


def test_route_forward_with_tied_logits(B, LY, dxo):
    """Logits on a coarse grid (many exact ties, both signs of zero): the ids must follow the tie rule."""
    import dataclasses
    wl = dataclasses.replace(WORKLOADS["C1"], T=32, E=128, k=8, d=256, f=128, group=128)
    g = np.random.default_rng(77)
    logits = np.round(g.standard_normal((wl.T, wl.E)) * 2).astype(np.float32) / 2
    logits[logits == 0] *= np.where(g.random(np.count_nonzero(logits == 0)) < 0.5, -1.0, 1.0).astype(np.float32)
    _route_forward_case(B, LY, dxo, wl, [0, 1, 2, 64, 127], 29, logits=logits)


@pytest.mark.parametrize("case", ["coarse grid", "all equal", "favourites are neighbours", "one lane and ties",
                                  "favourites 64 apart", "few above a sea of equals", "second pass"])
def test_route_forward_wide_layer_threshold_and_its_fallback(B, LY, dxo, case):
    """Layers of more than 128 experts select through a threshold and a short list per lane, and fall back to
    the plain selection when a lane's list overflows: logits built so that both ways run (many exact ties;
    every favourite of a token among 32 neighbouring experts, or among the 32 experts 64 * g + 4 * c + j that
    one lane of the selection holds; a few distinct values above a constant), all of them against the oracle's
    ids, weights and permutation."""
    import dataclasses
    T = 40 if case == "second pass" else 32
    wl = dataclasses.replace(WORKLOADS["C1"], T=T, E=512, k=10, d=256, f=128, group=128)
    g = np.random.default_rng(901)
    if case == "coarse grid":
        logits = np.round(g.standard_normal((T, wl.E)) * 2).astype(np.float32) / 2
        logits[logits == 0] *= np.where(g.random(np.count_nonzero(logits == 0)) < 0.5, -1.0, 1.0).astype(np.float32)
    elif case == "all equal":
        logits = np.full((T, wl.E), 0.25, np.float32)
        logits[1::2] = -3.0
    elif case == "favourites are neighbours":
        logits = g.standard_normal((T, wl.E)).astype(np.float32)
        for t in range(T):       # the ten largest inside one lane's 32 experts, a different lane per token
            lane = t % 16
            logits[t, 32 * lane + g.permutation(32)[:12]] += 8.0
    elif case == "one lane and ties":
        logits = g.standard_normal((T, wl.E)).astype(np.float32)
        for t in range(T):
            own = (64 * np.arange(8)[:, None] + 4 * (t % 16) + np.arange(4)[None, :]).ravel()
            logits[t, own[::2]] = 5.0                               # sixteen equal favourites in one lane's set
    elif case == "favourites 64 apart":
        logits = g.standard_normal((T, wl.E)).astype(np.float32)
        for t in range(T):
            own = (64 * np.arange(8)[:, None] + 4 * (t % 16) + np.arange(4)[None, :]).ravel()
            logits[t, own[g.permutation(32)[:12]]] += 8.0           # the ten largest inside one lane's set
    elif case == "few above a sea of equals":
        logits = np.zeros((T, wl.E), np.float32)
        for t in range(T):
            logits[t, g.permutation(wl.E)[:4]] = g.random(4).astype(np.float32) + 1.0   # 4 < k distinct leaders
    else:
        logits = (g.standard_normal((T, wl.E)) * 1.5).astype(np.float32)
    _route_forward_case(B, LY, dxo, wl, list(range(5, 512, 61)), 31, logits=logits)


def test_route_forward_c2_full_size_and_hotness(B, LY, dxo):
    """The 30B-shaped decode layer through dx_route_forward, with the hotness update inside the call."""
    wl = WORKLOADS["C2"]
    masters = W.layer_masters(wl, 0, 0)
    wg, wu, wd = masters
    resident = list(range(0, wl.E, 4))
    ctx = B.Context(L=2, E=wl.E, d=wl.d, f=wl.f, top_k=wl.k, group=wl.group, max_tokens=wl.T, route_updates_hotness=True)
    dev = [LY.bits_to_device(m) for m in masters]
    lws = [LY.LayerWeights(ctx, l, *dev, resident, wl.group) for l in range(2)]
    versions = [dxo.ExpertVersion.bf16(wg[e], wu[e], wd[e]) if e in set(resident)
                else dxo.ExpertVersion.int4_from_master(wg[e], wu[e], wd[e], wl.group) for e in range(wl.E)]
    rb = LY.RoutingBuffers(wl.T, wl.E, wl.k)
    c = np.zeros((2, wl.E), np.int64)
    y = torch.empty((wl.T, wl.d), dtype=torch.bfloat16, device="cuda")
    for step in range(3):
        for layer in range(2):
            x, lg = W.layer_inputs(wl, seed=0, layer=layer, step=step)
            print(f"route_forward C2 step {step} layer {layer}", flush=True)
            rb.route_forward(ctx, layer, torch.from_numpy(lg).cuda(), LY.bits_to_device(x), y)
            sync()
            ids, w, counts, offsets, perm = dxo.route(lg, wl.k)
            dxo.hotness_update(c[layer], counts)
            assert np.array_equal(rb.ids.cpu().numpy(), ids) and np.array_equal(rb.perm.cpu().numpy(), perm)
            assert np.array_equal(rb.offsets.cpu().numpy(), offsets)
            if step == 2:
                y_ref = dxo.moe_forward(versions, wl.d, wl.f, wl.group, x, ids, w)
                err = rel_l2(LY.device_to_bits(y), y_ref)
                print("  rel-L2", err, flush=True)
                assert err <= REL_L2_TOL
                used = assert_elementwise(dxo, LY.device_to_bits(y), y_ref, versions, wl.group, x, ids, w)
                print(f"  element-wise: largest error = {used:.2f} of its bound", flush=True)
    assert np.array_equal(ctx.dx_get_counters(), c)
    del lws
    ctx.close()


def test_route_forward_rejects_bad_arguments(B, LY):
    ctx = B.Context(L=1, E=8, d=64, f=64, top_k=2, group=32, max_tokens=4)
    rb = LY.RoutingBuffers(4, 8, 2)
    buf = torch.zeros(4096, dtype=torch.float32, device="cuda")
    with pytest.raises(B.DxError):
        ctx.dx_route_forward(1, None, buf, buf, 4, rb.ids, rb.w, rb.counts, rb.offsets, rb.perm, buf)   # layer
    with pytest.raises(B.DxError):
        ctx.dx_route_forward(0, None, buf, buf, 5, rb.ids, rb.w, rb.counts, rb.offsets, rb.perm, buf)   # T > max
    with pytest.raises(B.DxError):
        ctx.dx_route_forward(0, None, None, buf, 4, rb.ids, rb.w, rb.counts, rb.offsets, rb.perm, buf)  # null logits
    with pytest.raises(B.DxError):
        ctx.dx_route_forward(0, None, buf, buf, 4, rb.ids, rb.w, rb.counts, rb.offsets, rb.perm, buf)   # no versions published
    ctx.close()


def test_profiling_reports_every_kernel_of_a_forward_call(B, LY, dxo):
    """dx_set_profiling / dx_get_profile: decode calls (separate and as one call) and a prefill call are
    counted, every kernel reports a positive, plausible duration, reading clears the record, and the
    results are the same as without profiling."""
    import dataclasses
    for T, one_call in ((32, False), (32, True), (300, False)):
        wl = dataclasses.replace(WORKLOADS["C1"], T=T, E=8 if T <= 64 else 4)
        x, logits = W.layer_inputs(wl, seed=31)
        ly = Layer(B, LY, dxo, wl, [0, 2], seed=31)
        ctx, rb = ly.ctx, ly.rb
        xd, ld = LY.bits_to_device(x), torch.from_numpy(logits).cuda()
        y0 = torch.empty((T, wl.d), dtype=torch.bfloat16, device="cuda")
        y1 = torch.empty_like(y0)
        rb.route(ctx, 0, ld, T)
        rb.forward(ctx, 0, xd, y0, None, T)
        ctx.dx_set_profiling(True)
        for _ in range(3):
            if one_call:
                rb.route_forward(ctx, 0, ld, xd, y1, None, T)
            else:
                rb.route(ctx, 0, ld, T)
                rb.forward(ctx, 0, xd, y1, None, T)
        p = ctx.dx_get_profile()
        print(f"profile T={T} one_call={one_call}: {p}", flush=True)
        assert p["calls"] == 3
        for key in ("gate_up_ms", "down_ms", "combine_ms"):
            assert 0.0 < p[key] < 3 * 50.0, (key, p[key])          # three calls, far below 50 ms each
        assert p["empty_ms"] >= 0.0
        assert ctx.dx_get_profile()["calls"] == 0                   # reading clears
        ctx.dx_set_profiling(False)
        sync()
        assert torch.equal(y0, y1)
        ctx.close()


def test_profiling_stamps_the_kernels_of_thin_tiles_alone(B, LY, dxo):
    """A call of up to 128 tokens on tiles reports its kernels' own durations: the gate/up kernel's is the same whether the kernel that lists the tiles (4 us
    with its launch) runs in front of it, on a caller's routing arrays, or the routing wrote the list."""
    T, E, k, d, f = 128, 256, 10, 2304, 256
    ctx, keep, _, _ = _layer_of_few_versions(B, LY, dxo, "bf16-int4", E, k, d, f, 128, T, 37)
    g = torch.Generator(device="cuda").manual_seed(5)
    logits, x = torch.randn((T, E), generator=g, device="cuda"), torch.randn((T, d), generator=g, device="cuda").to(torch.bfloat16)
    rb, y, y1 = LY.RoutingBuffers(T, E, k), torch.empty_like(x), torch.empty_like(x)
    rb.route_forward(ctx, 0, logits, x, y)
    ctx.dx_set_profiling(True)
    us = {True: [], False: []}
    for rep in range(7):
        for routed in (True, False):
            for _ in range(20):
                if routed:
                    rb.route_forward(ctx, 0, logits, x, y1)
                else:
                    rb.forward(ctx, 0, x, y1)
            p = ctx.dx_get_profile()
            assert p["calls"] == 20 and p["down_ms"] > 0.0 and p["combine_ms"] > 0.0
            us[routed].append(p["gate_up_ms"] * 50)
    a, b = (float(np.median(v)) for v in us.values())
    print(f"gate/up behind routing {a:.2f} us, behind the list {b:.2f}", flush=True)
    assert abs(a - b) < 2.0, us
    ctx.dx_set_profiling(False)
    sync()
    assert torch.equal(y, y1)
    ctx.close()
    del keep


def test_route_forward_random_shapes_match_separate_calls(B, LY, dxo):
    """Seeded random decode shapes (tokens, experts, top-k, sizes, group, resident sets, with and without a
    shared expert): dx_route_forward gives the routing arrays of the oracle, bit for bit, and the same y
    bits as dx_route + dx_moe_forward.  (The layer output itself is checked against the oracle in the
    tests above; this one covers many shapes quickly.)"""
    import dataclasses
    g = np.random.default_rng(20251115)
    for case in range(36):
        group = int(g.choice([32, 64, 128]))
        d = group * int(g.integers(1, 9)) if group < 128 else 128 * int(g.choice([1, 2, 4, 8]))
        d = max(d, 64)
        f = group * int(g.integers(1, 5))
        if f % 16:
            f = (f // 16 + 1) * 16
        E = int(g.choice([1, 2, 5, 8, 16, 37, 64, 100, 128]))
        k = int(g.integers(1, min(E, 16) + 1))
        T = int(g.integers(1, 65))
        shared_f = int(g.choice([0, 0, f]))
        n_res = int(g.integers(0, E + 1))
        resident = sorted(g.choice(E, size=n_res, replace=False).tolist())
        wl = dataclasses.replace(WORKLOADS["C1"], T=T, E=E, k=k, d=d, f=f, group=group, shared_f=shared_f)
        print(f"case {case}: T={T} E={E} k={k} d={d} f={f} g={group} shared_f={shared_f} hi={n_res}", flush=True)
        x, logits = W.layer_inputs(wl, seed=100 + case)
        shared = W.shared_master(wl, 100 + case, 0) if shared_f else None
        ly = Layer(B, LY, dxo, wl, resident, seed=100 + case, shared=shared)
        ctx, rb = ly.ctx, ly.rb
        xd, ld = LY.bits_to_device(x), torch.from_numpy(logits).cuda()
        y_sep = torch.empty((T, d), dtype=torch.bfloat16, device="cuda")
        y_one = torch.full_like(y_sep, float("nan"))
        rb.route(ctx, 0, ld, T)
        rb.forward(ctx, 0, xd, y_sep, None, T)
        sync()
        w_sep = rb.w.clone()
        for t in (rb.ids, rb.counts, rb.offsets, rb.perm):
            t.fill_(-1)
        rb.route_forward(ctx, 0, ld, xd, y_one, None, T)
        sync()
        ids, w, counts, offsets, perm = dxo.route(logits, k)
        assert np.array_equal(rb.ids.cpu().numpy()[:T], ids)
        assert np.array_equal(rb.counts.cpu().numpy(), counts)
        assert np.array_equal(rb.offsets.cpu().numpy(), offsets)
        assert np.array_equal(rb.perm.cpu().numpy()[:T * k], perm)
        assert torch.equal(rb.w[:T], w_sep[:T])
        assert torch.equal(y_one, y_sep)
        ctx.close()


def test_forward_random_shapes_match_oracle(B, LY, dxo):
    """Seeded random layers in both regimes (1 to 400 tokens; streaming kernels, row tiles,
    shapes that fit the tiles and shapes that do not): every layer output within the bar of the oracle's,
    token by token within twice the bar."""
    import dataclasses
    g = np.random.default_rng(20251116)
    for case in range(24):
        group = int(g.choice([32, 64, 128]))
        d = int(g.choice([128, 256, 384, 512])) if group <= 64 else int(g.choice([128, 256, 512]))
        f = int(g.choice([64, 128, 192, 256, 384])) if group <= 64 else int(g.choice([128, 256, 384]))
        if d % group or f % group:
            d, f = 2 * group, 2 * group
        E = int(g.choice([1, 2, 3, 4, 8, 16, 32]))
        k = int(g.integers(1, min(E, 6) + 1))
        T = int(g.choice([1, 5, 31, 32, 33, 64, 100, 128, 129, 200, 257, 400]))
        shared_f = int(g.choice([0, 0, f]))
        n_res = int(g.integers(0, E + 1))
        resident = sorted(g.choice(E, size=n_res, replace=False).tolist())
        wl = dataclasses.replace(WORKLOADS["C1"], T=T, E=E, k=k, d=d, f=f, group=group, shared_f=shared_f)
        print(f"case {case}: T={T} E={E} k={k} d={d} f={f} g={group} shared_f={shared_f} hi={resident}", flush=True)
        x, logits = W.layer_inputs(wl, seed=200 + case)
        shared = W.shared_master(wl, 200 + case, 0) if shared_f else None
        ly = Layer(B, LY, dxo, wl, resident, seed=200 + case, shared=shared)
        y_gpu, y_ref = ly.run(x, logits)
        err = rel_l2(y_gpu, y_ref)
        print("  rel-L2", err, flush=True)
        assert err <= REL_L2_TOL
        yg = bf16_bits_to_f32(y_gpu).astype(np.float64)
        tok = np.linalg.norm(yg - y_ref, axis=1) / np.maximum(np.linalg.norm(y_ref, axis=1), 1e-30)
        assert tok.max() <= 2 * REL_L2_TOL
        ly.ctx.close()


def test_forward_random_shapes_int4_int2_pair(B, LY, dxo):
    """Seeded random layers of the int4 (high) / int2 (low) pair in both regimes, through dx_route_forward:
    routing bit-exact, layer output within the bar of the oracle's."""
    import dataclasses
    g = np.random.default_rng(20251117)
    for case in range(16):
        group = int(g.choice([64, 128]))
        d = int(g.choice([128, 256, 512]))
        f = int(g.choice([128, 256, 384]))
        E = int(g.choice([2, 4, 8, 16, 32]))
        k = int(g.integers(1, min(E, 6) + 1))
        T = int(g.choice([1, 7, 32, 33, 64, 100, 200, 300]))
        n_hi = int(g.integers(0, E + 1))
        hi_ids = sorted(g.choice(E, size=n_hi, replace=False).tolist())
        wl = dataclasses.replace(WORKLOADS["C1"], T=T, E=E, k=k, d=d, f=f, group=group)
        print(f"case {case}: T={T} E={E} k={k} d={d} f={f} g={group} int4={hi_ids}", flush=True)
        x, logits = W.layer_inputs(wl, seed=300 + case)
        ctx, lw, versions = _quant_pair_layer(B, LY, dxo, wl, hi_ids, 300 + case, T)
        rb = LY.RoutingBuffers(T, E, k)
        y = torch.empty((T, d), dtype=torch.bfloat16, device="cuda")
        rb.route_forward(ctx, 0, torch.from_numpy(logits).cuda(), LY.bits_to_device(x), y)
        sync()
        ids, w, counts, offsets, perm = dxo.route(logits, k)
        assert np.array_equal(rb.ids.cpu().numpy(), ids) and np.array_equal(rb.perm.cpu().numpy(), perm)
        y_ref = dxo.moe_forward(versions, d, f, group, x, ids, w)
        err = rel_l2(LY.device_to_bits(y), y_ref)
        print("  rel-L2", err, flush=True)
        assert err <= REL_L2_TOL
        del lw
        ctx.close()


@pytest.mark.parametrize("pair,T,d,f,group", [
    ("bf16-int4", 33, 2048, 256, 64),     # two groups per chunk, the self-routing kernel at the 30B layer's K
    ("bf16-int4", 20, 1152, 2176, 32),    # four groups per chunk; 9 and 17 chunks: K in rounds, a last chunk without a pair
    ("bf16-int4", 34, 1920, 1152, 128),   # 15 and 9 chunks
    ("bf16-int4", 7, 128, 896, 32),       # one and seven chunks: a chunk per wavefront
    ("bf16-int4", 21, 3584, 2560, 128),   # 28 chunks (two per wavefront in rounds, a short last round) and 20 (one per wavefront)
    ("bf16-int4", 40, 352, 608, 32),      # no multiple of 128: 11 chunks of 32 (one ragged round) and 19 (rounds)
    ("int4-int2", 20, 1152, 2176, 64),
    ("int4-int2", 35, 4096, 3584, 128),   # 32 and 28 chunks
    ("int4-int2", 5, 704, 1088, 64),      # 11 and 17 chunks of 64
    ("int4-int2", 33, 1920, 2048, 128),
    ("int4-int2", 3, 128, 896, 64),
    ("int4-int2", 18, 2048, 896, 64),
])
def test_decode_groups_and_chunk_counts(B, LY, dxo, pair, T, d, f, group):
    """Group sizes below the chunk of 128 elements, and numbers of chunks that leave a wavefront with half of its
    chunks or none: route_forward against the oracle, token by token within twice the bar."""
    import dataclasses
    wl = dataclasses.replace(WORKLOADS["C1"], T=T, E=4, k=2, d=d, f=f, group=group)
    x, logits = W.layer_inputs(wl, seed=51)
    if pair == "int4-int2":
        ctx, keep, versions = _quant_pair_layer(B, LY, dxo, wl, [0, 2], 51, T)
    else:
        ly = Layer(B, LY, dxo, wl, [0, 2], seed=51)
        ctx, keep, versions = ly.ctx, ly, ly.versions
    rb = LY.RoutingBuffers(T, wl.E, wl.k)
    y = torch.empty((T, d), dtype=torch.bfloat16, device="cuda")
    rb.route_forward(ctx, 0, torch.from_numpy(logits).cuda(), LY.bits_to_device(x), y)
    sync()
    ids, w, counts, offsets, perm = dxo.route(logits, wl.k)
    assert np.array_equal(rb.ids.cpu().numpy(), ids) and np.array_equal(rb.perm.cpu().numpy(), perm)
    y_ref = dxo.moe_forward(versions, d, f, group, x, ids, w)
    yg = bf16_bits_to_f32(LY.device_to_bits(y)).astype(np.float64)
    tok = np.linalg.norm(yg - y_ref, axis=1) / np.linalg.norm(y_ref, axis=1)
    assert rel_l2(LY.device_to_bits(y), y_ref) <= REL_L2_TOL and tok.max() <= 2 * REL_L2_TOL
    del keep
    ctx.close()


@pytest.mark.parametrize("pair,T,E,k,d,f,group,shared_f", [
    ("bf16-int4", 1, 8, 1, 256, 1664, 128, 0),     # one expert: eight wavefronts share 13 chunks
    ("bf16-int4", 1, 8, 3, 128, 896, 64, 128),     # two wavefronts to an expert, an odd number of chunks; the shared expert's one
    ("bf16-int4", 1, 32, 16, 256, 1792, 32, 256),  # more experts than wavefronts, K in three rounds of six chunks
    ("bf16-int4", 2, 4, 3, 256, 128, 128, 384),    # tokens that share experts: places inside a segment
    ("bf16-int4", 2, 64, 16, 2048, 128, 128, 128), # the most it takes: 32 pairs, 17 tasks to a block
    ("bf16-int4", 2, 4, 4, 4096, 1024, 128, 0),    # every expert selected by both tokens: the most chunks it takes then
    ("bf16-int4", 1, 8, 8, 128, 4096, 128, 0),     # too much for its eight blocks: the streaming kernel
    ("bf16-int4", 3, 16, 16, 128, 256, 128, 0),    # a token more than it takes
    ("int4-int2", 1, 8, 2, 256, 640, 64, 0),
    ("int4-int2", 2, 16, 9, 256, 384, 128, 0),
])
def test_forward_of_one_or_few_tokens(B, LY, dxo, pair, T, E, k, d, f, group, shared_f):
    """The down projection that combines in place (a call of a few tokens): route_forward and the separate calls give the
    same bits, and y is the oracle's within the bar, token by token within twice the bar."""
    import dataclasses
    wl = dataclasses.replace(WORKLOADS["C1"], T=T, E=E, k=k, d=d, f=f, group=group, shared_f=shared_f)
    x, logits = W.layer_inputs(wl, seed=61)
    shared = None
    if pair == "int4-int2":
        ctx, keep, versions = _quant_pair_layer(B, LY, dxo, wl, [0, 2], 61, T)
    else:
        masters = W.shared_master(wl, 61, 0) if shared_f else None
        ly = Layer(B, LY, dxo, wl, [0, 2], seed=61, shared=masters)
        ctx, keep, versions, shared = ly.ctx, ly, ly.versions, ly.shared
    rb = LY.RoutingBuffers(T, E, k)
    xd, ld = LY.bits_to_device(x), torch.from_numpy(logits).cuda()
    y = torch.full((T, d), float("nan"), dtype=torch.bfloat16, device="cuda")
    y1 = torch.empty_like(y)
    rb.route_forward(ctx, 0, ld, xd, y)
    rb.route(ctx, 0, ld)
    rb.forward(ctx, 0, xd, y1)
    sync()
    assert torch.equal(y, y1)
    ids, w, counts, offsets, perm = dxo.route(logits, k)
    assert np.array_equal(rb.ids.cpu().numpy(), ids) and np.array_equal(rb.perm.cpu().numpy(), perm)
    y_ref = dxo.moe_forward(versions, d, f, group, x, ids, w, shared=shared, shared_f=shared_f if shared else 0)
    yg = bf16_bits_to_f32(LY.device_to_bits(y)).astype(np.float64)
    tok = np.linalg.norm(yg - y_ref, axis=1) / np.linalg.norm(y_ref, axis=1)
    assert rel_l2(LY.device_to_bits(y), y_ref) <= REL_L2_TOL and tok.max() <= 2 * REL_L2_TOL
    del keep
    ctx.close()


@pytest.mark.parametrize("pair,T,E,k,d,f,group,shared_f", [
    ("bf16-int4", 1, 8, 2, 2176, 128, 64, 0),      # gate/up: a step of 2048 and 128 elements; rows no multiple of three
    ("int4-int2", 2, 8, 2, 2176, 640, 128, 0),
    ("bf16-int4", 2, 4, 4, 640, 128, 32, 0),       # every expert of both tokens, K less than a step
    ("bf16-int4", 2, 300, 10, 2048, 512, 128, 512),  # the wide selection
    ("bf16-int4", 2, 600, 3, 384, 256, 128, 256),  # more experts than the kernel routes
    ("bf16-int4", 1, 8, 8, 1536, 1280, 64, 256),   # more groups of rows than wavefronts
    ("bf16-int4", 2, 16, 2, 8192, 128, 128, 0),    # the longest rows
    ("bf16-int4", 1, 8, 2, 8320, 128, 128, 0),     # longer ones: the streaming kernel
    ("bf16-int4", 1, 8, 2, 192, 128, 64, 0),       # gate/up no multiple of 128: likewise
])
def test_forward_of_one_or_two_tokens_row_by_row(B, LY, dxo, pair, T, E, k, d, f, group, shared_f):
    """The edges of the gate/up kernel for one and two tokens, as above."""
    test_forward_of_one_or_few_tokens(B, LY, dxo, pair, T, E, k, d, f, group, shared_f)


@pytest.mark.parametrize("pair,T,E,k,d,f,group,shared_f", [
    ("bf16-int4", 2, 4, 4, 4096, 1152, 128, 0),    # a chunk too many for experts of both tokens: the streaming kernels
    ("bf16-int4", 2, 32, 8, 256, 256, 64, 0),      # short rows of two tokens: gate/up streams
    ("bf16-int4", 1, 8, 8, 256, 1024, 128, 0),     # one token, few blocks
    ("int4-int2", 1, 8, 8, 128, 1024, 128, 0),     # the most chunks for the fewest blocks
    ("bf16-int4", 1, 8, 8, 6144, 128, 64, 128),    # nine items, wavefronts with three each
    ("bf16-int4", 2, 16, 7, 4096, 128, 128, 128),  # two tokens, four wavefronts to a block
    ("bf16-int4", 2, 40, 16, 2048, 128, 128, 0),   # 16 items, eight wavefronts
])
def test_forward_of_one_or_two_tokens_choice_of_kernels(B, LY, dxo, pair, T, E, k, d, f, group, shared_f):
    """Both sides of the lines between the streaming kernels and those for one and two tokens, and blocks of fewer wavefronts than
    items, as above."""
    test_forward_of_one_or_few_tokens(B, LY, dxo, pair, T, E, k, d, f, group, shared_f)


@pytest.mark.parametrize("T,resident", [(1, [0, 1]), (2, [0, 1]), (2, [1])])
def test_forward_of_one_or_two_tokens_without_quantized_experts(B, LY, dxo, T, resident):
    """Rows that the streaming kernel cannot take in one round: layers without a quantized expert stream gate/up where there are
    many rows; route_forward, the separate calls and a caller's own table give the oracle's y."""
    import dataclasses
    wl = dataclasses.replace(WORKLOADS["C1"], T=T, E=2, k=2, d=2176, f=3328, group=128)
    x, logits = W.layer_inputs(wl, seed=87)
    ly = Layer(B, LY, dxo, wl, resident, seed=87)
    ids, w, *_ = dxo.route(logits, wl.k)
    y_ref = dxo.moe_forward(ly.versions, wl.d, wl.f, wl.group, x, ids, w)
    xd, ld = LY.bits_to_device(x), torch.from_numpy(logits).cuda()
    for call in ("one", "two", "table"):
        y = torch.full((T, wl.d), float("nan"), dtype=torch.bfloat16, device="cuda")
        if call == "one":
            ly.rb.route_forward(ly.ctx, 0, ld, xd, y)
        else:
            ly.rb.route(ly.ctx, 0, ld)
            ly.rb.forward(ly.ctx, 0, xd, y, table=None if call == "two" else ly.ctx.dx_handle_table(0))
        sync()
        yg = bf16_bits_to_f32(LY.device_to_bits(y)).astype(np.float64)
        assert (np.linalg.norm(yg - y_ref, axis=1) / np.linalg.norm(y_ref, axis=1)).max() <= 2 * REL_L2_TOL
    ly.ctx.close()


@pytest.mark.parametrize("T,E,k", [(1, 100, 8), (2, 512, 16)])
def test_hotness_of_one_or_two_tokens(B, LY, dxo, T, E, k):
    """The kernel that routes and multiplies adds the counts as well, and writes every array."""
    import dataclasses
    wl = dataclasses.replace(WORKLOADS["C1"], T=T, E=E, k=k, d=256, f=128, group=64)
    ctx = B.Context(L=1, E=E, d=256, f=128, top_k=k, group=64, max_tokens=T, route_updates_hotness=True)
    lw = LY.LayerWeights(ctx, 0, *[LY.bits_to_device(m) for m in W.layer_masters(wl, 71, 0)], [0, 3], 64)
    rb = LY.RoutingBuffers(T, E, k)
    y = torch.empty((T, 256), dtype=torch.bfloat16, device="cuda")
    c = np.zeros((1, E), np.int64)
    for step in range(3):
        x, logits = W.layer_inputs(wl, seed=71, step=step)
        rb.route_forward(ctx, 0, torch.from_numpy(logits).cuda(), LY.bits_to_device(x), y)
        sync()
        ids, w, counts, offsets, perm = dxo.route(logits, k)
        dxo.hotness_update(c[0], counts)
        for got, want in ((rb.ids, ids), (rb.counts, counts), (rb.offsets, offsets), (rb.perm, perm)):
            assert np.array_equal(got.cpu().numpy(), want)
        assert np.max(np.abs(rb.w.cpu().numpy() - w)) < 1e-6
    assert np.array_equal(ctx.dx_get_counters(), c)
    del lw
    ctx.close()


@pytest.mark.parametrize("T,E,k", [(1, 8, 3), (2, 4, 3), (2, 6, 6), (3, 4, 3)])
def test_forward_goes_by_offsets_and_perm_alone(B, LY, dxo, T, E, k):
    """dx_moe_forward on a permutation in another order inside the segments and with ids that say nothing: the pairs'
    experts are those of the segments, at every batch size (one and two tokens have a down kernel of their own)."""
    import dataclasses
    wl = dataclasses.replace(WORKLOADS["C1"], T=T, E=E, k=k, d=256, f=128, group=64)
    x, logits = W.layer_inputs(wl, seed=67)
    ly = Layer(B, LY, dxo, wl, [0, 2], seed=67)
    ctx, rb = ly.ctx, ly.rb
    rb.route(ctx, 0, torch.from_numpy(logits).cuda(), T)
    sync()
    offsets, perm = rb.offsets.cpu().numpy(), rb.perm.cpu().numpy()
    for e in range(E):
        perm[offsets[e]:offsets[e + 1]] = perm[offsets[e]:offsets[e + 1]][::-1].copy()
    rb.perm.copy_(torch.from_numpy(perm))
    rb.ids.fill_(0)
    y = torch.full((T, wl.d), float("nan"), dtype=torch.bfloat16, device="cuda")
    rb.forward(ctx, 0, LY.bits_to_device(x), y, None, T)
    sync()
    ids, w, *_ = dxo.route(logits, k)
    y_ref = dxo.moe_forward(ly.versions, wl.d, wl.f, wl.group, x, ids, w)
    yg = bf16_bits_to_f32(LY.device_to_bits(y)).astype(np.float64)
    tok = np.linalg.norm(yg - y_ref, axis=1) / np.linalg.norm(y_ref, axis=1)
    assert tok.max() <= 2 * REL_L2_TOL
    ctx.close()


@pytest.mark.parametrize("T,E,k,used", [(1, 1, 1, 1), (2, 5, 5, 2), (2, 64, 4, 3), (1, 65, 8, 8), (2, 256, 16, 20), (2, 300, 16, 300), (2, 700, 3, 4)])
def test_forward_of_one_or_two_tokens_on_any_segments(B, LY, dxo, T, E, k, used):
    """A caller's routing arrays with segments of any length (a token may name an expert more than once) and of any expert: the
    kernel for one or two tokens finds the expert of every place from the offsets, 256 experts at a time."""
    import dataclasses
    wl = dataclasses.replace(WORKLOADS["C1"], T=T, E=E, k=k, d=256, f=128, group=64)
    g = np.random.default_rng(100 * E + k)
    x = W.activations(wl, seed=83)
    some = np.append(g.choice(E - 1, used - 1, replace=False), E - 1)      # the last expert among them
    ids = some[g.integers(0, used, (T, k))].astype(np.int32)
    w = g.random((T, k))
    counts = np.bincount(ids.ravel(), minlength=E)
    ly = Layer(B, LY, dxo, wl, [0, E - 1], seed=83)
    rb = ly.rb
    rb.ids.copy_(torch.from_numpy(ids))
    rb.w.copy_(torch.from_numpy(w.astype(np.float32)))
    rb.offsets.copy_(torch.from_numpy(np.append(0, np.cumsum(counts)).astype(np.int32)))
    rb.perm.copy_(torch.from_numpy(np.argsort(ids.ravel(), kind="stable").astype(np.int32)))
    y = torch.full((T, wl.d), float("nan"), dtype=torch.bfloat16, device="cuda")
    rb.forward(ly.ctx, 0, LY.bits_to_device(x), y, None, T)
    sync()
    y_ref = dxo.moe_forward(ly.versions, wl.d, wl.f, wl.group, x, ids, w.astype(np.float32).astype(np.float64))
    yg = bf16_bits_to_f32(LY.device_to_bits(y)).astype(np.float64)
    assert (np.linalg.norm(yg - y_ref, axis=1) / np.linalg.norm(y_ref, axis=1)).max() <= 2 * REL_L2_TOL
    ly.ctx.close()


@pytest.mark.parametrize("T", [2, 40, 200])
def test_forward_takes_tokens_that_start_inside_16_bytes(B, LY, dxo, T):
    """x as a view that starts 4 bytes into a buffer: the same bits as an aligned copy where the streaming kernels run in both
    cases, within the bar of the oracle's where the copy would go to the tile kernels."""
    import dataclasses
    wl = dataclasses.replace(WORKLOADS["C1"], T=T, E=4, k=2, d=256, f=128, group=64)
    x, logits = W.layer_inputs(wl, seed=69)
    ly = Layer(B, LY, dxo, wl, [0, 2], seed=69)
    buf = torch.zeros(T * wl.d + 8, dtype=torch.bfloat16, device="cuda")
    assert buf.data_ptr() % 16 == 0
    xv = buf[2:2 + T * wl.d].view(T, wl.d)
    xv.copy_(LY.bits_to_device(x))
    y = torch.full((T, wl.d), float("nan"), dtype=torch.bfloat16, device="cuda")
    y_copy = torch.empty_like(y)
    ly.rb.route(ly.ctx, 0, torch.from_numpy(logits).cuda(), T)
    ly.rb.forward(ly.ctx, 0, xv, y, None, T)
    ly.rb.forward(ly.ctx, 0, xv.clone(), y_copy, None, T)
    sync()
    if T <= 128:
        assert torch.equal(y, y_copy)
    ids, w, *_ = dxo.route(logits, wl.k)
    y_ref = dxo.moe_forward(ly.versions, wl.d, wl.f, wl.group, x, ids, w)
    yg = bf16_bits_to_f32(LY.device_to_bits(y)).astype(np.float64)
    assert (np.linalg.norm(yg - y_ref, axis=1) / np.linalg.norm(y_ref, axis=1)).max() <= 2 * REL_L2_TOL
    ly.ctx.close()


def test_probe_read_runs_and_checks_its_arguments(B):
    ctx = B.Context(L=1, E=8, d=64, f=64, top_k=2, group=32, max_tokens=4)
    buf = torch.zeros(8 << 20, dtype=torch.uint8, device="cuda")
    ctx.dx_probe_read(buf, 8 << 20)
    ctx.dx_probe_read(buf, 0)                                   # nothing to read
    sync()
    with pytest.raises(B.DxError):
        ctx.dx_probe_read(buf, (8 << 20) - 1)                   # not whole MiB
    with pytest.raises(B.DxError):
        ctx.dx_probe_read(None, 1 << 20)
    with pytest.raises(B.DxError):
        ctx.dx_probe_read(buf.data_ptr() + 4, 1 << 20)          # misaligned
    ctx.close()
