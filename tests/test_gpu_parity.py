"""GPU parity: the HIP path (through the C ABI) against the float64 CPU oracle,
element by element on the same seeded inputs.

Tolerances (bf16 inputs, fp32 accumulation, one rounding of y to bf16):
normwise relative error <= 2e-3 and max elementwise relative error <= 1e-2 over
|y_ref| > 1e-2.  v is fp32 and is held to 1e-5 / 1e-3; the fp32 plumbing
configuration to 1e-5 / 1e-4.  Per-call contracts: lora_expand is compared with
y_in (as stored) + s (x A) B; the fused call with x W + s (x A) B end to end.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle
from paper_2411_00915_amd import binding as B
from paper_2411_00915_amd import device, workloads as wl

pytestmark = pytest.mark.gpu

BF16_TOL = (2e-3, 1e-2)
F32_TOL = (1e-5, 1e-4)
# v: fp32 sums of K <= 5120 exact products of O(1/sqrt(K)) size; the absolute error is a few 1e-6, which on
# entries just above the 1e-2 threshold is a relative error of a few 1e-4
V_TOL = (1e-5, 1e-3)
DEV = "cuda:0"


def _tol(w):
    return F32_TOL if w.dtype == "f32" else BF16_TOL


def _assert_close(got, ref, tol, what):
    nrm, elem = oracle.error_metrics(got, ref)
    print(f"    {what}: normwise {nrm:.3e} elementwise {elem:.3e}", flush=True)
    assert nrm <= tol[0], f"{what}: normwise {nrm:.3e} > {tol[0]}"
    assert elem <= tol[1], f"{what}: elementwise {elem:.3e} > {tol[1]}"


def _to_np(t):
    return t.detach().to(torch.float32).cpu().numpy()


def _y_in(w, seed=99):
    rng = np.random.default_rng(seed)
    y = rng.standard_normal((w.T, w.N), dtype=np.float32)
    return wl.round_to_bf16(y) if w.dtype == "bf16" else y


def _launched(call):
    """names of the library's kernels that call() launches"""
    B.lora_timing_begin()
    try:
        call()
    finally:
        names = set(B.lora_timing_end())
    return names


def run_delta_case(w, variant=B.LORA_VARIANT_AUTO, ld_pad=0, check_beta0=True, rows=None):
    """shrink + expand through the ABI vs the oracle.  `rows` limits the oracle
    comparison of y to a sample of tokens (v is always checked in full)."""
    print(f"  case {w.name} T={w.T} K={w.K} N={w.N} variant={variant} ld_pad={ld_pad}", flush=True)
    dl = device.to_device(w, DEV, with_w=False)
    tdt = device.torch_dtype(w)
    plan = device.make_plan(w, variant)
    view = B.lora_plan_export(plan)
    R, v_bytes, _ = B.lora_plan_query(plan)
    tok = oracle.token_adapter(w.T, w.seg_indptr, w.seg_adapter)
    ad = oracle.Adapters(w.adapter_rank, w.adapter_scale, w.A, w.B)
    ldx, ldy = w.K + ld_pad, w.N + ld_pad
    x = torch.zeros((w.T, ldx), dtype=tdt, device=DEV)
    x[:, :w.K] = dl.x
    CANARY = -12345.0
    P = view["v_parts"]
    assert v_bytes == P * w.T * R * 4
    v = torch.full((P, max(w.T, 1), R), CANARY, dtype=torch.float32, device=DEV)
    y0 = _y_in(w)
    y = torch.full((max(w.T, 1), ldy), 7.0, dtype=tdt, device=DEV)
    y[:w.T, :w.N] = torch.from_numpy(y0).to(DEV, tdt)

    B.lora_shrink(plan, x, ldx, dl.At_ptrs, v)
    B.lora_expand(plan, v, dl.Bt_ptrs, y, ldy, 1.0)
    torch.cuda.synchronize()

    v_parts = _to_np(v)[:, :w.T]
    assert all(np.array_equal(v_parts[p] == CANARY, v_parts[0] == CANARY) for p in range(P))
    v_np = np.where(v_parts[0] == CANARY, CANARY, v_parts.astype(np.float64).sum(axis=0)).astype(np.float32)
    v_ref = oracle.shrink(w.x, tok, ad, apply_scale=True, R=R)
    ranks_tok = np.where(tok >= 0, w.adapter_rank[np.clip(tok, 0, None)], 0) if w.num_adapters else np.zeros(w.T, int)
    valid = np.arange(R)[None, :] < ranks_tok[:, None]
    assert np.all(v_np[~valid] == CANARY), "v written outside [0, r_a) or for a token without adapter"
    if valid.any():
        _assert_close(np.where(valid, v_np, 0.0), v_ref, V_TOL if w.dtype == "bf16" else F32_TOL, "v")

    y_np = _to_np(y)[:w.T]
    assert np.all(y_np[:, w.N:] == 7.0), "y written beyond column N"
    no_ad = ranks_tok == 0
    assert np.array_equal(y_np[no_ad, :w.N], y0[no_ad]), "rows without adapter must stay bit-identical"
    sel = np.arange(w.T) if rows is None else np.asarray(rows)
    if w.T:
        y_ref = oracle.expand(w.x, tok, ad, w.N, y_in=y0[sel].astype(np.float64), rows=sel)
        _assert_close(y_np[sel, :w.N], y_ref, _tol(w), "expand beta=1")

    if check_beta0 and w.T:
        y2 = torch.full((w.T, ldy), 3.0, dtype=tdt, device=DEV)
        B.lora_expand(plan, v, dl.Bt_ptrs, y2, ldy, 0.0)
        torch.cuda.synchronize()
        y2_np = _to_np(y2)
        assert np.all(y2_np[no_ad] == 3.0) and np.all(y2_np[:, w.N:] == 3.0)
        d_ref = oracle.expand(w.x, tok, ad, w.N, rows=sel)
        act = ~no_ad[sel]
        if act.any():
            _assert_close(y2_np[sel, :w.N][act], d_ref[act], _tol(w), "expand beta=0")
        # run-to-run determinism (no atomics anywhere in the path)
        v_b = torch.full_like(v, CANARY)
        y_b = torch.full((w.T, ldy), 3.0, dtype=tdt, device=DEV)
        B.lora_shrink(plan, x, ldx, dl.At_ptrs, v_b)
        B.lora_expand(plan, v_b, dl.Bt_ptrs, y_b, ldy, 0.0)
        torch.cuda.synchronize()
        assert torch.equal(v_b, v) and torch.equal(y_b, y2), "two runs differ bitwise"
    torch.cuda.synchronize()
    plan.destroy()
    return view


def _forward_rows(w, view, n_sample, seed):
    """Rows of the oracle comparison for the big configurations: one seeded row out of every 16 consecutive rows of
    the order the fused GEMM walks (so every 16-row MFMA block of every wavefront of every 256-row tile is hit), the
    first and last token of every segment (at most n_sample of them) and n_sample seeded rows on top."""
    rng = np.random.default_rng(seed)
    order = view["gemm_order"] if view["gemm_order"].shape[0] == w.T else np.arange(w.T)
    nblk = (w.T + 15) // 16
    pick = np.minimum(np.arange(nblk) * 16 + rng.integers(0, 16, nblk), w.T - 1)
    edge = np.unique(np.concatenate([w.seg_indptr[:-1], w.seg_indptr[1:] - 1]))
    edge = edge[(edge >= 0) & (edge < w.T)]
    if edge.size > n_sample:
        edge = rng.choice(edge, n_sample, replace=False)
    rest = rng.choice(w.T, min(n_sample, w.T), replace=False)
    return np.unique(np.concatenate([order[pick], edge, rest])).astype(np.int64)


def run_forward_case(w, n_sample=None, seed=5, variant=B.LORA_VARIANT_AUTO):
    """base GEMM alone and the fused forward vs the oracle (on a row sample for the big configurations, see
    _forward_rows), then the fused forward on ALL rows against base GEMM + lora_delta of the same library."""
    dl = device.to_device(w, DEV, with_w=True)
    tdt = device.torch_dtype(w)
    plan = device.make_plan(w, variant)
    view = B.lora_plan_export(plan)
    R, v_bytes, ws_bytes = B.lora_plan_query(plan)
    tok = oracle.token_adapter(w.T, w.seg_indptr, w.seg_adapter)
    ad = oracle.Adapters(w.adapter_rank, w.adapter_scale, w.A, w.B)
    rows = np.arange(w.T) if (n_sample is None or n_sample >= w.T) else _forward_rows(w, view, n_sample, seed)
    print(f"  forward {w.name} T={w.T} K={w.K} N={w.N} oracle rows={rows.size}", flush=True)
    ws = torch.empty(max(ws_bytes, 256), dtype=torch.uint8, device=DEV)
    y = torch.full((w.T, w.N), 9.0, dtype=tdt, device=DEV)
    B.lora_base_gemm(w.T, w.K, w.N, dl.dtype, dl.x, w.K, dl.Wt, w.K, y, w.N)
    torch.cuda.synchronize()
    base_ref = oracle.base(w.x, w.W, rows=rows)
    _assert_close(_to_np(y)[rows], base_ref, _tol(w), "base gemm")
    y_base = y.clone()

    y.fill_(9.0)
    B.lora_fused_forward(plan, dl.x, w.K, dl.Wt, w.K, dl.At_ptrs, dl.Bt_ptrs, y, w.N, ws, ws.numel())
    torch.cuda.synchronize()
    y_ref = oracle.forward(w.x, w.W, tok, ad, rows=rows)
    _assert_close(_to_np(y)[rows], y_ref, _tol(w), "fused forward")

    # Every row, GPU against GPU: y_fused = rnd(xW + d), y_base = rnd(xW), y_delta = rnd(d) with one rounding each
    # (bf16: relative 2^-8; fp32: 2^-24) on top of fp32 accumulation noise, so element by element
    # |y_fused - (y_base + y_delta)| <= u (|y_fused| + |y_base| + |y_delta|) + accumulation slack.
    # A wrong row, a dropped or doubled adapter stage or a stale operand is an O(1) error.
    if w.T:
        v = torch.zeros(max(v_bytes // 4, 4), dtype=torch.float32, device=DEV)
        y_delta = torch.zeros((w.T, w.N), dtype=tdt, device=DEV)
        B.lora_delta(plan, dl.x, w.K, dl.At_ptrs, dl.Bt_ptrs, v, y_delta, w.N, 0.0)
        torch.cuda.synchronize()
        u = 2.0 ** -8 if w.dtype == "bf16" else 2.0 ** -24
        slack = 1e-4 if w.dtype == "bf16" else 1e-5
        yf, yb, yd = y.float(), y_base.float(), y_delta.float()
        excess = (yf - (yb + yd)).abs() - (1.01 * u * (yf.abs() + yb.abs() + yd.abs()) + slack)
        worst = float(excess.max())
        ranks_tok = np.where(tok >= 0, w.adapter_rank[np.clip(tok, 0, None)], 0) if w.num_adapters else np.zeros(w.T, int)
        none = torch.from_numpy(ranks_tok == 0).to(DEV)
        same = float((y[none] == y_base[none]).float().mean()) if bool(none.any()) else 1.0
        nrm = float(torch.linalg.norm(yf - (yb + yd)) / torch.linalg.norm(yb + yd).clamp_min(1e-30))
        print(f"    fused vs base gemm + lora_delta, all {w.T} rows: normwise {nrm:.3e}, worst excess over the "
              f"rounding bound {worst:.3e}; rows without adapter bit-identical to the base GEMM: {same:.4f}", flush=True)
        assert worst <= 0.0, "fused forward differs from base GEMM + delta by more than the three roundings allow"
        if bool(none.any()):      # no delta: the same product, at most the last bit apart (summation order)
            assert bool(((y[none].float() - y_base[none].float()).abs() <= 2 * u * y_base[none].float().abs() + slack).all())
    plan.destroy()


# ---------------------------------------------------------------- configurations
def test_cfg1_tiny_fp32():
    w = wl.cfg1()
    run_delta_case(w)
    run_forward_case(w)


def test_cfg2_decode():
    w = wl.cfg2()
    view = run_delta_case(w)
    assert view["kernel_family"] == B.LORA_VARIANT_TILED
    run_delta_case(w, B.LORA_VARIANT_GENERAL, check_beta0=False)
    run_forward_case(w)


@pytest.mark.parametrize("projection", [0, 1, 2, 3])
def test_cfg3_prefill(projection):
    w = wl.cfg3(projection)
    run_delta_case(w, check_beta0=(projection == 0))
    run_forward_case(w, n_sample=128)


def test_cfg4_mixed():
    w = wl.cfg4()
    run_delta_case(w, rows=np.arange(0, w.T, 4))
    run_forward_case(w, n_sample=192)


def test_cfg4d_mixed_with_decode_requests():
    w = wl.cfg4d()
    run_delta_case(w, rows=np.arange(0, w.T, 4), check_beta0=False)
    run_forward_case(w, n_sample=192)


@pytest.mark.parametrize("shape", ["attn", "mlp"])
def test_cfg5_large(shape):
    w = wl.cfg5(shape)
    run_delta_case(w, rows=np.arange(0, w.T, 8), check_beta0=False)
    run_forward_case(w, n_sample=128)


@pytest.mark.parametrize("T,K,N,kernel", [(3585, 128, 3600, "tiled"), (3585, 120, 3600, "tiled"), (3600, 72, 3592, "tiled"),
                                           (3600, 160, 3592, "ring"), (3585, 200, 3600, "ring")])
def test_large_tile_gemm_ragged_shapes(T, K, N, kernel):
    """The 256 x 256 tile kernels on ragged T and N with few stages: register-staged with two of 64 k, whole, with one chunk
    missing and with one chunk only in the last; the ring with three and four.  Base GEMM and fused forward, with mixed
    ranks, tokens without adapter and several adapters per tile."""
    w = wl.random_case(700 + K, T, K, N, 40, (8, 16, 24, 32, 64, 128), max_seg=90, frac_none=0.15, scales=(0.5, 2.0))
    assert f"gemm_{kernel}_kernel<delta>" in _launched(lambda: run_forward_case(w, n_sample=160))


@pytest.mark.parametrize("T,K,N,ldx,ranks,kernel", [
    (300, 264, 520, 7200000, (8, 64), "gemm_tiled_kernel<delta>"), (300, 256, 520, 7200000, (128,), "gemm_tiled_kernel<delta>"),
    (3600, 264, 3600, 600000, (8, 64), "gemm_tiled_kernel<delta>"), (3600, 256, 3600, 600000, (16, 128), "gemm_tiled_kernel<delta>"),
    (40, 264, 136, 54000000, (12, 100), "gemm_general_kernel")])
def test_gemm_of_operands_past_four_gigabytes(T, K, N, ldx, ranks, kernel):
    """x with rows so far apart that its last ones start past 2^32 bytes: the register-staged kernel in both tile sizes with
    more than two stages, with and without a K tail, and the general kernel for other ranks; base GEMM and fused forward."""
    w = wl.random_case(720 + T + K, T, K, N, 9, ranks, max_seg=40, frac_none=0.15, scales=(0.5, 2.0))
    dl = device.to_device(w, DEV, with_w=True)
    assert 2 ** 32 <= 2 * T * ldx < 2 ** 32 + 2 ** 26
    x = torch.empty((T, ldx), dtype=torch.bfloat16, device=DEV)
    x[:, :K] = dl.x
    plan = device.make_plan(w)
    ws = torch.empty(max(B.lora_plan_query(plan)[2], 256), dtype=torch.uint8, device=DEV)
    y = torch.full((T, N), 9.0, dtype=torch.bfloat16, device=DEV)
    rows = np.unique(np.concatenate([np.arange(0, T, max(1, T // 150)), [T - 1]]))
    tok = oracle.token_adapter(w.T, w.seg_indptr, w.seg_adapter)
    ad = oracle.Adapters(w.adapter_rank, w.adapter_scale, w.A, w.B)
    B.lora_base_gemm(T, K, N, dl.dtype, x, ldx, dl.Wt, K, y, N)
    torch.cuda.synchronize()
    _assert_close(_to_np(y)[rows], oracle.base(w.x, w.W, rows=rows), BF16_TOL, "base gemm")
    y.fill_(9.0)
    assert kernel in _launched(lambda: B.lora_fused_forward(plan, x, ldx, dl.Wt, K, dl.At_ptrs, dl.Bt_ptrs, y, N, ws, ws.numel()))
    _assert_close(_to_np(y)[rows], oracle.forward(w.x, w.W, tok, ad, rows=rows), BF16_TOL, "fused forward")
    plan.destroy()


@pytest.mark.parametrize("T,K,N", [(2900, 32, 2568), (3000, 72, 1544), (5000, 128, 1160), (1400, 264, 5000), (700, 200, 9000)])
def test_products_of_few_stages(T, K, N):
    """Base products that the register-staged 128 x 128 tiles take: one stage to five, with and without a K tail, ragged T
    and N; against the oracle on a sample of rows."""
    w = wl.random_case(760 + K, T, K, N, 1, (8,), max_seg=T, frac_none=1.0)
    dl = device.to_device(w, DEV, with_w=True)
    y = torch.full((T + 1, N), 9.0, dtype=torch.bfloat16, device=DEV)
    names = _launched(lambda: B.lora_base_gemm(T, K, N, dl.dtype, dl.x, K, dl.Wt, K, y, N))
    assert names == {"gemm_tiled_kernel"}
    rows = np.unique(np.concatenate([np.arange(0, T, max(1, T // 200)), [T - 1]]))
    _assert_close(_to_np(y)[rows], oracle.base(w.x, w.W, rows=rows), BF16_TOL, "base gemm")
    assert bool((y[T] == 9.0).all()) and bool((y[:T] != 9.0).any(dim=1).all())


# every tile of the small GEMM for bf16 (ranks of the tuned kernels and others) and for fp32: see
# test_planner.test_small_gemm_shapes_cover_every_tile
SMALL_GEMM_SHAPES = [(1, 8, 8), (1, 4096, 4096), (15, 72, 40), (17, 1000, 1096), (33, 64, 16), (47, 520, 4104), (65, 128, 2056),
                     (100, 3208, 1000), (129, 584, 4096), (257, 72, 1000), (500, 640, 1480), (511, 136, 72), (16, 1000, 1096),
                     (34, 200, 2056), (45, 520, 6008), (46, 264, 6008), (47, 520, 1480), (48, 200, 4104), (90, 264, 5000), (91, 200, 5000),
                     (131, 520, 2504), (190, 264, 5000), (191, 264, 5000)]


def _small_gemm_case(T, K, N, dtype):
    # ranks up to the largest that are no multiple of the MFMA step, or aligned ones
    ranks = (1, 5, 8, 20, 64, 100, 256) if T % 2 else (8, 16, 64)
    return wl.random_case(1500 + T + K, T, K, N, 9, ranks, dtype=dtype, max_seg=5, frac_none=0.15, scales=(0.5, 2.0, -1.0))


@pytest.mark.parametrize("T,K,N", SMALL_GEMM_SHAPES)
def test_small_batch_gemm_tiles_and_remainders(T, K, N):
    """The GEMM that splits K over the wavefronts of a workgroup: every tile shape its rule picks, remainders of
    tokens and features, fewer units of K than wavefronts, K tails of one chunk, tokens without adapter, mixture mode."""
    w = _small_gemm_case(T, K, N, "bf16")
    names = _launched(lambda: run_forward_case(w))
    assert bool(names & {"gemm_small_kernel<delta>", "layer_small_kernel"}) == (B.lora_gemm_choice(T, K, N, B.LORA_BF16, True)[0] == 1)
    if T > 16:
        run_mixture_case(w, 2)


@pytest.mark.parametrize("adapters,ranks,max_seg", [
    (40, (8, 16, 64), 1), (40, (4, 12, 20), 1), (64, (100, 128), 1), (64, (100, 36), 1), (2, (8, 128), 90), (2, (12, 100), 90), (12, (24, 72), 9)])
@pytest.mark.parametrize("T,K,N,tile", [
    (125, 264, 4104, (4, 4)), (95, 264, 4096, (2, 4)), (90, 264, 4104, (4, 2)), (75, 136, 2056, (2, 2)), (75, 200, 3000, (4, 1)),
    (25, 264, 2056, (1, 2)), (25, 136, 1096, (1, 1))])
def test_small_batch_deltas_in_items_and_in_pairs(T, K, N, tile, adapters, ranks, max_seg):
    """Both ways to share out bf16 deltas, in every tile that has them: many adapters with a row or two each, few that go over
    blocks and tiles, ranks of one step and more, with and without those of the tuned kernels; mixture mode's removal in both."""
    assert B.lora_gemm_choice(T, K, N, B.LORA_BF16, True) == (1, *tile)
    w = wl.random_case(1900 + T + K + adapters, T, K, N, adapters, ranks, max_seg=max_seg, frac_none=0.1, scales=(0.5, 2.0, -1.0))
    run_forward_case(w)
    run_mixture_case(w, int(np.bincount(np.clip(w.seg_adapter, 0, None), minlength=adapters).argmax()))


@pytest.mark.parametrize("wait", [True, False])
@pytest.mark.parametrize("T,K,N,tile,max_seg", [
    (1, 1024, 1000, (1, 1), 1), (7, 72, 264, (1, 1), 5), (25, 1096, 3992, (1, 2), 5), (37, 584, 4096, (2, 2), 5), (16, 520, 11008, (4, 1), 5),
    (20, 512, 13824, (4, 2), 5), (40, 520, 13816, (4, 4), 5), (200, 264, 4104, (4, 2), 5), (61, 1032, 4096, (2, 2), 61),
    (250, 1096, 4096, (4, 4), 150)])
def test_small_batch_shrink_and_gemm_in_one_launch(T, K, N, tile, max_seg, wait):
    """Every tile that takes the shrink into its launch, K tails, one K part and more, remainders of tokens and features,
    tokens without adapter, requests of many tokens and high ranks, factors on 16-byte boundaries and off them.  Every call
    has another x: v of the call before would show.  wait=False: the product never waits for the shrink and computes v itself."""
    assert B.lora_gemm_choice(T, K, N, B.LORA_BF16, True)[1:] == tile
    w = wl.random_case(1700 + T + K, T, K, N, 40 if T == 200 else 9, (8, 16, 40, 64) if max_seg <= 5 else (16, 104, 128),
                       max_seg=max_seg, frac_none=0.15 if T > 1 else 0.0, scales=(0.5, 2.0, -1.0))
    dl = device.to_device(w, DEV, with_w=True)
    plan = device.make_plan(w, tuning=None if wait else {"fused_wait_us": 1})
    _, _, ws_bytes = B.lora_plan_query(plan)
    ad = oracle.Adapters(w.adapter_rank, w.adapter_scale, w.A, w.B)
    tok = oracle.token_adapter(w.T, w.seg_indptr, w.seg_adapter)
    keep = [torch.empty(a.size + 8, dtype=torch.bfloat16, device=DEV) for a in w.A]
    for i, (buf, a) in enumerate(zip(keep, w.A)):
        buf[i % 8:i % 8 + a.size] = torch.from_numpy(np.ascontiguousarray(a.T).ravel()).to(DEV, torch.bfloat16)
    odd = torch.tensor([buf.data_ptr() + 2 * (i % 8) for i, buf in enumerate(keep)], dtype=torch.int64, device=DEV)
    ws = torch.full((ws_bytes,), 255, dtype=torch.uint8, device=DEV)          # (fp32: NaN)
    y = torch.full((T + 1, N), 9.0, dtype=torch.bfloat16, device=DEV)
    for call, At in enumerate((dl.At_ptrs, odd, dl.At_ptrs)):
        x = wl.round_to_bf16(np.random.default_rng(call).standard_normal((T, K)).astype(np.float32))
        xd = torch.from_numpy(x).to(DEV, torch.bfloat16)
        names = _launched(lambda: B.lora_fused_forward(plan, xd, K, dl.Wt, K, At, dl.Bt_ptrs, y, N, ws, ws.numel()))
        torch.cuda.synchronize()
        assert names == {"layer_small_kernel"}, "one launch"
        _assert_close(_to_np(y)[:T], oracle.forward(x, w.W, tok, ad), BF16_TOL, f"fused forward, call {call}")
    assert bool((y[T] == 9.0).all()), "written beyond the last token"
    plan.destroy()


@pytest.mark.parametrize("T,K,N,tile,adapters,rank,one", [
    (64, 520, 4096, (2, 2), 64, 128, False), (62, 520, 2048, (1, 2), 64, 128, False), (48, 520, 4096, (2, 2), 30, 128, True),
    (51, 520, 1024, (1, 1), 32, 64, False), (20, 520, 1024, (1, 1), 11, 64, True), (256, 520, 4096, (4, 4), 256, 64, True)])
def test_small_batch_shrinks_that_crowd_the_product_run_before_it(T, K, N, tile, adapters, rank, one):
    """One launch for shrink and product only where the shrink's workgroups leave the product's their place."""
    assert B.lora_gemm_choice(T, K, N, B.LORA_BF16, True) == (1, *tile)
    w = wl.random_case(1850 + T, T, K, N, adapters, (rank,), max_seg=1)
    dl = device.to_device(w, DEV, with_w=True)
    plan = device.make_plan(w)
    ws = torch.zeros(B.lora_plan_query(plan)[2], dtype=torch.uint8, device=DEV)
    y = torch.zeros((T, N), dtype=torch.bfloat16, device=DEV)
    names = _launched(lambda: B.lora_fused_forward(plan, dl.x, K, dl.Wt, K, dl.At_ptrs, dl.Bt_ptrs, y, N, ws, ws.numel()))
    assert names == ({"layer_small_kernel"} if one else {"shrink_tiled_kernel", "gemm_small_kernel<delta>"})
    ad = oracle.Adapters(w.adapter_rank, w.adapter_scale, w.A, w.B)
    _assert_close(_to_np(y), oracle.forward(w.x, w.W, oracle.token_adapter(w.T, w.seg_indptr, w.seg_adapter), ad), BF16_TOL, "fused forward")
    plan.destroy()


@pytest.mark.parametrize("T,K,N", [(25, 1096, 3992), (37, 584, 4096), (20, 512, 13824), (200, 264, 4104), (64, 4096, 4096)])
def test_small_batch_one_launch_without_waiting_computes_v_itself(T, K, N):
    """Which of its two sources the product takes v from, shown by values that only one of them can sum.  x is zero but for
    2^127, -2^127 next to each other at the start of K and again behind its middle, where every factor is 1 and W is 0.  The
    shrink adds neighbours first: v = 0, y = 0.  The product's own sum runs over K with elements 0 and 2 of every eight apart,
    each reaching 2^128: NaN in every output of a token with an adapter.  fused_wait_us = 1 is no waiting and no looking."""
    w = wl.random_case(1800 + T, T, K, N, 9, (8, 16, 40, 64), max_seg=5, frac_none=0.2, scales=(1.0,))
    dl = device.to_device(w, DEV, with_w=True)
    h = (K + 63) // 64 // 2 * 64
    cols = torch.tensor([0, 2, h, h + 2], device=DEV)
    x = torch.zeros((T, K), dtype=torch.bfloat16, device=DEV)
    x[:, cols] = torch.tensor([2.0 ** 127, -2.0 ** 127] * 2, dtype=torch.bfloat16, device=DEV)
    dl.Wt[:, cols] = 0
    keep = [torch.from_numpy(np.ascontiguousarray(a.T)).to(DEV, torch.bfloat16) for a in w.A]
    for a in keep:
        a[:, cols] = 1
    At = torch.tensor([a.data_ptr() for a in keep], dtype=torch.int64, device=DEV)
    tok = torch.from_numpy(oracle.token_adapter(w.T, w.seg_indptr, w.seg_adapter)).to(DEV)
    for wait in (True, False):
        plan = device.make_plan(w, tuning=None if wait else {"fused_wait_us": 1})
        ws = torch.zeros(B.lora_plan_query(plan)[2], dtype=torch.uint8, device=DEV)
        for _ in range(3):
            y = torch.full((T, N), 9.0, dtype=torch.bfloat16, device=DEV)
            B.lora_fused_forward(plan, x, K, dl.Wt, K, At, dl.Bt_ptrs, y, N, ws, ws.numel())
            torch.cuda.synchronize()
            own = torch.isnan(y) & (tok >= 0)[:, None]
            assert bool((y[tok < 0] == 0).all()), "tokens without adapter"
            if wait:
                assert bool((y == 0).all()), "v of the shrink"
            else:
                assert bool(own[tok >= 0].all()), "v of the product's own"
        plan.destroy()


@pytest.mark.parametrize("T,K,N", SMALL_GEMM_SHAPES + [(70, 100, 77)])
def test_fp32_gemm_tiles_and_remainders(T, K, N):
    """The same kernel in fp32, also with an N that is no multiple of 4.  A sum of n = K + rank fp32 additions whose
    partial sums stay below 4 (outputs of unit variance) carries a rounding error of at most 2^-24 * 4 * sqrt(n / 3) in
    standard deviation; five of them over the smallest |y| that is compared, 1e-2: the elementwise bound."""
    w = _small_gemm_case(T, K, N, "f32")
    dl = device.to_device(w, DEV, with_w=True)
    plan = device.make_plan(w)
    _, _, ws_bytes = B.lora_plan_query(plan)
    ad = oracle.Adapters(w.adapter_rank, w.adapter_scale, w.A, w.B)
    tok = oracle.token_adapter(w.T, w.seg_indptr, w.seg_adapter)
    tol = (1e-5, 5 * 2.0 ** -24 * 4 * np.sqrt((K + 256) / 3) / 1e-2)
    ws = torch.empty(max(ws_bytes, 256), dtype=torch.uint8, device=DEV)
    y = torch.full((T + 1, N), 9.0, dtype=torch.float32, device=DEV)
    B.lora_base_gemm(T, K, N, dl.dtype, dl.x, K, dl.Wt, K, y, N)
    torch.cuda.synchronize()
    _assert_close(_to_np(y)[:T], oracle.base(w.x, w.W), tol, "base gemm")
    y.fill_(9.0)
    B.lora_fused_forward(plan, dl.x, K, dl.Wt, K, dl.At_ptrs, dl.Bt_ptrs, y, N, ws, ws.numel())
    torch.cuda.synchronize()
    _assert_close(_to_np(y)[:T], oracle.forward(w.x, w.W, tok, ad), tol, "fused forward")
    assert bool((y[T] == 9.0).all()), "written beyond the last token"
    plan.destroy()


def _check_f32_delta(w, ld_pad=0, shift=0):
    """lora_shrink, lora_expand and lora_delta in fp32 against the oracle (bound: see
    test_fp32_gemm_tiles_and_remainders).  shift: the factors lie `shift` elements past 16-byte boundaries."""
    dl = device.to_device(w, DEV, with_w=False)
    At, Bt, keep = dl.At_ptrs, dl.Bt_ptrs, []
    if shift:
        ptrs = []
        for M in [a.T for a in w.A] + [b.T for b in w.B]:
            buf = torch.empty(M.size + 8, dtype=torch.float32, device=DEV)
            buf[shift:shift + M.size] = torch.from_numpy(np.ascontiguousarray(M).ravel()).to(DEV)
            keep.append(buf)
            ptrs.append(buf.data_ptr() + 4 * shift)
        At, Bt = (torch.tensor(q, dtype=torch.int64, device=DEV) for q in (ptrs[:w.num_adapters], ptrs[w.num_adapters:]))
    plan = device.make_plan(w, B.LORA_VARIANT_TILED)                   # (small problems would take the general expand)
    R, v_bytes, _ = B.lora_plan_query(plan)
    P = B.lora_plan_export(plan)["v_parts"]
    tok = oracle.token_adapter(w.T, w.seg_indptr, w.seg_adapter)
    ad = oracle.Adapters(w.adapter_rank, w.adapter_scale, w.A, w.B)
    tol = (1e-5, 5 * 2.0 ** -24 * 4 * np.sqrt((w.K + 256) / 3) / 1e-2)
    x = torch.full((w.T, w.K + ld_pad), float("nan"), dtype=torch.float32, device=DEV)
    x[:, :w.K] = torch.from_numpy(np.asarray(w.x, dtype=np.float32)).to(DEV)
    v = torch.full((P, w.T, R), float("nan"), dtype=torch.float32, device=DEV)
    assert v.numel() * 4 == v_bytes
    y0 = torch.from_numpy(_y_in(w)).to(DEV)
    y = torch.full((w.T + 1, w.N + ld_pad), 7.0, dtype=torch.float32, device=DEV)
    ref = oracle.expand(w.x, tok, ad, w.N, y_in=_y_in(w).astype(np.float64))
    none = torch.from_numpy(np.where(tok >= 0, w.adapter_rank[np.clip(tok, 0, None)], 0) == 0).to(DEV)
    B.lora_shrink(plan, x, w.K + ld_pad, At, v)
    rank_tok = np.where(tok >= 0, w.adapter_rank[np.clip(tok, 0, None)], 0)
    valid = np.arange(R)[None, :] < rank_tok[:, None]
    v_np = v.double().sum(0).cpu().numpy()
    assert np.array_equal(~np.isnan(v_np), valid), "v written outside [0, r_a), or not inside"
    _assert_close(np.where(valid, v_np, 0.0), oracle.shrink(w.x, tok, ad, apply_scale=True, R=R), tol, "v")
    for call in ("expand", "delta"):
        for beta in (1.0, 0.0):
            y.fill_(7.0)
            y[:w.T, :w.N] = y0
            if call == "expand":
                B.lora_expand(plan, v, Bt, y, w.N + ld_pad, beta)
            else:
                B.lora_delta(plan, x, w.K + ld_pad, At, Bt, v, y, w.N + ld_pad, beta)
            torch.cuda.synchronize()
            assert bool((y[:w.T, w.N:] == 7.0).all()) and bool((y[w.T] == 7.0).all()), "written outside y"
            assert torch.equal(y[:w.T, :w.N][none], y0[none]), "rows without adapter must stay bit-identical"
            got, want = _to_np(y)[:w.T, :w.N], ref - (0.0 if beta else _y_in(w).astype(np.float64))
            active = ~none.cpu().numpy()
            _assert_close(got[active], want[active], tol, f"{call} beta={beta}")
    plan.destroy()


@pytest.mark.parametrize("T,K,N,ranks,max_seg", [
    (1, 4, 1, (1,), 1), (5, 64, 130, (8, 16), 2), (64, 256, 256, (8,), 16), (33, 252, 127, (64, 33, 1), 9), (40, 268, 513, (5, 48, 17), 30),
    (257, 1024, 1000, (8, 64), 12), (300, 3208, 264, (8, 16, 100, 256), 150), (1000, 132, 520, (3, 20, 64, 128), 500),
    (2100, 512, 256, (64, 128), 2100)])
def test_fp32_adapter_kernels_tiles_and_remainders(T, K, N, ranks, max_seg):
    """The fp32 matrix-core shrink (each of its tiles, K parts, K tails, ranks off 4 and 16), expand (16- and 64-token
    tiles, ranks beyond a load group, N off 4 and 64) and the two in one launch, with padded and odd leading dimensions
    (no 16-byte rows of y, the general shrink) and with factors that are aligned to an element only."""
    w = wl.random_case(1700 + T + K, T, K, N, 5, ranks, dtype="f32", max_seg=max_seg, frac_none=0.15, scales=(0.5, 2.0, -1.0))
    for ld_pad, shift in ((0, 0), (4, 1), (3, 0), (0, 3)):
        _check_f32_delta(w, ld_pad, shift)


@pytest.mark.parametrize("T,K,N,ranks", [(64, 256, 256, (8,)), (33, 252, 127, (64, 33, 1)), (90, 512, 4096, (17, 40)), (40, 4096, 264, (64, 16))])
def test_fp32_delta_leaves_the_v_of_shrink(T, K, N, ranks):
    """lora_delta writes the caller's v as lora_shrink does, bit for bit, in one launch (the first three) as in two."""
    w = wl.random_case(1750 + T + K, T, K, N, 5, ranks, dtype="f32", max_seg=9, frac_none=0.15, scales=(0.5, 2.0, -1.0))
    dl = device.to_device(w, DEV, with_w=False)
    plan = device.make_plan(w)
    n = B.lora_plan_query(plan)[1] // 4
    v = [torch.full((n,), 777.0, dtype=torch.float32, device=DEV) for _ in range(2)]
    y = torch.zeros((T, N), dtype=torch.float32, device=DEV)
    B.lora_shrink(plan, dl.x, K, dl.At_ptrs, v[0])
    B.lora_delta(plan, dl.x, K, dl.At_ptrs, dl.Bt_ptrs, v[1], y, N, 0.0)
    torch.cuda.synchronize()
    assert bool((v[0] != 777.0).any()) and torch.equal(v[0], v[1])
    plan.destroy()


@pytest.mark.parametrize("T,K,ranks,dtype,merged", [
    (64, 256, (8,), "f32", None), (33, 512, (64, 16), "f32", None), (60, 512, (8, 64), "bf16", None), (200, 1024, (8, 12, 200), "bf16", None),
    (64, 256, (8,), "f32", 1), (60, 512, (8, 64), "bf16", 1)])
def test_delta_in_place_and_side_by_side(T, K, ranks, dtype, merged):
    """lora_delta with y = x (K = N), or y a few rows behind x in one buffer, gives the bits of lora_shrink followed by
    lora_expand on buffers of their own; x and y as columns of one buffer those of lora_delta on buffers of their own.  Also
    lora_delta_static."""
    w = wl.random_case(1770 + T + K, T, K, K, 5, ranks, dtype=dtype, max_seg=9, frac_none=0.15, scales=(0.5, 1.0, -1.0))
    dl = device.to_device(w, DEV, with_w=False)
    tdt = device.torch_dtype(w)
    plan = B.lora_plan(T, w.seg_indptr, w.seg_adapter, w.adapter_rank, w.adapter_scale, K, K, dl.dtype, merged_adapter=merged)
    v = torch.zeros(B.lora_plan_query(plan)[1] // 4, dtype=torch.float32, device=DEV)
    B.lora_plan_upload(plan)
    x = dl.x[:, :K].contiguous()

    def apart(x, y, beta):
        y = y.clone()
        B.lora_shrink(plan, x, K, dl.At_ptrs, v)
        B.lora_expand(plan, v, dl.Bt_ptrs, y, K, beta)
        return y

    def call(static, x, ldx, y, ldy, beta):
        if static:
            B.lora_delta_static(plan, x, ldx, dl.At_ptrs, dl.Bt_ptrs, y, ldy, beta)
        else:
            B.lora_delta(plan, x, ldx, dl.At_ptrs, dl.Bt_ptrs, v, y, ldy, beta)

    for static in (False, True) if merged is None else (False,):
        for beta in (1.0, 0.0):
            both = x.clone()
            call(static, both, K, both, K, beta)
            assert torch.equal(both, apart(x, x, beta)), "in place"
            rows = torch.randn((T + 8, K), device=DEV).to(tdt)
            want = apart(rows[:T].clone(), rows[8:].clone(), beta)
            call(static, rows, K, rows[8:], K, beta)
            assert torch.equal(rows[8:], want), "rows of one buffer"
            columns = torch.randn((T, 2 * K + 8), device=DEV).to(tdt)
            columns[:, :K] = x
            want = columns[:, K:2 * K].contiguous()
            call(static, x, K, want, K, beta)
            call(static, columns, 2 * K + 8, columns[:, K:], 2 * K + 8, beta)
            assert torch.equal(columns[:, K:2 * K], want) and torch.equal(columns[:, :K], x), "columns of one buffer"
    plan.destroy()


@pytest.mark.parametrize("T,K,ranks,max_seg", [
    (1, 8, (1,), 1), (3, 72, (2, 5), 1), (20, 1000, (10, 101, 256), 2), (50, 520, (1, 17, 33), 20), (64, 4096, (174, 2), 4),
    (200, 648, (256, 130), 60), (300, 136, (9,), 300), (900, 2120, (4, 100, 255), 200), (3000, 264, (129, 256), 900)])
def test_any_rank_shrink_tiles_and_remainders(T, K, ranks, max_seg):
    """The shrink of bf16 batches with ranks off the tuned kernels: tiles from 16 x 16 to 64 x 64, K parts, fewer units of
    64 k than wavefronts, K tails, remainders of tokens and ranks; factors on 16-byte boundaries and off them (the
    kernel's own general path)."""
    w = wl.random_case(2000 + T + K, T, K, 64, 7, ranks, max_seg=max_seg, frac_none=0.15, scales=(0.5, 2.0, -1.0))
    dl = device.to_device(w, DEV, with_w=False)
    tok = oracle.token_adapter(w.T, w.seg_indptr, w.seg_adapter)
    ad = oracle.Adapters(w.adapter_rank, w.adapter_scale, w.A, w.B)
    ptrs, keep = [], []
    for i, a in enumerate(w.A):
        buf = torch.empty(a.size + 8, dtype=torch.bfloat16, device=DEV)
        buf[i % 7 + 1:i % 7 + 1 + a.size] = torch.from_numpy(np.ascontiguousarray(a.T).ravel()).to(DEV, torch.bfloat16)
        keep.append(buf)
        ptrs.append(buf.data_ptr() + 2 * (i % 7 + 1))
    plan = device.make_plan(w)
    R, v_bytes, _ = B.lora_plan_query(plan)
    P = B.lora_plan_export(plan)["v_parts"]
    x = torch.full((w.T, w.K + 8), float("nan"), dtype=torch.bfloat16, device=DEV)
    x[:, :w.K] = dl.x
    valid = np.arange(R)[None, :] < np.where(tok >= 0, w.adapter_rank[np.clip(tok, 0, None)], 0)[:, None]
    ref = oracle.shrink(w.x, tok, ad, apply_scale=True, R=R)
    for At in (dl.At_ptrs, torch.tensor(ptrs, dtype=torch.int64, device=DEV)):
        v = torch.full((P, w.T, R), float("nan"), dtype=torch.float32, device=DEV)
        B.lora_shrink(plan, x, w.K + 8, At, v)
        torch.cuda.synchronize()
        v_np = v.double().sum(0).cpu().numpy()
        assert np.array_equal(~np.isnan(v_np), valid), "v written outside [0, r_a), or not inside"
        if valid.any():
            _assert_close(np.where(valid, v_np, 0.0), ref, V_TOL, "v")
    plan.destroy()


@pytest.mark.parametrize("dtype,rank,K", [("f32", 16, 71582792), ("bf16", 17, 143165584)])
def test_shrink_of_factors_past_four_gigabytes(dtype, rank, K):
    """The last row of an adapter's At starts past 2^32 bytes behind its first.  Row j of At is one at 100 + j places
    (sums of ones are exact) and zero elsewhere, so a row taken from another place of the matrix shows."""
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    At = torch.zeros((rank, K), dtype=tdt, device=DEV)
    assert (rank - 1) * K * At.element_size() > 2 ** 32
    for j in range(rank):
        At[j, 1000 * j:1000 * j + 100 + j] = 1.0
    x = torch.ones((1, K), dtype=tdt, device=DEV)
    plan = B.lora_plan(1, np.array([0, 1], np.int32), np.array([0], np.int32), np.array([rank], np.int32), np.array([2.0], np.float32),
                       K, 8, B.LORA_F32 if dtype == "f32" else B.LORA_BF16)
    R, v_bytes, _ = B.lora_plan_query(plan)
    v = torch.zeros((v_bytes // (4 * R), R), dtype=torch.float32, device=DEV)
    B.lora_shrink(plan, x, K, torch.tensor([At.data_ptr()], dtype=torch.int64, device=DEV), v)
    torch.cuda.synchronize()
    assert v.sum(0)[:rank].tolist() == [2.0 * (100 + j) for j in range(rank)]
    plan.destroy()


@pytest.mark.parametrize("T,N,ranks,max_seg", [
    (1, 64, (1,), 1), (3, 64, (3, 256), 1), (20, 72, (1, 2, 5, 7), 3), (33, 204, (12, 100, 4), 9), (90, 1000, (9, 33, 65, 129), 30),
    (150, 4100, (255, 31, 256), 60), (400, 520, (17, 63, 127, 8, 256), 200), (1200, 2056, (4, 100, 12, 256, 20, 48), 400)])
def test_any_rank_expand(T, N, ranks, max_seg):
    """The expand for ranks that are no multiple of 8 or above 128: rows of Bt that start and end inside 16-byte chunks,
    the last rows of the matrix (whose chunks would reach past it), every number of token blocks, short feature ranges,
    N off 8 and 64, and factors aligned to an element only; against the oracle and against the general kernel."""
    w = wl.random_case(1800 + T + N, T, 128, N, 5, ranks, max_seg=max_seg, frac_none=0.15, scales=(0.5, 2.0, -1.0))
    ldy = (N + 7) // 8 * 8 + 8
    dl = device.to_device(w, DEV, with_w=False)
    tok = oracle.token_adapter(w.T, w.seg_indptr, w.seg_adapter)
    ad = oracle.Adapters(w.adapter_rank, w.adapter_scale, w.A, w.B)
    ref = oracle.expand(w.x, tok, ad, w.N, y_in=_y_in(w).astype(np.float64))
    rank_tok = np.where(tok >= 0, w.adapter_rank[np.clip(tok, 0, None)], 0)
    none = torch.from_numpy(rank_tok == 0).to(DEV)
    y0 = torch.from_numpy(_y_in(w)).to(DEV, torch.bfloat16)
    ptrs, keep = [], []
    for i, b in enumerate(w.B):                       # Bt_a at 2, 4 .. bytes past a 16-byte boundary
        buf = torch.empty(b.size + 8, dtype=torch.bfloat16, device=DEV)
        buf[i % 7 + 1:i % 7 + 1 + b.size] = torch.from_numpy(np.ascontiguousarray(b.T).ravel()).to(DEV, torch.bfloat16)
        keep.append(buf)
        ptrs.append(buf.data_ptr() + 2 * (i % 7 + 1))
    shifted = torch.tensor(ptrs, dtype=torch.int64, device=DEV)
    out = {}
    for variant in (B.LORA_VARIANT_TILED, B.LORA_VARIANT_GENERAL):
        plan = device.make_plan(w, variant)
        _, v_bytes, _ = B.lora_plan_query(plan)
        v = torch.full((v_bytes // 4,), float("nan"), dtype=torch.float32, device=DEV)
        B.lora_shrink(plan, dl.x, w.K, dl.At_ptrs, v)
        for beta in (1.0, 0.0):
            for Bt in (dl.Bt_ptrs, shifted):
                y = torch.full((w.T + 1, ldy), 7.0, dtype=torch.bfloat16, device=DEV)
                y[:w.T, :w.N] = y0
                B.lora_expand(plan, v, Bt, y, ldy, beta)
                torch.cuda.synchronize()
                assert bool((y[:w.T, w.N:] == 7.0).all()) and bool((y[w.T] == 7.0).all()), "written outside y"
                assert torch.equal(y[:w.T, :w.N][none], y0[none]), "rows without adapter must stay bit-identical"
                active = ~none.cpu().numpy()
                got, want = _to_np(y)[:w.T, :w.N], ref - (0.0 if beta else _y_in(w).astype(np.float64))
                _assert_close(got[active], want[active], BF16_TOL, f"variant {variant} beta {beta}")
                out.setdefault(beta, y.clone())
                # one rounding each of sums that differ by their order alone (and by v's split, 2^-16): a bf16 ulp apart at most
                assert bool(((out[beta].float() - y.float()).abs() <= 2.0 ** -7 * y.float().abs() + 1e-4).all())
        plan.destroy()


@pytest.mark.parametrize("T,N,ranks,dtype,kernel", [
    (16, 7700, (91, 92), "bf16", "expand_rows_kernel"), (16, 7400, (91, 92), "bf16", "expand_general_kernel"),
    (700, 1160, (7, 8), "f32", "expand_rows_kernel"), (700, 1060, (7, 8), "f32", "expand_general_kernel"), (700, 40, (17, 20), "f32", "expand_rows_kernel")])
def test_expand_takes_the_general_kernel_where_it_is_faster(T, N, ranks, dtype, kernel):
    """Either side of the line between the general and the any-rank expand; both against the oracle."""
    w = wl.random_case(1850 + T + N, T, 2304, N, 3, ranks, dtype=dtype, max_seg=60, scales=(0.5, -1.0))
    weight = int((w.adapter_rank[oracle.token_adapter(w.T, w.seg_indptr, w.seg_adapter)] + 8).sum()) * N
    assert (weight >= 12000000) == (kernel == "expand_rows_kernel") or ranks == (17, 20), weight
    names = _launched(lambda: run_delta_case(w))
    assert kernel in names and len([n for n in names if "expand" in n]) == 1, names


@pytest.mark.parametrize("T,N,ranks", [
    (960, 4100, (4, 20, 31)), (1040, 4100, (32, 1)), (1100, 4100, (12,)), (2600, 4100, (4, 20)), (2600, 1000, (4, 31)), (2600, 4352, (9, 32, 17)),
    (1550, 4100, (90, 100)), (3000, 2060, (84, 100)), (3500, 4100, (255, 200)), (750, 4100, (4, 100, 256)), (333, 2060, (12, 131, 7))])
def test_any_rank_expand_of_one_step(T, N, ranks):
    """Ranks of one MFMA step: about 1000 and 2600 tiles of 16 tokens x 256 features, from where two and four blocks of
    features share a tile, and their remainders (N of 4, 17 and a bit, and 17 blocks); higher ranks of about one length, where two or four
    blocks make a full round of tiles; ranks above 128 in tiles of 16 tokens among short ones; against the oracle and, every value,
    against one rounding of the general kernel's sum."""
    w = wl.random_case(1850 + T + N, T, 64, N, 3, ranks, max_seg=90, frac_none=0.1, scales=(0.5, 2.0, -1.0))
    dl = device.to_device(w, DEV, with_w=False)
    tok = oracle.token_adapter(w.T, w.seg_indptr, w.seg_adapter)
    ad = oracle.Adapters(w.adapter_rank, w.adapter_scale, w.A, w.B)
    out = []
    for variant in (B.LORA_VARIANT_AUTO, B.LORA_VARIANT_GENERAL):
        plan = device.make_plan(w, variant)
        v = torch.zeros(max(B.lora_plan_query(plan)[1] // 4, 4), dtype=torch.float32, device=DEV)
        y = torch.from_numpy(_y_in(w)).to(DEV, torch.bfloat16)
        names = _launched(lambda: B.lora_delta(plan, dl.x, w.K, dl.At_ptrs, dl.Bt_ptrs, v, y, N, 1.0))
        assert ("expand_rows_kernel" in names) == (variant == B.LORA_VARIANT_AUTO), names
        out.append(_to_np(y))
        plan.destroy()
    _assert_close(out[0], oracle.expand(w.x, tok, ad, w.N, y_in=_y_in(w).astype(np.float64)), BF16_TOL, "delta")
    # two roundings of sums that agree to fp32's accuracy: one unit in the last place, 2^-7 at most
    assert np.all(np.abs(out[0] - out[1]) <= 2.0 ** -7 * np.abs(out[1]) + 1e-4)


@pytest.mark.parametrize("T,K,N,ranks,max_seg,parts,shapes", [
    (300, 1024, 4104, (16, 64), 150, 1, {(4, 1), (2, 1)}), (500, 1024, 4104, (128,), 500, 1, {(2, 1), (2, 2)}),
    (600, 1024, 8200, (24, 128), 200, 1, {(2, 2), (2, 3), (8, 2), (8, 3)}),
    (900, 1024, 8200, (64, 8), 400, 1, {(2, 0), (2, 1), (4, 0), (4, 1), (8, 0), (8, 1)}),
    (1300, 1024, 8200, (16, 64, 128), 300, 1, {(2, 1), (4, 1), (4, 3)}), (1500, 1024, 9000, (64,), 700, 1, {(2, 0), (2, 3), (4, 0)}),
    (700, 1024, 13832, (128,), 700, 1, {(2, 1), (2, 2)}), (9000, 1024, 8200, (16,), 1500, 2, {(1, 1), (1, 2), (2, 1), (2, 2)}),
    (16500, 1024, 4104, (64, 16), 2000, 2, {(1, 1), (2, 3)}), (16500, 1024, 4360, (64,), 2000, 2, {(1, 2), (1, 3)}),
    (7500, 2048, 9000, (128,), 2000, 4, {(1, 2), (1, 3), (2, 1), (2, 2)}), (7500, 2048, 9064, (16, 128, 64), 2000, 4, {(1, 0), (1, 2)}),
    (9000, 2048, 4104, (16, 64), 900, 4, {(2, 1), (2, 2), (4, 0), (4, 1)}), (2500, 8192, 4104, (128, 64), 700, 4, {(2, 1), (2, 3), (4, 1), (4, 2)})])
def test_streaming_expand_of_whole_rounds_of_stages_and_what_is_left(T, K, N, ranks, max_seg, parts, shapes):
    """Tiles whose feature ranges the planner makes as long as the rounds of the compute units ask for: one, two, four and eight
    64-feature chunks a stage, each with whole rounds of four stages and with one, two and three stages left (shapes: chunks and
    stages left, of all tiles), behind v in one, two and four K parts; remainders of tokens and features; beta 0 and 1; nothing
    written between the rows of y."""
    w = wl.random_case(2500 + T + N, T, K, N, 4, ranks, max_seg=max_seg, frac_none=0.1, scales=(0.5, 2.0, -1.0))
    dl = device.to_device(w, DEV, with_w=False)
    tok = oracle.token_adapter(w.T, w.seg_indptr, w.seg_adapter)
    ad = oracle.Adapters(w.adapter_rank, w.adapter_scale, w.A, w.B)
    plan = device.make_plan(w)
    view = B.lora_plan_export(plan)
    chunks = view["expand_tiles"][:, 5] >> 4 & 15
    assert view["v_parts"] == parts and set(zip(chunks.tolist(), (-(-view["expand_tiles"][:, 4] // (64 * chunks)) % 4).tolist())) == shapes
    v = torch.zeros(B.lora_plan_query(plan)[1] // 4, dtype=torch.float32, device=DEV)
    y0 = torch.from_numpy(_y_in(w)).to(DEV, torch.bfloat16)
    rows = np.arange(T) if T * N < 1 << 24 else np.sort(np.random.default_rng(T).choice(T, size=1 << 11, replace=False))
    ref = oracle.expand(w.x, tok, ad, N, rows=rows)
    has = np.where(tok >= 0, w.adapter_rank[np.clip(tok, 0, None)], 0) > 0
    for beta in (1.0, 0.0):
        y = torch.full((T, N + 8), 9.0, dtype=torch.bfloat16, device=DEV)
        y[:, :N] = y0
        names = _launched(lambda: B.lora_delta(plan, dl.x, w.K, dl.At_ptrs, dl.Bt_ptrs, v, y, N + 8, beta))
        assert "expand_stream_kernel" in names, names
        assert bool((y[:, N:] == 9.0).all()) and torch.equal(y[torch.from_numpy(~has), :N], y0[torch.from_numpy(~has)])
        got, was = _to_np(y[rows, :N]), _to_np(y0[rows]).astype(np.float64)
        _assert_close(got[has[rows]], (ref + was * beta)[has[rows]], BF16_TOL, f"delta, beta {beta}")
    plan.destroy()


def _one_adapter_plan(T, K, N, rank, variant=B.LORA_VARIANT_TILED):
    return B.lora_plan(T, np.array([0, T], np.int32), np.array([0], np.int32), np.array([rank], np.int32), np.array([1.0], np.float32),
                       K, N, B.LORA_BF16, variant)


@pytest.mark.parametrize("rank", [2, 12, 100, 256])
def test_any_rank_expand_uses_all_bits_of_v(rank):
    """v holds 1 + 2^-10 + 2^-23 and 1 + 2^-10, Bt the same power of two with opposite signs: in fp32 every product and sum
    is exact and 2^-23 of it is left; with less than the 24 bits of v, nothing."""
    T, N = 37, 200
    plan = _one_adapter_plan(T, 64, N, rank)
    R, v_bytes, _ = B.lora_plan_query(plan)
    v = torch.zeros((v_bytes // (4 * T * R), T, R), dtype=torch.float32, device=DEV)
    Bt = torch.zeros((N, rank), dtype=torch.bfloat16, device=DEV)
    b = 2.0 ** (torch.arange(N, device=DEV) % 7).float()
    j0, j1 = 0, rank - 1
    v[0, :, j0], v[0, :, j1] = 1 + 2.0 ** -10 + 2.0 ** -23, 1 + 2.0 ** -10
    Bt[:, j0], Bt[:, j1] = b.bfloat16(), -b.bfloat16()
    y = torch.full((T, N), 5.0, dtype=torch.bfloat16, device=DEV)
    B.lora_expand(plan, v, torch.tensor([Bt.data_ptr()], dtype=torch.int64, device=DEV), y, N, 0.0)
    torch.cuda.synchronize()
    assert torch.equal(y.float(), (b * 2.0 ** -23).expand(T, N))
    plan.destroy()


def _non_finite_rows(T, R, N, rank):
    """v rows and a Bt whose products are infinities, NaN and numbers that a v beyond bf16's largest value leads to"""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(rank)
    v = torch.randn((T, R), generator=gen, device=DEV)
    Bt = torch.randn((N, rank), generator=gen, device=DEV).abs().clamp_min(0.1).bfloat16()
    inf, top = float("inf"), float(np.float32(3.4e38))                 # (bf16 rounds 3.4e38 to infinity)
    v[0, 0], v[1, rank - 1], v[2, 0], v[3, 0] = inf, -inf, float("nan"), top
    v[4, 0], v[4, rank - 1] = inf, -inf
    v[5, :] = 1.0                                                      # one bf16 term, the others zero
    Bt[:, 0] = torch.where(torch.arange(N, device=DEV) % 5 == 0, 0.0, 2.0 ** -10).bfloat16()      # (row 0 of v: infinity times zero)
    Bt[7, rank // 2], Bt[8, rank // 2] = inf, -inf
    return v, Bt


@pytest.mark.parametrize("rank", [2, 12, 100, 256])
def test_any_rank_expand_of_infinities(rank):
    """Infinities and NaN in v and Bt come out as from fp32 products: against the general kernel."""
    T, N = 21, 203
    out = []
    for variant in (B.LORA_VARIANT_TILED, B.LORA_VARIANT_GENERAL):
        plan = _one_adapter_plan(T, 64, N, rank, variant)
        R, v_bytes, _ = B.lora_plan_query(plan)
        rows, Bt = _non_finite_rows(T, R, N, rank)
        v = torch.zeros((v_bytes // (4 * T * R), T, R), dtype=torch.float32, device=DEV)
        v[0] = rows
        y = torch.ones((T, N), dtype=torch.bfloat16, device=DEV)
        B.lora_expand(plan, v, torch.tensor([Bt.data_ptr()], dtype=torch.int64, device=DEV), y, N, 1.0)
        torch.cuda.synchronize()
        out.append(y.float())
        plan.destroy()
    got, want = out
    assert bool(torch.isinf(want[0]).any()) and bool(torch.isfinite(want[3]).any()) and bool(torch.isinf(want[6:, 7]).all())
    assert torch.equal(torch.isnan(got), torch.isnan(want))
    assert torch.equal(got[torch.isinf(want)], want[torch.isinf(want)]) and torch.equal(torch.isinf(got), torch.isinf(want))
    f = torch.isfinite(want)
    assert bool(((got[f] - want[f]).abs() <= 2.0 ** -7 * want[f].abs() + 1e-4).all())


def test_large_batch_expand_writes_nothing_past_an_n_off_eight():
    """N no multiple of 8 under a padded leading dimension, a batch that would take the streaming kernels: the columns
    between N and ldy stay as they are."""
    run_delta_case(wl.random_case(1900, 1100, 1024, 204, 9, (16, 64), max_seg=200, frac_none=0.1, scales=(1.0, -0.5)), ld_pad=4)


@pytest.mark.parametrize("T,dtype,ranks", [(90, "f32", (8, 20)), (90, "bf16", (5, 100)), (700, "bf16", (5, 100))])
def test_general_variant_runs_the_general_kernels(T, dtype, ranks):
    """A plan made with LORA_VARIANT_GENERAL, in fp32 or with ranks off the tuned kernels: no matrix-core kernel runs."""
    w = wl.random_case(2400 + T, T, 264, 520, 6, ranks, dtype=dtype, max_seg=7, frac_none=0.2)
    dl = device.to_device(w, DEV, with_w=True)
    plan = device.make_plan(w, B.LORA_VARIANT_GENERAL)
    ws = torch.empty(max(B.lora_plan_query(plan)[2], 256), dtype=torch.uint8, device=DEV)
    y = torch.empty((T, w.N), dtype=device.torch_dtype(w), device=DEV)
    names = _launched(lambda: B.lora_fused_forward(plan, dl.x, w.K, dl.Wt, w.K, dl.At_ptrs, dl.Bt_ptrs, y, w.N, ws, ws.numel()))
    assert names == {"shrink_general_kernel", "gemm_general_kernel"}
    tok = oracle.token_adapter(w.T, w.seg_indptr, w.seg_adapter)
    ad = oracle.Adapters(w.adapter_rank, w.adapter_scale, w.A, w.B)
    _assert_close(_to_np(y), oracle.forward(w.x, w.W, tok, ad), _tol(w), "fused forward")
    plan.destroy()


ANY_RANK_FUSED = [(40, 520, 12, "gemm_small_kernel<delta>"), (100, 1000, 100, "gemm_small_kernel<delta>"),
                  (700, 5000, 12, "gemm_mid_kernel<delta>"), (520, 2000, 256, "gemm_mid_kernel<delta>")]


def _fused_one_adapter(x, W, At, Bt, variant=B.LORA_VARIANT_AUTO):
    """lora_fused_forward of one adapter on every second request of three tokens; (output, kernels)"""
    (T, K), (N, r) = x.shape, Bt.shape
    offsets = np.append(np.arange(0, T, 3), T).astype(np.int32)
    plan = B.lora_plan(T, offsets, (np.arange(len(offsets) - 1) % 2 - 1).astype(np.int32), np.array([r], np.int32), np.array([1.0], np.float32),
                       K, N, B.LORA_BF16, variant)
    ws = torch.empty(max(B.lora_plan_query(plan)[2], 256), dtype=torch.uint8, device=DEV)
    y = torch.full((T, N), 7.0, dtype=torch.bfloat16, device=DEV)
    A, Bp = (torch.tensor([m.data_ptr()], dtype=torch.int64, device=DEV) for m in (At, Bt))
    names = _launched(lambda: B.lora_fused_forward(plan, x, K, W, K, A, Bp, y, N, ws, ws.numel()))
    plan.destroy()
    return y.float(), names, torch.arange(T, device=DEV) // 3 % 2 == 1


@pytest.mark.parametrize("T,N,rank,kernel", ANY_RANK_FUSED)
def test_any_rank_fused_forward_uses_all_bits_of_v(T, N, rank, kernel):
    """v is 1 + 2^-10 + 2^-23 and 1 + 2^-10 (exact sums of At), Bt the same power of two with opposite signs, W zero: in
    fp32 2^-23 of it is left; with less than the 24 bits of v, nothing."""
    K = 264
    x, W = torch.ones((T, K), device=DEV).bfloat16(), torch.zeros((N, K), dtype=torch.bfloat16, device=DEV)
    At, Bt = torch.zeros((rank, K), dtype=torch.bfloat16, device=DEV), torch.zeros((N, rank), dtype=torch.bfloat16, device=DEV)
    At[0, 0], At[0, 100], At[0, 200] = 1.0, 2.0 ** -10, 2.0 ** -23
    At[rank - 1, 0], At[rank - 1, 100] = 1.0, 2.0 ** -10
    b = 2.0 ** (torch.arange(N, device=DEV) % 7).float()
    Bt[:, 0], Bt[:, rank - 1] = b.bfloat16(), -b.bfloat16()
    y, names, on = _fused_one_adapter(x, W, At, Bt)
    assert kernel in names
    assert torch.equal(y, torch.where(on[:, None], b * 2.0 ** -23, 0.0))


@pytest.mark.parametrize("T,N,rank,kernel", ANY_RANK_FUSED)
def test_any_rank_fused_forward_of_infinities(T, N, rank, kernel):
    """An infinite v, one beyond bf16's largest value, and infinities in Bt come out as from fp32 products: against the
    general kernel.  (v overflows in its sum; x itself is finite.)"""
    K = 264
    gen = torch.Generator(device=DEV)
    gen.manual_seed(T)
    x, W = torch.randn((T, K), generator=gen, device=DEV).bfloat16(), (torch.randn((N, K), generator=gen, device=DEV) / 16).bfloat16()
    x[:, :40] = 0.0
    At = (torch.randn((rank, K), generator=gen, device=DEV) / 16).bfloat16()
    Bt = torch.randn((N, rank), generator=gen, device=DEV).abs().clamp_min(0.1).bfloat16()
    At[:, :40] = 0.0
    At[0, 0], At[rank - 1, 1], At[:, 2] = 2.0 ** 100, -2.0 ** 100, 1.0
    for i in range(10):
        At[0, 20 + i] = 2.0 ** (127 - i)                               # their sum: beyond bf16's largest value, below fp32's
    Bt[:, 0] = torch.where(torch.arange(N, device=DEV) % 5 == 0, 0.0, 2.0 ** -10).bfloat16()
    Bt[7, rank // 2], Bt[8, rank // 2] = float("inf"), -float("inf")
    x[3, 0] = x[4, 1] = x[5, 0] = x[5, 1] = 2.0 ** 100                 # (requests of three tokens, the second and fourth on the adapter)
    x[9, 20:30] = 1.0
    x[10, 40:], x[10, 2] = 0.0, 1.0                                    # v = 1 everywhere: one bf16 term, the others zero
    got, names, on = _fused_one_adapter(x, W, At, Bt)
    want, general, _ = _fused_one_adapter(x, W, At, Bt, B.LORA_VARIANT_GENERAL)
    assert kernel in names and "gemm_general_kernel" in general
    assert bool(torch.isinf(want[3]).any()) and bool(torch.isnan(want[3]).any()) and bool(torch.isfinite(want[9, 9:]).all())
    assert bool(torch.isinf(want[10, 7])) and bool(torch.isfinite(want[~on]).all())
    assert torch.equal(torch.isnan(got), torch.isnan(want))
    assert torch.equal(got[torch.isinf(want)], want[torch.isinf(want)]) and torch.equal(torch.isinf(got), torch.isinf(want))
    f = torch.isfinite(want)
    assert bool(((got[f] - want[f]).abs() <= 2.0 ** -7 * want[f].abs() + 1e-3).all())


@pytest.mark.parametrize("T,N,dtype,ranks,kernel", [
    (90, 520, "f32", (8, 20), "small"), (90, 520, "bf16", (8, 16), "small"), (90, 520, "bf16", (5, 100), "small"),
    (700, 5000, "bf16", (8, 16), "mid"), (700, 5000, "bf16", (5, 100), "mid"), (3585, 3600, "bf16", (8, 16), "ring"),
    (95, 4096, "bf16", (8, 16), "small"), (2049, 3080, "bf16", (8, 16), "mid"), (2049, 3080, "bf16", (5, 100), "mid")])
def test_fused_forward_keeps_an_adapters_infinities_to_its_tokens(T, N, dtype, ranks, kernel):
    """One adapter's factors hold infinities and NaN: the tokens of all other adapters, and of none, come out bit for bit
    as with that adapter's factors finite (small GEMM, medium of 128 or 192 and of 256 features, ring, fp32 and any rank)."""
    w = wl.random_case(2300 + T + ranks[0], T, 264, N, 6, ranks, dtype=dtype, max_seg=7, frac_none=0.2)
    dl = device.to_device(w, DEV, with_w=True)
    tdt = device.torch_dtype(w)
    plan = device.make_plan(w)
    ws = torch.empty(max(B.lora_plan_query(plan)[2], 256), dtype=torch.uint8, device=DEV)
    tok = oracle.token_adapter(w.T, w.seg_indptr, w.seg_adapter)
    bad = int(tok[tok >= 0][0])
    out, keep = [], []
    for fill in (None, float("inf"), float("nan")):
        Bt = dl.Bt_ptrs
        if fill is not None:
            keep.append(torch.full((w.N, int(w.adapter_rank[bad])), fill, dtype=tdt, device=DEV))
            Bt = Bt.clone()
            Bt[bad] = keep[-1].data_ptr()
        y = torch.empty((w.T, w.N), dtype=tdt, device=DEV)
        names = _launched(lambda: B.lora_fused_forward(plan, dl.x, w.K, dl.Wt, w.K, dl.At_ptrs, Bt, y, w.N, ws, ws.numel()))
        assert names & {f"gemm_{kernel}_kernel<delta>", f"layer_{kernel}_kernel"}
        assert (T == 2049) == (kernel == "mid" and B.lora_gemm_choice(T, w.K, N, B.LORA_BF16, True)[0] == 7)
        out.append(y)
    others = torch.from_numpy(tok != bad).to(DEV)
    assert bool(others.any()) and bool(torch.isfinite(out[0]).all())
    for y in out[1:]:
        assert torch.equal(y[others], out[0][others])
        assert not bool(torch.isfinite(y[~others]).any())
    plan.destroy()


@pytest.mark.parametrize("T,K,N,ranks", [
    (600, 8, 3000, (8, 16)), (513, 72, 4104, (8, 16, 64)), (640, 264, 2000, (24, 128)), (1025, 328, 2056, (1, 5, 20, 100, 256)),
    (777, 136, 5000, (8, 64)), (777, 200, 5000, (16, 128)), (700, 264, 5000, (3, 8, 100)), (777, 1160, 5000, (8, 64, 128)),
    (1111, 640, 5120, (16, 64)), (1111, 264, 5120, (16, 64)), (1300, 200, 776, (8, 12, 64)), (2049, 1032, 1032, (64,)), (1400, 328, 1544, (16, 32))])
def test_medium_batch_gemm_stages_and_remainders(T, K, N, ranks):
    """The GEMM of 128-token tiles in both widths: fewer stages than its ring holds, as many, one more, K tails of one
    chunk and of all but one; remainders of tokens and features; any rank; tokens without adapter, mixture mode."""
    # (scales of one magnitude s: rounding W' costs u sqrt(1 + s_m^2) and y itself u sqrt(1 + s_own^2), so mixture mode
    # stays within u sqrt(2) = 2.4e-3 of plain inference, under run_mixture_case's bound, only where s_m is not the larger)
    w = wl.random_case(1600 + T + K, T, K, N, 12, ranks, max_seg=60, frac_none=0.15, scales=(1.0, -1.0))
    assert "gemm_mid_kernel<delta>" in _launched(lambda: run_forward_case(w, n_sample=256))
    run_mixture_case(w, 2, n_sample=256)


@pytest.mark.parametrize("T,K,N,kernel", [
    (557, 2056, 1896, 6), (250, 1400, 4104, 6), (125, 2104, 11000, 6), (300, 2112, 4096, 6), (385, 4096, 4088, 6), (65, 4152, 13000, 6),
    (640, 8, 4096, 2), (650, 264, 4104, 2), (700, 1096, 4104, 2), (1300, 72, 776, 2), (1100, 200, 5000, 3), (1100, 264, 5000, 3), (1280, 1096, 4096, 3),
    (1025, 1608, 968, 6), (1100, 2104, 904, 6), (2049, 1672, 520, 6), (4097, 1544, 232, 6), (12289, 1992, 72, 6),
    (513, 1544, 4104, 2), (385, 2104, 5000, 2), (513, 1600, 4096, 2), (1100, 1544, 4104, 3), (777, 2104, 5000, 3), (1100, 1600, 4096, 3)])
def test_medium_base_gemm_k_steps_in_two_halves(T, K, N, kernel):
    """Products without adapters in the 64, 128 and 192 features of the medium GEMM, whose wavefronts take one of a stage's two
    k-steps each: K tails of one chunk, of all but one and none, fewer stages than the ring holds (where the choice goes
    there), remainders of tokens and features, one token past a tile; rows apart; and the fused forward of a batch without
    adapters."""
    assert B.lora_gemm_choice(T, K, N, B.LORA_BF16, False)[0] == kernel
    w = wl.random_case(1750 + T + K, T, K, N, 1, (8,), max_seg=T, frac_none=1.0)
    w.seg_adapter[:] = -1
    dl = device.to_device(w, DEV, with_w=True)
    ref = oracle.base(w.x, w.W)
    y = torch.full((T + 1, N), 9.0, dtype=torch.bfloat16, device=DEV)
    assert _launched(lambda: B.lora_base_gemm(T, K, N, dl.dtype, dl.x, K, dl.Wt, K, y, N)) == {"gemm_mid_kernel"}
    _assert_close(_to_np(y)[:T], ref, BF16_TOL, "base gemm")
    plan = device.make_plan(w)
    ws = torch.empty(max(B.lora_plan_query(plan)[2], 256), dtype=torch.uint8, device=DEV)
    z = torch.full((T + 1, N), 9.0, dtype=torch.bfloat16, device=DEV)
    B.lora_fused_forward(plan, dl.x, K, dl.Wt, K, dl.At_ptrs, dl.Bt_ptrs, z, N, ws, ws.numel())
    torch.cuda.synchronize()
    assert torch.equal(z, y) and bool((y[T] == 9.0).all())
    plan.destroy()
    # rows apart, each by another distance: the same tiles, the same sums; nothing written between the rows of y
    xs, ws, ys = (torch.full((rows, width), 9.0, dtype=torch.bfloat16, device=DEV) for rows, width in ((T, K + 8), (N, K + 24), (T, N + 16)))
    xs[:, :K], ws[:, :K] = dl.x.view(T, K), dl.Wt.view(N, K)
    assert _launched(lambda: B.lora_base_gemm(T, K, N, dl.dtype, xs, K + 8, ws, K + 24, ys, N + 16)) == {"gemm_mid_kernel"}
    assert torch.equal(ys[:, :N], y[:T]) and bool((ys[:, N:] == 9.0).all())


@pytest.mark.parametrize("T,K,N,ranks", [
    (1300, 8, 5000, (8, 16)), (1153, 136, 5000, (24, 128)), (1500, 200, 4104, (1, 5, 20, 100, 256)), (2049, 264, 3080, (8, 64, 128)),
    (6000, 72, 1032, (64,)), (1500, 328, 4104, (16, 64))])
def test_wide_tiles_of_the_medium_gemm_with_adapters(T, K, N, ranks):
    """Tiles of 128 tokens x 256 features: fewer stages than the ring of three holds, as many, more; K tails of one chunk, of
    all but one and half; one token past a tile, remainders of tokens and features; any rank, tokens without adapter, mixture mode."""
    assert B.lora_gemm_choice(T, K, N, B.LORA_BF16, True)[0] == 7
    w = wl.random_case(2100 + T + K, T, K, N, 12, ranks, max_seg=60, frac_none=0.15, scales=(1.0, -1.0))
    assert "gemm_mid_kernel<delta>" in _launched(lambda: run_forward_case(w, n_sample=256))
    run_mixture_case(w, 2, n_sample=256)


@pytest.mark.parametrize("T,K,N", [(1153, 1096, 5000), (1500, 1536, 4104), (1300, 1544, 5000), (2049, 1592, 3080), (1500, 1600, 4104), (3325, 2104, 2056)])
def test_wide_tiles_of_the_medium_base_gemm(T, K, N):
    """... without adapters, up to 24 stages in one chain of k-steps and above in two, with and without a K tail; rows apart,
    nothing written behind the last row or between the rows of y."""
    assert B.lora_gemm_choice(T, K, N, B.LORA_BF16, False)[0] == 7
    w = wl.random_case(2300 + T + K, T, K, N, 1, (8,), max_seg=T)
    dl = device.to_device(w, DEV, with_w=True)
    y = torch.full((T + 1, N), 9.0, dtype=torch.bfloat16, device=DEV)
    assert _launched(lambda: B.lora_base_gemm(T, K, N, dl.dtype, dl.x, K, dl.Wt, K, y, N)) == {"gemm_mid_kernel"}
    _assert_close(_to_np(y)[:T], oracle.base(w.x, w.W), BF16_TOL, "base gemm")
    assert bool((y[T] == 9.0).all())
    xs, ws, ys = (torch.full((rows, width), 9.0, dtype=torch.bfloat16, device=DEV) for rows, width in ((T, K + 8), (N, K + 24), (T, N + 16)))
    xs[:, :K], ws[:, :K] = dl.x.view(T, K), dl.Wt.view(N, K)
    B.lora_base_gemm(T, K, N, dl.dtype, xs, K + 8, ws, K + 24, ys, N + 16)
    assert torch.equal(ys[:, :N], y[:T]) and bool((ys[:, N:] == 9.0).all())


@pytest.mark.parametrize("T,K,N", [(640, 8, 4096), (1300, 72, 776), (650, 264, 4104), (640, 1536, 4096), (1100, 200, 5000), (1280, 1480, 4096),
                                   (1280, 1536, 4096)])
def test_short_medium_products_are_summed_in_one_chain(T, K, N):
    """Up to 24 stages the base product goes through K step by step, as the product with adapters does (two sums, one for either
    k-step, take longer to meet than they save): the bits of the fused forward whose adapter adds zeros."""
    assert B.lora_gemm_choice(T, K, N, B.LORA_BF16, False)[0] == B.lora_gemm_choice(T, K, N, B.LORA_BF16, True)[0] in (2, 3)
    w = wl.random_case(1900 + T + K, T, K, N, 1, (8,), max_seg=T, frac_none=0.0)
    dl = device.to_device(w, DEV, with_w=True)
    zeros = torch.zeros((N, 8), dtype=torch.bfloat16, device=DEV)
    Bt_ptrs = torch.full((1,), zeros.data_ptr(), dtype=torch.int64, device=DEV)
    plan = device.make_plan(w)
    ws = torch.empty(B.lora_plan_query(plan)[2], dtype=torch.uint8, device=DEV)
    y, z = (torch.full((T, N), 9.0, dtype=torch.bfloat16, device=DEV) for _ in range(2))
    assert _launched(lambda: B.lora_base_gemm(T, K, N, dl.dtype, dl.x, K, dl.Wt, K, y, N)) == {"gemm_mid_kernel"}
    assert "gemm_mid_kernel<delta>" in _launched(
        lambda: B.lora_fused_forward(plan, dl.x, K, dl.Wt, K, dl.At_ptrs, Bt_ptrs, z, N, ws, ws.numel()))
    assert torch.equal(y, z)
    plan.destroy()


@pytest.mark.parametrize("K", [136, 184, 192, 248, 320, 648])
def test_ring_gemm_shortest_rings_and_k_tails(K):
    """The 256 x 256 ring at its fewest stages (three of 64 k: prologue and drain only), one and two more, with and
    without chunks past K in the last stage (one chunk in, one chunk missing); ragged T and N, so that the last tiles
    clamp their rows; base GEMM, fused forward and mixture mode."""
    w = wl.random_case(740 + K, 3585, K, 3600, 24, (8, 32, 64, 128), max_seg=120, frac_none=0.1, scales=(0.5, 2.0))
    run_forward_case(w, n_sample=96)
    run_mixture_case(w, 3, n_sample=96)


@pytest.mark.parametrize("K,kernel", [(256, "ring"), (120, "tiled")])
def test_large_tile_gemm_with_hundreds_of_adapters_per_tile(K, kernel):
    """Single-token segments of 400 adapters: a 256-row tile carries about 250 adapters.  The ring kernel's wavefronts then
    walk about 60 adapters each for their 64 rows; the register-staged kernel has far more adapter stages than it caches
    per tile (256), so that it reads the stages beyond its list from memory."""
    w = wl.random_case(811, 3840, K, 3328, 400, (32, 64), max_seg=1, frac_none=0.05)
    assert f"gemm_{kernel}_kernel<delta>" in _launched(lambda: run_forward_case(w, n_sample=160))


@pytest.mark.parametrize("shape", ["decode", "prefill"])
def test_hip_graph_replays_match_the_eager_calls(shape):
    """lora_delta and lora_fused_forward captured into a HIP graph: every replay, with eager calls of the same plan
    and synchronisations in between, gives bit for bit what the eager calls give (the single-launch decode kernel
    keeps hand-off counters across launches; the streaming and GEMM kernels set function attributes on first use)."""
    if shape == "decode":      # one launch for shrink + expand
        w = wl.random_case(901, 180, 512, 768, 24, (8, 16, 32, 64), max_seg=3, frac_none=0.1)
    else:                      # streaming shrink / expand, ring GEMM with adapter stages
        w = wl.random_case(902, 3600, 1024, 3600, 12, (16, 32, 64, 128), max_seg=300, frac_none=0.1)
    dl = device.to_device(w, DEV, with_w=True)
    tdt = device.torch_dtype(w)
    plan = device.make_plan(w)
    R, v_bytes, ws_bytes = B.lora_plan_query(plan)
    B.lora_plan_upload(plan)
    y0 = torch.from_numpy(_y_in(w)).to(DEV, tdt)

    def buffers():
        return (torch.zeros(max(v_bytes // 4, 1), dtype=torch.float32, device=DEV), y0.clone(),
                torch.empty(w.T, w.N, dtype=tdt, device=DEV), torch.empty(max(ws_bytes, 256), dtype=torch.uint8, device=DEV))

    def run(v, y, yf, ws, stream=None):
        B.lora_delta(plan, dl.x, w.K, dl.At_ptrs, dl.Bt_ptrs, v, y, w.N, 1.0, stream)
        B.lora_fused_forward(plan, dl.x, w.K, dl.Wt, w.K, dl.At_ptrs, dl.Bt_ptrs, yf, w.N, ws, ws.numel(), stream)

    v_e, y_e, yf_e, ws_e = buffers()
    run(v_e, y_e, yf_e, ws_e)                                  # eager: also the first use of every kernel
    torch.cuda.synchronize()

    v_g, y_g, yf_g, ws_g = buffers()
    g = torch.cuda.CUDAGraph()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        with torch.cuda.graph(g, stream=side):
            run(v_g, y_g, yf_g, ws_g, side)
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    for replay in range(4):
        y_g.copy_(y0)                                          # lora_delta accumulates onto y
        yf_g.fill_(3.0)
        v_g.fill_(-7.0)
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(y_g, y_e), f"lora_delta: replay {replay} differs from the eager call"
        assert torch.equal(yf_g, yf_e), f"lora_fused_forward: replay {replay} differs from the eager call"
        v2, y2, yf2, ws2 = buffers()                           # eager work of the same plan between the replays
        run(v2, y2, yf2, ws2)
        torch.cuda.synchronize()
        assert torch.equal(y2, y_e) and torch.equal(yf2, yf_e)
    plan.destroy()


# ---------------------------------------------------------------- edge cases
@pytest.mark.parametrize("variant", [B.LORA_VARIANT_TILED, B.LORA_VARIANT_GENERAL])
def test_ragged_small_cases(variant):
    # several tiles and ragged tails: K not a multiple of 32, N not of 64 / 16,
    # tokens without adapter, empty segments, heterogeneous scales, all ranks
    for seed, (T, K, N) in enumerate([(37, 72, 200), (150, 328, 1000), (9, 64, 24), (300, 520, 72)]):
        w = wl.random_case(100 + seed, T, K, N, 7, (8, 16, 24, 32, 40, 64, 128), max_seg=40,
                           frac_none=0.25, scales=(0.5, 1.0, 2.0, -1.5, 3.25), empty_segments=True)
        run_delta_case(w, variant)
        run_delta_case(w, variant, ld_pad=8, check_beta0=False)
        run_forward_case(w, variant=variant)


def test_fused_forward_with_a_single_k_stage():
    # K of at most 64 is one stage of the register-staged GEMM: the first stage fetched ahead is then already an
    # adapter stage, whose descriptors every thread reads from LDS (a missing barrier there once let a workgroup read
    # them before they were written; found by a random sweep).  Many adapters per tile, plain and mixture mode, different
    # batches back to back; batches so large that this kernel takes them, and small ones, which the small and medium
    # GEMMs take.
    for seed, (T, K, N, n_a, ranks, large) in enumerate([(3700, 64, 3400, 9, (64,), True), (3585, 40, 3600, 300, (8, 16, 32), True),
                                                         (3600, 64, 3592, 5, (128,), True), (3850, 32, 3336, 120, (8, 64), True),
                                                         (700, 64, 200, 9, (64,), False), (300, 40, 328, 30, (8, 16, 32), False),
                                                         (520, 64, 136, 5, (128,), False), (130, 32, 72, 12, (8, 64), False)]):
        w = wl.random_case(600 + seed, T, K, N, n_a, ranks, max_seg=3, frac_none=0.1, scales=(1.0, 2.0, -0.5))
        names = _launched(lambda: run_forward_case(w, n_sample=min(T, 160), variant=B.LORA_VARIANT_TILED))
        assert ("gemm_tiled_kernel<delta>" in names) == large, names
        run_mixture_case(w, seed % n_a, n_sample=min(T, 96))


def test_seeded_sweep_of_random_batches():
    # Many small batches drawn from a seeded generator -- token counts from one to a few thousand, K from one GEMM
    # stage to 4096, ragged N, one to 150 adapters, aligned and odd rank sets, segment lengths from decode to
    # prefill -- through lora_delta (both kernel families decide for themselves), the single launch with and without
    # its fallback, the fused forward and mixture mode.  (A sweep like this found the missing barrier that
    # test_fused_forward_with_a_single_k_stage pins.)
    rng = np.random.default_rng(20241128)
    rank_sets = [(8, 16, 32, 64), (8, 64), (16, 128), (8, 16, 24, 40, 128), (64,), (128,), (3, 12, 100), (8, 20, 256), (4, 8)]
    for i in range(36):
        T = int(rng.choice([1, 7, 33, 100, 256, 300, 700, 1500, 2600]))
        K = int(rng.choice([64, 328, 1024, 2048, 4096]))
        N = int(rng.choice([64, 200, 1000, 2048, 4096]))
        n_a = int(rng.choice([1, 3, 9, 40, 150]))
        ranks = rank_sets[int(rng.integers(len(rank_sets)))]
        max_seg = int(rng.choice([1, 2, 12, 64, 300, 1024]))
        frac_none, empty = float(rng.choice([0.0, 0.2])), bool(rng.integers(2))
        m = int(rng.integers(n_a))
        if T * N < 400:
            continue                                # the normwise bound is a statement about many roundings
        w = wl.random_case(7000 + i, T, K, N, n_a, ranks, max_seg=max_seg, frac_none=frac_none,
                           scales=(0.5, 2.0, -1.5), empty_segments=empty)
        print(f"[{i}] T={T} K={K} N={N} adapters={n_a} ranks={ranks} max_seg={max_seg}", flush=True)
        run_delta_case(w, check_beta0=bool(i % 2))
        if i % 3 == 0:
            run_forward_case(w, n_sample=min(T, 96))
        if i % 4 == 1:
            _delta_case(w)
            _delta_case(w, fallback=True)
        # (mixture's identity check against unmerged inference assumes an update that does not dwarf W)
        if i % 5 == 0 and K >= 1024 and max(ranks) <= 64 and all(r % 8 == 0 for r in ranks):
            run_mixture_case(w, m, n_sample=min(T, 64))


def test_large_token_counts():
    # four times the tokens of the largest benchmark configuration (64-bit row offsets, tile lists of tens of
    # thousands of entries, thousands of adapter groups); the oracle checks v in full and y on sampled rows
    rng = np.random.default_rng(9)
    for seed, (T, K, N, n_a, ranks, max_seg) in enumerate([(65536, 1024, 2048, 512, (8, 16, 32, 64, 128), 64),
                                                           (50000, 2048, 1024, 2000, (8, 16), 1)]):
        w = wl.random_case(800 + seed, T, K, N, n_a, ranks, max_seg=max_seg, frac_none=0.05, scales=(2.0, -0.5))
        run_delta_case(w, check_beta0=False, rows=np.sort(rng.choice(T, size=256, replace=False)))
        run_forward_case(w, n_sample=160)


def test_streaming_kernels_ragged_cases():
    # the prefill-sized (streaming) shrink / expand kernels forced onto small ragged batches: adapter
    # groups from 1 to a few hundred tokens (every tile shape: 8, 4, 2, 1 token blocks), all ranks up to
    # 128, K with a ragged last stage and a ragged last k-step, N with a ragged last chunk, tokens without
    # adapter, padded leading dimensions, K split over 1, 2, 4 workgroups, short and long feature ranges
    before = B.lora_tuning_get()
    B.lora_timing_begin()
    try:
        cases = [(420, 1096, 200, 3, 300), (333, 2048, 1352, 9, 90), (700, 2120, 72, 5, 40), (129, 1024, 64, 1, 1000)]
        settings = [dict(shrink_stream_wgs=1, expand_stream_stages=16), dict(shrink_stream_wgs=1 << 20, expand_stream_stages=1),
                    dict(shrink_stream_wgs=512, expand_stream_stages=2)]
        for seed, (T, K, N, n_a, max_seg) in enumerate(cases):
            w = wl.random_case(500 + seed, T, K, N, n_a, (8, 16, 24, 32, 40, 64, 96, 128), max_seg=max_seg,
                               frac_none=0.15, scales=(0.5, 1.0, 2.0, -1.5), empty_segments=True)
            for st in settings:
                B.lora_tuning_set(**before)
                B.lora_tuning_set(shrink_stream_min_tokens=1, **st)
                run_delta_case(w, B.LORA_VARIANT_TILED, check_beta0=(st is settings[0]))
            run_delta_case(w, B.LORA_VARIANT_TILED, ld_pad=8, check_beta0=False)
            run_forward_case(w, variant=B.LORA_VARIANT_TILED)
    finally:
        B.lora_tuning_set(**before)
        launched = B.lora_timing_end()
    assert {"shrink_stream_kernel", "expand_stream_kernel"} <= set(launched), sorted(launched)
    assert not {"shrink_tiled_kernel", "expand_tiled_kernel"} & set(launched), sorted(launched)


def test_general_kernels_take_odd_layouts():
    w = wl.random_case(200, 45, 77, 53, 5, (1, 3, 5, 12, 200, 256), max_seg=9, frac_none=0.2,
                       scales=(1.0, 2.0, -0.5))
    run_delta_case(w)                              # odd K, N, ranks: general family
    run_delta_case(w, ld_pad=3, check_beta0=False)
    run_forward_case(w)
    wf = wl.random_case(201, 33, 40, 48, 3, (4, 8), dtype="f32", max_seg=6, frac_none=0.2)
    run_delta_case(wf)
    run_forward_case(wf)


def test_degenerate_batches():
    # no tokens at all
    w = wl.random_case(300, 0, 64, 64, 2, (8,))
    run_delta_case(w)
    # every token without adapter: y must equal its input bit for bit, fused = x W
    w = wl.random_case(301, 40, 64, 128, 2, (8, 16), frac_none=1.0)
    run_delta_case(w)
    run_forward_case(w)
    # one long segment, one adapter, maximum tiled rank
    w = wl.random_case(302, 257, 256, 192, 1, (128,), max_seg=1000)
    run_delta_case(w)
    # single token
    w = wl.random_case(303, 1, 128, 64, 3, (8, 64))
    run_delta_case(w)
    run_forward_case(w)


def test_tiled_request_with_unaligned_leading_dimension_is_refused():
    w = wl.random_case(304, 20, 64, 64, 2, (8,))
    dl = device.to_device(w, DEV, with_w=False)
    plan = device.make_plan(w, B.LORA_VARIANT_TILED)
    R, _, _ = B.lora_plan_query(plan)
    x = torch.zeros((w.T, w.K + 3), dtype=torch.bfloat16, device=DEV)
    v = torch.zeros(B.lora_plan_query(plan)[1] // 4, dtype=torch.float32, device=DEV)
    with pytest.raises(B.LoraError) as e:
        B.lora_shrink(plan, x, w.K + 3, dl.At_ptrs, v)
    assert e.value.status == B.LORA_ERR_UNSUPPORTED
    torch.cuda.synchronize()
    plan.destroy()


@pytest.mark.parametrize("T,K,N,n_a,ranks,max_seg", [
    (128, 1096, 512, 1, (16,), 128), (140, 4104, 264, 1, (8,), 140), (130, 4104, 72, 1, (128,), 128), (210, 1160, 264, 2, (24, 40), 105),
    (535, 2056, 264, 5, (64,), 107), (400, 4104, 200, 4, (128,), 100), (1500, 1032, 200, 2, (128, 8), 750), (1000, 4096, 256, 8, (128,), 125),
    (1100, 2056, 200, 11, (16, 128), 100), (1400, 4104, 200, 4, (128,), 350), (1900, 2056, 200, 4, (128,), 350)])
def test_batches_of_few_streaming_tiles_split_k_over_wavefronts(T, K, N, n_a, ranks, max_seg):
    # each tile and depth that choose_rows_shrink picks from, 1, 2 and 4 K parts; K off a unit of 64, fewer units than are
    # in flight, remainders of tokens and ranks; the expand that reads as many parts
    w = wl.random_case(2600 + T + K, T, K, N, n_a, ranks, max_seg=max_seg, frac_none=0.05, scales=(2.0, -0.5))
    names = _launched(lambda: run_delta_case(w))
    assert "shrink_rows_kernel" in names and "shrink_stream_kernel" not in names
    run_forward_case(w, n_sample=96)


@pytest.mark.parametrize("T,K,N,ranks,max_seg", [(1505, 11008, 512, (64,), 400), (1931, 5120, 264, (64,), 600), (1812, 13824, 264, (64,), 300)])
def test_batches_of_few_streaming_tiles_keep_them_where_little_is_gained(T, K, N, ranks, max_seg):
    w = wl.random_case(2650 + T, T, K, N, 2, ranks, max_seg=max_seg, frac_none=0.0)
    names = _launched(lambda: run_delta_case(w))
    assert "shrink_stream_kernel" in names and "shrink_rows_kernel" not in names


# ---------------------------------------------------------------- shape table
NO_TABLE = [dict(tokens=0, k=1, n=1, max_rank=8, group_class=0, tunables={})]      # matches no batch


@pytest.mark.parametrize("name", ["cfg2", "cfg4"])
def test_shape_table_entries_change_the_plan_and_keep_parity(name):
    """The shape table (section 4.3.2) is consulted inside lora_plan_create: under an entry for the configuration's
    shape class the plan carries the entry's tunables, its tile lists differ from those the defaults give, and it
    passes parity -- with an entry made up here, and with the shipped table's own entry where it has one for the
    class (the offline search keeps an entry only where it beat the defaults on two machines)."""
    w = wl.CONFIGS[name](with_w=False)
    rows = None if w.T <= 1024 else np.arange(0, w.T, 8)
    rc = 8
    while rc < int(w.adapter_rank.max()):
        rc *= 2
    try:
        B.lora_tuning_table_set(NO_TABLE)
        plain = device.make_plan(w)
        vp = B.lora_plan_export(plain)
        plain.destroy()
        assert vp["tuning_source"] == 0 and vp["tuning"] == B.lora_tuning_get()
        made_up = dict(shrink_small_jb=2, expand_wave_bytes=4096, fused_delay=8) if name == "cfg2" else \
            dict(shrink_stream_wgs=4096, expand_stream_stages=2)
        tables = [("made up", [dict(tokens=w.T, k=w.K, n=w.N, max_rank=rc, group_class=0 if name == "cfg2" else 1, tunables=made_up)])]
        B.lora_tuning_table_set([])
        shipped = device.make_plan(w)
        has_entry = B.lora_plan_export(shipped)["tuning_source"] == 1
        shipped.destroy()
        print(f"  shipped table has an entry for {w.name}'s class: {has_entry}", flush=True)
        if has_entry:
            tables.append(("shipped", []))
        for label, table in tables:
            B.lora_tuning_table_set(table)
            p = device.make_plan(w)
            vs = B.lora_plan_export(p)
            p.destroy()
            assert vs["tuning_source"] == 1
            changed = {k for k in B.TUNING_FIELDS if vs["tuning"][k] != vp["tuning"][k]}
            assert changed, f"{label}: the entry changes no tunable"
            if label == "made up":
                assert all(vs["tuning"][k] == val for k, val in made_up.items())
            assert (vs["shrink_tiles"].shape != vp["shrink_tiles"].shape or vs["expand_tiles"].shape != vp["expand_tiles"].shape or
                    not np.array_equal(vs["shrink_tiles"], vp["shrink_tiles"]) or not np.array_equal(vs["expand_tiles"], vp["expand_tiles"]) or
                    vs["shrink_waves"] != vp["shrink_waves"]), f"{label}: entry {changed} left the plan as it was"
            view = run_delta_case(w, rows=rows, check_beta0=False)
            assert view["tuning_source"] == 1
            if name == "cfg2":
                _delta_case(w)                                           # the single launch under that entry
    finally:
        B.lora_tuning_table_set([])


# ---------------------------------------------------------------- one launch for both steps
def _delta_case(w, fallback=False):
    """lora_delta (single launch when the plan allows) vs the oracle and vs shrink + expand."""
    print(f"  delta {w.name} T={w.T} K={w.K} N={w.N} fallback={fallback}", flush=True)
    before = B.lora_tuning_get()
    try:
        if fallback:
            B.lora_tuning_set(fused_wait_us=1)      # never wait: every expand block recomputes its v rows
        dl = device.to_device(w, DEV, with_w=False)
        plan = device.make_plan(w)
    finally:
        B.lora_tuning_set(**before)
    tdt = device.torch_dtype(w)
    _, v_bytes, _ = B.lora_plan_query(plan)
    view = B.lora_plan_export(plan)
    waves = view["shrink_waves"]
    fused = view["kernel_family"] == B.LORA_VARIANT_TILED and view["expand_tiles"].shape[0] > 0 and \
        bool(np.all((view["expand_tiles"][:, 5] >> 8) & 0xfff > 0))
    tok = oracle.token_adapter(w.T, w.seg_indptr, w.seg_adapter)
    ad = oracle.Adapters(w.adapter_rank, w.adapter_scale, w.A, w.B)
    y0 = _y_in(w)
    v = torch.zeros(max(v_bytes // 4, 4), dtype=torch.float32, device=DEV)
    for beta in (1.0, 0.0):
        y_a = torch.from_numpy(y0).to(DEV, tdt)
        y_b = y_a.clone()
        for rep in range(3):                            # repeated launches reuse the plan's hand-off counters
            y_a.copy_(torch.from_numpy(y0).to(DEV, tdt))
            B.lora_delta(plan, dl.x, w.K, dl.At_ptrs, dl.Bt_ptrs, v, y_a, w.N, beta)
        B.lora_shrink(plan, dl.x, w.K, dl.At_ptrs, v)
        B.lora_expand(plan, v, dl.Bt_ptrs, y_b, w.N, beta)
        torch.cuda.synchronize()
        ranks_tok = np.where(tok >= 0, w.adapter_rank[np.clip(tok, 0, None)], 0)
        act = ranks_tok > 0
        ref = oracle.expand(w.x, tok, ad, w.N, y_in=(y0.astype(np.float64) if beta else None))
        got = _to_np(y_a)
        assert np.array_equal(got[~act], y0[~act]), "rows without adapter must stay bit-identical"
        if act.any():
            _assert_close(got[act], ref[act], _tol(w), f"lora_delta beta={beta}")
        if not fallback:
            # same arithmetic; bitwise equal when both paths slice K over 4 wavefronts, otherwise the fp32
            # summation order of v differs and a few y entries may round the other way
            if waves == 4 or not fused:
                assert torch.equal(y_a, y_b), "single launch and shrink+expand differ bitwise"
            else:
                assert oracle.error_metrics(_to_np(y_a), _to_np(y_b))[0] <= 5e-4
    torch.cuda.synchronize()
    plan.destroy()


def test_single_launch_delta_decode_config():
    w = wl.cfg2(with_w=False)
    plan = device.make_plan(w)
    plan.destroy()
    _delta_case(w)
    _delta_case(w, fallback=True)


def test_single_launch_delta_small_and_mixed_cases():
    for seed, (T, K, N, ranks) in enumerate([(37, 72, 200, (8, 16, 24, 32, 40, 64)), (120, 520, 1000, (8, 64)),
                                             (9, 4096, 256, (16,)), (300, 328, 72, (8, 16, 128))]):
        w = wl.random_case(400 + seed, T, K, N, 9, ranks, max_seg=12, frac_none=0.2,
                           scales=(0.5, 2.0, -1.5), empty_segments=True)
        _delta_case(w)                                  # rank 128 or big groups: falls back to two launches inside
        _delta_case(w, fallback=True)
    wf = wl.random_case(410, 33, 40, 48, 3, (4, 8), dtype="f32", max_seg=6, frac_none=0.2)
    _delta_case(wf)
    # more adapters than a wavefront has lanes, and exactly one
    wm = wl.random_case(411, 200, 1024, 320, 150, (8, 16, 32, 64), max_seg=2, scales=(1.0, 2.0))
    _delta_case(wm)
    _delta_case(wm, fallback=True)
    _delta_case(wl.random_case(412, 5, 2048, 128, 1, (64,), max_seg=8))


def test_single_launch_delta_large_decode_batch():
    # a decode batch several times the size of cfg2: far more workgroups than fit the GPU at once, so expand
    # blocks are dispatched long after their shrink blocks, and many adapter groups share the counters' table
    w = wl.random_case(413, 1536, 2048, 2048, 384, (8, 16, 32, 64), max_seg=1, scales=(1.0, 2.0, -0.5))
    _delta_case(w)


def test_traced_single_launch_gives_the_same_result_and_ordered_stamps():
    # the instrumented build of the single-launch kernel (lora_trace_set): same arithmetic as the ordinary build,
    # so the same bits in y; every workgroup's stamps are set and in phase order; a buffer that is too small
    # for the plan is an error and launches nothing
    w = wl.cfg2(with_w=False)
    dl = device.to_device(w, DEV, with_w=False)
    plan = device.make_plan(w)
    view = B.lora_plan_export(plan)
    assert (view["expand_tiles"][:, 5] >> 8).any(), "cfg2 is expected to run as one launch"
    S, E = view["shrink_tiles"].shape[0], view["expand_tiles"].shape[0]
    _, v_bytes, _ = B.lora_plan_query(plan)
    v = torch.zeros(v_bytes // 4, dtype=torch.float32, device=DEV)
    y0 = torch.from_numpy(wl.bf16_bits(wl.round_to_bf16(
        np.random.default_rng(5).standard_normal((w.T, w.N), dtype=np.float32))).view(np.int16)).to(DEV).view(torch.bfloat16)
    y_plain, y_traced = y0.clone(), y0.clone()
    B.lora_delta(plan, dl.x, w.K, dl.At_ptrs, dl.Bt_ptrs, v, y_plain, w.N, 1.0)
    trace = torch.zeros(S + E, 8, dtype=torch.int64, device=DEV)
    small = torch.zeros(S + E - 1, 8, dtype=torch.int64, device=DEV)
    try:
        B.lora_trace_set(small)
        with pytest.raises(B.LoraError) as err:
            B.lora_delta(plan, dl.x, w.K, dl.At_ptrs, dl.Bt_ptrs, v, y_traced, w.N, 1.0)
        assert err.value.status == B.LORA_ERR_WORKSPACE
        B.lora_trace_set(trace)
        B.lora_delta(plan, dl.x, w.K, dl.At_ptrs, dl.Bt_ptrs, v, y_traced, w.N, 1.0)
    finally:
        B.lora_trace_set(None)
    torch.cuda.synchronize()
    assert torch.equal(y_plain.view(torch.int16), y_traced.view(torch.int16))
    assert int(small.abs().sum()) == 0
    t = trace.cpu().numpy()
    sh, ex = t[:S], t[S:]
    assert (sh[:, :5] > 0).all() and (np.diff(sh[:, :5], axis=1) >= 0).all()
    assert (ex[:, :5] > 0).all() and (np.diff(ex[:, :5], axis=1) >= 0).all()
    done = ex[:, 5] > 0
    assert done.any() and (ex[done, 5] >= ex[done, 4]).all()
    assert set(np.unique(ex[:, 7])) <= {0, 1}
    assert (sh[:, 5] == 0).all() and (sh[:, 7] == 0).all()
    where = t[:, 6]
    assert ((where >> 32) < 8).all() and len(np.unique(where >> 32)) == 8, "every XCD takes part in a launch of this size"
    span_us = (t[:, :6].max() - t[:, 0].min()) * 1e3 / B.lora_trace_tick_khz()
    assert 1.0 < span_us < 1000.0, span_us                    # one launch of some microseconds
    # and the ordinary build again afterwards, untouched by the episode
    y_again = y0.clone()
    B.lora_delta(plan, dl.x, w.K, dl.At_ptrs, dl.Bt_ptrs, v, y_again, w.N, 1.0)
    torch.cuda.synchronize()
    assert torch.equal(y_plain.view(torch.int16), y_again.view(torch.int16))
    plan.destroy()


# ---------------------------------------------------------------- mixture mode (merged adapter + de-LoRA branch)
def run_mixture_case(w, m, n_sample=None, seed=11, variant=B.LORA_VARIANT_AUTO):
    """Mixture inference (section 4.4.1): adapter m is merged into the base weight (W' = W + s_m A_m B_m, stored in
    the workload's dtype), requests of m run on W' alone, every other request runs its own branch plus the removal
    of m.  The library gets the plain segment table, the plain pointer tables and `merged_adapter = m`; no
    concatenated matrix is built anywhere.  Checked:
      - lora_fused_forward on W' against the oracle on the same inputs (one rounding: the usual tolerance), and
        against plain unmerged inference on W (the identity of section 4.4.1; W' carries one more rounding);
      - lora_shrink's two shares of v against the oracle;
      - lora_delta (beta 1 and 0) against its contract: the removal is added first, the tokens' own branches are
        accumulated onto it, each pass rounding y once; rows of m's tokens stay bit-identical."""
    import dataclasses
    from oracle import plan_ref
    tdt = device.torch_dtype(w)
    rnd = wl.round_to_bf16 if w.dtype == "bf16" else (lambda a: np.asarray(a, np.float32))
    W_merged = rnd(oracle.merge(w.W, w.A[m], w.B[m], float(w.adapter_scale[m])).astype(np.float32))
    wm = dataclasses.replace(w, W=W_merged)
    dl = device.to_device(wm, DEV, with_w=True)
    plan = device.make_plan(w, variant, merged_adapter=m)
    view = B.lora_plan_export(plan)
    R, v_bytes, ws_bytes = B.lora_plan_query(plan)
    assert view["merged_adapter"] == m
    own_seg, removal = plan_ref.mixture_tables(w.T, w.seg_indptr, w.seg_adapter, w.adapter_rank, m)
    tok_plain = oracle.token_adapter(w.T, w.seg_indptr, w.seg_adapter)
    tok_own = oracle.token_adapter(w.T, w.seg_indptr, own_seg)
    tok_rem = np.where(removal, m, -1).astype(np.int32)
    ad = oracle.Adapters(w.adapter_rank, w.adapter_scale, w.A, w.B)
    neg = w.adapter_scale.copy()
    neg[m] = -neg[m]
    ad_neg = oracle.Adapters(w.adapter_rank, neg, w.A, w.B)
    rows = np.arange(w.T) if (n_sample is None or n_sample >= w.T) else _forward_rows(w, view, n_sample, seed)
    print(f"  mixture {w.name} merged={m} T={w.T} K={w.K} N={w.N} removal tokens={int(removal.sum())} "
          f"own-branch tokens={view['num_active']} oracle rows={rows.size}", flush=True)

    # whole layer in one call
    ws = torch.empty(max(ws_bytes, 256), dtype=torch.uint8, device=DEV)
    y = torch.full((w.T, w.N), 9.0, dtype=tdt, device=DEV)
    B.lora_fused_forward(plan, dl.x, w.K, dl.Wt, w.K, dl.At_ptrs, dl.Bt_ptrs, y, w.N, ws, ws.numel())
    torch.cuda.synchronize()
    own_delta = oracle.expand(w.x, tok_own, ad, w.N, rows=rows)
    rem_delta = oracle.expand(w.x, tok_rem, ad_neg, w.N, rows=rows)
    y_ref = oracle.base(w.x, W_merged, rows=rows) + own_delta + rem_delta
    _assert_close(_to_np(y)[rows], y_ref, _tol(w), "mixture fused forward vs oracle on the merged weight")
    y_plain = oracle.forward(w.x, w.W, tok_plain, ad, rows=rows)
    nrm, _ = oracle.error_metrics(_to_np(y)[rows], y_plain)
    print(f"    mixture fused forward vs plain unmerged inference: normwise {nrm:.3e}", flush=True)
    # two independent roundings (W' and y) of 1.7e-3 normwise each
    assert nrm <= (3e-3 if w.dtype == "bf16" else 1e-5)

    # the two shares of v
    v = torch.full((max(v_bytes // 4, 4),), -12345.0, dtype=torch.float32, device=DEV)
    B.lora_shrink(plan, dl.x, w.K, dl.At_ptrs, v)
    torch.cuda.synchronize()
    v_np = v.cpu().numpy()
    vtol = V_TOL if w.dtype == "bf16" else F32_TOL
    for what, tok, a_, P, Rr, off in (("own", tok_own, ad, view["v_parts"], R, 0),
                                      ("removal", tok_rem, ad_neg, view["unmerge_v_parts"],
                                       view["unmerge_v_row_stride"], view["unmerge_v_offset"] // 4)):
        if not (tok >= 0).any():
            continue
        parts = v_np[off:off + P * w.T * Rr].reshape(P, w.T, Rr).astype(np.float64).sum(axis=0)
        ranks_tok = np.where(tok >= 0, w.adapter_rank[np.clip(tok, 0, None)], 0)
        valid = np.arange(Rr)[None, :] < ranks_tok[:, None]
        _assert_close(np.where(valid, parts, 0.0), oracle.shrink(w.x, tok, a_, apply_scale=True, R=Rr), vtol, f"mixture v ({what})")

    # lora_delta: two accumulating passes
    y0 = _y_in(w)
    is_m = ~removal
    for beta in (1.0, 0.0):
        yd = torch.from_numpy(y0).to(DEV, tdt)
        v.fill_(-12345.0)
        B.lora_delta(plan, dl.x, w.K, dl.At_ptrs, dl.Bt_ptrs, v, yd, w.N, beta)
        torch.cuda.synchronize()
        yd_np = _to_np(yd)
        assert np.array_equal(yd_np[is_m], y0[is_m]), "rows of the merged adapter's tokens must stay bit-identical"
        sel = rows[removal[rows]]
        if not sel.size:
            continue
        z1 = beta * y0[sel].astype(np.float64) + oracle.expand(w.x, tok_rem, ad_neg, w.N, rows=sel)
        own = oracle.expand(w.x, tok_own, ad, w.N, rows=sel)
        # Two roundings of y: the removal's pass leaves rnd(z1), z1 = beta y + removal, the own pass rnd(rnd(z1) + own).
        # Element by element against the exact z1 + own: |got - (z1 + own)| <= u |z1| + u |z1 + own| (+ fp32
        # accumulation slack) -- where the two terms cancel the result inherits the first rounding's error, which
        # a relative error of the small result would not bound.  Normwise against the two steps taken with the
        # oracle's values (the intermediate rounded as stored): one rounding apart, the usual tolerance.
        u = 2.0 ** -8 if w.dtype == "bf16" else 2.0 ** -24
        slack = 1e-4 if w.dtype == "bf16" else 1e-5
        nrm, _ = oracle.error_metrics(yd_np[sel], rnd(z1.astype(np.float32)).astype(np.float64) + own)
        excess = float((np.abs(yd_np[sel] - (z1 + own)) - (1.01 * u * (np.abs(z1) + np.abs(z1 + own)) + slack)).max())
        print(f"    mixture lora_delta beta={beta:g}: normwise {nrm:.3e}, worst excess over the two-rounding bound "
              f"{excess:.3e}", flush=True)
        assert nrm <= _tol(w)[0] and excess <= 0.0
    plan.destroy()


def test_mixture_mode_tiny_fp32_general_kernels():
    run_mixture_case(wl.cfg1(), 2)


def test_mixture_mode_small_cases():
    # unsorted segments, tokens without adapter, a rank-0 adapter, ragged sizes; merged adapter with few / many tokens
    w = wl.random_case(431, 300, 512, 328, 6, (8, 16, 32, 64), max_seg=40, frac_none=0.2, scales=(1.0, 2.0, -0.5))
    run_mixture_case(w, 1)
    run_mixture_case(w, 4, variant=B.LORA_VARIANT_GENERAL)
    # every token is the merged adapter's: nothing to compute
    T = 64
    one = wl.random_case(432, T, 256, 192, 2, (16,), max_seg=64)
    one = __import__("dataclasses").replace(one, seg_adapter=np.zeros_like(one.seg_adapter))
    run_mixture_case(one, 0)


def test_mixture_mode_cfg2_decode():
    w = wl.cfg2()
    counts = np.bincount(w.seg_adapter[w.seg_adapter >= 0], minlength=w.num_adapters)
    run_mixture_case(w, int(np.argmax(counts)))


def test_mixture_mode_cfg3_prefill():
    run_mixture_case(wl.cfg3(0), 1, n_sample=128)


def test_mixture_mode_cfg4_mixed():
    w = wl.cfg4()
    lens = np.diff(w.seg_indptr)
    counts = np.bincount(w.seg_adapter[w.seg_adapter >= 0], weights=lens[w.seg_adapter >= 0], minlength=w.num_adapters)
    run_mixture_case(w, int(np.argmax(counts)), n_sample=160)      # the most popular adapter is the merged one


@pytest.mark.parametrize("T,K,N,ranks,merged_rank,max_seg", [
    (130, 1024, 264, (8, 128), 8, 140), (257, 1160, 192, (8, 128), 128, 70), (1100, 4096, 328, (16, 64), 64, 300),
    (1500, 1032, 200, (64, 24), 24, 5)])
def test_mixture_mode_shrinks_of_both_batches_in_one_launch(T, K, N, ranks, merged_rank, max_seg):
    # widths of the two batches that differ either way, K parts of their own, K off the 128 of a stage
    w = wl.random_case(433 + T, T, K, N, 5, ranks, max_seg=max_seg, frac_none=0.1)
    m = int(np.argmax(w.adapter_rank == merged_rank))
    dl = device.to_device(w, DEV, with_w=False)
    plan = device.make_plan(w, merged_adapter=m)
    v = torch.zeros(B.lora_plan_query(plan)[1] // 4, dtype=torch.float32, device=DEV)
    B.lora_timing_begin()
    B.lora_shrink(plan, dl.x, w.K, dl.At_ptrs, v)
    torch.cuda.synchronize()
    assert {name: r["count"] for name, r in B.lora_timing_end().items()} == {"shrink_stream_kernel": 1}
    plan.destroy()
    run_mixture_case(w, m)


# ---------------------------------------------------------------- mode switch (merge / unmerge)
def _merge_case(L, N, K, r, scale, dtype="bf16", variant=B.LORA_VARIANT_AUTO, ld_pad=0, seed=0, check_layers=None):
    print(f"  merge case L={L} N={N} K={K} r={r} s={scale} {dtype} variant={variant} ld_pad={ld_pad}", flush=True)
    rng = np.random.default_rng(700 + seed)
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    rnd = wl.round_to_bf16 if dtype == "bf16" else (lambda a: np.asarray(a, np.float32))
    W = [rnd(rng.standard_normal((K, N), dtype=np.float32) * K ** -0.5) for _ in range(L)]
    A = [rnd(rng.standard_normal((K, r), dtype=np.float32) * K ** -0.5) for _ in range(L)]
    Bm = [rnd(rng.standard_normal((r, N), dtype=np.float32) * max(r, 1) ** -0.5) for _ in range(L)]
    ldw = K + ld_pad
    Wt = [torch.full((N, ldw), 7.0, dtype=tdt, device=DEV) for _ in range(L)]
    for l in range(L):
        Wt[l][:, :K] = torch.from_numpy(np.ascontiguousarray(W[l].T)).to(DEV, tdt)
    At = [torch.from_numpy(np.ascontiguousarray(a.T)).to(DEV, tdt).contiguous() for a in A]      # [r, K]
    Bt = [torch.from_numpy(np.ascontiguousarray(b.T)).to(DEV, tdt).contiguous() for b in Bm]     # [N, r]
    ptrs = lambda ts: torch.tensor([t.data_ptr() for t in ts] or [0], dtype=torch.int64, device=DEV)
    pW, pA, pB = ptrs(Wt), ptrs(At), ptrs(Bt)
    code = B.LORA_BF16 if dtype == "bf16" else B.LORA_F32
    B.lora_merge(L, N, K, r, scale, code, pW, ldw, pA, pB, variant)
    torch.cuda.synchronize()
    tol = BF16_TOL if dtype == "bf16" else F32_TOL
    layers = range(L) if check_layers is None else check_layers
    for l in layers:
        got = _to_np(Wt[l])
        assert np.all(got[:, K:] == 7.0), "written beyond column K"
        ref = oracle.merge(W[l], A[l], Bm[l], scale)                       # [K, N] float64
        _assert_close(got[:, :K], ref.T, tol, f"merged layer {l}")
    # unmerge: back to the original weights, to within the rounding of the two stores
    B.lora_merge(L, N, K, r, -scale, code, pW, ldw, pA, pB, variant)
    torch.cuda.synchronize()
    for l in layers:
        got = _to_np(Wt[l])[:, :K]
        if dtype != "bf16" or not r:
            _assert_close(got, W[l].T.astype(np.float64), tol, f"unmerged layer {l}")
        else:
            # not bit-exact: the merged weight was rounded to bf16 (half a step of |W'|, relative 2^-8 at
            # most), and so is the restored one (2^-8 of |W|)
            nrm, _ = oracle.error_metrics(got, W[l].T)
            bound = 2.0 ** -8 * (1.0 + np.linalg.norm(oracle.merge(W[l], A[l], Bm[l], scale)) / np.linalg.norm(W[l]))
            print(f"    unmerged layer {l}: normwise {nrm:.3e} (bound {bound:.3e})", flush=True)
            assert nrm <= bound
        if dtype == "bf16" and r:
            ulp = np.maximum(np.abs(W[l].T), 2.0 ** -126) * 2.0 ** -7       # one bf16 step at |w| (upper bound)
            big = np.maximum(ulp, np.abs(scale) * 2.0 ** -7 * np.abs(oracle.merge(0 * W[l], A[l], Bm[l], 1.0).T))
            assert np.all(np.abs(got - W[l].T) <= 2.5 * big + 1e-30), "unmerge is off by more than the two roundings"


def test_mode_switch_merge_unmerge():
    # streaming kernel: every rank class, ragged N (not a multiple of 128 / 16), ragged K (last stage, last
    # k-chunk), padded leading dimension, several layers; then the general kernel on the same and on odd shapes
    for seed, (L, N, K, r, s) in enumerate([(3, 192, 256, 8, 2.0), (2, 130, 1096, 96, -0.75), (1, 520, 2120, 128, 0.5),
                                            (4, 128, 64, 32, 1.0), (2, 1000, 328, 64, 2.0), (1, 16, 8, 16, 3.0)]):
        _merge_case(L, N, K, r, s, variant=B.LORA_VARIANT_TILED, seed=seed)
        _merge_case(L, N, K, r, s, variant=B.LORA_VARIANT_TILED, ld_pad=8, seed=seed)
        _merge_case(L, N, K, r, s, variant=B.LORA_VARIANT_GENERAL, seed=seed)
    _merge_case(2, 53, 77, 5, 1.5, ld_pad=3)                     # odd everything: general kernel
    _merge_case(2, 40, 48, 200, 0.25)                            # rank above 128: general kernel
    _merge_case(2, 33, 40, 4, 2.0, dtype="f32")
    _merge_case(0, 64, 64, 8, 1.0)
    _merge_case(2, 64, 64, 0, 1.0)
    with pytest.raises(B.LoraError):
        _merge_case(1, 53, 77, 5, 1.0, variant=B.LORA_VARIANT_TILED)


def test_mode_switch_model_sized():
    # the paper's mode-switch workload: every layer of a 7B-class model (32 x 4096 x 4096, rank 64) in one launch;
    # two layers are compared with the oracle in full
    _merge_case(32, 4096, 4096, 64, 2.0, check_layers=[0, 31])


# ---------------------------------------------------------------- vision task heads
def test_vision_task_heads_batched_through_the_shrink():
    # Vision task heads (paper section 4.2.2): a linear layer per adapter that maps the final feature of a
    # request's last token to C_a task outputs; heads of different width run in one batch.  In this library
    # that is the shrink with "rank" = C_a, Ht_a stored [C_a, K] like At_a, and scale 1: logits land in v.
    for seed, (classes, variant) in enumerate([((2, 5, 10, 101, 174, 256), B.LORA_VARIANT_AUTO),     # shrink alone tiled
                                               ((8, 16, 24, 64, 128), B.LORA_VARIANT_TILED)]):      # everything tiled
        w = wl.random_case(900 + seed, 96, 4096, 64, len(classes), classes, max_seg=1, frac_none=0.1,
                           scales=(1.0,), with_w=False)
        w.adapter_rank = np.asarray(classes, dtype=np.int32)         # one head of every width
        rng = np.random.default_rng(910 + seed)
        w.A = [wl.round_to_bf16(rng.standard_normal((w.K, c), dtype=np.float32) * w.K ** -0.5) for c in classes]
        w.B = [np.zeros((c, w.N), np.float32) for c in classes]
        dl = device.to_device(w, DEV, with_w=False)
        plan = device.make_plan(w, variant)
        R, v_bytes, _ = B.lora_plan_query(plan)
        view = B.lora_plan_export(plan)
        # widths of any kind run on the MFMA shrink (the rank demands of the tuned kernels are the expand's)
        assert view["shrink_kernel_family"] == B.LORA_VARIANT_TILED and view["shrink_tiles"].shape[0] > 0
        P = view["v_parts"]
        v = torch.full((P, w.T, R), -12345.0, dtype=torch.float32, device=DEV)
        B.lora_shrink(plan, dl.x, w.K, dl.At_ptrs, v)
        torch.cuda.synchronize()
        tok = oracle.token_adapter(w.T, w.seg_indptr, w.seg_adapter)
        ref = oracle.shrink(w.x, tok, oracle.Adapters(w.adapter_rank, w.adapter_scale, w.A, w.B), apply_scale=True, R=R)
        got = _to_np(v)
        width = np.where(tok >= 0, w.adapter_rank[np.clip(tok, 0, None)], 0)
        valid = np.arange(R)[None, :] < width[:, None]
        logits = np.where(valid, got.astype(np.float64).sum(axis=0), 0.0)
        assert np.all(got[0][~valid] == -12345.0), "written outside a head's C_a outputs"
        _assert_close(logits, ref, V_TOL, f"task-head logits, widths {classes}")
        # the decision a head exists for: the arg max agrees wherever the oracle's top two are not a near tie
        for t in np.nonzero(width > 1)[0]:
            top = np.sort(ref[t, :width[t]])[-2:]
            if top[1] - top[0] > 1e-3 * max(1.0, abs(top[1])):
                assert int(np.argmax(logits[t, :width[t]])) == int(np.argmax(ref[t, :width[t]]))
        plan.destroy()

