"""GPU parity of the FP8 block (all four projections on per-row E4M3 operands) through the C ABI.

Two kinds of check:
* exact, per projection, on the device's own operands: the row quantiser bit for bit, every FP8
  operand's codes and scales against the oracle's quantisation of the rows they came from, and each
  projection's output to float32-accumulation accuracy -- a wrong code, scale, column or K range
  moves an output by O(1);
* statistical, end to end, against the oracle's FP8 block (which quantises the exact float64
  activations): the device's activations carry bf16-level rounding, so a few percent of their E4M3
  codes differ by one step from the oracle's, with a bound derived from that rate (parity_util)."""
import numpy as np
import pytest
import torch

from oracle import hilo_oracle as O
from paper_2606_13898_amd import hilo, inputs
from paper_2606_13898_amd.pipeline import DeviceBlock

from parity_util import assert_close, check_selection, float_report, oracle_for, to_np
from schedule_model import FP8_SHAPES

pytestmark = pytest.mark.gpu


def _rows_for_quantiser(rng, dtype):
    """Rows that reach every branch of the quantiser: ordinary Gaussian rows, an all-zero row, a
    row whose amax is one huge outlier (most codes subnormal or zero), a row of one repeated value
    (every code 448), tiny values, and values exactly halfway between E4M3 neighbours after
    scaling (ties to even)."""
    x = rng.standard_normal((37, 96)).astype(np.float32) * 0.05
    x[3] = 0.0
    x[5] = rng.standard_normal(96).astype(np.float32) * 1e-3
    x[5, 17] = 30.0
    x[7] = -0.75
    x[9] *= 1e-6
    # row 11: amax 448 -> inv 1, so the scaled values are the values themselves; 1.0625 and
    # 1.1875 are ties between neighbouring codes (1.0 / 1.125 and 1.125 / 1.25)
    x[11] = 1.0
    x[11, 0], x[11, 1], x[11, 2], x[11, 3] = 448.0, 1.0625, 1.1875, -1.0625
    if dtype == torch.bfloat16:
        x = torch.from_numpy(x).to(torch.bfloat16).float().numpy()  # values the bf16 input holds
    return x


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16], ids=["f32", "bf16"])
def test_quantize_rows_bitwise(dtype):
    print(f"[parity-fp8] quantize rows dtype={dtype}", flush=True)
    x = _rows_for_quantiser(np.random.default_rng(3), dtype)
    xd = torch.from_numpy(x).to(dtype).cuda()
    codes = torch.empty(x.shape, dtype=torch.uint8, device="cuda")
    scale = torch.empty(x.shape[0], dtype=torch.float32, device="cuda")
    hilo.hilo_quantize_rows(xd, codes, scale)
    torch.cuda.synchronize()
    want_c, want_s = O.quantize_rows(x)
    np.testing.assert_array_equal(codes.cpu().numpy(), want_c)
    np.testing.assert_array_equal(scale.cpu().numpy(), want_s)
    assert (want_c[11, :4] == np.array([0x7e, 0x38, 0x3a, 0xb8], dtype=np.uint8)).all()
    assert (want_c[3] == 0).all() and want_s[3] == 0.0


def _code_order(c):
    """Position of an E4M3 code on the number line (codes of one sign are monotone in magnitude)."""
    c = c.astype(np.int64)
    return np.where(c & 0x80, -(c & 0x7F), c & 0x7F)


def _align(x):
    return -(-x // 256) * 256


def _ws_h(Tmax, D):
    """Bytes of the workspace's first region: bf16 rows, or FP8 codes plus row scales."""
    return max(_align(Tmax * D * 2), _align(Tmax * D) + _align(Tmax * 4))


def _gather(db, off, stride, rows, nbytes):
    """Bytes [off + r * stride, + nbytes) of the workspace for every r in rows -> uint8 [rows][nbytes]."""
    idx = off + np.asarray(rows, dtype=np.int64)[:, None] * stride + np.arange(nbytes)[None, :]
    return db.ws[torch.from_numpy(idx).to(db.ws.device)].cpu().numpy()


def _bf16_rows(db, off, rows, C):
    u8 = np.ascontiguousarray(_gather(db, off, 2 * C, rows, 2 * C))
    return torch.from_numpy(u8.view(np.uint16).astype(np.int32) << 16).view(torch.float32).numpy().astype(np.float64)


def _codes_scales(db, off, Tmax, rows, C):
    codes = _gather(db, off, C, rows, C)
    sc = np.ascontiguousarray(_gather(db, off + _align(Tmax * C), 4, rows, 4)).view(np.float32)[:, 0]
    return codes, sc


def _segment_of(cu, L, rows):
    """(sample, stream) of every packed row."""
    cu = np.asarray(cu)
    s = np.searchsorted(cu, rows, side="right") - 1
    sig = (rows >= cu[s + 1] - L).astype(np.int64)
    return s, sig


def _w8(db, sig, name, sname):
    return O.dequant_rows(db.weights8[sig][name].cpu().numpy(), db.weights8[sig][sname].cpu().numpy())


def _bias(db, sig, name):
    return db.weights[sig][name].float().cpu().numpy().astype(np.float64)


def _check_codes_of(codes, scales, x, what):
    """Codes and scales the device formed from the rows x it stored: bit for bit."""
    want_c, want_s = O.quantize_rows(x.astype(np.float32))
    np.testing.assert_array_equal(codes, want_c, err_msg=f"{what} codes")
    np.testing.assert_array_equal(scales, want_s, err_msg=f"{what} scales")


def _check_codes_near(codes, scales, h, what):
    """Codes of a row the device normalised in float32 against the oracle's quantisation of the same
    row normalised in float64 from the device's own input: they differ only where the two layer
    norms round a scaled value to different sides of a code boundary (then by one step)."""
    want_c, want_s = O.quantize_rows(h.astype(np.float32))
    np.testing.assert_allclose(scales, want_s, rtol=1e-5, err_msg=f"{what} scales")
    same = codes == want_c
    frac = float(same.mean())
    assert frac >= 0.995, f"{what}: only {frac:.4f} of the codes match"
    step = np.abs(_code_order(codes[~same]) - _code_order(want_c[~same]))
    assert (step <= 1).all(), f"{what}: a differing code is not a neighbour of the oracle's"
    return frac


def _check_qk_codes(codes, exps, want, hd):
    """The FP8 q and k the QKV projection wrote (E4M3 codes, one power-of-two exponent per (row,
    head)) against the float64 product of the same codes.  The device quantises its float32
    accumulation, whose error reaches ~1e-4 of the sum of |terms| (a fraction of 1e-3 of the row's
    RMS here); so every dequantised code must lie within half an E4M3 step of the exact value (2^-4
    of it; below the normal range half the subnormal step, 2^-10 of the row scale) plus 1e-3 of the
    row's RMS, the exponent must be the oracle's power-of-two scale of the exact row except where
    the row's amax sits within that error of 448 2^k (then one off), and most codes must match the
    oracle's quantisation of the exact row."""
    heads2 = exps.shape[1]
    same_c = total = 0
    same_e = np.zeros(exps.shape, bool)
    worst = 0.0
    for j in range(heads2):
        cols = slice(j * hd, (j + 1) * hd)
        w = want[:, cols]
        wc, wk = O.quantize_rows_pow2(w.astype(np.float32))
        same_e[:, j] = exps[:, j] == wk
        assert (np.abs(exps[:, j] - wk) <= 1).all(), "a q / k exponent off by more than one"
        got = O.dequant_rows_pow2(codes[:, cols], exps[:, j])
        rms = np.sqrt(np.mean(w ** 2, axis=1, keepdims=True))
        tol = 2.0 ** -4 * np.abs(w) + np.exp2(exps[:, j:j + 1] - 10.0) + 1e-3 * rms
        err = np.abs(got - w)
        worst = max(worst, float((err / tol).max()))
        assert (err <= tol).all(), f"q / k head {j}: {int((err > tol).sum())} codes off, worst {err.max():.3g}"
        eq = codes[:, cols] == wc
        same_c += int(eq[same_e[:, j]].sum())
        total += int(same_e[:, j].sum()) * hd
    print(f"[parity-fp8] q/k codes equal {same_c / max(total, 1):.5f}, exponents equal {same_e.mean():.5f}, "
          f"worst error / bound {worst:.3f}", flush=True)
    assert same_e.mean() >= 0.99, f"q / k exponents: only {same_e.mean():.4f} match"
    assert same_c >= 0.97 * total, f"q / k codes: only {same_c / total:.4f} match"


def _check_bf16_output(got, want, what):
    """A projection output the device rounded to bf16 against the float64 product of the same
    codes: within one bf16 ulp (the rounding, which an accumulation error can push over a midpoint)
    plus float32-accumulation error."""
    tol = 2.0 ** -8 * np.abs(want) + 1e-3 * np.sqrt(np.mean(want ** 2))
    bad = np.abs(got - want) > tol
    assert not bad.any(), f"{what}: {int(bad.sum())} outputs off, worst {np.abs(got - want).max():.3g}"


def _check_update(got, want, what):
    """A float32 residual update z_out - z_in against the float64 product of the same codes: float32
    accumulation (the FP8 MFMA's own rounding stays below ~1.3e-4 of each 64-term chunk's sum of
    |terms|) is far inside any FP8 effect; a wrong code, scale or column is an O(1) error."""
    ma, rel = float_report(got, want)
    lim = 1e-2 * np.abs(want).max()
    assert rel <= 2e-3 and ma <= lim, f"{what}: max_abs {ma:.3g} (<= {lim:.3g}), rel {rel:.3g}"
    return ma, rel


def fp8_block_checked(db, wl, rows=None):
    """Runs the FP8 attention and MLP halves on db (its z holds the compressed sequence) and checks
    all four projections exactly on the device's own operands at `rows` (all rows when None).
    Workspace after hilo_attention_fp8: the normalised rows' codes and scales first, the QKV output
    next (its first rows then overwritten by the attention output's codes and scales), the attention
    output's bf16 rows behind the bf16 block's regions; after hilo_mlp_fp8: h2's codes first, the
    hidden bf16 rows next, their codes and scales behind.  Returns (z0, z1, z2) at `rows`."""
    s = wl.shape
    cu = to_np(db.cu)
    T = int(cu[-1])
    Tmax, D, F, L = db.T, s.dim, s.mlp_dim, s.text_len
    rows = np.arange(T) if rows is None else np.asarray(rows)
    hsz = _ws_h(Tmax, D)
    base = hilo.hilo_workspace_bytes(db.shape)
    smp, sig = _segment_of(cu, L, rows)
    z0_all = to_np(db.z)[:T].astype(np.float64)
    z0 = z0_all[rows]

    db.attention(fp8=True)
    torch.cuda.synchronize()
    z1_all = to_np(db.z)[:T].astype(np.float64)
    z1 = z1_all[rows]
    # QKV: h's codes (normalised in float32 on the device) against the oracle's from the same z
    hc, hs = _codes_scales(db, 0, Tmax, rows, D)
    h = np.empty((rows.size, D))
    for k, (a, b) in enumerate(zip(smp, sig)):
        h[k] = O.layer_norm(z0[k:k + 1])[0] * (1.0 + wl.mod[a, b, 1]) + wl.mod[a, b, 0]
    frac_h = _check_codes_near(hc, hs, h, "h")
    # the QKV output (rows of 6 D bytes: q and k codes, their scale bytes, v in bf16) survives past
    # the attention output's codes and scales
    first_qkv = -(-(_align(Tmax * D) + _align(Tmax * 4)) // (6 * D))
    keep = rows >= first_qkv
    if keep.any():
        raw = _gather(db, hsz, 6 * D, rows[keep], 6 * D)
        want = np.empty((int(keep.sum()), 3 * D))
        hd = O.dequant_rows(hc[keep], hs[keep])
        for st in (0, 1):
            m = sig[keep] == st
            if m.any():
                want[m] = hd[m] @ _w8(db, st, "w_qkv", "s_qkv").T + _bias(db, st, "b_qkv")
        v = np.ascontiguousarray(raw[:, 4 * D:]).view(np.uint16).astype(np.int32) << 16
        v = torch.from_numpy(v).view(torch.float32).numpy().astype(np.float64)
        _check_bf16_output(v, want[:, 2 * D:], "QKV projection (v)")
        _check_qk_codes(raw[:, :2 * D], raw[:, 2 * D:2 * D + 2 * s.heads].astype(np.int64) - 127,
                        want[:, :2 * D], s.head_dim)
    # attention output projection: a's codes from the device's bf16 a, then the residual update
    a_bf = _bf16_rows(db, base, rows, D)
    ac, as_ = _codes_scales(db, hsz, Tmax, rows, D)
    _check_codes_of(ac, as_, a_bf, "attention output")
    ad = O.dequant_rows(ac, as_)
    want = np.empty((rows.size, D))
    for k, (a, b) in enumerate(zip(smp, sig)):
        want[k] = wl.mod[a, b, 2] * (ad[k] @ _w8(db, b, "w_o", "s_o").T + _bias(db, b, "b_o"))
    _check_update(z1 - z0, want, "attention output projection")

    db.mlp(fp8=True)
    torch.cuda.synchronize()
    z2 = to_np(db.z)[:T].astype(np.float64)[rows]
    # MLP up: h2's codes from the device's own z1, then GELU(h2 W1^T + b1) rounded to bf16
    h2c, h2s = _codes_scales(db, 0, Tmax, rows, D)
    h2 = np.empty((rows.size, D))
    for k, (a, b) in enumerate(zip(smp, sig)):
        h2[k] = O.layer_norm(z1[k:k + 1])[0] * (1.0 + wl.mod[a, b, 4]) + wl.mod[a, b, 3]
    frac_h2 = _check_codes_near(h2c, h2s, h2, "h2")
    hid = _bf16_rows(db, hsz, rows, F)
    h2d = O.dequant_rows(h2c, h2s)
    want = np.empty_like(hid)
    for st in (0, 1):
        m = sig == st
        if m.any():
            want[m] = O.gelu_tanh(h2d[m] @ _w8(db, st, "w1", "s1").T + _bias(db, st, "b1"))
    _check_bf16_output(hid, want, "MLP up projection")
    # MLP down: the hidden rows' codes from the device's bf16 rows, then the residual update
    gc, gs = _codes_scales(db, base, Tmax, rows, F)
    _check_codes_of(gc, gs, hid, "hidden")
    gd = O.dequant_rows(gc, gs)
    want = np.empty((rows.size, D))
    for k, (a, b) in enumerate(zip(smp, sig)):
        want[k] = wl.mod[a, b, 5] * (gd[k] @ _w8(db, b, "w2", "s2").T + _bias(db, b, "b2"))
    _check_update(z2 - z1, want, "MLP down projection")
    print(f"[parity-fp8] exact projections on {rows.size} rows ({int(keep.sum())} QKV rows): "
          f"h codes equal {frac_h:.5f}, h2 codes equal {frac_h2:.5f}", flush=True)
    return z0, z1, z2


def _check_fp8_weights(db, wl):
    db.prepare_fp8()
    for k in range(2):  # weight codes and scales bit for bit
        for name_w, name_s in (("w_qkv", "s_qkv"), ("w_o", "s_o"), ("w1", "s1"), ("w2", "s2")):
            want_c, want_s = O.quantize_rows(np.asarray(wl.weights[k][name_w], dtype=np.float32))
            np.testing.assert_array_equal(db.weights8[k][name_w].cpu().numpy(), want_c)
            np.testing.assert_array_equal(db.weights8[k][name_s].cpu().numpy(), want_s)


def _updates_vs_oracles(tag, Z, z1, z2, ref, ref16):
    """The device follows the FP8 block, not the bf16 one.  On each half's update of z the FP8 and
    bf16 oracles differ by the quantisation itself (two operands at ~2^-3.5 / sqrt(12) relative
    each: ~3.6%, more through the attention).  The device's difference from the FP8 oracle comes
    from its bf16-level activation noise flipping ~5% of the output and down projections' codes by
    one step: sqrt(0.05) * 2^-3.5 ~ 2%, i.e. ~0.45 of that gap, where a device multiplying bf16
    operands would sit at 1.0.  The bound is halfway, 0.75."""
    for half, got, want8, want16 in (("attention", z1 - Z, ref["z1"] - Z, ref16["z1"] - Z),
                                     ("mlp", z2 - z1, ref["z2"] - ref["z1"], ref16["z2"] - ref16["z1"])):
        _, e8 = float_report(got, want8)
        _, gap = float_report(want8, want16)
        print(f"[parity-fp8] {tag} {half} update: rel to FP8 oracle {e8:.3g}, FP8 vs bf16 oracle {gap:.3g}",
              flush=True)
        assert e8 < 0.75 * gap, f"{half}: device update is not closer to the FP8 oracle ({e8:.3g} vs {gap:.3g})"


@pytest.mark.parametrize("name", ["small128", "small64"])
def test_fp8_block_parity(name):
    print(f"[parity-fp8] block workload={name}", flush=True)
    wl = inputs.make_workload(name)
    db = DeviceBlock(wl)
    ref = oracle_for(wl, fp8=True)
    ref16 = oracle_for(wl)
    _check_fp8_weights(db, wl)
    db.score()
    db.select(hilo.TOPK)
    db.compress()
    torch.cuda.synchronize()
    check_selection(db, ref)
    T = int(ref["cu"][-1])
    Z = ref["Z"][:T]
    _, z1, z2 = fp8_block_checked(db, wl)
    assert_close(z1, ref["z1"], "fp8", f"{name} z after FP8 attention")
    assert_close(z2, ref["z2"], "fp8", f"{name} z after FP8 mlp")
    _updates_vs_oracles(name, Z, z1, z2, ref, ref16)
    db.decompress()
    torch.cuda.synchronize()
    assert_close(to_np(db.y_img), ref["y_img"], "fp8", f"{name} y_img")
    assert_close(to_np(db.y_txt), ref["y_txt"], "fp8", f"{name} y_txt")


# The schedules of the FP8 tilings (QKV 256 x 256 with FP8 q / k, the others 192 x 192) that schedule_model.py
# lists beside each shape (checked in test_gemm_schedule.py): stream-K tails (partials in the bf16 fragment
# layout, finished by the fixup, for QKV through the FP8 q / k epilogue), whole waves, long K in whole tiles
# and in pieces.
@pytest.mark.parametrize("name", list(FP8_SHAPES))
def test_fp8_gemm_schedules(name):
    shp = FP8_SHAPES[name][0]
    print(f"[parity-fp8] FP8 GEMM schedules shape={shp}", flush=True)
    wl = inputs.make_workload("splitk", shape=shp, seed=5, keep_frac=1.0)
    db = DeviceBlock(wl)
    ref = oracle_for(wl, fp8=True)
    db.prepare_fp8()
    db.score()
    db.select(hilo.TOPK)
    db.compress()
    torch.cuda.synchronize()
    check_selection(db, ref)
    T = int(ref["cu"][-1])
    rows = np.unique(np.random.default_rng(7).choice(T, min(T, 96), replace=False))
    fp8_block_checked(db, wl, rows)
    db.decompress()
    torch.cuda.synchronize()
    assert_close(to_np(db.z)[:T], ref["z2"], "fp8", "z after FP8 block")
    assert_close(to_np(db.y_img), ref["y_img"], "fp8", "y_img")


# the FP8 tiles' K loop runs windows of 128 values in pairs on 192 x 192 tiles: one, two and three windows (MLP
# down with mlp_dim 128, 256, 384), row tails around a tile's edge, and both head dims of the QKV epilogue
@pytest.mark.parametrize("mlp,hd,grid,text", [(128, 128, 14, 1), (256, 64, 28, 65), (384, 128, 16, 191)])
def test_fp8_window_counts(mlp, hd, grid, text):
    print(f"[parity-fp8] windows mlp={mlp} hd={hd} grid={grid} text={text}", flush=True)
    shp = inputs.BlockShape(1, 1, grid, grid, text, 256, 256 // hd, hd, mlp, "bf16")
    wl = inputs.make_workload("fp8windows", shape=shp, seed=11, keep_frac=0.9)
    db = DeviceBlock(wl)
    db.prepare_fp8()
    db.score()
    db.select(hilo.TOPK)
    db.compress()
    torch.cuda.synchronize()
    fp8_block_checked(db, wl)


@pytest.mark.parametrize("name", ["small128", "small64"])
def test_fp8_fused_compress_norm(name):
    """The FP8 block with its attention half's first row norm in the compress pass
    (hilo_compress_norm_fp8 + hilo_attention_fp8_normed, the benchmark's FP8 step): z, y_img and
    y_txt bit for bit those of hilo_compress + hilo_attention_fp8."""
    print(f"[parity-fp8] fused compress + norm workload={name}", flush=True)
    wl = inputs.make_workload(name)
    db = DeviceBlock(wl)
    db.run(hilo.TOPK, fp8=True, fused=False)
    torch.cuda.synchronize()
    T = int(db.cu[-1])
    z_u, yi_u, yt_u = db.z[:T].clone(), db.y_img.clone(), db.y_txt.clone()
    db.run(hilo.TOPK, fp8=True, fused=True)
    torch.cuda.synchronize()
    assert int(db.cu[-1]) == T
    assert torch.equal(db.z[:T], z_u), "z differs from the unfused calls"
    assert torch.equal(db.y_img, yi_u), "y_img differs from the unfused calls"
    assert torch.equal(db.y_txt, yt_u), "y_txt differs from the unfused calls"


def test_fp8_full_size_sampled():
    """The 1024 px workload (2766 tokens at 40% kept, dim 3072, MLP 12288) in the benchmark's launch
    configuration: all four projections exact on the device's own operands at sampled rows, then the
    block outputs against the oracle's FP8 block at those rows."""
    from test_parity_full_gpu import _sample_rows

    print("[parity-fp8] full size m1024", flush=True)
    wl = inputs.make_workload("m1024")
    s = wl.shape
    db = DeviceBlock(wl)
    db.prepare_fp8()
    db.score()
    db.select(hilo.TOPK)
    db.compress()
    torch.cuda.synchronize()
    front = oracle_for(wl, with_block=False)
    check_selection(db, front)
    rows = _sample_rows(front["counts"], front["cu"], front["seg"], s.images, s.text_len, per_seg=16)
    Z = front["Z"][rows]
    _, z1, z2 = fp8_block_checked(db, wl, rows)
    q8 = O.quantize_fp8_weights(wl.weights)
    w1, w2 = O.block(front["Z"], front["cu"], s.text_len, s.heads, wl.weights, wl.mod, rows, q8)
    ma, rel = assert_close(z2, w2, "fp8", "m1024 FP8 z at sampled rows")
    print(f"[parity-fp8] m1024: {rows.size} rows, max_abs {ma:.3g}, rel_l2 {rel:.3g}", flush=True)
    b1, b2 = O.block(front["Z"], front["cu"], s.text_len, s.heads, wl.weights, wl.mod, rows)
    _updates_vs_oracles("m1024", Z, z1, z2, {"z1": w1, "z2": w2}, {"z1": b1, "z2": b2})


def _pack_qkv8(q, k, v, heads):
    """Host side of hilo_attention_core_fp8's input: q and k quantised per (token, head) with
    power-of-two scales (the oracle's quantize_rows_pow2), v rounded to bf16, in rows of 6 D bytes.
    Returns (packed uint8 [T][6D], q codes, q exponents, k codes, k exponents, v as float64)."""
    T, D = q.shape
    hd = D // heads
    qc = np.empty((T, D), np.uint8); kc = np.empty_like(qc)
    qe = np.empty((T, heads), np.int64); ke = np.empty_like(qe)
    for h in range(heads):
        cols = slice(h * hd, (h + 1) * hd)
        qc[:, cols], qe[:, h] = O.quantize_rows_pow2(q[:, cols].astype(np.float32))
        kc[:, cols], ke[:, h] = O.quantize_rows_pow2(k[:, cols].astype(np.float32))
    vb = torch.from_numpy(v.astype(np.float32)).to(torch.bfloat16)
    buf = np.zeros((T, 6 * D), np.uint8)
    buf[:, :D], buf[:, D:2 * D] = qc, kc
    buf[:, 2 * D:2 * D + heads] = (qe + 127).astype(np.uint8)
    buf[:, 2 * D + heads:2 * D + 2 * heads] = (ke + 127).astype(np.uint8)
    buf[:, 4 * D:] = vb.view(torch.int16).numpy().view(np.uint8).reshape(T, 2 * D)
    return buf, qc, qe, kc, ke, vb.float().numpy().astype(np.float64)


@pytest.mark.gpu
@pytest.mark.parametrize("hd,lens,heads", [(128, [1, 17, 64, 65, 200], 2), (128, [150, 300, 3], 2),
                                           (64, [3, 130, 31], 4), (128, [1100] * 3, 24),
                                           (64, [1000] * 8, 8)])
def test_fp8_attention_core_ragged(hd, lens, heads):
    """The FP8-score attention core alone on codes formed on the host: against the oracle's
    attention from the same codes (attend_codes) at the bf16 core's tolerance -- the probabilities
    and v are bf16 as there, and the FP8 products are exact with float32 accumulation."""
    print(f"[parity-fp8] FP8 attention core hd={hd} heads={heads} lens={lens}", flush=True)
    D = heads * hd
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    T = int(cu[-1])
    rng = np.random.default_rng(hd + 7 * len(lens))
    q, k, v = (rng.standard_normal((T, D)) for _ in range(3))
    buf, qc, qe, kc, ke, vd = _pack_qkv8(q, k, v, heads)
    want = np.empty((T, D))
    for a, b in zip(cu[:-1], cu[1:]):
        want[a:b] = O.attend_codes(qc[a:b], qe[a:b], kc[a:b], ke[a:b], vd[a:b], heads)
    maxlen = max(lens)
    W = 2 * ((maxlen + 3) // 4)
    shp = hilo.hilo_shape(len(lens), 1, 2, W, 0, D, heads, hd, 4 * D, hilo.BF16)
    out = torch.zeros(T, D, dtype=torch.bfloat16, device="cuda")
    ws = torch.empty(hilo.hilo_workspace_bytes(shp), dtype=torch.uint8, device="cuda")
    hilo.hilo_attention_core_fp8(shp, torch.from_numpy(buf).cuda(), torch.from_numpy(cu).cuda(), out, ws)
    torch.cuda.synchronize()
    assert_close(to_np(out), want, "bf16", f"FP8 attention core hd={hd}")


def _random_fp8_shape(i):
    """Case i of a fixed seeded draw of valid FP8 block shapes: dim 256-1024, heads of 64 or 128,
    mlp_dim any multiple of 128 up to 4 dim, batch 1-2, one or two grids, even grids 4..32 a side,
    no text or 1..199 text tokens, any kept fraction."""
    rng = np.random.default_rng([104729, i])
    hd = int(rng.choice([64, 128]))
    dim = 256 * int(rng.integers(1, 5))
    mlp = 128 * int(rng.integers(2, 4 * dim // 128 + 1))
    shp = inputs.BlockShape(int(rng.integers(1, 3)), int(rng.integers(1, 3)), 2 * int(rng.integers(2, 17)),
                            2 * int(rng.integers(2, 17)), int(rng.choice([0, int(rng.integers(1, 200))])),
                            dim, dim // hd, hd, mlp, "bf16")
    return shp, float(rng.uniform(0.0, 1.0)), int(rng.integers(0, 1 << 30))


@pytest.mark.parametrize("i", range(4))
def test_fp8_random_shapes(i):
    """The FP8 block on seeded random shapes: the exact per-projection checks on sampled rows, then z
    and y against the oracle's FP8 block."""
    shp, keep, seed = _random_fp8_shape(i)
    print(f"[parity-fp8] random{i} {shp} keep={keep:.2f} seed={seed}", flush=True)
    wl = inputs.make_workload(f"fp8random{i}", shape=shp, seed=seed, keep_frac=keep)
    db = DeviceBlock(wl)
    ref = oracle_for(wl, fp8=True)
    db.prepare_fp8()
    db.score()
    db.select(hilo.TOPK)
    db.compress()
    torch.cuda.synchronize()
    check_selection(db, ref)
    T = int(ref["cu"][-1])
    rows = np.unique(np.random.default_rng(7).choice(T, min(T, 64), replace=False))
    fp8_block_checked(db, wl, rows)
    db.decompress()
    torch.cuda.synchronize()
    assert_close(to_np(db.z)[:T], ref["z2"], "fp8", "z after FP8 block")
    assert_close(to_np(db.y_img), ref["y_img"], "fp8", "y_img")
    if shp.text_len:
        assert_close(to_np(db.y_txt), ref["y_txt"], "fp8", "y_txt")
