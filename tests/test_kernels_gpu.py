"""Single kernels at the sizes where their tiling can go wrong, against the float64 oracle."""
import numpy as np
import pytest
import torch

from oracle import hilo_oracle as O
from paper_2606_13898_amd import hilo, inputs
from parity_util import assert_close, to_np
from schedule_model import MLP_SHAPES

pytestmark = pytest.mark.gpu


def _cu(lens):
    return np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)


# 16 queries per workgroup, 16-key tiles dealt to 8 waves: waves without a tile, a lone last key,
# whole rounds of tiles, and more units than an XCD's share
@pytest.mark.parametrize("hd,lens,heads", [(64, [1, 15, 16, 17, 0, 33], 2), (128, [2, 127, 128, 129], 2),
                                           (64, [257, 600], 4), (128, [511], 1)])
def test_attention_core_f32(hd, lens, heads):
    print(f"[kernel] float32 attention core hd={hd} heads={heads} lens={lens}", flush=True)
    cu, D = _cu(lens), heads * hd
    qkv = np.random.default_rng(hd + len(lens)).standard_normal((int(cu[-1]), 3 * D)).astype(np.float32)
    shp = hilo.hilo_shape(len(lens), 1, 2, 2 * ((max(lens) + 3) // 4), 0, D, heads, hd, 4 * D, hilo.F32)
    out = torch.full((int(cu[-1]), D), float("nan"), device="cuda")
    hilo.hilo_attention_core(shp, torch.from_numpy(qkv).cuda(), torch.from_numpy(cu).cuda(), out)
    torch.cuda.synchronize()
    assert_close(to_np(out), O.attention_core(qkv, cu, heads), "f32", "float32 attention core")


# the bf16 core gives a problem of I key steps (units of 128 or 256 queries x tiles of 64 keys) to ranges of 2
# to 4 or 8 steps: an empty one, a single step, odd counts around 2 steps a range, the growing range (128 to 512
# steps), and the last size below a range for every workgroup; head dim 64 then has 512 ranges (5808 steps) and
# 768 (22704)
@pytest.mark.parametrize("hd,lens,heads", [(64, [0], 2), (64, [1], 2), (64, [65, 0, 129], 1), (64, [320, 361], 2),
                                           (64, [1100], 4), (64, [600], 24), (64, [1400], 24), (64, [2700], 24),
                                           (128, [1], 2), (128, [193, 64], 3), (128, [257, 320], 2),
                                           (128, [704], 8), (128, [600], 24)])
def test_attention_core_bf16(hd, lens, heads):
    print(f"[kernel] bf16 attention core hd={hd} heads={heads} lens={lens}", flush=True)
    cu, D = _cu(lens), heads * hd
    qkv = torch.from_numpy(np.random.default_rng(hd + sum(lens)).standard_normal((max(1, int(cu[-1])), 3 * D)))
    qkv = qkv.to(torch.bfloat16)
    shp = hilo.hilo_shape(len(lens), 1, 2, 2 * ((max(lens) + 7) // 4), 0, D, heads, hd, 4 * D, hilo.BF16)
    out = torch.full((qkv.shape[0], D), 7.0, dtype=torch.bfloat16, device="cuda")
    hilo.hilo_attention_core_noalloc(shp, qkv.cuda(), torch.from_numpy(cu).cuda(), out)
    torch.cuda.synchronize()
    if cu[-1] == 0:
        assert (out == 7.0).all()
        return
    assert_close(to_np(out), O.attention_core(qkv.float().numpy(), cu, heads), "bf16", "bf16 attention core")


def run_mlp(shape, lens, seed, rows=None):
    """hilo_mlp on packed rows of the given sample lengths -> (z after, oracle's z), for `rows` if given."""
    rng = np.random.default_rng(seed)
    cu, D = _cu(lens), shape.dim
    z = rng.standard_normal((int(cu[-1]), D)).astype(np.float32)
    w = inputs.block_weights(rng, D, shape.mlp_dim, shape.dtype)
    mod = inputs.modulation(rng, shape.batch, D)
    dt = torch.float32 if shape.dtype == "f32" else torch.bfloat16
    dev = [{k: torch.from_numpy(v).to(dt).cuda() for k, v in s.items()} for s in w]
    sh = hilo.make_shape(shape)
    zd = torch.from_numpy(z).cuda()
    ws = torch.empty(hilo.hilo_workspace_bytes(sh), dtype=torch.uint8, device="cuda")
    hilo.hilo_mlp(sh, zd, torch.from_numpy(cu).cuda(), hilo.mlp_weights(dev), torch.from_numpy(mod).cuda(), ws)
    torch.cuda.synchronize()
    rows = np.arange(int(cu[-1])) if rows is None else rows
    return to_np(zd)[rows], O.mlp(z[rows].astype(np.float64), rows, cu, shape.text_len, w, mod)


# 32 x 32 tiles, K split over 4 waves in steps of 16 (D 64: one step per wave; 192: three, less than
# a load chunk), row tails on either side of a tile's edge, with and without text rows
@pytest.mark.parametrize("dim,mlp,lens,text", [(64, 64, [1, 32, 33], 0), (192, 320, [40, 103, 64], 31),
                                               (256, 1024, [97, 66], 33)])
def test_mlp_f32(dim, mlp, lens, text):
    print(f"[kernel] float32 MLP dim={dim} mlp={mlp} lens={lens} text={text}", flush=True)
    shape = inputs.BlockShape(len(lens), 1, 2, 2 * ((max(lens) + 3) // 4), text, dim, dim // 64, 64, mlp, "f32")
    got, want = run_mlp(shape, lens, 3)
    assert_close(got, want, "f32", "float32 MLP")


# the bf16 projections choose their tile and plan from the row counts: schedule_model.py says which each of
# these shapes reaches, and test_gemm_schedule.py checks that it does
@pytest.mark.parametrize("dim,mlp,lens,text", [shape for shape, _ in MLP_SHAPES])
def test_mlp_bf16(dim, mlp, lens, text):
    print(f"[kernel] bf16 MLP dim={dim} mlp={mlp} lens={lens} text={text}", flush=True)
    shape = inputs.BlockShape(len(lens), 1, 2, 2 * ((max(lens) + 3) // 4), text, dim, dim // 64, 64, mlp, "bf16")
    T = sum(lens)
    rows = None if T < 2500 and dim < 512 else np.sort(np.random.default_rng(5).choice(T, 160, replace=False))
    got, want = run_mlp(shape, lens, 4, rows)
    assert_close(got, want, "bf16", "bf16 MLP")


# one key of every 64-key tile outweighs the tile's others by 2^40, so a short problem's probabilities are 1 or
# nothing in units of their tile's maximum and the output's only rounding in 16 bits is its own (half of 2^-7 relative);
# the maxima rise, fall and fall by more than the reference may.  Ranges of 2, 4 and 8 tiles, whole and cut units,
# and a last tile of one key.
@pytest.mark.parametrize("hd,n,heads", [(64, 128, 2), (64, 256, 32), (64, 512, 64), (64, 449, 24), (128, 128, 2),
                                        (128, 321, 12), (128, 256, 64)])
def test_attention_core_bf16_short_precision(hd, n, heads):
    print(f"[kernel] bf16 attention core precision hd={hd} heads={heads} n={n}", flush=True)
    rng = np.random.default_rng(hd + n + heads)
    D, tiles = heads * hd, (n + 63) // 64
    qkv = np.zeros((n, 3, heads, hd), np.float32)
    unit = np.sqrt(hd) * np.log(2.0)  # a score of one in base 2
    qkv[:, 0, :, 0] = inputs.to_bf16_values(rng.uniform(0.75, 1.25, (n, heads)).astype(np.float32))
    level = rng.choice([0.0, 1.3, -1.7, 2.9, -0.6, -30.0], (tiles, heads))
    level[rng.integers(tiles, size=heads), np.arange(heads)] = 0.0
    score = np.repeat(level, 64, axis=0)[:n] - 60.0
    for t in range(tiles):
        score[rng.integers(64 * t, min(n, 64 * t + 64), size=heads), np.arange(heads)] = level[t]
    qkv[:, 1, :, 0] = inputs.to_bf16_values((score * unit).astype(np.float32))
    qkv[:, 2] = inputs.to_bf16_values(rng.standard_normal((n, heads, hd)).astype(np.float32))
    qkv, cu = qkv.reshape(n, 3 * D), _cu([n])
    shp = hilo.hilo_shape(1, 1, 2, 2 * ((n + 3) // 4), 0, D, heads, hd, 4 * D, hilo.BF16)
    out = torch.empty(n, D, dtype=torch.bfloat16, device="cuda")
    hilo.hilo_attention_core_noalloc(shp, torch.from_numpy(qkv).to(torch.bfloat16).cuda(), torch.from_numpy(cu).cuda(), out)
    torch.cuda.synchronize()
    want = O.attention_core(qkv, cu, heads)
    over = np.abs(to_np(out).astype(np.float64) - want) - (2.0 ** -8 * np.abs(want) + 1e-5 * np.abs(qkv[:, 2 * D:]).max())
    assert over.max() <= 0, (over.max(), (over > 0).mean())


# an infinite value of the last key, with its 16-key tile and its wave's turn partly past the sequence: every
# query's output is infinite in that dim and finite in the others
@pytest.mark.parametrize("hd,n", [(64, 17), (64, 130), (128, 31)])
def test_attention_core_f32_infinite_value(hd, n):
    print(f"[kernel] float32 attention core, infinite value hd={hd} n={n}", flush=True)
    qkv, cu = np.random.default_rng(n).standard_normal((n, 3 * hd)).astype(np.float32), _cu([n])
    qkv[n - 1, 2 * hd + 5] = np.inf
    want = O.attention_core(np.where(np.isinf(qkv), 0, qkv), cu, 1)
    shp = hilo.hilo_shape(1, 1, 2, 2 * ((n + 3) // 4), 0, hd, 1, hd, 4 * hd, hilo.F32)
    out = torch.empty(n, hd, device="cuda")
    hilo.hilo_attention_core(shp, torch.from_numpy(qkv).cuda(), torch.from_numpy(cu).cuda(), out)
    torch.cuda.synchronize()
    got = to_np(out)
    assert np.all(got[:, 5] == np.inf)
    assert_close(np.delete(got, 5, 1), np.delete(want, 5, 1), "f32", "finite dims")


# scores of -inf that fill a wave's only tile (a lone last key) or several:
# these keys count nothing and every output is finite
@pytest.mark.parametrize("hd,n,keys", [(64, 17, [16]), (64, 300, list(range(16, 32))), (128, 145, [144]),
                                       (128, 40, list(range(16, 40)))])
def test_attention_core_f32_infinite_scores(hd, n, keys):
    print(f"[kernel] float32 attention core, scores of -inf hd={hd} n={n}", flush=True)
    qkv, cu = np.random.default_rng(n).standard_normal((n, 3 * hd)).astype(np.float32), _cu([n])
    qkv[:, 7] = np.abs(qkv[:, 7]) + 0.1   # the queries' component that meets the keys' -inf
    qkv[keys, hd + 7] = -np.inf
    shp = hilo.hilo_shape(1, 1, 2, 2 * ((n + 3) // 4), 0, hd, 1, hd, 4 * hd, hilo.F32)
    out = torch.empty(n, hd, device="cuda")
    hilo.hilo_attention_core(shp, torch.from_numpy(qkv).cuda(), torch.from_numpy(cu).cuda(), out)
    torch.cuda.synchronize()
    q, k, v = (qkv[:, i * hd:(i + 1) * hd].astype(np.float64) for i in range(3))
    score = q @ k.T / np.sqrt(hd)
    p = np.exp(score - score.max(1, keepdims=True))
    assert_close(to_np(out), p / p.sum(1, keepdims=True) @ v, "f32", "float32 attention core")
