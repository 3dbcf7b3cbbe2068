"""Attention on its own: a model of one layer whose logits are the attention output, over a cache that the test writes."""
import numpy as np
import pytest
import torch

import synth_inputs as si

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
QUERY = 2048                       # the large component of every query; the other one is 1


def _model(heads, kv_heads, hd, dtype="bf16"):
    """Every query is (.., 1, 2048, 0 ..): the two components turn by less than 1e-20 at any position.  New tokens' keys and values are zero; the
    attention output is added to a hidden state of ones and read through a unit matrix."""
    d = heads * hd
    shape = si.ModelShape(1, d, heads, kv_heads, hd, 32, d, dtype, rms_eps=0.0, rope_theta=1e30)
    zero = lambda *n: np.zeros(n, np.float32)
    qkv, eye = zero(shape.qkv_rows, d), np.eye(d, dtype=np.float32)
    half = hd // 2
    for h in range(heads):
        qkv[h * hd + half - 1, 0], qkv[h * hd + half - 2, 0] = QUERY, 1
    w = {"embed": np.ones((d, d), np.float32), "L0.w_qkv": qkv, "L0.w_o": eye, "L0.w_gu": zero(64, d), "L0.w_d": zero(d, 32), "unembed": eye}
    if dtype == "bf16":
        w = {k: si.f32_to_bf16_bits(v) for k, v in w.items()}
    w.update({k: np.ones(d, np.float32) for k in ("L0.g_attn", "L0.g_ffn", "g_final")})
    return shape, w


def _run(heads, kv_heads, hd, batch, gamma, beam, lens, keys, values, fused_pass=0, dtype="bf16"):
    """Logits [batch][rows][heads * hd] over a cache of lens[s] tokens, keys / values [batch][n][kv_heads][hd]; every row sees itself alone
    beside them."""
    from paper_2407_09722_amd.engine import DeviceModel, Engine
    shape, w = _model(heads, kv_heads, hd, dtype)
    m = DeviceModel(shape, w, DEV)
    n = keys.shape[1]
    eng = Engine(m, m, batch=batch, gamma=gamma, beam=beam, mode="mmtad", max_context=n + 64, prefill_rows=1, fused_pass=fused_pass)
    at = eng.tkv.page_table.cpu().numpy()[:, np.arange(n) // 16] * 16 + np.arange(n) % 16
    for to, x in ((eng.tkv.k, keys), (eng.tkv.v, values)):
        flat = to.view(-1, kv_heads, hd)
        flat[torch.from_numpy(at.astype(np.int64)).to(DEV)] = torch.from_numpy(x).to(DEV, to.dtype)
    eng.tkv.len.copy_(torch.tensor(lens, dtype=torch.int32))
    M = eng.M
    eng.t_parent.fill_(0)
    eng.t_depth.fill_(1)
    eng.t_mask.copy_(torch.from_numpy(np.left_shift(np.uint64(1), np.arange(M, dtype=np.uint64)).astype(np.int64)).expand(batch, M))
    eng.verify_phase()
    torch.cuda.synchronize()
    out = eng.logits.cpu().numpy().astype(np.float64)
    eng.close()
    return out


def _expected(heads, kv_heads, hd, lens, keys, values, rows):
    out = []
    for s, n in enumerate(lens):
        k, v = keys[s, :n].astype(np.float64), values[s, :n].astype(np.float64)
        score = (k[:, :, hd // 2 - 1] * QUERY + k[:, :, hd // 2 - 2]) / np.sqrt(hd)                  # [n][kv_heads]
        score = np.concatenate([score, np.zeros((1, kv_heads))])                                     # the row itself: key and value zero
        p = np.exp(score - score.max(0))
        o = np.einsum("nh,nhd->hd", p[:-1], v) / p.sum(0)[:, None]
        h = 1 + np.repeat(o, heads // kv_heads, 0).reshape(-1)
        out.append(np.tile(h / np.sqrt((h * h).mean()), (rows, 1)))
    return np.stack(out)


# the attention output is kept as two bfloat16 terms, 2^-17 of it (it lies within the values, 4.5 at most); the sums in float32 add less than a tenth of that
TOLERANCE = 4.5 * 2**-17


@pytest.mark.parametrize("hd,heads,kv_heads,batch,gamma,beam,n,fused_pass", [
    (64, 4, 4, 1, 1, 1, 9000, 0),      # key splits merged in the attention launch
    (64, 8, 8, 32, 3, 2, 2000, 0),     # one row group
    (128, 8, 8, 32, 3, 2, 2000, 0),
    (64, 16, 8, 16, 4, 3, 2000, 0),    # 26 (query head, row) pairs a KV head: two row groups
    (128, 16, 8, 16, 4, 3, 2000, 0),
    (64, 8, 2, 2, 4, 4, 2000, 0),      # 68: waves that share their tiles
    (128, 6, 2, 2, 4, 3, 2000, 0),     # 39
    (64, 4, 4, 1, 3, 2, 9000, 2),      # the one-launch pass
    (128, 4, 4, 2, 3, 1, 9000, 2),
])
def test_scores_in_the_hundred_thousands(hd, heads, kv_heads, batch, gamma, beam, n, fused_pass):
    """The maximum a row's probabilities refer to moves while keys of hundreds of thousands of octaves are added up: what was added before has
    to be scaled by the very difference of the two references.  (Scores are whole numbers below 2^24, exact in float32.)"""
    print(f"scores hd {hd} heads {heads}/{kv_heads} batch {batch} rows {1 + gamma * beam} n {n} fused {fused_pass}", flush=True)
    rows = 1 + gamma * beam
    r = np.random.default_rng(hd + heads + rows)
    keys, values = np.zeros((batch, n, kv_heads, hd)), r.standard_normal((batch, n, kv_heads, hd)).astype(np.float16)
    half, place = hd // 2, np.arange(n)[None, :, None]
    step = int(np.ceil(8.5 * np.log(2) * np.sqrt(hd)))                                               # a little more than eight octaves
    rises = (place > 0.6 * n) & (r.random((batch, n, kv_heads)) < 1 / 48)
    again = (place > 0.85 * n) & (r.random((batch, n, kv_heads)) < 1 / 96)
    keys[..., half - 1] = 2000 + r.integers(0, 2, (batch, 1, kv_heads))
    keys[..., half - 2] = r.integers(0, 4, (batch, n, kv_heads)) + step * (rises * 1 + again * 1)
    lens = [n - 7 * s for s in range(batch)]
    got = _run(heads, kv_heads, hd, batch, gamma, beam, lens, keys, values, fused_pass)
    want = _expected(heads, kv_heads, hd, lens, keys, values, rows)
    err = np.abs(got - want).max()
    print(f"largest error {err:.2e}", flush=True)
    assert err < TOLERANCE


@pytest.mark.parametrize("hd,heads,kv_heads,batch,gamma,beam,n", [
    (64, 40, 40, 4, 4, 1, 2100),       # 160 items of one row group: the splits run slowest, the heads are turned
    (64, 12, 12, 8, 4, 3, 2100),       # 96
    (128, 24, 24, 4, 4, 5, 1300),      # 96 of two row groups
    (64, 24, 24, 4, 5, 8, 1700),       # 96 of many rows
    (64, 40, 8, 5, 5, 8, 1100),        # 160: four chunks of rows a head
    (128, 16, 8, 8, 7, 4, 900),        # 64: the splits of an item side by side
    (128, 64, 8, 8, 4, 4, 600),        # 192, some sequences split, some whole
])
def test_grids_of_sequences_of_different_lengths(hd, heads, kv_heads, batch, gamma, beam, n):
    """More and fewer workgroups than compute units, sequences that use all, some or one of the splits a launch offers."""
    print(f"grid hd {hd} heads {heads}/{kv_heads} batch {batch} rows {1 + gamma * beam} n {n}", flush=True)
    r = np.random.default_rng(heads + n)
    keys, values = np.zeros((batch, n, kv_heads, hd)), r.standard_normal((batch, n, kv_heads, hd)).astype(np.float16)
    keys[..., hd // 2 - 2] = r.integers(-16, 17, (batch, n, kv_heads))
    lens = [n, 1, n // 2, 130, n // 4, n - 1, 449, 300][:batch]
    got = _run(heads, kv_heads, hd, batch, gamma, beam, lens, keys, values, 0)
    assert np.abs(got - _expected(heads, kv_heads, hd, lens, keys, values, 1 + gamma * beam)).max() < TOLERANCE


@pytest.mark.parametrize("hd,heads,kv_heads,batch,gamma,beam,n", [
    (64, 8, 8, 16, 8, 1, 1300),        # 9 rows: one key split, five or six rounds of blocks, the last of 20 keys
    (128, 8, 8, 8, 4, 3, 1100),        # 13 rows, two splits of two or three rounds
    (64, 16, 4, 3, 3, 5, 900),         # three splits
    (128, 8, 2, 4, 7, 8, 700),         # 57 rows: one split
    (64, 2, 2, 1, 4, 1, 9000),         # 32 splits, some with a second round
])
def test_float32_waves_of_several_blocks(hd, heads, kv_heads, batch, gamma, beam, n):
    """The float32 kernel's key loop: running maxima that move from block to block, the next block's places, a last block that is cut."""
    print(f"float32 hd {hd} heads {heads}/{kv_heads} batch {batch} rows {1 + gamma * beam} n {n}", flush=True)
    r = np.random.default_rng(heads + n)
    keys, values = np.zeros((batch, n, kv_heads, hd), np.float32), r.standard_normal((batch, n, kv_heads, hd)).astype(np.float32)
    keys[..., hd // 2 - 2] = r.standard_normal((batch, n, kv_heads)) * 12 + np.arange(n)[None, :, None] * (40 / n) * r.choice([-1, 0, 1], (batch, 1, kv_heads))
    lens = [n - (97 * s) % (n // 2) for s in range(batch)]
    got = _run(heads, kv_heads, hd, batch, gamma, beam, lens, keys, values, dtype="fp32")
    err = np.abs(got - _expected(heads, kv_heads, hd, lens, keys, values, 1 + gamma * beam)).max()
    print(f"largest error {err:.2e}", flush=True)
    assert err < 1e-5  # of values up to 4.5 with weights from scores up to 10: a few units in the last place of each
