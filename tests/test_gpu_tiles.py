"""The many-row product on every tile shape it is built for, with every epilogue, whole and with a cut reduction, against
float64.  Each tile meets rows, strips and k tiles that do not fill it; what lies beyond the outputs stays as it was."""
import numpy as np
import pytest
import torch

import synth_inputs as si
from tests import _tiles as T

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
EPS = 1e-5
KEPT = -12345.0   # what the outputs' surroundings hold


def _dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).to(DEV)


def _bf16(x):
    return si.bf16_bits_to_f32(si.f32_to_bf16_bits(x))


def _offsets(R, K):
    """Element offsets [plane][row][k] of the operand-fragment order of more than 24 rows."""
    plane, r, k = np.meshgrid(np.arange(2), np.arange(R), np.arange(K), indexing="ij")
    return (((k // 32 * ((R + 7) // 8) + r // 8) * 64 + (k % 32) // 8 * 16 + plane * 8 + r % 8) * 8) + k % 8


def _frag_elems(R, K):
    return (K + 31) // 32 * ((R + 7) // 8) * 512


class Product:
    """Operands of one product, and its float64 value with the bound on the sum of its terms."""

    def __init__(self, R, N, K, seed, pack, head_dim=0, factors=False):
        from paper_2407_09722_amd import binding as mb
        g = np.random.default_rng(seed)
        W = _bf16((g.standard_normal((N, K)) * 0.05).astype(np.float32))
        X = g.standard_normal((R, K)).astype(np.float32)
        hi = _bf16(X)
        lo = _bf16(X - hi)
        planes = np.zeros(_frag_elems(R, K), np.uint16)
        planes[_offsets(R, K).ravel()] = np.concatenate([si.f32_to_bf16_bits(hi).ravel(), si.f32_to_bf16_bits(lo).ravel()])
        row_major = _dev(si.f32_to_bf16_bits(W).view(np.int16))
        self.W = torch.empty_like(row_major)
        mb.mtad_pack_matrix(pack, row_major, self.W, N, K, head_dim)
        self.X = _dev(planes.view(np.int16))
        x = hi.astype(np.float64) + lo
        self.value, self.scale = x @ W.T.astype(np.float64), np.abs(x) @ np.abs(W).T.astype(np.float64)
        self.args = T.GemmArgs(W=self.W.data_ptr(), X=self.X.data_ptr(), R=R, N=N, K=K, ncg=(R + 7) // 8, eps=EPS)
        self.keep = []
        if factors:
            ssq = g.uniform(0.5, 1.5, (R, 3)).astype(np.float32) * K / 3
            inv = 1.0 / np.sqrt(ssq.astype(np.float64).sum(1, keepdims=True) / K + EPS)
            self.value, self.scale = self.value * inv, self.scale * inv
            self.set(ssq=_dev(ssq))
            self.args.NP = 3
        part = torch.empty(4 * R * N, device=DEV)
        self.set(part=part)
        self.args.part_floats = part.numel()
        self.g = g

    def set(self, **tensors):
        for k, t in tensors.items():
            self.keep.append(t)
            setattr(self.args, k, t.data_ptr())

    def close(self, got, want=None, extra=0.0):
        want = self.value if want is None else want
        err = np.abs(got.astype(np.float64) - want)
        bound = 2e-6 * self.scale + 1e-6 + extra     # a float32 chain of up to 2 K terms in some order
        assert np.all(err <= bound), f"max err {err.max()}, {np.argwhere(err > bound)[:4].tolist()}"


def _store(R, NT, K, tile, ks, seed):
    from paper_2407_09722_amd import binding as mb
    N = 16 * NT
    p = Product(R, N, K, seed, mb.MTAD_PACK_PLAIN)
    for accumulate in (0, 1):
        Y0 = p.g.standard_normal((R + 2, N + 16)).astype(np.float32)
        Y = _dev(Y0)
        p.set(Y=Y)
        p.args.ldy, p.args.accumulate = N + 16, accumulate
        lse = torch.full((R + 1, NT, 2), KEPT, device=DEV)
        if ks == 1 and not accumulate:
            p.set(lse_part=lse)
        else:
            p.args.lse_part = None
        assert T.launch(p.args, T.STORE, tile, ks) == 0
        torch.cuda.synchronize()
        got = Y.cpu().numpy()
        p.close(got[:R, :N], p.value + Y0[:R, :N] if accumulate else p.value)
        assert np.array_equal(got[R:], Y0[R:]) and np.array_equal(got[:, N:], Y0[:, N:])
        if ks == 1 and not accumulate:
            part = lse.cpu().numpy().astype(np.float64)
            strips = got[:R, :N].astype(np.float64).reshape(R, NT, 16)
            assert np.array_equal(part[:R, :, 0], strips.max(2))
            assert np.allclose(part[:R, :, 1], np.exp(strips - strips.max(2, keepdims=True)).sum(2), rtol=4e-6)  # 16 float32 exponentials
            assert np.all(part[R:] == KEPT)


def _resid(R, NT, K, tile, ks, seed):
    from paper_2407_09722_amd import binding as mb
    N = 16 * NT
    p = Product(R, N, K, seed, mb.MTAD_PACK_PLAIN)
    h0, gain = p.g.standard_normal((R + 2, N)).astype(np.float32), (1 + 0.1 * p.g.standard_normal(N)).astype(np.float32)
    h, planes = _dev(h0), _dev(np.full(_frag_elems(R, N) + 512, 0x5A5A, np.int16))
    ssq = torch.full((R * NT + 8,), KEPT, device=DEV)
    p.set(h=h, g_next=_dev(gain), planes_out=planes, ssq_out=ssq)
    assert T.launch(p.args, T.RESID, tile, ks) == 0
    torch.cuda.synchronize()
    got = h.cpu().numpy()
    p.close(got[:R], p.value + h0[:R], extra=2.0 ** -23 * np.abs(h0[:R]))
    assert np.array_equal(got[R:], h0[R:])
    bits, at = planes.cpu().numpy().view(np.uint16), _offsets(R, N)
    terms = si.bf16_bits_to_f32(bits[at.ravel()]).reshape(at.shape).astype(np.float64)
    want = got[:R].astype(np.float64) * gain
    assert np.all(np.abs(terms[0] + terms[1] - want) <= 2.0 ** -15 * np.abs(want))
    untouched = np.ones(bits.size, bool)
    untouched[at.ravel()] = False
    assert np.all(bits[untouched] == 0x5A5A)
    s, q = ssq.cpu().numpy().astype(np.float64), got[:R].astype(np.float64) ** 2
    n = R * NT if ks == 1 else R
    assert np.allclose(s[:n], (q.reshape(R, NT, 16).sum(2) if ks == 1 else q.sum(1)).ravel(), rtol=1e-5)
    assert np.all(s[n:] == KEPT)


def _swiglu(R, NT, K, tile, ks, seed):
    from paper_2407_09722_amd import binding as mb
    NT += NT & 1                                       # gate and up halves of whole strips
    f = 8 * NT
    p = Product(R, 2 * f, K, seed, mb.MTAD_PACK_GATE_UP, factors=True)
    act = _dev(np.full(_frag_elems(R, f) + 512, 0x5A5A, np.int16))
    p.set(act_out=act)
    assert T.launch(p.args, T.SWIGLU, tile, ks) == 0
    torch.cuda.synchronize()
    bits, at = act.cpu().numpy().view(np.uint16), _offsets(R, f)
    terms = si.bf16_bits_to_f32(bits[at.ravel()]).reshape(at.shape).astype(np.float64)
    gate, up, e = p.value[:, :f], p.value[:, f:], 2e-6 * p.scale + 1e-6
    silu = gate / (1 + np.exp(-gate))
    want = silu * up
    bound = 1.1 * np.abs(up) * e[:, :f] + np.abs(silu) * e[:, f:] + 2.0 ** -15 * np.abs(want) + 1e-6   # |silu'| <= 1.1
    err = np.abs(terms[0] + terms[1] - want)
    assert np.all(err <= bound), f"max err {err.max()}"
    untouched = np.ones(bits.size, bool)
    untouched[at.ravel()] = False
    assert np.all(bits[untouched] == 0x5A5A)


def _qkv(R, NT, K, tile, ks, seed):
    from paper_2407_09722_amd import binding as mb
    R -= R & 1                                         # two sequences
    hd, KVH, page, layer = (64, 2, 4, 1) if NT % 8 else (128, 1, 8, 0)
    H = max(1, NT * 16 // hd - 2 * KVH)
    heads, half, Rseq = H + 2 * KVH, hd // 2, R // 2
    p = Product(R, heads * hd, K, seed, mb.MTAD_PACK_QKV, head_dim=hd, factors=True)
    angle = p.g.uniform(0, 6.28, (R, half))
    rope = np.stack([np.cos(angle), np.sin(angle)], -1).astype(np.float32)
    pages = (Rseq + page) // page + 1
    slot = np.tile(np.arange(Rseq, dtype=np.int32) + 1, 2)
    slot[[0, R - 1]] = -1                              # rows that are not stored
    slot[1] = pages * page                             # a row that does not fit: status bit, nothing stored
    table = p.g.permutation(2 * pages).astype(np.int32).reshape(2, pages)
    cache = [torch.full((2, 2 * pages, page, KVH, hd), KEPT, dtype=torch.float16, device=DEV) for _ in range(2)]
    q, status = torch.full((R + 1, H * hd), KEPT, device=DEV), torch.zeros(1, dtype=torch.int32, device=DEV)
    p.set(q_out=q, rope=_dev(rope), slot=_dev(slot), status=status)
    a, table_d, lens = p.args, _dev(table), torch.zeros(2, dtype=torch.int32, device=DEV)
    a.kv = T.KvView(cache[0].data_ptr(), cache[1].data_ptr(), table_d.data_ptr(), lens.data_ptr(), page, pages, 2 * pages, KVH, hd, 2 * pages * page * KVH * hd)
    a.layer, a.Rseq, a.n_heads = layer, Rseq, H
    assert T.launch(a, T.QKV, tile, ks) == 0
    torch.cuda.synchronize()
    x, e = p.value.reshape(R, heads, hd).copy(), (2e-6 * p.scale + 1e-6).reshape(R, heads, hd)
    c, s = (rope[:, None, :, i].astype(np.float64) for i in range(2))
    turned = x[:, :H + KVH]
    x1, x2 = turned[..., :half].copy(), turned[..., half:].copy()
    turned[..., :half], turned[..., half:] = x1 * c - x2 * s, x2 * c + x1 * s
    e = e + np.concatenate([e[..., half:], e[..., :half]], -1) + 2.0 ** -22 * np.abs(x)
    got = q.cpu().numpy().astype(np.float64)
    assert np.all(np.abs(got[:R] - x[:, :H].reshape(R, -1)) <= e[:, :H].reshape(R, -1)) and np.all(got[R:] == KEPT)
    assert int(status.item()) == 1
    for which, t in enumerate(cache):
        got = t.cpu().numpy()
        want = np.full(got.shape, KEPT)
        tol = np.zeros(got.shape)
        first = H + which * KVH
        for m in range(R):
            if 0 <= slot[m] < pages * page:
                at = (layer, table[m // Rseq, slot[m] // page], slot[m] % page)
                want[at], tol[at] = x[m, first:first + KVH], e[m, first:first + KVH] + 2.0 ** -11 * np.abs(x[m, first:first + KVH]) + 2.0 ** -25
        assert np.all(np.abs(got - np.where(tol > 0, want, np.float16(KEPT))) <= tol)


@pytest.mark.parametrize("tile", T.TILES, ids=lambda t: f"{t[0]}x{t[1]}{'tall' if t[2] else ''}")
def test_every_tile_with_every_epilogue(tile):
    A, B, tall = tile
    rows, strips = 64 * B or 32, A << tall
    for n, (R, NT, KT, ks) in enumerate([(max(25, rows - 5), strips + 3, 2, 1),         # one tile of rows, strips left over, fewer k tiles than the ring holds
                                         (rows + 27, strips * 2, 21, 1),                # a second tile of rows, an odd count of k tiles, more than the ring holds
                                         (rows, strips - 1, 18, 1),                     # full rows, one strip too few
                                         (rows + 9, strips + 4, 20, 3)]):               # ranges of 7, 7 and 6 k tiles
        for epi, check in enumerate((_store, _resid, _swiglu, _qkv)):
            print(f"tile {tile} R={R} strips={NT} k tiles={KT} ranges={ks} epilogue={epi}", flush=True)
            nt = NT if epi != T.QKV else max(5, NT // 8 if n & 1 else NT // 4) * (8 if n & 1 else 4)   # whole heads of 128 or 64
            check(R, nt, 32 * KT, tile, ks, seed=100 * A + 10 * B + n)


@pytest.mark.parametrize("tile,KT", [((5, 3, 1), 2), ((5, 3, 1), 9), ((7, 4, 1), 5)], ids=lambda x: "-".join(map(str, x)) if isinstance(x, tuple) else str(x))
def test_more_tiles_than_compute_units(tile, KT):
    """Workgroups that take a second tile, of the same rows or of others, with fewer and more k tiles than the ring holds; rows and strips left over."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    A, B, _ = tile
    R, NT = 4 * 64 * B + 27, 2 * A * (cus // 5 + 2) + 4                # five tiles of rows, the last one apart from the four that share weights
    assert 5 * ((NT + 2 * A - 1) // (2 * A)) > cus
    for epi, check in enumerate((_store, _resid, _swiglu, _qkv)):
        print(f"tile {tile} R={R} strips={NT} k tiles={KT} epilogue={epi}", flush=True)
        check(R, NT // 8 * 8 if epi == T.QKV else NT, 32 * KT, tile, 1, seed=KT)


@pytest.mark.parametrize("tile", [(7, 0, 0), (8, 0, 0), (7, 1, 0), (8, 1, 0)], ids=lambda t: f"{t[0]}x{t[1]}")
@pytest.mark.parametrize("N", [16368, 16400])   # the last width at 8192 terms whose weights go through the caches, and one whose weights pass them by
def test_weights_that_no_cache_holds(tile, N):
    """Against the float64 product of the same operands on the device (the matrix is too large for the host)."""
    from paper_2407_09722_amd import binding as mb
    K, R = 8192, 29 if tile[1] == 0 else 41
    print(f"tile {tile} N={N}", flush=True)
    g = torch.Generator(device=DEV).manual_seed(N)
    W = torch.empty(N, K, dtype=torch.bfloat16, device=DEV).normal_(0, 0.05, generator=g)
    X = torch.empty(R, K, device=DEV).normal_(generator=g)
    hi = X.bfloat16()
    lo = (X - hi.float()).bfloat16()
    planes = torch.zeros(_frag_elems(R, K), dtype=torch.bfloat16, device=DEV)
    planes[_dev(_offsets(R, K).ravel())] = torch.stack([hi, lo]).ravel()
    packed, Y = torch.empty_like(W), torch.full((R + 1, N), KEPT, device=DEV)
    mb.mtad_pack_matrix(mb.MTAD_PACK_PLAIN, W, packed, N, K, 0)
    a = T.GemmArgs(W=packed.data_ptr(), X=planes.data_ptr(), R=R, N=N, K=K, ncg=(R + 7) // 8, Y=Y.data_ptr(), ldy=N)
    assert T.launch(a, T.STORE, tile, 1) == 0
    x, w = hi.double() + lo.double(), W.double()
    want, scale = x @ w.T, x.abs() @ w.abs().T
    torch.cuda.synchronize()
    assert bool(((Y[:R].double() - want).abs() <= 2e-6 * scale + 1e-6).all()) and bool((Y[R] == KEPT).all())


def test_tiles_that_do_not_exist_or_fit_are_refused():
    from paper_2407_09722_amd import binding as mb
    p = Product(40, 80, 96, 1, mb.MTAD_PACK_PLAIN)
    Y = torch.full((40, 80), KEPT, device=DEV)
    p.set(Y=Y)
    p.args.ldy = 80
    for tile, ks in (((9, 1, 0), 1), ((3, 1, 0), 1), ((4, 2, 0), 1), ((8, 2, 1), 1), ((8, 5, 0), 1), ((8, -1, 0), 1), ((8, 0, 1), 1), ((5, 3, 2), 1), ((8, 1, 0), 0), ((8, 1, 0), 4), ((8, 1, 0), 9)):
        assert T.launch(p.args, T.STORE, tile, ks) == -1, (tile, ks)
    p.args.part_floats = 2 * 40 * 80 - 1
    assert T.launch(p.args, T.STORE, (8, 1, 0), 2) == -1
    torch.cuda.synchronize()
    assert bool((Y == KEPT).all())


def test_a_device_with_too_little_lds_is_refused():
    """Checked on the host before the launch, also when the same kernel has run before."""
    from paper_2407_09722_amd import binding as mb
    p = Product(40, 80, 96, 1, mb.MTAD_PACK_PLAIN)
    Y = torch.full((40, 80), KEPT, device=DEV)
    p.set(Y=Y)
    p.args.ldy = 80
    for tile in ((8, 1, 0), (5, 4, 1)):
        assert T.launch(p.args, T.STORE, tile, 1, lds=64 << 10) == -1
        torch.cuda.synchronize()
        assert bool((Y == KEPT).all())
        assert T.launch(p.args, T.STORE, tile, 1, lds=160 << 10) == 0 and T.launch(p.args, T.STORE, tile, 1) == 0
        torch.cuda.synchronize()
        p.close(Y.cpu().numpy())
        assert T.launch(p.args, T.STORE, tile, 1, lds=64 << 10) == -1
        Y.fill_(KEPT)
