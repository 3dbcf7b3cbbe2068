"""The decoder pass of a small model in one launch, at the edges of its units, splits and waits."""
import ctypes as C

import numpy as np
import pytest
import torch

import synth_inputs as si
from tests._parity import run_pair
from tests.test_gpu_attention import TOLERANCE, _expected, _run
from tests.test_gpu_path import _weights

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _relay(eng, draft, rows, absent=0, patience=0):
    """Workgroups of such a pass (0: a launch a step); absent ones never start, and are counted out after patience * 10 ns."""
    from paper_2407_09722_amd import binding as mb
    return mb.lib().mtad_test_relay(eng.ctx, draft, rows, absent, C.c_uint(patience))


def _any(eng):
    """Every pass that can run in one launch does so, whether or not that is the faster form."""
    from paper_2407_09722_amd import binding as mb
    mb.lib().mtad_test_relay_any(eng.ctx)
    eng.workspace = torch.empty(mb.mtad_workspace_bytes(eng.ctx), dtype=torch.uint8, device=DEV)
    mb.mtad_bind_workspace(eng.ctx, eng.workspace)


@pytest.fixture
def in_one_launch(monkeypatch):
    """Engines made by the test take it for every verify pass and every draft step of at most 8 rows, and say so."""
    from paper_2407_09722_amd import engine

    class Engine(engine.Engine):
        def __init__(self, *args, **more):
            super().__init__(*args, **more)
            _any(self)
            for draft, rows in ((0, self.M), (1, self.gamma + 1), (1, self.beam)):
                assert self.B * rows > 8 or _relay(self, draft, rows) > 0

    monkeypatch.setattr(engine, "Engine", Engine)


@pytest.mark.parametrize("dtype,heads,kv_heads,hd,ffn,layers,batch,gamma,beam,n", [
    ("fp32", 1, 1, 64, 8, 1, 1, 1, 1, 1),        # one layer, a reduction of 8 terms, an empty cache
    ("fp32", 2, 1, 64, 1032, 3, 1, 6, 1, 40),    # 129 strips of gate and up: the last unit has one of two
    ("fp32", 6, 2, 64, 344, 2, 1, 7, 1, 40),     # 8 rows, 24 pairs a KV head
    ("fp32", 3, 3, 128, 200, 2, 4, 1, 1, 70),    # 4 sequences of 2 rows
    ("fp32", 2, 1, 128, 344, 2, 1, 5, 2, 520),   # draft steps of two beams; a second split of the keys
    ("bf16", 1, 1, 64, 32, 1, 1, 1, 1, 1),
    ("bf16", 6, 2, 64, 1056, 3, 1, 7, 1, 40),    # 132 strips of gate and up; 33 k tiles of down over 8 waves
    ("bf16", 12, 12, 64, 160, 2, 4, 1, 1, 30),   # 144 strips of q, k and v: two a unit
    ("fp32", 12, 12, 64, 160, 2, 4, 1, 1, 30),
    ("bf16", 2, 2, 64, 160, 2, 8, 1, 1, 30),     # 16 rows a step at a time; draft steps of 8 sequences
    ("bf16", 5, 1, 128, 352, 2, 2, 3, 2, 270),   # 20 pairs a KV head: three units of 8, 8 and 4; a second split
    ("bf16", 2, 2, 128, 96, 40, 1, 4, 3, 20),    # many layers
])
def test_pass_against_the_oracle(in_one_launch, dtype, heads, kv_heads, hd, ffn, layers, batch, gamma, beam, n):
    """Every iteration, logits and cache, of a target whose passes are of that kind; the draft's beam steps likewise."""
    from paper_2407_09722_amd.engine import DeviceModel
    ts = si.ModelShape(layers, heads * hd, heads, kv_heads, hd, ffn, 512, dtype)
    ds = si.ModelShape(1, 64, 1, 1, 64, 160, 512, dtype)
    wt, wd = _weights(ts, 61, "target", boost=2.0), _weights(ds, 61, "draft", boost=2.0)
    prompt = np.random.default_rng(n).integers(0, ts.vocab, (batch, n)).astype(np.int32)
    print(f"one launch {dtype} {heads}/{kv_heads} x {hd} ffn {ffn} layers {layers} batch {batch} gamma {gamma} beam {beam} n {n}", flush=True)
    tm, dm = DeviceModel(ts, wt, DEV), DeviceModel(ds, wd, DEV)
    st = run_pair(ts, ds, wt, wd, prompt, 2 * gamma + 2, gamma=gamma, beam=beam, mode="mtad", tau=0.0, seed=5, check_kv=True, prefill_rows=16, fused_pass=1,
                  device_models=(tm, dm))
    assert st["excused"] == 0 and all(e == gamma for e in st["eta"])


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("hd,heads,kv_heads,batch,gamma,beam,n", [
    (64, 4, 4, 1, 1, 1, 9000),       # eight splits of several rounds of blocks
    (128, 2, 2, 1, 3, 2, 4100),      # 7 rows
    (64, 4, 2, 2, 3, 1, 1025),       # a split of one key
    (128, 6, 2, 4, 1, 1, 257),       # empty and nearly empty caches beside a second split
])
def test_long_caches(in_one_launch, dtype, hd, heads, kv_heads, batch, gamma, beam, n):
    """Splits of the keys, their merge, running maxima that move from block to block, sequences shorter than a split."""
    print(f"long {dtype} hd {hd} heads {heads}/{kv_heads} batch {batch} rows {1 + gamma * beam} n {n}", flush=True)
    r = np.random.default_rng(heads + n)
    keys, values = np.zeros((batch, n, kv_heads, hd), np.float32), r.standard_normal((batch, n, kv_heads, hd)).astype(np.float16).astype(np.float32)
    if dtype == "fp32":
        keys[..., hd // 2 - 2] = r.standard_normal((batch, n, kv_heads)) * 12 + np.arange(n)[None, :, None] * (40 / n) * r.choice([-1, 0, 1], (batch, 1, kv_heads))
    else:  # whole numbers, exact in the cache: two octaves' worth of steps up and down
        keys[..., hd // 2 - 1] = 1000
        keys[..., hd // 2 - 2] = r.integers(0, 4, (batch, n, kv_heads)) + np.round(np.arange(n)[None, :, None] * (40 / n) * r.choice([-1, 0, 1], (batch, 1, kv_heads)))
    lens = [n, 0, 1, n - 64][:batch]
    got = _run(heads, kv_heads, hd, batch, gamma, beam, lens, keys, values, 1, dtype)
    err = np.abs(got - _expected(heads, kv_heads, hd, lens, keys, values, 1 + gamma * beam)).max()
    print(f"largest error {err:.2e}", flush=True)
    assert err < (1e-5 if dtype == "fp32" else TOLERANCE)


def _engine(dtype, hd=64, rows=4, n=600, prompt=None):
    from paper_2407_09722_amd.engine import DeviceModel, Engine
    shape = si.ModelShape(3, 4 * hd, 4, 2, hd, 352, 512, dtype)
    m = DeviceModel(shape, _weights(shape, 7, "target", boost=2.0), DEV)
    eng = Engine(m, m, batch=1, gamma=rows - 1, beam=1, mode="mtad", max_context=n + 100, device=DEV, fused_pass=1)
    _any(eng)
    eng.prefill(np.random.default_rng(2).integers(0, 512, (1, prompt or n)).astype(np.int32))
    eng.draft_phase()
    eng.verify_phase()
    torch.cuda.synchronize()
    return eng


def _verify(eng, absent=0, patience=20000):
    """A pass over other tokens, with all workgroups (what it leaves behind is wrong for the one that is looked at), then that one."""
    _relay(eng, 0, 4, 0, 20000)
    eng.t_tok.bitwise_xor_(1)
    eng.verify_phase()
    other = eng.logits.clone()
    eng.t_tok.bitwise_xor_(1)
    _relay(eng, 0, 4, absent, patience)
    eng.verify_phase()
    assert not torch.equal(other, eng.logits)
    torch.cuda.synchronize()
    return eng.logits.cpu(), eng.tkv.k.cpu(), eng.tkv.v.cpu()


@pytest.mark.parametrize("dtype,hd", [("fp32", 64), ("fp32", 128), ("bf16", 64), ("bf16", 128)])
def test_workgroups_that_do_not_start(dtype, hd):
    """Those that are there count the others out and do all units themselves, bit for bit the same; one is enough; then all are back."""
    from paper_2407_09722_amd import binding as mb
    eng = _engine(dtype, hd)
    want = _verify(eng)
    n = _relay(eng, 0, 4)
    assert n > 8
    for absent in (1, n // 2, n - 1, 0, n - 3):
        print(f"{dtype} {hd}: {absent} of {n} absent", flush=True)
        got = _verify(eng, absent, 300)                 # 3 us
        assert mb.mtad_device_status(eng.ctx) == 0
        assert all(torch.equal(a, b) for a, b in zip(got, want)), absent
    for patience in (1, 30, 1000, 3000):                # all there, but some have waited too long for others at some place of the pass
        for _ in range(20):
            got = _verify(eng, 0, patience)
            assert torch.equal(got[0], want[0]), patience
    assert mb.mtad_device_status(eng.ctx) == 0
    eng.close()


@pytest.mark.parametrize("dtype,hd", [("fp32", 64), ("bf16", 128)])
def test_waits_that_fail_in_a_merge(dtype, hd):
    """Few workgroups, several attention units each, some of which merge the splits of others: they leave from a merge's wait or from that of
    the unit after it, and whoever takes part again gives the same bits."""
    from paper_2407_09722_amd import binding as mb
    eng = _engine(dtype, hd, n=2040)
    want = _verify(eng)
    n = _relay(eng, 0, 4)
    for absent in (n - 2, n - 3, n - 5, n - 7):
        for patience in (1, 300):
            print(f"{dtype} {hd}: {absent} of {n} absent, patience {patience}", flush=True)
            got = _verify(eng, absent, patience)
            assert mb.mtad_device_status(eng.ctx) == 0
            assert all(torch.equal(a, b) for a, b in zip(got, want)), (absent, patience)
    eng.close()


def _state(eng):
    """Numbers of the last pass, of the last one that was given up, of the last one whose workgroups were counted, and passes that started over."""
    from paper_2407_09722_amd import binding as mb
    out = (C.c_uint32 * 4)()
    assert mb.lib().mtad_test_relay_state(eng.ctx, out) == 0
    return list(out)


def _status(eng):
    from paper_2407_09722_amd import binding as mb
    bits = C.c_uint32()
    mb.lib().mtad_device_status(eng.ctx, C.byref(bits), None)
    return bits.value


def test_which_passes_start_over():
    """With workgroups that never start all do, with all of them there none does, however short the patience."""
    eng = _engine("bf16")
    n = _relay(eng, 0, 4)
    for absent, patience in ((1, 300), (0, 1), (n - 1, 1), (0, 300), (n // 2, 300), (0, 3000)):
        _relay(eng, 0, 4, absent, patience)
        before = _state(eng)
        for _ in range(5):
            eng.verify_phase()
        now = _state(eng)
        assert now[0] == before[0] + 5 and now[3] - before[3] == (5 if absent else 0), (absent, patience)
    eng.close()


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
def test_workgroups_that_are_counted_and_all_there(dtype):
    """Attention over so long a cache that whoever waits for it runs out of patience in layer 0 of every pass: all are there, so the pass goes on."""
    from paper_2407_09722_amd import binding as mb
    eng = _engine(dtype, n=100000, prompt=600)
    eng.tkv.k.normal_(generator=torch.Generator(DEV).manual_seed(1))
    eng.tkv.v.normal_(generator=torch.Generator(DEV).manual_seed(2))
    eng.tkv.len.fill_(100000)
    _relay(eng, 0, 4, 0, 0xFFFFFFFF)
    eng.verify_phase()
    torch.cuda.synchronize()
    want, counted = eng.logits.cpu(), 0
    for patience in (1, 100, 1000):
        _relay(eng, 0, 4, 0, patience)
        for _ in range(5):
            before = _state(eng)
            eng.verify_phase()
            now = _state(eng)
            assert torch.equal(eng.logits.cpu(), want) and now[3] == before[3], patience
            counted += now[2] == now[0]
    print(f"{dtype}: counted in {counted} of 15 passes", flush=True)
    assert counted > 0 and mb.mtad_device_status(eng.ctx) == 0
    # counted, found to be all there, and then given up while they wait: the pass ends, and the next one is right
    _relay(eng, 0, 4, 0, 1)
    for ticks in (2, 3000, 5000):
        print(f"{dtype}: given up after {ticks} ticks", flush=True)
        mb.lib().mtad_test_relay_give_up(eng.ctx, C.c_uint(ticks))
        eng.verify_phase()
        now = _state(eng)
        print(f"{dtype}: {now}, status {_status(eng):#x}", flush=True)
        assert now[1] == now[0] or ticks > 2
    mb.lib().mtad_test_relay_give_up(eng.ctx, C.c_uint(20000000))
    eng.verify_phase()
    torch.cuda.synchronize()
    assert torch.equal(eng.logits.cpu(), want) and _status(eng) == 8
    eng.close()


def test_a_pass_that_lasts_is_not_given_up():
    """Three workgroups for a ragged batch, which share the long sequence's heads unevenly: they wait for each other in every layer, and the pass is
    several times as long as one wait may last."""
    from paper_2407_09722_amd import binding as mb
    from paper_2407_09722_amd.engine import DeviceModel, Engine
    shape, draft, n = si.ModelShape(8, 17 * 64, 17, 17, 64, 704, 512, "bf16"), si.ModelShape(1, 64, 1, 1, 64, 160, 512, "bf16"), 12000
    eng = Engine(DeviceModel(shape, _weights(shape, 3, "target"), DEV), DeviceModel(draft, _weights(draft, 3, "draft"), DEV), batch=8, gamma=1, beam=1,
                 mode="mtad", max_context=n + 100, prefill_rows=8, device=DEV)
    eng.tkv.k.normal_(generator=torch.Generator(DEV).manual_seed(1))
    eng.tkv.v.normal_(generator=torch.Generator(DEV).manual_seed(2))
    eng.tkv.len.copy_(torch.tensor([n, 5, 40, 17, 100, 64, 3, 80], dtype=torch.int32))

    def one():
        ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        ev[0].record()
        mb.mtad_verify_tree(eng.ctx, eng.target.desc, eng.tkv.desc, eng.root_tok, eng.ar_tree, eng.logp_cond, eng.row_lse, eng.logits, None)
        ev[1].record()
        torch.cuda.synchronize()
        return eng.logits[:, 0].cpu(), ev[0].elapsed_time(ev[1])

    _any(eng)
    groups = _relay(eng, 0, 1, 0, 300)
    assert groups > 3
    one()
    want, _ = one()
    _relay(eng, 0, 1, groups - 3, 300)
    mb.lib().mtad_test_relay_give_up(eng.ctx, C.c_uint(100000))           # 1 ms
    before = _state(eng)
    got, ms = one()
    now = _state(eng)
    print(f"{groups} workgroups, 3 there: {ms:.1f} ms, {now}, status {_status(eng)}", flush=True)
    assert now[3] == before[3] + 1 and ms > 2 and _status(eng) == 0 and torch.equal(got, want)
    eng.close()


@pytest.mark.parametrize("layers", [12, 24, 48])
@pytest.mark.parametrize("heads,kv_heads,ffn,dtype,several", [(12, 12, 2048, "bf16", (1, 5, 8)), (12, 1, 2048, "bf16", (1, 5, 8)), (16, 16, 2816, "bf16", (1, 5)),
                                                              (8, 8, 1408, "fp32", (1, 5))])
def test_long_passes_do_not_start_over(layers, heads, kv_heads, ffn, dtype, several):
    """Passes of many layers, longer than what a workgroup's patience ever was, on models some of whose workgroups have attention units only: at the
    patience that a program has, with nothing else on the machine, none starts over."""
    from paper_2407_09722_amd import binding as mb
    from paper_2407_09722_amd.engine import DeviceModel, Engine
    shape = si.ModelShape(layers, heads * 64, heads, kv_heads, 64, ffn, 512, dtype)
    one = si.make_weights(shape.with_layers(1), 3, "target", threads=8)
    m = DeviceModel(shape, {n: one[n if n in one else "L0." + n.split(".")[1]] for n in si.tensor_names(shape)}, DEV)
    eng = Engine(m, m, batch=1, gamma=7, beam=1, mode="mtad", max_context=400, device=DEV)
    _any(eng)
    eng.prefill(np.random.default_rng(2).integers(0, 512, (1, 300)).astype(np.int32))
    eng.draft_phase()
    for rows in several:
        tree = eng.ar_tree if rows == 1 else mb.mtad_tree(rows, eng.tree.tok, eng.tree.parent, eng.tree.depth, eng.tree.src_beam, eng.tree.anc_mask, eng.tree.qref)
        assert _relay(eng, 0, rows) > 0
        before, ev = _state(eng), [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        ev[0].record()
        for _ in range(5):
            mb.mtad_verify_tree(eng.ctx, m.desc, eng.tkv.desc, eng.root_tok, tree, eng.logp_cond, eng.row_lse, eng.logits, None)
        ev[1].record()
        now = _state(eng)
        print(f"{dtype} {layers} layers, {heads} on {kv_heads} x 64, ffn {ffn}, {rows} rows: {ev[0].elapsed_time(ev[1]) * 200:.0f} us a pass", flush=True)
        assert now[0] == before[0] + 5 and now[3] == before[3], (rows, now, before)
    assert mb.mtad_device_status(eng.ctx) == 0
    eng.close()


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
def test_tags_that_come_round(dtype):
    """26 bits of a pass's number are in its words' tags.  Passes on both sides of the place where they come round, the words never written
    before among them, and words that the pass 2^26 earlier left: neither may be taken for a result."""
    from paper_2407_09722_amd import binding as mb
    eng = _engine(dtype)
    n, absent = _relay(eng, 0, 4), lambda a: _relay(eng, 0, 4, a, 300)
    eng.verify_phase()
    want = eng.logits.cpu()
    token = eng.t_tok[0, 1].clone()

    def passes(first, last, missing):
        assert mb.lib().mtad_test_relay_epoch(eng.ctx, C.c_uint32(first - 1 & 0xFFFFFFFF)) == 0
        absent(missing)
        for e in range(first, last + 1):
            eng.verify_phase()
            assert torch.equal(eng.logits.cpu(), want), (hex(e), missing)
            assert _state(eng)[0] == e & 0xFFFFFFFF

    # (no number twice.)  Starting over, the second copy of the words has never been written
    for first, missing in ((0x3fffffe, n - 2), (0x7fffffe, 0), (0xfffffffe, n - 2)):
        print(f"{dtype}: from pass {first:#x}, {missing} missing", flush=True)
        passes(first, first + 5, missing)
    # words of another pass in both copies, 2^26 passes earlier
    eng.t_tok[0, 1] = token ^ 1
    assert mb.lib().mtad_test_relay_epoch(eng.ctx, C.c_uint32(0xc000004)) == 0
    for missing in (n - 2, 0):
        absent(missing)
        eng.verify_phase()
        assert not torch.equal(eng.logits.cpu(), want)
    eng.t_tok[0, 1] = token
    passes(0xffffffe, 0x10000006, n - 2)
    passes(0x10000007, 0x10000008, 0)
    assert mb.mtad_device_status(eng.ctx) == 0
    eng.close()


def test_a_pass_that_is_given_up():
    """A workgroup missing and nobody allowed to count it out: the pass ends all the same, the status says so, and the next one is right."""
    from paper_2407_09722_amd import binding as mb
    eng = _engine("bf16")
    want = _verify(eng)
    _relay(eng, 0, 4, 1, 0xFFFFFFFF)
    eng.verify_phase()
    bits = C.c_uint32()
    mb.lib().mtad_device_status(eng.ctx, C.byref(bits), None)
    assert bits.value == 8
    assert all(torch.equal(a, b) for a, b in zip(_verify(eng), want))
    eng.close()


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
def test_streams_of_fewer_compute_units(dtype):
    """On a stream that has not all compute units a pass is launched a step at a time, on one that has them it is not; neither starts over, eager
    or captured."""
    from paper_2407_09722_amd import binding as mb
    hip, eng = C.CDLL("libamdhip64.so"), _engine(dtype)
    groups, cus = _relay(eng, 0, 4), torch.cuda.get_device_properties(0).multi_processor_count
    eng.verify_phase()
    relay = eng.logits.cpu()
    mb.mtad_set_fused_pass(eng.ctx, 0)
    eng.verify_phase()
    steps = eng.logits.cpu()
    mb.mtad_set_fused_pass(eng.ctx, 1)
    assert not torch.equal(relay, steps)                # the two forms add in different orders
    for n in (groups // 2, groups, cus - 1, cus):
        words = (cus + 31) // 32
        mask = (C.c_uint32 * words)(*[((1 << max(0, min(32, n - 32 * i))) - 1) for i in range(words)])
        made = C.c_void_p()
        assert hip.hipExtStreamCreateWithCUMask(C.byref(made), C.c_uint32(words), mask) == 0
        stream = torch.cuda.ExternalStream(made.value)
        before = _state(eng)
        print(f"{dtype}: {groups} workgroups, {n} compute units", flush=True)
        for _ in range(3):
            eng.logits.zero_()
            torch.cuda.synchronize()
            eng.verify_phase(stream=stream)
            now = _state(eng)
            assert torch.equal(eng.logits.cpu(), relay if n == cus else steps), n
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            eng.verify_phase(stream=stream)
        for _ in range(3):
            eng.logits.zero_()
            torch.cuda.synchronize()
            with torch.cuda.stream(stream):
                graph.replay()
            now = _state(eng)
            assert torch.equal(eng.logits.cpu(), relay if n == cus else steps), n
        assert now[3] == before[3] and mb.mtad_device_status(eng.ctx) == 0, n
        del graph
        torch.cuda.synchronize()
        assert hip.hipStreamDestroy(made) == 0
    eng.close()


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
def test_captured_iterations(dtype):
    """Iterations replayed from a graph, with eager work between, and two engines on streams of their own at the same time."""
    from paper_2407_09722_amd import binding as mb
    from paper_2407_09722_amd.engine import DeviceModel, Engine
    shape = si.ModelShape(2, 256, 4, 2, 64, 352, 512, dtype)
    draft = si.ModelShape(1, 64, 1, 1, 64, 160, 512, dtype)
    tm, dm = DeviceModel(shape, _weights(shape, 9, "target"), DEV), DeviceModel(draft, _weights(draft, 9, "draft"), DEV)
    prompt = np.random.default_rng(4).integers(0, 512, (2, 33)).astype(np.int32)

    def engine():
        e = Engine(tm, dm, batch=2, gamma=3, beam=3, mode="mtad", max_context=128, device=DEV, fused_pass=1)
        e.prefill(prompt)
        torch.cuda.synchronize()
        return e

    eager, want = engine(), []
    assert _relay(eager, 0, 4) > 0 and _relay(eager, 1, 3) > 0
    for _ in range(6):
        eager.iteration(0.3, sample_beam=True, seed=9)
        torch.cuda.synchronize()
        want.append((eager.emitted(), eager.logits.cpu()))
    rep = engine()
    graph = rep.capture_iteration(0.3, sample_beam=True, seed=9)
    scratch = torch.zeros(1 << 16, device=DEV)
    for i in range(6):
        graph.replay()
        scratch.add_(1.0)
        torch.cuda.synchronize()
        assert rep.emitted() == want[i][0] and torch.equal(rep.logits.cpu(), want[i][1]), i
    pair = [(engine(), torch.cuda.Stream()) for _ in range(2)]
    for i in range(6):
        for e, s in pair:
            e.iteration(0.3, sample_beam=True, seed=9, stream=s)
        torch.cuda.synchronize()
        for e, _ in pair:
            assert e.emitted() == want[i][0] and torch.equal(e.logits.cpu(), want[i][1]), i
    for e in (eager, rep, pair[0][0], pair[1][0]):
        assert mb.mtad_device_status(e.ctx) == 0
        e.close()


@pytest.mark.parametrize("heads,kv_heads,rows,batch", [(16, 16, 3, 1), (16, 16, 4, 1), (16, 16, 2, 2), (16, 4, 4, 1), (16, 4, 5, 1), (16, 2, 2, 1)])
def test_large_layers(heads, kv_heads, rows, batch):
    """Layers of 64 MiB and more: 4 rows or more with at most 16 query heads x rows a KV head take the other one-launch pass, the rest the
    steps; either side of both lines is what both forms give."""
    from paper_2407_09722_amd import binding as mb
    from paper_2407_09722_amd.engine import DeviceModel, Engine
    shape = si.ModelShape(1, 2048, heads, kv_heads, 128, 4608, 512, "bf16")
    m = DeviceModel(shape, si.make_weights(shape, 5, "target", threads=8), DEV)
    eng = Engine(m, m, batch=batch, gamma=rows - 1, beam=1, mode="mtad", max_context=300, device=DEV)
    eng.prefill(np.random.default_rng(2).integers(0, 512, (batch, 200)).astype(np.int32))
    eng.draft_phase()
    got = []
    for on in (0, 1, 2):
        mb.mtad_set_fused_pass(eng.ctx, on)
        eng.verify_phase()
        torch.cuda.synchronize()
        got.append(eng.logits.cpu().double())
    for other in (got[0], got[2]):  # operands of two bf16 terms, 2^-17, through two products a row
        assert (got[1] - other).norm() <= 2**-15 * other.norm()
    assert mb.mtad_device_status(eng.ctx) == 0
    eng.close()
