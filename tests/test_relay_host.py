"""Which passes of small models run in one launch: shapes that were measured on both sides, a launch a step / one launch in us."""
import ctypes as C

import pytest

import synth_inputs as si


def _groups(layers, heads, kv_heads, hd, ffn, dtype, batch, rows, context):
    """Workgroups of the one-launch pass, 0 where the steps are launched one by one (256 compute units where there is no device to ask)."""
    from paper_2407_09722_amd import binding as mb
    s = si.ModelShape(layers, heads * hd, heads, kv_heads, hd, ffn, 1024, dtype)
    desc = mb.mtad_model(s.n_layers, s.d_model, s.n_heads, s.n_kv_heads, s.head_dim, s.d_ffn, s.vocab, int(dtype == "bf16"), s.rms_eps, s.rope_theta, None)
    ctx = mb.mtad_create(mb.mtad_config(batch, max(1, rows - 1), 1, mb.MTAD_MODE_MTAD, 8, context + 128), desc, desc)
    n = mb.lib().mtad_test_relay(ctx, 0, rows, 0, C.c_uint(0))
    mb.mtad_destroy(ctx)
    return n


@pytest.mark.parametrize("layers,heads,kv_heads,hd,ffn,dtype,batch,rows,context", [
    (1, 8, 8, 128, 3264, "bf16", 1, 5, 448),      # 42.5 / 47.0
    (2, 8, 8, 128, 3264, "bf16", 1, 5, 448),      # 69.9 / 76.4
    (12, 8, 8, 128, 3264, "bf16", 1, 5, 448),     # 359 / 382
    (2, 8, 4, 128, 2912, "bf16", 1, 4, 2379),     # 1.10
    (2, 4, 2, 128, 1824, "bf16", 2, 4, 2742),     # 1.09
    (1, 4, 4, 128, 1888, "bf16", 1, 8, 55),       # 36.7 / 39.0
    (1, 4, 2, 128, 1280, "bf16", 1, 8, 2854),     # 40.8 / 46.1
    (2, 4, 4, 128, 1600, "bf16", 1, 8, 2163),     # 67.2 / 70.7
    (12, 16, 8, 64, 3296, "bf16", 4, 1, 1036),    # 1.16
    (12, 20, 5, 64, 3200, "bf16", 1, 5, 43),      # 1.10
    (2, 16, 16, 64, 3520, "bf16", 1, 4, 158),     # 62.5 / 64.6
    (2, 16, 16, 64, 2720, "bf16", 1, 2, 3169),    # 61.6 / 64.6
    (12, 16, 16, 64, 3520, "bf16", 1, 4, 158),    # 313 / 319
    (12, 10, 10, 64, 2112, "bf16", 4, 1, 1169),   # 1.07
    (1, 8, 4, 64, 1824, "fp32", 1, 4, 64),        # 36.6 / 38.5
    (4, 4, 1, 64, 768, "fp32", 2, 4, 2209),       # 1.16
    (2, 4, 2, 64, 832, "fp32", 4, 2, 45),         # 1.08
    (2, 2, 1, 128, 992, "fp32", 4, 2, 3088),      # 1.08
])
def test_slower_in_one_launch(layers, heads, kv_heads, hd, ffn, dtype, batch, rows, context):
    assert _groups(layers, heads, kv_heads, hd, ffn, dtype, batch, rows, context) == 0


@pytest.mark.parametrize("layers,heads,kv_heads,hd,ffn,dtype,batch,rows,context", [
    (12, 12, 12, 64, 2048, "bf16", 1, 1, 255),    # 269 / 174
    (2, 12, 12, 64, 2048, "bf16", 1, 5, 255),     # 61 / 57
    (12, 12, 12, 64, 2048, "bf16", 1, 5, 255),    # 308 / 252
    (12, 12, 12, 64, 2048, "bf16", 1, 5, 3400),   # 373 / 314
    (48, 12, 12, 64, 2048, "bf16", 1, 8, 255),    # 1206 / 1023
    (2, 12, 12, 64, 3072, "bf16", 1, 4, 513),     # a draft step: 79.0 / 77.5
    (2, 12, 12, 64, 3072, "bf16", 1, 4, 2100),    # 90.2 / 79.5
    (2, 10, 10, 64, 2496, "bf16", 1, 5, 3552),    # 0.90
    (4, 8, 8, 64, 1376, "bf16", 1, 5, 300),       # 112 / 94
    (48, 16, 16, 64, 2816, "bf16", 1, 1, 700),    # 1210 / 899
    (24, 24, 24, 64, 4096, "bf16", 1, 1, 256),    # 713 / 639
    (12, 4, 4, 128, 1600, "bf16", 1, 8, 2163),    # 342 / 324
    (2, 6, 6, 128, 2880, "bf16", 1, 1, 2590),
    (4, 4, 4, 64, 688, "fp32", 1, 5, 77),         # 101 / 84
    (2, 2, 2, 64, 344, "fp32", 1, 5, 77),
    (12, 8, 8, 64, 1408, "fp32", 1, 5, 300),      # 336 / 295
    (2, 4, 4, 128, 1376, "fp32", 1, 2, 300),
])
def test_faster_in_one_launch(layers, heads, kv_heads, hd, ffn, dtype, batch, rows, context):
    assert _groups(layers, heads, kv_heads, hd, ffn, dtype, batch, rows, context) > 0
