"""How attention cuts its work, on the host."""
import ctypes as C

import numpy as np
import pytest

from paper_2407_09722_amd import binding as mb

XCDS, CUS = 8, 256


def _places(rows, kv_heads, chunks, batch, offered, spread):
    at = (C.c_int * (4 * kv_heads * chunks * batch * offered))()
    mb.lib().mtad_test_attention_places(rows, kv_heads, chunks, batch, offered, int(spread), at)
    return np.array(at).reshape(-1, 4)                                   # split, head, sequence, chunk


@pytest.mark.parametrize("rows,chunks", [(0, 1), (1, 1), (1, 5)])
@pytest.mark.parametrize("kv_heads,batch", [(1, 1), (1, 7), (2, 4), (5, 3), (8, 8), (12, 8), (32, 4), (40, 4), (40, 1)])
def test_every_item_has_its_workgroups_and_the_xcds_share_them(rows, chunks, kv_heads, batch):
    items = kv_heads * chunks * batch
    for offered in (1, 2, 3, 4, 6, 8, 10, 32):
        spread = 4 * items > CUS and offered * items > CUS
        at = _places(rows, kv_heads, chunks, batch, offered, spread)
        assert len(np.unique(at, axis=0)) == len(at) == items * offered
        assert at.min() == 0 and tuple(at.max(0)) == (offered - 1, kv_heads - 1, batch - 1, chunks - 1)
        if not spread:
            continue
        for used in range(1, offered + 1):                               # the splits that sequences of one length make use of
            share = np.bincount(np.flatnonzero(at[:, 0] < used) % XCDS, minlength=XCDS)
            assert share.max() <= -(-items * used // XCDS)


def _splits(hd, pairs, kv_heads, batch, causal=0, n_splits=32, keys=4096):
    """Splits offered, splits that so many keys use, items."""
    out = (C.c_int * 3)()
    mb.lib().mtad_test_attention_splits(hd, pairs, kv_heads, batch, causal, n_splits, keys, out)
    return tuple(out)


@pytest.mark.parametrize("hd", [64, 128])
@pytest.mark.parametrize("pairs", [1, 16, 17, 33, 49, 64, 130])
def test_an_uneven_fill_is_split_evenly(hd, pairs):
    """The compute unit with the most work holds at most a tenth and a rounding more of an item than with the best number of splits."""
    most = 2 if pairs == 17 or pairs <= 16 and hd == 128 else 4 if pairs <= 16 else 3
    for batch in (1, 2, 3, 4, 5, 8, 16):
        for kv_heads in (1, 2, 4, 5, 8, 12, 20, 24, 32, 40, 48, 64):
            splits, _, items = _splits(hd, pairs, kv_heads, batch)
            assert 1 <= splits <= 32
            if items * -(-CUS // items) == CUS or items < 16:
                continue
            load = lambda s: -(-items * s // CUS) / s
            assert load(splits) <= 1.12 * min(load(s) for s in range(1, max(1, CUS * most // items) + 1)), (batch, kv_heads, splits, items)


@pytest.mark.parametrize("hd,pairs,kv_heads,batch,splits", [(128, 41, 40, 4, 3), (64, 41, 40, 4, 3), (128, 41, 40, 5, 2), (128, 33, 48, 4, 4), (128, 57, 24, 4, 5), (64, 1, 40, 2, 6),
                                                            (64, 1, 40, 8, 3), (64, 9, 12, 8, 5), (128, 5, 32, 4, 2), (128, 5, 32, 8, 1)])
def test_measured_numbers_of_splits(hd, pairs, kv_heads, batch, splits):
    assert _splits(hd, pairs, kv_heads, batch)[0] == splits
    assert _splits(hd, pairs, kv_heads, batch, n_splits=2)[0] == min(2, splits)


@pytest.mark.parametrize("hd,pairs,kv_heads,batch,causal,least", [(128, 64, 4, 32, 0, 448), (128, 128, 4, 16, 0, 448), (64, 116, 8, 8, 0, 640), (128, 300, 32, 1, 1, 544),
                                                                  (64, 8 * 300, 4, 1, 1, 960), (64, 33, 32, 4, 0, 640), (128, 41, 40, 4, 0, 448),
                                                                  (128, 64, 4, 31, 0, 256), (64, 57, 8, 4, 0, 256), (128, 5, 32, 4, 0, 256), (64, 1, 40, 4, 0, 256)])
def test_short_contexts_are_not_split(hd, pairs, kv_heads, batch, causal, least):
    """Items of many rows that give every other compute unit a workgroup are split later than others."""
    used = lambda keys: _splits(hd, pairs, kv_heads, batch, causal, keys=keys)[1]
    assert used(1) == used(least - 1) == 1 < used(least)


def test_float32_splits_fill_the_machine_once():
    for batch in (1, 2, 4, 8, 16):
        for heads in (1, 2, 4, 8, 16):
            for rows in (1, 5, 8, 9, 25, 57):
                for keys in (1, 256, 257, 700, 4100, 12000):
                    s, items = mb.lib().mtad_test_f32_attention_splits(batch, heads, rows, keys), batch * heads * -(-rows // 8)
                    assert s == 1 or (s - 1) * items < CUS and (s - 1) * 256 < keys and s <= 32
                    assert s in (32, -(-keys // 256)) or s * items >= CUS
