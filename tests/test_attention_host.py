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
