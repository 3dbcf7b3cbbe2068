"""How much workspace a context accepts."""
import ctypes as C

import pytest

import synth_inputs as si


def _context(mb, name, prefill_rows):
    w = si.WORKLOADS[name]
    desc = lambda s: mb.mtad_model(s.n_layers, s.d_model, s.n_heads, s.n_kv_heads, s.head_dim, s.d_ffn, s.vocab, int(s.dtype == "bf16"), s.rms_eps, s.rope_theta, None)
    mode = mb.MTAD_MODE_MMTAD if w.mode == "mmtad" else mb.MTAD_MODE_MTAD
    return mb.mtad_create(mb.mtad_config(w.batch, w.gamma, w.beam, mode, prefill_rows, 4096), desc(w.target), desc(w.draft))


# what contexts needed when a prompt ran in chunks of prefill_rows rows and nothing larger: a program with a buffer of that size keeps working
@pytest.mark.parametrize("name,prefill_rows,enough", [("C1", 8, 1675264), ("C1", 64, 4363776), ("C2", 8, 56592896), ("C2", 64, 65428224), ("C3", 8, 95010560),
                                                      ("C3", 64, 137797632), ("C4", 64, 137797632), ("C5", 32, 263961344), ("C5", 64, 351216384)])
def test_the_buffer_of_short_prompt_chunks_is_enough(name, prefill_rows, enough):
    from paper_2407_09722_amd import binding as mb
    import torch
    if torch.cuda.is_available():
        pytest.skip("binds an address that is none: only where no device could follow it")
    ctx = _context(mb, name, prefill_rows)
    bind = lambda n: mb.lib().mtad_bind_workspace(ctx, C.c_void_p(1 << 20), n)
    best = mb.mtad_workspace_bytes(ctx)
    assert bind(enough) != mb.MTAD_ECAP                 # (the device memory cannot be cleared here: MTAD_EHIP)
    assert mb.mtad_workspace_bytes(ctx) == best         # what is bound does not change what would be best
    assert bind(enough // 8) == mb.MTAD_ECAP and bind(best) != mb.MTAD_ECAP
    mb.mtad_destroy(ctx)
