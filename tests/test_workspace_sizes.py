"""Workspace sizes, on the host: one workspace sized by a call's largest row count serves every
smaller call (rounds commit a varying number of rows), so no reported size is below the need of
a call with fewer rows.  The need is what the call itself states when it refuses an empty
workspace, before it touches a device."""
import ctypes
import re

import pytest

from paper_2606_26744_amd import hdf

FAKE = ctypes.c_void_p(4096)     # never dereferenced: every call below is refused first


def _refused_need(status):
    assert hdf.STATUS[status] == "HDF_E_WORKSPACE"
    return int(re.search(rb"workspace of (\d+) bytes", hdf.lib().hdf_last_error()).group(1))


def _drafter(dt, d, hd, d_ff):
    w = hdf.Drafter()
    w.dtype, w.n_layers, w.d, w.n_heads, w.head_dim = dt, 1, d, d // hd, hd
    w.d_ff, w.vocab, w.eps, w.rope_max_pos = d_ff, 1000, 1e-6, 0
    one = (ctypes.c_void_p * 1)(4096)
    for f in ("attn_norm", "w_qkv", "w_o", "mlp_norm", "w_gate_up", "w_down"):
        setattr(w, f, ctypes.cast(one, ctypes.POINTER(ctypes.c_void_p)))
    w.tok_emb, w.ctx_norm, w.final_norm, w.rope_cs = FAKE, None, None, None
    return w, one


def _never_short(rows, need, size):
    """size(n) covers need(n') for every n' <= n of `rows` (increasing); the first fault."""
    most = 0
    for n in rows:
        most = max(most, need(n))
        assert size(n) >= most, (n, size(n), most)


@pytest.mark.parametrize("dt", [hdf.HDF_BF16, hdf.HDF_F32])
@pytest.mark.parametrize("d,hd,d_ff", [(256, 64, 512), (512, 64, 1024), (1024, 64, 4096), (2304, 128, 6144),
                                       (4096, 128, 12288)])
@pytest.mark.parametrize("n_seq,B", [(1, 16), (4, 16), (8, 16), (5, 33), (64, 16)])
def test_draft_block_workspace_serves_fewer_rows(dt, d, hd, d_ff, n_seq, B):
    L = hdf.lib()
    w, keep = _drafter(dt, d, hd, d_ff)
    p = ctypes.byref(w)

    def need(n):
        return _refused_need(L.hdf_draft_block(p, n_seq, B, FAKE, 2048, FAKE, FAKE, n, FAKE, FAKE, FAKE,
                                               1 << 20, FAKE, FAKE, FAKE, 0, None))
    rows = list(range(0, 700)) + list(range(700, 2060, 7)) + list(range(2060, 40000, 997))
    _never_short(rows, need, lambda n: L.hdf_draft_block_workspace(p, n_seq, B, n, 2048))


@pytest.mark.parametrize("dt", [hdf.HDF_BF16, hdf.HDF_F32])
@pytest.mark.parametrize("m,d", [(1, 576), (1, 2048), (2, 256), (4, 64), (4, 576), (4, 1024), (8, 128),
                                 (4, 4096)])
def test_fc_reduce_workspace_serves_fewer_rows(dt, m, d):
    L = hdf.lib()

    def need(n):
        return _refused_need(L.hdf_fc_reduce(FAKE, FAKE, None, n, m, d, dt, FAKE, FAKE, 0, None))
    rows = list(range(1, 700)) + list(range(700, 2060, 7)) + list(range(2060, 16384, 61)) + [16384]
    _never_short(rows, need, lambda n: L.hdf_fc_reduce_workspace(n, m, d, dt))
    # above a chunk the size is that of the whole chunks alone
    for n in (16385, 30000):
        assert L.hdf_fc_reduce_workspace(n, m, d, dt) >= need(n)
