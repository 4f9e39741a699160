"""The binding's packed cache descriptor, on the CPU: the bytes it passes are those of a KvDesc filled field by field."""
import ctypes
import os

import pytest
import torch

import paper_2606_00144_amd as bd


def _field_by_field(k, v, lens, table, L):
    d = bd.KvDesc()
    d.k, d.v, d.seq_lens = k.data_ptr(), (v.data_ptr() if v is not None else None), lens.data_ptr()
    d.num_seqs, d.num_kv_heads, d.head_dim = lens.shape[0], k.shape[1], 128
    d.stride_head, d.stride_tok = k.stride(1), k.stride(2)
    if table is None:
        d.max_seq_len, d.stride_seq = (k.shape[2] if L is None else L), k.stride(0)
    else:
        d.page_table, d.page_size, d.max_pages_per_seq = table.data_ptr(), k.shape[2], table.shape[1]
        d.num_pages, d.stride_page = k.shape[0], k.stride(0)
        d.max_seq_len = table.shape[1] * k.shape[2] if L is None else L
    return bytes(d)


@pytest.mark.parametrize("L", [None, 7, 2 ** 31 - 1, 2 ** 31, 2 ** 33 + 5, -1])
@pytest.mark.parametrize("paged,with_v,token_major", [(False, True, False), (False, False, False), (False, True, True),
                                                      (True, True, False), (True, False, True)])
def test_descriptor_bytes(paged, with_v, token_major, L):
    k = torch.zeros(5, 2, 24, 128, dtype=torch.bfloat16)
    if token_major:
        k = k.transpose(1, 2).contiguous().transpose(1, 2)
    v = torch.zeros_like(k) if with_v else None
    lens = torch.zeros(3 if paged else 5, dtype=torch.int32)
    table = torch.zeros(3, 4, dtype=torch.int32) if paged else None
    want = _field_by_field(k, v, lens, table, L)      # a size beyond its field keeps its low bits
    assert bytes(bd.kv_desc(k, v, lens, table, L)) == want
    assert bd._kv(k, v, lens, table, L)[0] == want


@pytest.mark.parametrize("paged", [False, True])
@pytest.mark.parametrize("L", [None, 7, 2 ** 31 - 1, 2 ** 31, 2 ** 33 + 5, -1])
def test_descriptor_sizes(paged, L):
    # the sizes that outputs and scratch are allocated by are those of the descriptor's own fields
    k = torch.zeros(5, 2, 24, 128, dtype=torch.bfloat16)
    lens = torch.zeros(3 if paged else 5, dtype=torch.int32)
    table = torch.zeros(3, 4, dtype=torch.int32) if paged else None
    d = bd.kv_desc(k, None, lens, table, L)
    assert bd._kv(k, None, lens, table, L)[1:] == (d.num_seqs, d.num_kv_heads, d.max_seq_len)


def test_descriptor_refusals():
    k = torch.zeros(5, 2, 24, 128, dtype=torch.bfloat16)
    lens = torch.zeros(5, dtype=torch.int32)
    for bad in [dict(k=k[..., :64]), dict(k=k.float()), dict(k=k[0]), dict(k=k.transpose(2, 3)), dict(v=k[:, :, :8]),
                dict(v=k.float()), dict(seq_lens=lens.long()), dict(seq_lens=lens[:, None]), dict(seq_lens=lens[:4]),
                dict(page_table=lens), dict(page_table=torch.zeros(4, 2, dtype=torch.int32)),
                dict(page_table=torch.zeros(5, 2, dtype=torch.int64))]:
        kw = dict(k=k, v=None, seq_lens=lens, page_table=None)
        kw.update(bad)
        with pytest.raises(bd.BdError):
            bd.kv_desc(**kw)


def test_library_descriptor_argument():
    # lib()'s entries take a KvDesc (itself, byref or a pointer) or NULL and refuse anything else.  Every call that
    # gets through is refused by the library's own checks (head_dim), so nothing is launched.
    if not os.path.exists(bd.library_path):
        from paper_2606_00144_amd import build
        build.build_library()
    L = bd.lib()
    d = bd.kv_desc(torch.zeros(5, 2, 24, 128, dtype=torch.bfloat16), None, torch.zeros(5, dtype=torch.int32))
    d.head_dim = 64
    rest = {name: [None if t is ctypes.c_void_p else 0 for t in sig[1][1:]] for name, sig in bd._SIGNATURES.items()
            if name in ("bd_select_kv", "bd_select_kv_chunks", "bd_cache_append", "bd_sparse_decode_attn",
                        "bd_multiview_attn", "bd_multiview_attn_bwd", "bd_verify_attn", "bd_verify_attn_noalloc")}
    assert len(rest) == 8
    rest["bd_select_kv_chunks"][4] = 1                     # chunk is checked before the descriptor
    for name, args in rest.items():
        for good in (d, ctypes.byref(d), ctypes.pointer(d)):
            assert getattr(L, name)(good, *args) == bd.BD_ERR_UNSUPPORTED, name
        assert getattr(L, name)(None, *args) == bd.BD_ERR_INVALID_ARG, name
        for bad in (ctypes.addressof(d), bytes(d), bytearray(d), "kv", ctypes.byref(ctypes.c_int64()), 1.0):
            with pytest.raises(ctypes.ArgumentError):
                getattr(L, name)(bad, *args)


def test_workspace_get_is_asked_by_every_call():
    # a caller's own Workspace.get (a subclass's, or an object that has nothing else) decides the scratch of each
    # call, also where a large enough buffer is there and where none is needed
    like, asked = torch.zeros(1), []

    class Own(bd.Workspace):
        def get(self, nbytes, device):
            asked.append((nbytes, torch.device(device)))
            self.buf = None                         # a fresh buffer per call
            return super().get(nbytes, device)

    class Bare:
        def __init__(self):
            self.mine = torch.zeros(4096, dtype=torch.uint8)

        def get(self, nbytes, device):
            asked.append((nbytes, torch.device(device)))
            return self.mine if nbytes else None

    for ws in (Own(), Bare()):
        asked.clear()
        for n in (1000, 500, 0):
            p, size = bd._ws("op", n, like, 0, ws)
            assert (p is None and size == 0) if n == 0 else (p % 256 == 0 and size >= n)
        assert asked == [(n, like.device) for n in (1000, 500, 0)]
    kept = bd.Workspace()
    first = bd._ws("op", 1000, like, 0, kept)
    assert bd._ws("op", 500, like, 0, kept) == first and kept.buf.numel() == 1256


def test_default_scratch_is_kept_and_grown():
    # without a caller's workspace: one buffer per (operation, device, stream), kept while it is large enough
    like = torch.zeros(1)
    key = ("test_default_scratch", like.get_device(), 7)
    try:
        assert bd._ws(key[0], 0, like, 7, None) == (None, 0)
        p, size = bd._ws(key[0], 1000, like, 7, None)
        assert p % 256 == 0 and size >= 1000
        assert bd._ws(key[0], 500, like, 7, None) == (p, size)
        assert bd._ws(key[0], 0, like, 7, None) == (None, 0)
        p, size = bd._ws(key[0], 5000, like, 7, None)
        assert p % 256 == 0 and size >= 5000 and not bd._default_ws[key].buf.any()
        assert ("test_default_scratch", like.get_device(), 8) not in bd._default_ws
    finally:
        bd._default_ws.pop(key, None)
