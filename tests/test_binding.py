"""The binding's packed cache descriptor, on the CPU: the bytes it passes are those of a KvDesc filled field by field."""
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
