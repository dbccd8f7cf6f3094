"""GPU parity: traj_confidence_topk against the fp64 oracle.

conf within 1e-4 absolute; idx bit-exact (equal values rank the lower index).
"""

import numpy as np
import pytest
import torch

import oracle
import paper_2608_27514_amd as tsp
from synthetic import WORKLOADS, decode_inputs, make_logits, seed_for, torch_dtype
from helpers import CONF_ATOL

pytestmark = pytest.mark.gpu


def _check(logits_gpu, k, rows=None, label=""):
    conf, idx = tsp.confidence_topk(logits_gpu, k)
    torch.cuda.synchronize()
    if rows is None:
        rows = np.arange(logits_gpu.shape[0])
    host = logits_gpu[torch.as_tensor(rows, device=logits_gpu.device)].float().cpu().numpy()
    rc, ri = oracle.confidence_topk(host, k)
    gc = conf.cpu().numpy()[rows]
    gi = idx.cpu().numpy()[rows]
    assert np.array_equal(gi, ri), f"{label}: idx mismatch in {int((gi != ri).any(axis=1).sum())} rows"
    err = np.abs(gc - rc).max()
    assert err <= CONF_ATOL, f"{label}: conf err {err}"
    return conf, idx


def test_tiny_fp32_full():
    wl = WORKLOADS[1]
    d = decode_inputs(wl, seed_for(1))
    lg = make_logits(d["row_margin"], d["row_top"], wl.V, torch.float32, seed_for(1)).cuda()
    _check(lg, wl.k, label="tiny-fp32")


def test_8b_siblings_full_size():
    """256 rows x 126464 bf16 -- the short-batch launch (8 waves per row), every row checked."""
    wl = WORKLOADS[2]
    d = decode_inputs(wl, seed_for(2))
    lg = make_logits(d["row_margin"], d["row_top"], wl.V, torch.bfloat16, seed_for(2)).cuda()
    _check(lg, 3, label="8b-siblings")


@pytest.mark.parametrize("rows", [1, 5, 40, 127])
def test_split_rows_full_vocab(rows):
    """Fewer than 128 rows: each row is split across workgroups and the partial records merged."""
    wl = WORKLOADS[2]
    d = decode_inputs(wl, seed_for(2, 1))
    lg = make_logits(d["row_margin"][:rows], d["row_top"][:rows], wl.V, torch.bfloat16, seed_for(2, 1)).cuda()
    assert tsp.confidence_topk_workspace_size(lg, 3) > 0
    _check(lg, 3, label=f"split rows={rows}")


@pytest.mark.parametrize("cid", [3, 4])
def test_full_size_sampled_rows(cid):
    wl = WORKLOADS[cid]
    d = decode_inputs(wl, seed_for(cid))
    lg = make_logits(d["row_margin"], d["row_top"], wl.V, torch.bfloat16, seed_for(cid), device="cuda")
    rows = np.random.default_rng(cid).choice(lg.shape[0], size=96, replace=False)
    rows = np.concatenate([[0, lg.shape[0] - 1], rows])
    _check(lg, 3, rows=rows, label=wl.name)


def test_batched_full_size_sampled_rows():
    wl = WORKLOADS[5]
    d = decode_inputs(wl, seed_for(5))
    lg = make_logits(d["row_margin"], d["row_top"], wl.V, torch.bfloat16, seed_for(5), device="cuda",
                     row_chunk=2048)
    rows = np.random.default_rng(5).choice(lg.shape[0], size=64, replace=False)
    rows = np.concatenate([[0, lg.shape[0] - 1], rows])
    _check(lg, 3, rows=rows, label=wl.name)
    del lg
    torch.cuda.empty_cache()


@pytest.mark.parametrize("k", [1, 2, 3, 4, 5, 8])
def test_exact_ties_every_k(k):
    rows, V = 300, 5000
    lg = make_logits(np.zeros(rows), np.zeros((rows, 3), dtype=np.int64), V, torch.bfloat16, 77 + k,
                     mode="ties").cuda()
    _check(lg, k, label=f"ties k={k}")


def test_raw_margin_rows_and_few_rows_split():
    wl = WORKLOADS[2].with_(N=1, parents=(-1,))
    d = decode_inputs(wl, 5)
    for rows in (1, 3, 32):
        lg = make_logits(d["row_margin"][:rows], d["row_top"][:rows], wl.V, torch.bfloat16, 9, mode="raw").cuda()
        _check(lg, 3, label=f"raw rows={rows}")


def test_strided_and_unaligned_rows_use_scalar_path():
    rows, V = 64, 3001
    base = make_logits(np.zeros(rows), np.zeros((rows, 3), dtype=np.int64), V + 67, torch.bfloat16, 4,
                       mode="ties").cuda()
    strided = base[:, :V]              # row stride 3068 elements (16-byte aligned)
    _check(strided, 3, label="strided")
    unaligned = base[:, 1:V + 1]       # base pointer off by 2 bytes
    _check(unaligned, 4, label="unaligned")
    f32 = make_logits(np.zeros(rows), np.zeros((rows, 3), dtype=np.int64), V + 5, torch.float32, 5,
                      mode="ties").cuda()[:, 1:V + 1]
    _check(f32, 2, label="fp32 unaligned")


# 4096 / 8200 / 12300 give 1, 2 and 3 full workgroup sweeps (bf16; fp32 twice as many) with
# and without a remainder, so the double-buffered sweep loop and its odd tail are exercised.
@pytest.mark.parametrize("V", [1, 7, 255, 1000, 2049, 4096, 8200, 12300])
def test_small_and_ragged_vocab(V):
    rng = np.random.default_rng(V)
    x = torch.from_numpy(rng.standard_normal((40, V)).astype(np.float32))
    for dt in (torch.float32, torch.bfloat16):
        _check(x.to(dt).cuda(), min(3, V), label=f"V={V} {dt}")


# The two short-batch launches: 128..511 rows stream 32768 bf16 (16384 fp32) values per sweep,
# 512..4095 rows 8192 (4096).  Each vocabulary gives 1, 3 or 5 whole sweeps (the two-sweep ring
# with and without an odd remainder) plus a ragged tail of whole vectors and single values.
@pytest.mark.parametrize("rows,V", [(130, 32776), (130, 98311), (130, 163848), (520, 8200), (520, 24583),
                                    (520, 41000)])
def test_short_batch_launches_ragged_vocab(rows, V):
    rng = np.random.default_rng(rows * 7 + V)
    x = torch.from_numpy(rng.standard_normal((rows, V)).astype(np.float32) * 2.0)
    for dt in (torch.float32, torch.bfloat16):
        _check(x.to(dt).cuda(), 3, label=f"rows={rows} V={V} {dt}")


# Rows that start anywhere inside a 16-byte vector: an odd stride moves the start from row to row
# through every offset, under each launch shape (split rows, 8, 4 and 1 waves per row); V = 1 .. 5 is
# shorter than the run up to the first aligned vector; up to 1024 values workgroups of 4 waves read
# one by one.
@pytest.mark.parametrize("rows,V", [(40, 1), (40, 5), (40, 12301), (130, 16391), (130, 32999), (520, 4099),
                                    (520, 20011), (4100, 1031), (4100, 9), (3, 126463), (40, 257), (130, 1024),
                                    (130, 1025), (520, 1023), (520, 1027), (4100, 1024)])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_rows_at_every_alignment(rows, V, dtype):
    rng = np.random.default_rng(rows + V)
    stride = V + 2 if V % 2 else V + 1
    x = torch.full((rows * stride + 1,), 1e30, dtype=dtype)  # the padding between rows would win
    x = x.as_strided((rows, V), (stride, 1), 1)
    x.copy_(torch.from_numpy(rng.standard_normal((rows, V)).astype(np.float32)))
    base = torch.empty(rows * stride + 1, dtype=dtype, device="cuda")
    base.copy_(x.as_strided((rows * stride + 1,), (1,), 0))
    sample = np.unique(np.concatenate([np.arange(min(rows, 40)), rng.choice(rows, size=min(rows, 60), replace=False)]))
    _check(base.as_strided((rows, V), (stride, 1), 1), min(3, V), rows=sample, label=f"rows={rows} V={V} {dtype}")


def test_negative_infinity_entries():
    x = torch.full((4, 300), -float("inf"))
    x[:, 5] = 1.0
    x[1, 7] = 1.0
    x[2, 299] = 3.0
    x[3, :] = torch.linspace(-3, 3, 300)
    x[3, ::2] = -float("inf")
    _check(x.cuda(), 3, label="-inf fp32")
    _check(x.to(torch.bfloat16).cuda(), 3, label="-inf bf16")


def test_zero_rows_is_a_no_op():
    x = torch.empty((0, 100), dtype=torch.bfloat16, device="cuda")
    conf, idx = tsp.confidence_topk(x, 3)
    assert conf.shape == (0, 3)


def test_bad_arguments_raise():
    x = torch.zeros((2, 5), dtype=torch.float32, device="cuda")
    with pytest.raises(tsp.TrajSpecError):
        tsp.confidence_topk(x, 9)
    with pytest.raises(tsp.TrajSpecError):
        tsp.confidence_topk(x, 6)
