"""The 64-row kernel at the edges of its tiles, stages and pipeline, against
the oracle: row counts around its 8-, 16- and 32-row groups, odd head counts
(its query rows are loaded row by row), stage counts below and above the ring,
strided query rows, and scores that keep raising the running maxima.

Tolerances are the parity bar of gpu_helpers.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2606_01502_amd import mla, workloads as W
from tests import gpu_helpers as G

pytestmark = pytest.mark.gpu


def _ref(w):
    return oracle.partial(w.q_lat, w.q_pe, w.ckv, w.kpe, w.table, w.sel, w.scale, w.ckv_scale,
                          w.kpe_scale, tokens=w.tokens)


def _check(w, what, **kw):
    print("case:", what, flush=True)
    out, lse = G.run_partial(G.upload(w), w.scale, row_tile=64, tokens=w.tokens, **kw)
    G.assert_parity(out, lse, *_ref(w), what)


@pytest.mark.parametrize("kv", ["bf16", "fp8", "fp8split"])
@pytest.mark.parametrize("mq,h", [(1, 1), (1, 8), (5, 3), (1, 17), (1, 31), (7, 7), (1, 64), (1, 65), (3, 43)])
def test_row_edges(mq, h, kv):
    w = W.random_case(900 + 7 * mq + h, R=2, Mq=mq, H=h, P=12, NB=9, K=3)
    if kv != "bf16":
        w = w.to_fp8(kv == "fp8")
    _check(w, f"rows {mq}x{h} {kv}")


@pytest.mark.parametrize("kv", ["bf16", "fp8", "fp8split"])
@pytest.mark.parametrize("k", [1, 31, 32, 33, 64, 65, 95, 97, 191, 193, 225])
def test_stage_counts_tokens(k, kv):
    # 32 tokens a stage: one stage, a full ring and beyond it, ragged ends
    w = W.random_case(930 + k, R=2, Mq=1, H=40, P=16, NB=11, K=k, tokens=True)
    if kv != "bf16":
        w = w.to_fp8(kv == "fp8")
    _check(w, f"tokens {k} {kv}", n_splits=1)


@pytest.mark.parametrize("kv", ["bf16", "fp8"])
@pytest.mark.parametrize("blocks", [0, 1, 2, 3, 4, 7])
def test_stage_counts_blocks(blocks, kv):
    w = W.random_case(960 + blocks, R=3, Mq=2, H=24, P=16, NB=11, K=8, n_valid=[blocks, 8, 0],
                      pad_pattern="interleaved")
    if kv != "bf16":
        w = w.to_fp8()
    _check(w, f"blocks {blocks} {kv}", n_splits=1)


@pytest.mark.parametrize("kv", ["bf16", "fp8"])
def test_per_row_counters_past_the_query_rows(kv):
    # so many logical blocks that the compaction's counters reach the place of
    # the query rows (and, for fp8, past the ring)
    w = W.random_case(980, R=1, Mq=64, H=1, P=64, NB=1100, K=6, per_row=True)
    if kv != "bf16":
        w = w.to_fp8()
    _check(w, f"per-row counters {kv}", n_splits=1)


@pytest.mark.parametrize("wire", [False, True])
def test_strided_queries_and_rising_maxima(wire):
    # blocks of growing magnitude: most stages raise some row's maximum by more
    # than the rescale threshold; the queries are slices of wider tensors
    w = W.random_case(990, R=2, Mq=3, H=10, P=20, NB=12, K=12)
    for r in range(2):
        w.sel[r] = np.arange(12)
        for j in range(12):
            b = w.table[r, j]
            f = np.float32(0.25 * 1.45 ** j)
            w.ckv[b] = W.f32_to_bf16_bits(W.bf16_bits_to_f32(w.ckv[b]) * f)
    t = G.upload(w)
    wide = torch.zeros((2, 5, 13, 512 + 64), dtype=torch.bfloat16, device="cuda")
    wide[:, 1:4, 2:12, :512] = t["q_lat"]
    wide[:, 1:4, 2:12, 512:] = t["q_pe"]
    ref_o, ref_l = _ref(w)
    for ns in (1, 3):
        print(f"case: strided wire={wire} splits={ns}", flush=True)
        out, lse = mla.sparse_partial_attn(wide[:, 1:4, 2:12, :512], wide[:, 1:4, 2:12, 512:], t["ckv"],
                                           t["kpe"], t["table"], t["sel"], w.scale, n_splits=ns,
                                           row_tile=64, wire=wire)
        torch.cuda.synchronize()
        lse = lse.double().cpu().numpy()
        if wire:
            lse = lse[..., 0] + np.log(lse[..., 1])
        G.assert_parity(out.double().cpu().numpy(), lse, ref_o, ref_l, f"wire={wire} splits={ns}")


@pytest.mark.parametrize("kind", ["blocks", "tokens", "per_row"])
@pytest.mark.parametrize("kv", ["bf16", "fp8", "fp8split"])
@pytest.mark.parametrize("mq,h", [(16, 1), (2, 16), (3, 11)])
def test_half_tiles(mq, h, kv, kind):
    # 16, 32 and 33 rows: the last takes both row halves; from one stage to
    # beyond the ring, blocks of growing magnitude so that maxima rise
    k = {"blocks": 9, "tokens": 289, "per_row": 5}[kind]
    w = W.random_case(1010 + 7 * mq + h, R=2, Mq=mq, H=h, P=16, NB=11, K=k, tokens=kind == "tokens",
                      per_row=kind == "per_row")
    for j in range(11):
        b = w.table[0, j]
        w.ckv[b] = W.f32_to_bf16_bits(W.bf16_bits_to_f32(w.ckv[b]) * np.float32(0.25 * 1.5 ** j))
    if kv != "bf16":
        w = w.to_fp8(kv == "fp8")
    for ns in (1, 3):
        _check(w, f"half tile {mq}x{h} {kv} {kind} splits={ns}", n_splits=ns)


@pytest.mark.parametrize("shared_q", [False, True])
def test_per_row_lists_beyond_the_scratch(shared_q):
    # 64 query rows x 16 slots a tile, a full list: in two splits the rows of all
    # jobs together would exceed the allocation-free entry's scratch
    R, Mq, K, NB = 600, 64, 16, 24
    print(f"case: per-row beyond scratch shared_q={shared_q}", flush=True)
    w = W.random_case(1100, R=R, Mq=Mq, H=1, P=40, NB=NB, K=K, per_row=True)
    t = G.upload(w)
    n_q = R // 2 if shared_q else R
    args = (t["q_lat"][:n_q], t["q_pe"][:n_q], t["ckv"], t["kpe"], t["table"], t["sel"], w.scale)
    for rt in (0, 64):
        out, lse = mla.sparse_partial_attn(*args, row_tile=rt, no_alloc=True)
        ref_o, ref_l = mla.sparse_partial_attn(*args, row_tile=128, n_splits=1)
        torch.cuda.synchronize()
        # the split rows' fp16 rounding and the weights' to bf16, in both plans
        err = (out - ref_o).abs().amax(-1) / ref_o.abs().amax(-1).clamp_min(1e-30)
        assert float(err.max()) <= 2 * (2 ** -8 + 2 ** -11), float(err.max())
        same = (lse == ref_l) | ((lse - ref_l).abs() <= 1e-4)
        assert bool(same.all())


@pytest.mark.parametrize("mq,h,k", [(8, 8, 64), (8, 8, 65), (16, 4, 64), (8, 8, 128), (8, 8, 129),
                                    (3, 64, 512), (3, 64, 513), (70, 1, 8), (70, 1, 9)])
def test_long_per_row_lists(mq, h, k):
    # a tile's slots at and past 512 (the eight-wave kernel's list) and 1024 (the
    # longest: ranges of slots from there on)
    w = W.random_case(1130 + mq + k, R=2, Mq=mq, H=h, P=80, NB=2 * k + 3 if h < 64 else 600, K=k,
                      per_row=True, shared_frac=0.5, allow_dup=True)
    for ns in (0, 1, 3):
        _check(w, f"long list {mq}x{h} K={k} splits={ns}", n_splits=ns)


@pytest.mark.parametrize("R,Mq,H,K,NB,n_q", [(300, 4, 16, 400, 500, 300), (200, 8, 8, 400, 600, 2),
                                             (1, 32768, 1, 12, 24, 1)])
def test_allocation_free_calls_with_long_lists(R, Mq, H, K, NB, n_q):
    # many jobs, jobs that share few query rows, and one job of many rows
    print(f"case: no_alloc R={R} Mq={Mq} H={H} K={K} n_q={n_q}", flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(1150 + R)

    def normal(*shape):
        return torch.randn(shape, generator=g, device="cuda").bfloat16()

    P = 700
    q_lat, q_pe, ckv, kpe = normal(n_q, Mq, H, 512), normal(n_q, Mq, H, 64), normal(P, 64, 512), normal(P, 64, 64)
    table = torch.stack([torch.randperm(P, generator=g, device="cuda")[:NB] for _ in range(R)]).int()
    sel = torch.rand((R, Mq, NB), generator=g, device="cuda").topk(K).indices.int()
    out, lse = mla.sparse_partial_attn(q_lat, q_pe, ckv, kpe, table, sel, 576 ** -0.5, no_alloc=True)
    torch.cuda.synchronize()
    for r, i in ((0, 0), (R - 1, Mq - 1), (R // 2, Mq // 2)):
        blk = table[r][sel[r, i].long()].long()
        k_lat, k_pe = ckv[blk].reshape(-1, 512).double().cpu(), kpe[blk].reshape(-1, 64).double().cpu()
        s = (q_lat[r % n_q, i].double().cpu() @ k_lat.T + q_pe[r % n_q, i].double().cpu() @ k_pe.T) * 576 ** -0.5
        G.assert_parity(out[r, i].double().cpu().numpy(), lse[r, i].double().cpu().numpy(),
                        (torch.softmax(s, -1) @ k_lat).numpy(), torch.logsumexp(s, -1).numpy(), f"job {r} row {i}")


@pytest.mark.parametrize("h", [8, 40])
def test_normaliser_is_a_correctly_rounded_reciprocal(h):
    # zero queries: every weight is 1, and job r's first token alone has a value
    # (1 in every column), so that a row is 1 / (r + 1); r + 1 runs over the
    # counts of a list
    print(f"case: normaliser h={h}", flush=True)
    R = 1024
    dev = G.device()
    ckv = torch.zeros((17, 64, 512), dtype=torch.bfloat16, device=dev)
    ckv[16, 0] = 1.0
    kpe = torch.zeros((17, 64, 64), dtype=torch.bfloat16, device=dev)
    table = torch.arange(17, dtype=torch.int32, device=dev).expand(R, 17).contiguous()
    sel = torch.arange(-1, R - 1, dtype=torch.int32, device=dev).expand(R, R).contiguous()
    sel[:, 0] = 16 * 64
    sel[torch.arange(R, device=dev)[None, :] > torch.arange(R, device=dev)[:, None]] = -1
    q = torch.zeros((R, 1, h, 512), dtype=torch.bfloat16, device=dev)
    out, lse = mla.sparse_partial_attn(q, q[..., :64].contiguous(), ckv, kpe, table, sel, 1.0, n_splits=1,
                                       row_tile=64, tokens=True)
    torch.cuda.synchronize()
    want = (1.0 / np.arange(1, R + 1, dtype=np.float64)).astype(np.float32)
    assert np.array_equal(out.cpu().numpy(), np.broadcast_to(want[:, None, None, None], (R, 1, h, 512)))


@pytest.mark.parametrize("kind", ["blocks", "tokens", "per_row"])
@pytest.mark.parametrize("kv", ["bf16", "fp8", "fp8split"])
@pytest.mark.parametrize("h", [8, 24])
def test_maxima_of_whole_blocks(h, kv, kind):
    """A row's maximum is taken over the 64 tokens of its first block, so that the
    heaviest of them weighs 1, exact in bf16.  Here that token is in the second
    half and 256 / 1.5 times as heavy as the others: 1.5 / 256 is exact too,
    170.67 (its weight against the first half's maximum) would round to 171 and
    move the row by 5e-4.  fp32 scores and sums leave 2^-16."""
    print(f"case: maxima of blocks h={h} {kv} {kind}", flush=True)
    dev = G.device()
    heavy = 41
    lat = torch.zeros((3, 64, 512))
    pe = torch.zeros((3, 64, 64))
    lat[:2, heavy] = 1.0  # block 2: nobody's heavy token (scores 0)
    pe[:2, heavy, 0] = 1.0
    kw = {}
    if kv == "bf16":
        ckv, kpe = lat.bfloat16().to(dev), pe.bfloat16().to(dev)
    else:
        ckv, kpe = (t.to(torch.float8_e4m3fn).view(torch.uint8).to(dev) for t in (lat, pe))
        one = torch.ones(3, device=dev)
        kw = dict(ckv_scale=one, kpe_scale=one if kv == "fp8" else one.clone())
    mq = 2 if kind == "per_row" else 1
    q_lat = torch.zeros((1, mq, h, 512), dtype=torch.bfloat16, device=dev)
    q_pe = torch.zeros((1, mq, h, 64), dtype=torch.bfloat16, device=dev)
    q_pe[..., 0] = 1.0
    table = torch.tensor([[2, 1, 0]], dtype=torch.int32, device=dev)
    if kind == "tokens":
        sel = torch.arange(64, 128, dtype=torch.int32, device=dev)[None]
    elif kind == "blocks":
        sel = torch.tensor([[1]], dtype=torch.int32, device=dev)
    else:  # the second row's first block is the second of the tile's list
        sel = torch.tensor([[[0, -1], [2, -1]]], dtype=torch.int32, device=dev)
    out, lse = mla.sparse_partial_attn(q_lat, q_pe, ckv, kpe, table, sel, float(np.log(256 / 1.5)), n_splits=1,
                                       row_tile=64, tokens=kind == "tokens", **kw)
    torch.cuda.synchronize()
    want = 1.0 / (1.0 + 63 * 1.5 / 256)
    assert float((out[0, mq - 1].double() / want - 1).abs().max()) <= 2 ** -16
    if kind == "per_row":
        assert float(out[0, 0].abs().max()) == 0.0
