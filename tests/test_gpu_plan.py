"""Automatic plans (splits and row tile chosen by the library) around whole
waves of workgroups, against one split and against the oracle on sampled jobs:
the split rows of one call are rounded to fp16 or kept in fp32, so two plans
agree to the library's parity bound."""
import numpy as np
import pytest
import torch

from paper_2606_01502_amd import mla
from tests import gpu_helpers as G

pytestmark = pytest.mark.gpu

SCALE = 576 ** -0.5


def _inputs(R, Mq, H, K, NB, tokens, per_row, seed):
    g = torch.Generator(device=G.device())
    g.manual_seed(seed)

    def normal(*shape):
        return torch.randn(shape, generator=g, device=G.device()).bfloat16()

    P = 96
    table = torch.stack([torch.randperm(P, generator=g, device=G.device())[:NB] for _ in range(R)])
    n_ids = NB * 64 if tokens else NB
    lists = R * Mq if per_row else R
    sel = torch.stack([torch.randperm(n_ids, generator=g, device=G.device())[:K]
                       for _ in range(lists)])
    if per_row:
        sel = sel.view(R, Mq, K)
    return dict(q_lat=normal(R, Mq, H, 512), q_pe=normal(R, Mq, H, 64), ckv=normal(P, 64, 512) * 0.5,
                kpe=normal(P, 64, 64) * 0.5, table=table.int(), sel=sel.int())


# (jobs, query rows, heads, slots, blocks of the table): grids that just fit a
# wave of 256 workgroups, just pass it, and pass two and three
@pytest.mark.parametrize("R,Mq,H,K,NB,tokens,per_row", [
    (20, 1, 128, 40, 40, False, False), (86, 1, 64, 12, 40, False, False),
    (128, 1, 16, 9, 40, False, False), (129, 1, 16, 9, 40, False, False),
    (257, 1, 16, 24, 40, False, False), (300, 1, 128, 10, 40, False, False),
    (24, 1, 128, 700, 40, True, False), (130, 1, 64, 129, 8, True, False),
    (1, 100, 16, 16, 64, False, True), (1, 130, 20, 6, 90, False, True)])
def test_automatic_plans(R, Mq, H, K, NB, tokens, per_row):
    print(f"case: plan R={R} Mq={Mq} H={H} K={K} tokens={tokens} per_row={per_row}", flush=True)
    t = _inputs(R, Mq, H, K, NB, tokens, per_row, 7000 + R + K)
    args = (t["q_lat"], t["q_pe"], t["ckv"], t["kpe"], t["table"], t["sel"], SCALE)
    out, lse = mla.sparse_partial_attn(*args, tokens=tokens)
    ref_o, ref_l = mla.sparse_partial_attn(*args, tokens=tokens, n_splits=1)
    torch.cuda.synchronize()
    # weights are rounded to bf16 (2^-9) and split rows to fp16 (2^-11 of the
    # row's largest), in each of the two plans
    err = (out - ref_o).abs().amax(-1) / ref_o.abs().amax(-1)
    assert float(err.max()) <= 2 * (2 ** -8 + 2 ** -11), float(err.max())
    assert float((lse - ref_l).abs().max()) <= 1e-4
    # float64 attention of the first and the last job's last query row
    for r in (0, R - 1):
        ids = t["sel"][r, Mq - 1] if per_row else t["sel"][r]
        if tokens:
            blk = t["table"][r][(ids // 64).long()].long()
            k_lat, k_pe = t["ckv"][blk, (ids % 64).long()], t["kpe"][blk, (ids % 64).long()]
        else:
            blk = t["table"][r][ids.long()].long()
            k_lat, k_pe = t["ckv"][blk].reshape(-1, 512), t["kpe"][blk].reshape(-1, 64)
        k_lat, k_pe = k_lat.double().cpu(), k_pe.double().cpu()
        s = (t["q_lat"][r, Mq - 1].double().cpu() @ k_lat.T + t["q_pe"][r, Mq - 1].double().cpu() @ k_pe.T) * SCALE
        want_l = torch.logsumexp(s, -1)
        want = torch.softmax(s, -1) @ k_lat
        got = out[r, Mq - 1].double().cpu()
        e = (got - want).abs().amax(-1) / want.abs().amax(-1)
        assert float(e.max()) <= 2 ** -8 + 2 ** -11, float(e.max())
        assert float((lse[r, Mq - 1].double().cpu() - want_l).abs().max()) <= 1e-4


@pytest.mark.parametrize("R,H,K,tokens", [(300, 16, 64, False), (269, 8, 96, False), (258, 16, 1000, True)])
def test_sums_stay_in_fp32(R, H, K, tokens):
    """More jobs than compute units, a few of them in a last wave: one split that
    sums in registers covers the chip, and other plans keep its fp32.  With zero
    queries every weight is 1, exact in bf16, and a row is the mean of its
    tokens: fp32 sums of 4096 terms stay within 2^-16 of the row's largest value
    (a row rounded to fp16 is off by up to 2^-12 of it)."""
    print(f"case: fp32 sums R={R} H={H} K={K} tokens={tokens}", flush=True)
    t = _inputs(R, 1, H, min(K, 96) if not tokens else K, 96 if not tokens else 30, tokens, False, 7300 + R)
    out, lse = mla.sparse_partial_attn(torch.zeros_like(t["q_lat"]), torch.zeros_like(t["q_pe"]), t["ckv"], t["kpe"],
                                       t["table"], t["sel"], SCALE, tokens=tokens)
    torch.cuda.synchronize()
    for r in (0, R // 2, R - 1):
        ids = t["sel"][r].long()
        rows = (t["ckv"][t["table"][r][ids // 64].long(), ids % 64] if tokens
                else t["ckv"][t["table"][r][ids].long()].reshape(-1, 512))
        want = rows.double().mean(0)
        err = (out[r, 0].double() - want).abs().amax() / want.abs().amax()
        assert float(err) <= 2 ** -16, float(err)
        assert float((lse[r].double() - np.log(rows.shape[0])).abs().max()) <= 1e-5


@pytest.mark.parametrize("R,H,K,cover,tile", [(300, 16, 64, 1, 64), (136, 128, 64, 2, 128)])
def test_captured_with_the_covering_plan_s_workspace(R, H, K, cover, tile):
    """A call that covers the chip in fewer splits than its plan takes is
    captured with no more workspace than those need (none for one split), and
    gives their result; replays repeat it, with eager work between them."""
    print(f"case: capture R={R} H={H} K={K}", flush=True)
    t = _inputs(R, 1, H, K, K, False, False, 7400 + R)
    args = (t["q_lat"], t["q_pe"], t["ckv"], t["kpe"], t["table"], t["sel"], SCALE)
    ref = mla.sparse_partial_attn(*args, n_splits=cover, row_tile=tile)  # (on another stream)
    out, lse = torch.empty_like(ref[0]), torch.empty_like(ref[1])
    torch.cuda.synchronize()
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        if cover > 1:
            mla.sparse_partial_attn(*args, out, lse, n_splits=cover, row_tile=tile)
            stream.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=stream):
            mla.sparse_partial_attn(*args, out, lse)
        for rep in range(3):
            out.fill_(float("nan"))
            lse.fill_(float("nan"))
            stream.synchronize()
            g.replay()
            stream.synchronize()
            assert torch.equal(out, ref[0]) and torch.equal(lse, ref[1]), rep
            mla.sparse_partial_attn(*args)  # eager: the plan's own workspace
            stream.synchronize()
    torch.cuda.synchronize()


def test_capture_without_the_covering_workspace_is_refused():
    print("case: capture refused", flush=True)
    t = _inputs(136, 1, 128, 64, 64, False, False, 7450)
    out = torch.empty((136, 1, 128, 512), device=G.device())
    lse = torch.empty((136, 1, 128), device=G.device())
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        g = torch.cuda.CUDAGraph()
        with pytest.raises(mla.MlaError) as e:
            with torch.cuda.graph(g, stream=stream):
                mla.sparse_partial_attn(t["q_lat"], t["q_pe"], t["ckv"], t["kpe"], t["table"], t["sel"], SCALE, out, lse)
        assert e.value.status == mla.MLA_ERR_UNSUPPORTED and "capture" in str(e.value)
    torch.cuda.synchronize()
