"""Performance cases of the library: what its callers have it do, over the
sizes, selection kinds and cache types they use.

Every case goes through the Python binding's public entry points on inputs
that are already on the GPU.  Partial and merge calls are prepared once
(`prepare_partial`, `prepare_merge`), as a serving loop over static buffers
holds them; the FETCH copies have no prepared form and are called directly
with their output buffers given.

Fields of a case (those that its kind uses):
  kind    blocks  partial attention over one block selection per job
          rows    one job whose Mq query rows are requesters of one holder
                  chunk; `sparse` gives each row a selection of its own
          tokens  partial attention over an indexer's single tokens
          route   partial attention of every (request, chunk) job of a batch,
                  then the requester's merge of each request's parts
          fetch   the scattered gather of a token selection over all layers,
                  and the splice of the payload into a requester's pools
  R, Mq, H        jobs (route: requests), query rows per job, heads
  NB, K           logical blocks per job's chunk, selection slots (tokens
                  for kinds tokens and fetch)
  valid           slots that hold an id (the rest are empty)
  hits            route: chunks that each request is routed to
  kv              bf16 | fp8 (one scale per block) | fp8split (separate
                  latent and RoPE scales)
  draw_ids        uniform | zipf | all
  wire            route: the partials in the 1032-byte bf16 wire form
  L, start, delta, pairing   fetch: layers, the splice's place and rotation
"""
import math

import numpy as np
import torch

from paper_2606_01502_amd import mla

DLAT, DPE, BLOCK = 512, 64, 64
SCALE = 1.0 / math.sqrt(192.0)
ROPE_BASE = 10000.0


# ---------------------------------------------------------------- the cases
def listed():
    return [
        # the smallest call: one 16-head share of one request over a 256-token
        # chunk with empty slots; launches and latency are all there is
        dict(name="tiny", kind="blocks", R=1, Mq=1, H=16, NB=4, K=4, valid=2, kv="bf16",
             draw_ids="uniform", sigma=1.0),
        # one routed request at full width: 128 heads, the top-2048 budget
        # (32 blocks) of a 4096-token chunk
        dict(name="one-request", kind="blocks", R=1, Mq=1, H=128, NB=64, K=32, valid=32,
             kv="bf16", draw_ids="uniform", sigma=0.5),
        # a tensor-parallel share (16 of 128 heads) of 16 requests with four
        # rows each (speculative tokens) on long chunks, hot blocks first
        dict(name="few-head", kind="blocks", R=16, Mq=4, H=16, NB=512, K=32, valid=32,
             kv="bf16", draw_ids="zipf", sigma=1.0),
        # odd sizes: rows that fill no tile, a slot count that no split
        # divides, empty slots, an fp8 cache with separate RoPE scales
        dict(name="ragged-fp8", kind="blocks", R=5, Mq=3, H=40, NB=150, K=53, valid=47,
             kv="fp8split", draw_ids="uniform", sigma=0.5),
        # a decode batch: 64 requests, each routed to 4 chunks of one holder,
        # and the merge of the 4 parts
        dict(name="batched-merge", kind="route", R=64, Mq=1, H=128, NB=128, K=32, valid=32,
             hits=4, chunks=256, kv="bf16", draw_ids="uniform", sigma=0.5, wire=False),
        # dense decode over long resident contexts, without a selection, from
        # a bf16 cache and from an fp8 cache: the largest calls
        dict(name="dense-local", kind="blocks", R=32, Mq=1, H=128, NB=1024, K=1024, valid=1024,
             kv="bf16", draw_ids="all", sigma=0.5),
        dict(name="dense-local-fp8", kind="blocks", R=32, Mq=1, H=128, NB=1024, K=1024,
             valid=1024, kv="fp8", draw_ids="all", sigma=0.5),
        # one holder chunk of 2048 tokens serving 256 requesters' 16-head
        # shares, all of it attended by each
        dict(name="holder-dense", kind="rows", R=1, Mq=256, H=16, NB=32, K=32, valid=32,
             kv="bf16", draw_ids="all", sigma=0.5, sparse=False),
        # the same holder under sparse selection: 64 requesters, each with
        # its own 32 of 128 blocks, hot blocks shared
        dict(name="holder-sparse", kind="rows", R=1, Mq=64, H=16, NB=128, K=32, valid=32,
             kv="bf16", draw_ids="zipf", sigma=0.5, sparse=True),
        # a token-level indexer's top-2048 of 32K-token chunks, 64 requests
        dict(name="tokens", kind="tokens", R=64, Mq=1, H=128, NB=512, K=2048, valid=2048,
             kv="bf16", draw_ids="uniform", sigma=0.5),
        # a small batch whose partials cross a link: wire-form rows, three
        # chunks a request, an odd number of heads and slots
        dict(name="wire-route", kind="route", R=12, Mq=2, H=24, NB=96, K=19, valid=19, hits=3,
             chunks=40, kv="bf16", draw_ids="uniform", sigma=0.5, wire=True),
        # the move-the-cache side: 2048 selected tokens of a 27-layer model
        # gathered, then spliced and re-rotated at an unaligned position
        dict(name="fetch", kind="fetch", L=27, K=2048, NB=512, start=37, delta=4096, pairing=0),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["blocks", "blocks", "dense", "rows", "tokens", "route", "fetch"])
    kv = rng.choice(["bf16", "bf16", "fp8", "fp8split"])
    if kind == "blocks":
        R, Mq, H = _log(rng, 1, 64), rng.randint(1, 4), rng.choice([8, 16, 24, 32, 40, 64, 128])
        K = _log(rng, 2, 64)
        NB = min(512, max(K, _log(rng, K, 16 * K)))
        return dict(kind="blocks", R=R, Mq=Mq, H=H, NB=NB, K=K, valid=rng.randint((K + 1) // 2, K),
                    kv=kv, draw_ids=rng.choice(["uniform", "zipf"]), sigma=0.5)
    if kind == "dense":
        R, NB = _log(rng, 1, 32), _log(rng, 48, 1024)
        return dict(kind="blocks", R=R, Mq=1, H=rng.choice([64, 128]), NB=NB, K=NB, valid=NB,
                    kv=kv, draw_ids="all", sigma=0.5)
    if kind == "rows":
        n, sparse = _log(rng, 6, 256), rng.random() < 0.5
        NB = rng.randint(64, 160) if sparse else rng.randint(16, 64)
        K = rng.randint(16, 32) if sparse else NB
        return dict(kind="rows", R=1, Mq=n, H=rng.choice([16, 20, 32]), NB=NB, K=K, valid=K,
                    kv="bf16" if sparse else kv, draw_ids="zipf" if sparse else "all", sigma=0.5,
                    sparse=sparse)
    if kind == "tokens":
        K = _log(rng, 64, 2048)
        return dict(kind="tokens", R=_log(rng, 1, 64), Mq=1, H=rng.choice([16, 64, 128]),
                    NB=min(512, (K + 63) // 64 * rng.choice([2, 4, 8, 16])), K=K,
                    valid=rng.randint(K * 3 // 4, K), kv=kv, draw_ids="uniform", sigma=0.5)
    if kind == "route":
        hits, K = rng.randint(2, 6), rng.randint(4, 32)
        return dict(kind="route", R=_log(rng, 2, 48), Mq=rng.randint(1, 2),
                    H=rng.choice([16, 24, 64, 128]), NB=rng.randint(K, 128), K=K, valid=K,
                    hits=hits, chunks=rng.randint(16, 128), kv=kv, draw_ids="uniform", sigma=0.5,
                    wire=rng.random() < 0.5)
    K = _log(rng, 55, 4096)
    return dict(kind="fetch", L=rng.choice([1, 4, 27, 61]), K=K,
                NB=(K + 63) // 64 * rng.choice([2, 4, 8]), start=rng.randint(0, 4000),
                delta=rng.randint(-4096, 32768), pairing=rng.randint(0, 1))


# ---------------------------------------------------------------- inputs
def _normal(g, shape, sigma):
    return torch.randn(shape, generator=g, device="cuda", dtype=torch.bfloat16).mul_(sigma)


def _pools(g, P, kv, sigma):
    """(ckv, kpe, ckv_scale, kpe_scale): a pool of P blocks ~ N(0, sigma)."""
    if kv == "bf16":
        return (_normal(g, (P, BLOCK, DLAT), sigma), _normal(g, (P, BLOCK, DPE), sigma), None,
                None)
    ckv = torch.empty((P, BLOCK, DLAT), dtype=torch.uint8, device="cuda")
    kpe = torch.empty((P, BLOCK, DPE), dtype=torch.uint8, device="cuda")
    cs = torch.empty(P, dtype=torch.float32, device="cuda")
    ks = cs if kv == "fp8" else torch.empty_like(cs)
    for lo in range(0, P, 4096):
        hi = min(P, lo + 4096)
        x = torch.randn((hi - lo, BLOCK, DLAT + DPE), generator=g, device="cuda").mul_(sigma)
        parts = [(x[..., :DLAT], ckv, cs), (x[..., DLAT:], kpe, ks)]
        if kv == "fp8":
            cs[lo:hi] = x.abs().amax(dim=(1, 2)) / 448.0
        for v, codes, s in parts:
            if kv != "fp8":
                s[lo:hi] = v.abs().amax(dim=(1, 2)) / 448.0
            q = (v / s[lo:hi, None, None]).clamp_(-448.0, 448.0)
            codes[lo:hi] = q.to(torch.float8_e4m3fn).view(torch.uint8)
    return ckv, kpe, cs, ks


def _ids(rs, rows, n, k, how):
    """k distinct sorted ids below n for each of `rows` lists; zipf(1.1)
    weights the first positions."""
    if how == "all":
        return np.tile(np.arange(k, dtype=np.int32), (rows, 1))
    key = rs.gumbel(size=(rows, n))
    if how == "zipf":
        key -= 1.1 * np.log(np.arange(1, n + 1))
    top = np.argpartition(-key, k - 1, axis=1)[:, :k] if k < n else np.tile(np.arange(n), (rows, 1))
    return np.sort(top, axis=1).astype(np.int32)


def _slots(ids, K):
    """The ids in the first of K slots, the rest empty (-1)."""
    s = np.full(ids.shape[:-1] + (K,), -1, np.int32)
    s[..., :ids.shape[-1]] = ids
    return s


def _gpu(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _inputs(case, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    rs = np.random.default_rng([seed, 77])
    if case["kind"] == "fetch":
        L, K, NB = case["L"], case["K"], case["NB"]
        nb = (case["start"] + K + BLOCK - 1) // BLOCK + 1
        return dict(src_ckv=_normal(g, (L, NB, BLOCK, DLAT), 0.5),
                    src_kpe=_normal(g, (L, NB, BLOCK, DPE), 0.5),
                    src_table=_gpu(rs.permutation(NB).astype(np.int32)),
                    sel=_gpu(_ids(rs, 1, NB * BLOCK, K, "uniform")[0]),
                    ckv=_normal(g, (L, nb + 2, BLOCK, DLAT), 0.5),
                    kpe=_normal(g, (L, nb + 2, BLOCK, DPE), 0.5),
                    table=_gpu(rs.permutation(nb + 2)[:nb].astype(np.int32)))
    R, Mq, H, NB, K = (case[k] for k in ("R", "Mq", "H", "NB", "K"))
    n_ids = NB * BLOCK if case["kind"] == "tokens" else NB
    if case["kind"] == "route":
        hits, C = case["hits"], case["chunks"]
        P = C * NB
        perm = rs.permutation(P).astype(np.int32).reshape(C, NB)
        # jobs are slot-major: job = hit * R + request
        chunks = np.argsort(rs.random((R, C)), axis=1)[:, :hits].T.reshape(-1)
        table = perm[chunks]
        sel = _slots(_ids(rs, hits * R, n_ids, case["valid"], case["draw_ids"]), K)
    elif case["kind"] == "rows":
        P = 2 * NB
        table = rs.permutation(P)[:NB].astype(np.int32)[None]
        if case["sparse"]:
            sel = _slots(_ids(rs, Mq, n_ids, case["valid"], case["draw_ids"]), K)[None]
        else:
            sel = _slots(_ids(rs, 1, n_ids, case["valid"], case["draw_ids"]), K)
    else:
        P = R * NB
        table = rs.permutation(P).astype(np.int32).reshape(R, NB)
        sel = _slots(_ids(rs, R, n_ids, case["valid"], case["draw_ids"]), K)
    ckv, kpe, cs, ks = _pools(g, P, case["kv"], case["sigma"])
    return dict(q_lat=_normal(g, (R, Mq, H, DLAT), 1.0), q_pe=_normal(g, (R, Mq, H, DPE), 1.0),
                ckv=ckv, kpe=kpe, cs=cs, ks=ks, table=_gpu(table), sel=_gpu(sel))


def prepare(case, seed):
    t = _inputs(case, seed)
    if case["kind"] == "fetch":
        t["pay_ckv"] = torch.empty((case["L"], case["K"], DLAT), dtype=torch.bfloat16, device="cuda")
        t["pay_kpe"] = torch.empty((case["L"], case["K"], DPE), dtype=torch.bfloat16, device="cuda")
        t["case"] = case
        return t
    route = case["kind"] == "route"
    wire = route and case["wire"]
    partial = mla.prepare_partial(t["q_lat"], t["q_pe"], t["ckv"], t["kpe"], t["table"], t["sel"],
                                  SCALE, ckv_scale=t["cs"], kpe_scale=t["ks"],
                                  tokens=case["kind"] == "tokens", wire=wire)
    state = dict(case=case, inputs=t, partial=partial)
    if route:
        out, lse = partial.result
        R = case["R"]
        state["merge"] = mla.prepare_merge([out[j * R:(j + 1) * R] for j in range(case["hits"])],
                                           [lse[j * R:(j + 1) * R] for j in range(case["hits"])],
                                           out_lse=True)
    return state


def run(state):
    case = state["case"]
    if case["kind"] == "fetch":
        s = state
        mla.fetch_gather(s["src_ckv"], s["src_kpe"], s["src_table"], s["sel"],
                         out_ckv=s["pay_ckv"], out_kpe=s["pay_kpe"])
        mla.fetch_splice(s["pay_ckv"], s["pay_kpe"], s["ckv"], s["kpe"], s["table"],
                         case["start"], case["delta"], ROPE_BASE, case["pairing"])
        return s["pay_ckv"], s["pay_kpe"], s["ckv"], s["kpe"]
    out, lse = state["partial"]()
    if case["kind"] != "route":
        return out, lse
    merged, merged_lse = state["merge"]()
    return out, lse, merged, merged_lse


# ---------------------------------------------------------------- bounds
def work(case):
    if case["kind"] == "fetch":
        # gather and splice: every selected token read and written by each
        return dict(bytes=4 * case["L"] * case["K"] * (DLAT + DPE) * 2, flops=0)
    R, Mq, H, NB = case["R"], case["Mq"], case["H"], case["NB"]
    jobs = R * case["hits"] if case["kind"] == "route" else R
    per_id = 1 if case["kind"] == "tokens" else BLOCK
    token_bytes = (DLAT + DPE) * (2 if case["kv"] == "bf16" else 1)
    blocks_read = jobs * case["valid"]
    if case["kind"] == "rows":
        blocks_read = min(NB, case["valid"] * (Mq if case["sparse"] else 1))
    out_row = DLAT * 2 + 8 if case.get("wire") else DLAT * 4 + 4
    n_rows = jobs * Mq * H
    b = blocks_read * per_id * token_bytes + R * Mq * H * (DLAT + DPE) * 2 + n_rows * out_row
    if case["kind"] == "route":
        b += n_rows * out_row + R * Mq * H * (DLAT * 4 + 4)
    return dict(bytes=b, flops=n_rows * case["valid"] * per_id * 2 * (DLAT + DPE + DLAT))


def tolerance(case):
    if case["kind"] == "fetch":
        # the gather and the latent rows are copies; a rotated RoPE value may
        # round to the neighbouring bf16
        return dict(rel=2e-4, max=0.02)
    # the weights enter the second product in bf16, the scores' sums are in
    # 32 bits; wire-form rows are themselves rounded to bf16
    return dict(rel=8e-3, max=0.08)


# ---------------------------------------------------------------- 64-bit values
def _attend(q_lat, q_pe, k_lat, k_pe):
    """(out, max, lse) of rows [n, .] over tokens [T, .], all float64."""
    s = (q_lat @ k_lat.T + q_pe @ k_pe.T) * float(np.float32(SCALE))
    m = s.amax(dim=1)
    p = torch.exp(s - m[:, None])
    ell = p.sum(dim=1)
    return (p @ k_lat) / ell[:, None], m, ell


def exact(case, seed):
    t = _inputs(case, seed)
    if case["kind"] == "fetch":
        sel, tab = t["sel"].long(), t["src_table"].long()
        blk, off = tab[sel // BLOCK], sel % BLOCK
        pay_ckv, pay_kpe = t["src_ckv"][:, blk, off], t["src_kpe"][:, blk, off]
        i = torch.arange(DPE // 2, device="cuda", dtype=torch.float64)
        ang = case["delta"] * ROPE_BASE ** (-2.0 * i / DPE)
        c, s = torch.cos(ang), torch.sin(ang)
        v = pay_kpe.double()
        x, y = (v[..., 0::2], v[..., 1::2]) if case["pairing"] == 0 else (v[..., :32], v[..., 32:])
        nx, ny = x * c - y * s, x * s + y * c
        turned = torch.stack([nx, ny], -1).flatten(-2) if case["pairing"] == 0 else torch.cat([nx, ny], -1)
        pos = case["start"] + torch.arange(case["K"], device="cuda")
        blk, off = t["table"].long()[pos // BLOCK], pos % BLOCK
        ckv, kpe = t["ckv"].double(), t["kpe"].double()
        ckv[:, blk, off] = pay_ckv.double()
        kpe[:, blk, off] = turned
        return pay_ckv, pay_kpe, ckv, kpe
    R, Mq, H = case["R"], case["Mq"], case["H"]
    jobs = t["table"].shape[0]
    sel, table = t["sel"].cpu().numpy(), t["table"].cpu().numpy()

    def tokens_of(r, ids):
        """The job's selected tokens as float64 (latent, RoPE) rows."""
        if case["kind"] == "tokens":
            blk, off = _gpu(table[r, ids // BLOCK]).long(), _gpu(ids % BLOCK).long()
            k, kp = t["ckv"][blk, off][:, None], t["kpe"][blk, off][:, None]
        else:
            blk = _gpu(table[r, ids]).long()
            k, kp = t["ckv"][blk], t["kpe"][blk]
        if t["cs"] is not None:
            k = k.view(torch.float8_e4m3fn).to(torch.float32).double() * t["cs"][blk].double()[:, None, None]
            kp = kp.view(torch.float8_e4m3fn).to(torch.float32).double() * t["ks"][blk].double()[:, None, None]
        return k.double().reshape(-1, DLAT), kp.double().reshape(-1, DPE)

    out = torch.zeros((jobs, Mq, H, DLAT), dtype=torch.float64, device="cuda")
    m = torch.zeros((jobs, Mq, H), dtype=torch.float64, device="cuda")
    ell = torch.zeros_like(m)
    for r in range(jobs):
        ql, qp = t["q_lat"][r % R].double(), t["q_pe"][r % R].double()
        if sel.ndim == 3:
            for i in range(Mq):
                kv = tokens_of(r, sel[r, i][sel[r, i] >= 0])
                out[r, i], m[r, i], ell[r, i] = _attend(ql[i], qp[i], *kv)
        else:
            kv = tokens_of(r, sel[r][sel[r] >= 0])
            o, mm, ee = _attend(ql.reshape(-1, DLAT), qp.reshape(-1, DPE), *kv)
            out[r], m[r], ell[r] = o.view(Mq, H, DLAT), mm.view(Mq, H), ee.view(Mq, H)
    lse = m + torch.log(ell)
    stat = torch.stack([m, ell], -1) if case.get("wire") else lse
    if case["kind"] != "route":
        return out, stat
    parts = lse.view(case["hits"], R, Mq, H)
    merged_lse = torch.logsumexp(parts, 0)
    w = torch.exp(parts - merged_lse[None])
    merged = (w[..., None] * out.view(case["hits"], R, Mq, H, DLAT)).sum(0)
    return out, stat, merged, merged_lse
