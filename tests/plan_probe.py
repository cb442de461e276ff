"""The library's plans on the CPU: csrc/mla_plan.h compiled here with g++ into
a small program that reads calls and prints their plans."""
import os
import random
import subprocess
from dataclasses import dataclass

from paper_2606_01502_amd import build as B

CUS = 256
SCRATCH = 64 << 20

_MAIN = r"""
#include "mla_plan.h"
#include <cstdio>
static void show(const mla::Planner& p, const mla::Plan& q) {
  std::printf(" %d %lld %lld %lld %d %.17g %d %llu %d %lld", q.row_groups, (long long)q.row_tiles,
              (long long)q.S, (long long)q.sps, (int)q.by_id, q.us, (int)p.ws_half(q.S),
              (unsigned long long)(q.S > 1 ? p.ws_size(q.S) : 0),
              (int)q.long_lists, (long long)p.tile_qrows);
}
int main() {
  long long R, Mq, H, NB, K, tok, pr, fp8, ns, rt, rg, S;
  while (std::scanf("%lld %lld %lld %lld %lld %lld %lld %lld %lld %lld %lld %lld", &R, &Mq, &H, &NB,
                    &K, &tok, &pr, &fp8, &ns, &rt, &rg, &S) == 12) {
    const mla::Planner p({R, Mq, H, NB, K, tok != 0, pr != 0, fp8 != 0, (int)ns, (int)rt, 256});
    if (p.refused) { std::printf("refused\n"); continue; }
    show(p, p.choose());
    show(p, p.cover);
    // the plan of S splits and rg row groups beside it
    if (rg) show(p, p.plan_of((int)rg, S));
    std::printf("\n");
  }
}
"""


@dataclass
class Call:
    R: int
    Mq: int
    H: int
    NB: int
    K: int
    tokens: bool = False
    per_row: bool = False
    fp8: bool = False
    n_splits: int = 0
    row_tile: int = 0

    @property
    def rows(self):
        return self.Mq * self.H


@dataclass
class Plan:
    row_groups: int
    row_tiles: int
    S: int
    sps: int
    by_id: bool
    us: float
    half: bool
    ws: int
    long_lists: bool
    tile_qrows: int


def build(tmp):
    src, exe = os.path.join(tmp, "plan.cc"), os.path.join(tmp, "plan")
    with open(src, "w") as f:
        f.write(_MAIN)
    rocm = os.path.dirname(os.path.dirname(B.HIPCC))
    subprocess.run(["g++", "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I",
                    os.path.join(rocm, "include"), "-I", B.CSRC, "-o", exe, src], check=True)
    return exe


def _parse(v):
    return Plan(int(v[0]), int(v[1]), int(v[2]), int(v[3]), v[4] == "1", float(v[5]), v[6] == "1", int(v[7]),
                v[8] == "1", int(v[9]))


def plans(exe, calls, beside=None):
    """[(plan, the covering plan, the plan of beside[i] = (row groups, splits) or
    None)], None where refused."""
    lines = []
    for i, c in enumerate(calls):
        rg, S = beside[i][:2] if beside and beside[i] else (0, 0)
        lines.append(f"{c.R} {c.Mq} {c.H} {c.NB} {c.K} {int(c.tokens)} {int(c.per_row)} {int(c.fp8)} "
                     f"{c.n_splits} {c.row_tile} {rg} {S}")
    out = subprocess.run([exe], input="\n".join(lines) + "\n", check=True, capture_output=True, text=True)
    rows = out.stdout.splitlines()
    assert len(rows) == len(calls)
    res = []
    for ln in rows:
        v = ln.split()
        res.append(None if v[0] == "refused" else (_parse(v[:10]), _parse(v[10:20]), _parse(v[20:]) if len(v) > 20 else None))
    return res


def cover_rule(c):
    """(row groups, splits, whether splits go by logical block) by coverage: 128-row tiles where a job has more
    than 64 rows and the splits hold 8 blocks and more, and the smallest number
    of splits of at least two blocks that gives every compute unit a workgroup."""
    Kb = (c.K + 63) // 64 if c.tokens else c.K
    rg = 2 if c.rows > 64 else 1

    def tiles(g):
        return (c.rows + 64 * g - 1) // (64 * g)

    if c.row_tile:
        rg = c.row_tile // 64
    elif rg == 2:
        units = c.R * tiles(2)
        if Kb < 8 * min((CUS + units - 1) // units, max(Kb // 2, 1)):
            rg = 1

    def span(g):
        w = 64 * g
        return max((min(r0 + w, c.rows) - 1) // c.H - r0 // c.H + 1 for r0 in range(0, c.rows, w))

    tq = 1
    if c.per_row:
        if rg == 2 and span(2) > 64:
            rg = 1
        tq = span(rg)
    units = c.R * tiles(rg)
    S = max(1, (CUS + units - 1) // units)
    cap = 512 if c.per_row and c.fp8 else 1024
    if c.per_row and tq > 1 and c.K * tq <= cap:
        return rg, min(S, max(min(c.NB, c.K * tq) // 2, 1)), True
    S = min(S, max(Kb // 2, 1))
    if S == 2 and Kb <= 5:
        S = 1
    if c.tokens:
        S = max(S, (c.K + 1023) // 1024)
        sps = min(max(64, -(-c.K // S) + 63 & ~63), 1024)
    else:
        S = max(S, (c.K * tq + cap - 1) // cap)
        sps = max(1, (c.K + S - 1) // S)
        if c.per_row:
            sps = min(sps, max(1, cap // tq))
    return rg, max(1, (c.K + sps - 1) // sps), False


def draw(rng, kinds=("blocks", "tokens", "per_row")):
    def log(lo, hi):
        return int(round(2 ** rng.uniform(lo, hi)))
    kind = rng.choice(kinds)
    fp8 = rng.random() < 0.4
    H = rng.choice([1, 3, 8, 16, 24, 40, 64, 65, 128, 200])
    if kind == "per_row":
        Mq, K = log(0, 9), log(0, 9)
        NB = min(K * rng.choice([1, 2, 4]) + rng.randint(0, 9), 73696 // min(64, 128 // H + 2))
        return Call(log(0, 10), Mq, H, max(NB, 1), K, per_row=True, fp8=fp8)
    K = log(0, 12) if kind == "tokens" else log(0, 11)
    return Call(log(0, 12), log(0, 2), H, K, K, tokens=kind == "tokens", fp8=fp8)
