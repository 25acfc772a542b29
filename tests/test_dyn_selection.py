"""Frontier and selection kernels of the dynamic tree, their source compiled for the CPU (kernel_on_cpu.h): between two barriers
the threads may run in any order, and every index stays in its array, whatever the scores are.  Oracle: sorting."""
import math
import os
import random
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
MAX_CAND, MAX_FRONT, MAX_DEPTH, MAX_NODES = 256, 64, 8, 128

MAIN = r"""
int main() {
  int n_cases;
  if (scanf("%d", &n_cases) != 1) return 2;
  for (int q = 0; q < n_cases; ++q) {
    DynTree t;
    int R, seed, j, m[2] = {1, 0};
    if (scanf("%d %d %d %d %d %d %d", &t.C, &t.D, &t.topk, &t.N, &R, &seed, &j) != 7) return 2;
    for (int i = 0; i < t.D + 2; ++i) if (scanf("%d", &t.off[i]) != 1) return 2;
    for (int i = 0; i < t.D + 1; ++i) if (scanf("%d", &t.F[i]) != 1) return 2;
    std::vector<int> tok(2 * t.C), par(2 * t.C), front(2 * CLOVER_MAX_DEPTH * DYN_MAX_FRONT, -5), tab(6 * 2 * R, -5), iv(4 * R, -5), out(2 * R, -5);
    std::vector<float> score(2 * t.C, 0.f);
    std::vector<unsigned long long> anc(4 * R, 5);
    for (int i = 0; i < t.C; ++i) { tok[i] = 1000 + i; char b[64]; if (scanf("%d %63s", &par[i], b) != 2) return 2; score[i] = strtof(b, nullptr); }
    t.cand_tok = {"cand_tok", tok.data(), (long)tok.size()}; t.cand_par = {"cand_par", par.data(), (long)par.size()};
    t.cand_score = {"cand_score", score.data(), (long)score.size()}; t.frontier = {"frontier", front.data(), (long)front.size()};
    Global<int>* tabs[6] = {&t.t_parent, &t.t_rank, &t.t_depth, &t.t_first_child, &t.t_n_child, &t.t_keep};
    for (int i = 0; i < 6; ++i) *tabs[i] = {"table", tab.data() + i * 2 * R, R};      // (sequence 0's rows: what lies behind is another's)
    t.t_anc = {"t_anc", anc.data(), 2 * R}; t.t_iv = {"t_iv", iv.data(), 2 * R};
    const Global<int> mm{"m", m, 2}, tokens{"tree_tokens", out.data(), R};
    if (j > 0) {
      launch(2, 256, seed, [&] { dyn_frontier_kernel(t, j, mm); });
      for (int i = 0; i < t.F[j]; ++i) printf("%d ", front[j * DYN_MAX_FRONT + i]);
    } else {
      launch(2, DYN_MAX_CAND, seed, [&] { dyn_finalize_kernel(t, R, mm, tokens); });
      for (int u = 0; u < t.N; ++u) {
        printf("%d ", out[u]);
        for (int i = 0; i < 6; ++i) printf("%d ", tab[i * 2 * R + u]);
        printf("%llu %llu %d %d ", anc[2 * u], anc[2 * u + 1], iv[2 * u], iv[2 * u + 1]);
      }
    }
    printf("\n");
  }
}
"""


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    src = open(os.path.join(ROOT, "paper_2408_00264_amd", "csrc", "kernels_dyn.hip")).read()
    head = open(os.path.join(ROOT, "paper_2408_00264_amd", "csrc", "clover_internal.h")).read()
    kernels = [re.search(r"^__global__ [^\n]*void %s\(.*?^}" % name, src, re.S | re.M)[0] for name in ("dyn_frontier_kernel", "dyn_finalize_kernel")]
    text = re.search(r"^struct DynTree \{.*?^\};", head, re.S | re.M)[0] + "\n" + re.search(r"^__device__ [^\n]*rank_score.*", src, re.M)[0] + "\n" + "\n".join(kernels)

    def shared(d):                                      # __shared__ T a[N], b[N][M], c;
        names = [re.fullmatch(r"\s*(\w+)((?:\[[^\]]+\])*)\s*", part) for part in d[2].split(",")]
        return " ".join("static Shared<%s, %s> %s{\"%s\"};" % (d[1], ", ".join(re.findall(r"\[([^\]]+)\]", n[2])) or "1", n[1], n[1]) for n in names)
    text = re.sub(r"__shared__ ((?:unsigned long long)|\w+) ([^;]*);", shared, text)
    text = re.sub(r"\b(?:const )?((?:unsigned long long)|int|float)\s*\*\s*(?:__restrict__ )?(\w+)((?:, \*\w+)*)", lambda d: "Global<%s> %s%s" % (d[1], d[2], d[3].replace("*", "")), text)
    consts = "".join(f"constexpr int {n} = {v};\n" for n, v in (("DYN_MAX_CAND", MAX_CAND), ("DYN_MAX_FRONT", MAX_FRONT), ("CLOVER_MAX_DEPTH", MAX_DEPTH), ("CLOVER_MAX_NODES", MAX_NODES)))
    d = tmp_path_factory.mktemp("dyn")
    (d / "k.cpp").write_text('#include "kernel_on_cpu.h"\n#include <unistd.h>\n' + consts + text + MAIN)
    subprocess.run(["g++", "-std=c++17", "-O1", "-w", "-include", "unistd.h", "-I", os.path.join(ROOT, "tests"), str(d / "k.cpp"), "-o", str(d / "k")], check=True)

    def go(cases):
        r = subprocess.run([str(d / "k")], input=f"{len(cases)}\n" + "\n".join(cases), capture_output=True, text=True, timeout=100)
        assert r.returncode == 0, r.stdout[-300:]
        return [list(map(int, line.split())) for line in r.stdout.splitlines()]
    return go


def _tree(rng, topk, frontier, D, score):
    """candidates' parents and scores as the ranking kernels leave them; score(parent's) draws a child's"""
    off, F, par, sc = [0, 1], [1], [0], [0.0]
    front = [0]
    for j in range(1, D + 1):
        for p in front:
            kids = sorted((score(sc[p]) for _ in range(topk)), key=lambda v: math.inf if v != v else v, reverse=True)
            par += [p] * topk
            sc += kids
        off.append(len(par))
        F.append(min(frontier, off[j + 1] - off[j]))
        front = sorted(range(off[j], off[j + 1]), key=lambda c: (-_order(sc[c]), c))[:F[j]]
    return off, F, par, sc


def _order(v):
    return -math.inf if v != v else v                   # a score that is no number comes last


def _line(off, F, par, sc, topk, D, N, R, seed, j):
    f = lambda v: "nan" if v != v else repr(float(v))
    return " ".join(map(str, [len(par), D, topk, N, R, seed, j] + off + F)) + "\n" + "\n".join(f"{p} {f(s)}" for p, s in zip(par, sc))


def _expected(off, par, sc, topk, D, N):
    C = len(par)
    keep = sorted(sorted(range(C), key=lambda c: (-math.inf if c == 0 else -_order(sc[c]), c))[:N])
    depth = lambda c: sum(c >= off[j] for j in range(1, D + 1))
    rank = lambda c: 0 if c == 0 else (c - off[depth(c)]) % topk
    nid = {0: 0}
    for j in range(1, D + 1):
        for c in sorted((c for c in keep if depth(c) == j), key=lambda c: (nid[par[c]], rank(c))):
            nid[c] = len(nid)
    order = sorted(nid, key=nid.get)
    parent = [-1] + [nid[par[c]] for c in order[1:]]
    anc, size = [], [1] * N
    for u in range(N):
        anc.append((anc[parent[u]] if u else 0) | 1 << u)
    for u in range(N - 1, 0, -1):
        size[parent[u]] += size[u]
    ent = [0] * N
    for u in range(N):
        e = ent[u] + 1
        for v in range(N):
            if parent[v] == u:
                ent[v], e = e, e + size[v]
    out = []
    for u, c in enumerate(order):
        kids = [v for v in range(N) if parent[v] == u]
        out += [1000 + c, parent[u], rank(c), depth(c), kids[0] if kids else 0, len(kids), c, anc[u] & (1 << 64) - 1, anc[u] >> 64, ent[u], ent[u] + size[u] - 1]
    return out


# (children per expansion, expansions per depth, depths, nodes)
SHAPES = [(4, 3, 3, 16), (16, 1, 8, 100), (8, 8, 4, 64), (1, 1, 1, 2), (16, 16, 1, 1), (2, 64, 7, 128), (10, 6, 5, 128)]
SCORES = {"spread": lambda rng: lambda p: p - rng.random() * 4,
          "ties": lambda rng: lambda p: p - rng.randrange(2),
          "minus infinity": lambda rng: lambda p: p - rng.choice([1.0, math.inf]),
          "some no number": lambda rng: lambda p: rng.choice([p - rng.random(), math.nan]),
          "no number": lambda rng: lambda p: math.nan}


@pytest.mark.parametrize("kind", SCORES)
def test_selection(run, kind):
    rng = random.Random(kind)
    lines, want = [], []
    for topk, frontier, D, N in SHAPES:
        off, F, par, sc = _tree(rng, topk, frontier, D, SCORES[kind](rng))
        if len(par) > MAX_CAND or N > len(par):
            continue
        for seed in range(6):                           # orders of the threads
            lines.append(_line(off, F, par, sc, topk, D, N, N, seed, 0))
            want.append(_expected(off, par, sc, topk, D, N))
            for j in range(1, D):
                lines.append(_line(off, F, par, sc, topk, D, N, N, seed, j))
                want.append(sorted(range(off[j], off[j + 1]), key=lambda c: (-_order(sc[c]), c))[:F[j]])
    assert len(lines) > 40
    for line, got, w in zip(lines, run(lines), want):
        assert got == w, line.split("\n")[0]
