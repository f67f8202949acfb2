"""Workloads of the framework, through its public entry points.

Each case is a dict of plain values. The kinds:

  search  `roots` breadth-first searches, one after another, on one resident
          graph: levels, (select, max) parents and, with `stats`, the message
          statistics of every level. `memory` "library" uses csbfs.Engine,
          "caller" csbfs.WorkspaceSearch on the caller's tensors.
  batch   one batched search of `roots` roots (csbfs.BatchEngine).
  serve   a burst of `queries` queries, spread evenly over a pool of graphs,
          submitted to a running csbfs.Server and awaited.
  build   tuple list to partitioned graph (csbfs.Graph), read back block by
          block.
  encode  sieve + WAH-64 compression of one frontier bitmap.
  decode  the same stream back into a bitmap.

Graphs are synthetic: "rmat" (n = 2^scale, edgefactor 16, initiator 0.57 /
0.19 / 0.19 / 0.05, ids permuted) or "er" (independent uniform endpoints).
They are drawn on the GPU from the seed alone, because a scale-26 tuple list
takes minutes of host time otherwise.
"""
import math

import numpy as np
import torch

from paper_1208_5542_amd import csbfs

RMAT_A, RMAT_B, RMAT_C = 0.57, 0.19, 0.19
CHUNK = 1 << 25  # tuples (or bits) drawn at a time
STAT_KEYS = ("frontier", "edges", "view_bits", "sieved_bits", "unsieved_bits", "raw_bytes", "wah_unsieved_bytes",
             "wah_sieved_bytes", "self_bytes", "max_rank_bytes", "pulled", "direction")
STAT_LEVELS = 48  # level statistics returned per search, zero past its depth


# ------------------------------------------------------------------ cases --

def _search(name, graph, n, tuples, p, roots=1, stats=False, memory="library", sieve=True):
    return {"name": name, "kind": "search", "graph": graph, "n": n, "tuples": tuples, "p": p, "roots": roots,
            "stats": stats, "memory": memory, "sieve": sieve}


def listed():
    return [
        # the smallest search a program makes: a graph of a thousand vertices
        # on one partition, with its level statistics; all latency
        _search("search_rmat10_p1", "rmat", 1 << 10, 16 << 10, 1, stats=True),
        # a lone query on a small resident graph (the smallest of the serving pool)
        _search("search_rmat16_p4", "rmat", 1 << 16, 16 << 16, 4),
        # flat degrees and more levels: the serving pool's uniform graph
        _search("search_er20_p4", "er", 1 << 20, 8 << 20, 4),
        # a vertex count that is no power of two, three processors, the
        # caller's own memory, messages without the sieve (Alg. 2)
        _search("search_er_ragged_p3", "er", 3 * 64 * 2049, 3 * 64 * 2049 * 16 + 77, 3, stats=True,
                memory="caller", sieve=False),
        # the 4 x 4 grid workload
        _search("search_rmat22_p4", "rmat", 1 << 22, 16 << 22, 4, roots=4),
        # the headline workload: scale 26 on the 8 x 8 grid
        _search("search_rmat26_p8", "rmat", 1 << 26, 16 << 26, 8, roots=4),
        # a small group of queries answered together
        {"name": "batch_rmat18_p4_b8", "kind": "batch", "graph": "rmat", "n": 1 << 18, "tuples": 16 << 18, "p": 4,
         "roots": 8, "stats": True},
        # the batched workload: 64 roots at scale 24
        {"name": "batch_rmat24_p4_b64", "kind": "batch", "graph": "rmat", "n": 1 << 24, "tuples": 16 << 24, "p": 4,
         "roots": 64, "stats": False},
        # a burst of queries over small resident graphs
        {"name": "serve_burst", "kind": "serve", "graph": "rmat", "scales": "16,18,20", "p": 4, "queries": 96,
         "slots": 4},
        # a new graph of a million vertices: tuples to the partitioned grid
        {"name": "build_rmat20_p4", "kind": "build", "graph": "rmat", "n": 1 << 20, "tuples": 16 << 20, "p": 4},
        # one message of the scale-26 grid (2^23 bits) in a sparse level
        {"name": "encode_2p23", "kind": "encode", "nbits": 1 << 23, "density": 0.004, "mask": 0.7},
        # a whole ragged frontier of a large graph coming back from a wide level
        {"name": "decode_2p28", "kind": "decode", "nbits": (1 << 28) + 77, "density": 0.06, "mask": 0.9},
    ]


def draw(rng):
    def logint(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(("search",) * 5 + ("batch", "batch", "serve", "build", "encode", "decode"))
    if kind in ("search", "batch", "build"):
        if rng.random() < 0.6:
            top = {"search": 24, "batch": 21, "build": 21}[kind]
            scale = rng.randint(10, top)
            n, p, graph = 1 << scale, rng.choice((1, 2, 4, 4 if kind == "build" else 8)), "rmat"
            tuples = 16 * n
        else:
            p, graph = rng.randint(1, 5 if kind == "build" else 8), "er"
            n = 64 * p * logint(16, (1 << 21) // (64 * p))
            tuples = int(n * rng.uniform(4, 20)) + rng.randint(0, 99)
        if kind == "search":
            return {"kind": kind, "graph": graph, "n": n, "tuples": tuples, "p": p, "roots": rng.randint(1, 4),
                    "stats": rng.random() < 0.5, "memory": rng.choice(("library", "caller")),
                    "sieve": rng.random() < 0.8}
        if kind == "batch":
            return {"kind": kind, "graph": graph, "n": n, "tuples": tuples, "p": p, "roots": logint(2, 64),
                    "stats": rng.random() < 0.5}
        return {"kind": kind, "graph": graph, "n": n, "tuples": tuples, "p": p}
    if kind == "serve":
        scales = sorted(rng.sample(range(12, 21), rng.randint(1, 3)))
        return {"kind": kind, "graph": "rmat", "scales": ",".join(map(str, scales)), "p": rng.choice((1, 2, 4)),
                "queries": logint(4, 160), "slots": rng.choice((1, 2, 4))}
    return {"kind": kind, "nbits": logint(1 << 12, 1 << 28), "density": round(math.exp(rng.uniform(-10, -0.7)), 6),
            "mask": rng.choice((0.0, 0.3, 0.7, 0.95))}


# ----------------------------------------------------------------- inputs --

def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _tuples(graph, n, m, g):
    """(src, dst, touched): the tuple list and the vertices with a tuple that is no self-loop."""
    src = torch.empty(m, dtype=torch.int64, device="cuda")
    dst = torch.empty(m, dtype=torch.int64, device="cuda")
    touched = torch.zeros(n, dtype=torch.bool, device="cuda")
    perm = torch.randperm(n, generator=g, device="cuda") if graph == "rmat" else None
    scale = n.bit_length() - 1
    for a in range(0, m, CHUNK):
        k = min(CHUNK, m - a)
        if graph == "rmat":
            u = torch.zeros(k, dtype=torch.int32, device="cuda")
            v = torch.zeros(k, dtype=torch.int32, device="cuda")
            for _ in range(scale):
                r = torch.rand(k, generator=g, device="cuda")
                low = r >= RMAT_A + RMAT_B
                right = torch.where(low, r >= RMAT_A + RMAT_B + RMAT_C, r >= RMAT_A)
                u.mul_(2).add_(low)
                v.mul_(2).add_(right)
            src[a:a + k] = perm[u]
            dst[a:a + k] = perm[v]
        else:
            src[a:a + k] = torch.randint(n, (k,), generator=g, device="cuda")
            dst[a:a + k] = torch.randint(n, (k,), generator=g, device="cuda")
        real = src[a:a + k] != dst[a:a + k]
        touched[src[a:a + k][real]] = True
        touched[dst[a:a + k][real]] = True
    return src, dst, touched


def _roots(touched, count, g):
    at = touched.nonzero().flatten()
    return at[torch.randint(at.numel(), (count,), generator=g, device="cuda")].tolist()


def _pack(bits):
    """Bit k of the vector is bit k % 64 of word k / 64."""
    weight = torch.ones(64, dtype=torch.int64, device="cuda") << torch.arange(64, device="cuda")
    pad = torch.nn.functional.pad(bits, (0, -bits.numel() % 64))
    return (pad.view(-1, 64).to(torch.int64) * weight).sum(dim=1)


def _bitmap(nbits, density, g):
    return torch.cat([_pack(torch.rand(min(CHUNK, nbits - a), generator=g, device="cuda") < density)
                      for a in range(0, nbits, CHUNK)])


def _piece(case, seed):
    g = _gen(seed)
    bits = _bitmap(case["nbits"], case["density"], g)
    return bits, _bitmap(case["nbits"], case["mask"], g) if case["mask"] else None


def _graph(case, seed):
    g = _gen(seed)
    src, dst, touched = _tuples(case["graph"], case["n"], case["tuples"], g)
    roots = _roots(touched, case.get("roots", 1), g)
    return csbfs.Graph(src, dst, case["n"], case["p"]), roots


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("encode", "decode"):
        nbits = case["nbits"]
        bits, mask = _piece(case, seed)
        ws = csbfs.wah_workspace(nbits)
        state = {"kind": kind, "nbits": nbits, "ws": ws, "bits": bits, "mask": mask}
        if kind == "decode":
            state["words"] = csbfs.wah_encode(bits, nbits, mask=mask, workspace=ws).clone()
        else:
            state["words"] = torch.zeros(csbfs.wah_capacity(nbits), dtype=torch.int64, device="cuda")
            state["count"] = torch.zeros(1, dtype=torch.int64, device="cuda")
        return state
    if kind == "build":
        src, dst, _ = _tuples(case["graph"], case["n"], case["tuples"], _gen(seed))
        return {"kind": kind, "src": src, "dst": dst, "n": case["n"], "p": case["p"]}
    if kind == "serve":
        server = csbfs.Server(slots=case["slots"], max_batch=64, max_levels=256, hbm_budget=32 << 30)
        scales = [int(s) for s in case["scales"].split(",")]
        state = {"kind": kind, "server": server, "graphs": [], "ids": [], "roots": [], "out": []}
        per = -(-case["queries"] // len(scales))
        for k, scale in enumerate(scales):
            gc = {"graph": case["graph"], "n": 1 << scale, "tuples": 16 << scale, "p": case["p"], "roots": per}
            graph, roots = _graph(gc, seed * 64 + k)
            state["graphs"].append(graph)
            state["ids"].append(server.add_graph(graph))
            state["roots"].append(roots)
            state["out"].append(torch.empty((per, 1 << scale), dtype=torch.int32, device="cuda"))
        return state
    graph, roots = _graph(case, seed)
    n, k = case["n"], case["roots"]
    state = {"kind": kind, "graph": graph, "roots": roots, "stats": case["stats"],
             "level": torch.empty((k, n), dtype=torch.int32, device="cuda")}
    if kind == "batch":
        state["engine"] = csbfs.BatchEngine(graph, max_roots=k, max_levels=256)
        return state
    flags = 0 if case["sieve"] else csbfs.FLAG_NO_SIEVE
    state["parent"] = torch.empty((k, n), dtype=torch.int32, device="cuda")
    if case["memory"] == "caller":
        state["engine"] = csbfs.WorkspaceSearch(graph, csbfs.search_config(flags=flags, max_levels=256))
    else:
        state["engine"] = csbfs.Engine(graph, max_levels=256, flags=flags)
    return state


# ------------------------------------------------------------------- runs --

def _counts(stats):
    out = np.zeros((STAT_LEVELS, len(STAT_KEYS)), dtype=np.int64)
    rows = [[s[k] for k in STAT_KEYS] for s in stats[:STAT_LEVELS]]
    out[:len(rows)] = rows
    return out


def run(state):
    kind = state["kind"]
    if kind == "encode":
        # through the C ABI, as a sender that keeps the stream and its length on the device
        bits, mask, words, count, ws = (state[k] for k in ("bits", "mask", "words", "count", "ws"))
        rc = csbfs.lib().csbfs_wah_encode(bits.data_ptr(), None if mask is None else mask.data_ptr(), state["nbits"],
                                          words.data_ptr(), words.numel(), count.data_ptr(), ws.data_ptr(),
                                          ws.numel(), torch.cuda.current_stream().cuda_stream)
        assert rc == csbfs.OK, csbfs.strerror(rc)
        return {"words": words, "count": count}
    if kind == "decode":
        bits, status = csbfs.wah_decode_or(state["words"], state["nbits"], workspace=state["ws"])
        return {"bits": bits, "status": status}
    if kind == "build":
        g = csbfs.Graph(state["src"], state["dst"], state["n"], state["p"])
        blocks = [g.block(i, j) for i in range(g.p) for j in range(g.p)]
        out = {"directory": g.directory(), "rows": torch.stack([b[0] for b in blocks]),
               "columns": torch.cat([b[1] for b in blocks])}
        torch.cuda.current_stream().synchronize()  # the graph is freed below
        g.close()
        return out
    if kind == "serve":
        server, rids = state["server"], []
        for k in range(state["out"][0].shape[0]):  # graphs in turn, as mixed arrivals
            for gid, roots, out in zip(state["ids"], state["roots"], state["out"]):
                rids.append(server.submit(gid, roots[k], out[k]))
        infos = [server.wait(r) for r in rids]
        return {"level": state["out"], "status": max(-i["status"] for i in infos),
                "n_levels": [max(i["n_levels"] for i in infos)]}
    if kind == "batch":
        r = state["engine"].bfs(state["roots"], state["level"], with_stats=state["stats"])
        out = {"level": r.level, "n_levels": r.n_levels}
        if state["stats"]:
            out["stats"] = _counts(r.stats)
        return out
    out = {"level": state["level"], "parent": state["parent"], "n_levels": [], "stats": []}
    for k, root in enumerate(state["roots"]):
        r = state["engine"].bfs(root, state["level"][k], state["parent"][k], with_stats=state["stats"])
        out["n_levels"].append(r.n_levels)
        if state["stats"]:
            out["stats"].append(_counts(r.stats))
    return out


def work(case):
    """One pass: inputs read once, outputs written once. A search has to look
    at one adjacency id of every vertex and to write its results."""
    kind = case["kind"]
    if kind in ("encode", "decode"):
        d = case["density"] * (case["mask"] or 1.0)
        groups = case["nbits"] / 63
        literal = 1 - (1 - d) ** 63
        stream = 8 * groups * min(1.0, 2 * literal)  # a literal, and a fill before most of them
        plain = case["nbits"] / 8 * (2 if kind == "encode" and case["mask"] else 1)
        return {"bytes": plain + stream, "flops": 0}
    if kind == "serve":
        scales = [int(s) for s in case["scales"].split(",")]
        per = -(-case["queries"] // len(scales))
        return {"bytes": sum(per * 8 * (1 << s) for s in scales), "flops": 0}
    n, m, p = case["n"], case["tuples"], case["p"]
    if kind == "build":
        return {"bytes": 16 * m + 8 * m + 4 * p * n + p * n / 8, "flops": 0}
    if kind == "batch":
        return {"bytes": 4 * n + 4 * n * case["roots"], "flops": 0}
    return {"bytes": case["roots"] * (4 * n + 8 * n + p * n / 8), "flops": 0}


# ------------------------------------------------- the same without csbfs --

def _plain_search(src, dst, n, root, parents):
    level = torch.full((n,), -1, dtype=torch.int32, device="cuda")
    parent = torch.full((n,), -1, dtype=torch.int64, device="cuda")
    level[root], parent[root], depth = 0, root, 0
    s, d = torch.cat([src, dst]), torch.cat([dst, src])
    while True:
        hit = (level[s] == depth) & (level[d] < 0)
        if not bool(hit.any()):
            return level, parent.to(torch.int32) if parents else None, depth + 1
        if parents:
            parent.scatter_reduce_(0, d[hit], s[hit], "amax")
        depth += 1
        level[d[hit]] = depth


def _plain_encode(bits, nbits):
    """WAH-64: literal, fill and active words of a 0/1 array."""
    groups, rest = nbits // 63, nbits % 63
    value = np.zeros(groups, dtype=np.uint64)
    body = bits[: groups * 63].reshape(groups, 63).astype(np.uint64)
    for t in range(63):
        value |= body[:, t] << np.uint64(62 - t)
    cls = np.where(value == 0, 0, np.where(value == np.uint64((1 << 63) - 1), 1, 2))
    start = np.ones(groups, dtype=bool)
    start[1:] = (cls[1:] == 2) | (cls[1:] != cls[:-1])
    at = np.flatnonzero(start)
    run = np.diff(np.append(at, groups)).astype(np.uint64)
    fill = np.uint64(1 << 63) | (cls[at].astype(np.uint64) << np.uint64(62)) | run
    words = np.where(cls[at] == 2, value[at], fill)
    if rest:
        active = 0
        for b in bits[groups * 63:]:
            active = active * 2 + int(b)
        words = np.append(words, np.uint64(active))
    return words.view(np.int64)


def exact(case, seed):
    kind = case["kind"]
    if kind in ("encode", "decode"):
        nbits = case["nbits"]
        bits, mask = _piece(case, seed)
        bits = bits if mask is None else bits & mask
        if kind == "decode":
            return {"bits": bits, "status": 0}
        if nbits > 1 << 24:
            return None
        flat = np.unpackbits(bits.cpu().numpy().view(np.uint8), bitorder="little")[:nbits]
        words = _plain_encode(flat, nbits)
        out = np.zeros(nbits // 63 + 1, dtype=np.int64)
        out[:words.size] = words
        return {"words": torch.from_numpy(out), "count": torch.tensor([words.size])}
    if kind not in ("search", "batch") or case["n"] > 1 << 20 or case["n"] * case["roots"] > 1 << 22:
        return None
    g = _gen(seed)
    src, dst, touched = _tuples(case["graph"], case["n"], case["tuples"], g)
    found = [_plain_search(src, dst, case["n"], r, kind == "search") for r in _roots(touched, case["roots"], g)]
    level = torch.stack([f[0] for f in found])
    if kind == "batch":
        return {"level": level, "n_levels": max(f[2] for f in found), "stats": None}
    return {"level": level, "parent": torch.stack([f[1] for f in found]), "n_levels": [f[2] for f in found],
            "stats": None}
