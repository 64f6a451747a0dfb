"""The work that a user of this library has it do, as cases that can be timed and compared.

Five kinds of work, all through the public binding:

* ``search``: plaid_search on a resident index -- one query per call (interactive use, where a query's latency is what
  counts) up to whole batches (offline evaluation, re-ranking jobs), on collections from ten thousand passages to the
  8.8 million of the largest configuration, with the search hyperparameters of Table 2 of the paper (k = 10, 100, 1000),
  1- and 2-bit residuals, both noise readings of the synthetic generator, and optionally with reconstructed vectors scaled
  to unit length;
* ``static``: the same through plaid_search_static, which a serving loop with buffers of its own uses;
* ``vanilla``: plaid_search_vanilla, the retrieval that PLAID is compared with;
* ``decode``: plaid_decompress_passages, the stored passages back as vectors and bucket indices (re-ranking elsewhere);
* ``build``: the construction of an index from embeddings: nearest centroids, residual encoding, inverted lists.

Collections are drawn like the repository's benchmark workloads: unit-norm random centroids, Zipf(1.1) centroid popularity,
embeddings around their centroid ("literal": noise of sigma per coordinate, "calibrated": a noise vector of that norm, which
gives the scores of Section 3.4 of the paper), queries around random stored embeddings.
"""
import math

import numpy as np
import torch

import paper_2205_09707_amd as pl

DIM, QLEN = 128, 32
ZIPF = 1.1
SIGMA_D, SIGMA_Q = 0.15, 0.2
CHUNK = 1 << 22  # embeddings generated at a time


def _search(name, C, P, lo, hi, nbits, nq, nprobe, t_cs, ndocs, k, noise="calibrated", renormalize=False, kind="search"):
    return {"name": name, "kind": kind, "C": C, "P": P, "lo": lo, "hi": hi, "nbits": nbits, "nq": nq, "nprobe": nprobe,
            "t_cs": t_cs, "ndocs": ndocs, "k": k, "noise": noise, "renormalize": renormalize}


def listed():
    return [
        # a question typed into a search box over a small site: ten results, nothing to amortise a launch over
        _search("one_small", 1024, 10_000, 20, 60, 2, 1, 1, 0.5, 256, 10),
        # a serving loop with its own buffers over a departmental collection, one query at a time
        _search("one_serving", 16_384, 200_000, 30, 90, 2, 1, 1, 0.5, 256, 10, kind="static"),
        # one query, a hundred results (the first stage of a reader or a re-ranker)
        _search("one_mid", 65_536, 400_000, 30, 100, 2, 1, 2, 0.45, 1024, 100),
        # one query against a web-scale collection stored with one bit per dimension
        _search("one_large", 262_144, 8_800_000, 8, 128, 1, 1, 4, 0.4, 4096, 100),
        # requests collected for a few milliseconds: an uneven batch on a collection of uneven size, unit-length scoring
        _search("few_uneven", 10_007, 123_457, 8, 180, 1, 23, 2, 0.45, 1000, 77, renormalize=True),
        # an evaluation set against a small collection, ten results
        _search("batch_small", 16_384, 200_000, 30, 90, 2, 256, 1, 0.5, 256, 10),
        # an evaluation set against a mid-sized collection, a hundred results
        _search("batch_mid", 65_536, 400_000, 30, 100, 2, 512, 2, 0.45, 1024, 100),
        # the same where hardly a centroid reaches the pruning threshold (far-off queries)
        _search("batch_mid_literal", 65_536, 400_000, 30, 100, 2, 512, 2, 0.45, 1024, 100, noise="literal"),
        # an evaluation set against the largest collection, a thousand results
        _search("batch_large", 262_144, 8_800_000, 8, 128, 2, 150, 4, 0.4, 4096, 1000),
        # the baseline retrieval of the comparison, a small batch
        dict(_search("vanilla_few", 65_536, 400_000, 30, 100, 2, 16, 4, 0.0, 1 << 14, 1000), kind="vanilla"),
        # five thousand stored passages fetched back as vectors
        {"name": "decode_mid", "kind": "decode", "C": 65_536, "P": 400_000, "lo": 30, "hi": 100, "nbits": 2, "n": 5000,
         "noise": "calibrated"},
        # a shard of new documents encoded and indexed
        {"name": "build_shard", "kind": "build", "C": 32_768, "P": 9_000, "lo": 30, "hi": 100, "nbits": 2, "noise": "calibrated"},
    ]


def _log_uniform(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["search"] * 7 + ["static", "vanilla", "decode", "build"])
    top = {"search": 8_800_000, "static": 400_000, "vanilla": 400_000, "decode": 400_000, "build": 12_000}[kind]
    P = _log_uniform(rng, 10_000 if kind != "build" else 200, top)
    lo, hi = rng.choice([(20, 60), (30, 90), (30, 100), (8, 128)])
    if P < 1_000_000 and rng.random() < 0.2:
        lo, hi = 8, 180
    tokens = P * (lo + hi) / 2
    # centroids in proportion to the square root of the number of embeddings, as the configurations have it
    C = min(262_144, max(1024, int(rng.uniform(5, 14) * math.sqrt(tokens))))
    if rng.random() < 0.5:
        C = 1 << (C.bit_length() - 1)
    nbits = rng.choice([1, 2, 2])
    noise = rng.choice(["calibrated", "calibrated", "calibrated", "literal"])
    if kind == "decode":
        return {"kind": kind, "C": C, "P": P, "lo": lo, "hi": hi, "nbits": nbits, "n": _log_uniform(rng, 1, 8000), "noise": noise}
    if kind == "build":
        return {"kind": kind, "C": C, "P": P, "lo": lo, "hi": hi, "nbits": nbits, "noise": noise}
    k, nprobe, t_cs, ndocs = rng.choice([(10, 1, 0.5, 256), (100, 2, 0.45, 1024), (1000, 4, 0.4, 4096)])
    if rng.random() < 0.5:  # a user's own values around those of the table
        ndocs = rng.randint(3 * ndocs // 4, ndocs)
        k = rng.randint(max(1, k // 3), min(k, ndocs // 4))
    if kind == "vanilla":
        nq, t_cs, ndocs = _log_uniform(rng, 1, 16), 0.0, _log_uniform(rng, 1 << 10, 1 << 14)
    else:
        nq = 1 if kind == "static" or rng.random() < 0.35 else _log_uniform(rng, 2, 512)
        nq = max(1, min(nq, 150 * 8_800_000 // P))
    c = _search("", C, P, lo, hi, nbits, nq, nprobe, t_cs, ndocs, k, noise, kind != "vanilla" and rng.random() < 0.15, kind)
    del c["name"]
    return c


# ------------------------------------------------------------------------------------------------ inputs
def _popularity(C):
    p = np.arange(1, C + 1, dtype=np.float64) ** -ZIPF
    return p / p.sum()


class _Collection:
    """Centroids, passages and codes of a case; embeddings come chunk by chunk from their own random streams."""

    def __init__(self, case, seed):
        self.case, self.seed = case, seed
        self.dev = torch.device("cuda:0")
        g = self.generator(0)
        C, P = case["C"], case["P"]
        self.centroids = torch.nn.functional.normalize(torch.randn(C, DIM, generator=g, device=self.dev), dim=1).contiguous()
        # lengths: uniform, or around the middle of the range for the widest ranges (web passages); the same lengths whatever
        # the seed, in an order of its own, so that the number of embeddings is the case's
        lo, hi = case["lo"], case["hi"]
        g_len = torch.Generator(device=self.dev)
        g_len.manual_seed(P)
        if lo == 8:
            z = torch.randn(P, generator=g_len, device=self.dev) * 20 + 68
            lengths = z.round().clamp(lo, hi).long()
        else:
            lengths = torch.randint(lo, hi + 1, (P,), generator=g_len, device=self.dev)
        self.order = torch.randperm(P, generator=g, device=self.dev)  # lengths[order[p]] is passage p's
        lengths = lengths[self.order]
        self.doc_offsets = torch.zeros(P + 1, dtype=torch.int64, device=self.dev)
        self.doc_offsets[1:] = torch.cumsum(lengths, 0)
        self.N = int(self.doc_offsets[-1])
        self.cdf = torch.from_numpy(np.cumsum(_popularity(C))).to(self.dev)
        scale = 1.0 if case["noise"] == "literal" else 1 / math.sqrt(DIM)
        self.sigma_d, self.sigma_q = SIGMA_D * scale, SIGMA_Q * scale

    def generator(self, stream):
        g = torch.Generator(device=self.dev)
        g.manual_seed((self.seed * 1_000_003 + stream) & 0x7FFFFFFFFFFFFFFF)
        return g

    def chunk(self, i):
        """(first token, codes, embeddings) of chunk i."""
        n = min(CHUNK, self.N - i * CHUNK)
        g = self.generator(10 + i)
        codes = torch.searchsorted(self.cdf, torch.rand(n, generator=g, device=self.dev, dtype=torch.float64))
        codes = codes.clamp_(max=self.case["C"] - 1).int()
        x = torch.randn(n, DIM, generator=g, device=self.dev).mul_(self.sigma_d).add_(self.centroids[codes])
        return i * CHUNK, codes, torch.nn.functional.normalize(x, dim=1)

    def buckets(self):
        """Cut-offs and weights of the residual buckets: quantiles of the residuals of the first embeddings."""
        _, codes, x = self.chunk(0)
        m = min(x.shape[0], 1 << 15)
        r = (x[:m] - self.centroids[codes[:m]]).reshape(-1).sort().values
        B = 1 << self.case["nbits"]

        def at(q):
            return r[min(r.numel() - 1, int(q * r.numel()))]
        return (torch.stack([at(b / B) for b in range(1, B)]).contiguous(),
                torch.stack([at((2 * b + 1) / (2 * B)) for b in range(B)]).contiguous())


def _index(case, seed):
    """The index of a case and, for searches, its queries."""
    col = _Collection(case, seed)
    cutoffs, weights = col.buckets()
    codes = torch.empty(col.N, dtype=torch.int32, device=col.dev)
    residuals = torch.empty(col.N, 16 * case["nbits"], dtype=torch.uint8, device=col.dev)
    g = col.generator(1)
    n_src = QLEN * case.get("nq", 0)
    # (queries of collections of more than one chunk come from the embeddings of the first)
    src = torch.randint(0, min(col.N, CHUNK), (n_src,), generator=g, device=col.dev)
    sources = None
    for i in range((col.N + CHUNK - 1) // CHUNK):
        t0, c, x = col.chunk(i)
        codes[t0:t0 + c.numel()] = c
        residuals[t0:t0 + c.numel()] = pl.plaid_encode_residuals(col.centroids, x, c, cutoffs, case["nbits"])
        if i == 0:
            sources = x[src]
        del x
    ivf_offsets, ivf_pids = pl.plaid_build_ivf(codes, col.doc_offsets, case["C"])
    arrays = {"centroids": col.centroids, "doc_offsets": col.doc_offsets, "codes": codes, "residuals": residuals,
              "bucket_weights": weights, "ivf_offsets": ivf_offsets, "ivf_pids": ivf_pids}
    idx = pl.plaid_index_from_view(arrays, case["nbits"], device=0, copy=False)
    if case.get("renormalize"):
        pl.plaid_index_set_renormalize(idx, True)
    Q = None
    if n_src:
        Q = sources + torch.randn(n_src, DIM, generator=g, device=col.dev) * col.sigma_q
        Q = torch.nn.functional.normalize(Q, dim=1).reshape(case["nq"], QLEN, DIM).contiguous()
    return idx, Q, col


def prepare(case, seed):
    """What a user's program holds before the call."""
    kind = case["kind"]
    if kind == "build":
        # embeddings as an encoder delivers them, the trained centroids and bucket cut-offs
        col = _Collection(case, seed)
        x = torch.cat([col.chunk(i)[2] for i in range((col.N + CHUNK - 1) // CHUNK)])
        return {"case": case, "centroids": col.centroids, "x": x.contiguous(), "doc_offsets": col.doc_offsets,
                "cutoffs": col.buckets()[0], "N": col.N}
    idx, Q, col = _index(case, seed)
    state = {"case": case, "idx": idx, "Q": Q}
    if kind == "decode":
        # random passages, those with the first lengths of the list: as many embeddings whatever the seed
        pids = torch.argsort(col.order)[torch.arange(case["n"], device=col.dev) % case["P"]]
        lengths = col.doc_offsets[pids + 1] - col.doc_offsets[pids]
        state.update(pids=pids.int(), capacity=int(lengths.sum()))
    if kind == "static":
        state["ids"] = torch.empty((case["nq"], case["k"]), dtype=torch.int32, device=col.dev)
        state["scores"] = torch.empty((case["nq"], case["k"]), dtype=torch.float32, device=col.dev)
    return state


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "search":
        return pl.plaid_search(state["idx"], state["Q"], case["nprobe"], case["t_cs"], case["ndocs"], case["k"])
    if kind == "static":
        return pl.plaid_search_static(state["idx"], state["Q"], case["nprobe"], case["t_cs"], case["ndocs"], case["k"],
                                      state["ids"], state["scores"])
    if kind == "vanilla":
        return pl.plaid_search_vanilla(state["idx"], state["Q"], case["nprobe"], case["ndocs"], case["k"])
    if kind == "decode":
        return pl.plaid_decompress_passages(state["idx"], state["pids"], state["capacity"])
    codes = pl.plaid_assign_centroids(state["centroids"], state["x"])
    residuals = pl.plaid_encode_residuals(state["centroids"], state["x"], codes, state["cutoffs"], case["nbits"])
    offsets, pids = pl.plaid_build_ivf(codes, state["doc_offsets"], case["C"])
    # the lists go into an array with room for the longest they can be
    return codes, residuals, offsets, torch.nn.functional.pad(pids, (0, state["N"] - pids.numel()), value=-1)


# ------------------------------------------------------------------------------------------------ what a pass needs
def work(case):
    """Bytes and operations of one pass, from the distributions (expected values).

    Search: the centroids once, per query the S_cq products (2 * 128 * 32 * C operations), the inverted lists of the
    centroids that the query tokens lie at (each list once per call), codes of the passages of stage 3 and codes and
    residuals of those of stage 4 (each passage once per call), the products of stage 4, queries in and results out."""
    C, P = case["C"], case["P"]
    mean = 68.0 if case["lo"] == 8 else (case["lo"] + case["hi"]) / 2
    token = 16 * case["nbits"]
    if case["kind"] == "build":
        n = P * mean
        return {"bytes": n * (512 + 4 + token + 4) + C * 512 + P * 8, "flops": 2.0 * DIM * C * n}
    if case["kind"] == "decode":
        n = case["n"] * mean
        return {"bytes": n * (4 + token) + min(C, n) * 512 + n * (512 + 128) + case["n"] * 24, "flops": n * DIM}
    nq, ndocs = case["nq"], case["ndocs"]
    p = _popularity(C)
    entries = P * -np.expm1(mean * np.log1p(-p))  # expected length of each inverted list
    lists = float(np.sum(-np.expm1(QLEN * nq * np.log1p(-p)) * entries))

    def distinct(n):  # passages among n draws with each query's its own
        return P * -math.expm1(-n * nq / P)
    if case["kind"] == "vanilla":
        scored = min(ndocs, P)
        codes, full, tokens = 0.0, distinct(scored), nq * scored * mean
    else:
        n3 = min(max(1, ndocs // 4), P)
        codes, full, tokens = distinct(min(ndocs, P)), distinct(n3), nq * n3 * mean
    return {"bytes": C * 512 + 4 * lists + codes * (mean * 4 + 16) + full * mean * token + nq * (QLEN * DIM * 4 + 8 * case["k"]),
            "flops": 2.0 * DIM * QLEN * (C * nq + tokens)}


def tolerance(case):
    if case["kind"] in ("decode", "build"):
        return "exact"  # whole numbers, and vectors that are one fp32 addition per element
    # fp32 scores of 32 summed dot products: against the double-precision score kernels and against MaxSim in double on the
    # decompressed passages the largest relative differences seen are 5.8e-8 (2-norm) and 1.3e-7 (single score); ids change
    # places where scores tie within that (up to 0.0011 of the ids of a thousand results)
    return {"rel": 2.5e-7, "max": 1e-6, "differ": 0.004}
