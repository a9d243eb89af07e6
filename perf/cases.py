"""What the performance of this framework is measured on: the calls of a decoding step, through the
public binding, over the sizes they are used at.

A case names one kind of call and its sizes.  Lengths are part of a case (drawn from its
`lengths` number), so that every state of a case has the same work; tensors, page tables, tokens and
uniforms are drawn from the seed.

Kinds
  attn    fd_verify_draft_attn on bf16, head dim 128 or 64, page size a power of two >= 16
  exact   fd_verify_draft_attn on float32, and on bf16 with head dims or page sizes the matrix-core
          kernel does not take
  greedy  fd_accept_greedy
  sample  fd_accept_sample
  select  fd_draft_select
  step    one whole decoding step of a few layers in full parallel mode: plan, attention per layer,
          greedy acceptance, drafting of every block, branch selection, commit of the accepted rows
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2605_20022_amd import flexdraft as fd

VOCAB = 151936


def _attn(name, batch, kv, verify, mask_len, *, blocks=1, hq=32, hkv=8, dim=128, page=16, dtype="bf16", planned=True,
          shuffled=True, lengths=1, kind="attn"):
    return dict(name=name, kind=kind, dtype=dtype, batch=batch, hq=hq, hkv=hkv, dim=dim, page=page, kv_lo=kv[0], kv_hi=kv[1],
                k_lo=verify[0], k_hi=verify[1], mask_len=mask_len, blocks=blocks, planned=planned, shuffled=shuffled,
                lengths=lengths)


def _accept(name, kind, batch, rows, *, dtype="bf16", vocab=VOCAB, lengths=1):
    return dict(name=name, kind=kind, dtype=dtype, batch=batch, k_lo=rows[0], k_hi=rows[1], vocab=vocab, lengths=lengths)


def listed():
    return [
        # one interactive user: the bonus token and a block of 15 mask tokens over a contiguous cache
        _attn("attn_b1", 1, (2048, 2048), (1, 1), 15, planned=False, shuffled=False),
        # a served batch of mixed lengths, 8 drafts verified and 8 drafted, planned once per decoding step
        _attn("attn_ragged", 16, (512, 4096), (8, 8), 8),
        # the large-batch mode: verification alone, as many rows as the confidence left
        _attn("attn_verify_b128", 128, (1024, 8192), (1, 16), 0),
        # long documents
        _attn("attn_long", 4, (32768, 32768), (16, 16), 16),
        # full parallel mode, one mask block per hypothetical number of accepted drafts: 272 and 36 new rows
        _attn("attn_parallel_b2", 2, (2048, 8192), (16, 16), 16, blocks=0),
        _attn("attn_parallel_b8", 8, (2048, 8192), (4, 4), 8, blocks=0),
        # the same batch as attn_ragged on a model with a head dim of 64
        _attn("attn_dim64", 16, (512, 4096), (8, 8), 8, dim=64),
        # float32, as a model is checked or a small one served at full precision
        _attn("exact_f32", 4, (512, 2048), (8, 8), 8, dtype="f32", planned=False, kind="exact"),
        # acceptance after attn_ragged and attn_long, and the draft block's token pick for 32 sequences
        _accept("greedy_b16", "greedy", 16, (8, 8)),
        _accept("sample_b4", "sample", 4, (16, 16)),
        _accept("select_b32", "select", 32, (15, 15)),
        # one user's whole step in full parallel mode: 8 verify rows, 8 blocks of 8, four layers
        dict(_attn("step_b1", 1, (2048, 2048), (8, 8), 8, blocks=0, kind="step"), layers=4, vocab=VOCAB),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


_MOST_BYTES = 2.3e9                            # the largest listed case (attn_verify_b128)
_MOST_FLOPS = {"attn": 6.5e10, "exact": 2.2e9, "step": 3e10}


def draw(rng):
    kind = rng.choice(["attn", "attn", "attn", "exact", "greedy", "sample", "select", "step"])
    lengths = rng.randrange(1 << 20)
    if kind in ("greedy", "sample", "select"):
        batch = _log(rng, 1, 64 if kind == "greedy" else 32)
        hi = rng.randint(2, 16)
        vocab = rng.choice([VOCAB, VOCAB, 32000, 128256, _log(rng, 1000, VOCAB)])
        return {k: v for k, v in _accept("", kind, batch, (rng.randint(1, hi), hi), dtype=rng.choice(["bf16", "bf16", "bf16", "f32"]),
                                         vocab=vocab, lengths=lengths).items() if k != "name"}
    while True:
        if kind == "attn":
            batch, hi = _log(rng, 1, 128), _log(rng, 256, 32768)
            k = rng.randint(0, 16)
            c = _attn("", batch, (max(1, hi // rng.choice([1, 2, 4, 8])), hi), (min(k, rng.choice([k, 1])), k), rng.choice([0, 8, 15, 16, rng.randint(1, 16)]),
                      blocks=rng.choice([1, 1, 1, 0]), hq=rng.choice([32, 32, 16, 40, 64]), dim=rng.choice([128, 128, 128, 64]),
                      page=rng.choice([16, 16, 32, 64]), planned=rng.random() < 0.75, shuffled=rng.random() < 0.8, lengths=lengths)
        elif kind == "exact":
            dtype = rng.choice(["f32", "f32", "bf16"])
            hi = _log(rng, 64, 4096)
            k = rng.randint(1, 16)
            c = _attn("", _log(rng, 1, 16), (max(1, hi // rng.choice([1, 2, 4])), hi), (k, k), rng.choice([0, 4, 8, rng.randint(1, 16)]), kind="exact",
                      hq=rng.choice([32, 16, 4]), hkv=rng.choice([8, 4, 1]), dim=rng.choice([128, 64, 96]), dtype=dtype,
                      page=rng.choice([16, 1, 8]), planned=False, lengths=lengths)
            if c["hq"] % c["hkv"] or (dtype == "bf16" and c["dim"] != 96 and c["page"] == 16):
                continue
        else:
            k = rng.randint(2, 16)
            hi = _log(rng, 256, 8192)
            c = dict(_attn("", rng.randint(1, 4), (max(1, hi // 2), hi), (k, k), rng.randint(4, 16), blocks=0, kind="step",
                           hq=rng.choice([32, 16, 40]), lengths=lengths), layers=rng.randint(2, 4), vocab=VOCAB)
        del c["name"]
        kv_len, n = _lengths(c)[0], _lengths(c)[2]
        if int(n.sum()) == 0:
            continue
        w = work(c)
        if w["bytes"] <= _MOST_BYTES and w["flops"] <= _MOST_FLOPS[kind] and int(kv_len.sum()) > 0:
            return c


# ---- sizes of a case --------------------------------------------------------------------------
def _lengths(c):
    """(prefix lengths, verify rows, new rows, mask blocks) of every sequence."""
    r = np.random.default_rng(c["lengths"])
    kv = r.integers(c["kv_lo"], c["kv_hi"] + 1, size=c["batch"]).astype(np.int32)
    k = r.integers(c["k_lo"], c["k_hi"] + 1, size=c["batch"]).astype(np.int32)
    nb = np.maximum(k, 1) if c["blocks"] == 0 else np.full(c["batch"], c["blocks"], dtype=np.int32)
    return kv, k, (k + nb * c["mask_len"]).astype(np.int32), nb.astype(np.int32)


def _accept_rows(c):
    return np.random.default_rng(c["lengths"]).integers(c["k_lo"], c["k_hi"] + 1, size=c["batch"]).astype(np.int32)


def _attn_work(c, layers=1):
    kv, k, n, nb = _lengths(c)
    e = 2 if c["dtype"] == "bf16" else 4
    kv64, n64 = kv.astype(np.int64), n.astype(np.int64)
    rows = int(n64.sum())
    new_keys = n64 * n64 if c["blocks"] == 1 else n64 * (k + c["mask_len"])        # what the masks leave, at most
    b = int(kv64.sum()) * c["hkv"] * c["dim"] * 2 * e                             # the cache
    b += rows * (2 * c["hq"] + 2 * c["hkv"]) * c["dim"] * e + rows * c["hq"] * 4   # q, out, new K and V, lse
    f = int((n64 * kv64 + new_keys).sum()) * c["hq"] * c["dim"] * 4
    return {"bytes": b * layers, "flops": f * layers}


def work(case):
    c = case
    e = 2 if c["dtype"] == "bf16" else 4
    if c["kind"] in ("attn", "exact"):
        return _attn_work(c)
    if c["kind"] == "step":
        w = _attn_work(c, c["layers"])
        _, k, n, _ = _lengths(c)
        logits = int(n.sum()) * c["vocab"]
        append = int(k.sum()) * c["hkv"] * c["dim"] * 2 * e * 2 * c["layers"]
        return {"bytes": w["bytes"] + logits * e + append, "flops": w["flops"] + 4 * logits}
    logits = int(_accept_rows(c).sum()) * c["vocab"]
    # a comparison per logit; a comparison, an exponential and two additions more where probabilities are asked for
    return {"bytes": logits * e * (2 if c["kind"] == "sample" else 1), "flops": logits * {"greedy": 1, "select": 4, "sample": 8}[c["kind"]]}


def tolerance(case):
    # Against the same call in 64-bit arithmetic on the same inputs (relative 2-norm): bf16 outputs 1.7e-3 to
    # 2.4e-3 (the rounding of the probabilities and of the result, 2^-9 each), float32 outputs 4e-7 to 6e-7,
    # the confidences of the token pick 1.7e-7; four times that is allowed.  Tokens and lengths are whole numbers and stay as they are.
    if case["kind"] in ("greedy", "sample"):
        return "exact"
    if case["kind"] == "select":
        return {"rel": 7e-7}
    return {"rel": 2.3e-6} if case["dtype"] == "f32" else {"rel": 9e-3}


# ---- states -----------------------------------------------------------------------------------
def _i32(x):
    return torch.from_numpy(np.ascontiguousarray(x, dtype=np.int32)).cuda()


def _indptr(n):
    return np.concatenate([[0], np.cumsum(n)])


def _dtype(c):
    return torch.bfloat16 if c["dtype"] == "bf16" else torch.float32


def _prepare_attn(c, gen, host, layers=1, room=0):
    """Lengths and page tables shared by all layers, tensors for each; `room`: cache slots beyond the prefix.

    Queries and keys have unit variance, as after a per-head norm: scores spread like N(0, 1)."""
    kv, k, n, nb = _lengths(c)
    ps, dt = c["page"], _dtype(c)
    pages = (kv.astype(np.int64) + room + ps - 1) // ps
    used = int(pages.sum())
    pool = used + used // 32
    ids = host.permutation(pool)[:used] if c["shuffled"] else np.arange(used)
    R, D = int(n.sum()), c["dim"]
    randn = lambda *s: torch.randn(*s, generator=gen, device="cuda", dtype=dt)  # noqa: E731
    s = dict(page_indptr=_i32(_indptr(pages)), page_indices=_i32(ids), kv_len=_i32(kv), row_indptr=_i32(_indptr(n)),
             verify_len=_i32(k), mask_blocks=_i32(nb) if c["blocks"] != 1 else None,
             status=torch.zeros(1, dtype=torch.int32, device="cuda"), workspace=None, layers=[])
    for _ in range(layers):
        t = dict(q=randn(R, c["hq"], D), k_new=randn(R, c["hkv"], D), v_new=randn(R, c["hkv"], D),
                 k_cache=randn(pool, c["hkv"], ps, D), v_cache=randn(pool, c["hkv"], ps, D),
                 out=torch.empty(R, c["hq"], D, device="cuda", dtype=dt), lse=torch.empty(R, c["hq"], device="cuda"))
        t["args"] = fd.make_attn_args(t["q"], t["k_new"], t["v_new"], t["k_cache"], t["v_cache"], s["page_indptr"], s["page_indices"],
                                      s["kv_len"], s["row_indptr"], s["verify_len"], None, s["mask_blocks"], out=t["out"], lse=t["lse"],
                                      max_kv_len=int(kv.max()), max_new_rows=int(n.max()),
                                      flags=fd.FD_ATTN_PLANNED if c["planned"] else 0, status=s["status"])
        if s["workspace"] is None:
            s["workspace"] = fd.alloc_workspace(fd.fd_verify_draft_attn_workspace(t["args"]))
        t["args"].workspace = s["workspace"].data_ptr()
        t["args"].workspace_bytes = s["workspace"].numel()
        s["layers"].append(t)
    return s


def _greedy_tokens(logits, gen, vocab):
    """Tokens fed at the verify rows: each draft is what the row before it prefers, seven times in ten."""
    R = logits.shape[0]
    other = torch.randint(0, vocab, (R,), generator=gen, device="cuda")
    agree = torch.rand(R, generator=gen, device="cuda") < 0.7
    return torch.where(agree, logits.argmax(dim=1).roll(1), other).to(torch.int32)


def _peaked(rows, vocab, gen, dt):
    """A drafter's logits: unit normal and one raised entry a row, so that its probability is anything from a few percent to nearly one."""
    x = torch.randn(rows, vocab, generator=gen, device="cuda", dtype=dt)
    top = torch.randint(0, vocab, (rows, 1), generator=gen, device="cuda")
    up = 6 + 10 * torch.rand(rows, 1, generator=gen, device="cuda")
    return x.scatter_(1, top, (x.gather(1, top).float() + up).to(dt))


def _empty(n, dtype=torch.int32):
    return torch.empty(n, dtype=dtype, device="cuda")


def prepare(case, seed):
    c = case
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    host = np.random.default_rng(seed)
    s = dict(case=c)
    if c["kind"] in ("attn", "exact"):
        s.update(_prepare_attn(c, gen, host))
        if c["planned"]:
            fd.fd_verify_draft_plan(s["layers"][0]["args"])
        return s
    if c["kind"] == "step":
        s.update(_prepare_attn(c, gen, host, c["layers"], room=c["k_hi"]))
        _, k, n, nb = _lengths(c)
        B, V, R, M, blocks = c["batch"], c["vocab"], int(k.sum()), int((n - k).sum()), int(nb.sum())
        s["verify_logits"] = torch.randn(R, V, generator=gen, device="cuda", dtype=_dtype(c)) * 3
        s["mask_logits"] = _peaked(M, V, gen, _dtype(c))
        s["tokens"] = _greedy_tokens(s["verify_logits"], gen, V)
        s.update(verify_indptr=_i32(_indptr(k)), branch_indptr=_i32(_indptr(n - k)), kmax=int(k.max()),
                 block_indptr=_i32(np.arange(blocks + 1) * c["mask_len"]), accept_len=_empty(B), bonus=_empty(B), drafted=_empty(M),
                 confidence=_empty(M, torch.float32), keep_len=_empty(blocks),
                 next_tokens=_empty((B, c["mask_len"])), block=_empty(B), kv_len_out=[_empty(B) for _ in range(c["layers"])],
                 accept_ws=fd.alloc_workspace(fd.fd_accept_workspace(B, R, V, False)),
                 select_ws=fd.alloc_workspace(fd.fd_draft_select_workspace(M, V)))
        return s
    k = _accept_rows(c)
    B, V, R, dt = c["batch"], c["vocab"], int(k.sum()), _dtype(c)
    s.update(indptr=_i32(_indptr(k)), kmax=int(k.max()), accept_len=_empty(B), bonus=_empty(B))
    if c["kind"] == "select":
        s.update(logits=_peaked(R, V, gen, dt), tokens=_empty(R), confidence=_empty(R, torch.float32),
                 workspace=fd.alloc_workspace(fd.fd_draft_select_workspace(R, V)))
    elif c["kind"] == "greedy":
        s["logits"] = torch.randn(R, V, generator=gen, device="cuda", dtype=dt) * 3
        s.update(tokens=_greedy_tokens(s["logits"], gen, V), row_argmax=_empty(R),
                 workspace=fd.alloc_workspace(fd.fd_accept_workspace(B, R, V, False)))
    else:
        s["target"] = torch.randn(R, V, generator=gen, device="cuda", dtype=dt) * 2
        s["draft"] = (s["target"].float() + 0.5 * torch.randn(R, V, generator=gen, device="cuda")).to(dt)
        drawn = torch.multinomial(torch.softmax(s["draft"].float(), dim=1), 1, generator=gen).flatten().to(torch.int32)
        s.update(tokens=drawn.roll(1), u_accept=torch.rand(R, generator=gen, device="cuda"), u_resample=torch.rand(R, generator=gen, device="cuda"),
                 workspace=fd.alloc_workspace(fd.fd_accept_workspace(B, R, V, True)))
    return s


def run(state):
    s = state
    kind = s["case"]["kind"]
    if kind in ("attn", "exact"):
        t = s["layers"][0]
        fd.fd_verify_draft_attn(t["args"])
        return {"out": t["out"], "lse": t["lse"]}
    if kind == "greedy":
        fd.fd_accept_greedy(s["logits"], s["indptr"], s["tokens"], s["accept_len"], s["bonus"], max_rows_per_seq=s["kmax"],
                            row_argmax=s["row_argmax"], workspace=s["workspace"])
        return {"accept_len": s["accept_len"], "bonus": s["bonus"], "row_argmax": s["row_argmax"]}
    if kind == "sample":
        fd.fd_accept_sample(s["target"], s["draft"], s["indptr"], s["tokens"], s["u_accept"], s["u_resample"], s["accept_len"], s["bonus"],
                            temperature=1.0, max_rows_per_seq=s["kmax"], workspace=s["workspace"])
        return {"accept_len": s["accept_len"], "bonus": s["bonus"]}
    if kind == "select":
        fd.fd_draft_select(s["logits"], s["indptr"], s["tokens"], s["accept_len"], temperature=1.0, threshold=0.3, max_rows_per_seq=s["kmax"],
                           confidence=s["confidence"], workspace=s["workspace"])
        return {"tokens": s["tokens"], "confidence": s["confidence"], "keep_len": s["accept_len"]}
    fd.fd_verify_draft_plan(s["layers"][0]["args"])
    for t in s["layers"]:
        fd.fd_verify_draft_attn(t["args"])
    fd.fd_accept_greedy(s["verify_logits"], s["verify_indptr"], s["tokens"], s["accept_len"], s["bonus"], max_rows_per_seq=s["kmax"],
                        workspace=s["accept_ws"])
    fd.fd_draft_select(s["mask_logits"], s["block_indptr"], s["drafted"], s["keep_len"], temperature=1.0, threshold=0.3,
                       max_rows_per_seq=s["case"]["mask_len"], confidence=s["confidence"], workspace=s["select_ws"])
    fd.fd_select_branch(s["drafted"], s["branch_indptr"], s["mask_blocks"], s["accept_len"], s["next_tokens"], verify_len=s["verify_len"],
                        out_block=s["block"])
    for t, n in zip(s["layers"], s["kv_len_out"]):
        fd.fd_append_kv(t["args"], t["k_cache"], t["v_cache"], s["accept_len"], n)
    return {"out": [t["out"] for t in s["layers"]], "lse": [t["lse"] for t in s["layers"]], "accept_len": s["accept_len"], "bonus": s["bonus"],
            "drafted": s["drafted"], "confidence": s["confidence"], "keep_len": s["keep_len"], "next_tokens": s["next_tokens"], "block": s["block"],
            "k_cache": [t["k_cache"] for t in s["layers"]], "v_cache": [t["v_cache"] for t in s["layers"]], "kv_len": s["kv_len_out"]}
