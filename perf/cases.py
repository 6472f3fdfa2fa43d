"""The performance cases of the NN-select + encode path.

What users of this library run, through its public entry points, over the range
of sizes they run it at: whole ranking requests (`SelectEncode`,
`SelectEncodeEq2`), the NN search alone (`nn_select`), the encoder alone
(`encode`) and the serving mini-batch from host buffers (`Batcher`).  Shapes are
those of the workloads the repository names (synth/configs.py) or lie in their
ranges.  Embeddings are random unit rows, as L2-normalised item embeddings are
(bf16, or the int8 codes of the paper's storage, Sec. 3.2.1), weights are drawn
with standard deviation 1 / sqrt(fan in), so that attention is not uniform.

A case's `kind`:
  path    tav2_select_encode on device-resident requests
  eq2     tav2_select_encode_eq2 (the four token sources of Eq. 2)
  select  tav2_nn_select
  encode  tav2_encode on explicit tokens
  serve   host requests through a Batcher: collate, upload, select + encode,
          wait for the results
"""
import math
from types import SimpleNamespace

import numpy as np
import torch

from paper_2506_02267_amd import tav2

STEP_I8 = 0.65 / 127.0     # dequantisation step of the int8 storage (Sec. 3.2.1)


def _path(name, dtype, R, L_min, L, N, k, d, dm, heads, ffn, layers, rt=0, has_time=True,
          packed=True, kind="path", **more):
    """R requests of L_min..L lifelong rows and N candidates each (N_min..N where
    the case says so)."""
    c = dict(kind=kind, dtype=dtype, R=R, L_min=L_min, L=L, N=N, k=k, d=d, dm=dm, heads=heads,
             ffn=ffn, layers=layers, rt=rt, has_time=has_time, packed=packed, **more)
    return dict(c, name=name) if name else c


def _select(name, dtype, R, L_min, L, N, k, d):
    c = dict(kind="select", dtype=dtype, R=R, L_min=L_min, L=L, N=N, k=k, d=d)
    return dict(c, name=name) if name else c


def _encode(name, B, T, T_min, d, dm, heads, ffn, layers, mask=0):
    """B candidates of T positions, T_min..T of them valid."""
    c = dict(kind="encode", dtype="bf16", B=B, T=T, T_min=T_min, d=d, dm=dm, heads=heads, ffn=ffn,
             layers=layers, mask=mask)
    return dict(c, name=name) if name else c


def listed():
    return [
        # one ranking request at full scale: 16384 actions, 1000 candidates (the
        # repository's benchmark workload)
        _path("request", "bf16", 1, 16384, 16384, 1000, 256, 256, 256, 4, 1024, 2),
        # a batch of users with histories of very different lengths
        _path("ragged_batch", "bf16", 16, 1024, 16384, 500, 128, 256, 256, 4, 512, 2),
        # every token source of Eq. 2: lifelong, kept and searched real-time rows,
        # impressions
        _path("request_eq2", "bf16", 1, 16384, 16384, 1000, 256, 256, 256, 4, 1024, 2, rt=200,
              kind="eq2", keep=32, k_rt=32, imp=300, k_imp=64),
        # the heaviest: thousands of candidates per request, 512 tokens, 8 heads
        _path("heavy_batch", "bf16", 2, 16384, 16384, 4000, 512, 256, 256, 8, 1024, 2),
        # a small late-stage request: few candidates, a short history; latency
        _path("small_request", "bf16", 1, 3001, 3001, 24, 64, 256, 256, 4, 1024, 2, rt=20),
        # the paper's production model on its int8 storage, one batch of 256
        _path("production_i8", "i8", 1, 16384, 16384, 256, 128, 32, 64, 1, 32, 2, rt=64),
        # float32 serving of a tiny model (parity runs, small deployments)
        _path("tiny_f32", "f32", 1, 1024, 1024, 16, 32, 64, 64, 2, 128, 1, has_time=False),
        # retrieval only, int8 storage: 1000 candidates against one long history
        _select("search_i8", "i8", 1, 16384, 16384, 1000, 256, 32),
        # retrieval only over many short histories
        _select("search_short", "bf16", 32, 200, 4000, 100, 64, 64),
        # the production encoder alone at the production batch (256 x 192)
        _encode("encode_192", 256, 192, 192, 32, 64, 1, 32, 2),
        # the production encoder on long sequences of mixed valid lengths
        _encode("encode_long", 200, 1024, 300, 32, 64, 1, 32, 2),
        # a serving mini-batch from host memory: 8 requests of 16 candidates
        _path("serve_128", "i8", 8, 16384, 16384, 16, 128, 32, 64, 1, 32, 2, rt=64, kind="serve"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["path", "path", "production", "f32", "eq2", "select", "select", "encode",
                       "encode", "encode", "serve"])
    if kind in ("path", "eq2"):
        k = _log(rng, 17, 512)
        N = _log(rng, 9, 4000)
        R = max(1, min(_log(rng, 1, 16), 4000 * 512 // (N * (k + 200))))
        L = _log(rng, 300, 16384)
        d = rng.choice([64, 128, 256, 256])
        heads, ffn, layers = rng.choice([4, 4, 8]), rng.choice([512, 1024, 1024]), rng.choice([1, 2, 2])
        more = dict(has_time=rng.random() < 0.8, packed=rng.random() < 0.8)
        L_min = max(1, int(L * rng.choice([1.0, 0.3, 0.06])))
        if kind == "path":
            return _path(None, "bf16", R, L_min, L, N, k, d, 256, heads, ffn, layers,
                         rt=rng.choice([0, 0, rng.randint(1, 120)]), **more)
        rt = rng.randint(40, 300)
        return _path(None, "bf16", R, L_min, L, N, k, d, 256, heads, ffn, layers, rt=rt, kind="eq2",
                     keep=rng.randint(0, 64), k_rt=rng.choice([0, rng.randint(1, 64)]),
                     imp=rng.randint(50, 1000), k_imp=rng.choice([0, rng.randint(1, 100)]), **more)
    if kind == "production":
        R = _log(rng, 1, 32)
        L = _log(rng, 500, 16384)
        return _path(None, rng.choice(["bf16", "i8"]), R, max(1, int(L * rng.choice([1.0, 0.2]))), L,
                     _log(rng, 16, max(16, 4096 // R)), rng.randint(16, 256), 32, 64,
                     rng.choice([1, 1, 2]), 32, 2, rt=rng.choice([0, rng.randint(1, 100)]),
                     packed=rng.random() < 0.8)
    if kind == "f32":
        k = rng.randint(8, 40)
        return _path(None, "f32", _log(rng, 1, 8), 100, _log(rng, 120, 8000), _log(rng, 4, 200), k,
                     64, 64, 2, 128, rng.choice([1, 2]), rt=rng.choice([0, rng.randint(1, 20)]),
                     has_time=rng.random() < 0.5)
    if kind == "select":
        dtype = rng.choice(["bf16", "bf16", "i8", "i8", "f32"])
        R = _log(rng, 1, 64)
        L = _log(rng, 200, 16384)
        N = _log(rng, 8, max(8, (4000 if dtype != "f32" else 500) // R))
        return _select(None, dtype, R, max(1, int(L * rng.choice([1.0, 0.5, 0.06]))), L, N,
                       rng.choice([rng.randint(8, 256), rng.randint(8, 1024)]),
                       rng.choice([32, 32, 64, 128, 256]))
    if kind == "encode":
        if rng.random() < 0.35:
            T = _log(rng, 9, 700)
            return _encode(None, _log(rng, 8, max(8, min(2000, 1000000 // T))), T,
                           max(1, int(T * rng.choice([1.0, 0.5]))), rng.choice([64, 128, 256]), 256,
                           rng.choice([4, 8]), rng.choice([512, 1024]), 2,
                           mask=1 if T <= 128 and rng.random() < 0.3 else 0)
        T = _log(rng, 17, 2048)
        ffn, layers = rng.choice([(32, 2), (32, 2), (64, 1), (128, 1)])
        return _encode(None, _log(rng, 8, max(8, min(4096, 500000 // T))), T,
                       max(1, int(T * rng.choice([1.0, 0.5, 0.1]))), rng.choice([32, 32, 64]), 64,
                       rng.choice([1, 1, 2]), ffn, layers,
                       mask=1 if T <= 64 and rng.random() < 0.3 else 0)
    R = _log(rng, 1, 32)
    L = _log(rng, 1000, 16384)
    return _path(None, "i8", R, max(1, int(L * rng.choice([1.0, 0.3]))), L, 16, rng.randint(32, 192),
                 32, 64, 1, 32, 2, rt=64, kind="serve")


# ------------------------------------------------------------------ inputs
def _torch_dtype(case):
    return {"bf16": torch.bfloat16, "f32": torch.float32, "i8": torch.int8}[case["dtype"]]


def _code(case):
    return {"bf16": tav2.BF16, "f32": tav2.F32, "i8": tav2.I8}[case["dtype"]]


def _unit(g, rows, d):
    e = torch.randn((rows, d), generator=g, device=g.device)
    return e / e.norm(dim=1, keepdim=True)


def _rows(g, rows, d, dtype):
    e = _unit(g, rows, d)
    if dtype == torch.int8:
        return (e / STEP_I8).round().clamp(-127, 127).to(torch.int8)
    return e.to(dtype)


def _seq(case, g, lengths):
    """Packed sequences of the given lengths on the generator's device; time buckets
    rise within a request (row 0 is the newest action)."""
    rows, dev = int(sum(lengths)), g.device
    emb = _rows(g, rows, case["d"], _torch_dtype(case))
    act = torch.randint(0, 8, (rows,), generator=g, device=dev, dtype=torch.uint8)
    time = None
    if case.get("has_time", True):
        who = torch.repeat_interleave(torch.arange(len(lengths), device=dev),
                                      torch.tensor(lengths, device=dev), output_size=rows)
        time = torch.randint(0, 64, (rows,), generator=g, device=dev) + 64 * who
        time = (torch.sort(time).values % 64).to(torch.uint8)
    offset = np.concatenate([[0], np.cumsum(lengths)[:-1]]).astype(np.int64)
    return tav2.DeviceSeq(emb=emb, act=act, time=time, offset=torch.from_numpy(offset).to(dev),
                          length=torch.tensor(lengths, dtype=torch.int32, device=dev),
                          max_len=int(max(lengths)), dtype=_code(case))


def _lengths(case, r):
    n = [int(x) for x in r.integers(case["L_min"], case["L"] + 1, size=case["R"])]
    n[0] = case["L"]
    return n


def _counts(case):
    """Candidates of each request: the requests of a batch differ, between 3/4 N and N
    (those of a serving mini-batch do not)."""
    R, N = case["R"], case["N"]
    return [N if case["kind"] == "serve" else N - 37 * i % (N // 4 + 1) for i in range(R)]


def _inputs(case, seed, device="cuda"):
    """The request batch of a path, eq2, select or serve case."""
    r = np.random.default_rng(seed)
    g = torch.Generator(device=device)
    g.manual_seed(seed)
    seq = _seq(case, g, _lengths(case, r))
    R = case["R"]
    counts = _counts(case)
    off = np.concatenate([[0], np.cumsum(counts)]).astype(np.int64)
    cemb = _rows(g, int(off[-1]), case["d"],
                 torch.float32 if case["dtype"] == "f32" else torch.bfloat16)
    cands = tav2.DeviceCands(emb=cemb, offset=torch.from_numpy(off).to(device), max_count=max(counts))
    rt = _seq(case, g, [case["rt"]] * R) if case.get("rt") else None
    imp = _seq(case, g, [case["imp"]] * R) if case.get("imp") else None
    return SimpleNamespace(seq=seq, cands=cands, rt=rt, imp=imp, counts=counts)


def _tokens(case):
    """Positions of the encoder."""
    if case["kind"] == "encode":
        return case["T"]
    if case["kind"] == "eq2":
        return case["k"] + min(case["keep"], case["rt"]) + case["k_rt"] + case["k_imp"]
    return case["k"] + case["rt"]


def _weights(case, seed):
    """Host weights, the layout DeviceWeights takes."""
    r = np.random.default_rng(seed + 7919)
    dm, ff, d = case["dm"], case["ffn"], case["d"]
    bf16 = case["dtype"] != "f32"

    def mat(rows, cols, std):
        a = (r.standard_normal((rows, cols), dtype=np.float32) * np.float32(std))
        return torch.from_numpy(a).bfloat16().float().numpy() if bf16 else a

    def vec(n, mean=0.0):
        return (mean + 0.05 * r.standard_normal(n, dtype=np.float32)).astype(np.float32)

    layers = [SimpleNamespace(W_qkv=mat(3 * dm, dm, dm ** -0.5), b_qkv=vec(3 * dm),
                              W_o=mat(dm, dm, dm ** -0.5), b_o=vec(dm), ln1_g=vec(dm, 1.0),
                              ln1_b=vec(dm), W_1=mat(ff, dm, dm ** -0.5), b_1=vec(ff),
                              W_2=mat(dm, ff, ff ** -0.5), b_2=vec(dm), ln2_g=vec(dm, 1.0),
                              ln2_b=vec(dm)) for _ in range(case["layers"])]
    T = _tokens(case)
    # token and candidate rows are unit vectors: a projection of std 1 gives
    # features of the size of the side tables' (0.5)
    return SimpleNamespace(d_in=d, d_model=dm, n_heads=case["heads"], d_ffn=ff, max_pos=T,
                           dtype="bf16" if bf16 else "f32", W_in=mat(dm, 2 * d, 1.0), b_in=vec(dm),
                           E_act=mat(8, dm, 0.5),
                           E_time=mat(64, dm, 0.5) if case.get("has_time", True) else None,
                           E_pos=mat(T, dm, 0.5), layers=layers, W_pool=mat(dm, dm, dm ** -0.5),
                           b_pool=vec(dm))


def _explicit(case, seed):
    """Tokens of an encode case."""
    r = np.random.default_rng(seed)
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    B, T, d = case["B"], case["T"], case["d"]
    emb = _rows(g, B * T, d, torch.bfloat16).view(B, T, d)
    act = torch.randint(0, 8, (B, T), generator=g, device="cuda", dtype=torch.uint8)
    time = torch.sort(torch.randint(0, 64, (B, T), generator=g, device="cuda"), 1).values
    valid = r.integers(case["T_min"], T + 1, size=B).astype(np.int32)
    tok = tav2.DeviceTokens(emb=emb, act=act, time=time.to(torch.uint8),
                            valid_len=torch.from_numpy(valid).cuda(), dtype=tav2.BF16)
    return tok, _rows(g, B, d, torch.bfloat16)


# ------------------------------------------------------------------ the passes
def prepare(case, seed):
    kind = case["kind"]
    if kind == "encode":
        tok, cand = _explicit(case, seed)
        w = tav2.DeviceWeights(_weights(case, seed), pack=True)
        out = torch.empty((case["B"], 2 * case["dm"]), dtype=torch.float32, device="cuda")
        return SimpleNamespace(kind=kind, tok=tok, cand=cand, w=w, out=out, ws=tav2.Workspace(),
                               mask=case["mask"])
    if kind == "serve":
        return _prepare_serve(case, seed)
    x = _inputs(case, seed)
    total = x.cands.total
    if kind == "select":
        return SimpleNamespace(kind=kind, x=x, k=case["k"], ws=tav2.Workspace(),
                               idx=torch.empty((total, case["k"]), dtype=torch.int32, device="cuda"),
                               score=torch.empty((total, case["k"]), dtype=torch.float32,
                                                 device="cuda"))
    w = tav2.DeviceWeights(_weights(case, seed), pack=case["packed"])
    if kind == "eq2":
        call = tav2.SelectEncodeEq2(x.seq, x.rt, case["keep"], case["k_rt"], x.imp, case["k_imp"],
                                    x.cands, case["k"], w)
    else:
        call = tav2.SelectEncode(x.seq, x.rt, x.cands, case["k"], w)
    return SimpleNamespace(kind=kind, x=x, w=w, call=call)


def _prepare_serve(case, seed):
    """Requests as host arrays (what a feature service hands over), the batcher, the
    model and the output buffers a serving thread keeps."""
    x = _inputs(case, seed, device="cpu")
    reqs = []
    for r in range(case["R"]):
        a, n = int(x.seq.offset[r]), int(x.seq.length[r])
        b, m = int(x.rt.offset[r]), case["rt"]
        c = int(x.cands.offset[r])
        cand = x.cands.emb[c:c + case["N"]].view(torch.int16).numpy()
        reqs.append((x.seq.emb[a:a + n].numpy(), x.seq.act[a:a + n].numpy(),
                     x.seq.time[a:a + n].numpy(), x.rt.emb[b:b + m].numpy(),
                     x.rt.act[b:b + m].numpy(), x.rt.time[b:b + m].numpy(), cand))
    total, k, dm = case["R"] * case["N"], case["k"], case["dm"]
    bt = tav2.Batcher(_code(case), case["d"], True, max_requests=case["R"],
                      max_rows=case["R"] * case["L"], max_rt_rows=case["R"] * case["rt"],
                      max_cands=total)
    w = tav2.DeviceWeights(_weights(case, seed), pack=case["packed"])
    dev = dict(device="cuda")
    return SimpleNamespace(kind="serve", reqs=reqs, bt=bt, w=w, k=k, ws=tav2.Workspace(),
                           idx=torch.empty((total, k), dtype=torch.int32, **dev),
                           score=torch.empty((total, k), dtype=torch.float32, **dev),
                           out=torch.empty((total, 2 * dm), dtype=torch.float32, **dev))


def run(state):
    kind = state.kind
    if kind == "encode":
        return tav2.encode(state.tok, state.cand, state.w, out=state.out, ws=state.ws,
                           flags=state.mask)
    if kind == "select":
        return tav2.nn_select(state.x.seq, state.x.cands, state.k, state.idx, state.score, state.ws)
    if kind == "serve":
        bt = state.bt
        bt.reset()
        for q in state.reqs:
            if not bt.add(*q):
                raise RuntimeError("the mini-batch does not fit the batcher")
        bt.upload()
        s, r, c = bt.views()
        tav2.select_encode_structs(s, r, c, state.k, state.w, state.idx, state.score, state.out,
                                   state.ws)
        # the batcher's arena may be filled again only after its upload has finished
        torch.cuda.current_stream().synchronize()
        return state.idx, state.score, state.out
    return state.call()


# ------------------------------------------------------------------ what a pass needs
def _mean_count(case):
    """Candidates and expected sequence rows of the batch."""
    return sum(_counts(case)), case["L"] + (case["R"] - 1) * (case["L_min"] + case["L"]) / 2


def _encoder_work(case, cands, T):
    """(flops, bytes of the weights) of `cands` candidates with T valid tokens."""
    dm, ff, d = case["dm"], case["ffn"], case["d"]
    layer = 2 * T * dm * (3 * dm + dm + 2 * ff) + 2 * dm * T * (T + 1)
    if case.get("mask"):
        layer += 2 * dm * T * (T - 1)
    flops = 2 * T * d * dm + 2 * d * dm + case["layers"] * layer + 2 * T * dm * dm
    eb = 4 if case["dtype"] == "f32" else 2
    wb = eb * (2 * d * dm + dm * dm + case["layers"] * dm * (4 * dm + 2 * ff) + (72 + T) * dm)
    return cands * flops, wb


def work(case):
    kind = case["kind"]
    if kind == "encode":
        B, T = case["B"], (case["T"] + case["T_min"]) / 2
        flops, wb = _encoder_work(case, B, T)
        return {"bytes": B * (T * (2 * case["d"] + 2) + 2 * case["d"] + 8 * case["dm"]) + wb,
                "flops": flops}
    cands, rows = _mean_count(case)
    eb = {"bf16": 2, "f32": 4, "i8": 1}[case["dtype"]]
    R, d, k = case["R"], case["d"], case["k"]
    flops = 2.0 * d * cands * rows / R
    nbytes = rows * d * eb + cands * d * max(eb, 2) + cands * k * 8
    if kind == "select":
        return {"bytes": nbytes, "flops": flops}
    if kind == "eq2":
        rest = max(0, case["rt"] - case["keep"])
        flops += 2.0 * d * cands * ((rest if case["k_rt"] else 0) + (case["imp"] if case["k_imp"] else 0))
        nbytes += R * d * eb * case["imp"] + cands * (case["k_rt"] + case["k_imp"]) * 8
    nbytes += R * d * eb * case["rt"] + 2 * rows + cands * 8 * case["dm"]
    k_valid = min(k, (case["L_min"] + case["L"]) / 2)
    f, wb = _encoder_work(case, cands, _tokens(case) - k + k_valid)
    return {"bytes": nbytes + wb, "flops": flops + f}


def tolerance(case):
    # Four times what the path shows against 64 bits over these ranges: scores 2.5e-7
    # (32-bit sums of up to 256 products), float32 outputs 2.9e-7, outputs of the bf16
    # encoders 2e-3 to 3e-3.  Rows whose 32-bit scores differ in the last bits only may
    # swap ranks, up to 1.4e-4 of the rows (one swap among 16 x 32 is 4e-3), and the
    # swapped tokens then move that candidate's outputs by up to 0.8 of their rms.
    if case["kind"] == "select":
        return {"rel": 1e-6, "max": 6e-6, "differ": 4e-3}
    if case["dtype"] == "f32":
        return {"rel": 1.2e-6, "max": 6e-6, "differ": 4e-3}
    if case["kind"] == "encode":
        return {"rel": 1.2e-2, "max": 0.06}
    return {"rel": 1.2e-2, "max": 0.95, "differ": 4e-3}


# ------------------------------------------------------------------ the same in 64 bits
def _scores64(case, seq, r, cand):
    a, n = int(seq.offset[r]), int(seq.length[r])
    e = seq.emb[a:a + n].double()
    s = cand.double() @ e.t()
    if case["dtype"] == "i8":
        s = s / e.norm(dim=1).clamp(min=1e-300)
    return s


def _topk64(case, seq, r, cand, k, first=0):
    """Rows [first, ..) of request r: (idx, score) padded to k, and how many are real."""
    s = _scores64(case, seq, r, cand)[:, first:]
    m = min(k, s.shape[1])
    v, i = torch.sort(s, dim=1, descending=True, stable=True)
    idx = torch.full((cand.shape[0], k), -1, dtype=torch.int64, device=s.device)
    score = torch.full((cand.shape[0], k), -math.inf, dtype=torch.float64, device=s.device)
    idx[:, :m], score[:, :m] = i[:, :m], v[:, :m]
    return idx, score, m


def _encode64(case, w, emb, act, time, cand, valid):
    """Encoder in 64 bits: emb [n, T, d], valid [n]."""
    D = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(emb.device).double()  # noqa: E731
    n, T, d = emb.shape
    dm, H = case["dm"], case["heads"]
    W_in = D(w.W_in)
    x = emb @ W_in[:, :d].t() + (cand @ W_in[:, d:].t())[:, None] + D(w.b_in)
    x = x + D(w.E_act)[act.long()] + D(w.E_pos)[:T]
    if w.E_time is not None:
        x = x + D(w.E_time)[time.long()]
    p = torch.arange(T, device=emb.device)
    seen = p[None, None, :] < valid[:, None, None]
    if not case.get("mask"):
        seen = seen & (p[None, :, None] >= p[None, None, :])
    ln = lambda v, g, b: torch.nn.functional.layer_norm(v, (dm,), D(g), D(b), 1e-5)  # noqa: E731
    for L in w.layers:
        q, k, v = (t.reshape(n, T, H, dm // H).transpose(1, 2).contiguous()
                   for t in (x @ D(L.W_qkv).t() + D(L.b_qkv)).split(dm, dim=2))
        s = q @ k.transpose(2, 3).contiguous() / math.sqrt(dm // H)
        s = s.masked_fill(~seen[:, None], -math.inf)
        o = torch.softmax(s, 3) @ v
        o = o.transpose(1, 2).reshape(n, T, dm)
        x = ln(x + o @ D(L.W_o).t() + D(L.b_o), L.ln1_g, L.ln1_b)
        h = torch.relu(x @ D(L.W_1).t() + D(L.b_1))
        x = ln(x + h @ D(L.W_2).t() + D(L.b_2), L.ln2_g, L.ln2_b)
    y = (x @ D(w.W_pool).t() + D(w.b_pool)).masked_fill((p[None] >= valid[:, None])[:, :, None],
                                                        -math.inf).amax(1)
    last = x[torch.arange(n, device=emb.device), (valid - 1).clamp(min=0)]
    return torch.cat([y, last], 1)


def _chunks(case, n, T):
    """Candidates at a time, so that a score tensor stays below about 1 GB."""
    step = max(1, int(1.2e8 // (case["heads"] * T * T + 8 * T * case["dm"] + T * case["ffn"])))
    return [(a, min(n, a + step)) for a in range(0, n, step)]


def exact(case, seed):
    kind = case["kind"]
    if kind == "encode":
        tok, cand = _explicit(case, seed)
        w, T = _weights(case, seed), case["T"]
        return torch.cat([_encode64(case, w, tok.emb[a:b].double(), tok.act[a:b], tok.time[a:b],
                                    cand[a:b].double(), tok.valid_len[a:b].long())
                          for a, b in _chunks(case, case["B"], T)])
    x = _inputs(case, seed, device="cpu" if kind == "serve" else "cuda")
    if kind == "serve":
        for s in (x.seq, x.rt):
            s.emb, s.act, s.time = s.emb.cuda(), s.act.cuda(), s.time.cuda()
        x.cands.emb = x.cands.emb.cuda()
    w = None if kind == "select" else _weights(case, seed)
    scale = STEP_I8 if case["dtype"] == "i8" else 1.0
    idx, score, out = [], [], []
    c0 = 0
    for r, n in enumerate(x.counts):
        cand = x.cands.emb[c0:c0 + n]
        c0 += n
        i, s, m = _topk64(case, x.seq, r, cand, case["k"])
        parts, ids, scs = [(x.seq, i[:, :m].flip(1), 0)], [i], [s]
        if kind == "eq2":
            keep = min(case["keep"], case["rt"])
            parts.append((x.rt, torch.arange(keep - 1, -1, -1, device="cuda").expand(n, keep), 0))
            if case["k_rt"]:
                i, s, m = _topk64(case, x.rt, r, cand, case["k_rt"], case["keep"])
                parts.append((x.rt, i[:, :m].flip(1), case["keep"]))
                ids, scs = ids + [i], scs + [s]
            if case["k_imp"]:
                i, s, m = _topk64(case, x.imp, r, cand, case["k_imp"])
                parts.append((x.imp, i[:, :m].flip(1), 0))
                ids, scs = ids + [i], scs + [s]
        elif kind != "select" and x.rt is not None:
            rows = case["rt"]
            parts.append((x.rt, torch.arange(rows - 1, -1, -1, device="cuda").expand(n, rows), 0))
        idx.append(torch.cat(ids, 1))
        score.append(torch.cat(scs, 1))
        if kind == "select":
            continue
        T = sum(p[1].shape[1] for p in parts)
        for a, b in _chunks(case, n, T):
            at = [p[1][a:b] + p[2] + int(p[0].offset[r]) for p in parts]
            emb = torch.cat([p[0].emb[j] for p, j in zip(parts, at)], 1).double() * scale
            act = torch.cat([p[0].act[j] for p, j in zip(parts, at)], 1)
            time = None
            if w.E_time is not None:
                time = torch.cat([p[0].time[j] for p, j in zip(parts, at)], 1)
            valid = torch.full((b - a,), T, device="cuda", dtype=torch.long)
            out.append(_encode64(case, w, emb, act, time, cand[a:b].double(), valid))
    if kind == "select":
        return torch.cat(idx), torch.cat(score)
    return torch.cat(idx), torch.cat(score), torch.cat(out)
