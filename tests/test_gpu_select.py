"""GPU parity of tav2_nn_select (Eq. 3) against the oracle: indices and scores
bit for bit, on the five workloads (every candidate of each) and on edge cases
(ragged, empty and short requests, k = 1 and k = K_MAX, heavy ties, padded
layout, every register-tile size of the short-row top-k, the fused search for
long rows with short rows in its batch, ties inside its survivor lists, inputs
that send it to its exhaustive fallback, and the float32 streaming top-k)."""
import numpy as np
import pytest
import torch

import oracle
import synth
from helpers import assert_select_equal, launched_sites, oracle_select, upload
from paper_2506_02267_amd import tav2 as T

pytestmark = pytest.mark.gpu


def run_select(inp, k):
    seq, _, cands = upload(inp)
    idx, score = T.nn_select(seq, cands, k)
    torch.cuda.synchronize()
    return idx, score


@pytest.mark.parametrize("cid", [1, 2, 3, 4, 5])
def test_full_workload_all_candidates(cid):
    """Every candidate of every workload (32,000 at ragged, 64,000 at stress)."""
    w = synth.WORKLOADS[cid]
    inp = synth.make_inputs(w)
    print(f"select workload {w.name}: all {inp.total} candidates", flush=True)
    idx, score = run_select(inp, w.k)
    ref_i, ref_s = oracle_select(inp, w.k)
    assert_select_equal(idx, score, ref_i, ref_s)


def custom_inputs(lengths, counts, d=64, dtype="bf16", levels=8, seed=0):
    """Requests with the given lengths and candidate counts (grid values)."""
    rng = np.random.default_rng(seed)
    w = synth.scaled(synth.SINGLE, R=len(lengths), d=d, dtype=dtype, N=max(counts) if counts else 0)
    off = np.zeros(len(lengths), dtype=np.int64)
    off[1:] = np.cumsum(lengths)[:-1]
    rows = int(np.sum(lengths))
    seq = synth.SeqBatch(emb=rng.integers(-levels, levels + 1, (rows, d)).astype(np.float32) / 8,
                         act=rng.integers(0, 8, rows).astype(np.uint8),
                         time=np.sort(rng.integers(0, 64, rows)).astype(np.uint8),
                         offset=off, length=np.asarray(lengths, dtype=np.int32))
    coff = np.zeros(len(counts) + 1, dtype=np.int64)
    coff[1:] = np.cumsum(counts)
    cand = rng.integers(-levels, levels + 1, (int(coff[-1]), d)).astype(np.float32) / 8
    return synth.Inputs(w=w, seq=seq, cand=cand, cand_offset=coff)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_ragged_short_and_empty_requests(dtype):
    inp = custom_inputs([0, 5, 300, 2000, 64], [3, 4, 7, 5, 2], dtype=dtype)
    for k in (1, 64, 301):
        idx, score = run_select(inp, k)
        ref_i, ref_s = oracle.nn_select_batch(inp.seq, inp.cand, inp.cand_offset, k)
        assert_select_equal(idx, score, ref_i, ref_s)


def test_short_rows_in_a_long_batch():
    # the batch's longest request selects the streaming top-k kernel; its shorter
    # requests take that kernel's other branches (every row kept at <= 2048 rows,
    # sampled threshold just above)
    inp = custom_inputs([5000, 100, 3000, 0, 2048, 2049], [3, 4, 5, 2, 3, 3], seed=7)
    for k in (1, 64, 301, 1024):
        idx, score = run_select(inp, k)
        ref_i, ref_s = oracle.nn_select_batch(inp.seq, inp.cand, inp.cand_offset, k)
        assert_select_equal(idx, score, ref_i, ref_s)


def test_request_without_candidates():
    inp = custom_inputs([100, 200, 300], [4, 0, 3])
    idx, score = run_select(inp, 16)
    ref_i, ref_s = oracle.nn_select_batch(inp.seq, inp.cand, inp.cand_offset, 16)
    assert_select_equal(idx, score, ref_i, ref_s)


@pytest.mark.parametrize("d", [48, 32])
@pytest.mark.parametrize("L", [100, 1500, 3000, 6000, 16384, 20000, 32768])
def test_each_register_tile_size(L, d):
    """The top-k over score rows in memory (up to 4096 rows) and the search with scores on
    chip; up to 8192 rows of d 32, the search in one launch."""
    inp = custom_inputs([L], [9], d=d, levels=2, seed=L)
    k = min(1024, L)
    idx, score = run_select(inp, k)
    seq, _, cands = upload(inp)
    sites = launched_sites(lambda: T.nn_select(seq, cands, k))
    assert ("nn_resident" in sites) == (d == 32 and L <= 8192)
    assert ("topk" in sites) == (L <= 4096 and d == 48) and ("nn_select" in sites) == (L > 4096 and "nn_resident" not in sites)
    ref_i, ref_s = oracle.nn_select_batch(inp.seq, inp.cand, inp.cand_offset, k)
    assert_select_equal(idx, score, ref_i, ref_s)


def test_heavy_ties_and_k_max():
    inp = custom_inputs([4096, 3000], [6, 6], d=16, levels=1, seed=3)   # values in {-1/8, 0, 1/8}
    for k in (1, 2, 1024):
        idx, score = run_select(inp, k)
        ref_i, ref_s = oracle.nn_select_batch(inp.seq, inp.cand, inp.cand_offset, k)
        assert_select_equal(idx, score, ref_i, ref_s)


@pytest.mark.parametrize("k", [1, 256, 1024])
def test_sampled_threshold_with_tied_rows(k):
    # long rows (the top-k takes its threshold from a sample of the keys): every
    # embedding row appears three times in a row, so ties fall inside the
    # compacted candidate set and are resolved by row in the radix select
    inp = custom_inputs([16384, 9000], [5, 4], d=64, levels=8, seed=11)
    for r0, n in zip(inp.seq.offset, inp.seq.length):
        e = inp.seq.emb[r0:r0 + n]
        e[:] = np.repeat(e[0::3], 3, axis=0)[:n]
    idx, score = run_select(inp, k)
    ref_i, ref_s = oracle.nn_select_batch(inp.seq, inp.cand, inp.cand_offset, k)
    assert_select_equal(idx, score, ref_i, ref_s)


@pytest.mark.parametrize("case", ["all_equal", "sample_misses_top"])
def test_sampled_threshold_falls_back(case):
    # inputs for which the sample gives no usable threshold, so every candidate
    # takes the exhaustive fallback: all scores equal (16384 survivors, far above
    # the list capacity), or the largest scores only on rows the sample never
    # looks at (the sample of a 16384-row request is the 32-row blocks starting at
    # multiples of 512: big scores on rows = 2 mod 4 outside those blocks, about
    # 3600 of them, again above the capacity)
    inp = custom_inputs([16384], [4], d=32, levels=8, seed=5)
    e = inp.seq.emb
    if case == "all_equal":
        e[:] = e[0]
    else:
        rows = np.arange(e.shape[0])
        big = (rows % 4 == 2) & (rows % 512 >= 64)
        e[:] = -np.abs(e)
        e[big] = np.abs(e[big]) + 1.0
        inp.cand[:] = np.abs(inp.cand) + 0.125
    idx, score = run_select(inp, 512)
    ref_i, ref_s = oracle.nn_select_batch(inp.seq, inp.cand, inp.cand_offset, 512)
    assert_select_equal(idx, score, ref_i, ref_s)


@pytest.mark.parametrize("lengths", [[4096, 300], [4097, 5], [6000, 4000, 0, 1]])
def test_materialised_and_fused_paths_meet(lengths):
    # the longest request decides the path: at most 4096 rows keep the score rows
    # in memory (register top-k), beyond it the scores stay on chip
    inp = custom_inputs(lengths, [3] * len(lengths), d=48, seed=sum(lengths))
    for k in (1, 100, 1024):
        idx, score = run_select(inp, k)
        ref_i, ref_s = oracle.nn_select_batch(inp.seq, inp.cand, inp.cand_offset, k)
        assert_select_equal(idx, score, ref_i, ref_s)


def test_many_candidate_tiles_with_a_ragged_tail():
    # 3 requests x 300 candidates: three 128-candidate tiles, the last one partial
    inp = custom_inputs([9000, 16384, 5000], [300, 300, 300], d=64, seed=41)
    idx, score = run_select(inp, 256)
    ref_i, ref_s = oracle_select(inp, 256)
    assert_select_equal(idx, score, ref_i, ref_s)


@pytest.mark.parametrize("L", [5000, 20000])
def test_f32_long_rows_stream_topk(L):
    # float32 sequences keep the materialised score rows at every length: rows of
    # more than 4096 keys take the streaming top-k
    inp = custom_inputs([L, 700], [5, 3], d=32, dtype="f32", seed=L + 1)
    for k in (1, 256, 1024):
        idx, score = run_select(inp, k)
        ref_i, ref_s = oracle.nn_select_batch(inp.seq, inp.cand, inp.cand_offset, k)
        assert_select_equal(idx, score, ref_i, ref_s)


def test_zero_scores_are_positive_zero():
    inp = custom_inputs([50], [3], d=16)
    inp.seq.emb[:] = 0.0
    inp.cand[0] = -1.0
    idx, score = run_select(inp, 10)
    s = score.cpu().numpy()
    assert np.all(s == 0) and not np.any(np.signbit(s))
    np.testing.assert_array_equal(idx.cpu().numpy(), np.tile(np.arange(10), (3, 1)))


def test_padded_layout_equals_packed_and_batch_equals_single():
    w = synth.scaled(synth.RAGGED, R=5, L_range=(700, 3000), N=11, k=128)
    inp = synth.make_inputs(w)
    idx, score = run_select(inp, 128)
    padded = synth.Inputs(w=w, seq=synth.to_padded(inp.seq, pad_to=3072), cand=inp.cand,
                          cand_offset=inp.cand_offset)
    i2, s2 = run_select(padded, 128)
    assert torch.equal(idx, i2) and torch.equal(score.view(torch.int32), s2.view(torch.int32))
    for r in range(w.R):
        a, b = int(inp.cand_offset[r]), int(inp.cand_offset[r + 1])
        one = synth.Inputs(w=w, seq=synth.SeqBatch(
            emb=inp.seq.emb[inp.seq.rows(r)], act=inp.seq.act[inp.seq.rows(r)],
            time=inp.seq.time[inp.seq.rows(r)], offset=np.zeros(1, np.int64),
            length=inp.seq.length[r:r + 1].copy()), cand=inp.cand[a:b],
            cand_offset=np.array([0, b - a], dtype=np.int64))
        i1, s1 = run_select(one, 128)
        assert torch.equal(i1, idx[a:b]) and torch.equal(s1, score[a:b])


def test_repeated_runs_and_streams_are_bitwise_identical():
    w = synth.scaled(synth.STRESS, R=2, N=300, k=512)
    inp = synth.make_inputs(w)
    seq, _, cands = upload(inp)
    outs = []
    for i in range(3):
        st = torch.cuda.Stream()
        with torch.cuda.stream(st):
            outs.append(T.nn_select(seq, cands, 512, stream=st))
        st.synchronize()
    for i, s in outs[1:]:
        assert torch.equal(i, outs[0][0]) and torch.equal(s, outs[0][1])


@pytest.mark.parametrize("N,L,k", [
    (3, 1, 1), (3, 40, 64), (5, 1020, 256), (5, 1021, 256), (5, 1021, 257), (5, 1024, 1000),
    (5, 1025, 64), (600, 1025, 64), (5, 2044, 512), (5, 2045, 512), (600, 2049, 700),
    (5, 4096, 1024), (600, 4096, 256)])
@pytest.mark.parametrize("ties", ["none", "some", "all"])
def test_short_row_bins(N, L, k, ties):
    """Rows of up to 4096 keys, placed by bins: every workgroup shape, key counts around
    what a thread's four rows cover, k around the thread count and above the row; scores
    with few ties, with a third of the rows equal (a bin past its limit), and all equal
    (the bitwise search)."""
    print(f"short rows N={N} L={L} k={k} ties={ties}", flush=True)
    w = synth.scaled(synth.SINGLE, L=L, N=N, k=k, d=64)
    inp = synth.make_inputs(w, seed=L + k)
    if ties != "none":
        n = L if ties == "all" else max(1, L // 3)
        pick = np.random.default_rng(L).permutation(L)[:n]
        inp.seq.emb[pick] = inp.seq.emb[0]
    seq, _, cands = upload(inp)
    idx, score = T.nn_select(seq, cands, k)
    torch.cuda.synchronize()
    ids = np.unique(np.r_[np.arange(min(N, 8)), np.arange(0, N, 61), N - 1])
    ref_i, ref_s = oracle_select(inp, k, ids=ids)
    assert_select_equal(idx, score, ref_i, ref_s, ids=ids)


@pytest.mark.parametrize("dtype", ["bf16", "i8"])
@pytest.mark.parametrize("copies,k", [(300, 64), (700, 64), (700, 1024)])
def test_long_row_bins_with_equal_scores(dtype, copies, k):
    """Long rows whose best survivors include many equal scores: within the bins' limit
    (300 copies of one row) and past it (700: the radix select)."""
    print(f"long rows {dtype} copies={copies} k={k}", flush=True)
    base = synth.SELECT_I8 if dtype == "i8" else synth.SINGLE
    w = synth.scaled(base, L=9000, N=6, k=k, d=64, tie_frac=0.0)
    inp = synth.make_inputs(w, seed=copies)
    rows = np.random.default_rng(copies).permutation(9000)[:copies]
    c0 = inp.cand[0]
    best = int(np.argmax(inp.seq.emb.astype(np.float64) @ c0))
    inp.seq.emb[rows] = inp.seq.emb[best]
    seq, _, cands = upload(inp)
    idx, score = T.nn_select(seq, cands, k)
    torch.cuda.synchronize()
    ref_i, ref_s = oracle_select(inp, k)
    assert_select_equal(idx, score, ref_i, ref_s)


@pytest.mark.parametrize("dtype,d", [("i8", 32), ("bf16", 32), ("i8", 64)])
@pytest.mark.parametrize("L,k", [(1, 4), (1023, 1024), (2049, 700), (4096, 1024), (8192, 33),
                                 (16384, 256)])
@pytest.mark.parametrize("ties", ["none", "some", "all"])
def test_resident_rows(dtype, d, L, k, ties):
    """The search with every product in registers: the edges of its rows per thread, fewer
    rows than places, a ragged second request, equal scores past the bins' limit."""
    print(f"resident {dtype} d={d} L={L} k={k} {ties}", flush=True)
    base = synth.SELECT_I8 if dtype == "i8" else synth.SINGLE
    w = synth.scaled(base, R=3, L=L, N=4, k=k, d=d, tie_frac=0.0)
    inp = synth.make_inputs(w, seed=L + d)
    inp.seq.length[1:] = [L // 3, 0]
    if ties != "none":
        n = min(L, 900) if ties == "some" else L
        rows = np.random.default_rng(L).permutation(L)[:n]
        best = int(np.argmax(inp.seq.emb[:L].astype(np.float64) @ inp.cand[0]))
        inp.seq.emb[rows] = inp.seq.emb[best]
    seq, _, cands = upload(inp)
    idx, score = T.nn_select(seq, cands, k)
    torch.cuda.synchronize()
    ref_i, ref_s = oracle_select(inp, k)
    assert_select_equal(idx, score, ref_i, ref_s)


@pytest.mark.parametrize("dtype,d", [("i8", 32), ("bf16", 32), ("i8", 64)])
@pytest.mark.parametrize("L", [90, 700, 3000, 5000, 8192])
def test_resident_equals_the_general_search(dtype, d, L):
    """The same candidates alone (every product in registers) and three times over (too
    many for that): bit for bit the same, also for infinite, huge, tiny, zero and
    not-a-number candidates, over requests with an all-zero row each (int8: its score is 0
    whatever the candidate)."""
    print(f"resident against general {dtype} d={d} L={L}", flush=True)
    g = torch.Generator().manual_seed(L + d)
    n, k = 200, 100
    if dtype == "i8":
        emb = torch.randint(-127, 128, (2 * L, d), generator=g, dtype=torch.int8)
        emb[[5, L + 5]] = 0                       # a row without a norm in each request
    else:
        emb = torch.randn(2 * L, d, generator=g).bfloat16()
    cand = torch.randn(n, d, generator=g)
    cand[0] = 0.0
    cand[1, 3] = float("inf")
    cand[2, 4] = -float("inf")
    cand[3] *= 1e38
    cand[4] *= 1e-39
    cand[5, 0] = float("nan")
    cand[6, :2] = torch.tensor([float("inf"), -float("inf")])
    cand = cand.bfloat16().cuda()
    seq = T.DeviceSeq(emb=emb.cuda(), act=torch.zeros(2 * L, dtype=torch.uint8, device="cuda"), time=None,
                      offset=torch.tensor([L, 0], device="cuda"),
                      length=torch.tensor([L, L - 37], dtype=torch.int32, device="cuda"), max_len=L,
                      dtype=T.I8 if dtype == "i8" else T.BF16)

    def search(c, per):
        off = torch.tensor([0, per, 2 * per], device="cuda")
        i, s = T.nn_select(seq, T.DeviceCands(emb=c, offset=off, max_count=per), k)
        torch.cuda.synchronize()
        return i.cpu(), s.cpu().view(torch.int32)

    h = n // 2
    i1, s1 = search(cand, h)
    big = torch.cat([cand[:h]] * 3 + [cand[h:]] * 3)
    i3, s3 = search(big, 3 * h)
    for r in range(2):
        for rep in range(3):
            a, b = slice(r * h, r * h + h), slice((3 * r + rep) * h, (3 * r + rep + 1) * h)
            assert torch.equal(i1[a], i3[b])
            assert torch.equal(s1[a], s3[b])
    if dtype == "i8":
        # request 0's seven extreme candidates: wherever its zero row was selected, it scored 0
        hit = (i1[:7] == 5)
        assert torch.all(s1[:7][hit] == 0)
        if k >= L:
            assert torch.all(hit.any(1))


@pytest.mark.parametrize("n", [1, 31, 33])
@pytest.mark.parametrize("d", [16, 240, 256, 272, 400, 512])
def test_direct_scores_of_wide_rows(d, n):
    """Few score tiles: products straight from memory, 16 k-blocks in flight (all of them up
    to d 256; past it, partly and wholly refilled).  Against the oracle, and the same
    candidates among enough others for the staged kernel: the same bits."""
    print(f"direct scores d={d} n={n}", flush=True)
    lengths = [300, 65, 0, 1]
    assert sum(-(-max(lengths) // 256) * -(-c // 128) for c in [n] * 4) * d < 8192
    inp = custom_inputs(lengths, [n] * 4, d=d, seed=d + n)
    ref_i, ref_s = oracle.nn_select_batch(inp.seq, inp.cand, inp.cand_offset, 50)
    idx, score = run_select(inp, 50)
    assert_select_equal(idx, score, ref_i, ref_s)
    # request 0 (2 tiles of 256 rows) alone, its candidates repeated past 8192 / d tiles
    rep = -(-(128 * (4096 // d + 2)) // n)
    one = synth.Inputs(w=inp.w, seq=synth.SeqBatch(emb=inp.seq.emb[:300], act=inp.seq.act[:300],
                       time=inp.seq.time[:300], offset=np.zeros(1, np.int64),
                       length=inp.seq.length[:1].copy()), cand=np.tile(inp.cand[:n], (rep, 1)),
                       cand_offset=np.array([0, n * rep], np.int64))
    i2, s2 = run_select(one, 50)
    for at in (0, n * (rep // 2), n * (rep - 1)):
        assert torch.equal(i2[at:at + n], idx[:n])
        assert torch.equal(s2[at:at + n].view(torch.int32), score[:n].view(torch.int32))


def ranged_inputs(dist, L, N, d, dtype, seed):
    """One request of L rows whose score against candidate 0 is the value drawn from `dist`
    (exact in fp32: two columns of at most 17 bits together), against the others that value
    times a power of two and a sign."""
    rng = np.random.default_rng(seed)
    a = {"both_signs": rng.normal(size=L), "negative": -1 - rng.random(L), "narrow": 1 + rng.random(L) / 128,
         "outlier": rng.normal(size=L), "octaves": rng.normal(size=L),
         "two_values": np.where(rng.random(L) < 0.3, 3.0, -2.0)}[dist]
    hi = np.round(a * 16) / 16
    lo = np.round(np.clip(a - hi, -1 / 32, 1 / 32) * 2 ** 13) / 2 ** 13
    if dist == "outlier":
        hi[L // 2], lo[L // 2] = 2.0 ** 28, 0
        hi[L // 3], lo[L // 3] = -2.0 ** 28, 0
    elif dist == "octaves":
        hi, lo = np.sign(a) * 2.0 ** rng.integers(-20, 20, L), np.zeros(L)
    elif dist == "two_values":
        lo[:] = 0
    w = synth.scaled(synth.SINGLE, R=1, d=d, dtype=dtype, N=N)
    emb = np.zeros((L, d), np.float32)
    emb[:, 0], emb[:, 1] = hi, lo
    cand = np.zeros((N, d), np.float32)
    cand[:, :2] = (np.where(np.arange(N) % 3 == 2, -1, 1) * 2.0 ** (np.arange(N) % 7 - 3 * (np.arange(N) > 0)))[:, None]
    cand[0, :2] = 1
    seq = synth.SeqBatch(emb=emb, act=rng.integers(0, 8, L).astype(np.uint8),
                         time=np.sort(rng.integers(0, 64, L)).astype(np.uint8), offset=np.zeros(1, np.int64),
                         length=np.array([L], np.int32))
    return synth.Inputs(w=w, seq=seq, cand=cand, cand_offset=np.array([0, N], np.int64))


@pytest.mark.parametrize("dist", ["both_signs", "negative", "narrow", "outlier", "octaves", "two_values"])
@pytest.mark.parametrize("dtype,d,L,N", [
    ("bf16", 16, 900, 3), ("bf16", 16, 2000, 4), ("bf16", 16, 2000, 600), ("bf16", 16, 4096, 5),
    ("bf16", 16, 4000, 600), ("f32", 16, 3000, 4),                     # score rows in memory
    ("bf16", 32, 900, 3), ("bf16", 32, 4000, 5), ("bf16", 32, 8192, 4),   # one launch
    ("bf16", 48, 9000, 4)])                                            # scores on chip
def test_score_ranges(dist, dtype, d, L, N):
    """Placement by bins over ranges of scores that one set of equal bins does not resolve:
    both signs (four bins to a factor of two), one value far out on either side, 40 powers of
    two, two values; and narrow ones.  k from one row to nearly every row."""
    print(f"score ranges {dist} {dtype} d={d} L={L} N={N}", flush=True)
    inp = ranged_inputs(dist, L, N, d, dtype, seed=L + N)
    ids = np.arange(N) if N <= 8 else np.unique(np.r_[0:8, np.arange(0, N, 97), N - 1])
    for k in sorted({1, 64, 256, 257, min(L - 1, 1000)}):
        idx, score = run_select(inp, k)
        ref_i, ref_s = oracle_select(inp, k, ids=ids)
        assert_select_equal(idx, score, ref_i, ref_s, ids=ids)


@pytest.mark.parametrize("dtype,d,L,N", [
    ("bf16", 16, 700, 4), ("bf16", 16, 2000, 600), ("bf16", 16, 4000, 3),   # score rows in memory
    ("f32", 16, 1100, 3), ("bf16", 32, 1500, 4)])                           # (the last: one launch)
@pytest.mark.parametrize("group", [31, 33, 127, 129, 255, 513, 650])
def test_equal_scores_at_the_last_place(group, dtype, d, L, N):
    """A group of rows of one score around the k-th place, of sizes about those at which
    placement by bins hands over (32, 128, 512), with k at its ends, inside it and where the
    group is about half of k; the scores around it are all different."""
    print(f"equal group {group} {dtype} d={d} L={L} N={N}", flush=True)
    inp = ranged_inputs("both_signs", L, N, d, dtype, seed=group)
    rng = np.random.default_rng(group)
    e = inp.seq.emb
    e[rng.choice(L, group, replace=False), :2] = (1.0, 2.0 ** -13)
    above = int((e[:, :2].sum(1) > 1.0 + 2.0 ** -13).sum())
    ids = np.arange(N) if N <= 8 else np.unique(np.r_[0:8, N - 1])
    for k in sorted({above, above + 1, above + group // 2, above + group, above + group + 1, 2 * group}):
        if not 1 <= k <= min(L, 1024):
            continue
        idx, score = run_select(inp, k)
        ref_i, ref_s = oracle_select(inp, k, ids=ids)
        assert_select_equal(idx, score, ref_i, ref_s, ids=ids)
