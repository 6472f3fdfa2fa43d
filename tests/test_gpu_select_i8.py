"""GPU parity of tav2_nn_select over int8 sequence codes, whose rows are
dequantised and L2-normalised inside the score kernel (Sec. 3.4.2, fused
sequence dequantisation), against the oracle: indices and scores bit for bit
(the dot products and sums of squares are exact, the square root and the
division rounded to nearest on both sides).  Cases: the 16k-row single-request
workload with all of its candidates (the launch the benchmark times), ragged
batches over several candidate tiles with ragged tails, k past the row count,
the narrowest and widest embeddings, all-zero and duplicated rows.  Where a case is meant
for one of the search's paths (score rows in memory, scores on chip, one launch), the path
taken is checked."""
import numpy as np
import pytest
import torch

import oracle
import synth
from helpers import assert_select_equal, launched_sites, upload
from paper_2506_02267_amd import tav2 as T

pytestmark = pytest.mark.gpu


# the sites of each path
PATHS = {"memory": {"score_i8", "topk"},
         "chip": {"nn_sample", "nn_threshold", "nn_filter", "nn_select", "nn_fallback"},
         "one_launch": {"nn_resident"}}


def check_inputs(inp, k, path=None):
    seq, _, cands = upload(inp)
    assert seq.emb.dtype == torch.int8 and cands.emb.dtype == torch.bfloat16
    idx, score = T.nn_select(seq, cands, k)
    torch.cuda.synchronize()
    if path:
        assert launched_sites(lambda: T.nn_select(seq, cands, k, idx, score)) == PATHS[path]
    ref_i, ref_s = oracle.nn_select_batch(inp.seq, inp.cand, inp.cand_offset, k)
    assert_select_equal(idx, score, ref_i, ref_s)


def check(w, seed=None, zero_every=0, path=None):
    inp = synth.make_inputs(w, seed=seed)
    if zero_every:
        inp.seq.emb[::zero_every] = 0
    print(f"select_i8 R={w.R} L={w.L or w.L_range} d={w.d} N={w.N} k={w.k} {path}", flush=True)
    check_inputs(inp, w.k, path)


def test_full_size_all_candidates():
    check(synth.SELECT_I8, zero_every=1021)


def test_several_long_requests_large_k():
    """Four 16k-row requests with 2000 candidates each and k = 512."""
    w = synth.scaled(synth.SELECT_I8, R=4, N=2000, k=512)
    check(w, seed=25, zero_every=2003)


@pytest.mark.parametrize("d,N,path", [(48, 5, "chip"), (32, 300, "chip"), (32, 5, "one_launch")])
@pytest.mark.parametrize("case", ["all_equal", "sample_misses_top"])
def test_fused_search_falls_back(case, d, N, path):
    """Inputs whose sample gives no usable threshold: every candidate takes the
    exhaustive fallback, whose recomputed scores must match the oracle's (and the same
    inputs where the search in one launch takes them)."""
    w = synth.scaled(synth.SELECT_I8, d=d, N=N, k=512)
    print(f"select_i8 fallback {case} d={d} N={N} {path}", flush=True)
    inp = synth.make_inputs(w, seed=26)
    e = inp.seq.emb
    if case == "all_equal":
        e[:] = e[7]
    else:
        rows = np.arange(e.shape[0])
        big = (rows % 4 == 2) & (rows % 512 >= 64)
        e[:] = -np.abs(e)
        e[big] = np.abs(e[big])
        inp.cand[:] = np.abs(inp.cand) + 0.125
    check_inputs(inp, w.k, path)


@pytest.mark.parametrize("d,R,Lr,N,k,seed,path", [
    # 2 candidate tiles, ragged tails, short rows: wide codes, or more candidates than the
    # search in one launch takes; and few enough
    (128, 3, (1, 700), 130, 64, 21, "memory"),
    (32, 3, (1, 700), 200, 64, 21, "memory"),
    (32, 3, (1, 700), 130, 64, 21, "one_launch"),
    (256, 2, (300, 2100), 40, 256, 22, "memory"),   # wide codes, k above some row counts
    (16, 2, (37, 37), 1, 100, 23, "memory"),        # narrowest rows, k > L (padding)
    (512, 1, (5000, 5000), 9, 33, 24, "chip"),      # widest rows, long rows
    # longest request 4096: score rows in memory; 4097: scores on chip, short rows inside
    (128, 3, (4096, 4096), 50, 128, 27, "memory"),
    (128, 3, (4097, 4097), 50, 128, 28, "chip"),
    (64, 3, (4000, 4096), 100, 128, 27, "memory"),
    (64, 3, (4000, 4096), 50, 128, 27, "one_launch"),
    (64, 3, (4000, 4097), 50, 128, 28, "one_launch"),
])
def test_ragged_batches(d, R, Lr, N, k, seed, path):
    w = synth.scaled(synth.SELECT_I8, R=R, L=None, L_range=Lr, d=d, N=N, k=k, tie_frac=0.05)
    check(w, seed=seed, zero_every=13, path=path)


def test_short_rows_inside_a_long_batch():
    """A request of 4097 rows decides for scores on chip; shorter ones go with it."""
    w = synth.scaled(synth.SELECT_I8, R=3, L=4097, N=50, d=128, k=128, tie_frac=0.05)
    inp = synth.make_inputs(w, seed=29)
    inp.seq.length[:] = [4097, 4096, 700]
    inp.seq.emb[::13] = 0
    print("select_i8 short rows inside a long batch", flush=True)
    check_inputs(inp, w.k, "chip")
