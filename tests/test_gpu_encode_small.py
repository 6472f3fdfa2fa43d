"""GPU parity of the d_model-64 encoder (the paper's production shape, Sec.
3.2.2, run as one kernel with every weight on chip, Sec. 3.4.2) against the
oracle: explicit tokens at 64 to 2048 positions with ragged valid lengths, one
and two heads, one and two layers, the causal and the unmasked mode, and the
whole select + encode path on the paper workload.  Pooled outputs within
max-abs 2e-2 (bf16 operands, fp32 accumulation)."""
import numpy as np
import pytest
import torch

import synth
from helpers import (BF16_TOL, max_abs, oracle_encode_tokens, upload_tokens)
from test_gpu_encode import check_workload
from paper_2506_02267_amd import tav2 as T

pytestmark = pytest.mark.gpu


def weights_for(T_, d=32, n_heads=1, d_ffn=32, n_layers=2, has_time=True, seed=None):
    """Encoder weights of the paper workload's shape, sized for T_ positions."""
    w = synth.scaled(synth.PAPER, k=T_, rt_len=0, d=d, n_heads=n_heads, d_ffn=d_ffn,
                     n_layers=n_layers, has_time=has_time)
    return synth.make_weights(w, seed=seed)


def ragged_lengths(total, T_, rng):
    """Valid lengths over [0, T_] with the edges of 64-position steps (63, 64, 65,
    127, 128, 129, ...; among them those of the encoder's tiles of 16 tokens, its pairs of
    32 keys and its blocks of up to 192 positions) and the extremes (0, 1, T_) present."""
    edges = [0, 1, T_]
    for e in range(64, T_ + 1, 64):
        edges += [e - 1, e, e + 1]
    edges = [e for e in edges if 0 <= e <= T_]
    vl = rng.integers(0, T_ + 1, size=total)
    vl[:len(edges)] = edges[:total]
    return vl.astype(np.int32)


def run_and_check(tb, W, flags=T.MASK_CAUSAL, ids=None, tol=BF16_TOL):
    tok, cand = upload_tokens(tb)
    out = T.encode(tok, cand, T.DeviceWeights(W), flags=flags)
    torch.cuda.synchronize()
    ref = oracle_encode_tokens(tb, W, ids=ids, causal=flags == T.MASK_CAUSAL)
    err = max_abs(out, ref, ids=ids)
    print(f"  max abs error {err:.3e} (bound {tol})", flush=True)
    assert err <= tol
    if ids is None:
        empty = np.flatnonzero(tb.valid_len == 0)
        assert torch.all(out[torch.from_numpy(empty).to(out.device)] == 0)
    return out


@pytest.mark.parametrize("T_,total", [(64, 48), (192, 64), (256, 40), (1000, 12), (2048, 8)])
def test_paper_shape_ragged(T_, total):
    """d 32, one head, FFN 32, two layers; one block of up to 192 positions, and up to
    eleven, every edge of 64 among the valid lengths."""
    print(f"encode_small T={T_} total={total}", flush=True)
    rng = np.random.default_rng(T_)
    tb = synth.make_tokens(total, T_, 32, seed=T_, valid_len=ragged_lengths(total, T_, rng))
    run_and_check(tb, weights_for(T_))


@pytest.mark.parametrize("case", ["two_heads", "one_layer_ffn96", "no_time_d64",
                                  "two_heads_one_layer_d256"])
def test_other_shapes(case):
    """Two heads of 32; an FFN wider than 64 (its hidden rows in a region of their
    own); d 64 without the time feature; d 256."""
    T_ = 300
    kw = {"two_heads": dict(n_heads=2),
          "one_layer_ffn96": dict(n_layers=1, d_ffn=96),
          "no_time_d64": dict(d=64, has_time=False),
          "two_heads_one_layer_d256": dict(n_heads=2, n_layers=1, d=256)}[case]
    print(f"encode_small {case}", flush=True)
    rng = np.random.default_rng(7)
    d = kw.get("d", 32)
    tb = synth.make_tokens(24, T_, d, has_time=kw.get("has_time", True), seed=11,
                           valid_len=ragged_lengths(24, T_, rng))
    run_and_check(tb, weights_for(T_, **kw))


def test_many_candidates_persistent_loop():
    """2,500 candidates at 192 positions: about ten candidates per workgroup, one after the
    other over the same keys and values in LDS; every 16th candidate and the last checked."""
    total, T_ = 2500, 192
    print(f"encode_small persistent total={total}", flush=True)
    rng = np.random.default_rng(3)
    tb = synth.make_tokens(total, T_, 32, seed=5, valid_len=rng.integers(1, T_ + 1, total))
    ids = np.unique(np.r_[np.arange(0, total, 16), total - 1])
    run_and_check(tb, weights_for(T_), ids=ids)


@pytest.mark.parametrize("n_heads", [1, 2])
def test_unmasked_one_block(n_heads):
    """TAV2_MASK_NONE (up to 64 positions): every valid token sees every valid
    token, padding excluded."""
    print(f"encode_small unmasked heads={n_heads}", flush=True)
    rng = np.random.default_rng(n_heads)
    tb = synth.make_tokens(40, 64, 32, seed=21, valid_len=ragged_lengths(40, 64, rng))
    run_and_check(tb, weights_for(64, n_heads=n_heads), flags=T.MASK_NONE)


def test_unmasked_past_one_block_is_unsupported():
    tb = synth.make_tokens(2, 65, 32, seed=1)
    tok, cand = upload_tokens(tb)
    with pytest.raises(T.Tav2Error) as e:
        T.encode(tok, cand, T.DeviceWeights(weights_for(65)), flags=T.MASK_NONE)
    assert e.value.status == -4   # TAV2_ERR_UNSUPPORTED


def test_paper_workload_select_encode():
    """The whole path on the paper workload: NN top-128 over a 16k lifelong
    sequence of 32-d embeddings plus 64 real-time actions (192 positions), 256
    candidates, every candidate checked."""
    check_workload(synth.PAPER)


@pytest.mark.parametrize("kw", [dict(), dict(n_heads=2, d=64)])
def test_packed_weights_equal_unpacked(kw):
    """Weights packed once (as operand fragments, copied into LDS as they stand)
    give the outputs of the weights read as given, bit for bit."""
    d = kw.get("d", 32)
    tb = synth.make_tokens(64, 192, d, seed=4, valid_len=np.random.default_rng(4).integers(0, 193, 64))
    tok, cand = upload_tokens(tb)
    W = weights_for(192, **kw)
    a = T.encode(tok, cand, T.DeviceWeights(W))
    b = T.encode(tok, cand, T.DeviceWeights(W, pack=True))
    torch.cuda.synchronize()
    assert torch.equal(a, b)


def test_int8_code_tokens():
    """Explicit tokens stored as int8 codes (Sec. 3.2.1): the encoder takes their
    dequantised values (the oracle: codes x 0.65 / 127 in float64)."""
    rng = np.random.default_rng(8)
    tb = synth.make_tokens(48, 192, 32, seed=8, valid_len=ragged_lengths(48, 192, rng), codes=True)
    run_and_check(tb, weights_for(192))


def test_paper_int8_workload_select_encode():
    """The paper's production path on its int8 storage: NN top-128 with fused
    dequantisation and L2 normalisation over 16k codes, the 64 real-time code
    rows kept, the encoder on the dequantised rows; every candidate checked."""
    check_workload(synth.PAPER_I8)


def test_repeated_runs_bitwise_identical():
    tb = synth.make_tokens(300, 192, 32, seed=2)
    tok, cand = upload_tokens(tb)
    dw = T.DeviceWeights(weights_for(192))
    first = T.encode(tok, cand, dw).clone()
    for _ in range(2):
        assert torch.equal(T.encode(tok, cand, dw), first)


@pytest.mark.parametrize("T_,total,kw", [
    (1, 9, {}), (15, 600, {}), (16, 300, dict(n_heads=2)), (17, 520, {}), (33, 300, {}),
    (128, 270, {}), (129, 30, {}), (191, 30, dict(n_heads=2)), (193, 30, {}), (257, 20, {}),
    (385, 12, dict(d=64)), (577, 8, dict(n_layers=1, d_ffn=160)),
    (200, 20, dict(n_layers=1, d=256)), (100, 20, dict(n_layers=1, d_ffn=96, d=128)),
    # what of W_in and W_pool is held next to 6 key pairs; a candidate's projection shared by
    # its waves: one to twelve of them, several candidates side by side, several blocks
    (192, 30, dict(d=64)), (180, 300, dict(n_layers=1, d=96)), (192, 30, dict(n_layers=1, d=256)),
    (16, 600, dict(n_layers=1, d=256)), (40, 600, dict(n_layers=1, d=160, n_heads=2)),
    (129, 300, dict(n_layers=1, d=224)), (400, 270, dict(n_layers=1, d=192, n_heads=2)),
    (300, 9, dict(n_layers=1, d=128))])
def test_tile_and_block_edges(T_, total, kw):
    """Waves of 16 tokens, pairs of 32 keys, one block of up to 192 positions or several
    of about one size, several short candidates to a workgroup (more than one per CU),
    and weights that leave no room for all of W_in and W_pool on chip; packed weights too."""
    print(f"encode_small edges T={T_} total={total} {kw}", flush=True)
    rng = np.random.default_rng(T_)
    edges = [e for e in (0, 1, 15, 16, 17, 31, 32, 33, T_ - 1, T_) if 0 <= e <= T_]
    vl = rng.integers(0, T_ + 1, size=total)
    vl[:min(total, len(edges))] = edges[:total]
    tb = synth.make_tokens(total, T_, kw.get("d", 32), seed=T_, valid_len=vl.astype(np.int32))
    ids = np.unique(np.r_[np.arange(min(total, 24)), np.arange(0, total, 17), total - 1])
    W = weights_for(T_, **kw)
    out = run_and_check(tb, W, ids=ids)
    tok, cand = upload_tokens(tb)
    assert torch.equal(T.encode(tok, cand, T.DeviceWeights(W, pack=True)), out)


def test_tables_aligned_to_8_bytes_only():
    """The side tables need 8-byte alignment only."""
    tb = synth.make_tokens(40, 100, 32, seed=3)
    tok, cand = upload_tokens(tb)
    dw = T.DeviceWeights(weights_for(100), pack=True)
    ref = T.encode(tok, cand, dw).clone()
    kept = []
    for name in ("E_act", "E_time"):
        src = next(t for t in dw.keep if t.data_ptr() == getattr(dw.s, name))
        buf = torch.empty(src.numel() + 4, dtype=src.dtype, device=src.device)
        buf[4:].copy_(src.reshape(-1))
        kept.append(buf)
        setattr(dw.s, name, buf.data_ptr() + 8)
    assert torch.equal(T.encode(tok, cand, dw), ref)


def one_value_inputs(T_, n_heads, total=3):
    """Tokens and weights (one layer, d 64) whose last query's attention output is one
    value V over the softmax's sum: its own key scores 0 (weight exactly 1), every other key
    has V = 0 and a weight just under the midpoint of 1/2 and the next bf16, 0.4 % above
    what it rounds to.  Returns the batch, the weights and the exact last rows (float64, the
    attention output rounded once to bf16, as the kernel's output projection takes it)."""
    dm, dh = 64, 64 // n_heads
    W = weights_for(T_, d=dm, n_heads=n_heads, n_layers=1)
    for a in (W.b_in, W.E_act, W.E_time, W.E_pos, W.b_pool):
        a[:] = 0
    W.W_in[:] = np.concatenate([np.eye(dm), np.zeros((dm, dm))], axis=1)
    L = W.layers[0]
    for a in (L.W_qkv, L.b_qkv, L.b_o, L.W_1, L.b_1, L.W_2, L.b_2, L.ln1_b, L.ln2_b):
        a[:] = 0
    L.ln1_g[:] = L.ln2_g[:] = 1
    L.W_o[:] = np.eye(dm)
    bf = synth.round_to_bf16
    # score of the other keys: x[1] + x[2] through the head's first two dimensions
    t = np.log(0.5 + 2.0 ** -9 - 2.0 ** -13) * np.sqrt(dh)
    hi = float(bf(np.array([t], np.float32))[0])
    lo = float(bf(np.array([t - hi], np.float32))[0])
    p = np.exp((hi + lo) / np.sqrt(dh))
    for h in range(n_heads):
        L.b_qkv[h * dh:h * dh + 2] = 1
        L.W_qkv[dm + h * dh, 1] = L.W_qkv[dm + h * dh + 1, 2] = 1
    vl = np.array([T_, T_ - 1, T_ - 2])[:total].astype(np.int32)
    emb = np.zeros((total, T_, dm), np.float32)
    emb[:, :, 1], emb[:, :, 2] = hi, lo
    # V: of the bf16 between 1.5 l and 1.97 l the one whose V / l lies nearest to a bf16 (its
    # rounding then hangs on no last bits, and 0.36 % more is past the midpoint to the next)
    last = np.where(np.arange(dm) % 2, 1.0, -0.5)
    last[0], last[1:3] = 1, 0
    exact = []
    for n in range(total):
        l = 1 + (vl[n] - 1) * p
        v = np.unique(bf(np.linspace(1.5 * l, 1.97 * l, 800).astype(np.float32))).astype(np.float64)
        o = bf((v / l).astype(np.float32)).astype(np.float64)
        best = int(np.argmin(np.abs(v / l - o)))
        assert abs(v[best] / l - o[best]) < 2.0 ** -10 * 0.9   # a spacing is 2^-7, a midpoint 2^-8
        emb[n, vl[n] - 1] = last
        emb[n, vl[n] - 1, 0] = v[best]
        # V = x[0] in the upper half of every head
        up = np.arange(dm) % dh >= dh // 2
        L.W_qkv[2 * dm + np.flatnonzero(up), 0] = 1
        x = emb[n, vl[n] - 1].astype(np.float64) + up * o[best]
        for _ in range(2):
            x = (x - x.mean()) / np.sqrt(x.var() + 1e-5)
        exact.append(x)
    tb = synth.make_tokens(total, T_, dm, seed=1, valid_len=vl)
    tb.emb[:], tb.cand[:] = emb, 0
    return tb, W, np.array(exact)


@pytest.mark.parametrize("n_heads", [1, 2])
@pytest.mark.parametrize("T_", [20, 64, 190, 192, 300])
def test_softmax_sums_are_not_rounded(T_, n_heads):
    """The softmax's row sums are sums of fp32 exponentials: summed after their rounding
    to bf16 they would be 0.4 % too small here, and the attention output the next bf16.
    Bound: fp32 arithmetic on values below 8 (2^-20), against 2e-3 for that fault."""
    print(f"encode_small softmax sums T={T_} heads={n_heads}", flush=True)
    tb, W, exact = one_value_inputs(T_, n_heads)
    tok, cand = upload_tokens(tb)
    out = T.encode(tok, cand, T.DeviceWeights(W)).cpu().numpy().astype(np.float64)
    err = np.abs(out[:, 64:] - exact).max()
    print(f"  max abs error {err:.3e}", flush=True)
    assert err <= 2e-5


@pytest.mark.parametrize("T_,flags", [(64, T.MASK_CAUSAL), (64, T.MASK_NONE), (300, T.MASK_CAUSAL)])
def test_scores_that_overflow_downwards(T_, flags):
    """Keys whose scores are below the fp32 range (-inf) have weight 0, also where the first
    32 keys that a query looks at are all of that kind (causal: the 32 around its own
    position; unmasked: the first 32)."""
    print(f"encode_small overflowing scores T={T_} flags={flags}", flush=True)
    W = weights_for(T_, d=64, n_layers=1, seed=9)
    L = W.layers[0]
    W.W_in[:] = np.concatenate([np.eye(64), np.zeros((64, 64))], axis=1)
    for a in (W.b_in, W.E_act, W.E_time, W.E_pos):
        a[:] = 0
    L.W_qkv[:64], L.b_qkv[:128] = 0, 0
    L.W_qkv[64:128] = 0
    L.W_qkv[64, 1], L.b_qkv[0] = -1e20, 1e20      # score -1e40 x[1]
    L.W_qkv[:] = synth.round_to_bf16(L.W_qkv)
    L.W_qkv[128:] *= 16
    tb = synth.make_tokens(4, T_, 64, seed=6, valid_len=[T_, T_ - 1, T_ - 9, 40])
    p = np.arange(T_)
    tb.emb[:, :, 1] = (p < 32) if flags == T.MASK_NONE else (p % 64 >= 32)
    run_and_check(tb, W, flags=flags)
