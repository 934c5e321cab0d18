"""Every query-group size the decode attention is built for, against the float64 oracle.

The decode attention is instantiated per G = n_q_heads / n_kv_heads (1 to 8) and
head_dim (64, 128); the workload shapes reach G = 4, 5 and 8.  Small two-layer
stages with the head cover the rest, G = 1 (multi-head attention, the degenerate
case) included, and one Qwen3-style variant: chunked prefill from tokens,
ragged batched decode, and the head's greedy token.  Every call goes through the
C ABI.
"""
import numpy as np
import pytest

import synth
from oracle import OracleStage
from tests import gemm_calls as gc
from tests.helpers import SeededModel, argmax_agrees, assert_hidden_close

pytestmark = pytest.mark.gpu

CASES = [  # (n_q_heads, n_kv_heads, head_dim, qk_norm)
    (4, 4, 64, False),    # G = 1
    (4, 2, 128, False),   # G = 2
    (6, 2, 64, False),    # G = 3
    (12, 2, 128, False),  # G = 6
    (14, 2, 64, False),   # G = 7
    (6, 3, 128, True),    # G = 2, per-head q/k norms, query width 768 against hidden 256
]


@pytest.fixture(scope="module")
def torch():
    import torch as t
    if not t.cuda.is_available():
        pytest.skip("no GPU")
    return t


@pytest.fixture(scope="module")
def st():
    from paper_2609_34045_amd import stage
    return stage


def host(t):
    return t.float().cpu().numpy().astype(np.float64)


@pytest.mark.parametrize("nq,nkv,hd,qkn", CASES, ids=[f"g{c[0] // c[1]}_hd{c[2]}{'_qknorm' if c[3] else ''}" for c in CASES])
def test_group_size(torch, st, nq, nkv, hd, qkn):
    shape = synth.ModelShape(2, 256, nq, nkv, hd, 512, 300, 1e-5, 1e4, qk_norm=qkn)
    cfg = 50 + nq + nkv + hd // 64
    model = SeededModel(shape, cfg)
    g = st.Stage(shape, 0, 2, model.layer, model.head())
    kv = g.kv(3, 200)
    o = OracleStage(shape, 0, 2, model.layer, model.head(), max_users=3, max_ctx=200)
    worst = 0.0
    for u, n in ((0, 70), (1, 5), (2, 130)):  # prompts: several splits, one tiny, several key blocks
        toks = synth.tokens(cfg, u, n, shape.vocab)
        for c0 in range(0, n, 48):
            part = toks[c0:c0 + 48]
            y = g.prefill(kv, u, c0, tokens=torch.from_numpy(part).cuda())
            worst = max(worst, assert_hidden_close(host(y), o.prefill(u, c0, tokens=part), what=f"prefill {u}@{c0}"))
    for step, users in enumerate(([0, 1, 2], [2, 0], [1], [0, 1, 2])):
        pos = [kv.len(u) for u in users]
        x = synth.hidden_states(cfg, synth.STREAM_DECODE_HIDDEN, step, len(users), shape.hidden)
        y = g.decode(kv, users, pos, hidden=torch.from_numpy(x).cuda())
        ref = o.decode(users, pos, hidden=x)
        worst = max(worst, assert_hidden_close(host(y), ref, what=f"decode {step}"))
        lg = host(g.head_logits(y))
        lr = o.logits(ref)
        tg = host(g.head_argmax(y)).astype(np.int64)
        for b in range(len(users)):
            assert argmax_agrees(int(tg[b]), int(np.argmax(lr[b])), lr[b], lg[b])
    print(f"G={nq // nkv} hd={hd} qk_norm={qkn} max row rel err", worst)
    kv.close()
    g.close()


@pytest.mark.parametrize("ffn,T", [(16384, 512), (16384, 300), (1408, 512)], ids=["f16384_t512", "f16384_t300", "f1408_t512"])
def test_prefill_swiglu_tile_widths(torch, st, ffn, T):
    """Layers with a wide SwiGLU projection against the float64 oracle: an FFN of 16384 at full and ragged chunks, and one of
    1408, which ends in a partial column tile of 256.

    Which tile each takes is the plan's choice; test_gpu_gemm_tiles.py compares every one.  One layer, a prefill from
    hidden rows on an empty cache; every output row is compared.
    """
    shape = synth.ModelShape(1, 256, 4, 2, 64, ffn, 300, 1e-5, 1e4)
    cfg = 60 + ffn % 97
    model = SeededModel(shape, cfg)
    g = st.Stage(shape, 0, 1, model.layer, None)
    kv = g.kv(1, T)
    h = synth.hidden_states(cfg, synth.STREAM_PREFILL_HIDDEN, 0, T, shape.hidden)
    y = g.prefill(kv, 0, 0, hidden=torch.from_numpy(h).cuda())
    o = OracleStage(shape, 0, 1, model.layer, None, max_users=1, max_ctx=T)
    err = assert_hidden_close(host(y), o.prefill(0, 0, hidden=h), what=f"prefill ffn {ffn} T {T}")
    print(f"ffn={ffn} T={T} prefill max row rel err", err)
    kv.close()
    g.close()


@pytest.mark.parametrize("T", [300, 512], ids=["t300", "t512"])
def test_prefill_splitk_tile_widths(torch, st, T):
    """A layer whose projections split K at full and ragged row tiles, against the float64 oracle.

    H 6144, 32 query heads and 8 KV heads of 128, FFN 8192: the slices of the QKV, output and down projections meet in
    the RoPE and row-norm kernels and in the output store.  Which tiles they take is the plan's choice;
    test_gpu_gemm_tiles.py compares every one.  One layer, a prefill from hidden rows on an empty cache; every output
    row is compared.
    """
    shape = synth.ModelShape(1, 6144, 32, 8, 128, 8192, 300, 1e-5, 1e4)
    cfg = 77
    model = SeededModel(shape, cfg)
    g = st.Stage(shape, 0, 1, model.layer, None)
    kv = g.kv(1, T)
    h = synth.hidden_states(cfg, synth.STREAM_PREFILL_HIDDEN, 0, T, shape.hidden)
    y = g.prefill(kv, 0, 0, hidden=torch.from_numpy(h).cuda())
    o = OracleStage(shape, 0, 1, model.layer, None, max_users=1, max_ctx=T)
    err = assert_hidden_close(host(y), o.prefill(0, 0, hidden=h), what=f"prefill T {T}")
    print(f"split-K tile widths T={T} prefill max row rel err", err)
    kv.close()
    g.close()


@pytest.mark.parametrize("T", [1, 32, 33, 64, 65, 128, 129, 257])
def test_prefill_row_tiles(torch, st, T):
    """A layer at chunk lengths around the row tiles' heights, against the float64 oracle.

    The plan takes tiles of 32 x 128 up to 128 tokens and of 256 x 128 above (test_gpu_gemm_tiles.py compares every tile);
    query width 320 and FFN 1088 are no multiples of 128; K = 256, 320 and 1088 give one to four K slices, down to
    slices of four and five 64-deep steps.
    """
    shape = synth.ModelShape(1, 256, 5, 1, 64, 1088, 300, 1e-5, 1e4)
    cfg = 78
    model = SeededModel(shape, cfg)
    g = st.Stage(shape, 0, 1, model.layer, None)
    kv = g.kv(1, T)
    h = synth.hidden_states(cfg, synth.STREAM_PREFILL_HIDDEN, 0, T, shape.hidden)
    y = g.prefill(kv, 0, 0, hidden=torch.from_numpy(h).cuda())
    o = OracleStage(shape, 0, 1, model.layer, None, max_users=1, max_ctx=T)
    # what the layer adds to the rows (a few percent of them: a lost block would pass unseen in the sum)
    err = assert_hidden_close(host(y) - h, o.prefill(0, 0, hidden=h) - h, what=f"prefill T {T}")
    print(f"row tiles T={T} prefill max row rel err", err)
    kv.close()
    g.close()


@pytest.mark.parametrize("slices", range(1, 9))
def test_prefill_slices(torch, st, slices):
    """Every number of K slices that the RoPE, the row norms and the output store add, against what two layers of the
    float64 oracle add."""
    k, T = 256 * slices, 20
    shape = synth.ModelShape(2, k, 4 * slices, slices, 64, k, 300, 1e-5, 1e4)
    for n in (6 * slices * 64, k):  # QKV; output and down
        assert gc.plan(st.load_library(), gc.PARTIAL, T, n, k, 1 << 22).slices == slices
    model = SeededModel(shape, 98)
    g = st.Stage(shape, 0, 2, model.layer, None)
    kv = g.kv(1, T)
    h = synth.hidden_states(98, synth.STREAM_PREFILL_HIDDEN, 0, T, k)
    y = g.prefill(kv, 0, 0, hidden=torch.from_numpy(h).cuda())
    o = OracleStage(shape, 0, 2, model.layer, None, max_users=1, max_ctx=T)
    assert_hidden_close(host(y) - h, o.prefill(0, 0, hidden=h) - h, what=f"{slices} slices")
    kv.close()
    g.close()


def test_prefill_shorter_chunk_after_longer(torch, st):
    """A chunk's results do not depend on the chunks before it, whose workspace is laid out otherwise: chunks of 300, 256,
    40 and 130 tokens on one stage give the bits that each gives on a stage of its own.  (That a shorter chunk fits where
    a longer one ran is checked on the host, test_prefill_workspace.py.)"""
    shape = synth.ModelShape(1, 1024, 8, 2, 64, 8192, 300, 1e-5, 1e4)
    cfg = 79
    model = SeededModel(shape, cfg)
    chunks = [300, 256, 40, 130]
    g = st.Stage(shape, 0, 1, model.layer, None)
    kv = g.kv(len(chunks), max(chunks))
    for u, T in enumerate(chunks):
        h = torch.from_numpy(synth.hidden_states(cfg, synth.STREAM_PREFILL_HIDDEN, u, T, shape.hidden)).cuda()
        y = g.prefill(kv, u, 0, hidden=h)
        own = st.Stage(shape, 0, 1, model.layer, None)
        own_kv = own.kv(1, T)
        assert torch.equal(y, own.prefill(own_kv, 0, 0, hidden=h)), T
        own_kv.close()
        own.close()
    kv.close()
    g.close()


@pytest.mark.parametrize("fold", [True, False], ids=["gain_folded", "gain_apart"])
@pytest.mark.parametrize("io", ["float32", "bfloat16"])
@pytest.mark.parametrize("rows", [5, 33, 64, 129, 300])
def test_logits_of_many_rows(torch, st, rows, io, fold):
    """More rows than one GEMV pass takes (the matrix-core logits), at the edges of their tiles and chunks.

    Rows of very different scales (1e-30 to 1e15, and values 1e-6 of their row's
    largest), one of zeros, one with an infinity and one with a NaN, over a
    vocabulary that ends in a partial tile.  Against the GEMV on the same rows, four at a
    time: either is about 1e-7 (two-norm) off exact sums over the stored matrix, single logits
    within ten times that, so they differ by no more than 2e-6 of a row's largest (without the low
    parts of fp32 rows by 2e-4); and the rows' relative error against float64 (their matrix as stored, fp16 with
    the gain) stays under 1e-3.
    """
    shape = synth.ModelShape(1, 320, 5, 1, 64, 64, 777, 1e-5, 1e4)
    cfg = 80
    model = SeededModel(shape, cfg)
    head = dict(model.head())
    if not fold:  # one product beyond fp16 keeps the gain out of the matrix
        gain = np.array(head["final_norm"], copy=True)
        gain[7] = 0x4974  # 1e6 in bf16
        head["final_norm"] = gain
    g = st.Stage(shape, 0, 1, model.layer, head)
    o = OracleStage(shape, 0, 1, model.layer, head, max_users=1, max_ctx=1)
    x = synth.hidden_states(cfg, synth.STREAM_DECODE_HIDDEN, 0, rows, shape.hidden)
    x[0, ::3] *= 1e-6
    x[1] *= 1e15
    x[2] *= 1e-30
    x[3] = 0
    x = torch.from_numpy(x).to(getattr(torch, io)).cuda()
    whole = g.head_logits(x)
    g.sync()
    parts = torch.cat([g.head_logits(x[r:r + 4].contiguous()) for r in range(0, rows, 4)])
    ref = o.logits(x.double().cpu().numpy())
    got, want = host(whole), host(parts)
    keep = np.array([r for r in range(rows) if r != 3])
    scale = np.max(np.abs(want[keep]), axis=1, keepdims=True)
    assert np.all(np.isfinite(got))
    assert np.max(np.abs(got[keep] - want[keep]) / scale) <= 2e-6
    assert np.max(np.abs(got[keep] - ref[keep]) / np.max(np.abs(ref[keep]), axis=1, keepdims=True)) <= 1e-3
    assert not got[3].any()
    x[0, 5] = float("inf")
    x[rows - 1, 9] = float("nan")
    bad = g.head_logits(x)
    with pytest.raises(st.KFError) as e:
        g.sync()
    assert e.value.status == st.KF_ERANGE
    assert torch.isnan(bad[0]).all() and torch.isnan(bad[rows - 1]).all()
    assert torch.equal(bad[1:rows - 1], whole[1:rows - 1])
    g.close()


@pytest.mark.parametrize("nq,nkv,hd,T", [(6, 2, 64, 1), (6, 2, 64, 45), (5, 1, 128, 20), (8, 1, 64, 130), (4, 4, 128, 129)],
                         ids=["g3_t1", "g3_t45", "g5_t20", "g8_t130", "g1_t129"])
def test_prefill_short_chunk_over_long_cache(torch, st, nq, nkv, hd, T):
    """Short chunks over 3000 cached keys: the attention's keys go to up to 23 workgroups per tile of 128 rows
    (tokens x query heads of a KV head), past the 16 splits merged in one pass, with tiles that end inside a
    token (G = 3, 5), in rows without a token, and waves without rows.  Values of unit variance, so that the
    attention carries what the layer adds; compared with the float64 oracle's addition."""
    shape = synth.ModelShape(1, 256, nq, nkv, hd, 64, 300, 1e-5, 1e4)
    cfg, n0 = 81 + nq, 3000
    model = SeededModel(shape, cfg)
    k, v = synth.injected_kv(shape, cfg, 0, 0, n0)
    v[7::211] = (0x40C0, )  # some values of 6: each split's share of the weights shows
    h = synth.hidden_states(cfg, synth.STREAM_PREFILL_HIDDEN, 0, T, shape.hidden)
    o = OracleStage(shape, 0, 1, model.layer, None, max_users=1, max_ctx=n0 + T)
    o.kv.inject(0, 0, 0, k, v)
    o.kv.set_len(0, n0)
    g = st.Stage(shape, 0, 1, model.layer, None)
    kv = g.kv(1, n0 + T)
    kv.write(0, 0, 0, torch.from_numpy(k.view(np.int16)).cuda(), torch.from_numpy(v.view(np.int16)).cuda())
    kv.set_len(0, n0)
    y = g.prefill(kv, 0, n0, hidden=torch.from_numpy(h).cuda())
    err = assert_hidden_close(host(y) - h, o.prefill(0, n0, hidden=h) - h, what=f"short chunk T {T}")
    print(f"G={nq // nkv} hd={hd} T={T} over {n0} keys: max row rel err of the addition", err)
    kv.close()
    g.close()


@pytest.mark.parametrize("H", [1984, 2048, 8192, 8320])
@pytest.mark.parametrize("io", ["tokens", "bfloat16", "float32"])
def test_prefill_row_norm_widths(torch, st, H, io):
    """The prefill's row norm around its row sizes (256 or 1024 threads, the row in registers up to H = 8192,
    the rest through memory), on each kind of stage input; compared with what the float64 oracle's layer adds."""
    shape = synth.ModelShape(1, H, 2, 1, 64, 192, 50, 1e-5, 1e4)
    cfg, T = 95, 3
    model = SeededModel(shape, cfg)
    head = model.head() if io == "tokens" else None
    g = st.Stage(shape, 0, 1, model.layer, head)
    o = OracleStage(shape, 0, 1, model.layer, head, max_users=1, max_ctx=T)
    kv = g.kv(1, T)
    if io == "tokens":
        toks = synth.tokens(cfg, 0, T, shape.vocab)
        y, ref = g.prefill(kv, 0, 0, tokens=torch.from_numpy(toks).cuda()), o.prefill(0, 0, tokens=toks)
        x = (head["embed"][toks].astype(np.uint32) << 16).view(np.float32).astype(np.float64)
    else:
        t = torch.from_numpy(synth.hidden_states(cfg, synth.STREAM_PREFILL_HIDDEN, 0, T, H)).to(getattr(torch, io))
        x = host(t)
        y, ref = g.prefill(kv, 0, 0, hidden=t.cuda()), o.prefill(0, 0, hidden=x)
    # bf16 rows come back rounded to 2^-9 of their values, the additions are about a twentieth of them
    rtol = 2 ** -9 * np.max(np.abs(ref)) / np.min(np.max(np.abs(ref - x), axis=1)) + 5e-3 if io == "bfloat16" else 5e-3
    err = assert_hidden_close(host(y) - x, ref - x, rtol=rtol, what=f"H {H} {io}")
    print(f"H={H} {io} max row rel err of the addition", err, "of", rtol)
    kv.close()
    g.close()
