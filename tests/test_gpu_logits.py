"""kf_head_logits over more rows than one GEMV pass takes (the matrix-core logits)."""
import numpy as np
import pytest

import synth
from tests.helpers import SeededModel

pytestmark = pytest.mark.gpu


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


def head_stage(st, hidden, vocab, cfg, edit=None):
    """A stage whose layer is not used, and its head's tensors."""
    shape = synth.ModelShape(1, hidden, 1, 1, 64, 64, vocab, 1e-5, 1e4)
    model = SeededModel(shape, cfg)
    head = {k: np.array(v, copy=True) for k, v in model.head().items()}
    if edit:
        edit(head)
    return shape, head, st.Stage(shape, 0, 1, model.layer, head)


@pytest.mark.parametrize("io", ["float32", "bfloat16"])
@pytest.mark.parametrize("hidden,vocab", [(320, 777), (512, 40003)])
def test_equal_rows_give_equal_logits(torch, st, hidden, vocab, io):
    """Equal LM-head rows in different column tiles give exactly equal logits (the lowest index then wins an argmax),
    equal hidden rows in different row tiles equal rows, and a row the same bits in a call of 5 rows as in one of
    600 (several chunks): every element sums its products in one order whatever tile it lies in."""
    cols = [3, 130, 300, 511, 512, 770] + ([9000, vocab - 1] if vocab > 9000 else [])

    def twins(head):
        head["lm_head"][cols] = head["lm_head"][3]

    shape, _, g = head_stage(st, hidden, vocab, 82, twins)
    x = synth.hidden_states(82, synth.STREAM_DECODE_HIDDEN, 0, 600, hidden)
    same = [1, 4, 33, 63, 70, 140, 255, 256, 399, 599]
    x[same] = x[1]
    x = torch.from_numpy(x).to(getattr(torch, io)).cuda()
    whole = g.head_logits(x)
    for rows in (5, 33, 64, 65, 97, 128, 129, 200, 256, 300, 600):
        y = g.head_logits(x[:rows].contiguous())
        assert torch.equal(y[:, cols], y[:, 3:4].expand(-1, len(cols))), rows
        r = [i for i in same if i < rows]
        assert torch.equal(y[r], y[1:2].expand(len(r), -1)), rows
        assert torch.equal(y, whole[:rows]), rows
    g.sync()
    g.close()


def test_rows_of_extreme_magnitude(torch, st):
    """Rows near and below the smallest normal fp32 values, against 64-bit sums over the matrix as stored (1e-5 of the
    largest logit: fp32's own spacing there is 1e-7), and a row with one product of value and gain beyond fp32, which
    gives infinities as the GEMV of up to four rows does."""
    def edit(head):
        head["final_norm"][7] = 0x7149  # 1e30 in bf16: the gain stays out of the matrix

    shape, head, g = head_stage(st, 320, 777, 84, edit)
    x = synth.hidden_states(84, synth.STREAM_DECODE_HIDDEN, 0, 40, 320)
    x[:, 7] = 0
    x[5] *= 1e-38
    x[6] *= 1e-40
    x[9, 7], x[10, 7] = 1e10, -1e10
    gain, w = ((head[k].astype(np.uint32) << 16).view(np.float32) for k in ("final_norm", "lm_head"))
    ref = (x[5:7] * gain.astype(np.float64) / np.sqrt(shape.rms_eps)) @ w.astype(np.float16).astype(np.float64).T
    x = torch.from_numpy(x).cuda()
    whole = host(g.head_logits(x))
    parts = host(g.head_logits(x[8:12].contiguous()))
    assert np.isinf(parts[1:3]).all() and np.array_equal(whole[9:11], parts[1:3])
    for r in (0, 1):
        assert np.max(np.abs(whole[5 + r] - ref[r])) <= 1e-5 * np.max(np.abs(ref[r])), r
    g.sync()
    g.close()


@pytest.mark.parametrize("rows,io,limit", [(5, "float32", 1.6e-7), (100, "float32", 1.6e-7), (256, "float32", 1.6e-7),
                                           (20, "bfloat16", 1.2e-7), (300, "bfloat16", 1.2e-7)])
def test_sums_as_exact_as_the_gemv(torch, st, rows, io, limit):
    """4096 products a logit, against 64-bit sums over the matrix as stored.  The GEMV of up to four rows is 1.2e-7 (bf16
    rows 1.0e-7) off in the 2-norm, a few roundings of 2^-24 / sqrt(3); one chain of matrix instructions over all
    of K 5.8e-7 (4.2e-7), the high parts of fp32 rows alone about 1e-4.  The limits are a third above the GEMV's."""
    shape, head, g = head_stage(st, 4096, 700, 86)
    gain, w = ((head[k].astype(np.uint32) << 16).view(np.float32) for k in ("final_norm", "lm_head"))
    x = torch.from_numpy(synth.hidden_states(86, synth.STREAM_DECODE_HIDDEN, 0, rows, 4096)).to(getattr(torch, io))
    xd = x.double().numpy()
    ref = (xd / np.sqrt(np.mean(xd * xd, axis=1, keepdims=True) + shape.rms_eps)) @ (w * gain).astype(np.float16).astype(np.float64).T
    x = x.cuda()
    err = lambda y, r: np.linalg.norm(host(y) - r) / np.linalg.norm(r)  # noqa: E731
    many, gemv = err(g.head_logits(x), ref), err(g.head_logits(x[:4].contiguous()), ref[:4])
    print(f"{rows} {io} rows: {many:.2e}, four {gemv:.2e}")
    assert gemv <= limit and many <= limit
    g.sync()
    g.close()


@pytest.mark.parametrize("io", ["float32", "bfloat16"])
@pytest.mark.parametrize("rows", [5, 40, 300])
def test_rows_of_wide_range(torch, st, rows, io):
    """Rows with one value 2^20 or 2^40 times the others, and rows spread over ten decades, among ordinary ones.  In every other
    LM-head row that value's weight is zero, so its logits rest on the small values alone: each row's error there
    against 64-bit sums stays at the GEMV's (as above; a fixed number of bits below the largest value gives 2e-6 and
    more)."""
    def edit(head):
        head["lm_head"][::2, 11] = 0

    hidden = 1024
    shape, head, g = head_stage(st, hidden, 777, 87, edit)
    gain, w = ((head[k].astype(np.uint32) << 16).view(np.float32) for k in ("final_norm", "lm_head"))
    rng = np.random.default_rng(87)
    x = rng.standard_normal((rows, hidden))
    x[1, 11], x[rows - 1, 11] = 2.0 ** 20, -2.0 ** 40
    x[rows // 2::9] *= 10 ** rng.uniform(-10, 0, x[rows // 2::9].shape)
    x = torch.from_numpy(x.astype(np.float32)).to(getattr(torch, io))
    xd = x.double().numpy()
    ref = (xd / np.sqrt(np.mean(xd * xd, axis=1, keepdims=True) + shape.rms_eps)) @ (w * gain).astype(np.float16).astype(np.float64).T
    y = host(g.head_logits(x.cuda()))
    for cols in (slice(0, None, 2), slice(1, None, 2)):
        err = np.linalg.norm((y - ref)[:, cols], axis=1) / np.linalg.norm(ref[:, cols], axis=1)
        print(f"{rows} {io}: largest row error {err.max():.2e}")
        assert err.max() <= 2.5e-7, (int(err.argmax()), err.max())  # a row's error varies more than that of many rows
    g.sync()
    g.close()


def test_first_call_under_capture(torch, st):
    """Nine rows as a stage's first call of more than four, while its stream is being captured: four at a time, without
    the workspace; after an eager call a capture takes the many-row path.  Both graphs replayed among eager work."""
    shape, head, g = head_stage(st, 320, 777, 85)
    x = torch.from_numpy(synth.hidden_states(85, synth.STREAM_DECODE_HIDDEN, 0, 9, 320)).cuda()
    fours = torch.cat([g.head_logits(x[r:r + 4].contiguous()) for r in range(0, 9, 4)])
    main, side = torch.cuda.current_stream(), torch.cuda.Stream()
    torch.cuda.synchronize()

    def captured():
        graph, y = torch.cuda.CUDAGraph(), torch.empty(9, 777, device="cuda")
        g.set_stream(side)
        with torch.cuda.graph(graph, stream=side):
            g.head_logits(x, out=y)
        g.set_stream(main)
        return graph, y

    def check(graph, y, want):
        for _ in range(3):
            y.zero_()
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(y, want)
            g.head_logits(x[:4].contiguous())
            torch.cuda.synchronize()

    first = captured()
    check(*first, fours)
    many = g.head_logits(x)
    torch.cuda.synchronize()
    second = captured()
    check(*second, many)
    check(*first, fours)
    g.sync()
    g.close()
