"""GPU parity on a mid-size bf16 decoder (2 layers, d 2048, 16 q / 4 kv heads
of 128, FFN 8192, V 8192).  Its projections split K across the waves of a
block, and the down projection (K = 8192) also across blocks (the last block
of a column group reducing the partials).

Bar (bf16): logits within 2e-2 absolute of the oracle (fp64 with the same
bf16 rounding points); tokens equal except where the oracle's top-2 logit gap
is below 1e-3.
"""
import numpy as np
import pytest

import jf_inputs
from oracle import jacobi as ojac
from oracle import multiblock as omb
from oracle.model import DecoderOracle

pytestmark = pytest.mark.gpu

SHAPE = dict(n_layers=2, d_model=2048, n_heads=16, n_kv_heads=4, head_dim=128, d_ffn=8192,
             vocab=8192, rope_base=1000000.0, rms_eps=1e-6, dtype="bf16")
LOGIT_TOL = 2e-2
GAP_EXEMPT = 1e-3


@pytest.fixture(scope="module")
def env():
    import torch
    from paper_2512_14681_amd import decode, jf
    assert torch.cuda.is_available()
    w = jf_inputs.model_weights(SHAPE, seed=5)
    prompt = jf_inputs.prompt(6, 80, SHAPE["vocab"])
    model = jf.Model(SHAPE, w, max_rows=64, max_ctx=512)
    return dict(w=w, prompt=prompt, model=model, dec=decode.Decoder(model))


def teacher_forced(env, tokens):
    """Oracle logits of every position of `tokens` in one causal pass."""
    m = DecoderOracle(SHAPE, env["w"])
    R = len(tokens)
    z, _ = m.forward(np.asarray(tokens), np.arange(R), np.tri(R, dtype=bool))
    return z


def gaps(z):
    s = np.sort(z, axis=1)
    return s[:, -1] - s[:, -2]


def test_step_logits(env):
    import torch
    dec = env["dec"]
    dec.reset()
    p = dec.prefill(env["prompt"])
    n = 16
    draft = [p] + [ojac.pad_id(3, 80 + i, SHAPE["vocab"]) for i in range(1, n)]
    d_draft = torch.tensor(draft, dtype=torch.int32, device="cuda")
    d_next = torch.zeros(n, dtype=torch.int32, device="cuda")
    d_log = torch.empty((n, SHAPE["vocab"]), dtype=torch.float32, device="cuda")
    env["model"].jf_jacobi_step(d_draft, n, 1, 3, dec.d_argmax, dec.d_result, d_next, d_log)
    z = d_log.cpu().numpy()
    g = dec.d_argmax[:n].cpu().numpy()
    zo = teacher_forced(env, list(env["prompt"]) + draft)[79:79 + n + 1]
    # row i of the step predicts the token after draft[i]: oracle position 80 + i
    zo = zo[1:]
    err = np.abs(z - zo).max()
    assert err < LOGIT_TOL, err
    ok = (g == zo.argmax(1)) | (gaps(zo) < GAP_EXEMPT)
    assert ok.all()


@pytest.mark.parametrize("n", [80, 96])
def test_step_logits_column_slice_rows(env, n):
    """Steps of 65 to 96 rows run every projection on the many-row GEMM (QKV and
    O with split K and the ordered reduction): all rows' logits against the
    teacher-forced oracle."""
    import torch
    from paper_2512_14681_amd import decode, jf
    model = jf.Model(SHAPE, env["w"], max_rows=96, max_ctx=512)
    dec = decode.Decoder(model)
    p = dec.prefill(env["prompt"])
    draft = [p] + [ojac.pad_id(4, 80 + i, SHAPE["vocab"]) for i in range(1, n)]
    d_draft = torch.tensor(draft, dtype=torch.int32, device="cuda")
    d_next = torch.zeros(n, dtype=torch.int32, device="cuda")
    d_log = torch.empty((n, SHAPE["vocab"]), dtype=torch.float32, device="cuda")
    model.jf_jacobi_step(d_draft, n, 1, 4, dec.d_argmax, dec.d_result, d_next, d_log)
    z = d_log.cpu().numpy()
    g = dec.d_argmax[:n].cpu().numpy()
    zo = teacher_forced(env, list(env["prompt"]) + draft)[80:80 + n]
    err = np.abs(z - zo).max()
    assert err < LOGIT_TOL, err
    assert ((g == zo.argmax(1)) | (gaps(zo) < GAP_EXEMPT)).all()


@pytest.mark.parametrize("n", [17, 32, 49, 65, 161, 257])
def test_step_logits_ragged_many_rows(env, n):
    """One row past a row-tile boundary of the many-row GEMM: the split-K
    reduction, the RoPE / cache-write, SwiGLU and residual epilogues with a
    last row tile of one row, in one and in several row chunks.  Bars as for
    every bf16 step."""
    import torch
    from paper_2512_14681_amd import decode, jf
    model = jf.Model(SHAPE, env["w"], max_rows=272, max_ctx=512)
    dec = decode.Decoder(model)
    p = dec.prefill(env["prompt"])
    draft = [p] + [ojac.pad_id(4, 80 + i, SHAPE["vocab"]) for i in range(1, n)]
    d_draft = torch.tensor(draft, dtype=torch.int32, device="cuda")
    d_next = torch.zeros(n, dtype=torch.int32, device="cuda")
    d_log = torch.empty((n, SHAPE["vocab"]), dtype=torch.float32, device="cuda")
    model.jf_jacobi_step(d_draft, n, 1, 4, dec.d_argmax, dec.d_result, d_next, d_log)
    z = d_log.cpu().numpy()
    g = dec.d_argmax[:n].cpu().numpy()
    zo = teacher_forced(env, list(env["prompt"]) + draft)[80:80 + n]
    err = np.abs(z - zo).max()
    assert err < LOGIT_TOL, err
    assert ((g == zo.argmax(1)) | (gaps(zo) < GAP_EXEMPT)).all()


@pytest.mark.parametrize("n", [10, 13, 15, 16])
def test_step_logits_few_rows_of_a_wide_ffn(n):
    """10 to 16 rows of a decoder whose gate/up projection (2560 column tiles)
    is on the many-row GEMM there, ragged and full."""
    import torch
    from paper_2512_14681_amd import decode, jf
    shape = dict(n_layers=1, d_model=256, n_heads=4, n_kv_heads=2, head_dim=64, d_ffn=20480, vocab=1024,
                 rope_base=10000.0, rms_eps=1e-6, dtype="bf16")
    w = jf_inputs.model_weights(shape, seed=8)
    prompt = jf_inputs.prompt(9, 20, shape["vocab"])
    dec = decode.Decoder(jf.Model(shape, w, max_rows=64, max_ctx=128))
    p = dec.prefill(prompt)
    draft = [p] + [ojac.pad_id(4, 20 + i, shape["vocab"]) for i in range(1, n)]
    d_draft = torch.tensor(draft, dtype=torch.int32, device="cuda")
    d_next = torch.zeros(n, dtype=torch.int32, device="cuda")
    d_log = torch.empty((n, shape["vocab"]), dtype=torch.float32, device="cuda")
    dec.m.jf_jacobi_step(d_draft, n, 1, 4, dec.d_argmax, dec.d_result, d_next, d_log)
    z = d_log.cpu().numpy()
    m = DecoderOracle(shape, w)
    T = 20 + n
    zo, _ = m.forward(np.asarray(list(prompt) + draft), np.arange(T), np.tri(T, dtype=bool))
    zo = zo[20:]
    assert np.abs(z - zo).max() < LOGIT_TOL
    assert ((dec.d_argmax[:n].cpu().numpy() == zo.argmax(1)) | (gaps(zo) < GAP_EXEMPT)).all()


@pytest.mark.parametrize("n", [49, 90])
def test_step_logits_with_buffers_off_a_16_byte_boundary(env, n):
    """Packed weights and workspace 8 bytes past a 16-byte boundary (the
    workspace holds 64-bit words): every projection's epilogue on the kernel
    for such operands, with and without split K."""
    import ctypes
    import torch
    from paper_2512_14681_amd import decode, jf

    class Shifted(jf.Model):
        def __init__(self, shape, weights, max_rows, max_ctx):
            self.torch, self.shape, self.stream, self.V = torch, dict(shape), None, shape["vocab"]
            self.cfg = jf.config(shape, max_rows, max_ctx)
            self.raw = [torch.empty(b + 8, dtype=torch.uint8, device="cuda") for b in jf.query_sizes(self.cfg)]
            assert all(t.data_ptr() % 16 == 0 for t in self.raw)
            self.packed, self.kv, self.ws = self.raw[0][8:], self.raw[1][:-8], self.raw[2][8:]
            dev = [torch.from_numpy(np.ascontiguousarray(weights[k]).view(np.int16)).to("cuda")
                   for k in jf.weight_names(shape)]
            ptrs = (ctypes.c_void_p * len(dev))(*[t.data_ptr() for t in dev])
            self.h = ctypes.c_void_p()
            jf.check(jf.lib().jf_model_load(ctypes.byref(self.cfg), ptrs, len(dev), jf._ptr(self.packed),
                                            jf._ptr(self.kv), jf._ptr(self.ws), jf._stream(), ctypes.byref(self.h)))

    dec = decode.Decoder(Shifted(SHAPE, env["w"], 96, 512))
    p = dec.prefill(env["prompt"])
    draft = [p] + [ojac.pad_id(4, 80 + i, SHAPE["vocab"]) for i in range(1, n)]
    d_draft = torch.tensor(draft, dtype=torch.int32, device="cuda")
    d_next = torch.zeros(n, dtype=torch.int32, device="cuda")
    d_log = torch.empty((n, SHAPE["vocab"]), dtype=torch.float32, device="cuda")
    dec.m.jf_jacobi_step(d_draft, n, 1, 4, dec.d_argmax, dec.d_result, d_next, d_log)
    z = d_log.cpu().numpy()
    g = dec.d_argmax[:n].cpu().numpy()
    zo = teacher_forced(env, list(env["prompt"]) + draft)[80:80 + n]
    err = np.abs(z - zo).max()
    assert err < LOGIT_TOL, err
    assert ((g == zo.argmax(1)) | (gaps(zo) < GAP_EXEMPT)).all()


@pytest.mark.parametrize("n,mode", [(16, "window"), (8, "block")])
def test_decode_matches_oracle_argmax(env, n, mode):
    dec = env["dec"]
    dec.reset()
    toks, acc = dec.generate_jacobi(env["prompt"], n, 40, mode=mode, pad_seed=4)
    z = teacher_forced(env, list(env["prompt"]) + toks)
    pred = z[79:79 + 40].argmax(1)       # greedy prediction of every generated slot
    bad = (pred != np.asarray(toks)) & (gaps(z[79:79 + 40]) >= GAP_EXEMPT)
    assert not bad.any(), np.nonzero(bad)
    assert all(a >= 1 for a in acc)


def test_multiblock_outputs_greedy_tokens(env):
    dec = env["dec"]
    dec.reset()
    toks, tr = dec.generate_multiblock(env["prompt"], 8, 3, 0.5, 40, pad_seed=6)
    z = teacher_forced(env, list(env["prompt"]) + toks)
    pred = z[79:79 + 40].argmax(1)
    bad = (pred != np.asarray(toks)) & (gaps(z[79:79 + 40]) >= GAP_EXEMPT)
    assert not bad.any()
    assert max(t["R"] for t in tr) > 8


def test_repeat_is_bitwise_deterministic(env):
    """Split-K partials are summed in a fixed order: two runs agree exactly."""
    import torch
    dec = env["dec"]
    outs = []
    for _ in range(2):
        dec.reset()
        p = dec.prefill(env["prompt"])
        d = torch.tensor([p] + list(range(1, 16)), dtype=torch.int32, device="cuda")
        d_log = torch.empty((16, SHAPE["vocab"]), dtype=torch.float32, device="cuda")
        env["model"].jf_jacobi_step(d, 16, 1, 0, dec.d_argmax, dec.d_result, dec.d_next, d_log)
        outs.append(d_log.cpu().numpy())
    assert np.array_equal(outs[0], outs[1])


@pytest.mark.parametrize("n", [1, 5, 16])
def test_fused_attention_launch_equals_four_launches(env, n):
    """Steps of at most 16 rows run QKV + attention + O of a layer as one
    persistent launch (JF_OPT_FUSED_ATTENTION); the same step with the four
    separate launches gives the same logits (to fp32 summation order: both
    agree with the oracle within the bar), the same argmax away from
    near-ties, and no sync error."""
    import torch
    from paper_2512_14681_amd import jf
    dec, model = env["dec"], env["model"]
    outs = []
    for fused in (1, 0):
        model.jf_model_set_option(jf.JF_OPT_FUSED_ATTENTION, fused)
        dec.reset()
        p = dec.prefill(env["prompt"])
        draft = [p] + [ojac.pad_id(3, 80 + i, SHAPE["vocab"]) for i in range(1, n)]
        d_draft = torch.tensor(draft, dtype=torch.int32, device="cuda")
        d_next = torch.zeros(n, dtype=torch.int32, device="cuda")
        d_log = torch.empty((n, SHAPE["vocab"]), dtype=torch.float32, device="cuda")
        model.jf_jacobi_step(d_draft, n, 1, 3, dec.d_argmax, dec.d_result, d_next, d_log)
        res = dec.d_result.cpu().numpy()
        assert res[3] == 0, res
        outs.append((d_log.cpu().numpy(), dec.d_argmax[:n].cpu().numpy(), res.copy(), draft))
    model.jf_model_set_option(jf.JF_OPT_FUSED_ATTENTION, 0)
    (z1, g1, r1, draft), (z0, g0, r0, _) = outs
    assert np.abs(z1 - z0).max() < 1e-3
    zo = teacher_forced(env, list(env["prompt"]) + draft)[80:80 + n]
    assert np.abs(z1 - zo).max() < LOGIT_TOL
    ok = (g1 == zo.argmax(1)) | (gaps(zo) < GAP_EXEMPT)
    assert ok.all()
    assert ((g1 == g0) | (gaps(zo) < GAP_EXEMPT)).all()


def test_fused_attention_repeat_is_bitwise_deterministic(env):
    """The fused launch merges waves, key splits and K-blocks in a fixed
    order: two identical steps agree bit for bit."""
    import torch
    from paper_2512_14681_amd import jf
    dec = env["dec"]
    env["model"].jf_model_set_option(jf.JF_OPT_FUSED_ATTENTION, 1)
    outs = []
    for _ in range(2):
        dec.reset()
        p = dec.prefill(env["prompt"])
        d = torch.tensor([p] + list(range(1, 12)), dtype=torch.int32, device="cuda")
        d_log = torch.empty((12, SHAPE["vocab"]), dtype=torch.float32, device="cuda")
        env["model"].jf_jacobi_step(d, 12, 1, 0, dec.d_argmax, dec.d_result, dec.d_next, d_log)
        outs.append(d_log.cpu().numpy())
    env["model"].jf_model_set_option(jf.JF_OPT_FUSED_ATTENTION, 0)
    assert np.array_equal(outs[0], outs[1])


@pytest.mark.parametrize("cands,pseudo", [(3, 1), (7, 0)])
def test_multiblock_step_beyond_256_rows(env, cands, pseudo):
    """Steps of more than 256 rows: blocks of n = 64 with the real-active draft,
    `cands` recycled 64-token candidates under its root and `pseudo` chained
    pseudo-active blocks (App. A Alg. 1).  (3, 1) is the paper's chosen
    multi-block point, block 64 x verification 4 at K = 2 (App. E): 320 rows;
    (7, 0) is 512 rows, the engine's maximum.  Every row's logits against
    the oracle, and the device's verification, winner and path from its own
    argmax."""
    import torch
    from oracle import tree as otree
    from paper_2512_14681_amd import jf
    V, n = SHAPE["vocab"], 64
    R = n * (1 + cands + pseudo)
    model = jf.Model(SHAPE, env["w"], max_rows=jf.JF_MAX_ROWS, max_ctx=704)
    from paper_2512_14681_amd import decode
    dec = decode.Decoder(model)
    p = dec.prefill(env["prompt"])
    C = len(env["prompt"])
    segs = [(0, n, -1, jf.JF_ROLE_RA, 1)]
    for c in range(cands):
        segs.append((n * (1 + c), n, 0, jf.JF_ROLE_CAND, 0))
    for b in range(pseudo):
        first = n * (1 + cands + b)
        segs.append((first, n, n - 1 if b == 0 else first - 1, jf.JF_ROLE_PSEUDO, 0))
    rng = np.random.default_rng(R)
    tokens = [p] + [int(t) for t in rng.integers(0, V, R - 1)]
    d_tok = torch.tensor(tokens, dtype=torch.int32, device="cuda")
    d_arg = torch.zeros(R, dtype=torch.int32, device="cuda")
    d_seg = torch.zeros(jf.JF_MAX_SEGMENTS, dtype=torch.int32, device="cuda")
    d_res = torch.zeros(4, dtype=torch.int32, device="cuda")
    d_path = torch.zeros(R, dtype=torch.int32, device="cuda")
    d_log = torch.empty((R, V), dtype=torch.float32, device="cuda")
    model.jf_multiblock_step(d_tok, R, segs, d_arg, d_seg, d_res, d_path, d_log)
    z = d_log.cpu().numpy()
    g = d_arg.cpu().numpy()
    ora = DecoderOracle(SHAPE, env["w"])
    ora.prefill(np.asarray(env["prompt"]))
    osegs = [otree.Segment(*s) for s in segs]
    parent, pos, vis = otree.build(osegs, R, C)
    zo, _ = ora.forward(np.asarray(tokens), pos, vis)
    err = np.abs(z - zo).max()
    assert err < LOGIT_TOL, err
    assert ((g == zo.argmax(1)) | (gaps(zo) < GAP_EXEMPT)).all()
    m_dev = list(d_seg.cpu().numpy()[:len(segs)])
    res = d_res.cpu().numpy()
    assert m_dev == otree.verify(np.asarray(tokens), g, parent, osegs)
    assert (res[1], [int(x) for x in d_path.cpu().numpy()[:res[0]]]) == otree.winner_path(osegs, m_dev, parent)
