"""GPU parity of the chunked transformer state encoder (Sec. 3.3) against the
CPU oracle, through the C ABI: the small backbone on whole batches (empty,
one-chunk and many-chunk programs, a ragged last chunk), the CodeBERT-shaped
backbone on a batch whose programs cover one and several 512-token windows,
token-id validation, determinism, and the encoder feeding the evaluator.

Comparison: per program ||g - o||_2 / ||o||_2 (the latent rule), 1e-4 in
fp32 and 2e-2 in bf16."""
import numpy as np
import pytest

import synth
from oracle import text_encoder as TE
from oracle import wm_oracle as O

from parity_util import TOL, latent_rel

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def wm():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2606_09312_amd as wm
    wm.load_library()
    return wm


_models = {}


def model_for(wm, name, prec):
    key = (name, prec)
    if key not in _models:
        w = synth.TEXT_WORKLOADS[name]
        W = synth.make_text_weights(w, 500)
        _models[key] = (wm.TextModel(w, W, precision=prec), W, w)
    return _models[key]


def run(wm, model, tokens, off):
    t = torch.from_numpy(np.ascontiguousarray(tokens, dtype=np.int32)).cuda()
    out = wm.encode_text(model, t, off)
    wm.device_status(out["ws"])
    return out["z0"].cpu().numpy().astype(np.float64)


def programs_of(tokens, off):
    return [tokens[off[s]:off[s + 1]] for s in range(len(off) - 1)]


@pytest.mark.parametrize("prec", ["fp32", "bf16"])
def test_small_backbone_whole_batch(wm, prec):
    model, W, w = model_for(wm, "tiny_text", prec)
    tokens, off = synth.make_programs(w, 11)
    # an empty program, one shorter than the window, one exactly a window
    lens = np.diff(off)
    lens[0], lens[1], lens[2] = 0, 17, w.window
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    tokens = np.random.default_rng(3).integers(0, w.vocab, size=int(off[-1])).astype(np.int32)
    print(f"[text] tiny_text {prec} lens={list(lens)} chunks={model.chunks(off)}", flush=True)
    g = run(wm, model, tokens, off)
    ref = TE.encode(W, programs_of(tokens, off), w.window, w.stride, w.heads, prec)
    rel = latent_rel(g, ref)
    assert rel.max() <= TOL[prec], f"z0 rel err {rel.max():.3e}"
    np.testing.assert_allclose(g[0], W["bp"], rtol=0, atol=0)      # empty program: the bias
    print(f"  max rel {rel.max():.2e}", flush=True)


def test_codebert_backbone(wm):
    """CodeBERT shape (12 layers, 768 wide, 12 heads, 512-token windows with
    stride 256): programs of 1, 300, 512, 700 and 1100 tokens (1, 1, 1, 2, 4
    chunks)."""
    model, W, w = model_for(wm, "codebert", "bf16")
    lens = np.array([1, 300, 512, 700, 1100])
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    tokens = np.random.default_rng(5).integers(0, w.vocab, size=int(off[-1])).astype(np.int32)
    print(f"[text] codebert bf16 chunks={model.chunks(off)}", flush=True)
    g = run(wm, model, tokens, off)
    ref = TE.encode(W, programs_of(tokens, off), w.window, w.stride, w.heads, "bf16")
    rel = latent_rel(g, ref)
    assert rel.max() <= TOL["bf16"], f"z0 rel err {rel.max():.3e}"
    print(f"  max rel {rel.max():.2e}", flush=True)


@pytest.mark.parametrize("prec,hidden,heads,window", [
    ("fp32", 96, 1, 64), ("bf16", 96, 1, 64), ("bf16", 64, 2, 544), ("fp32", 64, 2, 544), ("fp32", 192, 3, 160)])
def test_other_shapes(wm, prec, hidden, heads, window):
    """Head widths without fused attention (96) and windows past the fused bf16
    one (general path), and the float32 fused attention over several key and
    query blocks with a ragged last one."""
    w = synth.TextWorkload(name="other", S=5, vocab=300, hidden=hidden, heads=heads, ffn=160, layers=2,
                           window=window, stride=window // 2, d=32, len_lo=0, len_hi=3 * window)
    W = synth.make_text_weights(w, 81)
    model = wm.TextModel(w, W, precision=prec)
    tokens, off = synth.make_programs(w, 83)
    print(f"[text] other {prec} {hidden}/{heads} window {window} lens={np.diff(off)}", flush=True)
    g = run(wm, model, tokens, off)
    ref = TE.encode(W, programs_of(tokens, off), w.window, w.stride, w.heads, prec)
    rel = latent_rel(g, ref)
    assert rel.max() <= TOL[prec], f"z0 rel err {rel.max():.3e}"
    if prec == "fp32":          # six plane products: float32 accuracy, far inside the tolerance
        assert rel.max() <= 5e-6, f"z0 rel err {rel.max():.3e}"


@pytest.mark.parametrize("S,n", [(3, 70), (40, 190), (200, 190)])
def test_product_tiles(wm, S, n):
    """Each tile size of the bf16 products (64 x 64, 128 x 64 and 256 x 256 tiles
    for few, more and many rows), with row counts that no tile divides and
    output widths (128, 256, 384) below, at and above one 256-column tile."""
    w = synth.TextWorkload(name="tiles", S=S, vocab=500, hidden=128, heads=4, ffn=256, layers=2, window=64,
                           stride=32, d=64, len_lo=1, len_hi=n)
    W = synth.make_text_weights(w, 71)
    model = wm.TextModel(w, W, precision="bf16")
    tokens, off = synth.make_programs(w, 73)
    print(f"[text] tiles S={S} chunks={model.chunks(off)} tokens={len(tokens)}", flush=True)
    g = run(wm, model, tokens, off)
    ref = TE.encode(W, programs_of(tokens, off), w.window, w.stride, w.heads, "bf16")
    rel = latent_rel(g, ref)
    assert rel.max() <= TOL["bf16"], f"z0 rel err {rel.max():.3e}"


@pytest.mark.parametrize("S,n,hidden,heads,ffn", [
    (3, 70, 32, 1, 64), (4, 90, 96, 3, 160), (200, 190, 96, 3, 160), (256, 230, 32, 1, 96)])
def test_float32_product_tiles(wm, S, n, hidden, heads, ffn):
    """The float32 products with few and many tiles and ragged last ones, contractions of 1 to 5 slices (shorter and longer than the ring of
    three) and output widths whose last 64-column tile holds 32 columns.  The bound is
    that of the float32 shapes above."""
    w = synth.TextWorkload(name="tiles32", S=S, vocab=500, hidden=hidden, heads=heads, ffn=ffn, layers=2, window=64,
                           stride=32, d=64, len_lo=1, len_hi=n)
    W = synth.make_text_weights(w, 91)
    model = wm.TextModel(w, W, precision="fp32")
    tokens, off = synth.make_programs(w, 93)
    print(f"[text] fp32 tiles S={S} chunks={model.chunks(off)} tokens={len(tokens)}", flush=True)
    g = run(wm, model, tokens, off)
    ref = TE.encode(W, programs_of(tokens, off), w.window, w.stride, w.heads, "fp32")
    rel = latent_rel(g, ref)
    assert rel.max() <= 5e-6, f"z0 rel err {rel.max():.3e}"


def test_float32_overflowing_scores(wm):
    """Scores that overflow to -inf have weight 0, also where they fill the first
    key blocks: the first 40 tokens' keys against every query, then 50 ordinary ones."""
    H, W_ = 64, 96
    w = synth.TextWorkload(name="inf", S=1, vocab=3, hidden=H, heads=2, ffn=64, layers=1, window=W_, stride=W_, d=32,
                           len_lo=90, len_hi=90)
    W = {k: np.array(v) for k, v in synth.make_text_weights(w, 97).items()}
    # tokens 0 and 1 have no feature 0 after the LayerNorm (mean 0), token 2 has
    W["pos_emb"][:] = 0
    W["tok_emb"][:] = np.where(np.arange(H) % 2, -1.0, 1.0)
    W["tok_emb"][1, 8:] *= 2.0
    W["tok_emb"][:2, :2] = 0
    W["tok_emb"][2, :2] = 4.0, -4.0
    W["ln0_g"][:], W["ln0_b"][:] = 1, 0
    wqkv = W["wqkv"][0]
    wqkv[0, :], wqkv[H, :] = 0, 0                 # q[0] = 1e20, k[0] = -1e20 h[0]
    W["bqkv"][0, 0], W["bqkv"][0, H] = 1e20, 0
    wqkv[H, 0] = -1e20
    model = wm.TextModel(w, W, precision="fp32")
    tokens = np.concatenate([np.full(40, 2), np.tile([0, 1], 25)]).astype(np.int32)
    off = np.array([0, 90], np.int32)
    g = run(wm, model, tokens, off)
    ref = TE.encode(W, [tokens], w.window, w.stride, w.heads, "fp32")
    assert np.isfinite(ref).all()
    rel = latent_rel(g, ref)
    assert rel.max() <= 5e-6, f"z0 rel err {rel.max():.3e}"


def test_float32_values_past_the_largest_bf16(wm):
    """A hidden value between the largest bf16 and the largest float32 that no
    output takes up (its column of W2 is zero) changes nothing."""
    w = synth.TextWorkload(name="big", S=1, vocab=50, hidden=64, heads=2, ffn=96, layers=1, window=64, stride=64, d=32,
                           len_lo=60, len_hi=60)
    W = {k: np.array(v) for k, v in synth.make_text_weights(w, 99).items()}
    W["w2"][0, :, 5] = 0
    tokens = np.random.default_rng(9).integers(0, 50, 60).astype(np.int32)
    off = np.array([0, 60], np.int32)
    a = run(wm, wm.TextModel(w, W, precision="fp32"), tokens, off)
    W["b1"][0, 5] = 3.4e38
    b = run(wm, wm.TextModel(w, W, precision="fp32"), tokens, off)
    np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("prec,per", [("fp32", 6), ("bf16", 2)])
def test_model_memory(wm, prec, per):
    """A model of the packed paths holds its layer matrices once, as the products
    read them: 6 bytes per weight (three bf16 planes) in float32, 2 in bf16; everything
    else is float32.  16 MiB are allowed for the allocator's granularity."""
    w = synth.TextWorkload(name="mem", S=1, vocab=1000, hidden=768, heads=12, ffn=3072, layers=6, window=512,
                           stride=256, d=256, len_lo=1, len_hi=1)
    W = synth.make_text_weights(w, 95)
    mats = sum(W[k].size for k in ("wqkv", "wo", "w1", "w2"))
    rest = sum(v.size for v in W.values()) - mats
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    before = torch.cuda.mem_get_info()[0]
    model = wm.TextModel(w, W, precision=prec)
    used = before - torch.cuda.mem_get_info()[0]
    model.close()
    print(f"[text] memory {prec}: {used / 2 ** 20:.0f} MiB for {mats} matrix weights", flush=True)
    assert used <= per * mats + 4 * rest + (16 << 20)


def test_token_out_of_range_is_reported(wm):
    model, W, w = model_for(wm, "tiny_text", "fp32")
    off = np.array([0, 5], dtype=np.int32)
    tokens = np.array([1, 2, w.vocab, 3, 4], dtype=np.int32)
    t = torch.from_numpy(tokens).cuda()
    out = wm.encode_text(model, t, off)
    with pytest.raises(wm.WMError) as e:
        wm.device_status(out["ws"])
    assert e.value.status == 5
    wm.device_status(out["ws"])          # cleared


def test_deterministic_and_independent_of_batch(wm):
    """Repeated calls give identical bits; a program's latent does not depend
    on the other programs of the batch."""
    model, W, w = model_for(wm, "tiny_text", "bf16")
    tokens, off = synth.make_programs(w, 19)
    a = run(wm, model, tokens, off)
    b = run(wm, model, tokens, off)
    np.testing.assert_array_equal(a, b)
    s = 3
    one = run(wm, model, tokens[off[s]:off[s + 1]], np.array([0, off[s + 1] - off[s]], dtype=np.int32))
    np.testing.assert_array_equal(one[0], a[s])


def test_encoder_feeds_the_evaluator(wm):
    """The encoded programs are the initial latents of a rollout batch: the
    evaluator run on the GPU latents matches the oracle run on the oracle's
    encodings (bf16 end to end, within the latent tolerance)."""
    model, Wt, wt = model_for(wm, "tiny_text", "bf16")
    tokens, off = synth.make_programs(wt, 23)
    z0 = run(wm, model, tokens, off)
    z0_ref = TE.encode(Wt, programs_of(tokens, off), wt.window, wt.stride, wt.heads, "bf16")
    base = synth.workload("tiny")
    w = synth.scaled(base, B=wt.S * 40, S=wt.S)
    W = synth.make_weights(w, 1000)
    ev = wm.Model(wm.model_dims(w), W, precision="bf16")
    I = synth.make_inputs(w, 29)
    I["z0"] = z0.astype(np.float32)
    from parity_util import run_evaluate
    g = run_evaluate(ev, w, I, 4)
    Iref = dict(I, z0=z0_ref)
    ref = O.evaluate(W, Iref, 4, "bf16")
    assert latent_rel(g["zT"], ref["zT"]).max() <= TOL["bf16"]
