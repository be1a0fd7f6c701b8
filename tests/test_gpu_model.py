"""End-to-end GPU parity against the oracle: encoder output codes and cross
keys/values bit-exact, decode-step logits (bar: 1e-3 relative; bit-exact
expected), greedy token sequences identical on the tiny and mobile workloads,
hipGraph replay identical to eager launches, beam search identical on small
models and on sampled sentences of the batched beam workloads."""
import dataclasses

import numpy as np
import pytest

import oracle
from synth import generate as G

from .conftest import model_blob

pytestmark = pytest.mark.gpu
RTOL = 1e-3

SMALL_PRE = G.ModelConfig("small-preln", 64, 4, 128, 2, 2, 500, ln_post=0, seed=77, random_gamma=True)
SMALL_POST = G.ModelConfig("small-postln", 64, 2, 128, 2, 2, 300, ln_post=1, seed=78, random_gamma=True,
                           weight_std=0.1)
DIVERSE = G.ModelConfig("diverse-preln", 128, 2, 256, 3, 2, 700, ln_post=0, seed=81, random_gamma=True,
                        weight_std=0.1)


@pytest.fixture(scope="module")
def torch_dev():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a visible GPU"
    return torch, torch.device("cuda:0")


_models = {}


def _pair(name_or_cfg, flags=0):
    """(oracle model, GPU model) for a named workload model or a ModelConfig
    (flags: the GPU model's load flags)."""
    from paper_2306_04235_amd import mnmt

    key = (name_or_cfg if isinstance(name_or_cfg, str) else name_or_cfg.name, flags)
    if key not in _models:
        blob = model_blob(name_or_cfg) if isinstance(name_or_cfg, str) else G.build_model(name_or_cfg)
        _models[key] = (oracle.Model(blob), mnmt.Model(blob, flags=flags))
    return _models[key]


def _t(torch, dev, a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(dev)


def _greedy_check(torch, dev, cfg, src, lens, steps, stop_at_eos=False, check_logits=True, flags=0):
    from paper_2306_04235_amd import mnmt

    om, gm = _pair(cfg, flags)
    B, S = src.shape
    print(f"greedy {cfg if isinstance(cfg, str) else cfg.name} B={B} S={S} steps={steps}", flush=True)
    sess = mnmt.Session(gm, B, S, steps, 1)
    ts, tl = _t(torch, dev, src), _t(torch, dev, lens)
    o_out, o_len, o_logits = om.greedy(src, lens, steps, stop_at_eos=stop_at_eos, want_logits=True)
    # encoder output and cross keys/values, bit-exact on valid rows
    sess.encode(ts, tl)
    torch.cuda.synchronize()
    enc = sess.tensor("enc_out", torch.int8, (B, S, gm.info.d_model)).cpu().numpy()
    o_enc = om.encode(src, lens)
    for b in range(B):
        assert np.array_equal(enc[b, : lens[b]], o_enc[b, : lens[b]]), f"encoder output, sentence {b}"
    for l in range(gm.info.n_dec):
        kv = sess.tensor(f"cross_kv.{l}", torch.int8, (B, S, 2 * gm.info.d_model)).cpu().numpy()
        o_kv = om.cross_kv(o_enc, lens, l)
        for b in range(B):
            assert np.array_equal(kv[b, : lens[b]], o_kv[b, : lens[b]]), f"cross kv layer {l} sentence {b}"
    # teacher-forced decode steps through the C ABI: logits and tokens
    if check_logits and not stop_at_eos:
        prev = None
        for t in range(steps):
            nxt, logits = sess.decode_step(prev, want_logits=True)
            z = logits.cpu().numpy()
            ref = o_logits[:, t]
            assert np.allclose(z, ref, rtol=RTOL, atol=RTOL * np.abs(ref).max()), f"logits step {t}"
            assert np.array_equal(z.view(np.uint32), ref.view(np.uint32)), f"logits bits step {t}"
            assert np.array_equal(nxt.cpu().numpy(), o_out[:, t]), f"tokens step {t}"
            prev = _t(torch, dev, o_out[:, t])
    # whole translation, eager and captured in a graph (replayed twice)
    for use_graph in (False, True, True):
        out, out_len, _ = sess.translate(ts, tl, beam=1, max_steps=steps, stop_at_eos=stop_at_eos,
                                         use_graph=use_graph)
        torch.cuda.synchronize()
        assert np.array_equal(out.cpu().numpy(), o_out), f"greedy tokens (graph={use_graph})"
        assert np.array_equal(out_len.cpu().numpy(), o_len)
    # each step's winning arg-max key (recorded by the step that commits the
    # token): the high word is the order-preserving key of the maximum logit
    if not stop_at_eos:
        keys = sess.tensor("out_key", torch.int64, (steps, B)).cpu().numpy().view(np.uint64)
        assert np.array_equal(keys.T, _argmax_keys(o_logits)), "arg-max keys (maximum logit bits and index)"
    # no kernel of the translation chain gave up waiting for its predecessor
    assert int(sess.tensor("chain_err", torch.int32, (1,)).cpu().numpy()[0]) == 0
    sess.status()
    sess.close()
    return o_out


def _argmax_keys(z):
    """Packed arg-max keys of fp32 logits [..., V]: order-preserving 32-bit key of
    the maximum << 32 | (0xFFFFFFFF - index of its first occurrence)."""
    idx = z.argmax(axis=-1)
    m = np.take_along_axis(z, idx[..., None], axis=-1)[..., 0]
    u = m.astype(np.float32).view(np.uint32).astype(np.uint64)
    hi = np.where(u & 0x80000000, ~u & 0xFFFFFFFF, u | 0x80000000)
    return (hi << np.uint64(32)) | (np.uint64(0xFFFFFFFF) - idx.astype(np.uint64))


def test_tiny_postln_greedy(torch_dev):
    torch, dev = torch_dev
    src, lens = G.workload_inputs(G.WORKLOADS["tiny"])
    _greedy_check(torch, dev, "TINY", src, lens, 16)


def test_small_models_batched_greedy(torch_dev):
    torch, dev = torch_dev
    for cfg in (SMALL_PRE, SMALL_POST, DIVERSE):
        src, lens = G.make_sources(cfg.vocab, 5, [1, 7, 12, 3, 12], seed=21, s_max=12)
        _greedy_check(torch, dev, cfg, src, lens, 10)
        _greedy_check(torch, dev, cfg, src, lens, 10, stop_at_eos=True, check_logits=False)


def test_one_and_two_row_greedy(torch_dev):
    # 1 or 2 rows take the three-kernels-per-layer decoder step
    torch, dev = torch_dev
    for cfg in (SMALL_PRE, SMALL_POST, DIVERSE):
        for B in (1, 2):
            src, lens = G.make_sources(cfg.vocab, B, (3, 12), seed=24 + B, s_max=12)
            _greedy_check(torch, dev, cfg, src, lens, 10)
            _greedy_check(torch, dev, cfg, src, lens, 10, stop_at_eos=True, check_logits=False)


def test_two_row_greedy_longest_sequences(torch_dev):
    # 128 source positions and 128 target steps: the longest attention of the
    # 2-row step; one position more moves both lengths to the general path
    torch, dev = torch_dev
    src, lens = G.make_sources(SMALL_POST.vocab, 2, [128, 77], seed=26, s_max=128)
    _greedy_check(torch, dev, SMALL_POST, src, lens, 128)
    src, lens = G.make_sources(SMALL_POST.vocab, 2, [129, 5], seed=27, s_max=129)
    _greedy_check(torch, dev, SMALL_POST, src, lens, 129, check_logits=False)


def test_greedy_batch_above_gemv_limit(torch_dev):
    # 12 rows: the output projection runs on matrix cores, arg-max separately
    torch, dev = torch_dev
    src, lens = G.make_sources(DIVERSE.vocab, 12, (2, 20), seed=22, s_max=20)
    _greedy_check(torch, dev, DIVERSE, src, lens, 9)


@pytest.mark.parametrize("V", [63, 4100, 32772])
def test_row_argmax_widths(torch_dev, V):
    """The arg-max of stored logits (9 rows): a vocabulary that is no multiple
    of 4, one within a single round of 16-byte loads, and one just past it;
    repeated embedding rows tie the maximum (the smallest index wins)."""
    torch, dev = torch_dev
    cfg = dataclasses.replace(DIVERSE, name=f"argmax-{V}", vocab=V, emb_distinct=41)
    src, lens = G.make_sources(V, 9, (2, 9), seed=29, s_max=9)
    _greedy_check(torch, dev, cfg, src, lens, 3)


def test_diverse_model_output_depends_on_the_source(torch_dev):
    # the higher-variance test model's translations differ between sources
    torch, dev = torch_dev
    src, lens = G.make_sources(DIVERSE.vocab, 3, (8, 14), seed=23, s_max=14)
    out = _greedy_check(torch, dev, DIVERSE, src, lens, 12, check_logits=False)
    assert len({tuple(r) for r in out}) > 1


def test_mobile_greedy_latency_workload(torch_dev):
    torch, dev = torch_dev
    src, lens = G.workload_inputs(G.WORKLOADS["mobile"])
    _greedy_check(torch, dev, "MOBILE", src, lens, 30)


def test_serial_steps_match_the_kernel_chain(torch_dev, monkeypatch):
    """The batch-1 steps run as a chain of kernels over two streams, each
    waiting on its predecessor's flags; with MNMT_SERIAL_STEPS=1 (read at
    session creation) they run in one stream.  Both give the oracle's tokens."""
    torch, dev = torch_dev
    from paper_2306_04235_amd import mnmt

    om, gm = _pair("MOBILE")
    src, lens = G.workload_inputs(G.WORKLOADS["mobile"])
    o_out, o_len = om.greedy(src, lens, 30)[:2]
    ts, tl = _t(torch, dev, src), _t(torch, dev, lens)
    for serial in ("0", "1"):
        monkeypatch.setenv("MNMT_SERIAL_STEPS", serial)
        sess = mnmt.Session(gm, 1, src.shape[1], 30, 1)
        for use_graph in (False, True):
            out, out_len, _ = sess.translate(ts, tl, beam=1, max_steps=30, use_graph=use_graph)
            torch.cuda.synchronize()
            assert np.array_equal(out.cpu().numpy(), o_out), f"serial={serial} graph={use_graph}"
            assert np.array_equal(out_len.cpu().numpy(), o_len)
        assert int(sess.tensor("chain_err", torch.int32, (1,)).cpu().numpy()[0]) == 0
        sess.close()


def test_kernel_chain_many_sentences(torch_dev, monkeypatch):
    """Two dozen different batch-1 sentences (10-30 source tokens) through the
    kernel chain, in graph replays as the benchmark runs them, against the
    one-stream steps of the same kernels (about 5,000 flag hand-offs, each
    consumer reading what its predecessors wrote on other compute units),
    and the first four against the oracle."""
    torch, dev = torch_dev
    from paper_2306_04235_amd import mnmt

    om, gm = _pair("MOBILE")
    rng = np.random.default_rng(2024)
    lens_all = rng.integers(10, 31, 24)
    outs = {}
    for serial in ("1", "0"):
        monkeypatch.setenv("MNMT_SERIAL_STEPS", serial)
        sess = mnmt.Session(gm, 1, 30, 30, 1)
        got = []
        for k, n in enumerate(lens_all):
            src, lens = G.make_sources(G.MOBILE.vocab, 1, [int(n)], seed=500 + k, s_max=30)
            out, out_len, _ = sess.translate(_t(torch, dev, src), _t(torch, dev, lens), beam=1, max_steps=30,
                                             use_graph=True)
            torch.cuda.synchronize()
            got.append((out.cpu().numpy().copy(), out_len.cpu().numpy().copy()))
            if serial == "0" and k < 4:
                o_out, o_len = om.greedy(src, lens, 30)[:2]
                assert np.array_equal(got[-1][0], o_out) and np.array_equal(got[-1][1], o_len), f"sentence {k}"
        assert int(sess.tensor("chain_err", torch.int32, (1,)).cpu().numpy()[0]) == 0
        sess.close()
        outs[serial] = got
    for k, (a, b) in enumerate(zip(outs["0"], outs["1"])):
        assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1]), f"sentence {k}"


LAUNCH_FORMS = {"step": {"MNMT_STEP_LAUNCH": "1"}, "layer": {}, "three": {"MNMT_MERGED_LAYERS": "0"}}


@pytest.mark.parametrize("form", list(LAUNCH_FORMS))
def test_layer_launch_forms(torch_dev, monkeypatch, form):
    """The batch-1 translation's decode step in one launch (two-layer models
    of width 256 with a 32000-word vocabulary: both layers' self-
    attention, cross-attention and FFN blocks and the logits blocks, handing
    off through the counted words and flags inside it; MNMT_STEP_LAUNCH=1),
    one launch per decoder layer and one for the logits (the default), or
    with MNMT_MERGED_LAYERS=0 three launches per layer (read at session
    creation).  Per-step logits bits and tokens equal the oracle's at one and
    two rows, pre- and post-LN, with 4-bit weights, shared layers and widths
    64-512, eager and in graph replays."""
    import dataclasses

    torch, dev = torch_dev
    from paper_2306_04235_amd import mnmt

    for k, v in LAUNCH_FORMS[form].items():
        monkeypatch.setenv(k, v)
    src, lens = G.workload_inputs(G.WORKLOADS["mobile"])
    _greedy_check(torch, dev, "MOBILE", src, lens, 30)
    mob4 = dataclasses.replace(G.MOBILE, name="mobile-w4", w_bits=4)
    _greedy_check(torch, dev, mob4, src, lens, 30, flags=mnmt.LOAD_PACKED_4BIT_ONLY)
    for cfg, B, n, seed in ((SMALL_POST, 2, [9, 4], 121), (DIVERSE, 2, [14, 11], 122), (SHARED, 1, [12], 123),
                            (WIDE512, 1, [20], 124), (WIDE384, 2, [25, 19], 125), (VARIED, 2, [30, 21], 126)):
        src, lens = G.make_sources(cfg.vocab, B, n, seed=seed, s_max=max(n))
        _greedy_check(torch, dev, cfg, src, lens, 12)


def test_merged_layers_many_sentences(torch_dev, monkeypatch):
    """Two dozen batch-1 sentences in graph replays through the one-launch
    step against the per-layer launches and the three-kernel layers (all on
    the counted hand-off), the first four also against the oracle."""
    torch, dev = torch_dev
    from paper_2306_04235_amd import mnmt

    om, gm = _pair("MOBILE")
    rng = np.random.default_rng(2025)
    lens_all = rng.integers(10, 31, 24)
    outs = {}
    for form, env in LAUNCH_FORMS.items():
        monkeypatch.setenv("MNMT_STEP_LAUNCH", env.get("MNMT_STEP_LAUNCH", "0"))
        monkeypatch.setenv("MNMT_MERGED_LAYERS", env.get("MNMT_MERGED_LAYERS", "1"))
        sess = mnmt.Session(gm, 1, 30, 30, 1)
        got = []
        for k, n in enumerate(lens_all):
            src, lens = G.make_sources(G.MOBILE.vocab, 1, [int(n)], seed=700 + k, s_max=30)
            out, out_len, _ = sess.translate(_t(torch, dev, src), _t(torch, dev, lens), beam=1, max_steps=30,
                                             use_graph=True)
            torch.cuda.synchronize()
            got.append((out.cpu().numpy().copy(), out_len.cpu().numpy().copy()))
            if form == "step" and k < 4:
                o_out, o_len = om.greedy(src, lens, 30)[:2]
                assert np.array_equal(got[-1][0], o_out) and np.array_equal(got[-1][1], o_len), f"sentence {k}"
        assert int(sess.tensor("chain_err", torch.int32, (1,)).cpu().numpy()[0]) == 0
        sess.close()
        outs[form] = got
    for other in ("layer", "three"):
        for k, (a, b) in enumerate(zip(outs[other], outs["step"])):
            assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1]), f"{other}: sentence {k}"


@pytest.mark.parametrize("form", ["step", "layer"])
def test_many_translations_in_one_session(torch_dev, monkeypatch, form):
    """130 batch-1 translations of one sentence in one session, each alone
    in a graph replay: the tags that the chained step kernels hand off by
    (translation counter, step) wrap around more than once, and every
    translation must still equal the oracle's with no chain wait giving up
    (a tag that once coincided with that of the cleared slots derailed every
    64th translation)."""
    torch, dev = torch_dev
    from paper_2306_04235_amd import mnmt

    for k, v in LAUNCH_FORMS[form].items():
        monkeypatch.setenv(k, v)
    om, gm = _pair("MOBILE")
    src, lens = G.workload_inputs(G.WORKLOADS["mobile"])
    o_out, o_len = om.greedy(src, lens, 30)[:2]
    sess = mnmt.Session(gm, 1, 30, 30, 1)
    ts, tl = _t(torch, dev, src), _t(torch, dev, lens)
    err = sess.tensor("chain_err", torch.int32, (1,))
    for k in range(130):
        out, out_len, _ = sess.translate(ts, tl, beam=1, max_steps=30, use_graph=True)
        torch.cuda.synchronize()
        assert int(err.cpu().numpy()[0]) == 0, f"translation {k}: a chained wait gave up"
        assert np.array_equal(out.cpu().numpy(), o_out) and np.array_equal(out_len.cpu().numpy(), o_len), k
    sess.status()
    sess.close()


WIDE384 = G.ModelConfig("wide-384", 384, 6, 768, 2, 1, 600, ln_post=0, seed=83, random_gamma=True, weight_std=0.05)
WIDE512 = G.ModelConfig("wide-512", 512, 8, 1024, 2, 1, 600, ln_post=0, seed=84, random_gamma=True, weight_std=0.05)


def test_small_encoder_wide_models(torch_dev):
    """The batch-1 encoder kernels at widths 384 (two sentences, 50 rows: 8 rows
    per wave, attention within each sentence) and 512 (one sentence of 20)."""
    torch, dev = torch_dev
    src, lens = G.make_sources(WIDE384.vocab, 2, [25, 19], seed=41, s_max=25)
    _greedy_check(torch, dev, WIDE384, src, lens, 8)
    src, lens = G.make_sources(WIDE512.vocab, 1, [20], seed=42, s_max=20)
    _greedy_check(torch, dev, WIDE512, src, lens, 8)


@pytest.mark.parametrize("cfg", [G.PAPER_10MB, G.PAPER_20MB], ids=lambda c: c.name)
def test_paper_model_shapes_greedy(torch_dev, cfg):
    """The paper's MobileNMT-10MB / 20MB settings (vocabulary 8000, width 256 /
    384, 4 / 6 heads of 64, FFN 512 / 768, 12 + 2 layers): batch 1, 30 source
    tokens, 30 greedy steps, tokens and logits against the oracle."""
    torch, dev = torch_dev
    src, lens = G.make_sources(cfg.vocab, 1, [30], seed=2010 + cfg.d_model, s_max=30)
    _greedy_check(torch, dev, cfg, src, lens, 30)


def _beam_check(torch, dev, cfg, src, lens, W, steps, alpha, sample=None, parallel=False, flags=0):
    from paper_2306_04235_amd import mnmt

    from .oracle_pool import beam_many

    om, gm = _pair(cfg, flags)
    B, S = src.shape
    print(f"beam {cfg if isinstance(cfg, str) else cfg.name} B={B} S={S} W={W} T={steps}", flush=True)
    sess = mnmt.Session(gm, B, S, steps, W)
    ts, tl = _t(torch, dev, src), _t(torch, dev, lens)
    results = []
    for use_graph in (False, True):
        out, out_len, score = sess.translate(ts, tl, beam=W, max_steps=steps, alpha=alpha, use_graph=use_graph)
        torch.cuda.synchronize()
        results.append((out.cpu().numpy(), out_len.cpu().numpy(), score.cpu().numpy()))
    assert all(np.array_equal(results[0][i], results[1][i]) for i in range(3)), "graph replay differs from eager"
    out, out_len, score = results[0]
    idx = np.arange(B) if sample is None else np.asarray(sample)
    if parallel:  # one oracle process per sentence, up to 16 at a time
        mcfg = getattr(G, cfg) if isinstance(cfg, str) else cfg
        o_out, o_len, o_score = beam_many(mcfg, src, lens, idx, W, steps, alpha)
    else:
        o_out, o_len, o_score = om.beam(src[idx], lens[idx], W, steps, alpha)
    assert np.array_equal(out_len[idx], o_len)
    assert np.array_equal(out[idx], o_out)
    assert np.array_equal(score[idx].view(np.uint32), o_score.view(np.uint32))
    sess.close()


VARIED_BEAM = G.ModelConfig("varied-256-beam", 256, 4, 1024, 2, 2, 2000, ln_post=0, seed=1104, random_gamma=True,
                            weight_std=0.2)


# a long feed-forward (K 2048): W2's split partial sums are added by the next
# layer's fused self-attention prologue, which stores the updated rows into
# the second residual buffer
SPLIT_BEAM = G.ModelConfig("split-preln-beam", 128, 4, 2048, 2, 3, 700, ln_post=0, seed=94, random_gamma=True,
                           weight_std=0.1)


@pytest.mark.parametrize("cfg", [DIVERSE, VARIED_BEAM, SPLIT_BEAM], ids=lambda c: c.name)
def test_batched_layernorm_forms(torch_dev, monkeypatch, cfg):
    """Pre-LN beam search above 64 rows (19 sentences of beam 4: 76 rows, a
    ragged last tile of 16 rows).  The first two models run the row-wise
    decoder, which the switches below do not touch: its widths, lengths and
    hypotheses.  The third runs operator by operator (as the models of
    test_operator_path_layernorm_forms): the LayerNorms in the prologue of the
    kernels they feed (each block of the one-round-trip GEMM normalizes its
    rows) and, with MNMT_LN_FUSED=0 (read at session creation), as kernels of
    their own; the self-attention computing its rows' Q/K/V and, with
    MNMT_QKV_FUSED=0, the projection as a GEMM; the fused self-attention's
    128- and 256-position classes over 100 and 200 steps; every sentence
    against the oracle."""
    torch, dev = torch_dev
    src, lens = G.make_sources(cfg.vocab, 19, (2, 24), seed=97, s_max=24)
    for fused in ("1", "0"):
        monkeypatch.setenv("MNMT_LN_FUSED", fused)
        _beam_check(torch, dev, cfg, src, lens, 4, 12, 0.6, parallel=True)
    monkeypatch.setenv("MNMT_LN_FUSED", "1")
    monkeypatch.setenv("MNMT_QKV_FUSED", "0")
    _beam_check(torch, dev, cfg, src, lens, 4, 12, 0.6, parallel=True)
    monkeypatch.setenv("MNMT_QKV_FUSED", "1")
    # eight hypotheses per sentence (two rows per wave in the fused
    # self-attention, the K > 8 bound of the top-k), 9 sentences (72 rows)
    src8, lens8 = G.make_sources(cfg.vocab, 9, (2, 24), seed=96, s_max=24)
    _beam_check(torch, dev, cfg, src8, lens8, 8, 12, 0.6, parallel=True)
    # two and six hypotheses per sentence above 64 rows (40 and 12 sentences)
    src2, lens2 = G.make_sources(cfg.vocab, 40, (2, 24), seed=95, s_max=24)
    _beam_check(torch, dev, cfg, src2, lens2, 2, 12, 0.6, parallel=True)
    src6, lens6 = G.make_sources(cfg.vocab, 12, (2, 24), seed=94, s_max=24)
    _beam_check(torch, dev, cfg, src6, lens6, 6, 12, 0.6, parallel=True)
    # the longer key-length classes of the fused self-attention (up to 128 and
    # 256 target positions), 17 sentences (68 rows)
    src, lens = G.make_sources(cfg.vocab, 17, (1, 40), seed=98, s_max=40)
    for steps in (100, 200):
        _beam_check(torch, dev, cfg, src, lens, 4, steps, 0.6, parallel=True)


# models whose EOS row of the embedding is drawn larger, so that hypotheses
# and greedy sentences end at varied steps (the search's end-of-sentence
# rules: finished hypotheses, length penalty, finished sentences skipped)
VARIED_EOS = dataclasses.replace(VARIED_BEAM, name="varied-256-eos", eos_gain=3.0)
DIVERSE_EOS = dataclasses.replace(DIVERSE, name="diverse-eos", eos_gain=4.0)


def test_end_of_sentence_search(torch_dev):
    """Beam search and greedy search with stop_at_eos on models that emit EOS
    at varied steps (the oracle's lengths range from 1 to the maximum):
    batched beam above and below 64 rows, small-model beam at widths 2, 4, 6
    (all in the row-wise decoder), and greedy at 1, 2 and 5 rows (the chained
    batch-1 step, the 2-row step and the row-wise decoder)."""
    torch, dev = torch_dev
    src, lens = G.make_sources(VARIED_EOS.vocab, 19, (2, 24), seed=97, s_max=24)
    for W in (4, 2):
        _beam_check(torch, dev, VARIED_EOS, src, lens, W, 20, 0.6, parallel=True)
    src, lens = G.make_sources(DIVERSE_EOS.vocab, 4, [5, 1, 9, 9], seed=31, s_max=9)
    for W in (2, 4, 6):
        _beam_check(torch, dev, DIVERSE_EOS, src, lens, W, 16, 0.6)
    for B, seed in ((1, 45), (1, 48), (2, 42), (5, 45)):
        src, lens = G.make_sources(VARIED_EOS.vocab, B, (3, 30), seed=seed, s_max=30)
        _greedy_check(torch, dev, VARIED_EOS, src, lens, 20, stop_at_eos=True, check_logits=False)
    # the oracle's lengths do vary (the test exercises the end-of-sentence rules)
    om, _ = _pair(VARIED_EOS)
    src, lens = G.make_sources(VARIED_EOS.vocab, 19, (2, 24), seed=97, s_max=24)
    _, o_len, _ = om.beam(src[:6], lens[:6], 4, 20, 0.6)
    assert o_len.min() < 20 and o_len.max() > 1


HEAD16 = G.ModelConfig("head-16", 128, 8, 256, 1, 1, 600, ln_post=0, seed=88, random_gamma=True, weight_std=0.1)
HEAD128 = G.ModelConfig("head-128", 256, 2, 512, 1, 1, 600, ln_post=1, seed=89, random_gamma=True, weight_std=0.08)


@pytest.mark.parametrize("cfg", [HEAD16, HEAD128], ids=lambda c: c.name)
def test_attention_length_and_head_classes(torch_dev, cfg):
    """Attention over 64, 128 and 256 keys against the oracle, up to the maximum
    lengths (256 source tokens, 256 target positions), in the row-wise kernels
    (heads of 16) and operator by operator (heads of 128, whose length classes
    these are): greedy at 3 rows and beam search at 8 rows, with a one-token
    source among long ones."""
    torch, dev = torch_dev
    src, lens = G.make_sources(cfg.vocab, 3, [256, 131, 1], seed=90, s_max=256)
    _greedy_check(torch, dev, cfg, src, lens, 200, check_logits=False)
    src, lens = G.make_sources(cfg.vocab, 3, [100, 65, 7], seed=91, s_max=100)
    _greedy_check(torch, dev, cfg, src, lens, 100)
    src, lens = G.make_sources(cfg.vocab, 2, [150, 1], seed=92, s_max=150)
    _beam_check(torch, dev, cfg, src, lens, 4, 140, 0.6)


def test_postln_beam_above_64_rows(torch_dev):
    """Post-LN beam search above 64 rows (the normalized rows replace the
    residual stream): 76 rows of a d-64 model in the row-wise decoder, and 68
    rows of a d-256 model with 128-wide heads, operator by operator (LayerNorm
    kernels, and a cross-attention that computes its query rows itself),
    against the oracle on every sentence."""
    torch, dev = torch_dev
    src, lens = G.make_sources(SMALL_POST.vocab, 19, (2, 24), seed=99, s_max=24)
    _beam_check(torch, dev, SMALL_POST, src, lens, 4, 12, 0.6, parallel=True)
    src, lens = G.make_sources(HEAD128.vocab, 17, (2, 40), seed=100, s_max=40)
    _beam_check(torch, dev, HEAD128, src, lens, 4, 12, 0.6, parallel=True)


ODD_VOCAB = G.ModelConfig("odd-vocab", 64, 4, 128, 1, 1, 501, ln_post=0, seed=79, random_gamma=True, weight_std=0.1)


# every width and feed-forward ratio of the row-wise decoder, int8 and 4-bit
# weights, pre- and post-LN, heads of 16 to 64, shared layers
ROWS = [
    G.ModelConfig("rows-64-post", 64, 4, 128, 2, 2, 300, ln_post=1, seed=301, random_gamma=True, weight_std=0.1),
    G.ModelConfig("rows-64-w4", 64, 2, 256, 2, 1, 301, ln_post=0, seed=302, random_gamma=True, weight_std=0.1, w_bits=4),
    G.ModelConfig("rows-128", 128, 2, 512, 2, 2, 300, ln_post=0, seed=303, random_gamma=True, weight_std=0.1),
    G.ModelConfig("rows-128-post-shared", 128, 8, 256, 2, 3, 300, ln_post=1, seed=304, weight_std=0.1, share_every=1),
    G.ModelConfig("rows-256-w4", 256, 8, 512, 2, 2, 300, ln_post=0, seed=305, random_gamma=True, weight_std=0.1, w_bits=4),
    G.ModelConfig("rows-256-shared", 256, 4, 1024, 2, 3, 300, ln_post=0, seed=306, weight_std=0.1, share_every=2),
    G.ModelConfig("rows-384", 384, 6, 1536, 2, 1, 300, ln_post=0, seed=307, random_gamma=True, weight_std=0.05),
    G.ModelConfig("rows-384-w4", 384, 8, 768, 2, 1, 300, ln_post=1, seed=308, weight_std=0.05, w_bits=4),
    G.ModelConfig("rows-512", 512, 16, 1024, 2, 1, 300, ln_post=0, seed=309, random_gamma=True, weight_std=0.05),
    G.ModelConfig("rows-512-w4", 512, 8, 2048, 2, 2, 300, ln_post=0, seed=310, weight_std=0.05, w_bits=4),
]


@pytest.mark.parametrize("cfg", ROWS, ids=lambda c: c.name)
def test_row_wise_decoder_shapes(torch_dev, cfg):
    """The row-wise decoder against the oracle: greedy with every step's logits
    (5 rows; 67 source positions and 66 steps, past one group of 64 keys) and
    beam search of width 3 (21 rows, histories that cross rows)."""
    torch, dev = torch_dev
    src, lens = G.make_sources(cfg.vocab, 5, [67, 64, 65, 1, 30], seed=311, s_max=67)
    _greedy_check(torch, dev, cfg, src, lens, 66)
    src, lens = G.make_sources(cfg.vocab, 7, (2, 24), seed=312, s_max=24)
    _beam_check(torch, dev, cfg, src, lens, 3, 9, 0.6)


@pytest.mark.parametrize("cfg,B,W,steps", [(ROWS[0], 530, 1, 3), (ROWS[2], 257, 1, 4), (ROWS[4], 100, 6, 5),
                                           (ROWS[1], 1100, 1, 2), (ROWS[8], 90, 8, 2)],
                         ids=lambda v: getattr(v, "name", str(v)))
def test_row_wise_decoder_rows_per_block(torch_dev, cfg, B, W, steps):
    """More than 256 rows: several rows per block (2, 3 and, past the four
    rows of a 64-wide block, two rounds of blocks), a last block that is not
    full, blocks that cross sentences, more (row, head) pairs than waves."""
    torch, dev = torch_dev
    src, lens = G.make_sources(cfg.vocab, B, (1, 9), seed=313, s_max=9)
    if W == 1:
        _greedy_check(torch, dev, cfg, src, lens, steps)
    else:
        _beam_check(torch, dev, cfg, src, lens, W, steps, 0.6)


@pytest.mark.parametrize("i,V,B", [(1, 6161, 3), (2, 6400, 20), (8, 8001, 9), (6, 6146, 290)])
def test_wide_vocabulary_logits(torch_dev, i, V, B):
    """The output projection from the fragment-order embedding (vocabularies
    of more than 24 blocks of 256): widths 64 to 512, a last tile cut by V."""
    torch, dev = torch_dev
    cfg = dataclasses.replace(ROWS[i], name=f"{ROWS[i].name}-{V}", vocab=V)
    src, lens = G.make_sources(V, B, (1, 6), seed=316, s_max=6)
    _greedy_check(torch, dev, cfg, src, lens, 2)


@pytest.mark.parametrize("cfg,B,S", [(ROWS[0], 70, 64), (ROWS[4], 3, 130), (ROWS[2], 300, 30), (ROWS[9], 70, 60),
                                     (ROWS[7], 2, 33)], ids=lambda v: getattr(v, "name", str(v)))
def test_row_wise_encoder(torch_dev, cfg, B, S):
    """The row-wise encoder against the oracle: 16 and 32 rows per block, more
    than 8192 rows (two rounds), 64, 128 and 256 key classes, one block of a
    sentence all padding, 66 rows."""
    torch, dev = torch_dev
    rng = np.random.Generator(np.random.PCG64(314))
    lens = rng.integers(1, S + 1, B).astype(np.int32)
    lens[0], lens[-1] = S, 1
    src, lens = G.make_sources(cfg.vocab, B, lens, seed=315, s_max=S)
    _greedy_check(torch, dev, cfg, src, lens, 2)


def test_small_models_beam(torch_dev):
    torch, dev = torch_dev
    for cfg in (SMALL_PRE, SMALL_POST, DIVERSE, ODD_VOCAB):  # odd vocabulary: the one-wave-per-row top-k
        src, lens = G.make_sources(cfg.vocab, 4, [5, 1, 9, 9], seed=31, s_max=9)
        for W in (2, 4, 6):
            _beam_check(torch, dev, cfg, src, lens, W, 8, 0.6)


TIES3 = G.ModelConfig("ties-3", 64, 4, 128, 1, 1, 3000, ln_post=0, seed=86, emb_distinct=3)
TIES1 = G.ModelConfig("ties-1", 64, 4, 128, 1, 1, 2048, ln_post=0, seed=87, emb_distinct=1)


def test_beam_tied_logits(torch_dev):
    """Embedding rows repeated so the logits come in groups of equal values:
    1000 equal best scores per row (the filtered top-k list near its 1024
    capacity) and 2048 (every score equal: the overflow path).  Ties go to the
    lower flat index on both sides."""
    torch, dev = torch_dev
    for cfg in (TIES3, TIES1):
        src, lens = G.make_sources(cfg.vocab, 3, [6, 2, 7], seed=33, s_max=7)
        for W in (2, 4, 8):
            _beam_check(torch, dev, cfg, src, lens, W, 6, 0.6)


def test_4bit_weight_models(torch_dev):
    """The paper's W-E-A 4-8-8 setting (4-bit linear weights, 8-bit embedding
    and activations): batch-1 greedy on the mobile shape and on a small model,
    batched greedy and beam search on the small one, all against the oracle."""
    import dataclasses

    torch, dev = torch_dev
    mob4 = dataclasses.replace(G.MOBILE, name="mobile-w4", w_bits=4)
    src, lens = G.workload_inputs(G.WORKLOADS["mobile"])
    _greedy_check(torch, dev, mob4, src, lens, 30)
    div4 = dataclasses.replace(DIVERSE, name="diverse-w4", w_bits=4)
    src, lens = G.make_sources(div4.vocab, 1, [9], seed=31, s_max=9)
    _greedy_check(torch, dev, div4, src, lens, 10)
    src, lens = G.make_sources(div4.vocab, 3, [9, 5, 7], seed=31, s_max=9)
    _greedy_check(torch, dev, div4, src, lens, 10)
    _beam_check(torch, dev, div4, src, lens, 2, 8, 0.6)


def test_4bit_packed_only_models(torch_dev):
    """MNMT_LOAD_PACKED_4BIT_ONLY: the 4-bit weights stay packed on the device
    (half the int8 model's linear-weight bytes) and the batch-1 decoder and
    small-batch encoder kernels widen them in registers: per-step logits and
    tokens equal the oracle's on the mobile shape and on the varied model at
    one and two rows."""
    import dataclasses

    from paper_2306_04235_amd import mnmt

    torch, dev = torch_dev
    mob4 = dataclasses.replace(G.MOBILE, name="mobile-w4", w_bits=4)
    _, gm_full = _pair(mob4)
    _, gm = _pair(mob4, mnmt.LOAD_PACKED_4BIT_ONLY)
    _, gm8 = _pair("MOBILE")
    assert gm.arena.numel() < gm8.arena.numel() < gm_full.arena.numel()
    src, lens = G.workload_inputs(G.WORKLOADS["mobile"])
    _greedy_check(torch, dev, mob4, src, lens, 30, flags=mnmt.LOAD_PACKED_4BIT_ONLY)
    var4 = dataclasses.replace(VARIED, name="varied-w4", w_bits=4)
    for B in (1, 2):
        src, lens = G.make_sources(var4.vocab, B, [30, 21][:B], seed=95 + B, s_max=30)
        out = _greedy_check(torch, dev, var4, src, lens, 30, flags=mnmt.LOAD_PACKED_4BIT_ONLY)
        assert len(set(out[0].tolist())) >= 3


def test_4bit_packed_only_batched_paths(torch_dev):
    """Packed-only 4-bit models on the batched paths, which then read the
    packed codes too (the row-wise kernels a copy of them in fragment order,
    the cross keys' and values' projections the rows): 3-row greedy steps,
    beam search on a small model, and the mobile beam workload (64 sentences
    of 10-60 tokens), a dozen sentences of it against the oracle, shortest and
    longest included."""
    from paper_2306_04235_amd import mnmt

    torch, dev = torch_dev
    flags = mnmt.LOAD_PACKED_4BIT_ONLY
    div4 = dataclasses.replace(DIVERSE, name="diverse-w4", w_bits=4)
    src, lens = G.make_sources(div4.vocab, 3, [9, 5, 7], seed=31, s_max=9)
    _greedy_check(torch, dev, div4, src, lens, 10, flags=flags)
    _beam_check(torch, dev, div4, src, lens, 2, 8, 0.6, flags=flags)
    src, lens = G.make_sources(div4.vocab, 12, [9, 5, 7, 16, 3, 11, 8, 8, 2, 16, 12, 6], seed=32, s_max=16)
    _greedy_check(torch, dev, div4, src, lens, 6, flags=flags)
    # above 64 rows at d 128
    src, lens = G.make_sources(div4.vocab, 19, (2, 16), seed=34, s_max=16)
    _beam_check(torch, dev, div4, src, lens, 4, 10, 0.6, parallel=True, flags=flags)
    mob4 = dataclasses.replace(G.MOBILE, name="mobile-w4", w_bits=4)
    w = G.WORKLOADS["mobile_beam"]
    src, lens = G.workload_inputs(w)
    order = np.argsort(lens, kind="stable")
    idx = sorted({int(order[0]), int(order[-1]), *range(0, 64, 6)})
    _beam_check(torch, dev, mob4, src, lens, w.beam, w.steps, w.alpha, sample=idx, parallel=True, flags=flags)


SPLIT_PRE = G.ModelConfig("split-preln", 128, 4, 2048, 2, 2, 700, ln_post=0, seed=91, random_gamma=True,
                          weight_std=0.1)
SPLIT_POST = G.ModelConfig("split-postln", 64, 2, 1536, 1, 2, 500, ln_post=1, seed=92, random_gamma=True,
                           weight_std=0.1)


@pytest.mark.parametrize("cfg", [SPLIT_PRE, SPLIT_POST], ids=lambda c: c.name)
def test_split_k_feed_forward(torch_dev, cfg):
    """Feed-forward widths of 1536 and 2048 in the batched decoder: W2's K is
    split over blocks whose int32 partial sums the next LayerNorm kernel adds
    before the residual update (pre-LN with gamma != 1: the updated rows are
    stored, post-LN: the normalized rows replace them; the final LayerNorm
    too).  Batched greedy (12 rows) and beam search against the oracle, and
    the same with packed 4-bit weights."""
    from paper_2306_04235_amd import mnmt

    torch, dev = torch_dev
    src, lens = G.make_sources(cfg.vocab, 12, [9, 5, 7, 16, 3, 11, 8, 8, 2, 16, 12, 6], seed=93, s_max=16)
    _greedy_check(torch, dev, cfg, src, lens, 8)
    _beam_check(torch, dev, cfg, src[:5], lens[:5], 4, 8, 0.6)
    c4 = dataclasses.replace(cfg, name=cfg.name + "-w4", w_bits=4)
    _beam_check(torch, dev, c4, src[:5], lens[:5], 4, 8, 0.6, flags=mnmt.LOAD_PACKED_4BIT_ONLY)


SHARED = G.ModelConfig("shared-preln", 64, 4, 128, 4, 3, 500, ln_post=0, seed=82, random_gamma=True,
                       weight_std=0.1, share_every=1)
SHARED_256 = G.ModelConfig("shared-256", 256, 4, 1024, 6, 2, 32000, ln_post=0, seed=1103, random_gamma=True,
                           weight_std=0.2, share_every=2)


def test_cross_layer_sharing_models(torch_dev):
    """Cross-layer parameter sharing (Section 2.2): layers that reuse another
    layer's parameters (aliased device pointers, stored once) on every path --
    the batch-1 chained step and encoder, the row-wise kernels, beam search -- against the oracle."""
    torch, dev = torch_dev
    for B in (1, 2, 5, 12):
        src, lens = G.make_sources(SHARED.vocab, B, (3, 12), seed=60 + B, s_max=12)
        _greedy_check(torch, dev, SHARED, src, lens, 9)
    src, lens = G.make_sources(SHARED.vocab, 4, [5, 1, 9, 9], seed=31, s_max=9)
    _beam_check(torch, dev, SHARED, src, lens, 4, 8, 0.6)
    src, lens = G.make_sources(SHARED_256.vocab, 1, [30], seed=64, s_max=30)
    _greedy_check(torch, dev, SHARED_256, src, lens, 30)


FACTOR = G.ModelConfig("factorized-256", 256, 4, 512, 2, 2, 2000, ln_post=0, seed=83, random_gamma=True,
                       weight_std=0.2, emb_dim=128)
FACTOR_POST = G.ModelConfig("factorized-post", 128, 2, 256, 2, 1, 700, ln_post=1, seed=84, weight_std=0.1,
                            emb_dim=64)


def test_factorized_embedding_models(torch_dev):
    """Embedding factorization (Section 2.1): rows of width E projected to the
    model width on the way in (k_embed_proj) and the final rows projected back
    (an int8 linear layer over the transposed matrix) before the tied logits,
    in greedy search of 1 row (operator by operator), 5 and 12 rows (the
    row-wise decoder; per-step logits bits via mnmt_decode_step) and in beam
    search, against the oracle."""
    torch, dev = torch_dev
    for cfg in (FACTOR, FACTOR_POST):
        om, gm = _pair(cfg)
        assert gm.info.emb_dim == cfg.emb_dim and om.emb_dim == cfg.emb_dim
        for B in (1, 5, 12):
            src, lens = G.make_sources(cfg.vocab, B, (3, 16), seed=70 + B, s_max=16)
            _greedy_check(torch, dev, cfg, src, lens, 10)
        src, lens = G.make_sources(cfg.vocab, 4, [5, 1, 9, 9], seed=31, s_max=9)
        _beam_check(torch, dev, cfg, src, lens, 4, 8, 0.6)


def test_mobile_beam_workload_all_sentences(torch_dev):
    """The batched beam workload on the mobile model: all 64 sentences (10-60
    source tokens, beam 4, 64 steps) against the oracle, run one sentence per
    host process."""
    torch, dev = torch_dev
    w = G.WORKLOADS["mobile_beam"]
    src, lens = G.workload_inputs(w)
    _beam_check(torch, dev, "MOBILE", src, lens, w.beam, w.steps, w.alpha, parallel=True)


def test_base_beam_workload_sentences(torch_dev):
    """The base-model beam workload (128 sentences of 20-64 tokens, beam 4, 80
    steps): the shortest and longest sources and 22 more spread over the
    batch, against the oracle in host processes."""
    torch, dev = torch_dev
    w = G.WORKLOADS["base_beam"]
    src, lens = G.workload_inputs(w)
    order = np.argsort(lens, kind="stable")
    idx = sorted({int(order[0]), int(order[-1]), *range(0, 128, 6)})
    assert len(idx) >= 16
    _beam_check(torch, dev, "BASE", src, lens, w.beam, w.steps, w.alpha, sample=idx, parallel=True)


VARIED = G.ModelConfig("varied-256", 256, 4, 1024, 2, 2, 32000, ln_post=0, seed=1102, random_gamma=True,
                       weight_std=0.2)


@pytest.mark.parametrize("B", [1, 2])
def test_varied_output_chained_translate(torch_dev, B):
    """The path the latency benchmark times -- width 256, vocabulary 32000, two
    decoder layers: the two-stream kernel chain, the commit folded into the
    next step and the 4-tile logits kernel of the chain, replayed from a graph
    -- on a model whose greedy outputs vary from step to step (the workload
    model repeats its input token), against the oracle's tokens and the bits
    of every step's maximum logit."""
    torch, dev = torch_dev
    src, lens = G.make_sources(VARIED.vocab, B, [30, 17][:B], seed=90 + B, s_max=30)
    out = _greedy_check(torch, dev, VARIED, src, lens, 30)
    for b in range(B):
        assert len(set(out[b].tolist())) >= 4, "the varied model should not repeat one token"


def test_beam_session_rejects_decode_step(torch_dev):
    torch, dev = torch_dev
    from paper_2306_04235_amd import mnmt

    _, gm = _pair("TINY")
    sess = mnmt.Session(gm, 2, 8, 4, 2)
    src = torch.full((2, 8), 5, dtype=torch.int32, device=dev)
    lens = torch.full((2,), 8, dtype=torch.int32, device=dev)
    sess.encode(src, lens)
    with pytest.raises(mnmt.MnmtError) as e:
        sess.decode_step()
    assert e.value.status == mnmt.E_UNSUPPORTED
    sess.close()


def test_chain_error_word_marks_outputs(torch_dev):
    """A chained kernel whose bounded wait gives up sets the session's error
    word; here the host sets that word itself (no kernel waits in vain).  The
    next translations report length -1 until mnmt_session_status raises
    E_TIMEOUT and clears it."""
    torch, dev = torch_dev
    from paper_2306_04235_amd import mnmt

    om, gm = _pair("TINY")
    src, lens = G.workload_inputs(G.WORKLOADS["tiny"])
    o_out, o_len = om.greedy(src, lens, 16)
    sess = mnmt.Session(gm, 1, src.shape[1], 16, 1)
    ts, tl = _t(torch, dev, src), _t(torch, dev, lens)
    sess.status()
    err = sess.tensor("chain_err", torch.int32, (1,))
    err.fill_(1)
    torch.cuda.synchronize()
    for use_graph in (False, True):
        out, out_len, _ = sess.translate(ts, tl, beam=1, max_steps=16, use_graph=use_graph)
        torch.cuda.synchronize()
        assert int(out_len.cpu()[0]) == -1
    with pytest.raises(mnmt.MnmtError) as e:
        sess.status()
    assert e.value.status == mnmt.E_TIMEOUT
    out, out_len, _ = sess.translate(ts, tl, beam=1, max_steps=16, use_graph=True)
    torch.cuda.synchronize()
    assert np.array_equal(out.cpu().numpy(), o_out) and np.array_equal(out_len.cpu().numpy(), o_len)
    sess.status()
    sess.close()


def test_session_capacity_errors(torch_dev):
    torch, dev = torch_dev
    from paper_2306_04235_amd import mnmt

    _, gm = _pair("TINY")
    sess = mnmt.Session(gm, 2, 8, 4, 1)
    src = torch.full((3, 8), 5, dtype=torch.int32, device=dev)
    lens = torch.full((3,), 8, dtype=torch.int32, device=dev)
    with pytest.raises(mnmt.MnmtError) as e:
        sess.translate(src, lens, max_steps=4)
    assert e.value.status == mnmt.E_CAPACITY
    with pytest.raises(mnmt.MnmtError) as e:
        sess.translate(src[:2], lens[:2], max_steps=5)
    assert e.value.status == mnmt.E_CAPACITY
    with pytest.raises(mnmt.MnmtError) as e:
        mnmt.Session(gm, 1, 8, 4, 9)  # beam above the supported width
    assert e.value.status == mnmt.E_INVALID_ARG
    sess.encode(src[:1], lens[:1])
    for _ in range(4):
        sess.decode_step()
    with pytest.raises(mnmt.MnmtError) as e:
        sess.decode_step()
    assert e.value.status == mnmt.E_CAPACITY
    sess.close()


def test_session_over_memory_of_queued_work(torch_dev):
    """A session whose workspace takes memory that kernels queued earlier still
    write (freed and handed out again in stream order): it starts after them."""
    import ctypes

    torch, dev = torch_dev
    from paper_2306_04235_amd import mnmt

    cfg = ROWS[2]
    om, gm = _pair(cfg)
    src, lens = G.make_sources(cfg.vocab, 5, [67, 64, 65, 1, 30], seed=311, s_max=67)
    ts, tl = _t(torch, dev, src), _t(torch, dev, lens)
    o_out, o_len = om.greedy(src, lens, 6)[:2]
    n = ctypes.c_size_t()
    sc = mnmt.SessionCfg(5, 67, 6, 1)
    assert mnmt.lib().mnmt_session_bytes(gm.handle, ctypes.byref(sc), ctypes.byref(n)) == 0
    old = torch.empty(n.value, dtype=torch.uint8, device=dev)
    work = torch.empty(1 << 28, dtype=torch.uint8, device=dev)
    torch.cuda.synchronize()
    for k in range(50):
        work.fill_(k)
    old.fill_(0x5A)
    del old  # (the allocator hands the block out again for an equal size)
    sess = mnmt.Session(gm, 5, 67, 6, 1)
    out, out_len, _ = sess.translate(ts, tl, max_steps=6)
    torch.cuda.synchronize()
    assert np.array_equal(out.cpu().numpy(), o_out) and np.array_equal(out_len.cpu().numpy(), o_len)
    sess.close()


OPER = G.ModelConfig("oper-256", 256, 4, 768, 2, 2, 300, ln_post=0, seed=321, random_gamma=True, weight_std=0.1)


@pytest.mark.parametrize("cfg,B", [(ROWS[2], 12), (ROWS[5], 5), (ROWS[8], 5), (FACTOR, 12), (OPER, 12)],
                         ids=lambda v: getattr(v, "name", str(v)))
def test_replayed_decode_step(torch_dev, cfg, B):
    """One decode step captured in the caller's graph decodes the next position
    at each replay (the step index lives in device memory): logits of every
    step against the oracle, with eager work of the caller between replays."""
    torch, dev = torch_dev
    from paper_2306_04235_amd import mnmt

    om, gm = _pair(cfg)
    steps = 7
    src, lens = G.make_sources(cfg.vocab, B, (2, 20), seed=322, s_max=20)
    o_out, _, o_logits = om.greedy(src, lens, steps, want_logits=True)
    sess = mnmt.Session(gm, B, 20, steps, 1)
    ts, tl = _t(torch, dev, src), _t(torch, dev, lens)
    sess.encode(ts, tl)
    sess.decode_step()  # (the first call outside a capture)
    sess.encode(ts, tl)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        nxt, logits = sess.decode_step(want_logits=True)
    other = torch.ones(1000, device=dev)
    for t in range(steps):
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(nxt.cpu().numpy(), o_out[:, t]), f"tokens of step {t}"
        ref = np.ascontiguousarray(o_logits[:, t])
        assert np.array_equal(logits.cpu().numpy().view(np.uint32), ref.view(np.uint32)), f"logits of step {t}"
        other.mul_(1.01)
    sess.close()


@pytest.mark.parametrize("B", [2, 70])
def test_lengths_outside_the_range_are_clamped(torch_dev, B):
    """Source lengths below 1 read as 1 and above S as S, in the small and the
    row-wise encoder: the same bytes as with the clamped lengths (the buffers
    hold another batch's rows before, so that a row left out shows)."""
    torch, dev = torch_dev
    from paper_2306_04235_amd import mnmt

    cfg = ROWS[2]
    _, gm = _pair(cfg)
    S, d = 16, cfg.d_model
    rng = np.random.Generator(np.random.PCG64(323))
    lens = rng.integers(1, S + 1, B).astype(np.int32)
    lens[:2] = [0, S + 9]
    if B > 8:
        lens[4:8] = [-5, -2**31, 2**31 - 1, 0]
    ok = np.clip(lens, 1, S).astype(np.int32)
    src, _ = G.make_sources(cfg.vocab, B, [S] * B, seed=324, s_max=S)
    other, _ = G.make_sources(cfg.vocab, B, [S] * B, seed=325, s_max=S)
    out = []
    for n in (ok, lens):
        sess = mnmt.Session(gm, B, S, 2, 1)
        sess.encode(_t(torch, dev, other), _t(torch, dev, np.full(B, S, np.int32)))
        sess.encode(_t(torch, dev, src), _t(torch, dev, n))
        nxt, z = sess.decode_step(want_logits=True)
        enc = sess.tensor("cross_kv.0", torch.int8, (B, S, 2 * d)).cpu().numpy()
        out.append((np.concatenate([enc[b, : ok[b]] for b in range(B)]), nxt.cpu().numpy(), z.cpu().numpy()))
        sess.close()
    for a, b in zip(*out):
        assert np.array_equal(a, b)


def test_sessions_share_copies_of_shared_layers(torch_dev):
    """A batch session's copies of the layers' weights: layers that share
    parameters share them, in the encoder too (pre- and post-LN), and the
    results are those of the same model with every layer written out."""
    import ctypes

    from tests.test_oracle_model import _unshare

    torch, dev = torch_dev
    from paper_2306_04235_amd import mnmt

    base = dataclasses.replace(SHARED_256, vocab=500, n_enc=6, n_dec=3)
    for post in (0, 1):
        blob = G.build_model(dataclasses.replace(base, name=f"shared-copies-{post}", ln_post=post))
        models = [mnmt.Model(blob), mnmt.Model(_unshare(blob))]
        src, lens = G.make_sources(500, 5, (3, 30), seed=326, s_max=30)
        sizes, outs = [], []
        for m in models:
            n = ctypes.c_size_t()
            sc = mnmt.SessionCfg(5, 30, 8, 1)
            assert mnmt.lib().mnmt_session_bytes(m.handle, ctypes.byref(sc), ctypes.byref(n)) == 0
            sizes.append(n.value)
            sess = mnmt.Session(m, 5, 30, 8, 1)
            out = sess.translate(_t(torch, dev, src), _t(torch, dev, lens), max_steps=8)
            keys = sess.tensor("out_key", torch.int64, (8, 5))
            torch.cuda.synchronize()
            outs.append((out[0].cpu().numpy(), keys.cpu().numpy()))
            sess.close()
        d, F = base.d_model, base.d_ffn
        enc, dec = 4 * d * d + 2 * d * F, 6 * d * d + 2 * d * F  # weights of a pass and of a decoder layer
        # 7 encoder passes against 4 (two ends, (0, 1), (1, 0)); 3 decoder layers against 2 (post-LN: 3)
        saved = 3 * enc + (0 if post else dec)
        assert saved <= sizes[1] - sizes[0] < saved + 4 * 65536
        assert all(np.array_equal(a, b) for a, b in zip(*outs))
        for m in models:
            m.close()


@pytest.mark.parametrize("cfg,B,steps", [
    (ROWS[5], 4090, 3), (ROWS[4], 4090, 3), (ROWS[6], 3070, 3), (ROWS[9], 2050, 3), (ROWS[8], 1300, 3),
    (ROWS[2], 2000, 3), (ROWS[0], 1020, 4),  # 16, 16, 12, 9, 6, 8 and 4 rows per block
    (ROWS[9], 4090, 200),  # 16 rows per block, from 128 positions on 8 (LDS)
], ids=lambda v: getattr(v, "name", str(v)))
def test_row_wise_decoder_many_rows_per_block(torch_dev, cfg, B, steps):
    """Greedy search with up to 16 rows per block and a last block that is not
    full: a sample of sentences from all over the batch against the oracle,
    and the logits of single steps (whose launches are laid out for the
    longest target)."""
    torch, dev = torch_dev
    from paper_2306_04235_amd import mnmt

    om, gm = _pair(cfg)
    src, lens = G.make_sources(cfg.vocab, B, (1, 9), seed=327, s_max=9)
    idx = np.unique(np.concatenate([[0, 15, 16, B // 2, B - 11, B - 1],
                                    np.random.default_rng(B).integers(0, B, 24 if steps < 10 else 2)]))
    print(f"greedy {cfg.name} B={B} steps={steps}", flush=True)
    o_out, _, o_logits = om.greedy(src[idx], lens[idx], steps, want_logits=True)
    sess = mnmt.Session(gm, B, 9, steps, 1)
    ts, tl = _t(torch, dev, src), _t(torch, dev, lens)
    at = torch.from_numpy(idx).to(dev)
    out, _, _ = sess.translate(ts, tl, max_steps=steps)
    assert np.array_equal(out[at].cpu().numpy(), o_out)
    sess.encode(ts, tl)
    for t in range(3):
        nxt, z = sess.decode_step(want_logits=True)
        assert np.array_equal(nxt[at].cpu().numpy(), o_out[:, t])
        ref = np.ascontiguousarray(o_logits[:, t])
        assert np.array_equal(z[at].cpu().numpy().view(np.uint32), ref.view(np.uint32)), f"logits of step {t}"
    sess.close()


@pytest.mark.parametrize("i,B,W", [(5, 511, 8), (9, 300, 7)])
def test_row_wise_decoder_many_rows_per_block_beam(torch_dev, i, B, W):
    """Beam search with 16 and 9 rows per block, blocks that cross sentences."""
    torch, dev = torch_dev
    src, lens = G.make_sources(ROWS[i].vocab, B, (1, 9), seed=328, s_max=9)
    idx = np.unique(np.concatenate([[0, 1, B // 2, B - 1], np.random.default_rng(B).integers(0, B, 12)]))
    _beam_check(torch, dev, ROWS[i], src, lens, W, 5, 0.6, sample=idx)


FEW_ROWS = [
    dataclasses.replace(ROWS[9], name="few-512-2048", w_bits=8), ROWS[9], ROWS[8],
    dataclasses.replace(ROWS[9], name="few-512-2048-post", w_bits=8, ln_post=1),
    dataclasses.replace(ROWS[8], name="few-512-1024-post-w4", w_bits=4, ln_post=1), ROWS[6],
]


@pytest.mark.parametrize("cfg", FEW_ROWS, ids=lambda c: c.name)
def test_few_rows_of_wide_models(torch_dev, cfg):
    """Rows on both sides of the line between the row-wise decoder and the
    launches per operator: greedy search of 3, 4 and 5 rows, beam search of one
    sentence with 2 to 4 hypotheses, widths 384 and 512, both feed-forward
    ratios, int8 and 4-bit, pre- and post-LN."""
    torch, dev = torch_dev
    for B in (3, 4, 5):
        src, lens = G.make_sources(cfg.vocab, B, (2, 14), seed=330 + B, s_max=14)
        _greedy_check(torch, dev, cfg, src, lens, 6)
    for W in (2, 3, 4):
        src, lens = G.make_sources(cfg.vocab, 1, [11], seed=340 + W, s_max=11)
        _beam_check(torch, dev, cfg, src, lens, W, 7, 0.6)


# shapes the row-wise kernels do not take (feed-forward neither 2 nor 4 times
# the width), which run operator by operator
OPER_128 = G.ModelConfig("oper-128", 128, 4, 384, 2, 3, 700, ln_post=0, seed=351, random_gamma=True, weight_std=0.1)
OPER_64_POST = G.ModelConfig("oper-64-post", 64, 4, 192, 2, 2, 300, ln_post=1, seed=352, random_gamma=True,
                             weight_std=0.1)
OPER_512 = G.ModelConfig("oper-512", 512, 8, 1536, 2, 2, 300, ln_post=0, seed=353, random_gamma=True, weight_std=0.05)


def _w4(cfg):
    return dataclasses.replace(cfg, name=cfg.name + "-w4", w_bits=4)


@pytest.mark.parametrize("cfg", [OPER, OPER_128, _w4(OPER), _w4(OPER_128)], ids=lambda c: c.name)
def test_operator_path_layernorm_forms(torch_dev, monkeypatch, cfg):
    """Pre-LN beam search above 64 rows, operator by operator, at widths 128
    and 256: the LayerNorms in the prologue of the kernels they feed and, with
    MNMT_LN_FUSED=0, as kernels of their own; the self-attention computing its
    rows' Q/K/V and, with MNMT_QKV_FUSED=0, the projection as a GEMM; 2 to 8
    hypotheses, up to 128 and 256 target positions; 4-bit weights read
    packed."""
    from paper_2306_04235_amd import mnmt

    torch, dev = torch_dev
    flags = mnmt.LOAD_PACKED_4BIT_ONLY if cfg.w_bits == 4 else 0
    src, lens = G.make_sources(cfg.vocab, 19, (2, 24), seed=354, s_max=24)
    for ln, qkv in (("1", "1"), ("0", "1"), ("1", "0")):
        monkeypatch.setenv("MNMT_LN_FUSED", ln)
        monkeypatch.setenv("MNMT_QKV_FUSED", qkv)
        _beam_check(torch, dev, cfg, src, lens, 4, 12, 0.6, parallel=True, flags=flags)
    monkeypatch.setenv("MNMT_QKV_FUSED", "1")
    for B, W in ((9, 8), (40, 2)):
        src, lens = G.make_sources(cfg.vocab, B, (2, 24), seed=355 + W, s_max=24)
        _beam_check(torch, dev, cfg, src, lens, W, 8, 0.6, parallel=True, flags=flags)
    src, lens = G.make_sources(cfg.vocab, 17, (1, 40), seed=364, s_max=40)
    for steps in (100, 140):
        _beam_check(torch, dev, cfg, src, lens, 4, steps, 0.6, sample=range(0, 17, 4), parallel=True, flags=flags)


@pytest.mark.parametrize("cfg", [OPER, OPER_128, OPER_64_POST, OPER_512, _w4(OPER)], ids=lambda c: c.name)
def test_operator_path_greedy(torch_dev, cfg):
    """Greedy search operator by operator: 3 to 8 rows (the LayerNorm in the
    GEMV), 12 rows (the matrix cores), and the encoder above 64 rows."""
    torch, dev = torch_dev
    for B in (3, 5, 8, 12):
        src, lens = G.make_sources(cfg.vocab, B, (2, 30), seed=370 + B, s_max=30)
        _greedy_check(torch, dev, cfg, src, lens, 7)
