"""GPU edge cases of the rollout path, each checked against the CPU oracle or
against the state the library reports: empty calls, prompts of one token and at
KV-block boundaries, ragged decode batches (a different subset of sequences
each step), sequence ids reused after termination, KV-pool exhaustion and the
max_seq_len limit during decode, and a weight update with nothing in flight."""
import numpy as np
import pytest

from paper_2505_24298_amd import synth

pytestmark = pytest.mark.gpu

LOGIT_TOL = 2e-2
LOGP_TOL = 1e-2


@pytest.fixture(scope="module")
def torch():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    return torch


@pytest.fixture(scope="module")
def binding():
    from paper_2505_24298_amd import binding
    binding.lib()
    return binding


def _f16(a):
    return np.asarray(a, dtype=np.float32).astype(np.float16).astype(np.float32)


def _f16_weights(w):
    out = dict(embed=_f16(w["embed"]), lm_head=_f16(w["lm_head"]), final_norm=_f16(w["final_norm"]),
               layers=[])
    for lw in w["layers"]:
        out["layers"].append({k: _f16(v) for k, v in lw.items()})
    return out


def _engine(binding, cfg, w, **kw):
    args = dict(max_seqs=8, max_seq_len=96, max_batch_tokens=64, kv_blocks=64, convert_weights=True)
    args.update(kw)
    eng = binding.Areal(cfg, **args)
    eng.load_weights(binding.weights_to_device(w, bf16=False), 0)
    return eng


def _oracle(cfg, w, seed=0):
    from oracle import rollout
    return rollout.RolloutWorker(cfg, _f16_weights(w), version=0, seed=seed)


def _check_step(torch, eng, wk, ids, logits, seed=0):
    """Compare the GPU logits for the next token of `ids` with the oracle's, let
    the oracle draw, force its tokens on the GPU sampler; returns the tokens."""
    positions = [len(wk.tokens[s]) for s in ids]
    ref_logits, ref_tok = wk.step(ids)
    got = logits.cpu().numpy()
    assert np.abs(got - ref_logits).max() <= LOGIT_TOL
    forced = torch.from_numpy(ref_tok).to(logits.device)
    toks, lb, lf = eng.sample_logprob(logits, ids, positions, 1.0, 1.0, seed, forced_tokens=forced)
    ref_lb = np.array([wk.logp_behav[s][-1] for s in ids])
    assert np.abs(lb.cpu().numpy() - ref_lb).max() <= LOGP_TOL
    return toks


def test_empty_calls_are_noops(torch, binding):
    cfg = synth.shape("tiny")
    w = synth.make_weights(cfg, 0)
    eng = _engine(binding, cfg, w)
    before = eng.kv_blocks()
    lg = eng.prefill([], [])
    assert tuple(lg.shape) == (0, cfg["vocab"])
    empty_tok = torch.zeros(0, dtype=torch.int32, device="cuda")
    lg = eng.decode_step([], empty_tok)
    assert tuple(lg.shape) == (0, cfg["vocab"])
    t, lb, lf = eng.sample_logprob(torch.zeros((0, cfg["vocab"]), device="cuda"), [], [])
    assert t.numel() == 0 and lb.numel() == 0
    assert eng.kv_blocks() == before
    # the context still works afterwards
    wk = _oracle(cfg, w)
    p = synth.make_prompts(cfg, 1, 1, 9, 9, seed=1)
    wk.add(0, p[0])
    _check_step(torch, eng, wk, [0], eng.prefill([0], p))
    eng.close()


def test_prompts_of_one_token_and_at_block_boundaries(torch, binding):
    """Prompt lengths 1, 15, 16, 17, 31, 32, 33 (KV blocks hold 16 tokens); 20
    generated tokens take every sequence across at least one block boundary."""
    cfg = synth.shape("tiny")
    w = synth.make_weights(cfg, 11)
    lens = [1, 15, 16, 17, 31, 32, 33]
    rng = np.random.default_rng(3)
    prompts = [rng.integers(0, cfg["vocab"], size=n).astype(np.int32) for n in lens]
    ids = list(range(len(lens)))
    eng = _engine(binding, cfg, w, max_batch_tokens=48)
    wk = _oracle(cfg, w)
    for s, p in zip(ids, prompts):
        wk.add(s, p)
    logits = eng.prefill(ids, prompts)
    for _ in range(20):
        toks = _check_step(torch, eng, wk, ids, logits)
        logits = eng.decode_step(ids, toks)
    for s in ids:
        assert eng.seq_len(s) == lens[s] + 20
        assert eng.get_tokens(s).tolist() == wk.tokens[s]
    total, free = eng.kv_blocks()
    assert total - free == sum((n + 20 + 15) // 16 for n in lens)
    eng.close()


def test_ragged_decode_batches(torch, binding):
    """Each step decodes a different subset of the live sequences, in a
    different order: rows of a pass are independent of their position in it."""
    cfg = synth.shape("tiny")
    w = synth.make_weights(cfg, 12)
    prompts = synth.make_prompts(cfg, 5, 1, 5, 40, seed=8)
    ids = [4, 1, 3, 0, 2]
    eng = _engine(binding, cfg, w)
    wk = _oracle(cfg, w)
    for s, p in zip(ids, prompts):
        wk.add(s, p)
    first = eng.prefill(ids, prompts)
    # every sequence must take its first token from the prefill logits
    toks = _check_step(torch, eng, wk, ids, first)
    pending = {s: toks[i:i + 1] for i, s in enumerate(ids)}       # sampled, not yet appended
    rng = np.random.default_rng(5)
    for step in range(12):
        k = int(rng.integers(1, len(ids) + 1))
        subset = [int(s) for s in rng.permutation(ids)[:k]]
        tok_in = torch.cat([pending[s] for s in subset])
        logits = eng.decode_step(subset, tok_in)
        toks = _check_step(torch, eng, wk, subset, logits)
        for i, s in enumerate(subset):
            pending[s] = toks[i:i + 1]
    for s in ids:
        assert eng.get_tokens(s).tolist() == wk.tokens[s][:-1]   # the last draw is still pending
    eng.close()


def test_sequence_id_reuse_after_termination(torch, binding):
    cfg = synth.shape("tiny")
    w = synth.make_weights(cfg, 13)
    pa, pb = synth.make_prompts(cfg, 2, 1, 20, 40, seed=4)
    eng = _engine(binding, cfg, w, max_seqs=2, kv_blocks=8)
    wk = _oracle(cfg, w)
    wk.add(0, pa)
    logits = eng.prefill([0], [pa])
    for _ in range(5):
        toks = _check_step(torch, eng, wk, [0], logits)
        logits = eng.decode_step([0], toks)
    eng.free_seq(0)
    assert eng.seq_len(0) == -1 and eng.kv_blocks() == (8, 8)
    with pytest.raises(binding.ArealError) as e:
        eng.decode_step([0], toks)                                # terminated
    assert e.value.code == binding.E_STATE
    wk2 = _oracle(cfg, w)
    wk2.add(0, pb)
    logits = eng.prefill([0], [pb])                               # same id, new prompt
    for _ in range(5):
        toks = _check_step(torch, eng, wk2, [0], logits)
        logits = eng.decode_step([0], toks)
    assert eng.get_tokens(0).tolist() == wk2.tokens[0]
    v = eng.get_versions(0)
    assert v.tolist() == [-1] * len(pb) + [0] * 5
    eng.close()


def test_kv_exhaustion_during_decode_leaves_state(torch, binding):
    cfg = synth.shape("tiny")
    w = synth.make_weights(cfg, 14)
    rng = np.random.default_rng(6)
    prompts = [rng.integers(0, cfg["vocab"], size=16).astype(np.int32) for _ in range(2)]
    eng = _engine(binding, cfg, w, kv_blocks=3)                   # 2 blocks taken by the prompts
    wk = _oracle(cfg, w)
    for s, p in enumerate(prompts):
        wk.add(s, p)
    logits = eng.prefill([0, 1], prompts)
    toks = _check_step(torch, eng, wk, [0, 1], logits)
    with pytest.raises(binding.ArealError) as e:
        eng.decode_step([0, 1], toks)                             # both need a second block, one is free
    assert e.value.code == binding.E_NOMEM
    assert eng.seq_len(0) == 16 and eng.seq_len(1) == 16 and eng.kv_blocks() == (3, 1)
    eng.free_seq(1)
    logits = eng.decode_step([0], toks[:1])                       # now it fits
    assert eng.seq_len(0) == 17
    wk.finish(1)
    _check_step(torch, eng, wk, [0], logits)
    eng.close()


def test_max_seq_len_limit(torch, binding):
    cfg = synth.shape("tiny")
    w = synth.make_weights(cfg, 15)
    p = synth.make_prompts(cfg, 1, 1, 30, 30, seed=2)
    eng = _engine(binding, cfg, w, max_seq_len=32)
    wk = _oracle(cfg, w)
    wk.add(0, p[0])
    with pytest.raises(binding.ArealError) as e:
        eng.prefill([1], [np.zeros(33, dtype=np.int32)])          # longer than max_seq_len
    assert e.value.code == binding.E_NOMEM and eng.seq_len(1) == -1
    logits = eng.prefill([0], p)
    for _ in range(2):                                            # positions 30 and 31: the last two
        toks = _check_step(torch, eng, wk, [0], logits)
        logits = eng.decode_step([0], toks)
    assert eng.seq_len(0) == 32
    toks = _check_step(torch, eng, wk, [0], logits)               # logits at full length are still right
    with pytest.raises(binding.ArealError) as e:
        eng.decode_step([0], toks)
    assert e.value.code == binding.E_NOMEM and eng.seq_len(0) == 32
    eng.close()


def test_weight_update_with_nothing_in_flight(torch, binding):
    cfg = synth.shape("tiny")
    w = synth.make_weights(cfg, 16)
    w2 = synth.perturb_weights(w, 1001, scale=5e-3, round_bf16=False)
    eng = _engine(binding, cfg, w)
    live, logits, retok = eng.update_weights_interrupt(binding.weights_to_device(w2, bf16=False), 7)
    assert live.tolist() == [] and retok == 0
    with pytest.raises(binding.ArealError) as e:                  # versions only go up
        eng.update_weights_interrupt(binding.weights_to_device(w, bf16=False), 7)
    assert e.value.code == binding.E_STATE
    from oracle import rollout
    wk = rollout.RolloutWorker(cfg, _f16_weights(w2), version=7, seed=0)
    p = synth.make_prompts(cfg, 2, 1, 10, 20, seed=9)
    for s in (0, 1):
        wk.add(s, p[s])
    logits = eng.prefill([0, 1], p)                               # runs under the new weights
    toks = _check_step(torch, eng, wk, [0, 1], logits)
    eng.decode_step([0, 1], toks)
    assert eng.get_versions(0)[-1] == 7
    eng.close()


def test_pending_token_keeps_the_old_version_across_a_weight_update(torch, binding):
    """A weight update that lands between sampling and the decode step: the sampled tokens
    join their sequences through areal_append_tokens (old version tag, no forward pass), the
    update recomputes every prefix with them, and the logits that follow are the oracle's
    under the new weights.  A decode step on a sequence with an appended token and no
    update is refused.  Sequences cross a KV-block boundary with the appended token."""
    cfg = synth.shape("tiny")
    w = synth.make_weights(cfg, 21)
    w2 = synth.perturb_weights(w, 1002, scale=5e-3, round_bf16=False)
    eng = _engine(binding, cfg, w)
    wk = _oracle(cfg, w)
    prompts = [np.arange(5, 5 + n, dtype=np.int32) for n in (16, 31, 9)]     # the 17th / 32nd token opens a block
    ids = [0, 1, 2]
    for s, p in zip(ids, prompts):
        wk.add(s, p)
    logits = eng.prefill(ids, prompts)
    toks = _check_step(torch, eng, wk, ids, logits)              # sampled under version 0, not yet appended
    free_before = eng.kv_blocks()[1]
    eng.append_tokens(ids, toks)
    assert eng.kv_blocks()[1] == free_before - 1                 # sequence 0 opened its second block
    with pytest.raises(binding.ArealError) as e:
        eng.decode_step(ids, toks)
    assert e.value.code == binding.E_STATE
    wk.update_weights(_f16_weights(w2), 3)
    live, logits, retok = eng.update_weights_interrupt(binding.weights_to_device(w2, bf16=False), 3)
    assert live.tolist() == ids and retok == sum(len(wk.tokens[s]) for s in ids)
    for step in range(3):
        toks = _check_step(torch, eng, wk, ids, logits.contiguous())
        logits = eng.decode_step(ids, toks)
    for s in ids:
        assert eng.get_tokens(s).tolist() == wk.tokens[s]
        v = eng.get_versions(s)
        assert v[len(prompts[s]):].tolist() == [0, 3, 3, 3] == wk.versions[s]
    eng.close()


def test_shared_prompt_prefix_with_interrupt_and_early_termination(torch, binding):
    """Four samples of each of two prompts (lengths 37 and 48: the second ends on
    a block boundary) admitted in one call: the samples share the prompt's full
    KV blocks.  The first sample of a prompt (whose rows computed the shared
    blocks) terminates early; a weight update then recomputes every live prefix,
    the shared part once; decoding goes on.  Logits against the oracle throughout."""
    from oracle import rollout
    cfg = synth.shape("tiny")
    w = synth.make_weights(cfg, 31)
    w2 = synth.perturb_weights(w, 1002, scale=5e-3, round_bf16=False)
    rng = np.random.default_rng(12)
    base = [rng.integers(0, cfg["vocab"], size=n).astype(np.int32) for n in (37, 48)]
    prompts = [base[0]] * 4 + [base[1]] * 4
    ids = list(range(8))
    eng = _engine(binding, cfg, w, kv_blocks=40)
    wk = _oracle(cfg, w)
    for s, p in zip(ids, prompts):
        wk.add(s, p)
    logits = eng.prefill(ids, prompts)
    # 37 tokens: 3 blocks, 2 shared; 48 tokens: 3 blocks, 2 shared (one fewer than full)
    total, free = eng.kv_blocks()
    assert total - free == (3 + 3 * 1) + (3 + 3 * 1)
    for s in ids:
        assert eng.get_tokens(s).tolist() == prompts[s].tolist()
    live = list(ids)
    for step in range(20):
        toks = _check_step(torch, eng, wk, live, logits)
        if step == 3:                                  # the samples that computed the shared blocks leave
            for s in (0, 4):
                eng.free_seq(s)
                wk.finish(s)
            keep = [i for i, s in enumerate(live) if s not in (0, 4)]
            toks = toks[torch.tensor(keep, device=toks.device)].contiguous()
            live = [s for s in live if s not in (0, 4)]
        logits = eng.decode_step(live, toks)
        if step == 9:
            wk.update_weights(_f16_weights(w2), 1)
            got_live, logits, retok = eng.update_weights_interrupt(binding.weights_to_device(w2, bf16=False), 1)
            assert got_live.tolist() == live
            # each prompt's 32 shared positions are recomputed once, not three times
            assert retok == sum(len(wk.tokens[s]) for s in live) - 2 * 2 * 32
    for s in live:
        assert eng.get_tokens(s).tolist() == wk.tokens[s][:-1] or eng.get_tokens(s).tolist() == wk.tokens[s]
    for s in live:
        eng.free_seq(s)
    assert eng.kv_blocks() == (40, 40)
    eng.close()


def test_prompt_blocks_shared_across_prefill_calls(torch, binding):
    """The streaming regime admits the samples of a prompt one by one: a sequence whose prompt
    equals that of a sequence still live from an earlier call holds that sequence's prompt
    blocks and computes only the rest.  The first holder then terminates (its blocks stay with
    the others), a third sample arrives and shares with the second, a weight update recomputes
    the shared part once, a sequence with a different prompt of the same length shares nothing.
    Logits against the oracle throughout; block accounting at every step."""
    cfg = synth.shape("tiny")
    w = synth.make_weights(cfg, 33)
    w2 = synth.perturb_weights(w, 1004, scale=5e-3, round_bf16=False)
    rng = np.random.default_rng(14)
    P = rng.integers(0, cfg["vocab"], size=53).astype(np.int32)           # 4 blocks, 3 shared
    Q = P.copy()
    Q[20] = (Q[20] + 1) % cfg["vocab"]                                    # same length, one token differs
    eng = _engine(binding, cfg, w, kv_blocks=40)
    wk = _oracle(cfg, w)
    used = lambda: eng.kv_blocks()[0] - eng.kv_blocks()[1]
    wk.add(0, P)
    logits0 = eng.prefill([0], [P])
    assert used() == 4
    toks = _check_step(torch, eng, wk, [0], logits0)
    logits0 = eng.decode_step([0], toks)
    # second sample of P in a later call, together with a different prompt
    wk.add(1, P)
    wk.add(2, Q)
    lg = eng.prefill([1, 2], [P, Q])
    assert used() == 4 + 1 + 4                                            # 1: only its last block; 2: all four
    assert eng.get_tokens(1).tolist() == P.tolist()
    toks = _check_step(torch, eng, wk, [1, 2], lg)
    lg12 = eng.decode_step([1, 2], toks)
    toks = _check_step(torch, eng, wk, [0], logits0)
    logits0 = eng.decode_step([0], toks)
    # the first holder terminates: the shared blocks stay with sequence 1
    eng.free_seq(0)
    wk.finish(0)
    assert used() == 3 + 1 + 4
    wk.add(3, P)
    wk.add(4, P)
    lg3 = eng.prefill([3, 4], [P, P])                                     # two more samples in one call: both
    assert used() == 3 + 1 + 4 + 1 + 1                                    # share with sequence 1
    assert eng.get_tokens(3).tolist() == P.tolist() == eng.get_tokens(4).tolist()
    toks3 = _check_step(torch, eng, wk, [3, 4], lg3)
    toks = _check_step(torch, eng, wk, [1, 2], lg12)
    eng.decode_step([1, 2], toks)
    eng.decode_step([3, 4], toks3)
    eng.free_seq(4)
    wk.finish(4)
    # weight update: the shared part is recomputed once (48 positions counted once)
    wk.update_weights(_f16_weights(w2), 1)
    live, logits, retok = eng.update_weights_interrupt(binding.weights_to_device(w2, bf16=False), 1)
    assert live.tolist() == [1, 2, 3]
    assert retok == sum(len(wk.tokens[s]) for s in (1, 2, 3)) - 48
    for step in range(3):
        toks = _check_step(torch, eng, wk, [1, 2, 3], logits.contiguous())
        logits = eng.decode_step([1, 2, 3], toks)
    for s in (1, 2, 3):
        assert eng.get_tokens(s).tolist() == wk.tokens[s]
        eng.free_seq(s)
    assert used() == 0
    # nothing stale in the index: the same prompt again computes everything
    wk2 = _oracle(cfg, w2)
    wk2.add(0, P)
    lg = eng.prefill([0], [P])
    assert used() == 4
    _check_step(torch, eng, wk2, [0], lg)
    eng.close()


def test_activations_beyond_the_half_range_saturate(torch, binding):
    """Gate/up weights scaled so that the SwiGLU output exceeds 65,504, the largest half-
    precision number: the values the kernels round to half on their way to the matrix cores
    (normalised activations, q / k / v, attention output, SwiGLU output) saturate instead of
    turning into infinities, so prefill and decode logits stay finite and the sampler still
    returns tokens of the vocabulary.  (Without saturation the first such value makes the
    residual row, and every logit after it, NaN.)"""
    cfg = synth.shape("tiny")
    w = synth.make_weights(cfg, 41)
    for lw in w["layers"]:
        lw["wgate"] = lw["wgate"] * np.float32(3000.0)
        lw["wup"] = lw["wup"] * np.float32(3000.0)
    # the products really leave the range: float64 SwiGLU of the first block's input
    from oracle import decoder
    x = decoder.rmsnorm(w["embed"][:64], w["layers"][0]["norm_ffn"], cfg["rms_eps"])
    act = decoder.silu(x @ _f16(w["layers"][0]["wgate"]).T.astype(np.float64)) * (
        x @ _f16(w["layers"][0]["wup"]).T.astype(np.float64))
    assert np.abs(act).max() > 10 * 65504.0
    eng = _engine(binding, cfg, w)
    prompts = synth.make_prompts(cfg, 3, 1, 20, 40, seed=42)
    ids = [0, 1, 2]
    logits = eng.prefill(ids, prompts)
    for step in range(4):
        assert bool(torch.isfinite(logits).all())
        toks, lb, lf = eng.sample_logprob(logits, ids, [len(p) + step for p in prompts], 1.0, 1.0, 3)
        t = toks.cpu().numpy()
        assert ((t >= 0) & (t < cfg["vocab"])).all() and bool(torch.isfinite(lb).all())
        logits = eng.decode_step(ids, toks)
    assert bool(torch.isfinite(logits).all())
    eng.close()


def test_half_precision_weights_in_place_and_tied_output_projection(torch, binding):
    """A context without the conversion workspace reads fp16 parameter sets where
    they are (also across a weight update); the output projection may be the
    embedding matrix itself; bf16 sets are refused by such a context."""
    from oracle import rollout
    cfg = synth.shape("tiny")
    w = synth.make_weights(cfg, 61, qkv_bias=True)
    w["lm_head"] = w["embed"]                                     # tied
    w2 = synth.perturb_weights(w, 1004, scale=5e-3, round_bf16=False)
    w2["lm_head"] = w2["embed"]
    eng = binding.Areal(cfg, max_seqs=4, max_seq_len=96, max_batch_tokens=64, kv_blocks=24,
                        convert_weights=False)
    with pytest.raises(binding.ArealError) as e:
        eng.load_weights(binding.weights_to_device(w, bf16=False), 0)     # float32 needs the workspace
    assert e.value.code == binding.E_INVAL
    dw = binding.weights_to_device(w, f16=True)
    dw["lm_head"] = dw["embed"]                                   # the same device tensor
    eng.load_weights(dw, 0)
    wk = rollout.RolloutWorker(cfg, _f16_weights(w), version=0, seed=0)
    prompts = synth.make_prompts(cfg, 3, 1, 10, 40, seed=13)
    ids = [0, 1, 2]
    for s, p in zip(ids, prompts):
        wk.add(s, p)
    logits = eng.prefill(ids, prompts)
    for step in range(10):
        toks = _check_step(torch, eng, wk, ids, logits)
        logits = eng.decode_step(ids, toks)
        if step == 4:
            dw2 = binding.weights_to_device(w2, f16=True)
            dw2["lm_head"] = dw2["embed"]
            wk.update_weights(_f16_weights(w2), 1)
            _, logits, _ = eng.update_weights_interrupt(dw2, 1)
    _check_step(torch, eng, wk, ids, logits)
    eng.close()


@pytest.mark.parametrize("at", [1, 2, 4, 8])
def test_gains_read_in_place_start_at_any_element(torch, binding, at):
    """Half-precision gains anywhere in a larger buffer (`at` halves behind a 16-byte boundary), as views of a flat parameter
    buffer have them: steps of a few rows, whose products read them 16 bytes at a time, and a pass of many, against the oracle.
    Gains drawn between 0.5 and 1.5, so that a shift by one shows: logits of order 0.5, tolerance as stated."""
    from oracle import rollout
    cfg = synth.shape("tiny")
    w = synth.make_weights(cfg, 77, qkv_bias=True)
    rng = np.random.default_rng(at)
    gain = lambda: rng.uniform(0.5, 1.5, size=cfg["hidden"]).astype(np.float32)
    w["final_norm"] = gain()
    for lw in w["layers"]:
        lw["norm_attn"], lw["norm_ffn"] = gain(), gain()

    def moved(t):
        buf = torch.full((t.numel() + 64,), 7.0, dtype=t.dtype, device=t.device)
        buf[at:at + t.numel()] = t
        view = buf[at:at + t.numel()]
        assert view.data_ptr() % 16 == 2 * at % 16
        return view

    dw = binding.weights_to_device(w, f16=True)
    dw["final_norm"] = moved(dw["final_norm"])
    for lw in dw["layers"]:
        lw["norm_attn"], lw["norm_ffn"] = moved(lw["norm_attn"]), moved(lw["norm_ffn"])
    eng = binding.Areal(cfg, max_seqs=4, max_seq_len=96, max_batch_tokens=64, kv_blocks=24, convert_weights=False)
    eng.load_weights(dw, 0)
    wk = rollout.RolloutWorker(cfg, _f16_weights(w), version=0, seed=0)
    ids = [0, 1, 2]
    prompts = synth.make_prompts(cfg, 3, 1, 10, 40, seed=13)
    for s, p in zip(ids, prompts):
        wk.add(s, p)
    logits = eng.prefill(ids, prompts)
    for step in range(4):
        toks = _check_step(torch, eng, wk, ids, logits)
        logits = eng.decode_step(ids, toks)
        if step == 1:                     # one row from here on
            eng.free_seq(1)
            eng.free_seq(2)
            ids, logits = [0], logits[:1].contiguous()
    _check_step(torch, eng, wk, ids, logits)
    eng.close()
