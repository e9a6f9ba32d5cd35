"""CPU-only checks: the shared library loads, exports every symbol the headers
declare, and its host-side logic (KV allocator, pass planner, configuration
checks) behaves.  No GPU call is made."""
import ctypes as C
import os
import re

import numpy as np
import pytest

from paper_2505_24298_amd import binding, synth

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def L():
    return binding.lib()


@pytest.fixture(scope="module")
def HL():
    """Host-only entry points: from the main library, or from the sanitizer build when
    AREAL_HOST_LIB names it (test_host_logic_under_sanitizers runs this file that way)."""
    return binding.host_lib()


def _declared():
    names = set()
    for h in ("areal.h", "areal_host.h", "areal_ops.h"):
        src = open(os.path.join(ROOT, "include", h)).read()
        src = re.sub(r"/\*.*?\*/", "", src, flags=re.S)
        names |= set(re.findall(r"\b(areal_[a-z0-9_]+)\s*\(", src))
    return names


def test_every_declared_symbol_is_exported_and_bound(L):
    decl = _declared()
    assert {"areal_load_weights", "areal_prefill", "areal_decode_step",
            "areal_update_weights_interrupt", "areal_sample_logprob"} <= decl
    for n in decl:
        assert hasattr(L, n), n
    assert decl == set(binding._SIGNATURES)


def test_cfg_struct_matches_header_layout():
    # field order and widths as in areal_model_cfg
    assert [f[0] for f in binding.ModelCfg._fields_][:7] == [
        "n_layers", "hidden", "n_q_heads", "n_kv_heads", "head_dim", "ffn", "vocab"]
    assert C.sizeof(binding.ModelCfg) == 13 * 4 + 4 + 5 * 8     # 13 words, pad, 5 x 8 bytes


def test_workspace_and_block_bytes(L):
    cfg = binding.make_cfg(synth.shape("qwen2-1.5b"), 256, 8704, 8192, convert_weights=False)
    assert L.areal_kv_block_bytes(C.byref(cfg)) == 16 * 28672
    ws = L.areal_workspace_bytes(C.byref(cfg))
    assert 2 ** 20 < ws < 2 ** 31
    # space for a converted half-precision copy of a bf16 / float32 parameter set
    cfg_c = binding.make_cfg(synth.shape("qwen2-1.5b"), 256, 8704, 8192, convert_weights=True)
    extra = L.areal_workspace_bytes(C.byref(cfg_c)) - ws
    n_params = 1_543_656_960 + 151936 * 1536 + 28 * 1536      # + embedding, + second norm gain
    assert 2 * n_params <= extra <= 2 * n_params + 2 ** 20
    cfg7 = binding.make_cfg(synth.shape("qwen2-7b"), 64, 33792 + 16, 4096)
    assert L.areal_kv_block_bytes(C.byref(cfg7)) == 16 * 57344
    bad = binding.make_cfg(synth.shape("tiny", head_dim=48), 8, 128, 64)
    assert L.areal_workspace_bytes(C.byref(bad)) == 0
    bad = binding.make_cfg(synth.shape("tiny"), 8, 128, 4)        # fewer rows than sequences
    assert L.areal_workspace_bytes(C.byref(bad)) == 0


def test_create_rejects_bad_buffers_without_touching_the_gpu(L):
    cfg = binding.make_cfg(synth.shape("tiny"), 8, 128, 64)
    ctx = C.c_void_p()
    assert L.areal_create(C.byref(cfg), C.byref(ctx)) == binding.E_NOMEM     # no workspace
    assert b"workspace" in L.areal_last_error(None)
    assert L.areal_create(None, C.byref(ctx)) == binding.E_INVAL


# ------------------------------------------------------------- KV allocator
def _table(L, a, seq):
    buf = np.zeros(64, dtype=np.int32)
    n = L.areal_kvalloc_table(a, seq, buf.ctypes.data_as(binding._I32P), 64)
    return buf[:n].tolist()


def test_allocator_grows_on_block_boundaries_and_reuses(HL):
    L = HL
    a = L.areal_kvalloc_create(10, 4, 8)
    assert L.areal_kvalloc_free_blocks(a) == 10
    assert L.areal_kvalloc_reserve(a, 0, 16) == 0 and _table(L, a, 0) == [0]
    assert L.areal_kvalloc_reserve(a, 0, 16) == 0 and _table(L, a, 0) == [0]       # no growth
    assert L.areal_kvalloc_reserve(a, 0, 17) == 0 and _table(L, a, 0) == [0, 1]
    assert L.areal_kvalloc_reserve(a, 1, 40) == 0 and _table(L, a, 1) == [2, 3, 4]
    assert L.areal_kvalloc_free_blocks(a) == 5
    L.areal_kvalloc_release(a, 0)
    assert L.areal_kvalloc_free_blocks(a) == 7 and _table(L, a, 0) == []
    assert L.areal_kvalloc_reserve(a, 2, 33) == 0
    t2 = _table(L, a, 2)
    assert len(t2) == 3 and not set(t2) & set(_table(L, a, 1))
    L.areal_kvalloc_destroy(a)


def test_allocator_exhaustion_is_all_or_nothing(HL):
    L = HL
    a = L.areal_kvalloc_create(4, 2, 3)
    assert L.areal_kvalloc_reserve(a, 0, 3 * 16) == 0
    assert L.areal_kvalloc_reserve(a, 1, 2 * 16) == binding.E_NOMEM      # pool: 1 left, 2 needed
    assert _table(L, a, 1) == [] and L.areal_kvalloc_free_blocks(a) == 1
    assert L.areal_kvalloc_reserve(a, 0, 3 * 16 + 1) == binding.E_NOMEM  # per-sequence limit
    assert len(_table(L, a, 0)) == 3
    L.areal_kvalloc_destroy(a)


def test_allocator_never_leaks_or_double_books(HL):
    L = HL
    rng = np.random.default_rng(0)
    a = L.areal_kvalloc_create(200, 16, 40)
    L.areal_kvalloc_shuffle(a, 7)
    lens = [0] * 16
    for step in range(3000):
        s = int(rng.integers(0, 16))
        if lens[s] and rng.random() < 0.05:
            L.areal_kvalloc_release(a, s)
            lens[s] = 0
        else:
            want = lens[s] + int(rng.integers(1, 40))
            if L.areal_kvalloc_reserve(a, s, want) == 0:
                lens[s] = want
        tabs = [_table(L, a, q) for q in range(16)]
        flat = [b for t in tabs for b in t]
        assert len(flat) == len(set(flat))
        assert all(len(t) == -(-n // 16) for t, n in zip(tabs, lens))
        assert L.areal_kvalloc_free_blocks(a) == 200 - len(flat)
    for s in range(16):
        L.areal_kvalloc_release(a, s)
    assert L.areal_kvalloc_free_blocks(a) == 200
    L.areal_kvalloc_destroy(a)


# ------------------------------------------------------------- pass planner
def _plan(L, lens, max_rows):
    lens = np.asarray(lens, dtype=np.int32)
    out = np.zeros((1024, 6), dtype=np.int32)
    n = L.areal_plan_passes(len(lens), lens.ctypes.data_as(binding._I32P), max_rows,
                            out.ctypes.data_as(binding._I32P), 1024)
    return out[:n]

def test_planner_covers_every_position_once_in_order(HL):
    L = HL
    rng = np.random.default_rng(1)
    for trial in range(20):
        lens = rng.integers(1, 90, size=int(rng.integers(1, 12)))
        max_rows = int(rng.integers(8, 64))
        rec = _plan(L, lens, max_rows)
        rows_in_pass = {}
        nxt = [0] * len(lens)
        for p, span, pos0, ln, row0, out_index in rec:
            assert pos0 == nxt[span] and ln > 0
            nxt[span] += ln
            assert row0 == rows_in_pass.get(p, 0)
            rows_in_pass[p] = row0 + ln
            assert out_index == (span if nxt[span] == lens[span] else -1)
        assert nxt == lens.tolist()
        assert all(v <= max_rows for v in rows_in_pass.values())
        assert all(v == max_rows for k, v in rows_in_pass.items() if k != max(rows_in_pass))
        assert list(rec[:, 0]) == sorted(rec[:, 0]) and list(rec[:, 1]) == sorted(rec[:, 1])


def test_bench_refuses_more_than_one_gpu():
    """Every box has one GPU: bench.py --gpus N with N > 1 exits with a message
    before it touches the device."""
    import os
    import subprocess
    import sys
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, os.path.join(root, "bench.py"), "--gpus", "2"],
                       capture_output=True, text=True, timeout=120)
    assert r.returncode != 0 and "one MI355X" in r.stderr and r.stdout.strip() == ""


def test_host_logic_under_sanitizers():
    """The allocator, planner, gate and batching tests of this file once more, in a child
    process, against csrc/host_api.cpp built with -fsanitize=address,undefined (any report
    aborts the child)."""
    import subprocess
    import sys
    from paper_2505_24298_amd import build as b
    if os.environ.get("AREAL_HOST_LIB"):
        pytest.skip("already inside the sanitizer run")
    lib, runtimes = b.build_host_sanitized()
    assert runtimes, "sanitizer runtimes not found next to the host compiler"
    env = dict(os.environ, AREAL_HOST_LIB=lib, LD_PRELOAD=":".join(runtimes),
               ASAN_OPTIONS="detect_leaks=0:abort_on_error=1", UBSAN_OPTIONS="halt_on_error=1:print_stacktrace=1")
    r = subprocess.run([sys.executable, "-m", "pytest", os.path.abspath(__file__), "-q", "-x", "-p", "no:cacheprovider",
                        "-k", "allocator or planner or gate or kvalloc or dynamic_batching or stream"],
                       capture_output=True, text=True, env=env, cwd=ROOT, timeout=600)
    assert r.returncode == 0, r.stdout[-3000:] + r.stderr[-3000:]
    assert " passed" in r.stdout and "failed" not in r.stdout


def test_staleness_gate_matches_oracle_request_by_request():
    """The library's gate (budget form) against the oracle that applies the
    paper's inequality one request at a time, over random interleavings of
    submissions and version bumps, for every small (B, eta)."""
    from oracle import staleness
    L = binding.host_lib()
    rng = np.random.default_rng(3)
    for B in (1, 2, 5, 16):
        for eta in (0, 1, 4):
            g = L.areal_gate_create(B, eta)
            o = staleness.StalenessGate(B, eta)
            v = 0
            for _ in range(200):
                if rng.random() < 0.3:
                    v += int(rng.integers(0, 3))
                    assert L.areal_gate_set_version(g, v) == 0
                    o.set_version(v)
                n = int(rng.integers(0, 3 * B))
                assert L.areal_gate_budget(g) == _budget(o)
                assert L.areal_gate_submit(g, n) == o.submit(n)
                assert L.areal_gate_submitted(g) == o.submitted
            assert L.areal_gate_set_version(g, v - 1) == binding.E_STATE if v > 0 else True
            L.areal_gate_destroy(g)
    assert not L.areal_gate_create(0, 1) and not L.areal_gate_create(4, -1)


def _budget(o):
    """How many requests the oracle gate would admit now (on a copy)."""
    from oracle import staleness
    c = staleness.StalenessGate(o.B, o.eta, o.version)
    c.submitted = o.submitted
    return c.submit(10 ** 6)


def test_kvalloc_shared_prefix_refcounts():
    L = binding.host_lib()
    a = L.areal_kvalloc_create(10, 4, 8)
    assert L.areal_kvalloc_reserve(a, 0, 40) == 0 and _table(L, a, 0) == [0, 1, 2]
    assert L.areal_kvalloc_share(a, 1, 0, 2) == 0 and _table(L, a, 1) == [0, 1]
    assert L.areal_kvalloc_share(a, 2, 0, 2) == 0
    assert L.areal_kvalloc_share(a, 1, 0, 1) == binding.E_INVAL          # holder is not empty
    assert L.areal_kvalloc_share(a, 3, 0, 4) == binding.E_INVAL          # more than the source holds
    assert L.areal_kvalloc_reserve(a, 1, 40) == 0 and _table(L, a, 1) == [0, 1, 3]   # own third block
    assert L.areal_kvalloc_free_blocks(a) == 6
    L.areal_kvalloc_release(a, 0)                                        # the first holder leaves:
    assert L.areal_kvalloc_free_blocks(a) == 7                           # only its own block 2 returns
    L.areal_kvalloc_release(a, 1)
    assert L.areal_kvalloc_free_blocks(a) == 8                           # block 3; 0 and 1 still held by 2
    L.areal_kvalloc_release(a, 2)
    assert L.areal_kvalloc_free_blocks(a) == 10
    assert L.areal_kvalloc_reserve(a, 3, 160) == binding.E_NOMEM         # per-sequence limit 8 blocks
    assert L.areal_kvalloc_reserve(a, 3, 128) == 0 and len(set(_table(L, a, 3))) == 8
    L.areal_kvalloc_destroy(a)


def test_dynamic_batching_matches_oracle():
    """Algorithm 1 in the library against the oracle on random length sets
    (ties in length and in sequence count included) and on the edge cases."""
    from oracle import trainer_side
    L = binding.host_lib()
    rng = np.random.default_rng(11)
    for _ in range(200):
        n = int(rng.integers(0, 60))
        lens = rng.integers(1, 30, size=n).astype(np.int32)
        cap, k = int(rng.integers(10, 90)), int(rng.integers(1, 7))
        out = np.full(n, -1, dtype=np.int32)
        nb = L.areal_dynamic_batching(n, lens.ctypes.data_as(binding._I32P), cap, k,
                                      out.ctypes.data_as(binding._I32P))
        want = trainer_side.dynamic_batching(lens, cap, k)
        assert nb == len(want)
        for b, members in enumerate(want):
            assert sorted(np.nonzero(out == b)[0].tolist()) == sorted(members)
    bad = np.array([3, 0], dtype=np.int32)
    o = np.zeros(2, dtype=np.int32)
    assert L.areal_dynamic_batching(2, bad.ctypes.data_as(binding._I32P), 10, 1,
                                    o.ctypes.data_as(binding._I32P)) == binding.E_INVAL
    assert L.areal_dynamic_batching(2, bad.ctypes.data_as(binding._I32P), 0, 1,
                                    o.ctypes.data_as(binding._I32P)) == binding.E_INVAL


# ------------------------------------------------- streaming controller (host logic)
class _FakeTensor:
    def __getitem__(self, k):
        return self

    def contiguous(self):
        return self

    def to(self, d):
        return self


class _FakeTorch:
    """Just enough of torch for harness.streaming_rollout to run without a GPU."""
    float32, int32 = "f32", "i32"

    class cuda:
        class Event:
            def __init__(self, enable_timing=True):
                pass

            def record(self):
                pass

            def elapsed_time(self, other):
                return 1.0

        @staticmethod
        def synchronize():
            pass

    @staticmethod
    def empty(shape, dtype=None, device=None):
        return _FakeTensor()

    @staticmethod
    def empty_like(a):
        return a

    @staticmethod
    def from_numpy(a):
        return _FakeTensor()


class _FakeEngine:
    device = "cpu"

    def __init__(self):
        self.live = set()

    def prefill(self, ids, prompts, logits_out=None):
        assert not self.live & set(int(i) for i in ids)
        self.live.update(int(i) for i in ids)

    def sample_logprob(self, *a, **k):
        pass

    def decode_step(self, ids, *a, **k):
        assert set(int(i) for i in ids) <= self.live

    def free_seq(self, i):
        self.live.remove(int(i))

    def update_weights_interrupt(self, w, version, logits_out=None):
        return np.array(sorted(self.live), dtype=np.int32), None, 0


@pytest.mark.parametrize("eta", [0, 1, 2, 3, 5])
def test_streaming_controller_follows_the_oracle_event_loop(eta):
    """The refill loop of the streaming regime (slots, staleness gate through the C entry
    points, one weight update per finished training batch) with the GPU calls stubbed out:
    the same number of ticks as the oracle's plain event loop and every request submitted and
    completed under the versions that loop gives it (Section 5.1)."""
    from oracle import staleness
    from paper_2505_24298_amd import harness
    n_total, slots, B = 48, 8, 8
    for seed in range(6):
        outs = synth.output_lengths(n_total, 12, 1.0, 60, seed=seed)
        prompts = [np.zeros(3, dtype=np.int32)] * n_total
        eng = _FakeEngine()
        r = harness.streaming_rollout(eng, _FakeTorch, dict(vocab=16), binding.host_lib(), prompts, outs, slots, B,
                                      eta, [0, 1], 1.0, 1.0, 0)
        ticks, done = staleness.simulate_stream(n_total, B, eta, slots, outs)
        assert r["ticks"] == ticks and sorted(r["records"]) == sorted(done)
        assert r["gen_tokens"] == int(outs.sum()) and not eng.live


@pytest.mark.parametrize("own,group,nkv,max_slots,target,min_tokens", [
    ([1], 1, 2, 32, 0, 256), ([701], 1, 2, 32, 0, 256), ([33, 32, 31, 1], 1, 1, 32, 0, 256),
    ([65536] + [1] * 7, 1, 4, 32, 0, 256),                       # the longest context in 32 slots, next to one-token rows
    ([8150, 64, 1000], 1, 1, 32, 65536, 128), ([8150, 64, 1000], 1, 1, 32, 64, 2048),
    ([16384, 4000], 1, 2, 24, 65536, 128),                       # fewer slots: a set of rows takes the others
    (list(range(420, 676)), 16, 2, 32, 0, 256),                  # 16 prompts x 16 samples
    (list(range(1500, 4140, 30)), 1, 2, 32, 0, 256), ([5000] * 16, 16, 2, 32, 0, 256),   # one set: too big for one XCD
    ([300] * 30 + [9000] * 3, 3, 2, 32, 0, 256)])
def test_decode_plan_covers_every_token_once(own, group, nkv, max_slots, target, min_tokens):
    """areal_plan_decode: the segments of a row follow each other without gap from token 0 to the one it appends, at
    most max_slots of them and 2,048 tokens each; every XCD gets an eighth of the work to within a segment."""
    H = binding.host_lib()
    n = len(own)
    home = [i - i % group for i in range(n)]
    a, h = np.array(own, np.int32), np.array(home, np.int32)
    ptr = lambda x: x.ctypes.data_as(binding._I32P)
    out = np.zeros((4096, 4), np.int32)
    k = H.areal_plan_decode(n, ptr(a), ptr(h), nkv, max_slots, target, min_tokens, ptr(out), len(out))
    assert 0 < k <= len(out) and k % 8 == 0
    out = out[:k]
    units = -(-a.astype(int) // 32)
    load = np.zeros(8, int)
    seen = [[] for _ in range(n)]
    for q, (row, t0, m, slot) in enumerate(out.tolist()):
        if row < 0:
            continue
        assert 0 < m <= 2048 and m % 32 == 0 and t0 % 32 == 0
        seen[row].append((slot, t0, m))
        load[q % 8] += m // 32
    for i, s in enumerate(seen):
        s.sort()
        assert [x[0] for x in s] == list(range(len(s))) and len(s) <= max_slots
        at = 0
        for _, t0, m in s:
            assert t0 == at
            at += m
        assert at == units[i] * 32
        # all but a cut row's last segment are whole rounds of four waves of 32 tokens
        assert all(m % 128 == 0 for _, _, m in s[:-1])
    longest = max(m for s in seen for _, _, m in s) // 32
    assert load.sum() == units.sum() and load.max() <= units.sum() / 8 * 1.05 + longest
    if group == 16 and n == 256:                                 # the samples of a prompt on at most two XCDs
        where = [{q % 8 for q in range(k) if out[q, 0] // 16 == p and out[q, 0] >= 0} for p in range(16)]
        assert max(len(w) for w in where) <= 2
    assert H.areal_plan_decode(n, ptr(a), ptr(h), nkv, 0, 0, 0, ptr(out), 1) == binding.E_INVAL


@pytest.mark.parametrize("n_long,group", [(426, 256), (470, 256), (483, 128), (0, 1), (2063, 16), (3, 2063)])
def test_decode_plan_of_many_rows_is_bounded(n_long, group):
    """Long rows that share blocks next to many of one unit: no XCD gets more than a quarter above its share of
    the segments (the launch pads all to the deepest), and the segments' descriptors and block ids fit the space
    that a context has for them, whatever the lengths (22 bytes a row and unit of the longest, and 56)."""
    H = binding.host_lib()
    n, longest = 2063, 1709
    own = np.array([1539 + i * 37 % 171 for i in range(n_long)] + [17] * (n - n_long), np.int32)
    home = np.array([i - i % group for i in range(n)], np.int32)
    ptr = lambda x: x.ctypes.data_as(binding._I32P)
    for target, min_tokens in ((0, 256), (65536, 128), (64, 2048)):
        out = np.zeros((65536, 4), np.int32)
        k = H.areal_plan_decode(n, ptr(own), ptr(home), 2, 32, target, min_tokens, ptr(out), len(out))
        assert 0 < k <= len(out) and k % 8 == 0
        real = out[:k][out[:k, 0] >= 0]
        assert k <= 8 * (-(-len(real) // 8) * 5 // 4 + 4)
        ids = -(-(int(real[:, 2].max()) // 16) // 4) * 4
        units = -(-longest // 32)
        assert len(real) * (16 + 4 * ids) <= n * (14 * units + 8 * min(units, 64) + 56)


def test_tile_choice_for_the_decoder_shapes(L):
    """areal_op_gemm_choose (host only): the tile configuration and K split the library takes for
    the products of the 1.5B and 7B shapes, at the row counts where the rules change.  Pins the
    rules that were read off sweeps on the MI355X, so that an edit of one does not silently
    move another: configuration numbers as in gemm.hip's dispatch, where a number is one tile in every mode."""
    import ctypes as C

    def choose(M, N, K, mode):
        c, s = C.c_int32(), C.c_int32()
        assert L.areal_op_gemm_choose(M, N, K, mode, C.byref(c), C.byref(s)) == 0
        return c.value, s.value

    STORE, ADD, SWIGLU = 0, 1, 2
    H, F, V = 1536, 8960, 151936
    # prefill passes of 8,192 rows: 256 x 256 tiles; the down projection with its last round evened out
    assert choose(8192, 2048, H, STORE) == (19, 1)
    assert choose(8192, F, H, SWIGLU) == (19, 1)
    assert choose(8192, H, F, ADD) == (24, 1)
    assert choose(8192, 3584, 18944, ADD) == (24, 1)
    assert choose(8192, H, H, ADD) == (26, 1)                 # 256 x 192, as every residual add in that tile
    # decode steps: gate/up by row count, no K split (the SwiGLU epilogue needs whole sums)
    assert [choose(M, F, H, SWIGLU) for M in (24, 48, 100, 200)] == [(36, 1), (37, 1), (38, 1), (39, 1)]
    # narrow products split K; the down projection at few rows takes 64-column tiles
    assert choose(24, H, F, ADD) == (25, 8)
    assert choose(100, H, F, ADD) == (23, 8)
    for M in (8, 64, 256):
        cfg, splits = choose(M, 2048, H, STORE)
        assert cfg in (21, 22, 23) and 1 < splits <= 12
    # output projection: one work-group per column panel, never split
    assert [choose(M, V, H, STORE)[1] for M in (1, 100, 256)] == [1, 1, 1]
    # a ragged K (not a multiple of 64) falls back to the register-staged tiles
    assert choose(100, 1000, 344, STORE)[0] in (0, 2, 4)
    # invalid shapes are refused
    c, s = C.c_int32(), C.c_int32()
    assert L.areal_op_gemm_choose(0, 8, 8, 0, C.byref(c), C.byref(s)) != 0
    assert L.areal_op_gemm_choose(8, 8, 8, 3, C.byref(c), C.byref(s)) != 0


def test_passes_that_fill_the_chip_are_not_cut_along_k(L):
    """Above 256 rows a cut along K (float32 atomics: a pass then differs from run to run) is for launches that leave
    compute units idle, or where it saves enough by price.  At the
    1.5B shape every pass of more than 2,048 rows repeats; at the 7B shape all of more than 512 but for its down
    projection."""
    import ctypes as C

    def cut(M, N, K, mode):
        c, s = C.c_int32(), C.c_int32()
        assert L.areal_op_gemm_choose(M, N, K, mode, C.byref(c), C.byref(s)) == 0
        # 24 cuts tiles of 256 x 256; where its tiles of 192 columns fill whole rounds it cuts none
        return s.value > 1 or (c.value == 24 and (-(-N // 192) * -(-M // 256)) % 256 != 0)

    rows = sorted(set(range(257, 8193, 37)) | {r + d for r in range(512, 8193, 64) for d in (0, 1) if r + d <= 8192})
    for N, K, mode, above in ((2048, 1536, 0, 505), (1536, 1536, 1, 737), (1536, 8960, 1, 2048),
                              (4608, 3584, 0, 384), (3584, 3584, 1, 512)):
        assert not [M for M in rows if M > above and cut(M, N, K, mode)], (N, K)
    for lo, hi in ((1537, 1664), (2817, 3456), (3841, 4608), (6145, 6336), (6401, 6912)):
        assert not [M for M in rows if lo <= M <= hi and cut(M, 3584, 18944, 1)], (lo, hi)


def test_gate_up_tiles_by_rows_and_width(L):
    """Gate/up: the tile with the least to take in per compute unit, no taller than the launch needs; whole
    sums, so never a K split.  Narrow products never take a tile of more than twice the rows (of 32 at least)."""
    import ctypes as C

    def choose(M, N, K, mode):
        c, s = C.c_int32(), C.c_int32()
        assert L.areal_op_gemm_choose(M, N, K, mode, C.byref(c), C.byref(s)) == 0
        return c.value, s.value

    rows = (1, 32, 33, 64, 65, 96, 97, 128, 256, 257, 320, 321, 384)
    assert [choose(M, 8960, 1536, 2)[0] for M in rows] == [36, 36, 37, 37, 29, 29, 38, 38, 39, 33, 33, 34, 34]
    assert [choose(M, 18944, 3584, 2)[0] for M in rows[:9]] == [36, 36, 30, 30, 31, 31, 32, 32, 32]
    assert all(choose(M, N, 1536, 2)[1] == 1 for M in rows for N in (344, 8960))
    height = {22: 32, 23: 64, 25: 32, 35: 128, 21: 128}
    for N, K, mode in ((2048, 1536, 0), (1536, 1536, 1), (1536, 8960, 1), (3584, 18944, 1)):
        for M in (1, 16, 32, 33, 64, 65, 256):
            cfg, splits = choose(M, N, K, mode)
            assert height[cfg] <= 2 * max(M, 32) and 1 <= splits <= 12


@pytest.mark.parametrize("M,N,K,mode,want", [
    (132, 4608, 3584, 0, (23, 3)),       # 17.8 us; 19.0 in 128-row tiles
    (88, 3584, 18944, 1, (35, 6)),       # 34.1; 37.7 in (21, 8)
    (301, 3584, 3584, 1, (35, 2)),       # 21.3; 24.1 in (23, 1)
    (301, 3584, 18944, 1, (27, 4)),      # 64.3; 69.0 in (28, 8)
    (576, 1536, 8960, 1, (21, 4)),       # 32.5; 33.6 in (29, 2)
    (2048, 1536, 8960, 1, (27, 2)),      # 71.0; 76.0 in (35, 1)
    (2048, 3584, 18944, 1, (19, 2)),     # 246; 275 in (24, 1)
    (1600, 4608, 3584, 0, (20, 1)),      # 63.1; 69.8 in (28, 1)
    (832, 8960, 1536, 2, (20, 1))])      # 59.3; 63.9 in (28, 1)
def test_choices_that_the_sweeps_bear_out(L, M, N, K, mode, want):
    """Products for which a cheaper launch had been measured than the one that was taken."""
    import ctypes as C
    c, s = C.c_int32(), C.c_int32()
    assert L.areal_op_gemm_choose(M, N, K, mode, C.byref(c), C.byref(s)) == 0
    assert (c.value, s.value) == want


def test_long_k_choice_names_the_kernel_it_launches(L):
    """Residual adds with a long K: 24 is the launch that is evened out along K, 26 and 28 the whole tiles of
    256 x 192 and 192 x 256.  Where whole tiles are the cheaper ones the choice says so, also where 192-column
    tiles fill their rounds to nine tenths only."""
    import ctypes as C

    def choose(M, N, K):
        c, s = C.c_int32(), C.c_int32()
        assert L.areal_op_gemm_choose(M, N, K, 1, C.byref(c), C.byref(s)) == 0
        return c.value, s.value

    assert choose(6400, 3584, 18944) == choose(12400, 3584, 18944) == (24, 1)
    assert choose(5200, 4096, 11008) == (28, 1)                                  # 407 us; 427 evened out
    assert choose(2560, 4736, 8960) == choose(3457, 3456, 18944) == (26, 1)      # 250 and 252 tiles of 256 x 192
    assert choose(8192, 1536, 8960) == (24, 1)                                   # 256 of them: nothing to cut
    assert choose(8000, 1536, 8960) == choose(7000, 1536, 8960) == (28, 1)       # 252 and 222 of 192 x 256


def test_refused_products_stay_refused(L):
    """areal_op_gemm: a configuration that does not exist, or does not serve the mode or a ragged K, is refused
    whatever the shape, also where the shape would go to other tiles (odd widths of the gate/up product, K
    beyond 32-bit offsets).  The addresses are never used: nothing of this reaches a launch."""
    import ctypes as C
    p = [C.c_void_p(4096 * k) for k in range(1, 5)]
    n_cfg, INVAL = L.areal_op_gemm_num_configs(), binding.E_INVAL

    def refused(M, N, K, mode, cfg):
        return L.areal_op_gemm(None, *p, M, N, K, mode, cfg, 1) == INVAL

    assert all(refused(40, N, 128, 2, cfg) for N in (94, 95) for cfg in (22, 23, 24, 25, n_cfg, n_cfg + 70))
    assert all(refused(40, N, 72, 2, cfg) for N in (94, 95) for cfg in (7, 12, 21, 28))
    assert all(refused(3, 24, K, mode, n_cfg) for K in (128, 1 << 22) for mode in (0, 1))
    assert all(refused(3, 24, K, 0, 24) for K in (128, 1 << 22))
    assert all(refused(3, 24, (1 << 22) + 8, mode, 12) for mode in (0, 1, 2))


def test_products_of_a_few_rows_refuse_addresses_they_cannot_load_from(L):
    """areal_op_rows_product reads x, the gains and the weights 16 bytes at a time and stores single elements: what does not
    start there is refused before anything reaches a launch."""
    def rc(mode, x=16, gain=16, W0=16, W1=16, Cp=16):
        p = [C.c_void_p(4096 * k + at) for k, at in zip(range(1, 6), (x, gain, W0, W1, Cp))]
        gain_p = None if mode == 1 else p[1]
        W1_p = p[3] if mode == 2 else None
        return L.areal_op_rows_product(None, p[0], gain_p, 1e-6, p[2], W1_p, None, 24, 24, p[4], 1, 24, 128, mode)

    for mode in (0, 1, 2):
        bad = [dict(x=8), dict(W0=8), dict(Cp=1)] + [dict(Cp=2)] * (mode != 2) + [dict(W1=2)] * (mode == 2)
        bad += [dict(gain=at) for at in (2, 4, 8)] * (mode != 1)
        assert all(rc(mode, **b) == binding.E_INVAL for b in bad), mode


# ------------------------------------------------------------- addresses of the tiled products' loads
RANGE_CHECKS = {
    "lane offset alone": lambda lane, scalar, size: lane < size,
    "lane and scalar offset": lambda lane, scalar, size: lane + scalar < size,
    "lane offset against the rest, which wraps": lambda lane, scalar, size: lane < (size - scalar) % 2 ** 32,
}


def _load_faults(check, row, spread, rows, row_bytes, base, size, lane_off, row_scalar=0):
    """Lanes of one load (first and last K slab) that touch what does not exist or miss what does, if the range of a buffer
    load is checked as `check` says."""
    lane = np.arange(64, dtype=np.int64)
    r = lane >> 3
    r = row + (8 * (r >> 2) + (r & 3) if spread else r)
    chunk = ((lane & 7) ^ (lane >> 3)) * 16
    bad = 0
    for slab in (0, row_bytes - 128):
        scalar = row_scalar + slab
        taken = RANGE_CHECKS[check](lane_off, scalar, size)
        at = base + lane_off + scalar
        bad += int((taken & ((at < 0) | (at + 16 > rows * row_bytes))).sum())
        bad += int(((r < rows) & (~taken | (at != r * row_bytes + chunk + slab))).sum())
    return bad


@pytest.mark.parametrize("check", RANGE_CHECKS)
@pytest.mark.parametrize("row_bytes", [128, 3072, 37888])
def test_loads_of_edge_tiles_stay_inside_the_matrix(HL, check, row_bytes):
    """Every group of a tile of up to 256 rows, whatever part of the tile exists: no lane reads behind the operand's last row and
    every existing row is read where it lies, whichever offsets the hardware holds against a resource's range."""
    out = (C.c_uint32 * 66)()
    for rows in [1, 2, 7, 8, 9, 15, 16, 17, 23, 24, 31, 33, 63, 72, 100, 128, 255, 256]:
        for first in range(0, 256, 4):
            for kind in (0, 1, 2):
                assert HL.areal_plan_tile_load(first, kind, rows, row_bytes, out) == 0
                v = np.array(out[:], dtype=np.int64)
                assert _load_faults(check, first, kind == 1, rows, row_bytes, v[0], v[1], v[2:]) == 0, (rows, first, kind)
    assert HL.areal_plan_tile_load(0, 3, 8, 128, out) == HL.areal_plan_tile_load(0, 0, 0, 128, out) == binding.E_INVAL


def test_a_row_in_the_scalar_offset_would_not_be_inside():
    """The form that the loads must not have: one resource for a tile's rows, a group's place in the scalar offset.  It needs a
    check that includes the scalar offset and does not wrap."""
    lane = np.arange(64, dtype=np.int64)
    off = (lane >> 3) * 3072 + ((lane & 7) ^ (lane >> 3)) * 16
    faults = {c: _load_faults(c, 24, False, 20, 3072, 0, 20 * 3072, off, row_scalar=24 * 3072) for c in RANGE_CHECKS}
    assert faults["lane and scalar offset"] == 0
    assert faults["lane offset alone"] > 0 and faults["lane offset against the rest, which wraps"] > 0
