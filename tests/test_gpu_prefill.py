"""GPU parity of the bulk prefill (wkv_prefill) against the oracle's prefill: outputs of every
prompt row, the compressed cache (token positions, counts, merge counts, keys bit-exact; score
sums to 1e-9; merged values within the output tolerance), and decode steps that follow."""
import numpy as np
import pytest
import torch

from paper_2503_01330_amd import synth

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import parity
    from paper_2503_01330_amd import binding as wkv


def _run(cfg, P, decode_steps=0, units_sel=None, **kw):
    g = parity.gpu_prefill(cfg, P, units_sel=units_sel, **kw)
    try:
        okw = {k: kw[k] for k in ("n_sink", "score_mode", "merge_mode") if k in kw}
        stats = parity.compare_prefill(cfg, g, decode_steps=decode_steps, **okw)
    finally:
        g["cache"].close()
    print(f"\n  {cfg.name} P={P}: {stats}", flush=True)
    return stats


@pytest.mark.parametrize("dtype", ["fp16", "bf16"])
@pytest.mark.parametrize("d", [64, 128])
def test_prompt_lengths_around_the_tile_and_the_budget(dtype, d):
    """1 token, ragged tiles (15, 17, 100), prompt = budget, budget + 1 (where the prefill must equal
    token-by-token streaming), and several times the budget."""
    for P, m, R in ((1, 8, 1), (15, 20, 3), (17, 16, 2), (100, 100, 9), (101, 100, 9), (100, 37, 5), (333, 40, 1)):
        cfg = synth.StreamConfig(f"pre{P}", 8000 + P, 2, 3, d, dtype, P + 12, m, R)
        _run(cfg, P, decode_steps=12)


def test_prefill_equals_streaming_on_the_gpu_up_to_budget_plus_one():
    """The same property as the oracle's pin, on the library: a prompt of m + 1 tokens through
    wkv_prefill and through m + 1 calls of wkv_step gives the same cache."""
    cfg = synth.StreamConfig("pre-eq", 8100, 1, 4, 128, "fp16", 65, 64, 4)
    a = parity.gpu_prefill(cfg, 65)
    b = parity.gpu_stream(cfg)
    try:
        for what in (wkv.WKV_POS, wkv.WKV_COUNT, wkv.WKV_NMERGED, wkv.WKV_K, wkv.WKV_V):
            assert np.array_equal(a["cache"].state(what), b["cache"].state(what)), what
        np.testing.assert_allclose(a["cache"].state(wkv.WKV_SCORE_SUM), b["cache"].state(wkv.WKV_SCORE_SUM), rtol=1e-12)
        parity.check_outputs(a["out"], b["out"], cfg.dtype)
    finally:
        a["cache"].close(); b["cache"].close()


def test_sinks_eviction_only_and_cumulative_scores():
    cfg = synth.StreamConfig("pre-var", 8200, 1, 5, 128, "fp16", 300, 48, 8)
    _run(cfg, 280, decode_steps=20, n_sink=4)
    _run(cfg, 280, decode_steps=20, merge_mode=wkv.WKV_MERGE_NONE)
    _run(cfg, 280, decode_steps=20, merge_mode=wkv.WKV_MERGE_NONE, score_mode=wkv.WKV_SCORE_CUMULATIVE)


def test_long_runs_of_removed_tokens():
    """A tiny budget under a long prompt: almost everything is removed, runs of hundreds of tokens fold
    into one survivor in score order."""
    cfg = synth.StreamConfig("pre-runs", 8300, 1, 3, 64, "bf16", 1210, 6, 2)
    _run(cfg, 1200, decode_steps=10)


def _directed(cfg, slope, seed):
    """Prompts whose average scores are monotone in the token index: every query and key points
    along one direction per unit, and the logit of token i is proportional to slope * i.  slope > 0:
    every row attends to its newest tokens, abar_i ~ 1 / (P - i) ascends; slope < 0: every row
    attends to the oldest tokens, abar_i ~ exp(-c i) descends."""
    rng = np.random.default_rng(seed)
    T, U, d = cfg.steps, cfg.units, cfg.head_dim
    u = rng.standard_normal((1, U, d)).astype(np.float32)
    u *= np.sqrt(d) / np.linalg.norm(u, axis=-1, keepdims=True)
    ramp = np.arange(T, dtype=np.float32)[:, None, None] * slope
    q = np.broadcast_to(u, (T, U, d)) * 0.5
    k = u * ramp
    v = rng.standard_normal((T, U, d)).astype(np.float32)
    return q, k, v


@pytest.mark.parametrize("slope", [0.02, -0.02])
def test_monotone_scores_chains_and_fans(slope):
    """The two extreme shapes of the merge forest.  Ascending scores: every removed token folds
    into its right neighbour, one chain as long as the run (the weights are products up the
    chain).  Descending scores: the newest removed token goes first and every removed token is a
    child of the one survivor on the right (the weights are products over later siblings).  Runs
    of ~900 tokens span many 64-token blocks of the parent search."""
    cfg = synth.StreamConfig("pre-mono", 8600, 1, 3, 64, "fp16", 1000, 24, 4)
    g = parity.gpu_prefill(cfg, 990, arrays=_directed(cfg, slope, 8600))
    try:
        stats = parity.compare_prefill(cfg, g, decode_steps=10)
        pos = g["cache"].state(wkv.WKV_POS)
        gaps = np.diff(np.concatenate([np.full((pos.shape[0], 1), -1), pos], axis=1), axis=1)
        assert gaps.max() > 800, "expected one long run of removed tokens"
    finally:
        g["cache"].close()
    print(f"\n  slope {slope}: {stats}, longest run {int(gaps.max())}", flush=True)


def test_randomised_prompts():
    """Many small random configurations (prompt length, budget, window, sinks, rule variants, head
    size, dtype, unit count, workgroups per unit of the decode steps that follow)."""
    g = np.random.default_rng(20250302)
    for case in range(30):
        dtype = ["fp16", "bf16"][int(g.integers(2))]
        d = [64, 128][int(g.integers(2))]
        P = int(g.integers(1, 900))
        m = int(g.integers(1, 300))
        R = int(g.integers(1, m + 1)) if g.random() < 0.3 else int(g.integers(1, min(m, 40) + 1))
        n_sink = int(g.integers(0, min(5, m - R) + 1)) if g.random() < 0.4 else 0
        mode = int(g.integers(3))       # 0 merge, 1 evict-only, 2 cumulative score
        kw = {}
        if n_sink:
            kw["n_sink"] = n_sink
        if mode >= 1:
            kw["merge_mode"] = wkv.WKV_MERGE_NONE
        if mode == 2:
            kw["score_mode"] = wkv.WKV_SCORE_CUMULATIVE
        if g.random() < 0.25 and m >= 64:
            kw["split"] = [2, 4][int(g.integers(2))]
        batch, heads = int(g.integers(1, 3)), int(g.integers(1, 6))
        steps = int(g.integers(0, 9))
        cfg = synth.StreamConfig(f"rnd{case}", 8700 + case, batch, heads, d, dtype, P + steps, m, R)
        print(f"\n  case {case}: P={P} m={m} R={R} d={d} {dtype} units={batch * heads} {kw}", flush=True)
        _run(cfg, P, decode_steps=steps, **kw)


def test_prefill_then_sliced_decode():
    cfg = synth.StreamConfig("pre-split", 8400, 1, 2, 128, "fp16", 700, 300, 16)
    _run(cfg, 650, decode_steps=50, split=4)


def test_outputs_may_be_skipped():
    cfg = synth.StreamConfig("pre-noout", 8500, 1, 2, 128, "fp16", 200, 50, 4)
    g = parity.gpu_prefill(cfg, 200, want_out=False)
    try:
        parity.compare_prefill(cfg, g)
    finally:
        g["cache"].close()


def test_prompt_merges_with_a_zero_denominator():
    """Prompt tokens whose keys point away from every query get a score of exactly 0; runs of them
    are merged with undefined convex weights: averaged, and counted in the status."""
    units, d, m, R, P = 3, 64, 24, 4, 90
    cfg = synth.StreamConfig("pre-zero-den", 8650, 1, units, d, "fp16", P, m, R)
    g = np.random.default_rng(8650)
    q = (0.5 * g.standard_normal((P, units, d))).astype(np.float32)
    k = (0.5 * g.standard_normal((P, units, d))).astype(np.float32)
    v = g.standard_normal((P, units, d)).astype(np.float32)
    q[:, :, 0] = 200.0
    dead = np.zeros((P, units), bool)
    for u in range(units):
        t = 2 + u
        while t < P - 3:
            run = int(g.integers(1, 4))
            dead[t:t + run, u] = True
            t += run + int(g.integers(1, 4))
    k[:, :, 0] = np.where(dead, -200.0, 200.0)
    res = parity.gpu_prefill(cfg, P, arrays=(q, k, v))
    try:
        stats = parity.compare_prefill(cfg, res)
        status = res["cache"].state(wkv.WKV_STATUS)
    finally:
        res["cache"].close()
    print(f"\n  pre-zero-den: {stats} status {list(status)}", flush=True)
    assert status[0] > 0, "no merge with a zero denominator happened: the test shape is off"


def test_a_nan_in_one_unit_of_the_prompt_is_flagged_and_stays_in_that_unit():
    """A NaN in one unit's query of one prompt token: non-finite scores are counted in the status,
    that row's output is NaN, and the other units' outputs and compressed caches are bit for bit
    those of the clean prompt (units never interact, Section III-A)."""
    cfg = synth.StreamConfig("pre-nf", 8600, 1, 3, 64, "fp16", 150, 40, 8)
    P = 150
    q, k, v = (synth.storage_to_f32(x, cfg.dtype) for x in synth.Stream(cfg).steps(0, P))
    shape = (P, cfg.units, cfg.head_dim)

    def run(qa):
        g = parity.gpu_prefill(cfg, P, arrays=(qa.reshape(shape), k.reshape(shape), v.reshape(shape)))
        c = g["cache"]
        try:
            return dict(out=g["out"], K=c.state(wkv.WKV_K), V=c.state(wkv.WKV_V), a=c.state(wkv.WKV_SCORE_SUM),
                        pos=c.state(wkv.WKV_POS), status=c.state(wkv.WKV_STATUS))
        finally:
            c.close()

    clean = run(q)
    bad_q = q.copy().reshape(shape)
    bad_q[60, 1, 5] = np.nan
    dirty = run(bad_q)
    assert list(clean["status"]) == [0, 0]
    assert dirty["status"][1] > 0
    assert np.isnan(dirty["out"][60, 1]).all()
    others = [0, 2]
    assert np.array_equal(dirty["out"][:, others], clean["out"][:, others])
    for item in ("K", "V"):
        assert np.array_equal(dirty[item][others].view(np.uint16), clean[item][others].view(np.uint16))
    assert np.array_equal(dirty["a"][others], clean["a"][others])
    assert np.array_equal(dirty["pos"][others], clean["pos"][others])
    # the unit concerned is still compressed to the budget, newest token retained
    assert dirty["pos"].shape[1] == cfg.budget and (dirty["pos"][1, -1] == P - 1)


def test_argument_checks():
    code = synth.DTYPE_CODE
    x = torch.zeros(64, 2, 128, dtype=torch.float16, device="cuda")
    c = wkv.Cache(1, 2, 128, 16, 2, code["fp16"])
    try:
        with pytest.raises(wkv.WkvError) as e:
            wkv.wkv_prefill(c.h, x.data_ptr(), x.data_ptr(), x.data_ptr(), 0, 0)
        assert e.value.code == wkv.WKV_EINVAL
        with pytest.raises(wkv.WkvError) as e:
            wkv.wkv_prefill(c.h, x.data_ptr(), x.data_ptr(), x.data_ptr(), 0, wkv.WKV_MAX_PROMPT + 1)
        assert e.value.code == wkv.WKV_ESIZE
        with pytest.raises(wkv.WkvError) as e:
            wkv.wkv_prefill(c.h, x.data_ptr() + 2, x.data_ptr(), x.data_ptr(), 0, 8)
        assert e.value.code == wkv.WKV_EINVAL
        assert c.tokens == 0
        c.prefill(x, x, x)
        assert c.tokens == 64 and c.length == 16
        with pytest.raises(wkv.WkvError) as e:       # not empty any more
            c.prefill(x, x, x)
        assert e.value.code == wkv.WKV_EINVAL
    finally:
        c.close()
    for kw, dt, d in ((dict(), "fp32", 128), (dict(), "fp16", 256),
                      (dict(score_mode=wkv.WKV_SCORE_LAST, merge_mode=wkv.WKV_MERGE_NONE), "fp16", 128)):
        c = wkv.Cache(1, 2, d, 16, 2, code[dt], **kw)
        try:
            y = torch.zeros(8, 2, d, dtype={"fp32": torch.float32, "fp16": torch.float16}[dt], device="cuda")
            with pytest.raises(wkv.WkvError):
                c.prefill(y, y, y)
            assert c.tokens == 0
        finally:
            c.close()


def test_llama_shaped_prompt_sampled_units():
    """A 4096-token prompt into the stacked configuration's cache (batch 8 x 32 heads x 128 fp16,
    budget 410), every unit on the GPU, 3 sampled units through the oracle, then 64 decode steps."""
    cfg = synth.scaled(synth.CONFIGS["cfg3"], steps=4096 + 64, layers=1)
    sel = np.sort(np.random.default_rng(11).choice(cfg.units, 3, replace=False))
    stats = _run(cfg, 4096, decode_steps=64, units_sel=sel)
    assert stats["min_gap"] >= 0


@pytest.mark.parametrize("dtype", ["fp16", "bf16"])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("where", ["queries", "keys", "one row"])
def test_rows_that_span_more_than_the_digits(dtype, d, where):
    """Logits are formed from 8-bit digits of rows brought to integers below 2^31; a row with elements
    that are no integers at its scale must take the fp64 instruction.  Such a row here: one large
    element (times zero on the other side) and small ones below the last digit, which meet large
    elements, so that dropping what does not fit would move a logit by more than 1e-5 (score sums are held to
    1e-9).  Also a row of zeros and one of the smallest numbers.  130 tokens: a ragged last tile and
    several workgroups a unit."""
    P, m, R, U = 130, 48, 6, 3
    cfg = synth.StreamConfig("pre-span", 8700, 1, U, d, dtype, P + 12, m, R)
    g = np.random.default_rng(8700)
    q, k, v = (g.standard_normal((cfg.steps, U, d)).astype(np.float32) for _ in range(3))
    big, tiny = (2.0 ** 11, 2.0 ** -13) if dtype == "fp16" else (2.0 ** 10, 2.0 ** -18)
    rows = [97] if where == "one row" else [0, 1, 15, 16, 40, 63, 64, 100, 127, 129]
    side, other = (q, k) if where == "queries" else (k, q)
    side[rows] *= tiny
    other *= 20.0       # (small logits everywhere would make every output the mean of a hundred values, which cancels: the
                        # share of bit-exact bf16 outputs then falls with fp32 error / result, to 0.9989 at 130 tokens)
    side[:, :, 0] = other[:, :, 0] = 0.0
    side[rows, :, 0] = big
    other[3] = 0.0
    other[5] *= 2.0 ** -20 if dtype == "fp16" else 2.0 ** -120
    got = parity.gpu_prefill(cfg, P, arrays=(q, k, v))
    try:
        stats = parity.compare_prefill(cfg, got, decode_steps=8)
    finally:
        got["cache"].close()
    print(f"\n  {where}: {stats}", flush=True)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("P", [63, 64, 65, 66, 67, 127, 128, 129, 130, 257])
def test_sort_and_runs_at_their_edges(P, d):
    """The sort's steps leave a wave from 128 tokens on, and a run of 64 removed tokens or more is summed by a
    whole workgroup: prompts around powers of two, folded into one to three survivors and into seventeen
    (one more than a workgroup of the fold takes)."""
    for m, R in ((1, 1), (2, 1), (3, 2), (17, 5)):
        _run(synth.StreamConfig(f"pre-edge{P}", 8900 + P, 1, 3, d, "bf16", P + 3, m, R), P, decode_steps=3)


@pytest.mark.parametrize("dtype,d,P,units", [("fp16", 128, 129, 170), ("bf16", 64, 129, 170), ("fp16", 64, 129, 171), ("bf16", 128, 129, 171),
                                             ("bf16", 64, 1025, 63), ("fp16", 128, 1025, 64), ("bf16", 64, 1025, 1017),
                                             ("fp16", 128, 3073, 16), ("bf16", 64, 3073, 17)])
def test_prompts_of_many_units(dtype, d, P, units):
    """Up to 1536 tiles of 16 tokens a launch (4096 from 512 tokens on, where from 3072 on units count in rounds of eight) two waves share a tile (most prompts of these tests), then a
    wave has one: launches on either side.  An odd number of tiles, one row in the last tile, units that are no
    multiple of eight and a row that takes the fp64 instruction (one element far above the others).  Five units' inputs,
    repeated."""
    cfg = synth.StreamConfig("pre-two", 8800 + P, 1, units, d, dtype, P + 4, 100, 9)
    few = synth.Stream(synth.StreamConfig("pre-two", 8800 + P, 1, 5, d, dtype, P + 4, 100, 9))
    q, k, v = (synth.storage_to_f32(x, dtype).copy() for x in few.steps(0, cfg.steps))
    k[37, :, 1:] *= 2.0 ** -12 if dtype == "fp16" else 2.0 ** -26
    k[37, :, 0] = 128.0 if dtype == "fp16" else 9.0
    arrays = [x[:, np.arange(units) % 5] for x in (q, k, v)]
    got = parity.gpu_prefill(cfg, P, units_sel=[0, 1, 3, units // 2, units - 1], arrays=arrays)
    try:
        print(f"\n  {parity.compare_prefill(cfg, got, decode_steps=3)}", flush=True)
    finally:
        got["cache"].close()


@pytest.mark.parametrize("kw", [dict(split=1), dict(split=4), dict(split=1, replayable=1)])
def test_an_emptied_cache_is_a_fresh_one(kw):
    """Loading an empty state into a full cache (more log entries than slots, fewer slots than a block of the
    clearing kernel): the next prompt and the steps after it give what a fresh handle gives, bit for bit,
    and the eviction log starts afresh."""
    cfg = synth.StreamConfig("pre-empty", 9000, 1, 3, 64, "fp16", 90, 37, 5)
    a = parity.gpu_prefill(cfg, 60, **kw)
    b = parity.gpu_prefill(cfg, 60, **kw)
    try:
        tq, tk, tv, out = a["dev"]
        for t in range(60, 75):
            a["cache"].step(tq[t], tk[t], tv[t], out[t])
        U, d = cfg.units, cfg.head_dim
        rows = np.empty((U, 0, d), np.float16)
        a["cache"].load(0, rows, rows, np.empty((U, 0), np.float64), np.empty((U, 0), np.int32))
        assert a["cache"].tokens == 0 and a["cache"].length == 0
        with pytest.raises(RuntimeError):
            a["cache"].evictions(1)
        a["cache"].prefill(tq[:60], tk[:60], tv[:60], out[:60])
        for c, o in ((a["cache"], out), (b["cache"], b["dev"][3])):
            for t in range(60, 80):
                c.step(tq[t], tk[t], tv[t], o[t])
        torch.cuda.synchronize()
        assert torch.equal(out[:80], b["dev"][3][:80])
        for what in (wkv.WKV_POS, wkv.WKV_COUNT, wkv.WKV_NMERGED, wkv.WKV_K, wkv.WKV_V, wkv.WKV_SCORE_SUM):
            assert np.array_equal(a["cache"].state(what), b["cache"].state(what)), what
        assert all(np.array_equal(x, y) for x, y in zip(a["cache"].evictions(20), b["cache"].evictions(20)))
    finally:
        a["cache"].close(); b["cache"].close()


def test_more_survivors_than_a_launch_has_threads_for():
    """2796203 units x 33 survivors are 2^23 + 1 workgroups of 512 threads in the kernel that moves the rows: 2^32 + 512
    threads, of which one launch would run the last 512.  Five units' inputs, repeated: the step after the prompt gives every unit what the same unit gets
    in a small handle of the same launch form, bit for bit."""
    P, m, R, d = 35, 33, 3, 64
    gen = torch.Generator(device="cuda")
    gen.manual_seed(9100)
    base = torch.randn(P + 1, 5, d, generator=gen, device="cuda").half()

    def next_out(units):
        x = base[:, torch.arange(units, device="cuda") % 5].contiguous().view(P + 1, units, 1, d)
        cache = wkv.Cache(units, 1, d, m, R, wkv.WKV_FP16, split=1, threads=256, streaming=wkv.WKV_LOADS_CACHED, log_capacity=1)
        try:
            out = torch.empty_like(x[P])
            cache.prefill(x[:P], x[:P], x[:P], None)
            cache.step(x[P], x[P], x[P], out)
            torch.cuda.synchronize()
            return out.view(units, d)
        finally:
            cache.close()

    try:
        few, many = next_out(30000), next_out(2796203)
        assert torch.equal(few, few[:5].repeat(6000, 1))
        assert torch.equal(many[:2796200].view(-1, 5, d), few[:5].expand(559240, 5, d))
        assert torch.equal(many[2796200:], few[:3])
    finally:
        torch.cuda.empty_cache()


@pytest.mark.parametrize("replayable", [0, 1])
def test_emptying_a_cache_after_a_failed_call_of_the_caller(replayable):
    """An error that a HIP call of the program has left behind (a device that does not exist) is not this call's: emptying
    the cache works."""
    cache = wkv.Cache(1, 3, 64, 37, 5, wkv.WKV_FP16, replayable=replayable)
    rows = np.empty((3, 0, 64), np.float16)
    try:
        assert wkv._lib.hipSetDevice(1 << 20) != 0
        cache.load(0, rows, rows, np.empty((3, 0), np.float64), np.empty((3, 0), np.int32))
        assert cache.tokens == 0
    finally:
        wkv._lib.hipGetLastError()
        cache.close()


def test_two_threads_with_prompts_of_their_own_lengths():
    """Handles are used from a thread each: what one prompt's launches need (workgroup memory by its length) must not be
    taken back by another's.  A short and a long prompt, 40 times from two threads at once, each on its own stream."""
    import threading
    prompts = []
    for P, seed in ((120, 1), (4096, 2)):
        gen = torch.Generator(device="cuda")
        gen.manual_seed(seed)
        q, k, v = (torch.randn(P, 4, 1, 64, generator=gen, device="cuda").half() for _ in range(3))
        cache = wkv.Cache(4, 1, 64, 40, 4, wkv.WKV_FP16, max_prompt=P)
        want = torch.empty_like(q)
        cache.prefill(q, k, v, want)
        torch.cuda.synchronize()
        prompts.append((cache, q, k, v, want, cache.state(wkv.WKV_POS), cache.state(wkv.WKV_V)))
    rows = np.empty((4, 0, 64), np.float16)
    empty = (rows, rows, np.empty((4, 0), np.float64), np.empty((4, 0), np.int32))
    failed = []

    def work(cache, q, k, v, want, pos, vals):
        try:
            stream = torch.cuda.Stream()
            with torch.cuda.stream(stream):
                out = torch.empty_like(q)
                for _ in range(40):
                    cache.load(0, *empty)
                    cache.prefill(q, k, v, out)
                    stream.synchronize()
                    assert torch.equal(out, want) and np.array_equal(cache.state(wkv.WKV_POS), pos)
                    assert np.array_equal(cache.state(wkv.WKV_V), vals)
        except BaseException as e:                      # (an assertion in a thread does not reach pytest by itself)
            failed.append(e)

    threads = [threading.Thread(target=work, args=p) for p in prompts]
    try:
        for th in threads:
            th.start()
        for th in threads:
            th.join()
        assert not failed, failed
    finally:
        for p in prompts:
            p[0].close()


@pytest.mark.parametrize("what,limit", [("one channel", 1.25), ("two rows", 1.25), ("every row", 2.5)])
def test_time_with_uneven_keys(what, limit):
    """The time of a prompt may depend on its data only so far, against keys of normal numbers.  With one large channel (20), which
    8-bit digits still hold, or with an element beyond the digits in two of the first keys (2^-24 beside 2^11, where they end at 2^-19): a quarter more.  With such an
    element in every key, which leaves the fp64 instruction for everything: 2.5 times as long (2.35 was measured; that instruction alone, before there were
    digits, takes 2.38).  256 units x 4096 tokens, the fastest of six."""
    P, U, d, m = 4096, 256, 128, 256
    gen = torch.Generator(device="cuda")
    gen.manual_seed(9300)
    q, k, v = (torch.randn(P, U, 1, d, generator=gen, device="cuda") for _ in range(3))
    uneven_q, uneven_k = q.clone(), k.clone()
    if what == "one channel":
        uneven_k[..., 5] += 20.0
        uneven_q[..., 5] *= 0.05
    else:
        rows_beyond = [5, 20] if what == "two rows" else slice(0, P)
        uneven_k[rows_beyond, ..., 5] = 2048.0
        uneven_k[rows_beyond, ..., 6] = 2.0 ** -24
        uneven_q[..., 5] = 0.0
    cache = wkv.Cache(U, 1, d, m, 9, wkv.WKV_FP16, max_prompt=P, log_capacity=1)
    rows = np.empty((U, 0, d), np.float16)
    empty = (rows, rows, np.empty((U, 0), np.float64), np.empty((U, 0), np.int32))

    def fastest(q, k):
        q, k, w = q.half(), k.half(), v.half()
        out, best = torch.empty_like(q), float("inf")
        for _ in range(6):
            cache.load(0, *empty)
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            cache.prefill(q, k, w, out)
            b.record()
            b.synchronize()
            best = min(best, a.elapsed_time(b))
        return best

    try:
        even, uneven = fastest(q, k), fastest(uneven_q, uneven_k)
    finally:
        cache.close()
    print(f"\n  {what}: {uneven:.2f} ms against {even:.2f}", flush=True)
    assert uneven <= limit * even


@pytest.mark.parametrize("dtype", ["fp16", "bf16"])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("P,units", [(129, 170), (129, 171), (3073, 256)])
def test_marked_rows_in_every_launch_form(P, units, d, dtype):
    """The three launch forms (two waves a tile up to 1536 tiles of a short prompt; one; two tiles a wave from 49152 tiles on, if the
    prompt has 3072 tokens and rows of 256 bytes) at odd numbers of tiles a unit, so that the last wave has half a share; units that differ in the rows the digits do not hold: none, one key, a query in the first and
    in the second tile of a pair, both at once, every key, every query (which take the fp64 instruction for whole workgroups), all
    rows, and every key of the first 32 only.  What the digits would drop meets large elements and differs from row to row:
    dropped, it would move score sums by 8e-9 and more (as plain float64 on the CPU says), which are held to 1e-9."""
    T = P + 4
    g = np.random.default_rng(9400 + units)
    q, k, v = (g.standard_normal((T, 9, d)).astype(np.float32) for _ in range(3))
    q[..., 1] *= 8.0
    k[..., 1] *= 8.0
    everything = slice(0, T)

    def mark(x, rows, unit, big):
        n = x[rows, unit, 1].shape
        x[rows, unit, big] = 2.0 ** 11                      # the digits end at 2^-19
        x[rows, unit, 1] = 2.0 ** -20 * (1 + 2 * g.integers(0, 4, n))

    for unit, keys, queries in ((1, 37, None), (2, None, 5), (3, None, 21), (4, 37, 21), (5, everything, None), (6, None, everything),
                                (7, everything, everything), (8, slice(0, 32), None)):
        if keys is not None:
            q[:, unit, 0] = 0.0
        if queries is not None:
            k[:, unit, 2] = 0.0
        if keys is not None:
            mark(k, keys, unit, 0)
        if queries is not None:
            mark(q, queries, unit, 2)
    cfg = synth.StreamConfig("pre-marked", 9400, 1, units, d, dtype, T, 100, 9)
    sel = np.arange(9) if P > 1000 else np.concatenate([np.arange(9), np.arange(units - 9, units)])
    host = [synth.to_storage(x, dtype) for x in (q, k, v)]
    dev = [parity.to_device(x, dtype)[:, torch.arange(units, device="cuda") % 9].contiguous() for x in host]
    out = torch.zeros_like(dev[0])
    cache = wkv.Cache(1, units, d, 100, 9, synth.DTYPE_CODE[dtype], split=1)
    try:
        cache.prefill(*(x[:P] for x in dev), out[:P])
        torch.cuda.synchronize()
        q, k, v = (synth.storage_to_f32(x, dtype)[:, sel % 9] for x in host)
        got = dict(out=parity.out_to_f64(out[:P][:, torch.from_numpy(sel).cuda()], dtype), cache=cache, q=q, k=k, v=v, sel=sel,
                   dev=(*dev, out), P=P)
        print(f"\n  {parity.compare_prefill(cfg, got, decode_steps=3)}", flush=True)
    finally:
        cache.close()


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("dtype", ["fp16", "bf16"])
@pytest.mark.parametrize("P,units", [(129, 3), (129, 460), (3073, 256)])
def test_an_infinite_value_stays_out_of_the_tiles_before_it(P, units, dtype, d):
    """A row attends to no newer token: an infinity in the value of token 19 (the second tile of 16, also the second one of
    a wave that takes two) leaves the rows of the tile before it what they are without it, bit for bit, in each of the
    three launch forms."""
    t = torch.float16 if dtype == "fp16" else torch.bfloat16
    gen = torch.Generator(device="cuda")
    gen.manual_seed(9200)
    base = torch.randn(3, P, 5, d, generator=gen, device="cuda").to(t)
    q, k, v = (x[:, torch.arange(units, device="cuda") % 5].contiguous().view(P, units, 1, d) for x in base)
    outs = []
    for _ in range(2):
        cache = wkv.Cache(units, 1, d, 100, 9, synth.DTYPE_CODE[dtype], log_capacity=1)
        try:
            outs.append(torch.empty_like(q))
            cache.prefill(q, k, v, outs[-1])
            torch.cuda.synchronize()
        finally:
            cache.close()
        v[19, :, 0, 7] = float("inf")
    clean, with_inf = outs
    assert torch.equal(clean[:16], with_inf[:16])
    assert not torch.isfinite(with_inf[19:, :, 0, 7]).any()     # (infinite, or NaN where a part of the weight is 0)
    assert torch.isfinite(clean.float()).all()


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("dtype", ["fp16", "bf16"])
def test_logits_far_beyond_the_exponential(dtype, d):
    """Logits at least 3e5 apart and up to 7e7 (3e10 in the units the kernels count in, where a 32-bit integer ends at 2e9): every row
    attends to one token, all other weights are 0 exactly.  Elements are chosen so that logits are exact."""
    P, U, m = 129, 3, 100
    g = np.random.default_rng(9500)
    q, k = np.zeros((P + 8, U, d), np.float32), np.zeros((P + 8, U, d), np.float32)
    v = g.standard_normal((P + 8, U, d)).astype(np.float32)
    q[..., 3] = 2.0 ** 14
    for u in range(U):
        k[:, u, 3] = 256.0 * (g.permutation(P + 8) + 1)
    cfg = synth.StreamConfig("pre-huge", 9500, 1, U, d, dtype, P + 8, m, 9)
    got = parity.gpu_prefill(cfg, P, arrays=(q, k, v))
    try:
        print(f"\n  {parity.compare_prefill(cfg, got, decode_steps=5)}", flush=True)
    finally:
        got["cache"].close()


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("dtype", ["fp16", "bf16"])
@pytest.mark.parametrize("P,units", [(130, 3), (129, 171)])
def test_digits_at_their_edges(P, units, dtype, d):
    """Rows around the edges of the 8-bit digits: a largest element whose upper digit just fits, would be rounded up to 128, or is -128
    (2 - 2^-7, the format's last number below 2, and -2); tiles of which no row uses the lowest digit (multiples of 2^-5), one row does, or
    all do, against each other (whose products are left out only where neither side uses it); an element whose last bit is the integers'
    last one, and one beyond (marked).  Dropping a lowest digit would move a logit by 1e-6 and more; score sums are held to 1e-9.  One wave
    and two a tile."""
    g = np.random.default_rng(9600)
    T = P + 4
    q, k, v = (g.standard_normal((T, 4, d)).astype(np.float32) for _ in range(3))
    last = 2.0 - 2.0 ** (-10 if dtype == "fp16" else -7)
    tiny = 2.0 ** -9 if dtype == "fp16" else 2.0 ** -13       # times 1 + 2^-10 or + 2^-7: uses the lowest digit of a row whose largest is below 4
    ulp = 2.0 ** -10 if dtype == "fp16" else 2.0 ** -7
    for u in range(4):
        for x, other in ((q, k), (k, q)):
            x[:64, u] = np.clip(np.rint(x[:64, u] * 32) / 32, -3.0, 3.0)              # four tiles without the lowest digit
            x[5, u, 1], x[6, u, 1], x[7, u, 1], x[8, u, 1] = 2.0 - 2.0 ** -7, last, -last, -2.0
            x[5:9, u, 2:] *= 0.5                                                    # (below 2: those are the largest)
            if u in (1, 3):
                x[40, u, 3] = tiny * (1 + ulp) / 4                                  # one row of the third tile
            x[70:86, u, 4] = tiny * (1 + ulp) / 4                                   # every row of a tile, and its neighbours' some
            other[:, u, 3:5] *= 8.0                                                 # what they meet is large
        if u >= 2:
            # last bit 2^-24: the format's last one in fp16; in bf16 the last of integers whose largest is 2^6 and has 31 bits
            k[90, u, 0], k[90, u, 5], q[:, u, 0] = 2.0 ** 6, (2.0 ** -14 if dtype == "fp16" else 2.0 ** -17) * (1 + ulp), 0.0
            k[91, u, 0], k[91, u, 5] = 2.0 ** 11, 2.0 ** -14 * (1 + ulp)            # beyond: marked
    cfg = synth.StreamConfig("pre-digit", 9600, 1, 4, d, dtype, T, 60, 9)
    rep = np.arange(units) % 4
    big = synth.StreamConfig("pre-digit", 9600, 1, units, d, dtype, T, 60, 9)
    got = parity.gpu_prefill(big, P, arrays=tuple(np.ascontiguousarray(x[:, rep]) for x in (q, k, v)), units_sel=np.arange(min(units, 4)) if units > 4 else None)
    try:
        print(f"\n  {parity.compare_prefill(big, got, decode_steps=3)}", flush=True)
    finally:
        got["cache"].close()


@pytest.mark.parametrize("code", ["7FFF", "FFFF", "7FF9"])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("dtype", ["fp16", "bf16"])
@pytest.mark.parametrize("P,units", [(129, 170), (129, 171), (3073, 256)])
def test_a_nan_is_a_nan_whatever_its_bits(P, units, dtype, d, code):
    """NaNs at the top of the code range (memory filled with ones; other makers' conversions), in one element, in whole rows and in a row
    of zeros, of queries and of keys, in every launch form: what the call leaves is bit for bit what the format's usual NaN leaves, and the rows
    that are NaN are those that attend to one, or ask with one."""
    t = torch.float16 if dtype == "fp16" else torch.bfloat16
    gen = torch.Generator(device="cuda")
    gen.manual_seed(9700)
    base = [x.to(t) for x in torch.randn(3, P, 9, d, generator=gen, device="cuda")]
    usual = torch.tensor([float("nan")], dtype=t).view(torch.int16).item()
    given = np.array([int(code, 16)], np.uint16).view(np.int16).item()
    keys, queries = {}, {}                                     # unit: the first key, the queries that are NaN

    def prompt(nan):
        q, k, v = (x.clone() for x in base)
        q, k = q.view(torch.int16), k.view(torch.int16)
        k[37, 1, 5] = nan; keys[1] = 37
        q[50, 2, 7] = nan; queries[2] = [50]
        k[37, 3] = nan; keys[3] = 37
        q[21, 4] = nan; queries[4] = [21]
        k[:, 5] = nan; keys[5] = 0
        q[:, 6] = nan; queries[6] = list(range(P))
        k[100, 7] = 0; k[100, 7, 3] = nan; keys[7] = 100
        q[16, 8] = 0; q[16, 8, 3] = nan; queries[8] = [16]
        return [x.view(t)[:, torch.arange(units, device="cuda") % 9].contiguous() for x in (q, k, v)]

    got = []
    for nan in (usual, given):
        q, k, v = prompt(nan)
        out = torch.zeros_like(q)
        cache = wkv.Cache(1, units, d, 100, 9, synth.DTYPE_CODE[dtype], split=1, log_capacity=1)
        try:
            cache.prefill(q, k, v, out)
            torch.cuda.synchronize()
            got.append((out.float().cpu().numpy(), *(cache.state(w) for w in (wkv.WKV_SCORE_SUM, wkv.WKV_POS, wkv.WKV_STATUS))))
        finally:
            cache.close()
    for a, b in zip(*got):
        assert np.array_equal(a, b, equal_nan=a.dtype.kind == "f")
    want = np.zeros((P, 9), bool)
    for u, first in keys.items():
        want[first:, u] = True
    for u, rows in queries.items():
        want[rows, u] = True
    want = want[:, np.arange(units) % 9, None]
    assert np.array_equal(np.isnan(got[1][0]), np.broadcast_to(want, got[1][0].shape))


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("P,units,marked", [(130, 4, 0), (129, 171, 0), (129, 171, 1), (3073, 256, 0)])
@pytest.mark.parametrize("largest", [2.0 ** 126, 2.0 ** -110])
def test_values_at_both_ends_of_bf16(largest, P, units, marked, d):
    """Logits rise by 7 octaves of the weight after the first tiles, which is less than what moves the softmax reference, and the token they rise
    for has a value near the format's largest: the output is finite, and so must be all that is added up on the way.  And small values, whose products
    with the lowest parts of small weights are below the normal fp32 numbers (from 2^-118 on results are rounded to bf16's own subnormal numbers, where the bound below
    does not hold).  Every launch form; with marked: keys that take the fp64 instruction."""
    T, m = P + 4, 100
    g = np.random.default_rng(9800)
    q, k = (0.05 * g.standard_normal((T, 4, d)).astype(np.float32) for _ in range(2))
    v = g.uniform(0.5, 1.0, (T, 4, d)).astype(np.float32) * np.float32(largest) * np.where(g.random((T, 4, d)) < 0.5, -1, 1).astype(np.float32)
    if largest > 1.0:
        v *= np.float32(2.0 ** -9)
    q[..., 0] = np.sqrt(d)
    k[..., 0] = 0.0
    for u in range(4):
        t = 40 + 13 * u
        k[t, u, 0] = 7.0 * np.log(2.0)
        v[t, u] = g.uniform(0.5, 1.0, d) * largest
    if marked:
        k[:, :, 1] = 2.0 ** 10
        q[:, :, 1] = 0.0
        k[:, :, 2] = 2.0 ** -22
    cfg = synth.StreamConfig("pre-ends", 9800, 1, units, d, "bf16", T, m, 9)
    rep = np.arange(units) % 4
    got = parity.gpu_prefill(cfg, P, arrays=tuple(np.ascontiguousarray(x[:, rep]) for x in (q, k, v)), units_sel=np.arange(4))
    try:
        print(f"\n  {parity.compare_prefill(cfg, got)}", flush=True)
    finally:
        got["cache"].close()


@pytest.mark.parametrize("units", [(1 << 22) + 3, (1 << 24) - 1])
def test_prompts_of_more_units_than_a_launch_has_threads_for(units):
    """2^22 units and more are 2^32 threads in the kernel that ranks a unit's tokens, 2^24 - 1 (rounded up to whole partitions) in the two contractions
    as well.  Two tokens into one slot; five units' inputs, repeated: the step after the prompt gives every unit what the
    same unit gets in a smaller handle of the same launch form, bit for bit."""
    P, d = 2, 64
    gen = torch.Generator(device="cuda")
    gen.manual_seed(9900)
    base = torch.randn(P + 1, 5, d, generator=gen, device="cuda").half()

    def next_out(units):
        x = base[:, torch.arange(units, device="cuda") % 5].contiguous().view(P + 1, units, 1, d)
        cache = wkv.Cache(units, 1, d, 1, 1, wkv.WKV_FP16, split=1, threads=256, streaming=wkv.WKV_LOADS_CACHED, log_capacity=1)
        try:
            out = torch.empty_like(x[P])
            cache.prefill(x[:P], x[:P], x[:P], None)
            cache.step(x[P], x[P], x[P], out)
            torch.cuda.synchronize()
            return out.view(units, d)
        finally:
            cache.close()

    try:
        few, many = next_out(30000), next_out(units)
        assert torch.equal(few, few[:5].repeat(6000, 1))
        whole = units // 5 * 5
        assert torch.equal(many[:whole].view(-1, 5, d), few[:5].expand(units // 5, 5, d))
        assert torch.equal(many[whole:], few[:units - whole])
    finally:
        torch.cuda.empty_cache()
