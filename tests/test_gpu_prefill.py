"""GPU parity of the batched prefill initialisation (Sec. 3.3: the cache starts
with the last C prompt queries, each inserted with its Exact Top-K support over
its causal prefix) against the oracle's query-by-query prefill.

bf16 handles score U prompt positions x all heads per launch on the matrix
cores and select them from lists of the entries above a bound, or for short
prompts from stored score rows; the cache state they leave (normalised queries, supports, counts,
insertion count) must equal the oracle's, supports up to near-ties at the K
boundary (same rule as the decode parity tests)."""
import numpy as np
import pytest

from gpu_harness import Tally, check_selection, handle_of, params_of, to_dev, torch_cuda
from oracle import oracle as O
from paper_2607_27692_amd import retopk as R
from paper_2607_27692_amd.inputs import WORKLOADS, bf16_bits_to_f32, make_inputs, to_bf16_bits

pytestmark = pytest.mark.gpu


def _gpu_prefill(p, dtype, q_tail_raw, k_raw, v_raw, prefill_len):
    torch = torch_cuda()
    h = handle_of(p, dtype)
    n = q_tail_raw.shape[-2]
    h.prefill_init(to_dev(q_tail_raw), n, to_dev(k_raw), to_dev(v_raw), prefill_len)
    torch.cuda.synchronize()
    st = h.get_state()
    h.close()
    return st


def _check_slot(where, gsupp, osupp, q, krows, length, tally):
    if np.array_equal(gsupp, osupp):
        tally.exact += 1
        return
    universe = np.arange(length, dtype=np.int32)
    check_selection(gsupp, osupp, universe, O.scores(q, krows, universe), where, tally)


def _compare_states(p, gst, ost, heads, q_tail, k, prefill_len, tally):
    n = q_tail.shape[-2]
    C, G = p.cache_cap, p.n_q_heads // p.n_kv_heads
    assert gst["n_inserted"] == ost["n_inserted"] == n
    for bh in heads:
        b, h = divmod(bh, p.n_q_heads)
        for u in range(max(0, n - C), n):
            slot = u % C
            where = f"b={b} h={h} position u={u} (slot {slot})"
            length = prefill_len - n + u + 1
            _check_slot(where, gst["supp"][bh, slot], ost["supp"][bh, slot], q_tail[b, h, u],
                        k[b, h // G], length, tally)
            assert gst["cnt"][bh, slot] == ost["cnt"][bh, slot] == min(p.k, length), where
            gq, oq = gst["qbar"][bh, slot], ost["qbar"][bh, slot]
            assert np.abs(gq.view(np.int32) - oq.view(np.int32)).max() <= 1, f"{where}: q_bar"


def _mask(p, groups):
    G = p.n_q_heads // p.n_kv_heads
    heads = [b * p.n_q_heads + g * G + j for b in range(p.batch) for g in groups for j in range(G)]
    m = np.zeros(p.heads, np.uint8)
    m[heads] = 1
    return heads, m


def test_prefill_batched_16k():
    """Every prompt-tail query of KV groups 0 and 7 at 16K (256 positions)."""
    w = WORKLOADS["16k"]
    print(f"batched prefill {w.name}", flush=True)
    inp = make_inputs(w)
    p = params_of(w)
    heads, mask = _mask(p, [0, w.n_kv_heads - 1])
    qt, kf = inp.q_tail, inp.k
    orc = O.Oracle(p)
    orc.prefill_init(qt, kf, inp.v, w.prompt_len, head_mask=mask)
    gst = _gpu_prefill(p, w.dtype, inp.q_tail_raw, inp.k_raw, inp.v_raw, w.prompt_len)
    tally = Tally()
    _compare_states(p, gst, orc.get_state(), heads, qt, kf, w.prompt_len, tally)
    print(tally, flush=True)


@pytest.mark.parametrize("name, positions", [
    ("128k", (0, 1, 40, 41, 42, 81, 82, 255, 256, 492, 493, 510, 511)),
    ("128k_28x4_paper", (0, 1, 15, 16, 30, 31)),
])
def test_prefill_batched_128k_sampled(name, positions):
    """128K: 512 positions in several launches (positions on both sides of the
    launch boundaries and at the ends), and the 28 / 4 head layout with 32 slots;
    the first and last KV groups, against the oracle's Exact Top-K of each query
    over its causal prefix."""
    w = WORKLOADS[name]
    print(f"batched prefill {w.name}", flush=True)
    inp = make_inputs(w)
    p = params_of(w)
    heads, mask = _mask(p, [0, w.n_kv_heads - 1])
    gst = _gpu_prefill(p, w.dtype, inp.q_tail_raw, inp.k_raw, inp.v_raw, w.prompt_len)
    n = w.cache_cap
    assert gst["n_inserted"] == n
    qt, kf, vf = inp.q_tail, inp.k, inp.v      # widened once
    tally = Tally()
    for u in positions:
        length = w.prompt_len - n + u + 1
        _, osel, _ = O.exact(p, qt[:, :, u], kf, vf, length, head_mask=mask)
        for bh in heads:
            b, h = divmod(bh, w.n_q_heads)
            where = f"b={b} h={h} position u={u}"
            _check_slot(where, gst["supp"][bh, u], osel[b, h], qt[b, h, u], kf[b, h // w.group],
                        length, tally)
            assert gst["cnt"][bh, u] == w.k
            oq = O.normalize(qt[b, h, u])
            assert np.abs(gst["qbar"][bh, u].view(np.int32) - oq.view(np.int32)).max() <= 1
    print(tally, flush=True)


SHAPES = [
    # label, workload changes, prompt-tail positions beyond C
    ("g8_d64", dict(n_q_heads=8, n_kv_heads=1, head_dim=64, prompt_len=3000, k=64,
                    cache_cap=40, n_centers=32), 0),
    ("g1_d128", dict(n_q_heads=4, n_kv_heads=4, prompt_len=5000, k=100, cache_cap=24,
                     n_centers=48), 0),
    ("b2_more_than_c", dict(batch=2, n_q_heads=8, n_kv_heads=2, prompt_len=4100, k=128,
                            cache_cap=20, n_centers=32), 7),
    ("k_above_len", dict(n_q_heads=4, n_kv_heads=2, prompt_len=300, k=512, cache_cap=30,
                         n_centers=8), 0),
    # groups of 7 and 6 query heads (virtual queries u * G + j across tile edges)
    ("g7_d128", dict(n_q_heads=7, n_kv_heads=1, prompt_len=3500, k=96, cache_cap=36,
                     n_centers=16), 0),
    ("g6_d64_b2", dict(batch=2, n_q_heads=12, n_kv_heads=2, head_dim=64, prompt_len=2600,
                       k=64, cache_cap=20, n_centers=12), 3),
]


@pytest.mark.parametrize("label,change,extra", SHAPES, ids=[s[0] for s in SHAPES])
def test_prefill_batched_shapes(label, change, extra):
    """Group sizes 8 and 1, d = 64, batch 2, more prompt-tail queries than cache
    slots (the early ones are overwritten), K above the causal length (the whole
    prefix is the support), and groups of 7 and 6: all heads, all positions."""
    w = WORKLOADS["16k"].with_(**change)
    w = w.with_(cache_cap=w.cache_cap + extra)   # generate the extra positions too
    print(f"batched prefill {label}", flush=True)
    inp = make_inputs(w)
    p = params_of(w, cache_cap=w.cache_cap - extra)
    qt, kf = inp.q_tail, inp.k
    orc = O.Oracle(p)
    orc.prefill_init(qt, kf, inp.v, w.prompt_len)
    gst = _gpu_prefill(p, w.dtype, inp.q_tail_raw, inp.k_raw, inp.v_raw, w.prompt_len)
    tally = Tally()
    _compare_states(p, gst, orc.get_state(), list(range(p.heads)), qt, kf, w.prompt_len, tally)
    print(tally, flush=True)


@pytest.mark.parametrize("prompt_len", [6000, 9000])      # by score rows, by lists
def test_prefill_batched_equal_keys(prompt_len):
    """Identical key rows: every score of a query ties, so each support is the K
    lowest positions of its prefix (Top-K ties broken by index)."""
    w = WORKLOADS["16k"].with_(n_q_heads=8, n_kv_heads=2, prompt_len=prompt_len, k=300,
                               cache_cap=16, n_centers=8)
    print("batched prefill equal keys", flush=True)
    inp = make_inputs(w)
    k_raw = np.broadcast_to(inp.k_raw[:, :, :1], inp.k_raw.shape).copy()
    k_f32 = (k_raw.astype(np.uint32) << 16).view(np.float32)
    p = params_of(w)
    orc = O.Oracle(p)
    orc.prefill_init(inp.q_tail, k_f32, inp.v, w.prompt_len)
    ost = orc.get_state()
    assert (ost["supp"] == np.arange(w.k, dtype=np.int32)).all()
    gst = _gpu_prefill(p, w.dtype, inp.q_tail_raw, k_raw, inp.v_raw, w.prompt_len)
    assert np.array_equal(gst["supp"], ost["supp"])
    assert np.array_equal(gst["cnt"], ost["cnt"])


def _launches(p, dtype, q_tail_raw, k_raw, prefill_len):
    """State after a prefill, and its launches: (score products, bounds, selections)."""
    torch = torch_cuda()
    with handle_of(p, dtype) as h:
        h.profile(True)
        q, k = to_dev(q_tail_raw), to_dev(k_raw)
        h.prefill_init(q, q_tail_raw.shape[-2], k, k, prefill_len)
        torch.cuda.synchronize()
        prof = h.profile_read()
        return h.get_state(), tuple(prof[x][0] for x in ("prefill_score", "retopk_filter", "retopk_final"))


BOUND_SHAPES = [
    # label, workload changes, equal key rows, whether lists are kept (prompts of 2 cap
    # rows on, cap = max(8 K, 4096))
    # the last prompt of score rows and the first of lists, of more positions than
    # fit between one and two lists' rows: prefixes from 4081 and 4082 rows on
    ("below_2cap", dict(n_q_heads=2, n_kv_heads=1, head_dim=64, prompt_len=8176, k=64,
                        cache_cap=4096, n_centers=16), None, False),
    ("from_2cap", dict(n_q_heads=2, n_kv_heads=1, head_dim=64, prompt_len=8177, k=512,
                       cache_cap=4096, n_centers=16), None, True),
    # K = 1, and K = 2048 (list capacity 16384, group maxima of single tiles)
    ("k1", dict(n_q_heads=4, n_kv_heads=1, prompt_len=9001, k=1, cache_cap=9, n_centers=16), None, True),
    ("k2048_d64", dict(n_q_heads=2, n_kv_heads=2, head_dim=64, prompt_len=33001, k=2048,
                       cache_cap=6, n_centers=16), None, True),
    # more than 4096 group maxima
    ("maxima_5000", dict(n_q_heads=4, n_kv_heads=2, prompt_len=40000, k=1024, cache_cap=5,
                         n_centers=16), None, True),
    # 140 virtual queries a group: two waves side by side, padded columns
    ("two_query_tiles", dict(n_q_heads=7, n_kv_heads=1, prompt_len=8203, k=40, cache_cap=20,
                             n_centers=16), None, True),
    # prefixes past one bitmap pass (131072 rows)
    ("two_bitmap_passes", dict(n_q_heads=2, n_kv_heads=1, head_dim=64, prompt_len=140003, k=64,
                               cache_cap=3, n_centers=64), None, True),
    # for about half of the queries the best keys are one run of equal rows longer than
    # a list
    ("overflow", dict(n_q_heads=4, n_kv_heads=2, prompt_len=9000, k=50, cache_cap=5,
                      n_centers=8), (1000, 7000), True),
]


@pytest.mark.parametrize("label,change,equal,lists", BOUND_SHAPES, ids=[s[0] for s in BOUND_SHAPES])
def test_prefill_batched_bounds_and_lists(label, change, equal, lists):
    """The bounded selection of the batched prefill where it can go wrong: the prompts
    it begins with, the smallest and largest K, padded query columns, many maxima, several
    bitmap passes, lists that overflow.  Supports exact up to near-ties, as in the other
    cases, and the launches tell which path ran."""
    w = WORKLOADS["16k"].with_(**change)
    print(f"batched prefill {label}", flush=True)
    inp = make_inputs(w)
    k_raw = inp.k_raw
    if equal is not None:
        k_raw = k_raw.copy()
        # equal rows, eight times as long as the others (bf16 exponent + 3): far above or
        # far below every other score of a query
        k_raw[:, :, equal[0]:equal[1]] = k_raw[:, :, equal[0]:equal[0] + 1] + (3 << 7)
    kf = (k_raw.astype(np.uint32) << 16).view(np.float32)
    p = params_of(w)
    orc = O.Oracle(p)
    orc.prefill_init(inp.q_tail, kf, inp.v, w.prompt_len)
    gst, (scores, bounds, selects) = _launches(p, w.dtype, inp.q_tail_raw, k_raw, w.prompt_len)
    tally = Tally()
    _compare_states(p, gst, orc.get_state(), list(range(p.heads)), inp.q_tail, kf, w.prompt_len,
                    tally)
    print(tally, f"launches {scores} {bounds} {selects}", flush=True)
    if not lists:
        assert bounds == 0 and scores == selects
    elif equal is None:
        assert scores == 2 * bounds and selects == bounds       # bound and list per launch
    else:
        assert scores == 1 + bounds and selects == bounds > 1   # lists again, no score rows


def _segments(k, rng, lead):
    """Rows 2000 .. 7999 in 6 segments of one score level each, far above the other rows
    for a query along `lead`: more rows than a list holds reach the bound that a sample
    of the keys gives."""
    for j, level in enumerate(rng.permutation(6)):
        k[:, :, 2000 + 1000 * j:3000 + 1000 * j] = (6.0 + 0.5 * level) * lead


def _masked(k, rng, lead):
    """The first 5000 rows masked with nearly the lowest bf16 value."""
    k[:, :, :5000] = -3.0e38


def _equal_run(k, rng, lead):
    """6000 equal rows above all others: ties far past a list's capacity."""
    k[:, :, 1000:7000] = 8.0 * lead


@pytest.mark.parametrize("keys, reruns", [(_segments, (1, 1)), (_masked, (0, 0)), (_equal_run, (1, 3))],
                         ids=["segments", "masked", "equal_run"])
@pytest.mark.parametrize("d", [64, 128])
def test_prefill_overflowing_lists(keys, reruns, d):
    """Lists that overflow are collected again above the K-th largest entry they hold,
    and no score row is stored; masked rows do not make a list overflow."""
    print(f"batched prefill {keys.__name__} d={d}", flush=True)
    rng = np.random.default_rng(d)
    L, K, C, Hq, Hkv = 17000, 512, 6, 4, 2
    lead = (np.abs(rng.standard_normal(d)) + 0.5).astype(np.float32)
    q = (0.2 * rng.standard_normal((1, Hq, C, d)) + lead).clip(0.05).astype(np.float32)
    k = rng.standard_normal((1, Hkv, L, d)).astype(np.float32)
    keys(k, rng, lead)
    q_raw, k_raw = to_bf16_bits(q), to_bf16_bits(k)
    q, k = bf16_bits_to_f32(q_raw), bf16_bits_to_f32(k_raw)
    p = O.Params(1, Hq, Hkv, d, L, K, C, 1, 0, 0.5, 0)
    gst, (scores, bounds, selects) = _launches(p, "bf16", q_raw, k_raw, L)
    tally = Tally()
    for bh in range(Hq):
        for u in range(C):
            length = L - C + u + 1
            # masked rows overflow fp32, which the fp64 order of the other rows never reaches
            universe = np.arange(5000 if keys is _masked else 0, length, dtype=np.int32)
            s = O.scores(q[0, bh, u], k[0, bh // (Hq // Hkv)], universe)
            want = np.sort(universe[np.lexsort((universe, -s))[:K]])
            got = gst["supp"][bh, u]
            assert gst["cnt"][bh, u] == K
            if np.array_equal(got, want):
                tally.exact += 1
            else:
                check_selection(got, want, universe, s, f"h={bh} position {u}", tally)
    print(tally, f"launches {scores} {bounds} {selects}", flush=True)
    assert scores == 1 + bounds and selects == bounds, "some positions stored score rows"
    assert reruns[0] <= bounds - 1 <= reruns[1]


def _workspace_case(seed):
    """A layer whose batched prefill takes the whole workspace (32 heads x 256 positions)."""
    torch = torch_cuda()
    w = WORKLOADS["16k"].with_(prompt_len=9000, cache_cap=256)
    gen = torch.Generator("cuda")
    gen.manual_seed(seed)
    k = torch.randn((1, w.n_kv_heads, w.max_len, w.head_dim), generator=gen, device="cuda").bfloat16()
    q = torch.randn((1, w.n_q_heads, w.cache_cap, w.head_dim), generator=gen, device="cuda").bfloat16()
    return w, k, q


def test_prefill_workspace_is_shared():
    """Handles of one device (layers of one model) keep one prefill workspace between
    them, and none once the last handle is gone."""
    torch = torch_cuda()
    print("prefill workspace of several handles", flush=True)
    w, k, q = _workspace_case(1)
    p = params_of(w)
    free = lambda: torch.cuda.mem_get_info()[0]  # noqa: E731
    before = free()
    handles = [handle_of(p, w.dtype) for _ in range(4)]
    held = before - free()                      # the handles' own memory
    kept = []
    for h in handles:
        h.prefill_init(q, w.cache_cap, k, k, w.prompt_len)
        kept.append(before - free() - held)
    assert kept[0] <= 300 << 20
    assert kept[-1] <= kept[0] + (16 << 20), f"{[x >> 20 for x in kept]} MiB kept"
    states = [h.get_state() for h in handles]
    for st in states[1:]:
        assert all(np.array_equal(st[x], states[0][x]) for x in ("qbar", "supp", "cnt"))
    for h in handles:
        h.close()
    assert before - free() <= 32 << 20, f"{(before - free()) >> 20} MiB left"


def test_prefill_on_two_threads():
    """Two threads prefill their own handles on their own streams, over and over: each
    gets what it gets alone."""
    import threading
    torch = torch_cuda()
    print("prefill on two threads", flush=True)
    cases = [_workspace_case(s) for s in (2, 3)]
    want, got, errors = [], [None, None], []
    for w, k, q in cases:
        with handle_of(params_of(w), w.dtype) as h:
            h.prefill_init(q, w.cache_cap, k, k, w.prompt_len)
            want.append(h.get_state())
    torch.cuda.synchronize()

    def work(i):
        try:
            w, k, q = cases[i]
            stream = torch.cuda.Stream()
            with handle_of(params_of(w), w.dtype) as h:
                for _ in range(8):
                    h.prefill_init(q, w.cache_cap, k, k, w.prompt_len, stream=stream)
                got[i] = h.get_state()
        except Exception as e:  # noqa: BLE001
            errors.append(e)

    threads = [threading.Thread(target=work, args=(i,)) for i in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
    for i in range(2):
        assert all(np.array_equal(got[i][x], want[i][x]) for x in ("qbar", "supp", "cnt")), i


def test_prefill_under_capture_is_refused():
    """A batched prefill waits for its own work, so a capturing stream is refused before
    anything is recorded; the capture and the handle stay usable."""
    torch = torch_cuda()
    print("prefill under capture", flush=True)
    w, k, q = _workspace_case(4)
    with handle_of(params_of(w), w.dtype) as h:
        h.prefill_init(q, w.cache_cap, k, k, w.prompt_len)
        want = h.get_state()
        x = torch.zeros(8, device="cuda")
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            with pytest.raises(R.RetopkError) as e:
                h.prefill_init(q, w.cache_cap, k, k, w.prompt_len)
            x.add_(1.0)
        assert e.value.code == -4
        for i in range(3):
            graph.replay()
            torch.cuda.synchronize()
            assert (x == i + 1).all()
        h.prefill_init(q, w.cache_cap, k, k, w.prompt_len)
        got = h.get_state()
        assert all(np.array_equal(got[x], want[x]) for x in ("qbar", "supp", "cnt"))
