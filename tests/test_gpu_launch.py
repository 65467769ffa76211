"""Launch machinery of the batched path: HIP-graph capture and replay of the
forward launch (qs_set_graphs) and the launch tuner with its cache
(qs_tune).  Neither may change a result bit: graph replays are compared with
eager launches of the same arguments, several times, with other eager work
and synchronisations between them; tuned launches with untuned ones.
"""
import numpy as np
import pytest

from paper_2308_09348_amd import workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def qs():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2308_09348_amd as qs
    return qs


def _np(d):
    return {k: v.cpu().numpy() for k, v in d.items()}


def _same(a, b, what):
    for k in a:
        assert np.array_equal(a[k], b[k]), (what, k)


def _case(**kw):
    p = workloads.scaled(workloads.focused_3d(), n_samples=9037, n_steps=256)
    p.update(kw)
    return p


def test_graph_replays_match_eager(qs):
    import torch
    eager = qs.Context(0)
    graph = qs.Context(0)
    graph.set_graphs(True)
    p = _case()
    other = _case(n_samples=3000, n_steps=128, rr_model="classical")
    ref = _np(eager.forward(p))
    for r in range(4):
        got = _np(graph.forward(p))
        _same(got, ref, f"replay {r}")
        # eager work on the same context and on torch between the replays
        eager.forward(other)
        torch.cuda.synchronize()
        x = torch.arange(1 << 20, device="cuda", dtype=torch.float64).sum()
        assert x.item() > 0
    # new per-shot parameters, same shapes: the replay copies the new shot table
    q = dict(p, a0=37.0, x_off_um=-1.0, gamma0=2300.0)
    _same(_np(graph.forward(q)), _np(eager.forward(q)), "new parameters")
    # another class of launch on the graph context is captured separately
    _same(_np(graph.forward(other)), _np(eager.forward(other)), "second graph")
    _same(_np(graph.forward(p)), ref, "first graph again")
    eager.close()
    graph.close()


def test_graph_replays_match_eager_batched(qs):
    eager = qs.Context(0)
    graph = qs.Context(0)
    graph.set_graphs(True)
    shots = [_case(n_samples=n, a0=a, shot=0) for n, a in ((5000, 20.0), (777, 60.0),
                                                           (12001, 45.0))]
    shots = [dict(s, chi_fp64=0.1) for s in shots]
    ref = [_np(o) for o in eager.forward_batched(shots)]
    for r in range(3):
        got = [_np(o) for o in graph.forward_batched(shots)]
        for k in range(len(shots)):
            _same(got[k], ref[k], f"replay {r} shot {k}")
        eager.forward(shots[1])
    eager.close()
    graph.close()


def test_tuner_choice_cache_and_results(qs, tmp_path):
    p = _case(n_samples=1 << 17, n_steps=128)
    plain = qs.Context(0)
    ref = _np(plain.forward(p))
    tuned = qs.Context(0)
    cache = tmp_path / "tune.txt"
    t = tuned.tune(p, cache_path=str(cache))
    assert not t["from_cache"]
    assert t["dep_tile"] in (1024, 2048, 4096, 8192)
    assert t["phase_cap"] in (0, 2, 3) and t["dep_cap"] in (0, 2, 4)
    assert 0 < t["phase_ms"] < 1e3 and 0 < t["deposit_ms"] < 1e3
    lines = cache.read_text().splitlines()
    assert len(lines) == 1 and lines[0].startswith("qscatter-tune-1 ")
    # the tuned launch gives the untuned bits
    _same(_np(tuned.forward(p)), ref, "tuned")
    # a new context reads the choice from the cache
    again = qs.Context(0)
    u = again.tune(p, cache_path=str(cache))
    assert u["from_cache"]
    assert (u["dep_tile"], u["phase_cap"], u["dep_cap"]) == (t["dep_tile"], t["phase_cap"],
                                                             t["dep_cap"])
    assert len(cache.read_text().splitlines()) == 1
    _same(_np(again.forward(p)), ref, "from cache")
    for c in (plain, tuned, again):
        c.close()


@pytest.mark.parametrize("tile", [1024, 8192])
def test_deposit_tile_leaves_results_unchanged(qs, tmp_path, tile):
    """A cache line forcing each extreme tile (and capped residency): the
    moments are summed per 1024-sample tile whatever the deposit item."""
    import re
    p = _case(n_samples=50001, deposit="gauss")
    plain = qs.Context(0)
    ref = _np(plain.forward(p))
    probe = qs.Context(0)
    cache = tmp_path / "tune.txt"
    probe.tune(p, cache_path=str(cache))
    line = cache.read_text().split()
    # replace the choice (fields 10-12 after the tag) with the forced one
    line[10:13] = [str(tile), "2", "2"]
    cache.write_text(" ".join(line) + "\n")
    forced = qs.Context(0)
    u = forced.tune(p, cache_path=str(cache))
    assert u["from_cache"] and u["dep_tile"] == tile and u["dep_cap"] == 2
    _same(_np(forced.forward(p)), ref, f"tile {tile}")
    assert re.match(r"qscatter-tune-1 \S+/\d+ ", cache.read_text())
    for c in (plain, probe, forced):
        c.close()


def test_tuner_on_a_batch(qs, tmp_path):
    """The class of a batch (shot count and total samples) is tuned as a
    whole; the tuned batched launch, replayed from a graph, gives the bits of
    the plain one."""
    shots = [_case(n_samples=n, a0=a) for n, a in ((3000, 15.0), (20000, 50.0), (9000, 80.0),
                                                   (1, 30.0))]
    plain = qs.Context(0)
    ref = [_np(o) for o in plain.forward_batched(shots)]
    tuned = qs.Context(0)
    cache = tmp_path / "tune.txt"
    t = tuned.tune(shots, cache_path=str(cache))
    assert not t["from_cache"] and t["dep_tile"] in (1024, 2048, 4096, 8192)
    key = cache.read_text().split()
    assert key[9] == "2"  # floor(log2 4 shots)
    tuned.set_graphs(True)
    for r in range(2):
        got = [_np(o) for o in tuned.forward_batched(shots)]
        for k in range(len(shots)):
            _same(got[k], ref[k], f"tuned batch, launch {r}, shot {k}")
    plain.close()
    tuned.close()


def test_graph_replays_follow_the_shadow_stride(qs):
    """The FP64-shadow launches of a captured batch take their item count from
    shadow_stride: a new stride that leaves every buffer size unchanged
    (16384 and 6400 samples, stride 64 then 63) must be captured anew, not
    replayed with the old count."""
    eager = qs.Context(0)
    graph = qs.Context(0)
    graph.set_graphs(True)
    base = [_case(n_samples=n, a0=a, shot=0, validate_fp64=True)
            for n, a in ((16384, 30.0), (6400, 45.0))]
    for stride in (64, 63, 64):
        shots = [dict(s, shadow_stride=stride) for s in base]
        ref = [_np(o) for o in eager.forward_batched(shots)]
        for r in range(2):
            got = [_np(o) for o in graph.forward_batched(shots)]
            for k in range(len(shots)):
                _same(got[k], ref[k], f"stride {stride} replay {r} shot {k}")
    eager.close()
    graph.close()


def test_profiled_calls_are_kept_for_the_sum(qs):
    """Kernel events are kept per profiled call (a ring of 64 sets): the sum
    over calls enqueued back to back equals the per-call durations read one
    by one, only the last 64 calls are summed, and profiled launches are
    never graph replays."""
    ctx = qs.Context(0)
    p = _case(n_samples=4000, n_steps=64)
    out = ctx.forward(p)
    with pytest.raises(qs.QScatterError):
        ctx.timings_sum()  # profiling off
    ctx.set_profiling(True)
    with pytest.raises(qs.QScatterError):
        ctx.timings_sum()  # no profiled call yet
    each = []
    for _ in range(3):
        ctx.forward(p, out=out, check=False)
        each.append(ctx.last_timings())
    n, tot = ctx.timings_sum()
    assert n == 3
    for k in tot:
        assert tot[k] == pytest.approx(sum(t[k] for t in each), rel=1e-12, abs=1e-9)
    assert tot["phase"] > 0 and tot["deposit"] > 0
    # back to back, read once: the ring keeps the last 64
    for _ in range(70):
        ctx.forward(p, out=out, check=False)
    n, tot = ctx.timings_sum()
    assert n == 64 and tot["phase"] > 0
    last = ctx.last_timings()
    assert 0 < last["phase"] <= tot["phase"]
    # switching profiling on again starts a new count
    ctx.set_profiling(True)
    ctx.forward(p, out=out, check=False)
    assert ctx.timings_sum()[0] == 1
    # profiled launches are not captured into graphs: they stay eager and count
    ctx.set_graphs(True)
    ctx.forward(p, out=out, check=False)
    ctx.forward(p, out=out, check=False)
    assert ctx.timings_sum()[0] == 3
    ctx.close()


@pytest.mark.parametrize("n", [1, 256, 257, 1025, 131_071, 262_145, (1 << 19) - 1])
def test_small_launch_deposit_items(qs, tmp_path, n):
    """Launches without a tuned choice take deposit items of 256, 512 or 1024
    samples by their size, and below 1024 write a row of moment sums per 256
    samples: the bits of items of 2048 samples (one row per 1024), and of the
    launch that allocates nothing."""
    p = _case(n_samples=n, n_steps=16)
    plain = qs.Context(0)
    ref = _np(plain.forward(p))
    _same(_np(plain.forward(p, noalloc=True)), ref, "noalloc")
    cache = tmp_path / "tune.txt"
    plain.tune(p, cache_path=str(cache))
    line = cache.read_text().split()
    line[10:13] = ["2048", "0", "0"]
    cache.write_text(" ".join(line) + "\n")
    forced = qs.Context(0)
    assert forced.tune(p, cache_path=str(cache))["dep_tile"] == 2048
    _same(_np(forced.forward(p)), ref, "items of 2048")
    assert ref["energy_hist"].sum() == n
    plain.close()
    forced.close()


@pytest.mark.parametrize("n_shots", [1, 2, 3, 4])
def test_shot_table_by_value_or_copied(qs, n_shots):
    """Small shot tables travel with the set-up kernel, larger ones are copied
    (the forward and the adjoint table pass 1 KB between two and four shots):
    the bits of one shot at a time either way."""
    import torch
    shots = [_case(n_samples=300 + 77 * k, n_steps=64, a0=10.0 + k) for k in range(n_shots)]
    ctx = qs.Context(0)
    ws = [torch.linspace(-1, 1, s["n_e"] + 2, dtype=torch.float64, device="cuda") for s in shots]
    outs, grads = ctx.forward_batched(shots), ctx.backward_batched(shots, ws)
    for k, s in enumerate(shots):
        one = dict(s, shot=shots[0]["shot"] + k)
        _same(_np(ctx.forward(one)), _np(outs[k]), k)
        assert torch.equal(ctx.backward(one, ws[k]), grads[k])
    ctx.close()


def test_status_words_of_many_threads(qs):
    """More threads than pinned status words read status words at once: each gets
    its own word's value (the rest by the blocking copy)."""
    import ctypes
    import torch
    from concurrent.futures import ThreadPoolExecutor
    from paper_2308_09348_amd import _lib
    ctx = qs.Context(0)
    words = torch.arange(40, dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)

    def read(k):
        return [_lib.lib().qs_sync_status(ctx._ptr, ctypes.c_void_p(words.data_ptr() + 4 * k),
                                          stream) for _ in range(20)]

    with ThreadPoolExecutor(40) as pool:
        got = list(pool.map(read, range(40)))
    assert got == [[k] * 20 for k in range(40)]
    ctx.close()


@pytest.mark.parametrize("n_samples,n_steps", [(1, 130), (64, 131), (65, 8), (300, 7), (1111, 9),
                                               (2500, 512), (513, 1), (700, 1023)])
@pytest.mark.parametrize("plane_wave", [False, True])
def test_small_launches_have_the_bits_of_large_ones(qs, n_samples, n_steps, plane_wave):
    """FP32 quantum passes of at most an item a CU give every wavefront of samples
    a helper for the amplitudes; beside a shot of 70,000 samples (274 items) the
    same shot goes through the general kernel.  Counts of steps at and between
    multiples of the helper's eight, odd and even; coarse and fine steps; samples
    at the edges of wavefronts and items."""
    shot = _case(n_samples=n_samples, n_steps=n_steps, a0=3.0 if n_steps < 100 else 30.0,
                 **({"w0_um": 0.0} if plane_wave else {}))
    ctx = qs.Context(0)
    big = dict(shot, n_samples=70_000)
    _same(_np(ctx.forward(shot)), _np(ctx.forward_batched([shot, big])[0]), "small")
    ctx.close()


@pytest.mark.parametrize("n", [5003, 50_001])
def test_tuned_small_launch_keeps_its_items(qs, tmp_path, n):
    """A small launch tuned to tiles of 1024 deposits as the untuned one does (in
    items of 256 samples here).  Items of 1024 themselves take 3.1 and 2.4 times as
    long, so that the fastest of 40 launches of either, in turn, tells them apart
    at 1.5."""
    p = _case(n_samples=n, n_steps=16)
    cache = tmp_path / "tune.txt"
    first, plain, tuned = qs.Context(0), qs.Context(0), qs.Context(0)
    first.tune(p, cache_path=str(cache))
    line = cache.read_text().split()
    line[10:13] = ["1024", "0", "0"]
    cache.write_text(" ".join(line) + "\n")
    assert tuned.tune(p, cache_path=str(cache))["dep_tile"] == 1024
    _same(_np(tuned.forward(p)), _np(plain.forward(p)), "tuned")
    both = (plain, tuned)
    out = []
    for ctx in both:
        ctx.set_profiling(True)
        out.append(ctx.forward(p))
    ms = [1e9, 1e9]
    for _ in range(40):
        for k, ctx in enumerate(both):
            ctx.forward(p, out=out[k], check=False)
            ms[k] = min(ms[k], ctx.last_timings()["deposit"])
    print(n, ms)
    assert ms[1] <= 1.5 * ms[0]
    for ctx in (first, plain, tuned):
        ctx.close()
