"""The split schedule's passes at the edges of their tiles: 64-sample flag
words, 512-sample tiles, groups of 32 tiles, segments of 1,152 tiles, and the
windows whose reach decides how neighbouring flags join (up to 64, beyond 64,
beyond a tile, beyond a group). Every entry form against the oracle, exactly:
the single-fill form (one kernel after the scan), a batch large enough for the
edge and copy passes, and the form without allocations."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover - CPU machines
    pytest.skip("no GPU", allow_module_level=True)

import paper_1611_04959_amd as daq  # noqa: E402
from gpu_util import assert_same, dev, log, make_fill, oracle_result, pad_stride, poison_out, run  # noqa: E402

WORD, TILE, GROUP, SEGMENT = 64, 512, 512 * 32, 512 * 1152
WINDOWS = [(0, 0), (8, 24), (31, 31), (31, 32), (40, 700), (6000, 300), (32768, 32768)]
LENGTHS = [1, WORD - 1, TILE - 1, TILE, TILE + 1, GROUP - 1, GROUP + 1, 3 * GROUP + 77, SEGMENT - 1, SEGMENT,
           SEGMENT + 1, 2 * SEGMENT + 12_345]


def _fill(rng, N, gap, kind):
    """Two channels of noise whose crossings sit at, before and after word, tile,
    group and segment edges, a whole window apart, and at the fill's ends."""
    x = rng.integers(995, 1006, size=(2, N)).astype(np.int16)
    if kind == "none":
        return pad_stride(x)
    if kind == "all":
        x[0, N // 3:] -= 500
        return pad_stride(x)
    at = {0, N - 1, N // 2}
    for edge in (WORD, TILE, GROUP, SEGMENT, 2 * SEGMENT):
        for d in (-1, 0, 1):
            at |= {edge + d, edge + d + gap, edge + d - gap, edge + d + gap + 1, edge + d - gap - 1}
    at |= set(rng.integers(0, N, max(1, N // 3000)).tolist())
    x[0, [t for t in at if 0 <= t < N]] -= 500
    return pad_stride(x)


def _params(pre, post, kind):
    return {"threshold": -200, "pre": pre, "post": post, "ped_samples": 1 if kind == "all" else 100}


@pytest.mark.parametrize("pre,post", WINDOWS)
@pytest.mark.parametrize("N", LENGTHS)
def test_edges_of_tiles_groups_and_segments(N, pre, post):
    rng = np.random.default_rng(N + 7 * pre + post)
    with daq.Context(0) as ctx:
        for kind in ("edges", "none", "all"):
            x = _fill(rng, N, pre + post + 1, kind)
            p = _params(pre, post, kind)
            ref = oracle_result(x, N, p)
            f = make_fill(dev(x), N, p)
            for mode in ("chop", "twopass", "batch"):
                log("N=%d pre=%d post=%d %s %s" % (N, pre, post, kind, mode))
                o = daq.alloc_out(f)
                run(ctx, mode, [f], [o])
                assert_same(o, ref, ctx="%s %s" % (kind, mode))
            log("N=%d pre=%d post=%d %s noalloc" % (N, pre, post, kind))
            o = daq.alloc_out(f)
            ctx.daq_process_batch_noalloc([f], [o])
            torch.cuda.synchronize()
            assert_same(o, ref, ctx="%s noalloc" % kind)


@pytest.mark.parametrize("n", [2, 4, 5, 8, 9, 16, 17, 70])
@pytest.mark.parametrize("threads", [256, 512])
def test_batches_around_the_emit_pass_limit(n, threads):
    """Mixed fills (empty ones, whole segments, capped outputs, find only) in
    batches that take the emit pass and batches that do not; twice in one
    context with other fills, so that nothing is left from the first."""
    rng = np.random.default_rng(n)
    with daq.Context(0) as ctx:
        ctx.set_schedule(threads, 8, 5, 0)
        for graphs in (True, False):
            ctx.set_graphs(graphs)
            fills, outs, refs = [], [], []
            for i in range(n):
                N = int(rng.choice([0, 1, 300, TILE, 5000, GROUP + 1, 40_000]))
                pre, post = WINDOWS[int(rng.integers(0, 5))]
                kind = ["edges", "none", "all"][int(rng.integers(0, 3))]
                x = _fill(rng, N, pre + post + 1, kind) if N else pad_stride(np.zeros((2, 8), np.int16))
                p = _params(pre, post, kind)
                f = make_fill(dev(x), N, p)
                fills.append(f)
                refs.append(oracle_result(x, N, p))
                o = daq.alloc_out(f, gather=i % 5 != 4)
                outs.append(poison_out(o))
            log("batch of %d graphs=%s threads=%d" % (n, graphs, threads))
            ctx.daq_process_batch(fills, outs)
            torch.cuda.synchronize()
            for i, (o, r) in enumerate(zip(outs, refs)):
                assert_same(o, r, ctx="fill %d graphs %s" % (i, graphs))


@pytest.mark.parametrize("tail", range(1, 10))
def test_last_words_of_one_two_and_many_runs(tail):
    """Packed rows that end 1 to 8 samples into a 16-byte word, that word made of
    one run, of two, and of runs of one and two samples."""
    rng = np.random.default_rng(tail)
    with daq.Context(0) as ctx:
        for C in (1, 4, 7, 54):
            for what in ("one", "two", "many"):
                x = rng.integers(995, 1006, size=(C, 3001)).astype(np.int16)
                at = list(range(100, 180)) if what == "many" else []
                step = {"one": [tail + 40], "two": [24 + tail // 2, 24 + (tail + 1) // 2], "many": [1] * tail}[what]
                t = 500
                for run_len in step:
                    at += range(t, t + run_len)
                    t += run_len + 3
                if what == "many":
                    at = at[:80:2] + at[80:]
                x[:, at] -= 500
                x = pad_stride(x)
                p = {"threshold": -200 * C, "pre": 0, "post": 0, "ped_samples": 50}
                ref = oracle_result(x, 3001, p)
                f = make_fill(dev(x), 3001, p)
                for mode in ("chop", "twopass"):
                    log("tail=%d C=%d %s %s" % (tail, C, what, mode))
                    o = daq.alloc_out(f)
                    run(ctx, mode, [f], [o])
                    assert_same(o, ref, ctx="%s %s" % (what, mode))
                outs = [daq.alloc_out(f) for _ in range(6)]
                ctx.daq_process_batch([f] * 6, outs)
                torch.cuda.synchronize()
                for o in outs:
                    assert_same(o, ref, ctx="%s batch" % what)


def test_many_batches_queued_behind_each_other():
    """Descriptor tables of 17 and more fills wait in a ring of 16 slots: 40
    different batches queued without a wait between them."""
    rng = np.random.default_rng(40)
    with daq.Context(0) as ctx:
        queued = []
        for k in range(40):
            fills, outs, refs = [], [], []
            for i in range(17 + k % 3):
                N = int(rng.integers(1, 2 * TILE))
                pre, post = WINDOWS[int(rng.integers(0, 3))]
                x = _fill(rng, N, pre + post + 1, "edges")
                p = _params(pre, post, "edges")
                f = make_fill(dev(x), N, p)
                fills.append(f)
                refs.append(oracle_result(x, N, p))
                outs.append(poison_out(daq.alloc_out(f)))
            queued.append((fills, outs, refs))
        torch.cuda.synchronize()
        log("40 batches")
        for fills, outs, _ in queued:
            ctx.daq_process_batch(fills, outs)
        torch.cuda.synchronize()
        for k, (_, outs, refs) in enumerate(queued):
            for i, (o, r) in enumerate(zip(outs, refs)):
                assert_same(o, r, ctx="batch %d fill %d" % (k, i))


@pytest.mark.parametrize("n", [3, 16, 20])
def test_a_captured_batch_keeps_its_descriptors(n):
    """A batch captured into a caller's graph, with other batches (and the same
    one) launched plainly between its replays."""
    rng = np.random.default_rng(n)

    def batch():
        fills, outs, refs = [], [], []
        for _ in range(n):
            N = int(rng.integers(1, 3 * TILE))
            x = _fill(rng, N, 33, "edges")
            p = _params(8, 24, "edges")
            f = make_fill(dev(x), N, p)
            fills.append(f)
            refs.append(oracle_result(x, N, p))
            outs.append(poison_out(daq.alloc_out(f)))
        return fills, outs, refs

    def check(b, what):
        torch.cuda.synchronize()
        for i, (o, r) in enumerate(zip(b[1], b[2])):
            assert_same(o, r, ctx="%s fill %d" % (what, i))
            poison_out(o)
        torch.cuda.synchronize()

    with daq.Context(0) as ctx:
        kept, other = batch(), batch()
        s = torch.cuda.Stream()
        with torch.cuda.stream(s):
            ctx.daq_process_batch(other[0], other[1])  # scratch grows here
        check(other, "warm-up")
        log("capture of %d" % n)
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            ctx.daq_process_batch(kept[0], kept[1])
        for k in range(3):
            with torch.cuda.stream(s):
                ctx.daq_process_batch(kept[0], kept[1])
            check(kept, "plain %d" % k)
            with torch.cuda.stream(s):
                ctx.daq_process_batch(other[0], other[1])
            check(other, "other %d" % k)
            with torch.cuda.stream(s):
                g.replay()
            check(kept, "replay %d" % k)
            with torch.cuda.stream(s):
                ctx.daq_process_batch(other[0], other[1])
            check(other, "other after replay %d" % k)


def test_pedestals_longer_than_the_scan_takes():
    """Pedestal sums up to 128 samples are the scan's; longer ones come from a
    kernel of their own, and change the threshold alike."""
    rng = np.random.default_rng(3)
    N = 20_011
    for C in (1, 5, 54, 70):
        for np_ in (1, 8, 127, 128, 129, 5000, 50_000):
            x = pad_stride(rng.integers(-32768, 32768, size=(C, N)).astype(np.int16))
            S = x[:, :N].astype(np.int64).sum(0)
            p = {"threshold": int(np.quantile(S, 0.03)), "pre": 3, "post": 9, "ped_samples": np_}
            ref = oracle_result(x, N, p)
            f = make_fill(dev(x), N, p)
            with daq.Context(0) as ctx:
                for mode in ("chop", "batch"):
                    log("pedestals C=%d np=%d %s" % (C, np_, mode))
                    o = daq.alloc_out(f)
                    run(ctx, mode, [f], [o])
                    assert_same(o, ref, ctx="C=%d np=%d %s" % (C, np_, mode))
