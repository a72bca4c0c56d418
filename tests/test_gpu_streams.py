"""Maps used on other streams than the one they were built on: what include/ts.h promises about that."""
import numpy as np
import pytest
import torch

from paper_2204_10319_amd import binding as ts
from workloads import features, conv_weights, shuffle_rows
from _util import np_dtype, to_dev, gpu_triples, oracle_map, oracle_conv, check_features

pytestmark = pytest.mark.gpu


def _coords(seed, n, side, batches=1):
    rng = np.random.Generator(np.random.PCG64(seed))
    flat = rng.choice(batches * side ** 3, size=n, replace=False)
    b, x, y, z = np.unravel_index(flat, (batches, side, side, side))
    return np.stack([b, x - side // 2, y, z], axis=1).astype(np.int32)


@pytest.mark.parametrize("dtype", [torch.float16, torch.float32])
@pytest.mark.parametrize("K,s,transposed", [(3, 1, False), (2, 2, False), (2, 2, True), (3, 2, False)])
def test_map_of_a_waiting_build_on_another_stream(K, s, transposed, dtype):
    """ts_build_kmap returns when its map is complete: another stream's layers (which read the tile order and the
    ranks the build's last kernel leaves) and pair lists come right after it, with nothing in between."""
    a, b = torch.cuda.Stream(), torch.cuda.Stream()
    nd = np_dtype(dtype)
    w = ts.ts_weights_prepare(to_dev(conv_weights(3, K ** 3, 64, 64, nd)))
    for i, n in enumerate((700, 9000, 60000, 3001)):
        coords = _coords(900 + i, n, 64, batches=2)
        dev = to_dev(coords)
        ref = ts.ts_build_kmap(dev, K, s, transposed)
        x = to_dev(features(i, ref.num_in, 64, nd))
        want = ts.ts_sparse_conv_prepared(x, w, ref)
        want_pairs = [p.clone() for p in ref.pairs()]
        torch.cuda.synchronize()
        for _ in range(3):
            with torch.cuda.stream(a):
                kmap = ts.ts_build_kmap(dev, K, s, transposed)
            with torch.cuda.stream(b):
                got = ts.ts_sparse_conv_prepared(x, w, kmap)
                pairs = kmap.pairs()
            b.synchronize()
            assert torch.equal(got, want)
            assert all(torch.equal(p, q) for p, q in zip(pairs, want_pairs))
        assert np.array_equal(gpu_triples(kmap), oracle_map(coords, K, s, transposed)[2])


@pytest.mark.parametrize("dtype", [torch.float16, torch.float32])
def test_map_whose_verdict_is_known_on_another_stream(dtype):
    """An asynchronous 3x3x3 build reports its verdict before its search has ended: after ts_kmap_status, layers,
    what the build put off, and sizes come on other streams; and sizes without a verdict before them."""
    a, b, c = (torch.cuda.Stream() for _ in range(3))
    nd = np_dtype(dtype)
    w = ts.ts_weights_prepare(to_dev(conv_weights(4, 27, 64, 64, nd)))
    for i, n in enumerate((500, 80000, 250000)):
        coords = _coords(950 + i, n, 90)
        dev = to_dev(coords)
        x = to_dev(features(i, n, 64, nd))
        ref = ts.ts_build_kmap(dev, 3, 1)
        want, sizes = ts.ts_sparse_conv_prepared(x, w, ref), ref.sizes()
        torch.cuda.synchronize()

        def build():
            with torch.cuda.stream(a):
                return ts.ts_build_kmap(dev, 3, 1, wait=False)

        def layer(kmap, stream):
            with torch.cuda.stream(stream):
                got = ts.ts_sparse_conv_prepared(x, w, kmap)
            stream.synchronize()
            return got

        assert torch.equal(layer(build().status(), b), want)
        kmap = build().status()
        with torch.cuda.stream(b):
            kmap.prepare()
        assert torch.equal(layer(kmap, c), want) and np.array_equal(kmap.sizes(), sizes)
        kmap = build()
        with torch.cuda.stream(b):
            pairs = kmap.pairs()
        b.synchronize()
        assert all(torch.equal(p, q) for p, q in zip(pairs, ref.pairs())) and np.array_equal(kmap.sizes(), sizes)
        assert torch.equal(layer(kmap, c), want)


@pytest.mark.parametrize("dtype", [torch.float16, torch.float32])
def test_row_order_of_a_map_in_use_on_other_streams(dtype):
    """The second layer on a large map enqueues the ordering of its rows: layers that follow at once on other streams,
    eager or recorded into a graph, give the bits of the natural order, as does the one that enqueued it."""
    a, b, c = (torch.cuda.Stream() for _ in range(3))
    nd = np_dtype(dtype)
    w = ts.ts_weights_prepare(to_dev(conv_weights(5, 27, 64, 64, nd)))
    for i, n in enumerate((40000, 200000)):
        dev, x = to_dev(_coords(970 + i, n, 80)), to_dev(features(i, n, 64, nd))
        want = ts.ts_sparse_conv_prepared(x, w, ts.ts_build_kmap(dev, 3, 1))
        outs = [torch.zeros_like(want) for _ in range(4)]
        graph = torch.cuda.CUDAGraph()
        for rep in range(3):
            kmap = ts.ts_build_kmap(dev, 3, 1)
            torch.cuda.synchronize()
            for out, stream in zip(outs, (a, b, c, a)):
                if dtype == torch.float16:
                    stream.wait_stream(a)      # fp16 layers on one map share its tile counters: one after the other
                    stream.wait_stream(b)
                    stream.wait_stream(c)
                with torch.cuda.stream(stream):
                    ts.ts_sparse_conv_prepared(x, w, kmap, out=out.zero_())
            torch.cuda.synchronize()
            assert all(torch.equal(out, want) for out in outs)
        with torch.cuda.graph(graph, stream=c):
            ts.ts_sparse_conv_prepared(x, w, kmap, out=outs[0])
        for _ in range(3):
            outs[0].zero_()
            graph.replay()
            assert torch.equal(ts.ts_sparse_conv_prepared(x, w, kmap), want)   # eager work between the replays
            torch.cuda.synchronize()
            assert torch.equal(outs[0], want)
        del graph


@pytest.mark.parametrize("dtype", [torch.float16, torch.float32])
@pytest.mark.parametrize("n,c", [(9000, 64), (9000, 128), (60000, 128)])
def test_row_order_of_a_map_that_goes_up_on_other_streams(n, c, dtype):
    """A 2x2x2 map that goes up is ordered by its second layer, or a wide first one: layers that follow at once on other streams,
    eager or recorded, give the bits of the natural order; a layer recorded first leaves the ordering to others."""
    streams = [torch.cuda.Stream() for _ in range(3)]
    nd = np_dtype(dtype)
    dev, w = to_dev(_coords(980, n, 40)), ts.ts_weights_prepare(to_dev(conv_weights(6, 8, c, 64, nd)))
    derived = ts.ts_build_kmap(dev, 2, 2).transpose()
    x = to_dev(features(7, derived.num_in, c, nd))
    want = ts.ts_sparse_conv_prepared(x, w, derived)
    outs = [torch.zeros_like(want) for _ in range(4)]
    for recorded_first in (False, True) if dtype == torch.float16 else (False,):   # (fetched fp32 layers make pair lists first)
        kmap = ts.ts_build_kmap(dev, 2, 2, True)
        graph = torch.cuda.CUDAGraph()
        torch.cuda.synchronize()
        if recorded_first:
            with torch.cuda.graph(graph, stream=streams[2]):
                ts.ts_sparse_conv_prepared(x, w, kmap, out=outs[0])
        for out, stream in zip(outs[1:], streams):
            for other in streams:
                stream.wait_stream(other)          # fp16 layers on one map share its tile counters
            with torch.cuda.stream(stream):
                ts.ts_sparse_conv_prepared(x, w, kmap, out=out.zero_())
        torch.cuda.synchronize()
        assert all(torch.equal(out, want) for out in outs[1:])
        if not recorded_first:
            with torch.cuda.graph(graph, stream=streams[2]):
                ts.ts_sparse_conv_prepared(x, w, kmap, out=outs[0])
        for _ in range(3):
            outs[0].zero_()
            graph.replay()
            assert torch.equal(ts.ts_sparse_conv_prepared(x, w, kmap), want)   # eager work between the replays
            torch.cuda.synchronize()
            assert torch.equal(outs[0], want)
        del graph


def _far_spread(seed, n):
    """Points whose box is too large for the bitmap of a 2x2x2 stride-2 build: it is built by sorting once its number of
    outputs is asked for."""
    rng = np.random.Generator(np.random.PCG64(seed))
    xyz = np.unique(rng.integers(-40000, 40000, (n, 3)) // 8, axis=0)
    xyz = np.concatenate([xyz, xyz + [[0, 0, 1]], [[60000, 60000, 60000], [-60000, -60000, -60000]]])
    xyz = np.unique(xyz, axis=0)
    return np.concatenate([np.zeros((len(xyz), 1)), xyz[rng.permutation(len(xyz))]], 1).astype(np.int32)


@pytest.mark.parametrize("dtype", [torch.float16, torch.float32])
@pytest.mark.parametrize("n", [300, 60000])
def test_map_rebuilt_when_its_outputs_are_asked_for_elsewhere(n, dtype):
    """The number of outputs of such a map is asked for on another stream, which rebuilds the map there; the stream it was
    built on uses it at once, as include/ts.h allows.  The same with a layer, first thing on the other stream."""
    a, b = torch.cuda.Stream(), torch.cuda.Stream()
    coords, nd, lib = _far_spread(n, n), np_dtype(dtype), ts.load_library()
    dev = to_dev(coords)
    x, w = features(1, len(coords), 32, nd), conv_weights(2, 8, 32, 64, nd)
    xd, wd = to_dev(x), ts.ts_weights_prepare(to_dev(w))
    want = oracle_conv(coords, x, w, 2, 2)
    for _ in range(3):
        with torch.cuda.stream(a):
            kmap = ts.ts_build_kmap(dev, 2, 2, wait=False)
        a.synchronize()
        ts.ts_set_stream(b)
        assert lib.ts_kmap_num_out(kmap.handle) == want.shape[0]
        with torch.cuda.stream(a):
            got = ts.ts_sparse_conv_prepared(xd, wd, kmap)
        a.synchronize()
        check_features(got, want, dtype)
        with torch.cuda.stream(a):
            kmap = ts.ts_build_kmap(dev, 2, 2, wait=False)
        a.synchronize()
        with torch.cuda.stream(b):      # a layer asks for itself
            got = ts.ts_sparse_conv_prepared(xd, wd, kmap)
        b.synchronize()
        check_features(got, want, dtype)
    assert np.array_equal(gpu_triples(kmap), oracle_map(coords, 2, 2)[2])


def test_a_count_that_fails_says_why():
    """No memory for the rebuild of such a map: that is the error of whatever asked for its outputs, then and later."""
    coords = to_dev(_far_spread(7, 5000))
    x, w = torch.zeros((coords.shape[0], 32), dtype=torch.float16, device="cuda"), torch.zeros((8, 32, 32), dtype=torch.float16, device="cuda")
    asks = [lambda m: m.num_out, lambda m: m.out_coords(), lambda m: ts.ts_sparse_conv(x, w, m), lambda m: m.out_box()]
    for first in asks:
        kmap = ts.ts_build_kmap(coords, 2, 2, wait=False)
        ts.ts_set_allocator(lambda size: 0, lambda ptr: None)
        try:
            for ask in [first] + asks:
                with pytest.raises(ts.TsError) as e:
                    ask(kmap)
                assert e.value.code == ts.TS_ERR_OOM
        finally:
            ts.ts_set_allocator(None, None)
        kmap.free()


@pytest.mark.parametrize("layer", [ts.ts_sparse_conv, ts.ts_sparse_conv_static])
def test_layer_recorded_on_a_map_still_being_built(layer):
    """A layer is recorded while the build of its 2x2x2 map, whose number of outputs nobody has asked for, waits on the
    device behind other work: it waits for the count without touching the capture.  Where that map has to be built by
    sorting, the layer is refused and the capture, the map and a later layer are none the worse."""
    side = torch.cuda.Stream()
    w = to_dev(conv_weights(8, 8, 32, 64, np.float16))
    heavy = torch.randn(4096, 4096, device="cuda")
    for coords, refused in ((_coords(990, 120000, 70), False), (_far_spread(991, 60000), True)):
        dev, x = to_dev(coords), to_dev(features(9, len(coords), 32, np.float16))
        with torch.cuda.stream(side):
            want = ts.ts_sparse_conv(x, w, ts.ts_build_kmap(dev, 2, 2), dataflow=ts.TS_DATAFLOW_FUSED)
            out = torch.zeros_like(want)
            layer(x, w, ts.ts_build_kmap(dev, 2, 2), out)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.stream(side):
            for _ in range(8):
                heavy @ heavy
            kmap = ts.ts_build_kmap(dev, 2, 2, wait=False)
            graph.capture_begin(capture_error_mode="thread_local")
            try:
                out.zero_()
                if refused:
                    with pytest.raises(ts.TsError) as e:
                        layer(x, w, kmap, out)
                    assert e.value.code == ts.TS_ERR_UNSUPPORTED
                else:
                    layer(x, w, kmap, out)
            finally:
                graph.capture_end()
        torch.cuda.synchronize()
        for _ in range(3):
            out.fill_(1)
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(out, torch.zeros_like(out) if refused else want)
            with torch.cuda.stream(side):
                assert torch.equal(ts.ts_sparse_conv(x, w, kmap, dataflow=ts.TS_DATAFLOW_FUSED), want)
            side.synchronize()
        del graph


def test_layer_without_allocations_does_not_build_the_map():
    """A 2x2x2 map over a box too large for the bitmap, whose number of outputs nobody has asked for, has yet to be built:
    ts_sparse_conv_static refuses it, asks for no memory, and leaves the map to whoever asks for the number."""
    coords = _far_spread(992, 3000)
    dev, x, w = to_dev(coords), to_dev(features(9, len(coords), 32, np.float16)), to_dev(conv_weights(8, 8, 32, 64, np.float16))
    want = ts.ts_sparse_conv(x, w, ts.ts_build_kmap(dev, 2, 2), dataflow=ts.TS_DATAFLOW_FUSED)
    kmap, out, asked = ts.ts_build_kmap(dev, 2, 2, wait=False), torch.zeros_like(want), []
    ts.ts_set_allocator(lambda size: asked.append(size) or 0, lambda ptr: None)
    try:
        for _ in range(2):
            with pytest.raises(ts.TsError) as e:
                ts.ts_sparse_conv_static(x, w, kmap, out)
            assert e.value.code == ts.TS_ERR_UNSUPPORTED and not asked
    finally:
        ts.ts_set_allocator(None, None)
    assert kmap.num_out == len(want)
    assert torch.equal(ts.ts_sparse_conv_static(x, w, kmap, out), want)


def test_sizes_asked_for_while_recording():
    """What a 3x3x3 build put off is not run inside a capture: the request is refused, and served after it."""
    side = torch.cuda.Stream()
    dev = to_dev(_coords(995, 5000, 30))
    sizes = ts.ts_build_kmap(dev, 3, 1).sizes()
    out = torch.zeros(64, device="cuda")
    with torch.cuda.stream(side):
        kmap = ts.ts_build_kmap(dev, 3, 1, wait=False)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        out.fill_(3)
        with pytest.raises(ts.TsError) as e:
            kmap.sizes()
        assert e.value.code == ts.TS_ERR_UNSUPPORTED
        kmap.status()
    graph.replay()
    torch.cuda.synchronize()
    assert out.eq(3).all() and np.array_equal(kmap.sizes(), sizes)
    del graph


def test_single_precision_layer_recorded_with_and_without_pair_lists():
    """A 64 -> 64 layer on few points is fetched, which takes the map's pair lists.  Recorded on a map that has none yet it
    takes no memory and is fused; once the layer has run eagerly the recording is what the eager layer is."""
    dev, x = to_dev(_coords(996, 3000, 30)), to_dev(features(9, 3000, 64, np.float32))
    plain = to_dev(conv_weights(8, 27, 64, 64, np.float32))
    w = ts.ts_weights_prepare(plain)
    ref = ts.ts_build_kmap(dev, 3, 1)
    fused, fetched = (ts.ts_sparse_conv(x, plain, ref, dataflow=d) for d in (ts.TS_DATAFLOW_FUSED, ts.TS_DATAFLOW_FETCH))
    assert not torch.equal(fused, fetched)
    out, side = torch.zeros_like(fused), torch.cuda.Stream()
    for wait in (True, False):
        kmap = ts.ts_build_kmap(dev, 3, 1, wait=wait)
        torch.cuda.synchronize()
        for want in (fused, fetched):
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph, stream=side):
                ts.ts_sparse_conv_prepared(x, w, kmap, out=out)
            for _ in range(3):
                out.zero_()
                graph.replay()
                torch.cuda.synchronize()
                assert torch.equal(out, want)
                assert torch.equal(ts.ts_sparse_conv_prepared(x, w, kmap), fetched)
                torch.cuda.synchronize()
            del graph


@pytest.mark.parametrize("n,side", [(3000, 30), (120000, 64)])
def test_sorted_rows_on_another_stream(n, side):
    """ts_kmap_sort_rows returns when the order is complete: a layer on another stream comes right after it.  The second map
    has more distinct bitmasks than the table ranks, so that its rows are sorted."""
    a, b = torch.cuda.Stream(), torch.cuda.Stream()
    dev, x = to_dev(_coords(980, n, side)), to_dev(features(6, n, 64, np.float16))
    w = ts.ts_weights_prepare(to_dev(conv_weights(7, 27, 64, 64, np.float16)))
    want = ts.ts_sparse_conv_prepared(x, w, ts.ts_build_kmap(dev, 3, 1).sort_rows())
    torch.cuda.synchronize()
    for _ in range(3):
        with torch.cuda.stream(a):
            kmap = ts.ts_build_kmap(dev, 3, 1).sort_rows()
        with torch.cuda.stream(b):
            got = ts.ts_sparse_conv_prepared(x, w, kmap)
        b.synchronize()
        assert torch.equal(got, want)
