"""GPU parity at the sizes where a launch rule or a kernel variant changes: edges of units, workgroups and grids,
remainders, and the smallest and largest array of each variant.  Oracle and tolerances as in test_gpu_parity.py."""
import numpy as np
import pytest

import oracle
from paper_1511_04561_amd import workloads
from tests.test_gpu_parity import Guarded, bounds_dev, check_encode_decode, check_error_stats, check_segments, dev, same_bits  # noqa: F401

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dq8():
    if not torch.cuda.is_available():
        pytest.fail("these tests need a GPU (select them with -m gpu on a GPU box)")
    from paper_1511_04561_amd import dq8 as mod
    mod.lib()  # a missing library is an error, not a skip
    mod.init()
    oracle.set_threads(16)
    return mod


@pytest.mark.parametrize("n,block", [
    (1, 0), (11 * 1024 + 5, 0),         # one workgroup of twelve wavefronts, some of them without work
    (12 * 1024, 0), (13 * 1024 + 1, 0),  # exactly one workgroup, and one wavefront more
    (40 * 5120 + 3, 5120),              # blocks that end inside a workgroup's runs: it holds several at the end
    (256 * 700, 700), (256 * 700 + 1, 700),  # the last workgroup forms the means, and one block too many for that
    (800 * 100, 100), (2500 * 1100 + 7, 1100),  # a block or two per wavefront; more blocks than the last workgroup has threads
    (12 * 1024 * 512 + 4099, 0),        # two units per wavefront, the grid full
    (12 * 1024 * 512 * 2 + 1, 6144 * 1024)])
def test_error_stats_shared_blocks(dq8, n, block):
    """Wavefronts that share blocks: combined in the workgroup, merged by atomics, means by the workgroup that ends last."""
    rng = np.random.Generator(np.random.PCG64(6100 + n % 97))
    x = (rng.standard_normal(n) * np.exp(rng.uniform(-6, 0, n))).astype(np.float32)
    x[::17] = 0.0
    check_error_stats(dq8, 0, x, block, tag="shared")
    nb = oracle.dq8_oracle.n_blocks(n, block)
    check_error_stats(dq8, 3, x, block, given=np.full(nb, 4.0, np.float32), tag="shared, given")


@pytest.mark.parametrize("n,block", [
    (2048 * 3 + 1001, 1001), (1001 * 40, 1001), (9 * 700 + 3, 9), (257 * 300 + 1, 257), (1023 * 33 + 2, 1023),  # a wavefront per block; last block of 1, 2, 3
    (1500 * 9 + 1, 1500), (2047 * 20 + 5, 2047), (3071 * 13 + 3, 3071), (1300 * 30 + 7, 1300), (3500 * 9 + 2, 3500),  # teams, and the general kernel
    (4096 * 7 + 1, 4096), (4096 * 7 + 4095, 4096), (4097 * 11, 4097), (6143 * 5 + 3, 6143), (12289 * 3 + 1, 12289), (16383 * 3 + 2, 16383),
    (4096 * 9 + 3, 0), (16385, 0), (100003, 0), (70000 * 3 + 1, 70000), (5, 0), (3, 0), (1003 * 4 + 3, 20000)])
@pytest.mark.parametrize("offset", [0, 1, 2, 3])
def test_blocks_that_start_at_any_element(dq8, n, block, offset):
    """Blocks, last blocks and arrays that are no whole number of quads or start at an address that is aligned for an element only."""
    rng = np.random.Generator(np.random.PCG64(7300 + n % 89))
    x = (rng.standard_normal(n) * np.exp(rng.uniform(-9, 0, n))).astype(np.float32)
    check_encode_decode(dq8, (n + offset) % 4, x, block, x_off=offset, c_off=offset, tag="offset %d" % offset)
    check_encode_decode(dq8, (n + offset + 1) % 4, x, block, x_off=offset, c_off=(offset + 1) % 4, tag="offsets %d" % offset)


@pytest.mark.parametrize("block,blocks", [(256, 40), (512, 3100), (1024, 1), (1024, 3073), (2048, 7), (4096, 1), (4096, 769), (8192, 5), (12288, 300)])
@pytest.mark.parametrize("rest,offset", [(0, 3), (1, 0), (3, 3), (4, 0), (255, 3)])
def test_maxima_of_blocks_of_whole_units(dq8, block, blocks, rest, offset):
    """One unit and several per wavefront and per block, a wavefront more than the grid, a shorter last block."""
    n = block * blocks + rest
    rng = np.random.Generator(np.random.PCG64(6900 + n % 91))
    x = (rng.standard_normal(n) * np.exp(rng.uniform(-9, 0, n))).astype(np.float32)
    x[rng.integers(0, n, 1 + n // 997)] *= -50.0  # the maxima of few elements, anywhere in their units
    want = np.maximum.reduceat(np.abs(x), np.arange(0, n, block))
    same_bits(dq8.absmax(dev(x, offset), block), want, "maxima")


@pytest.mark.parametrize("block,blocks", [(1, 3000), (3, 3000), (5, 9000), (9, 8193), (100, 700), (255, 9), (257, 8200), (500, 3), (1000, 30), (1025, 4100), (1500, 40),
                                          (1536, 9), (2048, 2100), (4000, 12)])
@pytest.mark.parametrize("rest,offset", [(0, 0), (1, 1), (3, 0), (4, 1)])
def test_given_scales_and_general_blocks(dq8, block, blocks, rest, offset):
    """Blocks whose scales are handed in or computed in the general kernel; a last block of fewer than four elements."""
    n = block * blocks + min(rest, block - 1)
    rng = np.random.Generator(np.random.PCG64(7700 + n % 93))
    x = (rng.standard_normal(n) * np.exp(rng.uniform(-9, 0, n))).astype(np.float32)
    kind = (block + rest) % 4
    check_encode_decode(dq8, kind, x, block, x_off=offset, c_off=3 * offset, tag="general")
    given = np.exp(rng.uniform(2, 4, oracle.dq8_oracle.n_blocks(n, block))).astype(np.float32)
    given[::7] = 0.0
    x[np.repeat(given, block)[:n] == 0.0] *= np.float32(0.1)
    want, _ = oracle.encode(kind, x, block, scales=given)
    gc = Guarded(n, np.uint8, offset)
    dq8.encode(kind, dev(x, offset), block, scales=dev(given), codes=gc.t, scales_given=True)
    same_bits(gc.t, want, "given scales")
    gc.check("given scales")


# units of 1024 and 4096 elements and a last one of four or more; 1 to 3 elements that are in none; a wavefront, a workgroup, more
# than the grid; the array from which maxima take 16 quads per lane (16 Mi elements), and a little less
@pytest.mark.parametrize("n", [3, 4, 5, 1027, 1028, 8 * 1024 + 1, 4096 * 1024 + 2, (1 << 24) - 1, (1 << 24) + 4099])
@pytest.mark.parametrize("offset", [0, 1, 3])
def test_segments_and_whole_arrays_at_any_element(dq8, n, offset):
    """Tensors back to back, and arrays with one scale, whose ends and starts are aligned for an element only."""
    rng = np.random.Generator(np.random.PCG64(8200 + n % 83 + offset))
    x = (rng.standard_normal(n) * np.exp(rng.uniform(-9, 0, n))).astype(np.float32)
    kind = (n + offset) % 4
    if n > 4096:
        check_encode_decode(dq8, kind, x, 0, x_off=offset, c_off=offset, tag="one block, offset %d" % offset)
    inner = np.concatenate([rng.integers(0, n + 1, 5), n - np.minimum(n, [1, 2, 5, 7]), np.minimum(n, [1, 2, 6])])
    bounds = np.concatenate([[0], np.sort(inner), [n]])
    check_segments(dq8, kind, x, bounds, x_off=offset, c_off=(offset + n) % 4, tag="any element")
    K, n_seg = (9 if n % 2 else 3), len(bounds) - 1
    cl = [rng.integers(0, 256, n).astype(np.uint8) for _ in range(K)]
    sl = [np.exp(rng.uniform(-8, 8, n_seg)).astype(np.float32) for _ in range(K)]
    want = oracle.decode_accumulate_avg_segments(kind, cl, sl, bounds, local=x)
    go = Guarded(n, np.float32, offset)
    dq8.decode_accumulate_avg_segments(kind, [dev(c, (offset + k) % 4) for k, c in enumerate(cl)], [dev(s) for s in sl], bounds_dev(bounds),
                                       out=go.t, local=dev(x, offset))
    same_bits(go.t, want, "segment average")
    go.check("segment average")


@pytest.mark.parametrize("n_seg", [2047, 2048, 4095])
@pytest.mark.parametrize("n", [(1 << 21) - 5, (1 << 21) + 1027, 5 * (1 << 20) + 3])
def test_many_segments(dq8, n_seg, n):
    """Up to and beyond the number of segments whose bounds fit twice beside the value tables; one workgroup per compute unit and more."""
    rng = np.random.Generator(np.random.PCG64(8600 + n % 83 + n_seg))
    x = (rng.standard_normal(n) * np.exp(rng.uniform(-9, 0, n))).astype(np.float32)
    bounds = np.concatenate([[0], np.sort(rng.integers(0, n + 1, n_seg - 1)), [n]])
    check_segments(dq8, n % 4, x, bounds, tag="many")
    K = 2 + n_seg % 2
    cl = [rng.integers(0, 256, n).astype(np.uint8) for _ in range(K)]
    sl = [np.exp(rng.uniform(-8, 8, n_seg)).astype(np.float32) for _ in range(K)]
    want = oracle.decode_accumulate_avg_segments(0, cl, sl, bounds)
    go = Guarded(n, np.float32)
    dq8.decode_accumulate_avg_segments(0, [dev(c) for c in cl], [dev(s) for s in sl], bounds_dev(bounds), out=go.t)
    same_bits(go.t, want, "segment average")
    go.check("segment average")


@pytest.mark.parametrize("K,local", [(0, True), (1, False), (1, True), (2, False), (3, True), (4, True), (9, False), (32, False), (32, True)])
def test_segment_average_of_any_number_of_workers(dq8, K, local):
    """Whole pairs of workers and a last one by itself, over several units per wavefront."""
    n, n_seg = 5 * (1 << 20) + 7, 40
    rng = np.random.Generator(np.random.PCG64(8800 + K))
    bounds = np.concatenate([[0], np.sort(rng.integers(0, n + 1, n_seg - 1)), [n]])
    x = rng.standard_normal(n).astype(np.float32) if local else None
    cl = [rng.integers(0, 256, n).astype(np.uint8) for _ in range(K)]
    sl = [np.exp(rng.uniform(-8, 8, n_seg)).astype(np.float32) for _ in range(K)]
    want = oracle.decode_accumulate_avg_segments(2, cl, sl, bounds, local=x)
    go = Guarded(n, np.float32)
    dq8.decode_accumulate_avg_segments(2, [dev(c, k % 4) for k, c in enumerate(cl)], [dev(s) for s in sl], bounds_dev(bounds), out=go.t,
                                       local=dev(x) if local else None)
    same_bits(go.t, want, "segment average")
    go.check("segment average")


@pytest.mark.parametrize("rest,offset", [(1025, 0), (2050, 1), (3075, 3), (1027, 0), (4095, 1)])
def test_segment_maxima_of_a_last_part_under_a_quad(dq8, rest, offset):
    """16 quads per lane, and a last unit with several segments whose last 1024 elements are 1, 2 or 3: every largest value stands
    where only that part, or only the one before it, sees it."""
    n = (1 << 24) + rest
    rng = np.random.Generator(np.random.PCG64(8700 + rest))
    x = rng.uniform(-1, 1, n).astype(np.float32)
    bounds = np.array([0, 5, n - 1030, n - 5, n - 2, n - 1, n])
    for i in (1, 2, 4, 7):
        x[n - i] = np.float32(-8 - i)
    want = np.maximum.reduceat(np.abs(x), bounds[:-1])
    gx, gs = Guarded(n, np.float32, offset, data=x), Guarded(len(bounds) - 1, np.float32)
    dq8.absmax_segments(gx.t, bounds_dev(bounds), scales=gs.t)
    same_bits(gs.t, want, "segment maxima")
    gs.check("segment maxima")


@pytest.mark.parametrize("block", [0, 4096])
@pytest.mark.parametrize("more", [-4097, -1, 0, 1, 5, 4096])
def test_expansion_at_the_longest_short_array(dq8, block, more):
    """Arrays with about as many units of 4096 elements as the chip has compute units: units of 1024 up to there."""
    n = 4096 * torch.cuda.get_device_properties(0).multi_processor_count + more
    rng = np.random.Generator(np.random.PCG64(8900 + more % 89))
    codes = rng.integers(0, 256, n).astype(np.uint8)
    scales = np.exp(rng.uniform(-8, 8, oracle.dq8_oracle.n_blocks(n, block))).astype(np.float32)
    go = Guarded(n, np.float32, more % 4)
    dq8.decode(more % 4, dev(codes, 1), dev(scales), block, out=go.t)
    same_bits(go.t, oracle.decode(more % 4, codes, scales, block), "expansion")
    go.check("expansion")


# slices of 4096 elements and a last one of 1, 2, 3 and more; the kernels that take 1, 2, 4, 8, 16 and 24 slices; the longest array and one more
@pytest.mark.parametrize("n", [4, 7, 4095, 4096, 4097, 8194, 16387, 16388, 32769, 65536, 65537, 98301, 98304, 98305])
@pytest.mark.parametrize("offset", [0, 3])
def test_short_arrays_in_one_launch(dq8, n, offset):
    """Arrays with one scale, and tensors back to back, whose maxima every workgroup forms by itself: segments shorter than a quad,
    empty ones at the start, inside and at the end, one that spans all slices, more segments than threads."""
    rng = np.random.Generator(np.random.PCG64(9100 + n % 97 + offset))
    x = (rng.standard_normal(n) * np.exp(rng.uniform(-9, 0, n))).astype(np.float32)
    kind = (n + offset) % 4
    for at in {0, n // 2, n - 1}:  # the maximum at either end and inside
        y = x.copy()
        y[at] = -3.0
        check_encode_decode(dq8, kind, y, 0, x_off=offset, c_off=offset, tag="one scale")
    check_encode_decode(dq8, (kind + 1) % 4, np.zeros(n, np.float32), 0, x_off=offset, c_off=offset, tag="zeros")
    inner = rng.integers(0, n + 1, 6)
    near = np.minimum(n, [1, 3, 4, 4095, 4096, 4096, 4099, 8191, 12288])
    for cuts in ([], [n // 3], inner, near, n - near, np.concatenate([[0, 0], inner, [n, n]]), rng.integers(0, n + 1, 2000)):
        bounds = np.concatenate([[0], np.sort(np.asarray(cuts, np.int64)), [n]])
        check_segments(dq8, (kind + len(bounds)) % 4, x, bounds, x_off=offset, c_off=(offset + n) % 4, tag="%d segments" % (len(bounds) - 1))


# bounds in registers up to 63 segments; scales of all workers in LDS up to 1024; at most 12 bounds inside a unit are counted one by
# one (the test after this one); all workers' codes requested at once (up to 4, up to 8) where no wavefront has a second unit
@pytest.mark.parametrize("n,n_seg,K", [(5003, 1, 3), (5003, 2, 8), (5003, 16, 4), (5003, 17, 5), (5003, 18, 9), (5003, 63, 2), (5003, 64, 3), (5003, 65, 4), (5003, 128, 8),
                                       (5003, 129, 8), (5003, 341, 3), (5003, 342, 3), (5003, 1024, 1), (5003, 1025, 1), (256 * 8 * 1024 - 3, 18, 8),
                                       (256 * 8 * 1024 + 1, 17, 5), (256 * 16 * 1024 + 5000, 65, 3)])
def test_segments_at_the_edges_of_their_tables(dq8, n_seg, K, n):
    """All bounds inside one unit, and spread over the array; workers averaged with and without a local term."""
    rng = np.random.Generator(np.random.PCG64(9500 + n % 97 + n_seg))
    x = (rng.standard_normal(n) * np.exp(rng.uniform(-9, 0, n))).astype(np.float32)
    kind = (n + n_seg) % 4
    cl = [rng.integers(0, 256, n).astype(np.uint8) for _ in range(K)]
    for low, high in ((1025, 2047), (0, n + 1)):
        bounds = np.concatenate([[0], np.sort(rng.integers(low, high, n_seg - 1)), [n]])
        check_segments(dq8, kind, x, bounds, tag="%d segments" % n_seg)
        sl = [np.exp(rng.uniform(-8, 8, n_seg)).astype(np.float32) for _ in range(K)]
        local = x if low else None
        want = oracle.decode_accumulate_avg_segments(kind, cl, sl, bounds, local=local)
        go = Guarded(n, np.float32)
        dq8.decode_accumulate_avg_segments(kind, [dev(c) for c in cl], [dev(s) for s in sl], bounds_dev(bounds), out=go.t,
                                           local=None if local is None else dev(local))
        same_bits(go.t, want, "segment average")
        go.check("segment average")


# 11 to 13 bounds inside a unit; four workers at a time from nine on
@pytest.mark.parametrize("n,n_seg,K", [(5003, 12, 3), (5003, 13, 4), (5003, 14, 6), (5003, 3, 16), (60000, 1, 32)])
def test_segments_at_the_limits_of_counting_and_of_workers_ahead(dq8, n_seg, K, n):
    test_segments_at_the_edges_of_their_tables(dq8, n_seg, K, n)


# more than 2047 segments in more than a unit for eight wavefronts of every compute unit: workgroups of sixteen, with and without workers
@pytest.mark.parametrize("n_seg,K", [(2047, 0), (2048, 0), (4095, 0), (2048, 1), (4095, 3)])
@pytest.mark.parametrize("more", [0, 1, 5000])
def test_averages_of_many_segments(dq8, n_seg, K, more):
    """The local term alone and with workers: every element is written, whichever workgroups the launch takes."""
    n = 256 * 8 * 1024 + more
    rng = np.random.Generator(np.random.PCG64(9600 + n_seg + K + more))
    bounds = np.concatenate([[0], np.sort(rng.integers(0, n + 1, n_seg - 1)), [n]])
    cl = [rng.integers(0, 256, n).astype(np.uint8) for _ in range(K)]
    sl = [np.exp(rng.uniform(-8, 8, n_seg)).astype(np.float32) for _ in range(K)]
    local = rng.standard_normal(n).astype(np.float32)
    want = oracle.decode_accumulate_avg_segments(more % 4, cl, sl, bounds, local=local)
    for off in (0, 1):
        go = Guarded(n, np.float32)
        dq8.decode_accumulate_avg_segments(more % 4, [dev(c) for c in cl], [dev(s) for s in sl], bounds_dev(bounds), out=go.t, local=dev(local, off))
        same_bits(go.t, want, "segment average")
        go.check("segment average")


def test_calls_marshalled_by_the_extension_and_by_python(dq8, monkeypatch):
    """Ordinary arguments go through the extension, any others are declined there before anything has happened; both ways give the
    same bytes, on a side stream too, and errors are those of dq8.py."""
    native = dq8._native
    n, nb, n_seg = 5003, 5, 3
    rng = np.random.Generator(np.random.PCG64(9900))
    x, bounds = dev(rng.standard_normal(n).astype(np.float32)), bounds_dev(np.array([0, 7, 4099, n]))
    codes, scales = [dev(rng.integers(0, 256, n).astype(np.uint8)) for _ in range(3)], [dev(np.full(nb, 0.5 + k, np.float32)) for k in range(3)]
    new = lambda m, t=torch.float32: torch.empty(m, dtype=t, device="cuda")  # noqa: E731
    calls = [("absmax", lambda: [x, 1024, None]), ("absmax", lambda: [x, 0, new(1)]),
             ("encode", lambda: [0, x, 1024, None, None, False]), ("encode", lambda: [1, x, 1024, scales[1], new(n, torch.uint8), True]),
             ("decode", lambda: [2, codes[0], scales[0], 1024, None]), ("absmax_segments", lambda: [x, bounds, None]),
             ("encode_segments", lambda: [3, x, bounds, None, new(n, torch.uint8), False]),
             ("decode_segments", lambda: [0, codes[1], scales[1], bounds, new(n)]),
             ("decode_accumulate_avg", lambda: [0, codes, scales, 1024, None, None]), ("decode_accumulate_avg", lambda: [0, (), (), 1024, None, x]),
             ("decode_accumulate_avg_segments", lambda: [1, codes, tuple(scales), bounds, None, x]),
             ("decode_avg_encode", lambda: [2, codes, scales, 1024, x, None, None]),
             ("error_stats", lambda: [0, x, 0, None, False, new((1, 4), torch.float64), new(2, torch.float64)])]
    flat = lambda r: [t.cpu().numpy().tobytes() for t in (r if isinstance(r, tuple) else (r,))]  # noqa: E731
    side = torch.cuda.Stream()
    for name, args in calls:
        got = getattr(native, name)(*args())
        assert got is not None, name
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            beside = getattr(native, name)(*args())
        side.synchronize()
        with monkeypatch.context() as m:
            m.setattr(dq8, "_native", dq8._Unbound())
            want = getattr(dq8, name)(*args())
        if name != "error_stats":
            assert flat(got) == flat(want) == flat(beside), name
        else:
            assert np.allclose(got[0].cpu().numpy(), want[0].cpu().numpy(), rtol=1e-12) and got[1] is not want[1]
        # an argument that is not ordinary: a tensor subclass, a wrong type, a strided view, an integer of another type
        class Sub(torch.Tensor):
            pass
        for i, a in enumerate(args()):
            odd = {torch.Tensor: lambda: [a.as_subclass(Sub), a.to(torch.float16), torch.stack([a, a], -1)[..., 0], a.cpu()],
                   int: lambda: [np.int64(a), -1], bool: lambda: [int(a)], list: lambda: [iter(a), a[:1] + [None], a * 11], type(None): lambda: ["x"]}.get(type(a), lambda: [])()
            for o in odd:
                if isinstance(o, torch.Tensor) and o.is_contiguous() and o.is_cuda and type(o) is torch.Tensor and o.dtype == a.dtype:
                    continue
                changed = args()
                changed[i] = o
                assert getattr(native, name)(*changed) is None, (name, i, o)
    assert native.encode(0, new(0), 0, None, None, False) is None and dq8.encode(0, new(0))[0].numel() == 0
    out = new(n)
    assert dq8.decode(2, codes[0], scales[0], 1024, out=out) is out
    with pytest.raises(ValueError, match="out too small"):
        dq8.decode(2, codes[0], scales[0], 1024, out=new(n - 1))
    with pytest.raises(dq8.Dq8Error, match="dq8_encode failed .status 2.: unknown data type 9"):
        dq8.encode(9, x)
    with pytest.raises(Exception):  # a transformed tensor has no address; the same with and without the extension
        torch.vmap(lambda v: dq8.absmax(v, 0))(x[:64].view(8, 8))


def test_transformed_tensors_are_declined_and_refused(dq8, monkeypatch):
    """The extension declines a tensor inside vmap, and dq8.py refuses it with its own error, with and without the extension."""
    x, native = torch.ones(64, device="cuda"), dq8._native
    assert not isinstance(native, dq8._Unbound)

    def transformed(v):  # has no address
        assert native.absmax(v, 0, None) is None
        return dq8.absmax(v, 0)

    for way in (native, dq8._Unbound()):
        monkeypatch.setattr(dq8, "_native", way)
        with pytest.raises(RuntimeError, match="Cannot access data pointer of Tensor"):
            torch.vmap(transformed)(x.view(8, 8))


@pytest.mark.parametrize("n,n_seg", [(98305, 1), (98305, 4), (98305, 63), (98305, 65), (8192 * 63 + 1, 33), (256 * 8192, 64), (256 * 8192 + 3, 1),
                                     (256 * 8192 + 3, 5), ((1 << 24) + 4099, 1), ((1 << 24) + 4099, 64)])
def test_compression_with_and_without_scratch_memory(dq8, monkeypatch, n, n_seg):
    """Maxima merged through scratch memory (the extension hands it in), and without (the code of dq8.py does not); segments that begin
    and end in the same unit, long ones, empty ones; scratch memory that holds the largest numbers before the call."""
    rng = np.random.Generator(np.random.PCG64(9700 + n % 97 + n_seg))
    x = (rng.standard_normal(n) * np.exp(rng.uniform(-9, 0, n))).astype(np.float32)
    kind, offset = (n + n_seg) % 4, n_seg % 3
    bounds = np.concatenate([[0], np.sort(rng.integers(0, n + 1, n_seg - 1)), [n]])
    bounds[n_seg // 2] = bounds[n_seg // 2 + 1]
    bounds[0] = 0
    torch.full((1 << 18,), 3e38, device="cuda")  # given back at once: the allocator's next blocks
    for _ in range(2):
        if n_seg == 1:
            check_encode_decode(dq8, kind, x, 0, x_off=offset, c_off=offset, tag="one scale")
        check_segments(dq8, kind, x, bounds, x_off=offset, c_off=offset, tag="%d segments" % n_seg)
        monkeypatch.setattr(dq8, "_native", dq8._Unbound())


def test_scratch_memory_of_the_c_calls(dq8):
    """Too few bytes are not used; a workspace at an odd address or on top of another array is refused."""
    import ctypes
    L, n, vp, sz = dq8.lib(), 200000, ctypes.c_void_p, ctypes.c_size_t
    L.dq8_workspace_bytes.restype = L.dq8_workspace_bytes_segments.restype = sz
    x = dev(np.random.Generator(np.random.PCG64(9800)).standard_normal(n).astype(np.float32))
    codes, scale, work = torch.empty(n, dtype=torch.uint8, device="cuda"), torch.empty(1, device="cuda"), torch.empty(4096, dtype=torch.uint8, device="cuda")
    bounds, stream = bounds_dev(np.array([0, n])), torch.cuda.current_stream().cuda_stream
    want = [t.cpu().numpy().tobytes() for t in dq8.encode(0, x)]
    need = L.dq8_workspace_bytes(sz(n), sz(0), 0)
    assert need == L.dq8_workspace_bytes_segments(sz(n), sz(1), 0) == 1024
    assert 0 == L.dq8_workspace_bytes(sz(n), sz(0), 1) == L.dq8_workspace_bytes(sz(n), sz(4096), 0) == L.dq8_workspace_bytes_segments(sz(n), sz(65), 0)

    def calls(w, size):
        return (L.dq8_encode_ws(0, vp(x.data_ptr()), sz(n), sz(0), vp(scale.data_ptr()), vp(codes.data_ptr()), 0, vp(w), sz(size), vp(stream)),
                L.dq8_encode_segments_ws(0, vp(x.data_ptr()), sz(n), vp(bounds.data_ptr()), sz(1), vp(scale.data_ptr()), vp(codes.data_ptr()), 0, vp(w),
                                         sz(size), vp(stream)))
    for w, size in ((work.data_ptr(), need), (work.data_ptr() + 4, need), (work.data_ptr() + 1, need - 1), (None, need)):
        codes.zero_()
        scale.zero_()
        assert calls(w, size) == (0, 0)
        assert [codes.cpu().numpy().tobytes(), scale.cpu().numpy().tobytes()] == want
    for w in (work.data_ptr() + 1, x.data_ptr() + 4 * n - 4, codes.data_ptr(), scale.data_ptr(), x.data_ptr() - need + 4):
        assert calls(w, need) == (3, 3)
    assert L.dq8_encode_segments_ws(0, vp(x.data_ptr()), sz(n), vp(bounds.data_ptr()), sz(1), vp(scale.data_ptr()), vp(codes.data_ptr()), 0,
                                    vp(bounds.data_ptr()), sz(need), vp(stream)) == 3


def test_scratch_memory_of_the_statistics(dq8):
    """dq8_error_stats_ws: the same statistics with enough scratch memory, with too little and with none; other arrays' memory is refused."""
    import ctypes
    L, n, vp, sz = dq8.lib(), 200000, ctypes.c_void_p, ctypes.c_size_t
    x = dev(np.random.Generator(np.random.PCG64(9800)).standard_normal(n).astype(np.float32))
    scale, stream = torch.empty(1, device="cuda"), torch.cuda.current_stream().cuda_stream
    L.dq8_workspace_bytes_stats.restype = sz
    need, work = L.dq8_workspace_bytes_stats(sz(n), sz(0), 0), torch.empty(1 << 15, dtype=torch.uint8, device="cuda")
    stats, means = torch.empty(4, dtype=torch.float64, device="cuda"), torch.empty(2, dtype=torch.float64, device="cuda")
    want = oracle.error_stats(0, x.cpu().numpy(), 0)[0]
    for w, size, rc in ((work.data_ptr(), need, 0), (work.data_ptr() + 8, need, 0), (work.data_ptr() + 4, need - 1, 0), (None, need, 0), (work.data_ptr() + 4, need, 3),
                        (stats.data_ptr(), need, 3), (means.data_ptr(), need, 3), (x.data_ptr() + 8, need, 3)):
        stats.fill_(-1.0)
        assert L.dq8_error_stats_ws(0, vp(x.data_ptr()), sz(n), sz(0), vp(scale.data_ptr()), 0, vp(stats.data_ptr()), vp(means.data_ptr()), vp(w), sz(size), vp(stream)) == rc
        assert np.allclose(stats.cpu().numpy(), want if rc == 0 else -1.0, rtol=1e-12, atol=0)


# whole units only, elements past them for one wavefront and for several; four wavefronts per workgroup up to four units per compute
# unit and one unit more; a second unit for some wavefronts
@pytest.mark.parametrize("n", [4097, 5 * 1024 + 63, 9 * 1024 + 65, 30 * 1024 + 1023, 1024 * 1024, 1025 * 1024 + 1, 6144 * 1024 + 1025])
@pytest.mark.parametrize("offset", [0, 1])
def test_error_stats_of_one_block(dq8, monkeypatch, n, offset):
    """With scratch memory (the same bytes in every call) and without; no zeros, few, and almost nothing else; a given scale of 0."""
    rng = np.random.Generator(np.random.PCG64(6300 + n % 97))
    x = (rng.standard_normal(n) * np.exp(rng.uniform(-6, 0, n))).astype(np.float32)
    few = x.copy()
    few[[0, n // 2, n - 1]] = 0.0

    def both(kind, y, given=None):
        got = check_error_stats(dq8, kind, y, 0, given=given, tag="scratch")
        assert got.tobytes() == check_error_stats(dq8, kind, y, 0, given=given, tag="again").tobytes()
        with monkeypatch.context() as m:
            m.setattr(dq8, "_native", dq8._Unbound())
            check_error_stats(dq8, kind, y, 0, given=given, tag="none")
        return got
    if offset:  # an address that is aligned for an element only
        t = dev(x, offset)
        stats, means = torch.empty((1, 4), dtype=torch.float64, device="cuda"), torch.empty(2, dtype=torch.float64, device="cuda")
        want, _ = oracle.error_stats(n % 4, x, 0)
        got = dq8.error_stats(n % 4, t, 0, stats=stats, means=means)[0].cpu().numpy()
        assert got[:, 2:].tobytes() == want[:, 2:].tobytes() and np.all(np.abs(got - want) <= 2 * n * 2.0 ** -53 * want)
        return
    both(n % 4, x)
    both((n + 1) % 4, few, np.array([4.0], np.float32))
    both(2, np.zeros(n, np.float32), np.array([0.0], np.float32))
    for at, v in ((0, 0.3), (n // 2, -1e-7), (n - 1, 0.77))[:3 if n < 1 << 20 else 0]:  # sums of one term that is not 0: the term itself
        one = np.zeros(n, np.float32)
        one[at] = v
        assert both(at % 2, one, np.array([0.9], np.float32)).tobytes() == oracle.error_stats(at % 2, one, 0, scales=np.array([0.9], np.float32))[0].tobytes()


# units of 4096 elements (from 10 Mi elements on) and of 1024; whole, and with a last one of 1, 3, 4 and 1027 elements; 63 segments and 64
@pytest.mark.parametrize("n", [(10 << 20) - 1, 10 << 20, (10 << 20) + 3, (10 << 20) + 4, (12 << 20) + 1027])
@pytest.mark.parametrize("n_seg", [2, 63, 64])
def test_long_sets_of_tensors(dq8, n, n_seg):
    """Segments that end inside a unit, several in one part of a unit, in its first and last quad, and in the array's last unit."""
    rng = np.random.Generator(np.random.PCG64(9950 + n % 97 + n_seg))
    x = (rng.standard_normal(n) * np.exp(rng.uniform(-9, 0, n))).astype(np.float32)
    close = 4096 * 700 + np.array([0, 1, 3, 1023, 1024, 1025, 2050, 4093, 4095, 4096 + 5, 8192])
    inner = np.sort(np.concatenate([rng.integers(0, n + 1, max(0, n_seg - 14)), close, [n - 1, n - 2]])[-(n_seg - 1):])
    check_segments(dq8, n % 4, x, np.concatenate([[0], inner, [n]]), x_off=n % 3, c_off=n % 4, tag="long")


# the larger units only where out is a multiple of 16 bytes
@pytest.mark.parametrize("n", [(10 << 20) - 1, 10 << 20, (10 << 20) + 3, (12 << 20) + 1027])
@pytest.mark.parametrize("n_seg", [63, 64])
def test_long_sets_of_tensors_are_expanded_at_any_float(dq8, n, n_seg):
    """The same bytes at every float, from codes at every byte."""
    rng = np.random.Generator(np.random.PCG64(9960 + n % 97 + n_seg))
    x = (rng.standard_normal(n) * np.exp(rng.uniform(-9, 0, n))).astype(np.float32)
    close = 4096 * 700 + np.array([0, 1, 3, 1023, 1024, 1025, 2050, 4093, 4095, 4096 + 5, 8192])
    inner = np.sort(np.concatenate([rng.integers(0, n + 1, n_seg - 14), close, [n - 1, n - 2]]))
    codes, scales = dq8.encode_segments(n % 4, dev(x), bounds_dev(np.concatenate([[0], inner, [n]])))
    expanded = []
    for off in (0, 1, 2, 3):
        go, at = Guarded(n, np.float32, off), torch.empty(n + off, dtype=torch.uint8, device="cuda")[off:]
        at.copy_(codes)
        dq8.decode_segments(n % 4, at, scales, bounds_dev(np.concatenate([[0], inner, [n]])), out=go.t)
        go.check("expansion")
        expanded.append(go.t)
    assert all(torch.equal(expanded[0].view(torch.int32), e.view(torch.int32)) for e in expanded[1:])
    same_bits(expanded[0], oracle.decode_segments(n % 4, codes.cpu().numpy(), scales.cpu().numpy(), np.concatenate([[0], inner, [n]])), "expansion")


# more workers than the team kernels take in these blocks: every mean of a last block that is no whole unit, or of codes at an odd address,
# is formed for the maximum and once more for the compression
@pytest.mark.parametrize("block,K", [(256, 9), (512, 16), (1000, 9), (1024, 16), (2048, 9), (2048, 16), (3000, 16), (4000, 11)])
@pytest.mark.parametrize("rest,odd", [(0, 1), (1, 0), (5, 1), (-4, 0), (-1, 1)])
def test_many_workers_in_blocks_of_any_length(dq8, block, K, rest, odd):
    """k_avg_block: whole and short units, aligned codes and codes at odd addresses, with and without a local term."""
    n = block * 5 + rest % block
    rng = np.random.Generator(np.random.PCG64(9980 + n % 97 + K))
    kind, nb = (n + K) % 4, -(-n // block)
    cl = [rng.integers(0, 256, n).astype(np.uint8) for _ in range(K)]
    sl = [np.exp(rng.uniform(-4, 4, nb)).astype(np.float32) for _ in range(K)]
    x = rng.standard_normal(n).astype(np.float32) if rest % 2 == 0 else None
    codes, scales = [dev(c, odd * (k % 4)) for k, c in enumerate(cl)], [dev(v) for v in sl]
    want = oracle.decode_accumulate_avg(kind, cl, sl, block, local=x)
    wc, ws = oracle.encode(kind, want, block)
    gc, gs = Guarded(n, np.uint8, odd), Guarded(nb, np.float32)
    dq8.decode_avg_encode(kind, codes, scales, block, local=None if x is None else dev(x, odd), scales=gs.t, codes=gc.t)
    same_bits(gc.t, wc, "codes of the average")
    same_bits(gs.t, ws, "scales of the average")
    gc.check("codes of the average")
    gs.check("scales of the average")


# what is left after the whole units: quads for all lanes, then up to two elements per lane one by one or quads again
@pytest.mark.parametrize("rest", [64, 65, 127, 128, 129, 131, 255, 256, 300, 384, 385, 511])
@pytest.mark.parametrize("block,K", [(1000, 13), (4096, 17), (3000, 32)])
def test_averages_of_many_workers_with_a_rest_of_any_length(dq8, block, K, rest):
    """More than eight workers, units by position and inside blocks; codes at multiples of 4, out and local of 16."""
    n = 1024 * 12 + rest
    rng = np.random.Generator(np.random.PCG64(9990 + rest + K))
    kind, nb = (rest + K) % 4, -(-n // block)
    cl = [rng.integers(0, 256, n).astype(np.uint8) for _ in range(K)]
    sl = [np.exp(rng.uniform(-4, 4, nb)).astype(np.float32) for _ in range(K)]
    x = rng.standard_normal(n).astype(np.float32) if rest % 2 else None
    go = Guarded(n, np.float32)
    dq8.decode_accumulate_avg(kind, [dev(c) for c in cl], [dev(s) for s in sl], block, out=go.t, local=None if x is None else dev(x))
    same_bits(go.t, oracle.decode_accumulate_avg(kind, cl, sl, block, local=x), "average")
    go.check("average")


# a last block of 1, 3, 4, 5 elements, one short of whole quads and one short of whole; teams of one to four wavefronts and a workgroup
# per block; all workers unrolled, in passes and in chunks (blocks of 4096 and more; other blocks with more than eight workers: above)
@pytest.mark.parametrize("block,K", [(512, 2), (1000, 4), (1024, 1), (2048, 8), (3000, 5), (3500, 3), (4096, 6), (4096, 7), (4096, 9), (4096, 16), (5000, 2), (8192, 8),
                                     (12288, 11), (16384, 7)])
@pytest.mark.parametrize("rest", [1, 3, 4, 5, 257, -2])
@pytest.mark.parametrize("local", [False, True])
def test_averages_with_a_last_block_of_any_length(dq8, block, K, rest, local):
    """Averages and averages compressed again whose last block is no whole number of quads, at any alignment of an element."""
    n = block * (5 if block < 8192 else 3) + rest % block
    rng = np.random.Generator(np.random.PCG64(9970 + n % 97 + K))
    kind, nb, off = (n + K) % 4, -(-n // block), (K + rest) % 4
    cl = [rng.integers(0, 256, n).astype(np.uint8) for _ in range(K)]
    sl = [np.exp(rng.uniform(-4, 4, nb)).astype(np.float32) for _ in range(K)]
    x = rng.standard_normal(n).astype(np.float32) if local else None
    want = oracle.decode_accumulate_avg(kind, cl, sl, block, local=x)
    codes, scales = [dev(c, (off + k) % 4 if rest % 2 else 0) for k, c in enumerate(cl)], [dev(s) for s in sl]
    mine = None if x is None else dev(x, off)
    go = Guarded(n, np.float32)
    dq8.decode_accumulate_avg(kind, codes, scales, block, out=go.t, local=mine)
    same_bits(go.t, want, "average")
    go.check("average")
    wc, ws = oracle.encode(kind, want, block)
    gc, gs = Guarded(n, np.uint8, off), Guarded(nb, np.float32)
    dq8.decode_avg_encode(kind, codes, scales, block, local=mine, scales=gs.t, codes=gc.t)
    same_bits(gc.t, wc, "codes of the average")
    same_bits(gs.t, ws, "scales of the average")
    gc.check("codes of the average")
    gs.check("scales of the average")
