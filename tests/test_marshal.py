"""The extension module that makes ordinary tensor calls does what the binding's own steps do:
the same results, outputs and errors for every form of the arguments."""
import ctypes
import sys
import threading
import types

import numpy as np
import pytest
import torch

import paper_2409_17264_amd as medha
from paper_2409_17264_amd import binding
from paper_2409_17264_amd import workloads as wl


def _outcome(call, buffers):
    """What a call returns, copied, or raises; the callers' outputs hold NaN before it."""
    for t in buffers:
        t.fill_(float("nan"))
    try:
        r = call()
    except Exception as e:  # noqa: BLE001
        return type(e), getattr(e, "code", None)
    torch.cuda.synchronize()
    return tuple(t.clone() for t in r)


def _same(a, b):
    if isinstance(a, tuple) and a and isinstance(a[0], torch.Tensor):
        assert isinstance(b, tuple) and len(a) == len(b)
        for x, y in zip(a, b):
            assert (x.dtype, x.shape, x.device, x.is_contiguous()) == (y.dtype, y.shape, y.device,
                                                                       y.is_contiguous())
            assert torch.equal(x, y)
    else:
        assert a == b


def _forms(x):
    """The same numbers as a scheduler may hold them."""
    x = np.asarray(x)
    wide = np.zeros(2 * len(x), x.dtype)
    wide[::2] = x
    raw = np.zeros(x.nbytes + 1, np.uint8)
    odd = raw[1:].view(x.dtype)
    odd[:] = x
    return [x, x.tolist(), tuple(x.tolist()), x.astype(np.int64), x.astype(np.int32),
            x.astype(np.float64), wide[::2], x.reshape(1, -1), odd, torch.from_numpy(x.copy()),
            x.astype(x.dtype.newbyteorder(">")), [x.tolist()], list(x), x.astype(np.uint32),
            # numpy keeps the low half of what int32 does not hold
            x.astype(np.int64) + (1 << 32), (x.astype(np.int64) + (1 << 32)).tolist()]


def test_calls_without_a_device_are_refused_as_before():
    b = wl.make_prefill_batch("cpu", 2, 1, 64, [20], [4], seed=1)
    pt = torch.from_numpy(b.page_table)
    with pytest.raises(AssertionError):
        medha.chunked_prefill_attn(b.q, b.k_pool, b.v_pool, pt, b.page_table_offs, b.prefix_len,
                                   b.chunk_len, b.scale)
    with pytest.raises(AssertionError):
        medha.lse_merge(torch.zeros(1, 1, 1, 4), torch.zeros(1, 1, 1))
    with pytest.raises(AssertionError):
        medha.kv_append(b.q[:, :1].contiguous(), b.q[:, :1].contiguous(), b.k_pool, b.v_pool, pt,
                        b.page_table_offs, b.prefix_len, b.chunk_len)


@pytest.mark.parametrize("module", [None, types.SimpleNamespace(torch_version="0.1")])
def test_plans_and_sizes_need_no_extension_module(monkeypatch, module):
    """A module that is not there, or was built for another torch, leaves the library usable."""
    package = sys.modules[medha.__name__]
    size = medha.chunked_prefill_workspace_bytes([20000], [500], 8, 1, 128)
    plan = medha.describe_plan([20000], [500], 8, 1, 128, 256)[1:]
    try:
        with monkeypatch.context() as m:
            m.setitem(sys.modules, medha.__name__ + "._marshal", module)
            m.delattr(package, "_marshal", raising=False)
            if module is not None:
                m.setattr(package, "_marshal", module, raising=False)
            m.setattr(binding, "_LIB", None)
            m.setattr(binding, "_NATIVE", None)
            with pytest.warns(RuntimeWarning, match="extension module"):
                assert medha.chunked_prefill_workspace_bytes([20000], [500], 8, 1, 128) == size
            assert medha.describe_plan([20000], [500], 8, 1, 128, 256)[1:] == plan
            assert binding._NATIVE.kv_append(*range(8)) is None
    finally:
        binding._LIB = None
        binding.load_library()
    assert binding._NATIVE.torch_version == torch.__version__


class _OnDevice(torch.Tensor):
    """A host tensor that says it is on the device, for checks that come before any launch."""

    is_cuda = property(lambda self: True)


def _on_device(t):
    return t.as_subclass(_OnDevice)


@pytest.mark.parametrize("d_q,d_kv", [(64, 128), (128, 64)])
def test_a_head_dim_that_is_not_the_caches_is_refused(monkeypatch, d_q, d_kv):
    """The library knows the cache's head dim only: it would read past q and write past out."""
    launched = []
    monkeypatch.setattr(binding, "_stream", lambda: launched.append(1))
    b = wl.make_prefill_batch("d", 2, 1, d_kv, [20], [4], seed=1)
    q = _on_device(torch.zeros(4, 2, d_q, dtype=torch.bfloat16))
    k, v, pt = _on_device(b.k_pool), _on_device(b.v_pool), _on_device(torch.from_numpy(b.page_table))
    offs, pre, chk, kl = b.page_table_offs, b.prefix_len, b.chunk_len, b.prefix_len + b.chunk_len
    out, lse = _on_device(torch.zeros(4, 2, d_q)), _on_device(torch.zeros(4, 2))
    ws = _on_device(torch.zeros(1 << 20, dtype=torch.uint8))
    for call in (
            lambda: medha.chunked_prefill_attn(q, k, v, pt, offs, pre, chk, 1.0, out, lse, ws),
            lambda: medha.chunked_prefill_attn_noalloc(q, k, v, pt, offs, pre, chk, 1.0, out, lse),
            lambda: medha.decode_partial_attn(q, k, v, pt, offs, [0], kl, 1.0, out[:1], lse[:1], ws),
            lambda: medha.chunk_partial_attn(q, k, v, pt, offs, [0], chk, kl, pre + 1, 1.0, out, lse,
                                             ws)):
        with pytest.raises(AssertionError):
            call()
    assert not launched


def test_memory_that_the_kernels_cannot_reach_is_refused(monkeypatch):
    launched = []
    monkeypatch.setattr(binding, "_stream", lambda: launched.append(1))
    b = wl.make_prefill_batch("host", 2, 1, 64, [20], [4], seed=1)
    good = dict(q=_on_device(b.q), k=_on_device(b.k_pool), v=_on_device(b.v_pool),
                pt=_on_device(torch.from_numpy(b.page_table)),
                out=_on_device(torch.zeros(4, 2, 64)), lse=_on_device(torch.zeros(4, 2)),
                ws=_on_device(torch.zeros(1 << 20, dtype=torch.uint8)))
    offs, pre, chk, kl = b.page_table_offs, b.prefix_len, b.chunk_len, b.prefix_len + b.chunk_len

    def calls(q, k, v, pt, out, lse, ws):
        yield lambda: medha.chunked_prefill_attn(q, k, v, pt, offs, pre, chk, 1.0, out, lse, ws)
        yield lambda: medha.decode_partial_attn(q, k, v, pt, offs, [0], kl, 1.0, out[:1], lse[:1],
                                                ws)
        yield lambda: medha.chunk_partial_attn(q, k, v, pt, offs, [0], chk, kl, pre + 1, 1.0, out,
                                               lse, ws)

    one = _on_device(torch.zeros(1, dtype=torch.uint8))
    for bad in (dict(k=b.k_pool), dict(v=b.v_pool), dict(out=torch.zeros(4, 2, 64)),
                dict(lse=torch.zeros(4, 2)), dict(ws=torch.zeros(1 << 20, dtype=torch.uint8)),
                # one byte that says it is a megabyte, and every other byte of two
                dict(ws=one.expand(1 << 20)), dict(ws=one.repeat(2 << 20)[::2])):
        for call in calls(**dict(good, **bad)):
            with pytest.raises(AssertionError):
                call()
    po, pl = _on_device(torch.zeros(2, 4, 2, 64)), _on_device(torch.zeros(2, 4, 2))
    with pytest.raises(AssertionError):
        medha.lse_merge(po, torch.zeros(2, 4, 2))
    for out, lse in ((torch.zeros(4, 2, 64), good["lse"]), (good["out"], torch.zeros(4, 2)),
                     (good["out"].bfloat16(), good["lse"])):
        with pytest.raises(AssertionError):
            medha.lse_merge(po, pl, out, lse)
    assert not launched
    # dense in another order, or nothing at all, is a workspace
    binding._check_workspace(_on_device(torch.zeros(64, 32, dtype=torch.uint8)).t())
    binding._check_workspace(torch.zeros(0, dtype=torch.uint8))


@pytest.mark.gpu
def test_results_outputs_and_errors_are_those_of_the_binding(monkeypatch):
    b = wl.make_prefill_batch("marshal", 8, 2, 128, [1500, 70, 0], [40, 1, 130], seed=11)
    q, k, v = b.q.cuda(), b.k_pool.cuda(), b.v_pool.cuda()
    pt = torch.from_numpy(b.page_table).cuda()
    offs, pre, chk = b.page_table_offs, b.prefix_len, b.chunk_len
    tokens = b.tokens
    new = wl.randn_bf16((tokens, 2, 128), 12, "cuda")
    kl = (pre + chk).astype(np.int32)
    qi = np.array([0, 3, 9], np.int32)
    rows = np.array([0, 40, 41], np.int32)
    f32 = dict(dtype=torch.float32, device="cuda")
    po, pl = torch.randn(3, 5, 8, 128, **f32), torch.randn(3, 5, 8, **f32)
    ws = torch.empty(64 << 20, dtype=torch.uint8, device="cuda")
    small = torch.empty(256, dtype=torch.uint8, device="cuda")

    def prefill(offs=offs, pre=pre, chk=chk, q=q, k=k, v=v, pt=pt, scale=b.scale, **o):
        return lambda: medha.chunked_prefill_attn(q, k, v, pt, offs, pre, chk, scale, **o)

    def decode(qi=qi, kl=kl, q=q, **o):
        return lambda: medha.decode_partial_attn(q, k, v, pt, offs, qi, kl, b.scale, **o)

    def chunk(rows=rows, chk=chk, kl=kl, v0=pre + 1, q=q, **o):
        return lambda: medha.chunk_partial_attn(q, k, v, pt, offs, rows, chk, kl, v0, b.scale, **o)

    def append(offs=offs, pre=pre, chk=chk, new=new):
        def run():
            kk, vv = k.clone(), v.clone()
            medha.kv_append(new, new, kk, vv, pt, offs, pre, chk)
            return kk, vv
        return run

    buffers = []

    def given(shape, names=("out", "lse"), **bad):
        buffers.extend((torch.empty(shape + (8, 128), **dict(f32, **bad)),
                        torch.empty(shape + (8,), **f32)))
        return dict(zip(names, buffers[-2:]))

    def partial(shape):
        return given(shape, names=("out_partial", "lse_partial"))

    calls = [prefill(), decode(), chunk(), append(), lambda: medha.lse_merge(po, pl)]
    for form in _forms(offs):
        calls += [prefill(offs=form), append(offs=form)]
    for form in _forms(pre):
        calls += [prefill(pre=form), append(pre=form)]
    for form in _forms(chk):
        calls += [prefill(chk=form), chunk(chk=form), append(chk=form)]
    for form in _forms(kl):
        calls += [decode(kl=form), chunk(kl=form)]
    for s in (1, 0, np.float32(0.1), np.float64(-0.3), torch.tensor(0.2)):
        calls.append(prefill(scale=s))
    for w in (ws, small, None):
        calls += [prefill(workspace=w), decode(workspace=w), chunk(workspace=w),
                  prefill(workspace=w, **given((tokens,))), decode(workspace=w, **partial((3,))),
                  chunk(workspace=w, **partial((tokens,)))]
    calls.append(lambda: medha.lse_merge(po, pl, **given((5,))))
    # refused, by the binding or by the library
    calls += [prefill(q=q.float()), prefill(q=q[:, ::2]), prefill(q=q[:-1]), prefill(k=k[:-1]),
              prefill(k=k.float()), prefill(k=k.reshape(-1)), prefill(pt=pt.long()),
              prefill(pt=pt[:-1]), prefill(pt=pt.cpu()), prefill(offs=offs[:-1]),
              prefill(pre=pre[:-1]), prefill(pre=-pre - 1), prefill(pre="x"), prefill(pre=None),
              prefill(scale=float("nan")), prefill(scale="x"), prefill(scale=None),
              prefill(**given((tokens + 1,))), prefill(**given((tokens,), dtype=torch.float64)),
              decode(qi=qi + 1000), decode(kl=-kl), decode(**partial((2,))), chunk(rows=rows + 1000),
              chunk(v0=pre[:-1]), append(new=new[:-1]), append(new=new.float()),
              lambda: medha.lse_merge(po, pl[:-1]), lambda: medha.lse_merge(po.half(), pl),
              lambda: medha.lse_merge(po[..., :6].contiguous(), pl)]
    # refused before any launch: another head dim than the cache's, workspaces that are no memory of
    # the device's or less of it than they say
    q64 = q[..., :64].contiguous()
    for w in (ws, None):
        calls += [prefill(q=q64, workspace=w), decode(q=q64, workspace=w), chunk(q=q64, workspace=w)]
    for w in (torch.zeros(1 << 20, dtype=torch.uint8), small[:1].expand(1 << 20), ws[::2]):
        calls += [prefill(workspace=w), decode(workspace=w), chunk(workspace=w)]
    refused = 0
    for i, call in enumerate(calls):
        native = _outcome(call, buffers)
        with monkeypatch.context() as m:
            m.setattr(binding, "_NATIVE", binding._LongWay)
            plain = _outcome(call, buffers)
        print(f"call {i}", flush=True)
        _same(native, plain)
        refused += isinstance(native, tuple) and isinstance(native[0], type)
    assert refused >= 28 + 15
    # the module makes the ordinary calls itself, and hands back the caller's outputs
    n = binding._NATIVE
    out, lse = given((tokens,)).values()
    r = n.chunked_prefill_attn(q, k, v, pt, offs, pre, chk, b.scale, out, lse, None)
    assert r[0] is out and r[1] is lse
    out, lse = given((3,)).values()
    r = n.decode_partial_attn(q, k, v, pt, offs, qi, kl, b.scale, out, lse, ws)
    assert r[0] is out and r[1] is lse
    out, lse = given((tokens,)).values()
    r = n.chunk_partial_attn(q, k, v, pt, offs, rows, chk, kl, pre + 1, b.scale, out, lse, ws)
    assert r[0] is out and r[1] is lse
    out, lse = given((5,)).values()
    r = n.lse_merge(po, pl, out, lse)
    assert r[0] is out and r[1] is lse
    assert n.kv_append(new, new, k, v, pt, offs, pre, chk) is True
    assert n.lse_merge(po, pl, None, None) is not None
    # with lengths as lists, tuples and 64-bit arrays, and with or without a workspace
    for form in (lambda x: x, lambda x: x.tolist(), lambda x: tuple(x.tolist()),
                 lambda x: x.astype(np.int64)):
        for w in (ws, None):
            lengths = [form(x) for x in (offs, rows, chk, kl, pre + 1, pre, qi)]
            o, r, c, n_keys, v0, p, i = lengths
            made = (n.chunked_prefill_attn(q, k, v, pt, o, p, c, b.scale, None, None, w),
                    n.decode_partial_attn(q, k, v, pt, o, i, n_keys, b.scale, None, None, w),
                    n.chunk_partial_attn(q, k, v, pt, o, r, c, n_keys, v0, b.scale, None, None, w))
            with monkeypatch.context() as m:
                m.setattr(binding, "_NATIVE", binding._LongWay)
                plain = (prefill(workspace=w)(), decode(workspace=w)(), chunk(workspace=w)())
            torch.cuda.synchronize()
            for x, y in zip(made, plain):
                _same(x, y)
    for bad in ([True, 1, 1], [1.0, 1, 1], [1 << 40, 1, 1], pre.astype(np.int64) + (1 << 32)):
        assert n.chunked_prefill_attn(q, k, v, pt, offs, bad, chk, b.scale, None, None, None) is None


def _five_calls():
    """scale -> the tensor calls, each of the form that the module makes itself."""
    b = wl.make_prefill_batch("five", 2, 1, 64, [20], [4], seed=1)
    q, k, v, pt = b.q.cuda(), b.k_pool.cuda(), b.v_pool.cuda(), torch.from_numpy(b.page_table).cuda()
    offs, pre, chk, kl = b.page_table_offs, b.prefix_len, b.chunk_len, b.prefix_len + b.chunk_len
    zero = np.zeros(1, np.int32)
    ws = torch.empty(1 << 20, dtype=torch.uint8, device="cuda")
    new = wl.randn_bf16((4, 1, 64), 2, "cuda")
    po = wl.randn_bf16((2, 4, 2, 64), 3, "cuda").float()
    pl = wl.randn_bf16((2, 4, 2), 4, "cuda").float()
    medha.kv_append(new, new, k, v, pt, offs, pre, chk)  # the later ones write the same again
    return {
        "prefill": lambda s=b.scale: medha.chunked_prefill_attn(q, k, v, pt, offs, pre, chk, s),
        "decode": lambda s=b.scale: medha.decode_partial_attn(q, k, v, pt, offs, zero, kl, s,
                                                              workspace=ws),
        "chunk": lambda s=b.scale: medha.chunk_partial_attn(q, k, v, pt, offs, zero, chk, kl, pre + 1,
                                                            s, workspace=ws),
        "merge": lambda: medha.lse_merge(po, pl),
        "append": lambda: medha.kv_append(new, new, k, v, pt, offs, pre, chk)}


def _as_one(results):
    """The five calls' results as one list of tensors (the append has none)."""
    return [t.clone() for r in results if r is not None for t in r]


@pytest.mark.gpu
def test_calls_go_to_the_current_stream_of_their_thread():
    """From another stream, and from threads with a stream each, over and over: the results of the
    default stream, behind work that the stream still has before it."""
    five = _five_calls()
    want = _as_one(call() for call in five.values())
    torch.cuda.synchronize()
    wrong = []

    def work():
        stream = torch.cuda.Stream()
        with torch.cuda.stream(stream):
            five = _five_calls()  # (a workspace of its own for every thread)
            for _ in range(20):
                got = _as_one(call() for call in five.values())
                stream.synchronize()
                if not all(map(torch.equal, got, want)):
                    wrong.append(1)

    work()
    threads = [threading.Thread(target=work) for _ in range(3)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong
    # the call waits for what its own stream has before it
    b = wl.make_prefill_batch("order", 8, 1, 128, [5000], [300], seed=3)
    q, k, v, pt = b.q.cuda(), b.k_pool.cuda(), b.v_pool.cuda(), torch.from_numpy(b.page_table).cuda()
    args = (k, v, pt, b.page_table_offs, b.prefix_len, b.chunk_len, b.scale)
    want = _as_one([medha.chunked_prefill_attn(q, *args)])
    torch.cuda.synchronize()
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        late = torch.zeros_like(q)
        busy = torch.randn(4096, 4096, device="cuda")
        for _ in range(20):
            busy = busy @ busy * 1e-3
        late.copy_(q)
        got = medha.chunked_prefill_attn(late, *args)
    stream.synchronize()
    assert all(map(torch.equal, got, want))


@pytest.mark.gpu
def test_calls_can_be_captured():
    """A graph of the five calls, replayed between eager work on other inputs."""
    five = _five_calls()
    want = _as_one(call() for call in five.values())
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        captured = [call() for call in five.values()]
    outputs = [t for r in captured if r is not None for t in r]
    other = wl.make_prefill_batch("other", 8, 2, 128, [900, 40], [30, 1], seed=9)
    q, k, v = other.q.cuda(), other.k_pool.cuda(), other.v_pool.cuda()
    pt = torch.from_numpy(other.page_table).cuda()
    for _ in range(5):
        for t in outputs:
            t.fill_(float("nan"))
        medha.chunked_prefill_attn(q, k, v, pt, other.page_table_offs, other.prefix_len,
                                   other.chunk_len, other.scale)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert all(map(torch.equal, outputs, want))


@pytest.mark.gpu
@pytest.mark.parametrize("error", [KeyboardInterrupt, TimeoutError])
def test_what_is_raised_inside_a_call_reaches_the_caller(monkeypatch, error):
    """Interrupts and signal handlers' errors come up where Python code runs: in the conversion of
    the scale and in the search for the stream.  They come up once."""
    raised = []

    def once(value):
        if not raised:
            raised.append(1)
            raise error()
        return value

    class Scale:
        def __float__(self):
            return once(0.125)

    five = _five_calls()
    device = torch.cuda.current_device
    monkeypatch.setattr(torch.cuda, "current_device", lambda: once(device()))
    for name, call in five.items():
        raised[:] = [1]
        call()  # (nothing raises: the module makes the call)
        raised.clear()
        with pytest.raises(error):
            call()
        call()
        if name in ("prefill", "decode", "chunk"):
            raised.clear()
            with pytest.raises(error):
                call(Scale())
            call(Scale())
    torch.cuda.synchronize()


@pytest.mark.gpu
@pytest.mark.parametrize("code", [-1, -2, -3, -4])
def test_an_error_with_work_enqueued_is_raised_and_not_tried_again(code):
    """Entry points that answer with an error code: a refusal goes the long way, to the library, and
    the call is made; a runtime error is the call's."""
    calls = []
    entry = ctypes.CFUNCTYPE(ctypes.c_int)(lambda: calls.append(1) or code)
    address = ctypes.cast(entry, ctypes.c_void_p).value
    five = _five_calls()
    binding.load_library()
    try:
        binding._NATIVE.bind(binding._stream, binding._check, *[address] * 8)
        for i, call in enumerate(five.values()):
            if code == -4:
                with pytest.raises(medha.MedhaError) as e:
                    call()
                assert e.value.code == code
            else:
                call()
            assert len(calls) == i + 1
    finally:
        binding._LIB = None
        binding.load_library()  # binds the library's own again
    for call in five.values():
        call()
    assert len(calls) == 5
    torch.cuda.synchronize()
