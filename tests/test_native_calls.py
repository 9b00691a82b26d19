"""The binding's host extension: it declines what is not an ordinary call, so that the general path words the refusal, and for an
ordinary one it does what the general path does."""
import importlib.util
import inspect
import os
import sysconfig

import pytest
import torch

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

ROUNDS = [
    dict(kind="round", codec="minmax", k=3, n=70001, chunk=2048),
    dict(kind="round", codec="sign", k=5, n=9000, chunk=1024),
    dict(kind="buckets", codec="sign", k=2, n=50000, buckets=3, chunk=1024, flatten=True, odd=True),
    dict(kind="gather", codec="minmax", k=2, n=30001, chunk=1536, odd=True),
    dict(kind="gather", codec="sign", k=3, n=30001, chunk=4096, odd=True),
    dict(kind="hier", codec="minmax", k=2, local=4, n=5001, chunk=1024),
    dict(kind="hier", codec="sign", k=1, local=2, n=40001, chunk=2048),
    dict(kind="topk", k=3, n=20001, chunk=2048, keep=64, opt="sgd"),
    dict(kind="topk", k=2, n=20001, chunk=1024, keep=8, opt="adam"),
    dict(kind="ring_fp", k=5, n=30001),
    dict(kind="ring_lp", k=32, n=9001, chunk=1024),
    dict(kind="peers", k=7, n=9001, chunk=1024, lp=True),
    dict(kind="peers", k=4, n=9001, chunk=1024, lp=False),
    dict(kind="share", n=30001, chunk=1024),
]


@pytest.fixture(scope="module")
def bg():
    import paper_2107_01499_amd as b
    return b


def natives(bg):
    return [n for n in dir(bg.binding._native) if n.startswith("bagua_")]


def test_every_native_call_takes_the_arguments_of_its_function(bg):
    names = natives(bg)
    assert len(names) == 25 and set(names) <= set(bg.binding.EXPORTS)
    for n in names:
        params = inspect.signature(getattr(bg, n)).parameters
        f = getattr(bg.binding._native, n)
        assert list(params)[-1] == "stream"
        for count in (0, len(params) - 1, len(params), len(params) + 1):
            assert f(*[None] * count) is False, (n, count)


class Sub(torch.Tensor):
    pass


def test_what_is_not_ordinary_is_declined_and_refused_as_before(bg):
    f = bg.binding._native.bagua_compress_minmax_u8
    x, r, c, m = torch.zeros(512), torch.zeros(512), torch.zeros(512, dtype=torch.uint8), torch.zeros(4)
    for args in ((x, r, 256, c, m), (x.as_subclass(Sub), r, 256, c, m), (x[::2], r, 256, c, m), (x.numpy(), r, 256, c, m), (x, r, 256.0, c, m),
                 (x.to("meta"), r, 256, c, m), (x.to_sparse(), r, 256, c, m), (x, r, -1, c, m), (x, r, 1 << 70, c, m)):
        assert f(*args, None) is False
    with pytest.raises(ValueError, match="contiguous GPU tensor"):
        bg.bagua_compress_minmax_u8(x, r, 256, c, m)
    with pytest.raises(ValueError, match="contiguous GPU tensor"):
        bg.bagua_decentralized_avg(bg.AVG_FP, [x, x], [r, r])
    with pytest.raises(ValueError, match="one per worker"):
        bg.bagua_decentralized_avg(bg.AVG_FP, [x, x], [r])
    with pytest.raises(AttributeError):
        bg.bagua_compress_minmax_u8(None, r, 256, c, m)


def test_an_extension_for_another_python_or_torch_is_not_loaded(bg):
    """The extension holds the layouts of torch's and Python's types, so its name has both versions in it."""
    from paper_2107_01499_amd import build
    path = build.native_path()
    assert bg.binding._native.__spec__.origin == path and os.path.exists(path)
    name = os.path.basename(path)
    assert torch.__version__ in name and sysconfig.get_config_var("SOABI") in name
    assert build.native_path(torch_version="0.0.0") != path and not os.path.exists(build.native_path(torch_version="0.0.0"))


def test_without_the_extension_the_general_path_makes_the_calls(bg):
    with pytest.warns(RuntimeWarning, match="host extension is not there"):
        none = bg.binding._load_native(os.path.join(ROOT, "there-is-none.so"))
    assert none.bagua_compress_minmax_u8(None, None, 256, None, None, None) is False


def test_where_the_extension_cannot_be_built_there_is_none(bg, tmp_path, monkeypatch):
    from paper_2107_01499_amd import build
    old = build.native_path(str(tmp_path))
    open(old, "w").close()
    monkeypatch.setattr(build, "CXX", str(tmp_path / "no-compiler"))
    with pytest.warns(RuntimeWarning, match="no-compiler is missing"):
        assert build.build_native(libdir=str(tmp_path)) is None
    assert not os.path.exists(old)


def _cases():
    spec = importlib.util.spec_from_file_location("perf_cases", os.path.join(ROOT, "perf", "cases.py"))
    mod = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(mod)
    return mod


def _flat(o):
    if o is None or isinstance(o, torch.Tensor):
        return [] if o is None else [o]
    return [t for v in o for t in _flat(v)]


@pytest.mark.gpu
@pytest.mark.parametrize("case", ROUNDS, ids=lambda c: "%s-%s" % (c["kind"], c.get("codec", c.get("opt", c.get("lp", "")))))
def test_both_paths_make_the_same_call(bg, case, monkeypatch):
    cases = _cases()
    got = []
    for native in (True, False):
        state = cases.prepare(case, 5)
        with monkeypatch.context() as patch:
            if native:   # nothing is left for the general path (a prepared batched call holds its entry point already)
                patch.setattr(bg.binding, "_lib", None)
            else:
                patch.setattr(bg.binding, "_native", type("Declines", (), {n: staticmethod(lambda *a: False) for n in natives(bg)}))
            got.append([t.clone() for _ in range(2) for t in _flat(cases.run(state))])
    assert len(got[0]) == len(got[1]) > 0
    for a, b in zip(*got):
        assert torch.equal(a.view(torch.uint8), b.view(torch.uint8))


@pytest.mark.gpu
def test_the_other_calls_and_a_stream_of_their_own(bg):
    g = torch.Generator(device="cuda").manual_seed(1)
    n, chunk = 5000, 1024
    xs = [torch.empty(n, device="cuda").normal_(generator=g) for _ in range(3)]
    torch.cuda.synchronize()
    s = torch.cuda.Stream()
    native, out = bg.binding._native, torch.zeros(n, device="cuda")
    torch.cuda.synchronize()
    assert native.bagua_centralized_avg_fp(xs, out, s)
    s.synchronize()
    assert torch.equal(out, ((xs[0] + xs[1]) + xs[2]) * torch.tensor(1.0 / 3.0, device="cuda"))
    idx, val = torch.zeros(5 * 1024, dtype=torch.int16, device="cuda"), torch.zeros(5 * 1024, device="cuda")
    with torch.cuda.stream(s):
        assert native.bagua_compress_topk_ef(xs[0], None, chunk, chunk, idx, val, None)
        assert native.bagua_decompress_topk(idx, val, n, chunk, chunk, out, None)
    s.synchronize()
    assert torch.equal(out, xs[0])
    ws = torch.empty(bg.bagua_flatten_workspace_bytes(1, n), dtype=torch.uint8, device="cuda")
    bg.bagua_flatten_plan([xs[1]], [0], n, ws)
    assert native.bagua_bucket_flatten_run(ws, 1, out, None)
    assert torch.equal(out, xs[1])
    assert native.bagua_bucket_unflatten_run(ws, 1, xs[2], None)
    assert torch.equal(xs[1], xs[2])
    with pytest.raises(bg.binding.BaguaError, match="BAGUA_ERR_INVALID_ARG") as e:   # refused by the entry point itself
        native.bagua_compress_topk_ef(xs[0], None, 100, 10, idx, val, None)
    assert e.value.status == 1
