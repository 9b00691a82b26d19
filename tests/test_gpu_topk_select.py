"""Where the top-K selection can go wrong: the K-th magnitude far below the largest, in one crowded bin, among ties; and
entry lists longer than a workgroup in the server step.  Bit for bit against the oracle."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def bg():
    import paper_2107_01499_amd as b
    assert torch.cuda.is_available()
    return b


def values(kind, n, seed):
    r = np.random.default_rng(seed)
    sign = np.where(r.random(n) < 0.5, -1, 1).astype(np.float32)
    if kind == "binades":       # 60 binades: almost all of a chunk lies below the first histogram
        return (sign * np.exp2(r.uniform(-50, 10, n))).astype(np.float32)
    if kind == "crowded":       # one element far above, the rest within 2^-14 of each other
        x = sign * (1.0 + r.random(n) * 2.0 ** -14).astype(np.float32)
        x[::700] = 1e6
        return x.astype(np.float32)
    if kind == "neighbours":    # consecutive bit patterns, many of them several times
        return sign * (np.uint32(0x3f800000) + r.integers(0, 300, n).astype(np.uint32)).view(np.float32)
    if kind == "zeros":         # mostly +0 and -0
        return (sign * np.where(r.random(n) < 0.02, r.standard_normal(n), 0.0)).astype(np.float32)
    if kind == "denormal":
        return sign * r.integers(0, 1 << 23, n).astype(np.uint32).view(np.float32)
    return (r.standard_normal(n) * 1e-3).astype(np.float32)


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a.view(np.int16) if a.dtype == np.uint16 else a)).cuda()


def same(t, want):
    return t.cpu().numpy().tobytes() == want.tobytes()


@pytest.mark.parametrize("kind", ["binades", "crowded", "neighbours", "zeros", "denormal", "normal"])
@pytest.mark.parametrize("C,keep", [(256, 255), (1024, 32), (1536, 700), (4096, 1), (4096, 128), (4096, 4095), (8192, 1024), (16384, 5000)])
def test_select(bg, oracle, kind, C, keep):
    n = 2 * C + C // 2 + 3
    print("select %s C=%d keep=%d" % (kind, C, keep), flush=True)
    x, res = values(kind, n, C + keep), np.zeros(n, np.float32)
    rg = dev(res)
    io, vo = oracle.compress_topk(x, res, C, keep)
    slots = bg.num_chunks(n, C) * keep
    ig, vg = torch.zeros(slots, dtype=torch.int16, device="cuda"), torch.zeros(slots, device="cuda")
    bg.bagua_compress_topk_ef(dev(x), rg, C, keep, ig, vg)
    assert same(ig, io) and same(vg, vo) and same(rg, res)


@pytest.mark.parametrize("k", [1, 3, 9])
@pytest.mark.parametrize("C,keep", [(256, 65), (1024, 64), (1024, 129), (1024, 257), (1024, 1000), (4096, 257), (4096, 2049), (16384, 8193), (16384, 16384)])
def test_server_lists(bg, oracle, k, C, keep):
    n = 2 * C - 5
    print("server lists k=%d C=%d keep=%d" % (k, C, keep), flush=True)
    enc = [oracle.compress_topk(values("normal", n, 31 * k + j), None, C, keep) for j in range(k)]
    eps = values("normal", n, 5)
    eg = dev(eps)
    io, vo, oo = oracle.drr_topk([e[0] for e in enc], [e[1] for e in enc], eps, n, C, keep, want_fp32=True)
    slots = bg.num_chunks(n, C) * keep
    ig, vg, og = torch.zeros(slots, dtype=torch.int16, device="cuda"), torch.zeros(slots, device="cuda"), torch.zeros(n, device="cuda")
    bg.bagua_decompress_reduce_recompress_topk([dev(e[0]) for e in enc], [dev(e[1]) for e in enc], keep, eg, n, C, ig, vg, og)
    assert same(ig, io) and same(vg, vo) and same(eg, eps) and same(og, oo)
