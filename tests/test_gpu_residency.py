"""Launches on either side of the lines from which the number of resident workgroups is bounded, against the oracle."""
import numpy as np
import pytest
import torch

from bagua_workloads import draw

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def bg():
    import paper_2107_01499_amd as b
    assert torch.cuda.is_available()
    return b


def same(t, want):
    return np.array_equal(t.cpu().numpy().view(np.uint32), want.view(np.uint32))


@pytest.mark.parametrize("k,n", [(1, (1 << 24) + 1), (2, (1 << 23) - 1), (2, (1 << 23) + 255), (3, 5592406), (5, 3355444), (8, (1 << 21) + 77), (16, (1 << 20) - 1), (16, 1 << 20)])
def test_ring_fp(bg, oracle, k, n):
    print("ring_fp k=%d n=%d" % (k, n), flush=True)
    xs = [draw("normal", n, 7 * k + i, "cpu", 0.02) for i in range(k)]
    out = [torch.full((n,), float("nan"), device="cuda") for _ in range(k)]
    bg.bagua_decentralized_avg(bg.AVG_FP, [x.cuda() for x in xs], out)
    want = oracle.ring_avg_fp([x.numpy() for x in xs])
    assert all(same(o, w) for o, w in zip(out, want))


@pytest.mark.parametrize("k,n", [(1, (1 << 26) - 1), (1, (1 << 26) + 3), (3, 22369621), (3, 22369622), (8, (1 << 23) - 7), (8, (1 << 23) + 2), (14, 4793491), (15, 100), (16, (1 << 22) + 1), (17, 3000)])
def test_ring_fp_rows_per_workgroup(bg, oracle, k, n):
    """Longer launches than those above, either side of 2^29 bytes, and the numbers of peers around the last with a kernel of its own."""
    test_ring_fp(bg, oracle, k, n)


@pytest.mark.parametrize("n,chunk", [((1 << 26), 2048), ((1 << 26) + 1, 2048), ((1 << 26) + 77, 16384), (3 * (1 << 24) * 2 - 5, 1536)])
def test_momentum_compression(bg, oracle, n, chunk):
    print("momentum n=%d C=%d" % (n, chunk), flush=True)
    g, m, r = (draw("normal", n, 91 + i, "cpu", s) for i, s in enumerate((1e-3, 1e-3, 1e-4)))
    bits, scale = torch.full(((n + 31) // 32,), -1, dtype=torch.int32, device="cuda"), torch.full((bg.num_chunks(n, chunk),), float("nan"), device="cuda")
    res = r.cuda()
    bg.bagua_momentum_sign_compress_ef(g.cuda(), m.cuda(), 0.9, res, chunk, bits, scale)
    want_r = r.numpy().copy()
    want_bits, want_scale = oracle.momentum_sign_compress_ef(g.numpy(), m.numpy(), 0.9, want_r, chunk)
    assert same(bits, want_bits) and same(scale, want_scale) and same(res, want_r)


@pytest.mark.parametrize("n,chunk", [((1 << 24) - 1, 4096), ((1 << 24) + 5, 4096), ((1 << 24) + 3072 * 7, 2816)])
def test_gossip_pairs(bg, oracle, n, chunk):
    print("gossip n=%d C=%d" % (n, chunk), flush=True)
    peer, nc = [1, 0, 2], bg.num_chunks(n, chunk)
    xs, hats = ([draw("normal", n, s + j, "cpu", 0.02) for j in range(3)] for s in (60, 70))
    hg, out = [h.cuda() for h in hats], [torch.full((n,), float("nan"), device="cuda") for _ in range(3)]
    codes, mm = [torch.full((n,), 255, dtype=torch.uint8, device="cuda") for _ in range(3)], [torch.full((2 * nc,), float("nan"), device="cuda") for _ in range(3)]
    bg.bagua_decentralized_avg_peers_lp([x.cuda() for x in xs], out, hg, codes, mm, peer, chunk)
    want_hat = [h.numpy().copy() for h in hats]
    want_out, want_codes, want_mm = oracle.peer_avg_lp([x.numpy() for x in xs], want_hat, peer, chunk)
    for j in range(3):
        assert same(out[j], want_out[j]) and same(hg[j], want_hat[j]) and same(mm[j], want_mm[j]) and np.array_equal(codes[j].cpu().numpy(), want_codes[j])


@pytest.mark.parametrize("n,chunk", [((5 << 23) - 3, 4096), ((5 << 23) + 5, 2816)])
def test_gossip_pairs_either_side_of_the_bound(bg, oracle, n, chunk):
    test_gossip_pairs(bg, oracle, n, chunk)


@pytest.mark.parametrize("codec", ["minmax", "sign"])
@pytest.mark.parametrize("chunk,sizes", [(2048, [(1 << 25) + 2048 * 3, 1000, (1 << 25) - 2048 * 2 - 1000]), (1536, [1 << 25, 77, (1 << 25) + 1]), (1024, [(1 << 26) - 1025, 1])])
def test_batched_worker_side(bg, oracle, codec, chunk, sizes):
    """Just below (1024: one chunk short) and above 2^26 elements in chunks of two, three and four waves, with short buckets among them."""
    print("batched %s C=%d" % (codec, chunk), flush=True)
    xs, rs = ([draw("normal", n, s + b, "cpu", sg).numpy() for b, n in enumerate(sizes)] for s, sg in ((80, 1e-3), (90, 1e-4)))
    words = [n if codec == "minmax" else (n + 31) // 32 for n in sizes]
    metas = [(2 if codec == "minmax" else 1) * bg.num_chunks(n, chunk) for n in sizes]
    codes = [torch.full((w,), -1 if codec == "sign" else 255, dtype=torch.int32 if codec == "sign" else torch.uint8, device="cuda") for w in words]
    meta, rg = [torch.full((m,), float("nan"), device="cuda") for m in metas], [torch.from_numpy(r).cuda() for r in rs]
    ws = torch.empty(bg.bagua_batch_workspace_bytes(len(sizes), 0), dtype=torch.uint8, device="cuda")
    call, want_of = (bg.bagua_compress_minmax_u8_batched, oracle.compress_minmax_u8) if codec == "minmax" else (bg.bagua_sign_compress_ef_batched, oracle.sign_compress_ef)
    call([torch.from_numpy(x).cuda() for x in xs], rg, chunk, codes, meta, ws)
    for b, x in enumerate(xs):
        want_r = rs[b].copy()
        want = want_of(x, want_r, chunk)
        assert np.array_equal(codes[b].cpu().numpy().view(np.uint8), want[0].view(np.uint8)) and same(meta[b], want[1]) and same(rg[b], want_r)


@pytest.mark.parametrize("codec", ["minmax", "sign"])
def test_batched_chunks_of_1024_beyond_the_line(bg, oracle, codec):
    test_batched_worker_side(bg, oracle, codec, 1024, [(1 << 28) - 3, 5])


@pytest.mark.parametrize("n,chunk", [(7 << 24, 2048), ((7 << 24) + 300, 2048), ((7 << 24) + 300, 1792)])
def test_momentum_either_side_of_the_line(bg, oracle, n, chunk):
    test_momentum_compression(bg, oracle, n, chunk)
