"""Launches around the number of chunks from which the workgroups take the chunks in another order than their own (2048; then
runs of 128, 32 and 4 chunks for chunk lengths up to 1024, up to 4096 and above), with and without chunks left over."""
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
    return np.array_equal(t.cpu().numpy().view(np.uint8), want.view(np.uint8))


def room(codec, n, nc):
    if codec == "minmax":
        return torch.full((n,), 255, dtype=torch.uint8, device="cuda"), torch.full((2 * nc,), float("nan"), device="cuda")
    return torch.full(((n + 31) // 32,), -1, dtype=torch.int32, device="cuda"), torch.full((nc,), float("nan"), device="cuda")


CASES = [(256, 2047 * 256), (256, 2047 * 256 + 1), (256, 2049 * 256), (1024, 3071 * 1024 - 5), (1280, 2048 * 1280), (1280, 2303 * 1280 + 700),
         (4352, 2048 * 4352), (4352, 2079 * 4352 + 3)]


@pytest.mark.parametrize("codec", ["minmax", "sign"])
@pytest.mark.parametrize("chunk,n", CASES)
def test_worker_side(bg, oracle, codec, chunk, n):
    print("order %s C=%d n=%d" % (codec, chunk, n), flush=True)
    nc = bg.num_chunks(n, chunk)
    xs = [draw("normal", n, 31 * chunk + j, "cpu", 1e-3) for j in range(2)]
    res = draw("normal", n, 31 * chunk + 9, "cpu", 1e-4)
    plain, fused, reduce_, gather, batched, want_reduce = (
        (bg.bagua_compress_minmax_u8, oracle.compress_minmax_u8, bg.bagua_reduce_compress_minmax_u8, bg.bagua_flatten_compress_minmax_u8,
         bg.bagua_compress_minmax_u8_batched, oracle.reduce_compress_minmax_u8) if codec == "minmax" else
        (bg.bagua_sign_compress_ef, oracle.sign_compress_ef, bg.bagua_reduce_compress_sign_ef, bg.bagua_flatten_sign_compress_ef,
         bg.bagua_sign_compress_ef_batched, oracle.reduce_compress_sign))
    xg = [x.cuda() for x in xs]
    want_r = res.numpy().copy()
    want = fused(xs[0].numpy(), want_r, chunk)

    codes, meta = room(codec, n, nc)
    r = res.cuda()
    plain(xg[0], r, chunk, codes, meta)
    assert same(codes, want[0]) and same(meta, want[1]) and same(r, want_r)

    codes, meta = room(codec, n, nc)
    r = res.cuda()
    ws = torch.empty(bg.bagua_flatten_workspace_bytes(1, n), dtype=torch.uint8, device="cuda")
    bg.bagua_flatten_plan([xg[0]], [0], n, ws)
    gather(ws, 1, r, n, chunk, codes, meta)
    assert same(codes, want[0]) and same(meta, want[1]) and same(r, want_r)

    codes, meta = room(codec, n, nc)
    r = res.cuda()
    cut = nc // 3 * chunk                                   # two buckets; a bucket's codes start at a whole chunk
    at = cut if codec == "minmax" else cut // 32
    mat = 2 * cut // chunk if codec == "minmax" else cut // chunk
    ws = torch.empty(bg.bagua_batch_workspace_bytes(2, 0), dtype=torch.uint8, device="cuda")
    batched([xg[0][:cut], xg[0][cut:]], [r[:cut], r[cut:]], chunk, [codes[:at], codes[at:]], [meta[:mat], meta[mat:]], ws)
    assert same(codes, want[0]) and same(meta, want[1]) and same(r, want_r)

    want_r = res.numpy().copy()
    want = want_reduce([x.numpy() for x in xs], want_r, chunk)
    codes, meta = room(codec, n, nc)
    r = res.cuda()
    reduce_(xg, r, chunk, codes, meta)
    assert same(codes, want[0]) and same(meta, want[1]) and same(r, want_r)


@pytest.mark.parametrize("k,chunk,n", [(2, 256, 2047 * 256 + 1), (3, 1024, 3071 * 1024 - 5), (4, 1280, 2303 * 1280 + 700), (2, 4352, 2079 * 4352 + 3),
                                       (5, 4608, 2051 * 4608 + 300), (2, 8448, 2053 * 8448 + 8)])
def test_ring(bg, oracle, k, chunk, n):
    print("order ring k=%d C=%d n=%d" % (k, chunk, n), flush=True)
    nc = bg.num_chunks(n, chunk)
    xs = [draw("normal", n, 17 * chunk + j, "cpu", 0.02) for j in range(k)]
    hats = [draw("normal", n, 17 * chunk + 50 + j, "cpu", 0.02) for j in range(k)]
    hg, out = [h.cuda() for h in hats], [torch.full((n,), float("nan"), device="cuda") for _ in range(k)]
    wire = [room("minmax", n, nc) for _ in range(k)]
    bg.bagua_decentralized_avg(bg.AVG_LP_MINMAX_U8, [x.cuda() for x in xs], out, hg, [w[0] for w in wire], [w[1] for w in wire], chunk)
    want_hat = [h.numpy().copy() for h in hats]
    want_out, want_codes, want_mm = oracle.ring_avg_lp([x.numpy() for x in xs], want_hat, chunk)
    for j in range(k):
        assert same(out[j], want_out[j]) and same(hg[j], want_hat[j]) and same(wire[j][0], want_codes[j]) and same(wire[j][1], want_mm[j])


@pytest.mark.parametrize("chunk,n", [(256, 2047 * 256 + 1), (1024, 3071 * 1024 - 5), (1280, 2303 * 1280 + 700), (4352, 2079 * 4352 + 3)])
def test_topk(bg, oracle, chunk, n):
    print("order topk C=%d n=%d" % (chunk, n), flush=True)
    keep, nc = chunk // 32, bg.num_chunks(n, chunk)
    x, res = draw("normal", n, 7 * chunk, "cpu", 1e-3), draw("normal", n, 7 * chunk + 1, "cpu", 1e-4)
    idx, val, r = torch.full((nc * keep,), -1, dtype=torch.int16, device="cuda"), torch.full((nc * keep,), float("nan"), device="cuda"), res.cuda()
    bg.bagua_compress_topk_ef(x.cuda(), r, chunk, keep, idx, val)
    want_r = res.numpy().copy()
    want_idx, want_val = oracle.compress_topk(x.numpy(), want_r, chunk, keep)
    assert same(idx, want_idx) and same(val, want_val) and same(r, want_r)


@pytest.mark.parametrize("chunk,n", [(4352, 2047 * 4352), (4352, 2079 * 4352 + 3), (8448, 2053 * 8448 + 8)])
def test_peers(bg, oracle, chunk, n):
    print("order peers C=%d n=%d" % (chunk, n), flush=True)
    peer, nc = [1, 0, 2], bg.num_chunks(n, chunk)
    xs = [draw("normal", n, 13 * chunk + j, "cpu", 0.02) for j in range(3)]
    hats = [draw("normal", n, 13 * chunk + 50 + j, "cpu", 0.02) for j in range(3)]
    hg, out = [h.cuda() for h in hats], [torch.full((n,), float("nan"), device="cuda") for _ in range(3)]
    wire = [room("minmax", n, nc) for _ in range(3)]
    bg.bagua_decentralized_avg_peers_lp([x.cuda() for x in xs], out, hg, [w[0] for w in wire], [w[1] for w in wire], peer, chunk)
    want_hat = [h.numpy().copy() for h in hats]
    want_out, want_codes, want_mm = oracle.peer_avg_lp([x.numpy() for x in xs], want_hat, peer, chunk)
    for j in range(3):
        assert same(out[j], want_out[j]) and same(hg[j], want_hat[j]) and same(wire[j][0], want_codes[j]) and same(wire[j][1], want_mm[j])


@pytest.mark.parametrize("chunk,n", [(256, 8193), (512, 512 * 8 - 1), (512, 512 * 8), (512, 512 * 17 + 300), (768, 768 * 33 + 5), (1024, 1024 * 40), (4096, 4096 * 23 + 256), (16384, 16384 * 19 - 1),
                                     (2048, 1 << 25), (2048, (1 << 25) + 1)])
def test_share_of_a_ring(bg, oracle, chunk, n):
    """Encode + mix of peer 1 of three; the rows are mixed in the order of the encode up to 2^25 elements."""
    print("order share C=%d n=%d" % (chunk, n), flush=True)
    xs = [draw("normal", n, 19 * chunk + j, "cpu", 0.02) for j in range(3)]
    hats = [draw("normal", n, 19 * chunk + 50 + j, "cpu", 0.02) for j in range(3)]
    want_hat = [h.numpy().copy() for h in hats]
    want_out, want_codes, want_mm = oracle.ring_avg_lp([x.numpy() for x in xs], want_hat, chunk)
    hg, out, x = [h.cuda() for h in hats], torch.full((n,), float("nan"), device="cuda"), xs[1].cuda()
    codes, mm = room("minmax", n, bg.num_chunks(n, chunk))
    bg.bagua_lp_encode(x, hg[1], chunk, codes, mm)
    assert same(codes, want_codes[1]) and same(mm, want_mm[1]) and same(hg[1], want_hat[1])
    sent = [(torch.from_numpy(want_codes[j]).cuda(), torch.from_numpy(want_mm[j]).cuda()) for j in (0, 2)]
    bg.bagua_lp_apply_mix(x, hg[1], hg[0], hg[2], *sent[0], *sent[1], chunk, out)
    assert same(out, want_out[1]) and same(hg[0], want_hat[0]) and same(hg[2], want_hat[2])


@pytest.mark.parametrize("codec", ["minmax", "sign"])
@pytest.mark.parametrize("chunk,n", [(256, 8193), (512, 512 * 8 - 1), (512, 512 * 17 + 300), (768, 768 * 33 + 5), (4096, 4096 * 23 + 256), (16384, 16384 * 19 - 1), (2048, 1 << 24),
                                     (2048, (1 << 24) + 1)])
def test_optimizer_steps(bg, oracle, codec, chunk, n):
    """The rows are updated in the order of the chunks up to 2^24 elements."""
    print("order steps %s C=%d n=%d" % (codec, chunk, n), flush=True)
    codes, meta = (oracle.compress_minmax_u8 if codec == "minmax" else oracle.sign_compress_ef)(draw("normal", n, 23 * chunk, "cpu", 1e-3).numpy(), None, chunk)
    cid = bg.CODEC_MINMAX_U8 if codec == "minmax" else bg.CODEC_SIGN1
    cg, mg = torch.from_numpy(codes.view(np.uint8 if codec == "minmax" else np.int32)).cuda(), torch.from_numpy(meta).cuda()
    p, m = draw("normal", n, 23 * chunk + 1, "cpu", 0.02), draw("normal", n, 23 * chunk + 2, "cpu", 1e-3)
    v = m * m + 1e-8
    pg, mo = p.cuda(), m.cuda()
    bg.bagua_decompress_sgd_step(cid, cg, mg, n, chunk, pg, mo, 1e-3, momentum=0.9, weight_decay=1e-4)
    want_p, want_m = p.numpy().copy(), m.numpy().copy()
    oracle.decompress_sgd_step(cid, codes, meta, n, chunk, want_p, want_m, 1e-3, momentum=0.9, weight_decay=1e-4)
    assert same(pg, want_p) and same(mo, want_m)
    pg, mo, vg = p.cuda(), m.cuda(), v.cuda()
    bg.bagua_decompress_adam_step(cid, cg, mg, n, chunk, pg, mo, vg, 1e-4, variance_frozen=True)
    want_p, want_m, want_v = p.numpy().copy(), m.numpy().copy(), v.numpy().copy()
    oracle.decompress_adam_step(cid, codes, meta, n, chunk, want_p, want_m, want_v, 1e-4, variance_frozen=True)
    assert same(pg, want_p) and same(mo, want_m) and same(vg, want_v)


@pytest.mark.parametrize("codec", ["minmax", "sign"])
@pytest.mark.parametrize("k_local", [2, 3])
@pytest.mark.parametrize("n", [1 << 25, (1 << 25) + 300])
def test_average_of_short_chunks(bg, oracle, codec, k_local, n):
    """Either side of the size from which three and more in a node keep the plain order."""
    print("order average %s k=%d n=%d" % (codec, k_local, n), flush=True)
    xs, res = [draw("normal", n, 41 + j, "cpu", 1e-3) for j in range(k_local)], draw("normal", n, 40, "cpu", 1e-4)
    call, want_of = ((bg.bagua_reduce_compress_minmax_u8, oracle.reduce_compress_minmax_u8) if codec == "minmax" else
                     (bg.bagua_reduce_compress_sign_ef, oracle.reduce_compress_sign))
    codes, meta = room(codec, n, bg.num_chunks(n, 512))
    r, want_r = res.cuda(), res.numpy().copy()
    call([x.cuda() for x in xs], r, 512, codes, meta)
    want = want_of([x.numpy() for x in xs], want_r, 512)
    assert same(codes, want[0]) and same(meta, want[1]) and same(r, want_r)


@pytest.mark.parametrize("n", [1 << 26, (1 << 26) + 4])
def test_gather_of_short_chunks(bg, oracle, n):
    print("order gather n=%d" % n, flush=True)
    x, res = draw("normal", n, 51, "cpu", 1e-3), draw("normal", n, 52, "cpu", 1e-4)
    codes, meta = room("minmax", n, bg.num_chunks(n, 512))
    r, want_r, xg = res.cuda(), res.numpy().copy(), x.cuda()
    ws = torch.empty(bg.bagua_flatten_workspace_bytes(2, n), dtype=torch.uint8, device="cuda")
    bg.bagua_flatten_plan([xg[:1000], xg[1000:]], [0, 1000], n, ws)
    bg.bagua_flatten_compress_minmax_u8(ws, 2, r, n, 512, codes, meta)
    want = oracle.compress_minmax_u8(x.numpy(), want_r, 512)
    assert same(codes, want[0]) and same(meta, want[1]) and same(r, want_r)
