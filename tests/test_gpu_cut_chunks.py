"""The chunk of a bucket that is cut short has a path of its own in short launches (one access per lane, the lane on the edge shifted): every
remainder around the width of an access and of a row, chunks that a wave's rows divide and do not, and the lines between the forms of
a launch, against the oracle, bit for bit.  The outputs lie between words that the call must not touch."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

# (chunk, length): lengths around one access (4), one row (256), a chunk and two
CUTS = [(C, m * C + r) for C, m in ((256, 0), (256, 3), (768, 2), (1536, 1), (2048, 2), (4096, 1), (8192, 1), (16384, 0), (16384, 1))
        for r in (1, 2, 3, 4, 5, 7, 63, 64, 65, 255)] + [(C, C - r) for C in (512, 2048, 4096, 8192) for r in (1, 2, 3, 4, 5, 255, 256, 257)]


@pytest.fixture(scope="module")
def bg():
    import paper_2107_01499_amd as b
    assert torch.cuda.is_available()
    return b


class Guarded:
    """A tensor with 64 words on either side that must keep their value."""

    def __init__(self, values):
        self.all = torch.full((values.size + 128,), 77, dtype=torch.from_numpy(values[:0]).dtype, device="cuda")
        self.t = self.all[64:64 + values.size]
        self.t.copy_(torch.from_numpy(values))

    def check(self, want, what):
        got = self.t.cpu().numpy()
        assert got.tobytes() == np.ascontiguousarray(want).tobytes(), what
        assert bool((self.all[:64] == 77).all()) and bool((self.all[64 + got.size:] == 77).all()), what + " (beside it)"


def vals(n, seed, sigma=1e-3):
    r = np.random.default_rng(seed)
    v = (r.standard_normal(n) * sigma).astype(np.float32)
    v[r.integers(0, n, max(1, n // 50))] = 0.0
    return v


def groups(items, size):
    return [items[i:i + size] for i in range(0, len(items), size)]


def server_minmax(bg, oracle, k, n, C, ef, out):
    enc = [oracle.compress_minmax_u8(vals(n, 3 * j + n), None, C) for j in range(k)]
    eps = vals(n, n, 1e-5)
    ci, mi = [torch.from_numpy(c).cuda() for c, _ in enc], [torch.from_numpy(m).cuda() for _, m in enc]
    e, co = Guarded(eps), Guarded(np.zeros(n, np.uint8))
    mo, o = Guarded(np.zeros(2 * bg.num_chunks(n, C), np.float32)), Guarded(np.zeros(n, np.float32))
    bg.bagua_decompress_reduce_recompress(0, ci, mi, e.t if ef else None, n, C, co.t, mo.t, o.t if out else None)
    eps_o = eps.copy() if ef else None
    cw, mw, ow = oracle.drr_minmax_u8([c for c, _ in enc], [m for _, m in enc], eps_o, C)
    what = "k=%d n=%d C=%d" % (k, n, C)
    co.check(cw, "codes " + what)
    mo.check(mw, "minmax " + what)
    if ef:
        e.check(eps_o, "eps " + what)
    if out:
        o.check(ow, "out " + what)


@pytest.mark.parametrize("cuts", groups(CUTS, 20), ids=lambda c: "%d-%d" % c[0])
@pytest.mark.parametrize("k", [1, 3, 4, 9, 32])
def test_server_step_minmax(bg, oracle, cuts, k):
    for i, (C, n) in enumerate(cuts):
        server_minmax(bg, oracle, k, n, C, ef=i % 3 != 0, out=i % 2 == 0)


@pytest.mark.parametrize("k,C,n", [
    (3, 2048, 1 << 20), (3, 2048, (1 << 20) + 1), (2, 768, (1 << 20) + 1),                         # one row per wave, two, an odd number
    (2, 4096, (1 << 22) - 77), (2, 4096, 1 << 22), (2, 4096, (1 << 22) + 77),                      # ahead, behind
    (5, 1536, (1 << 22) + 1541), (2, 8192, (1 << 22) + 5), (2, 16384, (1 << 20) + 3), (5, 2048, (1 << 25) + 2047),
    (3, 16384, 1 << 18), (3, 16384, (1 << 18) + 5), (2, 12288, (1 << 21) - 1), (2, 16384, (1 << 21) + 1), (2, 9216, 500001),
    (2, 16384, (1 << 26) + 1), (2, 1536, (1 << 26) + 2),                                           # the last with a body for the cut
])
def test_server_step_minmax_either_side_of_its_lines(bg, oracle, k, C, n):
    server_minmax(bg, oracle, k, n, C, ef=True, out=False)


@pytest.mark.parametrize("C,ns", [(2048, [3, 2048 * 5 + 1, 700001, 2]), (4096, [5, 4096, 4099, 12345]), (1536, [1536 * 3 + 4, 4, 9001]),
                                  (8192, [2000003, 2500001]), (4096, [1, 3000001])])
def test_server_step_minmax_batched(bg, oracle, C, ns):
    k = 3
    enc = [[oracle.compress_minmax_u8(vals(n, 3 * j + n), None, C) for j in range(k)] for n in ns]
    eps = [vals(n, n, 1e-5) for n in ns]
    e, co = [Guarded(v) for v in eps], [Guarded(np.zeros(n, np.uint8)) for n in ns]
    mo = [Guarded(np.zeros(2 * bg.num_chunks(n, C), np.float32)) for n in ns]
    ws = torch.empty(bg.bagua_batch_workspace_bytes(len(ns), k), dtype=torch.uint8, device="cuda")
    bg.bagua_decompress_reduce_recompress_batched(
        0, [[torch.from_numpy(c).cuda() for c, _ in b] for b in enc], [[torch.from_numpy(m).cuda() for _, m in b] for b in enc],
        [g.t for g in e], ns, C, [g.t for g in co], [g.t for g in mo], None, ws)
    for b in range(len(ns)):
        cw, mw, _ = oracle.drr_minmax_u8([c for c, _ in enc[b]], [m for _, m in enc[b]], eps[b], C)
        co[b].check(cw, "codes %d" % b)
        mo[b].check(mw, "minmax %d" % b)
        e[b].check(eps[b], "eps %d" % b)


def replicas(k, n, seed):
    base = vals(n, seed, 0.02)
    return [base + vals(n, seed + 1 + j) for j in range(k)], [base + vals(n, seed + 50 + j, 1e-4) for j in range(k)]


def ring_low_precision(bg, oracle, k, n, C, peer=None):
    x, hat = replicas(k, n, n + k)
    hat_o = [h.copy() for h in hat]
    hg, og = [Guarded(h) for h in hat], [Guarded(np.zeros(n, np.float32)) for _ in range(k)]
    cg, mg = [Guarded(np.zeros(n, np.uint8)) for _ in range(k)], [Guarded(np.zeros(2 * bg.num_chunks(n, C), np.float32)) for _ in range(k)]
    lists = [torch.from_numpy(v).cuda() for v in x], [g.t for g in og], [g.t for g in hg], [g.t for g in cg], [g.t for g in mg]
    if peer is None:
        bg.bagua_decentralized_avg(bg.AVG_LP_MINMAX_U8, *lists, C)
        want = oracle.ring_avg_lp(x, hat_o, C)
    else:
        bg.bagua_decentralized_avg_peers_lp(*lists, peer, C)
        want = oracle.peer_avg_lp(x, hat_o, peer, C)
    for i in range(k):
        what = " %d k=%d n=%d C=%d" % (i, k, n, C)
        og[i].check(want[0][i], "out" + what)
        hg[i].check(hat_o[i], "hat" + what)
        cg[i].check(want[1][i], "codes" + what)
        mg[i].check(want[2][i], "minmax" + what)


@pytest.mark.parametrize("cuts", groups(CUTS, 20), ids=lambda c: "%d-%d" % c[0])
@pytest.mark.parametrize("k,peer", [(5, None), (16, None), (2, [1, 0]), (5, [1, 0, 2, 4, 3]), (4, [1, 2, 3, 0])])   # two launches; gossip, one way
def test_rounds_in_low_precision(bg, oracle, cuts, k, peer):
    for C, n in cuts[::2 if k < 16 else 5]:
        ring_low_precision(bg, oracle, k, n, C, peer)


@pytest.mark.parametrize("k,C,n,peer", [
    (25, 4096, 24 * 24 * 1024, None), (25, 4096, 24 * 24 * 1024 + 1, None), (17, 1024, 16 * 24 * 1024 + 1, None), (25, 4352, (5 << 17) + 1, None), (5, 4096, 5 * 24 * 1024, None), (5, 4096, 5 * 24 * 1024 + 1, None), (8, 1536, 8 * 24 * 1024 - 3, None), (4, 4096, 65537, None),
    (32, 8192, 100001, None), (6, 16384, 6 * 80 * 1024 - 1, None), (6, 16384, 6 * 80 * 1024 + 1, None), (6, 6400, 120003, None),
    (2, 4096, (1 << 21) + 1, [1, 0]), (3, 4096, (1 << 21) + 1, [1, 0, 2]), (3, 2048, (1 << 23) + 5, [1, 0, 2]), (3, 16384, 1 << 21, [0, 2, 1]),
    (3, 4096, 300001, [0, 1, 2]), (2, 16384, 5 << 18, None), (2, 16384, (5 << 18) + 1, None), (3, 8192, (3 << 16) + 1, None), (16, 8192, 3 << 18, None),
    (2, 16384, 1 << 18, [1, 0]), (2, 16384, (1 << 18) + 1, [1, 0]), (7, 12544, 70001, [1, 0, 2, 4, 3, 6, 5]), (3, 16384, 3, [1, 0, 2]), (3, 16384, 1 << 18, None), (3, 16384, (1 << 18) + 1, None), (1, 16384, 1 << 18, None), (1, 16384, (1 << 18) + 1, None), (1, 12800, 70001, None), (3, 16384, 2, None), (4, 16384, 21 << 20, None), (4, 12800, (20 << 20) + 1, None)])
def test_rounds_in_low_precision_either_side_of_their_lines(bg, oracle, k, C, n, peer):
    ring_low_precision(bg, oracle, k, n, C, peer)


@pytest.mark.parametrize("n,C", [(1, 256), (3, 256), (4, 256), (4097, 4096), (70001, 8192), ((1 << 23) - 1, 4096), ((1 << 23) + 1, 2048)])
def test_encode_of_one_peer(bg, oracle, n, C):
    x, hat = replicas(1, n, n)
    h, c = Guarded(hat[0]), Guarded(np.zeros(n, np.uint8))
    m = Guarded(np.zeros(2 * bg.num_chunks(n, C), np.float32))
    bg.bagua_lp_encode(torch.from_numpy(x[0]).cuda(), h.t, C, c.t, m.t)
    _, cw, mw = oracle.ring_avg_lp(x, hat, C)
    c.check(cw[0], "codes")
    m.check(mw[0], "minmax")
    h.check(hat[0], "hat")


def worker_side(bg, oracle, n, C, k_local, ef):
    """Every worker-side call on the same values: compress, momentum, intra-node average and gather, both codecs."""
    xs, mom, res = [vals(n, n + j) for j in range(k_local)], vals(n, n + 40), vals(n, n + 41, 1e-5)
    xg, mg = [torch.from_numpy(x).cuda() for x in xs], torch.from_numpy(mom).cuda()
    ws = torch.empty(bg.bagua_flatten_workspace_bytes(2, n), dtype=torch.uint8, device="cuda")
    cut = n // 3
    bg.bagua_flatten_plan([xg[0][:cut], xg[0][cut:]], [0, cut], n, ws)
    nc = bg.num_chunks(n, C)
    minmax = [(lambda r, c, m: bg.bagua_compress_minmax_u8(xg[0], r, C, c, m), lambda r: oracle.compress_minmax_u8(xs[0], r, C)),
              (lambda r, c, m: bg.bagua_reduce_compress_minmax_u8(xg, r, C, c, m), lambda r: oracle.reduce_compress_minmax_u8(xs, r, C)),
              (lambda r, c, m: bg.bagua_flatten_compress_minmax_u8(ws, 2, r, n, C, c, m), lambda r: oracle.compress_minmax_u8(xs[0], r, C))]
    sign = [(lambda r, c, m: bg.bagua_sign_compress_ef(xg[0], r, C, c, m), lambda r: oracle.sign_compress_ef(xs[0], r, C)),
            (lambda r, c, m: bg.bagua_momentum_sign_compress_ef(xg[0], mg, 0.9, r, C, c, m),
             lambda r: oracle.momentum_sign_compress_ef(xs[0], mom, 0.9, r, C)),
            (lambda r, c, m: bg.bagua_reduce_compress_sign_ef(xg, r, C, c, m), lambda r: oracle.reduce_compress_sign(xs, r, C)),
            (lambda r, c, m: bg.bagua_flatten_sign_compress_ef(ws, 2, r, n, C, c, m), lambda r: oracle.sign_compress_ef(xs[0], r, C))]
    for i, (run, want) in enumerate(minmax + sign):
        what = "call %d n=%d C=%d" % (i, n, C)
        r, ro = Guarded(res), res.copy() if ef else None
        codes = Guarded(np.zeros(n, np.uint8) if i < 3 else np.zeros((n + 31) // 32, np.int32))
        meta = Guarded(np.zeros(2 * nc if i < 3 else nc, np.float32))
        run(r.t if ef else None, codes.t, meta.t)
        cw, mw = want(ro)
        codes.check(cw, "codes " + what)
        meta.check(mw, "meta " + what)
        if ef:
            r.check(ro, "residual " + what)


@pytest.mark.parametrize("cuts", groups(CUTS, 10), ids=lambda c: "%d-%d" % c[0])
@pytest.mark.parametrize("k_local", [1, 3, 9])
def test_worker_side(bg, oracle, cuts, k_local):
    for i, (C, n) in enumerate(cuts):
        worker_side(bg, oracle, n, C, k_local, ef=i % 3 != 0)


@pytest.mark.parametrize("n,C,k_local", [((1 << 20) - 1, 4096, 2), (1 << 20, 768, 5), ((1 << 20) + 1, 4096, 5), ((1 << 20) - 3, 8192, 9),
                                         ((1 << 20) + 3, 16384, 2), (1 << 21, 4096, 1), ((1 << 21) + 1, 1024, 1), ((1 << 25) - 5, 4096, 1)])
def test_worker_side_either_side_of_its_lines(bg, oracle, n, C, k_local):
    worker_side(bg, oracle, n, C, k_local, ef=True)


@pytest.mark.parametrize("C", [1024, 4096])
def test_compressions_batched(bg, oracle, C):
    ns = [1, 3, 4, 5, C - 1, C + 1, 3 * C + 257, 70001]
    xs, res = [vals(n, n) for n in ns], [vals(n, n + 1, 1e-5) for n in ns]
    ws = torch.empty(bg.bagua_batch_workspace_bytes(len(ns), 0), dtype=torch.uint8, device="cuda")
    for call, width, dtype, per, want in ((bg.bagua_compress_minmax_u8_batched, lambda n: n, np.uint8, 2, oracle.compress_minmax_u8),
                                          (bg.bagua_sign_compress_ef_batched, lambda n: (n + 31) // 32, np.int32, 1, oracle.sign_compress_ef)):
        r, codes = [Guarded(v) for v in res], [Guarded(np.zeros(width(n), dtype)) for n in ns]
        meta = [Guarded(np.zeros(per * bg.num_chunks(n, C), np.float32)) for n in ns]
        call([torch.from_numpy(x).cuda() for x in xs], [g.t for g in r], C, [g.t for g in codes], [g.t for g in meta], ws)
        for b, n in enumerate(ns):
            ro = res[b].copy()
            cw, mw = want(xs[b], ro, C)
            codes[b].check(cw, "codes n=%d" % n)
            meta[b].check(mw, "meta n=%d" % n)
            r[b].check(ro, "residual n=%d" % n)


# keep below, at and above the threads of a workgroup; a chunk cut short; early and late entries; chunks in parts and whole
@pytest.mark.parametrize("n,C,keep", [(3, 256, 1), (5001, 1024, 7), (70001, 1024, 256), (70001, 1024, 257), (40001, 2048, 2048), (300001, 16384, 1500), (20001, 5376, 100), (12801, 12800, 12800),
                                      (1 << 20, 4096, 128), ((1 << 20) + 1, 4096, 600), ((5 << 20) + 3, 4096, 513), ((1 << 26) + 5, 8192, 3),
                                      ((1 << 20) + 1, 8192, 1500), (1 << 21, 8192, 1024), ((1 << 21) + 1, 8192, 300), ((1 << 20) + 1, 16384, 1500), (10 << 20, 8192, 513), ((10 << 20) + 1, 8192, 300),
                                      (352 * 16384, 16384, 600), (352 * 16384 + 1, 16384, 600), (288 * 14336 + 7, 14336, 3585), (512 * 16384 - 255, 16384, 1025), (512 * 16384 + 1, 16384, 1025),
                                      (426 * 9216, 9216, 300), (768 * 9216 - 1, 9216, 577), (341 * 12288 + 4, 12288, 100)])
@pytest.mark.parametrize("opt", ["sgd", "adam"])
def test_optimizer_steps_after_topk(bg, oracle, n, C, keep, opt):
    optimizer_step_after_topk(bg, oracle, n, C, keep, opt, momentum=True, weight_decay=1e-4 if opt == "sgd" else 0.0, lr=1e-3 if opt == "sgd" else 1e-4)


# The other forms of the step: late entries in parts, whole chunks of two and of four rows per wave
@pytest.mark.parametrize("n,C,keep", [((1 << 21) + 1, 8192, 300), ((1 << 20) + 1, 8192, 300), (353 * 16384, 16384, 600)])
@pytest.mark.parametrize("form", [("sgd", True, 0.0, 1e-3), ("sgd", False, 1e-4, 1e-3), ("sgd", False, 0.0, -1e-3), ("adam", False, 1e-2, 1e-4), ("adam", True, 0.0, 1e-4),
                                  ("adam", True, 1e-2, 1e-4)], ids=["mom", "wd", "neither", "adam-wd", "frozen", "frozen-wd"])
def test_forms_of_the_optimizer_step_after_topk(bg, oracle, n, C, keep, form):
    opt, flag, wd, lr = form
    optimizer_step_after_topk(bg, oracle, n, C, keep, opt, momentum=flag, weight_decay=wd, lr=lr, frozen=opt == "adam" and flag)


def optimizer_step_after_topk(bg, oracle, n, C, keep, opt, momentum, weight_decay, lr, frozen=False):
    idx, val = oracle.compress_topk(vals(n, n), None, C, keep)
    param, m, v = vals(n, 1, 0.02), vals(n, 2), np.square(vals(n, 3)) + np.float32(1e-8)
    gp, gm, gv = Guarded(param), Guarded(m), Guarded(v)
    gi, gx = torch.from_numpy(idx.view(np.int16)).cuda(), torch.from_numpy(val).cuda()
    if opt == "sgd":
        mu = 0.9 if momentum else 0.0
        bg.bagua_decompress_sgd_step_topk(gi, gx, n, C, keep, gp.t, gm.t if momentum else None, lr, momentum=mu, weight_decay=weight_decay)
        oracle.decompress_sgd_step_topk(idx, val, n, C, keep, param, m if momentum else None, lr, mu, weight_decay)
    else:
        bg.bagua_decompress_adam_step_topk(gi, gx, n, C, keep, gp.t, gm.t, gv.t, lr, weight_decay=weight_decay, variance_frozen=frozen)
        oracle.decompress_adam_step_topk(idx, val, n, C, keep, param, m, v, lr, weight_decay=weight_decay, variance_frozen=frozen)
        gv.check(v, "v")
    gp.check(param, "param")
    gm.check(m, "m")


def server_sign(bg, oracle, k, n, C, ef, out):
    enc = [oracle.sign_compress_ef(vals(n, 3 * j + n), None, C) for j in range(k)]
    eps, nw = vals(n, n, 1e-5), (n + 31) // 32
    ci, mi = [torch.from_numpy(b.view(np.int32)).cuda() for b, _ in enc], [torch.from_numpy(s).cuda() for _, s in enc]
    e, co = Guarded(eps), Guarded(np.zeros(nw, np.int32))
    mo, o = Guarded(np.zeros(bg.num_chunks(n, C), np.float32)), Guarded(np.zeros(n, np.float32))
    bg.bagua_decompress_reduce_recompress(1, ci, mi, e.t if ef else None, n, C, co.t, mo.t, o.t if out else None)
    eps_o = eps.copy() if ef else None
    cw, mw, ow = oracle.drr_sign([b for b, _ in enc], [s for _, s in enc], eps_o, n, C)
    what = "k=%d n=%d C=%d" % (k, n, C)
    co.check(cw, "bits " + what)
    mo.check(mw, "scale " + what)
    if ef:
        e.check(eps_o, "eps " + what)
    if out:
        o.check(ow, "out " + what)


@pytest.mark.parametrize("k", list(range(1, 18)) + [23, 31, 32])   # whole groups of eight workers and every rest
def test_server_step_sign(bg, oracle, k):
    for i, (n, C) in enumerate([(1, 256), (300, 256), (5000, 2048), (12289, 4096), (70001, 8192), (70001, 16384), (9001, 1536)]):
        server_sign(bg, oracle, k, n, C, ef=i % 3 != 0, out=i % 2 == 0)


# Either side of the launches whose rest of workers comes one by one, and one worker.
@pytest.mark.parametrize("k,C,n", [(1, 2048, 5000), (3, 512, 1 << 21), (3, 512, (1 << 21) + 512), (9, 1024, (1 << 22) - 5), (14, 1024, 1 << 22), (2, 1024, (1 << 22) + 1),
                                   (5, 4096, 2880000), (5, 4096, 2885632), (6, 4096, 3 << 20), (11, 3072, 3 << 20), (2, 4096, (1 << 22) + 4096)])
def test_server_step_sign_either_side_of_its_lines(bg, oracle, k, C, n):
    server_sign(bg, oracle, k, n, C, ef=True, out=k % 2 == 0)


@pytest.mark.parametrize("k", [3, 7, 8])
def test_server_step_sign_batched(bg, oracle, k):
    C, ns = 2048, [1, 2048, 2049, 70001, 300]
    enc = [[oracle.sign_compress_ef(vals(n, 3 * j + n), None, C) for j in range(k)] for n in ns]
    eps = [vals(n, n, 1e-5) for n in ns]
    e, co = [Guarded(v) for v in eps], [Guarded(np.zeros((n + 31) // 32, np.int32)) for n in ns]
    mo, o = [Guarded(np.zeros(bg.num_chunks(n, C), np.float32)) for n in ns], [Guarded(np.zeros(n, np.float32)) for n in ns]
    ws = torch.empty(bg.bagua_batch_workspace_bytes(len(ns), k), dtype=torch.uint8, device="cuda")
    bg.bagua_decompress_reduce_recompress_batched(
        1, [[torch.from_numpy(b.view(np.int32)).cuda() for b, _ in w] for w in enc], [[torch.from_numpy(s).cuda() for _, s in w] for w in enc],
        [g.t for g in e], ns, C, [g.t for g in co], [g.t for g in mo], [g.t for g in o], ws)
    for b, n in enumerate(ns):
        cw, mw, ow = oracle.drr_sign([w for w, _ in enc[b]], [s for _, s in enc[b]], eps[b], n, C)
        co[b].check(cw, "bits %d" % b)
        mo[b].check(mw, "scale %d" % b)
        e[b].check(eps[b], "eps %d" % b)
        o[b].check(ow, "out %d" % b)


@pytest.mark.parametrize("n,C,keep", [((1 << 23) + 77, 1024, 32), ((1 << 23) + 1, 1536, 1), ((1 << 23) + 255, 768, 768), ((1 << 23) + 3, 256, 100), (1 << 23, 1024, 9)])
@pytest.mark.parametrize("ef", [True, False])
def test_topk_compression_either_side_of_its_joint_stores(bg, oracle, n, C, keep, ef):
    x, res = vals(n, n), vals(n, n + 1)
    r, slots = Guarded(res), bg.num_chunks(n, C) * keep
    idx, val = Guarded(np.zeros(slots, np.int16)), Guarded(np.zeros(slots, np.float32))
    bg.bagua_compress_topk_ef(torch.from_numpy(x).cuda(), r.t if ef else None, C, keep, idx.t, val.t)
    iw, vw = oracle.compress_topk(x, res if ef else None, C, keep)
    idx.check(iw.view(np.int16), "idx")
    val.check(vw, "val")
    r.check(res, "residual")
