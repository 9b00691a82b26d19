"""The chunk statistics, whose lanes and waves meet through data-parallel primitives: the extreme of a chunk is moved
over every lane, every element of a lane and every wave, so that no exchange between them can be missing."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def bg():
    import paper_2107_01499_amd as b
    assert torch.cuda.is_available()
    return b


def same(t, want):
    return np.array_equal(t.cpu().numpy().view(np.uint8), want.view(np.uint8))


def _chunks(chunk, count):
    """One chunk per extreme: chunk i holds its largest value at one position and its smallest at another."""
    x = torch.empty(count * chunk).uniform_(-1.0, 1.0, generator=torch.Generator().manual_seed(chunk))
    i = torch.arange(count)
    x[i * chunk + i * 257 % chunk] = 2.0 + i / 64.0            # 257: next row, next element
    x[i * chunk + (i * 257 + 131) % chunk] = -2.0 - i / 64.0
    return x


@pytest.mark.parametrize("chunk", [256, 512, 768, 1536, 2048, 4096, 5376, 8192, 16384])
def test_extreme_in_every_lane_and_wave(bg, oracle, chunk):
    count = 320
    x = _chunks(chunk, count)[:count * chunk - 3]              # the last chunk is cut short
    n = x.numel()
    want_r = np.zeros(n, np.float32)
    want_codes, want_mm = oracle.compress_minmax_u8(x.numpy(), want_r, chunk)
    codes, mm, res = torch.zeros(n, dtype=torch.uint8, device="cuda"), torch.zeros(2 * count, device="cuda"), torch.zeros(n, device="cuda")
    bg.bagua_compress_minmax_u8(x.cuda(), res, chunk, codes, mm)
    assert same(mm, want_mm) and same(codes, want_codes) and same(res, want_r)
    want_r = np.zeros(n, np.float32)
    want_bits, want_scale = oracle.sign_compress_ef(x.numpy(), want_r, chunk)
    bits, scale, res = torch.zeros((n + 31) // 32, dtype=torch.int32, device="cuda"), torch.zeros(count, device="cuda"), torch.zeros(n, device="cuda")
    bg.bagua_sign_compress_ef(x.cuda(), res, chunk, bits, scale)
    assert same(scale, want_scale) and same(bits, want_bits) and same(res, want_r)
