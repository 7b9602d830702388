"""GPU parity of the encoder's choices by launch size: up to 512 chunks the
analysis runs 1024 threads a chunk and the packer starts several waves on one
lane group from the analysis' sums; beyond, 512 and 256 threads (and staging
slots for launches with an XOR base).  The counting pass reduces its counters
every 2 MiB of a chunk.  Containers equal the oracle's byte for byte."""
import numpy as np
import pytest
import torch

import oracle
from paper_2411_05239_amd import zipnn as Z

pytestmark = pytest.mark.gpu

TORCH = {Z.ZIPNN_BF16: torch.bfloat16, Z.ZIPNN_FP32: torch.float32, Z.ZIPNN_U8: torch.uint8}


@pytest.fixture(scope="module")
def codec():
    c = Z.Codec(0)
    yield c
    c.close()


def _check(codec, dt, raw, p, base=None):
    """raw, base: uint8 arrays of whole words"""
    x = torch.from_numpy(raw.copy()).view(TORCH[dt]).cuda()
    b = torch.from_numpy(base.copy()).view(TORCH[dt]).cuda() if base is not None else None
    c = codec.compress(x, p, base=b)
    ref = oracle.compress(raw, dt, base=base, chunk_bytes=p.chunk_bytes, S=p.substream_syms, g=p.group,
                          L=p.max_code_len, policy=list(p.policy), skip=p.probe_skip, exp=bool(p.exponent))
    assert np.array_equal(c.cpu().numpy(), ref)
    out = torch.empty_like(x)
    codec.decompress(c, out, base=b)
    assert torch.equal(out.view(torch.uint8), x.view(torch.uint8))


def _words(rng, n, B):
    """an exponent-like, a delta-like and spread byte groups"""
    raw = rng.integers(0, 256, (n, B), dtype=np.uint8)
    raw[:, B - 1] = rng.choice(np.array([60, 61, 62, 63, 188, 189, 190, 64], np.uint8), n,
                               p=[.3, .2, .15, .1, .1, .08, .05, .02])
    if B > 1:
        raw[:, 0] = np.where(rng.random(n) < 0.85, 0, raw[:, 0])
    return raw.reshape(-1)


@pytest.mark.parametrize("delta", [False, True])
@pytest.mark.parametrize("dt,S,g", [(Z.ZIPNN_BF16, 32, 4), (Z.ZIPNN_BF16, 128, 2), (Z.ZIPNN_FP32, 16, 8),
                                    (Z.ZIPNN_U8, 64, 8)])
@pytest.mark.parametrize("extra", [0, 1])
def test_few_and_many_chunks(codec, dt, S, g, extra, delta):
    """512 chunks are few, 513 (the last of one element) are many."""
    B = Z.WIDTH[dt]
    n = 512 * 4096 // B + extra
    rng = np.random.default_rng(31 * dt + S + extra)
    raw = _words(rng, n, B)
    base = None
    if delta:
        base = rng.integers(0, 256, raw.size, dtype=np.uint8)
        raw = raw ^ base
    _check(codec, dt, raw, Z.make_params(dt, chunk_bytes=4096, S=S, g=g), base)


@pytest.mark.parametrize("W,tail", [(1, 0), (8, 3), (63, 1), (64, 0), (65, 2), (192, 5), (320, 0), (960, 7), (1024, 1)])
@pytest.mark.parametrize("zg", [False, True])
def test_ranges_of_a_lane_group(codec, W, tail, zg):
    """Lane groups cut into 16 / (lane groups) ranges of steps, with partial
    lane groups, a partial last group and, for ZG, lanes whose words stay
    unfinished over several ranges."""
    S, g = 64, 4
    n = W * S - tail
    rng = np.random.default_rng(W + tail)
    raw = np.zeros((n, 2), np.uint8)
    raw[:, 1] = rng.choice(np.array([1, 2, 3, 4, 5], np.uint8), n, p=[.9, .05, .03, .01, .01])
    raw[:, 0] = np.where(rng.random(n) < 0.03, rng.integers(0, 256, n), 0)
    p = Z.make_params(Z.ZIPNN_BF16, chunk_bytes=262144, S=S, g=g,
                      policy=[Z.ZIPNN_HUF, Z.ZIPNN_ZG if zg else Z.ZIPNN_HUF])
    _check(codec, Z.ZIPNN_BF16, raw.reshape(-1), p)


@pytest.mark.parametrize("dt", [Z.ZIPNN_BF16, Z.ZIPNN_FP32, Z.ZIPNN_U8])
@pytest.mark.parametrize("value", [0, 0x5A])
def test_largest_chunk_of_almost_one_value(codec, dt, value):
    """4 MiB chunks whose bytes are all but one the same: the largest counts
    that the shared counters and the code construction meet."""
    B = Z.WIDTH[dt]
    raw = np.full((4 << 20) + 16 * B, value, np.uint8)
    raw[12345 * B:12345 * B + B] = value ^ 1
    p = Z.make_params(dt, chunk_bytes=4 << 20, S=4096, g=4, policy=[Z.ZIPNN_HUF] * B)
    _check(codec, dt, raw, p)


@pytest.mark.parametrize("n_sym", [2, 63, 64, 65, 128, 255, 256])
@pytest.mark.parametrize("L", [8, 11])
def test_alphabet_sizes(codec, n_sym, L):
    """Code construction with one and four leaves a lane, ties and steep
    counts."""
    rng = np.random.default_rng(n_sym + L)
    syms = rng.permutation(256)[:n_sym].astype(np.uint8)
    for counts in (np.full(n_sym, 7), np.minimum(np.cumsum(np.arange(n_sym)) + 1, 3000),
                   np.minimum(2 ** np.minimum(np.arange(n_sym), 14), 6000), rng.integers(1, 5, n_sym)):
        raw = np.repeat(syms, counts)
        rng.shuffle(raw)
        raw = np.resize(raw, (raw.size + 15) // 16 * 16)
        _check(codec, Z.ZIPNN_U8, raw, Z.make_params(Z.ZIPNN_U8, chunk_bytes=1 << 20, S=256, L=L,
                                                     policy=[Z.ZIPNN_HUF]))


@pytest.mark.parametrize("spread", [0.0, 0.2, 0.35, 0.45, 0.6, 0.9])
@pytest.mark.parametrize("chunk,S", [(262144, 512), (65536, 128), (4096, 16)])
def test_nearly_uniform_groups(codec, spread, chunk, S):
    """AUTO where the best code lies just above or below the raw size: counts
    spread evenly, in a ramp, and in two levels."""
    rng = np.random.default_rng(int(100 * spread) + chunk)
    E = chunk // 2
    cols = []
    for w in (1 + spread * np.linspace(-1, 1, 256), np.where(np.arange(256) < 32, 1 + 4 * spread, 1.0)):
        cols.append(rng.choice(256, 2 * E + 33, p=w / w.sum()).astype(np.uint8))
    raw = np.stack([cols[0], cols[1]], axis=1).reshape(-1)
    _check(codec, Z.ZIPNN_BF16, raw, Z.make_params(Z.ZIPNN_BF16, chunk_bytes=chunk, S=S))


@pytest.mark.parametrize("dt", [Z.ZIPNN_BF16, Z.ZIPNN_FP32])
@pytest.mark.parametrize("chunk", [262144, 524288])
@pytest.mark.parametrize("S_div", [64, 128, 256, 512])
def test_streams_held_in_registers(codec, dt, chunk, S_div):
    """More than 512 chunks of the sizes whose coded streams stay in registers
    between the counting and the size pass, full and partial last chunk, with
    streams beyond the held ones coded in some chunks."""
    B = Z.WIDTH[dt]
    E = chunk // B
    if E // S_div > 4096:
        pytest.skip("S out of range")
    n = 513 * E + 1000
    g = torch.Generator(device="cuda")
    g.manual_seed(S_div + B)
    x = (torch.randn(n, generator=g, device="cuda") * 0.02).to(TORCH[dt])
    x.view(torch.uint8).view(-1, B)[5 * E:6 * E, 0] &= 3       # the lowest byte group of chunk 5 is compressible
    x[7 * E:7 * E + E // 2] = 0                               # zeros: a ZG candidate in chunk 7
    p = Z.make_params(dt, chunk_bytes=chunk, S=E // S_div)
    c = codec.compress(x, p)
    out = torch.empty_like(x)
    codec.decompress(c, out)
    assert torch.equal(out.view(torch.uint8), x.view(torch.uint8))
    # the first and the last chunks against the oracle, as tensors of their own:
    # a chunk's map entries do not depend on the others but for the offsets
    for a, b in ((0, 9 * E), (512 * E, n)):
        part = x[a:b].clone()
        ref = oracle.compress(part.cpu().view(torch.uint8).numpy(), dt, chunk_bytes=chunk, S=p.substream_syms, g=p.group,
                              L=p.max_code_len, policy=list(p.policy))
        nc = (b - a + E - 1) // E
        got = c[64 + 16 * B * (a // E):64 + 16 * B * (a // E + nc)].cpu().numpy().view(np.uint64).reshape(-1, 2)
        want = np.frombuffer(ref[64:64 + 16 * B * nc].tobytes(), np.uint64).reshape(-1, 2)
        assert np.array_equal(got[:, 1], want[:, 1])          # sizes and modes
        pb = 64 + 16 * B * 514
        pb = (pb + 127) // 128 * 128
        rb = (64 + 16 * B * nc + 127) // 128 * 128
        o = int(got[0, 0])
        size = ref.size - rb
        assert np.array_equal(c[pb + o:pb + o + size].cpu().numpy(), ref[rb:])


@pytest.mark.parametrize("skip", [0, 3])
@pytest.mark.parametrize("n", [0, 1, 5000])
def test_single_tensor_descriptor(codec, n, skip):
    """A single tensor's descriptor comes with the analysis' launch (an empty
    one's, which is not analysed, by a launch of its own); it leaves nothing
    of the descriptors of a larger batch before it, nor the other way."""
    p = Z.zipnn_default_params(Z.ZIPNN_BF16)
    p.chunk_bytes, p.substream_syms, p.probe_skip = 1024, 16, skip
    rng = np.random.default_rng(7 + n)
    raws = [_words(rng, m, 2) for m in (3000, n, 700)]
    xs = [torch.from_numpy(r).view(torch.bfloat16).cuda() for r in raws]
    for _ in range(2):
        arena, offs = codec.compress_batch(xs, p)
        for i, r in enumerate(raws):
            ref = oracle.compress(r, Z.ZIPNN_BF16, chunk_bytes=p.chunk_bytes, S=p.substream_syms, g=p.group,
                                  L=p.max_code_len, policy=list(p.policy), skip=skip, exp=False)
            assert np.array_equal(arena[offs[i]:offs[i] + ref.size].cpu().numpy(), ref)
            assert np.array_equal(codec.compress(xs[i], p).cpu().numpy(), ref)


def test_status_keeps_the_first_error(codec):
    """An error stays until it is cleared, whatever is decoded after it."""
    p = Z.zipnn_default_params(Z.ZIPNN_BF16)
    x = torch.from_numpy(_words(np.random.default_rng(3), 4096, 2)).view(torch.bfloat16).cuda()
    c = codec.compress(x, p)
    out = torch.empty_like(x)
    head = c[:64].cpu().numpy().tobytes()
    bad = c.clone()
    bad[64:] = 0xFF   # map entries of no known mode
    codec.decompress(bad, out, header=head, check=False)
    codec.decompress(c, out, header=head, check=False)
    assert codec.status(clear=False) == Z.ZIPNN_E_CORRUPT
    assert codec.status(clear=True) == Z.ZIPNN_E_CORRUPT
    assert codec.status(clear=True) == Z.ZIPNN_OK
    codec.decompress(c, out)
    assert torch.equal(out.view(torch.uint8), x.view(torch.uint8))
