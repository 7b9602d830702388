"""GPU decode at the edges of the loop's cases: lane groups with fewer than 64
sub-streams, coded streams that use up words faster than the ring's refill
points assume, and batches whose few plain containers join the launch of those
with ZG entries.  The decoded words equal the originals."""
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


def _oracle_container(raw, dt, p, base=None):
    ref = oracle.compress(raw, dt, base=base, chunk_bytes=p.chunk_bytes, S=p.substream_syms, g=p.group,
                          L=p.max_code_len, policy=list(p.policy))
    return torch.from_numpy(np.ascontiguousarray(ref)).cuda()


@pytest.mark.parametrize("dt", [Z.ZIPNN_BF16, Z.ZIPNN_FP32, Z.ZIPNN_U8])
@pytest.mark.parametrize("g", [2, 4, 8])
@pytest.mark.parametrize("kind", ["spread", "longest", "mixed"])
def test_words_used_up_fast(codec, dt, g, kind):
    """spread: 8 bits a symbol everywhere; longest: stretches of the rarest
    symbols, 11 bits each, so that every lane takes a word in most rounds;
    mixed: both beside each other in one lane group."""
    B = Z.WIDTH[dt]
    S, W = 256, 100          # two lane groups, the second partial
    n = S * W - 3
    rng = np.random.default_rng(100 * dt + g + len(kind))
    raw = rng.integers(0, 256, (n, B), dtype=np.uint8)
    if kind != "spread":
        # a steep histogram whose tail has the longest codes; the tail
        # symbols come in long runs
        hot = rng.choice(np.array([1, 2, 3], np.uint8), (n, B), p=[.6, .3, .1])
        runs = ((np.arange(n) // (g * W * 16)) % 5 == 4)[:, None]
        lanes = (np.arange(n) // g % W % 2 == 0)[:, None] if kind == "mixed" else True
        raw = np.where(runs & lanes, raw, hot).astype(np.uint8)
    p = Z.make_params(dt, chunk_bytes=1 << 18, S=S, g=g, policy=[Z.ZIPNN_HUF] * B)
    raw = raw.reshape(-1)
    out = torch.empty(n, dtype=TORCH[dt], device="cuda")
    codec.decompress(_oracle_container(raw, dt, p), out)
    assert np.array_equal(out.view(torch.uint8).cpu().numpy(), raw)


@pytest.mark.parametrize("W", [1, 2, 7, 63, 64, 65, 130])
@pytest.mark.parametrize("policy", [[Z.ZIPNN_HUF, Z.ZIPNN_RAW], [Z.ZIPNN_ZG, Z.ZIPNN_HUF], [Z.ZIPNN_ZG, Z.ZIPNN_ZG]])
@pytest.mark.parametrize("delta", [False, True])
def test_partial_lane_groups(codec, W, policy, delta):
    n = 64 * W - (W % 5)
    rng = np.random.default_rng(W)
    raw = np.zeros((n, 2), np.uint8)
    raw[:, 1] = rng.choice(np.array([0, 60, 61, 188], np.uint8), n, p=[.7, .15, .1, .05])
    raw[:, 0] = np.where(rng.random(n) < 0.3, rng.integers(0, 256, n), 0)
    raw = raw.reshape(-1)
    base = rng.integers(0, 256, raw.size, dtype=np.uint8) if delta else None
    x = raw ^ base if delta else raw
    p = Z.make_params(Z.ZIPNN_BF16, chunk_bytes=1 << 18, S=64, g=4, policy=policy)
    # the output is followed by words that must stay
    out = torch.full((n + 64,), 7.0, dtype=torch.bfloat16, device="cuda")
    b = torch.from_numpy(base.copy()).view(torch.bfloat16).cuda() if delta else None
    codec.decompress(_oracle_container(x, Z.ZIPNN_BF16, p, base), out[:n], base=b)
    assert np.array_equal(out[:n].view(torch.uint8).cpu().numpy(), x)
    assert bool((out[n:] == 7.0).all())


@pytest.mark.parametrize("plain", [1000, 40_000, 400_000])
def test_plain_containers_beside_zg(codec, plain):
    """Below an eighth of the bytes the plain containers join the launch of
    those with ZG entries, above it they have their own; a container whose
    flag changed since the batch was prepared is reported either way."""
    rng = np.random.default_rng(plain)
    xs, params = [], []
    pz = Z.make_params(Z.ZIPNN_BF16, chunk_bytes=65536, S=128, policy=[Z.ZIPNN_ZG, Z.ZIPNN_ZG])
    pp = Z.make_params(Z.ZIPNN_BF16, chunk_bytes=65536, S=128, policy=[Z.ZIPNN_HUF, Z.ZIPNN_RAW])
    for n, p in ((300_000, pz), (plain, pp), (200_001, pz), (333, pp)):
        raw = np.where(rng.random(2 * n) < 0.2, rng.integers(1, 256, 2 * n), 0).astype(np.uint8)
        xs.append(torch.from_numpy(raw).view(torch.bfloat16).cuda())
        params.append(p)
    cs = [codec.compress(x, p).clone() for x, p in zip(xs, params)]
    offs = [0]
    for c in cs:
        offs.append((offs[-1] + c.numel() + 127) // 128 * 128)
    arena = torch.zeros(offs[-1], dtype=torch.uint8, device="cuda")
    for c, o in zip(cs, offs):
        arena[o:o + c.numel()] = c
    outs = [torch.empty_like(x) for x in xs]
    batch = codec.prepare_batch(arena, offs, outs)
    for _ in range(2):
        for o in outs:
            o.zero_()
        batch.run(check=True)
        for x, o in zip(xs, outs):
            assert torch.equal(x.view(torch.int16), o.view(torch.int16))
    arena[offs[1] + 24] |= 2      # the plain container now claims ZG entries
    batch.run()
    assert codec.status(clear=True) == Z.ZIPNN_E_FORMAT
    batch.close()
