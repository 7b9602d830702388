"""The decoder's ring of stream words where its loops meet.

The loop over full groups refills a stream's ring at fixed steps and else only
when the next round could run past it; the loop over the last groups checks
once in CHECK rounds and needs at most half of the ring used up when it starts.
A step without a marked group decodes nothing and passes a refill point by: as
the last step of the first loop, after long codes, it leaves the ring nearly
used up."""
import numpy as np
import pytest
import torch

import oracle
from oracle import spec
from paper_2411_05239_amd import zipnn as Z

S, W, L = 1024, 64, 11
TORCH = {Z.ZIPNN_BF16: torch.bfloat16, Z.ZIPNN_FP32: torch.float32, Z.ZIPNN_U8: torch.uint8}


def _past_the_ring(lens, marked, B, g, n_w, refill_between):
    """How far past the ring's words the cursor of any lane group reads, for a
    ZG stream decoded by itself: lens (groups, g) code lengths."""
    RW = 256 if B == 4 else 512
    at = max(1, min(4, (8 if B == 4 else 16) // g))   # steps between refill points
    worst = -RW
    for w0 in range(0, n_w, 64):
        lanes = np.arange(w0, min(n_w, w0 + 64))
        steps = (len(lens) - 1 - lanes[0]) // n_w + 1
        n_fast = ((len(lens) - 1 - lanes[-1]) // n_w + 1) // 4 * 4
        bits, ptr, rb = np.zeros(len(lanes), int), 0, 0
        for e in range(steps):
            q = np.minimum(lanes + e * n_w, len(lens) - 1)
            on = (lanes + e * n_w < len(lens)) & marked[q]
            if e == n_fast and refill_between and ptr - rb >= RW // 2:
                rb += RW // 2
            if e < n_fast and not on.any():
                continue
            for pr in range(g // 2):
                need = on & (bits < 2 * L)
                worst = max(worst, ptr + int(need.sum()) - (rb + RW))
                ptr += int(need.sum())
                bits += 32 * need - np.where(on, lens[q, 2 * pr] + lens[q, 2 * pr + 1], 0)
                end = pr == g // 2 - 1
                if e < n_fast:
                    due = ptr - rb >= RW // 2 if end and e % at == at - 1 else ptr - rb > RW - 64
                else:
                    due = (end or (pr + 1) % (RW // 128) == 0) and ptr - rb >= RW // 2
                rb += RW // 2 if due else 0
    return worst


def _stream(g, seed, rare_steps, empty):
    """One stream of a chunk whose last three steps follow the loop over full
    groups of four: short codes, then steps of the longest codes, then (the
    loop's last step) nothing but the fill value, then the longest again."""
    T = S // g - 1
    rng = np.random.default_rng(seed)
    s = rng.choice(np.array([0, 1, 2], np.uint8), (T, W, g), p=[.6, .3, .1])
    s[rng.random((T, W)) < empty] = 0
    s[:seed] = 0
    n_fast = T // 4 * 4
    s[n_fast - 1 - rare_steps:n_fast - 1] = rng.integers(3, 256, (rare_steps, W, g))
    s[n_fast - 1] = 0
    s[n_fast:] = rng.integers(3, 256, (T - n_fast, W, g))
    return s.reshape(T * W, g)


def _lengths(s):
    marked = (s != 0).any(1)
    f = np.bincount(s[marked].reshape(-1), minlength=256)
    table = np.zeros(256, int)
    for sym, n in spec.pm_lengths({i: int(v) for i, v in enumerate(f)}, L).items():
        table[sym] = n
    return table[s], marked


def _reaching(B, g, count):
    """The first `count` streams that would run past a ring not refilled
    between the loops."""
    found = []
    for i in range(240):
        s = _stream(g, i % 12, 2 + i // 12 % 12, 0.3 * (i % 2))
        if _past_the_ring(*_lengths(s), B, g, W, False) > 0:
            found.append(s)
            if len(found) == count:
                return found
    raise AssertionError("no stream reaches the ring's end")


@pytest.mark.parametrize("B,g", [(1, 4), (1, 8), (4, 4)])
def test_streams_reach_the_end_of_the_ring(B, g):
    for s in _reaching(B, g, 4):
        assert _past_the_ring(*_lengths(s), B, g, W, True) <= 0


@pytest.mark.parametrize("B", [1, 4])
@pytest.mark.parametrize("g", [2, 4, 8])
def test_no_read_past_the_ring(B, g):
    rng = np.random.default_rng(10 * B + g)
    for _ in range(30):
        n_w, groups = int(rng.integers(1, 131)), int(rng.integers(1, 2500))
        lens = rng.choice(np.array([1, 2, 8, 11]), (groups, g), p=rng.dirichlet(np.ones(4)))
        marked = rng.random(groups) < rng.random()
        # stretches of steps alike: nothing marked, or the longest codes
        step = np.arange(groups) // n_w
        for _ in range(4):
            a = int(rng.integers(0, step[-1] + 1))
            at = (step >= a) & (step < a + rng.integers(1, 9))
            marked[at] = rng.random() < 0.5
            lens[at] = 11
        assert _past_the_ring(lens, marked, B, g, n_w, True) <= 0


@pytest.mark.gpu
@pytest.mark.parametrize("dt,g,delta", [(Z.ZIPNN_U8, 4, True), (Z.ZIPNN_U8, 8, True), (Z.ZIPNN_U8, 8, False),
                                        (Z.ZIPNN_BF16, 4, True), (Z.ZIPNN_BF16, 8, True), (Z.ZIPNN_FP32, 4, False),
                                        (Z.ZIPNN_FP32, 4, True), (Z.ZIPNN_FP32, 8, False)])
@pytest.mark.parametrize("streams", ["all", "last"])
def test_decode_at_the_end_of_the_ring(dt, g, delta, streams):
    """streams: all of the byte groups hold such a stream, or the last alone
    beside Huffman-coded ones (FP32: a set without a loop of its own)."""
    B = Z.WIDTH[dt]
    found = _reaching(4 if (B, g) == (4, 4) else 1, g, 4)
    rng = np.random.default_rng(B + g)
    codec = Z.Codec(0)
    for i in range(4):
        cols = [found[(i + k) % 4].reshape(-1) for k in range(B)]
        policy = [Z.ZIPNN_ZG] * B
        if streams == "last":
            for k in range(B - 1):
                cols[k] = rng.choice(np.array([7, 8, 9], np.uint8), cols[k].size, p=[.8, .1, .1])
                policy[k] = Z.ZIPNN_HUF
        x = np.stack(cols[::-1], axis=1).reshape(-1)   # stream k is byte B-1-k
        base = rng.integers(0, 256, x.size, dtype=np.uint8) if delta else None
        raw = x ^ base if delta else x
        c = oracle.compress(raw, dt, base=base, chunk_bytes=B << 16, S=S, g=g, L=L, policy=policy)
        assert c[64 + 16 * (B - 1) + 12] == oracle.MODE_ZG
        out = torch.empty(raw.size // B, dtype=TORCH[dt], device="cuda")
        b = torch.from_numpy(base).cuda().view(TORCH[dt]) if delta else None
        codec.decompress(torch.from_numpy(c).cuda(), out, base=b)
        assert np.array_equal(out.view(torch.uint8).cpu().numpy(), raw), (i, dt, g, delta, streams)
    codec.close()
