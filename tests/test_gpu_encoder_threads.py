"""One prepared encoder run by several threads, each on a stream of its own: the
runs share the scratch, the placement's count of finished tensors and the
arena, so they take place one after another, and leave nothing behind that a
later run on other data would trip over."""
import threading

import numpy as np
import pytest
import torch

from paper_2411_05239_amd import zipnn as Z

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("delta", [False, True])
def test_runs_from_several_threads(delta):
    codec = Z.Codec(0)
    g = torch.Generator().manual_seed(5)
    sizes = [5, 70_000, 4096, 0, 300_001, 128, 20_000, 9]
    xs = [torch.randn(n, generator=g).to(torch.bfloat16).cuda() for n in sizes]
    bases = [x.clone() for x in xs] if delta else None
    if delta:
        for x in xs:
            x[::9] += 0.5
    p = Z.make_params(Z.ZIPNN_BF16, chunk_bytes=4096, S=16)
    enc = codec.prepare_encoder(xs, p, bases)
    want_offs = list(enc.run())
    want = enc.arena[:want_offs[-1]].clone()
    torch.cuda.synchronize()
    seen, errors = [], []

    def work():
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                for _ in range(25):
                    seen.append(list(enc.run()))
        except Exception as e:  # noqa: BLE001
            errors.append(e)

    threads = [threading.Thread(target=work) for _ in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors
    assert len(seen) == 100 and all(o == want_offs for o in seen)
    assert torch.equal(enc.arena[:want_offs[-1]], want)
    # other data of other container sizes
    for x in xs:
        x.copy_(torch.arange(x.numel(), device="cuda").remainder(7).to(torch.bfloat16))
    offs = list(enc.run())
    arena, ref_offs = codec.compress_batch(xs, p, bases=bases)
    assert offs == list(ref_offs)
    for a, b in zip(offs[:-1], offs[1:]):
        assert np.array_equal(enc.arena[a:b].cpu().numpy()[:64], arena[a:b].cpu().numpy()[:64])
    outs = [torch.empty_like(x) for x in xs]
    batch = codec.prepare_batch(enc.arena, offs, outs, bases)
    batch.run(check=True)
    for x, o in zip(xs, outs):
        assert torch.equal(x.view(torch.int16), o.view(torch.int16))
    batch.close()
    enc.close()
    codec.close()
