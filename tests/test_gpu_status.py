"""The sticky status: the first error recorded stays until it is cleared, and
after that the next one is recorded."""
import numpy as np
import pytest
import torch

from paper_2411_05239_amd import zipnn as Z

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def setup():
    codec = Z.Codec(0)
    x = torch.randn(40_000, generator=torch.Generator().manual_seed(1)).to(torch.bfloat16).cuda()
    p = Z.make_params(Z.ZIPNN_BF16, chunk_bytes=4096, S=16)
    c = codec.compress(x, p).clone()
    corrupt, changed = c.clone(), c.clone()
    corrupt[64:72] = 0xFF      # the first map entry's place
    changed[24] |= 2           # the device's header claims ZG entries, the host's copy does not
    yield codec, x, c, {Z.ZIPNN_E_CORRUPT: corrupt, Z.ZIPNN_E_FORMAT: changed}
    codec.close()


@pytest.mark.parametrize("first,second", [(Z.ZIPNN_E_CORRUPT, Z.ZIPNN_E_FORMAT),
                                          (Z.ZIPNN_E_FORMAT, Z.ZIPNN_E_CORRUPT)])
def test_first_of_two_errors_stays(setup, first, second):
    codec, x, c, bad = setup
    out = torch.empty_like(x)
    head = c[:64].cpu().numpy().tobytes()
    for _ in range(3):   # recorded again after every clear
        for code in (first, second, first):
            codec.decompress(bad[code], out, header=head, check=False)
        assert codec.status(clear=False) == first
        codec.decompress(bad[second], out, header=head, check=False)
        assert codec.status(clear=True) == first
        assert codec.status(clear=True) == Z.ZIPNN_OK
        codec.decompress(bad[second], out, header=head, check=False)
        assert codec.status(clear=True) == second
        codec.decompress(c, out)
        assert torch.equal(out.view(torch.int16), x.view(torch.int16))


def test_errors_of_many_workgroups_and_streams(setup):
    """Errors of both kinds found side by side: one of them is recorded, and
    it stays the one reported while more come in."""
    codec, x, c, bad = setup
    head = c[:64].cpu().numpy().tobytes()
    streams = [torch.cuda.Stream() for _ in range(4)]
    outs = [torch.empty_like(x) for _ in streams]
    torch.cuda.synchronize()
    for turn in range(10):
        for i in range(8):
            with torch.cuda.stream(streams[i % 4]):
                b = bad[(Z.ZIPNN_E_CORRUPT, Z.ZIPNN_E_FORMAT)[(i + turn) % 2]]
                codec.decompress(b, outs[i % 4], header=head, check=False)
        torch.cuda.synchronize()
        code = codec.status(clear=False)
        assert code in bad
        for b in bad.values():
            codec.decompress(b, outs[0], header=head, check=False)
        assert codec.status(clear=True) == code
        assert codec.status(clear=False) == Z.ZIPNN_OK


def test_batch_reports_and_recovers(setup):
    """A batch whose containers fail in the plan and in the decode at once."""
    codec, x, c, bad = setup
    offs = [i * ((c.numel() + 127) // 128 * 128) for i in range(4)]
    arena = torch.zeros(offs[-1] + (c.numel() + 127) // 128 * 128, dtype=torch.uint8, device="cuda")
    for o in offs:
        arena[o:o + c.numel()] = c
    good = arena.clone()
    outs = [torch.empty_like(x) for _ in offs]
    batch = codec.prepare_batch(arena, offs + [arena.numel()], outs)
    for _ in range(3):
        arena[offs[1]:offs[1] + c.numel()] = bad[Z.ZIPNN_E_CORRUPT]
        arena[offs[2]:offs[2] + c.numel()] = bad[Z.ZIPNN_E_FORMAT]
        batch.run()
        # the plan runs before any chunk is decoded
        assert codec.status(clear=True) == Z.ZIPNN_E_FORMAT
        arena.copy_(good)
        for o in outs:
            o.zero_()
        batch.run(check=True)
        for o in outs:
            assert torch.equal(o.view(torch.int16), x.view(torch.int16))
    batch.close()
