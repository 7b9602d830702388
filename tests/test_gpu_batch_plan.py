"""How many launches a prepared batch makes: a few plain containers join those
with ZG entries by the sizes of the tensors, whatever room their outputs have."""
import ctypes

import pytest
import torch

from paper_2411_05239_amd import zipnn as Z

pytestmark = pytest.mark.gpu


def test_plan_follows_the_tensors_sizes():
    from torch.profiler import ProfilerActivity, profile

    codec = Z.Codec(0)
    L = Z.lib()
    g = torch.Generator().manual_seed(1)
    n = 2_000_000
    zg = (torch.randn(n, generator=g) * (torch.rand(n, generator=g) < 0.1)).to(torch.bfloat16).cuda()
    batches = []
    # below and above an eighth of the bytes; the plain tensor goes to the
    # start of a large pool, the other to a buffer of its size
    for plain in (4096, 1_000_000):
        xs = [zg, torch.randn(plain, generator=g).to(torch.bfloat16).cuda()]
        params = [Z.make_params(Z.ZIPNN_BF16, policy=[Z.ZIPNN_ZG] * 2),
                  Z.make_params(Z.ZIPNN_BF16, policy=[Z.ZIPNN_HUF, Z.ZIPNN_RAW])]
        cs = [codec.compress(x, p).clone() for x, p in zip(xs, params)]
        at = (cs[0].numel() + 127) // 128 * 128
        arena = torch.zeros(at + cs[1].numel(), dtype=torch.uint8, device="cuda")
        arena[:cs[0].numel()], arena[at:] = cs[0], cs[1]
        outs = [torch.empty_like(zg), torch.zeros(64 << 20, dtype=torch.uint8, device="cuda")]
        dst = (ctypes.c_void_p * 2)(*[o.data_ptr() for o in outs])
        cap = (ctypes.c_uint64 * 2)(*[o.numel() * o.element_size() for o in outs])
        h = ctypes.c_void_p()
        assert L.zipnn_batch_create(codec.ctx, arena.data_ptr(), (ctypes.c_uint64 * 3)(0, at, arena.numel()), 2, dst,
                                    cap, None, ctypes.byref(h)) == Z.ZIPNN_OK
        batches.append((h, xs, outs, arena))
    with profile(activities=[ProfilerActivity.CUDA]) as prof:
        for _ in range(3):
            for h, *_ in batches:
                assert L.zipnn_batch_decompress(h, None) == Z.ZIPNN_OK
        torch.cuda.synchronize()
    assert codec.status() == Z.ZIPNN_OK
    for h, xs, outs, _ in batches:
        for x, o in zip(xs, outs):
            assert torch.equal(o.view(torch.int16)[:x.numel()], x.view(torch.int16))
        L.zipnn_batch_destroy(h)
    codec.close()
    plans = sum(e.count for e in prof.key_averages() if "k_plan" in e.key)
    if not plans:
        pytest.skip("the profiler saw no kernels")
    assert plans == 3 * 1 + 3 * 2   # one plan for each class of containers
