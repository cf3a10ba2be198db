"""The binding's one-expression argument checks accept nothing that the named checks refuse."""

import pytest

import paper_2505_22918_amd as rt


class Fake:
    """A stand-in tensor: what the checks read, without a GPU."""

    def __init__(self, torch, shape, dtype, dev=0, contiguous=True):
        self.shape, self.dtype, self._dev, self._c = torch.Size(shape), dtype, dev, contiguous
        self.is_cuda = dev >= 0
        self.device = torch.device("cuda", dev) if dev >= 0 else torch.device("cpu")

    def get_device(self):
        return self._dev

    def is_contiguous(self):
        return self._c

    def dim(self):
        return len(self.shape)


def test_qkv_check():
    import torch

    good = lambda **kw: Fake(torch, **{**dict(shape=(1, 2, 64, 64), dtype=torch.bfloat16), **kw})
    d = rt._check_qkv(good(), good(), good())
    assert (d.B, d.H, d.T, d.D) == (1, 2, 64, 64)
    bad = [good(shape=(1, 2, 64, 72)), good(shape=(2, 64, 64)), good(dtype=torch.float16), good(dev=1), good(dev=-1),
           good(contiguous=False), None, 3]
    for x in bad:
        for at in range(3):
            args = [good(), good(), good()]
            args[at] = x
            with pytest.raises(ValueError):
                rt._check_qkv(*args)


def test_same_and_mask():
    import torch

    like = Fake(torch, (1, 2, 64, 64), torch.bfloat16)
    stat = lambda **kw: Fake(torch, **{**dict(shape=(1, 2, 64), dtype=torch.float32), **kw})
    assert rt._same(stat(), torch.float32, like.shape[:3], like)
    for x in (stat(shape=(1, 2, 65)), stat(dtype=torch.float64), stat(dev=1), stat(dev=-1), stat(contiguous=False), None, 3):
        assert not rt._same(x, torch.float32, like.shape[:3], like)
    idx = lambda dev: Fake(torch, (4,), torch.int32, dev)
    rt._mask_on(rt.BlockMask(idx(0), idx(0), 64, 1, 1), like)
    for a, b in ((1, 0), (0, 1), (-1, 0), (0, -1)):
        with pytest.raises(ValueError, match="mask"):
            rt._mask_on(rt.BlockMask(idx(a), idx(b), 64, 1, 1), like)
