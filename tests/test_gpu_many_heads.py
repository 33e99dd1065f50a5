"""More (batch, head) pairs than one launch of 256-thread workgroups covers
(2^32 threads), in one 4x4 block each: tensors whose pairs lie a few elements
apart and hold one value throughout, so that they fit in memory and every
output is that value, also that of the last pair."""
import pytest
import torch

pytestmark = pytest.mark.gpu

PAIRS = (1 << 24) + 8


@pytest.mark.parametrize("dtype,step,batch", [(torch.float32, 4, PAIRS // 8), (torch.float32, 4, 1),
                                              (torch.bfloat16, 8, PAIRS // 8)], ids=["f32", "f32-heads", "bf16"])
def test_last_pair(dtype, step, batch):
    from paper_2605_15684_amd import ssba
    heads = PAIRS // batch
    shape, strides = (batch, heads, 16, 64), (heads * step, step, 64, 1)
    mk = lambda x: torch.full(((PAIRS - 1) * step + 1024,), x, dtype=dtype, device="cuda")   # noqa: E731
    q, buf = torch.as_strided(mk(0.5), shape, strides), mk(-1.0)
    desc = ssba.desc_for(q, grid=(4, 4), tile=4, gate="dense")
    index = torch.zeros((*shape[:2], 1, 2), dtype=torch.int32, device="cuda")
    index[..., 0] = 1
    ssba.forward(q, q, q, index, desc, out=torch.as_strided(buf, shape, strides))
    torch.cuda.synchronize()
    assert bool((buf == 0.5).all())
