"""bf16 attention where a kernel's offsets end: row strides for which the
slice of one (batch, head) is the largest that the 32-bit (4x4 blocks: 31-bit)
byte offsets of a specialised kernel reach, and the next one, which the
generic kernel (64-bit offsets) takes; and the dense control of fewer than 64
tokens, which it takes too.  Against the fp64 oracle (2e-2 max-abs, as every
bf16 parity test), every row."""
import numpy as np
import pytest
import torch

from oracle import ssba_oracle as O
from paper_2605_15684_amd import _lib
from paper_2605_15684_amd.inputs import make_qkv, workload_from

from _parity import BF16_TOL, gpu_desc, oracle_index, oracle_kw, run_gpu, inputs, to64

pytestmark = pytest.mark.gpu


def _w(**kw):
    base = dict(batch=1, heads=1, grid_h=16, grid_w=16, head_dim=64, tile=4, keep=3, shift=(2, 2), n_text=5)
    base.update(kw)
    return workload_from(**base)


# workload, bytes that a slice (with this many rows more) has to stay below, kernels at and past the limit
CASES = [
    (_w(), 1 << 31, 0, "k_attn_tile4<64>", "k_attn_bf16<64, 2>"),
    (_w(head_dim=128), 1 << 31, 0, "k_attn_tile4<128>", "k_attn_bf16<128, 2>"),
    (_w(grid_h=72, grid_w=72, tile=8, keep=9), 1 << 32, 64, "k_attn_mfma_long<64, 3>", "k_attn_bf16<64, 3>"),
    (_w(grid_h=72, grid_w=72, tile=8, keep=66, head_dim=128, n_text=77), 1 << 32, 64, "k_attn_mfma_long<128, 3>",
     "k_attn_bf16<128, 3>"),
    (_w(grid_h=80, grid_w=208, tile=16, keep=2), 1 << 32, 64, "k_attn_mfma_long<64, 4>", "k_attn_bf16<64, 4>"),
    (_w(grid_h=80, grid_w=208, tile=16, keep=2, head_dim=128), 1 << 32, 64, "k_attn_mfma_long<128, 4>",
     "k_attn_bf16<128, 4>"),
]


def _ids(c):
    return f"D{c[0].head_dim}-b{c[0].tile}"


@pytest.mark.parametrize("past", [False, True], ids=["at", "past"])
@pytest.mark.parametrize("case", CASES, ids=_ids)
def test_row_stride_at_the_limit(case, past):
    from paper_2605_15684_amd import ssba
    w, limit, more, at_name, past_name = case
    st = 8 * ((limit - 1) // (16 * (w.seq_len + more))) + (8 if past else 0)   # rows start at multiples of 16 bytes
    q, k, v = make_qkv(w)
    idx = oracle_index(w, q, k)
    strided = []
    for t in (q, k, v, torch.zeros_like(q)):
        x = torch.empty_strided(t.shape, (st * w.seq_len, st * w.seq_len, st, 1), dtype=t.dtype, device="cuda")
        strided.append(x.copy_(t))
    desc = gpu_desc(w, strided[0])
    assert _lib.forward_kernel(desc) == (past_name if past else at_name)
    out = ssba.forward(*strided[:3], torch.from_numpy(idx).to("cuda"), desc, out=strided[3])
    torch.cuda.synchronize()
    got = out.cpu()
    del out, strided
    torch.cuda.empty_cache()
    ref = O.attention(to64(q), to64(k), to64(v), idx, **oracle_kw(w))
    assert float(np.abs(to64(got) - ref).max()) <= BF16_TOL


@pytest.mark.parametrize("w", [_w(grid_h=4, grid_w=4, n_text=1, keep=1), _w(grid_h=4, grid_w=12, n_text=15, keep=1),
                               _w(grid_h=4, grid_w=8, n_text=0, keep=1, head_dim=128, heads=3)],
                         ids=lambda w: f"{w.seq_len}-D{w.head_dim}")
def test_dense_control_of_few_tokens(w):
    (q, k, v), gpu = inputs(w)
    assert _lib.forward_kernel(gpu_desc(w, gpu[0]), dense=True) == f"k_attn_bf16<{w.head_dim}, 2>"
    _, out = run_gpu(w, *gpu, dense=True)
    idx = O.build_index(to64(q), to64(k), gate="dense", **oracle_kw(w))
    ref = O.attention(to64(q), to64(k), to64(v), idx, **oracle_kw(w))
    assert float(np.abs(to64(out) - ref).max()) <= BF16_TOL
