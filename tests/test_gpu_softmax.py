"""The running softmax of the bf16 kernels for more than 64 blocks and for 4x4
blocks: sums of probabilities before their rounding to bf16, and scores far
below and above the first ones."""
import numpy as np
import pytest
import torch

from oracle import ssba_oracle as O
from paper_2605_15684_amd.inputs import make_qkv, workload_from

from _parity import gpu_desc, oracle_kw, to64

pytestmark = pytest.mark.gpu


def _w(**kw):
    base = dict(batch=1, heads=1, grid_h=72, grid_w=72, head_dim=64, tile=8, keep=2, shift=(4, 4))
    base.update(kw)
    return workload_from(**base)


KERNELS = [_w(), _w(head_dim=128), _w(grid_h=80, grid_w=208, tile=16), _w(grid_h=80, grid_w=208, tile=16, head_dim=128),
           _w(tile=4, grid_h=36, grid_w=40, keep=8), _w(tile=4, grid_h=36, grid_w=40, keep=8, head_dim=128)]
kernels = pytest.mark.parametrize("w", KERNELS, ids=lambda w: f"b{w.tile}-D{w.head_dim}")


def _run(w, q, k, v):
    """Output and index of lists that hold the first `keep` blocks."""
    from paper_2605_15684_amd import ssba
    idx = np.full((1, 1, w.n_tiles, w.n_tiles + 1), -1, np.int32)
    idx[..., 0], idx[..., 1:1 + w.keep] = w.keep, np.arange(w.keep)
    qg, kg, vg = (t.to("cuda") for t in (q, k, v))
    out = ssba.forward(qg, kg, vg, torch.from_numpy(idx).to("cuda"), gpu_desc(w, qg))
    torch.cuda.synchronize()
    return out.cpu(), idx


def _frame(w):
    return torch.from_numpy(np.asarray(O.frame_tiles(w.grid_h, w.grid_w, w.tile, *w.shift)))


@kernels
def test_row_sums_are_32_bit(w):
    """Two keys of probability 1 and the rest of just under the middle between
    0.5 and the next bf16 value, all with value 1: the products with V take
    the rounded 0.5, the sum what it was."""
    q, k, v = (torch.zeros_like(t) for t in make_qkv(w))
    unit = np.log2(np.e) / np.sqrt(w.head_dim)
    q[..., 0], q[..., 1] = 8, 0.125
    k[..., 0] = -0.6875 if w.head_dim == 64 else -0.97265625
    k[..., 1] = torch.tensor((np.log2(0.50188) / unit - 8 * float(k[0, 0, 0, 0])) / 0.125).to(k.dtype)
    top = _frame(w)[0, [0, 8 if w.tile == 4 else 32]]   # one for each half of a 64-key chunk
    k[:, :, top] = 0
    v[:] = 1
    out, _ = _run(w, q, k, v)
    p = float(torch.exp2(unit * (to64(q)[0, 0, 0] @ to64(k)[0, 0, int(_frame(w)[1, 0])]) * torch.ones(1, dtype=torch.float64)))
    assert 0.5015 < p < 0.50194
    n = w.keep * w.tile * w.tile - 2
    want = torch.tensor((2 + n * 0.5) / (2 + n * p)).to(torch.bfloat16)
    assert want < 1 and bool((out == want).all())


@kernels
def test_a_first_block_far_below(w):
    """The first list entry's scores lie 10^7 log2 units below the second's,
    which differ by less than a rounding step of that distance."""
    q, k, v = make_qkv(w)
    q[..., 0], k[..., 0] = 1024, 0
    frame = _frame(w)
    k[0, 0, frame[0], 0] = -2.0 ** 17
    if w.tile == 4:   # two blocks a step
        k[0, 0, frame[1], 0] = -2.0 ** 17
    out, idx = _run(w, q, k, v)
    ref = O.attention(to64(q), to64(k), to64(v), idx, **oracle_kw(w))
    bound = O.attention(to64(q), to64(k), np.abs(to64(v)), idx, **oracle_kw(w)) / 128   # P and the output: 8 bits each
    assert (np.abs(to64(out) - ref) <= bound).all()


@kernels
def test_all_scores_far_below(w):
    """Every score is -4.6e29 / -3.2e29 log2 units: equal probabilities, not a row without keys."""
    q, k, v = make_qkv(w)
    q[..., 0], k[..., 0] = 2.0 ** 50, -2.0 ** 51
    out, idx = _run(w, q, k, v)
    seen = to64(v)[0, 0, _frame(w)[:w.keep].ravel()]
    bound = np.abs(seen).mean(0) / 256
    assert (np.abs(to64(out)[0, 0] - seen.mean(0)) <= bound).all()
