"""bf16 attention with more than 64 blocks per head: kept lists that end at,
just before and just after the 64 entries that pass through the lanes at a
time, uneven lists, ragged text and ids past the grid, against the fp64 oracle
(2e-2 max-abs, as every bf16 parity test; every row)."""
import numpy as np
import pytest
import torch

from oracle import ssba_oracle as O
from paper_2605_15684_amd import _lib
from paper_2605_15684_amd.inputs import workload_from

from _parity import BF16_TOL, gpu_desc, growing_inputs, inputs, oracle_index, oracle_kw, sample_rows, to64


def _w(**kw):
    base = dict(batch=1, heads=1, grid_h=72, grid_w=72, head_dim=64, tile=8, keep=64, shift=(4, 4))
    base.update(kw)
    return workload_from(**base)


CASES = [
    _w(grid_h=40, grid_w=104, keep=65),                                         # 65 blocks, all kept
    _w(keep=1), _w(keep=63), _w(keep=64), _w(keep=65, n_text=13), _w(keep=81, n_text=64),
    _w(grid_h=88, grid_w=96, keep=128, shift=(-3, 5)), _w(grid_h=88, grid_w=96, keep=129, n_text=77),
    _w(head_dim=128, keep=66, n_text=5), _w(head_dim=128, keep=64, heads=2, batch=4),
    _w(grid_h=80, grid_w=208, tile=16, keep=65, shift=(8, -8)),                 # 65 blocks of 16x16
    _w(grid_h=80, grid_w=208, tile=16, keep=3, n_text=9, head_dim=128),
]


def _ids(w):
    return f"{w.grid_h}x{w.grid_w}-D{w.head_dim}-b{w.tile}-k{w.keep}-t{w.n_text}"


def _forward(w, qg, kg, vg, idx):
    from paper_2605_15684_amd import ssba
    out = ssba.forward(qg, kg, vg, torch.from_numpy(idx).to("cuda"), gpu_desc(w, qg))
    torch.cuda.synchronize()
    return out.float().cpu().double().numpy()


@pytest.mark.gpu
@pytest.mark.parametrize("uneven", [False, True], ids=["topk", "uneven"])
@pytest.mark.parametrize("w", CASES, ids=_ids)
def test_long_lists(w, uneven):
    (q, k, v), gpu = inputs(w)
    idx = oracle_index(w, q, k)
    if uneven:   # block i keeps the first 1 + 7 i mod keep entries
        tb = w.n_tiles
        idx = idx.copy()
        idx.reshape(-1, tb, tb + 1)[:, :, 0] = 1 + 7 * np.arange(tb) % w.keep
    got = _forward(w, *gpu, idx)
    ref = O.attention(to64(q), to64(k), to64(v), idx, **oracle_kw(w))
    assert np.isfinite(got).all()
    assert float(np.abs(got - ref).max()) <= BF16_TOL


@pytest.mark.gpu
@pytest.mark.parametrize("w", [_w(keep=81, n_text=5), _w(keep=81, n_text=5, head_dim=128),
                               _w(grid_h=80, grid_w=208, tile=16, keep=65)], ids=_ids)
def test_scores_that_grow(w):
    """A new maximum in half of the rows after 1, 7, 30 and 64 blocks."""
    (q, k, v), idx, bound = growing_inputs(w, (1, 7, 30, 64))
    rows = np.arange(w.seq_len) if w.tile == 8 else sample_rows(w, np.random.default_rng(1))
    got = _forward(w, *(t.to("cuda") for t in (q, k, v)), idx)
    ref = O.attention(to64(q), to64(k), to64(v), idx, rows=rows, **oracle_kw(w))
    assert (np.abs(got - ref)[:, :, rows] <= bound[:, :, rows]).all()


@pytest.mark.gpu
@pytest.mark.parametrize("d,n_text", [(64, 3), (64, 77), (128, 77)])
def test_masked_keys_add_nothing(d, n_text):
    """Ids past the grid and the rows beside a ragged tail are not seen,
    whatever they hold: NaN rows where an id past the grid in the first 64
    entries, or a tail of the text, would read; an infinite value in the block
    that the lane of such an id held before the list's second part; and an
    infinite text value that the second text chunk would see again."""
    w = _w(grid_h=88, grid_w=96, keep=70, n_text=n_text, head_dim=d)
    (q, k, v), (qg, kg, _) = inputs(w)
    idx = oracle_index(w, q, k).copy()
    frame = np.asarray(O.frame_tiles(w.grid_h, w.grid_w, w.tile, *w.shift))
    hidden = np.unique(np.concatenate([np.arange(64), (96 * np.arange(8)[:, None] + np.arange(8)).ravel()]))
    v[:, :, w.n_text + torch.from_numpy(hidden)] = float("nan")
    ok = [t for t in range(w.n_tiles) if not np.isin(frame[t], hidden).any()]
    want = idx.copy()                                  # the same without the two ids
    want[..., 0], want[..., 1:69] = 68, ok[:68]
    idx[..., 0], idx[..., 1:71] = 70, np.insert(ok[:68], [5, 65], [5000, -3])   # entries 5 and 66
    assert idx[0, 0, 0, 6] == 5000 and idx[0, 0, 0, 67] == -3
    v[:, :, w.n_text + int(frame[ok[2]][9]), 7] = float("inf")                  # entry 2: the lane of entry 66
    inf = [7]
    if n_text > 64:
        v[:, :, 40, 9] = float("inf")
        inf.append(9)
    got = _forward(w, qg, kg, v.to("cuda"), idx)[:, :, w.n_text:]
    assert (got[..., inf] == np.inf).all()
    v[~torch.isfinite(v)] = 0
    ref = O.attention(to64(q), to64(k), to64(v), want, **oracle_kw(w))[:, :, w.n_text:]
    rest = [c for c in range(d) if c not in inf]
    assert float(np.abs(got - ref)[..., rest].max()) <= BF16_TOL


@pytest.mark.gpu
@pytest.mark.parametrize("n_text", [3, 77])
def test_infinite_value_in_the_last_rows(n_text):
    """A text row's last chunk starts at a multiple of 64 rows: the rows before it are seen once."""
    w = _w(keep=1, n_text=n_text)
    (q, k, v), (qg, kg, _) = inputs(w)
    idx = oracle_index(w, q, k)
    v[:, :, w.seq_len - 40, 9] = float("inf")
    got = _forward(w, qg, kg, v.to("cuda"), idx)[:, :, :n_text]
    assert (got[..., 9] == np.inf).all()
    v[~torch.isfinite(v)] = 0
    ref = O.attention(to64(q), to64(k), to64(v), idx, rows=np.arange(n_text), **oracle_kw(w))[:, :, :n_text]
    rest = [c for c in range(64) if c != 9]
    assert float(np.abs(got - ref)[..., rest].max()) <= BF16_TOL


def test_kernel_names():
    d = lambda **kw: _lib.forward_kernel(_desc(**kw))   # noqa: E731
    assert d() == "k_attn_mfma_long<64, 3>"
    assert d(tile=16, grid_h=128, grid_w=256, head_dim=128) == "k_attn_mfma_long<128, 4>"
    assert d(grid_w=64) == "k_attn_mfma<64, 3, false, false>"
    assert d(tile=4) == "k_attn_tile4<64>"
    assert d(tile=4, head_dim=128, dtype=_lib.DT_F32) == "k_attn_f32<128>"
    assert d(tile=4, grid_h=4, grid_w=4, keep=1, batch=(1 << 24) - 1) == "k_attn_tile4<64>"     # 2^32 threads
    assert d(tile=4, grid_h=4, grid_w=4, keep=1, batch=1 << 24) == "k_attn_bf16<64, 2>"
    # 32-bit (4x4: 31-bit) byte offsets inside one (batch, head) are the kernels' limits
    assert d(tile=4, stride_b=1 << 40, stride_h=1 << 36, stride_t=233016) == "k_attn_tile4<64>"
    assert d(tile=4, stride_b=1 << 40, stride_h=1 << 36, stride_t=233024) == "k_attn_bf16<64, 2>"
    assert d(stride_b=1 << 40, stride_h=1 << 36, stride_t=1 << 20) == "k_attn_bf16<64, 3>"


def _desc(**kw):
    d = _lib.SsbaDesc()
    base = dict(batch=1, heads=1, head_dim=64, grid_h=64, grid_w=72, tile=8, gate=_lib.GATE_TOPK, keep=4,
                win_h=1, win_w=1, dtype=_lib.DT_BF16)
    base.update(kw)
    for name, value in base.items():
        setattr(d, name, value)
    return d
