"""Helpers shared by the GPU parity tests: run a workload through the HIP
path (via the C ABI binding) and through the fp64 oracle on the same seeded
inputs."""
from __future__ import annotations

import numpy as np
import torch

from oracle import ssba_oracle as O
from paper_2605_15684_amd.inputs import Workload, make_qkv

BF16_TOL = 2e-2     # max-abs error allowed for bf16 inputs
F32_TOL = 1e-5      # max-abs error allowed for the fp32 path


def tol(w: Workload) -> float:
    return F32_TOL if w.dtype == "f32" else BF16_TOL


def oracle_kw(w: Workload) -> dict:
    return dict(grid_h=w.grid_h, grid_w=w.grid_w, tile=w.tile, shift=w.shift, n_text=w.n_text)


def gpu_desc(w: Workload, q: torch.Tensor):
    from paper_2605_15684_amd import ssba
    return ssba.desc_for(q, grid=(w.grid_h, w.grid_w), tile=w.tile, shift=w.shift,
                         n_text=w.n_text, gate=w.gate, keep=w.keep, window=w.window)


def inputs(w: Workload):
    """CPU tensors (dtype of the workload) and their GPU copies."""
    q, k, v = make_qkv(w)
    return (q, k, v), tuple(t.to("cuda") for t in (q, k, v))


def to64(t: torch.Tensor) -> np.ndarray:
    return t.detach().to("cpu").double().numpy()


def oracle_index(w: Workload, q, k) -> np.ndarray:
    return O.build_index(to64(q), to64(k), gate=w.gate, keep=w.keep, window=w.window, **oracle_kw(w))


def run_gpu(w: Workload, qg, kg, vg, dense: bool = False):
    """(index on CPU or None, output on GPU)."""
    from paper_2605_15684_amd import ssba
    desc = gpu_desc(w, qg)
    if dense:
        out = ssba.forward_dense(qg, kg, vg, desc)
        torch.cuda.synchronize()
        return None, out
    index, _ = ssba.build_index(qg, kg, desc)
    out = ssba.forward(qg, kg, vg, index, desc)
    torch.cuda.synchronize()
    return index.cpu().numpy(), out


def sample_rows(w: Workload, rng: np.random.Generator, n_random: int = 64) -> np.ndarray:
    """Query rows for sampled full-size checks: every text row (at most 80),
    the first, last and one random query block of the shifted frame, and
    random rows."""
    tiles = O.frame_tiles(w.grid_h, w.grid_w, w.tile, *w.shift)
    rows = [np.arange(min(w.n_text, 80))]
    for t in (0, tiles.shape[0] - 1, int(rng.integers(tiles.shape[0]))):
        blk = tiles[t]
        if blk.size > 64:
            blk = blk[rng.choice(blk.size, 64, replace=False)]
        rows.append(w.n_text + blk)
    rows.append(rng.integers(0, w.seq_len, n_random))
    return np.unique(np.concatenate(rows))


def max_err(gpu_out: torch.Tensor, ref: np.ndarray, heads, rows) -> float:
    g = gpu_out.detach().float().cpu()
    err = 0.0
    for b, h in heads:
        gg = g[b, h, rows].double().numpy()
        rr = ref[b, h, rows]
        assert np.isfinite(gg).all()
        err = max(err, float(np.abs(gg - rr).max()))
    return err


def growing_inputs(w: Workload, at, units: int = 24):
    """Inputs for which the running maximum of a list of the first `keep`
    blocks, ascending, grows by about `units` log2 units at each of the
    entries `at`, in every other query row; in the rows between, the same
    keys change nothing.  Each part's values are larger by what its
    probabilities lose later, so that it still shows in the output.  Returns
    (q, k, v), the index and the bound 2^-7 sum p |v| on the error of each
    output (P and the output are each rounded to 8 bits)."""
    q, k, v = make_qkv(w)
    frame = np.asarray(O.frame_tiles(w.grid_h, w.grid_w, w.tile, *w.shift))
    unit = 8.0 / np.sqrt(w.head_dim) * np.log2(np.e)      # log2 units of q0 = 8, k0 = 1
    step = float(np.ceil(units / unit))
    level = torch.zeros(w.seq_len)
    for t in range(w.n_tiles):
        level[w.n_text + torch.from_numpy(frame[t])] = float(sum(t >= x for x in at))
    q[..., 0] = 0
    q[:, :, ::2, 0] = 8
    k[..., 0] = (step * level).to(k.dtype)
    v *= torch.exp2(units * (len(at) - level))[:, None].to(v.dtype)
    index = np.full((w.batch, w.heads, w.n_tiles, w.n_tiles + 1), -1, np.int32)
    index[..., 0] = w.keep
    index[..., 1:1 + w.keep] = np.arange(w.keep)
    # A sum of 2^20 in a lane takes the new maximum: each growth passes it by itself.
    s = to64(q)[0, 0, w.n_text + np.arange(w.n_text % 2, w.t_img, 2)] @ to64(k)[0, 0, w.n_text + frame[:w.keep].ravel()].T
    s = (s * unit / 8).reshape(len(s), w.keep, -1)
    for e in at:
        assert (s[:, e].min(-1) - s[:, :e].max((-2, -1))).min() > 20
    bound = O.attention(to64(q), to64(k), np.abs(to64(v)), index, **oracle_kw(w)) / 128
    return (q, k, v), index, bound
