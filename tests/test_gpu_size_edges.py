"""GPU: kernels at the sizes where their partitioning can go wrong -- one tile, runs that end inside a wave, the
first size that needs a second pass of a loop -- against the oracle or against an independent kernel of the
library that the oracle pins elsewhere."""
import numpy as np
import pytest
import torch

from oracle import fgmp_oracle as orc
from paper_2504_14152_amd import fgmp, synth

pytestmark = pytest.mark.gpu
DEV = "cuda"


# ------------------------------------------------------------------ packing weights

def _run_lengths(mask: torch.Tensor, rows: int, K: int) -> torch.Tensor:
    """FP8 slots per 8 x 128 tile, in tile order, from a canonical mask."""
    n_rt, n_kt = -(-rows // 8), -(-(K // 16) // 8)
    m = torch.zeros((n_rt * 8, n_kt * 8), dtype=torch.int64, device=mask.device)
    m[:rows, : K // 16] = mask.to(torch.int64)
    return m.view(n_rt, 8, n_kt, 8).sum((1, 3)).flatten()


# (rows, K): one tile; fewer tiles than waves; tiles per wave that leave a ragged last run; 2 per wave; and, with
# one block per row, more than 512 x 16 x 64 tiles, where a wave walks its run in two batches
@pytest.mark.parametrize("rows,K", [(1, 16), (8, 144), (520, 2064), (70000, 144), (4200000, 16)])
@pytest.mark.parametrize("p", [0.0, 0.1, 1.0])
def test_packed_weights_hold_the_same_blocks_as_the_one_pass_layout(rows, K, p):
    g = torch.Generator(device=DEV).manual_seed(rows + K)
    w = torch.randn(rows, K, generator=g, device=DEV).to(torch.bfloat16)
    f = torch.exp(torch.randn(K, generator=g, device=DEV))
    s = float(w.abs().max()) / 448.0
    _, scores = fgmp.quantize_weights(w, f, float("inf"), s, want_scores=True)
    T = fgmp.threshold_for_fraction(scores, p)
    pw = fgmp.quantize_weights(w, f, T, s)
    px = fgmp.quantize_activations(w, f, T, s)       # strided layout: nothing shared with the packing pass
    for a, b in zip(fgmp.unpack_canonical(pw), fgmp.unpack_canonical(px)):
        assert torch.equal(a, b)
    mask = fgmp.unpack_canonical(px)[2]
    counts = _run_lengths(mask, rows, K)
    info = fgmp.packed_info(pw)
    assert info["n_fp8_blocks"] == int(counts.sum())
    n_tiles = counts.numel()
    off_T = 256 + n_tiles * 512                       # planes L, S, M precede T, each 256-byte aligned
    off_T = -(-off_T // 256) * 256 + n_tiles * 64
    off_T = -(-off_T // 256) * 256 + n_tiles * 8
    off_T = -(-off_T // 256) * 256
    plane_t = pw.buf[off_T: off_T + 4 * n_tiles].view(torch.int32).to(torch.int64)
    assert torch.equal(plane_t, torch.cumsum(counts, 0) - counts)
    off_H = -(-(off_T + 4 * n_tiles) // 256) * 256
    assert info["bytes_used"] == off_H + 8 * max(1, int(counts.sum()))
