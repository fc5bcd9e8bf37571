"""GPU parity of the fp32 transfer kernels where their tiling changes: one and
several groups of receiver heads, one and several chunks of the map row, inputs
that are no multiple of 16, row counts around the 32-row tile, tiles with more
alignment entries than LDS holds, and heads past the matrix-core kernel's 256
channels, against the fp64 oracle (rel-Fro <= 1e-5)."""

import numpy as np
import pytest

from paper_2609_32259_amd import synth

from _compare import Case

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch
    assert torch.cuda.is_available(), "GPU test needs a GPU"
    from paper_2609_32259_amd import heterofold
    heterofold.lib()
    return torch


def _check(torch, cfg, parts, mode):
    from paper_2609_32259_amd.path import TransferPath
    seg = synth.concat_segmentations(parts)
    S = synth.make_cache(cfg, seg, seed=70, device="cuda")
    A, bias = synth.make_maps(cfg, seed=70, device="cuda")
    rng = np.random.default_rng(70)
    rope = synth.rope_params(cfg, pos0_s=rng.integers(0, 99, seg.batch).astype(np.int32),
                             pos0_r=rng.integers(0, 99, seg.batch).astype(np.int32))
    wl = synth.Workload(cfg, seg, S, A, bias, rope, synth.make_opts(cfg, 70, "cuda"))
    print(f"[gpu-f32] {cfg.name} T_r={list(seg.r_len)}", flush=True)
    T_cap = int(seg.r_len.max()) + 3
    R = torch.full((seg.batch, cfg.L_r, 2, cfg.H_r, T_cap, cfg.d_h), 3.0, device="cuda")
    path = TransferPath(seg, S, A, bias, rope, cfg.L_r, cfg.H_r, mode=mode, R=R,
                        layer_map=cfg.layer_map, opts=wl.opts)
    path.step()
    torch.cuda.synchronize()
    Case(cfg, wl, R, mode, tag="gpu-f32").check_all()
    for b in range(seg.batch):
        assert bool((R[b, :, :, :, int(seg.r_len[b]):] == 3.0).all()), "rows past the end changed"


# d_h, H_s, H_r, layer map, key norm
SHAPES = [(128, 4, 4, "interp2", True),     # two head groups, two chunks
          (64, 5, 8, "neighbor3", True),    # three chunks of one tap each, two head groups
          (36, 3, 5, "neighbor3", False),   # 324 inputs: 4 past a multiple of 16; 18-channel halves
          (256, 2, 3, "interp2", False),    # one head per chunk and group
          (8, 1, 1, "interp2", False),      # 8 inputs and 8 outputs: less than one step and tile
          (260, 1, 2, "interp2", False)]    # past the matrix-core kernel


@pytest.mark.parametrize("d_h,H_s,H_r,layer_map,norm", SHAPES)
def test_f32_groups_chunks_and_row_edges(torch, d_h, H_s, H_r, layer_map, norm):
    cfg = synth.TINY_F32.with_(name=f"f32 d_h={d_h} {H_s}->{H_r} {layer_map}", d_h=d_h, H_s=H_s,
                               H_r=H_r, L_s=6, L_r=3, layer_map=layer_map, paper_opts=norm,
                               rope=(1.0e4, 5.0e5))
    rng = np.random.default_rng(71)
    parts = []
    for n in (31, 32, 33, 1, 64):  # identical tokenizations: T_r = T_s
        sb, se = synth.segment_tokens(rng, n, 1, 7)
        parts.append((sb, se, sb.copy(), se.copy()))
    _check(torch, cfg, parts, "ta")


def test_f32_tiles_beyond_staged_entries(torch):
    # 9-16 one-character sender tokens per receiver token: about 400 entries per
    # 32-row tile in the first sequence (LDS holds 256), 100 in the second
    cfg = synth.TINY_F32.with_(name="f32 many entries", L_s=3, L_r=4, rope=(1.0e4, 5.0e5))
    rng = np.random.default_rng(72)
    parts = []
    for n, s_hi, r_lo, r_hi in ((700, 1, 9, 16), (150, 7, 1, 8)):
        sb, se = synth.segment_tokens(rng, n, 1, s_hi)
        rb, re_ = synth.segment_chars(rng, int(se[-1]), r_lo, r_hi)
        parts.append((sb, se, rb, re_))
    _check(torch, cfg, parts, "overlap")
