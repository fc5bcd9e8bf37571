"""GPU: the tiled kernel's work items dealt in queues (one per XCD up to 96 row
tiles, plain order past that): queues of different lengths with more items than
workgroups, fewer (layer, role)s than queues, one item per workgroup, and both
sides of the limit; every layer and role against the fp64 oracle on windows of
rows, and no row past the end touched."""

import numpy as np
import pytest

from paper_2609_32259_amd import synth

from _compare import Case, windows

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch
    assert torch.cuda.is_available(), "GPU test needs a GPU"
    from paper_2609_32259_amd import heterofold
    heterofold.lib()
    return torch


# H_s, H_r, L_r, receiver rows (identical tokenizations), layer map
SHAPES = [(8, 8, 9, 2500, "interp2"),       # 18 maps in 8 queues, 720 items
          (8, 4, 9, 2500, "interp2"),
          (4, 8, 3, 6000, "interp2"),       # 6 maps: two queues empty, 564 items
          (8, 8, 1, 96 * 64, "interp2"),    # 96 tiles: 2 queues hold all 192 items
          (8, 8, 1, 96 * 64 + 1, "interp2"),   # 97 tiles: plain order
          (8, 8, 1, 128 * 64, "interp2"),
          (8, 8, 1, 128 * 64 + 1, "interp2"),  # more items than workgroups
          (8, 8, 5, 60, "interp2"),         # 10 items, one each
          (8, 2, 9, 700, "interp2"),        # one item per workgroup, uneven: plain order
          (8, 2, 4, 700, "interp2"),        # one item per workgroup, even: queues
          (16, 8, 4, 500, "interp2"),
          (4, 4, 9, 500, "neighbor3")]


@pytest.mark.parametrize("H_s,H_r,L_r,T,layer_map", SHAPES)
def test_every_item_is_done_once(torch, H_s, H_r, L_r, T, layer_map):
    from paper_2609_32259_amd.path import TransferPath
    cfg = synth.LLAMA8B_14B_8K.with_(name=f"order {H_s}->{H_r} L_r={L_r} T={T}", H_s=H_s, H_r=H_r,
                                     L_s=4, L_r=L_r, layer_map=layer_map)
    rng = np.random.default_rng(T)
    sb, se = synth.segment_tokens(rng, T, 1, 7)
    seg = synth.concat_segmentations([(sb, se, sb.copy(), se.copy())])
    S = synth.make_cache(cfg, seg, seed=90, device="cuda")
    A, bias = synth.make_maps(cfg, seed=90, device="cuda")
    wl = synth.Workload(cfg, seg, S, A, bias, synth.rope_params(cfg))
    print(f"[gpu-order] {cfg.name}", flush=True)
    R = torch.full((1, L_r, 2, H_r, T + 5, 128), float("nan"), dtype=torch.bfloat16, device="cuda")
    TransferPath(seg, S, A, bias, wl.rope, L_r, H_r, R=R, layer_map=layer_map, staged=False).step()
    torch.cuda.synchronize()
    assert bool(torch.isfinite(R[:, :, :, :, :T]).all()) and bool(R[:, :, :, :, T:].isnan().all())
    Case(cfg, wl, R, "overlap", tag="gpu-order").check_all(
        windows_of=lambda b, T_r: windows(T_r, 64, rng, n_mid=1, width=96))
