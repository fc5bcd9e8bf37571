"""GPU: two receiver heads and more than eight sender heads give the same bits
whichever way a tile is built.

Those shapes build a tile from its staged entries in LDS, or, where the sender
cache spans 2 GiB or more, straight from the alignment table.  Both add an entry
with the same operations in the same order, so the receiver cache of a cache with
far-apart heads has to equal that of the packed one bit for bit."""

import numpy as np
import pytest

from paper_2609_32259_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch
    assert torch.cuda.is_available(), "GPU test needs a GPU"
    from paper_2609_32259_amd import heterofold
    heterofold.lib()
    return torch


def _far_heads(torch, S):
    """S with its heads so far apart that a (layer, role) spans 2 GiB."""
    B, L, two, H, T, d = S.shape
    step = ((1 << 30) // (H - 1) // 8 + 1) * 8   # elements, 16-byte aligned
    assert B == 1 and step >= L * two * T * d and (H - 1) * step * 2 >= 1 << 31
    view = torch.zeros(H * step, dtype=S.dtype, device="cuda").as_strided(
        S.shape, (0, two * T * d, T * d, step, d, 1))
    view.copy_(S)
    return view


# H_s, H_r, layer map, keys stored before RoPE, longest sender token (1: about 5
# entries a row, and runs of rows wider than the rotation table in LDS)
SHAPES = [(8, 2, "interp2", False, 7), (8, 2, "interp2", False, 1), (2, 2, "interp2", False, 7),
          (16, 2, "interp2", False, 7), (16, 4, "neighbor3", False, 7), (9, 8, "interp2", False, 7),
          (16, 8, "interp2", False, 1), (8, 2, "neighbor3", True, 7)]


@pytest.mark.parametrize("H_s,H_r,layer_map,pre,longest", SHAPES)
def test_staged_entries_and_the_alignment_table_give_the_same_bits(torch, H_s, H_r, layer_map, pre,
                                                                   longest):
    from paper_2609_32259_amd.path import TransferPath
    cfg = synth.LLAMA8B_14B_8K.with_(name=f"bits {H_s}->{H_r} {layer_map} {longest}", H_s=H_s,
                                     H_r=H_r, L_s=3, L_r=4, layer_map=layer_map, batch=1,
                                     sender_keys_post_rope=not pre, paper_opts=pre)
    rng = np.random.default_rng(H_s + H_r)
    sb, se = synth.segment_tokens(rng, 300, 1, longest)
    rb, re_ = synth.segment_chars(rng, int(se[-1]), 4 if longest == 1 else 1, 6)
    seg = synth.concat_segmentations([(sb, se, rb, re_)])
    S = synth.make_cache(cfg, seg, seed=17, device="cuda")
    A, bias = synth.make_maps(cfg, seed=17, device="cuda")
    rope = synth.rope_params(cfg, pos0_s=np.array([1000], np.int32), pos0_r=np.array([9], np.int32))
    print(f"[gpu-bits] {cfg.name}", flush=True)
    out = [TransferPath(seg, s, A, bias, rope, cfg.L_r, H_r, layer_map=layer_map,
                        opts=synth.make_opts(cfg, 17, "cuda"), staged=False).step()
           for s in (S, _far_heads(torch, S))]
    torch.cuda.synchronize()
    assert bool(out[0].isfinite().all()) and bool(out[0].any())
    assert torch.equal(out[0].view(torch.int16), out[1].view(torch.int16))
