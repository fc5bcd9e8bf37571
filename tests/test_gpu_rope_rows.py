"""GPU: the RoPE tables hold only the rows a call reads -- the first 16 of the
sender's and each side's from its smallest start position on.  Start positions
around 16, apart within a batch, and a workspace full of NaN before the call."""

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


@pytest.mark.parametrize("kind", ["fused", "staged", "two heads", "f32"])
@pytest.mark.parametrize("pos0_s,pos0_r", [((15, 40), (0, 3)), ((16, 16), (33, 1)), ((17, 900), (5, 5)),
                                           ((2000, 17), (70, 4000))])
def test_rope_rows_around_the_first_sixteen(torch, kind, pos0_s, pos0_r):
    from paper_2609_32259_amd.path import TransferPath
    if kind == "f32":
        cfg = synth.TINY_F32.with_(name="rope rows", rope=(1.0e4, 5.0e5), batch=2, n_chars=300)
    else:
        cfg = synth.LLAMA8B_14B_8K.with_(name=f"rope rows {kind}", L_s=3, L_r=2, T_s=70, batch=2,
                                         H_r=2 if kind == "two heads" else 8)
    wl = synth.make_workload(cfg, seed=80, device="cuda")
    rope = synth.rope_params(cfg, pos0_s=np.array(pos0_s, np.int32), pos0_r=np.array(pos0_r, np.int32))
    wl = synth.Workload(cfg, wl.seg, wl.S, wl.A, wl.bias, rope)
    print(f"[gpu-rope-rows] {kind} {pos0_s} {pos0_r}", flush=True)
    path = TransferPath(wl.seg, wl.S, wl.A, wl.bias, rope, cfg.L_r, cfg.H_r, staged=kind == "staged")
    path.transfer_ws.fill_(0xFF)  # NaN in fp32 and bf16
    R = path.step()
    torch.cuda.synchronize()
    Case(cfg, wl, R, "overlap", tag="gpu-rope-rows").check_all()
