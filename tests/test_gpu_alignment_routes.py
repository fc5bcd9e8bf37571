"""GPU alignment on each of its routes: one workgroup (up to 1024 rows of up to 4
sequences that overlap few sender tokens), two launches, and three launches (past
1024 workgroups of 256 rows).  Small cases
against the oracle, bit for bit; the largest against the closed form of two
tokenizations that tile one text (an entry per interval between neighbouring
boundaries), as the oracle is a per-token loop."""

import numpy as np
import pytest

from oracle import alignment as al
from paper_2609_32259_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hf():
    import torch
    assert torch.cuda.is_available(), "GPU test needs a GPU"
    from paper_2609_32259_amd import heterofold
    heterofold.lib()
    return heterofold


def _run(hf, seg, mode):
    import torch
    t = lambda a: torch.as_tensor(np.ascontiguousarray(a, np.int32), device="cuda")  # noqa: E731
    out = hf.hf_build_alignment(seg.s_cu, seg.r_cu, t(seg.s_beg), t(seg.s_end), t(seg.r_beg),
                                t(seg.r_end), mode)
    torch.cuda.synchronize()
    rp = out.row_ptr.cpu().numpy()
    return (rp, out.col[:int(rp[-1])].cpu().numpy(), out.num[:int(rp[-1])].cpu().numpy(),
            out.den[:int(seg.r_cu[-1])].cpu().numpy())


def _tokens(rng, n_chars, n):
    """n tokens that tile n_chars characters."""
    end = np.sort(rng.choice(np.arange(1, n_chars), n - 1, replace=False))
    end = np.concatenate([end, [n_chars]]).astype(np.int32)
    return np.concatenate([[0], end[:-1]]).astype(np.int32), end


@pytest.mark.parametrize("mode", ["overlap", "ta"])
@pytest.mark.parametrize("rows", [(1,), (1023,), (1024,), (1025,), (500, 0, 524), (500, 0, 525),
                                  (0, 1024, 0), (256, 256, 257, 1)])
def test_alignment_around_the_one_workgroup_limit(hf, rows, mode):
    rng = np.random.default_rng(sum(rows))
    parts = []
    for i, n in enumerate(rows):
        if n == 0:  # sender tokens without receiver tokens, between the others
            sb, se = synth.segment_tokens(rng, 30, 1, 7)
            parts.append((sb, se, np.zeros(0, np.int32), np.zeros(0, np.int32)))
            continue
        chars = 5 * n + 3
        rb, re_ = _tokens(rng, chars, n)
        sb, se = synth.segment_messy(rng, chars, 1, 7)
        if i == 0:  # a run of empty sender tokens first: rows before any partner fall back past it
            k = 300
            sb, se = np.concatenate([np.zeros(k, np.int32), sb]), np.concatenate([np.zeros(k, np.int32), se])
        parts.append((sb, se, rb, re_))
    seg = synth.concat_segmentations(parts)
    print(f"[gpu-align] rows={rows} {mode}", flush=True)
    exp = al.build_alignment_batched(seg.s_cu, seg.r_cu, seg.s_beg, seg.s_end, seg.r_beg, seg.r_end,
                                     mode)
    for g, e in zip(_run(hf, seg, mode), exp):
        assert np.array_equal(g, e)


# sequences, rows of each, sender tokens of each: both sides of 4 sequences, and of the
# products of rows and sender tokens past 256 rows
@pytest.mark.parametrize("mode", ["overlap", "ta"])
@pytest.mark.parametrize("B,n,m", [(4, 60, 70), (5, 60, 70), (64, 16, 20), (1, 256, 20000),
                                   (1, 257, 16320), (1, 257, 16321), (2, 512, 2048), (2, 512, 2049)])
def test_alignment_around_the_one_workgroup_rule(hf, B, n, m, mode):
    rng = np.random.default_rng(B * n + m)
    parts = []
    for _ in range(B):
        chars = m + 5 * n  # tokens of 1 character or a few; most rows have no shared end
        parts.append(_tokens(rng, chars, m) + _tokens(rng, chars, n))
    seg = synth.concat_segmentations(parts)
    print(f"[gpu-align] B={B} rows={n} senders={m} {mode}", flush=True)
    exp = al.build_alignment_batched(seg.s_cu, seg.r_cu, seg.s_beg, seg.s_end, seg.r_beg, seg.r_end,
                                     mode)
    for g, e in zip(_run(hf, seg, mode), exp):
        assert np.array_equal(g, e)


@pytest.mark.parametrize("mode", ["overlap", "ta"])
@pytest.mark.parametrize("n", [256 * 1024, 256 * 1024 + 1])
def test_alignment_around_the_two_launch_limit(hf, n, mode):
    rng = np.random.default_rng(n)
    chars = 4 * n + 1
    sb, se = _tokens(rng, chars, n + 7)
    rb, re_ = _tokens(rng, chars, n)
    print(f"[gpu-align] n={n} {mode}", flush=True)
    rp, col, num, den = _run(hf, synth.concat_segmentations([(sb, se, rb, re_)]), mode)
    if mode == "overlap":
        cut = np.unique(np.concatenate([se, re_]))
        beg = np.concatenate([[0], cut[:-1]])
        row = np.searchsorted(re_, beg, side="right")
        assert np.array_equal(rp, np.concatenate([[0], np.cumsum(np.bincount(row, minlength=n))]))
        assert np.array_equal(col, np.searchsorted(se, beg, side="right"))
        assert np.array_equal(num, cut - beg)
        assert np.array_equal(den, re_ - rb)
        return
    i = np.searchsorted(se, re_)
    hit = se[i] == re_
    last = np.maximum.accumulate(np.where(hit, np.arange(n), -1))
    assert np.array_equal(col, np.where(last >= 0, i[np.maximum(last, 0)], 0))
    assert np.array_equal(rp, np.arange(n + 1)) and bool((num == 1).all()) and bool((den == 1).all())
