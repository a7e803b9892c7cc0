"""GPU LM head: oracle parity, and the same logits bits for a row however
the batch is formed -- which, fed to the log-prob, gives a reuse ratio of
exactly one end to end (Section 3.1)."""
import numpy as np
import pytest

import oracle
from paper_2609_35140_amd import inputs

pytestmark = pytest.mark.gpu
gu = pytest.importorskip("gpu_util")


@pytest.fixture(scope="module")
def ua():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_35140_amd import uattn
    uattn.lib()
    return uattn


@pytest.mark.parametrize("T,V,H", [(300, 1000, 512), (129, 257, 64), (1, 4099, 1024), (256, 512, 4096)])
def test_matches_oracle(ua, T, V, H):
    h = inputs.normal_bf16((T, H), 1.0, 94, T, V)
    w = inputs.normal_bf16((V, H), float(2.0 / np.sqrt(H)), 95, T, V)
    got = gu.host_bits(ua.lm_head(gu.dev(h), gu.dev(w)))
    ref = oracle.logits_fp64(h, w)
    err = np.abs(oracle.bf16_to_f64(got) - ref)
    # bf16 output rounding plus fp32 accumulation over H terms
    bound = 2.0 ** -8 * np.abs(ref) + H * 2.0 ** -24 * oracle.abs_dot(h, w)
    exact = np.mean(got == oracle.logits_bf16(h, w))
    print(f"T={T} V={V} H={H}: {exact:.4f} equal to the rounded fp64 logits, max err {err.max():.3g}", flush=True)
    assert np.all(err <= bound) and exact > 0.95


def test_rows_are_batch_invariant_and_ratio_is_one(ua):
    import torch
    T, V, H = 640, 1500, 1024
    h = gu.dev(inputs.normal_bf16((T, H), 1.0, 96))
    w = gu.dev(inputs.normal_bf16((V, H), 0.0625, 97))
    full = ua.lm_head(h, w)
    tg = gu.dev_i32(inputs.targets(T, V, tag=98))
    lp_full = ua.logprob(full, tg)
    g = inputs.rng(99)
    for n in (1, 2, 7, 128, 129, 300):
        idx = torch.from_numpy(g.permutation(T)[:n]).cuda()
        part = ua.lm_head(h[idx].contiguous(), w)
        assert torch.equal(part.view(torch.int16), full[idx].view(torch.int16)), n
        lp = ua.logprob(part, tg[idx].contiguous())
        assert torch.equal(lp.view(torch.int32), lp_full[idx].view(torch.int32)), n
        assert bool((torch.exp(lp.double() - lp_full[idx].double()) == 1.0).all())
    # a row alone
    one = ua.lm_head(h[5:6], w)
    assert torch.equal(one.view(torch.int16), full[5:6].view(torch.int16))


@pytest.mark.parametrize("T,V,H,it", [(300, 1000, 512, 1.0), (129, 257, 64, 1.0), (1, 4099, 1024, 0.7),
                                       (256, 512, 4096, 1.0), (70, 20000, 256, 1.3)])
def test_fused_logprob_matches_oracle(ua, T, V, H, it):
    import torch
    h = inputs.normal_bf16((T, H), 1.0, 94, T, V)
    w = inputs.normal_bf16((V, H), float(2.0 / np.sqrt(H)), 95, T, V)
    tg = inputs.targets(T, V, tag=T)
    hd, wd, td = gu.dev(h), gu.dev(w), gu.dev_i32(tg)
    lp = ua.lm_head_logprob(hd, wd, td, inv_temperature=it).cpu().numpy().astype(np.float64)
    ref, bound = oracle.lm_head_logprob_fp64(h, w, tg, it)
    err = np.abs(lp - ref)
    print(f"T={T} V={V} H={H} it={it}: max err {err.max():.3g}, max err/bound {np.max(err / bound):.3f}, "
          f"median bound {np.median(bound):.3g}", flush=True)
    assert np.all(err <= bound)
    # the same logits through the two-call path: both fp32 log-softmaxes of identical logits
    logits = torch.empty((T, (V + 7) // 8 * 8), dtype=torch.bfloat16, device="cuda")[:, :V]
    lp2 = ua.lm_head_logprob(hd, wd, td, inv_temperature=it, logits=logits)
    assert torch.equal(logits.view(torch.int16), ua.lm_head(hd, wd).view(torch.int16))
    two = ua.logprob(logits, td, inv_temperature=it)
    assert float((lp2.double() - two.double()).abs().max()) < 2e-5


@pytest.mark.parametrize("V,H", [(255, 64), (257, 192), (321, 256), (1000, 640)])
def test_tile_shapes_give_the_same_bits(ua, V, H):
    """The tile shape follows the number of rows (16, 64 and 128 are its steps, of a call and of its last tile of 256) and
    the width (chunks of 64, 128, 256): rows of a small call equal the same rows of a large one, with and without stored
    logits."""
    import torch
    T = 700
    h = gu.dev(inputs.normal_bf16((T, H), 1.0, 96, H))
    w = gu.dev(inputs.normal_bf16((V, H), 0.25, 97, H))
    tg = gu.dev_i32(inputs.targets(T, V, tag=H))
    full, full_lp = ua.lm_head(h, w), ua.lm_head_logprob(h, w, tg)
    for n in (1, 15, 16, 17, 63, 64, 65, 127, 128, 129, 256, 257, 320, 321, 384, 385, 513):
        part = ua.lm_head(h[:n], w)
        assert torch.equal(part.view(torch.int16), full[:n].view(torch.int16)), n
        stored = torch.empty((n, (V + 7) // 8 * 8), dtype=torch.bfloat16, device="cuda")[:, :V]
        lp = ua.lm_head_logprob(h[:n], w, tg[:n], logits=stored)
        assert torch.equal(lp.view(torch.int32), full_lp[:n].view(torch.int32)), n
        assert torch.equal(stored.view(torch.int16), full[:n].view(torch.int16)), n


@pytest.mark.parametrize("which,stride,V", [("hidden", 1 << 22, 300), ("hidden", (1 << 22) + 8, 300),
                                            ("hidden", (1 << 22) + 8, 25600), ("weight", 1 << 22, 130),
                                            ("weight", (1 << 22) + 8, 130)])
def test_far_strides_give_the_same_bits(ua, which, stride, V):
    """Rows whose distance is the largest that 32-bit byte offsets inside a tile reach, and one step past it (tiles of 128
    tokens while they fit the GPU at once, else of 256): the bits of contiguous rows, plain and fused."""
    import torch
    T, H = 330, 128
    h = inputs.normal_bf16_device((T, H), 1.0, 99, 1)
    w = inputs.normal_bf16_device((V, H), 0.25, 99, 2)
    tg = gu.dev_i32(inputs.targets(T, V, tag=V))
    want, want_lp = ua.lm_head(h, w), ua.lm_head_logprob(h, w, tg)
    rows = T if which == "hidden" else V
    far = torch.empty((rows - 1) * stride + H, dtype=torch.bfloat16, device="cuda").as_strided((rows, H), (stride, 1))
    far.copy_(h if which == "hidden" else w)
    h, w = (far, w) if which == "hidden" else (h, far)
    assert torch.equal(ua.lm_head(h, w).view(torch.int16), want.view(torch.int16))
    assert torch.equal(ua.lm_head_logprob(h, w, tg).view(torch.int32), want_lp.view(torch.int32))


@pytest.mark.parametrize("V", [200, 4096, 4097, 8193])
def test_fused_logprob_fold_runs(ua, V):
    """1, 16, 17 and 33 vocabulary tiles: runs of one, full and empty runs of the fold."""
    T, H = 20, 64
    h = inputs.normal_bf16((T, H), 1.0, 94, T, V)
    w = inputs.normal_bf16((V, H), 0.25, 95, T, V)
    tg = inputs.targets(T, V, tag=V)
    lp = ua.lm_head_logprob(gu.dev(h), gu.dev(w), gu.dev_i32(tg)).cpu().numpy().astype(np.float64)
    ref, bound = oracle.lm_head_logprob_fp64(h, w, tg, 1.0)
    assert np.all(np.abs(lp - ref) <= bound)


def test_fused_logprob_rows_are_batch_invariant(ua):
    import torch
    T, V, H = 640, 1500, 1024
    h = gu.dev(inputs.normal_bf16((T, H), 1.0, 96))
    w = gu.dev(inputs.normal_bf16((V, H), 0.0625, 97))
    tg = gu.dev_i32(inputs.targets(T, V, tag=98))
    full = ua.lm_head_logprob(h, w, tg)
    g = inputs.rng(99, 1)
    for n in (1, 2, 7, 128, 129, 257, 300):
        idx = torch.from_numpy(g.permutation(T)[:n]).cuda()
        part = ua.lm_head_logprob(h[idx].contiguous(), w, tg[idx].contiguous())
        assert torch.equal(part.view(torch.int32), full[idx].view(torch.int32)), n
        assert bool((torch.exp(part.double() - full[idx].double()) == 1.0).all())
    # repeated calls, and a target outside the vocabulary
    again = ua.lm_head_logprob(h, w, tg)
    assert torch.equal(again.view(torch.int32), full.view(torch.int32))
    bad = tg.clone()
    bad[3] = V
    bad[5] = -1
    out = ua.lm_head_logprob(h, w, bad)
    assert bool(torch.isnan(out[3])) and bool(torch.isnan(out[5]))
    keep = torch.ones(T, dtype=torch.bool, device="cuda")
    keep[3] = keep[5] = False
    assert torch.equal(out[keep].view(torch.int32), full[keep].view(torch.int32))
