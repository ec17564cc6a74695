"""Index build at the edges of its tiles: segments of one key, of one 16-key
sub-tile and of one 64-key block, each one key more and less; every width of
the feature slices that a workgroup takes (few items take narrow slices,
many take wide ones), both head dims and both Omega types. Each summary is
checked against the fp64 oracle (relative error 1e-4 per element, the
exponent's fp32 rounding, as for every summary of the suite), and a segment
that an append closes (narrow slices) against the rebuild (wide ones) bit
for bit."""
import dataclasses

import numpy as np
import pytest
import torch

import _harness as H
import paper_2503_10571_amd as radar
from oracle import radar_oracle as orc

pytestmark = pytest.mark.gpu

SIZES = [1, 15, 16, 17, 32, 33, 63, 64, 65, 97, 100, 129]


def _case(c, n, d, pairs, segs, dtype=torch.bfloat16, n_sink=0, seed=0):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    t = n_sink + segs * c
    cfg = radar.Config(1, pairs, pairs, d, n, c, c, t + 3, dtype, n_sink)
    K = torch.randn(1, pairs, t + 3, d, generator=g, device="cuda").to(dtype)
    omega = torch.randn(n, d, generator=g, device="cuda").to(dtype).float()
    return cfg, K, omega, t


def _check(cfg, K, omega, t, summ, heads):
    for h in heads:
        ref = orc.segment_summaries(H.f64(K[0, h, :t]), H.f64(omega), cfg.seg_len,
                                    offset=cfg.n_sink)
        got = H.f64(summ[0, h, :ref.shape[0]])
        err = np.max(np.abs(got - ref) / ref)
        assert err <= H.SUMM_TOL, (h, err)


@pytest.mark.parametrize("c", SIZES)
@pytest.mark.parametrize("d", [64, 128])
def test_block_edges(c, d):
    print(f"[case] build c={c} d={d}", flush=True)
    cfg, K, omega, t = _case(c, 256, d, 2, 5, n_sink=3, seed=c)
    summ = radar.new_summaries(cfg, "cuda")
    radar.build_index(cfg, K, omega, t, summ)
    _check(cfg, K, omega, t, summ, range(2))
    half = dataclasses.replace(cfg, omega_dtype=torch.bfloat16)
    again = radar.new_summaries(cfg, "cuda")
    radar.build_index(half, K, omega.to(torch.bfloat16), t, again)
    assert torch.equal(summ, again)


@pytest.mark.parametrize("n", [64, 128, 256, 512, 1024, 2048])
@pytest.mark.parametrize("segs", [1, 9, 70, 300])
def test_slice_widths(n, segs):
    print(f"[case] build n={n} segs={segs}", flush=True)
    cfg, K, omega, t = _case(40, n, 128, 8, segs, seed=n + segs)
    summ = radar.new_summaries(cfg, "cuda")
    radar.build_index(cfg, K, omega, t, summ)
    _check(cfg, K, omega, t, summ, [0, 7])


@pytest.mark.parametrize("c,n,d,pairs,segs", [
    (300, 256, 64, 16, 266), (300, 256, 128, 8, 300), (129, 512, 128, 3, 198), (647, 1024, 128, 6, 6),
    (100, 128, 64, 32, 120), (70, 2048, 128, 4, 35), (1000, 64, 128, 2, 9), (64, 256, 128, 16, 129)])
def test_plans_agree(c, n, d, pairs, segs):
    """One pair alone (few items: narrow slices, segments split over waves)
    and all pairs together (wide slices, a wave per segment, a last round in a
    launch of its own) give the same bits."""
    print(f"[case] plans c={c} n={n} d={d} pairs={pairs} segs={segs}", flush=True)
    cfg, K, omega, t = _case(c, n, d, pairs, segs, seed=c)
    summ = radar.new_summaries(cfg, "cuda")
    radar.build_index(cfg, K, omega, t, summ)
    _check(cfg, K, omega, min(t, 3 * c), summ[:, :, :3], [0])
    one = dataclasses.replace(cfg, n_q_heads=1, n_kv_heads=1)
    for p in {0, pairs // 2, pairs - 1}:
        alone = radar.new_summaries(one, "cuda")
        radar.build_index(one, K[:, p].contiguous(), omega, t, alone)
        assert torch.equal(alone[0, 0], summ[0, p]), p


@pytest.mark.parametrize("c,n,d", [(33, 64, 64), (100, 256, 128), (64, 512, 128), (130, 2048, 64)])
def test_close_equals_rebuild(c, n, d):
    print(f"[case] close c={c} n={n} d={d}", flush=True)
    cfg, K, omega, t = _case(c, n, d, 16, 40, n_sink=1, seed=c)
    V = torch.zeros_like(K)
    full, grown = (radar.new_summaries(cfg, "cuda") for _ in range(2))
    radar.build_index(cfg, K, omega, t, full)
    radar.build_index(cfg, K, omega, t - 1, grown)
    k_new = K[:, :, t - 1].clone()
    radar.append(cfg, K, V, k_new, k_new, omega, t - 1, grown)
    assert torch.equal(full, grown)
    radar.build_index(cfg, K, omega, t - 1, grown)
    pos = torch.tensor([t - 1], device="cuda")
    grown[:, :, t // c - 1] = 0
    radar.append(cfg, K, V, k_new, k_new, omega, 0, grown, pos=pos)
    assert torch.equal(full, grown)
    # a row that closes nothing leaves the summaries alone
    radar.append(cfg, K, V, k_new, k_new, omega, 0, grown, pos=pos - 2)
    assert torch.equal(full, grown)
