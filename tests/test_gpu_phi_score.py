"""phi(q) and the segment scores at the edges of their tiles and slices: every
feature count, candidate counts around the row blocks of a wave and of a
workgroup, every group size, both head dims, few and many pairs (few take
feature slices and narrow workgroups; 260 of eight heads hold all of phi(q), 64
KB, in one slice), on the paths whose scores run as a
kernel of their own and on the fused one. All candidates are selected (k =
256), so every score comes back; they are held to the suite's 1e-5 of the fp64
oracle, and a bf16 Omega has to give the bits of its fp32 copy."""
import dataclasses

import numpy as np
import pytest
import torch

import _harness as H
import paper_2503_10571_amd as radar
from oracle import radar_oracle as orc

pytestmark = pytest.mark.gpu


def _run(path, cfg, q, K, omega, summ, t, k):
    radar.set_decode_path(path)
    try:
        sel = torch.empty(cfg.batch, cfg.n_q_heads, k, dtype=torch.int32, device="cuda")
        sc = torch.empty(cfg.batch, cfg.n_q_heads, k, device="cuda")
        out = radar.decode(cfg, q, K, K, omega, summ, t, k, selected=sel, scores=sc)
    finally:
        radar.set_decode_path(radar.PATH_AUTO)
    return out, sel, sc


@pytest.mark.parametrize("n", [64, 128, 256, 512, 1024, 2048])
@pytest.mark.parametrize("n_cand,G,d,pairs", [
    (1, 1, 64, 1), (15, 2, 128, 2), (16, 4, 128, 1), (17, 8, 64, 1), (63, 4, 64, 3),
    (64, 1, 128, 40), (65, 8, 128, 2), (127, 2, 64, 1), (128, 4, 128, 2), (129, 1, 64, 2),
    (255, 4, 128, 1), (256, 8, 128, 1), (129, 4, 64, 300), (30, 8, 128, 260)])
def test_scores(n, n_cand, G, d, pairs):
    c, w = 3, 2
    t = n_cand * c + w
    cfg = radar.Config(1, G * pairs, pairs, d, n, c, w, t + 3, torch.bfloat16)
    g = torch.Generator(device="cuda")
    g.manual_seed(n + n_cand)
    K = torch.randn(1, pairs, t + 3, d, generator=g, device="cuda").to(torch.bfloat16)
    q = torch.randn(1, G * pairs, d, generator=g, device="cuda").to(torch.bfloat16)
    omega = torch.randn(n, d, generator=g, device="cuda").to(torch.bfloat16).float()
    summ = radar.new_summaries(cfg, "cuda")
    radar.build_index(cfg, K, omega, t, summ)
    half = dataclasses.replace(cfg, omega_dtype=torch.bfloat16)
    heads = sorted({0, G * pairs - 1})
    for path in (radar.PATH_SCORED, radar.PATH_SPLIT, radar.PATH_FUSED, radar.PATH_AUTO):
        print(f"[case] scores n={n} n_cand={n_cand} G={G} d={d} pairs={pairs} path={path}",
              flush=True)
        out, sel, sc = _run(path, cfg, q, K, omega, summ, t, 256)
        out2, sel2, sc2 = _run(path, half, q, K, omega.to(torch.bfloat16), summ, t, 256)
        assert torch.equal(sel, sel2) and torch.equal(out, out2)
        assert torch.equal(sc[..., :n_cand], sc2[..., :n_cand])
        for h in heads:
            s64 = H.f64(summ[0, h // G, :n_cand])
            ref = orc.segment_scores(orc.random_features(H.f64(q[0, h]), H.f64(omega)), s64)
            ids = sel[0, h, :n_cand].cpu().numpy()
            assert sorted(ids) == list(range(n_cand))
            err = np.max(np.abs(H.f64(sc[0, h, :n_cand]) - ref[ids]) / ref[ids])
            assert err <= H.SCORE_TOL, (path, h, err)


@pytest.mark.parametrize("n", [64, 256, 512, 1024, 2048])
@pytest.mark.parametrize("G,d,dtype", [(1, 128, torch.bfloat16), (2, 64, torch.bfloat16),
                                       (4, 128, torch.bfloat16), (8, 128, torch.bfloat16),
                                       (1, 128, torch.float32), (2, 128, torch.float32),
                                       (4, 64, torch.float32)])
@pytest.mark.parametrize("n_cand", [40, 130])
def test_scores_do_not_depend_on_the_call(n, G, d, dtype, n_cand):
    """A sequence's scores are the same bits alone and in a batch (of equal
    and of longer sequences, with tables below and above 64 MB), with another
    capacity, and on every path."""
    c, w, k = 2, 2, n_cand
    t = n_cand * c + w
    big = (1 << 26) // (n_cand * n * 4) + 1          # pairs of a 64 MB table
    g = torch.Generator(device="cuda")
    g.manual_seed(n + G)

    def normal(*shape):
        return torch.randn(*shape, generator=g, device="cuda").to(dtype)

    long = 2400 if n == 2048 else t + 40              # 1200 candidates beside them
    omega = normal(n, d).to(torch.bfloat16).to(torch.float32)
    key, query = normal(1, 1, long, d), normal(1, G, d)
    want = None
    for B, cap, ragged in [(1, t, False), (1, 8 * t, False), (3, t + 1, False), (5, long, True),
                           (big, t, False), (big // 2 + 1, t + 9, False)]:
        if B * cap * d * key.element_size() > 1 << 29:
            continue
        cfg = radar.Config(B, G, 1, d, n, c, w, cap, dtype)
        K = normal(B, 1, cap, d)
        K[:, :, :t] = key[:, :, :t]
        q = normal(B, G, d)
        q[B // 2] = query[0]
        lens = None
        if ragged:
            lens = torch.full((B,), cap, dtype=torch.int64, device="cuda")
            lens[B // 2] = t
        t_max = cap if ragged else t
        summ = radar.new_summaries(cfg, "cuda")
        radar.build_index(cfg, K, omega, t_max, summ)
        for path in (radar.PATH_AUTO, radar.PATH_SPLIT, radar.PATH_FUSED, radar.PATH_SELECT,
                     radar.PATH_SCORED):
            print(f"[case] same scores n={n} G={G} d={d} {dtype} B={B} cap={cap} path={path}",
                  flush=True)
            radar.set_decode_path(path)
            try:
                sel = torch.empty(B, G, k, dtype=torch.int32, device="cuda")
                sc = torch.empty(B, G, k, device="cuda")
                radar.decode(cfg, q, K, K, omega, summ, t_max, k, selected=sel, scores=sc,
                             lens=lens)
            finally:
                radar.set_decode_path(radar.PATH_AUTO)
            got = (sel[B // 2].clone(), sc[B // 2].clone())
            want = want or got
            assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])


TYPES = [(64, torch.bfloat16), (128, torch.bfloat16), (64, torch.float32), (128, torch.float32)]
COUNTS = [64, 128, 256, 512, 1024, 2048]


@pytest.mark.parametrize("size,n", [("large", n) for n in COUNTS] +
                         [("few", n) for n in COUNTS if n >= 512])
@pytest.mark.parametrize("G", [1, 2, 4, 8])
def test_two_kernels(n, G, size):
    """phi(q) and the scores as two kernels, which take tables from 64 MB and
    more than 1024 candidates where slices are wanted (n >= 512, few pairs),
    with a shorter second sequence; every feature count and group size, and
    between them every head dim and type."""
    d, dtype = TYPES[(COUNTS.index(n) + G.bit_length()) % 4]
    n_cand = 301 if size == "large" else 1061
    pairs = (1 << 26) // (n_cand * n * 4) // 2 + 1 if size == "large" else 1
    c, w, k = 1, 1, 200
    t = n_cand * c + w
    print(f"[case] two kernels n={n} G={G} d={d} {dtype} {size} pairs={2 * pairs}", flush=True)
    cfg = radar.Config(2, G * pairs, pairs, d, n, c, w, t + 2, dtype)
    g = torch.Generator(device="cuda")
    g.manual_seed(n + G)
    K = torch.randn(2, pairs, t + 2, d, generator=g, device="cuda").to(dtype)
    q = torch.randn(2, G * pairs, d, generator=g, device="cuda").to(dtype)
    omega = torch.randn(n, d, generator=g, device="cuda").to(torch.bfloat16).float()
    lens = torch.tensor([t, t - 66], device="cuda")
    summ = radar.new_summaries(cfg, "cuda")
    radar.build_index(cfg, K, omega, t, summ)
    runs = [(cfg, omega)]
    if dtype == torch.bfloat16:
        runs.append((dataclasses.replace(cfg, omega_dtype=dtype), omega.to(dtype)))
    got = []
    for path in (radar.PATH_SPLIT, radar.PATH_SCORED):
        for cf, om in runs:
            radar.set_decode_path(path)
            radar.profile_enable(True)
            try:
                sel = torch.empty(2, G * pairs, k, dtype=torch.int32, device="cuda")
                sc = torch.empty(2, G * pairs, k, device="cuda")
                radar.decode(cf, q, K, K, om, summ, t, k, selected=sel, scores=sc, lens=lens)
                assert radar.profile_read()["phi_q"][1] == 1
            finally:
                radar.profile_enable(False)
                radar.profile_read()
                radar.set_decode_path(radar.PATH_AUTO)
            got.append((sel, sc))
    for sel, sc in got[1:]:
        assert torch.equal(sel, got[0][0]) and torch.equal(sc, got[0][1])
    sel, sc = got[0]
    for b, count in ((0, n_cand), (1, n_cand - 66)):
        for h in {0, G - 1, G * (pairs // 2), G * pairs - 1}:
            s64 = H.f64(summ[b, h // G, :count])
            ref = orc.segment_scores(orc.random_features(H.f64(q[b, h]), H.f64(omega)), s64)
            ids = sel[b, h].cpu().numpy()
            H.check_selection(ids, ref, k, count)
            err = np.max(np.abs(H.f64(sc[b, h]) - ref[ids]) / ref[ids])
            assert err <= H.SCORE_TOL, (b, h, err)
