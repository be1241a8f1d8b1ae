"""GPU parity of nat_advantage / nat_select / nat_compact against the oracle:
bit-exact masks, indices, cut points, offsets and weights (Sec. 3.1, Sec. 4, Eq. 6-9)."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

import synth_inputs as si
from oracle import grpo as ogrpo
from oracle import select as osel
from nat_testlib import (DEV, assert_select_compact_equal, hip_select_compact, oracle_select_compact, to_dev)


@pytest.fixture(scope="module")
def stage():
    from paper_2603_06619_amd.stage import LossStage
    return LossStage(DEV)


EDGE_LENGTHS = [1, 2, 63, 64, 65, 0, 127, 128, 129, 4095, 4096, 4097, 1, 0, 300]


@pytest.mark.parametrize("scheme,kw", [
    (osel.FULL, {}), (osel.URS, dict(p=0.5)), (osel.URS, dict(p=0.25)), (osel.URS, dict(p=1.0)),
    (osel.URS, dict(p=0.37)), (osel.RPC, dict(C=1)), (osel.RPC, dict(C=100)), (osel.RPC, dict(C=10 ** 6)),
    (osel.DET, dict(beta=0.5)), (osel.DET, dict(beta=1.0))])
def test_edge_lengths_all_schemes(stage, scheme, kw):
    cu = np.concatenate([[0], np.cumsum(EDGE_LENGTHS)]).astype(np.int64)
    for seed in (0, 1, 0xDEADBEEFCAFE):
        o = oracle_select_compact(cu, scheme, seed=seed, step=3, base=17, **kw)
        h = hip_select_compact(stage, cu, scheme, seed=seed, step=3, base=17, **kw)
        assert_select_compact_equal(h, o, int(cu[-1]))


def test_many_seeds_small_batches(stage):
    rng = np.random.default_rng(0)
    for trial in range(60):
        B = int(rng.integers(1, 12))
        T = rng.integers(0, 200, B)
        cu = np.concatenate([[0], np.cumsum(T)]).astype(np.int64)
        scheme = int(rng.integers(0, 4))
        kw = dict(p=float(rng.choice([0.1, 0.5, 0.9])), C=int(rng.choice([1, 5, 50])), beta=float(rng.choice([0.3, 0.5])),
                  seed=int(rng.integers(0, 2 ** 63)), step=int(rng.integers(0, 2 ** 32)), base=int(rng.integers(0, 10 ** 6)))
        o = oracle_select_compact(cu, scheme, n_rollouts=B + 3, **kw)
        h = hip_select_compact(stage, cu, scheme, n_rollouts=B + 3, **kw)
        assert_select_compact_equal(h, o, int(cu[-1]))


def test_mixed_schemes_per_rollout_and_gather(stage):
    lay = si.batch_layout("wide_head_stress", 5, P=6, G=4)
    cu = lay["cu_seqlens"]
    N = lay["N"]
    spr = np.where((np.arange(24) // 4) % 2 == 0, osel.URS, osel.DET).astype(np.int32)
    rng = np.random.default_rng(1)
    hidden = rng.standard_normal((N, 64), dtype=np.float32)
    ids = rng.integers(0, 1000, N).astype(np.int32)
    old = rng.standard_normal(N).astype(np.float32)
    o = oracle_select_compact(cu, osel.URS, p=0.5, beta=0.5, seed=9, spr=spr)
    for tdt in (torch.float32, torch.bfloat16):
        h = hip_select_compact(stage, cu, osel.URS, p=0.5, beta=0.5, seed=9, spr=spr,
                               hidden=to_dev(hidden, tdt), ids=to_dev(ids), old_logp=to_dev(old))
        assert_select_compact_equal(h, o, N)
        nk = o["n_kept"]
        ref_rows = to_dev(hidden, tdt)[torch.from_numpy(o["kept_idx"]).long().to(DEV)]
        assert torch.equal(h["hidden_k"][:nk], ref_rows)
        assert np.array_equal(h["ids_k"].cpu().numpy()[:nk], ids[o["kept_idx"]])
        assert np.array_equal(h["old_logp_k"].cpu().numpy()[:nk], old[o["kept_idx"]])


@pytest.mark.parametrize("name,scheme,kw", [
    ("qwen3_8b_head_rpc", osel.RPC, dict(C=1)),
    ("qwen3_8b_long_cot", osel.URS, dict(p=0.5)),
    ("qwen3_8b_long_cot", osel.RPC, dict(C=100)),
    ("wide_head_stress", osel.DET, dict(beta=0.5))])
def test_full_size_batches_bit_exact(stage, name, scheme, kw):
    lay = si.batch_layout(name, 1000 * si.WORKLOAD_ORDER.index(name))
    cu = lay["cu_seqlens"]
    o = oracle_select_compact(cu, scheme, seed=77, step=1, **kw)
    h = hip_select_compact(stage, cu, scheme, seed=77, step=1, **kw)
    assert_select_compact_equal(h, o, lay["N"])
    if scheme == osel.RPC and kw["C"] == 1:
        # expected retained fraction about one half (Sec. 4, uniform cutoff)
        assert 0.35 < o["n_kept"] / lay["N"] < 0.65


def test_empty_batch_and_all_dropped(stage):
    cu = np.array([0, 0, 0], dtype=np.int64)
    h = hip_select_compact(stage, cu, osel.URS, p=0.5)
    assert h["n_kept"] == 0 and h["cu_kept"].cpu().tolist() == [0, 0, 0]
    cu = np.array([0, 1, 2, 3], dtype=np.int64)          # DET with beta=.5 on length-1 rollouts keeps nothing
    o = oracle_select_compact(cu, osel.DET, beta=0.5)
    h = hip_select_compact(stage, cu, osel.DET, beta=0.5)
    assert o["n_kept"] == 0
    assert_select_compact_equal(h, o, 3)


def test_advantage_matches_eq2(stage):
    rng = np.random.default_rng(3)
    for P, G in [(1, 1), (2, 4), (16, 8), (8, 16), (5, 70), (3, 130)]:
        R = si.draw_rewards(P, G, rng, equal_reward_frac=0.3)
        if G > 8:
            R = R + rng.random((P, G)).astype(np.float32)
            R[0] = 2.0
        adv = stage.advantage(to_dev(R.reshape(-1)), P, G, 1e-6).cpu().numpy().reshape(P, G)
        ref = ogrpo.advantages(R, 1e-6)
        assert np.abs(adv - ref).max() <= 2e-6 * max(1.0, np.abs(ref).max())
        assert (adv[np.ptp(R, axis=1) == 0] == 0).all()       # equal rewards: exactly zero


@pytest.mark.parametrize("scheme,kw", [(osel.FULL, {}), (osel.URS, dict(p=0.5)), (osel.RPC, dict(C=100)),
                                        (osel.DET, dict(beta=0.5))])
def test_zero_advantage_rollouts_are_dropped(stage, scheme, kw):
    # the paper's second model workload: a quarter of the prompts have all-equal rewards; Eq. 2 on the device
    # gives exactly 0 there, and those rollouts keep nothing
    lay = si.batch_layout("qwen2p5_math_7b_head", 5000)
    cu, B, P, G = lay["cu_seqlens"], lay["B"], lay["P"], lay["G"]
    adv_dev = stage.advantage(to_dev(lay["rewards"].reshape(-1)), P, G)
    adv = adv_dev.cpu().numpy()
    adv_ref = ogrpo.advantages(lay["rewards"]).reshape(-1)
    assert np.array_equal(adv == 0, adv_ref == 0) and (adv == 0).sum() >= B // 4
    o = oracle_select_compact(cu, scheme, seed=3, step=2, drop=adv_ref, **kw)
    h = hip_select_compact(stage, cu, scheme, seed=3, step=2, drop=adv, **kw)
    assert_select_compact_equal(h, o, lay["N"])
    full = oracle_select_compact(cu, scheme, seed=3, step=2, **kw)
    assert o["n_kept"] < full["n_kept"]


@pytest.mark.parametrize("n_tiles,extra", [(1, -1), (1, 0), (1, 1), (2, 1023), (128, 0), (128, 1), (1024, 0), (1024, 1)])
def test_compaction_at_tile_and_scan_boundaries(stage, n_tiles, extra):
    # tiles of 4096 positions; up to 512 of them a scatter block counts the earlier mask words itself, beyond that it adds up
    # the counts of tiles and groups of tiles.  Rollouts: runs of empty and one-token ones at edges of tiles and spans
    N = 4096 * n_tiles + extra
    rng = np.random.default_rng(N)
    edges = np.concatenate([[0, 0, 1, 1023, 1024, 1025, 4095, 4095, 4096, 4096, 4097], rng.integers(0, N, 70)])
    cu = np.concatenate([[0], np.sort(np.minimum(edges, N)), np.full(3, N)]).astype(np.int64)
    ids = rng.integers(0, 1 << 30, N).astype(np.int32)
    old = rng.standard_normal(N).astype(np.float32)
    for scheme, kw in ((osel.URS, dict(p=0.4)), (osel.RPC, dict(C=7)), (osel.FULL, {})):
        o = oracle_select_compact(cu, scheme, seed=5, step=1, **kw)
        h = hip_select_compact(stage, cu, scheme, seed=5, step=1, ids=to_dev(ids), old_logp=to_dev(old), **kw)
        assert_select_compact_equal(h, o, N)
        k = o["kept_idx"]
        assert np.array_equal(h["ids_k"].cpu().numpy()[:len(k)], ids[k])
        assert np.array_equal(h["old_logp_k"].cpu().numpy()[:len(k)], old[k])


@pytest.mark.parametrize("N", [1, 4096, 9000, 4096 * 129 + 5, 4096 * 1025 + 3])
def test_compaction_offsets_of_long_runs_of_empty_rollouts(stage, N):
    # a tile's block writes the offsets of all rollouts that start in it, 1024 (256 above 512 tiles) x 4 at a time: runs of
    # empty rollouts around multiples of that, at the start, at a tile's edge, inside and at N
    rng = np.random.default_rng(N)
    inside = rng.integers(0, N + 1, 40)
    runs = [(0, 1022), (min(4095, N), 1024), (min(4096, N), 4097), (min(4097, N), 8192), (N // 2, 30000), (N, 9000)]
    cu = np.sort(np.concatenate([[0, N], inside] + [np.full(n, pos) for pos, n in runs])).astype(np.int64)
    o = oracle_select_compact(cu, osel.DET, beta=0.5)
    assert_select_compact_equal(hip_select_compact(stage, cu, osel.DET, beta=0.5), o, N)


@pytest.mark.parametrize("n_tiles,extra,B", [(512, 0, 254), (512, 1, 255), (528, 0, 256), (529, -4095, 300), (90, 77, 255),
                                               (1281, -4095, 4000), (1537, 77, 9000), (1792, 0, 300), (1793, -4095, 300)])
def test_compaction_where_counting_changes(stage, n_tiles, extra, B):
    # up to and beyond the tiles whose blocks count the mask words themselves, whole and begun groups of 16 tiles, as many rollouts
    # as one round of the search takes, and blocks of four and eight wavefronts; a mask that is not 16-byte aligned gives the same
    import paper_2603_06619_amd as nat
    N = 4096 * n_tiles + extra
    rng = np.random.default_rng(N)
    cu = np.concatenate([[0], np.sort(rng.integers(0, N + 1, B - 1)), [N]]).astype(np.int64)
    o = oracle_select_compact(cu, osel.URS, p=0.4, seed=5, step=1)
    h = hip_select_compact(stage, cu, osel.URS, p=0.4, seed=5, step=1)
    assert_select_compact_equal(h, o, N)
    shifted = torch.zeros(h["mask_bits"].numel() + 1, dtype=torch.int32, device=DEV)[1:]
    shifted.copy_(h["mask_bits"])
    assert shifted.data_ptr() % 16 == 4
    again = {k: torch.full_like(h[k], -1) for k in ("kept_idx", "kept_seq", "kept_w", "cu_kept", "n_kept_dev")}
    nat.nat_compact(nat.SelectParams(nat.URS, p=0.4, seed=5, step=1), B, shifted, to_dev(cu), B, N, *again.values(), None,
                    torch.empty(nat.compact_workspace_bytes(N), dtype=torch.uint8, device=DEV))
    nk = o["n_kept"]
    for k, v in again.items():
        assert torch.equal(v[:nk], h[k][:nk]), k
        if k.startswith("kept"):
            assert bool((v[nk:] == -1).all()), k
    # the same tokens weighted by given probabilities
    for v in again.values():
        v.fill_(-1)
    pi = torch.full((N,), 0.4, dtype=torch.float64, device=DEV)
    nat.nat_compact_pi(B, h["mask_bits"], pi, to_dev(cu), B, N, *again.values(), None,
                       torch.empty(nat.compact_workspace_bytes(N), dtype=torch.uint8, device=DEV))
    for k, v in again.items():
        assert torch.equal(v[:nk], h[k][:nk]) or (k == "kept_w" and float((v[:nk] / h[k][:nk] - 1).abs().max()) <= 2.0 ** -23), k
        if k.startswith("kept"):
            assert bool((v[nk:] == -1).all()), k
