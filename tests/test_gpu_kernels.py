"""Sizes at which single kernels can go wrong (tile edges, remainders, shortest and longest loops),
against the fp64 oracle."""
import dataclasses

import numpy as np
import pytest
import torch  # before the library: both use the HIP runtime that torch loads

from gpu_common import O, WL, build_instance, compare_full, ensure_library, params_for, rlk, run_gpu, run_oracle, to_host

pytestmark = pytest.mark.gpu


def _all_policy(dtype, tokens, d, V):
    """2 rollouts of one group, `tokens` trained tokens in all."""
    cfg = WL.get_config("small_bf16").with_(
        name=f"edge_{dtype}_{tokens}x{d}x{V}", dtype=dtype, groups=1, rollouts_per_group=2, len_min=tokens // 2,
        len_max=tokens // 2, d=d, V=V, w_std=d ** -0.5)
    st = WL.make_structure(cfg)
    if tokens % 2:  # one more token in the last rollout
        cu = st.cu_seqlens.copy()
        cu[-1] += 1
        grow = lambda a: np.concatenate([a, a[:1]])
        st = dataclasses.replace(st, cu_seqlens=cu, lengths=np.diff(cu).astype(np.int64), targets=grow(st.targets),
                                 noise=grow(st.noise), mask=grow(st.mask))
    return cfg, dataclasses.replace(st, mask=np.ones_like(st.mask))


# K slices of the forward: 1, 2, 3 (whole and with a tail); token and vocabulary tiles one short of, at and
# one past the tile's and its halves' edges; bf16 calls of more than 16,384 rows read W^T in the dhidden GEMM, the
# others W itself
@pytest.mark.parametrize("dtype,tokens,d,V", [
    ("bf16", 2, 8, 1), ("bf16", 127, 64, 129), ("bf16", 129, 72, 255), ("bf16", 255, 128, 256), ("bf16", 256, 136, 257),
    ("bf16", 257, 192, 513), ("bf16", 300, 520, 1), ("bf16", 8192, 136, 321),
    ("bf16", 16384, 136, 321), ("bf16", 16385, 136, 321), ("f32", 127, 8, 129), ("f32", 129, 32, 257), ("f32", 257, 40, 255), ("f32", 255, 96, 300)])
@pytest.mark.parametrize("entropy", [0.0, 1e-2])
def test_gemm_tile_edges(dtype, tokens, d, V, entropy):
    ensure_library()
    cfg, st = _all_policy(dtype, tokens, d, V)
    inst = build_instance(cfg, structure=st)
    p = params_for(cfg, entropy_coef=entropy)
    compare_full(inst, run_gpu(inst, p), run_oracle(inst, p), p, tag="edges")



# W as the head of a larger allocation: what lies behind its last row must not reach any output.  The
# probabilities of vocabulary rows past V are zero, so only NaN there shows a read (0 x NaN), in the K-major
# dhidden GEMM (bf16) above all, whose last K slice holds 1, 63 and 1 rows of W here, or all 64
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("V", [1, 63, 65, 256, 257, 320, 321])
def test_rows_behind_w_are_not_read(dtype, V):
    ensure_library()
    cfg, st = _all_policy(dtype, 100, 136, V)
    inst = build_instance(cfg, structure=st)
    p = params_for(cfg)
    out = []
    for fill in (0.0, float("nan")):
        buf = torch.full((V + 512, cfg.d), fill, dtype=inst["W"].dtype, device="cuda")
        buf[:V] = inst["W"]
        out.append(run_gpu(dict(inst, W=buf[:V]), p))
    for k in ("dh", "dW", "logp", "ent"):
        assert bool(torch.isfinite(out[1][k]).all()) and torch.equal(out[0][k], out[1][k]), k
    assert out[0]["loss"] == out[1]["loss"]


# fp32 tiles are 256 x 64: token, feature and vocabulary edges of them; K split over many, few and no workgroups
@pytest.mark.parametrize("tokens,d,V", [(2, 8, 1), (63, 64, 256), (64, 72, 512), (65, 56, 257), (1030, 264, 4100), (4200, 520, 8300)])
@pytest.mark.parametrize("entropy", [0.0, 1e-2])
def test_fp32_gemm_tile_edges(tokens, d, V, entropy):
    ensure_library()
    cfg, st = _all_policy("f32", tokens, d, V)
    inst = build_instance(cfg, structure=st)
    p = params_for(cfg, entropy_coef=entropy)
    ref = run_oracle(inst, p)
    compare_full(inst, run_gpu(inst, p), ref, p, tag="fp32")
    # added to a preset dW of the gradients' size, aligned to 16 bytes or to its elements only
    pa = params_for(cfg, entropy_coef=entropy, accumulate_dW=True)
    scale = float(np.abs(ref["dW"]).max()) or 1.0
    preset = scale * torch.randn(V * d, generator=torch.Generator(device="cuda").manual_seed(V), device="cuda")
    want = to_host(preset).astype(np.float64).reshape(V, d) + ref["dW"]
    for off in (0, 1):
        buf = torch.empty(V * d + 4, device="cuda")
        dW = buf[off:off + V * d].copy_(preset).view(V, d)
        run_gpu(inst, pa, dW=dW)
        # the gradient's own error and one rounding of a sum of up to six times its size
        assert np.abs(to_host(dW) - want).max() <= (1e-5 + 6 * 2.0 ** -24) * scale, off


def _bounded_call_is_the_same(dtype, tokens, d, V, outputs):
    """Every second token trained: a call bounded by their number (half the chunk rows) against one without, and
    the per-token outputs of one in chunks of 1,024 rows."""
    ensure_library()
    cfg, st = _all_policy(dtype, tokens, d, V)
    mask = np.ones_like(st.mask)
    mask[1::2] = 0
    inst = build_instance(cfg, structure=dataclasses.replace(st, mask=mask))
    p = params_for(cfg)
    free, bounded = run_gpu(inst, p), run_gpu(inst, p, max_policy_tokens=(tokens + 1) // 2)
    assert free["flags"] == bounded["flags"] == 0
    for k in outputs:
        assert torch.equal(free[k], bounded[k]), k
        assert int(torch.count_nonzero(free[k])) > 0
    chunked = run_gpu(inst, params_for(cfg, chunk_rows=1024))
    assert chunked["stats"]["n_chunks"] > free["stats"]["n_chunks"]
    for k in ("logp", "ent"):
        assert torch.equal(free[k], chunked[k]), k
    assert free["loss"] == bounded["loss"] == chunked["loss"]


# dhidden of 16 and of 8 output tiles has one split plan: 16 parts of 8 K slices
def test_fp32_dhidden_of_shapes_that_share_a_split_plan():
    _bounded_call_is_the_same("f32", 4096, 256, 4096, ("logp", "ent", "dh"))


# dhidden of 40 x 9 tiles from W itself, the tile rows of the partial last wave split over K in a second launch; the
# last K slice holds 17 rows of W
def test_k_major_dhidden_with_a_split_tail():
    ensure_library()
    cfg, st = _all_policy("bf16", 10000, 2056, 2001)
    inst = build_instance(cfg, structure=st)
    p = params_for(cfg)
    compare_full(inst, run_gpu(inst, p, max_policy_tokens=10000), run_oracle(inst, p), p, tag="K-major tail")


# bf16: W^T without the bound, W itself (K-major) with it: the same products in the same order
def test_bf16_dhidden_from_w_and_from_its_transpose_are_the_same():
    _bounded_call_is_the_same("bf16", 32768, 136, 250, ("logp", "ent", "dh"))


# Forward and unsplit dhidden take 256 x 256 tiles or such of 64 columns by the rows of the batch: 528 tiles of the
# forward (264 of the trained rows) and 1,040 (520), 512 of dhidden (256)
@pytest.mark.parametrize("tokens,d,V,outputs", [(4096, 264, 8448, ("logp", "ent")), (4096, 264, 16640, ("logp", "ent")),
                                                (16384, 2048, 300, ("logp", "ent", "dh"))])
def test_fp32_tile_width_does_not_follow_the_bound(tokens, d, V, outputs):
    _bounded_call_is_the_same("f32", tokens, d, V, outputs)


# 32 output tiles (128 of 64 columns), 188 K slices in 8 parts: two fp32 sums of 384 products each.  The gradients
# are 0.6e-6 off in all, 1.1e-6 and more if a sum runs over the whole vocabulary
def test_fp32_gradient_sums_stay_short():
    ensure_library()
    cfg, st = _all_policy("f32", 4096, 512, 6000)
    inst = build_instance(cfg, structure=st)
    p = params_for(cfg)
    m = compare_full(inst, run_gpu(inst, p), run_oracle(inst, p), p, tag="fp32 sums")
    assert m["dh_rel"] <= 9e-7 and m["dW_rel"] <= 9e-7


@pytest.mark.parametrize("accumulate", [False, True])
def test_dw_aligned_to_its_elements_only(accumulate):
    """dW may start at any fp32 element: the wide stores of the dW GEMM are not taken there.  The same
    sums in the same order, so the result is that of an aligned dW."""
    ensure_library()
    cfg, st = _all_policy("bf16", 300, 2048, 8200)  # 33 x 8 output tiles: the GEMM itself writes dW
    inst = build_instance(cfg, structure=st)
    p = params_for(cfg, accumulate_dW=accumulate)
    base = torch.randn(cfg.V * cfg.d + 1, generator=torch.Generator(device="cuda").manual_seed(3), device="cuda")
    out = []
    for off in (0, 1):
        buf = torch.empty_like(base)
        dW = buf[off:off + cfg.V * cfg.d].view(cfg.V, cfg.d).copy_(base[:cfg.V * cfg.d].view(cfg.V, cfg.d))
        run_gpu(inst, p, dW=dW)
        out.append(to_host(dW))
    np.testing.assert_array_equal(out[0], out[1])
    assert np.isfinite(out[0]).all() and np.abs(out[0]).max() > 0


# one pass takes 8 rows per thread of 256 or 1,024 threads (short and long mean length); groups of 8 rows
# straddle the rollouts; off = 1 starts the arrays at an element that is not 16-byte aligned
@pytest.mark.parametrize("lens", [(0, 1, 7, 8, 9, 15, 17), (2047, 2048, 2049, 3, 0, 1), (8191, 5, 8193, 8192), (20001, 1)])
@pytest.mark.parametrize("off", [0, 1])
def test_gae_and_value_loss_row_groups(lens, off):
    ensure_library()
    rng = np.random.default_rng(len(lens) + off)
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    N, R = int(cu[-1]), len(lens)
    mask = (rng.random(N) < 0.4).astype(np.uint8)
    vals, rew = rng.standard_normal(N).astype(np.float32), rng.standard_normal(R).astype(np.float32)
    gid = np.arange(R, dtype=np.int32)
    gid[1] = -1

    def dev(a):
        buf = torch.empty(a.shape[0] + off, dtype=torch.as_tensor(a).dtype, device="cuda")
        buf[off:].copy_(torch.as_tensor(a))
        return buf[off:]

    v, m, c, g = dev(vals), dev(mask), torch.as_tensor(cu, device="cuda"), torch.as_tensor(gid, device="cuda")
    out = [dev(np.full(N, np.nan, np.float32)) for _ in range(3)]
    adv, ret = rlk.gae(v, torch.as_tensor(rew, device="cuda"), m, c, g, 0.99, 0.95, adv=out[0], returns=out[1])
    loss, dv = rlk.value_loss(v, ret, m, c, g, dvalues=out[2])
    # the C entry takes gamma and lambda as fp32; fp64 scans, one rounding to fp32
    ra, rr = O.gae(vals, rew, mask, cu, gid, float(np.float32(0.99)), float(np.float32(0.95)))
    np.testing.assert_allclose(to_host(adv), ra, rtol=0, atol=2e-7 * np.abs(ra).max())
    np.testing.assert_allclose(to_host(ret), rr, rtol=0, atol=2e-7 * np.abs(rr).max())
    rl, rdv = O.value_loss(vals, to_host(ret), mask, cu, gid)
    assert abs(float(loss.item()) - rl) <= 2e-7 * abs(rl)
    np.testing.assert_allclose(to_host(dv), rdv, rtol=0, atol=2e-7 * np.abs(rdv).max())


def test_value_loss_of_many_rollouts():
    """More partial sums than the gradient's workgroups add up by themselves (1,024)."""
    ensure_library()
    rng = np.random.default_rng(5)
    R = 1500
    cu = np.concatenate([[0], np.cumsum(rng.integers(0, 12, R))]).astype(np.int32)
    N = int(cu[-1])
    mask, vals, rets = (rng.random(N) < 0.5).astype(np.uint8), rng.standard_normal(N).astype(np.float32), rng.standard_normal(N).astype(np.float32)
    d = lambda a: torch.as_tensor(a, device="cuda")
    loss, dv = rlk.value_loss(d(vals), d(rets), d(mask), d(cu))
    rl, rdv = O.value_loss(vals, rets, mask, cu)
    assert abs(float(loss.item()) - rl) <= 2e-7 * abs(rl)
    np.testing.assert_allclose(to_host(dv), rdv, rtol=0, atol=2e-7 * np.abs(rdv).max())


# more than 1,024 rollouts: a wavefront per rollout up to a mean length of 256 (single ones take several passes), a
# workgroup of four beyond
@pytest.mark.parametrize("R,mean", [(1025, 6), (1030, 256), (1030, 260)])
@pytest.mark.parametrize("off", [0, 1])
def test_gae_and_value_loss_of_many_rollouts(R, mean, off):
    ensure_library()
    rng = np.random.default_rng(R + mean)
    lens = rng.integers(0, mean, R)
    lens[3], lens[R - 1] = 513, 1100
    lens[5] += max(0, R * mean - int(lens.sum()))
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    N = int(cu[-1])
    mask = (rng.random(N) < 0.5).astype(np.uint8)
    vals, rets, rew = (rng.standard_normal(n).astype(np.float32) for n in (N, N, R))

    def dev(a):
        return torch.as_tensor(np.concatenate([a[:off], a]), device="cuda")[off:]

    v, t, m, c = dev(vals), dev(rets), dev(mask), torch.as_tensor(cu, device="cuda")
    loss, dv = rlk.value_loss(v, t, m, c)
    rl, rdv = O.value_loss(vals, rets, mask, cu)
    assert abs(float(loss.item()) - rl) <= 2e-7 * abs(rl)
    np.testing.assert_allclose(to_host(dv), rdv, rtol=0, atol=2e-7 * np.abs(rdv).max())
    adv, ret = rlk.gae(v, torch.as_tensor(rew, device="cuda"), m, c, torch.zeros(R, dtype=torch.int32, device="cuda"), 0.99, 0.95)
    ra, rr = O.gae(vals, rew, mask, cu, np.zeros(R, np.int32), float(np.float32(0.99)), float(np.float32(0.95)))
    np.testing.assert_allclose(to_host(adv), ra, rtol=0, atol=2e-7 * np.abs(ra).max())
    np.testing.assert_allclose(to_host(ret), rr, rtol=0, atol=2e-7 * np.abs(rr).max())


# rows of fewer than 256 16-byte chunks are dealt among the threads (8 features: 256 rows side by side; 1,360:
# one row and a rest of idle threads), wider ones take several passes; 128 rows per workgroup, of fewer than 16,257
# rows in windows of 32 chunks
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("lens,d", [((1,), 8), ((100, 27), 64), ((128,), 680), ((33, 0, 96), 1360), ((500, 13), 2048), ((61, 70), 4104),
                                    ((16000, 300), 64), ((16256,), 264), ((16257,), 264), ((16400,), 2072)])
@pytest.mark.parametrize("accumulate", [False, True])
def test_value_head_row_and_column_splits(dtype, lens, d, accumulate):
    ensure_library()
    rng = np.random.default_rng(d)
    gen = torch.Generator(device="cuda").manual_seed(d)
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    N, R = int(cu[-1]), len(lens)
    mask = (rng.random(N) < 0.6).astype(np.uint8)
    gid = np.zeros(R, np.int32)
    gid[R - 1] = -1 if R > 1 else 0
    r = lambda *shape: torch.randn(*shape, generator=gen, device="cuda")
    h, w, dv, dh0 = r(N, d).to(dtype), r(d).to(dtype), r(N), r(N, d).to(dtype)
    m, c, g = (torch.as_tensor(a, device="cuda") for a in (mask, cu, gid))
    values = rlk.value_head_fwd(h, w, 0.25, m, c, g)
    dh = dh0.clone()
    _, dw, db = rlk.value_head_bwd(h, w, m, c, g, dv, dhidden=dh, accumulate=accumulate)
    _, dw1, db1 = rlk.value_head_bwd(h, w, m, c, g, dv)  # without dhidden: the same sums
    on = ((mask != 0) & np.repeat(gid >= 0, lens)).astype(np.float64)[:, None]
    H, Wv, G = to_host(h).astype(np.float64), to_host(w).astype(np.float64), to_host(dv).astype(np.float64)[:, None] * on
    want = (to_host(dh0) if accumulate else 0.0) + G * Wv
    # fp32 sums of at most d (forward) or 128 (per workgroup) products; bf16 rows rounded once more
    eps = 2.0 ** -8 if dtype == torch.bfloat16 else 2.0 ** -23
    np.testing.assert_allclose(to_host(values)[:, None], (H @ Wv[:, None] + 0.25) * on, rtol=0, atol=2.0 ** -24 * d ** 0.5 * 8 * 4)
    np.testing.assert_allclose(to_host(dh), want, rtol=eps, atol=eps * 1e-2)
    np.testing.assert_allclose(to_host(dw), (G * H).sum(0), rtol=2.0 ** -23, atol=2.0 ** -24 * 128 * 8 * max(1.0, N / 128) ** 0.5)
    assert abs(float(db.item()) - G.sum()) <= 2.0 ** -23 * max(1.0, abs(G.sum()))
    assert torch.equal(dw, dw1) and torch.equal(db, db1)
    if accumulate:
        assert torch.equal(dh[torch.as_tensor(on[:, 0] == 0, device="cuda")], dh0[torch.as_tensor(on[:, 0] == 0, device="cuda")])


# one workgroup up to 1,024 rollouts, 64 to 4 lanes per group of up to 64 and a wavefront per larger one (G = 0: one
# of half the rollouts beside groups of one); beyond, runs of 1,024 (whole, a short last one, all sixteen)
@pytest.mark.parametrize("R,G", [(1, 1), (63, 4), (64, 64), (65, 1), (260, 1), (300, 2), (1024, 1), (1024, 64), (1024, 68),
                                 (1024, 0), (1023, 7), (1024, 1024), (1025, 3), (2048, 16), (5000, 5000), (16384, 1),
                                 (16383, 97)])
def test_group_advantage_run_edges(R, G):
    ensure_library()
    rng = np.random.default_rng(R + G)
    key = np.arange(R) // G if G else np.maximum(np.arange(R) - R // 2, 0)
    gid = rng.permutation(key).astype(np.int32) * 5 + 2
    gid[rng.random(R) < 0.05] = -3
    rew = (rng.integers(0, 4, R) / 4).astype(np.float32)
    idx, count = torch.full((R,), 9, dtype=torch.int32, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda")
    adv = rlk.group_advantage(torch.as_tensor(rew, device="cuda"), torch.as_tensor(gid, device="cuda"), group_index=idx,
                              n_groups=count)
    ref = O.group_advantage(rew, gid, float(np.float32(1e-6)))
    np.testing.assert_array_equal(to_host(idx), ref["group_index"])
    assert int(count.item()) == ref["n_groups"]
    a = to_host(adv).astype(np.float64)
    # fp64 sums, one rounding to fp32
    np.testing.assert_allclose(a, ref["adv"], rtol=2.0 ** -23, atol=1e-12)
    assert np.all(a[ref["adv"] == 0] == 0)


# 1,024 tokens per block, 4 per thread; above 1,024 blocks a scan launch instead of each block's own sums
@pytest.mark.parametrize("N,R", [(1, 1), (1023, 3), (1024, 1), (1025, 2), (4099, 1000), (1 << 20, 7), ((1 << 20) + 1, 5)])
def test_compaction_block_edges(N, R):
    ensure_library()
    rng = np.random.default_rng(N)
    cu = np.concatenate([[0], np.sort(rng.integers(0, N + 1, R - 1)), [N]]).astype(np.int32)
    mask = (rng.random(N) < 0.4).astype(np.uint8)
    gid = rng.integers(-1, 3, R).astype(np.int32)
    d = lambda a: torch.as_tensor(a, device="cuda")
    idx, tokr, n_pol, n_eff, ws = rlk.compact(d(cu), d(mask), d(gid))
    widx, wtokr, wn = O.compact(mask, cu, gid)
    n = int(n_eff.item())
    assert n == widx.size and rlk.check_status(ws) == 0
    np.testing.assert_array_equal(to_host(idx)[:n], widx)
    np.testing.assert_array_equal(to_host(tokr)[:n], wtokr)
    np.testing.assert_array_equal(to_host(n_pol), wn)


# the merge takes blocks of 64 tokens for the 8,192 chunk rows without the bound, of 16 for the 4,096 with it
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("V", [300, 17 * 256, 70 * 256, 330 * 256 + 1])
def test_combine_does_not_depend_on_the_chunk_rows(dtype, V):
    _bounded_call_is_the_same(dtype, 8192, 64, V, ("logp", "ent"))


# the merge of the vocabulary tiles: blocks of 16 tokens up to 4,096 chunk rows and of 64 above, tiles dealt in
# strides of 64 or 16 and batches of four: fewer tiles than strides, one past a batch, several batches
@pytest.mark.parametrize("tokens,V", [(1, 64 * 256 + 1), (15, 300), (17, 257 * 256), (4096, 15 * 256 + 3), (4097, 17 * 256),
                                      (4200, 65 * 256 + 1)])
def test_combine_strides(tokens, V):
    ensure_library()
    gen = torch.Generator(device="cuda").manual_seed(V)
    h, W = (torch.randn(n, 64, generator=gen, device="cuda").bfloat16() for n in (tokens, V))
    W[V // 2] *= 4  # the largest logits lie in one tile
    y = torch.randint(0, V, (tokens,), generator=gen, device="cuda", dtype=torch.int32)
    cu, mask = torch.tensor([0, tokens], dtype=torch.int32, device="cuda"), torch.ones(tokens, dtype=torch.uint8, device="cuda")
    logp, ent = torch.empty(tokens, device="cuda"), torch.empty(tokens, device="cuda")
    rlk.logprob_fwd(h, W, y, mask, cu, logp=logp, entropy=ent)
    for r in range(0, tokens, 1024):
        z = torch.log_softmax(h[r:r + 1024].double() @ W.double().T, 1)
        lp, H = z.gather(1, y[r:r + 1024, None].long())[:, 0], -(z.exp() * z).sum(1)
        # fp32 logits of up to 64 products, |z| up to about 100; one rounding of the results
        for got, want in ((logp, lp), (ent, H)):
            assert float((got[r:r + 1024].double() - want).abs().max()) <= 2.0 ** -23 * 100 * 4
